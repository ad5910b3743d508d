"""What the host code of the library enqueues, seen on the CPU: libkge.so runs in a process of its own against a stand-in
for the HIP runtime (hip_recorder.cpp) that records launches instead of making them."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2004_08532_amd", "libkge.so")

DRIVER = r'''
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
rec.recorder_events.restype = ctypes.c_char_p
i32, i64, f32, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_void_p
MODELS = ["transe_l2", "transe_l1", "distmult", "complex", "rotate", "rescal", "transr"]

class Config(ctypes.Structure):
    _fields_ = [("model", i32), ("device", i32), ("num_entities", i64), ("num_relations", i64), ("ent_dim", i32),
                ("rel_dim", i32), ("max_batch", i32), ("max_neg_per_chunk", i32), ("max_chunks", i32), ("gemm_input", i32),
                ("adagrad_mode", i32), ("adagrad_eps", f32), ("adv_temperature", f32), ("validate_indices", i32),
                ("loss", i32)]

lib.kge_workspace_bytes.restype = i64
lib.kge_workspace_bytes.argtypes = [vp]
lib.kge_graph_captures.restype = i64
lib.kge_graph_captures.argtypes = [vp]
lib.kge_destroy.argtypes = [vp]
lib.kge_train_steps.argtypes = [vp] * 5 + [vp] * 3 + [i64, vp, i64, i64, vp, i64, f32, f32, vp, vp]

class Library:
    """One context of `model` with b positives in chunks of g, k corrupting entities each, rows of D floats."""
    def __init__(self, model, b=64, g=16, k=24, D=64, relations=20, **kw):
        m = MODELS.index(model)
        rel = {"rotate": D // 2, "rescal": D * D, "transr": D + D * D}.get(model, D)
        self.b, self.g, self.k = b, g, k
        cfg = Config(model=m, num_entities=1000, num_relations=relations, ent_dim=D, rel_dim=rel, max_batch=b, max_neg_per_chunk=k,
                     max_chunks=b // g, **kw)
        self.ctx = vp()
        assert lib.kge_create(ctypes.byref(cfg), ctypes.byref(self.ctx)) == 0
        rec.recorder_clear()

    def steps(self, n, sides=True):
        """kge_train_steps of n steps on a stream of its own; the status and what was enqueued."""
        p = 4096  # (an address that nothing reads)
        host_sides = (i32 * n)(*[s % 2 for s in range(n)]) if sides else None
        rec.recorder_clear()
        rc = lib.kge_train_steps(self.ctx, p, p, p, p, p, p, p, self.b, p, self.k, self.g, host_sides, n, 12.0, 0.1, p, p)
        return rc, rec.recorder_events().decode().splitlines()

'''


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    out = tmp_path_factory.mktemp("recorder") / "librecorder.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "hip_recorder.cpp"), "-o", str(out)],
                   check=True)
    return str(out)


def drive(recorder, body):
    """Run `body` (which prints one JSON value) after DRIVER in a process without torch."""
    r = subprocess.run([sys.executable, "-c", DRIVER + body, recorder, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
    return json.loads(r.stdout.splitlines()[-1])


@pytest.mark.parametrize("chunk", [1, 16])
@pytest.mark.parametrize("model", ["transe_l2", "transe_l1", "distmult", "complex", "rotate", "rescal", "transr"])
def test_a_longer_call_needs_no_code_that_a_short_one_has_not_loaded(recorder, model, chunk):
    """The runtime loads the code of a source file when a kernel of it is first launched, which takes milliseconds for a large
    one.  A program that warms up with a few steps must not meet that in its first long call."""
    first, later = drive(recorder, f'''
x = Library({model!r}, g={chunk})
calls = [x.steps(n) for n in (5, 20, 20, 300)]
assert all(rc == 0 for rc, _ in calls)
print(json.dumps([calls[0][1], sum((e for _, e in calls[1:]), [])]))
''')
    loaded = {e.split()[1] for e in first if e.startswith("kernel")}
    new = [e for e in later if e.startswith("kernel") and e.split()[1] not in loaded]
    assert any(e.startswith("graph") for e in later)
    assert loaded and not new, new


@pytest.mark.parametrize("model,k", [("transe_l2", 24), ("transr", 24), ("rotate", 5000)])  # (the last: sorted on a second stream)
def test_a_graph_is_built_when_the_steps_of_a_short_call_are_enqueued(recorder, model, k):
    """First call of 20 steps: launched kernel by kernel, the graph only built.  The next replays it, and both run every step."""
    one, first, second, captures = drive(recorder, f'''
x = Library({model!r}, k={k})
print(json.dumps([x.steps(1), x.steps(20), x.steps(20), lib.kge_graph_captures(x.ctx)]))
''')
    assert one[0] == first[0] == second[0] == 0 and captures == 1
    assert all(e.startswith("kernel") for e in first[1]) and len(first[1]) == 20 * len(one[1])
    assert run_kernels(second[1]) == 20 * len(one[1]) and second[1][-1] == f"graph {16 * len(one[1])}"


def run_kernels(events):
    """Kernels of training steps in what a call enqueued, graphs counted by the kernels they hold."""
    return sum(int(e.split()[1]) if e.startswith("graph") else 1 for e in events
               if e != "copy" and "k_set_step_block" not in e)


@pytest.mark.parametrize("nth", [1, 2])
@pytest.mark.parametrize("n_steps", [16, 20, 64, 300, 65_536 + 97])
@pytest.mark.parametrize("call", ["hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate", "hipGraphUpload",
                                  "hipGraphLaunch", "hipMemcpyAsync", "capture: hipLaunchKernel"])
def test_a_graph_that_fails_leaves_no_step_out(recorder, call, n_steps, nth):
    """When building or starting a graph fails, the call still runs each of its steps once."""
    launch = call.startswith("capture")
    name = call.split()[-1]
    one, got = drive(recorder, f'''
x = Library("distmult")
one = x.steps(1)
unit = 16 if {n_steps} < 64 else 32
plain = {n_steps} if {n_steps} < 256 else unit + {n_steps} % unit
got = []
for _ in range(3):
    # a launch inside of the capture: the kernels before it are those of the plain start
    rec.recorder_fail({name!r}.encode(), len(one[1]) * plain + 3 if {launch} else {nth})
    got.append(x.steps({n_steps}))
print(json.dumps([one, got]))
''')
    for rc, events in got if not launch else got[:1]:
        assert rc == 0 and run_kernels(events) == n_steps * len(one[1])


def test_transr_projections_in_one_launch_with_the_gradients_where_no_kernel_comes_between(recorder):
    """Steps with the logistic loss and uniform weights, rows of up to 128 floats and at most 1024 scores per row run in units; kge_score, kge_rank
    and all other steps have the projections in a launch of their own, and those steps a kernel for V and one for the back-projection."""
    units, others, scores = drive(recorder, '''
lib.kge_score.argtypes = [vp] * 6 + [i64, vp, i64, i64, i32, f32, vp, vp, vp]
lib.kge_rank.argtypes = [vp] * 6 + [i64, vp, i64, i64, i32, f32, vp, vp]

def kernels(events):
    return sorted({k for e in events for k in ("project_units", "k_transr_projectI", "transr_dp", "transr_back") if k in e})

def forward(x, name, outputs):
    p = 4096
    rec.recorder_clear()
    assert getattr(lib, name)(x.ctx, p, p, p, p, p, x.b, p, x.k, x.g, 0, 12.0, p, *[p] * outputs) == 0
    return kernels(rec.recorder_events().decode().splitlines())

def step(**kw):
    return kernels(Library("transr", **{"k": 64, **kw}).steps(1)[1])

x = Library("transr", k=64)
print(json.dumps([[step(), step(D=128), step(k=1024), step(k=1, D=4), step(relations=1)],
                  [step(adv_temperature=1.0), step(loss=1), step(D=132), step(k=1025)],
                  [forward(x, "kge_score", 2), forward(x, "kge_rank", 1)]]))
''')
    assert units == 5 * [["project_units"]]
    assert others == 4 * [["k_transr_projectI", "transr_back", "transr_dp"]]
    assert scores == 2 * [["k_transr_projectI"]]


# (model, chunk, options, b, k of the first steps, k of the later ones): every form of the step, and changes of form on one context
PROFILED = [(m, g, "", 64, 24, 24) for m in ("transe_l2", "transe_l1", "distmult", "complex", "rotate", "rescal", "transr") for g in (1, 16)] + [
    ("transr", 16, "", 64, 1100, 24), ("transr", 16, "", 64, 24, 1100), ("transr", 16, "D=136, ", 64, 24, 24), ("transr", 16, "loss=1, ", 64, 24, 24),
    ("transe_l2", 16, "adv_temperature=1.0, ", 64, 24, 24), ("rescal", 16, "D=200, ", 64, 24, 24), ("distmult", 16, "", 64, 24, 5000),
    ("distmult", 16, "", 64, 5000, 24), ("transe_l2", 1, "D=400, ", 512, 256, 8)]


@pytest.mark.parametrize("model,chunk,options,b,k,later", PROFILED)
def test_profile_counts_the_kernels_that_ran(recorder, model, chunk, options, b, k, later):
    """kge_profile's times of steps whose kernels take 1 ms each: a slot gets a millisecond from every step that launches its kernel
    and nothing from the others, and no error is left behind."""
    codes, rows, pending = drive(recorder, f'''
lib.kge_profile.argtypes = [vp, i32]
lib.kge_profile_read.argtypes = [vp, ctypes.POINTER(ctypes.c_double), ctypes.POINTER(i64)]
x = Library({model!r}, b={b}, g={chunk}, {options}k=max({k}, {later}))
assert lib.kge_profile(x.ctx, 1) == 0
def read():
    ms, n = (ctypes.c_double * 9)(), i64()
    assert lib.kge_profile_read(x.ctx, ms, ctypes.byref(n)) == 0
    return list(ms) + [n.value]
codes, rows = [], [read()]
for k in ({k}, {later}):
    x.k = k
    for n in (1, 3):
        codes.append(x.steps(n)[0])
        rows.append(read())
print(json.dumps([codes, rows, rec.hipGetLastError()]))
''')
    assert codes == [0] * 4 and pending == 0
    for n, before, after in zip((1, 3, 1, 3), rows, rows[1:]):
        added = [y - x for x, y in zip(before, after)]
        assert added[9] == n and set(added[:9]) <= {0, n} and added[6] == n, added
    first, second = ([y - x for x, y in zip(rows[i], rows[i + 1])][:9] for i in (0, 2))
    assert (first == second) == (k == later), (first, second)


# (b, g, k, D, relations, rows per workgroup) whose (chunk, rows) pairs are 24, 6, 20, 104, 130, 300 and 2, and few units: the last
# shape has more workgroups of 64 rows than the chip holds at a time, the one in front of it just as many
@pytest.mark.parametrize("b,g,k,D,relations,rows", [
    (1024, 128, 300, 100, 1345, 128), (800, 400, 300, 64, 60, 128), (1024, 256, 640, 128, 1345, 128), (1300, 100, 1000, 100, 1345, 128),
    (1040, 16, 256, 100, 1345, 128), (1300, 13, 300, 48, 1345, 128), (1000, 1000, 200, 32, 1345, 128), (1024, 128, 256, 4, 2, 64),
    (3, 1, 1, 4, 2, 64), (64, 32, 1024, 100, 7, 64), (512, 16, 128, 100, 4, 64), (528, 16, 128, 100, 4, 128)])
def test_ranges_of_transr_units_fill_the_chip(recorder, b, g, k, D, relations, rows):
    """No grid whose last round of workgroups is a small part of the chip, and no more partial rows than there is room for."""
    rc, events = drive(recorder, f'''
print(json.dumps(Library("transr", b={b}, g={g}, k={k}, D={D}, relations={relations}).steps(1)))
''')
    events = [e for e in events if "k_transr_project_units" in e]
    assert rc == 0 and (len(events) == 1 if k <= 1024 else not events)
    if not events:
        return
    wgs = int(events[0].split()[3])
    base, slots, most = b // g * -(-k // rows), 512 if D <= 32 else 256, min(g, relations) + g // 32
    segments = wgs // base
    assert wgs == base * segments and 1 <= segments <= most
    assert segments * (b // g) * k <= b // g * k + (b // g + 768) * 64
    if wgs > slots:
        assert wgs / (-(-wgs // slots) * slots) > 0.75, (wgs, slots)
    elif segments < most:
        assert wgs > 0.75 * slots, (wgs, slots)


# (b, g, k, D) and whether the tiles of the forward product are in the gather launch: the limits on tiles and on keys
FRONT = {
    "complex": [(1024, 128, 384, 64, True), (1024, 128, 416, 64, False), (1024, 128, 384, 256, True), (1024, 128, 416, 256, False),
                (1024, 256, 768, 264, True), (1024, 256, 800, 264, False), (1024, 128, 640, 400, True), (1024, 128, 672, 400, False)],
    "transe_l2": [(1024, 128, 512, 64, True), (1024, 128, 544, 64, False), (1024, 128, 640, 400, True), (1024, 128, 672, 400, False),
                  (1024, 256, 768, 400, True), (2048, 128, 256, 400, True), (2048, 128, 288, 400, False)],
    "distmult": [(1024, 128, 512, 128, True), (1024, 128, 544, 128, False), (1024, 128, 768, 400, True), (1024, 128, 800, 400, False),
                 (16, 16, 8160, 8, True), (16, 16, 8161, 8, False), (1024, 128, 768, 512, True), (1024, 128, 768, 516, False)],
    "transe_l1": [(1024, 128, 512, 64, True), (1024, 128, 768, 400, True)],
    "rescal": [(1024, 128, 512, 64, True), (1024, 128, 768, 200, True)],
}


@pytest.mark.parametrize("model", sorted(FRONT))
def test_forward_product_in_the_gather_launch_where_it_is_the_faster_one(recorder, model):
    got = drive(recorder, f'''
got = []
for b, g, k, D, _ in {FRONT[model]!r}:
    rc, events = Library({model!r}, b=b, g=g, k=k, D=D).steps(1)
    assert rc == 0
    got.append([any("k_front" in e for e in events), any("k_gather" in e for e in events)])
print(json.dumps(got))
''')
    assert [f for f, _ in got] == [s[4] for s in FRONT[model]]
    assert [g for _, g in got] == [not s[4] for s in FRONT[model]]


# (b, g, k) and whether the forward product is the one on larger tiles of the bf16 matrix cores: few tiles, chunks of few
# positives, tiles that reach far past a chunk's rows or columns
@pytest.mark.parametrize("loss", ["adv_temperature=0.0", "adv_temperature=1.0", "loss=1"])
@pytest.mark.parametrize("b,g,k,split", [(1000, 1000, 1504, True), (1000, 1000, 1472, False), (2048, 256, 1024, True),
                                         (1504, 32, 1024, True), (1513, 17, 528, True), (1504, 16, 1024, False), (2048, 4, 96, False),
                                         (3072, 2, 32, False), (2048, 2, 64, False), (48_128, 32, 32, False), (48_128, 32, 64, False),
                                         (48_128, 32, 86, True), (3072, 96, 544, False), (2016, 96, 800, True)])
def test_split_forward_product_where_its_tiles_are_filled(recorder, b, g, k, split, loss):
    rc, events = drive(recorder, f'''
print(json.dumps(Library("transe_l2", b={b}, g={g}, k={k}, D=400, {loss}).steps(1)))
''')
    assert rc == 0
    assert any("k_gemm_split_fwd" in e for e in events) == split
    assert any("k_gemm_fwd" in e for e in events) != split


# (b, g, k, D) and whether scores, ranks and training steps take tiles of 64 x 64: 1024 tiles of 32 x 32 (1280 for scores of short rows), tiles
# that are filled, no few workgroups past the first or second 256
WIDE = [(1000, 1000, 1024, 400, 1, 1, 1), (1000, 1000, 1023, 400, 1, 1, 1), (992, 992, 1024, 400, 0, 0, 0), (1024, 1024, 1025, 400, 0, 1, 0),
        (1024, 1024, 1216, 400, 0, 1, 0), (1024, 1024, 1280, 400, 1, 1, 1), (1024, 1024, 1088, 800, 0, 0, 0), (1024, 1024, 1280, 800, 1, 1, 1),
        (1024, 1024, 1088, 128, 0, 1, 0), (1024, 1024, 1280, 128, 1, 1, 1), (1024, 1024, 2112, 400, 0, 1, None), (1024, 1024, 2112, 800, 0, 1, None),
        (1024, 1024, 2304, 400, 1, 1, None), (1024, 1024, 3136, 400, 1, 1, None), (2016, 96, 1024, 400, 0, 0, None), (2013, 33, 800, 100, 0, 0, None)]


@pytest.mark.parametrize("b,g,k,D,score,rank,step", WIDE)
def test_wide_tiles_where_they_fill_the_chip(recorder, b, g, k, D, score, rank, step):
    got = drive(recorder, f'''
lib.kge_score.argtypes = [vp] * 6 + [i64, vp, i64, i64, i32, f32, vp, vp, vp]
lib.kge_rank.argtypes = [vp] * 6 + [i64, vp, i64, i64, i32, f32, vp, vp]
x, p, got = Library("distmult", b={b}, g={g}, k={k}, D={D}, adv_temperature=1.0), 4096, []
for name, outputs in (("kge_score", 2), ("kge_rank", 1)):
    rec.recorder_clear()
    assert getattr(lib, name)(x.ctx, p, p, p, p, p, x.b, p, x.k, x.g, 0, 12.0, p, *[p] * outputs) == 0
    got.append(rec.recorder_events().decode())
got.append("\\n".join(x.steps(1)[1]))
print(json.dumps([["k_gemm_fwd_wide" in e, "k_gemm_fwd" in e, "k_gemm_split_fwd" in e] for e in got]))
''')
    assert got[:2] == [[bool(score), True, False], [bool(rank), True, False]]
    assert got[2] == ([False, False, True] if step is None else [bool(step), True, False])


# chunks of one positive, steps launched one by one: (model, b, k, D) and whether the keys are sorted beside k_ind, with a fork
# and a join: more positives than the chip holds workgroups of k_ind, and enough work
@pytest.mark.parametrize("model,b,k,D,beside", [
    ("distmult", 1024, 1024, 400, False), ("distmult", 1280, 256, 400, True), ("distmult", 1280, 200, 400, False),
    ("complex", 2048, 512, 400, True), ("transe_l1", 2048, 512, 400, True), ("transe_l2", 2048, 256, 400, True),
    ("transe_l2", 2048, 128, 400, False), ("distmult", 512, 256, 800, False), ("complex", 1024, 256, 640, True),
    ("distmult", 1024, 64, 800, False), ("rotate", 768, 256, 400, False), ("rotate", 800, 256, 400, True),
    ("rotate", 1024, 192, 400, True), ("rotate", 2048, 128, 256, False)])
def test_keys_of_chunks_of_one_positive_sorted_beside_where_that_is_shorter(recorder, model, b, k, D, beside):
    waits = drive(recorder, f'''
assert Library({model!r}, b={b}, g=1, k={k}, D={D}).steps(1)[0] == 0
print(json.dumps(rec.recorder_waits()))
''')
    assert waits == (2 if beside else 0)


@pytest.mark.parametrize("shape", ["b=20_000, g=100, k=4, D=1024", "b=1 << 20, g=1 << 10, k=1024, D=4, relations=1_000_000"])
def test_transr_steps_of_very_many_workgroups(recorder, shape):
    """Workspaces of 80 and 60 GB: more workgroups of the relation update, or of the projections, than one dimension of a grid
    takes."""
    rc, events = drive(recorder, f'''
print(json.dumps(Library("transr", {shape}).steps(1)))
''')
    assert not [e for e in events if e.startswith("refused")] and rc == 0


@pytest.mark.parametrize("model,b,g,k,D,most", [("rotate", 1024, 1, 256, 400, 1.4e9),      # 118 M floats of partial rows
                                                ("transe_l1", 1024, 8, 256, 400, 0.4e9),   # 26 M floats
                                                ("rotate", 1024, 1024, 1024, 1024, 0.5e9)])  # 256 MB of them, not 0.5 GB
def test_workspace_holds_the_partial_rows_that_a_step_can_write(recorder, model, b, g, k, D, most):
    size = drive(recorder, f'''
print(json.dumps(lib.kge_workspace_bytes(Library({model!r}, b={b}, g={g}, k={k}, D={D}).ctx)))
''')
    assert size < most


@pytest.mark.parametrize("options,mega", [("", 675), ("adv_temperature=1.0, ", 1187), ("loss=1, ", 1187), ("D=132, ", 1226)])
def test_transr_workspace_holds_what_its_steps_keep(recorder, options, mega):
    """b 1024, k 1024, D 128: V takes 537 MB.  Projections (as much again) only where there are steps that keep them; the gradients of
    the positives in parts of 16 rows (35 MB) only where a step writes such parts, of 64 rows (9 MB) elsewhere."""
    size = drive(recorder, f'''
print(json.dumps(lib.kge_workspace_bytes(Library("transr", b=1024, g=1024, k=1024, **dict(dict(D=128), **dict({options}))).ctx)))
''')
    assert 0.99 * mega < size / 1e6 < mega, size
