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
    def __init__(self, model, b=64, g=16, k=24, D=64, **kw):
        m = MODELS.index(model)
        rel = {"rotate": D // 2, "rescal": D * D, "transr": D + D * D}.get(model, D)
        self.b, self.g, self.k = b, g, k
        cfg = Config(model=m, num_entities=1000, num_relations=20, ent_dim=D, rel_dim=rel, max_batch=b, max_neg_per_chunk=k,
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
    first, second = drive(recorder, f'''
lib_ = Library({model!r}, g={chunk})
first, second = lib_.steps(5), lib_.steps(20)
assert first[0] == 0 and second[0] == 0
print(json.dumps([first[1], second[1]]))
''')
    loaded = {e.split()[1] for e in first if e.startswith("kernel")}
    new = [e for e in second if e.startswith("kernel") and e.split()[1] not in loaded]
    assert any(e.startswith("graph") for e in second)
    assert loaded and not new, new
