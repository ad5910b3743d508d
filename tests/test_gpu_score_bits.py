"""The bits of the positives' scores.  The rank of a positive among candidates that tie with it hangs on the last bit of its score,
so the order of the sum and which product is fused with its addition are part of what the library computes: here they are
formed one operation at a time (a fused multiply-add in 64 bits of significand, then rounded) and compared exactly.  RotatE's sines and
cosines are the GPU's; TransR has another kernel."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

F = np.float32
GAMMA = 12.0


@pytest.fixture(scope="module")
def kge():
    import paper_2004_08532_amd as k
    return k


def fma(x, y, z):
    return (np.longdouble(1) * x * y + z).astype(F)


def square4(x):
    return fma(x[3], x[3], fma(x[2], x[2], fma(x[0], x[0], x[1] * x[1])))


def wave_sum(lanes):
    s = lanes
    for o in (32, 16, 8, 4, 2, 1):
        s = s + s[:, np.arange(64) ^ o]
    return s[:, 0]


def pieces(x):
    """Rows -> for every round of 64 lanes the four floats [row, lane] of each lane's 16 bytes, zeros past the end, and the lanes."""
    b, n = x.shape
    rounds = -(-n // 256)
    y = np.zeros((b, 256 * rounds), F)
    y[:, :n] = x
    return [[y[:, 256 * i + e:256 * (i + 1):4] for e in range(4)] for i in range(rounds)]


def complex_product(a, r, head):
    (are, aim), (rre, rim) = np.split(a, 2, 1), r
    ri = -rim if head else rim
    return fma(are, rre, -(aim * ri)), fma(are, ri, aim * rre)


def scores(model, E, R, h, r, t, head):
    a, c = (E[t], E[h]) if head else (E[h], E[t])
    acc = np.zeros((h.size, 64), F)
    if model in ("complex", "rotate"):
        if model == "rotate":
            th = torch.from_numpy(R[r]).cuda()
            rel = torch.cos(th).cpu().numpy(), torch.sin(th).cpu().numpy()
        else:
            rel = np.split(R[r], 2, 1)
        ore, oim = complex_product(a, rel, head)
        cre, cim = np.split(c, 2, 1)
        for x, y, u, v in zip(*(pieces(z) for z in (ore, oim, cre, cim))):
            for e in range(4):
                if model == "complex":
                    acc = acc + fma(x[e], u[e], y[e] * v[e])
                else:
                    qre, qim = x[e] - u[e], y[e] - v[e]
                    acc = acc + np.sqrt(fma(qre, qre, qim * qim))
    else:
        o = a * R[r] if model == "distmult" else a - R[r] if head else a + R[r]
        for i, (x, y) in enumerate(zip(pieces(o), pieces(c))):
            u = [x[e] - y[e] for e in range(4)]
            if model == "transe_l2":
                first = fma(u[0], u[0], u[1] * u[1]) if i == 0 else fma(u[1], u[1], fma(u[0], u[0], acc))
                acc = fma(u[3], u[3], fma(u[2], u[2], first))
            for e in range(4):
                if model == "distmult":
                    acc = fma(x[e], y[e], acc)
                elif model == "transe_l1":
                    acc = acc + np.abs(u[e])
    s = wave_sum(acc)
    assert s.dtype == F
    return s if model in ("distmult", "complex") else F(GAMMA) - (np.sqrt(s) if model == "transe_l2" else s)


@pytest.mark.parametrize("D", [8, 72, 256, 264, 520, 1024])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("model", ["transe_l2", "transe_l1", "distmult", "complex", "rotate"])
def test_bits_of_the_scores_of_positives(kge, model, side, D):
    gen = np.random.default_rng(D + side)
    b, g, k = 300, 100, 8
    Dr = D // 2 if model == "rotate" else D
    E, R = (gen.uniform(-0.7, 0.7, s).astype(F) for s in ((500, D), (9, Dr)))
    h, r, t = (gen.integers(0, n, b) for n in (500, 9, 500))
    neg = gen.integers(0, 500, b // g * k)
    dev = lambda x: torch.from_numpy(x).cuda()
    pos, ng = torch.empty(b, device="cuda"), torch.empty((b, k), device="cuda")
    ctx = kge.KgeContext(model, 500, 9, D, Dr, max_batch=b, max_neg_per_chunk=k, max_chunks=b // g)
    try:
        ctx.score(dev(E), dev(R), dev(h), dev(r), dev(t), dev(neg), k, g, side, GAMMA, pos, ng)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    want = scores(model, E, R, h, r, t, side == 1)
    assert np.array_equal(pos.cpu().numpy().view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("D", [8, 256, 260, 400])
def test_bits_of_the_scores_of_positives_rescal(kge, D):
    """Identity matrices: o is the head's row."""
    gen = np.random.default_rng(D)
    b = 256
    E = gen.uniform(-0.7, 0.7, (500, D)).astype(F)
    R = np.eye(D, dtype=F).reshape(1, -1)
    h, t = gen.integers(0, 500, b), gen.integers(0, 500, b)
    dev = lambda x: torch.from_numpy(x).cuda()
    pos, ng = torch.empty(b, device="cuda"), torch.empty((b, 8), device="cuda")
    ctx = kge.KgeContext("rescal", 500, 1, D, D * D, max_batch=b, max_neg_per_chunk=8, max_chunks=1)
    try:
        ctx.score(dev(E), dev(R), dev(h), dev(np.zeros(b, np.int64)), dev(t), dev(t[:8]), 8, b, 0, GAMMA, pos, ng)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    acc = np.zeros((b, 64), F)
    for x, y in zip(pieces(E[h]), pieces(E[t])):
        first = fma(x[1], y[1], x[0] * y[0]) if D <= 256 else fma(x[0], y[0], x[1] * y[1])
        acc = acc + fma(x[3], y[3], fma(x[2], y[2], first))
    assert np.array_equal(pos.cpu().numpy().view(np.int32), wave_sum(acc).view(np.int32))


# (336, 336, 320 and 578 tiles of 64 x 64; fewer than 320 of them, or 1280 of 32 x 32, would be scored on 32 x 32)
@pytest.mark.parametrize("b,k,D", [(1000, 1300, 400), (1025, 1290, 36), (1020, 1280, 132), (1060, 2120, 4)])
@pytest.mark.parametrize("model", ["transe_l2", "distmult", "complex"])
def test_negative_scores_hang_on_the_pair_alone(kge, model, b, k, D):
    """One chunk is scored on tiles of 64 x 64, chunks of 20 (half of such tiles' rows would be missing) on tiles of 32 x 32: the
    same bits, and ranks, with blocks of K past the end, short last ones and ragged edges.  Candidates that are the replaced entity tie."""
    if model == "complex" and D % 8:
        D += 4
    gen = np.random.default_rng(3)
    n, g = 3000, 20
    b -= b % g
    E = torch.from_numpy(gen.uniform(-1, 1, (n, D)).astype(F)).cuda()
    R = torch.from_numpy(gen.uniform(-1, 1, (5, D)).astype(F)).cuda()
    h, t, neg = (torch.from_numpy(gen.integers(0, n, m)).cuda() for m in (b, b, k))
    neg[::7] = t[:neg[::7].numel()]
    r = torch.from_numpy(gen.integers(0, 5, b)).cuda()
    got = {}
    for chunk, ids in ((b, neg), (g, neg.repeat(b // g))):
        ctx = kge.KgeContext(model, n, 5, D, D, max_batch=b, max_neg_per_chunk=k, max_chunks=b // chunk)
        pos, out = torch.empty(b, device="cuda"), torch.empty((b, k), device="cuda")
        ranks = torch.empty(b, dtype=torch.int32, device="cuda")
        try:
            ctx.score(E, R, h, r, t, ids, k, chunk, 0, GAMMA, pos, out)
            ctx.rank(E, R, h, r, t, ids, k, chunk, 0, GAMMA, ranks)
            torch.cuda.synchronize()
        finally:
            ctx.close()
        got[chunk] = out.cpu().numpy(), ranks.cpu().numpy(), pos.cpu().numpy()
    np.testing.assert_array_equal(got[b][0], got[g][0])
    np.testing.assert_array_equal(got[b][1], got[g][1])
    np.testing.assert_array_equal(got[b][1], 1 + (got[b][0] > got[b][2][:, None]).sum(1))


@pytest.mark.parametrize("adv", [0.0, 1.0])
@pytest.mark.parametrize("model", ["transe_l2", "distmult"])
def test_training_steps_on_the_tiles_of_the_scores(kge, model, adv):
    """Coefficients with their loss, and scores and distances for the loss kernel, of 64 x 64 tiles in training steps."""
    from harness import configs
    from parity_util import Pair
    from test_gpu_parity import ragged, run_steps
    w = ragged(model, n_entities=60_001, n_triples=20_000, batch=1020, chunk=340, neg_per_chunk=1100, ent_dim=140, rel_dim=140, steps=1,
               adv_temperature=adv)
    p = Pair(w, kge)
    try:
        run_steps(p, configs.BatchStream(w), 1)
    finally:
        p.close()
