"""fp32 products on the bf16 matrix cores, operands in three parts: errors small enough that none of the six products of parts that are
formed may be missing, infinities and NaN as in fp32, and the training steps that take them (k_gemm_split_fwd: 1504 tiles of 32 x 32
and more; k_transr_back and k_transr_mgrad: rows of more than 64 floats)."""
import numpy as np
import pytest
import torch

from harness import configs
from parity_util import Pair
from test_gpu_parity import ragged, run_steps
from test_gpu_precision import ULP, gradients, gradients64

F_RMS = 6.0  # root mean square of the scores below
# Error of a sum relative to the sums' root mean square.  Roundings of the sum and of the coefficient: measured 0.5e-7 (36 products) to
# 0.9e-7 (372); TransR, with the roundings of projections, coefficients and V: 1.4e-7 to 2.2e-7.  Without the smallest of the six
# products of parts: at least 1.8 times the limit (emulated)
LIMIT = 3e-7

gpu = pytest.mark.gpu


@pytest.fixture(scope="module")
def kge():
    import paper_2004_08532_amd as k
    return k


def bf16(x):
    return torch.from_numpy(x.astype(np.float32)).bfloat16().float().numpy()


def parts(x):
    p0 = bf16(x)
    p1 = bf16(x - p0)
    return p0, p1, bf16(x - p0 - p1)


def rows(gen, n, D):
    """Rows whose products of D terms have the root mean square F_RMS."""
    a = np.sqrt(3 * F_RMS / np.sqrt(D))
    return gen.uniform(-a, a, (n, D)).astype(np.float32)


@pytest.mark.parametrize("D", [64, 400])
def test_every_product_of_parts_matters(D):
    """Emulation: the six products in 64 bits, all of them and without each one in turn."""
    gen = np.random.default_rng(1)
    x, y = rows(gen, 200, D), rows(gen, 300, D)
    want = x.astype(np.float64) @ y.astype(np.float64).T
    kept = [(0, 0), (0, 1), (1, 0), (0, 2), (2, 0), (1, 1)]
    terms = {(i, j): parts(x)[i].astype(np.float64) @ parts(y)[j].astype(np.float64).T for i, j in kept}
    err = lambda left_out: np.sqrt(np.mean((sum(v for k, v in terms.items() if k != left_out) - want) ** 2)) / F_RMS
    assert err(None) < 0.1 * LIMIT
    assert min(err(k) for k in kept) > 1.8 * LIMIT, {k: err(k) for k in kept}


MARKED = 32  # positives of a chunk whose coefficients are read back


def marked_step(kge, b, g, k, D, change=None):
    """A DistMult step whose positives o = h and corrupting rows n are random in D floats.  MARKED positives of every chunk have a 1 in a
    column of their own behind these, where all other rows have zeros: there the gradient of a corrupting row is that positive's
    coefficient W alone.  Returns W / w and the scores in 64 bits, [chunk, marked positive, corrupting row], and the losses."""
    gen = np.random.default_rng(9)
    chunks = b // g
    n = chunks * k
    E = np.zeros((2 * b + n, D + MARKED), np.float32)
    E[:b, :D], E[2 * b:, :D] = rows(gen, b, D), rows(gen, n, D)
    marked = np.stack([np.sort(np.append(gen.choice(g - 1, MARKED - 1, replace=False), g - 1)) for _ in range(chunks)])
    E[(g * np.arange(chunks)[:, None] + marked).ravel(), D + np.tile(np.arange(MARKED), chunks)] = 1
    if change:
        change(E, marked)
    ids = np.arange(2 * b + n)
    dev = lambda v: torch.from_numpy(v).cuda()
    ctx = kge.KgeContext("distmult", E.shape[0], 1, D + MARKED, D + MARKED, max_batch=b, max_neg_per_chunk=k, max_chunks=chunks)
    dE, dR, out = dev(E.copy()), torch.ones((1, D + MARKED), device="cuda"), torch.zeros(1, device="cuda")
    sE, sR = torch.zeros_like(dE), torch.zeros_like(dR)
    try:
        ctx.train_step(dE, sE, dR, sR, dev(ids[:b]), dev(np.zeros(b, np.int64)), dev(ids[b:2 * b]), dev(ids[2 * b:]), k, g, 0, 12.0, 0.1,
                       loss_out=out)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    got = np.sqrt(sE[2 * b:, D:].double().cpu().numpy()).reshape(chunks, k, MARKED).transpose(0, 2, 1) * (b * k)
    with np.errstate(invalid="ignore"):
        f = np.stack([E[c * g:(c + 1) * g, :D].astype(np.float64) @ E[2 * b + c * k:2 * b + (c + 1) * k, :D].astype(np.float64).T
                      for c in range(chunks)])
        loss = np.log(2) + np.logaddexp(0, f).mean()  # (scores of positives: 0)
    return got, np.take_along_axis(f, marked[:, :, None], 1), out.item(), loss


SHAPES = [(1000, 1000, 1504, 64), (1000, 500, 1600, 372), (1056, 33, 1500, 100), (1024, 32, 1505, 200), (1513, 89, 1000, 36)]


@gpu
@pytest.mark.parametrize("b,g,k,D", SHAPES)
def test_scores_behind_the_coefficients(kge, b, g, k, D):
    got, f, loss, want_loss = marked_step(kge, b, g, k, D)
    use = (f < 0) & (f > -12)  # (further out W says little of f in 32 bits, or its square is small)
    err = np.log(got[use] / (1 - got[use])) - f[use]
    rms = np.sqrt(np.mean(err ** 2)) / F_RMS
    print("\n[precision] split product", b, g, k, D, "scores %.2g, loss %.2g" % (rms, loss / want_loss - 1))
    assert rms < LIMIT
    # softplus by hardware exp2 and log2, two roundings each, at random signs, and the roundings of the sums (measured: up to 1.7)
    assert abs(loss / want_loss - 1) < 16 * ULP


@gpu
@pytest.mark.parametrize("b,g,k,D", SHAPES[1:4])
def test_infinities_and_nan(kge, b, g, k, D):
    """An infinity in a row makes its scores infinities of either sign, a NaN makes them NaN, and no other score changes."""
    def change(E, marked):
        chunk0, chunk1 = 2 * b, 2 * b + k
        E[chunk0 + 5, 3], E[chunk0 + k - 1, D - 1] = np.inf, -np.inf
        E[g + marked[1, 7], 0], E[g + marked[1, 8], D - 1] = -np.inf, np.inf
        E[chunk1 + 2, 1] = np.nan

    got, f, _, _ = marked_step(kge, b, g, k, D, change)
    assert np.isnan(f[1, :, 2]).all() and np.isnan(f).sum() == MARKED and np.isinf(f).sum() == 2 * MARKED + 2 * (k - 1)
    assert np.isnan(got[1, :, 2]).all() and np.isnan(got).sum() == MARKED
    for sign, w in ((np.inf, 1.0), (-np.inf, 0.0)):
        assert (f == sign).sum() > 20
        np.testing.assert_allclose(got[f == sign], w, rtol=4 * ULP)
    use = np.isfinite(f) & (f < 0) & (f > -12)
    err = np.log(got[use] / (1 - got[use])) - f[use]
    assert np.sqrt(np.mean(err ** 2)) / F_RMS < LIMIT


@gpu
@pytest.mark.parametrize("loss", ["logistic", "adv", "ranking"])
@pytest.mark.parametrize("b,g,k,D", [(1035, 345, 1500, 72), (1024, 32, 1505, 104)])
@pytest.mark.parametrize("model", ["transe_l2", "distmult", "complex"])
def test_training_steps(kge, model, b, g, k, D, loss):
    """Coefficients in the epilogue, scores and distances for the loss kernel; tiles of 64 and of 32 rows; several K blocks, a ragged
    last one."""
    w = ragged(model, n_entities=60_001, n_triples=20_000, batch=b, chunk=g, neg_per_chunk=k, ent_dim=D, rel_dim=D, steps=1,
               adv_temperature=1.0 if loss == "adv" else 0.0, loss="ranking" if loss == "ranking" else "logistic")
    p = Pair(w, kge)
    try:
        run_steps(p, configs.BatchStream(w), 1)
    finally:
        p.close()


@gpu
@pytest.mark.parametrize("D,k", [(68, 70), (100, 128), (128, 65), (136, 96)])
def test_transr_gradients(kge, D, k):
    """Random matrices and rows, scores of a few units; items of 1, 5, 17, 33 and 97 positives: entities (the back-projection), translations
    and matrices (sums over corrupting rows and positives), each as a whole."""
    gen = np.random.default_rng(5)
    runs = [97, 33, 5, 1, 17]
    g = sum(runs)
    r = gen.permutation(np.repeat(np.arange(len(runs)), runs))
    E = gen.uniform(-1, 1, (2 * g + k, D)).astype(np.float32)
    R = gen.uniform(-1, 1, (len(runs), D + D * D)).astype(np.float32)
    R[:, D:] *= 3 / D  # a distance^2 of about 2 D / 3 * 3 / D
    ids = gen.permutation(2 * g + k)
    R[:, :D] *= 0.1
    args = (E, R, ids[:g], r, ids[g:2 * g], ids[2 * g:].reshape(1, k), g, 2.0, 0.0, "logistic")
    (gE, gR), (wE, wR) = gradients(kge, "transr", *args), gradients64("transr", *args)
    err = [float(np.linalg.norm(x - y) / np.linalg.norm(y)) for x, y in ((gE, wE), (gR[:, :D], wR[:, :D]), (gR[:, D:], wR[:, D:]))]
    print("\n[precision] transr", D, k, "entities %.1e translations %.1e matrices %.1e" % tuple(err))
    assert max(err) < LIMIT, err


@gpu
@pytest.mark.parametrize("D,k", [(20, 40), (68, 129), (100, 70), (112, 33)])
def test_transr_infinite_corrupting_row(kge, D, k):
    """An infinity in a corrupting row makes its scores minus infinity: nothing of it in the loss or in the other rows' gradients,
    whether or not the columns of the projections are a multiple of the tiles."""
    gen = np.random.default_rng(8)
    g = 40
    E = gen.uniform(-1, 1, (2 * g + k, D)).astype(np.float32)
    R = gen.uniform(-1, 1, (3, D + D * D)).astype(np.float32)
    R[:, :D] *= 0.1
    R[:, D:] *= 3 / D  # scores of a few units, as above
    ids = np.arange(2 * g + k)
    bad = 2 * g + k - 2
    E[bad, D - 1] = np.inf
    h, r, t, neg = ids[:g], gen.integers(0, 3, g), ids[g:2 * g], ids[2 * g:]
    dev = lambda v: torch.from_numpy(v).cuda()
    ctx = kge.KgeContext("transr", *E.shape[:1], 3, D, D + D * D, max_batch=g, max_neg_per_chunk=k, max_chunks=1)
    dE, dR, out = dev(E.copy()), dev(R.copy()), torch.zeros(1, device="cuda")
    sE = torch.zeros_like(dE)
    try:
        ctx.train_step(dE, sE, dR, torch.zeros_like(dR), dev(h), dev(r), dev(t), dev(neg), k, g, 0, 2.0, 0.1, loss_out=out)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    others = neg[neg != bad]
    E64, R64 = (torch.from_numpy(x).double().requires_grad_() for x in (E, R))
    M = R64[r, D:].reshape(g, D, D)
    o = (M @ E64[h].unsqueeze(-1)).squeeze(-1) + R64[r, :D]
    fp = 2.0 - (o - (M @ E64[t].unsqueeze(-1)).squeeze(-1)).square().sum(-1)
    f = 2.0 - (o[:, None] - torch.einsum("gde,ke->gkd", M, E64[others])).square().sum(-1)
    loss = (torch.nn.functional.softplus(-fp).sum() + torch.nn.functional.softplus(f).sum() / k) / g
    loss.backward()
    assert abs(out.item() / loss.item() - 1) < 64 * ULP  # (roundings of the scores, a few units each)
    got, want = sE[others].double().sqrt().cpu().numpy(), E64.grad[others].abs().numpy()
    assert np.linalg.norm(got - want) / np.linalg.norm(want) < LIMIT
