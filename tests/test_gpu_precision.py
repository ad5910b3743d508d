"""Gradients of one training step against 64-bit autograd, on tables whose coordinates are multiples of a power of two, few
enough bits that rows o, differences and scores are exact in 32 bits.  What is left is the error of the coefficients, of the
sums and of the directions, and the limits below are the roundings on that way.  With an accumulator that starts at zero
Adagrad leaves S = g^2, so |g| can be read back for every element of the tables."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -24  # largest relative error of one rounding to 32 bits


@pytest.fixture(scope="module")
def kge():
    import paper_2004_08532_amd as k
    return k


def score64(model, E, R, h, r, x):
    """Scores of (h, r, x) over the last dimension, without the margin: minus the distance.  (Tail corrupted.)"""
    if model == "transr":
        D = E.shape[1]
        M = R[r][..., D:].reshape(*r.shape, D, D)
        q = torch.matmul(M, (E[h] - E[x]).unsqueeze(-1)).squeeze(-1) + R[r][..., :D]
        return -(q * q).sum(-1)
    q = E[h] + R[r] - E[x]
    if model == "transe_l1":
        return -q.abs().sum(-1)
    return -(q * q).sum(-1).sqrt()


def gradients64(model, E, R, h, r, t, neg, chunk, gamma, alpha, loss):
    E, R = (torch.from_numpy(x).double().requires_grad_() for x in (E, R))
    h, r, t, neg = (torch.from_numpy(x) for x in (h, r, t, neg))
    k = neg.shape[1]
    fp = gamma + score64(model, E, R, h, r, t)
    rows = neg.repeat_interleave(chunk, 0)
    f = gamma + score64(model, E, R, h[:, None].expand(-1, k), r[:, None].expand(-1, k), rows)
    w = torch.softmax(alpha * f.detach(), 1) if alpha > 0 else torch.full_like(f, 1.0 / k)
    if loss == "ranking":
        total = (w * torch.relu(gamma - fp[:, None] + f)).sum()
    else:
        total = torch.nn.functional.softplus(-fp).sum() + (w * torch.nn.functional.softplus(f)).sum()
    (total / h.shape[0]).backward()
    return E.grad.abs().numpy(), R.grad.abs().numpy()


def gradients(kge, model, E, R, h, r, t, neg, chunk, gamma, alpha, loss):
    b, k = h.shape[0], neg.shape[1]
    ctx = kge.KgeContext(model, E.shape[0], R.shape[0], E.shape[1], R.shape[1], max_batch=b, max_neg_per_chunk=k,
                         max_chunks=b // chunk, adv_temperature=alpha, loss=loss)
    dE, dR = (torch.from_numpy(x.copy()).cuda() for x in (E, R))
    sE, sR = torch.zeros_like(dE), torch.zeros_like(dR)
    h, r, t, neg = (torch.from_numpy(x).cuda() for x in (h, r, t, neg.reshape(-1)))
    try:
        ctx.train_step(dE, sE, dR, sR, h, r, t, neg, k, chunk, 0, gamma, 0.1)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    return sE.double().sqrt().cpu().numpy(), sR.double().sqrt().cpu().numpy()


def worst_row(got, want):
    """Largest relative error (2-norms) of a row."""
    size = np.linalg.norm(want, axis=1)
    err = np.linalg.norm(got - want, axis=1)
    assert not err[size == 0].any()
    return float((err[size > 0] / size[size > 0]).max())


# uniform weights, rows of up to 128 floats: units; others: products of two, three and four column tiles, W from the loss kernel or not
@pytest.mark.parametrize("D,k,alpha", [(100, 70, 0.0), (32, 256, 0.0), (136, 33, 0.0), (32, 70, 0.5), (48, 40, 0.5), (100, 70, 0.5)])
def test_transr_rows_close_to_each_other(kge, D, k, alpha):
    """Every o is within a hundredth of its length of every projection, as in a trained table; items of 17, 32, 33 and 97
    positives (sums or products in 64 bits) and of 5 (sums).  No term o - P may lose digits to the length of o and P."""
    rng = np.random.default_rng(3)
    runs = [97, 33, 5, 32, 17]
    g = sum(runs)
    r = rng.permutation(np.repeat(np.arange(len(runs)), runs))
    E = (1 + rng.integers(-16, 17, (2 * g + k, D)) / 4096).astype(np.float32)
    R = np.zeros((len(runs), D + D * D), np.float32)
    R[:, :D] = rng.integers(-4, 5, (len(runs), D)) / 4096
    R[:, D:] = np.eye(D).reshape(-1)
    ids = rng.permutation(2 * g + k)
    args = (E, R, ids[:g], r, ids[g:2 * g], ids[2 * g:].reshape(1, k), g, 0.5, alpha, "logistic")
    (gE, gR), (wE, wR) = gradients(kge, "transr", *args), gradients64("transr", *args)
    err = worst_row(gE, wE), worst_row(gR[:, :D], wR[:, :D])
    print("\n[precision] transr", D, k, alpha, "entities %.1e translations %.1e" % err)
    # coefficients: hardware exp2 and reciprocal of an argument below 1, four roundings; terms and their sum (errors of
    # either sign, so that the norm of a row has that of its largest terms), Adagrad's square and its root.  Softmax weights, with
    # scores within 0.01 of each other: another exp2 (2), its sum (3) and division (2), product with the coefficient (1)
    assert max(err) <= (16 if alpha == 0 else 24) * ULP, err


def far_negatives(model, b, g, k, D=8):
    """Positives of small scores, negatives (no two of them the same row) of scores between -36 and -24 at a margin of 12."""
    rng = np.random.default_rng(4)
    n = b // g * k
    if model == "transe_l2":  # one coordinate apart, so that distances are exact
        far = np.zeros((n, D))
        far[np.arange(n), rng.integers(0, D, n)] = rng.integers(38 * 4, 46 * 4, n) / 4
    else:
        step = {"transe_l1": [4.75, 5.0, 5.25, 5.5], "transr": [2.0, 2.25, 2.5]}[model]
        far = rng.choice(step, (n, D)) * rng.choice([-1.0, 1.0], (n, D))
    E = np.concatenate([np.zeros((b, D)), np.zeros((b, D)), far]).astype(np.float32)
    E[np.arange(b, 2 * b), rng.integers(0, D, b)] = 0.25
    R = np.zeros((3, D + D * D if model == "transr" else D), np.float32)
    if model == "transr":
        R[:, D:] = np.eye(D).reshape(-1)
    return E, R, np.arange(b), rng.integers(0, 3, b), np.arange(b, 2 * b), np.arange(2 * b, 2 * b + n).reshape(b // g, k), g, 12.0


@pytest.mark.parametrize("k", [1024, 1056])
@pytest.mark.parametrize("model,g,alpha", [("transe_l1", 2, 0.0), ("transe_l1", 2, 0.5), ("transe_l1", 1, 0.0),
                                           ("transe_l1", 1, 0.5), ("transe_l2", 1, 0.5), ("transr", 2, 0.0)])
def test_coefficients_of_far_negatives(kge, model, g, alpha, k):
    """W = w sigmoid(f) / b of scores around -30, where the argument of the hardware exp2 has lost four bits."""
    args = far_negatives(model, 4, g, k) + (alpha, "logistic")
    err = worst_row(gradients(kge, model, *args)[0], gradients64(model, *args)[0])
    print("\n[precision] far negatives", model, g, alpha, k, "%.1f roundings" % (err / ULP))
    # rows of more than 1024 scores: library exp (2), division, weight, product with it (3), their sum over positives and
    # its square (2); softmax: exp (2), sum (3), division (1).  Others: and half an ulp of 36 log2(e) (27), reciprocal (2)
    assert err <= (14 if k > 1024 else 43) * ULP, err / ULP


@pytest.mark.parametrize("g", [1, 4])
def test_coefficients_are_divided_by_the_distance(kge, g):
    """TransE-L2 with the ranking loss, weights 1 / 256, distances 3, 5, 7 ...: the gradient of a corrupting row is the weight
    divided by the distance, rounded once, times the distance."""
    D, b, k = 8, 4, 64
    n = b // g * k
    d = (2 * np.arange(n) + 3).astype(np.float32)
    E = np.zeros((2 * b + n, D), np.float32)
    E[2 * b + np.arange(n), np.arange(n) % D] = d
    h, t = np.arange(b), np.arange(b, 2 * b)
    E[t, 0] = 1.0
    got = gradients(kge, "transe_l2", E, np.zeros((1, D), np.float32), h, np.zeros(b, np.int64), t,
                    np.arange(2 * b, 2 * b + n).reshape(b // g, k), g, 1024.0, 0.0, "ranking")[0]
    want = (np.float32(1 / (b * k)) / d * np.float32(g) * d) ** 2  # the state, in 32 bits
    assert np.array_equal(got[2 * b + np.arange(n), np.arange(n) % D], np.sqrt(want.astype(np.float64)))


@pytest.mark.parametrize("scale", [2.0 ** -140, 2.0 ** -100, 2.0 ** -70, 1.0, 2.0 ** 66])
@pytest.mark.parametrize("g", [1, 24])
def test_signs_of_small_and_large_differences(kge, g, scale):
    """TransE-L1: the gradient depends on the sign of o - n alone, however small or large the coordinates are (the smallest
    scale: differences below the normal numbers), 0 where they are equal."""
    D, b, k = 24, 48, 40
    rng = np.random.default_rng(6)
    E = (rng.integers(-8, 9, (2 * b + b // g * k, D)) * scale).astype(np.float32)
    R = (rng.integers(-2, 3, (3, D)) * scale).astype(np.float32)
    ids = rng.permutation(E.shape[0])
    args = (E, R, ids[:b], rng.integers(0, 3, b), ids[b:2 * b], ids[2 * b:].reshape(b // g, k), g, 64.0 * max(scale, 1.0), 0.0, "ranking")
    (gE, gR), (wE, wR) = gradients(kge, "transe_l1", *args), gradients64("transe_l1", *args)
    # sums of terms +-w and 0, w = 1 / (b k): one rounding per term of a sum that never passes 1 / b in a row of o
    for got, want in ((gE, wE), (gR, wR)):
        np.testing.assert_allclose(got, want, rtol=1e-5, atol=64 * ULP / b)


@pytest.mark.parametrize("b,g,k,D", [(1024, 1024, 1536, 36), (1000, 500, 1600, 104), (1056, 33, 1500, 64), (1024, 32, 1505, 100)])
def test_forward_product_of_many_tiles(kge, b, g, k, D):
    """Loss and gradients of steps of 1504 tiles of 32 x 32 and more (sums of products of parts of the operands) against 64 bits:
    ragged tiles, chunks of 32 rows, numbers at the end of the floats whose products are finite."""
    gen = np.random.default_rng(9)
    n = b // g * k
    E = gen.uniform(-0.5, 0.5, (2 * b + n, D)).astype(np.float32)
    E[b:, 0] = gen.uniform(1, 2, b + n) * 1e-28  # replaced and corrupting rows
    E[0, 0], E[g - 1, 0], E[b - 1, 0] = 3.4e38, -3.4e38, 3.4e38  # rounds to infinity in 8 bits
    ids = np.arange(2 * b + n)
    h, t, m = ids[:b], ids[b:2 * b], ids[2 * b:]
    x, c, y = (E[i].astype(np.float64) for i in (h, t, m))
    f = np.concatenate([x[i:i + g] @ y[i // g * k:(i // g + 1) * k].T for i in range(0, b, g)])
    fp = (x * c).sum(1)
    loss = np.logaddexp(0, -fp).mean() + np.logaddexp(0, f).mean()
    with np.errstate(over="ignore"):
        w = 1 / (1 + np.exp(-f)) / (b * k)
    dy = np.concatenate([w[i:i + g].T @ x[i:i + g] for i in range(0, b, g)])[:, 1:]
    ctx = kge.KgeContext("distmult", E.shape[0], 1, D, D, max_batch=b, max_neg_per_chunk=k, max_chunks=b // g)
    dev = lambda v: torch.from_numpy(v).cuda()
    dE, dR, out = dev(E.copy()), torch.ones((1, D), device="cuda"), torch.zeros(1, device="cuda")
    sE, sR = torch.zeros_like(dE), torch.zeros_like(dR)
    try:
        ctx.train_step(dE, sE, dR, sR, dev(h), dev(np.zeros(b, np.int64)), dev(t), dev(m), k, g, 0, 12.0, 0.1, loss_out=out)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    got = np.sqrt(sE[2 * b:, 1:].cpu().numpy().astype(np.float64))
    err = np.linalg.norm(got - np.abs(dy)) / np.linalg.norm(dy)
    print("\n[precision] forward product", b, g, k, D, "loss %.3g, gradients %.3g" % (out.item() / loss - 1, err))
    # a score of a few units is off by a few roundings, its coefficient (0.5 and less) by as much and by the 27 to 30 roundings of
    # its own, both at random signs; a gradient is a sum of g of them and a root of its square
    assert abs(out.item() / loss - 1) < 64 * ULP
    assert err < 64 * ULP


@pytest.mark.parametrize("k", [16, 40, 256])
def test_transr_sums_over_the_positives_of_a_unit(kge, k):
    """32 positives of one relation with the identity for its matrix, every o - P of one sign: V, the sum over the positives, is the
    gradient of a corrupting row, and dL/do, the sum over the corrupting rows, that of a kept entity."""
    rng = np.random.default_rng(7)
    g, D = 32, 64
    E = np.concatenate([rng.integers(8, 25, (g, D)), rng.integers(0, 17, (g, D)), -rng.integers(0, 9, (k, D))]).astype(np.float32) / 64
    R = np.zeros((1, D + D * D), np.float32)
    R[0, D:] = np.eye(D).reshape(-1)
    ids = np.arange(2 * g + k)
    args = (E, R, ids[:g], np.zeros(g, np.int64), ids[g:2 * g], ids[2 * g:].reshape(1, k), g, 9.0, 0.0, "logistic")
    got, want = gradients(kge, "transr", *args)[0], gradients64("transr", *args)[0]
    rms = lambda rows: float(np.sqrt(np.mean((got[rows] / want[rows] - 1) ** 2))) / ULP
    err = rms(ids[2 * g:]), rms(ids[:g])
    print("\n[precision] transr sums", k, "over positives %.2f, over corrupting rows %.2f roundings" % err)
    # summed in 64 bits; then the rounding of the sum (root mean square 0.4 of the largest one), of its square, and what is left of
    # those of the coefficients in a mean of 32, or of k (measured 0.50 to 0.55, 0.66 to 0.73).  One after the other in 32 bits the 32
    # terms alone leave 0.4 sqrt(32 / 3) = 1.3 (measured 1.5)
    assert err[0] < 0.8, err
    assert err[1] < 1.0, err
