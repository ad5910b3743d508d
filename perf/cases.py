"""The work that programs give this library, as cases that can be timed and compared.

A case is one pass through the public entry points on tables and ids that are already on the GPU:

  kind "train"   kge_train_steps (a block of mini-batches staged ahead of time) or, with steps = 1, kge_train_step
                 (a training loop that makes one call per mini-batch); outputs: both tables, both optimizer states, losses
  kind "score"   kge_score of positives and their corrupted triples; outputs: the scores
  kind "rank"    kge_rank of positives against candidates, then kge_rank_metrics; outputs: ranks and metrics
  kind "sample"  kge_sample_steps, the ids of a block of mini-batches; outputs: the ids and sides

Letters: b positives per mini-batch in C chunks of g, k corrupting entities per chunk, D floats per entity row.  The
listed shapes are those of harness/configs.py and bench.py.  Tables and Adagrad accumulators are drawn as they look in
the middle of a training run (scores around the margin, accumulators of some hundred earlier updates), entity
degrees are Zipf-distributed as in harness/graphs.py, and ids come from kge_sample_steps.
"""
import functools
import math

import numpy as np
import torch

import paper_2004_08532_amd as kge
from harness import graphs, sampler

GAMMA, LR = 12.0, 0.1  # every configuration of this repository uses these

_DEFAULTS = dict(kind="train", model="transe_l2", entities=14_951, relations=1_345, zipf=1.0, dim=400, batch=1024,
                 chunk=128, k=256, degree=0, side="tail", steps=1, bf16=False, adv=0.0, loss="logistic", rowwise=False)


def _case(**kw):
    return dict(_DEFAULTS, **kw)


def listed():
    fb15k = dict(side="alternate")                                                      # FB15k-sized graph
    freebase = dict(entities=10_000_000, relations=14_824, batch=1000, chunk=1000, k=200)  # Freebase batch shape; the
    # table (16 GB, as much again for its state) is cut so that several states fit, and is still far beyond every cache
    return [
        # the smallest mini-batch in use, one call per step on the default stream: a first program, or a debugging run
        _case(name="tiny-step", entities=1_000, relations=20, zipf=1.1, dim=64, batch=256, chunk=32, k=64),
        # small benchmark graphs, where most published comparisons are made
        _case(name="fb15k-distmult", model="distmult", steps=100, **fb15k),
        # models with a matrix per relation, at the row lengths such models are trained with
        _case(name="fb15k-rescal", model="rescal", dim=200, steps=50, **fb15k),
        _case(name="fb15k-transr", model="transr", dim=100, steps=20, **fb15k),
        # the same graph with negatives drawn per positive, the comparison run for joint sampling
        _case(name="fb15k-independent", chunk=1, steps=4, **fb15k),
        # mid-sized graph, self-adversarial weights, negatives in proportion to degree
        _case(name="medium-rotate", model="rotate", entities=2_500_000, relations=800, zipf=0.9, degree=256, adv=1.0,
              steps=50),
        # large batches in mixed precision
        _case(name="large-bf16", entities=5_000_000, relations=800, zipf=0.9, batch=2048, chunk=256, k=1024, bf16=True,
              steps=50),
        # the headline workload of bench.py
        _case(name="freebase-transe", steps=100, **freebase),
        # the other common way to train there: one accumulator per row to save memory, one call per mini-batch
        _case(name="freebase-complex-rowwise", model="complex", rowwise=True, **freebase),
        # margin-based training of the oldest model at odd sizes: nothing a multiple of a tile
        _case(name="ragged-transe_l1", model="transe_l1", entities=40_943, relations=18, dim=212, batch=690, chunk=115, k=93,
              loss="ranking", side="alternate", steps=4),
        # link-prediction evaluation, 1000 uniform and 1000 degree-proportional candidates for every positive
        _case(name="rank-protocol2", kind="rank", k=2000, degree=1000, **{n: v for n, v in freebase.items() if n != "k"}),
        # step 1 of the loop for a block of steps
        _case(name="sample-1000", kind="sample", steps=1000, **freebase),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    """One more case: kind, model and options at the rates of use, sizes log-uniform, odd ones included."""
    c = _case(kind=rng.choice(["train"] * 7 + ["score", "rank", "sample"]))
    c["model"] = rng.choice(["transe_l2", "transe_l2", "distmult", "complex", "rotate", "rotate", "transe_l1", "rescal", "transr"])
    matrix, products = c["model"] in ("rescal", "transr"), c["model"] in ("transe_l2", "distmult", "complex")
    c["relations"] = _log(rng, 10, 1_500 if matrix else 15_000)
    unit = 8 if c["model"] in ("complex", "rotate") else 4
    c["dim"] = unit * _log(rng, 32 // unit, {"rescal": 256, "transr": 128}.get(c["model"], 800) // unit)
    c["entities"] = _log(rng, 1_000, min(10_000_000, 4_000_000_000 // c["dim"]))
    while math.gcd(c["entities"], 2_654_435_761) != 1:
        c["entities"] += 1
    c["zipf"] = rng.choice([0.9, 1.0, 1.1])
    c["chunk"] = _log(rng, 16, 1_000)
    c["batch"] = c["chunk"] * _log(rng, max(1, 200 // c["chunk"]), max(1, 2_048 // c["chunk"]))
    c["k"] = _log(rng, 16, 2_000 if c["kind"] == "rank" else 1_024)
    if c["kind"] == "train" and not matrix and rng.random() < 0.08:  # negatives of each positive's own
        c["chunk"], c["batch"], c["k"], c["dim"] = 1, _log(rng, 64, 1_024), _log(rng, 16, 256), min(c["dim"], 400)
    c["degree"] = rng.choice([0, 0, c["k"] // 2, c["k"]])
    c["side"] = rng.choice(["tail", "head", "alternate"])
    if c["kind"] == "train":
        c["adv"] = rng.choice([0.0, 0.0, 1.0])
        c["loss"] = rng.choice(["logistic"] * 5 + ["ranking"])
        c["rowwise"] = not matrix and rng.random() < 0.2
        c["steps"] = rng.choice([1, _log(rng, 4, 100), _log(rng, 4, 100)])
        if c["model"] == "transe_l1":  # a gradient of signs: what rounding changes in one step grows fast over many
            c["steps"] = min(c["steps"], 4)
    if c["kind"] == "sample":
        c["steps"] = _log(rng, 1, 1_000)
    c["bf16"] = products and c["kind"] == "train" and rng.random() < 0.25
    while c["kind"] != "sample" and _cost(c) > 8e-3:  # no more than the largest listed case
        if c["steps"] > 1:
            c["steps"] = c["steps"] * 3 // 4
        else:
            c["k"] = max(16, c["k"] * 3 // 4)
            c["degree"] = min(c["degree"], c["k"])
            if c["k"] == 16:
                break
    return c


# ---------------------------------------------------------------------------------------------------------------


def _rel_dim(c):
    D = c["dim"]
    return {"rotate": D // 2, "rescal": D * D, "transr": D + D * D}.get(c["model"], D)


def _draw_zipf(n, count, s, g):
    """Ids of `count` Zipf-distributed endpoints among n (the continuous inverse of the rank's distribution), spread over
    the table by the bijection of harness/graphs.py."""
    u = torch.rand(count, dtype=torch.float64, device="cuda", generator=g)
    rank = (n + 1.0) ** u if s == 1.0 else (((n + 1.0) ** (1 - s) - 1) * u + 1) ** (1 / (1 - s))
    rank = (rank.to(torch.int64) - 1).clamp_(0, n - 1)
    return (rank * graphs._SCRAMBLE_A + graphs._SCRAMBLE_B) % n


def _uniform(shape, lo, hi, g):
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=g)


def _tables(c, g):
    """Entity and relation tables with scores around the margin, as trained embeddings give."""
    D, m = c["dim"], c["model"]
    a = {"transe_l2": GAMMA / math.sqrt(D), "transe_l1": (GAMMA + 2) / D, "rotate": (GAMMA + 2) / D, "rescal": 0.3,
         "transr": 3.0 / math.sqrt(D)}.get(m, 0.8)
    E = _uniform((c["entities"], D), -a, a, g)
    if m == "rotate":
        return E, _uniform((c["relations"], D // 2), -math.pi, math.pi, g)
    if m in ("rescal", "transr"):  # entries of the matrices: rows keep their length
        R = _uniform((c["relations"], _rel_dim(c)), -2 / math.sqrt(D), 2 / math.sqrt(D), g)
        if m == "transr":
            R[:, :D].mul_(a * math.sqrt(D) / 2)
        return E, R
    return E, _uniform((c["relations"], D), -a, a, g)


def _accumulator(c, table, relation, g):
    """Adagrad state after a few hundred updates by gradients of the size this model has at this batch size."""
    per_positive = {"transe_l2": 1 / math.sqrt(c["dim"]), "transe_l1": 1.0, "rotate": 0.7, "rescal": 0.04 if relation else 0.2,
                    "transr": 0.2 if relation else 0.8}.get(c["model"], 0.2)
    if relation:  # a relation row meets many positives of a mini-batch
        per_positive *= 1 + c["batch"] / c["relations"]
    s = 400 * (per_positive / c["batch"]) ** 2
    return _uniform((table.shape[0],) if c["rowwise"] else table.shape, 0.5 * s, 1.5 * s, g)


@functools.lru_cache(maxsize=1)
def _stream():
    """The stream a training program keeps for its steps (kge_train_steps replays HIP graphs there)."""
    return torch.cuda.Stream()


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n_chunks, b, k, steps = c["batch"] // c["chunk"], c["batch"], c["k"], c["steps"]
    n = 1_000_000 if c["kind"] == "sample" else 2 * b * max(steps, 10)
    triples = torch.stack([_draw_zipf(c["entities"], n, c["zipf"], g), _draw_zipf(c["relations"], n, 1.0, g),
                           _draw_zipf(c["entities"], n, c["zipf"], g)], dim=1).contiguous()
    ids = [torch.empty((steps, b), dtype=torch.int64, device="cuda") for _ in range(3)]
    ids.append(torch.empty((steps, n_chunks * k), dtype=torch.int64, device="cuda"))
    s = dict(kind=c["kind"], ids=ids, k=k, chunk=c["chunk"], batch=b)
    sampling = (seed, triples, c["entities"], b, n_chunks, k, c["degree"], c["side"], 0, steps, *ids)
    if c["kind"] == "sample":
        s["sides"] = torch.empty(steps, dtype=torch.int32, device="cuda")
        s["sampling"] = (*sampling, s["sides"])
        return s
    kge.kge_sample_steps(*sampling)
    s["side"] = sampler.side_of_step(c["side"], 0)
    s["E"], s["R"] = _tables(c, g)
    s["ctx"] = kge.KgeContext(c["model"], c["entities"], c["relations"], c["dim"], _rel_dim(c), max_batch=b,
                              max_neg_per_chunk=k, max_chunks=n_chunks, gemm_input=int(c["bf16"]),
                              adv_temperature=c["adv"], adagrad_mode=int(c["rowwise"]), loss=c["loss"])
    if c["kind"] == "train":
        s["SE"], s["SR"] = _accumulator(c, s["E"], False, g), _accumulator(c, s["R"], True, g)
        s["losses"] = torch.zeros(steps, dtype=torch.float32, device="cuda")
        s["sides"] = None if c["side"] == "tail" else np.array([sampler.side_of_step(c["side"], i) for i in range(steps)], dtype=np.int32)
    elif c["kind"] == "score":
        s["pos"] = torch.empty(b, dtype=torch.float32, device="cuda")
        s["neg"] = torch.empty((b, k), dtype=torch.float32, device="cuda")
    else:
        s["ranks"] = torch.empty(b, dtype=torch.int32, device="cuda")
        s["metrics"] = torch.empty(5, dtype=torch.float64, device="cuda")
    return s


def run(state):
    s = state
    h, r, t, neg = s["ids"]
    if s["kind"] == "sample":
        kge.kge_sample_steps(*s["sampling"])
        return {"h": h, "r": r, "t": t, "neg": neg, "sides": s["sides"]}
    if s["kind"] == "score":
        s["ctx"].score(s["E"], s["R"], h[0], r[0], t[0], neg[0], s["k"], s["chunk"], s["side"], GAMMA, s["pos"], s["neg"])
        return {"pos": s["pos"], "neg": s["neg"]}
    if s["kind"] == "rank":
        s["ctx"].rank(s["E"], s["R"], h[0], r[0], t[0], neg[0], s["k"], s["chunk"], s["side"], GAMMA, s["ranks"])
        kge.kge_rank_metrics(s["ranks"], s["metrics"])
        return {"ranks": s["ranks"], "metrics": s["metrics"]}
    tables = s["E"], s["SE"], s["R"], s["SR"]
    if h.shape[0] == 1:
        s["ctx"].train_step(*tables, h[0], r[0], t[0], neg[0], s["k"], s["chunk"], s["side"], GAMMA, LR, loss_out=s["losses"])
    else:
        s["ctx"].train_steps(*tables, h, r, t, neg, s["k"], s["chunk"], s["sides"], GAMMA, LR, loss_out=s["losses"],
                             stream=_stream())
    return {"E": s["E"], "SE": s["SE"], "R": s["R"], "SR": s["SR"], "losses": s["losses"]}


# ---------------------------------------------------------------------------------------------------------------


def _distinct(n, s, count):
    """Expected number of distinct ids among `count` Zipf-distributed ones (s = 0: uniform) of n."""
    if count == 0:
        return 0.0
    edges = np.unique(np.floor(np.geomspace(1, n + 1, 4000)))  # blocks of ranks of nearly the same probability
    mid, width = (edges[:-1] + edges[1:] - 1) / 2, np.diff(edges)
    p = mid ** -s
    p /= (p * width).sum()
    return float((width * -np.expm1(count * np.log1p(-np.minimum(p, 1 - 1e-12)))).sum())


def work(case):
    """Bytes: a training step reads and writes every distinct row and its accumulator once and reads its ids; scoring
    reads the distinct rows and writes the scores; sampling reads the triples and writes the ids.  Flops: the chunked
    products (2bkD forward, 4bkD backward; b k D^2 with a matrix per relation) or the elementwise reductions in their
    place, and the matrix-vector products of the positives."""
    c = case
    D, Dr, b, k, steps = c["dim"], _rel_dim(c), c["batch"], c["k"], c["steps"]
    n_neg = b // c["chunk"] * k
    ids = 8 * (3 * b + n_neg)
    if c["kind"] == "sample":
        return {"bytes": steps * (24 * b + ids + 4), "flops": 0}
    degree = b // c["chunk"] * c["degree"]
    rows = min(c["entities"], _distinct(c["entities"], c["zipf"], 2 * b) + _distinct(c["entities"], 0.0, n_neg - degree))
    rels = _distinct(c["relations"], 1.0, b)
    forward = {"rotate": 3.0 * b * k * D, "transe_l1": 3.0 * b * k * D, "transr": 2.0 * b * k * D * D}.get(c["model"], 2.0 * b * k * D)
    vectors = 2.0 * b * D * D * {"rescal": 1, "transr": 2}.get(c["model"], 0)
    if c["kind"] != "train":
        out = 4 * b * (k + 1) if c["kind"] == "score" else 4 * b
        return {"bytes": 4 * (rows * D + rels * Dr) + ids + out, "flops": forward + vectors}
    per_row = 8 if c["rowwise"] else 16
    touched = rows * D * per_row + rels * Dr * per_row + (8 * (rows + rels) if c["rowwise"] else 0)
    return {"bytes": steps * (touched + ids + 4), "flops": steps * 3 * (forward + vectors)}


def _cost(c):
    """Seconds that a pass may be taken to need when sizes are drawn: launches, memory traffic and arithmetic at rates well
    below the card's."""
    w = work(c)
    copies = 2e1 * c["batch"] // c["chunk"] * c["k"] * c["dim"]  # rows of the corrupting entities and their gradients
    return c["steps"] * (5e-5 + copies / 1e12) + w["bytes"] / 1e12 + w["flops"] / (3e13 if c["model"] in ("rotate", "transe_l1") else 5e13)


def tolerance(case):
    """Scores are sums of up to D products in fp32.  A training pass adds what rounding in one step does to the next (a
    few parts in 10^7 of the tables' norms).  More where an element can land on the other side: bf16 operands (a
    coefficient rounds to either neighbour), RotatE (the gradient of a coordinate pair is a unit vector), TransE-L1 (it
    is a sign) and the kink of the ranking loss.  Ranks count comparisons of scores that can be equal to rounding."""
    if case["kind"] == "sample":
        return "exact"
    if case["kind"] == "score":
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "rank":
        return {"rel": 1e-3, "max": 1e-2, "differ": 0.01}
    if case["model"] in ("transe_l1", "rotate"):
        return {"rel": 5e-3 if case["model"] == "transe_l1" else 1e-3, "max": 0.9}
    if case["bf16"]:
        return {"rel": 1e-3, "max": 0.02}
    if case["loss"] == "ranking":
        return {"rel": 2e-5, "max": 0.05}
    return {"rel": 1e-5, "max": 1e-3}
