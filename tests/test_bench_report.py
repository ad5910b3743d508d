"""What bench.py reports of every kernel from the profiled times: the scoring product has a rate in every form of the step."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench
from harness import configs

SLOTS = ["gather", "neg_score", "loss", "neg_backward", "chain", "sort", "update", "phi", "rel_update"]


def report(name, us):
    w = configs.ALL[name]
    h, r, t, neg, _ = configs.BatchStream(w.scaled(n_entities=100_000), materialise=False).steps(0, 2)
    work = bench.algorithmic_work(w, h, r, t, neg)
    return w, work, bench.kernel_report(w, {s: 1e-3 * 50 * us.get(s, 0.0) for s in SLOTS}, 50, work)


def test_scoring_product_in_the_gather_launch():
    w, work, k = report("freebase-transe_l2", {"gather": 13.3, "neg_backward": 12.4, "update": 9.5})
    flops = 2.0 * w.batch * w.neg_per_chunk * w.ent_dim / 13.3e-6 / 1e12
    assert k["neg_score"]["achieved"] == pytest.approx(flops) and k["neg_score"]["bound"] == "mfma"
    assert k["neg_score"]["frac"] == pytest.approx(flops / bench.FP32_MATRIX_PEAK_TFLOPS)
    assert k["neg_score"]["launch"] == "gather" and k["neg_score"]["avg_us"] == 0.0
    both = {x["bound"]: x for x in (k["gather"], k["gather"]["other"])}
    assert both["mfma"]["achieved"] == pytest.approx(flops)
    assert both["hbm"]["achieved"] == pytest.approx(work["gather"]["bytes"] / 13.3e-6 / 1e9)
    assert k["gather"]["frac"] >= k["gather"]["other"]["frac"]


def test_scoring_product_in_a_launch_of_its_own():
    w, work, k = report("large", {"gather": 14.0, "neg_score": 12.0, "neg_backward": 20.0, "update": 21.0})
    assert k["neg_score"]["achieved"] == pytest.approx(work["neg_score"]["flops"] / 12e-6 / 1e12)
    assert k["neg_score"]["peak"] == bench.BF16_MATRIX_PEAK_TFLOPS and "launch" not in k["neg_score"]
    assert k["gather"]["bound"] == "hbm" and "other" not in k["gather"]
    assert "achieved" not in k["loss"]  # did not run


def test_elementwise_models_are_rated_by_the_vector_units():
    _, work, k = report("medium", {"gather": 8.0, "neg_score": 14.8, "neg_backward": 29.0, "chain": 7.0, "update": 14.0})
    assert k["neg_score"]["bound"] == "alu" and k["neg_score"]["peak"] == bench.FP32_VECTOR_PEAK_TFLOPS


@pytest.mark.parametrize("us", [{"neg_score": 75.0, "chain": 5.0}, {"neg_score": 60.0, "neg_backward": 65.0, "chain": 30.0}])
def test_transr_products_in_one_launch_or_two(us):
    w, work, k = report("small-transr", {"gather": 10.7, "update": 8.3, "phi": 16.6, "rel_update": 15.7, **us})
    product = work["neg_score"]["flops"]  # 2 k D^2 per (chunk, relation) that occurs
    assert w.batch / 4 < product / (2.0 * w.neg_per_chunk * w.ent_dim ** 2) < w.batch
    if "neg_backward" in us:
        assert k["neg_backward"]["achieved"] == pytest.approx(product / 65e-6 / 1e12)
        assert k["neg_score"]["achieved"] == pytest.approx(product / 60e-6 / 1e12)
    else:
        assert "achieved" not in k["neg_backward"]
        assert k["neg_score"]["achieved"] == pytest.approx(2 * product / 75e-6 / 1e12)
    assert k["chain"]["achieved"] == pytest.approx(20.0 * w.batch * w.ent_dim / us["chain"] / 1e3)  # GB/s
