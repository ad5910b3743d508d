"""Benchmark of the KGE training step on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME] [--entities N]

One "step" is one whole mini-batch step through the C ABI (gather, positive and chunked negative scoring, loss,
backward, duplicate reduction, sparse Adagrad) on synthetic inputs that are resident in HBM before the timed
region starts.  The default workload is the Freebase-scale configuration (86,054,151 entities, 14,824 relations,
TransE-L2, dim 400, b = 1000, one chunk of 1000, k = 200) with the full entity table and its Adagrad state in HBM.
Prints ONE JSON line.  The roofline object is for the kernel with the largest share of the step; the per-kernel
times behind it are measured in this process (kge_profile: every kernel is launched with a start and a stop
event that take the dispatch's own timestamps) over a second pass of the same kind of steps, and all of them are
listed under "kernels".  "traffic" is bytes per launch from hardware counters, read from the summary under
profiles/ (null for a workload that has none).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X HBM3E
FP32_MATRIX_PEAK_TFLOPS = 157.3
BF16_MATRIX_PEAK_TFLOPS = 2500.0
FP32_VECTOR_PEAK_TFLOPS = 157.3


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10000)
    ap.add_argument("--warmup", type=int, default=200)
    ap.add_argument("--workload", default="freebase-transe_l2")
    ap.add_argument("--entities", type=int, default=0, help="override the entity count (debugging)")
    ap.add_argument("--profile-steps", type=int, default=500)
    ap.add_argument("--cpu-steps", type=int, default=48,
                    help="steps of the single-thread oracle timing (the all-cores build runs eight times as many)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-other-workloads", dest="other_workloads", action="store_false",
                    help="skip the short runs of the other configurations that the default run appends")
    ap.add_argument("--rowwise-state", action="store_true",
                    help="Adagrad with one accumulator per row (adagrad_mode 1) instead of the element-wise state")
    ap.add_argument("--calibration-copy-mib", type=int, default=0,
                    help="also run one plain device copy of this size, as the known-size kernel that scales the "
                         "FETCH_SIZE / WRITE_SIZE counters of a rocprofv3 --pmc run")
    return ap.parse_args()


def algorithmic_work(w, h, r, t, neg, rowwise=False):
    """Per-step algorithmic bytes / flops of every kernel, averaged over the given steps (ids on the host).

    gather : every gathered row read once and every staged row (o_i, corrupting rows) written once
    update : per distinct row, table and state read and written (4 rows) plus every gradient row read once
    GEMMs  : 2 b k D flops forward, 4 b k D backward; pair kernels: b k D_c pair-coordinates
    """
    n = h.shape[0]
    D, Dr, b, k, C = w.ent_dim, w.rel_dim, w.batch, w.neg_per_chunk, w.n_chunks
    ue = np.mean([np.unique(np.concatenate([h[s], t[s], neg[s].reshape(-1)])).size for s in range(n)])
    ur = np.mean([np.unique(r[s]).size for s in range(n)])
    n_keys = 2 * b + C * k
    # elementwise-reduce models: flops per (positive, negative, coordinate): RotatE forward 2 sub, mul, fma, sqrt, add
    # (the transcendental counted once), backward per side the same difference and norm plus scale and two fma; L1
    # sub, abs, add forward and sub, select, add per side backward
    pair_fwd = {"rotate": 6.0, "transe_l1": 3.0}.get(w.model)
    pair_bwd = {"rotate": 2 * 9.0, "transe_l1": 2 * 3.0}.get(w.model)
    coords = D // 2 if w.model == "rotate" else D
    rescal = w.model in ("rescal", "transr")  # relation rows hold D x D matrices, read by their own kernels
    transr = w.model == "transr"  # products batched over the items, the (chunk, relation) that occur: 2 items k D^2 flops each
    items = np.mean([sum(np.unique(c).size for c in r[s].reshape(C, -1)) for s in range(n)]) if transr else 0
    # RESCAL: matrices that the chain rule reads for how many positives.  Rows of 148 to 256 floats: once for each relation of 16
    # positives and more (the update does the others)
    chain_b, chain_m = b, b
    if w.model == "rescal" and 148 <= D <= 256:
        runs = [np.unique(r[s], return_counts=True)[1] for s in range(n)]
        chain_b, chain_m = (np.mean([f(c[c >= 16]) for c in runs]) for f in (np.sum, np.size))
    return {
        "gather": {"bytes": 4.0 * ((2 * b + C * k) * D + (0 if rescal else b * Dr)) + 4.0 * (b + C * k) * D},
        "phi": {"bytes": 4.0 * b * (Dr + 2 * D)},
        "rel_update": {"bytes": ur * 16.0 * Dr + 8.0 * b * D},
        "update": {"bytes": ue * (8.0 * D + 8.0 if rowwise else 16.0 * D) + n_keys * 4.0 * D +
                            (0 if rescal else ur * (8.0 * Dr + 8.0 if rowwise else 16.0 * Dr) + b * 4.0 * Dr)},
        "neg_score": {"flops": pair_fwd * b * k * coords if pair_fwd else 2.0 * k * D * (items * D if transr else b)},
        "neg_backward": {"flops": pair_bwd * b * k * coords if pair_bwd else
                         (2.0 * items * k * D * D if transr else 4.0 * b * k * D)},
        # (TransR: o and p read, dL/do, dL/dp and the translation's gradient written)
        "chain": {"bytes": 4.0 * 5 * b * D if transr else 4.0 * (8 * chain_b * D + chain_m * Dr) if rescal else 4.0 * (6 * b * D + 2 * b * Dr)},
        "loss": {"bytes": 8.0 * b * k},
        "sort": {"bytes": 8.0 * (n_keys + b)},
        "unique_entity_rows": float(ue), "unique_relation_rows": float(ur),
    }


def kernel_report(w, ms, nsteps, work):
    """Average time of every kernel and what it achieves of the card's peaks.  In steps of few tiles the gather launch forms
    the negative scores too: it is then rated by its bytes and by the flops of the scoring product, the closer of the two to
    its peak first ("other" is the other one), and "neg_score", which has no launch of its own, carries the rate of the
    product over that whole launch.  Where TransR forms scores and the negatives' gradient rows in one launch, timed as
    "neg_score", that is rated by both products and "neg_backward" has neither time nor rate."""
    gemm = w.model in ("transe_l2", "distmult", "complex", "rescal", "transr")
    flop_peak = (BF16_MATRIX_PEAK_TFLOPS if w.bf16_inputs else FP32_MATRIX_PEAK_TFLOPS) if gemm else FP32_VECTOR_PEAK_TFLOPS

    def rates(work_of, us):
        found = []
        if us > 0 and "bytes" in work_of:
            found.append(dict(bound="hbm", achieved=work_of["bytes"] / (us * 1e-6) / 1e9, peak=HBM_PEAK_GBS, unit="GB/s"))
        if us > 0 and "flops" in work_of:
            found.append(dict(bound="mfma" if gemm else "alu", achieved=work_of["flops"] / (us * 1e-6) / 1e12, peak=flop_peak,
                              unit="TFLOP/s"))
        for r in found:
            r["frac"] = r["achieved"] / r["peak"]
        return sorted(found, key=lambda r: -r["frac"])

    avg_us = {name: 1e3 * total / max(nsteps, 1) for name, total in ms.items()}
    # (chunks of one positive have one kernel for scores and gradients, timed as neg_backward)
    merged = avg_us.get("neg_score") == 0 and avg_us.get("gather", 0) > 0 and w.chunk > 1
    one_pass = w.model == "transr" and avg_us.get("neg_score", 0) > 0 and avg_us.get("neg_backward") == 0
    kernels = {}
    for name, us in avg_us.items():
        work_of = work.get(name, {})
        if one_pass and name == "neg_score":
            work_of = {"flops": work_of["flops"] + work["neg_backward"]["flops"]}
        if merged and name == "gather":
            work_of = {**work_of, **work["neg_score"]}
        found = rates(work_of, us)
        kernels[name] = {"avg_us": us, **(found[0] if found else {}), **({"other": found[1]} if len(found) > 1 else {})}
    if merged:
        kernels["neg_score"].update(rates(work["neg_score"], avg_us["gather"])[0], launch="gather")
    return kernels


def measured_traffic(workload):
    """HBM-side bytes per launch of every kernel, from the rocprofv3 counter summary under profiles/ (two --pmc
    runs, scaled by a plain copy of known size; the file states the commands).  {} if there is none for this
    workload."""
    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{workload}.txt")
    out = {}
    if os.path.exists(path):
        for line in open(path):
            f = line.split()
            if len(f) == 6 and not line.startswith("#"):
                out[f[0]] = 1024.0 * (float(f[2]) * float(f[4]) + float(f[3]) * float(f[5]))
    return out


def cpu_baseline(w, steps, torch=None, dev=None):
    """The oracle, as it stands, timed on the host: same batch shape, entity table cut down to 5,000,000 rows (the
    full tables do not fit a host run of seconds; a smaller working set flatters the CPU).  Two figures: the parity
    oracle itself (one thread) and the same C file compiled with OpenMP (positives dealt to the threads,
    thread-private accumulators), which uses every core the box gives this process: "value" is that one, "cores" the
    threads it ran on.  The initial tables are drawn on the device when there is one (seconds instead of minutes)
    and copied to the host: they are inputs, the oracle computes everything else."""
    import oracle
    from harness import configs

    n_ent = min(w.n_entities, 5_000_000)
    wc = w.scaled(n_entities=n_ent)
    bs = configs.BatchStream(wc, materialise=False)
    if torch is not None and dev is not None:
        Ed, Rd = configs.init_tables(wc, device=dev)
        E0, R0 = Ed.cpu().numpy(), Rd.cpu().numpy()
        del Ed, Rd
        torch.cuda.empty_cache()
    else:
        E0, R0 = configs.init_tables(wc)
    out = {}
    for key, omp, n in (("single_thread", False, steps), ("all_cores", True, 8 * steps)):
        E, R = E0.copy(), R0.copy()
        SE, SR = np.zeros_like(E), np.zeros_like(R)
        batches = [bs.step(s) for s in range(n)]
        threads = oracle.threads(openmp=omp)
        t0 = time.perf_counter()
        for h, r, t, neg, side in batches:
            oracle.train_step(wc.model, E, SE, R, SR, h, r, t, neg, wc.neg_per_chunk, wc.chunk, side, wc.gamma, wc.lr,
                              adv_temperature=wc.adv_temperature, bf16_inputs=wc.bf16_inputs, openmp=omp)
        dt = time.perf_counter() - t0
        out[key] = {"value": n * wc.batch / dt, "unit": "triples/s", "cores": threads, "steps": n, "seconds": round(dt, 1)}
        del E, SE, R, SR
    sample = (f"{out['all_cores']['steps']} steps (all cores) and {out['single_thread']['steps']} steps (one thread) of the "
              f"same batch shape (b={wc.batch}, g={wc.chunk}, k={wc.neg_per_chunk}, dim={wc.ent_dim}) over a "
              f"{n_ent:,}-entity table on the host, {out['all_cores']['seconds']} s + {out['single_thread']['seconds']} s")
    return {"value": out["all_cores"]["value"], "unit": "triples/s", "cores": out["all_cores"]["cores"], "kind": "oracle",
            "sample": sample, "host_cpus": os.cpu_count(), "single_thread": out["single_thread"]}


def time_other_workload(kge, torch, configs, name, steps, warmup):
    """Triples/s of another configuration of the same benchmark family (same entry point, same replayed steps, ids
    resident on the device); no per-kernel pass."""
    dev = torch.device("cuda", 0)
    w = configs.ALL[name]
    bs = configs.BatchStream(w, materialise=w.n_triples > 0 and w.n_triples <= 50_000_000)
    h, r, t, neg, sides = bs.steps(0, warmup + steps)
    neg = neg.reshape(neg.shape[0], -1)
    dh, dr, dt_, dn = (torch.from_numpy(x).to(dev) for x in (h, r, t, neg))
    E, R = configs.init_tables(w, device=dev)
    SE, SR = torch.zeros_like(E), torch.zeros_like(R)
    ctx = kge.KgeContext(w.model, w.n_entities, w.n_relations, w.ent_dim, w.rel_dim, max_batch=w.batch,
                         max_neg_per_chunk=w.neg_per_chunk, max_chunks=w.n_chunks, gemm_input=int(w.bf16_inputs),
                         adv_temperature=w.adv_temperature)
    losses = torch.zeros(warmup + steps, dtype=torch.float32, device=dev)
    stream = torch.cuda.Stream(device=dev)
    all_tail = bool((sides == 0).all())

    def prepare(lo, hi):
        args = (E, SE, R, SR, dh[lo:hi], dr[lo:hi], dt_[lo:hi], dn[lo:hi], w.neg_per_chunk, w.chunk,
                None if all_tail else np.ascontiguousarray(sides[lo:hi], dtype=np.int32), w.gamma, w.lr)
        return lambda: ctx.train_steps(*args, loss_out=losses[lo:hi], stream=stream)

    torch.cuda.synchronize(dev)  # tables and ids were written on the default stream; the steps run on `stream`
    prepare(0, warmup)()
    timed = prepare(warmup, warmup + steps)
    torch.cuda.synchronize(dev)
    t0 = time.perf_counter()
    timed()
    torch.cuda.synchronize(dev)
    elapsed = time.perf_counter() - t0
    ctx.close()
    del timed
    return {"workload": name, "model": w.model, "dtype": "bf16-in/f32-acc" if w.bf16_inputs else "f32",
            "batch": w.batch, "chunk": w.chunk, "neg_per_chunk": w.neg_per_chunk, "dim": w.ent_dim,
            "entities": w.n_entities, "triples_per_s": steps * w.batch / elapsed, "us_per_step": 1e6 * elapsed / steps,
            "steps": steps}


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no sharding, no collectives); use --gpus 1", file=sys.stderr)
        sys.exit(2)
    import torch

    import paper_2004_08532_amd as kge
    from harness import configs

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = torch.device("cuda", 0)
    w = configs.ALL[args.workload]
    if args.entities:
        w = w.scaled(n_entities=args.entities, name=w.name + f"-{args.entities}ent")
    state_cols = (1, 1) if args.rowwise_state else (w.ent_dim, w.rel_dim)
    need = (w.n_entities * (w.ent_dim + state_cols[0]) + w.n_relations * (w.rel_dim + state_cols[1])) * 4
    free, _total = torch.cuda.mem_get_info(dev)
    if need + (4 << 30) > free:
        print(f"bench.py: workload {w.name} needs {need / 2**30:.1f} GiB of HBM, {free / 2**30:.1f} GiB free",
              file=sys.stderr)
        sys.exit(3)

    K, W, P = args.steps, args.warmup, args.profile_steps
    t_setup = time.perf_counter()
    bs = configs.BatchStream(w, materialise=w.n_triples > 0 and w.n_triples <= 50_000_000)
    h, r, t, neg, sides = bs.steps(0, W + K + P)
    neg = neg.reshape(neg.shape[0], -1)
    dh, dr, dt_, dn = (torch.from_numpy(x).to(dev) for x in (h, r, t, neg))
    E, R = configs.init_tables(w, device=dev)
    if args.rowwise_state:
        SE = torch.zeros(w.n_entities, dtype=torch.float32, device=dev)
        SR = torch.zeros(w.n_relations, dtype=torch.float32, device=dev)
    else:
        SE, SR = torch.zeros_like(E), torch.zeros_like(R)
    ctx = kge.KgeContext(w.model, w.n_entities, w.n_relations, w.ent_dim, w.rel_dim, max_batch=w.batch,
                         max_neg_per_chunk=w.neg_per_chunk, max_chunks=w.n_chunks, gemm_input=int(w.bf16_inputs),
                         adv_temperature=w.adv_temperature, adagrad_mode=int(args.rowwise_state))
    losses = torch.zeros(W + K + P, dtype=torch.float32, device=dev)
    if args.calibration_copy_mib > 0:
        src = torch.ones(args.calibration_copy_mib << 18, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        del src, dst
    torch.cuda.synchronize(dev)
    setup_s = time.perf_counter() - t_setup

    stream = torch.cuda.Stream(device=dev)  # a capturable stream: kge_train_steps replays HIP graphs on it
    all_tail = bool((sides == 0).all())

    def prepare(lo, hi):
        """The call for steps lo .. hi - 1 with its arguments marshalled (views of the resident id arrays); calling the
        result enqueues the steps on `stream`."""
        args = (E, SE, R, SR, dh[lo:hi], dr[lo:hi], dt_[lo:hi], dn[lo:hi], w.neg_per_chunk, w.chunk,
                None if all_tail else np.ascontiguousarray(sides[lo:hi], dtype=np.int32), w.gamma, w.lr)
        loss_view = losses[lo:hi]
        return lambda: ctx.train_steps(*args, loss_out=loss_view, stream=stream)

    def run(lo, hi):
        prepare(lo, hi)()

    run(0, W)
    timed = prepare(W, W + K)
    torch.cuda.synchronize(dev)
    t0 = time.perf_counter()
    timed()
    t_enqueued = time.perf_counter() - t0
    torch.cuda.synchronize(dev)
    elapsed = time.perf_counter() - t0

    # second pass: the same kind of steps with HIP events around every kernel
    kernels = {}
    roofline = None
    if P > 0:
        ctx.profile(True)
        run(W + K, W + K + P)
        ms, nsteps = ctx.profile_read()
        ctx.profile(False)
        work = algorithmic_work(w, h[W + K:], r[W + K:], t[W + K:], neg[W + K:], args.rowwise_state)
        kernels = kernel_report(w, ms, nsteps, work)
        traffic = measured_traffic(w.name)
        for name, ent in kernels.items():
            ent["traffic"] = traffic.get(name)
        on_stream = {n: e for n, e in kernels.items() if n != "sort"}  # the sort overlaps on its own stream
        dom = max(on_stream, key=lambda n: on_stream[n]["avg_us"])
        d = kernels[dom]
        roofline = {"kernel": dom, "bound": d.get("bound"), "achieved": d.get("achieved"), "peak": d.get("peak"),
                    "unit": d.get("unit"), "frac": d.get("frac"), "traffic": d.get("traffic"), "avg_us": d["avg_us"],
                    "other": d.get("other"),
                    "unique_entity_rows_per_step": work["unique_entity_rows"],
                    "unique_relation_rows_per_step": work["unique_relation_rows"]}

    # step 1 on the device (not part of the timed step: the step's ids are resident before it starts): ids of K steps
    # from a synthetic triple list, one launch
    # the triple list: the positives of this run's steps (drawn from the graph's generating distribution, so the list
    # has its degree skew), at most 16 M of them
    n_tr = min(16_000_000, dh.numel())
    tr = torch.stack([dh.reshape(-1)[:n_tr], dr.reshape(-1)[:n_tr], dt_.reshape(-1)[:n_tr]], dim=1).contiguous()
    sh = torch.empty((K, w.batch), dtype=torch.int64, device=dev)
    sr, st_ = torch.empty_like(sh), torch.empty_like(sh)
    sn = torch.empty((K, w.n_chunks * w.neg_per_chunk), dtype=torch.int64, device=dev)
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for rep in range(2):
        ev0.record()
        kge.kge_sample_steps(w.seed, tr, w.n_entities, w.batch, w.n_chunks, w.neg_per_chunk, 0, w.side_mode, 0, K, sh, sr,
                             st_, sn)
        ev1.record()
        torch.cuda.synchronize(dev)
    sample_ms = ev0.elapsed_time(ev1)
    ids_per_step = 3 * w.batch + w.n_chunks * w.neg_per_chunk
    sampling = {"us_per_step": 1e3 * sample_ms / K, "ids_per_s": K * ids_per_step / (sample_ms * 1e-3),
                "note": f"kge_sample_steps, {K} steps in one launch, list of {n_tr:,} synthetic triples"}
    # link-prediction evaluation (forward only), the paper's second protocol (Sec. 5): every positive is ranked among
    # 1000 candidates drawn uniformly and 1000 drawn in proportion to degree (the corrupted-side entities of the
    # evaluation batch itself), both sides; the candidate sets come from kge_sample_steps
    k_eval, n_eval = 2000, 200
    ectx = kge.KgeContext(w.model, w.n_entities, w.n_relations, w.ent_dim, w.rel_dim, max_batch=w.batch,
                          max_neg_per_chunk=k_eval, max_chunks=1, gemm_input=int(w.bf16_inputs))
    eh = torch.empty((n_eval, w.batch), dtype=torch.int64, device=dev)
    er, et = torch.empty_like(eh), torch.empty_like(eh)
    en = torch.empty((n_eval, k_eval), dtype=torch.int64, device=dev)
    kge.kge_sample_steps(w.seed + 17, tr, w.n_entities, w.batch, 1, k_eval, k_eval // 2, "alternate", 0, n_eval, eh, er, et, en)
    ranks = torch.empty(w.batch, dtype=torch.int32, device=dev)
    metrics = torch.zeros(5, dtype=torch.float64, device=dev)
    for rep in range(2):
        ev0.record()
        for s_ in range(n_eval):
            ectx.rank(E, R, eh[s_], er[s_], et[s_], en[s_], k_eval, w.batch, s_ & 1, w.gamma, rank_out=ranks)
        kge.kge_rank_metrics(ranks, metrics)
        ev1.record()
        torch.cuda.synchronize(dev)
    eval_ms = ev0.elapsed_time(ev1)
    evaluation = {"ranked_triples_per_s": n_eval * w.batch / (eval_ms * 1e-3), "us_per_call": 1e3 * eval_ms / n_eval,
                  "note": f"kge_rank, b={w.batch}, {k_eval // 2} uniform + {k_eval // 2} degree-proportional candidates per "
                          f"positive (ids from kge_sample_steps), alternating sides, {n_eval} calls"}
    ectx.close()
    del tr, sh, sr, st_, sn, eh, er, et, en

    captures = ctx.graph_captures()
    loss_first = float(losses[W].item())
    loss_last = float(losses[W + K - 1].item())
    ctx.close()

    # the other configurations of the benchmark family, for the record (not the headline value): each is timed the
    # same way on its own tables, after the Freebase-scale tables have been given back
    del timed, E, SE, R, SR  # (the prepared call holds the tables too)
    torch.cuda.empty_cache()
    others = []
    if args.other_workloads and args.workload == "freebase-transe_l2":
        for name in ("small-distmult", "small-complex", "medium", "large", "freebase-complex", "small-rescal",
                     "small-transr"):
            others.append(time_other_workload(kge, torch, configs, name, 2000, 100))
            torch.cuda.empty_cache()

    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(w, args.cpu_steps, torch, dev)

    out = {
        "metric": "positive triples/sec per MI355X at fixed negs",
        "value": K * w.batch / elapsed,
        "unit": "triples/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": W,
        "ms_per_step": 1e3 * elapsed / K,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16-in/f32-acc" if w.bf16_inputs else "f32",
        "data": "synthetic",
        "config": {"workload": w.name + ("+rowwise-adagrad-state" if args.rowwise_state else ""), "model": w.model, "entities": w.n_entities, "relations": w.n_relations,
                   "dim": w.ent_dim, "batch": w.batch, "chunk": w.chunk, "neg_per_chunk": w.neg_per_chunk,
                   "table_plus_state_GiB": round(need / 2 ** 30, 2), "setup_s": round(setup_s, 1),
                   "host_enqueue_ms_per_step": 1e3 * t_enqueued / K, "graph_captures": captures,
                   "loss_first": loss_first, "loss_last": loss_last},
        "roofline": roofline,
        "kernels": kernels,
        "sampling": sampling,
        "evaluation": evaluation,
        "other_workloads": others,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out))


if __name__ == "__main__":
    main()
