#!/usr/bin/env python3
"""Benchmark of LINE edge-sampled SGD on one MI355X.

    python bench.py [--gpus 1] [--steps 5] [--warmup 1] [--workload C2]

One step = the whole hot path over the workload's synthetic graph, arcs already in HBM:
validate the arcs and count out-degrees, build both alias tables (binary64 normalisation
and prefix sums), initialise the embedding tables, then train all T edge samples (Philox
draws, row gathers, dot products, scatter updates) with the Hogwild kernel.  ``value`` is
T / (median step time) in edge samples per second.

Default workload (C2): directed R-MAT scale 20 (2^20 nodes, 2^24 unique arcs, 1 % held
out), lognormal(0, 1) weights, d = 128, K = 5, first + second order, binary32 tables,
T = 2e8, eta 0.025 decaying linearly to 0.  After the timed steps the same hot path runs
with bfloat16 tables (C3) for the BF16-over-FP32 speedup, and the held-out AUC of both
is compared with the binary64 oracle's.  The C3 embedding error is measured on the first
2^20 samples in SNAPSHOT mode against the oracle's binary64 SNAPSHOT run.

Prints one JSON line.  ``--gpus`` above 1 is refused: the library runs on one GPU.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "edge samples/sec at d=128,K=5 + HBM GB/s; BF16 vs FP32 at equal AUC"
PEAK_HBM_GBS = 8000.0
GOLDEN = os.path.join(ROOT, "tests", "golden")


def algorithmic_bytes_per_sample(d: int, K: int, orders: int, elem_bytes: int) -> int:
    """Bytes the method must move per edge sample: per order, (2 + K) rows read and
    written (vertex row, positive context row, K negative context rows), plus one
    32-byte edge alias record (threshold, alias, both arcs' endpoints) and K 16-byte
    negative alias records."""
    n_orders = bin(orders).count("1")
    return n_orders * 2 * (2 + K) * d * elem_bytes + 32 + 16 * K


TRAFFIC_PROFILE = os.path.join(ROOT, "profiles", "k_hogwild_c2_fp32_hbm_traffic.md")


# The sources the C2 Hogwild training kernel and its launch are built from: the tile and
# launch code, the handle and alias build (the hot-row thresholds), the binary32
# orders-1+2 translation unit, the C header and the build flags.  The batched and
# SNAPSHOT sources and the other dtype/order units do not enter this kernel.
KERNEL_SOURCES = [
    "paper_2604_09419_amd/csrc/common.hpp", "paper_2604_09419_amd/csrc/handle.hpp",
    "paper_2604_09419_amd/csrc/scan.hpp", "paper_2604_09419_amd/csrc/table.hpp",
    "paper_2604_09419_amd/csrc/tile.hpp",
    "paper_2604_09419_amd/csrc/sgd_kernels.hpp", "paper_2604_09419_amd/csrc/alias.hip",
    "paper_2604_09419_amd/csrc/api.hip", "paper_2604_09419_amd/csrc/misc.hip",
    "paper_2604_09419_amd/csrc/sgd_f32_o3.hip", "include/linehip.h", "paper_2604_09419_amd/build.py",
]


def _code_only(text: str, python: bool) -> str:
    """Source text without comments and with whitespace collapsed, so that the hash below
    changes with the code, not with its comments (string literals are kept verbatim)."""
    import re
    if python:
        pat = re.compile(r'("(?:\\.|[^"\\])*"|\'(?:\\.|[^\'\\])*\')|#[^\n]*')
    else:
        pat = re.compile(r'("(?:\\.|[^"\\])*"|\'(?:\\.|[^\'\\])*\')|//[^\n]*|/\*.*?\*/', re.S)
    text = pat.sub(lambda m: m.group(1) or " ", text)
    return " ".join(text.split())


def kernel_sources_sha256(root: str = ROOT) -> str:
    """SHA-256 over KERNEL_SOURCES (path, NUL, code without comments, NUL each)."""
    import hashlib
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES:
        h.update(rel.encode())
        h.update(b"\0")
        with open(os.path.join(root, rel), encoding="utf-8") as fh:
            h.update(_code_only(fh.read(), rel.endswith(".py")).encode())
        h.update(b"\0")
    return h.hexdigest()


def measured_traffic(path: str, kernel_config: dict, total_samples: int):
    """HBM bytes per launch of the training kernel from a committed rocprofv3 counter
    summary (FETCH_SIZE + WRITE_SIZE, each scaled by a plain copy's reading), or None
    when the kernel sources, the kernel configuration or T differ from those the
    counters were taken with."""
    if not os.path.exists(path):
        return None
    rec = {}
    with open(path) as f:
        for line in f:
            k, sep, v = line.strip().partition(": ")
            if sep:
                rec[k] = v.strip()
    try:
        cfg = [int(x) for x in rec["kernel_config"].split()]
        ok = (rec["kernel_sources_sha256"] == kernel_sources_sha256()
              and cfg == [kernel_config["lanes_per_sample"], kernel_config["units_per_lane"],
                          kernel_config["blocks_per_cu"]]
              and int(rec["total_samples"]) == int(total_samples))
        return float(rec["traffic_bytes_per_launch"]) if ok else None
    except (KeyError, ValueError):
        return None


def log(msg: str) -> None:
    print(msg, file=sys.stderr, flush=True)


def workload(name: str):
    from synth import CONFIGS, config_graph
    cfg = dict(CONFIGS[name])
    t0 = time.time()
    g, hs, hd, neg = config_graph(name)
    log(f"[bench] {name}: n={g.n} m={g.m} generated in {time.time() - t0:.1f}s")
    return cfg, g, hs, hd, neg


# Random-walk pair source of the walk legs (Sec. IV-B): walk length 100 and window 2 (Sec.
# V-A), walks per batch 1024 (about 10^5 pairs per batch, the paper's batch sizes).
WALK = dict(walk_length=100, window=2, walks_per_batch=1024)


def run_gpu_leg(cfg, g, dtype, steps, warmup, seed, tune_cache, hot_shadow=False, walks=None, pool=False):
    """Time `steps` full passes (after `warmup`); return timings and the trainer.  With
    `walks`, every pass also builds the walk rows, and training takes its positive pairs
    from random walks (their generation inside the timed training call); with `pool` as
    well, every pass collects a pair pool of the default size after the walk rows, and
    training draws its pairs from it."""
    import torch
    from paper_2604_09419_amd import Trainer
    T = int(cfg["T"])
    tr = Trainer(g.n, g.src, g.dst, g.w, d=cfg["d"], K=cfg["K"], orders=cfg["orders"], dtype=dtype,
                 eta0=cfg["eta0"], seed=seed, total_samples=T, build=False, init=False, hot_shadow=hot_shadow)
    # Tuning happens once, outside the timed region, with the step size scaled to zero.
    tr.build_alias()
    tr.tune(probe=min(T, 20_000_000), cache_path=tune_cache)
    step_ms, kern_ms = [], []
    for i in range(warmup + steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        from paper_2604_09419_amd import _lib
        _lib.lh_set_graph(tr.h, tr.n, tr.m, tr.src.data_ptr(), tr.dst.data_ptr(), tr.w.data_ptr())
        tr.build_alias()
        if walks:
            tr.build_walks(**walks)
        if pool:
            tr.build_pool()
        tr.init_embeddings()
        tr.train_steps(0, T)
        tr.synchronize()
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) * 1e3
        km = tr.last_train_ms()
        if i >= warmup:
            step_ms.append(dt)
            kern_ms.append(km)
        kind = " pool" if pool else " walks" if walks else ""
        log(f"[bench] {dtype}{kind} step {i} ({'warmup' if i < warmup else 'timed'}): "
            f"{dt:.1f} ms, train kernel {km:.1f} ms")
    tr.check()
    return tr, step_ms, kern_ms


def walk_legs(args, cfg, g, hs, hd, neg, seed, T, pool=False):
    """C2 with positive pairs from random walks (WALK), or with `pool` from a pair pool
    collected from them (Sec. IV-C, Augmented-Pair), binary32 and bfloat16 tables: step and
    training-call rates (walk generation included), and held-out AUCs against the
    oracle's binary64 SEQ run on the same pairs."""
    import torch
    out = {"pairs": (f"pair pool of the default size for T collected from random walks {WALK}" if pool
                     else f"random walks {WALK}")}
    gold_path = os.path.join(GOLDEN, "c2_pool_oracle_auc.json" if pool else "c2_walk_oracle_auc.json")
    gold = json.load(open(gold_path)) if os.path.exists(gold_path) else None
    for dtype in ("fp32", "bf16"):
        tr, steps_ms, kern_ms = run_gpu_leg(cfg, g, dtype, max(1, args.steps), 1, seed, args.tune_cache,
                                            hot_shadow=args.hot_shadow, walks=WALK, pool=pool)
        leg = {"samples_per_s": T / (median(steps_ms) * 1e-3), "train_call_samples_per_s": T / (median(kern_ms) * 1e-3),
               "kernel_config": tr.kernel_config()}
        if not args.no_auc:
            leg["auc"] = held_out_auc(tr, hs, hd, neg, cfg["orders"])
            if gold:
                leg["auc_within_0.005_of_oracle"] = all(abs(v - gold["auc_" + k]) <= 0.005
                                                        for k, v in leg["auc"].items())
            log(f"[bench] {dtype} {'pool' if pool else 'walks'} AUC {leg['auc']}")
        out[dtype] = leg
        tr.close()
        del tr
        torch.cuda.empty_cache()
    if gold:
        out["auc_oracle_binary64"] = {k[4:]: v for k, v in gold.items() if k.startswith("auc_")
                                      and not k.startswith("auc_init")}
    return out


def node_classification(args):
    """Sec. V-A's quality metric on the labelled stand-in graph (synth.labels.SBM): Micro-
    and Macro-F1 of a one-vs-rest logistic regression on 10 % of the labels, for vertex
    embeddings trained on the GPU with arc-draw pairs, random-walk pairs and pairs from a
    pair pool (Sec. IV-C, Augmented-Pair), beside the oracle's stored values."""
    import torch
    from paper_2604_09419_amd import LH_TABLE_U, Trainer
    from synth.labels import node_classification_f1, sbm_workload
    g, labels, c = sbm_workload()
    out = {"workload": f"stochastic block model: {g.n} nodes, {c['classes']} classes, mean degree "
                       f"{c['mean_degree']}, p_in {c['p_in']}; d={c['d']}, K={c['K']}, second order, "
                       f"{c['epochs']} epochs (T={c['T']})"}
    for dtype in ("fp32", "bf16"):
        for pairs in ("arcs", "walks", "pool"):
            tr = Trainer(g.n, g.src, g.dst, g.w, d=c["d"], K=c["K"], orders=c["orders"], dtype=dtype,
                         eta0=c["eta0"], seed=c["train_seed"], total_samples=c["T"])
            if pairs in ("walks", "pool"):
                tr.build_walks(**WALK)
            if pairs == "pool":
                tr.build_pool()
            tr.train_steps(0, c["T"])
            ms = tr.last_train_ms()
            micro, macro = node_classification_f1(tr.read(LH_TABLE_U).cpu().numpy(), labels, c["split_seed"])
            out[f"{dtype}_{pairs}"] = {"micro_f1": micro, "macro_f1": macro, "train_ms": ms}
            tr.close()
            del tr
            torch.cuda.empty_cache()
    gold_path = os.path.join(GOLDEN, "sbm_oracle_f1.json")
    pool_path = os.path.join(GOLDEN, "sbm_pool_oracle_f1.json")
    if os.path.exists(gold_path) and os.path.exists(pool_path):
        gold = json.load(open(gold_path))
        gold.update({k: v for k, v in json.load(open(pool_path)).items() if k in ("pool", "pool_bf16")})
        out["oracle"] = {k: {"micro_f1": gold[k]["micro"], "macro_f1": gold[k]["macro"]}
                         for k in ("arcs", "walks", "pool", "arcs_bf16", "walks_bf16", "pool_bf16") if k in gold}
        # the tolerance of the tests: max(0.01, 3 sd of the oracle's F1 over training seeds)
        def ok(v, ref):
            return all(abs(v[f"{a}_f1"] - ref[a]) <= max(0.01, 3.0 * ref[f"sd_{a}"]) for a in ("micro", "macro"))
        # bfloat16 runs against the oracle with bfloat16 storage
        def ref_of(k):
            dtype, pairs = k.split("_")
            return gold[pairs if dtype == "fp32" else pairs + "_bf16"]
        out["within_tolerance_of_oracle"] = all(ok(v, ref_of(k)) for k, v in out.items()
                                                if isinstance(v, dict) and "micro_f1" in v)
    return out


def held_out_auc(tr, hs, hd, neg, orders):
    import numpy as np
    from paper_2604_09419_amd import LH_TABLE_C, LH_TABLE_U, LH_TABLE_U1

    def dots(A, B, u, v):
        return np.einsum("ij,ij->i", A[u].astype(np.float64), B[v].astype(np.float64))

    def auc(p, q):
        from scipy.stats import rankdata
        r = rankdata(np.concatenate([p, q]))
        return float((r[: p.size].sum() - p.size * (p.size + 1) / 2) / (p.size * q.size))

    out = {}
    if orders & 2:
        U = tr.read(LH_TABLE_U).cpu().numpy()
        C = tr.read(LH_TABLE_C).cpu().numpy()
        out["uc"] = auc(dots(U, C, hs, hd), dots(U, C, hs, neg))
        uu = (dots(U, U, hs, hd), dots(U, U, hs, neg))
        out["uu"] = auc(*uu)
    if orders & 1:
        U1 = tr.read(LH_TABLE_U1).cpu().numpy()
        o1 = (dots(U1, U1, hs, hd), dots(U1, U1, hs, neg))
        out["o1"] = auc(*o1)
    if orders == 3:
        out["concat"] = auc(uu[0] + o1[0], uu[1] + o1[1])
    return out


def host_threads():
    """Threads for the oracle's CPU legs: every core in this process's affinity mask, or
    fewer when OMP_NUM_THREADS says so (a shared host can give one GPU's job a fixed share of
    its cores that way).  Returns (threads, affinity core count, reason for a cap)."""
    cores = len(os.sched_getaffinity(0))
    omp = os.environ.get("OMP_NUM_THREADS", "")
    if omp.isdigit() and 0 < int(omp) < cores:
        return int(omp), cores, f"OMP_NUM_THREADS={omp} (the host's share for this job)"
    return cores, cores, ""


def median(xs):
    xs = sorted(xs)
    n = len(xs)
    return xs[n // 2] if n % 2 else 0.5 * (xs[n // 2 - 1] + xs[n // 2])


def _timed_chunks(run, first, count, chunks=5, say=None):
    """Run samples [first, first + count) as `chunks` consecutive equal parts; return each
    part's rate (samples/s)."""
    rates = []
    per = count // chunks
    for i in range(chunks):
        t = time.perf_counter()
        run(first + i * per, per)
        rates.append(per / (time.perf_counter() - t))
        if say:
            say(f"part {i + 1} of {chunks}: {rates[-1]:.4g} samples/s")
    return rates


def cpu_baseline(cfg, g, seed, target_s=15.0, chunks=5, label="same workload"):
    """The oracle's binary32 Hogwild mode on every host core this process may use, over a
    bounded prefix of the same sample stream, timed as `chunks` consecutive parts: the
    reported value is the median part's rate."""
    import oracle
    threads, cores, cap = host_threads()
    t0 = time.time()

    def say(msg):
        log(f"[bench] oracle: {msg} ({time.time() - t0:.1f}s)")

    tb = oracle.Tables(g.n, g.src, g.dst, g.w, progress=say)
    d, K, orders, T = cfg["d"], cfg["K"], cfg["orders"], int(cfg["T"])
    U = C = U1 = None
    if orders & 2:
        U = oracle.init_table(0, g.n, d, seed, 0)
        say("U initialised")
        C = oracle.init_table(1, g.n, d, seed, 0)
        say("C initialised")
    if orders & 1:
        U1 = oracle.init_table(2, g.n, d, seed, 0)
        say("U1 initialised")
    prep_s = time.time() - t0
    log(f"[bench] oracle tables ready in {prep_s:.1f}s, {threads} threads")

    def run(first, count):
        oracle.train_hogwild_f32(tb, U, C, U1, d, K, orders, T, seed, 0, first, count, threads)

    probe = 200_000
    t1 = time.perf_counter()
    run(0, probe)
    rate = probe / (time.perf_counter() - t1)
    count = int(min(max(rate * target_s, chunks * probe), T - probe))
    rates = _timed_chunks(run, probe, count, chunks, say)
    del U, C, U1, tb
    per = count // chunks
    return {"value": median(rates), "unit": "edge samples/s", "cores": threads, "kind": "oracle",
            "affinity_cores": cores, "thread_cap": cap or None, "chunk_rates": rates,
            "table_prep_s": prep_s,
            "sample": f"samples [{probe}, {probe + chunks * per}) of the {label} and seed, timed as "
                      f"{chunks} consecutive parts of {per} samples (median part reported), binary32 "
                      f"lock-free mode of the oracle, {threads} OpenMP threads of {cores} in the "
                      "affinity mask; alias build and init excluded"}


def oracle_seq_timings(g2, cfg2, seed2, c2_prefix=1_000_000, chunks=5):
    """The oracle's single-thread binary64 SEQ mode (the one the stored AUC references come
    from): C1 in full, `chunks` times, and a prefix of C2 as `chunks` consecutive parts.
    Median rates (samples/s)."""
    import oracle
    from synth import CONFIGS, config_graph
    out = {}
    cfg1 = CONFIGS["C1"]
    g1, _, _, _ = config_graph("C1")
    t1 = oracle.Tables(g1.n, g1.src, g1.dst, g1.w)
    T1 = int(cfg1["T"])
    rates = []
    for _ in range(chunks):
        m = oracle.Model(t1, d=cfg1["d"], K=cfg1["K"], orders=cfg1["orders"], T=T1, seed=cfg1["seed"],
                         eta0=cfg1["eta0"])
        t = time.perf_counter()
        m.train(0, T1, "seq")
        rates.append(T1 / (time.perf_counter() - t))
    out["C1"] = {"value": median(rates), "runs": rates, "threads": 1,
                 "sample": f"all T = {T1} samples, {chunks} runs from the initial tables"}
    t2 = oracle.Tables(g2.n, g2.src, g2.dst, g2.w)
    m = oracle.Model(t2, d=cfg2["d"], K=cfg2["K"], orders=cfg2["orders"], T=int(cfg2["T"]), seed=seed2,
                     eta0=cfg2["eta0"])
    rates = _timed_chunks(lambda f, c: m.train(f, c, "seq"), 0, c2_prefix, chunks)
    out["C2"] = {"value": median(rates), "runs": rates, "threads": 1,
                 "sample": f"samples [0, {c2_prefix}) as {chunks} consecutive parts"}
    out["unit"] = "edge samples/s"
    out["kind"] = "oracle binary64 SEQ"
    return out


def c3_embedding_error(cfg, g, seed, count=1 << 20, batch=65536):
    """||X - X64||_F / ||X64||_F per table after the first `count` samples in SNAPSHOT mode
    (batch B): bfloat16 tables and binary32 tables on the GPU against the oracle's binary64
    SNAPSHOT run, with the floor of rounding X64 to nearest bfloat16."""
    import numpy as np
    import torch
    import oracle
    from paper_2604_09419_amd import LH_TABLE_C, LH_TABLE_U, LH_TABLE_U1, Trainer
    t0 = time.time()
    tb = oracle.Tables(g.n, g.src, g.dst, g.w)
    m = oracle.Model(tb, d=cfg["d"], K=cfg["K"], orders=cfg["orders"], T=int(cfg["T"]), seed=seed,
                     eta0=cfg["eta0"])
    m.train(0, count, "snapshot", batch)
    log(f"[bench] oracle SNAPSHOT of {count} samples in {time.time() - t0:.1f}s")
    refs = {"U": (LH_TABLE_U, m.U), "C": (LH_TABLE_C, m.C), "U1": (LH_TABLE_U1, m.U1)}
    out = {"samples": count, "batch": batch, "mode": "snapshot"}

    def fro(x, ref):
        return float(np.linalg.norm(x.astype(np.float64) - ref) / np.linalg.norm(ref))

    for dtype in ("bf16", "fp32"):
        tr = Trainer(g.n, g.src, g.dst, g.w, d=cfg["d"], K=cfg["K"], orders=cfg["orders"], dtype=dtype,
                     eta0=cfg["eta0"], seed=seed, total_samples=int(cfg["T"]), mode="snapshot", batch=batch)
        tr.train_steps(0, count)
        tr.check()
        out[dtype] = {k: fro(tr.read(t).cpu().numpy(), ref) for k, (t, ref) in refs.items() if ref is not None}
        tr.close()
        del tr
        torch.cuda.empty_cache()
    out["nearest_bf16_floor"] = {
        k: fro(torch.tensor(ref, dtype=torch.float32).to(torch.bfloat16).float().numpy(), ref)
        for k, (_, ref) in refs.items() if ref is not None}
    return out


def _lib_batch_config(bt):
    from paper_2604_09419_amd import _lib
    return _lib.lh_batch_config(bt.b)


def bench_batched(args):
    """C4: 64 power-law graphs (bfloat16, second order, d in {64, 128}) trained in one
    persistent hipGraph-captured launch, against 64 one-graph launches."""
    import torch
    from paper_2604_09419_amd import BatchTrainer, Trainer
    from synth import batch_graph_specs
    from synth.graphs import rmat_graph_gpu
    specs = batch_graph_specs()
    stream = torch.cuda.Stream()
    trainers = []
    t0 = time.time()
    for sp in specs:
        src, dst, w = rmat_graph_gpu(sp["scale"], sp["n"], sp["m"], sp["seed"] + 100_000)
        tr = Trainer(sp["n"], src, dst, w, d=sp["d"], K=5, orders=2, dtype="bf16", seed=sp["seed"],
                     graph_id=sp["g"], total_samples=sp["T"], stream=stream, hot_shadow=args.hot_shadow)
        trainers.append(tr)
    torch.cuda.synchronize()
    log(f"[bench] C4: 64 graphs generated and built in {time.time() - t0:.1f}s")
    total_T = sum(sp["T"] for sp in specs)
    algo_bytes = sum(sp["T"] * algorithmic_bytes_per_sample(sp["d"], 5, 2, 2) for sp in specs)
    bt = BatchTrainer(trainers)
    t0 = time.time()
    bt.tune(cache_path=args.tune_cache)
    tuning = _lib_batch_config(bt)
    log(f"[bench] C4 tiling {tuning} ({time.time() - t0:.1f}s)")
    bt.capture()
    times = []
    for i in range(args.warmup + args.steps):
        for tr in trainers:
            tr.init_embeddings()
        bt.launch()
        ms = bt.last_ms()
        if i >= args.warmup:
            times.append(ms)
        log(f"[bench] C4 batched launch {i}: {ms:.1f} ms")
    assert bt.done() == [sp["T"] for sp in specs]
    seq_ms = 0.0
    for tr in trainers:
        tr.init_embeddings()
        tr.train_steps(0, tr.T)
        seq_ms += tr.last_train_ms()
    ms = median(times)
    achieved = algo_bytes / (ms * 1e-3) / 1e9
    return {
        "metric": "edge samples/sec, 64 graphs in one persistent hipGraph launch (bf16 tables)",
        "value": total_T / (ms * 1e-3), "unit": "edge samples/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "table_dtype": "bf16", "data": "synthetic",
        "config": {"workload": "C4: 64 directed R-MAT graphs, n log-uniform 1e3..2e6, mean degree 8..32, "
                               "lognormal weights, d in {64,128}, K=5, second order, bf16 tables, T_g = 20 m_g",
                   "graphs": len(specs), "total_samples": total_T, "sum_m": sum(sp["m"] for sp in specs),
                   "hot_shadow": args.hot_shadow, "tiling": tuning, "tiling_from": "lh_batch_tune"},
        "sequential_launches": {"ms": seq_ms, "samples_per_s": total_T / (seq_ms * 1e-3),
                                "batched_speedup": seq_ms / ms},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                     "frac": achieved / PEAK_HBM_GBS, "traffic": None, "kernel": "k_batch (bf16)"},
    }


def bench_large(args):
    """C5: directed R-MAT scale 26 (2^26 nodes, 2^30 arcs), bfloat16, second order, 1e10
    samples.  C5U: the uniform-endpoint control at the same shape (no hub rows, so every row
    is cold: the kernel's raw random gather/scatter rate)."""
    import torch
    from paper_2604_09419_amd import Trainer
    from synth.graphs import rmat_graph_gpu, uniform_graph_gpu
    from synth import CONFIGS
    name = args.workload
    cfg = CONFIGS[name]
    t0 = time.time()
    if name == "C5U":
        src, dst, w = uniform_graph_gpu(cfg["n"], cfg["m_unique"], cfg["seed"])
    else:
        src, dst, w = rmat_graph_gpu(cfg["scale"], cfg["n"], cfg["m_unique"], cfg["seed"])
    torch.cuda.synchronize()
    log(f"[bench] {name} graph generated on the GPU in {time.time() - t0:.1f}s")
    host_graph = None
    if args.cpu_slice:
        from synth.graphs import Graph
        host_graph = Graph(n=cfg["n"], src=src.cpu().numpy(), dst=dst.cpu().numpy(), w=w.cpu().numpy())
        log(f"[bench] {name} graph copied to the host ({time.time() - t0:.1f}s)")
    T = int(cfg["T"]) if args.c5_samples is None else int(args.c5_samples)
    tr = Trainer(cfg["n"], src, dst, w, d=cfg["d"], K=cfg["K"], orders=cfg["orders"], dtype="bf16",
                 seed=cfg["seed"], total_samples=T, build=False, init=False, hot_shadow=args.hot_shadow)
    del src, dst, w
    tb = time.time()
    tr.build_alias()
    build_s = time.time() - tb
    walk_s = None
    if args.walks:
        tw = time.time()
        tr.build_walks(**WALK)
        walk_s = time.time() - tw
        log(f"[bench] {name} walk rows built in {walk_s:.2f}s")
    tr.init_embeddings()
    tr.train_steps(0, T)
    ms = tr.last_train_ms()
    tr.check()
    bps = algorithmic_bytes_per_sample(cfg["d"], cfg["K"], cfg["orders"], 2)
    achieved = bps * T / (ms * 1e-3) / 1e9
    graph = ("uniform random endpoints (control), unit weights" if name == "C5U"
             else "directed R-MAT scale 26, lognormal weights")
    kcfg = tr.kernel_config()
    cpu = None
    if host_graph is not None:
        tr.close()
        del tr
        torch.cuda.empty_cache()
        cpu = cpu_baseline(dict(cfg, T=T), host_graph, cfg["seed"], label=f"{name} workload")
        log(f"[bench] cpu baseline {cpu['value']:.3e} samples/s")
    out = {
        "metric": f"edge samples/sec at d=128,K=5 ({name}, bf16{', random-walk pairs' if args.walks else ''})",
        "value": T / (ms * 1e-3),
        "unit": "edge samples/s", "n_gpus": 1, "steps": 1, "warmup": 0, "ms_per_step": ms,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "table_dtype": "bf16", "data": "synthetic",
        "config": {"workload": f"{name}: {graph}, 67108864 nodes, 2^30 arcs, d=128, K=5, second order, "
                               "bf16 tables", "T": T,
                   "kernel_config": kcfg, "alias_build_s": build_s, "hot_shadow": args.hot_shadow,
                   "pairs": f"random walks {WALK}, walk rows built in {walk_s:.2f} s" if args.walks else "arc draws"},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                     "frac": achieved / PEAK_HBM_GBS, "traffic": None, "kernel": "k_hogwild (bf16, order 2)",
                     "bytes_per_sample": bps},
    }
    if cpu is not None:
        out["cpu_baseline"] = cpu
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="C2", choices=["C2", "C4", "C5", "C5U"])
    ap.add_argument("--c5-samples", type=float, default=None, help="override T for C5 and C5U")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle CPU baseline")
    ap.add_argument("--cpu-slice", action="store_true",
                    help="C5 and C5U: also time the oracle's binary32 lock-free mode on the host over a "
                         "bounded prefix (builds the oracle's tables for 2^30 arcs: minutes, ~130 GB of "
                         "host memory)")
    ap.add_argument("--no-bf16", action="store_true", help="skip the bfloat16 leg")
    ap.add_argument("--no-auc", action="store_true")
    ap.add_argument("--no-c3-error", action="store_true", help="skip the C3 embedding-error leg")
    ap.add_argument("--no-walks", action="store_true", help="skip the random-walk and pair-pool legs")
    ap.add_argument("--no-f1", action="store_true", help="skip the node-classification leg")
    ap.add_argument("--walks", action="store_true",
                    help="C5 and C5U: positive pairs from random walks (the training call includes the walks)")
    ap.add_argument("--hot-shadow", action="store_true",
                    help="bfloat16 runs: hot rows accumulate in a binary32 shadow per launch")
    ap.add_argument("--tune-cache", default=os.path.join(ROOT, "paper_2604_09419_amd", "tune_cache.json"))
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain device copy of 2 GiB three times (HBM counter scale)")
    args = ap.parse_args()

    if args.copy_calibration:
        import torch
        n = 1 << 31
        a = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(1)
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_per_dispatch": n}), flush=True)
        return

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on one GPU only: the library has no multi-GPU path "
              "(the sharded design is described, not built).", file=sys.stderr)
        sys.exit(2)

    import torch
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    os.makedirs(os.path.dirname(args.tune_cache), exist_ok=True)

    if args.workload == "C4":
        print(json.dumps(bench_batched(args)), flush=True)
        return
    if args.workload in ("C5", "C5U"):
        print(json.dumps(bench_large(args)), flush=True)
        return

    cfg, g, hs, hd, neg = workload(args.workload)
    seed = cfg["seed"]
    tr, step_ms, kern_ms = run_gpu_leg(cfg, g, "fp32", args.steps, args.warmup, seed, args.tune_cache)
    T = int(cfg["T"])
    ms_step = median(step_ms)
    ms_kern = median(kern_ms)
    bps = algorithmic_bytes_per_sample(cfg["d"], cfg["K"], cfg["orders"], 4)
    achieved = bps * T / (ms_kern * 1e-3) / 1e9
    traffic = measured_traffic(TRAFFIC_PROFILE, tr.kernel_config(), T)

    result = {
        "metric": METRIC,
        "value": T / (ms_step * 1e-3),
        "unit": "edge samples/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": "C2: directed R-MAT scale 20 (a,b,c=0.57,0.19,0.19), 1048576 nodes, "
                        f"{g.m} training arcs (1% of 2^24 held out), lognormal(0,1) weights, d=128, K=5, "
                        "orders 1+2, binary32 tables, T=2e8 edge samples, eta 0.025 linear decay, Hogwild",
            "n": g.n, "m": g.m, "d": cfg["d"], "K": cfg["K"], "orders": cfg["orders"], "T": T,
            "kernel_config": tr.kernel_config(),
        },
        "train_only": {"samples_per_s": T / (ms_kern * 1e-3), "ms": ms_kern},
        "roofline": {
            "bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
            "frac": achieved / PEAK_HBM_GBS, "traffic": traffic,
            "kernel": "k_hogwild (binary32, orders 1+2)", "bytes_per_sample": bps,
            "algorithmic_bytes_per_launch": bps * T,
            "traffic_over_algorithmic": None if traffic is None else traffic / (bps * T),
        },
    }
    if not args.no_auc:
        t0 = time.time()
        result["auc_fp32"] = held_out_auc(tr, hs, hd, neg, cfg["orders"])
        log(f"[bench] fp32 AUC {result['auc_fp32']} ({time.time() - t0:.1f}s)")
    tr.close()
    del tr
    torch.cuda.empty_cache()

    if not args.no_bf16:
        tb, bsteps, bkern = run_gpu_leg(cfg, g, "bf16", max(1, args.steps), 1, seed, args.tune_cache,
                                        hot_shadow=args.hot_shadow)
        bms = median(bkern)
        bstep = median(bsteps)
        bbps = algorithmic_bytes_per_sample(cfg["d"], cfg["K"], cfg["orders"], 2)
        bach = bbps * T / (bms * 1e-3) / 1e9
        result["bf16"] = {
            "samples_per_s": T / (bstep * 1e-3),
            "train_only_samples_per_s": T / (bms * 1e-3),
            "speedup_train_vs_fp32": ms_kern / bms,
            "speedup_step_vs_fp32": ms_step / bstep,
            "kernel_config": tb.kernel_config(),
            "hot_shadow": args.hot_shadow,
            "roofline": {"bound": "hbm", "achieved": bach, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                         "frac": bach / PEAK_HBM_GBS, "bytes_per_sample": bbps},
        }
        if not args.no_auc:
            result["bf16"]["auc"] = held_out_auc(tb, hs, hd, neg, cfg["orders"])
            log(f"[bench] bf16 AUC {result['bf16']['auc']}")
        tb.close()
        del tb
        torch.cuda.empty_cache()

    if not args.no_walks:
        result["walks"] = walk_legs(args, cfg, g, hs, hd, neg, seed, T)
        result["pool"] = walk_legs(args, cfg, g, hs, hd, neg, seed, T, pool=True)
    if not args.no_f1:
        result["node_classification"] = node_classification(args)
        log(f"[bench] node classification {result['node_classification']}")

    gold_path = os.path.join(GOLDEN, "c2_oracle_auc.json")
    if os.path.exists(gold_path):
        gold = json.load(open(gold_path))
        ref = {k[4:]: v for k, v in gold.items() if k.startswith("auc_") and not k.startswith("auc_init")}
        result["auc_oracle_binary64"] = ref
        # every score within 0.005 of the oracle's, for each dtype that was measured
        for key, got in (("fp32", result.get("auc_fp32")), ("bf16", result.get("bf16", {}).get("auc"))):
            if got:
                result.setdefault("auc_within_0.005_of_oracle", {})[key] = all(
                    abs(v - ref[k]) <= 0.005 for k, v in got.items())

    if not args.no_c3_error and not args.no_bf16:
        result["c3_embedding_error"] = c3_embedding_error(cfg, g, seed)
        log(f"[bench] C3 embedding error {result['c3_embedding_error']}")

    if not args.no_cpu:
        result["cpu_baseline"] = cpu_baseline(cfg, g, seed)
        log(f"[bench] cpu baseline {result['cpu_baseline']['value']:.3e} samples/s")
        result["cpu_baseline"]["seq_binary64"] = oracle_seq_timings(g, cfg, seed)
        log(f"[bench] oracle SEQ timings {result['cpu_baseline']['seq_binary64']}")

    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
