#!/usr/bin/env python3
"""Benchmark of the all-pairs Needleman-Wunsch hot path on one MI355X.

Default workload (the paper's scale): 600,000 synthetic words (40-symbol
Zipf(1.1) alphabet, lengths clip(Poisson(8), 1, 32)), scoring +1/-1, gap -1;
one step = the whole all-pairs pass producing every word's top-32 neighbours
(int16 score, int32 index, ties by lower index) and the global score
histogram: n(n-1)/2 = 1.8e11 pairs, every pair scored once.

    python bench.py [--steps K] [--warmup W] [--workload paper|mid|small|batched|diag|edges|export] [--cpu-seconds S]

Prints one JSON line.  --gpus N with N > 1 exits: the benchmark measures one GPU.
"""
from __future__ import annotations

import argparse
import concurrent.futures as cf
import json
import os
import platform
import subprocess
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "all-pairs NW GCUPS + pairs/s at 600k words; served query p50/p99 latency"
# Scores are exact integers: held in bit planes (words up to 48 symbols under
# symmetric scorings of weights 0..7), else as whole numbers in binary16 halves.
# The roofline of the packed binary16 DP kernels.  Every cell needs one packed add and one
# packed three-input max per two cells (two pairs share a register, one in
# each 16-bit half), i.e. one VALU lane-instruction per cell, and nothing in
# the recurrence can fuse the add into the max.  The ceiling is therefore the
# VALU issue rate: 256 CUs x 64 lanes x 2.4 GHz lane-instructions/s, one cell
# each.  `frac` is measured cells/s over that ceiling.
PEAK_ISSUE_CELLS = 256 * 64 * 2.4e9
# The roofline of the bit-plane kernels (csrc/nw_bits.h): a cell of 32 pairs
# takes 7 three-input functions where every match weighs 3 and every mismatch
# 1 (two planes), and 22 with three planes.  The rate at which the card issues
# them (v_bitop3_b32, more than the packed unit's) is measured in the same run
# (nw_function_issue_rate); over the functions of a cell it is the ceiling.
BIT_FUNCTIONS = {2: 7, 3: 22}


def bit_planes(planes: int) -> int:
    """Planes the kernels of a workload hold: none where NW_DP=packed keeps the packed ones."""
    return 0 if os.environ.get("NW_DP") == "packed" else planes


# The algorithmic operation count of a cell (2 adds, 2 maxes, 1 similarity
# lookup: Algorithm 1 with max(up, left) + p hoisted) against the nominal
# packed 16-bit rate (256 x 64 x 2 halves x 2.4 GHz).  Reported beside the
# roofline for reference only: the kernels issue fewer instructions than these
# operations (the change of variables drops the gap adds, max3 does two maxes,
# the similarity is an LDS read), so this ratio is not bounded by 1.
OPS_PER_CELL = 5
PEAK_16BIT_OPS = 256 * 64 * 2 * 2.4e9


def roofline(cells: float, seconds: float, kernel: str, traffic=None, algorithmic_bytes=None, planes=0,
             function_rate=None) -> dict:
    """The roofline record of a DP kernel pass that updates `cells` cells in
    `seconds`; planes: 2 or 3 for the bit-plane kernels (function_rate: their
    functions per second as measured), 0 for the packed ones."""
    rate = cells / seconds
    peak = 32 * function_rate / BIT_FUNCTIONS[planes] if planes else PEAK_ISSUE_CELLS
    rec = {"bound": "alu", "achieved": round(rate / 1e12, 3), "peak": round(peak / 1e12, 3),
           "unit": "10^12 DP cells/s (VALU issue ceiling: " +
                   (f"{BIT_FUNCTIONS[planes]} functions per 32 cells)" if planes else "one packed lane-instruction per cell)"),
           "frac": round(rate / peak, 4),
           "traffic": None if traffic is None else round(traffic),
           "kernel": kernel,
           "ops_16bit": {"ops_per_cell": OPS_PER_CELL, "achieved_Tops": round(OPS_PER_CELL * rate / 1e12, 2),
                         "nominal_peak_Tops": round(PEAK_16BIT_OPS / 1e12, 2),
                         "ratio": round(OPS_PER_CELL * rate / PEAK_16BIT_OPS, 4),
                         "note": "algorithmic op count over the nominal packed rate; not a roofline fraction"}}
    if traffic is not None and algorithmic_bytes:
        rec["algorithmic_bytes"] = round(algorithmic_bytes)
        rec["traffic_over_algorithmic"] = round(traffic / algorithmic_bytes, 2)
    return rec

# HBM bytes of the main pass from rocprofv3 FETCH_SIZE / WRITE_SIZE runs, kept in
# this summary together with the SHA-256 of the sources the kernel was built from
COUNTER_SUMMARY = os.path.join(ROOT, "profiles", "topk_main_paper600k_counters.md")
MAIN_PASS_SOURCES = ["nw_internal.h", "nw_bits.h", "nw_tile_common.h", "nw_topk.h", "k_topk.h", "k_topk_bits.h",
                     "k_launch.hip", "k_bits_inst.hip", "nw_api.cpp"]
# the same for the 50,000-word int8 triangle (k_tri_bits)
TRI_COUNTER_SUMMARY = os.path.join(ROOT, "profiles", "tri_bits_mid50k_counters.md")
TRI_SOURCES = ["nw_internal.h", "nw_bits.h", "nw_tile_common.h", "k_tri_bits.h", "k_launch.hip", "k_tri_bits_inst.hip",
               "nw_api.cpp"]


def sources_sha256(names) -> str:
    import hashlib
    h = hashlib.sha256()
    for name in names:
        with open(os.path.join(ROOT, "paper_2509_01654_amd", "csrc", name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    return h.hexdigest()


def main_pass_sources_sha256() -> str:
    return sources_sha256(MAIN_PASS_SOURCES)


def _summary_fields(prefix, path=None):
    try:
        text = open(path or COUNTER_SUMMARY, encoding="utf-8").read()
    except OSError:
        return {}
    fields = {}
    for line in text.splitlines():
        if line.startswith(prefix):
            for kv in line[len(prefix):].split():
                k, _, val = kv.partition("=")
                fields[k] = val
    return fields


def counter_traffic(path=None, sources=None):
    """(bytes fetched, bytes written) per pass from a counter summary (the main
    pass by default), or None when there is none or the kernel sources changed
    since it was taken."""
    fields = _summary_fields("traffic:", path)
    if fields.get("sources_sha256") != sources_sha256(sources or MAIN_PASS_SOURCES):
        return None
    return float(fields["fetch_bytes"]), float(fields["write_bytes"])


def measured_rate(issue, torch, blocks=2048, trips=4096, runs=3):
    """The lane-instruction rate the chip sustains during this run: the launch of
    nw.packed_issue_rate (the packed DP's add + max3 pair) or
    nw.function_issue_rate (the bit planes' function), independent chains, every
    CU at full occupancy, timed with events on the current stream; the best of
    `runs` after one warm-up launch."""
    issue(blocks, trips)
    best = 0.0
    for _ in range(runs):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        n_instr = issue(blocks, trips)
        e1.record()
        torch.cuda.synchronize()
        best = max(best, n_instr / (e0.elapsed_time(e1) / 1e3))
    return best


def counter_issue():
    """VALU and LDS figures of the main pass from the same summary (same gate)."""
    fields = _summary_fields("counters:")
    if fields.pop("sources_sha256", None) != main_pass_sources_sha256():
        return None
    return {k: float(v) for k, v in fields.items()}


# The paper's own GPU timings (a GTX 1060, i8 output, the device-to-host copy
# included): context for the numbers here, not a baseline of this metric.
PAPER_CONTEXT = {"gpu": "NVIDIA GTX 1060 6 GB (paper, Section 5)",
                 "runs": [{"words": 20000, "ms": 484, "pairs_per_s": 4.1e8},
                          {"words": 107000, "s": 21.3, "pairs_per_s": 2.7e8}],
                 "note": "i8 triangle incl. D2H copy; no GCUPS, top-k, batched or served numbers are published"}


def host_cpu_model() -> str:
    try:
        out = subprocess.run(["lscpu"], capture_output=True, text=True).stdout
        for line in out.splitlines():
            if line.startswith("Model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or "unknown"


def cpu_baseline(v, k, gpu_scores, gpu_index, budget_s):
    """The oracle on a bounded sample of rows (each row: all n-1 partners).

    Returns the baseline record and whether the sampled rows match the GPU."""
    import numpy as np
    import oracle
    threads = oracle.default_threads()
    sim = oracle.sim_matrix(v.alphabet, 1, -1)
    L = v.lengths
    total_l = int(L.sum())
    rng = np.random.default_rng(12345)
    order = rng.permutation(v.n)
    done, cells, t_used, ok = 0, 0, 0.0, True
    while t_used < budget_s and done < v.n:
        rows = order[done:done + threads]
        t0 = time.perf_counter()
        # the oracle splits rows over its threads; one row per call runs single-threaded,
        # so a batch of `threads` single-row calls runs side by side
        res = [None] * len(rows)
        with cf.ThreadPoolExecutor(max_workers=len(rows)) as ex:
            futs = {ex.submit(oracle.topk_rows, v.symbols, v.offsets, sim, -1, k, int(r), int(r) + 1, None, 1): t
                    for t, r in enumerate(rows)}
            for f in cf.as_completed(futs):
                res[futs[f]] = f.result()
        t_used += time.perf_counter() - t0
        for t, r in enumerate(rows):
            ws, wi, _ = res[t]
            ok &= bool((gpu_index[r] == wi[0]).all() and (gpu_scores[r] == ws[0]).all())
            cells += int(L[r]) * (total_l - int(L[r]))
        done += len(rows)
    rec = {"value": cells / t_used / 1e9, "unit": "GCUPS", "cores": threads, "kind": "oracle",
           "sample": f"{done} random rows x all {v.n - 1} partners each (top-{k} kept in a sorted list), "
                     f"{cells:.3e} cells in {t_used:.1f} s on {host_cpu_model()}",
           "pairs_per_s": done * (v.n - 1) / t_used}
    return rec, ok, done


def serve(nw, dv, rates, nq, main_ms, cells):
    """Served form: open-loop Poisson arrivals against the resident dictionary."""
    import numpy as np
    import synth
    k = 16
    srv = nw.Server(dv, k=k, max_batch=256, num_slots=4)
    # warm the server's kernels
    wq = synth.query_words(512, seed=49)
    srv.replay(wq.symbols, wq.offsets, np.linspace(0, 0.01, wq.n))
    out = []
    total_l = int(dv.offsets[-1])
    for t, rate in enumerate(rates):
        q = synth.query_words(nq, seed=50 + t)
        arr = synth.poisson_arrivals(rate, q.n, seed=150 + t)
        b0, _ = srv.stats()
        t0 = time.perf_counter()
        sc, ix, lat = srv.replay(q.symbols, q.offsets, arr)
        wall = time.perf_counter() - t0
        b1, _ = srv.stats()
        qcells = int(q.lengths.sum()) * total_l
        out.append({"offered_qps": rate, "queries": q.n, "achieved_qps": round(q.n / wall, 1),
                    "p50_ms": round(float(np.percentile(lat, 50)) * 1e3, 3),
                    "p99_ms": round(float(np.percentile(lat, 99)) * 1e3, 3),
                    "batches": b1 - b0, "gcups_while_serving": round(qcells / wall / 1e9, 1)})
    srv.close()
    return {"workload": "top-16 per query against the resident 600,000-word dictionary; queries drawn like the "
                        "dictionary, open-loop Poisson arrivals; latency = completion - scheduled arrival",
            "k": k, "max_batch": 256, "slots": 4, "rates": out,
            "plain_main_pass_gcups": round(cells / (main_ms / 1e3) / 1e9, 1)}


def bench_batched(args, nw, synth, torch, dev):
    """Eight vocabularies (1k..100k words, lengths 1..8 .. 1..48, 64-symbol
    substitution matrix, gap -2), every triangle as int16: one graph-captured
    persistent run per step, against per-dictionary plain launches."""
    import numpy as np
    vocabs, S = synth.batched_configs()
    sc = nw.Scoring(64, submat=S, gap=-2)
    dvs = [nw.Vocab(v.symbols, v.offsets, sc, device=dev) for v in vocabs]
    pairs = sum(d.num_pairs for d in dvs)
    cells = sum(d.num_cells for d in dvs)
    # the autotuner's cache of best settings per device and workload signature
    import tempfile
    cache = os.environ.get("NW_AUTOTUNE_CACHE") or os.path.join(tempfile.gettempdir(), "nw_autotune.jsonl")
    t0 = time.perf_counter()
    b = nw.Batch(dvs, torch.int16, autotune=True, cache_path=cache)
    tune_s = time.perf_counter() - t0

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1)
    # comparisons first (so the timed replays are the last kernels of a trace):
    # the plain per-dictionary calls, and the persistent form, on the same outputs
    plain_ms = float(np.sum([timed(lambda d=d, o=o: d.all_pairs_scores(dtype=torch.int16, out=o))
                             for d, o in zip(dvs, b.outs)]))
    pb = nw.Batch(dvs, torch.int16, class_width=1, wg_per_cu=4, pairs_per_item=16, use_graph=True, outs=b.outs)
    persistent_ms = timed(pb.run)
    pb.close()
    for _ in range(args.warmup):
        b.run()
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record()
    for _ in range(args.steps):
        b.run()
    ev1.record()
    torch.cuda.synchronize()
    ms = ev0.elapsed_time(ev1) / args.steps
    items, launches = b.info()
    return {
        "metric": METRIC, "value": round(cells / (ms / 1e3) / 1e9, 1), "unit": "GCUPS", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 3), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "int16", "data": "synthetic",
        "pairs_per_s": pairs / (ms / 1e3),
        "config": {"workload": "batched: 8 vocabularies 1k..100k words, uniform lengths 1..8 .. 1..48, 64-symbol "
                               "seeded symmetric matrix in [-3,3] (diag +3), gap -2, every triangle as int16",
                   "pairs": pairs, "cells": cells, "options": b.options, "items": items, "launches": launches,
                   "autotune_s": round(tune_s, 1)},
        "roofline": roofline(cells, ms / 1e3,
                             (("k_tri_bits" if bit_planes(3) else "k_tri_code") + " (every dictionary's launches"
                              + (", graph replay)" if b.options["use_graph"] else ", eager on forked streams)")
                              if b.options["class_width"] == 0 else "k_tri_persist (graph replay)"),
                             planes=bit_planes(3) if b.options["class_width"] == 0 else 0,
                             function_rate=measured_rate(nw.function_issue_rate, torch)),
        "output_GB_per_s": round(2 * pairs / (ms / 1e3) / 1e9, 1),
        "plain_per_dictionary_ms": round(plain_ms, 3),
        "plain_gcups": round(cells / (plain_ms / 1e3) / 1e9, 1),
        "persistent_form_ms": round(persistent_ms, 3),
    }


def _time(fn, torch, steps):
    fn()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        fn()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / steps


def bench_diag(args, nw, synth, torch, dev):
    """Anti-diagonal kernel against the register-row kernel on the longest
    batched vocabulary (100,000 words, lengths 1..48), and alone on words of
    up to 255 symbols."""
    vocabs, S = synth.batched_configs()
    sc = nw.Scoring(64, submat=S, gap=-2)
    v = vocabs[-1]
    dv = nw.Vocab(v.symbols, v.offsets, sc, device=dev)
    out = torch.empty(dv.num_pairs, dtype=torch.int16, device=dev)
    t_row = _time(lambda: dv.all_pairs_scores(dtype=torch.int16, out=out), torch, args.steps)
    t_diag = _time(lambda: dv.all_pairs_scores_diag(dtype=torch.int16, out=out), torch, args.steps)
    lv = synth.uniform_vocab(20000, seed=90, alphabet=64, min_len=1, max_len=255)
    dl = nw.Vocab(lv.symbols, lv.offsets, sc, device=dev)
    out2 = torch.empty(dl.num_pairs, dtype=torch.int16, device=dev)
    t_long = _time(lambda: dl.all_pairs_scores(dtype=torch.int16, out=out2), torch, args.steps)
    return {"workload": "anti-diagonal vs register-row kernel", "steps": args.steps,
            "short_words": {"words": dv.n, "lengths": "1..48", "cells": dv.num_cells,
                            "register_row_ms": round(t_row, 3), "anti_diagonal_ms": round(t_diag, 3),
                            "register_row_gcups": round(dv.num_cells / t_row / 1e6, 1),
                            "anti_diagonal_gcups": round(dv.num_cells / t_diag / 1e6, 1)},
            "long_words": {"words": dl.n, "lengths": "1..255", "cells": dl.num_cells, "ms": round(t_long, 3),
                           "gcups": round(dl.num_cells / t_long / 1e6, 1)}}


def bench_edges(args, nw, synth, torch, dev):
    """Threshold edges of the 600,000-word dictionary in the normalised slice
    [60, 100] (the slice of the paper's ego networks): every pair scored, the
    passing pairs appended as (i, j, score)."""
    v = synth.plain_config("paper")
    dv = nw.Vocab(v.symbols, v.offsets, nw.Scoring(40, 1, -1, -1), device=dev)
    cnt = torch.empty(1, dtype=torch.int64, device=dev)
    _, _, _, total = dv.all_pairs_edges(60, 100, True, 1, cap=0, count=cnt)
    cap = total + 1024
    out = (torch.empty(cap, dtype=torch.int32, device=dev), torch.empty(cap, dtype=torch.int32, device=dev),
           torch.empty(cap, dtype=torch.int16, device=dev))

    def step():
        return dv.all_pairs_edges(60, 100, True, 1, cap=cap, out=out, count=cnt)[3]

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        c = step()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    assert c == total
    cells, E = dv.num_cells, dv.num_pairs
    return {"metric": METRIC, "value": round(cells / (ms / 1e3) / 1e9, 1), "unit": "GCUPS", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 3), "higher_is_better": True,
            "scaling": "weak", "vs_baseline": None, "dtype": "int16", "data": "synthetic",
            "pairs_per_s": E / (ms / 1e3),
            "config": {"workload": "threshold edges, normalised weight in [60, 100], 600,000 words (Zipf-40, "
                                   "clip(Poisson 8, 1, 32), +1/-1, gap -1)", "n_words": dv.n, "pairs": E,
                       "cells": cells, "edges": total},
            "edges_per_s": total / (ms / 1e3), "edge_bytes_per_s": 10 * total / (ms / 1e3),
            "roofline": roofline(cells, ms / 1e3, "k_edges_bits (every LA)" if bit_planes(2) else "k_edges_tiled (every LA)",
                                 planes=bit_planes(2), function_rate=measured_rate(nw.function_issue_rate, torch))}


def bench_export(args, nw, synth, torch, dev):
    """The whole int8 triangle of the 600,000-word dictionary streamed to page-
    locked host memory in 1 GiB chunks (nw_export_triangle); the consumer only
    touches each chunk.  The rate includes the device-to-host copies."""
    v = synth.plain_config("paper")
    dv = nw.Vocab(v.symbols, v.offsets, nw.Scoring(40, 1, -1, -1), device=dev)
    chunk = 1 << 30
    ws = torch.empty(2 * chunk, dtype=torch.uint8, device=dev)
    host = torch.empty(2 * chunk, dtype=torch.uint8, pin_memory=True)
    got = [0]

    def consume(b0, scores):
        got[0] += len(scores)

    def step():
        dv.export_triangle(consume, dtype=torch.int8, chunk_pairs=chunk, ws=ws, host=host)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    got[0] = 0
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    E, cells = dv.num_pairs, dv.num_cells
    assert got[0] == E * args.steps
    return {"metric": METRIC, "value": round(cells / (ms / 1e3) / 1e9, 1), "unit": "GCUPS", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 3), "higher_is_better": True,
            "scaling": "weak", "vs_baseline": None, "dtype": "int16", "data": "synthetic",
            "pairs_per_s": E / (ms / 1e3),
            "config": {"workload": "streamed int8 triangle export to host, 600,000 words (Zipf-40, clip(Poisson 8, "
                                   "1, 32), +1/-1, gap -1), 1 GiB chunks", "n_words": dv.n, "pairs": E,
                       "cells": cells, "bytes": E},
            "host_GB_per_s": round(E / (ms / 1e3) / 1e9, 2)}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", choices=["paper", "mid", "small", "batched", "diag", "edges", "export"],
                    default="paper")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--serve-rates", default="2000,5000,10000,20000,50000",
                    help="offered query rates (q/s) for the served form; empty to skip")
    ap.add_argument("--serve-queries", type=int, default=20000)
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run a plain 1 GiB device copy 4 times (calibrates HBM byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path.",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2509_01654_amd as nw
    import synth

    torch.cuda.set_device(0)
    dev = torch.device("cuda:0")
    if args.calibrate_copy:
        src = torch.ones(1 << 30, dtype=torch.uint8, device=dev)
        dst = torch.empty_like(src)
        for _ in range(4):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"calibration": "device copy", "bytes_read_per_copy": 1 << 30,
                          "bytes_written_per_copy": 1 << 30, "copies": 4}), flush=True)
        return
    if args.workload == "batched":
        print(json.dumps(bench_batched(args, nw, synth, torch, dev)), flush=True)
        return
    if args.workload == "diag":
        print(json.dumps(bench_diag(args, nw, synth, torch, dev)), flush=True)
        return
    if args.workload == "edges":
        print(json.dumps(bench_edges(args, nw, synth, torch, dev)), flush=True)
        return
    if args.workload == "export":
        print(json.dumps(bench_export(args, nw, synth, torch, dev)), flush=True)
        return
    v = synth.plain_config(args.workload)
    dv = nw.Vocab(v.symbols, v.offsets, nw.Scoring(40, 1, -1, -1), device=dev)
    E, cells = dv.num_pairs, dv.num_cells
    k = 32
    stream = torch.cuda.current_stream()

    if args.workload == "paper":
        ws = torch.empty(dv.topk_workspace_bytes(k), dtype=torch.uint8, device=dev)
        out = (torch.empty((dv.n, k), dtype=torch.int16, device=dev),
               torch.empty((dv.n, k), dtype=torch.int32, device=dev),
               torch.empty(dv.bounds[1] - dv.bounds[0] + 1, dtype=torch.int64, device=dev))

        def step():
            dv.all_pairs_topk(k, ws=ws, out=out)
    else:
        tri = torch.empty(E, dtype=torch.int8, device=dev)

        def step():
            dv.all_pairs_scores(dtype=torch.int8, out=tri)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    phases = []
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev0.record(stream)
    for _ in range(args.steps):
        step()
        if args.workload == "paper":
            phases.append(dv.topk_phase_times())
    ev1.record(stream)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_per_step = (t1 - t0) * 1e3 / args.steps
    value = cells / (ms_per_step / 1e3) / 1e9

    rec = {
        "metric": METRIC,
        "value": round(value, 1),
        "unit": "GCUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int16",
        "data": "synthetic",
        "pairs_per_s": E / (ms_per_step / 1e3),
    }
    if args.workload == "paper":
        pre, main_ms, sel = (float(np.mean([p[i] for p in phases])) for i in range(3))
        rec["config"] = {"workload": "all-pairs top-32 neighbours + score histogram, 600,000 words "
                                     "(Zipf-40, clip(Poisson 8, 1, 32), +1/-1, gap -1)",
                         "n_words": dv.n, "k": k, "pairs": E, "cells": cells}
        rec["phase_ms"] = {"threshold_prepass": round(pre, 3), "main_pass": round(main_ms, 3),
                           "select": round(sel, 3)}
        rec["overflow_words"] = dv.topk_overflow_words()
        rec["paper_context"] = PAPER_CONTEXT
        tr = counter_traffic()
        # algorithmic bytes of the main pass: the words read once (48-byte
        # slots) and every word's top-k list written once (int16 + int32)
        alg_bytes = dv.n * 48 + dv.n * k * 6
        function_rate = measured_rate(nw.function_issue_rate, torch)
        rec["roofline"] = roofline(cells, main_ms / 1e3,
                                   "k_topk_bits (all-pairs main pass, every class)" if bit_planes(2)
                                   else "k_topk_code (all-pairs main pass, every length)",
                                   None if tr is None else tr[0] + tr[1], alg_bytes, planes=bit_planes(2),
                                   function_rate=function_rate)
        rec["roofline"]["function_peak"] = {
            "kernel": "k_function_rate (nw_function_issue_rate: the bit planes' function, independent chains)",
            "lane_functions_per_s": round(function_rate / 1e12, 3), "unit": "10^12 lane-functions per s"}
        rate = measured_rate(nw.packed_issue_rate, torch)
        rec["roofline"]["packed_peak"] = {
            "kernel": "k_packed_rate (nw_packed_issue_rate: the packed DP's add + max3, independent chains)",
            "cells_per_s": round(rate / 1e12, 3), "unit": "10^12 packed lane-instructions (= cells of the packed DP) per s",
            "note": "the packed kernels' measured ceiling; the bit planes pass it"}
        iss = counter_issue()
        if iss is not None:
            rec["roofline"]["counters"] = iss
        if tr is not None:
            rec["roofline"]["traffic_detail"] = {
                "unit": "HBM bytes per main pass (calibrated rocprofv3 FETCH_SIZE + WRITE_SIZE)",
                "fetch": round(tr[0]), "write": round(tr[1]),
                "GB_per_s": round((tr[0] + tr[1]) / (main_ms / 1e3) / 1e9, 1),
                "frac_of_hbm_peak": round((tr[0] + tr[1]) / (main_ms / 1e3) / 8e12, 4)}
        if args.serve_rates:
            rec["served"] = serve(nw, dv, [float(r) for r in args.serve_rates.split(",")], args.serve_queries,
                                  rec["phase_ms"]["main_pass"], cells)
        sc, ix, h = out
        hist = h.cpu().numpy()
        assert int(hist.sum()) == E, "histogram does not count every pair once"
        if not args.no_cpu:
            cb, ok, rows = cpu_baseline(v, k, sc.cpu().numpy().astype(np.int32), ix.cpu().numpy(), args.cpu_seconds)
            rec["cpu_baseline"] = cb
            rec["parity_sample"] = {"rows": rows, "bit_exact": ok}
    else:
        rec["config"] = {"workload": f"all-pairs int8 triangle, {dv.n:,} words (Zipf-40, clip(Poisson 7, 1, 20), "
                                     "+1/-1, gap -1)", "n_words": dv.n, "pairs": E, "cells": cells}
        tr = counter_traffic(TRI_COUNTER_SUMMARY, TRI_SOURCES) if args.workload == "mid" else None
        # algorithmic bytes: one int8 score written per pair, the words read once
        rec["roofline"] = roofline(cells, ms_per_step / 1e3, "k_tri_bits (every LA)" if bit_planes(2) else "k_tri_code",
                                   None if tr is None else tr[0] + tr[1], E + dv.n * 48, planes=bit_planes(2),
                                   function_rate=measured_rate(nw.function_issue_rate, torch))
        if tr is not None:
            # algorithmic bytes: one int8 score written per pair; the words read are ~1 MB
            rec["roofline"]["traffic_detail"] = {
                "unit": "HBM bytes per triangle (calibrated rocprofv3 FETCH_SIZE + WRITE_SIZE)",
                "fetch": round(tr[0]), "write": round(tr[1]), "algorithmic_write": E,
                "write_over_algorithmic": round(tr[1] / E, 4),
                "GB_per_s": round((tr[0] + tr[1]) / (ms_per_step / 1e3) / 1e9, 1)}
        rec["output_GB_per_s"] = E / (ms_per_step / 1e3) / 1e9
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
