#!/usr/bin/env python3
"""Benchmark of the libah path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload collection|plain]

A step is one primer-pair query over the packed genome collection resident in
HBM: site scan (both strands, <= k mismatches, clamp), canonical sort,
melting temperature of every site, and amplicon calling.  Inputs are seeded
synthetic genomes built on the GPU before the timed region; packing them from
ASCII is timed separately and reported as ``ingest``.  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import math
import multiprocessing as mp
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "genome Gbp/s scanned per primer pair at k mismatches; batched vs plain; p99 latency"
BATCHED_DESC = ("batched: 2,000 genomes (log-normal lengths clipped 0.5-12 Mbp) x 64 law pairs "
                "(L 15-30, degeneracy 2^0-2^10, k 0-3, windows 100-6000), one hipGraph replay per "
                "step, against the 64 pairs as sequential plain queries")
SERVE_DESC = ("serve: 100,000 genomes (log-normal lengths, median 4 Mbp, clipped 1-12 Mbp) resident "
              "in HBM, Poisson arrivals, each job one law pair (1,024-pair pool: L 15-30, degeneracy "
              "2^0-2^10, k 0-3) over a log-uniform subset of 10-100,000 genomes")
HBM_PEAK_GBS = 8000.0
SCAN_BYTES_PER_BP = 0.25  # 2-bit packed genome read once per query
# int32 VALU lane-ops/s: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz
ALU_PEAK_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12


def workload(name: str):
    from synth import plan

    if name == "plain":
        p = plan.plain()
        desc = ("plain: one 5 Mbp genome, GC 0.5, 5 planted 1.5 kbp operon copies at 1%; "
                "fwd 20 nt / rev 19 nt with 3 two-fold codes each; k=2, clamp 5, window 200-2000")
    else:
        p = plan.collection(1000, seed=13302)
        desc = ("collection: 1,000 genomes, log-normal lengths (median 4 Mbp, sigma 0.3, "
                "clipped 1-12 Mbp), GC U[0.3,0.7], 1-15 planted 1.5 kbp operons at 1%; "
                "V4-like pair 19/20 nt (degeneracy 4/8); k=2, no clamp, window 200-500")
    return p, desc


# ------------------------------------------------------------ CPU baseline --
def _gen(args):
    name, g = args
    from synth import fill

    p, _ = workload(name)
    return fill.genome_bytes(p, g)


def _oracle_one(args):
    name, g, seq = args
    from oracle import pair as opair
    from oracle import scan as oscan
    from oracle import tm as otm

    p, _ = workload(name)
    pr = p.pairs[0]
    h = oscan.scan_sequence(seq, pr.fwd, pr.rev, pr.k, pr.clamp)
    h["genome"] = 0  # the index of seq in the list fill_tm gets
    h = otm.fill_tm(h, [seq], [pr])
    h["genome"] = g
    a = opair.call_amplicons(h, [pr])
    return g, h, a


def host_cores():
    """(cores this process may run on, os.cpu_count())."""
    try:
        aff = len(os.sched_getaffinity(0))
    except AttributeError:
        aff = os.cpu_count() or 1
    return aff, os.cpu_count() or 1


def cpu_baseline(name: str, n_genomes: int, target_bp: float):
    """The oracle as it stands on the first genomes of the workload: on the
    host's cores (at most 16, one GPU's share of a shared host), and on one
    core.  Returns the figures and the oracle's records of the sample."""
    import concurrent.futures as cf

    import numpy as np

    p, _ = workload(name)
    ids, bp = [], 0
    for g in range(n_genomes):
        ids.append(g)
        bp += int(p.lengths[g])
        if bp >= target_bp:
            break
    aff, ncpu = host_cores()
    workers = max(1, min(16, aff, len(ids)))
    ctx = mp.get_context("spawn")
    with cf.ProcessPoolExecutor(workers, mp_context=ctx) as ex:
        seqs = list(ex.map(_gen, [(name, g) for g in ids]))
        t0 = time.perf_counter()
        out = list(ex.map(_oracle_one, [(name, g, s) for g, s in zip(ids, seqs)]))
        dt = time.perf_counter() - t0
    # one core: the same oracle in this process on the first genomes, about
    # a quarter of the sample
    t0 = time.perf_counter()
    one_bp, n_one = 0, 0
    for g, s in zip(ids, seqs):
        _oracle_one((name, g, s))
        one_bp += int(p.lengths[g])
        n_one += 1
        if one_bp >= bp / 4:
            break
    dt1 = time.perf_counter() - t0
    del seqs
    hits = np.concatenate([o[1] for o in out])
    amps, at = [], 0
    for o in out:
        a = o[2].copy()
        a["plus_hit"] += at
        a["minus_hit"] += at
        at += o[1].size
        amps.append(a)
    amps = np.concatenate(amps)
    return {
        "value": bp / dt / 1e9,
        "unit": "Gbp/s",
        "cores": workers,
        "kind": "oracle",
        "sample": (f"first {len(ids)} genomes of the same collection ({bp / 1e6:.1f} Mbp), "
                   f"oracle scan + Tm + pairing, one genome per task on {workers} worker "
                   f"processes; {dt:.2f} s wall"),
        "host_cores": {"affinity": aff, "os_cpu_count": ncpu, "workers": workers,
                       "note": "workers capped at 16, one GPU's share of the host"},
        "single_core": {"value": one_bp / dt1 / 1e9, "unit": "Gbp/s",
                        "sample": f"first {n_one} genomes ({one_bp / 1e6:.1f} Mbp) in one "
                                  f"process; {dt1:.2f} s"},
        "hits": int(hits.size),
    }, ids, hits, amps


def oracle_agreement(gh, ga, ids, oh, oa) -> dict:
    """The GPU records of the sample genomes (the first ones, so a prefix of
    the canonical output) against the oracle's: every site, every amplicon
    with its hit indices, and the Tm error."""
    import numpy as np

    n = len(ids)
    assert list(ids) == list(range(n))
    hsel = gh[gh["genome"] < n]
    asel = ga[ga["genome"] < n]
    got = [(int(x["genome"]), int(x["pos"]), int(x["strand_primer"]) >> 1,
            int(x["strand_primer"]) & 1, int(x["mm"])) for x in hsel]
    want = [(int(x["genome"]), int(x["pos"]), int(x["strand"]), int(x["primer"]), int(x["mm"]))
            for x in oh]
    ga_t = [(int(x["genome"]), int(x["start"]), int(x["end"]), int(x["orient"]),
             int(x["plus_hit"]), int(x["minus_hit"])) for x in asel]
    oa_t = [(int(x["genome"]), int(x["start"]), int(x["end"]), int(x["orient"]),
             int(x["plus_hit"]), int(x["minus_hit"])) for x in oa]
    equal = got == want and ga_t == oa_t
    err = (np.abs(hsel["tm"].astype(np.float64) - oh["tm"]) if got == want
           else np.array([np.inf]))
    return {"oracle_equal": bool(equal),
            "tm_error": {"max": float(err.max(initial=0.0)),
                         "mean": float(err.mean()) if err.size else 0.0, "n": int(err.size),
                         "unit": "C", "tolerance": 0.01},
            "genomes": n, "sites": len(want), "amplicons": len(oa_t)}


# ------------------------------------------------------------------ GPU --
def gpu_run(name: str, steps: int, warmup: int):
    import numpy as np
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu

    dev = torch.device("cuda:0")
    p, desc = workload(name)
    pr = p.pairs[0]
    ascii, off = gpu.fill_cuda(p, dev)
    torch.cuda.synchronize()
    # ingest: ASCII -> packed, timed on its own
    L.ah_profile_reset()
    L.ah_profile_enable(True)
    t0 = time.perf_counter()
    coll, _ = path.pack(ascii, off, p.lengths)
    torch.cuda.synchronize()
    pack_s = time.perf_counter() - t0
    L.ah_profile_enable(False)
    _, pack_ms = L.ah_profile_query("pack")
    del ascii
    torch.cuda.empty_cache()

    buf = path.alloc(coll, [pr], 1 << 22, 1 << 22, dev)
    jit0 = L.ah_jit_stats()
    for _ in range(max(1, warmup)):
        path.run(coll, [pr], buf)
    torch.cuda.synchronize()
    jit1 = L.ah_jit_stats()
    res_h = path.result(buf.hit_res)
    res_a = path.result(buf.amp_res)
    assert res_h["status"] == 0 and res_a["status"] == 0, (res_h, res_a)

    L.ah_profile_reset()
    L.ah_profile_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        path.run(coll, [pr], buf)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    L.ah_profile_enable(False)
    kern = {}
    for k in ("scan", "verify", "sort", "tm", "pair"):
        n, ms = L.ah_profile_query(k)
        kern[k] = ms / max(n, 1)
    traffic = None
    valu = None
    rec = os.path.join(ROOT, "profiles", f"ah_scan_kernel__{name}-{coll.n}.json")
    if os.path.exists(rec):
        import hashlib

        d = json.load(open(rec))
        sha = hashlib.sha256(L.ah_scan_program_source([pr], False).encode()).hexdigest()
        if d.get("program_sha256") == sha:  # counters were taken on this exact kernel
            traffic = d["traffic_bytes_per_dispatch"]
            valu = d.get("sq_insts_valu_per_dispatch")
    # the same pass captured once into a hipGraph and replayed
    graph = path.capture(coll, [pr], buf)
    for _ in range(max(1, warmup)):
        graph.replay()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        graph.replay()
    torch.cuda.synchronize()
    ms_graph = (time.perf_counter() - t0) * 1e3 / steps
    # the records compared with the oracle below are those of the last replay
    assert path.result(buf.hit_res)["count"] == res_h["count"]
    hits = path.hits_numpy(buf)
    amps = path.amps_numpy(buf)
    cands = L.ah_scan_candidate_stats(buf.scan_work, coll.n, buf.hit_cap)
    tm_ok = bool(np.all(np.isfinite(hits["tm"]))) if hits.size else True
    ms_step = dt * 1e3 / steps
    bp = coll.total_bp
    scan_bytes = SCAN_BYTES_PER_BP * bp
    achieved = scan_bytes / (kern["scan"] * 1e-3) / 1e9
    return {
        "bp": bp, "desc": desc, "ms_per_step": ms_step, "value": bp / (ms_step * 1e-3) / 1e9,
        "kernel_ms": kern, "hits": res_h["count"], "amplicons": res_a["count"], "tm_finite": tm_ok,
        "graph_replay": {"ms_per_step": ms_graph, "gbps": bp / (ms_graph * 1e-3) / 1e9},
        "scan_candidates": cands,
        "pack": {"ms": pack_ms, "wall_ms": pack_s * 1e3, "gbps": bp / (pack_ms * 1e-3) / 1e9},
        "jit": {"compiles": jit1[0] - jit0[0], "ms": jit1[1] - jit0[1]},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "kernel": "ah_scan_kernel", "algorithmic_bytes": scan_bytes,
                     "kernel_work": "filter over the packed genome, then each wave's exact "
                                    "count of its own candidates",
                     # the filter's VALU issue rate: the profiled instruction count of
                     # this exact program (64 lanes each) over the live kernel time
                     "valu_issue": None if valu is None else {
                         "achieved": valu * 64 / (kern["scan"] * 1e-3) / 1e12,
                         "peak": ALU_PEAK_TOPS, "unit": "T lane-ops/s",
                         "frac": valu * 64 / (kern["scan"] * 1e-3) / 1e12 / ALU_PEAK_TOPS,
                         "valu_insts_per_dispatch": valu}},
        "pair": {"fwd": pr.fwd, "rev": pr.rev, "k": pr.k, "clamp": pr.clamp,
                 "window": [pr.min_len, pr.max_len]},
        "genomes": coll.n, "hits_np": hits, "amps_np": amps,
    }


def tested_positions(pairs) -> int:
    """Primer positions that need a test (every position but N), summed over
    the four patterns of each pair (fwd and rev, both strands)."""
    return sum(2 * sum(1 for ch in (q.fwd + q.rev) if ch.upper() != "N") for q in pairs)


def alu_roofline(pairs, bp: int, scan_ms: float, scan_bytes: float) -> dict:
    """Scan kernel against the VALU peak.  Algorithmic work: every tested
    primer position of every pattern is one one-hot literal per packed word
    (32 windows), and one 3-input bitwise instruction folds two more literals
    into a running AND, so testing each position once takes half an
    instruction per position and word."""
    ops = tested_positions(pairs) * bp / 32.0 / 2.0
    achieved = ops / (scan_ms * 1e-3) / 1e12
    hbm = scan_bytes / (scan_ms * 1e-3) / 1e9
    return {"bound": "alu", "achieved": achieved, "peak": ALU_PEAK_TOPS, "unit": "Tops/s",
            "frac": achieved / ALU_PEAK_TOPS, "traffic": None, "kernel": "ah_scan_kernel",
            "algorithmic_ops": ops, "hbm_achieved_gbs": hbm, "hbm_frac": hbm / HBM_PEAK_GBS}


def gpu_batched(steps: int, warmup: int, n_genomes: int = 2000, n_pairs: int = 64,
                shape=None):
    """Batched form: n_pairs primer pairs in one pass (hipGraph replay of the
    whole scan -> Tm -> pairing sequence) against the same pairs one by one.
    ``shape`` (words per lane, patterns per group) pins the batched kernel's
    shape instead of autotuning it on a 200-genome sample."""
    import numpy as np
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu, plan

    dev = torch.device("cuda:0")
    p = plan.batched(n_genomes, n_pairs=n_pairs)
    pairs = p.pairs
    ascii, off = gpu.fill_cuda(p, dev)
    coll, _ = path.pack(ascii, off, p.lengths)
    torch.cuda.synchronize()
    del ascii
    torch.cuda.empty_cache()
    bp = coll.total_bp
    buf = path.alloc(coll, pairs, 1 << 25, 1 << 24, dev)
    sample = min(200, coll.n)
    tune_s = 0.0
    if shape is not None:
        L.ah_set_scan_tuning(pairs, shape)
    t0 = time.perf_counter()
    L.ah_scan_prepare(pairs)
    prep_s = time.perf_counter() - t0
    print(f"batched: {len(pairs)} pairs compiled in {prep_s:.1f} s", file=sys.stderr, flush=True)
    if shape is None:
        os.environ["AH_VERBOSE"] = "1"  # the autotuner reports each candidate on stderr
        t0 = time.perf_counter()
        shape, tune_ms = L.ah_autotune_scan(path.subset_view(coll, sample), L.primer_pairs(pairs),
                                            buf.hits, buf.hit_cap, buf.hit_res, buf.scan_work,
                                            repeats=2)
        tune_s = time.perf_counter() - t0
        os.environ.pop("AH_VERBOSE", None)
        print(f"batched: autotuned in {tune_s:.1f} s: {shape}", file=sys.stderr, flush=True)
    shape = L.ah_get_scan_tuning(pairs)
    for _ in range(max(1, warmup)):
        path.run(coll, pairs, buf)
    torch.cuda.synchronize()
    rh, ra = path.result(buf.hit_res), path.result(buf.amp_res)
    assert rh["status"] == 0 and ra["status"] == 0, (rh, ra)
    L.ah_profile_reset()
    L.ah_profile_enable(True)
    path.run(coll, pairs, buf)
    torch.cuda.synchronize()
    L.ah_profile_enable(False)
    kern = {k: L.ah_profile_query(k)[1] for k in ("scan", "sort", "tm", "pair")}
    graph = path.capture(coll, pairs, buf)
    graph.replay()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        graph.replay()
    torch.cuda.synchronize()
    ms_batched = (time.perf_counter() - t0) * 1e3 / steps
    assert path.result(buf.hit_res)["count"] == rh["count"]
    print(f"batched: {ms_batched:.2f} ms per step; the pairs one by one next", file=sys.stderr,
          flush=True)
    # the same pairs one by one (each its own specialised kernel, prepared
    # concurrently beforehand)
    t0 = time.perf_counter()
    L.prepare_many([[q] for q in pairs])
    prep_seq_s = time.perf_counter() - t0
    print(f"batched: {len(pairs)} single-pair kernels compiled in {prep_seq_s:.1f} s",
          file=sys.stderr, flush=True)
    widest = max(pairs, key=lambda q: L.ah_scan_workspace_bytes(coll.view(), [q], 1 << 25))
    one = path.alloc(coll, [widest], 1 << 25, 1 << 24, dev)
    for q in pairs:
        path.run(coll, [q], one)
    torch.cuda.synchronize()
    seq_steps = max(1, steps // 4)
    t0 = time.perf_counter()
    for _ in range(seq_steps):
        for q in pairs:
            path.run(coll, [q], one)
    torch.cuda.synchronize()
    ms_seq = (time.perf_counter() - t0) * 1e3 / seq_steps
    scan_bytes = SCAN_BYTES_PER_BP * bp
    return {
        "bp": bp, "genomes": coll.n, "pairs": len(pairs),
        "ms_per_step": ms_batched, "value": len(pairs) * bp / (ms_batched * 1e-3) / 1e9,
        "distinct_gbps": bp / (ms_batched * 1e-3) / 1e9,
        "sequential": {"ms_per_step": ms_seq,
                       "per_pair_gbps": len(pairs) * bp / (ms_seq * 1e-3) / 1e9},
        "speedup_vs_sequential": ms_seq / ms_batched,
        "hits": rh["count"], "amplicons": ra["count"], "kernel_ms": kern,
        "tuning": {"words_per_lane": shape[0], "patterns_per_group": shape[1],
                   "autotuned": tune_s > 0, "sample_genomes": sample if tune_s > 0 else 0,
                   "autotune_s": tune_s, "compile_s": prep_s,
                   "sequential_compile_s": prep_seq_s,
                   "sequential_words_per_lane": sorted({L.ah_get_scan_tuning([q])[0]
                                                        for q in pairs})},
        "roofline": alu_roofline(pairs, bp, kern["scan"], scan_bytes),
    }


def gpu_decoy(steps: int, warmup: int):
    """Decoy estimate (the analysis on the genomes reversed) in the same pass
    as the real pair: [pair, decoy of pair] in one call, against the pair
    alone and against two separate passes."""
    import dataclasses

    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu

    p, desc = workload("collection")
    dev = torch.device("cuda:0")
    ascii, off = gpu.fill_cuda(p, dev)
    coll, _ = path.pack(ascii, off, p.lengths)
    torch.cuda.synchronize()
    del ascii
    torch.cuda.empty_cache()
    pr = p.pairs[0]
    dec = dataclasses.replace(pr, decoy=True)
    bp = coll.total_bp

    def timed(pairs):
        buf = path.alloc(coll, pairs, 1 << 22, 1 << 22, dev)
        for _ in range(max(1, warmup)):
            path.run(coll, pairs, buf)
        torch.cuda.synchronize()
        L.ah_profile_reset()
        L.ah_profile_enable(True)
        t0 = time.perf_counter()
        for _ in range(steps):
            path.run(coll, pairs, buf)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / steps
        L.ah_profile_enable(False)
        kern = {k: L.ah_profile_query(k)[1] / max(L.ah_profile_query(k)[0], 1)
                for k in ("scan", "verify", "sort", "tm", "pair")}
        rh, ra = path.result(buf.hit_res), path.result(buf.amp_res)
        assert rh["status"] == 0 and ra["status"] == 0, (rh, ra)
        return ms, kern, path.hits_numpy(buf), path.amps_numpy(buf)

    ms_real, k_real, h_real, a_real = timed([pr])
    ms_dec, k_dec, h_dec, a_dec = timed([dec])
    ms_both, k_both, h_both, a_both = timed([pr, dec])
    n_real = int((a_both["pair"] == 0).sum())
    n_dec = int((a_both["pair"] == 1).sum())
    assert n_real == a_real.size and n_dec == a_dec.size
    # the long-amplicon pair of the streaming workload (192 + 768 oligos, k 3)
    # on the same genomes: random binding is common enough for decoy amplicons
    from synth import plan as splan

    lp = splan.stream(10).pairs[0]
    ms_l, _, _, a_l = timed([lp])
    ms_lb, _, h_lb, a_lb = timed([lp, dataclasses.replace(lp, decoy=True)])
    long_pair = {"fwd": lp.fwd, "rev": lp.rev, "k": lp.k, "window": [lp.min_len, lp.max_len],
                 "real_only_ms": ms_l, "one_pass_ms": ms_lb, "time_vs_real_only": ms_lb / ms_l,
                 "amplicons": {"real": int((a_lb["pair"] == 0).sum()),
                               "decoy": int((a_lb["pair"] == 1).sum())},
                 "sites": {"real": int((h_lb["pair"] == 0).sum()),
                           "decoy": int((h_lb["pair"] == 1).sum())}}
    long_pair["decoy_ratio"] = long_pair["amplicons"]["decoy"] / max(long_pair["amplicons"]["real"], 1)
    assert long_pair["amplicons"]["real"] == a_l.size
    return {
        "desc": desc.replace("collection:", "decoy: collection") +
        "; the pair and its decoy (every genome reversed) in one pass",
        "bp": bp, "genomes": coll.n, "value": bp / (ms_both * 1e-3) / 1e9, "ms_per_step": ms_both,
        "real_only": {"ms_per_step": ms_real, "kernel_ms": k_real},
        "two_passes_ms": ms_real + ms_dec,
        "one_pass": {"ms_per_step": ms_both, "kernel_ms": k_both},
        "time_vs_real_only": ms_both / ms_real,
        "amplicons": {"real": n_real, "decoy": n_dec},
        "sites": {"real": int((h_both["pair"] == 0).sum()), "decoy": int((h_both["pair"] == 1).sum())},
        "decoy_ratio": n_dec / max(n_real, 1),
        "long_amplicon_pair": long_pair,
        "roofline_scan": {"bound": "hbm", "achieved": SCAN_BYTES_PER_BP * bp /
                          (k_both["scan"] * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                          "frac": SCAN_BYTES_PER_BP * bp / (k_both["scan"] * 1e-3) / 1e9 /
                          HBM_PEAK_GBS, "traffic": None, "kernel": "ah_scan_kernel"},
    }


def gpu_fasta(steps: int, warmup: int):
    """FASTA records, sequence hashes and amplitypes of the amplicons of one
    query (after scan, Tm and pairing), for the V4-like pair and the
    long-amplicon pair on the 1000-genome collection."""
    import numpy as np
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu
    from synth import plan as splan

    p, desc = workload("collection")
    dev = torch.device("cuda:0")
    ascii, off = gpu.fill_cuda(p, dev)
    coll, _ = path.pack(ascii, off, p.lengths)
    torch.cuda.synchronize()
    del ascii
    torch.cuda.empty_cache()
    out = {}
    for name, pr in (("v4_like", p.pairs[0]), ("long_amplicon", splan.stream(10).pairs[0])):
        buf = path.alloc(coll, [pr], 1 << 22, 1 << 22, dev)
        path.run(coll, [pr], buf)
        torch.cuda.synchronize()
        n_amp = path.result(buf.amp_res)["count"]
        fb = path.fasta_alloc(coll, 1, buf.amp_cap, 16, dev)
        path.fasta(coll, 1, buf, fb)  # sizes the text
        torch.cuda.synchronize()
        need = path.result(fb.text_res)["required"]
        fb = path.fasta_alloc(coll, 1, buf.amp_cap, need, dev)
        for _ in range(max(1, warmup)):
            path.fasta(coll, 1, buf, fb)
        torch.cuda.synchronize()
        L.ah_profile_reset()
        L.ah_profile_enable(True)
        t0 = time.perf_counter()
        for _ in range(steps):
            path.fasta(coll, 1, buf, fb)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / steps
        L.ah_profile_enable(False)
        nk, kms = L.ah_profile_query("fasta")
        assert path.result(fb.text_res)["status"] == 0
        amps = path.amps_numpy(buf)
        bases = int((amps["end"].astype(np.int64) - amps["start"]).sum()) if amps.size else 0
        kernel_ms = kms / max(nk, 1)
        # bytes: the text written, the amplicon records read (24 B each) and
        # the packed words of the bases decoded (0.25 B per base)
        algo = need + 24 * n_amp + bases / 4
        out[name] = {"amplicons": n_amp, "text_bytes": need, "bases": bases, "ms": ms,
                     "kernel_ms": kernel_ms, "text_gbps": need / (kernel_ms * 1e-3) / 1e9,
                     "hbm_frac": algo / (kernel_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                     "distinct_amplitypes": int(np.unique(
                         fb.amplitype.cpu().numpy().view(np.uint64)[
                             fb.amplitype_n.cpu().numpy() > 0]).size)}
        del buf, fb
        torch.cuda.empty_cache()
    return {"desc": desc, "bp": coll.total_bp, "genomes": coll.n, **out}


def gpu_ingest(n_genomes: int = 250, width: int = 80):
    """Real-FASTA ingest: the first genomes of the collection written as FASTA
    (lines of `width` bases), then read on the host (16 threads), copied to
    the device through pinned memory and packed there."""
    import numpy as np
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu

    p, desc = workload("collection")
    p = p.subset(list(range(n_genomes)))
    dev = torch.device("cuda:0")
    ascii, off = gpu.fill_cuda(p, dev)
    raw = ascii.cpu().numpy()
    offs = off.cpu().numpy().astype(np.int64)
    parts = []
    for g in range(p.n):
        s = raw[offs[g]:offs[g + 1]]
        rows = -(-s.size // width)
        buf = np.full((rows, width + 1), ord("\n"), dtype=np.uint8)
        padded = np.zeros(rows * width, dtype=np.uint8)
        padded[: s.size] = s
        buf[:, :width] = padded.reshape(rows, width)
        body = buf.reshape(-1)
        keep = np.ones(body.size, bool)  # drop the padding of the last row
        pad = rows * width - s.size
        if pad:
            keep[body.size - 1 - pad: body.size - 1] = False
        parts.append(f">g{g} synthetic\n".encode() + body[keep].tobytes())
    text = b"".join(parts)
    del raw, ascii
    torch.cuda.empty_cache()
    L.fasta_read(b">warm\nACGT\n", pinned=True)  # the pinned allocator's first call
    t0 = time.perf_counter()
    host, soff, names = L.fasta_read(text, pinned=True)
    t_read = time.perf_counter() - t0
    assert len(names) == p.n and int(soff[-1]) == p.total_bp
    t_pin = 0.0  # read straight into pinned memory
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    d = host.to(dev, non_blocking=True)
    torch.cuda.synchronize()
    t_h2d = time.perf_counter() - t0
    d_off = torch.from_numpy(soff).to(dev)
    # the library's first kernel launch in the process loads its code object
    path.pack(d[:64], torch.tensor([0, 64], dtype=torch.int64, device=dev), np.array([64]),
              with_nmask=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    coll, _ = path.pack(d, d_off, np.diff(soff), with_nmask=True)
    torch.cuda.synchronize()
    t_pack = time.perf_counter() - t0
    t_all = t_read + t_pin + t_h2d + t_pack
    gb = len(text) / 1e9
    return {"desc": f"{p.n} genomes of the collection as FASTA ({width}-base lines), "
                    f"{len(text) / 1e9:.2f} GB of text", "text_bytes": len(text),
            "bases": p.total_bp, "read_s": t_read, "pin_copy_s": t_pin, "h2d_s": t_h2d,
            "pack_s": t_pack, "total_s": t_all, "text_gbps": gb / t_all,
            "read_gbps": gb / t_read, "h2d_gbps": p.total_bp / 1e9 / t_h2d,
            "pack_gbps": p.total_bp / 1e9 / t_pack, "threads": min(16, os.cpu_count() or 1)}


PCIE_PEAK_GBS = 64.0  # PCIe 5.0 x16, one direction, nominal


def gpu_stream(steps: int, warmup: int, n_genomes: int = 10000, chunk_words: int = 1 << 26,
               n_slots: int = 3, n_copy: int = 2):
    """Streaming form: the packed collection sits in pinned host memory and is
    copied to the GPU in chunks on ``n_copy`` copy streams while earlier
    chunks are scanned, scored and paired (one ah_stream_query per step)."""
    import numpy as np
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu, plan

    dev = torch.device("cuda:0")
    p = plan.stream(n_genomes)
    pr = p.pairs[0]
    t0 = time.perf_counter()
    hg = path.pack_to_host(lambda ids: gpu.fill_cuda(p.subset(ids), dev), p.lengths, dev)
    build_s = time.perf_counter() - t0
    bp = int(p.lengths.sum())
    packed_bytes = 8 * int(hg.word_off[-1])
    print(f"stream: host collection {bp / 1e9:.2f} Gbp, {packed_bytes / 1e9:.2f} GB packed, "
          f"built in {build_s:.1f} s", file=sys.stderr, flush=True)
    hit_cap, amp_cap = 1 << 24, 1 << 22
    buf = path.stream_alloc(hg, [pr], hit_cap, amp_cap, dev, chunk_words, n_slots)
    copies = [torch.cuda.Stream(dev) for _ in range(n_copy)]
    for _ in range(max(1, warmup)):
        path.stream_run(hg, [pr], buf, copy_streams=copies)
    torch.cuda.synchronize()
    rh, ra = path.result(buf.hit_res), path.result(buf.amp_res)
    assert rh["status"] == 0 and ra["status"] == 0, (rh, ra)
    L.ah_profile_reset()
    L.ah_profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(steps):
        path.stream_run(hg, [pr], buf, copy_streams=copies)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    L.ah_profile_enable(False)
    kern = {k: L.ah_profile_query(k)[1] / steps for k in ("scan", "sort", "tm", "pair")}
    hs, as_ = path.hits_numpy(buf), path.amps_numpy(buf)
    # copy-only reference: the same bytes, one chunk-sized pinned copy after another
    staging = torch.empty(min(packed_bytes, chunk_words * 8) // 4, dtype=torch.int32, device=dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    done = 0
    flat = hg.words
    while done < flat.numel():
        n = min(staging.numel(), flat.numel() - done)
        staging[:n].copy_(flat[done: done + n], non_blocking=True)
        done += n
    torch.cuda.synchronize()
    copy_gbs = packed_bytes / (time.perf_counter() - t0) / 1e9
    del staging
    # the same query on the collection resident in HBM, and full-size parity
    coll = path.to_device(hg, dev)
    rbuf = path.alloc(coll, [pr], hit_cap, amp_cap, dev)
    path.run(coll, [pr], rbuf)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        path.run(coll, [pr], rbuf)
    torch.cuda.synchronize()
    ms_res = (time.perf_counter() - t0) * 1e3 / steps
    same = bool(np.array_equal(path.hits_numpy(rbuf), hs) and
                np.array_equal(path.amps_numpy(rbuf), as_))
    gbs = packed_bytes / (ms * 1e-3) / 1e9
    return {
        "bp": bp, "genomes": n_genomes, "ms_per_step": ms, "value": bp / (ms * 1e-3) / 1e9,
        "packed_bytes": packed_bytes, "hits": rh["count"], "amplicons": ra["count"],
        "kernel_ms": kern, "host_build_s": build_s,
        "pair": {"fwd": pr.fwd, "rev": pr.rev, "k": pr.k, "clamp": pr.clamp,
                 "window": [pr.min_len, pr.max_len]},
        "chunk_words": chunk_words, "n_slots": n_slots, "copy_streams": n_copy,
        "copy_only_gbs": copy_gbs,
        "resident": {"ms_per_step": ms_res, "gbps": bp / (ms_res * 1e-3) / 1e9},
        "streamed_equals_resident": same,
        "roofline": {"bound": "pcie", "achieved": gbs, "peak": PCIE_PEAK_GBS, "unit": "GB/s",
                     "frac": gbs / PCIE_PEAK_GBS, "traffic": None,
                     "kernel": "host-to-device copies of the packed chunks",
                     "algorithmic_bytes": packed_bytes,
                     "copy_only_frac": gbs / copy_gbs},
    }


def _serve_pass(srv, p, jobs, mode: str, rate_start_delay: float = 0.05):
    """Run every job through the server.  mode "poisson": submit at the
    jobs' arrival times from a submitter thread; "burst": all at once;
    "serial": one at a time, each after the previous finished.  Returns
    per-job statuses and the makespan (first submission to last completion)."""
    import threading

    out = []
    if mode == "serial":
        t0 = srv.now()
        for _, pid, ids in jobs:
            j = srv.submit(p.pairs[pid], ids)
            st = srv.wait(120.0)
            assert st is not None and st["job"] == j and st["status"] == 0, st
            out.append(st)
            srv.release(j)
        return out, out[-1]["t_done"] - t0
    start = srv.now() + rate_start_delay
    err = []

    def submit_all():
        try:
            for ta, pid, ids in jobs:
                if mode == "poisson":
                    d = start + ta - srv.now()
                    if d > 0:
                        time.sleep(d)
                srv.submit(p.pairs[pid], ids)
        except Exception as e:  # surfaced below
            err.append(e)

    th = threading.Thread(target=submit_all)
    th.start()
    last = time.perf_counter()
    while len(out) < len(jobs):
        st = srv.wait(120.0)  # no job finishing for two minutes: stuck
        if st is None or err:
            break
        assert st["status"] == 0, st
        out.append(st)
        srv.release(st["job"])
        if time.perf_counter() - last > 10.0:
            print(f"serve: {mode} {len(out)}/{len(jobs)} jobs done", file=sys.stderr, flush=True)
            last = time.perf_counter()
    th.join()
    if err:
        raise err[0]
    assert len(out) == len(jobs), "a job did not finish"
    first = min(st["t_submit"] for st in out)
    return out, max(st["t_done"] for st in out) - first


def _lat_summary(sts):
    import numpy as np

    lat = np.array([st["t_done"] - st["t_submit"] for st in sts]) * 1e3
    wait = np.array([st["t_start"] - st["t_submit"] for st in sts]) * 1e3
    return {"p50_ms": float(np.percentile(lat, 50)), "p99_ms": float(np.percentile(lat, 99)),
            "mean_ms": float(lat.mean()), "max_ms": float(lat.max()),
            "queue_p50_ms": float(np.percentile(wait, 50)),
            "queue_p99_ms": float(np.percentile(wait, 99))}


def _pass_summary(sts, span, rate=None) -> dict:
    bases = sum(st["bases"] for st in sts)
    out = {"jobs": len(sts), "makespan_s": span, "jobs_per_s": len(sts) / span,
           "gbps": bases / span / 1e9, "latency": _lat_summary(sts),
           "hits": int(sum(st["hits"] for st in sts)),
           "amplicons": int(sum(st["amplicons"] for st in sts))}
    if rate is not None:
        out["offered_jobs_per_s"] = rate
    return out


def gpu_serve(n_genomes: int = 100000, n_jobs: int = 2000, sat_jobs: int = 240,
              main_frac: float = 0.7, sweep=(0.25, 0.5, 0.9), sweep_jobs: int = 500,
              cold_jobs: int = 200, pool_gb: float = 48.0, host_gb: int = 64, n_lanes: int = 4):
    """Serving form: the 100,000-genome collection resident in HBM; each job
    is one law pair over a log-uniform genome subset.  Protocol: saturation
    = jobs/s of a burst of the first ``sat_jobs`` jobs; then ``n_jobs``
    Poisson arrivals at ``main_frac`` x saturation, a sweep over the other
    fractions (the first ``sweep_jobs`` jobs each), all with every pair's
    kernel compiled beforehand (warm); then ``cold_jobs`` Poisson jobs at the
    main rate with every cached kernel dropped first, so that each new pair is
    compiled on the request path (cold)."""
    import numpy as np
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path
    from synth import gpu, plan

    dev = torch.device("cuda:0")
    p = plan.serving(n_genomes)
    t0 = time.perf_counter()
    coll = path.pack_resident(lambda ids: gpu.fill_cuda(p.subset(ids), dev), p.lengths, dev)
    build_s = time.perf_counter() - t0
    print(f"serve: resident {coll.total_bp / 1e9:.1f} Gbp, "
          f"{coll.words.numel() * 4 / 1e9:.1f} GB packed, built in {build_s:.1f} s",
          file=sys.stderr, flush=True)
    n_all = max(n_jobs, sat_jobs, sweep_jobs if sweep else 0, cold_jobs)
    base = plan.jobs(13306, n_all, 1.0, p.n, len(p.pairs))  # arrivals of a unit-rate process

    def at_rate(jobs, rate):  # the same Poisson process run at `rate` jobs/s
        return [(ta / rate, pid, ids) for ta, pid, ids in jobs]

    warm_ids = sorted({pid for _, pid, _ in
                       base[:max(n_jobs, sat_jobs, sweep_jobs if sweep else 0, 8)]})
    t0 = time.perf_counter()
    L.prepare_many([[p.pairs[i]] for i in warm_ids])
    compile_s = time.perf_counter() - t0
    print(f"serve: {len(warm_ids)} pair kernels compiled in {compile_s:.1f} s", file=sys.stderr,
          flush=True)
    cfg = dict(n_lanes=n_lanes, n_compilers=16, part_bases=1 << 32, max_part_hits=1 << 25,
               capacity_scale=2.0, host_pool_bytes=host_gb << 30)
    out = {"genomes": n_genomes, "total_bp": coll.total_bp, "build_s": build_s,
           "warm_compile_s": compile_s, "warm_distinct_pairs": len(warm_ids), "config": cfg,
           "pool_gb": pool_gb}
    srv = path.Server(coll, int(pool_gb * (1 << 30)), dev, **cfg)
    try:
        _serve_pass(srv, p, base[:8], "burst")  # warm-up: tables, staging buffers
        sts, span = _serve_pass(srv, p, base[:sat_jobs], "burst")
        sat = len(sts) / span
        out["saturation"] = _pass_summary(sts, span)
        print(f"serve: saturation {sat:.1f} jobs/s ({sat_jobs} jobs in a burst)",
              file=sys.stderr, flush=True)
        rate = main_frac * sat
        sts, span = _serve_pass(srv, p, at_rate(base[:n_jobs], rate), "poisson")
        out["main"] = dict(_pass_summary(sts, span, rate), fraction_of_saturation=main_frac)
        print(f"serve: {n_jobs} jobs at {rate:.1f}/s: p50 {out['main']['latency']['p50_ms']:.1f} "
              f"ms, p99 {out['main']['latency']['p99_ms']:.1f} ms", file=sys.stderr, flush=True)
        out["sweep"] = []
        for f in sweep:
            sts, span = _serve_pass(srv, p, at_rate(base[:sweep_jobs], f * sat), "poisson")
            out["sweep"].append(dict(_pass_summary(sts, span, f * sat), fraction_of_saturation=f))
            print(f"serve: sweep {f}: p50 {out['sweep'][-1]['latency']['p50_ms']:.1f} ms, p99 "
                  f"{out['sweep'][-1]['latency']['p99_ms']:.1f} ms", file=sys.stderr, flush=True)
        stats = srv.stats()
    finally:
        srv.close()
    out["server"] = {k: stats[k] for k in ("parts_run", "retries", "pool_bytes", "pool_high_water",
                                           "admission_waits", "lane_busy_s", "host_pool_bytes",
                                           "host_pool_high_water", "host_fallbacks", "gpu_s",
                                           "copy_s")}
    if cold_jobs:
        L.lib().ah_release_caches()  # every pair's kernel is compiled again, on request
        srv = path.Server(coll, int(pool_gb * (1 << 30)), dev, **cfg)
        try:
            rate = main_frac * sat
            sts, span = _serve_pass(srv, p, at_rate(base[:cold_jobs], rate), "poisson")
            out["cold"] = dict(_pass_summary(sts, span, rate), fraction_of_saturation=main_frac,
                               distinct_pairs=len({pid for _, pid, _ in base[:cold_jobs]}),
                               ready_p50_ms=float(np.percentile(
                                   [(st["t_ready"] - st["t_submit"]) * 1e3 for st in sts], 50)))
            print(f"serve: cold {cold_jobs} jobs: p50 {out['cold']['latency']['p50_ms']:.1f} ms, "
                  f"p99 {out['cold']['latency']['p99_ms']:.1f} ms", file=sys.stderr, flush=True)
        finally:
            srv.close()
    m = out["main"]
    out.update(value=m["gbps"], jobs_per_s=m["jobs_per_s"], ms_per_step=m["makespan_s"] * 1e3 / m["jobs"])
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="collection", choices=["collection", "plain"])
    ap.add_argument("--form", default="plain",
                    choices=["plain", "batched", "stream", "serve", "decoy", "fasta", "ingest"],
                    help="plain: one pair per query (the headline); batched: 64 pairs in one "
                         "pass vs one by one; stream: 10,000 genomes copied host -> HBM in "
                         "packed chunks during the query; serve: Poisson jobs over a resident "
                         "100,000-genome collection; decoy: the pair and its decoy estimate "
                         "(genomes reversed) in one pass; fasta: amplicon FASTA records, "
                         "sequence hashes and amplitypes; ingest: FASTA text read, copied and "
                         "packed")
    ap.add_argument("--jobs", type=int, default=2000,
                    help="serve: Poisson jobs at 0.7 x the measured saturation")
    ap.add_argument("--no-forms", action="store_true",
                    help="the headline query only: no batched and serving sub-objects")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-target-mbp", type=float, default=128.0)
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="after the run, launch one elementwise copy kernel of 1 GiB in / 1 GiB "
                         "out (reference for scaling rocprofv3 byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}): sharding the genomes over "
              "GPUs is designed but not implemented.", file=sys.stderr)
        sys.exit(2)
    if args.form == "batched":
        r = gpu_batched(args.steps, args.warmup)
        print(f"batched: {r['value']:.1f} Gbp/s per pair, {r['speedup_vs_sequential']:.2f}x vs "
              f"sequential, kernels {r['kernel_ms']}", file=sys.stderr, flush=True)
        print(json.dumps({
            "metric": METRIC, "value": r["value"], "unit": "Gbp/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": r["ms_per_step"],
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u32",
            "data": "synthetic",
            "config": {"workload": BATCHED_DESC,
                       "form": "batched", "genomes": r["genomes"], "total_bp": r["bp"],
                       "pairs": r["pairs"], "distinct_gbps": r["distinct_gbps"],
                       "sequential": r["sequential"],
                       "speedup_vs_sequential": r["speedup_vs_sequential"], "hits": r["hits"],
                       "amplicons": r["amplicons"], "kernel_ms": r["kernel_ms"],
                       "tuning": r["tuning"]},
            "roofline": r["roofline"], "cpu_baseline": None}))
        return
    if args.form == "ingest":
        r = gpu_ingest()
        print(f"ingest: {r}", file=sys.stderr, flush=True)
        print(json.dumps({
            "metric": "FASTA text GB/s ingested (read, copied to HBM, packed)",
            "value": r["text_gbps"], "unit": "GB/s", "n_gpus": 1, "steps": 1, "warmup": 0,
            "ms_per_step": r["total_s"] * 1e3, "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "u8", "data": "synthetic",
            "config": {"workload": r["desc"], "form": "ingest",
                       **{k: v for k, v in r.items() if k != "desc"}},
            "roofline": {"bound": "pcie", "achieved": r["h2d_gbps"], "peak": PCIE_PEAK_GBS,
                         "unit": "GB/s", "frac": r["h2d_gbps"] / PCIE_PEAK_GBS, "traffic": None,
                         "kernel": "host-to-device copy"},
            "cpu_baseline": None}))
        return
    if args.form == "fasta":
        r = gpu_fasta(args.steps, args.warmup)
        print(f"fasta: v4 {r['v4_like']}; long {r['long_amplicon']}", file=sys.stderr, flush=True)
        lng = r["long_amplicon"]
        print(json.dumps({
            "metric": "amplicon FASTA GB/s written (records, hashes, amplitypes)",
            "value": lng["text_gbps"], "unit": "GB/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": lng["ms"], "higher_is_better": True,
            "scaling": "weak", "vs_baseline": None, "dtype": "u8", "data": "synthetic",
            "config": {"workload": r["desc"] + "; FASTA of the amplicons of one query",
                       "form": "fasta", "genomes": r["genomes"], "total_bp": r["bp"],
                       "v4_like": r["v4_like"], "long_amplicon": lng},
            "roofline": {"bound": "hbm", "achieved": lng["hbm_frac"] * HBM_PEAK_GBS,
                         "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": lng["hbm_frac"],
                         "traffic": None, "kernel": "k_fasta_write"},
            "cpu_baseline": None}))
        return
    if args.form == "decoy":
        r = gpu_decoy(args.steps, args.warmup)
        print(f"decoy: {r['ms_per_step']:.3f} ms per pass with the decoy vs "
              f"{r['real_only']['ms_per_step']:.3f} alone ({r['time_vs_real_only']:.2f}x; two "
              f"passes {r['two_passes_ms']:.3f} ms); amplicons {r['amplicons']}, ratio "
              f"{r['decoy_ratio']:.4f}; long-amplicon pair {r['long_amplicon_pair']}",
              file=sys.stderr, flush=True)
        print(json.dumps({
            "metric": METRIC, "value": r["value"], "unit": "Gbp/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": r["ms_per_step"],
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u32",
            "data": "synthetic",
            "config": {"workload": r["desc"], "form": "decoy", "genomes": r["genomes"],
                       "total_bp": r["bp"], **{k: r[k] for k in (
                           "real_only", "one_pass", "two_passes_ms", "time_vs_real_only",
                           "amplicons", "sites", "decoy_ratio", "long_amplicon_pair")}},
            "roofline": r["roofline_scan"], "cpu_baseline": None}))
        return
    if args.form == "serve":
        r = gpu_serve(n_jobs=args.jobs)
        print(f"serve: {r['value']:.1f} Gbp/s, {r['jobs_per_s']:.1f} jobs/s at "
              f"{r['main']['fraction_of_saturation']} x saturation", file=sys.stderr, flush=True)
        print(json.dumps({
            "metric": METRIC, "value": r["value"], "unit": "Gbp/s", "n_gpus": 1,
            "steps": r["main"]["jobs"], "warmup": 8, "ms_per_step": r["ms_per_step"],
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u32",
            "data": "synthetic",
            "config": {"workload": SERVE_DESC, "form": "serve",
                       **{k: v for k, v in r.items() if k not in ("value", "ms_per_step")}},
            "roofline": None, "cpu_baseline": None}))
        return
    if args.form == "stream":
        r = gpu_stream(args.steps, args.warmup)
        print(f"stream: {r['value']:.1f} Gbp/s incl. PCIe, copies {r['roofline']['achieved']:.1f} "
              f"GB/s (copy only {r['copy_only_gbs']:.1f}), resident {r['resident']['gbps']:.1f} "
              f"Gbp/s, equal {r['streamed_equals_resident']}", file=sys.stderr, flush=True)
        print(json.dumps({
            "metric": METRIC, "value": r["value"], "unit": "Gbp/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": r["ms_per_step"],
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u32",
            "data": "synthetic",
            "config": {"workload": "stream: 10,000 genomes (log-normal lengths, median 4 Mbp, "
                                   "clipped 1-12 Mbp, GC 30-70%), long-amplicon pair (192 + 768 "
                                   "oligos, k 3, window 2000-5500), 2-bit packed collection in "
                                   "pinned host memory copied to HBM during every query",
                       "form": "stream", **{k: r[k] for k in (
                           "genomes", "packed_bytes", "pair", "hits", "amplicons", "kernel_ms",
                           "chunk_words", "n_slots", "copy_streams", "copy_only_gbs", "resident",
                           "streamed_equals_resident", "host_build_s")}, "total_bp": r["bp"]},
            "roofline": r["roofline"], "cpu_baseline": None}))
        return
    cpu = None
    if not args.no_cpu_baseline:
        cpu, cpu_ids, cpu_hits, cpu_amps = cpu_baseline(args.workload, 1000,
                                                        args.cpu_target_mbp * 1e6)
        print(f"cpu baseline: {cpu['value']:.4f} Gbp/s on {cpu['cores']} cores, "
              f"{cpu['single_core']['value']:.4f} on one", file=sys.stderr, flush=True)
    r = gpu_run(args.workload, args.steps, args.warmup)
    agree = None
    if cpu is not None:
        agree = oracle_agreement(r["hits_np"], r["amps_np"], cpu_ids, cpu_hits, cpu_amps)
        print(f"oracle agreement on the baseline's genomes: {agree}", file=sys.stderr, flush=True)
    del r["hits_np"], r["amps_np"]
    forms = {}
    if not args.no_forms and args.workload == "collection":
        import torch

        torch.cuda.empty_cache()
        # batched vs plain: the 64-pair workload in one pass against the same
        # pairs one by one (shape pinned to the autotuner's usual choice:
        # autotuning takes minutes)
        b = gpu_batched(max(3, args.steps // 4), 1, shape=(15, 16))
        forms["batched"] = {
            "workload": BATCHED_DESC, "genomes": b["genomes"], "total_bp": b["bp"],
            "pairs": b["pairs"], "per_pair_gbps": b["value"], "distinct_gbps": b["distinct_gbps"],
            "ms_per_step": b["ms_per_step"], "sequential": b["sequential"],
            "speedup_vs_sequential": b["speedup_vs_sequential"], "hits": b["hits"],
            "amplicons": b["amplicons"], "tuning": b["tuning"],
            "roofline": {k: b["roofline"][k] for k in ("bound", "achieved", "peak", "unit", "frac",
                                                       "hbm_frac")}}
        print(f"batched: {b['value']:.1f} Gbp/s per pair, {b['speedup_vs_sequential']:.2f}x vs "
              f"sequential", file=sys.stderr, flush=True)
        torch.cuda.empty_cache()
        # serving: a short run of the protocol (the full one: --form serve)
        sv = gpu_serve(n_jobs=240, sat_jobs=120, sweep=(), cold_jobs=40, host_gb=64)
        forms["serve"] = {"workload": SERVE_DESC + "; 120-job burst for saturation, 240 Poisson "
                                                   "jobs at 0.7 x saturation (warm), 40 with "
                                                   "every kernel compiled on request (cold)",
                          **{k: sv[k] for k in ("saturation", "main", "cold", "warm_compile_s",
                                                "warm_distinct_pairs", "build_s")}}
        print(f"serve: warm p99 {sv['main']['latency']['p99_ms']:.1f} ms, cold p99 "
              f"{sv['cold']['latency']['p99_ms']:.1f} ms", file=sys.stderr, flush=True)
    g = r["graph_replay"]
    print(f"gpu: {g['gbps']:.1f} Gbp/s, {g['ms_per_step']:.3f} ms/step replayed from a hipGraph "
          f"({r['value']:.1f} Gbp/s, {r['ms_per_step']:.3f} ms launched call by call), kernels "
          f"{r['kernel_ms']}", file=sys.stderr, flush=True)
    line = {
        "metric": METRIC,
        "value": g["gbps"],
        "unit": "Gbp/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": g["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u32",
        "data": "synthetic",
        "config": {
            "workload": r["desc"], "genomes": r["genomes"], "total_bp": r["bp"],
            "pair": r["pair"], "form": "plain", "hits": r["hits"], "amplicons": r["amplicons"],
            "kernel_ms": r["kernel_ms"], "scan_candidates": r["scan_candidates"],
            "launch": "one hipGraph replay per step of the whole path (scan, sort, Tm, pairing), "
                      "captured once; the same K steps launched call by call under 'eager'",
            "eager": {"ms_per_step": r["ms_per_step"], "gbps": r["value"]},
            "ingest_pack": r["pack"], "jit": r["jit"],
            "tm_dtype": "f32 (exact fixed-point stack sums, f64 salt/log terms)",
            "oracle_equal": None if agree is None else agree["oracle_equal"],
            "tm_error": None if agree is None else agree["tm_error"],
            "oracle_check": None if agree is None else {
                k: agree[k] for k in ("genomes", "sites", "amplicons")},
            **forms,
        },
        "roofline": r["roofline"],
        "cpu_baseline": cpu,
    }
    if args.calibrate_copy:
        import torch

        x = torch.ones(1 << 28, dtype=torch.int32, device="cuda:0")
        y = torch.empty_like(x)
        torch.add(x, 0, out=y)
        torch.cuda.synchronize()
        line["config"]["copy_calibration_bytes"] = 2 * x.numel() * 4
    print(json.dumps(line))


if __name__ == "__main__":
    main()
