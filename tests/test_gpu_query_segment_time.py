"""ah_query's tail over segments of tens of sites: a workgroup a segment, whatever
the segments' length, as far as there are workgroups.  Tiles that held two segments
where one was meant made a query over 30 segments of 100 sites take 1.53 times
one over segments of 50 (93 and 61 us); a workgroup each takes 1.22 times (73 and
60).  And one long segment among thousands, which its workgroup sorts in global
memory: 8 times the radix tail's time by one wave (1,109 and 138 us), 2.8-3.1 times by four
(399-433 and 138-143)."""
import time

import numpy as np
import pytest

from gpu_util import random_rate, say
from synth import gpu, plan

pytestmark = pytest.mark.gpu


def test_segments_of_a_hundred_sites_have_a_workgroup_each():
    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    pair = plan.PairSpec("ACGTRYACGTACAG", "TTGCANNGCATTGC", k=2, clamp=0, min_len=20, max_len=400)
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=dev)
    graphs = []
    for mean in (50, 100):
        length = int(mean / random_rate(pair))
        ascii = letters[torch.randint(0, 4, (30 * length,), device=dev, generator=g)]
        off = torch.arange(31, dtype=torch.int64, device=dev) * length
        coll, _ = path.pack(ascii, off, np.full(30, length))
        buf = path.alloc(coll, [pair], 1 << 17, 1 << 17, dev)
        path.run(coll, [pair], buf)
        torch.cuda.synchronize()
        r = path.result(buf.hit_res)
        assert r["status"] == 0 and r["count"] > 25 * mean
        graphs.append((path.capture(coll, [pair], buf), buf, coll))
    best = [1e9, 1e9]
    for _ in range(20):
        for i, (graph, _, _) in enumerate(graphs):
            graph.replay()
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                graph.replay()
            torch.cuda.synchronize()
            best[i] = min(best[i], (time.perf_counter() - t) / 20 * 1e6)
    say("segments of 50 and 100 sites: us a query", best)
    assert best[1] <= 1.38 * best[0]


def test_one_long_segment_among_thousands(monkeypatch):
    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    unit = b"ACGTTGCAAGCTTCGA"
    rev = (unit[8:] + unit[:8])[::-1].translate(bytes.maketrans(b"ACGT", b"TGCA")).decode()
    pair = plan.PairSpec(unit.decode(), rev, k=0, clamp=0, min_len=24, max_len=40)
    g = torch.Generator(device=dev)
    g.manual_seed(4)
    lengths = np.full(5000, 3000)
    lengths[2500] = 33_000
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=dev)
    ascii = letters[torch.randint(0, 4, (int(off[-1]),), device=dev, generator=g)]
    at = int(off[2500])
    ascii[at: at + 32_000] = torch.tensor(list(unit), dtype=torch.uint8, device=dev).repeat(2000)
    coll, _ = path.pack(ascii, torch.from_numpy(off).to(dev), lengths)
    got, best = [], []
    for segmented in (None, "0"):
        if segmented:
            monkeypatch.setenv("AH_QUERY_SEGMENTED", segmented)
        buf = path.alloc(coll, [pair], 1 << 17, 1 << 17, dev)
        buf.scan_work = torch.empty(buf.scan_work.numel() + (256 << 20), dtype=torch.uint8, device=dev)
        path.run(coll, [pair], buf)
        torch.cuda.synchronize()
        assert path.result(buf.hit_res)["status"] == 0 and path.result(buf.hit_res)["count"] >= 3900
        assert path.result(buf.amp_res)["status"] == 0 and path.result(buf.amp_res)["count"] >= 1900
        got.append((path.hits_numpy(buf).tobytes(), path.amps_numpy(buf).tobytes()))
        graph = path.capture(coll, [pair], buf)
        us = []
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            graph.replay()
            torch.cuda.synchronize()
            us.append((time.perf_counter() - t) * 1e6)
        best.append(min(us))
    say("one long segment: us a query, and by the radix tail", best)
    assert got[0] == got[1]
    assert best[0] <= 4 * best[1]


def test_few_sites_are_spread_over_the_workgroups(monkeypatch):
    """Two pairs at k = 2 and 3 and their decoys on 185 contigs, 1,300 sites of which many
    have some dozens of pairings: in tiles of 32 sites and more the query took
    0.75 times its time with the radix tail (110 and 147 us), and takes 0.53 times
    it in tiles of two."""
    import dataclasses

    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    pairs = [plan.PairSpec("CCACTTKCAGACARAC", "WNAATKCAWCKGNNTATCAAT", k=3, clamp=0, min_len=2184, max_len=3805),
             plan.PairSpec("CGACCTTWGTACATGCTCCGCGTGYGTRW", "NTGGYTCATNTAATCGAAAACCGKCT", k=2, clamp=0,
                           min_len=2184, max_len=3805)]
    pairs += [dataclasses.replace(p, decoy=True) for p in pairs]
    p = plan.tiny(9810, n_genomes=185, len_lo=15_000, len_hi=100_000, pair=pairs[0], n_copies=(1, 1), span=3000)
    ascii, off = gpu.fill_cuda(p, dev)
    coll, _ = path.pack(ascii, off, p.lengths)
    best = []
    for segmented in (None, "0"):
        if segmented:
            monkeypatch.setenv("AH_QUERY_SEGMENTED", segmented)
        buf = path.alloc(coll, pairs, 8000, 6000, dev)
        path.run(coll, pairs, buf)
        torch.cuda.synchronize()
        r = path.result(buf.hit_res)
        assert r["status"] == 0 and 500 < r["count"] < 4000
        graph = path.capture(coll, pairs, buf)
        us = []
        for _ in range(40):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(10):
                graph.replay()
            torch.cuda.synchronize()
            us.append((time.perf_counter() - t) / 10 * 1e6)
        best.append(min(us))
    say("few sites: us a query, and by the radix tail", best, r["count"])
    assert best[0] <= 0.64 * best[1]


def test_a_chromosome_full_of_a_repeat_among_thousands(monkeypatch):
    """Where there are more than 4,096 segments, a genome longer than 16.8 Mbp takes the query
    to the radix tail: one family of repeats gives it more sites than a workgroup
    should sort (16,000 here: 1.45 ms a query by segments, 0.25 on the radix tail)."""
    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    unit = b"ACGTTGCAAGCTTCGA"
    rev = (unit[8:] + unit[:8])[::-1].translate(bytes.maketrans(b"ACGT", b"TGCA")).decode()
    pair = plan.PairSpec(unit.decode(), rev, k=0, clamp=0, min_len=24, max_len=40)
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    lengths = np.full(5000, 3000)
    lengths[2500] = (1 << 24) + 1
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=dev)
    ascii = letters[torch.randint(0, 4, (int(off[-1]),), device=dev, generator=g)]
    for i in range(8):  # in eight places of 1,000 units
        at = int(off[2500]) + 2_000_000 * i
        ascii[at: at + 16_000] = torch.tensor(list(unit), dtype=torch.uint8, device=dev).repeat(1000)
    coll, _ = path.pack(ascii, torch.from_numpy(off).to(dev), lengths)
    got, best = [], []
    for segmented in (None, "0"):
        if segmented:
            monkeypatch.setenv("AH_QUERY_SEGMENTED", segmented)
        buf = path.alloc(coll, [pair], 1 << 17, 1 << 17, dev)
        buf.scan_work = torch.empty(buf.scan_work.numel() + (256 << 20), dtype=torch.uint8, device=dev)
        path.run(coll, [pair], buf)
        torch.cuda.synchronize()
        assert path.result(buf.hit_res)["status"] == 0 and path.result(buf.hit_res)["count"] >= 15_900
        assert path.result(buf.amp_res)["status"] == 0 and path.result(buf.amp_res)["count"] >= 7900
        got.append((path.hits_numpy(buf).tobytes(), path.amps_numpy(buf).tobytes()))
        graph = path.capture(coll, [pair], buf)
        us = []
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            graph.replay()
            torch.cuda.synchronize()
            us.append((time.perf_counter() - t) * 1e6)
        best.append(min(us))
    say("a repeat in a chromosome: us a query, and by the radix tail", best)
    assert got[0] == got[1]
    assert best[0] <= 1.5 * best[1]


def test_fewer_tiles_of_four_waves_among_many_segments(monkeypatch):
    """1,700 sites on 5,000 contigs: in a thousand tiles the query took 0.85 times its time
    with the radix tail (80.5 and 94.5 us), and takes 0.77 times it in 512 (72 and 93)."""
    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    pair = plan.PairSpec("ACGTRYACGTACAG", "TTGCANNGCATTGC", k=2, clamp=0, min_len=20, max_len=400)
    n = 5000
    length = int(1700 / n / random_rate(pair))
    g = torch.Generator(device=dev)
    g.manual_seed(9)
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=dev)
    ascii = letters[torch.randint(0, 4, (n * length,), device=dev, generator=g)]
    coll, _ = path.pack(ascii, torch.arange(n + 1, dtype=torch.int64, device=dev) * length, np.full(n, length))
    best = []
    for segmented in (None, "0"):
        if segmented:
            monkeypatch.setenv("AH_QUERY_SEGMENTED", segmented)
        buf = path.alloc(coll, [pair], 8000, 6000, dev)
        path.run(coll, [pair], buf)
        torch.cuda.synchronize()
        r = path.result(buf.hit_res)
        assert r["status"] == 0 and 1500 < r["count"] < 1900
        graph = path.capture(coll, [pair], buf)
        us = []
        for _ in range(40):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(10):
                graph.replay()
            torch.cuda.synchronize()
            us.append((time.perf_counter() - t) / 10 * 1e6)
        best.append(min(us))
    say("1,700 sites on 5,000 contigs: us a query, and by the radix tail", best, r["count"])
    assert best[0] <= 0.81 * best[1]
