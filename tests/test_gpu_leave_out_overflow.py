"""Filters that leave positions of a primer out, on sequence that repeats the
positions they keep: their candidates overfill the scan's slices many times over
while the sites are few.  The scan fills those slices again with the records of
sites and reports every site, as it does where the filter tests every position;
only records of sites that do not fit make an overflow, whose bound then suffices.
One and several groups of patterns, wave and tile mode, the count in the
filter and after it, with and without non-ACGT bases, against the oracle."""
import re

import numpy as np
import pytest

from gpu_util import say
from oracle import scan as oscan
from synth import plan

pytestmark = pytest.mark.gpu

LONG = "ACGTTGACACACACACACACACAC"  # kept of it: A..........C..AC.CACACAC
SETS = {
    "wave": [("CATGACACACACACACACAC", "GGATCCAAGTTCGACGTAAC", 0)],  # .....C..A..CACACACAC
    "tile": [(LONG, "GGATCCAAGTTCGACGTAACGTTGCA", 0)],
    "wave-groups": [("ACGTTGACACACACACACAC"[i:], "GGATCCAAGTTCGACGTAA", i % 2) for i in range(5)],
    "tile-groups": [(LONG[i:] + "ACGTACTTGCA"[:i], "GGATCCAAGTTCGACGTAACGTTGCA", i % 2) for i in range(5)],
}


@pytest.fixture(scope="module")
def dev():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return torch.device("cuda:0")


def _pairs(name):
    from paper_2509_13300_amd import _lib as L

    pairs = [plan.PairSpec(f, r, k=k, clamp=0, min_len=40, max_len=400) for f, r, k in SETS[name]]
    macro = dict(re.findall(r"#define AH_(\w+) (\d+)\n", L.ah_scan_program_source(pairs)))
    assert macro["REFILL"] == "1" and macro["WAVE"] == str(int(name.startswith("wave")))
    return pairs


def _revcomp(s):
    return s[::-1].translate(bytes.maketrans(b"ACGT", b"TGCA"))


def _collection(dev, seqs, mask):
    import torch

    from paper_2509_13300_amd import path

    lengths = np.array([s.size for s in seqs])
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    ascii = torch.from_numpy(np.concatenate(seqs)).to(dev)
    coll, _ = path.pack(ascii, torch.from_numpy(off).to(dev), lengths, with_nmask=mask)
    return coll


def _repeats(pairs, mask, n=30, length=180_000):
    """Genomes with tracts of (AC)n and its reverse complement, and planted sites,
    some inside the tracts."""
    rng = np.random.default_rng(len(pairs) + 2 * mask)
    seqs = []
    for g in range(n):
        s = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, length + 37 * g)].copy()
        tracts = []
        for unit in (b"AC", b"GT", b"CA"):
            at, m = int(rng.integers(0, length - 40_000)), int(rng.integers(500, 40_000))
            s[at: at + m] = np.frombuffer(unit * (m // 2 + 1), np.uint8)[:m]
            tracts.append(at + int(rng.integers(0, max(1, m - 60))))
        for at in tracts + [int(x) for x in rng.integers(0, length - 500, 3)]:
            p = pairs[int(rng.integers(len(pairs)))]
            f, r = p.fwd.encode(), _revcomp(p.rev.encode())
            span = int(rng.integers(80, 380))
            s[at: at + len(f)] = np.frombuffer(f, np.uint8)
            s[at + span: at + span + len(r)] = np.frombuffer(r, np.uint8)
        if mask:
            for at in rng.integers(0, length - 100, 20):
                s[at: at + int(rng.integers(1, 100))] = ord("N")
        seqs.append(s)
    return seqs


def _run(coll, pairs, cap, fused, dev):
    import torch

    from paper_2509_13300_amd import path

    buf = path.alloc(coll, 1, cap, 1 << 18, dev)  # the minimum list
    path.run(coll, pairs, buf, fused=fused)
    torch.cuda.synchronize()
    return buf


@pytest.mark.parametrize("mask", [False, True])
@pytest.mark.parametrize("name", list(SETS))
def test_repeats_do_not_overflow(dev, name, mask):
    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path

    pairs = _pairs(name)
    seqs = _repeats(pairs, mask)
    coll = _collection(dev, seqs, mask)
    print(name, mask, flush=True)
    fus, sep = _run(coll, pairs, 4096, True, dev), _run(coll, pairs, 4096, False, dev)
    got = path.hits_numpy(fus)
    stats = L.ah_scan_candidate_stats(fus.scan_work, coll.n, fus.hit_cap)
    say("repeats", name, mask, path.result(fus.hit_res), stats)
    for buf in (fus, sep):
        assert path.result(buf.hit_res)["status"] == 0 and path.result(buf.amp_res)["status"] == 0
    assert stats["full_slices"] == 0
    assert path.hits_numpy(sep).tobytes() == got.tobytes()
    assert path.amps_numpy(sep).tobytes() == path.amps_numpy(fus).tobytes()
    for q, pr in enumerate(pairs):
        want = oscan.scan_collection([s.tobytes() for s in seqs], [pr])
        mine = got[got["pair"] == q]
        assert mine.size == want.size > 0
        for f in ("genome", "pos", "mm"):
            assert np.array_equal(mine[f], want[f]), (q, f)
        assert np.array_equal(mine["strand_primer"] >> 1, want["strand"])
        assert np.array_equal(mine["strand_primer"] & 1, want["primer"])


@pytest.mark.parametrize("name", list(SETS))
def test_more_sites_than_the_slices_hold(dev, name, monkeypatch):
    """A genome that repeats a primer: the records of its sites alone overfill the
    slices.  An overflow with a bound, and a call with that capacity gives what
    the filter that tests every position (none left out) gives."""
    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path

    pairs = _pairs(name)
    unit = np.frombuffer(pairs[0].fwd.encode() + b"ACACACGTTGA", np.uint8)
    rng = np.random.default_rng(9)
    seqs = [np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, 150_000)].copy() for _ in range(60)]
    for s in seqs[7:57:5]:
        s[1000: 1000 + 4000 * unit.size] = np.tile(unit, 4000)
    coll = _collection(dev, seqs, False)
    print(name, flush=True)
    small = _run(coll, pairs, 1 << 16, True, dev)
    r = path.result(small.hit_res)
    assert L.ah_scan_candidate_stats(small.scan_work, coll.n, small.hit_cap)["full_slices"] > 0
    again = _run(coll, pairs, r["required"], True, dev)
    full = path.hits_numpy(again)
    say("sites overfill", name, r, full.size)
    assert r["status"] == -4 and r["required"] >= full.size >= 40_000
    assert path.result(again.hit_res)["status"] == 0
    monkeypatch.setenv("AH_SCAN_PREFILTER", "0")
    exact = _run(coll, pairs, r["required"], True, dev)
    assert path.result(exact.hit_res)["status"] == 0
    assert path.hits_numpy(exact).tobytes() == full.tobytes()
