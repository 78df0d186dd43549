"""The tiles of ah_query's segmented tail, byte for byte against the three
separate calls: many short segments (thousands of genomes, most of them without a
site), segments that fill tiles by themselves, segments longer than a tile's LDS in
either form (four waves where the capacity is above 2^17 sites and more than 32,768
are expected on genomes of the longest's length, else one), no site at all, and
overflows."""
import numpy as np
import pytest

from gpu_util import say
from synth import plan
from test_gpu_query import _both, dev  # noqa: F401

pytestmark = pytest.mark.gpu

NARROW, WIDE = 1 << 17, (1 << 17) + 1
SHORT = plan.PairSpec("ACGTACGTAC", "GGCCAATTGG", k=3, clamp=0, min_len=20, max_len=3000)


@pytest.mark.parametrize("cap", [NARROW, WIDE])
@pytest.mark.parametrize("n,pairs", [(4096, 1), (4097, 1), (5000, 3)])
def test_many_short_segments(dev, n, pairs, cap):  # noqa: F811
    p = plan.tiny(9400 + n, n_genomes=n, len_lo=30, len_hi=900, n_copies=(0, 1), span=100,
                  pair=plan.PairSpec("ACGTRYACGTAC", "TTGCANNGCATT", k=2, clamp=0, min_len=20, max_len=400))
    ps = [p.pairs[0]] + plan.law_pairs(9401, pairs - 1) + ([SHORT] if cap == WIDE else [])
    sep, fus = _both(p, ps, dev, hit_cap=cap, amp_cap=1 << 16, filter_tm=pairs == 3, min_tm=25.0)
    say("short segments", n, pairs, cap, sep[0]["count"], sep[1]["count"])
    assert sep[0]["status"] == 0 and sep[0]["count"] > 500 and fus == sep


@pytest.mark.parametrize("cap", [NARROW, WIDE])
@pytest.mark.parametrize("lengths", [[3000] * 200 + [60_000], [90_000, 120_000, 31, 60_000] + [10] * 40,
                                     [700_000, 5000] + [20] * 10])
def test_long_segments(dev, monkeypatch, lengths, cap):  # noqa: F811
    """From a few sites a segment to more than 4,096 (forced: left to itself the
    query expects segments this long and takes the radix tail)."""
    monkeypatch.setenv("AH_QUERY_SEGMENTED", "1")
    p = plan.tiny(9410 + len(lengths), n_genomes=len(lengths), len_lo=30, len_hi=60, pair=SHORT, n_copies=(0, 0))
    p = p.with_lengths(lengths)
    sep, fus = _both(p, [SHORT], dev, hit_cap=cap, amp_cap=1 << 21)
    per = np.bincount(np.frombuffer(sep[2], dtype=np.uint32).reshape(-1, 4)[:, 0], minlength=p.n)
    say("long segments", cap, "most", int(per.max()), "amplicons", sep[1]["count"])
    assert sep[0]["status"] == 0 and sep[1]["status"] == 0 and fus == sep
    assert max(lengths) < 700_000 or per.max() > 4096


@pytest.mark.parametrize("cap", [64, NARROW, WIDE])
def test_no_site_and_overflow(dev, monkeypatch, cap):  # noqa: F811
    monkeypatch.setenv("AH_QUERY_SEGMENTED", "1")
    none = plan.PairSpec("ACGTTGCAGCTAGGCTTACGATCC", "GGATTCCAGACCTTGACGTTAGCA", k=0, clamp=0, min_len=60, max_len=300)
    p = plan.tiny(9420, n_genomes=5, len_lo=2000, len_hi=9000, pair=none, n_copies=(0, 0))
    sep, fus = _both(p, [none], dev, hit_cap=cap, amp_cap=64)
    assert sep[0]["count"] == 0 and sep[0]["status"] == 0 and fus == sep
    if cap > 64:  # more sites than even the large capacity holds
        p = plan.tiny(9421, n_genomes=4, len_lo=2_000_000, len_hi=4_000_000, n_copies=(0, 0),
                      pair=plan.PairSpec("ACGTN", "GGCCN", k=1, clamp=0, min_len=20, max_len=40))
        sep, fus = _both(p, p.pairs, dev, hit_cap=cap, amp_cap=64)
        assert sep[0]["status"] == -4 and fus[0] == sep[0]
        assert (fus[1]["status"], fus[1]["count"], fus[1]["required"]) == (-4, 0, 0)
