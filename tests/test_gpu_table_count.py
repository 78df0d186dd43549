"""Programs of more than one pair count their candidates from a table of the
patterns: the shortest and longest primers, clamps up to the whole primer, every
IUPAC code, many mismatches, masked genomes, in wave and in tile mode, against the
oracle's scan (sites, strands and mismatches exactly)."""
import numpy as np
import pytest

from gpu_util import say
from oracle import scan as oscan
from synth import fill, gpu, plan

pytestmark = pytest.mark.gpu

FULL = "ACGTNRYSWKMBDHVACGTNRYSWKMBDHVAC"  # 32 positions
PAIRS = {
    "ends": [(FULL, FULL[::-1], 6, 2), ("ACGTA", "TTGCA", 0, 5), ("NNNNN", "RYSWK", 1, 0)],
    "wave": [("ACGTRYACGTACGG", "TTGCANNGCATTA", 2, 0), ("GGCCAATTGGCA", "ACGTTGCAACGT", 3, 3)],
    "many": [(FULL[i: i + 12 + i], FULL[3 * i: 3 * i + 14], i % 4, i % 3) for i in range(6)],
}


@pytest.mark.parametrize("nruns", [0, 6])
@pytest.mark.parametrize("name", list(PAIRS))
def test_table_count_matches_the_oracle(name, nruns):
    import torch

    from paper_2509_13300_amd import path

    pairs = [plan.PairSpec(f, r, k=k, clamp=c, min_len=20, max_len=60) for f, r, k, c in PAIRS[name]]
    p = plan.tiny(9500 + nruns + len(name), n_genomes=4, len_lo=20, len_hi=4000, pair=pairs[0], n_copies=(0, 1),
                  nruns=nruns, span=70)
    p = p.with_lengths([5, 33] + p.lengths[2:].tolist())
    dev = torch.device("cuda:0")
    ascii, off = gpu.fill_cuda(p, dev)
    coll, _ = path.pack(ascii, off, p.lengths, with_nmask=nruns > 0)
    buf = path.alloc(coll, pairs, 1 << 18, 16, dev)
    print(name, nruns, flush=True)
    path.run(coll, pairs, buf, do_tm=False, do_pair=False)
    got = path.hits_numpy(buf)
    assert path.result(buf.hit_res)["status"] == 0 and got.size > 0
    seqs = [fill.genome_bytes(p, g) for g in range(p.n)]
    for q, pr in enumerate(pairs):
        want = oscan.scan_collection(seqs, [pr])
        mine = got[got["pair"] == q]
        say("table count", name, nruns, q, "sites", mine.size)
        assert mine.size == want.size
        for f in ("genome", "pos", "mm"):
            assert np.array_equal(mine[f], want[f]), (q, f)
        assert np.array_equal(mine["strand_primer"] >> 1, want["strand"])
        assert np.array_equal(mine["strand_primer"] & 1, want["primer"])
