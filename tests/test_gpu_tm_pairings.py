"""Which pairings the Tm kernels evaluate: sites whose best pairing is surely the
representative are not enumerated, the others are (in their own lane, or dealt
over the wave).  Primers with degenerate ends (unpairing one changes the
outermost pair), with many degenerate positions, and clamped ones, against the
oracle's maximum over every oligo."""
import numpy as np
import pytest

from gpu_util import run_gpu, run_oracle, say
from oracle import tm as otm
from synth import plan

pytestmark = pytest.mark.gpu

# Tm in single precision against the FP64 oracle: the final operations (a
# rounded Delta-H, a rounded denominator, one division, one subtraction at
# ~350 K) are off by a few 2^-24 x 350 = 2e-5 K; 1e-4 leaves room for method 7's
# second rounding, and is far below what a missed pairing changes.
TOL = 1e-4

PAIRS = {
    "ends": ("YACGTTGCAAGCTTGR", "SATTGCCAGTWACCGTTK", 2, 0),
    "hot": ("NGGCGCGCCGSGCCGGCN", "NCCGGGCSCGGCCGGCGCN", 3, 0),
    "many": ("RYSWKMRYSWACGTKM", "NNACGTRYACGTNN", 3, 0),
    "clamp": ("YRACGTTGCAAGCTYR", "SWTTGCCAGTWACCGTTSK", 2, 3),
    "short": ("NNNNN", "RYWSK", 2, 0),
}


@pytest.mark.parametrize("salt", [0, 1, 5, 7])
@pytest.mark.parametrize("name", list(PAIRS))
def test_best_pairing_against_every_oligo(name, salt):
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path

    fwd, rev, k, clamp = PAIRS[name]
    pair = plan.PairSpec(fwd, rev, k=k, clamp=clamp, min_len=30, max_len=400)
    n = 2 if name == "short" else 6
    p = plan.tiny(8800 + len(name), n_genomes=n, len_lo=200, len_hi=400 if name == "short" else 6000, pair=pair,
                  n_copies=(1, 3) if name != "short" else (0, 1), gc_lo=0.4, gc_hi=0.6, nruns=3, span=60)
    dev = torch.device("cuda:0")
    print(name, salt, flush=True)
    _, buf = run_gpu(p, [pair], dev, tm=L.tm_params(saltcorr=salt))
    got = path.hits_numpy(buf)
    want, _ = run_oracle(p, [pair], tmp=otm.TmParams(saltcorr=salt))
    assert got.size == want.size > 0
    err = np.abs(got["tm"].astype(np.float64) - want["tm"])
    say("pairings", name, salt, "sites", got.size, "max error", float(np.nanmax(err)))
    assert np.array_equal(np.isnan(got["tm"]), np.isnan(want["tm"]))
    assert float(np.nanmax(err)) <= TOL
