"""Requests whose Tm denominator, Delta-S + R ln C + salt entropy, is not
negative for every pairing of a primer (strand concentrations from tens of mM on):
unpairing positions can then lift it past zero, where losing a stable stack
raises the Tm, so the maximum over the compatible oligos may be far from
the oligo that pairs everywhere.  Against the oracle's maximum over every
oligo, through the fused query and the separate calls, and the sites kept by a
minimum Tm."""
import numpy as np
import pytest

from gpu_util import amp_tuples, run_gpu, run_oracle, say
from oracle import tm as otm
from synth import plan

pytestmark = pytest.mark.gpu

# The stacks and initiations (at most six terms here) are held as floats below
# 32, off by up to 2^-20 each: 6e-6 in a denominator of 0.42 or more at these
# sites' maxima, and 6 x 2^-22 in a Delta-H of 0.2 or more; four roundings to
# float on top.  Below 2.2e-5 of the Tm in kelvin; 5e-5 leaves room.
REL_TOL = 5e-5

CASES = [
    ("ANGNT", "ASGRT", 2, 0, dict(dnac1=2e7, saltcorr=0)),
    ("ANGNT", "ASGRT", 2, 0, dict(dnac1=1e8, dnac2=5e7, saltcorr=0)),
    ("ANGNT", "ASGRT", 2, 0, dict(dnac1=6e7, saltcorr=4)),
    ("ANGNT", "ASGRT", 2, 0, dict(dnac1=3e7, saltcorr=5, Na=1000.0, Mg=0.0)),
    ("GNANC", "ASKTC", 2, 1, dict(dnac1=1e9, saltcorr=0)),
    ("GNANCNT", "CATNGNA", 3, 0, dict(dnac1=1e9, saltcorr=0)),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_denominator_past_zero_against_every_oligo(case):
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path

    fwd, rev, k, clamp, kw = CASES[case]
    pair = plan.PairSpec(fwd, rev, k=k, clamp=clamp, min_len=10, max_len=60)
    p = plan.tiny(9700, n_genomes=2, len_lo=200, len_hi=300, pair=pair, n_copies=(0, 1), span=30)
    dev = torch.device("cuda:0")
    min_tm = 100.0
    print(fwd, rev, kw, flush=True)
    coll, buf = run_gpu(p, [pair], dev, tm=L.tm_params(**kw), filter_tm=True, min_tm=min_tm)
    got, amps = path.hits_numpy(buf), path.amps_numpy(buf)
    want, want_amps = run_oracle(p, [pair], tmp=otm.TmParams(**kw), filter_tm=True, min_tm=min_tm)
    assert got.size == want.size > 0
    kelvin = want["tm"] + 273.15
    err = np.abs(got["tm"].astype(np.float64) - want["tm"])
    say("denominators", fwd, kw, "sites", got.size, "highest", float(want["tm"].max()),
        "worst relative error", float((err / np.abs(kelvin)).max()))
    assert want["tm"].max() > 200.0
    assert np.all(err <= REL_TOL * np.abs(kelvin))
    assert amp_tuples(amps) == amp_tuples(want_amps)
    sep = path.alloc(coll, [pair], 1 << 16, 1 << 16, dev)
    path.run(coll, [pair], sep, tm=L.tm_params(**kw), filter_tm=True, min_tm=min_tm, fused=False)
    assert path.hits_numpy(sep).tobytes() == got.tobytes()
    assert path.amps_numpy(sep).tobytes() == amps.tobytes()
