"""The numbers at which ah_query changes its launches, byte for byte against the
separate calls: 65,536 genomes (above, the tile prefix is three launches and the
clearing its own), 131,072 segments (above, the radix sort takes the sites), and 4,096
segments of several pairs (above, the segments' first slots are a launch of their own
and a tile has four waves)."""
import numpy as np
import pytest

from gpu_util import say
from synth import plan

pytestmark = pytest.mark.gpu

PAIRS = [plan.PairSpec("ACGTRYACGTACAG", "TTGCANNGCATTGC", k=2, clamp=0, min_len=20, max_len=100),
         plan.PairSpec("GGATCCTTGAGCAA", "CATTGACCRGATAC", k=1, clamp=0, min_len=20, max_len=100)]


@pytest.mark.parametrize("n,pairs", [(65_536, 1), (65_537, 1), (131_072, 1), (131_073, 1), (65_536, 2), (65_537, 2),
                                     (2048, 2), (2049, 2)])
def test_either_side_of_the_limits(n, pairs):
    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    pairs = PAIRS[:pairs]
    rng = np.random.default_rng(n + len(pairs))
    length = 120
    seq = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, (n, length))].copy()
    for q, p in enumerate(pairs):  # an amplicon in every seventh genome, the last one among them
        f = p.fwd.replace("R", "A").replace("Y", "C").replace("N", "G").encode()
        r = p.rev.replace("R", "A").replace("N", "G").encode()[::-1].translate(bytes.maketrans(b"ACGT", b"TGCA"))
        at = 5 + 50 * q
        seq[n - 1::-7, at: at + 14] = np.frombuffer(f, np.uint8)
        seq[n - 1::-7, at + 30: at + 44] = np.frombuffer(r, np.uint8)
    dev_seq = torch.from_numpy(seq.reshape(-1)).to(dev)
    off = torch.arange(n + 1, dtype=torch.int64, device=dev) * length
    coll, _ = path.pack(dev_seq, off, np.full(n, length))
    print(n, len(pairs), flush=True)
    out = []
    for fused in (False, True):
        buf = path.alloc(coll, pairs, 200_000, 100_000, dev)
        path.run(coll, pairs, buf, fused=fused)
        torch.cuda.synchronize()
        out.append((path.result(buf.hit_res), path.result(buf.amp_res), path.hits_numpy(buf).tobytes(),
                    path.amps_numpy(buf).tobytes()))
    say("limits", n, len(pairs), out[0][:2])
    assert out[0][0]["status"] == 0 and out[0][1]["status"] == 0
    assert out[0][1]["count"] >= n // 7 * len(pairs)
    last = np.frombuffer(out[0][2], dtype=np.uint32).reshape(-1, 4)[:, 0].max()
    assert last == n - 1
    assert out[0] == out[1]
