"""The FASTA writer at the lengths where its steps end: a lane takes eight bases, a
wave 512, and only the last lane of a sequence can have fewer.  Amplicons of either
strand of every residue mod 8 around one and two waves' steps and of the shortest
ones, at every offset in genomes whose segments end inside them, with N bases."""
import numpy as np
import pytest

from gpu_util import say
from oracle import fasta as ofasta
from synth import plan
from test_gpu_fasta import parse, same_header

pytestmark = pytest.mark.gpu

PAIR = plan.PairSpec("ACGTTGCAAGCT", "GGATCCTTGAGC", k=0, clamp=0, min_len=24, max_len=1100)
LENGTHS = list(range(24, 50)) + list(range(504, 521)) + list(range(1016, 1034))


@pytest.mark.parametrize("masked", [False, True])
def test_lengths_around_the_writers_steps(masked):
    import torch

    from paper_2509_13300_amd import path

    dev = torch.device("cuda:0")
    rng = np.random.default_rng(12 + masked)
    comp = bytes.maketrans(b"ACGT", b"TGCA")
    seqs = []
    for n in LENGTHS:
        for rc in (False, True):
            block = bytearray(np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, n)].tobytes())
            block[:12] = PAIR.fwd.encode()
            block[n - 12:] = PAIR.rev.encode()[::-1].translate(comp)
            block = bytes(block)
            if rc:
                block = block[::-1].translate(comp)
            block = np.frombuffer(block, np.uint8).copy()
            if masked and n > 40:
                block[rng.integers(12, n - 12, 3)] = ord("N")
            pads = [np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, int(m))] for m in rng.integers(0, 700, 2)]
            seqs.append(np.concatenate([pads[0], block, pads[1]]))
    lengths = np.array([s.size for s in seqs])
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    coll, _ = path.pack(torch.from_numpy(np.concatenate(seqs)).to(dev), torch.from_numpy(off).to(dev), lengths,
                        with_nmask=masked)
    buf = path.alloc(coll, [PAIR], 4096, 4096, dev)
    path.run(coll, [PAIR], buf)
    fb = path.fasta_alloc(coll, 1, buf.amp_cap, 1 << 20, dev)
    path.fasta(coll, 1, buf, fb)
    torch.cuda.synchronize()
    assert path.result(fb.text_res)["status"] == 0
    recs = ofasta.records([s.tobytes() for s in seqs], path.hits_numpy(buf), path.amps_numpy(buf))
    lens = {orient: {len(s) for h, s, _ in recs if orient in h} for orient in ("orient=FR", "orient=RF")}
    say("lengths", masked, len(recs), len(lens["orient=FR"]), len(lens["orient=RF"]))
    assert lens["orient=FR"] >= set(LENGTHS) and lens["orient=RF"] >= set(LENGTHS)
    got = parse(path.fasta_text(fb))
    assert len(got) == len(recs)
    for (gh, gs), (oh, os_, _) in zip(got, recs):
        same_header(gh, oh)
        assert gs == os_, gh
    assert [int(x) for x in fb.seq_hash[: len(recs)].cpu().numpy().view(np.uint64)] == [h for _, _, h in recs]
