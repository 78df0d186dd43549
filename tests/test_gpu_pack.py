"""Packing against the layout's definition, written out in numpy: every word,
mask word and count, halo words and padding included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def packed(seq):
    """(words [W, 2], mask [W]) of one sequence, from the layout: bit b of word
    t is base b * S + t, positions past the end read as A."""
    n = seq.size
    S = (n + 31) // 32
    W = (S + 31 + 1) // 2 * 2
    code = np.zeros(256, np.int64)
    good = np.zeros(256, bool)
    for i, ch in enumerate("ACGT"):
        for c in (ch, ch.lower()):
            code[ord(c)] = i
            good[ord(c)] = True
    pos = np.arange(32)[None, :] * S + np.arange(W)[:, None]
    inside = pos < n
    b = seq[np.where(inside, pos, 0)] if n else np.zeros(pos.shape, np.uint8)
    c = np.where(inside & good[b], code[b], 0)
    bad = inside & ~good[b]
    bit = 1 << np.arange(32, dtype=np.int64)
    words = np.stack([((c >> 1) * bit).sum(1), ((c & 1) * bit).sum(1)], axis=1)
    return words.astype(np.uint32), (bad * bit).sum(1).astype(np.uint32), int(((seq.size > 0) and (~good[seq]).sum()))


# around a group of four words, a wave's and a workgroup's run of groups, the
# shortest sequences (fewer bytes than a load) and empty ones
CASES = {
    "short": [1, 2, 3, 4, 5, 0, 7, 31, 32, 33, 63, 64, 65, 97, 0, 1],
    "groups": [32 * 4 - 1, 32 * 4, 32 * 4 + 1, 32 * 5, 32 * 7 + 31, 3, 32 * 8],
    "runs": [32 * 256 - 33, 32 * 256, 32 * 256 + 1, 32 * 1024, 32 * 1024 + 31, 32 * 993],
    "long": [3_000_017],
    "many": [int(x) for x in np.random.default_rng(5).integers(0, 900, 700)],
}


@pytest.mark.parametrize("kind", ["clean", "mixed", "noise"])
@pytest.mark.parametrize("name", list(CASES))
def test_pack_words_match_the_layout(name, kind):
    import torch

    from paper_2509_13300_amd import path

    lengths = np.array(CASES[name], dtype=np.int64)
    rng = np.random.default_rng(len(name) + len(kind))
    total = int(lengths.sum())
    alphabet = {"clean": b"ACGT", "mixed": b"ACGTacgt" * 30 + b"NRY-n", "noise": bytes(range(256))}[kind]
    seq = np.frombuffer(alphabet, np.uint8)[rng.integers(0, len(alphabet), total)]
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    dev = torch.device("cuda:0")
    ascii = torch.from_numpy(seq.copy()).to(dev)
    for with_nmask in (True, False):
        print(name, kind, with_nmask, flush=True)
        coll, non_acgt = path.pack(ascii, torch.from_numpy(off).to(dev), lengths, with_nmask=with_nmask)
        words = coll.words.cpu().numpy().view(np.uint32).reshape(-1, 2)
        woff = coll.word_off.cpu().numpy()
        assert np.array_equal(coll.len.cpu().numpy()[: lengths.size], lengths)
        for g in range(lengths.size):
            want, mask, bad = packed(seq[off[g]: off[g + 1]])
            assert np.array_equal(words[woff[g]: woff[g + 1]], want), (name, kind, g)
            if with_nmask:
                got = coll.nmask[woff[g]: woff[g + 1]].cpu().numpy().view(np.uint32)
                assert np.array_equal(got, mask), (name, kind, g)
                assert int(non_acgt[g]) == bad, (name, kind, g)
