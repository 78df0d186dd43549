"""Serving parts with full candidate slices: a first run leaves them as they are and the
part runs again with more room (filled again, they took the filter 20 times its time on
GC-rich contigs), and where that much room does not fit the pool, it runs again in
the same buffers with the slices filled again."""
import numpy as np
import pytest

from gpu_util import say
from synth import plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return torch.device("cuda:0")


def _contigs(dev, lengths, letters, seed):
    import torch

    from paper_2509_13300_amd import path

    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    table = torch.tensor(list(letters), dtype=torch.uint8, device=dev)
    ascii = table[torch.randint(0, len(letters), (int(off[-1]),), device=dev, generator=g)]
    return ascii, off, lambda a: path.pack(a, torch.from_numpy(off).to(dev), lengths)[0]


def _job(server, pair, n):
    server.submit(pair, np.arange(n, dtype=np.uint32))
    st = server.wait(60.0)
    assert st is not None and st["status"] == 0
    got = server.result(st)
    server.release(st["job"])
    return got


def test_full_slices_of_a_part_take_a_second_run(dev):
    import torch

    from paper_2509_13300_amd import _lib as L
    from paper_2509_13300_amd import path

    pair = plan.PairSpec("TTCCCCCAAYGCSCC", "WCGGNCGACATTTTSWGAGGAGGAYGACR", k=2, clamp=0, min_len=459, max_len=2762)
    n = 144
    lengths = np.exp(np.random.default_rng(5).uniform(np.log(9600), np.log(4.3e6), n)).astype(np.int64)
    ascii, _, pack = _contigs(dev, lengths, b"AACCCGGGTT", 5)  # 60% GC
    coll = pack(ascii)
    buf = path.alloc(coll, [pair], 1 << 20, 1 << 20, dev)
    server = path.Server(coll, 2 << 30, dev, n_lanes=1, host_pool_bytes=256 << 20)
    us = []
    for run in (lambda: path.run(coll, [pair], buf, fused=False), lambda: _job(server, pair, n)):
        run()
        torch.cuda.synchronize()
        L.ah_profile_reset()
        L.ah_profile_enable(True)
        for _ in range(10):
            run()
        torch.cuda.synchronize()
        L.ah_profile_enable(False)
        us.append(L.ah_profile_query("scan")[1] / 10 * 1e3)
    hits, amps = _job(server, pair, n)
    say("filter of a query and of a part, us", us, "retries", server.stats()["retries"], "sites", hits.size)
    assert server.stats()["retries"] == 12  # every job: the slices are full
    server.close()
    assert path.result(buf.hit_res)["status"] == 0 and path.result(buf.amp_res)["status"] == 0
    assert hits.tobytes() == path.hits_numpy(buf).tobytes()
    assert amps.tobytes() == path.amps_numpy(buf).tobytes()
    assert us[1] <= 5 * us[0]


def test_full_slices_of_a_part_in_a_small_pool(dev):
    """Half the windows of an (AC)n repeat pass the filter, which keeps A and C alone of the
    primer; a list of them all does not fit the pool."""
    import torch

    from paper_2509_13300_amd import path

    pair = plan.PairSpec("CATGACACACACACACACAC", "GGATCCAAGTTCGACGTAAC", k=0, clamp=0, min_len=40, max_len=400)
    lengths = np.full(4, 500_000)
    ascii, off, pack = _contigs(dev, lengths, b"ACGT", 6)
    for i in range(4):
        ascii[int(off[i]) + 1000: int(off[i]) + 451_000] = torch.tensor(list(b"AC"), dtype=torch.uint8, device=dev).repeat(225_000)
        for at, s in ((460_000, pair.fwd), (460_200, pair.rev[::-1].translate(str.maketrans("ACGT", "TGCA")))):
            ascii[int(off[i]) + at: int(off[i]) + at + 20] = torch.tensor(list(s.encode()), dtype=torch.uint8, device=dev)
    coll = pack(ascii)
    buf = path.alloc(coll, [pair], 1 << 21, 1 << 12, dev)
    path.run(coll, [pair], buf, fused=False)
    torch.cuda.synchronize()
    assert path.result(buf.hit_res)["status"] == 0 and path.result(buf.amp_res)["count"] == 4
    server = path.Server(coll, 16 << 20, dev, n_lanes=1, host_pool_bytes=16 << 20)
    hits, amps = _job(server, pair, 4)
    say("sites", hits.size, "retries", server.stats()["retries"])
    assert server.stats()["retries"] == 1
    server.close()
    assert hits.tobytes() == path.hits_numpy(buf).tobytes()
    assert amps.tobytes() == path.amps_numpy(buf).tobytes()
