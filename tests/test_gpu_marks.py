"""Record-start bits of a batch against numpy: one record, empty records, runs
of records at the edges of 32-base words and of the 32768-base blocks a
workgroup writes, more records than one search step covers, and stale words."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def expected(off):
    n = int(off[-1])
    bits = np.zeros((n + 31) // 32 * 32, dtype=np.uint8)
    inner = off[1:-1].astype(np.int64)
    bits[inner[inner < n]] = 1
    return np.packbits(bits.reshape(-1, 8), axis=1, bitorder="little").reshape(-1).view(np.uint32)


BLOCK = 32768
CASES = {
    "one record": [0, 100_003],
    "one base": [0, 1],
    "empty records": [0, 0, 0, 5, 5, 5, 70, 70],
    "block edges": [0, 31, 32, 33, BLOCK - 1, BLOCK, BLOCK, BLOCK + 1, 2 * BLOCK, 3 * BLOCK - 1, 3 * BLOCK, 5 * BLOCK + 7],
    "ends at a block": [0, BLOCK - 32, 2 * BLOCK],
    "nothing in the middle": [0, 10, 9 * BLOCK + 3, 9 * BLOCK + 4, 10 * BLOCK],
}


@pytest.mark.parametrize("name", list(CASES) + ["%d random" % n for n in (2, 63, 64, 65, 4097, 300_000)])
def test_marks(name):
    from paper_2606_24417_amd import Filter

    if name in CASES:
        off = np.array(CASES[name], dtype=np.uint64)
    else:
        n = int(name.split()[0])
        rng = np.random.default_rng(n)
        lens = rng.integers(0, 9 if n > 1000 else 5000, size=n)
        lens[-1] += 1
        off = np.concatenate(([0], np.cumsum(lens))).astype(np.uint64)
    d = torch.from_numpy(off.view(np.int64)).cuda()
    nwords = (int(off[-1]) + 31) // 32
    buf = torch.full((nwords + 8,), -1, dtype=torch.int32, device="cuda")
    Filter.mark_record_starts(d, int(off[-1]), starts=buf)
    torch.cuda.synchronize()
    got = buf.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:nwords], expected(off))
    assert (got[nwords:] == 0xFFFFFFFF).all(), "words past the batch written"


# from 2^24 words (537 Mbp) on a workgroup writes 4096 words; records at the
# edges of both sizes of block, dense at the start and sparse after
@pytest.mark.parametrize("nwords", [(1 << 24) - 1, (1 << 24) + 5000])
def test_marks_of_large_batches(nwords):
    from paper_2606_24417_amd import Filter

    n = nwords * 32 - 7
    rng = np.random.default_rng(nwords)
    edge = np.arange(32 * 2048, n - 2, 32 * 2048, dtype=np.int64)
    cut = np.concatenate([rng.integers(1, 3_000_000, 400_000), rng.integers(1, n, 300_000), edge[::3] - 1, edge[::5],
                          edge[::7] + 1])
    off = np.concatenate(([0], np.sort(cut), [n])).astype(np.uint64)
    d = torch.from_numpy(off.view(np.int64)).cuda()
    buf = torch.full((nwords + 8,), -1, dtype=torch.int32, device="cuda")
    Filter.mark_record_starts(d, n, starts=buf)
    torch.cuda.synchronize()
    got = buf.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:nwords], expected(off))
    assert (got[nwords:] == 0xFFFFFFFF).all(), "words past the batch written"
