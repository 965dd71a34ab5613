"""GPU parity of the binned insert (large batches: super-k-mers sorted by shard
range, then applied slice by slice) against the oracle, bit for bit: filters
with one and with two levels of bins, every shard size, windows that are cut
into several records, batches around the tile of 8192 k-mers, crowded shards
whose bins overflow, several batches into one filter, and the captured forms.
"""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(x):
    return torch.from_numpy(np.array(x, copy=True)).cuda()


def doff(off):
    return dev(np.asarray(off, dtype=np.uint64).view(np.int64))


def records(n, mean, seed, p_invalid=0.0005):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 2 * mean, size=max(1, n // mean))
    lens[::7] = rng.integers(0, 40, size=lens[::7].size)
    off = np.concatenate(([0], np.cumsum(lens))).astype(np.uint64)
    seq = synth.uniform_acgt(int(off[-1]), seed).copy()
    bad = rng.random(seq.size) < p_invalid
    seq[bad] = rng.choice(np.frombuffer(b"NnX-.", dtype=np.uint8), bad.sum())
    return seq, off


def check(params, S, batches, unaligned=False):
    from paper_2606_24417_amd import Filter

    k, s, m, H, bits = params
    p = oracle.Params(k, s, m, H, bits, shard_words=S)
    want = p.empty()
    f = Filter(k, s, m, H, bits, shard_words=S)
    for seq, off in batches:
        want = oracle.insert(p, want, seq, off)
        d = dev(np.concatenate([seq[:1], seq]))[1:] if unaligned else dev(seq)
        f.insert(d, doff(off) if off is not None else None)
    torch.cuda.synchronize()
    got = f.get_bits()
    f.close()
    bad = np.flatnonzero(got != want)
    assert bad.size == 0, "%d of %d words differ, first %s" % (bad.size, got.size, bad[:5].tolist())


# filters of 2^24 bits (64 slices, one level), 2^27 (512 slices, two levels)
# and 2^28; k, m classes: m = 16, m < 16, m > 16, k = 32; w from 6 to 32 (w > 16
# cuts super-k-mers into several records); every H up to 8
@pytest.mark.parametrize("bits,S", [(1 << 24, 4), (1 << 25, 16), (1 << 27, 4), (1 << 27, 8)])
@pytest.mark.parametrize("k,s,m,H", [(31, 28, 16, 4), (31, 28, 18, 4), (31, 26, 12, 8), (21, 15, 11, 3),
                                     (32, 26, 17, 7), (21, 15, 16, 2), (32, 20, 1, 1), (24, 1, 19, 5),
                                     (13, 9, 4, 6)])
def test_parameters_match_oracle(k, s, m, H, bits, S):
    print("case binned k=%d s=%d m=%d H=%d bits=%d S=%d" % (k, s, m, H, bits, S), flush=True)
    check((k, s, m, H, bits), S, [records(600_000, 900, k + 100 * m + S)])


# the batch ends inside, at and after a tile, with its last k-mers in one lane
@pytest.mark.parametrize("n", [131072 + 30, 131072 + 31, 17 * 8192 + 30, 17 * 8192 + 31, 17 * 8192 + 62, 20 * 8192 + 4111])
def test_lengths_around_tiles(n):
    print("case binned length", n, flush=True)
    seq = synth.uniform_acgt(n, n)
    check((31, 28, 16, 4, 1 << 24), 4, [(seq, None)])
    check((31, 28, 16, 4, 1 << 24), 4, [(seq, None)], unaligned=True)


# reads of 100 bp, one contig, and several batches on top of one another
def test_batches_accumulate():
    for bits in (1 << 24, 1 << 27):
        check((31, 28, 16, 4, bits), 4,
              [records(400_000, 100, 1), (synth.uniform_acgt(300_001, 2), None), records(500_000, 20_000, 3),
               (synth.uniform_acgt(5_000, 4), None)])


# repeats of period 1 to 7 and 40 crowd a few shards: equal neighbours are
# dropped, the others overflow their bin and are applied directly
@pytest.mark.parametrize("period", [1, 2, 3, 5, 7, 40, 1000])
@pytest.mark.parametrize("bits,S", [(1 << 24, 4), (1 << 27, 4), (1 << 27, 16)])
def test_crowded_shards(period, bits, S):
    print("case binned period", period, bits, S, flush=True)
    seq = synth.uniform_acgt(800_000, 10 + period).copy()
    seq[100_000:] = np.resize(seq[:period], 700_000)
    check((31, 28, 16, 4, bits), S, [(seq, None)])


# homopolymers of each base, and runs of N longer than a tile
def test_homopolymers_and_gaps():
    parts = [np.full(60_000, ord(c), dtype=np.uint8) for c in "ACGTNacgt"]
    parts += [synth.uniform_acgt(50_000, 5)]
    check((31, 28, 16, 4, 1 << 24), 4, [(np.concatenate(parts), None)])


# more k-mers than are binned at a time (2^27), against the atomic insert
def test_several_chunks():
    from paper_2606_24417_amd.sbf import INSERT_ATOMIC, Filter

    seq = dev(synth.background((1 << 27) + 100_003, 9))
    got = []
    for mode in (0, INSERT_ATOMIC):
        f = Filter(31, 28, 16, 4, 1 << 28)
        f.set_insert_mode(mode)
        f.insert(seq)
        torch.cuda.synchronize()
        got.append(f.get_bits())
        f.close()
    assert np.array_equal(got[0], got[1])


# filters from 2^34 bits on have 256 buckets and tiles of 16384 k-mers
@pytest.mark.parametrize("k,s,m,H,n", [(21, 15, 11, 4, 70_000_017), (21, 15, 16, 2, 68_000_000)])
def test_wide_tiles(k, s, m, H, n):
    from paper_2606_24417_amd.sbf import INSERT_ATOMIC, Filter

    print("case binned wide tile k=%d m=%d" % (k, m), flush=True)
    seq = synth.background(n, 11).copy()
    seq[1_000_000:1_400_000] = np.resize(seq[:40], 400_000)  # a crowded shard
    seq[2_000_000:2_050_000] = ord("A")
    seq[3_000_000::99_991] = ord("N")
    d, got = dev(seq), []
    for mode in (0, INSERT_ATOMIC):
        f = Filter(k, s, m, H, 1 << 34)
        f.set_insert_mode(mode)
        f.insert(d)
        torch.cuda.synchronize()
        got.append(f.get_bits())
        f.close()
    assert np.array_equal(got[0], got[1])


def test_captured_inserts():
    """sbf_graph_create captures the binned insert with its own scratch; a
    stream captured by the caller takes the two passes."""
    from paper_2606_24417_amd import Filter, Graph

    seq, off = records(400_000, 500, 21)
    p = oracle.Params(31, 28, 16, 4, 1 << 24)
    want = oracle.insert(p, p.empty(), seq, off)
    d, o = dev(seq), doff(off)
    f = Filter(31, 28, 16, 4, 1 << 24)
    g = Graph(f, ins=d, ins_off=o, clear_first=True)
    for _ in range(3):
        g.launch()
        torch.cuda.synchronize()
        assert np.array_equal(f.get_bits(), want)
    g.close()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        f.insert(d, o)  # allocates the stream's scratch before the capture
        f.set_tile(32, 0)
        f.insert(d, o)
        f.set_tile(0, 0)
    torch.cuda.synchronize()
    cg = torch.cuda.CUDAGraph()
    with torch.cuda.graph(cg, stream=st):
        f.clear()
        f.insert(d, o)
    for _ in range(3):
        cg.replay()
        torch.cuda.synchronize()
        assert np.array_equal(f.get_bits(), want)
        f.insert(d, o)
        torch.cuda.synchronize()
        assert np.array_equal(f.get_bits(), want)
    f.close()


# tiles in which no run starts: records shorter than k over several tiles, alone
# and between valid ones, a last tile that holds only the end of the last
# record, and valid bases that never make a k-mer
@pytest.mark.parametrize("bits,S", [(1 << 24, 4), (1 << 27, 4), (1 << 27, 16)])
@pytest.mark.parametrize("form", ["short", "between", "tail", "gaps"])
def test_tiles_without_runs(form, bits, S):
    print("case binned no runs", form, bits, S, flush=True)
    rng = np.random.default_rng(31)
    short = rng.integers(1, 31, size=14_000)
    if form == "gaps":
        seq = synth.uniform_acgt(200_000, 32).copy()
        seq[20_000:180_000:30] = ord("N")
        batch = (seq, None)
    else:
        if form == "short":
            lens = short
        elif form == "between":
            lens = np.concatenate([[60_000], short[:7_000], [50_000], short[7_000:], [40_000]])
        else:
            lens = np.array([20 * 8192 - 40, 60, 29])
        off = np.concatenate(([0], np.cumsum(lens))).astype(np.uint64)
        batch = (synth.uniform_acgt(int(off[-1]), 33), off)
    assert batch[0].size > 131072 + 31
    check((31, 28, 16, 4, bits), S, [batch])
    check((31, 28, 16, 4, bits), S, [(synth.uniform_acgt(150_000, 34), None), batch])


# crowded shards in tiles with more runs than their list holds (short windows),
# with more shards than fit the table of a round, and with every shard size
@pytest.mark.parametrize("k,s,m,H", [(31, 28, 16, 4), (21, 15, 16, 4), (31, 27, 16, 8), (32, 20, 1, 2)])
@pytest.mark.parametrize("period", [3, 40, 1000, 5000])
@pytest.mark.parametrize("bits,S", [(1 << 25, 4), (1 << 25, 16), (1 << 27, 8)])
def test_crowded_parameters(bits, S, period, k, s, m, H):
    print("case binned crowded", k, s, m, H, period, bits, S, flush=True)
    seq = np.resize(synth.uniform_acgt(period, 60 + period), 700_000)
    seq[300_000:300_005] = ord("N")
    check((k, s, m, H, bits), S, [(seq, None), (synth.uniform_acgt(200_000, 61), None)])


# A batch of few distinct super-k-mers takes about as long binned as with the
# two passes that the set tile selects (1.2 times; 12 times where each record
# that found its bucket full was tested in the filter by itself).
@pytest.mark.parametrize("period", [40, 1000])
def test_crowded_batches_are_not_slow(period):
    from paper_2606_24417_amd import Filter

    d = dev(np.resize(synth.uniform_acgt(period, 70 + period), 2_000_000))
    f = Filter(31, 28, 16, 4, 1 << 25, shard_words=16)
    took = []
    for tile in (0, 16):
        f.set_tile(tile, 0)
        times = []
        for _ in range(12):
            f.clear()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f.insert(d)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took.append(sorted(times)[len(times) // 2])
    f.close()
    print("binned %.3f ms, two passes %.3f ms" % tuple(took), flush=True)
    assert took[0] < 2.5 * took[1]


def test_capture_after_the_same_insert_as_warm_up():
    """One insert on a stream prepares that stream for the capture of the same
    insert, also where another stream has used the filter before."""
    from paper_2606_24417_amd import Filter

    seq, off = records(400_000, 500, 23)
    p = oracle.Params(31, 28, 16, 4, 1 << 24)
    want = oracle.insert(p, p.empty(), seq, off)
    d, o = dev(seq), doff(off)
    f = Filter(31, 28, 16, 4, 1 << 24)
    f.query(d, o)
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        f.insert(d, o)
    torch.cuda.synchronize()
    cg = torch.cuda.CUDAGraph()
    with torch.cuda.graph(cg, stream=st):
        f.clear()
        f.insert(d, o)
    for _ in range(3):
        cg.replay()
        torch.cuda.synchronize()
        assert np.array_equal(f.get_bits(), want)
        f.clear()
        f.insert(d, o)
        torch.cuda.synchronize()
        assert np.array_equal(f.get_bits(), want)
    f.close()


def test_growing_batches_do_not_wait():
    """A stream-ordered insert whose scratch grows returns while other work of
    the device is still running, and the earlier insert's records stay."""
    import time

    from paper_2606_24417_amd import Filter

    seqs = [synth.background(n, 90 + i) for i, n in enumerate((2_000_000, 5_000_000, 12_000_000))]
    ds = [dev(x) for x in seqs]
    p = oracle.Params(31, 28, 16, 4, 1 << 28)
    want = p.empty()
    for x in seqs:
        want = oracle.insert(p, want, x)
    warm = Filter(31, 28, 16, 4, 1 << 28)
    warm.insert(ds[0])
    f = Filter(31, 28, 16, 4, 1 << 28)
    other = torch.cuda.Stream()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    torch.cuda._sleep(10_000_000)
    b.record()
    torch.cuda.synchronize()
    cycles = int(10_000_000 * 500.0 / a.elapsed_time(b))  # half a second
    busy = torch.cuda.Event()
    with torch.cuda.stream(other):
        torch.cuda._sleep(cycles)
        busy.record()
    t0 = time.perf_counter()
    for d in ds:
        f.insert(d)
    took = time.perf_counter() - t0
    still = not busy.query()
    torch.cuda.synchronize()
    print("three growing inserts returned after %.1f ms" % (took * 1e3), flush=True)
    assert still and took < 0.25
    assert np.array_equal(f.get_bits(), want)
    f.insert(ds[0])
    assert np.array_equal(f.get_bits(), want)
    f.close()
    warm.close()


def test_growing_during_a_capture_elsewhere():
    """A large insert on its own stream, while another stream is captured."""
    from paper_2606_24417_amd import Filter

    seq = synth.background(3_000_000, 95)
    p = oracle.Params(31, 28, 16, 4, 1 << 28)
    want = oracle.insert(p, p.empty(), seq)
    d = dev(seq)
    small = d[:100_000]
    f, g = Filter(31, 28, 16, 4, 1 << 28), Filter(31, 28, 16, 4, 1 << 20)
    st, own = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    f.insert(small, stream=own)  # the stream's counters
    g.insert(small, stream=st)
    torch.cuda.synchronize()
    cg = torch.cuda.CUDAGraph()
    with torch.cuda.graph(cg, stream=st):
        g.clear()
        f.insert(d, stream=own)
        g.insert(small)
    torch.cuda.synchronize()
    assert np.array_equal(f.get_bits(), want)
    q = oracle.Params(31, 28, 16, 4, 1 << 20)
    want_small = oracle.insert(q, q.empty(), seq[:100_000])
    for _ in range(3):
        cg.replay()
        torch.cuda.synchronize()
        assert np.array_equal(g.get_bits(), want_small)
        g.insert(small)
        torch.cuda.synchronize()
    f.close()
    g.close()


@pytest.mark.parametrize("bits", [1 << 24, 1 << 31])
def test_scratch_is_given_back(bits):
    """Growing inserts keep a record scratch (0.2 GB here), which
    release_scratch returns; the filter goes on as before."""
    from paper_2606_24417_amd import Filter

    d = dev(synth.background(100_000_000 if bits > 1 << 24 else 4_000_000, 97))
    f = Filter(31, 28, 16, 4, bits)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for n in (2_000_000, d.numel() // 2, d.numel()):
        f.insert(d[:n])
    torch.cuda.synchronize()
    kept = torch.cuda.mem_get_info()[0]
    want = f.get_bits()
    f.release_scratch()
    after = torch.cuda.mem_get_info()[0]
    print("free memory: %d, %d after inserts, %d after the release" % (before, kept, after), flush=True)
    if bits > 1 << 24:
        assert before - kept > 100 << 20
    assert before - after < 8 << 20
    f.clear()
    f.insert(d)
    assert np.array_equal(f.get_bits(), want)
    f.close()


@pytest.mark.parametrize("k,s,m", [(31, 28, 16), (21, 15, 11), (21, 15, 16), (32, 26, 17)])
def test_small_filters_hold_their_first_records(k, s, m):
    """A filter of 8 MiB has room for the records of 16 bits per k-mer from its
    creation on, whatever the window, and none where nothing is binned."""
    from paper_2606_24417_amd import Filter

    n = (1 << 22) + k - 1
    seq = synth.background(n, 98)
    d = dev(seq)

    def used(H, insert):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        fs = [Filter(k, s, m, H, 1 << 26) for _ in range(8)]
        created = before - torch.cuda.mem_get_info()[0]
        if insert:
            for f in fs:
                f.insert(d)
            torch.cuda.synchronize()
        inserted = before - torch.cuda.mem_get_info()[0]
        words = fs[0].get_bits()
        for f in fs:
            f.close()
        return created, inserted, words

    used(4, True)  # the library's own allocations of a first run
    created, inserted, words = used(4, True)
    print("8 filters: %.1f MiB created, %.1f after inserts" % (created / 2**20, inserted / 2**20), flush=True)
    assert inserted == created
    p = oracle.Params(k, s, m, 4, 1 << 26)
    assert np.array_equal(words, oracle.insert(p, p.empty(), seq))
    assert used(9, False)[0] <= 8 * (12 << 20)  # generic kernels: 8 MiB and a granule each
