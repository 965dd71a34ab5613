"""Plan of the binned insert (host code of the library, no GPU): the records
that its buckets and slices have room for against the records of random
sequence, counted with numpy."""

import ctypes

import numpy as np
import pytest

from paper_2606_24417_amd import lib


class Geometry(ctypes.Structure):
    _fields_ = [("k", ctypes.c_uint32), ("s", ctypes.c_uint32), ("m", ctypes.c_uint32), ("H", ctypes.c_uint32),
                ("shard_words", ctypes.c_uint32), ("nshards", ctypes.c_uint64)]


class BinPlan(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_int) for n in ("slice_words_log2", "slice_shift", "bits1", "bits2")] +
                [("parts", ctypes.c_uint32), ("group", ctypes.c_uint32)] +
                [(n, ctypes.c_uint64) for n in ("chunk", "cap1", "cap2", "counts1", "counts2", "rec1", "rec2",
                                                "count_words", "bytes")])


def plan(k, s, m, H, bits, S, length, lane_family=False):
    """The library's plan for an insert of `length` bases, or None."""
    fn = lib()["_ZN3sbf11binned_planERKNS_8GeometryEmbRNS_7BinPlanE"]
    fn.restype = ctypes.c_bool
    fn.argtypes = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_bool, ctypes.c_void_p]
    g, p = Geometry(k, s, m, H, S, bits // (64 * S)), BinPlan()
    return p if fn(ctypes.byref(g), length, lane_family, ctypes.byref(p)) else None


def records_per_kmer(w, nmax, n=400_000):
    """Runs of one window minimum in n windows of random ranks, cut after nmax."""
    rank = np.random.default_rng(w).permutation(n + w - 1)
    low = np.lib.stride_tricks.sliding_window_view(rank, w).min(axis=1)
    start = np.flatnonzero(np.concatenate(([True], low[1:] != low[:-1])))
    length = np.diff(np.concatenate((start, [n])))
    return np.sum((length + nmax - 1) // nmax) / n


# Room is 1.12 times the expected records; the count above has a standard
# error below 0.5%, and a tile's end adds less than 0.1%.
@pytest.mark.parametrize("k,m", [(31, 16), (21, 16), (21, 11), (31, 18), (32, 17), (31, 15), (31, 14), (31, 12),
                                 (31, 8), (32, 16), (32, 8), (32, 1)])
@pytest.mark.parametrize("bits,S", [(1 << 24, 4), (1 << 31, 4), (1 << 31, 16), (1 << 36, 8)])
def test_buckets_hold_the_records_of_random_sequence(bits, S, k, m):
    length = bits // 16
    p = plan(k, 20, m, 4, bits, S, length)
    want = records_per_kmer(k - m + 1, min(16, 47 - k)) * min(p.chunk, length - k + 1)
    room = p.cap1 * p.parts << p.bits1
    assert room > 1.1 * want, "room for %d records of %d" % (room, want)
    if p.bits2:
        assert p.cap2 << (p.bits1 + p.bits2) > 1.3 * want


# The scratch that the header promises: at most 1 GiB plus 1.2 times the filter's
# size at k-m = 15, 1.7 times at k-m = 10, 2.75 times at any, whatever the batch.
@pytest.mark.parametrize("S", [4, 16])
@pytest.mark.parametrize("log2_bits", range(24, 39))
def test_scratch_stays_within_its_bound(log2_bits, S):
    bits = 1 << log2_bits
    planned = 0
    for k, m in [(31, 16), (32, 17), (31, 18), (31, 12), (21, 11), (21, 12), (21, 14), (21, 16), (13, 4), (32, 1)]:
        times = {16: 1.2, 11: 1.7}.get(k - m + 1 if k < 32 else 0, 2.75)
        for length in (bits // 100, bits // 32, bits // 16, bits // 15, bits // 8, bits, 1 << 40):
            p = plan(k, min(20, k), m, 4, bits, S, length)
            if p is None:
                continue
            planned += 1
            assert p.bytes <= times * bits / 8 + (1 << 30), (k, m, length)
            assert p.rec2 <= p.bytes and p.chunk % 16384 == 0
            # equal parts, smaller than the batch only by whole tiles
            nk = length - k + 1
            parts = -(-nk // p.chunk)
            assert 0 <= p.chunk * parts - nk < 16384 * (parts + 1)
    assert planned >= 20


# The launches that the benchmark states for its two workloads: 100 Mbp into 2^31
# bits and 3 Gbp into 2^36, in one part.
@pytest.mark.parametrize("name,bits,length", [("in_cache", 1 << 31, 100_000_000), ("out_of_cache", 1 << 36, 3_000_000_000)])
@pytest.mark.parametrize("S", [4, 8, 16])
def test_launches_of_the_benchmark(S, name, bits, length):
    import bench

    p = plan(31, 28, 16, 4, bits, S, length, lane_family=S == 4)
    assert p.chunk >= length - 30 and p.bits2 > 0
    assert 2 + 2 * ((1 << p.bits1) // p.group) == bench.BINNED_LAUNCHES[name]
