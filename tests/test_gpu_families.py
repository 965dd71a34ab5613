"""The kernels that a setting names are the ones that run: an explicit
wide-shard or run-time parameter family keeps every batch on its own kernels.
And those kernels, and the lane kernels by their tile or where the batch's size
selects them, give the oracle's filter and answers."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_24417_amd.sbf import (VARIANT_AUTO, VARIANT_GENERIC, VARIANT_PARAM, VARIANT_ROLLING, VARIANT_WIDE,  # noqa: E402
                                      Filter)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(x):
    return torch.from_numpy(np.array(x, copy=True)).cuda()


def doff(off):
    return dev(np.asarray(off, dtype=np.uint64).view(np.int64))


@pytest.mark.parametrize("S", [4, 16])
@pytest.mark.parametrize("variant,own", [(VARIANT_AUTO, False), (VARIANT_ROLLING, False), (VARIANT_WIDE, True),
                                         (VARIANT_PARAM, True)])
def test_explicit_families_do_not_bin(variant, own, S):
    """A binned insert of 50 Mbp keeps more than 200 MB of records."""
    d = dev(synth.background(50_000_000, 3))
    f = Filter(31, 28, 16, 4, 1 << 31, shard_words=S)
    f.variant = variant
    f.insert(d[:1000])
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    f.insert(d)
    torch.cuda.synchronize()
    kept = before - torch.cuda.mem_get_info()[0]
    f.close()
    assert (kept < 100 << 20) if own else (kept > 200 << 20)


# The lane kernels where no setting replaces them, and by a given tile, against
# the oracle: the batches have more tiles than the persistent grids have
# workgroups (1 or 4 per CU), so that workgroups take several tiles.
def against_oracle(params, S, ins, query, mode=0, tile=(0, 0), launch=None, variant=VARIANT_AUTO, qmode=0):
    p = oracle.Params(*params, shard_words=S)
    F = oracle.insert(p, p.empty(), *ins)
    want = oracle.query(p, F, *query)
    f = Filter(*params, shard_words=S)
    f.variant = variant
    f.set_insert_mode(mode)
    f.set_query_mode(qmode)
    f.set_tile(*tile)
    if launch is not None:
        f.set_launch(launch, launch)
    f.insert(dev(ins[0]), doff(ins[1]))
    torch.cuda.synchronize()
    words = f.get_bits()
    out = f.query(dev(query[0]), doff(query[1])).cpu().numpy()
    f.close()
    bad = np.flatnonzero(words != F)
    assert bad.size == 0, "%d of %d words differ, first %s" % (bad.size, words.size, bad[:5].tolist())
    bad = np.flatnonzero(out != want)
    assert bad.size == 0, "%d of %d answers differ, first %s" % (bad.size, out.size, bad[:5].tolist())
    return want


def noisy_records(n, mean, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 2 * mean, size=max(1, n // mean))
    off = np.concatenate(([0], np.cumsum(lens))).astype(np.uint64)
    seq = synth.uniform_acgt(int(off[-1]), seed).copy()
    bad = rng.random(seq.size) < 0.001
    seq[bad] = rng.choice(np.frombuffer(b"NnX-.", dtype=np.uint8), bad.sum())
    return seq, off


@pytest.mark.parametrize("tile,launch", [((32, 32), 4), ((64, 48), 1)])
def test_lane_kernels_on_persistent_grids(tile, launch):
    """The insert's store pass and repair and the lane query, by their tiles."""
    print("case lane persistent", tile, launch, flush=True)
    w = synth.in_cache_workload(scale=0.1)
    against_oracle((31, 28, 16, 4, w["bits"]), 4, w["insert"], w["query"], tile=tile, launch=launch)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("S", [4, 16])
def test_wide_kernels_on_persistent_grids(S, mode):
    print("case wide persistent", S, mode, flush=True)
    w = synth.in_cache_workload(scale=0.04)
    against_oracle((31, 28, 16, 4, w["bits"]), S, w["insert"], w["query"], mode=mode, launch=1, variant=VARIANT_WIDE)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("S", [4, 16])
def test_param_kernels_on_persistent_grids(S, mode):
    print("case param persistent", S, mode, flush=True)
    w = synth.in_cache_workload(scale=0.03)
    against_oracle((31, 26, 15, 5, w["bits"]), S, w["insert"], w["query"], mode=mode, launch=1, variant=VARIANT_PARAM)


# 4.2M to 12.6M k-mers are the lane query's at every compiled set; the insert
# is small for its filter and takes the two passes.
@pytest.mark.parametrize("k,s,m,H", [(31, 28, 16, 4), (31, 27, 16, 4), (31, 30, 16, 4), (31, 31, 16, 4),
                                     (31, 28, 18, 4), (31, 28, 16, 8)])
def test_lane_query_between_the_run_query_sizes(k, s, m, H):
    print("case lane query", k, s, m, H, flush=True)
    ins = noisy_records(1_200_000, 3000, k + s + m + H)
    q = noisy_records(4_000_000, 500, s + H)
    qs = np.concatenate([ins[0], q[0]])
    qo = np.concatenate([ins[1], q[1][1:] + ins[1][-1]])
    want = against_oracle((k, s, m, H, 1 << 28), 4, ins, (qs, qo))
    assert 4 * 256 * 4096 < qs.size <= 4 * 256 * 12288
    assert want.sum() > 1_000_000


@pytest.mark.parametrize("n", [30, 31, 77, 78, 79, 12317, 12318, 12319, 24605, 24606, 24607, 50_000])
@pytest.mark.parametrize("query_lane", [32, 48])
def test_lane_lengths_around_tiles(query_lane, n):
    print("case lane length", query_lane, n, flush=True)
    seq, off = synth.uniform_acgt(n, n), np.array([0, n], dtype=np.uint64)
    against_oracle((31, 28, 16, 4, 1 << 14), 4, (seq, off), (seq, off), tile=(32, query_lane))


# One invalid base in every fourth lane and one record start in every fourth
# (another phase), at the bases that decide validity where a lane's two 64-base
# windows meet and where lanes of 32 or 48 k-mers end.
@pytest.mark.parametrize("lane", [32, 48])
def test_lane_validity_at_window_seams(lane):
    print("case lane seams", lane, flush=True)
    at = [1, 30, 31, 32, 33, 47, 48, 61, 62, 63, 64, 77, 78]
    n = lane * 1600
    seq = synth.uniform_acgt(n, lane).copy()
    lanes = n // lane - 2
    for j, i in enumerate(range(0, lanes, 4)):
        seq[i * lane + at[j % len(at)]] = ord("N")
    starts = sorted({i * lane + at[j % len(at)] for j, i in enumerate(range(2, lanes, 4))})
    off = np.array([0] + starts + [n], dtype=np.uint64)
    want = against_oracle((31, 28, 16, 4, 1 << 23), 4, (seq, off), (seq, off), tile=(32, lane))
    assert want.sum() > n // 2


# The generic query on a batch that fills the GPU many times over, three times,
# against the default kernels (which the full-size tests compare with the
# oracle), and the filter that the generic insert builds.
@pytest.mark.parametrize("S", [4, 8, 16])
@pytest.mark.parametrize("k,s,m,H", [(31, 28, 16, 4), (21, 15, 11, 8)])
def test_generic_kernels_on_large_batches(k, s, m, H, S):
    print("case generic large", k, s, m, H, S, flush=True)
    w = synth.in_cache_workload(scale=0.1)
    d, o = dev(w["insert"][0]), doff(w["insert"][1])
    q, qo = dev(w["query"][0]), doff(w["query"][1])
    f, g = Filter(k, s, m, H, w["bits"], shard_words=S), Filter(k, s, m, H, w["bits"], shard_words=S)
    g.variant = VARIANT_GENERIC
    f.insert(d, o)
    g.insert(d, o)
    assert np.array_equal(f.get_bits(), g.get_bits())
    for off in (qo, None):
        want = f.query(q, off)
        for _ in range(3):
            assert torch.equal(g.query(q, off), want)
    f.close()
    g.close()
