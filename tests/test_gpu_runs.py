"""GPU parity of the run query kernels (one lane per super-k-mer, runs in order
of length) against the oracle, every answer: all shard sizes, front ends with
m = 16, below and above, windows of 6 to 32 m-mers, s-mer counts past 32 per
run, tiles with more runs than their list holds, lengths around the tile of
8192 k-mers, unaligned buffers, invalid bases and short records.
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


def records(n, mean, seed, p_invalid=0.001):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 2 * mean, size=max(1, n // mean))
    lens[::5] = rng.integers(0, 40, size=lens[::5].size)
    off = np.concatenate(([0], np.cumsum(lens))).astype(np.uint64)
    seq = synth.uniform_acgt(int(off[-1]), seed).copy()
    bad = rng.random(seq.size) < p_invalid
    seq[bad] = rng.choice(np.frombuffer(b"NnX-.", dtype=np.uint8), bad.sum())
    return seq, off


def check(params, S, ins, seq, off, shift=0):
    from paper_2606_24417_amd import Filter

    k, s, m, H, bits = params
    p = oracle.Params(k, s, m, H, bits, shard_words=S)
    F = oracle.insert(p, p.empty(), ins)
    want = oracle.query(p, F, seq, off)
    f = Filter(k, s, m, H, bits, shard_words=S)
    f.set_bits(F)
    d = dev(np.concatenate([seq[:1]] * shift + [seq]))[shift:]
    out = torch.full((want.size + 64,), 7, dtype=torch.uint8, device="cuda")
    f.query(d, doff(off) if off is not None else None, out=out[shift:])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    f.close()
    bad = np.flatnonzero(got[shift:shift + want.size] != want)
    assert bad.size == 0, "%d of %d answers differ, first %s" % (bad.size, want.size, bad[:5].tolist())
    assert (got[:shift] == 7).all() and (got[shift + want.size:] == 7).all(), "bytes outside the answers written"
    return want


@pytest.mark.parametrize("S", [4, 8, 16])
@pytest.mark.parametrize("k,s,m,H", [(31, 28, 16, 4), (31, 27, 16, 8), (31, 28, 18, 4), (31, 26, 12, 5), (21, 15, 11, 4),
                                     (32, 26, 17, 7), (21, 15, 16, 2), (32, 12, 1, 4), (24, 1, 19, 3), (32, 32, 16, 1),
                                     (13, 9, 4, 4)])
def test_parameters_match_oracle(k, s, m, H, S):
    print("case runs k=%d s=%d m=%d H=%d S=%d" % (k, s, m, H, S), flush=True)
    ins = synth.uniform_acgt(60_000, 7 * k + m)
    seq, off = records(90_000, 300, k + 100 * m + S)
    # every third stretch of the batch is inserted sequence
    at = np.arange(0, seq.size - 700, 2100)
    for a in at:
        b = a % (ins.size - 700)
        seq[a:a + 700] = ins[b:b + 700]
    want = check((k, s, m, H, 1 << 18), S, ins, seq, off)
    assert want.sum() > 0


@pytest.mark.parametrize("S", [4, 16])
@pytest.mark.parametrize("n", [31, 32, 62, 8192 + 30, 8192 + 31, 2 * 8192 + 30, 2 * 8192 + 63, 3 * 8192 + 4000])
def test_lengths_and_alignment(n, S):
    print("case runs length", n, S, flush=True)
    seq = synth.uniform_acgt(n, n)
    for shift in (0, 1, 8):
        want = check((31, 28, 16, 4, 1 << 16), S, seq, seq, None, shift)
        assert want.all()


# homopolymers and repeats (runs cut at 16 k-mers across lanes and tiles)
@pytest.mark.parametrize("S", [4, 8])
@pytest.mark.parametrize("period", [1, 2, 3, 7, 17, 40])
def test_repeats(period, S):
    print("case runs period", period, S, flush=True)
    seq = synth.uniform_acgt(40_000, 50 + period).copy()
    seq[5_000:] = np.resize(seq[:period], 35_000)
    seq[20_000:20_003] = ord("N")
    check((31, 28, 16, 4, 1 << 18), S, seq[:12_000], seq, None)
    check((31, 28, 12, 4, 1 << 18), S, seq[:12_000], seq, None)
