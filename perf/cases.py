"""Workloads of the Super Bloom filter's insert and query path, sized as the
repository's own benchmark and tests use it.

A case is a plain dict:
  op     "build": clear the filter and insert a sequence set (an index is
         built), "add": insert a further batch into a filter in use, "query":
         ask for every k-mer of a batch;
  form   "contig": one sequence, "reads": 150 bp reads, "lognormal": reads of
         log-normal length (median 500 bp), "mixed": half 150 bp reads, half
         long reads of 10 to 20 kbp;
  where  "device": tensors on the GPU, "host": numpy arrays, copied both ways
         inside the call;
  k, s, m, H, words, bits   the filter (words 64-bit words per shard);
  bases  bases of the batch.

`add` and `query` run against a filter that holds a genome at 16 bits per
k-mer.  Sequence is synthetic with 41% GC, up to 5% diverged repeat copies, a
few runs of N and soft-masked (lower-case) stretches; half of a query batch's
reads come from the genome with 1% substitutions, half are random.
"""

import numpy as np
import torch

from paper_2606_24417_amd import Filter

DEV = "cuda"
PAPER = dict(k=31, s=28, m=16, H=4, words=4)


def listed():
    def case(name, op, form, bases, bits, where="device", **geometry):
        return dict(PAPER, **geometry, name=name, op=op, form=form, where=where, bases=bases, bits=bits)

    return [
        # one small request against a resident index: latency and launches
        case("query_64_reads", "query", "reads", 64 * 150, 1 << 31),
        # a sequencer's batch streamed into an index that is being extended
        case("add_2000_reads", "add", "lognormal", 1_500_007, 1 << 31),
        # a bacterial-size genome into its own small filter
        case("build_1mbp", "build", "contig", 1_000_003, 1 << 24),
        # the benchmark's in-cache pair: 100 Mbp genome, 2M x 150 bp reads
        case("build_100mbp", "build", "contig", 100_000_000, 1 << 31),
        case("query_2m_reads", "query", "reads", 300_000_000, 1 << 31),
        # the benchmark's out-of-cache pair: human-size genome, 8 GiB filter
        case("build_3gbp", "build", "contig", 3_000_000_000, 1 << 36),
        case("query_3gbp_mixed", "query", "mixed", 3_000_000_000, 1 << 36),
        # shards of one 128-byte line: the lower false-positive rate at equal memory
        case("build_100mbp_16_words", "build", "contig", 100_000_000, 1 << 31, words=16),
        case("query_2m_reads_16_words", "query", "reads", 300_000_000, 1 << 31, words=16),
        # the parameter study's lowest false-positive rate at k = 31
        case("build_100mbp_s26", "build", "contig", 100_000_000, 1 << 31, s=26),
        # a shorter k, as assemblers use it
        case("query_k21", "query", "lognormal", 150_000_001, 1 << 31, k=21, s=15, m=11, H=4),
        # reads in host memory, answers back in host memory
        case("query_host_200k_reads", "query", "reads", 30_000_000, 1 << 31, where="host"),
    ]


def draw(rng):
    def log_uniform(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    geometry = rng.choice([
        dict(), dict(), dict(), dict(),                                   # the paper's default
        dict(s=27), dict(s=31), dict(m=18), dict(H=8),                    # its neighbours in the parameter study
        dict(s=26), dict(s=25, m=14, H=3), dict(m=12), dict(k=21, s=15, m=11), dict(k=32, s=26, m=17, H=8),
    ])
    case = dict(PAPER, **geometry)
    case["words"] = rng.choice([4, 4, 4, 4, 8, 16])
    case["op"] = rng.choice(["build", "query", "query", "add"])
    case["form"] = rng.choice(["contig", "reads", "lognormal", "mixed"])
    case["where"] = rng.choice(["device"] * 7 + ["host"])
    top = 400_000_000 if case["where"] == "device" else 40_000_000
    case["bases"] = log_uniform(2_000, top) | 1
    if case["op"] == "build":
        need = 16 * case["bases"]
        case["bits"] = 1 << max(16, (need - 1).bit_length())
    else:
        case["bits"] = 1 << rng.randrange(24, 34)
    return case


# --- inputs -------------------------------------------------------------------

def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + salt)
    return g


def _background(n, gen):
    """n bases, A and T 76/256 each, C and G 52/256 each."""
    letters = torch.full((256,), ord("A"), dtype=torch.uint8, device=DEV)
    letters[76:128], letters[128:180], letters[180:] = ord("C"), ord("G"), ord("T")
    out = torch.empty(n, dtype=torch.uint8, device=DEV)
    for a in range(0, n, 1 << 26):
        b = min(n, a + (1 << 26))
        r = torch.randint(0, 256, (b - a,), dtype=torch.int32, device=DEV, generator=gen)
        out[a:b] = torch.index_select(letters, 0, r)
    return out


def _substitute(seq, gen):
    """Every hundredth base, at random, drawn again."""
    for a in range(0, seq.numel(), 1 << 26):
        part = seq[a:a + (1 << 26)]
        hit = torch.randint(0, 100, (part.numel(),), dtype=torch.uint8, device=DEV, generator=gen) == 0
        part.copy_(torch.where(hit, _background(part.numel(), gen), part))


_REPEAT = 6000


def _genome(n, seed, salt):
    gen = _gen(seed, salt)
    seq = _background(n, gen)
    rng = np.random.default_rng([seed, salt])
    # repeat families of 3..6 kbp, 10..50 diverged copies each, none overlapping
    places = rng.permutation(n // _REPEAT)[: min(n // _REPEAT // 20, 4_000)]
    used = 0
    while used < places.size:
        length, copies = int(rng.integers(_REPEAT // 2, _REPEAT + 1)), int(rng.integers(10, 51))
        at = torch.from_numpy(places[used:used + copies] * _REPEAT).to(DEV)
        rows = _background(length, gen).repeat(at.numel(), 1)
        _substitute(rows.view(-1), gen)
        seq[at[:, None] + torch.arange(length, device=DEV)[None, :]] = rows
        used += copies
    for _ in range(min(64, n // 20_000)):
        a = int(rng.integers(0, n - 400))
        seq[a:a + int(rng.integers(1, 400))] = ord("N")
        a = int(rng.integers(0, n - 400))
        seq[a:a + 300] |= 0x20
    return seq


def _lengths(case, rng):
    n, form = case["bases"], case["form"]
    if form == "contig":
        return np.array([n], dtype=np.int64)
    if form == "reads":
        lens = np.full(n // 150, 150, dtype=np.int64)
    elif form == "lognormal":
        lens = np.clip(np.round(np.exp(rng.normal(np.log(500.0), 1.0, n // 400 + 16))), 100, 50_000).astype(np.int64)
    else:
        lens = np.concatenate([np.full(n // 300, 150, dtype=np.int64), rng.integers(10_000, 20_001, n // 20_000)])
    end = np.cumsum(lens)
    lens = lens[: int(np.searchsorted(end, n, side="right"))]
    rest = n - int(lens.sum())
    return np.concatenate([lens, [rest]]) if rest else lens


def _batch(case, seed, genome):
    """(sequence, offsets or None) of the case's batch on the GPU.  With a
    genome, every second read is sampled from it with 1% substitutions."""
    n = case["bases"]
    if case["form"] == "contig" and genome is None:
        return _genome(n, seed, 1), None
    rng = np.random.default_rng([seed, 2])
    lens = torch.from_numpy(_lengths(case, rng)).to(DEV)
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(lens, 0)
    gen = _gen(seed, 3)
    if genome is None:
        return _genome(n, seed, 1), off
    seq = _background(n, gen)
    if case["form"] == "contig":  # the first half is a diverged piece of the genome
        half = min(n // 2, genome.numel())
        seq[:half] = genome[:half]
        _substitute(seq[:half], gen)
        return seq, None
    start = (torch.rand(lens.numel(), device=DEV, dtype=torch.float64, generator=gen)
             * (genome.numel() - lens).clamp(min=1)).to(torch.int64)
    per = max(1, (1 << 25) * lens.numel() // max(n, 1))
    for r in range(0, lens.numel(), per):
        e = min(lens.numel(), r + per)
        a, b = int(off[r]), int(off[e])
        rec = torch.repeat_interleave(torch.arange(r, e, device=DEV), lens[r:e], output_size=b - a)
        src = torch.arange(a, b, device=DEV) - off[rec] + start[rec]
        hit = (rec % 2 == 0) & (src < genome.numel())
        seq[a:b] = torch.where(hit, genome[src.clamp(max=genome.numel() - 1)], seq[a:b])
    _substitute(seq, gen)
    return seq, off


def _resident(case):
    """Bases of the genome that an `add` or `query` filter holds."""
    return max(64, min(case["bits"] // 16, 3_000_000_000))


def _inputs(case, seed):
    genome = _genome(_resident(case), seed, 0) if case["op"] != "build" else None
    seq, off = _batch(case, seed, genome if case["op"] == "query" else None)
    return genome, seq, off


class _Words:
    """The filter's own bit array, for torch (the filter lives as long as a view)."""

    def __init__(self, f):
        self.filter = f
        self.__cuda_array_interface__ = dict(shape=(f.num_words,), typestr="<i8", version=2,
                                             data=(f.device_words_ptr, False))


def prepare(case, seed):
    f = Filter(case["k"], case["s"], case["m"], case["H"], case["bits"], case["words"])
    genome, seq, off = _inputs(case, seed)
    if genome is not None:
        f.insert(genome)
    if case["where"] == "host":
        seq = seq.cpu().numpy()
        off = off.cpu().numpy().view(np.uint64) if off is not None else None
    return dict(op=case["op"], filter=f, words=torch.as_tensor(_Words(f), device=DEV), seq=seq, off=off)


def run(state):
    f = state["filter"]
    if state["op"] == "query":
        return f.query(state["seq"], state["off"])
    if state["op"] == "build":
        f.clear()
    f.insert(state["seq"], state["off"])
    return state["words"]


# --- what a pass cannot do without ----------------------------------------------

def work(case):
    """Bytes: the batch, its answers, and each shard that a super-k-mer of the
    batch needs (mean length (w+1)/2 k-mers), read for a query, read and
    written for an insert, at most the whole filter.  Operations: the integer
    operations per k-mer of the rolling formulation."""
    k, s, m, H, words = (case[x] for x in ("k", "s", "m", "H", "words"))
    n, filter_bytes = case["bases"], case["bits"] // 8
    mean = dict(contig=n, reads=150, lognormal=800, mixed=297)[case["form"]]
    kmers = max(1.0, n - (k - 1) * n / max(mean, k))
    shards = min(filter_bytes, 8 * words * (kmers * 2 / (k - m + 2)))
    shared = 16 + 10 + H  # encode, m-mer hash, sliding minimum, shard; s-mer hash, bit addresses
    if case["op"] == "query":
        return dict(bytes=2 * n + shards, flops=kmers * (shared + 2 * H * (k - s + 1) + 1))
    cleared = filter_bytes if case["op"] == "build" else 0
    return dict(bytes=n + 2 * shards + cleared, flops=kmers * (shared + 16))


# --- the same in plain torch ---------------------------------------------------

def _i64(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _shr(x, n):
    return x if n == 0 else (x >> n) & ((1 << (64 - n)) - 1)


def _bits_of(case, seq, off, a, b):
    """k-mers a .. b-1 of the batch: validity and, per s-mer and hash index,
    the bit number in the filter."""
    k, s, m, H, words = (case[x] for x in ("k", "s", "m", "H", "words"))
    end = min(seq.numel(), b + k - 1)
    part = seq[a:end].to(torch.int64)
    pad = b + k - 1 - end
    if pad:
        part = torch.cat([part, torch.zeros(pad, dtype=torch.int64, device=DEV)])
    low = part | 0x20
    code = ((low == 0x63) * 1 + (low == 0x67) * 2 + (low == 0x74) * 3).to(torch.int64)
    bad = ((low != 0x61) & (code == 0)).to(torch.int64)
    gone = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(bad, 0)])
    valid = gone[k:] == gone[:-k]
    if off is not None:
        first = torch.zeros(part.numel(), dtype=torch.int64, device=DEV)
        inside = off[:-1]
        inside = inside[(inside > a) & (inside < a + part.numel())]
        first[inside - a] = 1
        rec = torch.cumsum(first, 0)
        valid &= rec[k - 1:] == rec[: rec.numel() - k + 1]

    def window(length):
        out = torch.zeros(part.numel() - length + 1, dtype=torch.int64, device=DEV)
        for i in range(length):
            out = (out << 2) | code[i: i + out.numel()]
        return out

    top = -(1 << 63)
    h = (window(m) * _i64(0x9E3779B97F4A7C15)) ^ top  # signed order of the flipped hash = unsigned order
    w, have = k - m + 1, 1
    while have < w:
        step = min(have, w - have)
        h = torch.minimum(h[: h.numel() - step], h[step:])
        have += step
    nshards = 1
    while nshards * 64 * words < case["bits"]:
        nshards *= 2
    shard = (h[: b - a] ^ top) & (nshards - 1)
    g = window(s)
    g = g ^ _shr(g, 30)
    g = g * _i64(0xBF58476D1CE4E5B9)
    g = g ^ _shr(g, 31)
    width = 64 // H
    for t in range(H):
        in_shard = (_shr(g, t * width) & 63) + 64 * (t % 4)
        if words > 4:
            in_shard = in_shard + 256 * (_shr(g, t * width + 6) & (words // 4 - 1))
        for j in range(k - s + 1):
            yield valid, shard * (64 * words) + in_shard[j: j + b - a]


_CHUNK = 1 << 24


def _exact_insert(case, filt, seq, off):
    n = seq.numel() - case["k"] + 1
    for a in range(0, n, _CHUNK):
        for valid, at in _bits_of(case, seq, off, a, min(n, a + _CHUNK)):
            filt[at[valid]] = True


def exact(case, seed):
    # one byte per filter bit on the GPU: up to 2^33 bits
    if case["bits"] > 1 << 33 or case["bases"] > 400_000_000:
        return None
    nshards = 1
    while nshards * 64 * case["words"] < case["bits"]:
        nshards *= 2
    filt = torch.zeros(nshards * 64 * case["words"], dtype=torch.bool, device=DEV)
    genome, seq, off = _inputs(case, seed)
    if genome is not None:
        _exact_insert(case, filt, genome, None)
    if case["op"] != "query":
        _exact_insert(case, filt, seq, off)
        bits = filt.view(-1, 64)
        words = torch.zeros(bits.shape[0], dtype=torch.int64, device=DEV)
        for i in range(64):
            words |= bits[:, i].to(torch.int64) << i
        return words
    n = seq.numel() if off is not None else max(0, seq.numel() - case["k"] + 1)
    out = torch.zeros(n, dtype=torch.uint8, device=DEV)
    for a in range(0, n, _CHUNK):
        b = min(n, a + _CHUNK)
        hit = None
        for valid, at in _bits_of(case, seq, off, a, b):
            found = filt[at]
            hit = valid & found if hit is None else hit & found
        out[a:b] = hit.to(torch.uint8)
    return out if case["where"] == "device" else out.cpu().numpy()
