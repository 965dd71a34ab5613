// Front end of the run kernels (kernels_binned.hip, query_runs.h): a workgroup
// stages a tile of WG x 32 k-mers, computes every k-mer's shard and finds the
// runs of consecutive valid k-mers with one shard (super-k-mers), cut to at most
// nmax k-mers.  Lane t owns k-mers 32t .. 32t+31; the sliding
// minimum over its m-mer hashes is a van Herk / Gil-Werman minimum held in
// registers (w = k-m+1 is a compile-time constant, k and m are not).
#pragma once

#include "sbf_device.h"
#include "sbf_tiles.h"

namespace sbf {
namespace {

constexpr int kRunL = 32;  // k-mers per lane

// LDS of a tile.
template <int WG, int LCAP>
struct RunTile {
  // the last lane's bases: 32 + k - 1 <= 63, and one granule for the funnel
  // shift of the last window
  static constexpr int NGRAN = (WG - 1) * 2 + 5;
  static constexpr int TILE = WG * kRunL;
  uint32_t codes[NGRAN];
  // validity bits of the staged bases, then the list of run starts
  union {
    uint32_t vb[NGRAN];
    uint16_t list[LCAP];
  };
  // low 32 bits of each k-mer's minimizer hash, whose low bits are its shard
  alignas(16) uint32_t shard[kRunL][WG];
  uint32_t change[WG];
  uint32_t stop[WG + 1];  // validity, then run starts and invalid k-mers
  uint32_t wsum[WG / 64];
};

// Run-time parameters of the front end.
struct RunGeo {
  int k;
  int m_shift;  // 32 - 2m for m <= 16, 64 - 2m above
  int nmax;     // k-mers per run, at most 16
  uint32_t shard_mask;
};

// Bit r: bits r .. r+n-1 of x are all set (n >= 1, uniform).
__device__ __forceinline__ uint64_t window_and_rt(uint64_t x, int n) {
  for (int have = 1; have < n;) {
    const int d = have < n - have ? have : n - have;
    x &= x >> d;
    have += d;
  }
  return x;
}

// Validity of the lane's 32 k-mers: the 64 bases from granule g0 cover them
// for k <= 32.
__device__ __forceinline__ uint32_t kmer_valid32(const uint32_t *s_vb, int g0, int k) {
  uint64_t vbits = 0, sbits = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t vb = s_vb[g0 + i];
    vbits |= (uint64_t)(vb & 0xFFFFu) << (16 * i);
    sbits |= (uint64_t)(vb >> 16) << (16 * i);
  }
  uint64_t kv = window_and_rt(vbits, k);
  // no record starts at r+1 .. r+k-1
  if (k > 1 && sbits >> 1) kv &= window_and_rt(~(sbits >> 1), k - 1);
  return (uint32_t)kv;
}

// Hash of the m-mer at window position j.  MK 0: m = 16; 1: m < 16; 2: m > 16.
template <int MK>
__device__ __forceinline__ uint64_t run_mmer_hash(const uint32_t *a, int j, int m_shift) {
  if constexpr (MK == 0) return minimizer_hash32_split(win32(a, j));
  if constexpr (MK == 1) return minimizer_hash32_split(win32(a, j) >> m_shift);
  return minimizer_hash((((uint64_t)win32(a, j) << 32) | win32(a, j + 16)) >> m_shift);
}

// Sixteen ASCII bases -> 32 bits of codes (first base in bits 31:30) and their
// valid bits: four encode4 at once, whose validity multiplies are left out for
// a granule of valid bases.
__device__ __forceinline__ void encode16(u32x4 v, uint32_t &code, uint32_t &valid) {
  uint32_t c[4], diff[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t x = v[w];
    const uint32_t c4 = ((x >> 1) ^ (x >> 2)) & 0x03030303u;
    diff[w] = (x | 0x20202020u) ^ __builtin_amdgcn_perm(0u, 0x74676361u, c4);  // letters by code
    c[w] = c4 * 0x40100401u;  // the word's 8 bits of codes in the top byte
  }
  const uint32_t c01 = __builtin_amdgcn_perm(c[0], c[1], 0x0C0C0703u);
  const uint32_t c23 = __builtin_amdgcn_perm(c[2], c[3], 0x0C0C0703u);
  code = (c01 << 16) | c23;
  valid = 0xFFFFu;
  if (diff[0] | diff[1] | diff[2] | diff[3]) {
    valid = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      uint32_t c8, v4;
      encode4(v[w], c8, v4);
      valid |= v4 << (4 * w);
    }
  }
}

// stage_granules for a run tile: inside an aligned sequence a lane loads all
// its granules before it encodes the first, and so waits for memory once.
template <int WG, int NGRAN>
__device__ __forceinline__ void stage_tile(const uint8_t *__restrict__ seq, uint64_t len, uint64_t base,
                                           const uint32_t *__restrict__ starts, bool aligned16,
                                           uint32_t *__restrict__ s_codes, uint32_t *__restrict__ s_vb) {
  constexpr int N = (NGRAN + WG - 1) / WG;
  if (!aligned16 || base + 16ull * NGRAN > len) {
    stage_granules<WG>(seq, len, base, starts, aligned16, NGRAN, s_codes, s_vb);
    return;
  }
  u32x4 v[N];
  uint32_t rs[N];
  const u32x4 *src = reinterpret_cast<const u32x4 *>(seq + base);
  // (a lane past the last granule loads that one again)
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int g = i * WG + (int)threadIdx.x;
    v[i] = __builtin_nontemporal_load(src + (g < NGRAN ? g : NGRAN - 1));
    rs[i] = 0;
  }
  if (starts != nullptr) {
    const uint32_t *sw = starts + (base >> 5);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int g = i * WG + (int)threadIdx.x;
      rs[i] = (sw[(g < NGRAN ? g : NGRAN - 1) >> 1] >> ((uint32_t)(g & 1) * 16u)) & 0xFFFFu;
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int g = i * WG + (int)threadIdx.x;
    if ((i + 1) * WG <= NGRAN || g < NGRAN) {
      uint32_t code, valid;
      encode16(v[i], code, valid);
      s_codes[g] = code;
      s_vb[g] = valid | (rs[i] << 16);
    }
  }
}

// Stage the tile from `base` on and find its runs: head has a bit per k-mer of
// the lane that starts a run, first is the number of runs in the lanes before,
// total that of the tile.  T.shard and T.stop are complete after the caller's
// next barrier.
template <int W, int MK, int WG, int LCAP>
__device__ __forceinline__ void find_runs(RunTile<WG, LCAP> &T, const uint8_t *__restrict__ seq, uint64_t len,
                                          uint64_t base, const uint32_t *__restrict__ starts, bool aligned16,
                                          const RunGeo &P, uint32_t &head, uint32_t &first, uint32_t &total) {
  constexpr int L = kRunL;
  const int t = threadIdx.x;
  stage_tile<WG, RunTile<WG, LCAP>::NGRAN>(seq, len, base, starts, aligned16, T.codes, T.vb);
  __syncthreads();

  const int g0 = t * 2;
  uint32_t change = 0;  // bit r: k-mer r's hash differs from k-mer r-1's
  const uint32_t kv = kmer_valid32(T.vb, g0, P.k);
  {
    uint32_t a[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) a[i] = T.codes[g0 + i];
    uint64_t suf[W];
    {
      uint64_t m = run_mmer_hash<MK>(a, W - 1, P.m_shift);
      suf[W - 1] = m;
#pragma unroll
      for (int i = W - 2; i >= 0; --i) {
        m = umin64(run_mmer_hash<MK>(a, i, P.m_shift), m);
        suf[i] = m;
      }
    }
    uint32_t prev = 0;
#pragma unroll
    for (int q = 0; q * W < L; ++q) {
      uint64_t pre = ~0ull;
#pragma unroll
      for (int i = 0; i < W; ++i) {
        const int r = q * W + i;
        if (r < L) {
          uint64_t mu = suf[i];
          if (i > 0) {
            const uint64_t h = run_mmer_hash<MK>(a, r + W - 1, P.m_shift);
            pre = umin64(pre, h);
            mu = umin64(mu, pre);
            suf[i - 1] = h;
          }
          const uint32_t sh = (uint32_t)mu;
          T.shard[r][t] = sh;
          // change = 2 change + (sh != prev)
          asm("v_cmp_ne_u32_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
              : "+v"(change)
              : "v"(sh), "v"(prev)
              : "vcc");
          prev = sh;
        }
      }
      if ((q + 1) * W < L) {
        uint64_t m = run_mmer_hash<MK>(a, (q + 1) * W + W - 1, P.m_shift);
        suf[W - 1] = m;
#pragma unroll
        for (int i = W - 2; i >= 0; --i) {
          m = umin64(suf[i], m);
          suf[i] = m;
        }
      }
    }
    change = __builtin_bitreverse32(change);
  }
  T.change[t] = change;
  T.stop[t] = kv;
  if (t == 0) T.stop[WG] = ~0u;
  __syncthreads();

  // Record starts among the lane's k-mers: a valid k-mer after an invalid one
  // or in another shard than the one before; runs of more than nmax k-mers
  // are cut.
  {
    const uint32_t pkv = t > 0 ? T.stop[t - 1] : 0u;
    const uint32_t pch = t > 0 ? T.change[t - 1] : 0u;
    const bool same = t > 0 && (pkv >> 31) && T.shard[L - 1][t > 0 ? t - 1 : 0] == T.shard[0][t];
    uint32_t fresh = (change & ~1u) | (same ? 0u : 1u);
    head = kv & (fresh | ~(kv << 1 | (same ? 1u : 0u)));
    if (same && (kv & 1u)) {
      // continues the previous lane's last run, of `tail` k-mers there (its
      // start is not in that lane: taken as too long)
      const uint32_t phead = pkv & ~1u & (pch | ~(pkv << 1));
      int tail = phead ? __clz((int)phead) + 1 : 64;
      while (tail > P.nmax && tail <= 32) tail -= P.nmax;
      const uint32_t stop = head | ~kv;
      const int lead = stop ? __ffs((int)stop) - 1 : 32;
      if (tail + lead > P.nmax) head |= 1u;
    }
    for (;;) {
      // k-mers whose nmax-1 predecessors and themselves continue a run: the
      // lowest is the run's k-mer number nmax
      uint32_t c = kv & ~head;
      for (int have = 1; have < P.nmax;) {
        const int d = have < P.nmax - have ? have : P.nmax - have;
        c &= c << d;
        have += d;
      }
      if (c == 0) break;
      head |= c & (0u - c);
    }
  }
  // positions of the lane's records in the tile's list
  const int lane = t & 63, wave = t >> 6;
  const uint32_t mine = (uint32_t)__popc(head);
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) T.wsum[wave] = incl;
  __syncthreads();
  T.stop[t] = head | ~kv;
  first = incl - mine;
  total = 0;
#pragma unroll
  for (int w = 0; w < WG / 64; ++w) {
    if (w < wave) first += T.wsum[w];
    total += T.wsum[w];
  }
}

// List the tile positions of runs number done .. done + LCAP - 1.
template <int WG, int LCAP>
__device__ __forceinline__ void list_runs(RunTile<WG, LCAP> &T, uint32_t head, uint32_t first, uint32_t done) {
  uint32_t at = first - done;
  while (head) {
    const int r = __ffs((int)head) - 1;
    if (at < (uint32_t)LCAP) T.list[at] = (uint16_t)(threadIdx.x * kRunL + r);
    ++at;
    head &= head - 1;
  }
}

// k-mers minus one (below 16) of the run from tile position q on.
template <int WG, int LCAP>
__device__ __forceinline__ uint32_t run_length1(const RunTile<WG, LCAP> &T, int q) {
  const uint64_t stop = (((uint64_t)T.stop[q / kRunL + 1] << 32) | T.stop[q / kRunL]) >> ((q & (kRunL - 1)) + 1);
  return (uint32_t)__ffs((int)(uint32_t)stop) - 1u;
}

// 48 bases from tile position q on, first base most significant.
template <int WG, int LCAP>
__device__ __forceinline__ void run_bases(const RunTile<WG, LCAP> &T, int q, uint32_t &x, uint32_t &y, uint32_t &z) {
  const uint32_t *a = T.codes + (q >> 4);
  const int off = (q & 15) * 2;
  x = (uint32_t)(((((uint64_t)a[0] << 32) | a[1]) << off) >> 32);
  y = (uint32_t)(((((uint64_t)a[1] << 32) | a[2]) << off) >> 32);
  z = (uint32_t)(((((uint64_t)a[2] << 32) | a[3]) << off) >> 32);
}

// s-mer bits of a launch.
struct BitGeo {
  int z;        // k - s
  int s_shift;  // 64 - 2s
  int H;
  int slice;    // 64 / H
  int sw_log2;  // log2 of the words per shard
};

// h_S of the s-mer at the top of (x, y); S > 0: s is known.
template <int S>
__device__ __forceinline__ uint64_t top_smer_hash(uint32_t x, uint32_t y, const BitGeo &B) {
  if constexpr (S > 16 && S < 32) {
    // below 2^62, v >> 30 has no high word
    const uint32_t hi = x >> (64 - 2 * S);
    uint32_t lo = __builtin_amdgcn_alignbit(x, y, 64 - 2 * S);
    lo ^= __builtin_amdgcn_alignbit(hi, lo, 30);
    const uint64_t v = (((uint64_t)hi << 32) | lo) * kSmerMul;
    return v ^ (v >> 31);
  } else {
    return smer_hash((((uint64_t)x << 32) | y) >> B.s_shift);
  }
}

// v[0 .. 15] in LDS: each becomes the sum of those before it (first wave).
__device__ __forceinline__ void scan16(uint32_t *v) {
  if (threadIdx.x < 64) {
    const uint32_t own = v[threadIdx.x & 15u];
    uint32_t incl = own;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 16);
      if ((threadIdx.x & 15u) >= (uint32_t)d) incl += o;
    }
    if (threadIdx.x < 16) v[threadIdx.x] = incl - own;
  }
}

// m classes (MK) of the compiled front ends: m = 16 (at k = 31), m <= 16, m > 16.
inline int run_mk(uint32_t k, uint32_t m) { return m > 16 ? 2 : k == 31 && m == 16 ? 0 : 1; }

// Compiled (w, m class) pairs: m = 16 at k = 31, and every w = k - m + 1 from
// 6 on for m <= 16 (MK 1) and m > 16 (MK 2).  Below 6 a batch has a record
// for every third k-mer or more.  Each w is its own unrolled minimum in
// registers; the 39 pairs times two tiles of the bin kernel and two query
// kernels per shard size make up most of the library (2.4 MB without them,
// 11.3 with) and of its build.
#define SBF_RUN_SETS(X)                                                                                  \
  X(16, 0) X(6, 1) X(7, 1) X(8, 1) X(9, 1) X(10, 1) X(11, 1) X(12, 1) X(13, 1) X(14, 1) X(15, 1)          \
  X(16, 1) X(17, 1) X(18, 1) X(19, 1) X(20, 1) X(21, 1) X(22, 1) X(23, 1) X(24, 1) X(25, 1) X(26, 1)      \
  X(27, 1) X(28, 1) X(29, 1) X(30, 1) X(31, 1) X(32, 1) X(6, 2) X(7, 2) X(8, 2) X(9, 2) X(10, 2) X(11, 2) \
  X(12, 2) X(13, 2) X(14, 2) X(15, 2) X(16, 2)

inline bool run_compiled(int w, int mk) {
#define SBF_MATCH(W_, MK_) \
  if (w == W_ && mk == MK_) return true;
  SBF_RUN_SETS(SBF_MATCH)
#undef SBF_MATCH
  return false;
}

inline int log2_of(uint64_t x) {
  int n = 0;
  while ((1ull << n) < x) ++n;
  return n;
}

inline RunGeo run_geo(const Geometry &g, int nmax) {
  RunGeo P;
  P.k = (int)g.k;
  P.m_shift = g.m > 16 ? 64 - 2 * (int)g.m : 32 - 2 * (int)g.m;
  P.nmax = nmax;
  P.shard_mask = (uint32_t)(g.nshards - 1);
  return P;
}

inline BitGeo bit_geo(const Geometry &g) {
  BitGeo B;
  B.z = (int)(g.k - g.s);
  B.s_shift = 64 - 2 * (int)g.s;
  B.H = (int)g.H;
  B.slice = 64 / (int)g.H;
  B.sw_log2 = log2_of(g.shard_words);
  return B;
}

// Runs that a tile's list holds, a whole number per lane: above the expected
// 2 / (w + 1) per k-mer of 8192 (968 at w = 16) and its spread, for w from 8 on.
template <int W>
constexpr int run_list_cap() { return W >= 16 ? 1280 : W >= 11 ? 1536 : W == 10 ? 1792 : 2048; }

}  // namespace
}  // namespace sbf
