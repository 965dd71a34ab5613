// Run query kernels for gfx950: each super-k-mer (run of valid k-mers with one
// shard, Section "Minimizers and Super-k-mers") of a tile is tested by one
// lane, which loads its shard once and hashes each of its s-mers once
// (Algorithm 2 with the shard shared by the whole run).  The tile's runs are
// taken in order of length, so that the lanes of a wave finish together.
//   * 4-word shards: the lane holds the shard in registers;
//   * 8- and 16-word shards: SW/2 lanes load a run's line together, one
//     16-byte piece each, into the wave's LDS rows, and the run's lane reads
//     the 32-bit word of each bit from its row.
// Answers are collected as bits in LDS and written as bytes (or bits), 32
// k-mers per lane.
// Bound by VALU issue in cache (62 instructions per position at 80%, the lane
// kernel 73 at 70%) and by random reads out of cache: 35 G super-k-mers/s, where
// two 16-byte loads per lane reach 41 G shards/s and lane pairs 48.7, each of
// them a 128-byte line (5.2 TB/s).  2M reads of 150 bp: 865 -> 654 us (4-word shards), 2004 -> 873 (16
// words); 150 Mbp at k = 21 1282 -> 497 us (before: the run-time parameter
// kernel); 3 Gbp of reads against 8 GiB 9.99 -> 9.07 ms.
#pragma once

#include "sbf_runs.h"

namespace sbf {
namespace {

// A run's shard in registers.  HC is H, or 0 where H (up to 8) is known only
// at run time.
template <int HC>
struct Sectors {
  uint64_t w[4];
  // 1 where every bit of the s-mer with hash g is set in the shard
  __device__ __forceinline__ uint32_t test(uint64_t g, const BitGeo &B) const {
    if constexpr (HC == 4) {
      const uint32_t lo = (uint32_t)g, hi = (uint32_t)(g >> 32);
      return (uint32_t)(w[0] >> (lo & 63u)) & (uint32_t)(w[1] >> ((lo >> 16) & 63u)) & (uint32_t)(w[2] >> (hi & 63u)) &
             (uint32_t)(w[3] >> ((hi >> 16) & 63u)) & 1u;
    } else {
      uint32_t hit = 1u;
#pragma unroll
      for (int h = 0; h < 8; ++h)
        if (HC == 8 || h < B.H) hit &= (uint32_t)(w[h & 3] >> ((uint32_t)(g >> (h * (HC ? 64 / HC : B.slice))) & 63u));
      return hit;
    }
  }
};

// A run's shard in the wave's LDS rows (pieces of 16 bytes, spread over the
// banks by swz): the row's byte offset with the swizzle folded in.
template <int SW, int HC>
struct Row {
  const uint8_t *rows;
  uint32_t at;
  __device__ __forceinline__ uint32_t test(uint64_t g, const BitGeo &B) const {
    constexpr uint32_t GROUPS = 32u * (SW / 4 - 1);
    uint32_t hit = 1u;
#pragma unroll
    for (int h = 0; h < (HC ? HC : 8); ++h) {
      if (HC || h < B.H) {
        const uint32_t a = (uint32_t)(g >> (h * (HC ? 64 / HC : B.slice)));
        const uint32_t off = (((a >> 1) & GROUPS) ^ (at ^ (uint32_t)(8 * (h & 2)))) | ((a >> 3) & 4u);
        hit &= *reinterpret_cast<const uint32_t *>(rows + off + 8 * (h & 1)) >> (a & 31u);
      }
    }
    return hit;
  }
};

// A run's shard in the filter itself (tiles with more runs than their list
// holds).
template <int SW>
struct Direct {
  const uint32_t *shard;
  __device__ __forceinline__ uint32_t test(uint64_t g, const BitGeo &B) const {
    uint32_t hit = 1u;
#pragma unroll 1
    for (int h = 0; h < B.H; ++h) {
      const uint32_t a = (uint32_t)(g >> (h * B.slice));
      const uint32_t word = (uint32_t)(h & 3) + 4u * ((a >> 6) & (SW / 4 - 1));
      hit &= shard[2 * word + ((a >> 5) & 1u)] >> (a & 31u);
    }
    return hit;
  }
};

// Answers of the wave's runs (one per lane) of n k-mers, whose bases are x, y,
// w: bit r is k-mer r's.  The lanes take steps (uniform, at least n + z for
// every lane) s-mers each, also those of shorter runs, so that the loop needs
// no lane masks.
template <int S, typename Shard>
__device__ __forceinline__ uint32_t run_answers(const Shard &shard, uint32_t x, uint32_t y, uint32_t w, uint32_t n,
                                                int steps, const BitGeo &B) {
  uint32_t hits = 0, more = 0;  // shifted in from the right: steps up to 32, and after
  auto one = [&](uint32_t &to, uint32_t hi, uint32_t lo) {
    to = (to << 1) | (shard.test(top_smer_hash<S>(hi, lo, B), B) & 1u);
  };
  auto walk = [&](uint32_t &to, int count) {
    int j = 0;
    for (; j + 4 <= count; j += 4) {
      one(to, x, y);
#pragma unroll
      for (int o = 1; o < 4; ++o)
        one(to, __builtin_amdgcn_alignbit(x, y, 32 - 2 * o), __builtin_amdgcn_alignbit(y, w, 32 - 2 * o));
      x = __builtin_amdgcn_alignbit(x, y, 24);
      y = __builtin_amdgcn_alignbit(y, w, 24);
      w <<= 8;
    }
    for (; j < count; ++j) {
      one(to, x, y);
      x = __builtin_amdgcn_alignbit(x, y, 30);
      y = __builtin_amdgcn_alignbit(y, w, 30);
      w <<= 2;
    }
  };
  walk(hits, steps < 32 ? steps : 32);
  uint64_t all = hits;
  if (steps > 32) {
    walk(more, steps - 32);
    all = (all << (steps - 32)) | more;
  }
  // s-mer j is bit steps-1-j; k-mer r needs s-mers r .. r+z: bit steps-1-z-r
  all = window_and_rt(all, B.z + 1);
  const uint32_t rev = __builtin_bitreverse32((uint32_t)all) >> (32 - (steps - B.z));
  return rev & ((1u << n) - 1u);
}

constexpr int kRunWG = 256;

template <int W, int MK, int SW, int HC, int S>
__global__ __launch_bounds__(kRunWG) __attribute__((amdgpu_waves_per_eu(4))) void query_runs_kernel(
    const uint8_t *__restrict__ seq, uint64_t len, const uint32_t *__restrict__ starts, int aligned16,
    const uint64_t *__restrict__ words, RunGeo P, BitGeo B, uint8_t *__restrict__ out, uint64_t n_out, int out_aligned16,
    int out_packed, TileQueue tq) {
  constexpr int WG = kRunWG;
  constexpr int LCAP = run_list_cap<W>();
  constexpr int RPT = LCAP / WG;
  using Tile = RunTile<WG, LCAP>;
  __shared__ Tile T;
  __shared__ uint32_t s_len[16];
  __shared__ uint32_t s_next_tile;
  const int t = threadIdx.x, lane = t & 63;

  acquire_device();
  uint64_t tile;
  for (bool first_tile = true; next_tile(tq, &s_next_tile, first_tile, tile); first_tile = false) {
    const uint64_t base = tile * (uint64_t)Tile::TILE;
    uint32_t head, first, total;
    find_runs<W, MK>(T, seq, len, base, starts, aligned16 != 0, P, head, first, total);
    uint32_t *s_ans = T.change;  // answer bits: lane t's 32 k-mers
    s_ans[t] = 0;
    for (uint32_t done = 0; done < total; done += LCAP) {
      const uint32_t here = total - done < (uint32_t)LCAP ? total - done : (uint32_t)LCAP;
      list_runs(T, head, first, done);
      if (t < 16) s_len[t] = 0;
      __syncthreads();
      {
        // counting sort of the list, longest runs first
        uint32_t q[RPT], bin[RPT], rank[RPT];
#pragma unroll
        for (int c = 0; c < RPT; ++c) {
          const uint32_t i = (uint32_t)(c * WG + t);
          q[c] = T.list[i < here ? i : 0];
          bin[c] = 15u - run_length1(T, (int)q[c]);
        }
#pragma unroll
        for (int c = 0; c < RPT; ++c)
          if ((uint32_t)(c * WG + t) < here) rank[c] = atomicAdd(&s_len[bin[c]], 1u);
        __syncthreads();
        scan16(s_len);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < RPT; ++c)
          if ((uint32_t)(c * WG + t) < here) T.list[s_len[bin[c]] + rank[c]] = (uint16_t)q[c];
      }
      __syncthreads();
      // a finished run's answers, from tile position q on
      auto put = [&](uint32_t q, uint32_t ans) {
        const uint64_t v = (uint64_t)ans << (q & 31u);
        if ((uint32_t)v) atomicOr(&s_ans[q >> 5], (uint32_t)v);
        if ((uint32_t)(v >> 32)) atomicOr(&s_ans[(q >> 5) + 1], (uint32_t)(v >> 32));
      };
      auto shard_of = [&](uint32_t q) { return T.shard[q & (kRunL - 1)][q / kRunL] & P.shard_mask; };
      // the wave's first run is its longest (a lane past the list takes run 0,
      // but then only the wave's first lane counts)
      auto steps_of = [&](uint32_t n) { return __builtin_amdgcn_readfirstlane((int)n) + B.z; };
      if constexpr (SW == 4) {
        // the next run's shard is loaded while this one is tested
        uint32_t q = T.list[(uint32_t)t < here ? t : 0];
        const uint4 *p = reinterpret_cast<const uint4 *>(words + 4ull * shard_of(q));
        uint4 lo = p[0], hi = p[1];
#pragma unroll 1
        for (uint32_t i = t; i - lane < here; i += WG) {
          const uint32_t q2 = T.list[i + WG < here ? i + WG : 0];
          p = reinterpret_cast<const uint4 *>(words + 4ull * shard_of(q2));
          const uint4 lo2 = p[0], hi2 = p[1];
          Sectors<HC> s;
          s.w[0] = ((uint64_t)lo.y << 32) | lo.x;
          s.w[1] = ((uint64_t)lo.w << 32) | lo.z;
          s.w[2] = ((uint64_t)hi.y << 32) | hi.x;
          s.w[3] = ((uint64_t)hi.w << 32) | hi.z;
          uint32_t x, y, w;
          run_bases(T, (int)q, x, y, w);
          const uint32_t n = run_length1(T, (int)q) + 1u;
          const uint32_t ans = run_answers<S>(s, x, y, w, n, steps_of(n), B);
          if (i < here) put(q, ans);
          q = q2;
          lo = lo2;
          hi = hi2;
        }
      } else if (total > (uint32_t)LCAP) {
#pragma unroll 1
        for (uint32_t i = t; i - lane < here; i += WG) {
          const uint32_t q = T.list[i < here ? i : 0];
          uint32_t x, y, w;
          run_bases(T, (int)q, x, y, w);
          const Direct<SW> s{reinterpret_cast<const uint32_t *>(words + (uint64_t)SW * shard_of(q))};
          const uint32_t n = run_length1(T, (int)q) + 1u;
          const uint32_t ans = run_answers<S>(s, x, y, w, n, steps_of(n), B);
          if (i < here) put(q, ans);
        }
      } else {
        constexpr int LPR = SW / 2;      // lanes per line, and loads per lane
        constexpr int RPL = 64 / LPR;    // lines per load
        uint32_t q[RPT], sh[RPT];
#pragma unroll
        for (int c = 0; c < RPT; ++c) {
          const uint32_t i = (uint32_t)(c * WG + t);
          q[c] = T.list[i < here ? i : 0];
          sh[c] = shard_of(q[c]);
        }
        __syncthreads();  // the rows go over the shards
        u32x4 *rows = reinterpret_cast<u32x4 *>(&T.shard[0][0]) + (t & ~63) * LPR;
        u32x4 piece[LPR];
        auto fetch = [&](uint32_t shard) {
#pragma unroll
          for (int x = 0; x < LPR; ++x) {
            const uint32_t s = __shfl(shard, x * RPL + lane / LPR, 64);
            piece[x] = *reinterpret_cast<const u32x4 *>(words + (uint64_t)s * SW + 2 * (lane % LPR));
          }
        };
        auto swz = [](int r) { return (uint32_t)(SW == 16 ? r & 7 : (r >> 1) & 3); };
        fetch(sh[0]);
#pragma unroll 1
        for (uint32_t i = t; i - lane < here; i += WG) {
#pragma unroll
          for (int x = 0; x < LPR; ++x) {
            const int r = x * RPL + lane / LPR;
            rows[r * LPR + (int)((uint32_t)(lane % LPR) ^ swz(r))] = piece[x];
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          const uint32_t at = q[0];
#pragma unroll
          for (int c = 0; c + 1 < RPT; ++c) {
            q[c] = q[c + 1];
            sh[c] = sh[c + 1];
          }
          fetch(sh[0]);  // the next round's lines (the last round's again after it)
          uint32_t x, y, w;
          run_bases(T, (int)at, x, y, w);
          const Row<SW, HC> s{reinterpret_cast<const uint8_t *>(rows),
                                (uint32_t)(lane * LPR * 16) | (swz(lane) << 4)};
          const uint32_t n = run_length1(T, (int)at) + 1u;
          const uint32_t ans = run_answers<S>(s, x, y, w, n, steps_of(n), B);
          if (i < here) put(at, ans);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
      }
      __syncthreads();
    }
    __syncthreads();
    const uint32_t ans = s_ans[t];
    const uint64_t pos0 = base + (uint64_t)t * kRunL;
    if (out_packed) {
      // one answer bit per k-mer; bits at or past n_out are cleared, bytes
      // past them not written
      if (pos0 < n_out) {
        const uint64_t left = n_out - pos0;
        const uint32_t bits = left < 32 ? ans & ((1u << left) - 1u) : ans;
        uint8_t *ob = out + pos0 / 8;
        if (left >= 32) {
          reinterpret_cast<uint16_t *>(ob)[0] = (uint16_t)bits;
          reinterpret_cast<uint16_t *>(ob)[1] = (uint16_t)(bits >> 16);
        } else {
          for (uint64_t j = 0; j < (left + 7) / 8; ++j) ob[j] = (uint8_t)(bits >> (8 * j));
        }
      }
      continue;
    }
    // one answer byte per k-mer: four bits x spread to bytes by x * 0x204081
    auto bytes4 = [&](int r) { return (((ans >> r) & 0xFu) * 0x204081u) & 0x01010101u; };
    if (out_aligned16 && pos0 + kRunL <= n_out) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
        *reinterpret_cast<uint4 *>(out + pos0 + 16 * c) =
            make_uint4(bytes4(16 * c), bytes4(16 * c + 4), bytes4(16 * c + 8), bytes4(16 * c + 12));
    } else {
      for (int r = 0; r < kRunL; ++r)
        if (pos0 + r < n_out) out[pos0 + r] = (uint8_t)((ans >> r) & 1u);
    }
  }
}

template <int W, int MK, int SW, int HC, int S>
hipError_t query_runs(const Geometry &g, const uint64_t *words, const SeqArgs &a, const LaunchShape &ls,
                      hipStream_t st) {
  const uint64_t tile = (uint64_t)kRunWG * kRunL;
  const RunGeo P = run_geo(g, 16);
  const BitGeo B = bit_geo(g);
  SBF_LAUNCH_TILES((query_runs_kernel<W, MK, SW, HC, S>), kRunWG, (a.n_out + tile - 1) / tile, 2, a.seq, a.len,
                   a.starts, (int)(((uintptr_t)a.seq & 15u) == 0), words, P, B, a.out, a.n_out,
                   (int)(((uintptr_t)a.out & 15u) == 0), a.packed);
  return hipSuccess;
}

// Shards of SW words, any compiled front end.
template <int SW>
hipError_t query_runs_any(const Geometry &g, const uint64_t *words, const SeqArgs &a, const LaunchShape &ls,
                          hipStream_t st) {
  if (a.n_out == 0) return hipSuccess;
  const int w = (int)(g.k - g.m + 1), mk = run_mk(g.k, g.m);
  // the paper's default s saves 3 of 22 instructions per s-mer
  if (w == 16 && mk == 0 && g.H == 4 && g.s == 28) return query_runs<16, 0, SW, 4, 28>(g, words, a, ls, st);
  if (w == 16 && mk == 0 && g.H == 8) return query_runs<16, 0, SW, 8, 0>(g, words, a, ls, st);
#define SBF_CALL(W_, MK_)                                                             \
  if (w == W_ && mk == MK_)                                                           \
    return g.H == 4 ? query_runs<W_, MK_, SW, 4, 0>(g, words, a, ls, st)              \
                    : query_runs<W_, MK_, SW, 0, 0>(g, words, a, ls, st);
  SBF_RUN_SETS(SBF_CALL)
#undef SBF_CALL
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace sbf
