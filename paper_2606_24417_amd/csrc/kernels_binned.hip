// Binned insert of large batches (shards of 4, 8 or 16 words, k <= 32, H <= 8)
// for gfx950.
//
// The two-pass insert (kernels_rolling.hip and the other families) reads and
// writes a random shard per super-k-mer, then reads every shard again to
// restore the bits that racing writes dropped; it is bound by those random
// accesses (a 128-byte line moves for every 32-byte shard).  For a batch that
// touches most of the filter it is cheaper to bring the super-k-mers to the
// filter in order:
//   1. bin_kernel walks the sequence once, finds the super-k-mers (runs of
//      valid k-mers with one shard) and appends each as a 16-byte record (its
//      bases, length and shard) to the bucket of its shard range;
//   2. split_kernel (filters of more than 256 slices) splits each bucket into
//      slices of 32 or 64 KB of the filter;
//   3. apply_kernel holds one slice in LDS, ORs the s-mer bits of the slice's
//      records into it and writes the slice back once.
// Every slice is read and written by one workgroup, so no update races with
// another and no repair pass is needed.  Records that find their bucket full (a
// batch far from the expected spread over shards) are gathered by shard in LDS
// and applied with atomic ORs of the bits that are missing, before any slice is
// read.
// Measured against the two passes (clear + insert): 100 Mbp into 256 MiB 880
// -> 412 us, with 16-word shards 2159 -> 468, 3 Gbp into 8 GiB 29.8 -> 13.6 ms,
// 1 Mbp into 2 MiB 76 -> 25 us.
#include "sbf_runs.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace sbf {
namespace {

constexpr int kBinTile = 512 * kRunL;       // k-mers of the largest tile
constexpr int kCountShift = 5;              // counters one 128-byte line apart
constexpr int kXcds = 8;
constexpr int kMaxBucketBits1 = 8;
constexpr int kMaxBucketBits2 = 11;
constexpr int kSplitWG = 512;
constexpr int kSplitPer = 8;                // records per lane
constexpr int kSplitTile = kSplitWG * kSplitPer;
constexpr uint32_t kApplyGrid = 512;        // two workgroups per CU (64 KB of LDS each), four of 32 KB

// k-mers binned at a time: up to these, more for a filter that has more memory
// itself
constexpr uint64_t kMinChunkKmers = 1ull << 27;
// batches up to these append to one part per bucket
constexpr uint64_t kOnePartKmers = 1ull << 25;
constexpr int kMinSliceBits = 6;  // fewer slices leave most of the GPU idle
// Batches that take the binned insert.  It reads and writes the whole filter,
// so it needs enough k-mers for the filter's size; measured (us, binned against
// two passes) at (31,28,16,4): 2^27 bits 0.15M k-mers 43/53, 4M 57/127; 2^28
// bits 1M 62/63, 2M 64/73; 2^31 bits 8M 162/143, 16M 184/228, 128M 496/1057;
// 2^33 bits 32M 547/404, 64M 638/683; 2^36 bits 400M 4804/3938.  The other
// kernel families' two passes take twice as long: at (31,26,16,4) 2^26 bits
// 0.15M 30/39; 2^27 bits 0.25M 43/41, 0.5M 42/49; 2^31 bits 4M 156/156, 8M
// 164/235; 2^33 bits 32M 547/723; 2^36 bits 256M 4271/5071; 16-word shards
// at (31,28,16,4) 2^31 bits 8M 167/259, 2^36 bits 256M 4277/5586.
constexpr uint64_t kMinBinnedKmers = 1ull << 17;
constexpr uint64_t kLaneSmallBits = 1ull << 27, kOtherSmallBits = 1ull << 26;
constexpr uint64_t kLaneBitsPerKmer = 112, kOtherBitsPerKmer = 256;

// A super-k-mer of at most 16 k-mers: its bases from the top of x down (2 bits
// each, at most 46), its number of k-mers minus one in the low 4 bits of z,
// its shard in w.
typedef u32x4 Record;

struct BinGeo {
  int bucket_shift;  // shard >> bucket_shift = bucket
  int nbuckets;
  int part_mask;     // parts per bucket minus one: 7 (an XCD each) or 0
};

// Appended records: region r holds cap records from r * cap on,
// counts[r << kCountShift] is the number of appends asked for (it may exceed
// cap).
struct Bins {
  Record *rec;
  uint32_t *counts;
  uint32_t cap;
};

// The records of a tile that found their region full (a lane's are rec[c] with
// bit c of pending set): their bits are gathered per shard in a table in LDS,
// lines then keys, and each word of the table is ORed into the filter where it
// has bits that are missing.  The loads bypass this XCD's caches (agent scope),
// so that the tiles of a crowded shard find their bits set instead of issuing
// atomics.  A record that finds no place in the table waits for the next round;
// the first of a round always finds one.
// Gathering matters because such tiles hold few shards, and looking before an
// OR because their lanes meet in one word.  Bound by the chain of hashes and LDS
// reads of a few busy waves.  Measured against testing each record's words in
// the filter one by one (us; clear + insert of 2 Mbp into 4 MiB of 16-word
// shards): repeats of period 40 975 -> 102, of 5000 277 -> 120; two passes 89
// and 94.  100 Mbp of period 171 into 256 MiB: 1.5 ms with 4-word shards, 1.7
// with 16 (two passes: 27.7 and 2.3).
constexpr uint32_t kNoShard = ~0u;  // binned filters have at most 2^30 shards
constexpr int kProbes = 8;

template <int WG, int N>
__device__ __forceinline__ void apply_overflow(const Record (&rec)[N], uint32_t pending, void *lds, uint32_t lds_bytes,
                                               uint32_t *s_more, uint64_t *words, BitGeo B) {
  const int t = threadIdx.x;
  const uint32_t nslots = lds_bytes / ((8u << B.sw_log2) + 4u);  // a line and its key
  const uint32_t line_words = nslots << B.sw_log2;
  uint64_t *lines = reinterpret_cast<uint64_t *>(lds);
  uint32_t *keys = reinterpret_cast<uint32_t *>(lines + line_words);
  const uint32_t groups = (1u << B.sw_log2) / 4u;
  for (;;) {
    for (uint32_t i = t; i < line_words; i += WG) lines[i] = 0;
    for (uint32_t i = t; i < nslots; i += WG) keys[i] = kNoShard;
    if (t == 0) *s_more = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const Record r = rec[c];
      if (!(pending >> c & 1u)) continue;
      uint32_t slot = __umulhi(r[3] * 0x9E3779B1u, nslots);
      bool found = false;
      for (int probe = 0; probe < kProbes && !found; ++probe) {
        if (probe) slot = slot + 1 < nslots ? slot + 1 : 0;
        const uint32_t had = atomicCAS(&keys[slot], kNoShard, r[3]);
        found = had == kNoShard || had == r[3];
      }
      if (!found) continue;
      pending &= ~(1u << c);
      uint32_t *line = reinterpret_cast<uint32_t *>(lines + (slot << B.sw_log2));
      const int count = (int)(r[2] & 15u) + 1 + B.z;
      uint32_t x = r[0], y = r[1], w = r[2];
#pragma unroll 1
      for (int j = 0; j < count; ++j) {
        const uint64_t g = top_smer_hash<0>(x, y, B);
        x = __builtin_amdgcn_alignbit(x, y, 30);
        y = __builtin_amdgcn_alignbit(y, w, 30);
        w <<= 2;
        // most bits are set by the lanes before, and ORs of one word go one by
        // one: look first, at four hash indices at a time
#pragma unroll 1
        for (int h0 = 0; h0 < B.H; h0 += 4) {
          uint32_t *p[4], bit[4], had[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t a = (uint32_t)(g >> ((h0 + i < B.H ? h0 + i : 0) * B.slice));
            p[i] = line + 2 * ((uint32_t)(h0 + i < B.H ? i : 0) + 4 * ((a >> 6) & (groups - 1))) + ((a >> 5) & 1u);
            bit[i] = 1u << (a & 31u);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) had[i] = __hip_atomic_load(p[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (!(had[i] & bit[i])) atomicOr(p[i], bit[i]);
        }
      }
    }
    if (pending) *s_more = 1;
    __syncthreads();
    for (uint32_t i = t; i < line_words; i += WG) {
      const uint32_t shard = keys[i >> B.sw_log2];
      const uint64_t m = lines[i];
      if (shard == kNoShard || m == 0) continue;
      uint64_t *word = words + ((uint64_t)shard << B.sw_log2) + (i & ((1u << B.sw_log2) - 1u));
      const uint64_t missing = m & ~__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (missing) atomic_or64(word, missing);
    }
    const uint32_t more = *s_more;
    if (!more) return;
    __syncthreads();  // before the table and the flag are cleared
  }
}

// Tiles of WG x 32 k-mers: 256 lanes, or 512 where there are 256 buckets.  A
// tile appends 2 / (w + 1) records per k-mer; at 256 buckets a tile of 8192
// k-mers appends less than four at a time to each, lines leave the L2 before
// they are full and the pass writes 1.5 times its records (3 Gbp: 4.65 ms
// with 256 lanes, 3.41 with 512; with 128 buckets 100 Mbp 0.113 and 0.120).
// LDS allows four workgroups of 256 lanes per CU, or two of 512; three of 256
// for w below 11, whose list is longer.
template <int W, int MK, int WG>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4))) void bin_kernel(
    const uint8_t *__restrict__ seq, uint64_t len, const uint32_t *__restrict__ starts, int aligned16, RunGeo P,
    BinGeo G, Bins out, uint64_t *__restrict__ words, BitGeo B) {
  // a tile with more runs only appends in two goes, so the list is shorter
  // than the query's
  constexpr int LCAP = W >= 16 ? 4 * WG : W >= 11 || WG > 256 ? 6 * WG : 8 * WG;
  using Tile = RunTile<WG, LCAP>;
  static_assert(LCAP % WG == 0 && LCAP * 16 <= kRunL * WG * 4, "whole records per lane, which fit over the shards");
  constexpr int RPT = LCAP / WG;
  __shared__ Tile T;
  __shared__ uint16_t s_before[1 << kMaxBucketBits1];  // a bucket's first record in the sorted tile
  __shared__ uint32_t s_over;                          // a region is full
  static_assert((1 << kMaxBucketBits1) <= WG, "a bucket per lane");

  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  uint32_t head, first, total;
  find_runs<W, MK>(T, seq, len, (uint64_t)blockIdx.x * Tile::TILE, starts, aligned16 != 0, P, head, first, total);
  uint32_t *s_hist = T.change;  // records per bucket, then where they go
  // each XCD appends to its own part of a bucket, so that the part's last
  // line fills up in that XCD's L2
  const uint32_t part = blockIdx.x & (uint32_t)G.part_mask, parts = (uint32_t)G.part_mask + 1u;

  // the record of the run from tile position q on
  auto record = [&](int q) {
    uint32_t x, y, z;
    run_bases(T, q, x, y, z);
    Record rec;
    rec[0] = x;
    rec[1] = y;
    rec[2] = (z & ~15u) | run_length1(T, q);
    rec[3] = T.shard[q & (kRunL - 1)][q / kRunL] & P.shard_mask;
    return rec;
  };
  s_hist[t] = 0;
  if (t == 0) s_over = 0;
  // no run starts in the tile (records shorter than k, invalid bases): the
  // list is empty and its storage still holds validity bits
  if (total == 0) return;
  list_runs(T, head, first, 0);
  __syncthreads();
  if (total <= (uint32_t)LCAP) {
    // The usual tile: its records are put in bucket order in LDS, over the
    // shards, so that consecutive lanes append consecutive records.
    Record rec[RPT];
    uint32_t rank[RPT];
#pragma unroll
    for (int c = 0; c < RPT; ++c) {
      const uint32_t i = (uint32_t)(c * WG + t);
      rec[c] = record(T.list[i < total ? i : 0]);
    }
    // A record equal to the one before it (long homopolymers and the like
    // are cut into equal records, all for one shard) adds nothing.
    uint32_t keep = 0;
#pragma unroll
    for (int c = 0; c < RPT; ++c) {
      const bool listed = (uint32_t)(c * WG + t) < total;
      bool same = __shfl_up(rec[c][3], 1, 64) == rec[c][3] && lane > 0 && listed;
      if (__ballot(same)) {
#pragma unroll
        for (int x = 0; x < 3; ++x) same = (__shfl_up(rec[c][x], 1, 64) == rec[c][x]) && same;
      }
      if (listed && !same) keep |= 1u << c;
    }
#pragma unroll
    for (int c = 0; c < RPT; ++c)
      if (keep >> c & 1u) rank[c] = atomicAdd(&s_hist[rec[c][3] >> G.bucket_shift], 1u);
    __syncthreads();
    const uint32_t n = t < G.nbuckets ? s_hist[t] : 0u;
    uint32_t upto = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(upto, d, 64);
      if (lane >= d) upto += o;
    }
    if (lane == 63) T.wsum[wave] = upto;
    // where the bucket's records go, and (in T.change) where they are in LDS
    const uint32_t place = n ? atomicAdd(&out.counts[(t * parts + part) << kCountShift], n) : 0u;
    __syncthreads();
    uint32_t before = upto - n, kept = 0;
#pragma unroll
    for (int w = 0; w < WG / 64; ++w) {
      if (w < wave) before += T.wsum[w];
      kept += T.wsum[w];
    }
    if (t < G.nbuckets) s_before[t] = (uint16_t)before;
    __syncthreads();
    Record *sorted = reinterpret_cast<Record *>(&T.shard[0][0]);
#pragma unroll
    for (int c = 0; c < RPT; ++c)
      if (keep >> c & 1u) sorted[s_before[rec[c][3] >> G.bucket_shift] + rank[c]] = rec[c];
    if (t < G.nbuckets) s_hist[t] = place - before;
    if (place + n > out.cap) s_over = 1;
    __syncthreads();
#pragma unroll 1
    for (uint32_t i = t; i < kept; i += WG) {
      const Record x = sorted[i];
      const uint32_t bucket = x[3] >> G.bucket_shift;
      const uint32_t pos = s_hist[bucket] + i;
      if (pos < out.cap) out.rec[(uint64_t)(bucket * parts + part) * out.cap + pos] = x;
    }
    if (s_over) {
      uint32_t pending = 0;
#pragma unroll
      for (int c = 0; c < RPT; ++c) {
        const uint32_t i = (uint32_t)(c * WG + t);
        rec[c] = sorted[i < kept ? i : 0];
        if (i < kept && s_hist[rec[c][3] >> G.bucket_shift] + i >= out.cap) pending |= 1u << c;
      }
      __syncthreads();  // the sorted records and the flag have been read
      apply_overflow<WG>(rec, pending, sorted, sizeof(T.shard), &s_over, words, B);
    }
    return;
  }
  // more records than the list holds: some at a time, appended as they come
  for (uint32_t done = 0;;) {
    const uint32_t here = total - done < (uint32_t)LCAP ? total - done : (uint32_t)LCAP;
    uint32_t rank[RPT];
#pragma unroll
    for (int c = 0; c < RPT; ++c) {
      const uint32_t i = (uint32_t)(c * WG + t);
      const int q = T.list[i < here ? i : 0];
      if (i < here) rank[c] = atomicAdd(&s_hist[(T.shard[q & (kRunL - 1)][q / kRunL] & P.shard_mask) >> G.bucket_shift], 1u);
    }
    __syncthreads();
    if (t < G.nbuckets) {
      const uint32_t n = s_hist[t];
      if (n) {
        const uint32_t place = atomicAdd(&out.counts[(t * parts + part) << kCountShift], n);
        if (place + n > out.cap) s_over = 1;
        s_hist[t] = place;
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < RPT; ++c) {
      const uint32_t i = (uint32_t)(c * WG + t);
      if (i < here) {
        const Record x = record(T.list[i]);
        const uint32_t bucket = x[3] >> G.bucket_shift;
        const uint32_t pos = s_hist[bucket] + rank[c];
        if (pos < out.cap) out.rec[(uint64_t)(bucket * parts + part) * out.cap + pos] = x;
      }
    }
    if (s_over) {
      Record rec[RPT];
      uint32_t pending = 0;
#pragma unroll
      for (int c = 0; c < RPT; ++c) {
        const uint32_t i = (uint32_t)(c * WG + t);
        rec[c] = record(T.list[i < here ? i : 0]);
        if (i < here && s_hist[rec[c][3] >> G.bucket_shift] + rank[c] >= out.cap) pending |= 1u << c;
      }
      // the table takes some rows of the shards, which are put back after
      constexpr int ROWS = LCAP * (int)sizeof(Record) / (WG * 4);
      uint32_t mine[ROWS];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) mine[r] = T.shard[r][t];
      __syncthreads();
      apply_overflow<WG>(rec, pending, &T.shard[0][0], LCAP * sizeof(Record), &s_over, words, B);
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ROWS; ++r) T.shard[r][t] = mine[r];
    }
    done += LCAP;
    if (done >= total) break;
    __syncthreads();
    s_hist[t] = 0;
    if (t == 0) s_over = 0;
    list_runs(T, head, first, done);
    __syncthreads();
  }
}

// Split the records of a group of buckets, from bucket b0 on, into the slices
// of each.  The tiles of one bucket run on one XCD (workgroups go to the XCDs
// in turn), so that the records appended to a slice gather in one L2, and a
// tile's records are put in slice order in LDS first, so that consecutive
// lanes append consecutive records: the 12 M records of 100 Mbp take 76 us (5
// TB/s read and written, the rate of a streaming copy) against 143 us appended
// as they come.
__global__ __launch_bounds__(kSplitWG) __attribute__((amdgpu_waves_per_eu(4))) void split_kernel(
    Bins in, Bins out, uint32_t b0, uint32_t tiles_per_region, int slice_shift, uint32_t slices_per_bucket,
    uint64_t *__restrict__ words, BitGeo B) {
  __shared__ Record s_rec[kSplitTile];
  __shared__ uint32_t s_hist[1 << kMaxBucketBits2];   // records per slice, then where they go
  __shared__ uint16_t s_first[1 << kMaxBucketBits2];  // a slice's first record in s_rec
  __shared__ uint32_t s_wsum[kSplitWG / 64];
  __shared__ uint32_t s_over;  // a slice's region is full
  const uint32_t per_bucket = tiles_per_region * kXcds;
  const uint32_t j = blockIdx.x / kXcds;
  const uint32_t bl = (j / per_bucket) * kXcds + (blockIdx.x & (kXcds - 1));  // bucket - b0
  const uint32_t region = (b0 + bl) * kXcds + j % kXcds;
  const uint32_t first = (j % per_bucket) / kXcds * kSplitTile;
  uint32_t n = in.counts[region << kCountShift];
  n = n < in.cap ? n : in.cap;
  if (first >= n) return;
  n = n - first < (uint32_t)kSplitTile ? n - first : (uint32_t)kSplitTile;
  const int t = threadIdx.x;
  for (uint32_t b = t; b < slices_per_bucket; b += kSplitWG) s_hist[b] = 0;
  if (t == 0) s_over = 0;
  const Record *src = in.rec + (uint64_t)region * in.cap + first;
  const uint32_t sub = slices_per_bucket - 1;
  Record r[kSplitPer];
  uint32_t rank[kSplitPer];
#pragma unroll
  for (int c = 0; c < kSplitPer; ++c) {
    const uint32_t i = (uint32_t)(c * kSplitWG + t);
    r[c] = src[i < n ? i : 0];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kSplitPer; ++c)
    if ((uint32_t)(c * kSplitWG + t) < n) rank[c] = atomicAdd(&s_hist[(r[c][3] >> slice_shift) & sub], 1u);
  __syncthreads();
  // lane t takes the slices_per_bucket / kSplitWG slices from t times that on
  constexpr int MAXPER = (1 << kMaxBucketBits2) / kSplitWG;
  const uint32_t per = slices_per_bucket > (uint32_t)kSplitWG ? slices_per_bucket / kSplitWG : 1u;
  const uint32_t sb = t * per;
  uint32_t mine = 0;
  for (uint32_t x = 0; x < per; ++x)
    if (sb + x < slices_per_bucket) mine += s_hist[sb + x];
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if ((t & 63) >= d) incl += o;
  }
  if ((t & 63) == 63) s_wsum[t >> 6] = incl;
  __syncthreads();
  uint32_t at = incl - mine;
#pragma unroll
  for (int w = 0; w < kSplitWG / 64; ++w)
    if (w < t >> 6) at += s_wsum[w];
  uint32_t place[MAXPER], end[MAXPER];
#pragma unroll
  for (int x = 0; x < MAXPER; ++x) {
    if ((uint32_t)x < per && sb + x < slices_per_bucket) {
      const uint32_t m = s_hist[sb + x];
      s_first[sb + x] = (uint16_t)at;
      place[x] = m ? atomicAdd(&out.counts[((uint64_t)(b0 + bl) * slices_per_bucket + sb + x) << kCountShift], m) - at
                   : 0u;
      at += m;
      end[x] = m ? at : 0u;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kSplitPer; ++c)
    if ((uint32_t)(c * kSplitWG + t) < n) s_rec[s_first[(r[c][3] >> slice_shift) & sub] + rank[c]] = r[c];
#pragma unroll
  for (int x = 0; x < MAXPER; ++x)
    if ((uint32_t)x < per && sb + x < slices_per_bucket) {
      s_hist[sb + x] = place[x];
      if (end[x] && place[x] + end[x] > out.cap) s_over = 1;
    }
  __syncthreads();
#pragma unroll 1
  for (uint32_t i = t; i < n; i += kSplitWG) {
    const Record x = s_rec[i];
    const uint32_t b = (x[3] >> slice_shift) & sub;
    const uint32_t pos = s_hist[b] + i;
    if (pos < out.cap) out.rec[((uint64_t)bl * slices_per_bucket + b) * out.cap + pos] = x;
  }
  if (s_over) {
    uint32_t pending = 0;
#pragma unroll
    for (int c = 0; c < kSplitPer; ++c) {
      const uint32_t i = (uint32_t)(c * kSplitWG + t);
      r[c] = s_rec[i < n ? i : 0];
      if (i < n && s_hist[(r[c][3] >> slice_shift) & sub] + i >= out.cap) pending |= 1u << c;
    }
    __syncthreads();  // the sorted records and the flag have been read
    apply_overflow<kSplitWG>(r, pending, s_rec, sizeof(s_rec), &s_over, words, B);
  }
}

// Apply the records of slices s0 .. s0 + nslices - 1, one slice at a time per
// workgroup.  A slice's records lie in `regions` regions of in, from region
// (slice - s0) * regions on; counts are indexed from slice 0.  The records are
// taken in order of length (a counting sort of their indices), so that the
// lanes of a wave finish together (320 -> 254 us for 100 Mbp, with fewer, larger
// launches; 198 us now, 42 VALU instructions per k-mer at 56% of issue: a
// workgroup waits between its sort, its records and its write-back, and four
// per CU do not hide all of it).
// With 8- and 16-word shards, whose bits are ORed one by one, sector c of shard
// i is at place c ^ x(i) in LDS, x from i's low bits: the lanes of a wave, which
// all OR the same sector at a time, then spread over all banks instead of a
// quarter of them (16 words, 100 Mbp: 344 -> 305 us; no change with the four
// 64-bit ORs per record of 4-word shards).
// S > 0: s is known.
template <int SW, int H, int SB, int S>
__global__ __launch_bounds__(1 << (SB - 4)) __attribute__((amdgpu_waves_per_eu(4))) void apply_kernel(
    Bins in, uint32_t s0, uint32_t nslices, uint32_t regions, uint64_t *__restrict__ words, BitGeo B) {
  constexpr int SWL = SW == 4 ? 2 : SW == 8 ? 3 : 4;
  constexpr int WORDS = 1 << SB;                      // 64-bit words of a slice
  constexpr int WG = 1 << (SB - 4);
  constexpr int PIECES = WORDS / 2 / WG;  // 16-byte pieces per lane
  constexpr int SLICE = 64 / H;
  constexpr int PER = 8;                              // records sorted per lane
  constexpr int CHUNK = PER * WG;
  __shared__ uint64_t s_words[WORDS];
  __shared__ uint16_t s_list[CHUNK];
  __shared__ uint32_t s_len[16];
  const int t = threadIdx.x;
  acquire_device();
  __syncthreads();
  u32x4 *acc = reinterpret_cast<u32x4 *>(s_words);
  auto swz = [](uint32_t shard) { return SW == 4 ? 0u : (shard >> (4 - SWL)) & 3u; };
  auto region_count = [&](uint32_t slice, uint32_t g) {
    const uint32_t n = in.counts[((uint64_t)(s0 + slice) * regions + g) << kCountShift];
    return n < in.cap ? n : in.cap;
  };
  // 16 minus the k-mers of the lane's records i = t, t + WG, ..
  auto lengths = [&](const Record *src, uint32_t here, uint32_t (&len)[PER]) {
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const uint32_t i = (uint32_t)(c * WG + t);
      len[c] = 15u - (reinterpret_cast<const uint32_t *>(src + (i < here ? i : 0))[2] & 15u);
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int c = 0; c < PIECES; ++c) acc[c * WG + t] = u32x4{0, 0, 0, 0};
  };
  // OR a record's s-mer bits into the slice.
  auto take = [&](const Record &r, auto looks) {
    constexpr bool look = decltype(looks)::value;
    const uint32_t shard = r[3] & ((WORDS >> SWL) - 1);
    uint64_t *dst = s_words + (shard << SWL);
    const uint32_t sx = swz(shard);
    const int count = (int)(r[2] & 15u) + 1 + B.z;
    uint32_t x = r[0], y = r[1], w = r[2];
    uint64_t m[4] = {0, 0, 0, 0};
    // (unrolled by 2, clear + insert of 100 Mbp into 16-word shards take 470 us
    // instead of 457)
#pragma unroll (SW > 4 ? 4 : 2)
    for (int j = 0; j < count; ++j) {
      const uint64_t g = top_smer_hash<S>(x, y, B);
      x = __builtin_amdgcn_alignbit(x, y, 30);
      y = __builtin_amdgcn_alignbit(y, w, 30);
      w <<= 2;
      uint32_t *p[H], bit[H], had[H];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const uint32_t a = (uint32_t)(g >> (h * SLICE));
        if constexpr (SW == 4) {
          m[h & 3] |= 1ull << (a & 63u);
        } else {
          // bytes from the shard on: sector, word group, half
          const uint32_t off = ((((uint32_t)h & 3u) ^ sx) << 3) + (((a >> 1) & (32u * (SW / 4 - 1))) | ((a >> 3) & 4u));
          p[h] = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(dst) + off);
          bit[h] = 1u << (a & 31u);
          if constexpr (look) had[h] = __hip_atomic_load(p[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          else atomicOr(p[h], bit[h]);
        }
      }
      if constexpr (SW > 4 && look) {
#pragma unroll
        for (int h = 0; h < H; ++h)
          if (!(had[h] & bit[h])) atomicOr(p[h], bit[h]);
      }
    }
    if constexpr (SW == 4) {
#pragma unroll
      for (int h = 0; h < (H < 4 ? H : 4); ++h)
        __hip_atomic_fetch_or(dst + ((uint32_t)h ^ sx), m[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
  if (SW > 4) clear();
  for (uint32_t sl = blockIdx.x; sl < nslices; sl += gridDim.x) {
    u32x4 *line = reinterpret_cast<u32x4 *>(words + ((uint64_t)(s0 + sl) << SB));
    // the slice's words are read now and used only at the end
    u32x4 old[PIECES];
#pragma unroll
    for (int c = 0; c < PIECES; ++c) old[c] = line[c * WG + t];
    if (SW == 4) clear();
    for (uint32_t g = 0; g < regions; ++g) {
      const Record *src = in.rec + ((uint64_t)sl * regions + g) * in.cap;
      const uint32_t n = region_count(sl, g);
      for (uint32_t first = 0; first < n; first += CHUNK, src += CHUNK) {
        const uint32_t here = n - first < CHUNK ? n - first : CHUNK;
        uint32_t len[PER], rank[PER];
        lengths(src, here, len);
        if (t < 16) s_len[t] = 0;
        __syncthreads();  // also: the previous records are applied, the words are cleared
#pragma unroll
        for (int c = 0; c < PER; ++c)
          if ((uint32_t)(c * WG + t) < here) rank[c] = atomicAdd(&s_len[len[c]], 1u);
        __syncthreads();
        scan16(s_len);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < PER; ++c) {
          const uint32_t i = (uint32_t)(c * WG + t);
          if (i < here) s_list[s_len[len[c]] + rank[c]] = (uint16_t)i;
        }
        __syncthreads();
        uint32_t i = t;
        Record r = src[i < here ? s_list[i] : 0];
        while (i < here) {
          i += WG;
          const Record next = src[i < here ? s_list[i] : 0];
          // ORs of one LDS word go one by one.  The lanes of a wave are rarely
          // of one shard, except in a batch with crowded shards: there a lane
          // looks first whether the bit is set.
          if (SW > 4 && __popcll(__ballot(r[3] == (uint32_t)__builtin_amdgcn_readfirstlane((int)r[3]))) > 5)
            take(r, std::true_type{});
          else
            take(r, std::false_type{});
          r = next;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < PIECES; ++c) {
      const uint32_t piece = (uint32_t)(c * WG + t);  // words 2p and 2p+1 of a shard
      const uint32_t sx = swz(piece >> (SWL - 1));
      const u32x4 a = acc[piece ^ (sx >> 1)];
      // another lane's place where sectors move: cleared by the lane that read it
      if (SW > 4) acc[piece ^ (sx >> 1)] = u32x4{0, 0, 0, 0};
      const u32x4 b = (sx & 1u) ? u32x4{a[2], a[3], a[0], a[1]} : a;
      *(coherent_u32x4 *)(line + piece) = old[c] | b;
    }
  }
}

uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }

// Records of one region holding a share of n expected ones: the spread over
// buckets of up to 2^11 shares stays within a few percent on genomes; finer
// shares (slices) spread more.
uint64_t region_cap(double expected, double slack) {
  return (uint64_t)std::ceil(expected * slack + 6.0 * std::sqrt(expected) + 64.0);
}

template <int W, int MK, int WG>
hipError_t launch_bin(const SeqArgs &a, uint64_t nk, const RunGeo &P, const BinGeo &G, const Bins &out,
                      uint64_t *words, const BitGeo &B, hipStream_t st) {
  constexpr uint64_t tile = (uint64_t)WG * kRunL;
  const unsigned grid = (unsigned)((nk + tile - 1) / tile);
  const int aligned = ((uintptr_t)a.seq & 15u) == 0;
  hipLaunchKernelGGL((bin_kernel<W, MK, WG>), dim3(grid), dim3(WG), 0, st, a.seq, a.len, a.starts, aligned, P, G, out,
                     words, B);
  return hipGetLastError();
}

template <int SW, int SB>
hipError_t launch_apply_sb(const Bins &in, uint32_t s0, uint32_t nslices, uint32_t regions, uint64_t *words,
                           const BitGeo &B, hipStream_t st) {
  const dim3 grid(std::min(nslices, kApplyGrid << (13 - SB))), wg(1 << (SB - 4));
#define SBF_APPLY(H_, S_)                                                                                          \
  hipLaunchKernelGGL((apply_kernel<SW, H_, SB, S_>), grid, wg, 0, st, in, s0, nslices, regions, words, B); break
  switch (B.H) {
    case 1: SBF_APPLY(1, 0);
    case 2: SBF_APPLY(2, 0);
    case 3: SBF_APPLY(3, 0);
    case 4:
      if (B.s_shift == 64 - 2 * 28) {
        SBF_APPLY(4, 28);
      }
      SBF_APPLY(4, 0);
    case 5: SBF_APPLY(5, 0);
    case 6: SBF_APPLY(6, 0);
    case 7: SBF_APPLY(7, 0);
    case 8: SBF_APPLY(8, 0);
    default: return hipErrorInvalidValue;
  }
#undef SBF_APPLY
  return hipGetLastError();
}

template <int SW>
hipError_t launch_apply(int slice_words_log2, const Bins &in, uint32_t s0, uint32_t nslices, uint32_t regions,
                        uint64_t *words, const BitGeo &B, hipStream_t st) {
  return slice_words_log2 == 12 ? launch_apply_sb<SW, 12>(in, s0, nslices, regions, words, B, st)
                                : launch_apply_sb<SW, 13>(in, s0, nslices, regions, words, B, st);
}

// Expected records per k-mer of random sequence: runs of one minimizer in
// windows of w, cut after nmax k-mers.  An m-mer is the minimum of at least l
// successive windows with the probability (w-l) (1/(w+l-1) - 1/(w+l)) +
// 1/(w+l-1), from its distances to the next smaller ones on both sides (2/(w+1)
// for l = 1, the density of runs; 1/(2w-1) for l = w); each nmax k-mers of a
// run make a record.
double records_per_kmer(int w, int nmax) {
  double sum = 0;
  for (int l = 1; l <= w; l += nmax)
    sum += (w - l) * (1.0 / (w + l - 1) - 1.0 / (w + l)) + 1.0 / (w + l - 1);
  return sum;
}

// k-mers of a record: 16, fewer where their bases would reach the low 4 bits
int record_kmers(uint32_t k) { return std::min(16, 47 - (int)k); }

}  // namespace

bool runs_supported(const Geometry &g) {
  const int w = (int)(g.k - g.m + 1);
  return g.nshards <= (1ull << 32) && g.k <= 32 && g.H <= 8 && run_compiled(w, run_mk(g.k, g.m));
}

bool binned_plan(const Geometry &g, uint64_t len, bool lane_family, BinPlan &p) {
  if (len < g.k || !runs_supported(g)) return false;
  const int w = (int)(g.k - g.m + 1);
  const uint64_t nk = len - g.k + 1;
  const int words_bits = log2_of(g.nshards) + log2_of(g.shard_words);
  const uint64_t nbits = 64ull << words_bits;
  if (nk < kMinBinnedKmers) return false;
  if (nbits > (lane_family ? kLaneSmallBits : kOtherSmallBits) &&
      nk < nbits / (lane_family ? kLaneBitsPerKmer : kOtherBitsPerKmer))
    return false;
  // 32 KB slices give the apply pass four independent workgroups per CU
  // (7% faster than two of 64 KB on a 256 MiB filter); beyond 2^14 slices the
  // split pass loses more with twice the slices.
  p.slice_words_log2 = words_bits - 12 <= 14 ? 12 : 13;
  p.slice_shift = p.slice_words_log2 - log2_of(g.shard_words);
  const int slice_bits = words_bits - p.slice_words_log2;
  if (slice_bits < kMinSliceBits || slice_bits > kMaxBucketBits1 + kMaxBucketBits2) return false;
  p.bits1 = slice_bits <= kMaxBucketBits1 ? slice_bits : std::min(kMaxBucketBits1, (slice_bits + 1) / 2);
  p.bits2 = slice_bits - p.bits1;
  const int nmax = record_kmers(g.k);
  const double density = records_per_kmer(w, nmax) + 1.0 / kBinTile;
  const uint64_t buckets = 1ull << p.bits1, slices = 1ull << slice_bits;
  auto lay_out = [&](uint64_t chunk) {
    p.chunk = (chunk + kBinTile - 1) / kBinTile * kBinTile;
    // a small batch does not fill eight parts of each bucket
    p.parts = p.bits2 == 0 && p.chunk <= kOnePartKmers ? 1 : kXcds;
    const double records = density * (double)p.chunk;
    p.cap1 = region_cap(records / (double)(buckets * p.parts), 1.12);
    p.cap2 = 0;
    p.counts1 = 0;
    uint64_t bytes = align256((buckets * p.parts * 4) << kCountShift);
    p.counts2 = bytes;
    p.group = (uint32_t)buckets;
    if (p.bits2) {
      bytes += align256((slices * 4) << kCountShift);
      p.cap2 = region_cap(records / (double)slices, 1.4);
      // buckets split and applied together: at most 1 GiB of records
      const uint64_t per_bucket = (p.cap2 << p.bits2) * sizeof(Record);
      while (p.group > (uint32_t)kXcds && p.group * per_bucket > (1ull << 30)) p.group /= 2;
    }
    p.count_words = bytes / 4;
    p.rec1 = bytes;
    bytes += align256(buckets * p.parts * p.cap1 * sizeof(Record));
    p.rec2 = bytes;
    if (p.bits2) bytes += align256(((uint64_t)p.group << p.bits2) * p.cap2 * sizeof(Record));
    p.bytes = bytes;
  };
  // bits/15 k-mers take 9.6 times their records per k-mer, 2 / (w + 1), in
  // filter sizes: 1.13 at w = 16, 1.6 at w = 11, 2.73 at w = 6.  Beyond 2.75
  // times the filter plus 1 GiB (short windows into filters below 256 MiB) the
  // batch takes equal parts that stay within it; each part reads and writes the
  // whole filter, so a tighter bound would cost the larger filters time.
  uint64_t chunk = std::min(nk, std::max(nbits / 15, kMinChunkKmers));
  const uint64_t most = nbits / 8 * 11 / 4 + (1ull << 30);
  for (lay_out(chunk); p.bytes > most; lay_out(chunk))
    chunk = (uint64_t)(0.99 * (double)chunk * (double)most / (double)p.bytes);
  const uint64_t nchunks = (nk + p.chunk - 1) / p.chunk;
  if (nchunks > 1) lay_out((nk + nchunks - 1) / nchunks);
  return p.cap1 < (1ull << 31) && p.cap2 < (1ull << 31);
}

hipError_t launch_insert_binned(const Geometry &g, uint64_t *words, const SeqArgs &a, const BinPlan &p, void *scratch,
                                hipStream_t st) {
  uint8_t *s = (uint8_t *)scratch;
  const BitGeo B = bit_geo(g);
  const int mk = run_mk(g.k, g.m), w = (int)(g.k - g.m + 1);
  const RunGeo P = run_geo(g, record_kmers(g.k));
  const BinGeo G{p.slice_shift + p.bits2, 1 << p.bits1, (int)p.parts - 1};
  const Bins b1{(Record *)(s + p.rec1), (uint32_t *)(s + p.counts1), (uint32_t)p.cap1};
  const Bins b2{(Record *)(s + p.rec2), (uint32_t *)(s + p.counts2), (uint32_t)p.cap2};
  const bool wide_tile = p.bits1 == kMaxBucketBits1 && p.bits2 > 0;
  const uint64_t nk_all = a.len - g.k + 1;
  for (uint64_t c0 = 0; c0 < nk_all; c0 += p.chunk) {
    // chunks start at whole tiles, so the sequence stays 16-byte aligned and
    // the record-start bits start at a word
    const uint64_t nk = std::min(p.chunk, nk_all - c0);
    SeqArgs c = a;
    c.seq = a.seq + c0;
    c.len = nk + g.k - 1;
    c.starts = a.starts ? a.starts + c0 / 32 : nullptr;
    hipError_t e = launch_fill_u32((uint32_t *)(s + p.counts1), p.count_words, 0u, st);
    if (e != hipSuccess) return e;
    e = hipErrorInvalidValue;
#define SBF_CALL(W_, MK_) \
  if (w == W_ && mk == MK_)                                            \
    e = wide_tile ? launch_bin<W_, MK_, 512>(c, nk, P, G, b1, words, B, st) \
                  : launch_bin<W_, MK_, 256>(c, nk, P, G, b1, words, B, st);
    SBF_RUN_SETS(SBF_CALL)
#undef SBF_CALL
    if (e != hipSuccess) return e;
    const uint32_t buckets = 1u << p.bits1;
    for (uint32_t b0 = 0; b0 < buckets; b0 += p.group) {
      Bins in = b1;
      uint32_t s0 = b0, nslices = buckets, regions = p.parts;
      if (p.bits2) {
        const uint32_t tiles = ((uint32_t)p.cap1 + kSplitTile - 1) / kSplitTile;
        hipLaunchKernelGGL(split_kernel, dim3(p.group * kXcds * tiles), dim3(kSplitWG), 0, st, b1, b2, b0, tiles,
                           p.slice_shift, 1u << p.bits2, words, B);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        in = b2;
        s0 = b0 << p.bits2;
        nslices = p.group << p.bits2;
        regions = 1;
      }
      switch (g.shard_words) {
        case 4: e = launch_apply<4>(p.slice_words_log2, in, s0, nslices, regions, words, B, st); break;
        case 8: e = launch_apply<8>(p.slice_words_log2, in, s0, nslices, regions, words, B, st); break;
        default: e = launch_apply<16>(p.slice_words_log2, in, s0, nslices, regions, words, B, st); break;
      }
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace sbf
