// HIP kernels of librk for gfx950 that follow the scan: prefix sums of the
// per-tile hit counts, slab compaction, the stable radix sort by pattern id,
// per-pattern offsets, direct window hashes and the stream-read roofline probe;
// plus the dispatch of the scan kernels (rk_scan.h, instantiated per family and
// geometry in the rk_scan_*.hip units).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "rk_dev.h"
#include "rk_internal.h"
#include "rk_runtime.h"

namespace rk {

// ---------------------------------------------------------- prefix sums (u64)
// Exclusive scan of u32 counts into u64 offsets: per-block local scans that
// start from the sum of the counts before them.  Up to kScanSelf blocks add
// the counts up themselves (the last one reads 240 KB, about 3 us, less than
// one more launch), up to kScanWG blocks the per-block sums of a kernel before
// (scan_block_sums), and beyond that a single-block scan of the sums
// (scan_sums_single) hands them.  Every block is kScanWG threads: a scan of
// one step is not held back until a whole CU is free while another step's
// scan fills the chip.
//
// TILES: the counts are a count pass's hits per tile; the total, the
// overflowed tiles and whether there are any come with the scan (TileTotals),
// so that a pass needs no counters of its own, no kernel to clear them and no
// copy to read them back, and the collect finds its offsets there: 38 us for
// count and collect of a 1 MiB text, 52 to 57 us with those.  The flag travels in
// the top bit of a block's sum.
constexpr int kScanWG = 256;
constexpr int kScanPer = 16;
constexpr int kScanBlock = kScanWG * kScanPer;  // items per block
constexpr uint64_t kScanSelf = 4;              // most blocks that add up the counts before them
constexpr uint64_t kOvfBit = 1ull << 63;

// most records of tile t's slab
__device__ __forceinline__ uint32_t slab_of(const TileTotals &tt, uint64_t t) {
  uint32_t S = tt.S[0];
#pragma unroll
  for (int p = 1; p < kMaxParts; ++p)
    if (p < (int)tt.nparts && t >= tt.tile0[p]) S = tt.S[p];
  return S;
}

// a + b where the top bits are flags
__device__ __forceinline__ uint64_t add_flagged(uint64_t a, uint64_t b) {
  return (((a & ~kOvfBit) + (b & ~kOvfBit)) & ~kOvfBit) | ((a | b) & kOvfBit);
}

// The total to the host, the last thing that a scan of nb blocks writes (a
// waiting host reads it as soon as it is there): every block passes here when
// its own writes are done, and the last one to pass writes the sum, which one
// thread (mine) brings.  Called by all threads.
template <bool TILES>
__device__ __forceinline__ void put_total(const TileTotals &tt, uint64_t nb, bool mine, uint64_t sum) {
  if (mine) __hip_atomic_store(tt.ctr, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // every wave's stores are in the L2; one thread writes it back (each fence
  // does, and the four waves' own took a microsecond or two of seven)
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  if (threadIdx.x) return;
  if (nb > 1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (__hip_atomic_fetch_add(tt.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != nb - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  const uint64_t t = __hip_atomic_load(tt.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (TILES) {
    __hip_atomic_store(tt.ctr, t & ~kOvfBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(tt.host + kHostOvf, t >> 63, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  __hip_atomic_store(tt.host + kHostTotal, t & ~kOvfBit, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <bool TILES>
__global__ __launch_bounds__(kScanWG) void scan_block_sums(const uint32_t *in, uint64_t n, uint64_t *bsum,
                                                           TileTotals tt) {
  __shared__ uint64_t red[kScanWG / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock;
  uint64_t s = 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    const uint64_t i = base + (uint64_t)j * kScanWG + threadIdx.x;
    const uint32_t v = i < n ? in[i] : 0u;
    s = add_flagged(s, TILES && v > slab_of(tt, i) ? v | kOvfBit : v);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) s = add_flagged(s, __shfl_xor(s, d, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0;
    for (int i = 0; i < kScanWG / 64; ++i) t = add_flagged(t, red[i]);
    bsum[blockIdx.x] = t;
  }
}

// Single block: exclusive scan of bsum[0..nb) in place (without the flags);
// bsum[nb] = the sum with them.
template <bool TILES>
__global__ __launch_bounds__(kScanWG) void scan_sums_single(uint64_t *bsum, uint64_t nb, TileTotals tt) {
  __shared__ uint64_t wsum[kScanWG / 64];
  __shared__ uint64_t carry;
  __shared__ uint32_t any;
  if (threadIdx.x == 0) {
    carry = 0;
    any = 0;
  }
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint64_t base = 0; base < nb; base += kScanWG) {
    const uint64_t i = base + threadIdx.x;
    const uint64_t b = i < nb ? bsum[i] : 0, v = b & ~kOvfBit;
    if (TILES && (b & kOvfBit)) any = 1;
    uint64_t x = v;
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t y = __shfl_up(x, d, 64);
      if (lane >= (uint32_t)d) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint64_t before = carry, tot = 0;
    for (int k = 0; k < kScanWG / 64; ++k) {
      before += (uint32_t)k < wave ? wsum[k] : 0;
      tot += wsum[k];
    }
    if (i < nb) bsum[i] = before + x - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[nb] = any ? carry | kOvfBit : carry;
}

// How a block of scan_local gets the sum before it.
enum ScanPrefix { kPrefixScanned, kPrefixSums, kPrefixCounts };

// kPrefixScanned: bsum is already scanned; kPrefixSums: bsum holds the blocks'
// own sums (at most kScanWG blocks), each block adds those before it;
// kPrefixCounts: each block adds the counts before it (`in` 16-byte aligned).
// TILES: every block lists its overflowed tiles.  The total goes to the host
// if it is asked for (tt.host).
template <ScanPrefix FROM, bool TILES>
__global__ __launch_bounds__(kScanWG) void scan_local(const uint32_t *in, uint64_t n, const uint64_t *bsum, uint64_t nb,
                                                      uint64_t *out, TileTotals tt) {
  __shared__ uint64_t wsum[kScanWG / 64];
  __shared__ uint64_t pre[kScanWG / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock, i0 = base + (uint64_t)threadIdx.x * kScanPer;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // each thread owns kScanPer consecutive items
  uint32_t v[kScanPer];
  const bool wide = ((uintptr_t)in & 15u) == 0 && ((uintptr_t)out & 15u) == 0 && i0 + kScanPer <= n;
  if (wide) {
#pragma unroll
    for (int j = 0; j < kScanPer; j += 4) {
      const uint4 q = *(const uint4 *)(in + i0 + j);
      v[j] = q.x;
      v[j + 1] = q.y;
      v[j + 2] = q.z;
      v[j + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) v[j] = i0 + j < n ? in[i0 + j] : 0u;
  }
  if (FROM != kPrefixScanned) {
    uint64_t p = 0;
    if (FROM == kPrefixSums) {
      p = threadIdx.x < blockIdx.x ? bsum[threadIdx.x] : 0;
    } else {
      // 16 loads in flight
      const uint4 *q = (const uint4 *)in + threadIdx.x;
      uint64_t ovf = 0;
#pragma unroll 4
      for (uint32_t b = 0; b < blockIdx.x; ++b) {
#pragma unroll
        for (int j = 0; j < kScanBlock / 4 / kScanWG; ++j) {
          const uint32_t i = b * (kScanBlock / 4) + j * kScanWG;
          const uint4 c = q[i];
          p += (uint64_t)c.x + c.y + c.z + c.w;
          if (TILES && blockIdx.x == nb - 1) {
            const uint64_t t = 4ull * (i + threadIdx.x);
            if (tt.nparts == 1)
              ovf |= max(max(c.x, c.y), max(c.z, c.w)) > tt.S[0] ? kOvfBit : 0;
            else
              ovf |= c.x > slab_of(tt, t) || c.y > slab_of(tt, t + 1) || c.z > slab_of(tt, t + 2) ||
                             c.w > slab_of(tt, t + 3)
                         ? kOvfBit
                         : 0;
          }
        }
      }
      p |= ovf;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) p = add_flagged(p, __shfl_xor(p, d, 64));
    if (lane == 0) pre[wave] = p;
  }
  uint64_t s = 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) s += v[j];
  uint64_t x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(x, d, 64);
    if (lane >= (uint32_t)d) x += y;
  }
  bool any = false;  // a tile of this thread overflowed
  if (TILES) {
    uint32_t over = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) over |= v[j] > slab_of(tt, i0 + j) ? 1u << j : 0u;
    any = over != 0;
    if (tt.nparts == 1) {
      // places for a wave's tiles at once (additions to one address are served
      // one after the other)
      const uint32_t c = __builtin_popcount(over);
      uint32_t at = c;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(at, d, 64);
        if (lane >= (uint32_t)d) at += y;
      }
      uint32_t first = 0;
      if (lane == 63 && at) first = atomicAdd(tt.ovf_count, at);
      at += __shfl(first, 63, 64) - c;
      for (; over; over &= over - 1) tt.ovf_list[at++] = i0 + __builtin_ctz(over);
    } else {
      for (; over; over &= over - 1) {
        const uint64_t t = i0 + __builtin_ctz(over);
        uint32_t part = 0;
        for (uint32_t q = 1; q < tt.nparts; ++q)
          if (t >= tt.tile0[q]) part = q;
        tt.ovf_list[tt.tile0[part] + atomicAdd(tt.ovf_count + part, 1u)] = t;
      }
    }
  }
  if (lane == 63) wsum[wave] = x;
  any = __syncthreads_or(any);
  uint64_t before = 0;
  if (FROM != kPrefixScanned) {
#pragma unroll
    for (int k = 0; k < kScanWG / 64; ++k) before = add_flagged(before, pre[k]);
    any = any || (before & kOvfBit);
    before &= ~kOvfBit;
  } else {
    before = bsum[blockIdx.x];
  }
#pragma unroll
  for (int k = 0; k < kScanWG / 64; ++k) before += (uint32_t)k < wave ? wsum[k] : 0;
  uint64_t run = before + x - s;
  if (wide) {
#pragma unroll
    for (int j = 0; j < kScanPer; j += 2) {
      *(ulonglong2 *)(out + i0 + j) = make_ulonglong2(run, run + v[j]);
      run += (uint64_t)v[j] + v[j + 1];
    }
  } else {
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      if (i0 + j < n) out[i0 + j] = run;
      run += v[j];
    }
  }
  if (tt.host) {
    const bool mine = blockIdx.x == nb - 1 && threadIdx.x == kScanWG - 1;
    if (FROM == kPrefixScanned && mine) run = bsum[nb];
    put_total<TILES>(tt, nb, mine, any ? run | kOvfBit : run);
  }
}

// ------------------------------------------------------------ slab compaction
// Copy every tile's staged hits to their final offset (tiles that overflowed
// their slab are rescanned instead).  offsets1 (a single pattern's offsets,
// else null) gets {0, total} from the first thread.
//
// compact_slabs: one wave per tile.
__global__ __launch_bounds__(256) void compact_slabs(const uint32_t *counts, const uint64_t *offs, uint64_t ntiles,
                                                     const uint64_t *slabs, uint32_t slab_cap, uint64_t *out,
                                                     uint64_t *offsets1, uint64_t total) {
  if (offsets1 && blockIdx.x == 0 && threadIdx.x == 0) {
    offsets1[0] = 0;
    offsets1[1] = total;
  }
  const uint64_t t = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= ntiles) return;
  const uint32_t c = counts[t];
  if (c == 0 || c > slab_cap) return;
  const uint64_t *src = slabs + t * (uint64_t)slab_cap;
  uint64_t *dst = out + offs[t];
  for (uint32_t i = threadIdx.x & 63; i < c; i += 64) dst[i] = src[i];
}

// compact_sparse (fewer hits than tiles): a wave takes 64 tiles, a lane
// each.  A lane copies its tile itself when it holds at most kLaneCopy
// records; the wave copies the larger ones, one after the other.
constexpr uint32_t kLaneCopy = 8;

__global__ __launch_bounds__(256) void compact_sparse(const uint32_t *counts, const uint64_t *offs, uint64_t ntiles,
                                                      const uint64_t *slabs, uint32_t slab_cap, uint64_t *out,
                                                      uint64_t *offsets1, uint64_t total) {
  if (offsets1 && blockIdx.x == 0 && threadIdx.x == 0) {
    offsets1[0] = 0;
    offsets1[1] = total;
  }
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t t0 = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64, t = t0 + lane;
  const uint32_t c = t < ntiles ? counts[t] : 0u;
  const bool ok = c != 0 && c <= slab_cap;
  const uint64_t o = ok ? offs[t] : 0;
  if (ok && c <= kLaneCopy) {
    const uint64_t *src = slabs + t * (uint64_t)slab_cap;
    uint64_t r[kLaneCopy];
#pragma unroll
    for (uint32_t i = 0; i < kLaneCopy; ++i)
      if (i < c) r[i] = src[i];
#pragma unroll
    for (uint32_t i = 0; i < kLaneCopy; ++i)
      if (i < c) out[o + i] = r[i];
  }
  uint64_t big = __ballot(ok && c > kLaneCopy);
  while (big) {
    const uint32_t l = (uint32_t)__builtin_ctzll(big);
    big &= big - 1;
    const uint32_t cl = __shfl(c, (int)l, 64);
    const uint64_t ol = __shfl(o, (int)l, 64);
    const uint64_t *src = slabs + (t0 + l) * (uint64_t)slab_cap;
    for (uint32_t i = lane; i < cl; i += 64) out[ol + i] = src[i];
  }
}

// -------------------------------------------------- stable radix by pattern id
// Records are pid << 40 | x.  One DB-bit digit of the pid per pass (8 bits,
// or 9..11 when a single pass covers every pid): a histogram per block of the
// input, the starts of every (digit, block), and the scatter.
//
// The input is an array of n records, rb to a block, or (TILES) the count
// pass's staging slabs: for dense hits the compaction is skipped and the
// records of a part's tiles are read where they are, in tile order (the order
// the compaction would have produced), a block taking G consecutive tiles.
// Tile t's counts[t] records are its slab (slabs + (t - tile0) * S) when they
// fit, else those of the collect's rescan, written at tile_off[t] of the direct
// buffer.
struct RecordSrc {
  TileSrc tiles;       // TILES
  const uint64_t *in;  // else
  uint64_t n;
  uint32_t rb;
};
constexpr int kRadixR = 16;  // records per lane in flight

// A wave walks its tiles as chunks of up to 64 records of one tile, the counts
// of 64 tiles loaded at once (a lane each): a round of chunks spans as many
// tiles as it takes, so that tiles of some hundred records keep as many loads
// in flight as large ones (a histogram of 130 K records in tiles of 100 to 270:
// 28 us in rounds of one tile's records, 4 us so).
struct TileChunks {
  const TileSrc &src;
  uint64_t t, t1;         // next tile, end
  uint32_t step, i;       // tiles between this wave's, index of t in batch
  uint32_t batch;         // the lane's tile's count
  uint32_t c = 0, j = 0;  // current tile: records, records handed out
  const uint64_t *in;

  __device__ __forceinline__ TileChunks(const TileSrc &s, uint64_t first, uint64_t end, uint32_t st)
      : src(s), t(first), t1(end), step(st), in(s.slabs) {
    load_batch();
  }
  __device__ __forceinline__ void load_batch() {
    const uint64_t q = t + (uint64_t)(threadIdx.x & 63) * step;
    batch = q < t1 ? src.counts[q] : 0u;
    i = 0;
  }
  // The next N chunks: records r[u] (clamped loads, all unconditional) of the
  // lanes below lim[u]; false when there are none left.
  template <int N>
  __device__ __forceinline__ bool load(uint64_t (&r)[N], uint32_t (&lim)[N]) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      while (j >= c && t < t1) {
        if (i == 64) load_batch();
        c = __builtin_amdgcn_readlane(batch, i);
        in = c <= src.S ? src.slabs + (t - src.tile0) * src.S : src.direct + src.tile_off[t];
        j = 0;
        t += step;
        ++i;
      }
      lim[u] = min(c - j, 64u);
      // (no chunk left: a record that is there, not used)
      const uint64_t *p = lim[u] ? in + j : src.slabs;
      r[u] = p[min(threadIdx.x & 63u, max(lim[u], 1u) - 1u)];
      j += lim[u];
    }
    return lim[0] != 0;
  }
};

// Histogram of a block, block-major (block b's ND counts contiguous).  Four
// waves, wave w taking the block's tiles w, w + 4, ..., or every fourth round
// of the array's records.
template <int DB, bool TILES>
__global__ __launch_bounds__(256) void radix_hist(RecordSrc src, uint32_t shift, uint32_t *ghist) {
  constexpr uint32_t ND = 1u << DB;
  __shared__ uint32_t h[ND];
  for (uint32_t i = threadIdx.x; i < ND; i += 256) h[i] = 0;
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t rec[kRadixR];
  if constexpr (TILES) {
    const uint64_t t0 = src.tiles.tile0 + (uint64_t)blockIdx.x * src.tiles.G;
    TileChunks q(src.tiles, t0 + w, min(t0 + src.tiles.G, src.tiles.tile0 + src.tiles.ntiles), 4);
    uint32_t lim[kRadixR];
    while (q.load(rec, lim)) {
#pragma unroll
      for (int u = 0; u < kRadixR; ++u)
        if (lane < lim[u]) atomicAdd(&h[(rec[u] >> shift) & (ND - 1u)], 1u);
    }
  } else {
    const uint64_t base = (uint64_t)blockIdx.x * src.rb, end = min(base + src.rb, src.n);
    for (uint64_t j = base + w * 64u * kRadixR; j < end; j += 4 * 64u * kRadixR) {
#pragma unroll
      for (int u = 0; u < kRadixR; ++u) rec[u] = src.in[min(j + u * 64u + lane, end - 1)];
#pragma unroll
      for (int u = 0; u < kRadixR; ++u)
        if (j + u * 64u + lane < end) atomicAdd(&h[(rec[u] >> shift) & (ND - 1u)], 1u);
    }
  }
  __syncthreads();
  const uint64_t b = (TILES ? src.tiles.blk0 : 0) + blockIdx.x;
  for (uint32_t d = threadIdx.x; d < ND; d += 256) ghist[b * ND + d] = h[d];
}

// The records to their place in the output (STRIP: the last pass, which writes
// their positions only), by blocks of four waves in rounds of kSortRound
// records that are sorted in LDS first: a wave takes kSortPer chunks of the round, each lane a record of each;
// the waves count their digits, the counts of all four give every (wave, digit)
// its place in the round and every digit its place in the output, and the
// waves rank their chunks in order (the lanes of one digit found by a ballot
// per bit).  Then consecutive lanes write consecutive records of a digit.
// Bound by the writes: a wave that writes 64 records as it finds them makes 64
// requests, most to lines of their own, which each leave the L2 before the
// next record of the digit comes (35 M records of 1,024 digits: 253 us, 167 us
// sorted; with rounds of 4,096 records, which leave room for two blocks a CU
// instead of three, 200 us).
constexpr uint32_t kSortPer = 12, kSortRound = 4 * 64 * kSortPer;

// Lanes (of the active ones) whose low DB bits of d are this lane's: four
// instructions a bit, the bit spread over a word, its ballot, and both halves
// of the mask without the lanes where the ballot differs.
template <int DB>
__device__ __forceinline__ uint64_t same_digit(uint32_t d) {
  const uint64_t all = __ballot(1);
  uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
#pragma unroll
  for (int b = 0; b < DB; ++b) {
    const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);
    const uint64_t m = __ballot(mine != 0);
    lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, mine, 0x90);          // lo & ~(m ^ mine)
    hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), mine, 0x90);
  }
  return (uint64_t)hi << 32 | lo;
}

template <int DB, bool TILES, bool STRIP>
__global__ __launch_bounds__(256) void radix_scatter(RecordSrc rsrc, uint32_t shift, const uint64_t *goff,
                                                     uint64_t *out) {
  constexpr uint32_t ND = 1u << DB, PER = ND / 256;
  __shared__ uint64_t sorted[kSortRound];
  __shared__ uint64_t delta[ND];           // a digit's place in the output less its place in the round
  __shared__ uint32_t cnt[4][ND];          // counts, then next places in the round
  __shared__ uint32_t first[TILES ? kSortTiles : 1];  // chunks of the block's tiles before each
  __shared__ uint32_t count[TILES ? kSortTiles : 1];  // records of each
  __shared__ uint32_t wsum[4];
  const uint32_t lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TileSrc &src = rsrc.tiles;
  const uint64_t base0 = (uint64_t)blockIdx.x * rsrc.rb;  // the array's first record
  const uint32_t nrec = TILES ? 0 : (uint32_t)min((uint64_t)rsrc.rb, rsrc.n - base0);
  const uint64_t t0 = src.tile0 + (uint64_t)blockIdx.x * src.G;
  const uint32_t ng = TILES ? (uint32_t)min((uint64_t)src.G, src.tile0 + src.ntiles - t0) : 0;
  // exclusive prefix sum over the block of each thread's v; *all: the sum
  auto block_scan = [&](uint32_t v, uint32_t *all) __attribute__((always_inline)) -> uint32_t {
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= (uint32_t)d) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      before += i < w ? wsum[i] : 0;
      sum += wsum[i];
    }
    *all = sum;
    return before + x - v;
  };
  uint32_t nch = (nrec + 63) / 64;
  if constexpr (TILES) {
    constexpr uint32_t Q = (kSortTiles + 255) / 256;
    uint32_t c[Q], v = 0;
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {
      const uint32_t i = threadIdx.x * Q + q;
      c[q] = i < ng ? src.counts[t0 + i] : 0u;
      if (i < kSortTiles) count[i] = c[q];
      v += (c[q] + 63) / 64;
    }
    uint32_t at = block_scan(v, &nch);
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {
      if (threadIdx.x * Q + q < kSortTiles) first[threadIdx.x * Q + q] = at;
      at += (c[q] + 63) / 64;
    }
  }
  uint64_t place[PER];  // next place in the output of digits threadIdx.x * PER ..
#pragma unroll
  for (uint32_t q = 0; q < PER; ++q) place[q] = goff[((TILES ? src.blk0 : 0) + blockIdx.x) * ND + threadIdx.x * PER + q];
  __syncthreads();
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  for (uint32_t q0 = 0; q0 < nch; q0 += 4 * kSortPer) {
    // the wave's chunks, one looked up by each of its first lanes
    const uint64_t *p = TILES ? src.slabs : rsrc.in;  // (no chunk: a record that is there, not used)
    uint32_t len = 0;
    const uint32_t q = q0 + w * kSortPer + min(lane, kSortPer - 1);
    if (q < nch) {
      if constexpr (TILES) {
        uint32_t lo = 0, hi = ng;
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (first[mid] <= q) lo = mid;
          else hi = mid;
        }
        const uint32_t c = count[lo], off = (q - first[lo]) * 64;
        const uint64_t t = t0 + lo;
        p = (c <= src.S ? src.slabs + (t - src.tile0) * src.S : src.direct + src.tile_off[t]) + off;
        len = min(c - off, 64u);
      } else {
        p = rsrc.in + base0 + 64ull * q;
        len = min(nrec - 64 * q, 64u);
      }
    }
    uint64_t rec[kSortPer];
    uint32_t lim[kSortPer];
#pragma unroll
    for (uint32_t u = 0; u < kSortPer; ++u) {
      lim[u] = __builtin_amdgcn_readlane(len, u);
      const uint64_t at = (uint64_t)__builtin_amdgcn_readlane((uint32_t)((uint64_t)p >> 32), u) << 32 |
                          (uint32_t)__builtin_amdgcn_readlane((uint32_t)(uint64_t)p, u);
      // (known to be global memory: a flat load would wait on LDS too)
      rec[u] = ((const __attribute__((address_space(1))) uint64_t *)at)[min(lane, max(lim[u], 1u) - 1u)];
    }
    for (uint32_t d = lane; d < ND; d += 64) cnt[w][d] = 0;
#pragma unroll
    for (uint32_t u = 0; u < kSortPer; ++u)
      if (lane < lim[u]) atomicAdd(&cnt[w][(uint32_t)(rec[u] >> shift) & (ND - 1u)], 1u);
    __syncthreads();
    uint32_t tot[PER], v = 0, n;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
      const uint32_t d = threadIdx.x * PER + i;
      tot[i] = cnt[0][d] + cnt[1][d] + cnt[2][d] + cnt[3][d];
      v += tot[i];
    }
    uint32_t at = block_scan(v, &n);
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
      const uint32_t d = threadIdx.x * PER + i;
      delta[d] = place[i] - at;
      place[i] += tot[i];
#pragma unroll
      for (uint32_t x = 0; x < 4; ++x) {
        const uint32_t c = cnt[x][d];
        cnt[x][d] = at;
        at += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kSortPer; ++u) {
      if (lane >= lim[u]) continue;
      const uint32_t d = (uint32_t)(rec[u] >> shift) & (ND - 1u);
      const uint64_t peers = same_digit<DB>(d);
      const uint32_t base = cnt[w][d];
      sorted[base + __builtin_popcountll(peers & lt_mask)] = rec[u];
      if ((peers >> lane) == 1ull) cnt[w][d] = base + __builtin_popcountll(peers);
    }
    __syncthreads();
    // (the next round writes delta and sorted only after its barriers)
    for (uint32_t i = threadIdx.x; i < n; i += 256) {
      const uint64_t r = sorted[i];
      out[delta[(uint32_t)(r >> shift) & (ND - 1u)] + i] = STRIP ? r & kPosMask : r;
    }
  }
}

// Start of every (digit, block) of a pass from its block-major
// histogram h[b][d] (nblk blocks, nd digits).  The blocks go in chunks of
// kDigitChunk: digit_chunk_sums sums each chunk's rows (csum[c][d]);
// digit_chunk_starts scans every digit's column over the chunks (crel[c][d]:
// the counts of digit d in the chunks before c) and writes the digit totals;
// digit_block_starts scans the totals across digits (where each digit starts)
// and writes goff[b][d] = that start + crel + the counts of digit d in the
// chunk's blocks before b.  Every access walks rows, 64 lanes over
// consecutive digits.
constexpr uint32_t kDigitChunk = 32;
constexpr uint32_t kDigitWaves = 4;  // waves of digit_chunk_starts, one block per 64 digits

__global__ __launch_bounds__(256) void digit_chunk_sums(const uint32_t *__restrict__ h, uint64_t nblk, uint32_t nd,
                                                        uint32_t *__restrict__ csum) {
  const uint64_t b0 = (uint64_t)blockIdx.x * kDigitChunk, b1 = min(b0 + kDigitChunk, nblk);
  for (uint32_t d = threadIdx.x; d < nd; d += 256) {
    uint32_t t = 0;
#pragma unroll 8
    for (uint64_t b = b0; b < b1; ++b) t += h[b * nd + d];
    csum[(uint64_t)blockIdx.x * nd + d] = t;
  }
}

// Block x covers digits 64x..64x+63 (one per lane); wave w takes a
// contiguous run of chunks, sums it, then writes its chunks' exclusive
// column prefixes from the sums of the waves before it.
__global__ __launch_bounds__(64 * kDigitWaves) void digit_chunk_starts(const uint32_t *__restrict__ csum,
                                                                        uint64_t nchunk, uint32_t nd,
                                                                        uint64_t *__restrict__ crel,
                                                                        uint64_t *__restrict__ dtot) {
  __shared__ uint64_t part[kDigitWaves][64];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t d = blockIdx.x * 64 + lane;
  const uint64_t per = (nchunk + kDigitWaves - 1) / kDigitWaves;
  const uint64_t c0 = min((uint64_t)w * per, nchunk), c1 = min(c0 + per, nchunk);
  uint64_t t = 0;
  if (d < nd)
#pragma unroll 8
    for (uint64_t c = c0; c < c1; ++c) t += csum[c * nd + d];
  part[w][lane] = t;
  __syncthreads();
  uint64_t run = 0;
  for (uint32_t i = 0; i < w; ++i) run += part[i][lane];
  if (d < nd) {
    for (uint64_t c = c0; c < c1; ++c) {
      crel[c * nd + d] = run;
      run += csum[c * nd + d];
    }
    if (w == kDigitWaves - 1) dtot[d] = run;
  }
}

// Chunk x's blocks, digits 256y..256y+255.  Every block scans the digit
// totals itself (nd is at most 2048); block (0, 0) also writes offsets, if
// asked for (the digit is the whole pid of a one-pass sort): offsets[j] = start
// of pid j, offsets[k] = n.
__global__ __launch_bounds__(256) void digit_block_starts(const uint32_t *__restrict__ h, uint64_t nblk, uint32_t nd,
                                                          const uint64_t *__restrict__ crel,
                                                          const uint64_t *__restrict__ dtot,
                                                          uint64_t *__restrict__ goff, uint32_t k, uint64_t n,
                                                          uint64_t *__restrict__ offsets) {
  constexpr uint32_t kPer = 8;  // digits per thread of the totals' scan (256 * 8 = 2048)
  __shared__ uint64_t start[256 * kPer];
  __shared__ uint64_t wsum[4];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t v[kPer], x = 0;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    const uint32_t d = threadIdx.x * kPer + i;
    v[i] = d < nd ? dtot[d] : 0;
    x += v[i];
  }
  const uint64_t mine = x;
  for (int sh = 1; sh < 64; sh <<= 1) {
    const uint64_t y = __shfl_up(x, sh, 64);
    if (lane >= (uint32_t)sh) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint64_t before = x - mine;
  for (uint32_t i = 0; i < wave; ++i) before += wsum[i];
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    start[threadIdx.x * kPer + i] = before;
    before += v[i];
  }
  __syncthreads();
  if (offsets && blockIdx.x == 0 && blockIdx.y == 0)
    for (uint32_t j = threadIdx.x; j <= k; j += 256) offsets[j] = j < k ? start[j] : n;
  const uint64_t b0 = (uint64_t)blockIdx.x * kDigitChunk, b1 = min(b0 + kDigitChunk, nblk);
  const uint32_t d = blockIdx.y * 256 + threadIdx.x;
  if (d >= nd) return;
  uint64_t run = start[d] + crel[(uint64_t)blockIdx.x * nd + d];
  uint32_t c[kDigitChunk];
#pragma unroll
  for (uint32_t i = 0; i < kDigitChunk; ++i) c[i] = b0 + i < b1 ? h[(b0 + i) * nd + d] : 0;
#pragma unroll
  for (uint32_t i = 0; i < kDigitChunk; ++i) {
    if (b0 + i < b1) goff[(b0 + i) * nd + d] = run;
    run += c[i];
  }
}

// All of it in one block, for up to kDigitOne blocks (one chunk): two launches
// less, for histograms that a block reads in a few microseconds.
constexpr uint32_t kDigitOne = 32;

__global__ __launch_bounds__(256) void digit_starts_one(const uint32_t *__restrict__ h, uint32_t nblk, uint32_t nd,
                                                        uint64_t *__restrict__ goff, uint32_t k, uint64_t n,
                                                        uint64_t *__restrict__ offsets) {
  constexpr uint32_t kPer = 8;  // digits per thread of the totals' scan (256 * 8 = 2048)
  __shared__ uint64_t start[256 * kPer];
  __shared__ uint64_t wsum[4];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t d = threadIdx.x; d < 256 * kPer; d += 256) {
    uint64_t t = 0;
    if (d < nd) {
#pragma unroll 8
      for (uint32_t b = 0; b < nblk; ++b) t += h[b * nd + d];
    }
    start[d] = t;
  }
  __syncthreads();
  uint64_t v[kPer], x = 0;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    v[i] = start[threadIdx.x * kPer + i];
    x += v[i];
  }
  const uint64_t mine = x;
  for (int sh = 1; sh < 64; sh <<= 1) {
    const uint64_t y = __shfl_up(x, sh, 64);
    if (lane >= (uint32_t)sh) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint64_t before = x - mine;
  for (uint32_t i = 0; i < wave; ++i) before += wsum[i];
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    start[threadIdx.x * kPer + i] = before;
    before += v[i];
  }
  __syncthreads();
  if (offsets)
    for (uint32_t j = threadIdx.x; j <= k; j += 256) offsets[j] = j < k ? start[j] : n;
  for (uint32_t d = threadIdx.x; d < nd; d += 256) {
    uint64_t run = start[d];
#pragma unroll 8
    for (uint32_t b = 0; b < nblk; ++b) {
      goff[b * nd + d] = run;
      run += h[b * nd + d];
    }
  }
}

// The records sorted by pid to offsets (a binary search per pid, the first
// blocks) and positions (the others, two records per thread).
__global__ __launch_bounds__(256) void sorted_results(const uint64_t *sorted, uint64_t n, uint32_t k, uint32_t oblocks,
                                                      uint64_t *offsets, uint64_t *pos) {
  if (blockIdx.x >= oblocks) {
    const uint64_t i = ((uint64_t)(blockIdx.x - oblocks) * 256 + threadIdx.x) * 2;
    if (i < n) pos[i] = sorted[i] & kPosMask;
    if (i + 1 < n) pos[i + 1] = sorted[i + 1] & kPosMask;
    return;
  }
  const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (j > k) return;
  if (j == k) {
    offsets[k] = n;
    return;
  }
  uint64_t lo = 0, hi = n;
  while (lo < hi) {
    const uint64_t mid = (lo + hi) >> 1;
    if ((sorted[mid] >> kPosBits) < j) lo = mid + 1;
    else hi = mid;
  }
  offsets[j] = lo;
}

// ------------------------------------------------------------- window hashes
__global__ void window_hashes_kernel(const uint8_t *text, uint64_t n, uint32_t m, const uint64_t *xs, uint64_t cnt,
                                     uint64_t *out) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  const uint64_t x = xs[i];
  if (m == 0 || x > n || n - x < m) {
    out[i] = ~0ull;
    return;
  }
  uint64_t s = 0;
  for (uint32_t j = 0; j < m; ++j) s = mul256_lazy(s) + text[x + j];
  out[i] = canon(s);
}

__global__ void fill_u32_kernel(uint32_t *p, uint64_t words, uint32_t v) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t *p, uint64_t words, uint32_t v, hipStream_t s) {
  if (words == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((uint32_t)((words + 255) / 256)), dim3(256), 0, s, p, words, v);
  return hipGetLastError();
}

// exclusive scan of n u32 counts into u64 offsets; tmp holds scan_tmp_words(n)
// u64; *total (optional, pinned host memory) receives the sum, after everything
// else, with *done a counter at zero
uint64_t scan_tmp_words(uint64_t n) { return (n + kScanBlock - 1) / kScanBlock + 2; }

template <bool TILES>
static hipError_t exclusive_scan(const uint32_t *in, uint64_t n, uint64_t *out, uint64_t *tmp, const TileTotals &tt,
                                 hipStream_t s) {
  // (nothing to scan: one block writes the total)
  const uint64_t nb = std::max<uint64_t>((n + kScanBlock - 1) / kScanBlock, tt.host ? 1 : 0);
  const dim3 g((uint32_t)nb), b(kScanWG);
  if (nb == 0) return hipSuccess;
  if (nb <= kScanSelf && ((uintptr_t)in & 15u) == 0) {
    hipLaunchKernelGGL((scan_local<kPrefixCounts, TILES>), g, b, 0, s, in, n, tmp, nb, out, tt);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((scan_block_sums<TILES>), g, b, 0, s, in, n, tmp, tt);
  if (nb <= (uint64_t)kScanWG) {
    hipLaunchKernelGGL((scan_local<kPrefixSums, TILES>), g, b, 0, s, in, n, tmp, nb, out, tt);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((scan_sums_single<TILES>), dim3(1), b, 0, s, tmp, nb, tt);
  hipLaunchKernelGGL((scan_local<kPrefixScanned, TILES>), g, b, 0, s, in, n, tmp, nb, out, tt);
  return hipGetLastError();
}

hipError_t launch_exclusive_scan(const uint32_t *in, uint64_t n, uint64_t *out, uint64_t *tmp, uint64_t *total,
                                 uint32_t *done, hipStream_t s) {
  TileTotals tt = {};
  tt.host = total;
  tt.done = done;
  tt.ctr = tmp + (n + kScanBlock - 1) / kScanBlock + 1;
  return exclusive_scan<false>(in, n, out, tmp, tt, s);
}

hipError_t launch_tile_scan(const uint32_t *in, uint64_t n, uint64_t *out, uint64_t *tmp, const TileTotals &tt,
                            hipStream_t s) {
  return exclusive_scan<true>(in, n, out, tmp, tt, s);
}

hipError_t launch_compact(const uint32_t *counts, const uint64_t *offs, uint64_t ntiles, const uint64_t *slabs,
                          uint32_t slab_cap, uint64_t *out, bool sparse, uint64_t *offsets1, uint64_t total,
                          hipStream_t s) {
  if (ntiles == 0) return hipSuccess;
  if (sparse)
    hipLaunchKernelGGL(compact_sparse, dim3((uint32_t)((ntiles + 255) / 256)), dim3(256), 0, s, counts, offs, ntiles,
                       slabs, slab_cap, out, offsets1, total);
  else
    hipLaunchKernelGGL(compact_slabs, dim3((uint32_t)((ntiles + 3) / 4)), dim3(256), 0, s, counts, offs, ntiles,
                       slabs, slab_cap, out, offsets1, total);
  return hipGetLastError();
}

// Starts of every (digit, block) of a pass into goff (block-major, like h) and,
// of a one-pass sort, of every digit into offsets (k + 1 entries; else null); cs: work of
// digit_cs_bytes(nblk * nd, nd) bytes.
static hipError_t digit_offsets(const uint32_t *h, uint64_t nblk, uint32_t nd, uint64_t *goff, uint8_t *cs,
                                uint32_t k, uint64_t n, uint64_t *offsets, hipStream_t s) {
  if (nd > 2048 || (offsets && k > nd)) return hipErrorInvalidValue;
  if (nblk <= kDigitOne) {
    hipLaunchKernelGGL(digit_starts_one, dim3(1), dim3(256), 0, s, h, (uint32_t)nblk, nd, goff, k, n, offsets);
    return hipGetLastError();
  }
  const uint64_t nchunk = (nblk + kDigitChunk - 1) / kDigitChunk;
  uint32_t *csum = (uint32_t *)cs;
  uint64_t *crel = (uint64_t *)(cs + ((nchunk * nd * 4 + 255) & ~255ull));
  uint64_t *dtot = crel + nchunk * nd;
  hipLaunchKernelGGL(digit_chunk_sums, dim3((uint32_t)nchunk), dim3(256), 0, s, h, nblk, nd, csum);
  hipLaunchKernelGGL(digit_chunk_starts, dim3((nd + 63) / 64), dim3(64 * kDigitWaves), 0, s, csum, nchunk, nd, crel,
                     dtot);
  hipLaunchKernelGGL(digit_block_starts, dim3((uint32_t)nchunk, (nd + 255) / 256), dim3(256), 0, s, h, nblk, nd, crel,
                     dtot, goff, k, n, offsets);
  return hipGetLastError();
}

uint64_t digit_cs_bytes(uint64_t nh, uint32_t nd) {
  const uint64_t cells = nh / kDigitChunk + nd;  // at least nchunk * nd for any nblk * nd <= nh
  return ((cells * 4 + 255) & ~255ull) + cells * 8 + nd * 8;
}

// Records per block of a pass of `bits` bits: 16,384 once there are 1,024 such
// blocks (longer runs per digit and block make the scatter's writes fuller
// lines; 32,768 leave too few blocks for the chip: 188 us against 167 for 35 M
// records of 1,024 digits), down to 2,048 to 8,192 for fewer (more blocks at
// work; a block's histogram and its scan then cost about as much as its
// records).
uint32_t radix_block_records(uint64_t n, uint32_t bits) {
  const uint64_t least = std::min<uint64_t>(8192, 8ull << bits);
  return (uint32_t)std::min<uint64_t>(16384, std::max<uint64_t>(least, n / 1024));
}

// One pass over the parts' tiles (nparts > 0, nblk blocks in all) or over `in`.
template <int DB, bool STRIP>
static hipError_t radix_pass(const TileSrc *parts, uint32_t nparts, uint64_t nblk, const uint64_t *in, uint64_t n,
                             uint32_t shift, uint32_t *ghist, uint64_t *goff, uint8_t *cs, uint32_t k,
                             uint64_t *offsets, uint64_t *out, hipStream_t s) {
  RecordSrc r = {};
  r.in = in;
  r.n = n;
  r.rb = radix_block_records(n, DB);
  if (!nparts) {
    nblk = (n + r.rb - 1) / r.rb;
    hipLaunchKernelGGL((radix_hist<DB, false>), dim3((uint32_t)nblk), dim3(256), 0, s, r, shift, ghist);
  }
  auto blocks = [](const TileSrc &t) { return dim3((uint32_t)((t.ntiles + t.G - 1) / t.G)); };
  for (uint32_t i = 0; i < nparts; ++i) {
    r.tiles = parts[i];
    if (r.tiles.ntiles)
      hipLaunchKernelGGL((radix_hist<DB, true>), blocks(r.tiles), dim3(256), 0, s, r, shift, ghist);
  }
  hipError_t e = digit_offsets(ghist, nblk, 1u << DB, goff, cs, k, n, offsets, s);
  if (e != hipSuccess) return e;
  if (!nparts)
    hipLaunchKernelGGL((radix_scatter<DB, false, STRIP>), dim3((uint32_t)nblk), dim3(256), 0, s, r, shift, goff, out);
  for (uint32_t i = 0; i < nparts; ++i) {
    r.tiles = parts[i];
    if (r.tiles.ntiles)
      hipLaunchKernelGGL((radix_scatter<DB, true, STRIP>), blocks(r.tiles), dim3(256), 0, s, r, shift, goff, out);
  }
  return hipGetLastError();
}

// Stable sort of n records by pid (bits 40.. of each record, pids below k),
// written out as per-pid offsets (k+1) and positions (n).  Up to 2,048 pids:
// one pass whose digit is the whole pid, scattering positions straight to
// their final place, with the offsets read from the scanned histogram.
// Beyond: 8-bit passes ping-ponging between b and a, then the offsets and
// positions from the sorted records.  The first pass reads the parts'
// tiles (nparts > 0; parts[i].G and blk0 set by the caller, nblk blocks in all)
// or a.  ghist and goff hold 2^DB entries per block of each pass.
hipError_t launch_radix(const TileSrc *parts, uint32_t nparts, uint64_t nblk, uint64_t *a, uint64_t *b, uint64_t n,
                        uint32_t k, uint32_t *ghist, uint64_t *goff, uint8_t *cs, uint64_t *offsets,
                        uint64_t *positions, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint32_t bits = pid_bits(k);
#define RK_ONE_PASS(DB) \
  radix_pass<DB, true>(parts, nparts, nblk, a, n, kPosBits, ghist, goff, cs, k, offsets, positions, s)
  if (bits <= 8) return RK_ONE_PASS(8);
  if (bits == 9) return RK_ONE_PASS(9);
  if (bits == 10) return RK_ONE_PASS(10);
  if (bits == 11) return RK_ONE_PASS(11);
#undef RK_ONE_PASS
  uint64_t *src = a, *dst = b;
  for (uint32_t done = 0; done < bits; done += 8) {
    hipError_t e = radix_pass<8, false>(parts, done ? 0 : nparts, nblk, src, n, kPosBits + done, ghist, goff, cs, k,
                                        nullptr, dst, s);
    if (e != hipSuccess) return e;
    uint64_t *t = src;
    src = dst;
    dst = t;
  }
  const uint32_t oblocks = (k + 256) / 256;  // k + 1 offsets
  hipLaunchKernelGGL(sorted_results, dim3(oblocks + (uint32_t)((n + 511) / 512)), dim3(256), 0, s, src, n, k, oblocks,
                     offsets, positions);
  return hipGetLastError();
}

hipError_t launch_window_hashes(const uint8_t *text, uint64_t n, uint32_t m, const uint64_t *xs, uint64_t cnt,
                                uint64_t *out, hipStream_t s) {
  if (cnt == 0) return hipSuccess;
  hipLaunchKernelGGL(window_hashes_kernel, dim3((uint32_t)((cnt + 255) / 256)), dim3(256), 0, s, text, n, m, xs, cnt,
                     out);
  return hipGetLastError();
}

// --------------------------------------------------------- scan dispatch
#define RK_SCAN_DISPATCH(fam, cfg, CALL)                       \
  switch (fam * 16 + cfg) {                                    \
    case kFamScreen1 * 16 + 0: return ScanGeom<kFamScreen1, 0>::CALL; \
    case kFamScreen1 * 16 + 1: return ScanGeom<kFamScreen1, 1>::CALL; \
    case kFamScreen1 * 16 + 2: return ScanGeom<kFamScreen1, 2>::CALL; \
    case kFamScreen1 * 16 + 3: return ScanGeom<kFamScreen1, 3>::CALL; \
    case kFamScreen * 16 + 0: return ScanGeom<kFamScreen, 0>::CALL;   \
    case kFamScreen * 16 + 1: return ScanGeom<kFamScreen, 1>::CALL;   \
    case kFamScreen * 16 + 2: return ScanGeom<kFamScreen, 2>::CALL;   \
    case kFamScreen * 16 + 3: return ScanGeom<kFamScreen, 3>::CALL;   \
    case kFamExact * 16 + 0: return ScanGeom<kFamExact, 0>::CALL;     \
    case kFamExact * 16 + 1: return ScanGeom<kFamExact, 1>::CALL;     \
    case kFamExact * 16 + 2: return ScanGeom<kFamExact, 2>::CALL;     \
    case kFamExact * 16 + 3: return ScanGeom<kFamExact, 3>::CALL;     \
    default: return hipErrorInvalidValue;                      \
  }

hipError_t scan_fit(int cfg, int fam, uint32_t img_cap, uint32_t block, ScanFit *f) {
  RK_SCAN_DISPATCH(fam, cfg, fit(img_cap, block, f))
}

hipError_t launch_scan(int cfg, int fam, const ScanParams &p, uint32_t grid, uint32_t block, hipStream_t s) {
  RK_SCAN_DISPATCH(fam, cfg, launch(p, grid, block, s))
}

// Launches (p != nullptr) or sizes (occupancy into *blocks) the single-bucket
// scan of geometry cfg and family fam.
hipError_t list_scan(int cfg, int fam, const ListParams *p, uint32_t grid, hipStream_t s, int *blocks) {
  RK_SCAN_DISPATCH(fam, cfg, list(p, grid, s, blocks))
}

static hipError_t prepare_scan_kernel(int fam, int cfg) { RK_SCAN_DISPATCH(fam, cfg, prepare()) }
static hipError_t prepare_list_kernel(int fam, int cfg) { RK_SCAN_DISPATCH(fam, cfg, list_prepare()) }

// Raises the dynamic LDS limit of every scan kernel once, outside any stream
// capture (a graph capture must not run first-time setup calls).
void prepare_scan_kernels() {
  for (int fam : {kFamScreen1, kFamScreen, kFamExact})
    for (int cfg = 0; cfg < kNumTileCfg; ++cfg) {
      (void)prepare_scan_kernel(fam, cfg);
      (void)prepare_list_kernel(fam, cfg);
    }
}

// ----------------------------------------------------- stream-read roofline
// Reads every 16-byte block of data[0..n) once (the scan's load width, fully
// coalesced, grid-stride) and folds it into one word per workgroup so that
// nothing is optimised away: the read-bandwidth ceiling the scan is held to.
// Each wave streams 1 KiB chunks (gw, gw + TW, ...; TW waves in the grid)
// into a private LDS ring of two sets of 8 slots with non-temporal LDS-DMA
// loads, the way the scans load their tiles: a batch of 8 is issued, then the
// previous batch is waited for and XOR-folded from LDS (every byte is read).
// Tail bytes (n % 1024) are folded by the first workgroup's first wave.
__device__ __forceinline__ uint32_t sr_lds(const void *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint8_t *)p;
}

__device__ __forceinline__ void sr_dma(const void *g, uint32_t m0) {
  __asm__ volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(g), "{m0}"(m0) : "memory");
}

__global__ __launch_bounds__(256) void stream_read_kernel(const uint8_t *data, uint64_t n, uint32_t *out) {
  __shared__ __attribute__((aligned(16))) uint8_t ring[4][2][8][1024];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t nchunks = n / 1024, gw = (uint64_t)blockIdx.x * 4 + w, tw = (uint64_t)gridDim.x * 4;
  uint32_t acc = 0, par = 0, prev = 0;
  for (uint64_t c0 = gw; c0 < nchunks; c0 += 8 * tw) {
    // the previous batch's reads of the set about to be refilled are done
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    uint32_t cnt = 0;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const uint64_t c = c0 + j * tw;
      if (c < nchunks) {
        sr_dma(data + c * 1024 + 16 * lane, __builtin_amdgcn_readfirstlane(sr_lds(&ring[w][par][j][0])));
        ++cnt;
      }
    }
    if (cnt == 8)
      __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8): the previous batch has landed
    else
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __asm__ volatile("" ::: "memory");
    for (uint32_t j = 0; j < prev; ++j) {
      const uint4 v = *(const uint4 *)&ring[w][par ^ 1][j][16 * lane];
      acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    prev = cnt;
    par ^= 1;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __asm__ volatile("" ::: "memory");
  for (uint32_t j = 0; j < prev; ++j) {
    const uint4 v = *(const uint4 *)&ring[w][par ^ 1][j][16 * lane];
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (blockIdx.x == 0 && w == 0 && nchunks * 1024 + 16 * lane < n) {
    const uint4 v = *(const uint4 *)(data + nchunks * 1024 + 16 * lane);
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  for (int d = 32; d >= 1; d >>= 1) acc ^= __shfl_xor(acc, d, 64);
  __shared__ uint32_t red[4];
  if (lane == 0) red[w] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = red[0] ^ red[1] ^ red[2] ^ red[3];
}

hipError_t launch_stream_read(const void *data, uint64_t n, uint32_t *out, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, s, (const uint8_t *)data, n, out);
  return hipGetLastError();
}

}  // namespace rk
