// The paper's own GPU procedure (Shah & Oza, Sec. 3.1), kept as a mode of its
// own so that the paper's experiments (threads per block, pattern length) can
// be rerun on MI355X next to the tiled scans:
//   - threads over text offsets x, numbered (block index) * (threads per block)
//     + thread index, the block index formed from a grid of up to three
//     dimensions as the paper does; a thread takes 16 consecutive offsets (the
//     paper's takes one);
//   - for each, it hashes the m bytes at T + x with the paper's shift-and-add
//     hash h <- (h << 1) + c, read straight from device memory (no tile), in a
//     32-bit word (the paper leaves the word width open; the hash is the
//     polynomial hash with d = 2, q = 2^32, in which all but the window's last
//     32 bytes have weight 0); the hash of a thread's first offset comes from
//     the window's bytes, the others' from it;
//   - if the hash equals the pattern's (computed once on the host) the m bytes
//     are compared, and the result array gets 1 at x for a match.
// Deviations: the result byte is written for every x (0 or 1), so the array
// needs no clearing; the device-side print of each match is not done.  The
// positions of the set bytes are gathered afterwards (rk_paper_positions) in
// ascending order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "../../include/rk.h"
#include "rk_dev.h"
#include "rk_internal.h"
#include "rk_runtime.h"

namespace rk {

// Offsets per thread: 16 consecutive ones, whose windows share their dwords.
constexpr uint32_t kPaperPer = 16;
constexpr uint32_t kPaperDwords = 13;  // hold the 31 + 16 bytes hashed, from any byte of the first

// Hashes of 16 consecutive windows whose last 32 bytes are bytes i..i+31 of e
// (i < 16): the first from its words K0..7 (word K0's bytes with the weights of
// w0, 0 before the window, the others with 8, 4, 2, 1), the others from the one
// before: 2 h + c, less the byte that leaves (SHORT: windows of fewer than 32
// bytes; the byte's weight is 0 in a longer one), which is byte out of word K0
// for the second window.
template <int K0, bool SHORT>
__device__ __forceinline__ void window_hashes16(const uint32_t *e, uint32_t w0, uint32_t out, uint32_t m,
                                                uint32_t *h) {
  uint32_t x = __builtin_amdgcn_udot4(e[K0], w0, 0u, false);
#pragma unroll
  for (int j = K0 + 1; j < 8; ++j) x = __builtin_amdgcn_udot4(e[j], 0x01020408u, x << 4, false);
  h[0] = x;
  uint32_t o[4] = {};
  if (SHORT) {
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = __builtin_amdgcn_alignbyte(e[K0 + j + 1], e[K0 + j], out);
  }
#pragma unroll
  for (int i = 1; i < 16; ++i) {
    x = (x << 1) + byte_at(e, 31 + i);
    if (SHORT) x -= byte_at(o, i - 1) << m;
    h[i] = x;
  }
}

// Every offset's hash from the text in device memory.  h <- (h << 1) + c in a
// 32-bit word gives byte i of the window the weight 2^(m-1-i), which is 0 for
// all but the last 32 bytes: those of a thread's first window are hashed four
// bytes at a time (the weights 8, 4, 2, 1 of a word's bytes are one byte dot
// product, word k back from the end weighs 16^k), the other windows follow from
// it, and their flags leave in one store.  Bound by the read of the text and the
// write of the flags: 320 MB with m = 25 at 1,024 threads per block take
// 0.145 ms (nothing but the two would take 0.11 ms); 0.19 ms with every window
// hashed from its words, one offset per thread took 1.30 ms with the same
// dwords and products (the blocks' start and load latency), 1.87 ms with a byte
// load per hashed byte (m = 800: 29 ms).
__global__ void paper_kernel(const uint8_t *T, uint64_t n, uint64_t nwin, const uint8_t *P, uint32_t m, uint32_t hx,
                             uint8_t *result, uint32_t *hash_out) {
  const uint64_t block = blockIdx.x + (uint64_t)blockIdx.y * gridDim.x + (uint64_t)gridDim.x * gridDim.y * blockIdx.z;
  const uint64_t x0 = (block * blockDim.x + threadIdx.x) * kPaperPer;
  if (x0 >= nwin) return;  // x <= n - m
  // the 32 bytes ending at each window's end: bytes x0 + m - 32 + [0, 47) of
  // the text, of which those before a shorter window weigh 0
  const uint32_t mis = (uint32_t)((uintptr_t)T + m) & 3u;  // of that byte, the same for every thread
  const int64_t base = (int64_t)x0 + m - 32 - mis;         // its dword, as an offset from T
  const int64_t lo = -(int64_t)((uintptr_t)T & 3u), hi = (int64_t)n - 1 - (int64_t)(((uintptr_t)T + n - 1) & 3u);
  uint32_t d[kPaperDwords], e[kPaperDwords - 1];
  if (base >= 0 && base + 4 * (int64_t)(kPaperDwords - 1) <= hi) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (uint32_t j = 0; j < 3; ++j) {
      const u32x4 q = *(const u32x4 *)(T + base + 16 * j);
      d[4 * j] = q.x;
      d[4 * j + 1] = q.y;
      d[4 * j + 2] = q.z;
      d[4 * j + 3] = q.w;
    }
    d[12] = *(const uint32_t *)(T + base + 48);
  } else {
    // near the ends of the text: dwords without a text byte are not read (the
    // nearest one that holds text is, and its bytes are not used)
#pragma unroll
    for (uint32_t j = 0; j < kPaperDwords; ++j) {
      const int64_t q = base + 4 * j;
      d[j] = *(const uint32_t *)(T + (q < lo ? lo : (q > hi ? hi : q)));
    }
  }
#pragma unroll
  for (uint32_t j = 0; j + 1 < kPaperDwords; ++j) e[j] = __builtin_amdgcn_alignbyte(d[j + 1], d[j], mis);
  const uint32_t lead = m < 32u ? 32u - m : 0u, k0 = lead >> 2;  // bytes and words before the window
  const uint32_t w0 = 0x01020408u & (0xFFFFFFFFu << (8u * (lead & 3u)));
  uint32_t h[kPaperPer];
  // (m is uniform: one case per wave)
  const uint32_t out = lead & 3u;
  if (m >= 32) {
    window_hashes16<0, false>(e, w0, out, m, h);
  } else {
    switch (k0) {
      case 0: window_hashes16<0, true>(e, w0, out, m, h); break;
      case 1: window_hashes16<1, true>(e, w0, out, m, h); break;
      case 2: window_hashes16<2, true>(e, w0, out, m, h); break;
      case 3: window_hashes16<3, true>(e, w0, out, m, h); break;
      case 4: window_hashes16<4, true>(e, w0, out, m, h); break;
      case 5: window_hashes16<5, true>(e, w0, out, m, h); break;
      case 6: window_hashes16<6, true>(e, w0, out, m, h); break;
      default: window_hashes16<7, true>(e, w0, out, m, h); break;
    }
  }
  uint32_t cand = 0, hit = 0;
#pragma unroll
  for (uint32_t i = 0; i < kPaperPer; ++i) cand |= (uint32_t)(h[i] == hx) << i;
  const uint32_t cnt = (uint32_t)min((uint64_t)kPaperPer, nwin - x0);
  cand &= 0xFFFFu >> (kPaperPer - cnt);
  while (cand) {
    const uint32_t i = __builtin_ctz(cand);
    cand &= cand - 1u;
    bool match = true;
    for (uint32_t j = 0; j < m; ++j)
      if (P[j] != T[x0 + i + j]) {
        match = false;
        break;
      }
    hit |= (uint32_t)match << i;
  }
  if (cnt == kPaperPer && ((uintptr_t)result & 15u) == 0) {
    uint4 f;  // bit i of a nibble to byte i of a word
    f.x = ((hit & 15u) * 0x00204081u) & 0x01010101u;
    f.y = ((hit >> 4 & 15u) * 0x00204081u) & 0x01010101u;
    f.z = ((hit >> 8 & 15u) * 0x00204081u) & 0x01010101u;
    f.w = ((hit >> 12) * 0x00204081u) & 0x01010101u;
    *(uint4 *)(result + x0) = f;
  } else {
    for (uint32_t i = 0; i < cnt; ++i) result[x0 + i] = (uint8_t)(hit >> i & 1u);
  }
  if (hash_out) {
#pragma unroll
    for (uint32_t i = 0; i < kPaperPer; ++i)
      if (i < cnt) hash_out[x0 + i] = h[i];
  }
}

// 16 bytes at any address, as dwords in memory order.
__device__ __forceinline__ void load16(const uint8_t *p, uint32_t *w) { __builtin_memcpy(w, p, 16); }

constexpr uint32_t kFlagWG = 256;
constexpr uint32_t kFlagRounds = 4;
constexpr uint32_t kFlagRound = kFlagWG * 16;              // flags per round: 16 consecutive ones per thread
constexpr uint32_t kFlagBlock = kFlagRound * kFlagRounds;  // flags per block

// Bit i set where byte i of the 16 flags at p (those below nf) is nonzero.
// Whole words are tested four flags at a time; the ragged end of the array
// reads single bytes.
__device__ __forceinline__ uint32_t flag_mask(const uint8_t *flags, uint64_t i, uint64_t nf) {
  uint32_t mask = 0;
  if (i + 16 <= nf) {
    uint32_t w[4];
    load16(flags + i, w);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t hi = ((((w[j] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w[j]) & 0x80808080u) >> 7;
      mask |= __builtin_amdgcn_udot4(hi, 0x08040201u, 0u, false) << (4 * j);
    }
  } else {
    for (uint32_t j = 0; j < 16 && i + j < nf; ++j) mask |= (uint32_t)(flags[i + j] != 0) << j;
  }
  return mask;
}

// Count of set flags per block of kFlagBlock.  Bound by the read of the
// flags: 16 bytes per lane, a wave's loads contiguous, the last flags first, as
// those written last are still in the cache behind the L2 (320 MB: 51 us right
// after the search that wrote them, 75 us with the first flags first or after
// other searches, 0.29 ms with one byte per lane and load).
__global__ __launch_bounds__(kFlagWG) void flag_counts(const uint8_t *flags, uint64_t nf, uint32_t *counts,
                                                       uint32_t *done) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *done = 0;  // of the scan that follows
  const uint32_t blk = gridDim.x - 1 - blockIdx.x;
  const uint64_t base = (uint64_t)blk * kFlagBlock + 16u * threadIdx.x;
  uint32_t c = 0;
#pragma unroll
  for (uint32_t j = 0; j < kFlagRounds; ++j) c += __builtin_popcount(flag_mask(flags, base + j * kFlagRound, nf));
  for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
  __shared__ uint32_t red[kFlagWG / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (uint32_t w = 0; w < kFlagWG / 64; ++w) t += red[w];
    counts[blk] = t;
  }
}

// Writes the positions of the set flags of each block, in ascending order,
// from the block's offset: the block walks its flags in rounds, a thread's 16
// flags ranked by a block prefix sum of the threads' counts.  A block without
// a set flag reads nothing (320 MB with 1,000 matches: 9 us, 344 us when
// every block read its flags byte by byte).
__global__ __launch_bounds__(kFlagWG) void flag_positions(const uint8_t *flags, uint64_t nf, const uint32_t *counts,
                                                          const uint64_t *offs, uint64_t *pos) {
  if (counts[blockIdx.x] == 0) return;
  __shared__ uint32_t wsum[kFlagWG / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kFlagBlock + 16u * threadIdx.x;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t o = offs[blockIdx.x];
  for (uint32_t j = 0; j < kFlagRounds; ++j) {
    const uint64_t i = base + j * kFlagRound;
    uint32_t mask = flag_mask(flags, i, nf);
    const uint32_t c = __builtin_popcount(mask);
    uint32_t x = c;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= (uint32_t)d) x += y;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (uint32_t w = 0; w < kFlagWG / 64; ++w) {
      before += w < wave ? wsum[w] : 0u;
      tot += wsum[w];
    }
    uint64_t at = o + before + x - c;
    while (mask) {
      pos[at++] = i + (uint32_t)__builtin_ctz(mask);
      mask &= mask - 1u;
    }
    o += tot;
  }
}

static rk_status paper_grid(rk_ctx *ctx, uint64_t nwin, uint32_t tpb, dim3 *grid) {
  const uint64_t blocks = ((nwin + kPaperPer - 1) / kPaperPer + tpb - 1) / tpb;
  // a dispatch holds at most 2^32 - 1 work-items per dimension
  const uint64_t gx = std::min<uint64_t>(blocks, 0xFFFFFFFFull / tpb);
  const uint64_t gy = (blocks + gx - 1) / gx;
  if (gy > 65535) return set_err(ctx, RK_EUNSUPPORTED, "text too long for one paper-mode launch");
  *grid = dim3((uint32_t)gx, (uint32_t)gy, 1);
  return RK_OK;
}

}  // namespace rk

using namespace rk;

extern "C" rk_status rk_paper_search(rk_ctx *ctx, const uint8_t *text_dev, uint64_t n, const uint8_t *pattern_dev,
                                     const uint8_t *pattern_host, uint32_t m, uint32_t threads_per_block,
                                     uint8_t *result_dev, uint32_t *hash_dev, rk_stream s) {
  if (!ctx) return RK_EINVAL;
  if (m == 0) return set_err(ctx, RK_EINVAL, "m = 0");
  if (threads_per_block == 0 || threads_per_block > 1024)
    return set_err(ctx, RK_EINVAL, "threads per block must be 1..1024");
  if (n < m) return RK_OK;  // no window
  if (!text_dev || !pattern_dev || !pattern_host || !result_dev) return set_err(ctx, RK_EINVAL, "null pointer");
  const uint64_t nwin = n - m + 1;
  // the pattern's hash, once on the host (Sec. 3.1)
  uint32_t hx = 0;
  for (uint32_t i = 0; i < m; ++i) hx = (hx << 1) + pattern_host[i];
  dim3 grid;
  rk_status st = paper_grid(ctx, nwin, threads_per_block, &grid);
  if (st != RK_OK) return st;
  if (hipSetDevice(ctx->device) != hipSuccess) return set_err(ctx, RK_EDEVICE, "hipSetDevice failed");
  hipStream_t hs = (hipStream_t)s;
  int slot = -1;
  hipError_t e = prof_begin(ctx, hs, 5, &slot);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(paper_kernel, grid, dim3(threads_per_block), 0, hs, text_dev, n, nwin, pattern_dev, m, hx,
                       result_dev, hash_dev);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = prof_end(ctx, hs, slot);
  return e == hipSuccess ? RK_OK : hip_err(ctx, e, "paper-mode launch");
}

extern "C" rk_status rk_paper_scratch_size(uint64_t nflags, uint64_t *bytes) {
  if (!bytes) return RK_EINVAL;
  const uint64_t nb = (nflags + kFlagBlock - 1) / kFlagBlock;
  *bytes = (nb * 4 + 255) / 256 * 256 + (nb * 8 + 255) / 256 * 256 + scan_tmp_words(nb) * 8 + 256;
  return RK_OK;
}

extern "C" rk_status rk_paper_positions(rk_ctx *ctx, const uint8_t *flags_dev, uint64_t nflags, void *scratch_dev,
                                        uint64_t scratch_bytes, uint64_t *positions_dev, uint64_t capacity,
                                        uint64_t *total_host, rk_stream s) {
  if (!ctx || !total_host) return RK_EINVAL;
  *total_host = 0;
  if (nflags == 0) return RK_OK;
  if (!flags_dev || !scratch_dev) return set_err(ctx, RK_EINVAL, "null pointer");
  uint64_t need = 0;
  rk_paper_scratch_size(nflags, &need);
  if (scratch_bytes < need) return set_err(ctx, RK_ENOSPACE, "scratch needs %llu bytes", (unsigned long long)need);
  if (hipSetDevice(ctx->device) != hipSuccess) return set_err(ctx, RK_EDEVICE, "hipSetDevice failed");
  hipStream_t hs = (hipStream_t)s;
  const uint64_t nb = (nflags + kFlagBlock - 1) / kFlagBlock;
  uint8_t *sc = (uint8_t *)scratch_dev;
  uint32_t *counts = (uint32_t *)sc;
  uint64_t *offs = (uint64_t *)(sc + (nb * 4 + 255) / 256 * 256);
  uint64_t *tmp = (uint64_t *)((uint8_t *)offs + (nb * 8 + 255) / 256 * 256);
  uint32_t *done = (uint32_t *)((uint8_t *)tmp + scan_tmp_words(nb) * 8);
  ctx->pinned[kHostTotal] = kNoTotal;
  hipLaunchKernelGGL(flag_counts, dim3((uint32_t)nb), dim3(kFlagWG), 0, hs, flags_dev, nflags, counts, done);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_exclusive_scan(counts, nb, offs, tmp, ctx->pinned, done, hs);
  if (e == hipSuccess) e = wait_total(ctx, hs);
  if (e != hipSuccess) return hip_err(ctx, e, "paper positions count");
  const uint64_t total = ctx->pinned[kHostTotal];
  *total_host = total;
  if (total > capacity) return set_err(ctx, RK_ENOSPACE, "positions capacity %llu < %llu matches",
                                       (unsigned long long)capacity, (unsigned long long)total);
  if (total == 0) return RK_OK;
  if (!positions_dev) return set_err(ctx, RK_EINVAL, "null positions");
  hipLaunchKernelGGL(flag_positions, dim3((uint32_t)nb), dim3(kFlagWG), 0, hs, flags_dev, nflags, counts, offs,
                     positions_dev);
  e = hipGetLastError();
  return e == hipSuccess ? RK_OK : hip_err(ctx, e, "paper positions launch");
}
