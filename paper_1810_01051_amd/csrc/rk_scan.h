// HIP kernels of librk for gfx950 (CDNA4, wave64).
//
// Hot path (Shah & Oza, Sec. 3.1, GPU procedure): every text window gets a
// polynomial hash, the hash is tested against the pattern-hash set and a hit
// is confirmed by comparing bytes.  The paper gives one thread per window and
// recomputes each window's hash from global memory; here a wave stages a
// sub-tile of the text (plus a 64-byte halo in front of it) in LDS with coalesced
// 16-byte loads, and each thread rolls the hash over C consecutive windows held
// in registers, so every text byte is read from HBM once.
//
// Window identity: a window is named by its END byte e (bytes e-m+1 .. e).
// A wave scans sub-tiles of 64 C bytes on its own: lane l owns the windows
// ending at sub-tile bytes [l*C, l*C + C).
//
// Two ways to test a window (same results):
//   exact  : the d=256, q=2^61-1 hash is rolled for every window
//            (H' = 256 H + in - out*256^m mod q, with a lazily reduced 64-bit
//            state; for one key of six bytes or more, four windows a step)
//            and compared with the set;
//   screen : the paper's shift-and-add hash h' = (h << s) + in mod 2^32 is
//            rolled for every window (s*m >= 32, so bytes older than the window
//            shift out and no out-term is needed) and compared with the set.
// One key is compared in a register; a set of keys is a bitmap in LDS, indexed
// by bits of the hash: one LDS read and a bit test per window.  A candidate
// window (its hash passed the set test) finds its pattern by the rank of its
// bit in a bitmap of the patterns' shift-add hashes, and is confirmed byte by
// byte against every pattern of that bit.
//
// Hits are appended in ascending window order per bucket to the staging slab
// of their tile (a run of sub-tiles that one wave scans in order); later
// kernels scan the tile counts, compact the slabs and sort stably by pattern
// id.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rk_dev.h"
#include "rk_internal.h"
#include "rk_runtime.h"

namespace rk {

// -------------------------------------------------------------- window tests
// Each pass walks the C windows of the calling thread.  The register array w
// holds 64 bytes before the thread's first window end (w[0..15]) followed by
// its C bytes (w[16..]).  ANY=true returns the OR over windows of the wave
// ballot of the test; ANY=false returns the per-thread candidate bit mask.
template <int C>
struct Bits {
  uint32_t b[(C + 31) / 32];
};

// Bit layout of Bits: window i is bit i%32 of word i/32.  The flags are
// shifted in from the top, one instruction each: the low bit of f.
template <int C>
__device__ __forceinline__ constexpr int word_windows(int j) {
  return (C - 32 * j) < 32 ? (C - 32 * j) : 32;
}
template <int C>
__device__ __forceinline__ void put_bit(Bits<C> &bits, uint32_t &acc, int i, uint32_t f) {
  acc = __builtin_amdgcn_alignbit(f, acc, 1);
  if ((i & 31) == 31 || i == C - 1) bits.b[i >> 5] = acc >> (32 - word_windows<C>(i >> 5));
}
// The same with the flags of a wave's lanes in a mask: shifted in from the
// bottom as an add with carry, then reversed.
template <int C>
__device__ __forceinline__ void put_mask(Bits<C> &bits, uint32_t &acc, int i, uint64_t f) {
  uint64_t carry;
  __asm__("v_addc_co_u32 %0, %1, %0, %0, %2" : "+v"(acc), "=s"(carry) : "s"(f));
  if ((i & 31) == 31 || i == C - 1) {
    bits.b[i >> 5] = __builtin_bitreverse32(acc) >> (32 - word_windows<C>(i >> 5));
    acc = 0;
  }
}

typedef __attribute__((address_space(3))) const uint32_t lds_word;
typedef __attribute__((address_space(3))) uint16_t lds_half;
typedef uint32_t rk_u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const rk_u32x4 lds_quad;
// LDS reads by byte address (no generic pointers: a read that the compiler
// merged with one from device memory would wait for the loads in flight).
__device__ __forceinline__ uint32_t lds32(uint32_t a) { return *(lds_word *)(uintptr_t)a; }
__device__ __forceinline__ uint32_t lds16(uint32_t a) { return *(lds_half *)(uintptr_t)a; }

// ---------------------------------------------------- LDS reads out of sight
// The tile pipeline issues the next tiles' loads-to-LDS before testing the
// current tile.  The compiler cannot tell that the current tile's LDS words
// are not the ones those loads write, so before any LDS read it can see it
// waits for every outstanding load -- the next tiles' included, which would
// end the overlap.  The tile words are therefore read by inline asm (pairs of
// dwords, then one wait for all of them inside the same statement, so that no
// word is used before it has arrived; the outputs are early-clobber, as the
// address is still read after the first word is written); the scan's
// wait_loads orders these reads after the tile has landed.
typedef uint32_t rk_u32x2 __attribute__((ext_vector_type(2)));

#define RK_DSP1 "ds_read2_b32 %0, %[a] offset0:0 offset1:1\n"
#define RK_DSP2 RK_DSP1 "ds_read2_b32 %1, %[a] offset0:2 offset1:3\n"
#define RK_DSP3 RK_DSP2 "ds_read2_b32 %2, %[a] offset0:4 offset1:5\n"
#define RK_DSP4 RK_DSP3 "ds_read2_b32 %3, %[a] offset0:6 offset1:7\n"
#define RK_DSP5 RK_DSP4 "ds_read2_b32 %4, %[a] offset0:8 offset1:9\n"
#define RK_DSP6 RK_DSP5 "ds_read2_b32 %5, %[a] offset0:10 offset1:11\n"
#define RK_DSP7 RK_DSP6 "ds_read2_b32 %6, %[a] offset0:12 offset1:13\n"
#define RK_DSP8 RK_DSP7 "ds_read2_b32 %7, %[a] offset0:14 offset1:15\n"
#define RK_DSP9 RK_DSP8 "ds_read2_b32 %8, %[a] offset0:16 offset1:17\n"
#define RK_DSP10 RK_DSP9 "ds_read2_b32 %9, %[a] offset0:18 offset1:19\n"
#define RK_DSP11 RK_DSP10 "ds_read2_b32 %10, %[a] offset0:20 offset1:21\n"
#define RK_DSP12 RK_DSP11 "ds_read2_b32 %11, %[a] offset0:22 offset1:23\n"
#define RK_DSP13 RK_DSP12 "ds_read2_b32 %12, %[a] offset0:24 offset1:25\n"
#define RK_DSP14 RK_DSP13 "ds_read2_b32 %13, %[a] offset0:26 offset1:27\n"
#define RK_DSP15 RK_DSP14 "ds_read2_b32 %14, %[a] offset0:28 offset1:29\n"
#define RK_DSP16 RK_DSP15 "ds_read2_b32 %15, %[a] offset0:30 offset1:31\n"
#define RK_DSP17 RK_DSP16 "ds_read2_b32 %16, %[a] offset0:32 offset1:33\n"
#define RK_DSP18 RK_DSP17 "ds_read2_b32 %17, %[a] offset0:34 offset1:35\n"
#define RK_DSP19 RK_DSP18 "ds_read2_b32 %18, %[a] offset0:36 offset1:37\n"
#define RK_DSP20 RK_DSP19 "ds_read2_b32 %19, %[a] offset0:38 offset1:39\n"
#define RK_DSP21 RK_DSP20 "ds_read2_b32 %20, %[a] offset0:40 offset1:41\n"
#define RK_DSP22 RK_DSP21 "ds_read2_b32 %21, %[a] offset0:42 offset1:43\n"
#define RK_DSP23 RK_DSP22 "ds_read2_b32 %22, %[a] offset0:44 offset1:45\n"
#define RK_DSP24 RK_DSP23 "ds_read2_b32 %23, %[a] offset0:46 offset1:47\n"
#define RK_DSO1(v) "=&v"(v[0])
#define RK_DSO2(v) RK_DSO1(v), "=&v"(v[1])
#define RK_DSO3(v) RK_DSO2(v), "=&v"(v[2])
#define RK_DSO4(v) RK_DSO3(v), "=&v"(v[3])
#define RK_DSO5(v) RK_DSO4(v), "=&v"(v[4])
#define RK_DSO6(v) RK_DSO5(v), "=&v"(v[5])
#define RK_DSO7(v) RK_DSO6(v), "=&v"(v[6])
#define RK_DSO8(v) RK_DSO7(v), "=&v"(v[7])
#define RK_DSO9(v) RK_DSO8(v), "=&v"(v[8])
#define RK_DSO10(v) RK_DSO9(v), "=&v"(v[9])
#define RK_DSO11(v) RK_DSO10(v), "=&v"(v[10])
#define RK_DSO12(v) RK_DSO11(v), "=&v"(v[11])
#define RK_DSO13(v) RK_DSO12(v), "=&v"(v[12])
#define RK_DSO14(v) RK_DSO13(v), "=&v"(v[13])
#define RK_DSO15(v) RK_DSO14(v), "=&v"(v[14])
#define RK_DSO16(v) RK_DSO15(v), "=&v"(v[15])
#define RK_DSO17(v) RK_DSO16(v), "=&v"(v[16])
#define RK_DSO18(v) RK_DSO17(v), "=&v"(v[17])
#define RK_DSO19(v) RK_DSO18(v), "=&v"(v[18])
#define RK_DSO20(v) RK_DSO19(v), "=&v"(v[19])
#define RK_DSO21(v) RK_DSO20(v), "=&v"(v[20])
#define RK_DSO22(v) RK_DSO21(v), "=&v"(v[21])
#define RK_DSO23(v) RK_DSO22(v), "=&v"(v[22])
#define RK_DSO24(v) RK_DSO23(v), "=&v"(v[23])

// reads NW consecutive dwords at LDS byte address a (4-byte aligned) into w
template <int NW>
__device__ __forceinline__ void lds_read_words(uint32_t *w, uint32_t a) {
  constexpr int P = NW / 2;
  static_assert(NW >= 2 && P <= 24, "word count within the generated forms");
  rk_u32x2 v[P];
  uint32_t last = 0;
  (void)last;
  if constexpr (P == 1) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP1 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO1(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP1 "s_waitcnt lgkmcnt(0)" : RK_DSO1(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 2) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP2 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO2(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP2 "s_waitcnt lgkmcnt(0)" : RK_DSO2(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 3) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP3 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO3(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP3 "s_waitcnt lgkmcnt(0)" : RK_DSO3(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 4) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP4 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO4(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP4 "s_waitcnt lgkmcnt(0)" : RK_DSO4(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 5) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP5 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO5(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP5 "s_waitcnt lgkmcnt(0)" : RK_DSO5(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 6) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP6 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO6(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP6 "s_waitcnt lgkmcnt(0)" : RK_DSO6(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 7) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP7 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO7(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP7 "s_waitcnt lgkmcnt(0)" : RK_DSO7(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 8) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP8 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO8(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP8 "s_waitcnt lgkmcnt(0)" : RK_DSO8(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 9) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP9 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO9(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP9 "s_waitcnt lgkmcnt(0)" : RK_DSO9(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 10) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP10 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO10(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP10 "s_waitcnt lgkmcnt(0)" : RK_DSO10(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 11) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP11 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO11(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP11 "s_waitcnt lgkmcnt(0)" : RK_DSO11(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 12) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP12 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO12(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP12 "s_waitcnt lgkmcnt(0)" : RK_DSO12(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 13) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP13 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO13(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP13 "s_waitcnt lgkmcnt(0)" : RK_DSO13(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 14) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP14 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO14(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP14 "s_waitcnt lgkmcnt(0)" : RK_DSO14(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 15) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP15 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO15(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP15 "s_waitcnt lgkmcnt(0)" : RK_DSO15(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 16) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP16 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO16(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP16 "s_waitcnt lgkmcnt(0)" : RK_DSO16(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 17) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP17 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO17(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP17 "s_waitcnt lgkmcnt(0)" : RK_DSO17(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 18) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP18 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO18(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP18 "s_waitcnt lgkmcnt(0)" : RK_DSO18(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 19) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP19 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO19(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP19 "s_waitcnt lgkmcnt(0)" : RK_DSO19(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 20) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP20 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO20(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP20 "s_waitcnt lgkmcnt(0)" : RK_DSO20(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 21) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP21 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO21(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP21 "s_waitcnt lgkmcnt(0)" : RK_DSO21(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 22) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP22 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO22(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP22 "s_waitcnt lgkmcnt(0)" : RK_DSO22(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 23) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP23 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO23(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP23 "s_waitcnt lgkmcnt(0)" : RK_DSO23(v) : [a] "v"(a) : "memory");
  } else if constexpr (P == 24) {
    if constexpr (NW & 1)
      __asm__ volatile(RK_DSP24 "ds_read_b32 %[l], %[a] offset:%[o]\n\ts_waitcnt lgkmcnt(0)"
                       : RK_DSO24(v), [l] "=&v"(last) : [a] "v"(a), [o] "n"(8 * P) : "memory");
    else
      __asm__ volatile(RK_DSP24 "s_waitcnt lgkmcnt(0)" : RK_DSO24(v) : [a] "v"(a) : "memory");
  }
#pragma unroll
  for (int j = 0; j < P; ++j) {
    w[2 * j] = v[j].x;
    w[2 * j + 1] = v[j].y;
  }
  if constexpr (NW & 1) w[NW - 1] = last;
}

__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(lds_word *)p; }

// The lane's bytes, loaded from the LDS sub-tile by each pass itself (so that
// the loads, and the byte extractions that follow them, are not shared between
// the test variants of a bucket and hoisted above the variant switch, which
// would keep every extracted byte of every variant live at once).  Passes take
// the LDS address of the lane's first window end (mine).
// Words before a lane's first window end that the screen passes read: the 16
// bytes their hash can reach back over.
constexpr int kWarm = 4;

// Shift-add hash state after the 16 bytes held in w[0..4), i.e. before the
// lane's first window end: h = sum_j b[15-j] << (S*j) mod 2^32 (bytes older
// than 32/S positions have shifted out).  For S = 2 four bytes at a time with
// one dot product each: the weights 4^3..4^0 of a word's bytes fit in bytes.
template <int S>
__device__ __forceinline__ uint32_t screen_init(const uint32_t *w) {
  if constexpr (S == 2) {
    uint32_t h = 0;
#pragma unroll
    for (int q = 0; q < kWarm; ++q) h = __builtin_amdgcn_udot4(w[q], 0x01041040u, h << 8, false);
    return h;
  } else {
    constexpr int WU = (32 + S - 1) / S - 1;  // bytes before the first window end that are still in the hash
    uint32_t h = 0;
#pragma unroll
    for (int j = 4 * kWarm - WU; j < 4 * kWarm; ++j) h = (h << S) + byte_at(w, j);
    return h;
  }
}

// OR of the wave ballots, kept as a sequential chain of scalar ORs (a
// reassociated OR tree would keep one SGPR pair per window alive).
__device__ __forceinline__ void any_or(uint64_t &any, uint64_t b) {
  any |= b;
  __asm__ volatile("" : "+s"(any));
}

// NT keys: the hash of every window compared with each.
template <int C, int S, bool ANY, int NT>
__device__ __forceinline__ void pass_list_screen(uint32_t mine, uint32_t msk, const uint32_t *tgt, uint64_t &any,
                                                 Bits<C> &bits) {
  uint32_t w[kWarm + C / 4];
  lds_read_words<kWarm + C / 4>(w, mine - 4 * kWarm);
  uint32_t h = screen_init<S>(w), acc = 0;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    h = (h << S) + byte_at(w, 4 * kWarm + i);
    const uint32_t v = (S == 8) ? (h & msk) : h;
    uint64_t f = ballot(v == tgt[0]);
#pragma unroll
    for (int t = 1; t < NT; ++t) f |= ballot(v == tgt[t]);
    if (ANY) any_or(any, f);
    else put_mask<C>(bits, acc, i, f);
  }
}

// Word of a bitmap (LDS address base) for value v and, as the lowest bit, v's
// bit in it.
__device__ __forceinline__ uint32_t filter_word(uint32_t base, uint32_t sh, uint32_t v) {
  return lds32(base + ((v >> sh) << 2));
}
__device__ __forceinline__ uint32_t filter_bit(uint32_t word, uint32_t v) { return word >> (v & 31u); }

// Windows per block of the bitmap tests: the LDS reads of a block's windows
// are all issued before the first of them is tested, so that their latencies
// overlap (C is a multiple of 4 in every geometry).
constexpr int kProbeBlock = 4;

// A set of keys: kMix times the hash of every window tested in the bucket's
// bitmap.  MASKED: windows shorter than the hash's span (one to three bytes),
// whose hash is masked before the product (below 2^24, as kMix is).
template <int C, int S, bool MASKED>
__device__ __forceinline__ void pass_filter_screen(uint32_t mine, uint32_t msk, uint32_t base, uint32_t sh,
                                                   Bits<C> &bits) {
  static_assert(C % kProbeBlock == 0, "whole probe blocks");
  uint32_t w[kWarm + C / 4];
  lds_read_words<kWarm + C / 4>(w, mine - 4 * kWarm);
  uint32_t h = screen_init<S>(w), acc = 0;
  if (!MASKED) h *= kMix;
#pragma unroll
  for (int i0 = 0; i0 < C; i0 += kProbeBlock) {
    uint32_t v[kProbeBlock], t[kProbeBlock];
#pragma unroll
    for (int j = 0; j < kProbeBlock; ++j) {
      const uint32_t c = byte_at(w, 4 * kWarm + i0 + j);
      h = (h << S) + (MASKED ? c : __umul24(c, kMix));
      v[j] = MASKED ? __umul24(h & msk, kMix) : h;
      t[j] = filter_word(base, sh, v[j]);
    }
#pragma unroll
    for (int j = 0; j < kProbeBlock; ++j) put_bit<C>(bits, acc, i0 + j, filter_bit(t[j], v[j]));
  }
}

// Exact rolling hash of the window ending before the first one of this
// thread: Horner over the 64 preceding bytes with the bytes older than the
// window (older than m positions) masked to zero -- leading zero digits do not
// change the polynomial.
__device__ __forceinline__ uint64_t exact_init(const uint32_t *w, uint32_t m) {
  uint64_t s = 0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int lead = 64 - (int)m - 4 * q;  // bytes of this word that precede the window
    if (lead >= 4) continue;                // wholly before the window: s stays 0 (m is uniform)
    const uint32_t keep = lead <= 0 ? 0xFFFFFFFFu : (0xFFFFFFFFu >> (8 * lead));
    s = mul2p32_lazy(s) + (__builtin_bswap32(w[q]) & keep);
  }
  return s;
}

// One exact rolling step: H(e) = 256 H(e-1) + in - out * 2^r  (r = 8m mod 61),
// with the 32-bit halves spelled out and the outgoing term specialised on
// where out * 2^r lands in the 61-bit word (r = 8m mod 61 is fixed per group):
// OUTK 0: bits r..r+7 in the low word (r <= 24), 1: in the high word
// (32 <= r <= 53), 2: anywhere (general rotation).
//   256 s mod q = ((s << 8) & q) + (s >> 53): the low byte of s << 8 is free
//   for the entering byte (byte k of the word inw, merged by one byte
//   permute); q - v = q ^ v for v <= q.
// The sum (256 s + in) + (q - out * 2^r) + (s >> 53) is two add-with-carry
// pairs (OUTK 0, 1).  s < 2^63 in, s < 2^62 + 2^11 out.
template <int OUTK>
__device__ __forceinline__ uint64_t exact_step_k(uint64_t s, uint32_t inw, uint32_t k, uint32_t out, uint32_t r) {
  const uint32_t lo = (uint32_t)s, hi = (uint32_t)(s >> 32);
  const uint32_t alo = __builtin_amdgcn_perm(lo, inw, 0x06050400u | k);  // (lo << 8) | byte k of inw
  const uint32_t ahi = __builtin_amdgcn_alignbit(hi, lo, 24) & 0x1FFFFFFFu;
  const uint32_t f = hi >> 21;
  if constexpr (OUTK == 2) {
    const uint64_t neg = kQ - rot61(out, r);
    return ((((uint64_t)ahi << 32) | alo) + neg) + f;
  } else {
    uint32_t x, h;
    if constexpr (OUTK == 0) {
      // (the high word of q comes in a VGPR: with the carry in VCC a literal
      // would be a second constant-bus read)
      __asm__("v_add_co_u32 %0, vcc, %2, %3\n\t"
              "v_addc_co_u32 %1, vcc, %6, %4, vcc\n\t"
              "v_add_co_u32 %0, vcc, %0, %5\n\t"
              "v_addc_co_u32 %1, vcc, 0, %1, vcc"
              : "=&v"(x), "=&v"(h)
              : "v"(alo), "v"(~(out << r)), "v"(ahi), "v"(f), "v"(0x1FFFFFFFu)
              : "vcc");
    } else {
      __asm__("v_add_co_u32 %0, vcc, -1, %2\n\t"
              "v_addc_co_u32 %1, vcc, %3, %4, vcc\n\t"
              "v_add_co_u32 %0, vcc, %0, %5\n\t"
              "v_addc_co_u32 %1, vcc, 0, %1, vcc"
              : "=&v"(x), "=&v"(h)
              : "v"(alo), "v"(0x1FFFFFFFu ^ (out << (r - 32))), "v"(ahi), "v"(f)
              : "vcc");
    }
    return ((uint64_t)h << 32) | x;
  }
}

__device__ __forceinline__ int out_kind(uint32_t r) { return r <= 24 ? 0 : ((r >= 32 && r <= 53) ? 1 : 2); }

// Out-stream: the byte leaving window i (the thread's i-th window end) sits m
// bytes before the entering one.  It is read as aligned LDS dwords starting
// o = 4*ceil(m/4) bytes before the thread's first window end and realigned by
// sh = o - m bytes with alignbyte, four windows per dword.
struct OutStream {
  uint32_t d;  // LDS address, 4-byte aligned
  uint32_t sh;
};

__device__ __forceinline__ OutStream out_stream(uint32_t mine, uint32_t m) {
  const uint32_t o = (m + 3u) & ~3u;
  return OutStream{mine - o, o - m};
}

// The exact rolling hash over the thread's C windows, the one loop every
// exact pass and the hash dump run: the state of the window ending before the
// thread's first one (exact_init), then one exact_step_k per window with the
// entering byte from w and the leaving byte from the out-stream dwords d;
// visit(i, s) sees the lazy state s of window i (congruent to its hash,
// s < 2^62 + 2^11).
template <int C, int OUTK, typename Visit>
__device__ __forceinline__ void roll_exact(const uint32_t *w, const uint32_t *d, OutStream os, uint32_t m, uint32_t r,
                                           Visit &&visit) {
  uint64_t s = exact_init(w, m);
  uint32_t dlo = d[0], ow = 0;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    if ((i & 3) == 0) {
      const uint32_t dhi = d[(i >> 2) + 1];
      ow = __builtin_amdgcn_alignbyte(dhi, dlo, os.sh);
      dlo = dhi;
    }
    s = exact_step_k<OUTK>(s, w[(64 + i) >> 2], (uint32_t)(i & 3), (ow >> (8 * (i & 3))) & 0xFFu, r);
    visit(i, s);
  }
}

// exact_mix in one instruction.
__device__ __forceinline__ uint32_t exact_mix2(uint64_t s) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const u16x2 k = {(unsigned short)kExactMixLo, (unsigned short)kExactMixHi};
  return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, (uint32_t)s), k, (uint32_t)(s >> 32), false);
}

// A set of keys: the lazy state of every window in the bucket's bitmap, which
// holds every lazy form of every key.
template <int C, int OUTK>
__device__ __forceinline__ void pass_filter_exact(uint32_t mine, OutStream os, uint32_t m, uint32_t r, uint32_t base,
                                                  uint32_t fsh, Bits<C> &bits) {
  uint32_t w[16 + C / 4], d[C / 4 + 1], acc = 0;
  lds_read_words<16 + C / 4>(w, mine - 64);
  lds_read_words<C / 4 + 1>(d, os.d);
  uint32_t v[kProbeBlock], t[kProbeBlock];
  roll_exact<C, OUTK>(w, d, os, m, r, [&](int i, uint64_t s) __attribute__((always_inline)) {
    // lazy state s = H + j*q for j in {0,1,2}
    v[i % kProbeBlock] = exact_mix2(s);
    t[i % kProbeBlock] = filter_word(base, fsh, v[i % kProbeBlock]);
    if (i % kProbeBlock == kProbeBlock - 1) {
#pragma unroll
      for (int j = 0; j < kProbeBlock; ++j) put_bit<C>(bits, acc, i + 1 - kProbeBlock + j, filter_bit(t[j], v[j]));
    }
  });
}

constexpr uint32_t kStepM = 6;

// out * 2^r mod q for a 32-bit word, r uniform; K: r <= 29 (0: nothing leaves
// the 61 bits), r >= 32 (1: the low word is only what wraps), else (2).
__device__ __forceinline__ int rot_kind(uint32_t r) { return r <= 29 ? 0 : r >= 32 ? 1 : 2; }
template <int K>
__device__ __forceinline__ uint64_t rot61_word(uint32_t v, uint32_t r) {
  if (K == 0) return (uint64_t)v << r;
  if (K == 1) return (uint64_t)((v << (r - 32u)) & 0x1FFFFFFFu) << 32 | v >> (61u - r);
  return rot61(v, r);
}

// NT keys of fewer than kStepM bytes: every window's state compared with each
// key's lazy forms H, H + q, H + 2q, whose low words are consecutive from tg
// (tg2) on (q is -1 in 32 bits).
template <int C, bool ANY, int OUTK, int NT>
__device__ __forceinline__ void pass_short_exact(uint32_t mine, OutStream os, uint32_t m, uint32_t r, uint32_t tg,
                                                 uint32_t tg2, uint64_t &any, Bits<C> &bits) {
  uint32_t w[16 + C / 4], d[C / 4 + 1], acc = 0, low = ~0u;
  lds_read_words<16 + C / 4>(w, mine - 64);
  lds_read_words<C / 4 + 1>(d, os.d);
  roll_exact<C, OUTK>(w, d, os, m, r, [&](int i, uint64_t s) __attribute__((always_inline)) {
    uint32_t x = (uint32_t)s - tg;
    if (NT == 2) x = min(x, (uint32_t)s - tg2);
    if (ANY) low = min(low, x);
    else put_mask<C>(bits, acc, i, ballot(x <= 2u));
  });
  if (ANY) any |= ballot(low <= 2u);
}

// NT keys: the hash of every window compared with each, four windows a step.
// With Y = 2^32 H for the hash H before the four, I and O the four entering and
// leaving bytes (the first one on top) and R(x) = x * 256^m mod q, the hash
// after j + 1 of them is, times 2^(24-8j),
//   X_j = Y + (I & top j + 1 bytes) - R(O & top j + 1 bytes)  (mod q)
// and R of the masked bytes is R(O) masked by R of the mask (a rotation).  So
// the rolling state moves once per four windows, and a window costs the low
// word of X_j: one mask each for I and R(O), one three-way sum.  It is compared
// with the low word of the key times 2^(24-8j): X_j + q is that plus 0, q or 2q
// (Y < 2^61 + 2^35), whose low words are consecutive from tg[j] (the second
// key's: tg2[j]) on.
// s < 2^62 + 2^35 after each step.
// The low word of X_j is another 32 of the hash's 61 bits for each j, and of a
// window of few bytes some of these are zero: more of its false matches go on
// to the candidates.  Keys below kStepM bytes keep the low word of the hash
// itself (1 GiB of four letters: 4 bytes 555 us, with steps 770, 5 bytes 560
// and 728, 6 bytes 560 and 520, 8 bytes 560 and 420).
// Bound by these operations: 8 a window where one 64-bit step per window
// took 12 (1 GiB, m = 32: 316 us against 434).
template <int C, bool ANY, int K, int NT>
__device__ __forceinline__ void pass_list_exact(uint32_t mine, OutStream os, uint32_t m, uint32_t r, const uint32_t *tg,
                                                const uint32_t *tg2, uint64_t &any, Bits<C> &bits) {
  uint32_t w[16 + C / 4], d[C / 4 + 1], acc = 0, low = ~0u;
  lds_read_words<16 + C / 4>(w, mine - 64);
  lds_read_words<C / 4 + 1>(d, os.d);
  uint64_t s = exact_init(w, m);
  const uint32_t osel = 0x00010203u + 0x01010101u * os.sh;  // bytes sh..sh + 3 of a pair of dwords, reversed
  uint32_t keep[3];  // what R leaves of R(O) outside the mask's image
#pragma unroll
  for (int j = 0; j < 3; ++j) keep[j] = ~(uint32_t)rot61_word<K>(0xFFFFFFFFu << (24 - 8 * j), r);
#pragma unroll
  for (int i = 0; i < C; i += 4) {
    const uint32_t in = __builtin_bswap32(w[16 + i / 4]);
    const uint64_t neg = kQ ^ rot61_word<K>(__builtin_amdgcn_perm(d[i / 4 + 1], d[i / 4], osel), r);
    const uint64_t y = mul2p32_lazy(s);
    uint32_t v[4], x[4];
#pragma unroll
    for (int j = 0; j < 3; ++j) v[j] = (uint32_t)y + (in & (0xFFFFFFFFu << (24 - 8 * j))) + ((uint32_t)neg | keep[j]);
    s = y + in + neg;
    v[3] = (uint32_t)s;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = v[j] - tg[j];
      if (NT == 2) x[j] = min(x[j], v[j] - tg2[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (ANY) low = min(low, x[j]);
      else put_mask<C>(bits, acc, i + j, ballot(x[j] <= 2u));
    }
  }
  if (ANY) any |= ballot(low <= 2u);
}

// Destination of a hash dump: the canonical hash of every window whose start
// x = e - m + 1 is a multiple of stride goes to out[x / stride] (x / stride < cap).
struct DumpDst {
  uint64_t *out;
  uint64_t stride;
  uint64_t cap;
};

// kDump: the exact pass's own rolling loop (roll_exact, same out-kind
// specialisation as the test passes), writing canonical states of sampled
// windows instead of testing them.
template <int C, int OUTK>
__device__ __forceinline__ void pass_dump_w(const uint32_t *w, const uint32_t *d, OutStream os, uint32_t m, uint32_t r,
                                            int64_t e0, uint64_t n, const DumpDst &dst) {
  const int64_t x0 = e0 - (int64_t)m + 1;
  // rem = x0 mod stride for the first window (x0 may be negative)
  const int64_t st = (int64_t)dst.stride;
  int64_t rem = x0 % st;
  if (rem < 0) rem += st;
  // slot of the next sampled window at or after x0 (x0 - rem is a multiple of st)
  int64_t slot = (x0 - rem) / st + (rem ? 1 : 0);
  roll_exact<C, OUTK>(w, d, os, m, r, [&](int i, uint64_t s) __attribute__((always_inline)) {
    const int64_t x = x0 + i;
    if (rem == 0) {
      if (x >= 0 && (uint64_t)x + m <= n && (uint64_t)slot < dst.cap) dst.out[slot] = canon(s);
      ++slot;
    }
    rem = (rem + 1 == st) ? 0 : rem + 1;
  });
}

template <int C>
__device__ __forceinline__ void pass_dump(uint32_t mine, OutStream os, uint32_t m, uint32_t r, int64_t e0, uint64_t n,
                                          const DumpDst &dst) {
  uint32_t w[16 + C / 4], d[C / 4 + 1];
  lds_read_words<16 + C / 4>(w, mine - 64);
  lds_read_words<C / 4 + 1>(d, os.d);
  const int k = out_kind(r);
  if (k == 0) pass_dump_w<C, 0>(w, d, os, m, r, e0, n, dst);
  else if (k == 1) pass_dump_w<C, 1>(w, d, os, m, r, e0, n, dst);
  else pass_dump_w<C, 2>(w, d, os, m, r, e0, n, dst);
}

// Runs the test pass of bucket D over the lane's windows, filling the lane's
// candidate mask; ANY=true (list kinds): the wave ballots ORed into any instead.  D.shift holds the screen shift in bits 0-7; base: LDS address of the
// bucket's bitmap.  run_few: the single-bucket kernel's keys, two to four in
// kFamScreen, one or two, the second with tgt2, in kFamExact.
template <int C, bool ANY, int NT>
__device__ __forceinline__ void run_list_screen(const BucketDesc &D, uint32_t mine, uint64_t &any, Bits<C> &bits) {
  const uint32_t sh = D.shift & 0xFFu;
  if (sh == 2) pass_list_screen<C, 2, ANY, NT>(mine, D.mask, D.tgt, any, bits);
  else if (sh == 3) pass_list_screen<C, 3, ANY, NT>(mine, D.mask, D.tgt, any, bits);
  else if (sh == 4) pass_list_screen<C, 4, ANY, NT>(mine, D.mask, D.tgt, any, bits);
  else pass_list_screen<C, 8, ANY, NT>(mine, D.mask, D.tgt, any, bits);
}

template <int C, bool ANY, int NT>
__device__ __forceinline__ void run_list_exact(const BucketDesc &D, uint32_t mine, OutStream os, uint32_t r,
                                               const uint32_t *tgt2, uint64_t &any, Bits<C> &bits) {
  if (D.m < kStepM) {
    const int k = out_kind(r);
    if (k == 0) pass_short_exact<C, ANY, 0, NT>(mine, os, D.m, r, D.tgt[3], tgt2[3], any, bits);
    else if (k == 1) pass_short_exact<C, ANY, 1, NT>(mine, os, D.m, r, D.tgt[3], tgt2[3], any, bits);
    else pass_short_exact<C, ANY, 2, NT>(mine, os, D.m, r, D.tgt[3], tgt2[3], any, bits);
  } else {
    const int k = rot_kind(r);
    if (k == 0) pass_list_exact<C, ANY, 0, NT>(mine, os, D.m, r, D.tgt, tgt2, any, bits);
    else if (k == 1) pass_list_exact<C, ANY, 1, NT>(mine, os, D.m, r, D.tgt, tgt2, any, bits);
    else pass_list_exact<C, ANY, 2, NT>(mine, os, D.m, r, D.tgt, tgt2, any, bits);
  }
}

template <int C, bool ANY, int FAM>
__device__ __forceinline__ void run_few(const BucketDesc &D, uint32_t mine, OutStream os, uint32_t r, uint32_t nkeys,
                                        const uint32_t *tgt2, uint64_t &any, Bits<C> &bits) {
  if constexpr (FAM == kFamScreen1) {
    run_list_screen<C, ANY, 1>(D, mine, any, bits);
  } else if constexpr (FAM == kFamScreen) {
    if (nkeys == 2) run_list_screen<C, ANY, 2>(D, mine, any, bits);
    else if (nkeys == 3) run_list_screen<C, ANY, 3>(D, mine, any, bits);
    else run_list_screen<C, ANY, 4>(D, mine, any, bits);
  } else {
    if (nkeys == 2) run_list_exact<C, ANY, 2>(D, mine, os, r, tgt2, any, bits);
    else run_list_exact<C, ANY, 1>(D, mine, os, r, tgt2, any, bits);
  }
}

template <int C, int FAM>
__device__ __forceinline__ void run_pass(const BucketDesc &D, uint32_t mine, OutStream os, uint32_t r,
                                         uint32_t base, Bits<C> &bits) {
  const uint32_t sh = D.shift & 0xFFu;
  uint64_t any = 0;  // (not used)
  if constexpr (FAM == kFamExact) {
    if (D.kind == kListExact) {
      run_list_exact<C, false, 1>(D, mine, os, r, D.tgt, any, bits);
    } else {
      const int k = out_kind(r);
      if (k == 0) pass_filter_exact<C, 0>(mine, os, D.m, r, base, D.test_sh, bits);
      else if (k == 1) pass_filter_exact<C, 1>(mine, os, D.m, r, base, D.test_sh, bits);
      else pass_filter_exact<C, 2>(mine, os, D.m, r, base, D.test_sh, bits);
    }
  } else {
    if (FAM == kFamScreen1 || D.kind == kListScreen) {
      run_list_screen<C, false, 1>(D, mine, any, bits);
    } else {
      if (sh == 2) pass_filter_screen<C, 2, false>(mine, 0, base, D.test_sh, bits);
      else if (sh == 3) pass_filter_screen<C, 3, false>(mine, 0, base, D.test_sh, bits);
      else if (sh == 4) pass_filter_screen<C, 4, false>(mine, 0, base, D.test_sh, bits);
      else if (D.mask == 0xFFFFFFFFu) pass_filter_screen<C, 8, false>(mine, 0, base, D.test_sh, bits);
      else pass_filter_screen<C, 8, true>(mine, D.mask, base, D.test_sh, bits);
    }
  }
}

// -------------------------------------------------------- wave-level helpers
// Inclusive prefix sum over the wave's lanes (DPP: shifts by 1, 2, 4, 8 within
// rows of 16, then each row's last lane added to the rows after it).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return (uint32_t)x;
}

// Number of set bits of b below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t b) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
}

// Orders this wave's LDS writes before its later reads of them (LDS accesses
// of one wave take effect in issue order; this keeps the compiler to it).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Shift-add value of four window bytes rw (memory order: the oldest in the
// low byte) with the oldest weighted 2^(3s), ..., the newest 1: one byte dot
// product for s = 2, two for s = 3 and 4, the big-endian word for s = 8.
__device__ __forceinline__ uint32_t screen_word(uint32_t rw, uint32_t shift) {
  if (shift == 2) return __builtin_amdgcn_udot4(rw, 0x01041040u, 0u, false);
  if (shift == 3)
    return (__builtin_amdgcn_udot4(rw, 0x00000840u, 0u, false) << 3) + __builtin_amdgcn_udot4(rw, 0x01080000u, 0u, false);
  if (shift == 4)
    return (__builtin_amdgcn_udot4(rw, 0x00000110u, 0u, false) << 8) + __builtin_amdgcn_udot4(rw, 0x01100000u, 0u, false);
  return __builtin_bswap32(rw);
}

// Shift-add hash of the window whose last 16 bytes are raw (memory order),
// as the screen pass holds it for that window end (its last ceil(32/s) bytes,
// masked as the group's hash is).
__device__ __forceinline__ uint32_t screen_key(const uint32_t (&raw)[4], uint32_t shift, uint32_t mask) {
  if (shift == 2) {
    uint32_t h = screen_word(raw[0], 2);
#pragma unroll
    for (int j = 1; j < 4; ++j) h = (h << 8) + screen_word(raw[j], 2);
    return h;
  }
  if (shift == 3) return (((screen_word(raw[1], 3) << 12) + screen_word(raw[2], 3)) << 12) + screen_word(raw[3], 3);
  if (shift == 4) return (screen_word(raw[2], 4) << 16) + screen_word(raw[3], 4);
  return screen_word(raw[3], 8) & mask;
}

// Compares the m bytes at a (device memory: the text, any alignment) with the
// pattern at pat (device memory, 4-byte aligned), four bytes per step; reads
// only the text dwords that hold bytes of [a, a + m).  For windows longer than
// the tile's front halo.
__device__ __forceinline__ bool window_equals_global(const uint8_t *a, const uint8_t *pat, uint32_t m) {
  const uint32_t mis = (uint32_t)(uintptr_t)a & 3u;
  const uint32_t *aw = (const uint32_t *)(a - mis);
  const uint32_t *pw = (const uint32_t *)pat;
  const uint32_t nd = (mis + m + 3u) >> 2;  // dwords holding window bytes
  uint32_t lo = aw[0];
  for (uint32_t q = 0; 4 * q < m; ++q) {
    const uint32_t hi = q + 1 < nd ? aw[q + 1] : 0u;  // bytes past the window are masked below
    const uint32_t rem = m - 4 * q;
    const uint32_t keep = rem >= 4 ? 0xFFFFFFFFu : ((1u << (8 * rem)) - 1u);
    if ((__builtin_amdgcn_alignbyte(hi, lo, mis) ^ pw[q]) & keep) return false;
    lo = hi;
  }
  return true;
}

// Whether r bytes (r <= 16 counts, more: all 16; r <= 0: none) at LDS address
// a equal the first of p.
__device__ __forceinline__ bool quad_equals(uint32_t a, const rk_u32x4 p, int r) {
  const uint32_t mis = a & 3u, aw = a & ~3u;
  uint32_t diff = 0, lo = lds32(aw);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t hi = lds32(aw + 4 * (j + 1));
    const int left = r - 4 * j;
    const uint32_t keep = left <= 0 ? 0u : (left >= 4 ? 0xFFFFFFFFu : (1u << (8 * left)) - 1u);
    diff |= (__builtin_amdgcn_alignbyte(hi, lo, mis) ^ p[j]) & keep;
    lo = hi;
  }
  return diff == 0;
}

// ------------------------------------------------------- tile staging (LDS DMA)
// One 16-byte chunk per active lane from device memory straight into LDS:
// lane i's chunk at g lands at dst + 16 i (LDS address dst, wave-uniform).  Issued in asm
// so that the compiler does not see an LDS write in flight: it would make
// every later LDS read wait for all such loads (vmcnt(0)), the reads of the
// tile being tested included, so that the next tile's loads would no longer
// overlap its test.  Every read of a slot is ordered after that slot's loads
// by the scan's own waits (wait_loads, wait_lds).
// (M0 holds the LDS address, placed there by the compiler; the s_nop is the
// wait state required between a write of M0 and the load that uses it.)  The
// loads are non-temporal (nt): the text is read once, and streaming it past
// the caches reads 4 GiB at 6.6 TB/s against 6.1 without the hint.
__device__ __forceinline__ void lds_dma16(const void *g, uint32_t dst) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst);
  __asm__ volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(g), "{m0}"(m0) : "memory");
}

// LDS of one wave: sub-tile slots (front halo, 64 C bytes, 16 bytes that the
// realigning reads may touch) and the candidate list.
template <int C>
constexpr uint32_t sub_slot_bytes() {
  return kFront + 64 * C + 16;
}
template <int C>
constexpr uint32_t wave_lds_bytes(uint32_t slots) {
  return slots * sub_slot_bytes<C>() + kWaveCand * 2;
}

// Issues the loads of one sub-tile into an LDS slot of the calling wave: text
// bytes [start - kFront, start + 64 C) as 16-byte chunks that the load unit
// writes straight into LDS (no register staging), whole-wave loads of 1 KiB
// and a partial one.  Chunks outside the text read the text's first chunk
// instead: those LDS bytes only feed windows that start before the text or end
// after it, which the edge masks drop.
template <int C>
__device__ __forceinline__ void dma_sub(uint32_t slot, const uint8_t *text, uint64_t n, uint64_t start) {
  constexpr uint32_t NCH = 4 + 4 * C, J = NCH / 64, REM = NCH % 64;
  const uint32_t lane = threadIdx.x & 63;
  if (start >= kFront && start + 64 * C <= n) {
    // interior: every chunk is text
    const uint8_t *base = text + (start - kFront) + 16u * lane;
#pragma unroll
    for (uint32_t j = 0; j < J; ++j) lds_dma16(base + 1024u * j, slot + 1024u * j);
    if (lane < REM) lds_dma16(base + 1024u * J, slot + 1024u * J);
    return;
  }
#pragma unroll 1
  for (uint32_t j = 0; j <= J; ++j) {
    const uint64_t g = start + 1024u * j + 16u * lane;  // chunk start + kFront
    const uint8_t *src = g >= kFront && g - kFront < n ? text + (g - kFront) : text;
    if (j < J || lane < REM) lds_dma16(src, slot + 1024u * j);
  }
}

// This wave's loads-to-LDS have landed.
__device__ __forceinline__ void wait_loads() { __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }
// This wave's LDS reads are done.
__device__ __forceinline__ void wait_lds() { __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// A record and the last 16 bytes of its pattern, zeros in front of a shorter
// one.
struct Looked {
  uint64_t rec;
  rk_u32x4 tail;
};

// Where a bucket's records are: in the LDS image, in device memory, or held in
// registers: one of one pattern, or those of a few keys (the records of their
// runs in device memory).  The candidate phase is compiled for each, so that
// the LDS one holds no load from memory that could be under way: a wait for
// one would be a wait for every hit stored before it.
enum RecordPlace { kRecLds, kRecGlobal, kRecOne, kRecKeys };

struct Records {
  uint32_t img;         // LDS address of the image
  const uint8_t *gimg;  // device image
  uint32_t lk[kFewScreen];  // kRecKeys: lookup keys (those not used repeat the first)
  Looked held[kFewScreen];  // and their records; kRecOne: the first
};

// Record i of a bucket's table.
template <RecordPlace AT>
__device__ __forceinline__ Looked table_record(const BucketDesc &D, const Records &R, uint32_t i) {
  Looked L;
  if constexpr (AT == kRecLds) {
    const uint32_t r = R.img + D.tab_off + 16u * D.ntab + 8u * i;
    L.tail = *(lds_quad *)(uintptr_t)(R.img + D.tab_off + 16u * i);
    L.rec = (uint64_t)lds32(r + 4) << 32 | lds32(r);
  } else {
    L.tail = *(const rk_u32x4 *)(R.gimg + D.tab_off + 16u * i);
    L.rec = *(const uint64_t *)(R.gimg + D.tab_off + 16u * D.ntab + 8u * i);
  }
  return L;
}

// The record of a bucket for the window whose last 16 bytes are raw: the rank
// of the window key's bit in the lookup bitmap (rec 0: the bit is not set).
// One-key buckets hold one record; of a few keys in registers a window whose
// key is none of them gets the first one's, which its bytes do not match.
template <RecordPlace AT, uint32_t KEYS>
__device__ __forceinline__ Looked bucket_lookup(const BucketDesc &D, const Records &R, const uint32_t (&raw)[4]) {
  if constexpr (AT == kRecOne) return R.held[0];
  if constexpr (AT == kRecKeys) {
    const uint32_t v = screen_key(raw, D.shift & 0xFFu, D.mask);
    Looked L = R.held[0];
#pragma unroll
    for (uint32_t j = 1; j < KEYS; ++j) {
      const bool is = v == R.lk[j];
      L.rec = is ? R.held[j].rec : L.rec;
#pragma unroll
      for (int i = 0; i < 4; ++i) L.tail[i] = is ? R.held[j].tail[i] : L.tail[i];
    }
    return L;
  }
  uint32_t ord = 0;
  bool in = true;
  if (D.kind == kTableScreen || D.kind == kTableExact) {
    const uint32_t v = screen_key(raw, D.shift & 0xFFu, D.mask) * kMix;
    const uint32_t i = v >> D.lk_sh;
    const uint32_t w = lds32(R.img + D.lk_off + 4u * i);
    const uint32_t below = lds16(R.img + D.lk_off + (4u << (32u - D.lk_sh)) + 2u * i);
    in = filter_bit(w, v) & 1u;
    ord = in ? below + __builtin_popcount(w & ((1u << (v & 31u)) - 1u)) : 0u;
  }
  Looked L = table_record<AT>(D, R, ord);
  if (!in) L.rec = 0;
  return L;
}

// The 16 bytes ending at LDS address end (memory order), from the five aligned
// dwords that hold them.
__device__ __forceinline__ void last_bytes(uint32_t end, uint32_t (&raw)[4]) {
  const uint32_t mis = (end + 1u) & 3u, aw = end - 15u - mis;
  const uint32_t d0 = lds32(aw), d1 = lds32(aw + 4), d2 = lds32(aw + 8), d3 = lds32(aw + 12), d4 = lds32(aw + 16);
  raw[0] = __builtin_amdgcn_alignbyte(d1, d0, mis);
  raw[1] = __builtin_amdgcn_alignbyte(d2, d1, mis);
  raw[2] = __builtin_amdgcn_alignbyte(d3, d2, mis);
  raw[3] = __builtin_amdgcn_alignbyte(d4, d3, mis);
}

// Whether the windows ending at sub-tile bytes er[q] (last 16 bytes raw[q])
// are occurrences of the patterns of L[q] (one pattern each; rec 0: none):
// they start inside the text and all their bytes are equal (Sec. 3.1).  The
// last 16 bytes are compared with the record's tail, the others of a longer
// pattern with the plan's bytes, which are loaded for all Q windows, as many
// as any lane needs, before the first is used.
template <RecordPlace AT, int Q>
__device__ __forceinline__ void verify(const BucketDesc &D, const Records &R, const Looked (&L)[Q],
                                       const uint32_t (&raw)[Q][4], const uint32_t (&er)[Q], uint32_t sub,
                                       uint64_t start, const uint8_t *gtext, bool (&ok)[Q]) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
  bool m16 = false;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t mj = om_len((uint32_t)L[q].rec);
    uint32_t diff = 0;
    if ((D.shift & 0xFFu) == 2) {  // no pattern below 16 bytes
      diff = (raw[q][0] ^ L[q].tail.x) | (raw[q][1] ^ L[q].tail.y) | (raw[q][2] ^ L[q].tail.z) | (raw[q][3] ^ L[q].tail.w);
    } else {
      // shorter than 16 bytes: the newest mj of them
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int nb = (int)mj - 4 * (3 - j);
        const uint32_t keep = nb <= 0 ? 0u : (nb >= 4 ? 0xFFFFFFFFu : 0xFFFFFFFFu << (8 * (4 - nb)));
        diff |= (raw[q][j] ^ L[q].tail[j]) & keep;
      }
    }
    ok[q] = L[q].rec != 0 && diff == 0 && start + er[q] + 1u >= mj;
    m16 = m16 || (ok[q] && mj > 16);
  }
  if (ballot(m16) == 0) return;
  bool m32 = false, m48 = false, m64 = false;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t mj = om_len((uint32_t)L[q].rec);
    m32 = m32 || (ok[q] && mj > 32);
    m48 = m48 || (ok[q] && mj > 48);
    m64 = m64 || (ok[q] && mj > kFront);
  }
  m32 = ballot(m32) != 0;
  m48 = ballot(m48) != 0;
  rk_u32x4 h[Q][3];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t pat = D.pat_off + om_off((uint32_t)L[q].rec);
    if (ok[q] && om_len((uint32_t)L[q].rec) > 16) {
      if (AT == kRecLds && (D.shift & (1u << 17))) {
        const uint32_t p = R.img + pat;
        h[q][0] = rk_u32x4{lds32(p), lds32(p + 4), lds32(p + 8), lds32(p + 12)};
        if (m32) h[q][1] = rk_u32x4{lds32(p + 16), lds32(p + 20), lds32(p + 24), lds32(p + 28)};
        if (m48) h[q][2] = rk_u32x4{lds32(p + 32), lds32(p + 36), lds32(p + 40), lds32(p + 44)};
      } else {
        h[q][0] = *(const u32x4 *)(R.gimg + pat);
        if (m32) h[q][1] = *(const u32x4 *)(R.gimg + pat + 16);
        if (m48) h[q][2] = *(const u32x4 *)(R.gimg + pat + 32);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t mj = om_len((uint32_t)L[q].rec), a = sub + kFront + er[q] + 1u - mj;
    if (ok[q] && mj > 16 && mj <= kFront) {
      ok[q] = quad_equals(a, h[q][0], (int)mj - 16);
      if (m32) ok[q] = ok[q] && quad_equals(a + 16, h[q][1], (int)mj - 32);
      if (m48) ok[q] = ok[q] && quad_equals(a + 32, h[q][2], (int)mj - 48);
    }
    // beyond the sub-tile's front halo: compared in the text itself (the LDS
    // part leads the device image, so offsets hold in both)
    if (ballot(m64) && ok[q] && mj > kFront)
      ok[q] = window_equals_global(gtext + (start + er[q] + 1u - mj), R.gimg + D.pat_off + om_off((uint32_t)L[q].rec), mj);
  }
}

// Candidate phase of one bucket on one sub-tile, by one wave.  bits holds the
// lane's candidate mask (window i: bit i%32 of word i/32).
// Windows that start before the text or end after it are dropped, the
// candidates are compacted into the wave's LDS list in window order, and each
// is checked by one lane: its key's record, then its bytes.  A bit that
// several patterns share is put off: its candidates go back to the front of
// the list and are checked after the others (a pattern's hits come all from
// the one or all from the other, so each keeps the window order).  Where the
// records fill device memory, runs are many and long: their pairs of a
// candidate and a pattern are taken a lane each (6,000 patterns of word text,
// runs of up to 8, 64 MiB: 371 us, 397 with as many rounds as the longest run
// of 64 candidates, a lane walking its own); the fewer ones of a table in LDS
// are walked (1,024 patterns, 1 GiB: 583 us in pairs, 565 walked).  Hits go to the tile's slab (up to cap records);
// tile_hits counts them all.  Returns the number of candidates (uniform).
//
// A wave works alone (no block barrier anywhere in the scan), so its LDS and
// memory latencies are covered by the other waves of the CU, whatever they
// are doing; records and pattern bytes in memory are loaded for 128 candidates
// at a time.
template <int C, RecordPlace AT, uint32_t KEYS = 1>
__device__ __forceinline__ uint32_t wave_candidates(Bits<C> &bits, const BucketDesc &D, uint32_t sub, uint64_t start,
                                                    uint64_t n, const Records &R, uint32_t cand,
                                                    uint64_t *slab, uint32_t cap, uint32_t &tile_hits,
                                                    const uint8_t *gtext, unsigned long long *pid_counts) {
  constexpr uint32_t SUB = 64 * C;
  constexpr int NB = (C + 31) / 32;
  const uint32_t lane = threadIdx.x & 63;
  // only windows with m-1 <= e <= n-1 exist
  if (start < (uint64_t)D.m - 1 || start + SUB > n) {
    // my windows i are valid for ilo <= i < ihi
    const int64_t e0 = (int64_t)start + lane * C;
    const int64_t lo64 = (int64_t)D.m - 1 - e0, hi64 = (int64_t)n - e0;
    const int ilo = (int)(lo64 < 0 ? 0 : (lo64 > C ? C : lo64));
    const int ihi = (int)(hi64 < 0 ? 0 : (hi64 > C ? C : hi64));
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int nw = word_windows<C>(j);
      int a = ilo - 32 * j, b2 = ihi - 32 * j;
      a = a < 0 ? 0 : (a > nw ? nw : a);
      b2 = b2 < 0 ? 0 : (b2 > nw ? nw : b2);
      // keep bits [a, b2)
      const uint32_t below_b = b2 >= 32 ? 0xFFFFFFFFu : ((1u << b2) - 1u);
      const uint32_t below_a = a >= 32 ? 0xFFFFFFFFu : ((1u << a) - 1u);
      bits.b[j] &= below_b & ~below_a;
    }
  }
  uint32_t cnt = 0;
#pragma unroll
  for (int j = 0; j < NB; ++j) cnt += __builtin_popcount(bits.b[j]);
  if (ballot(cnt != 0) == 0) return 0;
  const uint32_t incl = wave_incl_scan(cnt);
  const uint32_t ncand = __builtin_amdgcn_readlane(incl, 63);

  for (uint32_t r0 = 0; r0 < ncand; r0 += kWaveCand) {
    wave_lds_fence();  // the list's readers of the last round are done
    uint32_t idx = incl - cnt - r0;  // (wraps for entries of earlier rounds: not below kWaveCand)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      uint32_t bb = bits.b[j];
      const uint32_t first = lane * C + 32u * j;
      if (ncand <= kWaveCand) {
        while (bb) {
          *(lds_half *)(uintptr_t)(cand + 2u * idx++) = (uint16_t)(first + __builtin_ctz(bb));
          bb &= bb - 1u;
        }
      } else {
        for (; bb; bb &= bb - 1u, ++idx)
          if (idx < kWaveCand) *(lds_half *)(uintptr_t)(cand + 2u * idx) = (uint16_t)(first + __builtin_ctz(bb));
      }
    }
    wave_lds_fence();
    const uint32_t nc = min(kWaveCand, ncand - r0);
    auto window = [&](uint32_t i, uint32_t count, uint32_t &e_rel, uint32_t(&raw)[4])
        __attribute__((always_inline)) -> Looked {
      e_rel = lds16(cand + 2u * min(i + lane, count - 1));
      last_bytes(sub + kFront + e_rel, raw);
      Looked L = bucket_lookup<AT, KEYS>(D, R, raw);
      if (i + lane >= count) L.rec = 0;
      return L;
    };
    // a hit for each of the pattern's ids
    auto emit = [&](bool ok, uint64_t rec, uint32_t e_rel) __attribute__((always_inline)) {
      uint64_t hit = ballot(ok);
      if (hit == 0) return;
      const uint64_t x = start + e_rel + 1u - om_len((uint32_t)rec);
      const uint32_t nid = ok ? (rec_same(rec) ? same_count(rec) : 1u) : 0u;
      uint32_t pid = (uint32_t)(rec >> 32) & 0xFFFFFFu;
      const bool ids = ballot(ok && rec_same(rec)) != 0;
      for (uint32_t j = 0;;) {
        if (ids && nid > j && rec_same(rec)) {
          const uint32_t q = D.ids_off + 4u * (same_first(rec) + j);
          if (AT == kRecLds || (AT == kRecGlobal && (D.shift & (1u << 18)))) pid = lds32(R.img + q);
          else pid = *(const uint32_t *)(R.gimg + q);
        }
        if (nid > j) {
          const uint32_t o = tile_hits + lanes_below(hit);
          if (o < cap) slab[o] = ((uint64_t)pid << kPosBits) | x;
          if (pid_counts) atomicAdd(pid_counts + pid, 1ull);
        }
        tile_hits += (uint32_t)__builtin_popcountll(hit);
        if (!ids) break;
        ++j;
        hit = ballot(nid > j);
        if (!hit) break;
      }
    };
    constexpr int Q = AT == kRecOne ? 1 : 2;
    uint32_t nd = 0;  // put off (never past what has been read of the list)
    for (uint32_t i0 = 0; i0 < nc; i0 += 64 * Q) {
      Looked L[Q];
      uint32_t er[Q], raw[Q][4];
      bool ok[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (q == 0 || i0 + 64 * q < nc) {
          L[q] = window(i0 + 64 * q, nc, er[q], raw[q]);
        } else {
          L[q] = Looked{};
          er[q] = raw[q][0] = raw[q][1] = raw[q][2] = raw[q][3] = 0;
        }
      }
      if constexpr (AT != kRecOne) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const bool run = L[q].rec && !rec_one_pattern(L[q].rec);
          const uint64_t b = ballot(run);
          if (b) {
            if (run) {
              *(lds_half *)(uintptr_t)(cand + 2u * (nd + lanes_below(b))) = (uint16_t)er[q];
              L[q].rec = 0;
            }
            nd += (uint32_t)__builtin_popcountll(b);
          }
        }
      }
      verify<AT, Q>(D, R, L, raw, er, sub, start, gtext, ok);
#pragma unroll
      for (int q = 0; q < Q; ++q) emit(ok[q], L[q].rec, er[q]);
    }
    if constexpr (AT != kRecOne) {
      if (nd) wave_lds_fence();
      if constexpr (AT == kRecGlobal || AT == kRecKeys) {
        for (uint32_t i0 = 0; i0 < nd; i0 += 64) {
          // pairs of a candidate and a pattern of its run, 64 Q at a time, in
          // the candidates' order
          uint32_t e, last[4];
          const uint64_t run = window(i0, nd, e, last).rec;
          const uint32_t count = (uint32_t)(run >> 32), incl = wave_incl_scan(count);
          const uint32_t rel = (uint32_t)run - (incl - count);  // record of pair p: rel + p
          const uint32_t pairs = __builtin_amdgcn_readlane(incl, 63);
          for (uint32_t p0 = 0; p0 < pairs; p0 += 64 * Q) {
            Looked L[Q];
            uint32_t er[Q], raw[Q][4];
            bool ok[Q];
  #pragma unroll
            for (int q = 0; q < Q; ++q) {
              L[q] = Looked{};
              er[q] = raw[q][0] = raw[q][1] = raw[q][2] = raw[q][3] = 0;
              if (q > 0 && p0 + 64 * q >= pairs) continue;
              const uint32_t p = p0 + 64 * q + lane;
              // its candidate's lane: the first one whose incl is above p
              uint32_t o = 0;
  #pragma unroll
              for (uint32_t step = 32; step; step >>= 1)
                o += (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (o + step - 1), (int)incl) <= p ? step : 0;
              er[q] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * o, (int)e);
              const uint32_t r = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * o, (int)rel) + p;
              last_bytes(sub + kFront + er[q], raw[q]);
              L[q] = table_record<AT>(D, R, p < pairs ? r : 0);
              if (p >= pairs) L[q].rec = 0;
            }
            verify<AT, Q>(D, R, L, raw, er, sub, start, gtext, ok);
  #pragma unroll
            for (int q = 0; q < Q; ++q) emit(ok[q], L[q].rec, er[q]);
          }
        }
      } else {
        for (uint32_t i0 = 0; i0 < nd; i0 += 64) {
          Looked L[1];
          uint32_t er[1], raw[1][4];
          bool ok[1];
          const uint64_t run = window(i0, nd, er[0], raw[0]).rec;
          const uint32_t first = (uint32_t)run, count = (uint32_t)(run >> 32);
          for (uint32_t i = 0; ballot(i < count); ++i) {
            L[0] = table_record<AT>(D, R, i < count ? first + i : 0);
            if (i >= count) L[0].rec = 0;
            verify<AT, 1>(D, R, L, raw, er, sub, start, gtext, ok);
            emit(ok[0], L[0].rec, er[0]);
          }
        }
      }
    }
  }
  return ncand;
}

// Scalar loads of what the kernel does not write (p wave-uniform).
typedef const __attribute__((address_space(4))) uint32_t const_word;
__device__ __forceinline__ uint32_t const32(const void *p) { return *(const_word *)(uintptr_t)p; }
__device__ __forceinline__ uint64_t const64(const void *p) {
  return *(const __attribute__((address_space(4))) uint64_t *)(uintptr_t)p;
}

// Bucket descriptor b of the image at gimg (device memory).
__device__ __forceinline__ BucketDesc read_desc(const uint8_t *gimg, uint32_t b) {
  const_word *q = (const_word *)(uintptr_t)(gimg + sizeof(ImageHeader) + 64u * b);
  BucketDesc D;
  uint32_t *d = (uint32_t *)&D;
#pragma unroll
  for (int j = 0; j < 16; ++j) d[j] = q[j];
  return D;
}

// ------------------------------------------------------------ the scan kernel
//
// Work comes in runs of consecutive tiles of one instance; the waves of a
// block take a run's tiles in turn, each wave scanning its tile's sub-tiles in
// order.  The block shares the instance image in LDS, so its waves meet
// (barriers) when the image changes and, with a queue and several waves, when
// a run is popped; a block of one wave never waits for another.  A wave has
// one sub-tile slot: the next sub-tile's loads are issued when the last read
// of the current one is done, and the other waves' work covers them (a second
// slot would cost the waves that do so).
//
// LDS: [image: img_cap][queue word: 16][per wave: slot, candidates]
template <int WG, int C, int FAM>
__global__ __launch_bounds__(scan_block_max(C, FAM)) void scan_kernel(ScanParams p) {
  constexpr uint32_t SUB = 64 * C;
  constexpr int NB = (C + 31) / 32;
  static_assert(WG % 64 == 0, "a tile is at most WG / 64 sub-tiles");
  extern __shared__ __align__(16) uint8_t lds[];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), nw = blockDim.x >> 6;
  const uint32_t img = lds_addr(lds);
  uint32_t *popw = (uint32_t *)(lds + p.img_cap);
  const uint32_t sub = img + p.img_cap + 16 + wave * wave_lds_bytes<C>(1);
  const uint32_t cand = sub + sub_slot_bytes<C>(), mine = sub + kFront + lane * C;

  struct Item {
    uint64_t gt;         // tile
    uint64_t n, tstart;  // its text's length, its first byte
    const uint8_t *text;
    uint32_t inst;
  };
  // (the instance of a launch of one comes with the kernel's arguments)
  const InstDesc *const insts =
      p.inst ? p.inst
             : (const InstDesc *)((uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(ScanParams, one));
  if (!p.queue && p.ovf_count && blockIdx.x == 0 && tid == 0) *p.ovf_count = *p.done = 0;
  // the run this wave is in: its remaining tiles are tnext, tnext + nw, ...
  uint64_t next_run = blockIdx.x, tnext = 0, tbase = 0, rn = 0;
  const uint8_t *rtext = nullptr;
  uint32_t tleft = 0, rinst = kNoLink;
  const uint64_t nlist = p.nitems_dev ? min(p.nitems, (uint64_t)const32(p.nitems_dev)) : p.nitems;
  const uint64_t nruns = p.wave_items ? (nlist + nw - 1) / nw : p.nitems;

  // The wave's next tile: 1 (in it), 2 (none in this run, but its image is to
  // be switched to), 0 (no run left).
  auto next_item = [&](Item &it) __attribute__((always_inline)) -> uint32_t {
    if (tleft == 0) {
      uint64_t r = next_run;
      if (!p.queue) {
        next_run += gridDim.x;
      } else if (next_run == blockIdx.x) {
        next_run = ~0ull;  // the first run needs no pop
      } else {
        // the block's cursor hands out every ncur-th of the other runs
        const uint32_t ncur = min(gridDim.x, kCursors), c = blockIdx.x % ncur;
        uint32_t *q = p.queue + c * (kCursorStride / 4);
        uint32_t v = 0;
        if (nw == 1) {
          if (lane == 0) v = atomicAdd(q, 1u);
        } else {
          wg_barrier();
          if (tid == 0) popw[0] = atomicAdd(q, 1u);
          wg_barrier();
          v = popw[0];
        }
        r = gridDim.x + (uint64_t)uni(v) * ncur + c;
      }
      if (r >= nruns) return 0;
      uint64_t first;
      if (p.wave_items) {
        const uint64_t q = r * nw + wave;
        first = tnext = const64(p.items + (q < nlist ? q : nlist - 1));
        tleft = q < nlist && first >= p.item_lo && first < p.item_hi ? 1u : 0u;
      } else {
        uint32_t cnt;
        if (p.items) {
          const uint64_t v = const64(p.items + r);
          first = v & kItemTile;
          cnt = (uint32_t)(v >> kItemShift);
        } else {
          const uint64_t i = p.ninst > 1 ? r / p.inst_runs : 0, q = (r - i * p.inst_runs) * p.run;
          first = i * p.inst_tiles + q;
          cnt = (uint32_t)min((uint64_t)p.run, p.inst_tiles - q);
        }
        tleft = cnt > wave ? (cnt - wave + nw - 1u) / nw : 0u;
        tnext = first + wave;
      }
      uint32_t lo = 0, hi = p.ninst;  // instance owning the tile
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (const64(&insts[mid].tile_base) <= first) lo = mid;
        else hi = mid;
      }
      if (lo != rinst) {
        rinst = lo;
        rtext = (const uint8_t *)const64(&insts[lo].text);
        rn = const64(&insts[lo].n);
        tbase = const64(&insts[lo].tile_base);
      }
    }
    it.inst = rinst;
    if (tleft == 0) return 2;
    it.gt = tnext;
    it.text = rtext;
    it.n = rn;
    it.tstart = (tnext - tbase) * ((uint64_t)SUB * p.sub);
    tnext += nw;
    --tleft;
    return 1;
  };

  uint32_t cur_inst = kNoLink, nb = 0;
  const uint8_t *gimg = nullptr;  // current instance image in device memory
  Item cur;
  uint32_t st = next_item(cur);
  if (st == 1) dma_sub<C>(sub, cur.text, cur.n, cur.tstart);
  while (st) {
    if (cur.inst != cur_inst) {
      // the image's leading part goes to LDS; the rest is read in place
      if (nw > 1) wg_barrier();
      gimg = p.blob + const32(&insts[cur.inst].img_off);
      const uint4 *src = (const uint4 *)gimg;
      uint4 *dst = (uint4 *)lds;
      const uint32_t nq = const32(&insts[cur.inst].lds_bytes) / 16u;
      for (uint32_t q = tid; q < nq; q += blockDim.x) dst[q] = src[q];
      cur_inst = cur.inst;
      wg_barrier();
      nb = const32(gimg);  // ImageHeader::nbuckets
    }
    if (st == 2) {
      st = next_item(cur);
      if (st == 1) dma_sub<C>(sub, cur.text, cur.n, cur.tstart);
      continue;
    }
    uint64_t *slab = nullptr;
    if (p.out)
      slab = p.direct ? p.out + const64(p.tile_offsets + cur.gt) : p.out + (cur.gt - p.tile0) * (uint64_t)p.slab_cap;
    const uint32_t cap = p.direct ? 0xFFFFFFFFu : p.slab_cap;
    const uint32_t ns = (uint32_t)min((uint64_t)p.sub, (cur.n - cur.tstart + SUB - 1) / SUB);
    uint32_t tile_hits = 0;
    Item nx;
    for (uint32_t s = 0; s < ns; ++s) {
      const uint64_t start = cur.tstart + (uint64_t)s * SUB;
      if (s + 1 == ns) st = next_item(nx);  // (its reads are under way with the sub-tile's)
      wait_loads();                         // this sub-tile has landed
      for (uint32_t b = 0; b < nb; ++b) {
        const BucketDesc D = read_desc(gimg, b);
        const uint32_t r = (8u * D.m) % 61u;
        const OutStream os = out_stream(mine, D.m);
        if constexpr (FAM == kFamExact) {
          if (D.kind == kDump) {
            pass_dump<C>(mine, os, D.m, r, (int64_t)(start + lane * C), cur.n,
                         DumpDst{p.dump_out, p.dump_stride, p.dump_cap});
            continue;
          }
        }
        Bits<C> bits;
#pragma unroll
        for (int j = 0; j < NB; ++j) bits.b[j] = 0;
        run_pass<C, FAM>(D, mine, os, r, img + D.test_off, bits);
        const Records R{img, gimg, {}, {}};
        unsigned long long *const pc = p.direct ? nullptr : p.pid_counts;
        if (D.shift & (1u << 16))
          wave_candidates<C, kRecLds>(bits, D, sub, start, cur.n, R, cand, slab, cap, tile_hits, cur.text, pc);
        else
          wave_candidates<C, kRecGlobal>(bits, D, sub, start, cur.n, R, cand, slab, cap, tile_hits, cur.text, pc);
      }
      wait_lds();  // every read of the slot is done
      if (s + 1 < ns) dma_sub<C>(sub, cur.text, cur.n, start + SUB);
      else if (st == 1) dma_sub<C>(sub, nx.text, nx.n, nx.tstart);
    }
    if (lane == 0 && !p.direct) p.tile_counts[cur.gt] = tile_hits;
    cur = nx;
  }
}

// ------------------------------------------------- single-bucket scan kernel
// The same scan for the most common plan shapes: one text and one bucket with
// one key (one pattern, or one pattern under several ids) or a few (up to
// kFewScreen in screen mode, kFewExact in exact mode).  The bucket
// descriptor, the text and the keys' records come as kernel arguments, tiles
// are strided statically over the waves of the grid, and there is no image
// staging, work list or instance lookup, so a sub-tile costs little beyond its
// hash pass.  Count mode only (hits into per-tile slabs); a tile whose slab
// overflows is rescanned by the general kernel, from the image's tables.
//
// A sub-tile without a candidate is decided by the test pass alone (a compare
// and a scalar OR per window and key); after one with candidates the wave runs the
// mask pass straight away, until a sub-tile has none.  Two slots: the next
// sub-tile loads while this one is tested.
//
// LDS: per wave [slot 0][slot 1][candidates]
template <int WG, int C, int FAM>
__global__ __launch_bounds__(kListBlock) void scan_list_kernel(ListParams p) {
  constexpr uint32_t SUB = 64 * C, SLOT = sub_slot_bytes<C>();
  constexpr int NB = (C + 31) / 32;
  extern __shared__ __align__(16) uint8_t lds[];
  const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  const uint32_t slots = lds_addr(lds) + wave * wave_lds_bytes<C>(2);
  const uint32_t cand = slots + 2 * SLOT;
  const BucketDesc D = p.D;
  const uint32_t r = p.rot;
  const uint64_t W = (uint64_t)SUB * p.sub, stride = (uint64_t)gridDim.x * (kListBlock / 64);
  uint32_t slot = 0;
  bool dense = false;
  if (p.ovf_count && blockIdx.x == 0 && threadIdx.x == 0) *p.ovf_count = *p.done = 0;
  uint64_t t = (uint64_t)blockIdx.x * (kListBlock / 64) + wave;
  if (t < p.ntiles) dma_sub<C>(slots, p.text, p.n, t * W);
  for (; t < p.ntiles; t += stride) {
    const uint64_t tstart = t * W;
    const uint32_t ns = (uint32_t)min((uint64_t)p.sub, (p.n - tstart + SUB - 1) / SUB);
    uint32_t tile_hits = 0;
    for (uint32_t s = 0; s < ns; ++s) {
      const uint32_t sub = slots + slot * SLOT, mine = sub + kFront + lane * C;
      const uint64_t start = tstart + (uint64_t)s * SUB;
      wait_loads();
      const uint64_t nstart = s + 1 < ns ? start + SUB : (t + stride < p.ntiles ? (t + stride) * W : p.n);
      if (nstart < p.n) dma_sub<C>(slots + (slot ^ 1u) * SLOT, p.text, p.n, nstart);
      slot ^= 1u;
      const OutStream os = out_stream(mine, D.m);
      Bits<C> bits;
      if constexpr (FAM == kFamExact) {
        if (D.kind == kDump) {
          pass_dump<C>(mine, os, D.m, r, (int64_t)(start + lane * C), p.n,
                       DumpDst{p.dump_out, p.dump_stride, p.dump_cap});
          continue;
        }
      }
      uint64_t any = 0;
      if (!dense) {
        run_few<C, true, FAM>(D, mine, os, r, p.nkeys, p.tgt2, any, bits);
        if (any == 0) continue;
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) bits.b[j] = 0;
      run_few<C, false, FAM>(D, mine, os, r, p.nkeys, p.tgt2, any, bits);
      constexpr uint32_t KEYS = FAM == kFamScreen ? kFewScreen : FAM == kFamExact ? kFewExact : 1;
      Records R{0, p.gimg, {}, {}};
#pragma unroll
      for (uint32_t j = 0; j < KEYS; ++j) {
        R.lk[j] = p.key[j].lk;
        R.held[j] = Looked{p.key[j].rec, {p.key[j].tail[0], p.key[j].tail[1], p.key[j].tail[2], p.key[j].tail[3]}};
      }
      uint64_t *const slab = p.out + t * (uint64_t)p.slab_cap;
      uint32_t nc;
      if (FAM != kFamScreen && p.nkeys == 1 && rec_one_pattern(p.key[0].rec))
        nc = wave_candidates<C, kRecOne>(bits, D, sub, start, p.n, R, cand, slab, p.slab_cap, tile_hits, p.text,
                                         p.pid_counts);
      else
        nc = wave_candidates<C, kRecKeys, KEYS>(bits, D, sub, start, p.n, R, cand, slab, p.slab_cap, tile_hits, p.text,
                                                p.pid_counts);
      dense = nc != 0;
    }
    if (lane == 0 && D.kind != kDump) p.tile_counts[t] = tile_hits;
  }
}

// ------------------------------------------------------------------ launchers
template <int C>
constexpr uint32_t list_lds_bytes_t() {
  return kListBlock / 64 * wave_lds_bytes<C>(2);
}

template <int WG, int C, int FAM>
static hipError_t launch_scan_t(const ScanParams &p, uint32_t grid, uint32_t block, hipStream_t s) {
  // the dynamic LDS limit was raised by prepare_scan_kernels() at context creation
  const uint32_t lds = p.img_cap + 16 + block / 64 * wave_lds_bytes<C>(1);
  hipLaunchKernelGGL((scan_kernel<WG, C, FAM>), dim3(grid), dim3(block), lds, s, p);
  return hipGetLastError();
}

template <int WG, int C, int FAM>
static hipError_t launch_list_t(const ListParams &p, uint32_t grid, hipStream_t s) {
  constexpr uint32_t lds = list_lds_bytes_t<C>();
  hipLaunchKernelGGL((scan_list_kernel<WG, C, FAM>), dim3(grid), dim3(kListBlock), lds, s, p);
  return hipGetLastError();
}

// Geometry CFG of kTileCfgs as template arguments.
template <int CFG>
struct Geom {
  static constexpr int WG = kTileCfgs[CFG].wg, C = kTileCfgs[CFG].c;
};

template <int FAM, int CFG>
hipError_t ScanGeom<FAM, CFG>::launch(const ScanParams &p, uint32_t grid, uint32_t block, hipStream_t s) {
  return launch_scan_t<Geom<CFG>::WG, Geom<CFG>::C, FAM>(p, grid, block, s);
}

template <int FAM, int CFG>
hipError_t ScanGeom<FAM, CFG>::fit(uint32_t img_cap, uint32_t block, ScanFit *f) {
  constexpr int WG = Geom<CFG>::WG, C = Geom<CFG>::C;
  f->wave_lds = wave_lds_bytes<C>(1);
  f->max_block = scan_block_max(C, FAM);
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&f->blocks, (const void *)scan_kernel<WG, C, FAM>, block,
                                                      img_cap + 16 + block / 64 * f->wave_lds);
}

template <int FAM, int CFG>
hipError_t ScanGeom<FAM, CFG>::list(const ListParams *p, uint32_t grid, hipStream_t s, int *blocks) {
  constexpr int WG = Geom<CFG>::WG, C = Geom<CFG>::C;
  if (p) return launch_list_t<WG, C, FAM>(*p, grid, s);
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, (const void *)scan_list_kernel<WG, C, FAM>, kListBlock,
                                                      list_lds_bytes_t<C>());
}

template <int FAM, int CFG>
hipError_t ScanGeom<FAM, CFG>::prepare() {
  return hipFuncSetAttribute((const void *)scan_kernel<Geom<CFG>::WG, Geom<CFG>::C, FAM>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

template <int FAM, int CFG>
hipError_t ScanGeom<FAM, CFG>::list_prepare() {
  return hipFuncSetAttribute((const void *)scan_list_kernel<Geom<CFG>::WG, Geom<CFG>::C, FAM>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

// Explicit instantiation of the general kernel's launchers (X = launch) or
// the single-bucket kernel's (X = list) for family FAM and geometry CFG.
#define RK_INSTANTIATE_SCAN(FAM, CFG)                                                                     \
  template hipError_t ScanGeom<FAM, CFG>::launch(const ScanParams &, uint32_t, uint32_t, hipStream_t); \
  template hipError_t ScanGeom<FAM, CFG>::fit(uint32_t, uint32_t, ScanFit *);                           \
  template hipError_t ScanGeom<FAM, CFG>::prepare();
#define RK_INSTANTIATE_LIST(FAM, CFG)                                                                    \
  template hipError_t ScanGeom<FAM, CFG>::list(const ListParams *, uint32_t, hipStream_t, int *);      \
  template hipError_t ScanGeom<FAM, CFG>::list_prepare();

}  // namespace rk
