// Internal layouts shared by the host runtime and the HIP kernels of librk.
//
// Text windows are identified by their END byte e (window = T[e-m+1 .. e]):
// a tile owns the windows whose last byte falls inside it, so every thread
// ingests its own bytes at static register positions and the (m-1)-byte
// halo sits in front of the tile.  Start position x = e - m + 1.
#pragma once
#include <stdint.h>

namespace rk {

constexpr uint64_t kQ = (1ull << 61) - 1;  // Mersenne modulus 2^61 - 1
constexpr uint32_t kFront = 64;            // halo bytes kept in front of a tile (= kStreamM)
constexpr uint32_t kStreamM = 64;          // longest window hashed by a rolling stream; longer patterns are
                                           // keyed by their last kStreamM bytes
constexpr uint32_t kPosBits = 40;          // hit record = pid << 40 | start position
constexpr uint64_t kPosMask = (1ull << kPosBits) - 1;
constexpr uint32_t kWaveCand = 256;         // candidate slots in LDS per wave (window index in the sub-tile, u16)
constexpr uint32_t kListBlock = 256;       // threads of a single-bucket scan's block (its waves are independent)
constexpr uint32_t kNoLink = 0xFFFFFFFFu;

// Screen/test variants of one bucket (one pattern length inside one instance).
enum BucketKind : uint32_t {
  kListScreen = 0,   // screen mode, one key: shift-add hash compared with it
  kTableScreen = 1,  // screen mode: shift-add hash tested in the LDS bitmap
  kListExact = 2,    // exact mode, one key: lazy 61-bit hash compared with its lazy forms
  kTableExact = 3,   // exact mode: lazy state tested in the LDS bitmap
  kDump = 4,         // exact rolling state written out for sampled windows (no patterns)
};

// Group descriptor as laid out in an instance image (64 bytes).  A group is a
// set of patterns tested with one hash stream: one length class in exact mode
// (keyed on its shortest length), one screen-hash span in screen mode.
//
// Bitmaps have 2^(32 - sh) 32-bit words; a 32-bit value v sits in word v >> sh,
// bit v & 31.  The test bitmap holds what the stream tests (screen: the keys
// times kMix; exact: exact_mix of every lazy form of every key), the lookup
// bitmap the patterns' shift-add keys times kMix, whose bits in ascending
// order number the records; it is followed by u16 counts of the set bits
// before each word.  In screen groups the two are one.
struct BucketDesc {
  uint32_t m;          // the group's shortest length: the window its exact stream hashes
  uint32_t kind;       // BucketKind
  uint32_t shift;      // shift s of the screen or lookup hash in bits 0-7; in the LDS part: bit 16 tails and
                       // records, 17 pattern bytes, 18 ids
  uint32_t mask;       // screen-hash mask (all ones unless m < 4 with s = 8)
  uint32_t tgt[4];     // one screen key (four times); one exact key by the window's place in a step of four
  uint32_t test_off;   // table kinds: image offset of the test bitmap (LDS part)
  uint32_t test_sh;    // its sh
  uint32_t lk_off;     // table kinds: image offset of the lookup bitmap and its counts (LDS part)
  uint32_t lk_sh;      // the lookup bitmap's sh
  uint32_t tab_off;    // per record its pattern's last 16 bytes (zeros before a shorter one), then u64 records
  uint32_t ntab;       // records: one per lookup bit, then those of the bits' runs
  uint32_t ids_off;    // u32 pattern ids of the patterns that have several
  uint32_t pat_off;    // pattern bytes; om_pack offsets are relative to this
};
static_assert(sizeof(BucketDesc) == 64, "bucket descriptor is 64 bytes");

// Shift-add keys are looked up times this odd constant, mod 2^32.  The product
// rolls like the hash itself (p <- (p << s) + kMix c) at no cost: the
// multiplication by kMix takes the entering byte out of its word, which the
// hash needs an instruction for as well.  Its high bits spread like random
// ones: on word text with 1,024 patterns 1.5% of the windows pass an 8 KiB
// bitmap besides the matches, as many as bits are set; the high half of the
// hash itself lets 5.4% pass (sums of letters).
constexpr uint32_t kMix = 0x85EBCB;

// What the test bitmap of exact keys holds of a lazy state s: one dot product
// of its low word's halves with two constants plus its high word.  (The low
// word of a short window's hash is its last four bytes: alone it lets 56% of a
// DNA text pass the bitmap of 32 patterns of 8 to 15 bytes, 28% of word text
// that of 100, against 4% and 7% so.)
constexpr uint32_t kExactMixLo = 0x9E37, kExactMixHi = 0x79B1;
inline uint32_t exact_mix(uint64_t s) {
  const uint32_t lo = (uint32_t)s;
  return (lo & 0xFFFFu) * kExactMixLo + (lo >> 16) * kExactMixHi + (uint32_t)(s >> 32);
}

constexpr uint32_t kMinBitmap = 256, kMaxBitmap = 32 * 1024;  // bytes

// Pattern reference of an entry: byte offset in its group's pattern block
// (bits 0-21, so a group holds at most 4 MiB of pattern bytes) and length - 1
// (bits 22-31, lengths 1..1024).
constexpr uint32_t kOmOffBits = 22;
constexpr uint32_t kGroupPatBytes = 1u << kOmOffBits;
__host__ __device__ inline uint32_t om_pack(uint32_t off, uint32_t m) { return off | ((m - 1u) << kOmOffBits); }
__host__ __device__ inline uint32_t om_len(uint32_t om) { return (om >> kOmOffBits) + 1u; }
__host__ __device__ inline uint32_t om_off(uint32_t om) { return om & (kGroupPatBytes - 1u); }

// Record of a lookup bit (list kinds: of the one key): its pattern, or the run
// of records of several different patterns.
//   bit 63 set : one pattern with one id, in bits 32..55, off_m in bits 0..31
//   bits 63-62 = 01: one pattern with several ids: count - 1 in bits 54..61,
//                index of the first in the id list in bits 32..53, off_m in
//                bits 0..31
//   bits 63-62 = 00: records [first, first + count): count in bits 32..61 (0:
//                no record), first in bits 0..31
__host__ __device__ inline uint64_t rec_inline(uint32_t pid, uint32_t off_m) {
  return (1ull << 63) | ((uint64_t)pid << 32) | off_m;
}
__host__ __device__ inline uint64_t rec_run(uint32_t first, uint32_t count) {
  return ((uint64_t)count << 32) | first;
}
constexpr uint32_t kSameMaxCount = 256, kSameMaxFirst = 1u << 22;
__host__ __device__ inline uint64_t rec_ids(uint32_t first, uint32_t count, uint32_t off_m) {
  return (1ull << 62) | ((uint64_t)(count - 1u) << 54) | ((uint64_t)first << 32) | off_m;
}
__host__ __device__ inline bool rec_one_pattern(uint64_t rec) { return (rec >> 62) != 0; }
__host__ __device__ inline bool rec_same(uint64_t rec) { return (rec >> 62) == 1u; }
__host__ __device__ inline uint32_t same_count(uint64_t rec) { return (uint32_t)((rec >> 54) & 0xFFu) + 1u; }
__host__ __device__ inline uint32_t same_first(uint64_t rec) { return (uint32_t)(rec >> 32) & (kSameMaxFirst - 1u); }

// Header at the start of an instance image (16 bytes), followed by nb
// descriptors, the parts staged in LDS and the parts read from device memory.
struct ImageHeader {
  uint32_t nbuckets;
  uint32_t bytes;      // total image bytes (multiple of 16)
  uint32_t max_m;
  uint32_t lds_bytes;  // leading bytes staged in LDS (header, descriptors, bitmaps, small record tables)
};

// One instance of a scan job (48 bytes).
struct InstDesc {
  const uint8_t *text; // 16-byte aligned
  uint64_t n;
  uint64_t tile_base;  // global id of this instance's tile 0
  uint64_t ntiles;
  uint32_t img_off;    // byte offset of the instance image in the plan blob (16-aligned)
  uint32_t lds_bytes;  // leading image bytes the scan stages in LDS
  uint64_t pad;
};
static_assert(sizeof(InstDesc) == 48, "instance descriptor is 48 bytes");

// The work queue of a batch has kCursors cursors on a 128-byte line each:
// additions to one address are served one after the other, 15 ns a pop (with
// one cursor 1,024 instances of 2 GB spent 0.5 of 1.0 ms on pops).  For the
// same reason the scan adds its hits to no counter: the prefix sum over the
// tiles' counts, which the collect needs anyway, yields the total (every tile
// adding to one counter was the bound of dense scans, 0.8 ms for the 61,681
// tiles of a 1 GiB text).
constexpr uint32_t kCursors = 16, kCursorStride = 128;

// A run of consecutive tiles of one instance in a work list.
constexpr uint32_t kItemShift = 48;
constexpr uint64_t kItemTile = (1ull << kItemShift) - 1;

// Kernel parameters of the scan (passed by value).
struct ScanParams {
  const InstDesc *inst;       // nullptr: one instance, in `one`
  uint32_t ninst;
  uint32_t img_cap;           // LDS bytes reserved for an instance image
  const uint8_t *blob;        // instance images
  uint32_t sub;               // sub-tiles of 64 C bytes per tile
  const uint64_t *items;      // runs: first global tile id | tiles << kItemShift; wave_items: tile ids
  uint64_t nitems;            // runs (wave_items: listed tiles)
  const uint32_t *nitems_dev; // optional device-side bound on nitems (rescan list length)
  uint64_t inst_tiles;        // without items: tiles of each instance,
  uint64_t inst_runs;         // runs of each,
  uint32_t run;               // and tiles per run (the last one of an instance may have fewer)
  uint32_t wave_items;        // 1: items lists tiles, one for each wave in turn (one instance, or one-wave blocks);
  uint64_t item_lo, item_hi;  // those outside [item_lo, item_hi) are passed over
  uint32_t *tile_counts;      // hits per global tile
  uint64_t *out;              // count mode: slabs [tile][slab_cap]; direct mode: compact array
  const uint64_t *tile_offsets; // direct mode: first output slot of each tile
  uint32_t slab_cap;
  uint32_t direct;            // 1: rescan writing every hit at tile_offsets[tile]
  uint32_t *ovf_count, *done; // count mode without queue: set to zero (the tile scan's counters)
  uint32_t *queue;            // first of kCursors work-queue cursors, kCursorStride apart (nullptr: static striding)
  uint64_t *dump_out;         // kDump buckets: destination of sampled hashes
  uint64_t dump_stride;
  uint64_t dump_cap;
  unsigned long long *pid_counts; // count mode, optional: hits per global pattern id
  uint64_t tile0;             // count mode: global id of the first tile of out's slabs
  InstDesc one;               // inst == nullptr: the only instance
};

// Most keys that the single-bucket scan compares in registers: a compare a
// window each in screen mode, two operations in exact mode, against a probe of a
// bitmap and the candidates that pass a small one by chance (1 GiB of letters,
// patterns of 16 bytes, count and collect: two, three and four screen keys 238,
// 278 and 319 us, with the bitmap 405; two exact keys 379 and 787.  Where the
// keys recur, as on word text, four cost up to 515 us and the bitmap 440, three
// as much as it and two less).
constexpr uint32_t kFewScreen = 4, kFewExact = 2;

// A key of the single-bucket scan.
struct FewKey {
  uint32_t lk;       // its lookup key (shift-add), which tells the candidates apart
  uint32_t tail[4];  // its record's tail
  uint32_t pad;
  uint64_t rec;      // its record
};

// Kernel parameters of the single-bucket scan (one text, one bucket of a few
// keys, which sit in registers; count mode).
struct ListParams {
  const uint8_t *text;        // 16-byte aligned
  uint64_t n;
  uint64_t ntiles;
  const uint8_t *gimg;        // the instance image in device memory (verification tables)
  BucketDesc D;               // the bucket (offsets relative to gimg), of a list kind
  uint32_t rot;               // 8 m mod 61
  uint32_t slab_cap;
  uint32_t sub;               // sub-tiles of 64 C bytes per tile
  uint32_t nkeys;             // keys (the ones after them repeat the first)
  uint32_t tgt2[4];           // exact mode: what D.tgt is for the second key
  FewKey key[kFewScreen];
  uint32_t *tile_counts;
  uint64_t *out;              // slabs [tile][slab_cap]
  uint32_t *ovf_count, *done; // set to zero
  uint64_t *dump_out;         // kDump bucket: destination of sampled hashes (no counts then)
  uint64_t dump_stride;
  uint64_t dump_cap;
  unsigned long long *pid_counts; // optional: hits per pattern id
};

// Host-side geometry table (windows per lane c; a tile is wg * c bytes, wg / 64
// sub-tiles, in all but small texts).
struct TileCfg {
  uint32_t wg;
  uint32_t c;
};
constexpr int kNumTileCfg = 4;
constexpr TileCfg kTileCfgs[kNumTileCfg] = {{256, 68}, {256, 132}, {512, 68}, {256, 36}};

// Largest block of the general kernel: 1,024 threads leave 128 VGPRs a lane,
// which the exact family's words of a 132-window lane do not fit.
constexpr uint32_t scan_block_max(int c, int fam) { return c > 68 && fam == 2 ? 512u : 1024u; }

// Kernel families: each scan kernel is compiled for the bucket kinds one plan
// can hold, so that a single-pattern search does not pay the register budget
// of the multi-pattern and exact variants.
enum Family : int {
  kFamScreen1 = 0,  // list screen buckets only
  kFamScreen = 1,   // every screen kind
  kFamExact = 2,    // every exact kind and the hash dump
};

}  // namespace rk
