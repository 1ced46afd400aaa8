// Host runtime of librk: contexts, pattern preprocessing (plans), scratch
// layout, launch orchestration of the count and collect passes, profiling and
// the scan-geometry autotuner.  Every entry point of include/rk.h except the
// server lives here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../../include/rk.h"
#include "rk_internal.h"
#include "rk_runtime.h"

namespace rk {

// ------------------------------------------------------------ host arithmetic
// The library's own mod 2^61-1 arithmetic for d = 256 (pattern hashes are
// computed once on the host, Sec. 3.1).  256*s is a rotation of the 61-bit word.
static inline uint64_t h_mul256(uint64_t s) { return ((s << 8) & kQ) + (s >> 53); }
static inline uint64_t h_canon(uint64_t s) {
  uint64_t f = (s & kQ) + (s >> 61);
  return f >= kQ ? f - kQ : f;
}
uint64_t host_hash(const uint8_t *p, uint64_t m) {
  uint64_t s = 0;
  for (uint64_t i = 0; i < m; ++i) s = h_canon(h_mul256(s) + p[i]);
  return s;
}
// Screen shift of a group whose shortest pattern has m bytes: the smallest of
// 2, 3, 4, 8 whose hash covers at most m bytes (ceil(32/s) of them; one to
// three bytes are masked).  s = 1 is the paper's shift-and-add form.
static uint32_t screen_shift(uint32_t m) {
  if (m < 8) return 8;
  if (m < 11) return 4;
  if (m < 16) return 3;
  return 2;
}
static uint32_t screen_hash(const uint8_t *p, uint32_t m, uint32_t s, uint32_t mask) {
  uint32_t h = 0;
  for (uint32_t i = 0; i < m; ++i) h = (h << s) + p[i];
  return h & mask;
}

// ------------------------------------------------------------------ errors
rk_status set_err(rk_ctx *ctx, rk_status st, const char *fmt, ...) {
  if (ctx) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    ctx->err = buf;
  }
  return st;
}

rk_status hip_err(rk_ctx *ctx, hipError_t e, const char *what) {
  return set_err(ctx, RK_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(ctx, expr, what)                 \
  do {                                           \
    hipError_t e_ = (expr);                      \
    if (e_ != hipSuccess) return hip_err(ctx, e_, what); \
  } while (0)

static inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }
static inline uint32_t next_pow2(uint32_t v) {
  uint32_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

// ------------------------------------------------------------ image building
// An instance image holds, per group of patterns, the structures the scan
// probes for every window (a register target or a bitmap of keys) and those
// it reads for candidates only (lookup bitmap, records with pattern tails,
// entries and pattern bytes).
//
// Patterns are grouped by length class: their keys are taken from the end of
// the pattern, over as many bytes as the class's shortest one has (exact mode:
// the exact hash; screen mode: the shift-add hash, from which bytes older than
// 32/s positions have shifted out).
struct PatRef {
  uint32_t pid;
  const uint8_t *p;
  uint32_t m;
  uint64_t key;  // screen hash (screen groups) or exact hash (exact groups)
  uint32_t lk;   // shift-add key of the lookup
  uint32_t at;   // the lookup bit
};

struct GroupIn {
  bool screen;
  uint32_t shift, mask;  // of the screen hash (screen groups: tested; all groups: looked up)
  uint32_t m;            // exact groups: the length; screen groups: the shortest length
  std::vector<PatRef> pats;
};

// Length class of a pattern: 1, 2, 3, 4 (4..7 bytes), 5 (8..15), 6 (16 and
// more).  Screen and exact mode share them: a class is a group with a hash
// stream of its own, keyed on the last l bytes of each pattern, l the class's
// shortest length in exact mode (at most kStreamM; a class of one length
// hashes whole windows), what the shift covers of them in screen mode.
static uint32_t length_class(uint32_t m) { return m < 4 ? m : m < 8 ? 4 : m < 16 ? 5 : 6; }

// Classes that join the next shorter one, which saves their own pass over the
// text (a test of every window, about eight instructions in screen mode and
// sixteen in exact mode): the shorter keys let more windows pass, which is
// dear where the text repeats itself.  On word text a copied pattern's last
// eight bytes occur every 3,000 bytes, its last four every 300, and a
// candidate costs about 130 instructions: the pass is the dearer of the two up
// to some 100 long and 15 short patterns; half of each keeps clear of texts
// that repeat more.  Long patterns that join a class of no pattern below 11
// bytes keep keys of 11 bytes and more, which recur a fourth as often, and the
// exact pass is the dearer one, so those limits are higher (200 MiB of word
// text, lengths from 12 to 64: 80 patterns 303 -> 216 us exact and 156 -> 133
// screened, 300 patterns 346 -> 266 us exact; from 8 to 64: 80 patterns
// 336 -> 303 us exact, but 300 patterns 374 -> 555 us, which stay apart).
constexpr uint32_t kJoinKey = 11;
constexpr size_t kJoinShort = 8;
static size_t join_long(bool exact, uint32_t shortest) {
  if (shortest >= kJoinKey) return exact ? 512 : 256;
  return exact ? 96 : 64;
}

// Bytes of a bitmap for nbits set bits: at least 16 bytes a bit (a random
// window passes at most one time in 128) up to 1,024 bits, 4 bytes beyond,
// where the image's LDS would otherwise cost the scan more resident waves than
// the candidates saved are worth; at most kMaxBitmap.  (With 8 bytes a bit
// 1,024 sixteen-byte patterns scan 1 GiB in 591 us, with 16 in 556; 1,024
// instances of up to 32 patterns in 2 GB: 878 and 836 us, with 32 bytes 853.)
static uint32_t bitmap_bytes(size_t nbits) {
  const uint64_t want = nbits <= 1024 ? 16 * nbits : 4 * nbits;
  return std::min(kMaxBitmap, std::max(kMinBitmap, next_pow2((uint32_t)std::min<uint64_t>(want, kMaxBitmap))));
}

// A group serialised in two parts: what is staged in LDS (bitmaps, and the
// records with their tails when they fit) and what the kernel reads from the
// plan in device memory (entries, pattern bytes, larger record tables).
// Offsets in the descriptor are relative to the start of each part.
struct GroupBody {
  std::vector<uint8_t> lds, glob;
  BucketDesc D;
  bool tab_lds = false;  // records and tails are in the LDS part
  bool ids_lds = false;  // ids are in the LDS part
  bool pat_lds = false;  // pattern bytes are in the LDS part
  uint32_t npat = 0, max_m = 0;
  FewKeys few;
};
constexpr uint32_t kIdsLds = 8 * 1024;   // most bytes of ids staged in LDS (a load for every hit of a pattern's 2nd id on)
constexpr uint32_t kTabLds = 24 * 1024 + 512;  // largest record table staged in LDS (some 1,024 records)
constexpr uint32_t kPatLds = 2 * 1024;   // most pattern bytes staged in LDS

static uint32_t put_bytes(std::vector<uint8_t> &body, const void *p, size_t bytes) {
  const uint32_t off = (uint32_t)align_up(body.size(), 16);
  body.resize(off + align_up(bytes, 16), 0);
  if (bytes) memcpy(body.data() + off, p, bytes);
  return off;
}

// Serialises one group.  Returns false if it has more entries than a lookup
// counts or more pattern bytes than an entry addresses (the caller then splits
// the group).
static bool emit_group(const GroupIn &G, bool tab_lds, GroupBody &out) {
  std::vector<PatRef> P = G.pats;
  if (P.size() > 0xFFFFu) return false;
  BucketDesc &D = out.D;
  memset(&D, 0, sizeof D);
  D.m = G.m;
  D.shift = G.shift;
  D.mask = G.mask;
  out.npat = (uint32_t)P.size();
  for (const PatRef &r : P) out.max_m = std::max(out.max_m, r.m);
  // the keys the stream tests
  std::vector<uint64_t> dist;
  for (const PatRef &r : P) dist.push_back(r.key);
  std::sort(dist.begin(), dist.end());
  dist.erase(std::unique(dist.begin(), dist.end()), dist.end());
  const bool table = dist.size() > 1;
  std::vector<uint32_t> tkeys;
  for (uint64_t H : dist) {
    if (G.screen) {
      tkeys.push_back(table ? (uint32_t)H * kMix : (uint32_t)H);
      continue;
    }
    // every lazy form the rolling state can take
    for (uint64_t s = H; s < (1ull << 62) + (1ull << 11); s += kQ) tkeys.push_back(table ? exact_mix(s) : (uint32_t)s);
  }
  // exact: the lowest of three consecutive low words of key H times 2^(24-8j),
  // by the window's place j in its four
  auto target = [](uint64_t H, uint32_t j) {
    const uint32_t rot = 24 - 8 * j;
    return (uint32_t)(((H << rot) & kQ) | H >> (61 - rot)) - 2u;
  };
  FewKeys &F = out.few;
  if (dist.size() <= (G.screen ? kFewScreen : kFewExact)) {
    F.nkeys = (uint32_t)dist.size();
    for (uint32_t j = 0; j < 4; ++j) {
      F.tgt[j] = G.screen ? (uint32_t)dist[j < F.nkeys ? j : 0] : target(dist[0], j);
      F.tgt2[j] = G.screen ? 0u : target(dist.back(), j);
    }
  }
  if (!table) {
    D.kind = G.screen ? kListScreen : kListExact;
    memcpy(D.tgt, F.tgt, sizeof D.tgt);
    for (PatRef &r : P) r.at = 0;
  } else {
    D.kind = G.screen ? kTableScreen : kTableExact;
    // (exact: the lookup bitmap and its counts beside a test bitmap of any size
    // in one image; with fewer bits the records of a bit are more)
    const uint32_t tb = bitmap_bytes(tkeys.size());
    const uint32_t lb = G.screen ? tb : std::min(kMaxBitmap / 2, bitmap_bytes((P.size() + 3) / 4));
    std::vector<uint32_t> test(tb / 4, 0), look(lb / 4, 0);
    D.test_sh = 32 - (uint32_t)__builtin_ctz(tb / 4);
    D.lk_sh = 32 - (uint32_t)__builtin_ctz(lb / 4);
    for (uint32_t v : tkeys) test[v >> D.test_sh] |= 1u << (v & 31u);
    for (PatRef &r : P) {
      const uint32_t v = r.lk * kMix;
      r.at = (v >> D.lk_sh) * 32 + (v & 31u);
      look[r.at / 32] |= 1u << (r.at & 31u);
    }
    std::vector<uint16_t> below(lb / 4);
    uint32_t set = 0;
    for (size_t i = 0; i < look.size(); ++i) {
      below[i] = (uint16_t)set;
      set += (uint32_t)__builtin_popcount(look[i]);
    }
    D.lk_off = put_bytes(out.lds, look.data(), lb);
    put_bytes(out.lds, below.data(), below.size() * 2);  // right behind (lb is a multiple of 16)
    D.test_off = G.screen ? D.lk_off : put_bytes(out.lds, test.data(), tb);
  }
  // patterns of one lookup bit side by side, identical ones adjacent
  std::stable_sort(P.begin(), P.end(), [](const PatRef &a, const PatRef &b) {
    if (a.at != b.at) return a.at < b.at;
    if (a.m != b.m) return a.m < b.m;
    const int c = memcmp(a.p, b.p, a.m);
    if (c) return c < 0;
    return a.pid < b.pid;
  });
  // Pattern bytes, each at a 4-byte aligned offset (the kernel compares
  // dwords), identical patterns under several ids once; their records, in the
  // order of the patterns.
  struct One {
    uint32_t at;
    uint64_t rec;
    const PatRef *p;
  };
  std::vector<One> ones;
  std::vector<uint8_t> pb;
  std::vector<uint32_t> ids;
  for (size_t i = 0; i < P.size();) {
    size_t j = i + 1;
    while (j < P.size() && P[j].at == P[i].at && P[j].m == P[i].m && memcmp(P[j].p, P[i].p, P[i].m) == 0) ++j;
    const uint32_t om = om_pack((uint32_t)pb.size() & (kGroupPatBytes - 1), P[i].m);
    pb.insert(pb.end(), P[i].p, P[i].p + P[i].m);
    pb.resize(align_up(pb.size(), 4), 0);
    if (pb.size() > kGroupPatBytes) return false;  // split: records address 4 MiB of pattern bytes
    if (j == i + 1) ones.push_back({P[i].at, rec_inline(P[i].pid, om), &P[i]});
    for (size_t q = i; j > i + 1 && q < j; q += kSameMaxCount) {
      const uint32_t c = (uint32_t)std::min<size_t>(kSameMaxCount, j - q);
      ones.push_back({P[i].at, rec_ids((uint32_t)ids.size(), c, om), &P[i]});
      for (size_t t = q; t < q + c; ++t) ids.push_back(P[t].pid);
    }
    i = j;
  }
  pb.resize(pb.size() + 48, 0);  // the kernel reads 48 bytes from any pattern's start
  // one record per lookup bit: its pattern's, or a run of records behind them
  std::vector<One> tab;
  std::vector<std::pair<size_t, size_t>> runs;  // of ones; the record that refers to run i comes at tab index -1
  for (size_t i = 0; i < ones.size();) {
    size_t j = i + 1;
    while (j < ones.size() && ones[j].at == ones[i].at) ++j;
    tab.push_back(ones[i]);
    if (j > i + 1) {
      tab.back().rec = 0;
      runs.emplace_back(i, j);
    }
    i = j;
  }
  const size_t nord = tab.size();
  size_t run = 0;
  for (size_t i = 0; i < nord; ++i) {
    if (tab[i].rec) continue;
    const size_t lo = runs[run].first, hi = runs[run].second;
    ++run;
    tab[i].rec = rec_run((uint32_t)tab.size(), (uint32_t)(hi - lo));
    for (size_t q = lo; q < hi; ++q) tab.push_back(ones[q]);
  }
  // the record of each of a few keys: that of its patterns' lookup bit
  for (uint32_t j = 0; F.nkeys && j < kFewScreen; ++j) {
    const uint64_t key = dist[j < F.nkeys ? j : 0];
    const auto r = std::find_if(P.begin(), P.end(), [&](const PatRef &p) { return p.key == key; });
    const auto t = std::find_if(tab.begin(), tab.begin() + nord, [&](const One &o) { return o.at == r->at; });
    const uint32_t tail = std::min(t->p->m, 16u);
    F.key[j].lk = r->lk;
    memcpy((uint8_t *)F.key[j].tail + 16 - tail, t->p->p + t->p->m - tail, tail);
    F.key[j].rec = t->rec;
  }
  D.ntab = (uint32_t)tab.size();
  std::vector<uint8_t> tb(24 * tab.size(), 0);
  for (size_t i = 0; i < tab.size(); ++i) {
    const PatRef &r = *tab[i].p;
    const uint32_t t = std::min(r.m, 16u);
    memcpy(tb.data() + 16 * i + 16 - t, r.p + r.m - t, t);
    memcpy(tb.data() + 16 * tab.size() + 8 * i, &tab[i].rec, 8);
  }
  out.ids_lds = tab_lds && 4 * ids.size() <= kIdsLds;
  out.tab_lds = out.ids_lds && tb.size() <= kTabLds;
  out.pat_lds = tab_lds && pb.size() <= kPatLds;
  if (out.tab_lds) D.shift |= 1u << 16;
  if (out.pat_lds) D.shift |= 1u << 17;
  if (out.ids_lds) D.shift |= 1u << 18;
  D.tab_off = put_bytes(out.tab_lds ? out.lds : out.glob, tb.data(), tb.size());
  D.ids_off = put_bytes(out.ids_lds ? out.lds : out.glob, ids.data(), ids.size() * 4);
  D.pat_off = put_bytes(out.pat_lds ? out.lds : out.glob, pb.data(), pb.size());
  return true;
}

// Emits G, splitting its pattern list in halves while it does not fit.
static void expand_group(const GroupIn &G, bool tab_lds, std::vector<GroupBody> &bodies) {
  GroupBody gb;
  if ((emit_group(G, tab_lds, gb) && sizeof(ImageHeader) + 64 + align_up(gb.lds.size(), 16) <= kImgLimit) ||
      G.pats.size() < 2) {
    bodies.push_back(std::move(gb));
    return;
  }
  GroupIn a = G, b = G;
  const size_t h = G.pats.size() / 2;
  a.pats.assign(G.pats.begin(), G.pats.begin() + h);
  b.pats.assign(G.pats.begin() + h, G.pats.end());
  expand_group(a, tab_lds, bodies);
  expand_group(b, tab_lds, bodies);
}

// Packs groups greedily into virtual instances whose LDS part (header,
// descriptors, bitmaps, record tables) fits kImgLimit.  Image layout:
//   [ImageHeader][BucketDesc x nb][LDS parts ...][device-memory parts ...]
static rk_status build_images(rk_ctx *ctx, const std::vector<GroupIn> &groups, uint32_t src_inst,
                              std::vector<VInst> &vinsts, std::vector<uint8_t> &blob) {
  std::vector<GroupBody> bodies;
  for (const GroupIn &G : groups) expand_group(G, true, bodies);
  // records go to device memory rather than to another image (another scan)
  uint64_t all = sizeof(ImageHeader);
  for (const GroupBody &b : bodies) all += 64 + align_up(b.lds.size(), 16);
  if (all > kImgLimit) {
    bodies.clear();
    for (const GroupIn &G : groups) expand_group(G, false, bodies);
  }
  size_t i = 0;
  while (i < bodies.size()) {
    size_t j = i;
    uint64_t lds = 0;
    while (j < bodies.size()) {
      const uint64_t hdr = sizeof(ImageHeader) + 64 * (j - i + 1);
      const uint64_t add = align_up(bodies[j].lds.size(), 16);
      if (j > i && hdr + lds + add > kImgLimit) break;
      lds += add;
      ++j;
    }
    const uint32_t hdr = (uint32_t)(sizeof(ImageHeader) + 64 * (j - i));
    if (hdr + lds > kImgLimit)
      return set_err(ctx, RK_EUNSUPPORTED, "pattern group needs %llu bytes of LDS image (limit %u)",
                     (unsigned long long)(hdr + lds), kImgLimit);
    std::vector<uint8_t> img(hdr, 0);
    std::vector<uint32_t> lds_base(j - i), glob_base(j - i);
    for (size_t b = i; b < j; ++b) {
      lds_base[b - i] = (uint32_t)img.size();
      img.insert(img.end(), bodies[b].lds.begin(), bodies[b].lds.end());
      img.resize(align_up(img.size(), 16), 0);
    }
    const uint32_t lds_bytes = (uint32_t)img.size();
    for (size_t b = i; b < j; ++b) {
      glob_base[b - i] = (uint32_t)img.size();
      img.insert(img.end(), bodies[b].glob.begin(), bodies[b].glob.end());
      img.resize(align_up(img.size(), 16), 0);
    }
    uint32_t max_m = 0, npat = 0;
    bool only_one_list = true;
    for (size_t b = i; b < j; ++b) {
      BucketDesc d = bodies[b].D;
      npat += bodies[b].npat;
      if (d.kind == kTableScreen || d.kind == kTableExact) {
        d.test_off += lds_base[b - i];
        d.lk_off += lds_base[b - i];
      }
      d.tab_off += bodies[b].tab_lds ? lds_base[b - i] : glob_base[b - i];
      d.ids_off += bodies[b].ids_lds ? lds_base[b - i] : glob_base[b - i];
      d.pat_off += bodies[b].pat_lds ? lds_base[b - i] : glob_base[b - i];
      max_m = std::max(max_m, bodies[b].max_m);
      if (d.kind != kListScreen) only_one_list = false;
      memcpy(img.data() + sizeof(ImageHeader) + 64 * (b - i), &d, 64);
    }
    ImageHeader hd;
    hd.nbuckets = (uint32_t)(j - i);
    hd.bytes = (uint32_t)align_up(img.size(), 16);
    hd.max_m = max_m;
    hd.lds_bytes = lds_bytes;
    img.resize(hd.bytes, 0);
    memcpy(img.data(), &hd, sizeof hd);
    VInst v;
    v.src = src_inst;
    v.img_off = (uint32_t)align_up(blob.size(), 256);
    v.img_bytes = hd.bytes;
    v.lds_bytes = lds_bytes;
    v.nbuckets = hd.nbuckets;
    v.max_m = max_m;
    v.npat = npat;
    v.only_one_list = only_one_list;
    if (j == i + 1) v.few = bodies[i].few;
    blob.resize(v.img_off, 0);
    blob.insert(blob.end(), img.begin(), img.end());
    vinsts.push_back(v);
    i = j;
  }
  return RK_OK;
}

static rk_status validate_patterns(rk_ctx *ctx, const uint8_t *bytes, const uint64_t *offs, uint32_t k) {
  if (k > 0 && (!offs || (!bytes && offs[k] > offs[0])))
    return set_err(ctx, RK_EINVAL, "null pattern arrays");
  if (k > RK_MAX_PID) return set_err(ctx, RK_EUNSUPPORTED, "too many patterns (%u)", k);
  for (uint32_t j = 0; j < k; ++j) {
    if (offs[j + 1] <= offs[j]) return set_err(ctx, RK_EINVAL, "pattern %u has length 0", j);
    if (offs[j + 1] - offs[j] > RK_MAX_M)
      return set_err(ctx, RK_EUNSUPPORTED, "pattern %u has length %llu > %u", j,
                     (unsigned long long)(offs[j + 1] - offs[j]), RK_MAX_M);
  }
  return RK_OK;
}

// Groups one instance's patterns (global ids from pid_base) for a mode.
static std::vector<GroupIn> group_patterns(const uint8_t *bytes, const uint64_t *offs, uint32_t k,
                                           uint32_t pid_base, int mode) {
  std::map<uint32_t, GroupIn> by;
  for (uint32_t j = 0; j < k; ++j) {
    const uint32_t m = (uint32_t)(offs[j + 1] - offs[j]);
    PatRef r;
    r.pid = pid_base + j;
    r.p = bytes + offs[j];
    r.m = m;
    r.at = r.lk = 0;
    r.key = 0;
    by[length_class(m)].pats.push_back(r);
  }
  auto join = [&](uint32_t from, uint32_t to, size_t most) {
    auto f = by.find(from), t = by.find(to);
    if (f == by.end() || t == by.end() || f->second.pats.size() > most) return;
    t->second.pats.insert(t->second.pats.end(), f->second.pats.begin(), f->second.pats.end());
    by.erase(f);
  };
  if (by.count(5)) {
    uint32_t shortest = ~0u;
    for (const PatRef &r : by[5].pats) shortest = std::min(shortest, r.m);
    join(6, 5, join_long(mode == RK_MODE_EXACT, shortest));
  }
  join(5, 4, kJoinShort);
  std::vector<GroupIn> out;
  for (auto &kv : by) {
    GroupIn &G = kv.second;
    G.screen = mode != RK_MODE_EXACT;
    G.m = G.pats[0].m;
    for (const PatRef &r : G.pats) G.m = std::min(G.m, r.m);
    G.shift = screen_shift(G.m);
    G.mask = G.m < 4 ? (1u << (8 * G.m)) - 1u : 0xFFFFFFFFu;
    if (!G.screen) G.m = std::min(G.m, kStreamM);
    for (PatRef &r : G.pats) {
      r.lk = screen_hash(r.p, r.m, G.shift, G.mask);
      // exact keys: the exact hash of the last G.m bytes
      r.key = G.screen ? (uint64_t)r.lk : host_hash(r.p + r.m - G.m, G.m);
    }
    out.push_back(std::move(G));
  }
  return out;
}

// Images of one instance's patterns: every group of the instance shares its
// images (one scan of the text).
rk_status build_instance_images(rk_ctx *ctx, const uint8_t *bytes, const uint64_t *offs, uint32_t k,
                                uint32_t pid_base, int mode, uint32_t src, std::vector<VInst> &vinsts,
                                std::vector<uint8_t> &blob) {
  rk_status st = validate_patterns(ctx, bytes, offs, k);
  if (st != RK_OK) return st;
  if (k == 0) return RK_OK;  // nothing to scan for
  return build_images(ctx, group_patterns(bytes, offs, k, pid_base, mode), src, vinsts, blob);
}

void instance_buckets(const uint8_t *bytes, const uint64_t *offs, uint32_t k, int mode, uint32_t npat[kNumMClass]) {
  for (int c = 0; c < kNumMClass; ++c) npat[c] = 0;
  if (k == 0) return;
  for (const GroupIn &G : group_patterns(bytes, offs, k, 0, mode)) npat[m_class(G.m)] += (uint32_t)G.pats.size();
}

}  // namespace rk

using namespace rk;

// ===================================================================== C ABI
extern "C" {

const char *rk_status_string(rk_status s) {
  switch (s) {
    case RK_OK: return "RK_OK";
    case RK_EINVAL: return "RK_EINVAL";
    case RK_ENOMEM: return "RK_ENOMEM";
    case RK_EUNSUPPORTED: return "RK_EUNSUPPORTED";
    case RK_EDEVICE: return "RK_EDEVICE";
    case RK_ENOSPACE: return "RK_ENOSPACE";
    case RK_EBUSY: return "RK_EBUSY";
    case RK_ECANCELED: return "RK_ECANCELED";
    case RK_ETIMEDOUT: return "RK_ETIMEDOUT";
  }
  return "RK_UNKNOWN";
}

rk_status rk_ctx_create(int device, uint64_t d, uint64_t q, rk_ctx **out) {
  if (!out) return RK_EINVAL;
  *out = nullptr;
  if (q != kQ || d != 256) return RK_EUNSUPPORTED;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return RK_EDEVICE;
  if (hipSetDevice(device) != hipSuccess) return RK_EDEVICE;
  rk_ctx *c = new (std::nothrow) rk_ctx();
  if (!c) return RK_ENOMEM;
  c->device = device;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
    delete c;
    return RK_EDEVICE;
  }
  c->num_cu = prop.multiProcessorCount;
  c->arch = prop.gcnArchName;
  if (hipHostMalloc((void **)&c->pinned, 4096, hipHostMallocCoherent) != hipSuccess) {
    delete c;
    return RK_ENOMEM;
  }
  if (hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking) != hipSuccess) {
    hipHostFree(c->pinned);
    delete c;
    return RK_EDEVICE;
  }
  if (hipEventCreateWithFlags(&c->counted, hipEventDisableTiming) != hipSuccess) {
    hipStreamDestroy(c->aux);
    hipHostFree(c->pinned);
    delete c;
    return RK_EDEVICE;
  }
  for (int md = 0; md < 3; ++md) {
    for (int m = 0; m <= RK_MAX_M; ++m) c->tune[md][m] = -1;
    for (int a = 0; a < kNumMClass; ++a)
      for (int b = 0; b < kNumKClass; ++b) {
        c->tune_b[md][a][b] = -1;
        for (int g = 0; g < kNumTileCfg; ++g) c->tune_bms[md][a][b][g] = -1.0;
      }
  }
  prepare_scan_kernels();
  if (static_scratch_setup(c) != RK_OK) {
    hipEventDestroy(c->counted);
    hipStreamDestroy(c->aux);
    hipHostFree(c->pinned);
    delete c;
    return RK_EDEVICE;
  }
  *out = c;
  return RK_OK;
}

void rk_ctx_destroy(rk_ctx *ctx) {
  if (!ctx) return;
  hipSetDevice(ctx->device);
  for (auto &ev : ctx->prof_events) {
    hipEventDestroy(ev.a);
    hipEventDestroy(ev.b);
  }
  if (ctx->counted) hipEventDestroy(ctx->counted);
  if (ctx->pinned) hipHostFree(ctx->pinned);
  if (ctx->stage) hipHostFree(ctx->stage);
  if (ctx->copy) hipStreamDestroy(ctx->copy);
  if (ctx->aux) hipStreamDestroy(ctx->aux);
  delete ctx;
}

const char *rk_ctx_last_error(const rk_ctx *ctx) { return ctx ? ctx->err.c_str() : "null context"; }

rk_status rk_ctx_set_option(rk_ctx *ctx, int option, int64_t value) {
  if (!ctx) return RK_EINVAL;
  switch (option) {
    case RK_OPT_SLAB_CAP:
      if (value < 0 || value > (1 << 20)) return set_err(ctx, RK_EINVAL, "slab cap out of range");
      ctx->slab_cap = (uint32_t)value;
      return RK_OK;
    case RK_OPT_TILE_CFG:
      if (value < -1 || value >= kNumTileCfg) return set_err(ctx, RK_EINVAL, "tile cfg out of range");
      ctx->tile_cfg = (int)value;
      return RK_OK;
    case RK_OPT_GRID:
      if (value < 0 || value > (1 << 20)) return set_err(ctx, RK_EINVAL, "grid out of range");
      ctx->grid = (uint32_t)value;
      return RK_OK;
    case RK_OPT_PROFILE:
      ctx->profile = value != 0;
      return RK_OK;
    case RK_OPT_QUEUE:
      if (value < -1 || value > 1) return set_err(ctx, RK_EINVAL, "queue option is -1, 0 or 1");
      ctx->queue = (int)value;
      return RK_OK;
  }
  return set_err(ctx, RK_EINVAL, "unknown option %d", option);
}

int rk_tile_cfg_count(void) { return kNumTileCfg; }

rk_status rk_tile_cfg(int i, uint32_t *wg, uint32_t *c, uint32_t *tile) {
  if (i < 0 || i >= kNumTileCfg) return RK_EINVAL;
  if (wg) *wg = kTileCfgs[i].wg;
  if (c) *c = kTileCfgs[i].c;
  if (tile) *tile = kTileCfgs[i].wg * kTileCfgs[i].c;
  return RK_OK;
}

rk_status rk_hash(const rk_ctx *ctx, const uint8_t *s, uint64_t m, uint64_t *out) {
  (void)ctx;
  if (!out || (m && !s)) return RK_EINVAL;
  *out = host_hash(s, m);
  return RK_OK;
}

rk_status rk_plan_create(rk_ctx *ctx, const uint8_t *bytes, const uint64_t *offs, uint32_t k, int mode,
                         rk_plan **out) {
  if (!ctx || !out) return RK_EINVAL;
  *out = nullptr;
  rk_instance inst;
  inst.text_dev = nullptr;
  inst.n = 0;
  inst.bytes_host = bytes;
  inst.offsets_host = offs;
  inst.k = k;
  return plan_build(ctx, &inst, 1, mode, false, out);
}

rk_status rk_batch_plan_create(rk_ctx *ctx, const rk_instance *inst, uint32_t count, int mode, rk_plan **out) {
  if (!ctx || !out || (count && !inst)) return RK_EINVAL;
  *out = nullptr;
  return plan_build(ctx, inst, count, mode, true, out);
}

void rk_plan_destroy(rk_plan *plan) {
  if (!plan) return;
  hipSetDevice(plan->device);
  if (plan->dev) hipFree(plan->dev);
  delete plan;
}

uint32_t rk_plan_patterns(const rk_plan *plan) { return plan ? plan->k_total : 0; }
uint64_t rk_plan_text_bytes(const rk_plan *plan) { return plan ? plan->text_bytes : 0; }

rk_status rk_scratch_size(rk_ctx *ctx, const rk_plan *plan, uint64_t n, uint64_t *bytes) {
  if (!ctx || !plan || !bytes) return RK_EINVAL;
  Layout L;
  rk_status st = make_layout(ctx, plan, n, L);
  if (st != RK_OK) return st;
  *bytes = L.total;
  return RK_OK;
}

rk_status rk_work_size(rk_ctx *ctx, const rk_plan *plan, uint64_t total, uint64_t *bytes) {
  if (!ctx || !plan || !bytes) return RK_EINVAL;
  *bytes = work_bytes_for(plan, total);
  return RK_OK;
}

rk_status rk_count(rk_ctx *ctx, const rk_plan *plan, const uint8_t *text, uint64_t n, void *scratch,
                   uint64_t scratch_bytes, uint64_t *counts_dev, uint64_t *total_host, rk_stream s) {
  if (!ctx || !plan || !total_host) return RK_EINVAL;
  hipStream_t st = (hipStream_t)s;
  uint64_t total = 0;
  rk_status r = count_enqueue(ctx, plan, text, n, scratch, scratch_bytes, counts_dev, ctx->pinned, st);
  if (r != RK_OK) return r;
  r = count_finish(ctx, plan, scratch, st, &total);
  if (r != RK_OK) return r;
  *total_host = total;
  return RK_OK;
}

rk_status rk_collect(rk_ctx *ctx, const rk_plan *plan, const uint8_t *text, uint64_t n, void *scratch,
                     uint64_t scratch_bytes, void *work, uint64_t work_bytes, uint64_t *offsets,
                     uint64_t *positions, uint64_t capacity, rk_stream s) {
  if (!ctx || !plan) return RK_EINVAL;
  return collect_enqueue(ctx, plan, text, n, scratch, scratch_bytes, work, work_bytes, offsets, positions,
                         capacity, (hipStream_t)s);
}

rk_status rk_window_hashes(rk_ctx *ctx, const uint8_t *text, uint64_t n, uint32_t m, const uint64_t *xs,
                           uint64_t cnt, uint64_t *out, rk_stream s) {
  if (!ctx) return RK_EINVAL;
  if (cnt == 0) return RK_OK;
  if (!text || !xs || !out) return set_err(ctx, RK_EINVAL, "null pointer");
  if (m == 0) return set_err(ctx, RK_EINVAL, "m = 0");
  HIP_TRY(ctx, hipSetDevice(ctx->device), "hipSetDevice");
  HIP_TRY(ctx, launch_window_hashes(text, n, m, xs, cnt, out, (hipStream_t)s), "window_hashes launch");
  return RK_OK;
}

rk_status rk_ctx_profile(rk_ctx *ctx, int kernel, uint64_t *launches, double *total_ms) {
  if (!ctx) return RK_EINVAL;
  HIP_TRY(ctx, hipSetDevice(ctx->device), "hipSetDevice");
  uint64_t cnt = 0;
  double ms = 0;
  for (auto &ev : ctx->prof_events) {
    if (kernel != 3 && ev.kind != kernel) continue;
    HIP_TRY(ctx, hipEventSynchronize(ev.b), "hipEventSynchronize");
    float t = 0;
    HIP_TRY(ctx, hipEventElapsedTime(&t, ev.a, ev.b), "hipEventElapsedTime");
    ms += t;
    ++cnt;
  }
  if (launches) *launches = cnt;
  if (total_ms) *total_ms = ms;
  return RK_OK;
}

rk_status rk_ctx_profile_reset(rk_ctx *ctx) {
  if (!ctx) return RK_EINVAL;
  hipSetDevice(ctx->device);
  for (auto &ev : ctx->prof_events) {
    hipEventSynchronize(ev.b);
    ctx->free_events.push_back(ev);
  }
  ctx->prof_events.clear();
  return RK_OK;
}

}  // extern "C"
