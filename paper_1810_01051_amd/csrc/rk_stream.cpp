// Searches of texts that live in host memory or in a file, of any length
// (larger than device memory): the text goes to the device in pieces through
// two device buffers, each piece a one-text search with the plan's kernels.
//
// Piece i owns the windows starting in [i L, (i + 1) L) and holds the text
// bytes [i L, (i + 1) L + m_max - 1) (cut at n), where L = piece bytes -
// (m_max - 1): the same front/back overlap rule as tiles inside a search, so
// every window lies wholly inside the piece that owns it.  A piece's per-
// pattern lists come back ascending; positions at or past L belong to the
// next piece and are dropped; the rest are shifted by i L and appended, so the
// concatenation per pattern stays ascending.
//
// Overlap: the text is staged chunk by chunk through a ring of pinned host
// memory (up to 16 threads copy, or read from the file), an uploading thread
// sends the staged chunks to the device in order on a copy stream, and the
// caller's thread searches the pieces that are there, so that staging, link and
// search run at the same time.  The link (host-to-device bandwidth) bounds the
// whole search: 400 MiB of text in 9.6 ms, which the link alone takes 7.4 ms for.
// The ring and the copy stream are the context's, as pinning memory costs more
// than the link takes for as much text (two pinned buffers of a piece of 256 MiB
// each per call: 36 ms).
#include <hip/hip_runtime.h>

#include <fcntl.h>
#include <sched.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "../../include/rk.h"
#include "rk_internal.h"
#include "rk_runtime.h"

namespace rk {

namespace {

struct DevMem {
  void *p = nullptr;
  uint64_t bytes = 0;
  ~DevMem() {
    if (p) hipFree(p);
  }
  hipError_t ensure(uint64_t b) {
    if (b <= bytes && p) return hipSuccess;
    if (p) hipFree(p);
    p = nullptr;
    bytes = 0;
    const hipError_t e = hipMalloc(&p, std::max<uint64_t>(b, 256));
    if (e == hipSuccess) bytes = std::max<uint64_t>(b, 256);
    return e;
  }
};

// The source of the text: host memory or a file descriptor.
struct Source {
  const uint8_t *mem = nullptr;
  int fd = -1;
  uint64_t n = 0;
};

// Copies text bytes [off, off + len) of src to dst.  Returns false on a read
// error or a short file.
static bool stage(const Source &src, uint64_t off, uint64_t len, uint8_t *dst) {
  if (src.mem) {
    memcpy(dst, src.mem + off, len);
    return true;
  }
  for (uint64_t done = 0; done < len;) {
    const ssize_t r = pread(src.fd, dst + done, len - done, (off_t)(off + done));
    if (r <= 0) return false;
    done += (uint64_t)r;
  }
  return true;
}

// Threads that stage chunks: the CPUs this process may run on, at most 16.
// Staging from pageable memory is a host memcpy that one thread runs at a
// fraction of the host's memory bandwidth; with 8 threads it took longer than
// the host-to-device copy of the same bytes.
static int staging_threads() {
  cpu_set_t set;
  int n = 0;
  if (sched_getaffinity(0, sizeof set, &set) == 0) n = CPU_COUNT(&set);
  if (n <= 0) n = (int)std::thread::hardware_concurrency();
  return std::max(1, std::min(16, n));
}

// The ring: half of it is staged while the other half is on its way.  A chunk
// is an upload, large enough that the link is busy between one and the next; it
// is staged in blocks by as many threads.  (400 MiB of text: 9.6 ms with chunks of
// 8 MiB, 10.3 with 4, 12.0 with 2; two copy streams in turn take 9 to 20.)
constexpr uint64_t kStageChunk = 8ull << 20, kStageBlock = 512u << 10;
constexpr uint32_t kStageSlots = 4;

struct PieceOut {
  std::vector<uint64_t> off;  // k + 1, after dropping positions >= L
  std::vector<uint64_t> pos;  // shifted to text positions
};

// The way of the text to the device.  Worker threads take the chunks' blocks in
// order, each waiting until the chunk's slot of the ring is free; run(), on a
// thread of its own, uploads the staged chunks in order, records the event of a
// piece with its last chunk and frees the slots of the finished uploads; it
// waits with a piece until the piece before the last one was searched (their
// buffer is the same).  The owner waits for a piece's uploads to be enqueued, reports each
// searched piece, and stops everything on an error of its own.
struct Pipe {
  const Source &src;
  uint64_t n, L, piece, chunk, npieces;
  uint64_t per, nchunks, blocks;  // chunks of a whole piece, of all; blocks of a chunk
  uint8_t *ring;
  hipStream_t cs;
  uint8_t *text[2] = {nullptr, nullptr};
  hipEvent_t copied[2] = {nullptr, nullptr}, slot_ev[kStageSlots] = {};
  int device;

  std::mutex mu;
  std::condition_variable cv;
  std::atomic<uint64_t> next{0};  // blocks taken by workers
  uint64_t freed = 0;             // chunks whose slots are free again
  uint64_t enqueued = 0;          // pieces whose uploads are enqueued
  uint64_t searched = 0;          // pieces searched
  uint64_t staged[kStageSlots] = {};  // blocks of the slot's chunk that are there
  bool stop = false;
  int64_t bad = -1;               // first byte of a chunk that could not be read
  hipError_t err = hipSuccess;

  uint64_t piece_len(uint64_t i) const { return std::min(n, i * L + piece) - i * L; }
  // bytes of chunk c, and where they are in its piece
  uint64_t chunk_len(uint64_t c, uint64_t *at) const {
    *at = c % per * chunk;
    const uint64_t len = piece_len(c / per);
    return *at < len ? std::min(chunk, len - *at) : 0;
  }

  // stages block q of chunk c
  void fill(uint64_t c, uint64_t q) {
    uint64_t at;
    const uint64_t len = chunk_len(c, &at), from = std::min(len, q * kStageBlock), off = c / per * L + at + from;
    const bool ok = stage(src, off, std::min(len - from, kStageBlock), ring + c % kStageSlots * chunk + from);
    std::lock_guard<std::mutex> g(mu);
    const bool whole = ++staged[c % kStageSlots] == blocks;
    if (!ok) {
      if (bad < 0 || off < (uint64_t)bad) bad = (int64_t)off;
      stop = true;
    }
    if (whole || !ok) cv.notify_all();
  }

  void work() {
    for (;;) {
      const uint64_t q = next.fetch_add(1), c = q / blocks;
      if (c >= nchunks) return;
      {
        std::unique_lock<std::mutex> lk(mu);
        cv.wait(lk, [&] { return stop || c < freed + kStageSlots; });
        if (stop) return;
      }
      fill(c, q % blocks);
    }
  }

  void run() {
    hipError_t e = hipSetDevice(device);
    for (uint64_t c = 0; c < nchunks && e == hipSuccess; ++c) {
      const uint64_t i = c / per, b = i & 1, s = c % kStageSlots;
      {
        std::unique_lock<std::mutex> lk(mu);
        cv.wait(lk, [&] { return stop || (staged[s] == blocks && i < searched + 2); });
        if (stop) break;
        staged[s] = 0;
      }
      uint64_t at;
      const uint64_t len = chunk_len(c, &at);
      if (len) e = hipMemcpyAsync(text[b] + at, ring + s * chunk, len, hipMemcpyHostToDevice, cs);
      if (e == hipSuccess) e = hipEventRecord(slot_ev[s], cs);
      const bool whole = e == hipSuccess && (c + 1 == nchunks || (c + 1) % per == 0);
      if (whole) e = hipEventRecord(copied[b], cs);
      // half of the slots may wait for the link, half are the workers'
      const bool reap = e == hipSuccess && c + 1 >= kStageSlots / 2;
      if (reap) e = hipEventSynchronize(slot_ev[(c + 1 - kStageSlots / 2) % kStageSlots]);
      if (e != hipSuccess) break;
      std::lock_guard<std::mutex> g(mu);
      if (reap) freed = c + 2 - kStageSlots / 2;
      if (whole) enqueued = i + 1;
      if (reap || whole) cv.notify_all();
    }
    if (e == hipSuccess) return;
    std::lock_guard<std::mutex> g(mu);
    err = e;
    stop = true;
    cv.notify_all();
  }

  // Waits until piece i's uploads are enqueued; false when that will not be.
  bool wait_piece(uint64_t i) {
    std::unique_lock<std::mutex> lk(mu);
    cv.wait(lk, [&] { return stop || enqueued > i; });
    return enqueued > i;
  }
  void piece_searched() {
    std::lock_guard<std::mutex> g(mu);
    ++searched;
    cv.notify_all();
  }
  void cancel() {
    std::lock_guard<std::mutex> g(mu);
    stop = true;
    cv.notify_all();
  }
};

static rk_status run_pieces(rk_ctx *ctx, const rk_plan *plan, const Source &src, uint64_t piece_bytes,
                            rk_host_result **out) {
  const uint64_t n = src.n;
  const uint32_t k = plan->k_total;
  const uint64_t ov = plan->max_m ? plan->max_m - 1 : 0;
  if (piece_bytes < (1u << 16) || piece_bytes <= 2 * ov)
    return set_err(ctx, RK_EINVAL, "piece bytes %llu too small (at least 64 KiB and 2 (m_max - 1))",
                   (unsigned long long)piece_bytes);
  piece_bytes = (piece_bytes + 15) & ~15ull;
  const uint64_t L = piece_bytes - ov;
  const uint64_t npieces = n == 0 ? 0 : (n + L - 1) / L;
  if (hipSetDevice(ctx->device) != hipSuccess) return set_err(ctx, RK_EDEVICE, "hipSetDevice failed");
  DevMem text[2], scratch, work, offs, pos;
  rk_status st = RK_OK;
  std::vector<PieceOut> pieces;
  Pipe pipe{src, n, L, piece_bytes, std::min<uint64_t>(kStageChunk, piece_bytes), npieces};
  pipe.device = ctx->device;
  pipe.per = (piece_bytes + pipe.chunk - 1) / pipe.chunk;
  pipe.blocks = (pipe.chunk + kStageBlock - 1) / kStageBlock;
  pipe.nchunks = npieces ? (npieces - 1) * pipe.per + (pipe.piece_len(npieces - 1) + pipe.chunk - 1) / pipe.chunk : 0;
  auto fail = [&](hipError_t e, const char *what) { return hip_err(ctx, e, what); };
  hipError_t e = hipSuccess;
  if (!ctx->stage) {
    e = hipHostMalloc((void **)&ctx->stage, kStageSlots * kStageChunk, hipHostMallocDefault);
    if (e != hipSuccess) ctx->stage = nullptr;
  }
  if (e == hipSuccess && !ctx->copy) e = hipStreamCreateWithFlags(&ctx->copy, hipStreamNonBlocking);
  const hipStream_t ss = ctx->aux;
  pipe.ring = ctx->stage;
  pipe.cs = ctx->copy;
  // device buffers as large as the pieces are
  const uint64_t most = std::min<uint64_t>(piece_bytes, (n + 15) & ~15ull);
  for (int b = 0; b < 2 && e == hipSuccess; ++b) {
    e = hipEventCreateWithFlags(&pipe.copied[b], hipEventDisableTiming);
    if (e == hipSuccess && (uint64_t)b < npieces) e = text[b].ensure(most);
    pipe.text[b] = (uint8_t *)text[b].p;
  }
  for (uint32_t s = 0; s < kStageSlots && s < pipe.nchunks && e == hipSuccess; ++s)
    e = hipEventCreateWithFlags(&pipe.slot_ev[s], hipEventDisableTiming);
  uint64_t sb = 0;
  if (e == hipSuccess) {
    st = rk_scratch_size(ctx, plan, piece_bytes, &sb);
    if (st == RK_OK) st = rk_scratch_size(ctx, plan, most, &sb);
    if (st == RK_OK) e = scratch.ensure(sb);
  }
  if (e == hipSuccess) e = offs.ensure((uint64_t)(k + 1) * 8);
  if (e != hipSuccess) st = fail(e, "streamed search setup");
  std::vector<uint64_t> hoff(k + 1);
  std::vector<std::thread> threads;
  if (st == RK_OK && pipe.nchunks) {
    try {
      if (pipe.nchunks == 1) {  // nothing to overlap
        for (uint64_t q = 0; q < pipe.blocks; ++q) pipe.fill(0, q);
        pipe.run();
      } else {
        threads.emplace_back([&] { pipe.run(); });
        const uint64_t want = std::min<uint64_t>(staging_threads(), pipe.nchunks * pipe.blocks);
        for (uint64_t t = 0; t < want; ++t) threads.emplace_back([&] { pipe.work(); });
      }
    } catch (...) {
      if (threads.size() < 2) {  // without a worker nothing would come
        pipe.cancel();
        st = set_err(ctx, RK_ENOMEM, "staging threads");
      }
    }
  }
  try {
    for (uint64_t i = 0; i < npieces && st == RK_OK; ++i) {
      const int b = (int)(i & 1);
      const uint64_t a = i * L, len = pipe.piece_len(i);
      if (!pipe.wait_piece(i)) break;  // the reason follows below
      e = hipStreamWaitEvent(ss, pipe.copied[b], 0);
      if (e != hipSuccess) {
        st = fail(e, "piece upload");
        break;
      }
      uint64_t total = 0;
      st = rk_count(ctx, plan, (const uint8_t *)text[b].p, len, scratch.p, sb, nullptr, &total, ss);
      uint64_t wb = 0;
      if (st == RK_OK) {
        rk_work_size(ctx, plan, total, &wb);
        e = work.ensure(wb);
        if (e == hipSuccess) e = pos.ensure(std::max<uint64_t>(total, 1) * 8);
        if (e != hipSuccess)
          st = set_err(ctx, RK_ENOMEM, "device memory for %llu hits of a piece", (unsigned long long)total);
      }
      if (st == RK_OK)
        st = rk_collect(ctx, plan, (const uint8_t *)text[b].p, len, scratch.p, sb, work.p, wb, (uint64_t *)offs.p,
                        (uint64_t *)pos.p, total, ss);
      std::vector<uint64_t> raw(total);
      if (st == RK_OK) {
        e = hipMemcpyAsync(hoff.data(), offs.p, (k + 1) * 8, hipMemcpyDeviceToHost, ss);
        if (e == hipSuccess && total) e = hipMemcpyAsync(raw.data(), pos.p, total * 8, hipMemcpyDeviceToHost, ss);
        if (e == hipSuccess) e = hipStreamSynchronize(ss);
        if (e != hipSuccess) st = fail(e, "piece results");
      }
      if (st != RK_OK) break;
      pipe.piece_searched();
      // keep the windows this piece owns (start < L unless it is the last piece)
      const bool last = i + 1 == npieces;
      PieceOut po;
      po.off.assign(k + 1, 0);
      po.pos.reserve(total);
      for (uint32_t j = 0; j < k; ++j) {
        const uint64_t *s0 = raw.data() + hoff[j], *s1 = raw.data() + hoff[j + 1];
        const uint64_t *cut = last ? s1 : std::lower_bound(s0, s1, L);
        for (const uint64_t *q = s0; q < cut; ++q) po.pos.push_back(*q + a);
        po.off[j + 1] = po.pos.size();
      }
      pieces.push_back(std::move(po));
    }
  } catch (const std::bad_alloc &) {
    st = set_err(ctx, RK_ENOMEM, "host memory for the hits of a piece");
  }
  pipe.cancel();  // (after the last piece nothing is left to stop)
  for (auto &t : threads) t.join();
  if (st == RK_OK && pipe.bad >= 0)
    st = set_err(ctx, RK_EINVAL, "reading text bytes from %llu failed", (unsigned long long)pipe.bad);
  if (st == RK_OK && pipe.err != hipSuccess) st = fail(pipe.err, "piece upload");
  // nothing of this call is left on the streams when its buffers go
  hipStreamSynchronize(ss);
  if (ctx->copy) hipStreamSynchronize(ctx->copy);
  for (hipEvent_t ev : pipe.copied)
    if (ev) hipEventDestroy(ev);
  for (hipEvent_t ev : pipe.slot_ev)
    if (ev) hipEventDestroy(ev);
  if (st != RK_OK) return st;
  // per pattern: the pieces' lists in piece order
  uint64_t total = 0;
  for (const PieceOut &po : pieces) total += po.pos.size();
  rk_host_result *r = new (std::nothrow) rk_host_result();
  if (!r) return set_err(ctx, RK_ENOMEM, "result");
  r->k = k;
  r->total = total;
  r->offsets = new (std::nothrow) uint64_t[k + 1];
  r->positions = new (std::nothrow) uint64_t[std::max<uint64_t>(total, 1)];
  if (!r->offsets || !r->positions) {
    rk_host_result_free(r);
    return set_err(ctx, RK_ENOMEM, "result of %llu positions", (unsigned long long)total);
  }
  uint64_t o = 0;
  for (uint32_t j = 0; j < k; ++j) {
    r->offsets[j] = o;
    for (const PieceOut &po : pieces) {
      const uint64_t c = po.off[j + 1] - po.off[j];
      if (c) memcpy(r->positions + o, po.pos.data() + po.off[j], c * 8);
      o += c;
    }
  }
  r->offsets[k] = o;
  *out = r;
  return RK_OK;
}

}  // namespace

}  // namespace rk

using namespace rk;

extern "C" rk_status rk_search_host(rk_ctx *ctx, const rk_plan *plan, const uint8_t *text_host, uint64_t n,
                                    uint64_t piece_bytes, rk_host_result **out) {
  if (!ctx || !plan || !out) return RK_EINVAL;
  *out = nullptr;
  if (plan->batch) return set_err(ctx, RK_EINVAL, "streamed searches take single-text plans");
  if (n && !text_host) return set_err(ctx, RK_EINVAL, "null text");
  Source src;
  src.mem = text_host;
  src.n = n;
  return run_pieces(ctx, plan, src, piece_bytes, out);
}

extern "C" rk_status rk_search_file(rk_ctx *ctx, const rk_plan *plan, const char *path, uint64_t piece_bytes,
                                    rk_host_result **out) {
  if (!ctx || !plan || !out || !path) return RK_EINVAL;
  *out = nullptr;
  if (plan->batch) return set_err(ctx, RK_EINVAL, "streamed searches take single-text plans");
  const int fd = open(path, O_RDONLY);
  if (fd < 0) return set_err(ctx, RK_EINVAL, "cannot open %s", path);
  const off_t end = lseek(fd, 0, SEEK_END);
  if (end < 0) {
    close(fd);
    return set_err(ctx, RK_EINVAL, "cannot size %s", path);
  }
  Source src;
  src.fd = fd;
  src.n = (uint64_t)end;
  const rk_status st = run_pieces(ctx, plan, src, piece_bytes, out);
  close(fd);
  return st;
}

extern "C" void rk_host_result_free(rk_host_result *r) {
  if (!r) return;
  delete[] r->offsets;
  delete[] r->positions;
  delete r;
}
