// Host side of the stage path: argument checks, the per-launch tile depth of
// automatic plans, the device tables of a plan, and the dr_stage_chunk /
// dr_stage_all entry points (kernels in stage.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>

#include "dr_internal.h"
#include "kernels.h"

namespace dr {
namespace {

bool aligned16(const void* p) { return p && (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_shards(const dr_plan* p, const float* const* shards, const char* what) {
  if (!shards) return fail(DR_EINVAL, "%s: null shard array", what);
  for (int w = 0; w < p->layout.train_shards; ++w)
    if (!aligned16(shards[w])) return fail(DR_EINVAL, "%s: shard %d pointer is null or not 16-byte aligned", what, w);
  return DR_OK;
}

int check_device(const dr_plan* p, const char* what) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(DR_EHIP, "%s: hipGetDevice: %s", what, hipGetErrorString(e));
  if (dev != p->device) return fail(DR_EINVAL, "%s: plan lives on device %d, current device is %d", what, p->device, dev);
  return DR_OK;
}

// Tile order of a launch.  A short launch is mostly its start, when nothing of source, destination
// and tables has been touched for a while: in grouped order the chip works on one window of 512
// tiles, in contiguous order on eight places of the stream at once.  Once the launch runs, contiguous
// order is the faster one.  The line depends on the depth, not on what ran before the launch or
// which call makes it.  Grouped against contiguous, back to back / after 30 ms idle, GiB read and
// written, decoders of twelve widths and shard counts:
//   depth 2: 0.3-0.9 +0.4..-5 %; 1.1-1.8 +1..-4 / +3..-4; 2.2-2.7 +0.3..-3 / +1..-2; 3.3-4.7 +3..-3 / +3..-3;
//   5-6.7 +4..-3 / +4..-3; 7-16 +0.4..+2; 45 +1.8 / +1.3: by width from 1 GiB on, mostly a loss from 3;
//   depth 4: 0.3-0.9 0..-6 % / 0..-6; 1-2.7 +0.8..-4 / +2..-5; 3.3-4.7 +2..-3 / +2..-2; 5-6.7 +2..-2 / +2..-2
//   (a loss at one width only, from 1.6 GiB on); 7-8 0; 11-16 +0.4..+1.1; 45 +1.5 / +1.3;
//   depth 4, one chunk a launch: 0.2 -8 %, 0.8 -1.4, 3 -2, 6 -1.2, 12 +0.4, 24 +1.1, 45 +1.5 / +1.2.
constexpr uint64_t kGroupedBytes = 1ull << 30;
constexpr uint64_t kGroupedDeepBytes = 6ull << 30;

bool grouped_order(int depth, uint64_t bytes) {
  return bytes <= (depth == kVecItersLarge ? kGroupedDeepBytes : kGroupedBytes);
}

// Per-device state of the automatic tile depth (see pack_drain_ns in the
// internal header): when the packs launched so far should have drained.
std::atomic<int64_t> g_packs_drain_ns[kClockDevices];

int64_t host_ns() {
  return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch())
      .count();
}

// Index of the tiling of a one-chunk launch (dr_stage_chunk, the host relay): the deep one when the
// plan has it.  Measured on the 8B workload, 60 one-chunk launches of 256 MiB take 7.86 ms back to
// back and 8.14 ms after idle time at depth 4, against 7.88 / 8.56 ms at depth 2.
int chunk_tiling(const dr_plan* p) { return p->tiling[1].depth ? 1 : 0; }

// Index of the tiling that a whole-stream launch (dr_stage_all) starting now uses.
int pick_tiling(const dr_plan* p) {
  if (!p->tiling[1].depth || p->device < 0 || p->device >= kClockDevices) return 0;
  return pack_is_hot(host_ns(), g_packs_drain_ns[p->device].load(std::memory_order_relaxed)) ? 0 : 1;
}

// Advances the device's drain estimate past a pack of `bytes` algorithmic bytes whose launch has
// just returned (a slow launch, e.g. the first on a new stream, delays the pack's start, so the
// estimate starts no earlier than the return).  The estimate only picks between two bit-identical
// kernels, so a race between threads costs nothing else.
void note_pack(const dr_plan* p, uint64_t bytes) {
  if (p->device < 0 || p->device >= kClockDevices) return;
  std::atomic<int64_t>& drain = g_packs_drain_ns[p->device];
  drain.store(pack_drain_ns(host_ns(), drain.load(std::memory_order_relaxed), bytes), std::memory_order_relaxed);
}

// Whether a launch of ntiles tiles sums its chunks itself: the rule at kOwnSumTiles; the ticket has
// its word only where slots lie a line apart.
bool own_sums(const Tiling& tl, uint32_t ntiles, hipStream_t st) {
  static_assert(kOwnSumChunkTiles <= 64 * kTilesPerSumLine, "at most 64 slots: one wave collects them");
  if (ntiles > kOwnSumTiles || tl.max_chunk_tiles > kOwnSumChunkTiles || tl.sum_stride != kSlotLineWords) return false;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capture) != hipSuccess) (void)hipGetLastError();
  return capture == hipStreamCaptureStatusNone;
}

// Tiles [tile0, tile0 + ntiles) of tiling tl, which cover chunks [chunk0, chunk0 + nchunks) and move
// `bytes` in all, then their checksums from the accumulators of cs.
int launch(dr_plan* p, const Tiling& tl, uint32_t tile0, uint32_t ntiles, const float* const* shards, void* dst,
           uint64_t dst_bias, uint32_t chunk0, uint32_t nchunks, uint64_t bytes, const ChunkSum& cs, hipStream_t st,
           const char* what) {
  StageLaunch l = stage_launch(p, tl, shards, cs);
  l.dst = dst;
  l.dst_bias = dst_bias;
  l.tile0 = tile0;
  l.ntiles = ntiles;
  l.grouped = grouped_order(tl.depth, bytes);
  if (own_sums(tl, ntiles, st)) l.sum.chunk_tiles = tl.d_chunk_tile_begin;
  hipError_t e = launch_stage_kernel(l, st);
  if (e != hipSuccess) return fail(DR_EHIP, "%s: stage kernel launch: %s", what, hipGetErrorString(e));
  p->last_depth.store(tl.depth, std::memory_order_relaxed);
  if (l.sum.chunk_tiles) return DR_OK;
  e = launch_chunk_sums(l.sum, chunk0, nchunks, st);
  if (e != hipSuccess) return fail(DR_EHIP, "%s: chunk sum launch: %s", what, hipGetErrorString(e));
  return DR_OK;
}

// Chunk `chunk` with tiling tl into dst_chunk, its checksum into *ck.
int launch_one_chunk(dr_plan* p, const Tiling& tl, uint64_t chunk, const float* const* shards, void* dst_chunk,
                     dr_checksum* ck, hipStream_t st, const char* what) {
  int rc = clear_sums(p, tl, (uint32_t)chunk, 1, st, what);
  if (rc) return rc;
  rc = launch_chunk_into(p, tl, chunk, shards, dst_chunk, chunk_sum(p, tl, ck, (uint32_t)chunk), st, what);
  if (rc) mark_sums(p, tl);
  return rc;
}

std::atomic<bool>& sums_dirty(dr_plan* p, const Tiling& tl) {
  return p->sums_dirty[&tl == &p->tiling[0] ? 0 : &tl == &p->tiling[1] ? 1 : 2];
}

uint64_t chunk_out_bytes(const dr_plan* p, uint64_t chunk) {
  return chunk + 1 < p->info.num_chunks ? p->layout.chunk_bytes : p->info.last_chunk_bytes;
}

int alloc(void** dptr, size_t bytes, const char* what) {
  bytes = std::max<size_t>(bytes, 16);
  hipError_t e = hipMalloc(dptr, bytes);
  if (e != hipSuccess) {
    *dptr = nullptr;
    return fail(e == hipErrorOutOfMemory ? DR_ENOMEM : DR_EHIP, "hipMalloc(%s, %zu B): %s", what, bytes,
                hipGetErrorString(e));
  }
  return DR_OK;
}

template <typename T>
int upload(T** dptr, const std::vector<T>& host, const char* what) {
  if (int rc = alloc(reinterpret_cast<void**>(dptr), host.size() * sizeof(T), what)) return rc;
  if (!host.empty()) {
    const hipError_t e = hipMemcpy(*dptr, host.data(), host.size() * sizeof(T), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail(DR_EHIP, "hipMemcpy(%s): %s", what, hipGetErrorString(e));
  }
  return DR_OK;
}

}  // namespace

ChunkSum chunk_sum(const dr_plan* p, const Tiling& tl, dr_checksum* out, uint32_t out_chunk0) {
  ChunkSum cs{};
  cs.acc = p->d_acc + tl.acc0;
  cs.out = out;
  cs.sub = tl.sum_slots;
  cs.stride_words = tl.sum_stride;
  cs.out_chunk0 = out_chunk0;
  cs.chunk_bias = 0;
  return cs;
}

void mark_sums(dr_plan* p, const Tiling& tl) { sums_dirty(p, tl) = true; }

int clear_sums(dr_plan* p, const Tiling& tl, uint32_t chunk0, uint32_t nchunks, hipStream_t st, const char* what) {
  if (!sums_dirty(p, tl).load(std::memory_order_relaxed)) return DR_OK;
  const uint64_t words = (uint64_t)tl.sum_slots * tl.sum_stride;
  const hipError_t e = launch_zero_words(p->d_acc + tl.acc0 + chunk0 * words, nchunks * words, st);
  if (e != hipSuccess) return fail(DR_EHIP, "%s: clear launch: %s", what, hipGetErrorString(e));
  // a clear recorded into a graph has not run yet
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (nchunks + 1 == tl.chunk_tile_begin.size() && hipStreamIsCapturing(st, &capture) == hipSuccess &&
      capture == hipStreamCaptureStatusNone)
    sums_dirty(p, tl) = false;
  return DR_OK;
}

StageLaunch stage_launch(const dr_plan* p, const Tiling& tl, const float* const* shards, const ChunkSum& cs) {
  StageLaunch l{};
  l.segs = p->d_segs;
  l.tiles = tl.d_tiles;
  l.sum = cs;
  l.chunk_elems = p->layout.chunk_bytes / 2;
  l.depth = tl.depth;
  l.num_shards = p->layout.train_shards;
  l.shards = shards;
  return l;
}

int check_stage_args(const dr_plan* p, const float* const* shards, const void* dst, const void* cks,
                     const char* what) {
  if (int rc = check_shards(p, shards, what)) return rc;
  if (!aligned16(dst)) return fail(DR_EINVAL, "%s: destination is null or not 16-byte aligned", what);
  if (!aligned16(cks)) return fail(DR_EINVAL, "%s: checksum slots are null or not 16-byte aligned", what);
  if (!p->d_segs) return fail(DR_EINVAL, "%s: host-only plan has no device tables", what);
  return check_device(p, what);
}

int launch_chunk_into(dr_plan* p, const Tiling& tl, uint64_t chunk, const float* const* shards, void* dst_chunk,
                      const ChunkSum& cs, hipStream_t st, const char* what) {
  const uint32_t t0 = tl.chunk_tile_begin[chunk], t1 = tl.chunk_tile_begin[chunk + 1];
  return launch(p, tl, t0, t1 - t0, shards, dst_chunk, chunk * (p->layout.chunk_bytes / 2), (uint32_t)chunk, 1,
                3 * chunk_out_bytes(p, chunk), cs, st, what);
}

const Tiling& chunk_launch_tiling(const dr_plan* p) { return p->tiling[chunk_tiling(p)]; }

int launch_chunk(dr_plan* p, uint64_t chunk, const float* const* shards, void* dst_chunk, dr_checksum* ck,
                 void* st) {
  return launch_one_chunk(p, p->tiling[chunk_tiling(p)], chunk, shards, dst_chunk, ck,
                          static_cast<hipStream_t>(st), "chunk launch");
}

int upload_plan(dr_plan* p) {
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) return fail(DR_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  int rc;
  if ((rc = upload(&p->d_segs, p->segs, "segments"))) return rc;
  // per tiling: tiles, chunk index and the checksum accumulators, which start at zero (and every
  // launch leaves them at zero: ChunkSum)
  if (!p->moment_segs.empty() && (rc = upload(&p->d_moment_segs, p->moment_segs, "moment segments"))) return rc;
  uint64_t words = 0;
  for_each_tiling(p, [&](Tiling& tl) {
    if (rc) return;
    if ((rc = upload(&tl.d_tiles, tl.tiles, "tiles"))) return;
    if ((rc = upload(&tl.d_chunk_tile_begin, tl.chunk_tile_begin, "chunk tiles"))) return;
    tl.acc0 = words;
    words += (uint64_t)(tl.chunk_tile_begin.size() - 1) * tl.sum_slots * tl.sum_stride;
  });
  if (rc) return rc;
  if ((rc = alloc(reinterpret_cast<void**>(&p->d_acc), words * 8, "checksum accumulators"))) return rc;
  e = hipMemset(p->d_acc, 0, words * 8);
  if (e != hipSuccess) return fail(DR_EHIP, "hipMemset(checksum accumulators): %s", hipGetErrorString(e));
  e = hipDeviceSynchronize();
  if (e != hipSuccess) return fail(DR_EHIP, "hipDeviceSynchronize: %s", hipGetErrorString(e));
  // the static scratch of dr_stage_chunk_noalloc on this device, looked up here rather than in a call
  uint64_t* scratch = nullptr;
  if ((rc = scratch_on(p->device, &scratch))) return rc;
  p->info.device = p->device;
  return DR_OK;
}

void free_device(dr_plan* p) {
  if (p->d_segs) (void)hipFree(p->d_segs);
  if (p->d_acc) (void)hipFree(p->d_acc);
  if (p->d_moment_segs) (void)hipFree(p->d_moment_segs);
  p->d_segs = nullptr;
  p->d_acc = nullptr;
  p->d_moment_segs = nullptr;
  for_each_tiling(p, [](Tiling& tl) {
    if (tl.d_tiles) (void)hipFree(tl.d_tiles);
    if (tl.d_chunk_tile_begin) (void)hipFree(tl.d_chunk_tile_begin);
    tl.d_tiles = nullptr;
    tl.d_chunk_tile_begin = nullptr;
  });
}

}  // namespace dr

using namespace dr;

extern "C" int dr_stage_chunk(dr_plan* p, uint64_t chunk, const float* const* shards, void* dst_chunk,
                              dr_checksum* d_ck, void* stream) {
  clear_error();
  if (!p) return fail(DR_EINVAL, "dr_stage_chunk: null plan");
  if (p->kind != kRollout) return fail(DR_EINVAL, "dr_stage_chunk: not a rollout plan");
  if (chunk >= p->info.num_chunks)
    return fail(DR_ERANGE, "dr_stage_chunk: chunk %llu >= num_chunks %llu", (unsigned long long)chunk,
                (unsigned long long)p->info.num_chunks);
  if (int rc = check_shards(p, shards, "dr_stage_chunk")) return rc;
  if (!aligned16(dst_chunk)) return fail(DR_EINVAL, "dr_stage_chunk: dst_chunk is null or not 16-byte aligned");
  if (!aligned16(d_ck)) return fail(DR_EINVAL, "dr_stage_chunk: d_ck is null or not 16-byte aligned");
  if (!p->d_segs) return fail(DR_EINVAL, "dr_stage_chunk: host-only plan has no device tables");
  if (int rc = check_device(p, "dr_stage_chunk")) return rc;
  const Tiling& tl = p->tiling[chunk_tiling(p)];
  const int rc =
      launch_one_chunk(p, tl, chunk, shards, dst_chunk, d_ck, static_cast<hipStream_t>(stream), "dr_stage_chunk");
  if (rc == DR_OK) note_pack(p, 3 * chunk_out_bytes(p, chunk));
  return rc;
}

extern "C" int dr_stage_all(dr_plan* p, const float* const* shards, void* dst, dr_checksum* d_cks, void* stream) {
  clear_error();
  if (!p) return fail(DR_EINVAL, "dr_stage_all: null plan");
  if (p->kind != kRollout) return fail(DR_EINVAL, "dr_stage_all: not a rollout plan");
  if (int rc = check_shards(p, shards, "dr_stage_all")) return rc;
  if (!aligned16(dst)) return fail(DR_EINVAL, "dr_stage_all: dst is null or not 16-byte aligned");
  if (!aligned16(d_cks)) return fail(DR_EINVAL, "dr_stage_all: d_cks is null or not 16-byte aligned");
  if (!p->d_segs) return fail(DR_EINVAL, "dr_stage_all: host-only plan has no device tables");
  if (int rc = check_device(p, "dr_stage_all")) return rc;
  const Tiling& tl = p->tiling[pick_tiling(p)];
  const uint64_t bytes = 4 * p->info.n_elems + p->info.rollout_bytes;
  const uint32_t n = (uint32_t)p->info.num_chunks;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (int rc = clear_sums(p, tl, 0, n, st, "dr_stage_all")) return rc;
  const int rc = launch(p, tl, 0, (uint32_t)tl.tiles.size(), shards, dst, 0, 0, n, bytes, chunk_sum(p, tl, d_cks, 0),
                        st, "dr_stage_all");
  if (rc == DR_OK) note_pack(p, bytes);
  else mark_sums(p, tl);
  return rc;
}
