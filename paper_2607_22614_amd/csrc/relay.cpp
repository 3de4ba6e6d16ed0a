// The paper's state path (Sec. 3.3): the training rank's state goes to the
// new rank through host memory, cut into bounded chunks, with store and reload
// pipelined chunk by chunk.  Chunk c is packed straight into one of two pinned
// host buffers of B bytes (the stores cross PCIe: the store half of the path),
// and the buffer is reloaded into the chunk's place at the destination.  The
// transient memory is 2*B pinned and no device staging, whatever the model
// size.  Two forms share the pipeline: the weights to the rollout layout
// (stage kernel) and the training state to W' training shards (reshard kernel).
//
// Store and reload run in the same launch: launch i packs piece i of the stream
// (a chunk, or part of a large one) and reads back piece i - 1, in alternation
// in each workgroup, so both directions of the link stay busy and the launches
// follow one another on the caller's stream with nothing to wait for across
// queues.  A destination the kernels may not be able to write (memory of
// another device, or not device memory) is reloaded by copies on a
// plan-owned stream instead, ordered with events.
//
// Everything is enqueued; the call never blocks the host.  The result is valid
// once the caller's stream reaches this point, as for dr_stage_all.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dr_internal.h"
#include "kernels.h"

namespace dr {

void free_relay_resources(dr_plan* p) {
  if (p->relay_stream) (void)hipStreamSynchronize(static_cast<hipStream_t>(p->relay_stream));
  // the latest call's kernels, and with them every earlier call's, whatever device is current now
  if (p->relay_ev[4]) (void)hipEventSynchronize(static_cast<hipEvent_t>(p->relay_ev[4]));
  for (int i = 0; i < 5; ++i) {
    if (p->relay_ev[i]) (void)hipEventDestroy(static_cast<hipEvent_t>(p->relay_ev[i]));
    p->relay_ev[i] = nullptr;
  }
  if (p->relay_stream) (void)hipStreamDestroy(static_cast<hipStream_t>(p->relay_stream));
  p->relay_stream = nullptr;
  for (int i = 0; i < 2; ++i) {
    if (p->relay_pin[i]) (void)hipHostFree(p->relay_pin[i]);
    p->relay_pin[i] = nullptr;
  }
}

namespace {

int hip_fail(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? DR_ENOMEM : DR_EHIP, "host relay buffers: %s: %s", what,
              hipGetErrorString(e));
}

// The pinned buffers and the event that orders the calls on a plan.
int create_relay(dr_plan* p) {
  const size_t b = p->layout.chunk_bytes;
  for (int i = 0; i < 2; ++i) {
    hipError_t e = hipHostMalloc(&p->relay_pin[i], b, hipHostMallocDefault);  // mapped: kernels write and read it
    if (e != hipSuccess) return p->relay_pin[i] = nullptr, hip_fail(e, "hipHostMalloc(relay)");
  }
  hipEvent_t ev;
  const hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
  if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
  p->relay_ev[4] = ev;
  return DR_OK;
}

// The copy stream and events of reloads by copies.
int create_relay_copies(dr_plan* p) {
  hipStream_t s;
  hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);  // default priority
  if (e != hipSuccess) return hip_fail(e, "hipStreamCreate");
  p->relay_stream = s;
  for (int i = 0; i < 4; ++i) {
    hipEvent_t ev;
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
    p->relay_ev[i] = ev;
    // a recorded event: the first waits of the first call find it complete
    e = hipEventRecord(ev, s);
    if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
  }
  return DR_OK;
}

int relay_hip(hipError_t e, const char* what, const char* step) {
  return fail(e == hipErrorOutOfMemory ? DR_ENOMEM : DR_EHIP, "%s: %s: %s", what, step, hipGetErrorString(e));
}

// Whether kernels on the plan's device can write p: device memory of that device.
bool kernels_write(const dr_plan* plan, const void* p) {
  hipPointerAttribute_t a{};
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return a.type == hipMemoryTypeDevice && a.device == plan->device;
}

// The piece of the stream that a launch packs: tiles [t0, t1) of chunk c, of which chunk bytes
// [begin, end) can be reloaded once the launch is done.
struct Piece {
  uint64_t c;
  uint32_t t0, t1;
  uint64_t begin, end;
};

// The chunk byte, on the 16-byte grid of the reload, up to which everything lies in tiles before t.
uint64_t packed_before(const dr_plan* p, const Tiling& tl, uint32_t t, uint64_t chunk, uint32_t elem_bytes) {
  const Tile& tile = tl.tiles[t];
  const DevSeg& s = p->segs[tile.seg];
  uint64_t e = s.dst + (s.flags & DR_SEG_VEC4 ? 4ull * tile.unit0 : tile.unit0);
  if (!(s.flags & DR_SEG_VEC4) && tile.unit0) e -= s.dst & 3;  // the groups of an unaligned tile
  return (e * elem_bytes - chunk * p->layout.chunk_bytes) & ~15ull;
}

// Store and reload by kernels.  launch(piece, prev) enqueues the launch that packs *piece (null:
// nothing) into its chunk's pinned buffer and reloads *prev (null: nothing) from its own.  A buffer
// is packed again two chunks later, at least one launch after its last piece was reloaded.
template <typename Launch>
int relay_pieces(dr_plan* p, const Tiling& tl, uint32_t elem_bytes, uint32_t tile_bytes, Launch launch) {
  const uint32_t most = std::max<uint32_t>(1, kRelayPieceBytes / tile_bytes);
  Piece prev{};
  bool have = false;
  for (uint64_t c = 0; c < p->info.num_chunks; ++c) {
    const uint64_t len = c + 1 < p->info.num_chunks ? p->layout.chunk_bytes : p->info.last_chunk_bytes;
    const uint32_t c0 = tl.chunk_tile_begin[c], c1 = tl.chunk_tile_begin[c + 1];
    // equal pieces: a short one would leave the other direction of its launches without company
    const uint32_t pieces = std::max(1u, (c1 - c0 + most / 2) / most), per = (c1 - c0 + pieces - 1) / pieces;
    uint64_t begin = 0;
    for (uint32_t t = c0; t < c1;) {
      const uint32_t t1 = t + std::min(per, c1 - t);
      const Piece piece{c, t, t1, begin, t1 == c1 ? len : packed_before(p, tl, t1, c, elem_bytes)};
      if (int rc = launch(&piece, have ? &prev : nullptr)) return rc;
      prev = piece;
      have = true;
      begin = piece.end;
      t = t1;
    }
  }
  return launch(nullptr, &prev);
}

// The same, and the checksums behind the last launch.
template <typename Launch>
int relay_kernels(dr_plan* p, hipStream_t st, const char* what, const ChunkSum& cs, const Tiling& tl,
                  uint32_t elem_bytes, uint32_t tile_bytes, Launch launch) {
  const uint32_t n = (uint32_t)p->info.num_chunks;
  int rc = clear_sums(p, tl, 0, n, st, what);
  if (rc) return rc;
  rc = relay_pieces(p, tl, elem_bytes, tile_bytes, launch);
  if (rc == DR_OK) {
    const hipError_t e = launch_chunk_sums(cs, 0, n, st);
    if (e != hipSuccess) rc = relay_hip(e, what, "chunk sum launch");
  }
  if (rc) mark_sums(p, tl);
  return rc;
}

// Takes the plan's relay buffers for one call; released when the call returns.
struct RelayHeld {
  dr_plan* p = nullptr;
  ~RelayHeld() {
    if (p) p->relay_busy = false;
  }
  int take(dr_plan* plan, const char* what) {
    bool idle = false;
    if (!plan->relay_busy.compare_exchange_strong(idle, true))
      return fail(DR_EINVAL, "%s: another call on this plan is running on another thread", what);
    p = plan;
    if (!plan->relay_pin[0]) {
      if (int rc = create_relay(plan)) {
        free_relay_resources(plan);
        return rc;
      }
    }
    return DR_OK;
  }
};

// Refuses a stream that is being captured (a graph's replays would share the pinned buffers with the
// plan's other calls in no order), before anything is allocated or enqueued.
int check_not_capturing(hipStream_t st, const char* what) {
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const hipError_t e = hipStreamIsCapturing(st, &capture);
  if (e != hipSuccess) return relay_hip(e, what, "capture status");
  if (capture != hipStreamCaptureStatusNone)
    return fail(DR_EHIP, "%s: the stream is being captured; this call cannot be recorded into a graph", what);
  return DR_OK;
}

// Orders a call's work on st after the plan's previous call, and what follows after this one.
int relay_begin(dr_plan* p, hipStream_t st, const char* what) {
  const hipError_t e = hipStreamWaitEvent(st, static_cast<hipEvent_t>(p->relay_ev[4]), 0);
  return e == hipSuccess ? DR_OK : relay_hip(e, what, "wait previous call");
}
int relay_finish(dr_plan* p, hipStream_t st, const char* what) {
  const hipError_t e = hipEventRecord(static_cast<hipEvent_t>(p->relay_ev[4]), st);
  return e == hipSuccess ? DR_OK : relay_hip(e, what, "record end of call");
}

// Store by kernels, reload by copies, shared by the rollout and reshard plans.  pack(c, buf) enqueues on st the
// kernels that write chunk c into pinned buffer buf; reload(c, buf, in) enqueues on the plan's
// copy stream the host->device copies that move it to its destination.
template <typename Pack, typename Reload>
int relay_copies(dr_plan* p, hipStream_t st, const char* what, Pack pack, Reload reload) {
  if (!p->relay_stream) {
    if (int rc = create_relay_copies(p)) {
      free_relay_resources(p);
      return rc;
    }
  }
  hipStream_t in = static_cast<hipStream_t>(p->relay_stream);  // host -> device
  hipEvent_t* ev = reinterpret_cast<hipEvent_t*>(p->relay_ev);
  hipEvent_t* packed = ev;         // chunk packed into relay_pin[b]
  hipEvent_t* copied_in = ev + 2;  // relay_pin[b] reloaded: relay_pin[b] free
  hipEvent_t start = ev[4];        // the caller's earlier work on `st` (e.g. readers of the destination)
  hipError_t e;
#define DR_RELAY(call, step) \
  if ((e = (call)) != hipSuccess) return relay_hip(e, what, step)
  DR_RELAY(hipEventRecord(start, st), "record start");
  DR_RELAY(hipStreamWaitEvent(in, start, 0), "wait start");
  for (uint64_t c = 0; c < p->info.num_chunks; ++c) {
    const int b = (int)(c & 1);
    // relay_pin[b] still holds chunk c-2 until its reload has finished
    DR_RELAY(hipStreamWaitEvent(st, copied_in[b], 0), "wait pinned buffer");
    if (int rc = pack(c, p->relay_pin[b])) return rc;
    DR_RELAY(hipEventRecord(packed[b], st), "record packed");
    DR_RELAY(hipStreamWaitEvent(in, packed[b], 0), "wait packed");
    DR_RELAY(reload(c, static_cast<const char*>(p->relay_pin[b]), in), "host-to-device reload");
    DR_RELAY(hipEventRecord(copied_in[b], in), "record copied in");
  }
  DR_RELAY(hipStreamWaitEvent(st, copied_in[0], 0), "final wait");
  DR_RELAY(hipStreamWaitEvent(st, copied_in[1], 0), "final wait");
#undef DR_RELAY
  return DR_OK;
}

// The whole call around `run` (relay_kernels or relay_copies), in order with the plan's other calls.
template <typename Run>
int relay_call(dr_plan* p, hipStream_t st, const char* what, Run run) {
  if (int rc = check_not_capturing(st, what)) return rc;
  RelayHeld held;
  if (int rc = held.take(p, what)) return rc;
  if (int rc = relay_begin(p, st, what)) return rc;
  int rc = run();
  if (rc == DR_OK) rc = relay_finish(p, st, what);
  if (rc) {
    // What was enqueued still uses the pinned buffers.  No copy is left running (a later call that
    // reloads by kernels waits for none), and the next call is ordered after the kernels.
    if (p->relay_stream) (void)hipStreamSynchronize(static_cast<hipStream_t>(p->relay_stream));
    hipEvent_t end = static_cast<hipEvent_t>(p->relay_ev[4]);
    if (end && hipEventRecord(end, st) != hipSuccess) (void)hipStreamSynchronize(st);
    (void)hipGetLastError();
  }
  return rc;
}

}  // namespace
}  // namespace dr

using namespace dr;

extern "C" int dr_stage_through_host(dr_plan* p, const float* const* shards, void* dst, dr_checksum* d_cks,
                                     void* stream) {
  clear_error();
  const char* what = "dr_stage_through_host";
  if (!p) return fail(DR_EINVAL, "%s: null plan", what);
  if (p->kind != kRollout) return fail(DR_EINVAL, "%s: not a rollout plan", what);
  if (int rc = check_stage_args(p, shards, dst, d_cks, what)) return rc;
  const uint64_t B = p->layout.chunk_bytes, n = p->info.num_chunks;
  char* d = static_cast<char*>(dst);
  hipStream_t st = static_cast<hipStream_t>(stream);
  return relay_call(p, st, what, [&] {
    if (!kernels_write(p, dst))
      return relay_copies(
          p, st, what, [&](uint64_t c, void* buf) { return launch_chunk(p, c, shards, buf, d_cks + c, st); },
          [&](uint64_t c, const char* buf, hipStream_t in) {
            const uint64_t len = c + 1 < n ? B : p->info.last_chunk_bytes;
            return hipMemcpyAsync(d + c * B, buf, len, hipMemcpyHostToDevice, in);
          });
    const Tiling& tl = chunk_launch_tiling(p);
    const ChunkSum cs = chunk_sum(p, tl, d_cks, 0);
    const int rc = relay_kernels(p, st, what, cs, tl, 2, 2048 * tl.depth, [&](const Piece* pack, const Piece* reload) {
      StageLaunch l = stage_launch(p, tl, shards, cs);
      if (pack) {
        l.dst = p->relay_pin[pack->c & 1];
        l.dst_bias = pack->c * (B / 2);
        l.tile0 = pack->t0;
        l.ntiles = pack->t1 - pack->t0;
      }
      Reload r{};
      if (reload) {
        r.from = static_cast<const char*>(p->relay_pin[reload->c & 1]) + reload->begin;
        r.to = d + reload->c * B + reload->begin;
        r.groups = (uint32_t)((reload->end - reload->begin) / 16);
      }
      const hipError_t e = launch_stage_relay(l, r, st);
      return e == hipSuccess ? DR_OK : relay_hip(e, what, "relay kernel launch");
    });
    if (rc == DR_OK) p->last_depth.store(tl.depth, std::memory_order_relaxed);
    return rc;
  });
}

extern "C" int dr_reshard_through_host(dr_plan* p, const float* const* src_shards, float* const* dst_shards,
                                       dr_checksum* d_cks, void* stream) {
  clear_error();
  const char* what = "dr_reshard_through_host";
  if (int rc = check_reshard_args(p, src_shards, dst_shards, d_cks, what)) return rc;
  const uint64_t ce = p->layout.chunk_bytes / 4, S2 = p->dst_shard_elems, total = p->info.rollout_bytes / 4;
  hipStream_t st = static_cast<hipStream_t>(stream);
  return relay_call(p, st, what, [&] {
    if (!std::all_of(dst_shards, dst_shards + p->dst_shards, [&](const float* x) { return kernels_write(p, x); }))
      return relay_copies(
          p, st, what,
          [&](uint64_t c, void* buf) { return launch_reshard_chunk(p, c, src_shards, buf, d_cks + c, st, what); },
          [&](uint64_t c, const char* buf, hipStream_t in) {
            // the chunk's destination elements [e0, e1), cut at the destination shard boundaries
            const uint64_t e0 = c * ce, e1 = std::min(total, e0 + ce);
            for (uint64_t e = e0; e < e1;) {
              const uint64_t w = e / S2, n = std::min(e1, (w + 1) * S2) - e;
              hipError_t err = hipMemcpyAsync(dst_shards[w] + (e - w * S2), buf + (e - e0) * 4, n * 4,
                                              hipMemcpyHostToDevice, in);
              if (err != hipSuccess) return err;
              e += n;
            }
            return hipSuccess;
          });
    const Tiling& tl = p->tiling[0];
    const ChunkSum cs = chunk_sum(p, tl, d_cks, 0);
    return relay_kernels(p, st, what, cs, tl, 4, 4096 * tl.depth, [&](const Piece* pack, const Piece* reload) {
      ReshardLaunch l = reshard_launch(p, src_shards, dst_shards, cs);
      if (pack) {
        l.flat = static_cast<float*>(p->relay_pin[pack->c & 1]);
        l.flat_bias = pack->c * ce;
        l.tile0 = pack->t0;
        l.ntiles = pack->t1 - pack->t0;
      }
      Reload r{};
      if (reload) {
        r.from = static_cast<const char*>(p->relay_pin[reload->c & 1]) + reload->begin;
        r.elem0 = reload->c * ce + reload->begin / 4;
        r.groups = (uint32_t)((reload->end - reload->begin) / 16);
      }
      const hipError_t e = launch_reshard_relay(l, r, st);
      return e == hipSuccess ? DR_OK : relay_hip(e, what, "relay kernel launch");
    });
  });
}
