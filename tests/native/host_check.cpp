// The library's host code (plans, launches, the paths through host memory) on the CPU, over the
// stand-in runtime of fake_hip.h and plain loops in place of the kernels: what is enqueued, in what
// order, and what is left behind when a call fails or a plan goes away.
//   host_check copies|sums|destroy|order
//   host_check pieces L H Hq Hkv D F V  W T|-W' B depth   (prints how many pieces the call packs)
// Exit status 0 when everything holds.
#include "fake_hip.h"

#include <algorithm>
#include <cstdint>
#include <string>

#include "dr_internal.h"
#include "kernels.h"

static int errors = 0;
#define CHECK(c, ...)                                   \
  do {                                                  \
    if (!(c)) {                                         \
      if (errors < 20) {                                \
        std::fprintf(stderr, "FAIL %s: ", #c);          \
        std::fprintf(stderr, __VA_ARGS__);              \
        std::fprintf(stderr, "\n");                     \
      }                                                 \
      ++errors;                                         \
    }                                                   \
  } while (0)

namespace dr {

// The kernels as loops.  They read their tables when they run, like the kernels.
namespace {

struct StageRecord {  // every stage launch, in order
  uint32_t ntiles, groups;
  bool relay, grouped;
  int depth;
};
std::vector<StageRecord> launched;
struct ReshardRecord {
  uint32_t ntiles;
  bool whole_tiles;
};
std::vector<ReshardRecord> resharded;

uint16_t bf16(float x) {  // finite inputs
  uint32_t u;
  std::memcpy(&u, &x, 4);
  return (uint16_t)((u + 0x7FFF + ((u >> 16) & 1)) >> 16);
}

void add_sums(const ChunkSum& cs, uint32_t tile, uint32_t chunk, uint64_t s1, uint64_t s2) {
  fake::touch(cs.acc);
  uint64_t* slots = cs.acc + (uint64_t)(chunk - cs.chunk_bias) * cs.sub * cs.stride_words;
  slots[(tile & (cs.sub - 1)) * cs.stride_words] += s1;
  slots[(tile & (cs.sub - 1)) * cs.stride_words + 1] += s2;
}

void finish_chunk(const ChunkSum& cs, uint32_t chunk) {
  uint64_t* slots = cs.acc + (uint64_t)(chunk - cs.chunk_bias) * cs.sub * cs.stride_words;
  dr_checksum& out = cs.out[chunk - cs.out_chunk0];
  out.s1 = out.s2 = 0;
  for (uint32_t i = 0; i < cs.sub; ++i) {
    out.s1 += slots[i * cs.stride_words];
    out.s2 += slots[i * cs.stride_words + 1];
    slots[i * cs.stride_words] = slots[i * cs.stride_words + 1] = 0;
  }
}

// The elements of an unaligned tile lie on the destination's grid of 4: `lead` elements back from
// its first unit; the segment's last tile goes to the segment's end.
void stage_tiles(const StageLaunch& l, const std::vector<const float*>& shards) {
  for (uint32_t g = l.tile0; g < l.tile0 + l.ntiles; ++g) {
    const Tile t = l.tiles[g];
    const DevSeg& s = l.segs[t.seg];
    const uint64_t pos0 = s.dst - s.chunk * l.chunk_elems;
    uint64_t e0, e1;
    if (s.flags & DR_SEG_VEC4) {
      e0 = 4ull * t.unit0;
      e1 = 4ull * std::min(s.units, t.unit0 + kThreads * (uint32_t)l.depth);
    } else {
      const uint32_t lead = pos0 & 3;
      e0 = t.unit0 ? t.unit0 - lead : 0;
      e1 = t.unit0 + kScalarUnitsPerTile >= s.units ? s.units : t.unit0 + kScalarUnitsPerTile - lead;
    }
    uint16_t* out = static_cast<uint16_t*>(l.dst) + (s.dst - l.dst_bias);
    fake::touch(out + e0);
    uint64_t s1 = 0, s2 = 0;
    for (uint64_t e = e0; e < e1; ++e) {
      const uint16_t v = bf16(shards[s.shard][s.src + e / s.cols * s.stride + e % s.cols]);
      out[e] = v;
      const uint64_t pos = pos0 + e, w = (uint64_t)v << (pos & 1) * 16;
      s1 += w;
      s2 += ((pos >> 1) + 1) * w;
    }
    add_sums(l.sum, g, s.chunk, s1, s2);
    if (l.sum.chunk_tiles) {
      uint32_t& ticket = *reinterpret_cast<uint32_t*>(
          l.sum.acc + (uint64_t)(s.chunk - l.sum.chunk_bias) * l.sum.sub * l.sum.stride_words + kTicketWord);
      if (++ticket == l.sum.chunk_tiles[s.chunk + 1] - l.sum.chunk_tiles[s.chunk]) {
        ticket = 0;
        finish_chunk(l.sum, s.chunk);
      }
    }
  }
}

void reshard_tiles(const ReshardLaunch& l, const std::vector<const float*>& src, const std::vector<float*>& dst) {
  for (uint32_t g = l.tile0; g < l.tile0 + l.ntiles; ++g) {
    const Tile t = l.tiles[g];
    const DevSeg& s = l.segs[t.seg];
    const uint64_t pos0 = s.dst - s.chunk * l.chunk_elems;
    uint64_t s1 = 0, s2 = 0;
    for (uint64_t e = 4ull * t.unit0; e < 4ull * std::min(s.units, t.unit0 + kThreads * kReshardIters); ++e) {
      uint32_t w = 0;
      if (s.op != DR_OP_ZERO_F32) std::memcpy(&w, src[s.shard] + s.src + e, 4);
      float* out = l.flat ? l.flat + (s.dst - l.flat_bias) : dst[s.dst_shard] + (s.dst - s.dst_shard * l.dst_shard_elems);
      if (e == 4ull * t.unit0) fake::touch(out + e);
      std::memcpy(out + e, &w, 4);
      s1 += w;
      s2 += (pos0 + e + 1) * w;
    }
    add_sums(l.sum, g, s.chunk, s1, s2);
  }
}

}  // namespace

int scratch_on(int, uint64_t** out) { return *out = nullptr, DR_OK; }

hipError_t launch_stage_kernel(const StageLaunch& l, hipStream_t st) {
  if (launched.size() < 10000) launched.push_back({l.ntiles, 0, false, l.grouped, l.depth});
  std::vector<const float*> shards(l.shards, l.shards + l.num_shards);
  return fake::launch(st, [=] { stage_tiles(l, shards); });
}

hipError_t launch_stage_relay(const StageLaunch& l, const Reload& r, hipStream_t st) {
  if (launched.size() < 10000) launched.push_back({l.ntiles, r.groups, true, l.grouped, l.depth});
  std::vector<const float*> shards(l.shards, l.shards + l.num_shards);
  return fake::launch(st, [=] {  // the reload first or last: the launch leaves it open
    const bool first = l.tile0 & 1;
    for (int k = 0; k < 2; ++k) {
      if ((k == 0) != first && l.ntiles) stage_tiles(l, shards);
      if ((k == 0) == first && r.groups) {
        fake::touch(r.from);
        fake::touch(r.to);
        std::memcpy(r.to, r.from, 16ull * r.groups);
      }
    }
  });
}

hipError_t launch_chunk_sums(const ChunkSum& cs, uint32_t chunk0, uint32_t n, hipStream_t st) {
  return fake::launch(st, [=] {
    fake::touch(cs.acc);
    for (uint32_t c = chunk0; c < chunk0 + n; ++c) finish_chunk(cs, c);
  });
}

hipError_t launch_zero_words(uint64_t* p, uint64_t n, hipStream_t st) {
  return fake::launch(st, [=] {
    fake::touch(p);
    std::memset(p, 0, 8 * n);
  });
}

hipError_t launch_reshard_kernel(const ReshardLaunch& l, hipStream_t st) {
  resharded.push_back({l.ntiles, l.whole_tiles});
  std::vector<const float*> src(l.src, l.src + l.num_src);
  std::vector<float*> dst;
  if (l.dst) dst.assign(l.dst, l.dst + l.num_dst);
  return fake::launch(st, [=] { reshard_tiles(l, src, dst); });
}

hipError_t launch_reshard_relay(const ReshardLaunch& l, const Reload& r, hipStream_t st) {
  if (launched.size() < 10000) launched.push_back({l.ntiles, r.groups, true, false, 0});
  std::vector<const float*> src(l.src, l.src + l.num_src);
  std::vector<float*> dst(l.dst, l.dst + l.num_dst);
  return fake::launch(st, [=] {
    const bool first = l.tile0 & 1;
    for (int k = 0; k < 2; ++k) {
      if ((k == 0) != first && l.ntiles) reshard_tiles(l, src, dst);
      if ((k == 0) == first && r.groups) fake::touch(r.from);
      if ((k == 0) == first)
        for (uint64_t i = 0; i < 4ull * r.groups; ++i) {
          const uint64_t e = r.elem0 + i;
          std::memcpy(dst[e / l.dst_shard_elems] + e % l.dst_shard_elems, static_cast<const float*>(r.from) + i, 4);
        }
    }
  });
}

}  // namespace dr

using namespace dr;

namespace {

// A plan with sources and expected output (from one dr_stage_all or dr_reshard, checked elsewhere
// against the oracle's definition of the layout), and what a call on it produces.
struct Work {
  dr_plan* p = nullptr;
  std::vector<float*> src;
  std::vector<uint8_t> want;
  std::vector<dr_checksum> want_cks;
  uint8_t *dst = nullptr, *pinned = nullptr;
  dr_checksum* cks = nullptr;
  std::vector<float*> shards_of(uint8_t* at) {
    std::vector<float*> v;
    for (int w = 0; w < p->dst_shards; ++w) v.push_back(reinterpret_cast<float*>(at) + w * p->dst_shard_elems);
    return v;
  }
  void clear() {
    std::memset(dst, 0xEE, p->info.rollout_bytes);
    std::memset(pinned, 0xEE, p->info.rollout_bytes);
    std::memset(static_cast<void*>(cks), 0xEE, p->info.num_chunks * sizeof(dr_checksum));
  }
  bool right(const uint8_t* at) const {
    return !std::memcmp(at, want.data(), want.size()) &&
           !std::memcmp(cks, want_cks.data(), want_cks.size() * sizeof(dr_checksum));
  }
  int all(hipStream_t st) {
    if (p->kind == kRollout) return dr_stage_all(p, src.data(), dst, cks, st);
    return dr_reshard(p, src.data(), shards_of(dst).data(), cks, st);
  }
  int through_host(uint8_t* to, hipStream_t st) {
    if (p->kind == kRollout) return dr_stage_through_host(p, src.data(), to, cks, st);
    return dr_reshard_through_host(p, src.data(), shards_of(to).data(), cks, st);
  }
};

Work setup(const dr_model& m, int w, int to, uint64_t chunk, int depth = 0) {
  Work k;
  const dr_layout l{w, to, chunk, 0, depth, 0};
  const int rc = to < 0 ? dr_reshard_plan_create(&m, w, -to, chunk, &k.p) : dr_plan_create(&m, &l, &k.p);
  if (rc) std::fprintf(stderr, "plan: %s\n", dr_last_error()), std::exit(2);
  uint32_t x = 12345;
  for (int i = 0; i < w; ++i) {
    void* p;
    fake::add(&p, 4 * k.p->info.shard_elems, true);
    float* f = static_cast<float*>(p);
    for (uint64_t e = 0; e < k.p->info.shard_elems; ++e) f[e] = (float)((x = x * 1664525 + 1013904223) >> 8) - 8e6f;
    k.src.push_back(f);
  }
  void* p;
  fake::add(&p, k.p->info.rollout_bytes, true), k.dst = static_cast<uint8_t*>(p);
  fake::add(&p, k.p->info.rollout_bytes, false), k.pinned = static_cast<uint8_t*>(p);
  fake::add(&p, k.p->info.num_chunks * sizeof(dr_checksum), true), k.cks = static_cast<dr_checksum*>(p);
  k.clear();
  if (k.all(nullptr)) std::exit(2);
  (void)hipDeviceSynchronize();
  k.want.assign(k.dst, k.dst + k.p->info.rollout_bytes);
  k.want_cks.assign(k.cks, k.cks + k.p->info.num_chunks);
  return k;
}

hipStream_t stream() {
  hipStream_t s;
  (void)hipStreamCreateWithFlags(&s, 0);
  return s;
}

const dr_model kSmall{2, 64, 6, 3, 24, 3 * 37, 3 * 41};  // column slices of any alignment at T = 3

// f(n) for n = 1, 2, ... until it is false; f passes n to failing_call, which has enqueue n of one call fail.
template <typename F>
long each_failure(F f) {
  long n = 1;
  while (f(n)) ++n;
  return n - 1;
}
template <typename F>
int failing_call(long n, F call) {
  fake::enqueues = 0;
  fake::fail_at = n;
  const int rc = call();
  fake::fail_at = 0;
  return rc;
}

// A call that fails on the way leaves none of its reload copies running.
void check_copies() {
  for (int to : {3, -2}) {
    const long n = each_failure([&](long i) {
      Work k = setup(kSmall, 4, to, 4096);
      const hipStream_t st = stream();
      const int rc = failing_call(i, [&] { return k.through_host(k.pinned, st); });
      const fake::Stream* in = fake::of(static_cast<hipStream_t>(k.p->relay_stream));
      CHECK(!rc || !k.p->relay_stream || in->ops.empty(), "enqueue %ld: %zu left on the copy stream", i, in->ops.size());
      (void)hipDeviceSynchronize();
      if (!rc) CHECK(k.right(k.pinned), "through host");
      dr_plan_destroy(k.p);
      fake::release_for_good();
      return rc != 0;
    });
    CHECK(n > 100, "only %ld enqueues", n);
  }
}

// After a call that failed anywhere, the plan's later calls write the right checksums, and once a
// whole-stream call has run they enqueue no more than before the failure.
void check_sums() {
  enum { kAll, kChunk, kHost };
  const auto call = [](Work& k, int op, hipStream_t st) -> int {
    if (op == kHost) return k.through_host(k.dst, st);
    if (op == kAll || k.p->kind != kRollout) return k.all(st);
    for (uint64_t c = 0; c < k.p->info.num_chunks; ++c)
      if (int rc = dr_stage_chunk(k.p, c, k.src.data(), k.dst + c * k.p->layout.chunk_bytes, k.cks + c, st)) return rc;
    return DR_OK;
  };
  for (int late = 0; late < 2; ++late)
    for (int to : {3, -2})
      for (int depth : {2, 0})
        for (int op : {kAll, kChunk, kHost}) {
          if (to < 0 && (op == kChunk || depth)) continue;
          // chunks of few tiles (packed slots), and of enough to sum themselves
          for (uint64_t chunk : {4096u, 48u << 10}) {
            long before = 0;
            each_failure([&](long i) {
              Work k = setup(kSmall, 4, to, chunk, depth);
              fake::enqueues = 0;
              CHECK(!call(k, op, nullptr), "%s", dr_last_error());
              before = fake::enqueues;
              (void)hipDeviceSynchronize();
              const hipStream_t st = stream(), st2 = stream();
              fake::fail_late = late;
              const int rc = failing_call(i, [&] { return call(k, op, st); });
              fake::fail_late = false;
              const int after[] = {op, kChunk, kHost, kAll, op};
              for (int j = 0; j < 5; ++j) {
                (void)hipDeviceSynchronize();
                k.clear();
                fake::enqueues = 0;
                CHECK(!call(k, after[j], j & 1 ? st2 : st), "%s", dr_last_error());
                const long n = fake::enqueues;
                (void)hipDeviceSynchronize();
                CHECK(k.right(k.dst), "to %d, op %d, enqueue %ld failed, then call %d", to, op, i, j);
                // (an automatic plan has two tilings, each cleared by its own whole-stream call)
                CHECK(j < 4 || n <= before || (depth == 0 && to > 0), "%ld enqueues, %ld before", n, before);
              }
              dr_plan_destroy(k.p);
              fake::release_for_good();
              return rc != 0;
            });
          }
        }
}

// The pinned buffers outlive the work of the latest call when the plan goes away, whatever device is
// current, and when the copy stream of a later call cannot be made.
void check_destroy() {
  for (int to : {3, -2})
    for (bool copies : {false, true}) {
      Work k = setup(kSmall, 4, to, 4096);
      CHECK(!k.through_host(copies ? k.pinned : k.dst, stream()), "%s", dr_last_error());
      (void)hipSetDevice(1);
      dr_plan_destroy(k.p);
      (void)hipSetDevice(0);
      (void)hipDeviceSynchronize();
      CHECK(k.right(copies ? k.pinned : k.dst), "plan destroyed with device 1 current");
      fake::release_for_good();
    }
  for (long i = 1; i <= 8; ++i) {
    Work k = setup(kSmall, 4, 3, 4096);
    CHECK(!k.through_host(k.dst, stream()), "%s", dr_last_error());
    (void)failing_call(i, [&] { return k.through_host(k.pinned, stream()); });
    (void)hipDeviceSynchronize();
    CHECK(!std::memcmp(k.dst, k.want.data(), k.want.size()), "the first call, enqueue %ld of the second failed", i);
    k.clear();
    CHECK(!k.through_host(k.dst, stream()), "%s", dr_last_error());
    (void)hipDeviceSynchronize();
    CHECK(k.right(k.dst), "after enqueue %ld failed", i);
    dr_plan_destroy(k.p);
    fake::release_for_good();
  }
}

// The tile order follows a launch's depth and traffic, whichever call makes it: grouped up to 1 GiB
// at depth 2 and up to 6 GiB at depth 4.  The launches are only recorded, nothing runs.
void check_order() {
  const struct { int32_t vocab; double gib; } sizes[] = {  // one chunk; GiB read and written
      {2000, 0.1}, {20000, 0.9}, {25000, 1.2}, {80000, 3.7}, {120000, 5.5}, {140000, 6.5}, {200000, 9.2}};
  for (const auto& z : sizes)
    for (int depth : {0, 2, 4}) {
      const dr_model m{0, 4096, 32, 8, 128, 14336, z.vocab};
      const dr_layout l{1, 1, 1ull << 40, 0, depth, 0};
      dr_plan* p;
      CHECK(!dr_plan_create(&m, &l, &p), "%s", dr_last_error());
      const uint64_t bytes = 4 * p->info.n_elems + p->info.rollout_bytes;
      CHECK(std::abs(bytes / 1073741824.0 - z.gib) < 0.1, "%.2f GiB", bytes / 1073741824.0);
      float* src = reinterpret_cast<float*>(4096);  // never read
      dr_checksum* cks = reinterpret_cast<dr_checksum*>(4096);
      for (int chunk = 0; chunk < 2; ++chunk) {
        launched.clear();
        const int rc = chunk ? dr_stage_chunk(p, 0, &src, src, cks, nullptr) : dr_stage_all(p, &src, src, cks, nullptr);
        CHECK(!rc && launched.size() == 1, "%s", dr_last_error());
        const StageRecord& r = launched.back();
        CHECK(!depth || r.depth == depth, "depth %d", r.depth);
        CHECK(r.grouped == (z.gib < (r.depth == 4 ? 6 : 1)), "%.1f GiB, depth %d, chunk call %d: grouped %d", z.gib, r.depth,
              chunk, r.grouped);
      }
      fake::null_stream.ops.clear();
      dr_plan_destroy(p);
      fake::release_for_good();
    }
  // whole tiles per workgroup for a reshard of more than 44 GiB, and for chunks of as much
  for (int32_t vocab : {4000, 60000, 700000, 750000})
    for (uint64_t chunk : {1ull << 20, 1ull << 40}) {
      const dr_model m{0, 4096, 32, 8, 128, 14336, vocab};
      dr_plan* p;
      CHECK(!dr_reshard_plan_create(&m, 3, 2, chunk, &p), "%s", dr_last_error());
      float* at[3];
      for (float*& x : at) x = reinterpret_cast<float*>(4096);
      CHECK(!dr_reshard(p, at, at, reinterpret_cast<dr_checksum*>(4096), nullptr), "%s", dr_last_error());
      CHECK(resharded.back().whole_tiles == (vocab == 750000), "vocabulary %d: %d", vocab, resharded.back().whole_tiles);
      fake::null_stream.ops.clear();
      dr_plan_destroy(p);
      fake::release_for_good();
    }
}

// The path through host memory over one plan, twice: the pieces of its launches, each reloaded by the
// launch behind it, put the whole stream and its checksums in place.
void check_pieces(char** a) {
  const dr_model m{atoi(a[0]), atoi(a[1]), atoi(a[2]), atoi(a[3]), atoi(a[4]), atoi(a[5]), atoi(a[6])};
  Work k = setup(m, atoi(a[7]), atoi(a[8]), strtoull(a[9], nullptr, 10), atoi(a[10]));
  for (int i = 0; i < 2; ++i) {
    k.clear();
    launched.clear();
    CHECK(!k.through_host(k.dst, stream()), "%s", dr_last_error());
    (void)hipDeviceSynchronize();
    CHECK(k.right(k.dst), "through host");
    size_t packs = 0;
    for (const StageRecord& r : launched) packs += r.relay && r.ntiles;
    CHECK(launched.size() == packs + 1 && !launched.back().ntiles, "%zu launches", launched.size());
    if (!i) std::printf("pieces %zu\n", packs);
  }
  dr_plan_destroy(k.p);
  fake::release_for_good();
}

}  // namespace

int main(int argc, char** argv) {
  const std::string mode = argc > 1 ? argv[1] : "";
  if (mode == "copies") check_copies();
  else if (mode == "sums") check_sums();
  else if (mode == "destroy") check_destroy();
  else if (mode == "order") check_order();
  else if (mode == "pieces" && argc == 13) check_pieces(argv + 2);
  else return 2;
  CHECK(!fake::dead_accesses, "%d accesses to freed memory", fake::dead_accesses);
  std::printf("%s: %d errors\n", mode.c_str(), errors);
  return errors != 0;
}
