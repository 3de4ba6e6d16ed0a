// The tile kernels' index functions (tile_index.h) on the CPU, as the kernels call them.
//   index_check order                grouped and contiguous order, capped grids
//   index_check division
//   index_check parts               a reshard's parts cover every group of every segment once
//   index_check unaligned ROWS COLS STRIDE LEAD
// Exit status 0 when everything holds.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "tile_index.h"

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

using namespace dr;

// Every item once; the full windows' groups of G whole on one XCD.
template <uint32_t G, typename T>
static void check_group(T n) {
  std::vector<T> at(n, n);  // item -> workgroup
  for (T b = 0; b < n; ++b) {
    const T t = xcd_group<G>(b, n);
    CHECK(t < n && at[t] == n, "group %u, n %llu, workgroup %llu", G, (unsigned long long)n, (unsigned long long)b);
    if (t < n) at[t] = b;
  }
  for (T t = 0; t + 1 < n / (kXcds * G) * (kXcds * G); ++t)
    if ((t + 1) % G) CHECK(at[t] % kXcds == at[t + 1] % kXcds, "group %u, n %llu: items %llu", G, (unsigned long long)n, (unsigned long long)t);
}

static void check_order() {
  for (uint32_t n : {1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 1536, 4099, 8192, 10000}) {
    check_group<kTileGroup, uint32_t>(n);
    check_group<kPartGroup, uint64_t>(n);
    std::vector<bool> seen(n);
    for (uint32_t b = 0; b < n; ++b) {
      const uint32_t t = xcd_tile(b, n);
      CHECK(t < n && !seen[t], "contiguous, n %u, workgroup %u", n, b);
      if (t < n) seen[t] = true;
      if (b + kXcds < n) CHECK(xcd_tile(b + kXcds, n) == t + 1, "contiguous, n %u, workgroup %u", n, b);
    }
  }
}

static void check_division() {
  std::mt19937 rng(0);
  std::vector<uint32_t> cols = {3456, 3584, 4096, 4864, 27648, (1u << 30) - 1, 1u << 30};
  for (uint32_t c = 1; c < 2100; ++c) cols.push_back(c);
  for (int i = 0; i < 300; ++i) cols.push_back(1 + rng() % (1u << 30));
  for (uint32_t c : cols) {
    DevSeg s{};
    s.rows = 2, s.cols = c, s.stride = c + 3, s.magic = c == 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / c);
    std::vector<uint32_t> es = {0, 1, c - 1, c, c + 1, (1u << 30) - 1, (1u << 31) - 1, 0xFFFFFFFFu};
    for (int i = 0; i < 64; ++i) es.push_back(rng());
    for (uint32_t e : es) {
      uint32_t r, col;
      CHECK(div_cols(e, c, s.magic, &r) == e / c && r == e % c, "%u / %u", e, c);
      CHECK(elem_src(s, e, &col) == e / c * s.stride + e % c && col == e % c, "%u of rows of %u", e, c);
    }
  }
}

// reshard_tile's lanes over every tile and part of a segment of `units` groups
static void check_segment(uint64_t chunk_elems, uint32_t units) {
  const uint32_t parts = 1u << reshard_part_shift(chunk_elems);
  std::vector<int> moved(units);
  for (uint32_t unit0 = 0; unit0 < units; unit0 += kThreads * kReshardIters)  // the planner's tiles
    for (uint32_t part = 0; part < parts; ++part) {
      const uint32_t first = unit0 + part * kPartIters * kThreads;
      for (uint32_t i = 0; first < units && i < (uint32_t)kPartIters * kThreads; ++i)
        if (first + i < units) ++moved[first + i];
    }
  for (uint32_t u = 0; u < units; ++u) CHECK(moved[u] == 1, "chunk of %llu elements, %u groups: %u", (unsigned long long)chunk_elems, units, u);
}

static void check_parts() {
  for (uint32_t chunk_groups : {1, 255, 256, 511, 512, 513, 1023, 1024, 1025, 5000})
    for (uint32_t units : {1u, 2u, 511u, 512u, 513u, 1023u, 1024u, 1025u, 2048u, 2049u, chunk_groups})
      if (units <= chunk_groups) check_segment(4ull * chunk_groups, units);  // a segment lies in one chunk
}

// Which element every lane of every tile of an unaligned segment loads from where, and stores: each
// element once, from (e / cols) * stride + e % cols; no load outside the group's span.
static void check_unaligned(uint32_t rows, uint32_t cols, uint32_t stride, uint32_t lead) {
  DevSeg s{};
  s.rows = rows;
  s.cols = rows > 1 ? cols : rows * cols;
  s.stride = rows > 1 ? stride : s.cols;
  s.magic = s.cols == 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / s.cols);
  s.units = rows * cols;
  std::vector<int64_t> from(s.units, -1);
  std::vector<int> stored(s.units);
  const auto src = [&](uint32_t e) { return (int64_t)(e / s.cols) * s.stride + e % s.cols; };
  uint32_t col;
  for (uint32_t unit0 = 0; unit0 < s.units; unit0 += kScalarUnitsPerTile) {
    for (int k = 0; k < kScalarIters / 4; ++k)
      for (uint32_t lane = 0; lane < (uint32_t)kThreads; ++lane) {
        const int32_t e = group_elem(unit0, k, lane, lead);
        if (wide_group(s, e)) {
          const int64_t p = elem_src(s, e, &col), cut = group_cut(s, col);
          CHECK(whole_group(s, e) && p == src(e) && p + 3 <= src(e + 3), "first load of %d", e);
          if (cut < 4) CHECK(p + (s.stride - s.cols) + 3 == src(e + 3), "second load of %d", e);
          for (int j = 0; j < 4; ++j) from[e + j] = j < cut ? p + j : p + (s.stride - s.cols) + j;
        }
        if (whole_group(s, e)) CHECK((lead + e) % 4 == 0, "8-byte store of %d", e);
        for (int32_t x = e; x < e + 4; ++x) {
          if (x < 0 || (uint32_t)x >= s.units) continue;
          if (!wide_group(s, e)) from[x] = elem_src(s, x, &col);
          ++stored[x];
        }
      }
    for (uint32_t lane = 0; lane < (uint32_t)kThreads; ++lane) {
      uint32_t x;
      if (!tail_elem(s, unit0, lane, lead, &x)) continue;
      CHECK(x < s.units, "tail %u", x);
      from[x] = elem_src(s, x, &col);
      ++stored[x];
    }
  }
  for (uint32_t e = 0; e < s.units; ++e) CHECK(from[e] == src(e) && stored[e] == 1, "element %u: from %lld, stored %d times", e, (long long)from[e], stored[e]);
}

int main(int argc, char** argv) {
  const std::string mode = argc > 1 ? argv[1] : "";
  if (mode == "order") check_order();
  else if (mode == "division") check_division();
  else if (mode == "parts") check_parts();
  else if (mode == "unaligned" && argc == 6) check_unaligned(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]));
  else return 2;
  std::printf("%s: %d errors\n", mode.c_str(), errors);
  return errors != 0;
}
