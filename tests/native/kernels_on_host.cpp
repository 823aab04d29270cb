// Sorts through the library's own C entry points with every kernel run on the
// host (hip_emu/), under the address and undefined-behaviour sanitizers, each
// result compared with std::stable_sort.  Arguments: the case's name and the
// seed of the order in which waves and workgroups run (0: ascending).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <random>
#include <string>

#include "../../paper_2305_05245_amd/csrc/pss_dist.hpp"
#include "pss.h"

namespace {

int failures = 0;
#define CHECK(c, ...)                                                   \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::fprintf(stderr, "line %d: %s: ", __LINE__, #c);              \
      std::fprintf(stderr, __VA_ARGS__);                                \
      std::fprintf(stderr, "\n");                                       \
      ++failures;                                                       \
    }                                                                   \
  } while (0)

pss_ctx *ctx;
std::mt19937_64 rng;

uint32_t device_error() {
  uint32_t code = ~0u;
  CHECK(pss_device_check(ctx, &code) == PSS_OK, "device check");
  return code;
}

// A buffer of exactly `bytes` bytes, filled with 0xAB (its ends are checked by
// the address sanitizer).
struct Buffer {
  char *p;
  explicit Buffer(size_t bytes) : p((char *)std::malloc(bytes ? bytes : 1)) { std::memset(p, 0xAB, bytes); }
  ~Buffer() { std::free(p); }
  Buffer(const Buffer &) = delete;
};

// Segments of uint64 keys (values: their positions) sorted in one call; `sorted`
// tells which of them have to come out sorted.
template <typename Sorted>
void segments(const std::vector<uint64_t> &lens, uint64_t bound, bool kv, uint64_t distinct,
              uint32_t expect_error, Sorted sorted) {
  std::vector<uint64_t> off(1, 0);
  for (uint64_t l : lens) off.push_back(off.back() + l);
  const uint64_t n = off.back();
  std::vector<uint64_t> keys(n), out(n);
  std::vector<uint32_t> vals(n), vout(n);
  for (uint64_t i = 0; i < n; ++i) {
    keys[i] = distinct ? rng() % distinct * 0x9E3779B97F4A7C15ull : rng();
    vals[i] = (uint32_t)i;
  }
  const pss_tuning tu{2048, 4096, bound, 0, 0};
  const pss_val_t val = kv ? PSS_VAL_U32 : PSS_VAL_NONE;
  size_t need = 0;
  CHECK(pss_segmented_workspace_bytes(ctx, PSS_U64, val, n, (uint32_t)lens.size(), &tu, &need) == PSS_OK, "workspace");
  Buffer ws(need);
  const pss_status st = pss_segmented_sort(ctx, PSS_U64, val, keys.data(), out.data(), vals.data(), vout.data(), n,
                                           off.data(), (uint32_t)lens.size(), &tu, ws.p, need, nullptr);
  CHECK(st == PSS_OK, "%s", pss_last_error(ctx));
  CHECK(device_error() == expect_error, "device error word");
  for (size_t s = 0; s < lens.size(); ++s) {
    if (!sorted(s)) continue;
    std::vector<uint32_t> at(vals.begin() + off[s], vals.begin() + off[s + 1]);
    std::stable_sort(at.begin(), at.end(), [&](uint32_t a, uint32_t b) { return keys[a] < keys[b]; });
    for (uint64_t i = off[s]; i < off[s + 1]; ++i) {
      const uint32_t from = at[i - off[s]];
      if (out[i] != keys[from] || (kv && vout[i] != from)) {
        CHECK(false, "segment %zu of %zu, position %llu", s, lens.size(), (unsigned long long)(i - off[s]));
        break;
      }
    }
  }
}

// A segment longer than the bound on the segment length allows is left out and
// reported; the others are sorted, whichever wave finds it first.
void segment_left_out() {
  // no segment above one tile, some (merged), and one that is distributed
  const uint64_t bounds[] = {4096, 9000, 140000}, left_out[] = {9000, 140000, 17000000};
  for (int i = 0; i < 3; ++i) {
    std::vector<uint64_t> lens(200, 70);
    for (size_t s = 0; s < lens.size(); s += 23) lens[s] = 3000;
    lens[130] = bounds[i];
    lens[70] = left_out[i];
    segments(lens, bounds[i], true, 0, 16, [](size_t s) { return s != 70; });
  }
}

// One distribution sort of uint64 keys by the launches of plan d (whose arrays
// end at byte `bytes` of the workspace, after keys and values); true if the
// output is sorted.
bool distribution(const pss::DistPlan &d, size_t bytes, const std::vector<uint64_t> &keys, bool kv,
                  pss::DistCounters *ctr = nullptr) {
  const uint64_t n = keys.size();
  std::vector<uint64_t> out(n);
  std::vector<uint32_t> vals(n), vout(n);
  for (uint64_t i = 0; i < n; ++i) vals[i] = (uint32_t)i;
  Buffer ws(bytes), kws(n * 8), vws(n * 4);
  const pss::DistBufs b{keys.data(), vals.data(), kws.p, (uint32_t *)vws.p, out.data(), vout.data()};
  const int kt = PSS_U64;
  for (int l = 1; l <= d.levels; ++l) {
    CHECK(pss::launch_dist_sample(kt, d, l, b, n, ws.p, nullptr) == hipSuccess, "sample");
    if (!d.tiled(l)) {
      CHECK(pss::launch_dist_count(kt, d, l, b, ws.p, nullptr) == hipSuccess, "count");
      CHECK(pss::launch_dist_scan(kt, d, l, ws.p, nullptr) == hipSuccess, "scan");
      CHECK(pss::launch_dist_scatter(kt, kv, d, l, b, ws.p, nullptr) == hipSuccess, "scatter");
    } else {
      CHECK(pss::launch_dist_partition(kt, kv, d, l, b, ws.p, nullptr) == hipSuccess, "partition");
      if (l < d.levels) CHECK(pss::launch_dist_pieces(kt, d, l, ws.p, nullptr) == hipSuccess, "pieces");
      CHECK(pss::launch_dist_scan(kt, d, l, ws.p, nullptr) == hipSuccess, "scan");
    }
  }
  CHECK(pss::launch_dist_leaves(kt, kv, d, b, ws.p, nullptr) == hipSuccess, "leaves");
  CHECK(pss::launch_dist_rest(kt, kv, d, b, ws.p, nullptr) == hipSuccess, "rest");
  if (ctr) std::memcpy(ctr, ws.p + d.off_ctr, sizeof(*ctr));
  std::vector<uint32_t> at(vals);
  std::stable_sort(at.begin(), at.end(), [&](uint32_t x, uint32_t y) { return keys[x] < keys[y]; });
  for (uint64_t i = 0; i < n; ++i)
    if (out[i] != keys[at[i]] || (kv && vout[i] != at[i])) return false;
  return true;
}

bool distribution(const pss::DistPlan &d, size_t bytes, uint64_t n, bool kv, uint64_t distinct) {
  std::vector<uint64_t> keys(n);
  for (auto &k : keys) k = distinct ? rng() % distinct * 0x9E3779B97F4A7C15ull : rng();
  return distribution(d, bytes, keys, kv);
}

// A plan with too little room for its buckets: nothing is written past its
// arrays, and the error word says so.
void plan_bounds() {
  const uint64_t n = 150001;
  for (int shape = 0; shape < 3; ++shape)  // one level, two that scatter, two that gather
    for (bool kv : {false, true}) {
      const uint64_t len = shape == 0 ? n : shape == 1 ? 1 << 22 : 1 << 25;
      pss::DistPlan d = pss::dist_plan(n, len, 0, 0, len, 8, kv, 0, shape == 2);
      CHECK(d.levels == (shape == 0 ? 1 : 2) && d.gather == (shape == 2), "shape %d", shape);
      if (shape) d.root_p = 6;  // (keys for a second level)
      const size_t bytes = d.end;
      CHECK(distribution(d, bytes, n, kv, 0) && device_error() == 0, "shape %d as planned", shape);
      // (few values: buckets of the first level that are not cut again)
      CHECK(distribution(d, bytes, n, kv, 3) && device_error() == 0, "shape %d, three values", shape);
      auto lowered = [&](const char *what, uint64_t distinct, auto change) {
        pss::DistPlan low = d;
        change(low);
        (void)distribution(low, bytes, n, kv, distinct);
        CHECK(device_error() == 32, "shape %d, %s, %s", shape, kv ? "values" : "keys", what);
      };
      lowered("leaves", 0, [](pss::DistPlan &p) { p.max_leaves = 3; });
      if (shape == 0) lowered("big buckets", 0, [](pss::DistPlan &p) { p.root_p = 2, p.max_big = 1; });
      if (shape == 0) lowered("crowded leaves", 2000, [](pss::DistPlan &p) { p.max_rest = 1; });
      if (shape == 0) continue;
      lowered("nodes", 0, [](pss::DistPlan &p) { p.max_nodes[2] = 2; });
      lowered("columns", 0, [](pss::DistPlan &p) { p.max_cols = 13; });
      lowered("table", 0, [](pss::DistPlan &p) { p.max_table[2] = 100; });
      if (shape == 1) lowered("ranges", 0, [](pss::DistPlan &p) { p.max_ranges[2] = 2; });
      if (shape == 2 && kv) lowered("copies", 3, [](pss::DistPlan &p) { p.max_copies = 1; });
    }
}

// Buckets far above the cap: of two tiles to all of the array, with lengths at
// the edges of tiles and of pairs of runs.
void big_buckets() {
  for (uint64_t n : {30001, 65536, 65537, 81921, 150001})
    for (bool kv : {false, true})
      for (uint64_t distinct : {0, 300, 20000}) {
        pss::DistPlan d = pss::dist_plan(n, n, 0, 0, n, 8, kv, 0, false);
        d.root_p = 2;
        const size_t bytes = d.end;
        CHECK(distribution(d, bytes, n, kv, distinct), "%llu keys, %s, %llu values", (unsigned long long)n,
              kv ? "values" : "keys", (unsigned long long)distinct);
        CHECK(device_error() == 0, "device error word");
      }
}

// Segments on both sides of the longest that is merged, in calls with a bound on
// the length and without, where their mean length decides.
void segment_routes() {
  const std::vector<uint64_t> shorter = {100, 4096, 4097, 131071, 0, 131072, 5000, 9000};
  const std::vector<uint64_t> some = {100, 4096, 4097, 131071, 0, 131072, 131073, 9000};
  const std::vector<uint64_t> longer = {131073, 131072, 270000};
  // (more than one level can cut: the first one cuts those that it can, unless the
  // length is bounded and the keys are few, or the level leaves its tiles in place)
  const auto one_p = [](uint64_t n, uint64_t max_len) {
    return pss::dist_plan(n, max_len, 96, 131072, max_len, 8, true, 0, true).one_p;
  };
  CHECK(one_p(10000000, 10000000) == pss::kDistOneLevel && one_p(10000000, 1 << 20) == 0, "one level, 10^7");
  CHECK(one_p(1 << 24, 1 << 20) == 0 && one_p(1 << 25, 1 << 20) == pss::kDistOneLevel && one_p(1 << 25, 1 << 25) == 0, "one level, more");
  const std::vector<uint64_t> levels = {327680, 131073, 327681, 150001, 7};
  for (uint64_t distinct : {0, 900}) {
    segments(levels, 0, true, distinct, 0, [](size_t) { return true; });
    segments(shorter, 131072, true, distinct, 0, [](size_t) { return true; });
    segments(some, 131073, true, distinct, 0, [](size_t) { return true; });
    segments(some, 0, true, distinct, 0, [](size_t) { return true; });
    segments(longer, 0, true, distinct, 0, [](size_t) { return true; });
  }
}

// One leaf of n keys with `copies` of each: an array whose samples all fall on a
// smaller key that is most of it, so that the n keys are one bucket.
void one_leaf(uint64_t n, uint64_t copies, bool small, bool kv) {
  std::vector<uint64_t> keys;
  for (uint64_t i = 0; i < n; ++i) keys.push_back(1 + (small ? i / copies : i / copies * 0x9E3779B97F4A7C15ull >> 1));
  keys.resize(5 * n, 0);
  std::shuffle(keys.begin(), keys.end(), rng);
  pss::DistPlan d = pss::dist_plan(keys.size(), keys.size(), 0, 0, keys.size(), 8, kv, 0, false);
  const size_t bytes = d.end;
  d.root_p = 2;
  CHECK(distribution(d, bytes, keys, kv), "leaf of %llu keys, %llu copies, %s, %s", (unsigned long long)n,
        (unsigned long long)copies, small ? "small" : "wide", kv ? "values" : "keys");
  CHECK(device_error() == 0, "device error word");
}

// Leaves at the limits of a bin's keys and of the list of bins.
void leaf_bins() {
  for (uint64_t copies : {1, 2, 3, 6, 15, 16, 17, 96, 97, 255, 256})
    for (bool small : {false, true})
      for (bool kv : {false, true})
        for (uint64_t n : kv ? std::vector<uint64_t>{4093, 4096} : std::vector<uint64_t>{8191, 8192})
          one_leaf(n, copies, small, kv);
}

// Leaves whose bins are crowded by values of many copies, of all lengths: in
// pieces, in the output and in the workspace (buckets of a first level that
// scatters or gathers); and with big buckets among them.
void crowded_leaves() {
  for (uint64_t copies : {25, 50, 300, 3000})
    for (bool kv : {false, true}) {
      for (uint64_t l : {1023, 1024, 1025, 2500, 4096, 5000, 7169})
        if (!kv || l <= 4096) one_leaf(l, copies, false, kv);
      const uint64_t n = 100003;
      for (int shape = 0; shape < 3; ++shape) {
        const uint64_t len = shape == 0 ? n : shape == 1 ? 1 << 22 : 1 << 25;
        for (uint32_t root : {3u, 45u}) {
          pss::DistPlan d = pss::dist_plan(n, len, 0, 0, len, 8, kv, 0, shape == 2);
          const size_t bytes = d.end;
          d.root_p = root;
          if (shape == 0 && root > 3) continue;
          CHECK(distribution(d, bytes, n, kv, n / copies), "shape %d, root %u, %s, %llu copies", shape, root,
                kv ? "values" : "keys", (unsigned long long)copies);
          CHECK(device_error() == 0, "device error word");
        }
      }
    }
}

// More buckets aimed at than half of the slots, and values so frequent that each
// pick takes two splitters: as many picks as fit, so that few of the buckets
// between (4 of 1000 values, 3000 keys, with every slot used) are above the cap.
void doubled_splitters() {
  for (uint64_t n : {700001, 760001}) {
    const pss::DistPlan d = pss::dist_plan(n, n, 0, 0, n, 8, true, 0, false);
    CHECK(d.levels == 1, "%d levels", d.levels);
    std::vector<uint64_t> keys(n);
    for (auto &k : keys) k = rng() % 1000 * 0x9E3779B97F4A7C15ull;
    pss::DistCounters ctr;
    CHECK(distribution(d, d.end, keys, true, &ctr), "%llu keys", (unsigned long long)n);
    CHECK(ctr.big <= 4, "%llu keys: %u buckets above the cap", (unsigned long long)n, ctr.big);
    CHECK(device_error() == 0, "device error word");
  }
}

}  // namespace

int main(int argc, char **argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  emu::seed = argc > 2 ? (uint32_t)std::atoi(argv[2]) : 0;
  if (pss_create(0, &ctx) != PSS_OK) return 2;
  const struct { const char *name; void (*run)(); } cases[] = {
      {"segment_left_out", segment_left_out}, {"plan_bounds", plan_bounds}, {"big_buckets", big_buckets},
      {"crowded_leaves", crowded_leaves}, {"leaf_bins", leaf_bins}, {"segment_routes", segment_routes},
      {"doubled_splitters", doubled_splitters}};
  bool found = false;
  for (const auto &c : cases) {
    if (name != c.name) continue;
    found = true;
    c.run();
  }
  pss_destroy(ctx);
  if (!found) std::fprintf(stderr, "no case %s\n", name.c_str());
  if (failures || !found) return 1;
  std::printf("%s passed\n", name.c_str());
  return 0;
}
