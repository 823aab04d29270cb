// Plan and launchers of the distribution sort: an array longer than one LDS
// tile is cut into buckets by sampled splitters, level by level, until every
// bucket fits one workgroup, which sorts it in LDS.
#pragma once
#include <algorithm>

#include "pss_internal.hpp"

namespace pss {

// One tile of a level: kDistThreads * kDistItems keys.
constexpr int kDistThreads = 512;
constexpr int kDistItems = 12;
constexpr uint32_t kDistTile = kDistThreads * kDistItems;
// Buckets of one node: at most kDistMaxPicks sampled picks, of which each may
// add a second splitter (the next larger key, so that a frequent key gets a
// bucket of its own), capped at kDistSlots buckets.
constexpr uint32_t kDistMaxPicks = 384;
constexpr uint32_t kDistSlots = 512;
constexpr int kDistMaxLevels = 3;
// Keys one workgroup sorts in LDS, and the mean bucket the splitters aim at:
// half of it.  A bucket between every k-th of the samples then overflows with the
// odds of a gamma variable of order k above twice its mean: 1.8e-4 at k = 20 (a
// node of 384 buckets has 21 samples a bucket), 4e-6 at 32, 1e-10 at 64 (up to 128
// buckets); it is sorted all the same, by all workgroups in the last kernel.
constexpr uint32_t kDistCap = 8192, kDistCapKV = 4096;
constexpr uint32_t kDistTarget = 4096, kDistTargetKV = 2048;
// Most tiles of one range.
constexpr uint32_t kDistRangeTiles = 11;
// Shortest array whose last level gathers its keys.  Sampling gathered nodes
// and looking up their pieces costs more than the count and the scatter of
// short arrays, less than those of long ones (us, scattered and gathered, random
// keys; 2.4*10^7: int64 426 and 460, with values 654 and 666, int32 354 and 379, 508
// and 549; 2^25: 561 and 569, 895 and 857, 451 and 466, 701 and 708; 10^8: 1633 and
// 1421, 2543 and 2212, 1174 and 1123, 2032 and 1894; 5*10^7 is the one length above
// the line where int32 keys are still faster scattered, 610 and 642).
constexpr uint64_t kDistGatherMin = (uint64_t)1 << 25;
// Segments of up to as many buckets are cut by the first level alone where the
// plan has more levels for longer ones and the first one scatters (by two levels
// in brackets: 50 segments of 300007 int64 without a bound on the length, random
// 251 us (339), of 1000 values 427 (515), with values 325 and 600 (435 and 721)).
// Of wider ones it is slower where the segments are few, as a single workgroup
// samples each: 4 of 700000 int64, 171 buckets, 153 and 238 us (153 and 202); 2 of
// 900000, 220 buckets, 157 and 254 (146 and 187).
constexpr uint32_t kDistOneLevel = 160;
// With a bound on the length some segment needs the levels, and the others take
// one only if there are as many keys: sampling them for good adds to the chain of
// launches (96 requests, 1.7*10^7 u64 with values, most of them in requests that
// need two levels: 768 us (733); 384 requests, 5.8*10^7, 1553 (1588); 4096 arrays,
// 4.5*10^8 int64, 4630 (4856)).
constexpr uint64_t kDistOneKeys = (uint64_t)1 << 25;
// Most tiles of a node of the last level: a leaf lists one piece a tile in the
// LDS its keys take later.  Sampled nodes stay far below.
inline constexpr uint32_t dist_node_tiles(int kb, bool kv) {
  return (kv ? kDistCapKV : kDistCap) * (uint32_t)kb / 4;
}

// A stretch of keys being cut into buckets by one level.
struct DistNode {
  uint32_t off, len;  // its keys
  uint32_t p;         // buckets aimed at
  uint32_t nr;        // ranges, one workgroup each
  uint32_t cols;      // bucket slots reserved (at most 2 p)
  uint32_t sbase;     // first entry in the splitter and start arrays
  uint32_t tbase;     // first entry in the level's table
  uint32_t stride;    // table entries per bucket
  uint32_t nb;        // buckets (splitters + 1), set by the sampling kernel
  // gathered nodes: the node it was a bucket of, and the rows of that node's
  // table for this bucket and the next one (~0: the last bucket)
  uint32_t poff, plen, prow, pnext;
};
// The table of a level: keys of every bucket in every range ([bucket][range],
// uint32, made into prefix sums), or, for a level that leaves its tiles in
// place (DistPlan::tiled), where every bucket starts in every tile
// ([bucket][tile], uint16).
struct DistRange { uint32_t node, r; };  // (gathered level: those of copies only)
// A bucket (or at most cap keys of one) to be sorted or moved, with all that
// its workgroup needs to know.
struct DistLeaf {
  uint32_t off;        // its place in the output
  uint32_t len_flags;  // length, kLeaf* flags
  // last level: the node's keys, the bucket's first key here, and the table
  // rows of its starts and of the next bucket's (~0: the bucket is the last)
  uint32_t node_off, node_len, first, row, next_row;
  uint32_t pad;
  uint64_t below, above;  // kLeafInner: below <= key < above
};
// A bucket the last level left above the cap, moved to its place in the output.
struct DistBig {
  uint32_t off, len;
  uint32_t done;  // tasks of its sort that have ended
  uint32_t pad;
};
struct DistCounters {
  uint32_t nodes[kDistMaxLevels + 1], ranges[kDistMaxLevels + 1];
  uint32_t cols[kDistMaxLevels + 1], table[kDistMaxLevels + 1];
  uint32_t leaves, rest, big;
  // the last kernel's: crowded leaves sorted, and tasks claimed
  uint32_t rest_done, next_task;
  // gathered: buckets of the level before that are not cut again, and the most
  // ranges of one that is
  uint32_t copies, most_ranges;
  uint32_t failed;    // a bound of the plan did not hold
};

// DistLeaf::len_flags
constexpr uint32_t kLeafLenMask = 0xffffu;
constexpr uint32_t kLeafEqual = 1u << 16;  // one key value: unmapped, not sorted
constexpr uint32_t kLeafMove = 1u << 17;   // part of a big bucket: moved to the output
constexpr uint32_t kLeafInner = 1u << 18;  // the splitters around it bound its keys
constexpr int kLeafSrcShift = 19;          // where its keys are:
constexpr uint32_t kSrcWs = 0, kSrcOut = 1, kSrcPieces = 2;

// Host bounds and workspace layout (byte offsets) of one distribution sort.
struct DistPlan {
  bool on = false;
  int levels = 0;
  uint32_t cap = 0, target = 0;
  uint32_t root_p = 0;    // most buckets aimed at in a first-level node
  uint32_t n_segs = 0;    // segmented: segments (0: one array)
  uint32_t one_p = 0;     // the first level cuts segments of up to as many buckets for good
  // Two or more levels: the level before the last leaves its tiles in place
  // as well, and the last level gathers its keys from them, which takes the
  // place of a count and a scatter (if the tables fit the workspace).
  bool gather = false;
  bool tiled(int level) const { return level == levels || (gather && level == levels - 1); }
  uint32_t rl[kDistMaxLevels + 1] = {};  // keys of a range (whole tiles)
  uint32_t max_nodes[kDistMaxLevels + 1] = {}, max_ranges[kDistMaxLevels + 1] = {};
  uint32_t max_cols = 0, max_table[kDistMaxLevels + 1] = {}, max_leaves = 0, max_rest = 0, max_big = 0;
  uint32_t max_copies = 0;
  uint32_t leaf_grid = 0;  // workgroups of the leaf kernel: the leaves to expect
  size_t off_ctr = 0, off_nodes[kDistMaxLevels + 1] = {}, off_ranges[kDistMaxLevels + 1] = {};
  size_t off_ptable = 0, off_pre = 0;  // gathered: the level before's table, keys before every 8 tiles
  size_t off_spl = 0, off_start = 0, off_table = 0, off_leaves = 0, off_rest = 0, off_big = 0;
  size_t end = 0;  // first byte after the distribution's arrays
};

// Smallest p with p^levels >= units.
inline uint32_t dist_root(uint64_t units, int levels) {
  uint64_t p = 1;
  auto pow = [&](uint64_t x) {
    uint64_t y = 1;
    for (int i = 0; i < levels; ++i) y *= x;
    return y;
  };
  while (pow(p) < units) ++p;
  return (uint32_t)p;
}

// Plan of n keys in arrays of at most max_len > cap keys (one array: max_len =
// n and n_segs = 0; of n_segs segments, those above min_len >= cap keys), laid
// out from byte offset `off` on.  Arrays of up to `longest` keys are sorted too,
// with as many first-level buckets as they need, or kDistMaxPicks.  One level reaches
// kDistMaxPicks buckets of the target size; two levels are kept up to 144000
// (380 x 380).  Up to 65536 (2^28 keys) a first-level bucket half as large again
// as the mean still gets its share of second-level buckets; above, the larger ones
// get fewer than the target size asks for, and larger leaves or big buckets, as a
// third level would move every key once or twice more.
inline DistPlan dist_plan(uint64_t n, uint64_t max_len, uint32_t n_segs, uint64_t min_len,
                          uint64_t longest, int kb, bool kv, size_t off, bool gather) {
  DistPlan d;
  d.cap = kv ? kDistCapKV : kDistCap;
  d.target = kv ? kDistTargetKV : kDistTarget;
  d.n_segs = n_segs;
  const uint64_t units = (max_len + d.target - 1) / d.target;
  d.levels = units <= kDistMaxPicks ? 1 : units <= 144000 ? 2 : 3;
  d.gather = gather && d.levels > 1 && max_len >= kDistGatherMin;
  if (n_segs && d.levels > 1 && !d.tiled(1) && (max_len == n || n >= kDistOneKeys)) d.one_p = kDistOneLevel;
  d.root_p = std::max<uint32_t>(
      2, std::min(kDistMaxPicks, dist_root((longest + d.target - 1) / d.target, d.levels)));
  auto tiles = [](uint64_t x) { return (x + kDistTile - 1) / kDistTile; };
  uint64_t nodes = n_segs ? std::min<uint64_t>(n_segs, n / min_len + 1) : 1;
  uint64_t cols = n_segs ? 2 * (n / d.target) + 4 * nodes : std::min(kDistSlots, 2 * d.root_p);
  uint64_t leaves = 0, max_cols = 0, table_bytes = 0, ptable_bytes = 0;
  for (int l = 1; l <= d.levels; ++l) {
    const bool tiled = d.tiled(l);
    // A first level that scatters covers the array with two ranges a CU
    // (one round of workgroups); otherwise nodes are of uneven length, and
    // more, shorter ranges balance better.
    const uint64_t rt = l == 1 && !tiled ? tiles((n + 511) / 512)
                                        : std::min<uint64_t>(kDistRangeTiles, tiles((n + 2047) / 2048));
    d.rl[l] = (uint32_t)(rt * kDistTile);
    if (l > 1) {
      if (d.gather && l == d.levels) d.max_copies = (uint32_t)cols;
      nodes = std::min<uint64_t>(cols, n / d.cap + 1);
      cols = std::min<uint64_t>(2 * (n / d.target) + 4 * nodes, (uint64_t)kDistSlots * nodes);
    }
    d.max_nodes[l] = (uint32_t)nodes;
    d.max_ranges[l] = (uint32_t)(n / d.rl[l] + nodes + (l == d.levels ? d.max_copies : 0));
    max_cols = std::max(max_cols, cols);
    // rows of the table are its buckets: at most 2 root_p in the first level,
    // unless it cuts some segments for good, and kDistSlots later; tiles are
    // padded to 8 entries
    const uint64_t widest = l == 1 && !d.one_p ? std::min(kDistSlots, 2 * d.root_p) : kDistSlots;
    const uint64_t table =
        tiled ? widest * (n / kDistTile) + 9 * cols : widest * (n / d.rl[l]) + cols;
    d.max_table[l] = (uint32_t)std::min<uint64_t>(table, 0xffffffffu);
    if (tiled && l < d.levels) ptable_bytes = table * 2;
    else table_bytes = std::max(table_bytes, table * (tiled ? 2 : 4));
    leaves += cols;
  }
  d.max_cols = (uint32_t)max_cols;
  d.max_leaves = (uint32_t)(leaves + n / d.cap + 1);
  const uint64_t expect = n / d.target + n / d.target / 8 + d.max_nodes[d.levels] + 64;
  d.leaf_grid = (uint32_t)((std::min<uint64_t>(d.max_leaves, expect) + 7) / 8 * 8);
  d.max_rest = d.max_leaves;
  d.max_big = (uint32_t)(n / d.cap);
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) / 256 * 256;
    return o;
  };
  d.off_ctr = take(sizeof(DistCounters));
  for (int l = 1; l <= d.levels; ++l) {
    d.off_nodes[l] = take((size_t)(d.max_nodes[l] + (l == d.levels ? d.max_copies : 0)) * sizeof(DistNode));
    d.off_ranges[l] = take((size_t)d.max_ranges[l] * sizeof(DistRange));
  }
  d.off_spl = take((size_t)d.max_cols * kb);
  d.off_start = take((size_t)d.max_cols * 4);
  d.off_table = take((size_t)table_bytes);
  d.off_ptable = take((size_t)ptable_bytes);
  d.off_pre = take((size_t)ptable_bytes / 4);  // a uint32 for every 8 entries
  d.off_leaves = take((size_t)d.max_leaves * sizeof(DistLeaf));
  d.off_rest = take((size_t)d.max_rest * 4);
  d.off_big = take((size_t)d.max_big * sizeof(DistBig));
  d.end = off;
  return d;
}

// Keys and values of one distribution sort.
struct DistBufs {
  const void *in;
  const uint32_t *vin;
  void *ws;
  uint32_t *vws;
  void *out;
  uint32_t *vout;
};

// Segmented: reads the segment offsets, and writes the first level's nodes and
// ranges, of the segments above `merged` keys; those above `longest` are left out
// (the merge passes' planner reports them).  The steps of a level and the two
// kernels that end the sort follow.  Declared weak so that a host-only program can
// link the plan without the device code; a sort then fails (pss_api.hip), and is
// never run another way.
#define PSS_WEAK __attribute__((weak))
PSS_WEAK hipError_t launch_dist_segments(const DistPlan &d, const uint64_t *seg_off, uint64_t n,
                                         uint64_t merged, uint64_t longest, char *w, hipStream_t s);
PSS_WEAK hipError_t launch_dist_sample(int kt, const DistPlan &d, int level, const DistBufs &b,
                                       uint64_t n, char *w, hipStream_t s);
// before the last level
PSS_WEAK hipError_t launch_dist_count(int kt, const DistPlan &d, int level, const DistBufs &b,
                                      char *w, hipStream_t s);
PSS_WEAK hipError_t launch_dist_scan(int kt, const DistPlan &d, int level, char *w, hipStream_t s);
PSS_WEAK hipError_t launch_dist_scatter(int kt, bool kv, const DistPlan &d, int level,
                                        const DistBufs &b, char *w, hipStream_t s);
// levels that leave their tiles in place (launch_dist_scan follows)
PSS_WEAK hipError_t launch_dist_partition(int kt, bool kv, const DistPlan &d, int level,
                                          const DistBufs &b, char *w, hipStream_t s);
// after a partition that is not the last level's
PSS_WEAK hipError_t launch_dist_pieces(int kt, const DistPlan &d, int level, char *w,
                                       hipStream_t s);
PSS_WEAK hipError_t launch_dist_leaves(int kt, bool kv, const DistPlan &d, const DistBufs &b, char *w,
                                       hipStream_t s);
PSS_WEAK hipError_t launch_dist_rest(int kt, bool kv, const DistPlan &d, const DistBufs &b, char *w,
                                     hipStream_t s);
#undef PSS_WEAK

}  // namespace pss
