// Distribution sort for gfx950: arrays longer than one LDS tile.
//
// The merge passes of the single level move every key through HBM once per
// factor of 32 and through log2(F) rounds of LDS merges each time.  Here a
// level cuts a node (a stretch of keys) into up to 512 buckets instead:
//
//   sample     a few thousand stratified random keys of the node, sorted in
//              LDS; every (S/p)-th is a splitter.  A key seen twice at a
//              splitter also gives the next larger key, so that a frequent key
//              has a bucket of its own, which needs no further work.
//   partition  every tile is ordered by bucket in LDS and written back as one
//              piece, with a table of where each bucket starts in it: nothing
//              has to be counted first, and no partial cache lines are written.
//              A further level gathers its keys from the pieces the one before
//              left, for which "pieces" counts the keys before every 8 tiles
//   scan       where the buckets start; they become leaves (fit one workgroup,
//              or hold one key value only), nodes of the next level, or - if the
//              last level left one too large - big buckets
//
// and a leaf is sorted by one workgroup, which gathers it from its piece of
// every tile of the node.  The last two levels leave their tiles in place;
// before them, and for arrays too short to gather (kDistGatherMin), a level is
//
//   count      keys per bucket of every range
//   scatter    the same ranges, tile by tile: a tile is ordered by bucket in LDS
//              and leaves in runs of consecutive addresses, each bucket's at its
//              own place
//
// Samples are taken at hashed positions, so the order of the input does not
// matter, and any distribution of keys gives buckets of about the same size.
// Nothing depends on the sizes being met: a bucket left too large is sorted by
// all workgroups together, merging through memory.
//
// At 2^28 int64 uniform keys (ms): samples 0.21, first partition 0.85, gathered
// partition 1.26, leaves 1.43; the sort 3.72.  With a count (0.44) and a
// scatter (1.48) in place of the first partition, and 0.89 for a partition that
// need not gather, it took 4.50, and the merge plan's tile sort (1.71) and three
// merge passes (1.88 each with their searches) 7.31.  A piece is 24 keys of 8
// bytes there, at any multiple of 8, so that a gather reads 1.7 times its bytes
// in cache lines; a scatter writes as many partial lines, to 256 places at once.
//
// Key-value sorts place equal keys in input order at every step (the ranges
// are in order, and a tile's ranks follow it), keys-only sorts need not:
// equal keys are bit-identical.
#include "pss_device.hpp"
#include "pss_dist.hpp"

namespace pss {
namespace {

constexpr uint32_t kLutBins = 1024;
constexpr uint32_t kXcds = 8;
constexpr uint32_t kGang = 4;  // neighbouring nodes gathered on one XCD

// Arguments of one level's kernels.
struct Level {
  DistCounters *ctr;
  DistNode *nodes, *next_nodes;
  DistRange *ranges, *next_ranges;
  void *spl;
  uint32_t *start;
  void *table;
  DistLeaf *leaves;
  uint32_t *rest;  // leaves with a crowded bin
  DistBig *big;
  uint32_t level, levels, cap, target, rl, next_rl;
  uint32_t src;  // kSrc* of this level's leaves
  uint32_t node_tiles;  // most tiles of a last-level node
  uint32_t max_next_nodes, max_next_ranges, max_cols, max_next_table, max_leaves, max_rest, max_big;
  uint32_t root_len, root_p;  // level 1 of a single array (0: nodes are given)
  uint32_t tiled, next_tiled;  // its tiles are left in place
  uint32_t gather;  // its keys are gathered from the tiles of the level before
  uint32_t kv, max_copies;
  const uint16_t *ptable;  // gathered: the table of the level before,
  uint32_t *pre;           // and per bucket the keys before every 8 tiles
  uint32_t *err;  // device error word (kernels that report only)
};

// A bound of the plan does not hold: what would lie past it is not written, the
// error word is set, and every later kernel of the sort returns at once (it
// would meet nodes, ranges or leaves that were never written).
__device__ __forceinline__ void plan_failed(DistCounters *ctr, uint32_t *err) {
  atomicOr(&ctr->failed, 1u);
  atomicOr(err, kErrPlan);
}

// Inclusive sum over the wave's lanes, in DPP moves: shifts by 1, 2, 4 and 8
// lanes within rows of 16, then the last lane of row 0 to row 1 and of row 2
// to row 3, then that of row 1 to rows 2 and 3.
__device__ __forceinline__ uint32_t wave_sum_scan(uint32_t x) {
  int y = (int)x;
  y += __builtin_amdgcn_update_dpp(0, y, 0x111, 0xF, 0xF, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x112, 0xF, 0xF, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x114, 0xF, 0xF, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x118, 0xF, 0xF, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x142, 0xA, 0xF, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x143, 0xC, 0xF, false);
  return (uint32_t)y;
}

// Exclusive sum over the workgroup's threads; `wsum` needs NT / 64 entries and
// may be used again after the next barrier.
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *wsum, uint32_t &total) {
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t x = wave_sum_scan(v);
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (uint32_t w = 0; w < NT / 64; ++w) {
    const uint32_t c = wsum[w];
    before += w < wid ? c : 0u;
    total += c;
  }
  return before + x - v;
}

// ------------------------------------------------------------ gathering ---
// A gathered node's keys lie in its parent's tiles: eight tiles' pieces of
// them, as starts (s) and ends (e) in the tiles.
__device__ __forceinline__ uint32_t parent_tiles(const DistNode &nd) {
  return (nd.plen + kDistTile - 1) / kDistTile;
}

// The bucket's piece of tile t (row, next: the table's rows of the bucket and
// the next one) of a node of len keys.
__device__ __forceinline__ void piece_of(const uint16_t *table, uint32_t row, uint32_t next,
                                         uint32_t len, uint32_t t, uint32_t &s, uint32_t &e) {
  s = e = 0;
  if (t * kDistTile < len) {
    const uint32_t rem = len - t * kDistTile, whole = rem < kDistTile ? rem : kDistTile;
    s = table[row + t];
    e = next != ~0u ? table[next + t] : whole;
  }
}

// The pieces of tiles t .. t+7 (t a multiple of 8); empty past the last tile.
__device__ __forceinline__ void pieces_of_8(const uint16_t *table, uint32_t row, uint32_t next,
                                            uint32_t len, uint32_t t, uint32_t (&s)[8],
                                            uint32_t (&e)[8]) {
  const uint4 a = *reinterpret_cast<const uint4 *>(table + row + t);
  const uint4 z = *reinterpret_cast<const uint4 *>(table + (next != ~0u ? next : row) + t);
  const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
  for (uint32_t q = 0; q < 8; ++q) {
    const uint32_t at = (t + q) * kDistTile, rem = len > at ? len - at : 0u;
    const uint32_t whole = rem < kDistTile ? rem : kDistTile;
    s[q] = (x[q >> 1] >> (16 * (q & 1))) & 0xffffu;
    e[q] = next != ~0u ? (y[q >> 1] >> (16 * (q & 1))) & 0xffffu : whole;
    s[q] = rem ? s[q] : 0u;
    e[q] = rem ? e[q] : 0u;
  }
}

// Turns positions of a gathered node into addresses in the level's source; pre:
// the keys before each group of 8 tiles.
template <int N>
__device__ __forceinline__ void gathered_from(const Level &L, const DistNode &nd, uint32_t (&at)[N],
                                              const uint32_t *pre, uint32_t groups) {
  uint32_t g[N];  // the last group of 8 tiles whose keys start at or before the position
#pragma unroll
  for (int i = 0; i < N; ++i) g[i] = 0;
  for (uint32_t step = 1u << (31 - __clz(groups)); step; step >>= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t to = g[i] + step < groups ? g[i] + step : g[i];
      g[i] = pre[to] <= at[i] ? to : g[i];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    uint32_t s[8], e[8], rem = at[i] - pre[g[i]], where = 0;
    pieces_of_8(L.ptable, nd.prow, nd.pnext, nd.plen, g[i] * 8, s, e);
    bool found = false;
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) {
      const uint32_t c = e[q] - s[q];
      const bool here = !found && rem < c;
      where = here ? nd.poff + (g[i] * 8 + q) * kDistTile + s[q] + rem : where;
      found |= here;
      rem -= found ? 0u : c;
    }
    at[i] = where;
  }
}

// The same.  A thread's positions rise with the thread, so that a wave's lookups
// share cache lines; `lds` (`room` entries) takes the groups' starts if they
// fit, as every step of the search waits for the one before it.
template <int N>
__device__ __forceinline__ void gathered_at(const Level &L, const DistNode &nd, uint32_t (&at)[N],
                                            uint32_t *lds, uint32_t room) {
  const uint32_t groups = (parent_tiles(nd) + 7) / 8;
  const uint32_t *pre = L.pre + nd.prow / 8;
  if (groups <= room) {
    for (uint32_t i = threadIdx.x; i < groups; i += blockDim.x) lds[i] = pre[i];
    __syncthreads();
    gathered_from(L, nd, at, lds, groups);
    __syncthreads();
  } else {
    gathered_from(L, nd, at, pre, groups);
  }
}

// After a partition that is not the last level's: a bucket's keys before every
// eight tiles, and in all.  One workgroup a bucket (few nodes), or several
// buckets each.
constexpr int kPiecesThreads = 512;

__global__ __launch_bounds__(kPiecesThreads) void dist_pieces_kernel(Level L) {
  __shared__ uint32_t wsum[kPiecesThreads / 64];
  const uint32_t tid = threadIdx.x;
  if (blockIdx.x >= L.ctr->nodes[L.level] || L.ctr->failed) return;
  const DistNode nd = L.nodes[blockIdx.x];
  const uint32_t tiles = (nd.len + kDistTile - 1) / kDistTile;
  for (uint32_t b = blockIdx.y; b < nd.nb; b += gridDim.y) {
    const uint32_t row = nd.tbase + b * nd.stride;
    uint32_t run = 0;
    for (uint32_t t0 = 0; t0 < tiles; t0 += kPiecesThreads * 8) {
      const uint32_t t = t0 + tid * 8;
      uint32_t c = 0;
      if (t < tiles) {
        uint32_t s[8], e[8];
        pieces_of_8(L.ptable, row, b + 1 < nd.nb ? row + nd.stride : ~0u, nd.len, t, s, e);
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) c += e[q] - s[q];
      }
      uint32_t total;
      const uint32_t x = block_scan<kPiecesThreads>(c, wsum, total);
      if (t < tiles) L.pre[(row + t) / 8] = run + x;
      run += total;
      __syncthreads();
    }
    if (tid == 0) L.start[nd.sbase + b] = run;
  }
}

// ------------------------------------------------------------- segments ---
// Segmented distribution sort: one workgroup reads the segment offsets, checks
// them, and lists every segment of more than `merged` and at most `longest` keys
// as a node of the first level.  Invalid offsets (not starting at 0, decreasing,
// or ending beyond n) give no nodes and an error bit.
struct SegDistArgs {
  const uint64_t *off;
  uint32_t n_segs;
  uint64_t n, merged, longest;
  uint32_t target, rl, root_p, one_p, levels, tiled;
  DistCounters *ctr;
  DistNode *nodes;
  DistRange *ranges;
  uint32_t max_nodes, max_ranges, max_cols, max_table;
  uint32_t *err;  // device error word
};

__global__ __launch_bounds__(1024) void seg_dist_plan_kernel(SegDistArgs a) {
  __shared__ uint32_t bad, n_nodes, n_ranges, n_cols, n_table;
  const uint32_t tid = threadIdx.x;
  uint32_t *c = (uint32_t *)a.ctr;
  for (uint32_t i = tid; i < sizeof(DistCounters) / 4; i += 1024) c[i] = 0;
  if (tid == 0) {
    bad = (a.off[0] != 0 || a.off[a.n_segs] > a.n) ? 1u : 0u;
    n_nodes = n_ranges = n_cols = n_table = 0;
  }
  __syncthreads();
  for (uint32_t s = tid; s < a.n_segs; s += 1024)
    if (a.off[s + 1] < a.off[s]) atomicOr(&bad, 1u);
  __syncthreads();
  const bool ok = bad == 0;
  if (tid == 0 && !ok) atomicOr(a.err, kErrSegments);
  if (!ok) return;
  for (uint32_t s = tid; s < a.n_segs; s += 1024) {
    const uint64_t len64 = a.off[s + 1] - a.off[s];
    if (len64 <= a.merged || len64 > a.longest) continue;
    const uint32_t len = (uint32_t)len64;
    DistNode d;
    d.off = (uint32_t)a.off[s];
    d.len = len;
    const bool one = len <= a.one_p * a.target;
    d.p = node_picks(len, a.target, one ? 1 : (int)a.levels);
    d.p = one || d.p < a.root_p ? d.p : a.root_p;
    d.nr = (len + a.rl - 1) / a.rl;
    d.cols = node_cols(d.p);
    d.stride = node_stride(len, d.nr, a.tiled != 0);
    d.nb = 0;
    d.poff = d.plen = d.prow = d.pnext = 0;
    const uint32_t at = atomicAdd(&n_nodes, 1u), r0 = atomicAdd(&n_ranges, d.nr);
    d.sbase = atomicAdd(&n_cols, d.cols);
    d.tbase = atomicAdd(&n_table, d.cols * d.stride);
    if (at < a.max_nodes && r0 + d.nr <= a.max_ranges && d.sbase + d.cols <= a.max_cols &&
        d.tbase + d.cols * d.stride <= a.max_table) {
      a.nodes[at] = d;
      for (uint32_t r = 0; r < d.nr; ++r) a.ranges[r0 + r] = DistRange{at, r};
    } else {
      plan_failed(a.ctr, a.err);
    }
  }
  __syncthreads();
  if (tid == 0) {
    a.ctr->nodes[1] = n_nodes;
    a.ctr->ranges[1] = n_ranges;
    a.ctr->cols[1] = n_cols;
    a.ctr->table[1] = n_table;
  }
}

// ------------------------------------------------------------- sampling ---
// One workgroup per node; latency-bound (a few random loads a thread, then
// one LDS sort).  The picks come from S sorted samples, S a power of two of at
// least 20 per bucket, at most one tile.
template <int KT, int NT>
__global__ __launch_bounds__(NT) void dist_sample_kernel(const typename Key<KT>::U *__restrict__ src,
                                                         Level L, uint32_t p_lo, uint32_t p_hi) {
  using U = typename Key<KT>::U;
  constexpr uint32_t TILE = NT * kTileItems;
  __shared__ U sk[TileLds<false, NT>::SLOTS];
  __shared__ uint32_t wsum[NT / 64];
  const uint32_t tid = threadIdx.x;
  DistNode nd;
  if (L.root_len) {
    nd.off = 0;
    nd.len = L.root_len;
    nd.p = L.root_p;
    nd.nr = (nd.len + L.rl - 1) / L.rl;
    nd.cols = node_cols(nd.p);
    nd.sbase = 0;
    nd.tbase = 0;
    nd.stride = node_stride(nd.len, nd.nr, L.tiled != 0);
    nd.poff = nd.plen = nd.prow = nd.pnext = 0;
    uint32_t *c = (uint32_t *)L.ctr;
    for (uint32_t i = tid; i < sizeof(DistCounters) / 4; i += NT) c[i] = 0;
    for (uint32_t r = tid; r < nd.nr; r += NT) L.ranges[r] = DistRange{0u, r};
    __syncthreads();
    if (tid == 0) {
      L.ctr->nodes[1] = 1;
      L.ctr->ranges[1] = nd.nr;
    }
  } else {
    if (blockIdx.x >= L.ctr->nodes[L.level] || L.ctr->failed) return;
    nd = L.nodes[blockIdx.x];
    if (nd.p < p_lo || nd.p > p_hi) return;  // another tile size samples it
  }
  uint32_t want = 64 * nd.p < TILE ? 64 * nd.p : TILE;
  want = nd.len / 2 < want ? nd.len / 2 : want;
  const uint32_t lg = 31 - __clz(want), S = 1u << lg;
  U rk[kTileItems];
  uint32_t at[kTileItems];
#pragma unroll
  for (int i = 0; i < kTileItems; ++i) {
    const uint32_t j = i * NT + tid;
    uint32_t h = (j + 1) * 0x9E3779B1u ^ (nd.off + L.level) * 0x85EBCA6Bu;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    h *= 0x297A2D39u;
    h ^= h >> 15;
    // a hashed position of the j-th of S equal strata
    const uint64_t pos = ((uint64_t)j * nd.len + (((uint64_t)h * nd.len) >> 32)) >> lg;
    at[i] = j < S ? (uint32_t)pos : 0u;
  }
  if (L.gather) gathered_at(L, nd, at, reinterpret_cast<uint32_t *>(sk), (uint32_t)(sizeof(sk) / 4));
#pragma unroll
  for (int i = 0; i < kTileItems; ++i) {
    const U x = src[L.gather ? at[i] : nd.off + at[i]];
    rk[i] = i * NT + tid < S ? Key<KT>::map(x) : key_max<U>();
  }
  lds_sort_keys<U, NT>(rk, sk);
  // splitters of p picks; when frequent keys double them beyond the slots, those
  // of as many picks as fit doubled.  (Half the picks, 186 of 372 with 4 to 6 of
  // 1000 values between two, left 20 to 40 buckets above the cap: 1500000 int64 of
  // 1000 values 170 us, now 128; 48 segments of 4.6*10^6 u64 with values 464, now 363.)
  U *spl = (U *)L.spl + nd.sbase;
  uint32_t ns = 0;
  for (uint32_t p = nd.p;; p = nd.cols / 2) {
    const uint32_t last_pick = p - 2;  // picks 0 .. p-2
    U v = 0;
    uint32_t e = 0;
    bool first = false, next = false;
    if (tid <= last_pick) {
      const uint32_t at = (tid + 1) * S / p;
      v = sk[at];
      const U before = tid > 0 ? sk[tid * S / p] : U(0);
      const U after = tid < last_pick ? sk[(tid + 2) * S / p] : U(0);
      first = tid == 0 || before != v;
      const bool last = tid == last_pick || after != v;
      const bool dup = !(first && last) || (at > 0 && sk[at - 1] == v) ||
                       (at + 1 < S && sk[at + 1] == v);
      next = last && dup && v != key_max<U>() && !(tid < last_pick && after == v + 1);
      e = (first ? 1u : 0u) + (next ? 1u : 0u);
    }
    uint32_t total;
    const uint32_t to = block_scan<NT>(e, wsum, total);
    if (total < nd.cols) {  // (2 (p - 1) at most)
      if (first) spl[to] = v;
      if (next) spl[to + (first ? 1u : 0u)] = v + 1;
      ns = total;
      break;
    }
    __syncthreads();
  }
  if (tid == 0) {
    nd.nb = ns + 1;
    L.nodes[blockIdx.x] = nd;
  }
}

// ------------------------------------------------------- classification ---
// Bucket of a key: the number of splitters <= it.  A table over 1024 equal
// steps of the splitters' span gives the candidates of a key's step (none or
// one for keys spread evenly), a binary search the rest.
template <typename U> struct Classifier {
  U spl[kDistSlots + 1];
  uint32_t lut[kLutBins];  // splitters below the step | those up to its end << 16
};

template <typename U> struct ClassifierRegs {
  U first;
  uint32_t shift;
};

template <typename U>
__device__ __forceinline__ ClassifierRegs<U> classifier_load(Classifier<U> &c, const U *g,
                                                             uint32_t ns) {
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i <= kDistSlots; i += blockDim.x) c.spl[i] = i < ns ? g[i] : key_max<U>();
  __syncthreads();
  ClassifierRegs<U> r;
  r.first = c.spl[0];
  const uint64_t span = (uint64_t)(c.spl[ns - 1] - r.first);
  const int bits = span ? 64 - __clzll((long long)span) : 0;
  r.shift = bits > 10 ? (uint32_t)(bits - 10) : 0u;
  auto below = [&](uint32_t x) {  // splitters in steps before x
    uint32_t lo = 0, hi = ns;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if ((uint64_t)((c.spl[mid] - r.first) >> r.shift) < x) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  for (uint32_t x = tid; x < kLutBins; x += blockDim.x)
    c.lut[x] = below(x) | (x + 1 < kLutBins ? below(x + 1) : ns) << 16;
  __syncthreads();
  return r;
}

template <typename U, int N>
__device__ __forceinline__ void classify(const Classifier<U> &c, const ClassifierRegs<U> &r,
                                         const U (&k)[N], uint32_t (&b)[N]) {
  uint32_t hi[N];
  bool more = false;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const U d = k[i] - r.first;
    const U s = d >> r.shift;
    const uint32_t x = s < (U)(kLutBins - 1) ? (uint32_t)s : kLutBins - 1;
    const uint32_t e = c.lut[x];
    const bool under = k[i] < r.first;
    b[i] = under ? 0u : e & 0xffffu;
    hi[i] = under ? 0u : e >> 16;
    more |= b[i] < hi[i];
  }
  while (__any(more)) {
    more = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t mid = (b[i] + hi[i]) >> 1;
      const bool act = b[i] < hi[i], le = c.spl[mid] <= k[i];
      b[i] = act && le ? mid + 1 : b[i];
      hi[i] = act && !le ? mid : hi[i];
      more |= b[i] < hi[i];
    }
  }
}

// ---------------------------------------------------------------- count ---
// One workgroup per range: reads every key once (HBM-bound).
constexpr int kCountItems = 8;

template <int KT>
__global__ __launch_bounds__(kDistThreads) void dist_count_kernel(
    const typename Key<KT>::U *__restrict__ src, Level L) {
  using U = typename Key<KT>::U;
  __shared__ Classifier<U> cl;
  __shared__ uint32_t hist[kDistSlots];
  const uint32_t tid = threadIdx.x;
  if (blockIdx.x >= L.ctr->ranges[L.level] || L.ctr->failed) return;
  const DistRange rg = L.ranges[blockIdx.x];
  const DistNode nd = L.nodes[rg.node];
  for (uint32_t i = tid; i < kDistSlots; i += kDistThreads) hist[i] = 0;
  const ClassifierRegs<U> cr = classifier_load(cl, (const U *)L.spl + nd.sbase, nd.nb - 1);
  const uint32_t end = rg.r * L.rl + L.rl < nd.len ? rg.r * L.rl + L.rl : nd.len;
  const U *p = src + nd.off;
  for (uint32_t base = rg.r * L.rl; base < end; base += kDistThreads * kCountItems) {
    U k[kCountItems];
    uint32_t b[kCountItems];
#pragma unroll
    for (int i = 0; i < kCountItems; ++i) {
      const uint32_t idx = base + i * kDistThreads + tid;
      k[i] = p[idx < end ? idx : end - 1];
    }
#pragma unroll
    for (int i = 0; i < kCountItems; ++i) k[i] = Key<KT>::map(k[i]);
    classify(cl, cr, k, b);
#pragma unroll
    for (int i = 0; i < kCountItems; ++i) {
      const bool ok = base + i * kDistThreads + tid < end;
      // one bucket for the whole wave (ordered input): one addition, not 64
      // to the same address
      const uint32_t b0 = __builtin_amdgcn_readfirstlane(b[i]);
      if (__all(ok && b[i] == b0)) {
        if ((tid & 63) == 0) atomicAdd(&hist[b0], 64u);
      } else if (ok) {
        atomicAdd(&hist[b[i]], 1u);
      }
    }
  }
  __syncthreads();
  uint32_t *table = (uint32_t *)L.table + nd.tbase;
  for (uint32_t b = tid; b < nd.nb; b += kDistThreads) table[b * nd.stride + rg.r] = hist[b];
}

// ----------------------------------------------------------------- scan ---
// One wave per bucket of the root node, whose hundreds of ranges are too many
// for one thread: exclusive sums over the ranges in place, the total to start.
__global__ __launch_bounds__(256) void dist_columns_kernel(Level L) {
  if (L.ctr->failed) return;
  const DistNode nd = L.nodes[0];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t b = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= nd.nb) return;
  uint32_t *col = (uint32_t *)L.table + nd.tbase + b * nd.stride;
  uint32_t run = 0;
  for (uint32_t r0 = 0; r0 < nd.nr; r0 += 64) {
    const uint32_t r = r0 + lane;
    const uint32_t v = r < nd.nr ? col[r] : 0u;
    const uint32_t x = wave_sum_scan(v);
    if (r < nd.nr) col[r] = run + x - v;
    run += __shfl(x, 63, 64);
  }
  if (lane == 0) L.start[nd.sbase + b] = run;
}

// One workgroup per node, one thread per bucket.  Last level: a bucket's start
// is the sum of its starts in the node's tiles.
template <typename U>
__global__ __launch_bounds__(kDistSlots) void dist_scan_kernel(Level L, int summed) {
  __shared__ uint32_t wsum[kDistSlots / 64], wsum2[kDistSlots / 64];
  __shared__ uint32_t starts[kDistSlots + 1];
  __shared__ uint32_t leaf0;
  const uint32_t b = threadIdx.x;
  if (blockIdx.x >= L.ctr->nodes[L.level]) return;
  // (other workgroups of this launch may set the flag: one answer for all waves)
  if (__syncthreads_or(L.ctr->failed != 0)) return;
  const DistNode nd = L.nodes[blockIdx.x];
  const bool last = L.level == L.levels;
  uint32_t len = 0, off = nd.off;
  if (last) {
    if (b < nd.nb) {
      const uint16_t *col = (const uint16_t *)L.table + nd.tbase + b * nd.stride;
      const uint32_t tiles = (nd.len + kDistTile - 1) / kDistTile;
      for (uint32_t t = 0; t < tiles; t += 32) {  // entries past the tiles count nothing
        // (loaded together: the scan of 163 tiles takes 7.8 us, one at a time 9.1)
        uint4 q[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
          q[u] = t + 8 * u < tiles ? *reinterpret_cast<const uint4 *>(col + t + 8 * u) : uint4{};
#pragma unroll
        for (uint32_t i = 0; i < 32; ++i) {
          const uint4 &v = q[i >> 3];
          const uint32_t wd = (i & 6) == 0 ? v.x : (i & 6) == 2 ? v.y : (i & 6) == 4 ? v.z : v.w;
          off += t + i < tiles ? (wd >> (16 * (i & 1))) & 0xffffu : 0u;
        }
      }
      starts[b] = off;
    }
    if (b == 0) starts[nd.nb] = nd.off + nd.len;
    __syncthreads();
    if (b < nd.nb) len = starts[b + 1] - off;
  } else {
    if (b < nd.nb) {
      if (summed) {
        len = L.start[nd.sbase + b];
      } else {
        uint32_t *col = (uint32_t *)L.table + nd.tbase + b * nd.stride;
        for (uint32_t r0 = 0; r0 < nd.nr; r0 += 8) {
          uint32_t v[8];
#pragma unroll
          for (uint32_t i = 0; i < 8; ++i) v[i] = r0 + i < nd.nr ? col[r0 + i] : 0u;
#pragma unroll
          for (uint32_t i = 0; i < 8; ++i) {
            if (r0 + i < nd.nr) col[r0 + i] = len;
            len += v[i];
          }
        }
      }
    }
    uint32_t total;
    off = nd.off + block_scan<kDistSlots>(len, wsum, total);
    if (b < nd.nb) L.start[nd.sbase + b] = off;
  }
  const uint32_t ns = nd.nb - 1;
  const bool next_last = L.level + 1 == L.levels;
  bool equal = false;  // the bucket can hold one key value only
  bool node = false, big = false, copy = false, known = false;
  uint32_t pieces = 0;
  U lo = 0, hi = 0;
  if (b < nd.nb && len) {
    const U *spl = (const U *)L.spl + nd.sbase;
    lo = b > 0 ? spl[b - 1] : U(0);
    hi = b < ns ? spl[b] : U(0);
    equal = b < ns ? hi - lo == 1 : lo == key_max<U>();
    const bool fits = len <= L.cap;
    node = !last && !equal && !fits && !(next_last && len > L.node_tiles * kDistTile);
    big = !equal && !fits && !node;
    // (after a scatter a big bucket already lies in the output)
    pieces = node || (big && !L.tiled) ? 0u : (len + L.cap - 1) / L.cap;
    // in place before the last level: the last level's workgroups bring it to
    // its place in the workspace (keys of one value need not be read)
    known = equal && !L.kv;
    copy = L.tiled && !last && !node && !known;
  }
  uint32_t npieces;
  const uint32_t at = block_scan<kDistSlots>(pieces, wsum2, npieces);
  if (b == 0) leaf0 = npieces ? atomicAdd(&L.ctr->leaves, npieces) : 0u;
  __syncthreads();
  for (uint32_t q = 0; q < pieces; ++q) {
    const uint32_t o = q * L.cap, l = len - o < L.cap ? len - o : L.cap;
    const uint32_t to = leaf0 + at + q;
    if (to < L.max_leaves) {
      const uint32_t row = nd.tbase + b * nd.stride;
      L.leaves[to] = DistLeaf{off + o,
                              l | (copy ? kSrcWs : L.tiled ? kSrcPieces : L.src) << kLeafSrcShift | (equal ? kLeafEqual : 0u) |
                                  (big ? kLeafMove : 0u) | (b > 0 && b < ns ? kLeafInner : 0u),
                              nd.off, nd.len, o, row, b < ns ? row + nd.stride : ~0u, 0u, (uint64_t)lo,
                              (uint64_t)hi};
    } else {
      plan_failed(L.ctr, L.err);
    }
  }
  if (big) {
    const uint32_t to = atomicAdd(&L.ctr->big, 1u);
    if (to < L.max_big) L.big[to] = DistBig{off, len, 0u, 0u};
    else plan_failed(L.ctr, L.err);
  }
  if (node) {
    DistNode c;
    c.off = off;
    c.len = len;
    c.p = node_picks(len, L.target, (int)(L.levels - L.level));
    c.nr = (len + L.next_rl - 1) / L.next_rl;
    c.cols = node_cols(c.p);
    c.stride = node_stride(len, c.nr, L.next_tiled != 0);
    c.nb = 0;
    c.poff = nd.off;
    c.plen = nd.len;
    c.prow = nd.tbase + b * nd.stride;
    c.pnext = b < ns ? c.prow + nd.stride : ~0u;
    const uint32_t lv = L.level + 1;
    const uint32_t at_node = atomicAdd(&L.ctr->nodes[lv], 1u);
    // (a gathered level takes its nodes' ranges in turn, without a list)
    const bool list = !L.tiled;
    const uint32_t at_range = list ? atomicAdd(&L.ctr->ranges[lv], c.nr) : 0u;
    if (!list) atomicMax(&L.ctr->most_ranges, c.nr);
    c.sbase = atomicAdd(&L.ctr->cols[lv], c.cols);
    c.tbase = atomicAdd(&L.ctr->table[lv], c.cols * c.stride);
    // (the plan's bounds hold for any lengths)
    if (at_node < L.max_next_nodes && (!list || at_range + c.nr <= L.max_next_ranges) &&
        c.sbase + c.cols <= L.max_cols && c.tbase + c.cols * c.stride <= L.max_next_table) {
      L.next_nodes[at_node] = c;
      for (uint32_t r = 0; list && r < c.nr; ++r) L.next_ranges[at_range + r] = DistRange{at_node, r};
    } else {
      plan_failed(L.ctr, L.err);
    }
  }
  if (copy) {  // a node without splitters, listed after the others
    DistNode c{};
    c.off = off;
    c.len = len;
    c.nr = (len + L.next_rl - 1) / L.next_rl;
    c.nb = 1;
    c.poff = nd.off;
    c.plen = nd.len;
    c.prow = nd.tbase + b * nd.stride;
    c.pnext = b < ns ? c.prow + nd.stride : ~0u;
    const uint32_t at_copy = atomicAdd(&L.ctr->copies, 1u);
    const uint32_t at_range = atomicAdd(&L.ctr->ranges[L.level + 1], c.nr);
    if (at_copy < L.max_copies && at_range + c.nr <= L.max_next_ranges) {
      L.next_nodes[L.max_next_nodes + at_copy] = c;
      for (uint32_t r = 0; r < c.nr; ++r)
        L.next_ranges[at_range + r] = DistRange{L.max_next_nodes + at_copy, r};
    } else {
      plan_failed(L.ctr, L.err);
    }
  }
}

// ----------------------------------------------------------- tile ranks ---
// Position in its tile of a thread's i-th key.  Key-value: a wave's keys are
// consecutive, row by row, as the ranks follow that order.
template <bool KV> __device__ __forceinline__ uint32_t tile_at(int i) {
  const uint32_t tid = threadIdx.x;
  return KV ? (tid >> 6) * (64 * kDistItems) + i * 64 + (tid & 63) : i * kDistThreads + tid;
}

// Ranks of a tile's keys within their buckets: pos[i] gets the key's rank
// (key-value: among its wave's keys of the bucket; wh then holds how many keys
// of the bucket earlier waves have).  Returns the tile's keys of bucket tid.
template <bool KV>
__device__ __forceinline__ uint32_t tile_ranks(const uint32_t (&b)[kDistItems],
                                               uint32_t (&pos)[kDistItems], uint32_t count,
                                               uint32_t nbits, uint16_t *wh, uint32_t *hist) {
  constexpr int NT = kDistThreads, NI = kDistItems, NW = NT / 64;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if constexpr (KV) {
    for (uint32_t i = tid; i < NW * kDistSlots / 2; i += NT) reinterpret_cast<uint32_t *>(wh)[i] = 0;
    __syncthreads();
    uint16_t *my = wh + wid * kDistSlots;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bool ok = tile_at<KV>(i) < count;
      uint64_t peers = __ballot(ok);
      for (uint32_t bit = 0; bit < nbits; ++bit) {
        const bool one = (b[i] >> bit) & 1u;
        const uint64_t m = __ballot(one);
        peers &= one ? m : ~m;
      }
      const uint32_t below = __popcll(peers & (((uint64_t)1 << lane) - 1));
      const uint32_t seen = my[b[i]];
      wave_sync();
      if (ok && below == 0) my[b[i]] = (uint16_t)(seen + __popcll(peers));
      wave_sync();
      pos[i] = seen + below;
    }
    __syncthreads();
    uint32_t mine = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint32_t c = wh[w * kDistSlots + tid];
      wh[w * kDistSlots + tid] = (uint16_t)mine;
      mine += c;
    }
    return mine;
  } else {
    hist[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bool ok = tile_at<KV>(i) < count;
      // one bucket for the whole wave (ordered input): one addition
      const uint32_t b0 = __builtin_amdgcn_readfirstlane(b[i]);
      if (__all(ok && b[i] == b0)) {
        uint32_t r = 0;
        if (lane == 0) r = atomicAdd(&hist[b0], 64u);
        pos[i] = __builtin_amdgcn_readfirstlane(r) + lane;
      } else if (ok) {
        pos[i] = atomicAdd(&hist[b[i]], 1u);
      }
    }
    __syncthreads();
    return hist[tid];
  }
}

// -------------------------------------------------------------- scatter ---
// One workgroup per range, tile by tile in order.  A tile's keys are placed
// in LDS in bucket order, so that a bucket's share of the tile (24 keys at 256
// buckets) leaves as one run of addresses; the next tile continues the same
// runs, and L2 joins the lines they share.  76 KB of LDS: two workgroups a CU.
template <int KT, bool KV>
__global__ __launch_bounds__(kDistThreads, 4) void dist_scatter_kernel(
    const typename Key<KT>::U *__restrict__ src, const uint32_t *__restrict__ vsrc,
    typename Key<KT>::U *__restrict__ dst, uint32_t *__restrict__ vdst, Level L) {
  using U = typename Key<KT>::U;
  constexpr int NT = kDistThreads, NI = kDistItems, NW = NT / 64;
  __shared__ Classifier<U> cl;
  __shared__ U sk[kDistTile];
  __shared__ uint16_t sb[kDistTile];
  __shared__ uint32_t hist[kDistSlots], lofs[kDistSlots], gofs[kDistSlots], wsum[NW];
  // key-value: per-wave bucket counts, dead before the keys are placed
  uint16_t *wh = reinterpret_cast<uint16_t *>(sk);
  static_assert(NW * kDistSlots * 2 <= sizeof(sk), "wave counts fit the key area");
  static_assert(NT == (int)kDistSlots, "one thread per bucket");
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (blockIdx.x >= L.ctr->ranges[L.level] || L.ctr->failed) return;
  const DistRange rg = L.ranges[blockIdx.x];
  const DistNode nd = L.nodes[rg.node];
  const ClassifierRegs<U> cr = classifier_load(cl, (const U *)L.spl + nd.sbase, nd.nb - 1);
  uint32_t cursor = 0;
  if (tid < nd.nb)
    cursor = L.start[nd.sbase + tid] + ((const uint32_t *)L.table)[nd.tbase + tid * nd.stride + rg.r];
  const uint32_t end = rg.r * L.rl + L.rl < nd.len ? rg.r * L.rl + L.rl : nd.len;
  const U *p = src + nd.off;
  const uint32_t *vp = KV ? vsrc + nd.off : nullptr;
  const uint32_t nbits = 32 - __clz(nd.nb - 1);
  for (uint32_t base = rg.r * L.rl; base < end; base += kDistTile) {
    const uint32_t count = end - base < kDistTile ? end - base : kDistTile;
    U k[NI];
    uint32_t v[KV ? NI : 1], b[NI], pos[NI];
    auto at = [](int i) { return tile_at<KV>(i); };
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t j = at(i) < count ? at(i) : count - 1;
      k[i] = __builtin_nontemporal_load(&p[base + j]);
      if constexpr (KV) v[i] = __builtin_nontemporal_load(&vp[base + j]);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) k[i] = Key<KT>::map(k[i]);
    classify(cl, cr, k, b);
    const uint32_t mine = tile_ranks<KV>(b, pos, count, nbits, wh, hist);
    uint32_t total;
    const uint32_t lo = block_scan<NT>(mine, wsum, total);
    lofs[tid] = lo;
    gofs[tid] = cursor - lo;  // modulo 2^32: the sum below is in range
    cursor += mine;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      pos[i] += lofs[b[i]];
      if constexpr (KV) pos[i] += wh[wid * kDistSlots + b[i]];
    }
    if constexpr (KV) __syncthreads();  // wh is read before the keys overwrite it
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (at(i) < count) {
        sk[pos[i]] = k[i];
        sb[pos[i]] = (uint16_t)b[i];
      }
    }
    __syncthreads();
    uint32_t to[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t j = i * NT + tid;
      if (j < count) {
        to[i] = gofs[sb[j]] + j;
        dst[to[i]] = sk[j];
      }
    }
    if constexpr (KV) {
      __syncthreads();
      uint32_t *sv = reinterpret_cast<uint32_t *>(sk);
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (at(i) < count) sv[pos[i]] = v[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t j = i * NT + tid;
        if (j < count) vdst[to[i]] = sv[j];
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ partition ---
// One workgroup per range; every tile is ordered by bucket in LDS and written
// to its own place in the level's output, so stores are whole lines
// and nothing has to be counted first.  The starts of the buckets in the
// range's tiles are collected in LDS and leave as one short run per bucket.
//
// GATHER: the level's keys are gathered from the tiles of the level before,
// which takes the place of counting and scattering them there.  As in
// the leaves, the pieces of a tile are listed and a bit mask tells every
// position its piece.  A node without splitters is only brought to its place.
template <int KT, bool KV, bool GATHER>
__global__ __launch_bounds__(kDistThreads, 4) void dist_partition_kernel(
    const typename Key<KT>::U *__restrict__ src, const uint32_t *__restrict__ vsrc,
    typename Key<KT>::U *__restrict__ dst, uint32_t *__restrict__ vdst, Level L) {
  using U = typename Key<KT>::U;
  constexpr int NT = kDistThreads, NI = kDistItems, NW = NT / 64;
  __shared__ Classifier<U> cl;
  // (gathered: a tile may list the pieces of up to 8 tiles before its first)
  __shared__ U sk[kDistTile + (GATHER ? 16 : 0)];
  __shared__ uint32_t hist[kDistSlots], lofs[kDistSlots], wsum[NW];
  __shared__ uint16_t rows[kDistRangeTiles][kDistSlots];
  // key-value: per-wave bucket counts, dead before the keys are placed
  uint16_t *wh = reinterpret_cast<uint16_t *>(sk);
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t nranges = L.ctr->ranges[L.level];
  if (L.ctr->failed) return;
  // gathered: the next tile's first key is key cur_key of its node or later,
  // the first of the piece of the parent's tile cur_t
  __shared__ uint32_t mask[GATHER ? kDistTile / 32 : 1], next_t, next_key;
  __shared__ uint16_t row_piece[GATHER ? kDistTile / 64 : 1];
  uint32_t *piece = reinterpret_cast<uint32_t *>(sk);  // address - position
  // Gathered: every XCD takes a stretch of neighbouring nodes, all ranges of
  // kGang of them, then of the next kGang, so that workgroups that run together
  // read the cache lines where their nodes' pieces adjoin once.  (One range of
  // all nodes after the other: 1314 against 1238 us at 2^28 int64; the ranges
  // dealt out to the XCDs: 1267 against 1136 at 2^27 uint64 with values.)  The
  // copies' ranges follow.
  uint32_t nodes = 0, each = 0, most = 0, listed = 0;
  if constexpr (GATHER) {
    nodes = L.ctr->nodes[L.level];
    each = (nodes + kXcds - 1) / kXcds;
    most = L.ctr->most_ranges;
    listed = (each + kGang - 1) / kGang * kGang * most * kXcds;
  }
  for (uint32_t ri = blockIdx.x; ri < listed + nranges; ri += gridDim.x) {
  DistRange rg;
  if (ri < listed) {
    const uint32_t x = ri / kXcds, y = x / kGang;
    const uint32_t local = y / most * kGang + x % kGang;
    rg = DistRange{ri % kXcds * each + local, y % most};
    if (local >= each || rg.node >= nodes || rg.r >= L.nodes[rg.node].nr) continue;
  } else {
    rg = L.ranges[ri - listed];
  }
  __syncthreads();  // the last range's LDS is read no more
  const DistNode nd = L.nodes[rg.node];
  const bool cut = !GATHER || nd.nb > 1;
  ClassifierRegs<U> cr{};
  if (cut) cr = classifier_load(cl, (const U *)L.spl + nd.sbase, nd.nb - 1);
  const uint32_t begin = rg.r * L.rl, end = begin + L.rl < nd.len ? begin + L.rl : nd.len;
  const U *p = GATHER ? src : src + nd.off;
  const uint32_t *vp = KV ? (GATHER ? vsrc : vsrc + nd.off) : nullptr;
  U *q = dst + nd.off;
  uint32_t *vq = KV ? vdst + nd.off : nullptr;
  const uint32_t nbits = 32 - __clz(nd.nb - 1);
  uint32_t tile = 0, cur_t = 0, cur_key = 0;
  const uint32_t ptiles = GATHER ? parent_tiles(nd) : 0u;
  if constexpr (GATHER) {
    // the last group of 8 tiles whose keys start at or before the range's
    const uint32_t *pre = L.pre + nd.prow / 8;
    uint32_t lo = 0, m = (ptiles + 7) / 8;
    while (m > 1) {
      const uint32_t step = (m + 63) / 64, x = lane * step;
      const uint64_t le = __ballot(x < m && pre[lo + (x < m ? x : 0u)] <= begin);
      const uint32_t c = (uint32_t)__popcll(le) - 1;  // (the first one is)
      lo += c * step;
      m = m - c * step < step ? m - c * step : step;
    }
    cur_t = lo * 8;
    cur_key = pre[lo];
  }
  for (uint32_t base = begin; base < end; base += kDistTile, ++tile) {
    const uint32_t count = end - base < kDistTile ? end - base : kDistTile;
    auto at = [](int i) { return tile_at<KV>(i); };
    U k[NI];
    uint32_t v[KV ? NI : 1], b[NI], pos[NI];
    if constexpr (GATHER) {
      for (uint32_t i = tid; i < kDistTile / 32; i += NT) mask[i] = 0;
      __syncthreads();
      const uint32_t limit = base + count;
      uint32_t np = 0;
      do {
        const uint32_t t = cur_t + tid;
        uint32_t s, c;
        piece_of(L.ptable, nd.prow, nd.pnext, nd.plen, t, s, c);
        c -= s;
        // keys (at most 512 tiles of 6144: 22 bits) and non-empty pieces before
        uint32_t total;
        const uint32_t x = block_scan<NT>(c | (c ? 1u << 22 : 0u), wsum, total);
        const uint32_t first = cur_key + (x & 0x3fffffu), to = np + (x >> 22);
        if (c && first < limit && first + c > base) {
          const uint32_t from = first > base ? first - base : 0u;
          const uint32_t stop = first + c < limit ? first + c - base : count;
          piece[to] = nd.poff + t * kDistTile + s + base - first;  // modulo 2^32
          if (from & 63u) {
            const uint32_t bit = (from & 63u) - 1;
            atomicOr(&mask[(from >> 6) * 2 + (bit >> 5)], 1u << (bit & 31u));
          }
          for (uint32_t r = (from + 63) / 64; r * 64 < stop; ++r) row_piece[r] = (uint16_t)to;
        }
        if (c && first <= limit && limit - first < c) {
          next_t = t;
          next_key = first;
        }
        np += total >> 22;
        cur_t += NT;
        cur_key += total & 0x3fffffu;
        __syncthreads();
      } while (cur_key < limit && cur_t < ptiles);
      if (cur_key > limit) {  // a piece listed now continues in the next tile
        cur_t = next_t;
        cur_key = next_key;
      }
      uint32_t addr[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t j = at(i) < count ? at(i) : count - 1, r = j >> 6;
        const uint64_t m = (uint64_t)mask[r * 2] | (uint64_t)mask[r * 2 + 1] << 32;
        const uint32_t started = __popcll(m & (((uint64_t)1 << (j & 63u)) - 1));
        addr[i] = piece[row_piece[r] + started] + j;
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        k[i] = __builtin_nontemporal_load(&p[addr[i]]);
        if constexpr (KV) v[i] = __builtin_nontemporal_load(&vp[addr[i]]);
      }
      __syncthreads();  // the list is read before keys or counts overwrite it
      if (!cut) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if (at(i) < count) {
            q[base + at(i)] = k[i];
            if constexpr (KV) vq[base + at(i)] = v[i];
          }
        }
        continue;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t j = at(i) < count ? at(i) : count - 1;
        k[i] = __builtin_nontemporal_load(&p[base + j]);
        if constexpr (KV) v[i] = __builtin_nontemporal_load(&vp[base + j]);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) k[i] = Key<KT>::map(k[i]);
    }
    classify(cl, cr, k, b);
    const uint32_t mine = tile_ranks<KV>(b, pos, count, nbits, wh, hist);
    uint32_t total;
    const uint32_t lo = block_scan<NT>(mine, wsum, total);
    lofs[tid] = lo;
    rows[tile][tid] = (uint16_t)lo;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      pos[i] += lofs[b[i]];
      if constexpr (KV) pos[i] += wh[wid * kDistSlots + b[i]];
    }
    if constexpr (KV) __syncthreads();  // wh is read before the keys overwrite it
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (at(i) < count) sk[pos[i]] = k[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t j = i * NT + tid;
      if (j < count) q[base + j] = sk[j];
    }
    if constexpr (KV) {
      __syncthreads();
      uint32_t *sv = reinterpret_cast<uint32_t *>(sk);
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (at(i) < count) sv[pos[i]] = v[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t j = i * NT + tid;
        if (j < count) vq[base + j] = sv[j];
      }
    }
    __syncthreads();
  }
  if (cut && tid < nd.nb) {
    uint16_t *to = (uint16_t *)L.table + nd.tbase + tid * nd.stride + begin / kDistTile;
    for (uint32_t t = 0; t < tile; ++t) to[t] = rows[t][tid];
  }
  }
}

// --------------------------------------------------------------- leaves ---
// The same entry in every lane, in scalar registers.
__device__ __forceinline__ DistLeaf uniform(const DistLeaf &f) {
  DistLeaf u;
  const uint32_t *a = reinterpret_cast<const uint32_t *>(&f);
  uint32_t *b = reinterpret_cast<uint32_t *>(&u);
#pragma unroll
  for (uint32_t i = 0; i < sizeof(DistLeaf) / 4; ++i) b[i] = __builtin_amdgcn_readfirstlane(a[i]);
  return u;
}

// One workgroup sorts one leaf of at most CAP = NT * NI keys.  The keys are
// binned by interpolation between the bounds of the leaf (CAP bins, one key in
// two bins when the leaf has its target size), placed in bin order in LDS, and
// the bins of two keys or more (one in eleven at the target size) are listed
// and sorted, one thread each (counting every key's place within its bin
// instead looked at each bin as often as it has keys, in lockstep with the
// fullest of 256: 1.77 against 1.52 ms at 2^28 int64).  VALU instructions (123
// a key, 147 with values) and the latency of the gather bound it: 76 KB of LDS
// leave two workgroups a CU.  The loads are issued as their addresses are found,
// before the barrier that ends it: 1.52 -> 1.43 ms.  A leaf with a crowded bin (a key of rank
// kCrowded or more: many equal keys, or keys spread over many magnitudes) is
// left to the rest list.
//
// Keys of the last level are gathered: the leaf's piece of every tile of the
// node is found in the table, and a bit mask over the leaf's positions, set
// where a piece starts, tells every position its piece.
constexpr uint32_t kCrowded = 16;
// Bins of one key value: keys-only they need no sorting, and the byte of their
// count limits them; key-value every key counts the earlier ones of its bin.
template <bool KV> constexpr uint32_t kCrowdedDirect = KV ? 96 : 255;

// Sorts the n >= 2 keys of a bin in LDS, key-value by key and position: four
// in registers, any further ones (1 bin in 500 at the target size) by
// insertion.
template <typename U, bool KV>
__device__ __forceinline__ void sort_bin(U *sk, uint16_t *sidx, uint32_t n) {
  U k[4];
  uint32_t x[KV ? 4 : 1];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t a = j < (int)n ? j : 0;
    k[j] = sk[a];
    k[j] = j < (int)n ? k[j] : key_max<U>();
    if constexpr (KV) x[j] = j < (int)n ? (uint32_t)sidx[a] : 0xffffu;
  }
  auto order = [&](int a, int b) {
    bool sw = k[b] < k[a];
    if constexpr (KV) sw = sw || (k[b] == k[a] && x[b] < x[a]);
    const U ka = opaque(k[a]), kb = opaque(k[b]);
    k[a] = sw ? kb : ka;
    k[b] = sw ? ka : kb;
    if constexpr (KV) {
      const uint32_t xa = x[a], xb = x[b];
      x[a] = sw ? xb : xa;
      x[b] = sw ? xa : xb;
    }
  };
  order(0, 1);
  order(2, 3);
  order(0, 2);
  order(1, 3);
  order(1, 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (j < (int)n) {
      sk[j] = k[j];
      if constexpr (KV) sidx[j] = (uint16_t)x[j];
    }
  }
  for (uint32_t t = 4; t < n; ++t) {
    const U y = sk[t];
    const uint32_t z = KV ? sidx[t] : 0;
    uint32_t j = t;
    for (; j > 0; --j) {
      const U o = sk[j - 1];
      if (o < y) break;
      if constexpr (KV) {
        const uint32_t oz = sidx[j - 1];
        if (o == y && oz < z) break;
        sidx[j] = (uint16_t)oz;
      } else {
        if (o == y) break;
      }
      sk[j] = o;
    }
    sk[j] = y;
    if constexpr (KV) sidx[j] = (uint16_t)z;
  }
}

// Where the keys of a leaf that lies in pieces are: use(i, address) of the key at
// position at(i), for the steps i that are wanted (the same for a whole wave).
// `piece` (one entry a tile of the node) and the tables `mask` (a bit a
// position) and `row_piece` (an entry for 64) are scratch, free again on return.
template <int NT, int NI, typename At, typename Wanted, typename Use>
__device__ __forceinline__ void leaf_addresses(const Level &L, const DistLeaf &leaf, uint32_t *piece,
                                               uint32_t *mask, uint16_t *row_piece, uint32_t *wsum,
                                               At at, Wanted wanted, Use use) {
  constexpr uint32_t CAP = NT * NI;
  const uint32_t tid = threadIdx.x, len = leaf.len_flags & kLeafLenMask;
  const uint16_t *table = (const uint16_t *)L.table;
  const uint32_t tiles = (leaf.node_len + kDistTile - 1) / kDistTile;
  for (uint32_t i = tid; i < CAP / 32; i += NT) mask[i] = 0;
  uint32_t np = 0, run = 0;
  for (uint32_t t0 = 0; t0 < tiles && run < leaf.first + len; t0 += NT) {
    const uint32_t t = t0 + tid;
    uint32_t s, c;
    piece_of(table, leaf.row, leaf.next_row, leaf.node_len, t, s, c);
    c -= s;
    // keys (at most 512 tiles of 6144: 22 bits) and non-empty pieces before
    uint32_t total;
    const uint32_t x = block_scan<NT>(c | (c ? 1u << 22 : 0u), wsum, total);
    const uint32_t first = run + (x & 0x3fffffu), pi = np + (x >> 22);
    if (c) {
      // position of the piece's first key in the leaf; a piece that starts
      // before the leaf holds position 0
      const uint32_t pos = first > leaf.first ? first - leaf.first : 0u;
      const uint32_t stop = first + c > leaf.first ? first + c - leaf.first : 0u;
      piece[pi] = leaf.node_off + t * kDistTile + s + leaf.first - first;  // modulo 2^32
      if (stop && pos < len) {
        if (pos & 63u) {
          const uint32_t bit = (pos & 63u) - 1;
          atomicOr(&mask[(pos >> 6) * 2 + (bit >> 5)], 1u << (bit & 31u));
        }
        for (uint32_t r = (pos + 63) / 64; r * 64 < stop && r * 64 < len; ++r)
          row_piece[r] = (uint16_t)pi;
      }
    }
    run += total & 0x3fffffu;
    np += total >> 22;
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (wanted(i)) {  // (positions past the end: the last key)
      const uint32_t j = at(i) < len ? at(i) : len - 1;
      const uint32_t r = j >> 6;
      const uint64_t m = (uint64_t)mask[r * 2] | (uint64_t)mask[r * 2 + 1] << 32;
      const uint32_t started = __popcll(m & (((uint64_t)1 << (j & 63u)) - 1));
      use(i, piece[row_piece[r] + started] + j);
    }
  }
  __syncthreads();
}

template <int KT, bool KV, int NT, int NI>
__device__ __forceinline__ void sort_leaf(
    const typename Key<KT>::U *__restrict__ ws, const uint32_t *__restrict__ vws,
    typename Key<KT>::U *out, uint32_t *vout, const Level &L, uint32_t li) {
  using U = typename Key<KT>::U;
  constexpr uint32_t CAP = NT * NI, NBIN = CAP, NW = NT / 64;
  constexpr int BW = NBIN / 4 / NT;  // words of bin counts a thread scans
  static_assert(BW == 4 || BW == 2, "one vector of bin counts a thread");
  using Counts = std::conditional_t<BW == 4, uint4, uint2>;
  __shared__ U sk[CAP];
  __shared__ uint16_t sidx[KV ? CAP : 1];  // position of the key of a slot
  // bin counts, a byte each (a count past 255 runs into its neighbours, but
  // the leaf is crowded by then), and the keys before every four bins; later
  // the list of bins to sort
  constexpr uint32_t kList = NBIN / 4 + NBIN / 8;
  __shared__ __attribute__((aligned(16))) uint32_t bins[kList];
  uint16_t *bin4 = reinterpret_cast<uint16_t *>(bins + NBIN / 4);
  __shared__ U smin[NW], smax[NW];
  __shared__ uint32_t wsum[NW];
  // the gather's tables, dead before the keys are placed
  uint32_t *piece = reinterpret_cast<uint32_t *>(sk);  // address - position
  uint32_t *mask = bins;                               // CAP bits: a piece starts at the next position
  uint16_t *row_piece = reinterpret_cast<uint16_t *>(bins + CAP / 32);  // piece of position 64 r
  static_assert(dist_node_tiles(sizeof(U), KV) * 4 <= sizeof(sk), "pieces fit the key area");
  static_assert(CAP / 8 + CAP / 32 <= sizeof(bins), "mask and rows fit the bins");
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const DistLeaf leaf = uniform(L.leaves[li]);
  const uint32_t off = leaf.off, len = leaf.len_flags & kLeafLenMask;
  const uint32_t from = (leaf.len_flags >> kLeafSrcShift) & 3u;
  const bool inner = from == kSrcPieces && (leaf.len_flags & kLeafInner);
  U k[NI];
  uint32_t v[KV ? NI : 1];
  // the loads are all issued before any is used: clamped, not conditional;
  // steps of NT keys past the end are skipped throughout.  Keys in pieces are
  // loaded as their addresses are found, before the barrier that ends the search
  // (2^28 int64: 3.71 ms, after it 3.87; 2^27 uint64 with values 2.97 and 3.04).
  auto load = [&](int i, const U *p, const uint32_t *vp, uint32_t addr) {
    k[i] = __builtin_nontemporal_load(&p[addr]);
    if constexpr (KV) v[i] = __builtin_nontemporal_load(&vp[addr]);
  };
  auto wanted = [&](int i) { return i * NT < len; };
  if (from == kSrcPieces) {
    if (!KV && (leaf.len_flags & kLeafEqual)) {
      // one key value, known from the splitters: nothing to read
      const U x = (U)leaf.below;
      for (uint32_t i = tid; i < len; i += NT)
        __builtin_nontemporal_store(Key<KT>::unmap(x), &out[off + i]);
      return;
    }
    leaf_addresses<NT, NI>(L, leaf, piece, mask, row_piece, wsum, [&](int i) { return i * NT + tid; }, wanted,
                           [&](int i, uint32_t addr) { load(i, ws, vws, addr); });
  } else {
    const U *p = from == kSrcOut ? (const U *)out : ws;
    const uint32_t *vp = from == kSrcOut ? (const uint32_t *)vout : vws;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (wanted(i)) load(i, p, vp, off + (i * NT + tid < len ? i * NT + tid : len - 1));
  }
  if (leaf.len_flags & (kLeafEqual | kLeafMove)) {
    const bool equal = leaf.len_flags & kLeafEqual;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t idx = i * NT + tid;
      if (idx < len) {
        out[off + idx] = equal ? Key<KT>::unmap(k[i]) : k[i];
        if constexpr (KV) vout[off + idx] = v[i];
      }
    }
    return;
  }
  reinterpret_cast<Counts *>(bins)[tid] = Counts{};
  // Bounds of the keys: the splitters around the bucket, or (a node's first
  // and last bucket, and leaves of earlier levels) the smallest and largest
  // key.
  U mn, mx;
  if (inner) {
    mn = (U)leaf.below;
    mx = (U)leaf.above - 1;
    __syncthreads();
  } else {
    mn = mx = k[0];  // (clamped loads repeat the last key)
#pragma unroll
    for (int i = 1; i < NI; ++i) {
      if (i * NT < len) {
        mn = k[i] < mn ? k[i] : mn;
        mx = k[i] > mx ? k[i] : mx;
      }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      const U a = __shfl_xor(mn, d, 64), c = __shfl_xor(mx, d, 64);
      mn = a < mn ? a : mn;
      mx = c > mx ? c : mx;
    }
    if (lane == 0) {
      smin[wid] = mn;
      smax[wid] = mx;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t w = 0; w < NW; ++w) {
      const U a = smin[w], c = smax[w];
      mn = a < mn ? a : mn;
      mx = c > mx ? c : mx;
    }
  }
  // bin = floor(x * scale / 2^32) of x, the top 32 bits of the key's distance
  // from mn; the scale is a little below NBIN 2^32 / (top + 1), so that every
  // bin is below NBIN.  A span below NBIN gives every key value its own bin.
  const uint64_t span = (uint64_t)(mx - mn);
  const uint32_t sh = span >> 32 ? 32 - __clz((uint32_t)(span >> 32)) : 0u;
  const uint32_t top = (uint32_t)(span >> sh);
  const bool direct = top < NBIN;
  const uint32_t scale =
      direct ? 0u : (uint32_t)((float)NBIN * 4294967296.0f * (1.0f - 0x1p-20f) / ((float)top + 1.0f));
  uint32_t place[NI];  // bin, and rank in it << 16
  uint32_t worst = 0;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (i * NT < len) {
      const uint32_t x = (uint32_t)((uint64_t)(k[i] - mn) >> sh);
      const uint32_t bin = direct ? x : __umulhi(x, scale);
      place[i] = bin;
      if (i * NT + tid < len) {
        const uint32_t byte = (bin & 3u) * 8;
        const uint32_t r = (atomicAdd(&bins[bin >> 2], 1u << byte) >> byte) & 0xffu;
        place[i] |= r << 16;
        worst = r > worst ? r : worst;
      }
    }
  }
  if (__syncthreads_or(worst >= (direct ? kCrowdedDirect<KV> : kCrowded))) {
    // one key value between two sampled ones: the keys (and values) are in order
    if (tid == 0) smin[0] = k[0];
    __syncthreads();
    const U x = smin[0];
    bool other = false;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (i * NT < len) other |= k[i] != x;
    if (!__syncthreads_or(other)) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t idx = i * NT + tid;
        if (idx < len) {
          out[off + idx] = Key<KT>::unmap(x);
          if constexpr (KV) vout[off + idx] = v[i];
        }
      }
    } else if (tid == 0) {
      const uint32_t to = atomicAdd(&L.ctr->rest, 1u);
      if (to < L.max_rest) L.rest[to] = li;
      else plan_failed(L.ctr, L.err);
    }
    return;
  }
  // keys before every four bins, 16 bins a thread; and the bins of two keys or
  // more, each listed by its second key
  uint32_t at, listed;
  {
    uint32_t seconds = 0;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (i * NT < len) seconds += place[i] >> 16 == 1 ? 1u : 0u;
    const Counts q = reinterpret_cast<const Counts *>(bins)[tid];
    uint32_t c[BW + 1] = {};  // keys in the words before
    c[1] = __builtin_amdgcn_sad_u8(q.x, 0, 0);
    c[2] = __builtin_amdgcn_sad_u8(q.y, 0, c[1]);
    if constexpr (BW == 4) {
      c[3] = __builtin_amdgcn_sad_u8(q.z, 0, c[2]);
      c[4] = __builtin_amdgcn_sad_u8(q.w, 0, c[3]);
    }
    uint32_t total;
    const uint32_t x = block_scan<NT>(c[BW] | seconds << 16, wsum, total);
    const uint32_t run = x & 0xffffu;
#pragma unroll
    for (int j = 0; j < BW; j += 2)
      reinterpret_cast<uint32_t *>(bin4)[(tid * BW + j) / 2] = (run + c[j]) | (run + c[j + 1]) << 16;
    at = x >> 16;
    listed = direct ? 0u : total >> 16;  // (bins of one key value: see below)
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (i * NT < len) {
      const uint32_t bin = place[i] & 0xffffu, rank = place[i] >> 16;
      place[i] = 0;
      if (i * NT + tid < len) {
        const uint32_t w = bins[bin >> 2];
        const uint32_t s = __builtin_amdgcn_sad_u8(w & ~(~0u << (bin & 3u) * 8), 0, bin4[bin >> 2]);
        sk[s + rank] = k[i];
        if constexpr (KV) sidx[s + rank] = (uint16_t)(i * NT + tid);
        // a listed bin (or any, of one key value): first slot, and keys << 16
        if (rank == 1 || (KV && direct)) place[i] = s | ((w >> (bin & 3u) * 8) & 0xffu) << 16;
      }
    }
  }
  if constexpr (KV) {
    // the leaf may lie in the output: every load has returned before any
    // thread stores
#pragma unroll
    for (int i = 0; i < NI; ++i) asm volatile("" : "+v"(v[i]));
  }
  __syncthreads();
  // The keys of every listed bin are sorted in place by one thread.  The list
  // takes the place of the counts; a leaf of many pairs needs it twice.
  uint32_t *list = bins;
  for (uint32_t base = 0; base < listed; base += kList) {
    uint32_t to = at - base;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (i * NT < len && place[i]) {
        if (to < kList) list[to] = place[i];
        ++to;
      }
    }
    __syncthreads();
    const uint32_t m = listed - base < kList ? listed - base : kList;
    for (uint32_t e = tid; e < m; e += NT)
      sort_bin<U, KV>(sk + (list[e] & 0xffffu), sidx + (KV ? list[e] & 0xffffu : 0u), list[e] >> 16);
    __syncthreads();
  }
  if constexpr (KV) {
    if (direct) {
      // equal keys in the order of their positions (30011 int64 of 1000 values:
      // 59 us, with the bins sorted by insertion 124)
      uint32_t fin[NI], most = 0;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (i * NT >= len) place[i] = 0;
        fin[i] = place[i] & 0xffffu;
        most = place[i] >> 16 > most ? place[i] >> 16 : most;
      }
      for (uint32_t t = 0; t < most; ++t) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const bool in_bin = t < place[i] >> 16;
          const uint32_t x = sidx[(place[i] & 0xffffu) + (in_bin ? t : 0u)];
          fin[i] += in_bin && x < i * NT + tid ? 1u : 0u;
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (i * NT + tid < len) sidx[fin[i]] = (uint16_t)(i * NT + tid);
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const uint32_t idx = i * NT + tid;
    if (idx < len) __builtin_nontemporal_store(Key<KT>::unmap(sk[idx]), &out[off + idx]);
  }
  if constexpr (KV) {
    uint32_t *sv = reinterpret_cast<uint32_t *>(sk);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (i * NT + tid < len) sv[i * NT + tid] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t idx = i * NT + tid;
      if (idx < len) __builtin_nontemporal_store(sv[sidx[idx]], &vout[off + idx]);
    }
  }
}

// The grid is the count of leaves to expect: the bound on them is more than
// twice that, and empty workgroups cost (4096 int64 arrays: 2546 us with, 2445
// without).  Frequent keys and short segments may leave more.  Neighbouring
// leaves run on one XCD (workgroups go to the eight in turn): their pieces of
// a tile adjoin and share cache lines, which that XCD's L2 then reads once.
template <int KT, bool KV, int NT, int NI, int WAVES>
__global__ __launch_bounds__(NT, WAVES) void dist_leaf_kernel(
    const typename Key<KT>::U *__restrict__ ws, const uint32_t *__restrict__ vws,
    typename Key<KT>::U *out, uint32_t *vout, Level L) {
  const uint32_t nl = L.ctr->leaves;
  // a bound did not hold (the flag is not looked at, as this launch may set it:
  // the leaves that were written can be sorted)
  if (nl > L.max_leaves) return;
  const uint32_t each = (nl + kXcds - 1) / kXcds;
  for (uint32_t x = blockIdx.x; x < each * kXcds; x += gridDim.x) {
    const uint32_t li = x % kXcds * each + x / kXcds;
    if (li >= nl) continue;
    __syncthreads();  // the last leaf's LDS is read no more
    sort_leaf<KT, KV, NT, NI>(ws, vws, out, vout, L, li);
  }
}

// ----------------------------------------------------------------- rest ---
// The tile sort's network and merge rounds on len keys (and values) at p[addr[i]],
// where a thread's i-th is position tile_pos(tid, i) (a position past the end: any
// address of a key).  The sorted keys are left in sk (values in sv).
template <int NI>
__device__ __forceinline__ uint32_t tile_pos(uint32_t tid, int i) {  // (a wave's are consecutive)
  return (tid >> 6) * (64 * NI) + i * 64 + (tid & 63);
}

template <typename U, bool KV, int NT, int NI>
__device__ __forceinline__ void sort_tile(const U *p, const uint32_t *vp,
                                          const uint32_t (&addr)[NI], uint32_t len,
                                          U *sk, uint32_t *sv, uint32_t tid) {
  U k[NI];
  uint32_t v[NI];
  if ((tid >> 6) * (64 * NI) < len) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      k[i] = p[addr[i]];
      if constexpr (KV) v[i] = vp[addr[i]];
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bool ok = tile_pos<NI>(tid, i) < len;
      k[i] = ok ? k[i] : key_max<U>();
      if constexpr (KV) {  // consecutive positions a thread, through LDS
        sk[pad16(tile_pos<NI>(tid, i))] = k[i];
        sv[pad16(tile_pos<NI>(tid, i))] = ok ? v[i] : 0u;
      }
    }
    if constexpr (KV) {
      wave_sync();
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        k[i] = sk[pad16(tid * NI + i)];
        v[i] = sv[pad16(tid * NI + i)];
      }
    }
  }
  if constexpr (KV) lds_sort_pairs<U, NT, true, NI>(k, v, sk, sv, len, tid);
  else lds_sort_keys<U, NT, true>(k, sk, len, tid);
}

// How many of the first d keys of the merge of a[0, la) and b[0, lb) (ties to a)
// come from a; by one wave, 64 candidates at a time.
template <typename U>
__device__ __forceinline__ uint32_t wave_merge_path(const U *a, uint32_t la, const U *b, uint32_t lb,
                                                    uint32_t d) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t lo = d > lb ? d - lb : 0, hi = d < la ? d : la;
  while (lo < hi) {
    const uint32_t step = (hi - lo + 63) / 64, x = lo + lane * step;
    const uint32_t y = x < hi ? x : lo;
    // (true for a prefix of the candidates)
    const uint32_t c = (uint32_t)__popcll(__ballot(x < hi && a[y] <= b[d - 1 - y]));
    hi = lo + c * step < hi ? lo + c * step : hi;
    lo = c ? lo + (c - 1) * step + 1 : hi;
  }
  return lo;
}

// What the leaf kernel left: leaves with a crowded bin, each sorted like a tile by
// one workgroup (16 million int64 of 1000 values in segments of 100003, all leaves
// crowded: 378 us, uint64 with values 565; 438 and 766 when the leaf kernel wrote
// such leaves out, and this one sorted them as whole tiles, with values 16 keys a
// thread), and big buckets, above the cap.
//
// Big buckets come from samples that missed much of a node: about one bucket of
// ten thousand by chance, and then of two tiles, but the sampled positions can
// be computed, and an input that holds one key there has its whole array in
// two.  So their sorts are tasks that all workgroups share (1500000 uint64 keys
// of that kind: 552 us, by one workgroup a bucket 14611; random ones 92).  A
// bucket of T tiles has T tile sorts and then, for every doubling of the sorted
// runs, T merges of one tile's length, between the output and the workspace.
//
// Workgroups claim the tasks of all in one order: the crowded leaves (which lie
// in the workspace), then bucket by bucket, round by round.  A task waits until
// all before its round have ended: every task it waits for has a lower number,
// so some workgroup already works on it, and the lowest unfinished task never
// waits.
// (One thread's fences stand for the workgroup, between its barriers: fences of
// all waves write back and invalidate the L2 each, 1397 us.)
template <int KT, bool KV, int NT, int NI, int WAVES>
__global__ __launch_bounds__(NT, WAVES) void dist_rest_kernel(
    typename Key<KT>::U *ws, uint32_t *vws, typename Key<KT>::U *out, uint32_t *vout, Level L) {
  using U = typename Key<KT>::U;
  constexpr uint32_t CAP = NT * NI;
  using T = TileLds<KV, CAP / kTileItems>;
  __shared__ U sk[T::SLOTS];
  __shared__ uint32_t sv[KV ? T::SLOTS : 1];
  __shared__ uint32_t mask[CAP / 32], wsum[NT / 64];
  __shared__ uint16_t row_piece[CAP / 64];
  __shared__ uint32_t claimed, path[2];
  static_assert(dist_node_tiles(sizeof(U), KV) * 4 <= sizeof(sk), "pieces fit the key area");
  DistCounters *ctr = L.ctr;
  DistBig *big = L.big;
  const uint32_t no = ctr->rest, nbig = ctr->big;
  if (ctr->failed || no + nbig == 0) return;
  uint32_t e = 0, base = no;  // a bucket, and its first task
  for (;;) {
    // hidden from the optimiser, which otherwise computes every LDS address of the
    // sort before the loop and keeps it (240 registers, one workgroup a CU)
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    __syncthreads();  // the task before has no more use for the LDS
    if (tid == 0) claimed = atomicAdd(&ctr->next_task, 1u);
    __syncthreads();
    const uint32_t task = claimed;
    // the m keys of the task come from p (a merge's from o in the runs of src) and
    // go to dst, final or still mapped
    const U *p = out, *src = nullptr;
    const uint32_t *vp = vout, *vsrc = nullptr;
    U *dst = out;
    uint32_t *vdst = vout, *count = &ctr->rest_done;
    uint32_t m, o = 0, r = 0, len = 0, addr[NI];
    bool final = true;
    if (task < no) {
      const DistLeaf leaf = uniform(L.leaves[L.rest[task]]);
      const uint32_t from = (leaf.len_flags >> kLeafSrcShift) & 3u;
      m = leaf.len_flags & kLeafLenMask;
      p = from == kSrcOut ? out : ws;
      vp = from == kSrcOut ? vout : vws;
      dst += leaf.off;
      if constexpr (KV) vdst += leaf.off;
      if (from == kSrcPieces)
        leaf_addresses<NT, NI>(L, leaf, reinterpret_cast<uint32_t *>(sk), mask, row_piece, wsum,
                               [&](int i) { return tile_pos<NI>(tid, i); },
                               [&](int) { return tile_pos<NI>(tid, 0) - (tid & 63) < m; },
                               [&](int i, uint32_t at) { addr[i] = at; });
      else
#pragma unroll
        for (int i = 0; i < NI; ++i) addr[i] = leaf.off + (tile_pos<NI>(tid, i) < m ? tile_pos<NI>(tid, i) : 0u);
    } else {
      if (nbig == 0) return;
      uint32_t tiles, rounds;
      for (;;) {
        len = big[e].len;
        tiles = (len + CAP - 1) / CAP;
        rounds = 32 - __clz(tiles - 1);
        if (task < base + tiles * (1 + rounds)) break;
        base += tiles * (1 + rounds);
        if (++e == nbig) return;
      }
      const uint32_t off = big[e].off;
      r = (task - base) / tiles;
      o = (task - base) % tiles * CAP;
      m = len - o < CAP ? len - o : CAP;
      final = r == rounds;
      // round r leaves its runs in the output if the number of rounds to come is even
      const bool here = ((rounds - r) & 1) == 0;
      src = (here ? ws : out) + off;
      dst = (here ? out : ws) + off + o;
      if constexpr (KV) {
        vsrc = (here ? vws : vout) + off;
        vdst = (here ? vout : vws) + off + o;
      }
      count = &big[e].done;
      const uint32_t *before = r ? count : &ctr->rest_done;
      const uint32_t n = r ? tiles * r : no;
      if (tid == 0) {
        while (__hip_atomic_load(before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n)
          __builtin_amdgcn_s_sleep(8);
        __threadfence();
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NI; ++i) addr[i] = off + o + (tile_pos<NI>(tid, i) < m ? tile_pos<NI>(tid, i) : 0u);
    }
    if (r == 0) {
      sort_tile<typename Key<KT>::U, KV, NT, NI>(p, vp, addr, m, sk, sv, tid);
      for (uint32_t i = tid; i < m; i += NT) {
        dst[i] = final ? Key<KT>::unmap(sk[i]) : sk[i];
        if constexpr (KV) vdst[i] = sv[i];
      }
    } else {
      // outputs o .. o+m-1 of the runs' pairs (whose lengths are whole tiles)
      const uint32_t w = CAP << (r - 1), a0 = o / (2 * w) * (2 * w);
      const uint32_t la = len - a0 < w ? len - a0 : w, b0 = a0 + la;
      const uint32_t lb = len - b0 < w ? len - b0 : w;
      if (tid < 128) {  // (two waves)
        const uint32_t x = wave_merge_path(src + a0, la, src + b0, lb, o - a0 + (tid < 64 ? 0u : m));
        if ((tid & 63) == 0) path[tid >> 6] = x;
      }
      __syncthreads();
      const uint32_t pa = path[0], na = path[1] - pa, pb = o - a0 - pa;
      for (uint32_t i = tid; i < m; i += NT) {
        const uint32_t from = i < na ? a0 + pa + i : b0 + pb + (i - na);
        sk[i] = src[from];
        if constexpr (KV) sv[i] = vsrc[from];
      }
      __syncthreads();
      // NI outputs a thread, stored one by one (in registers until all are merged
      // they would not fit beside the sort's)
      const uint32_t at = tid * NI;
      uint32_t lo = at > m - na ? at - (m - na) : 0, hi = at < na ? at : na;
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (sk[mid] <= sk[na + at - 1 - mid]) lo = mid + 1;
        else hi = mid;
      }
      uint32_t xa = lo, xb = na + (at - lo);
#pragma unroll 1
      for (uint32_t i = at; i < at + NI && i < m; ++i) {
        const uint32_t x = xa < na && (xb >= m || sk[xa] <= sk[xb]) ? xa++ : xb++;
        dst[i] = final ? Key<KT>::unmap(sk[x]) : sk[x];
        if constexpr (KV) vdst[i] = sv[x];
      }
    }
    if (nbig) {  // (else no task waits)
      __syncthreads();
      if (tid == 0) {
        __threadfence();
        atomicAdd(count, 1u);
      }
    }
  }
}

// ------------------------------------------------------------ launchers ---
// Buffers of a level: the last level writes the workspace (the leaves go from
// there to the output), the ones before it alternate.
bool level_to_out(const DistPlan &d, int level) { return (d.levels - level) & 1; }

const void *level_src(const DistPlan &d, const DistBufs &b, int level) {
  return level == 1 ? b.in : level_to_out(d, level - 1) ? (const void *)b.out : (const void *)b.ws;
}
const uint32_t *level_vsrc(const DistPlan &d, const DistBufs &b, int level) {
  return level == 1 ? b.vin : level_to_out(d, level - 1) ? b.vout : b.vws;
}

hipError_t level_error_word(uint32_t **err) {
  int device = 0;
  const hipError_t e = hipGetDevice(&device);
  return e != hipSuccess ? e : error_word(device, err);
}

Level level_args(int kt, const DistPlan &d, int level, char *w) {
  Level L{};
  L.ctr = (DistCounters *)(w + d.off_ctr);
  L.nodes = (DistNode *)(w + d.off_nodes[level]);
  L.ranges = (DistRange *)(w + d.off_ranges[level]);
  L.spl = w + d.off_spl;
  L.start = (uint32_t *)(w + d.off_start);
  L.table = w + (d.tiled(level) && level < d.levels ? d.off_ptable : d.off_table);
  L.ptable = (const uint16_t *)(w + d.off_ptable);
  L.pre = (uint32_t *)(w + d.off_pre);
  L.tiled = d.tiled(level);
  L.next_tiled = d.tiled(level + 1);
  L.gather = d.gather && level == d.levels;
  L.kv = d.cap == kDistCapKV;
  L.max_copies = d.max_copies;
  L.leaves = (DistLeaf *)(w + d.off_leaves);
  L.rest = (uint32_t *)(w + d.off_rest);
  L.big = (DistBig *)(w + d.off_big);
  L.level = (uint32_t)level;
  L.levels = (uint32_t)d.levels;
  L.cap = d.cap;
  L.target = d.target;
  L.rl = d.rl[level];
  L.src = level == d.levels ? kSrcPieces : level_to_out(d, level) ? kSrcOut : kSrcWs;
  L.node_tiles = dist_node_tiles(key_bytes(kt), d.cap == kDistCapKV);
  L.max_cols = d.max_cols;
  L.max_leaves = d.max_leaves;
  L.max_rest = d.max_rest;
  L.max_big = d.max_big;
  if (level < d.levels) {
    L.next_nodes = (DistNode *)(w + d.off_nodes[level + 1]);
    L.next_ranges = (DistRange *)(w + d.off_ranges[level + 1]);
    L.next_rl = d.rl[level + 1];
    L.max_next_nodes = d.max_nodes[level + 1];
    L.max_next_ranges = d.max_ranges[level + 1];
    L.max_next_table = d.max_table[level + 1];
  }
  return L;
}

// Level 1 reads raw keys of type kt; later levels read mapped keys, which are
// unsigned integers.
int level_type(int kt, int level) { return level == 1 ? kt : key_bytes(kt) == 8 ? 2 : 0; }

template <typename F> hipError_t with_type(int kt, F &&f) {
  switch (kt) {
    case 0: return f(std::integral_constant<int, 0>{});
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_dist_segments(const DistPlan &d, const uint64_t *seg_off, uint64_t n, uint64_t merged,
                                uint64_t longest, char *w, hipStream_t s) {
  SegDistArgs a{};
  if (const hipError_t e = level_error_word(&a.err); e != hipSuccess) return e;
  a.off = seg_off;
  a.n_segs = d.n_segs;
  a.n = n;
  a.merged = merged;
  a.longest = longest;
  a.target = d.target;
  a.rl = d.rl[1];
  a.root_p = d.root_p;
  a.one_p = d.one_p;
  a.levels = (uint32_t)d.levels;
  a.tiled = d.tiled(1) ? 1u : 0u;
  a.ctr = (DistCounters *)(w + d.off_ctr);
  a.nodes = (DistNode *)(w + d.off_nodes[1]);
  a.ranges = (DistRange *)(w + d.off_ranges[1]);
  a.max_nodes = d.max_nodes[1];
  a.max_ranges = d.max_ranges[1];
  a.max_cols = d.max_cols;
  a.max_table = d.max_table[1];
  hipLaunchKernelGGL(seg_dist_plan_kernel, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_dist_sample(int kt, const DistPlan &d, int level, const DistBufs &b, uint64_t n,
                              char *w, hipStream_t s) {
  Level L = level_args(kt, d, level, w);
  if (level == 1 && !d.n_segs) {
    L.root_len = (uint32_t)n;
    L.root_p = d.root_p;
  }
  const dim3 grid(d.max_nodes[level]);
  return with_type(level_type(kt, level), [&](auto c) {
    constexpr int KT = decltype(c)::value;
    using U = typename Key<KT>::U;
    const U *src = (const U *)level_src(d, b, level);
    // 64 samples a bucket fit a tile of 2048 up to 32 buckets, which short
    // segments take: many of its workgroups fit a CU at once; 16384 samples for a root whose buckets are cut again
    // (their evenness decides how many buckets the next level can give each)
    const uint32_t few = 32, all = kDistMaxPicks;
    auto go = [&](auto nt, uint32_t lo, uint32_t hi) -> hipError_t {
      constexpr int NT = decltype(nt)::value;
      hipLaunchKernelGGL((dist_sample_kernel<KT, NT>), grid, dim3(NT), 0, s, src, L, lo, hi);
      return hipGetLastError();
    };
    using N128 = std::integral_constant<int, 128>;
    using N512 = std::integral_constant<int, 512>;
    using N1024 = std::integral_constant<int, 1024>;
    if (L.root_len)
      return d.root_p <= few ? go(N128{}, 0, all) : d.levels > 1 ? go(N1024{}, 0, all) : go(N512{}, 0, all);
    // (nodes of later levels are much alike, so one launch does when they need
    // the large tile)
    if (level > 1 && d.root_p > few) return go(N512{}, 0, all);
    const hipError_t e = go(N128{}, 0, few);
    if (e != hipSuccess) return e;
    return go(N512{}, few + 1, all);
  });
}

hipError_t launch_dist_count(int kt, const DistPlan &d, int level, const DistBufs &b, char *w,
                             hipStream_t s) {
  Level L = level_args(kt, d, level, w);
  return with_type(level_type(kt, level), [&](auto c) {
    constexpr int KT = decltype(c)::value;
    using U = typename Key<KT>::U;
    hipLaunchKernelGGL((dist_count_kernel<KT>), dim3(d.max_ranges[level]), dim3(kDistThreads), 0, s,
                       (const U *)level_src(d, b, level), L);
    return hipGetLastError();
  });
}

hipError_t launch_dist_scan(int kt, const DistPlan &d, int level, char *w, hipStream_t s) {
  Level L = level_args(kt, d, level, w);
  if (const hipError_t e = level_error_word(&L.err); e != hipSuccess) return e;
  const int columns = level == 1 && d.levels > 1 && !d.n_segs && !d.tiled(level);
  const int summed = columns || (d.tiled(level) && level < d.levels);
  if (columns) {
    hipLaunchKernelGGL(dist_columns_kernel, dim3((kDistSlots + 3) / 4), dim3(256), 0, s, L);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (key_bytes(kt) == 8)
    hipLaunchKernelGGL((dist_scan_kernel<uint64_t>), dim3(d.max_nodes[level]), dim3(kDistSlots), 0, s,
                       L, summed);
  else
    hipLaunchKernelGGL((dist_scan_kernel<uint32_t>), dim3(d.max_nodes[level]), dim3(kDistSlots), 0, s,
                       L, summed);
  return hipGetLastError();
}

hipError_t launch_dist_scatter(int kt, bool kv, const DistPlan &d, int level, const DistBufs &b,
                               char *w, hipStream_t s) {
  Level L = level_args(kt, d, level, w);
  const uint32_t *vsrc = level_vsrc(d, b, level);
  void *dst = level_to_out(d, level) ? b.out : b.ws;
  uint32_t *vdst = level_to_out(d, level) ? b.vout : b.vws;
  return with_type(level_type(kt, level), [&](auto c) {
    constexpr int KT = decltype(c)::value;
    using U = typename Key<KT>::U;
    const U *src = (const U *)level_src(d, b, level);
    if (kv)
      hipLaunchKernelGGL((dist_scatter_kernel<KT, true>), dim3(d.max_ranges[level]),
                         dim3(kDistThreads), 0, s, src, vsrc, (U *)dst, vdst, L);
    else
      hipLaunchKernelGGL((dist_scatter_kernel<KT, false>), dim3(d.max_ranges[level]),
                         dim3(kDistThreads), 0, s, src, vsrc, (U *)dst, vdst, L);
    return hipGetLastError();
  });
}

hipError_t launch_dist_partition(int kt, bool kv, const DistPlan &d, int level, const DistBufs &b,
                                 char *w, hipStream_t s) {
  Level L = level_args(kt, d, level, w);
  const uint32_t *vsrc = level_vsrc(d, b, level);
  void *dst = level_to_out(d, level) ? b.out : b.ws;
  uint32_t *vdst = level_to_out(d, level) ? b.vout : b.vws;
  // (buckets that are only brought to their place are rare)
  const uint32_t ranges = d.max_ranges[level] - (level == d.levels ? d.max_copies : 0);
  const dim3 grid((ranges + std::min<uint32_t>(d.max_copies, 64) + kXcds - 1) / kXcds * kXcds);
  return with_type(level_type(kt, level), [&](auto c) {
    constexpr int KT = decltype(c)::value;
    using U = typename Key<KT>::U;
    const U *src = (const U *)level_src(d, b, level);
    auto go = [&](auto with_values, auto gather) -> hipError_t {
      hipLaunchKernelGGL((dist_partition_kernel<KT, decltype(with_values)::value, decltype(gather)::value>),
                         grid, dim3(kDistThreads), 0, s, src, vsrc, (U *)dst, vdst, L);
      return hipGetLastError();
    };
    if constexpr (KT == 0 || KT == 2) {  // (mapped keys)
      if (L.gather) return kv ? go(std::true_type{}, std::true_type{}) : go(std::false_type{}, std::true_type{});
    }
    return kv ? go(std::true_type{}, std::false_type{}) : go(std::false_type{}, std::false_type{});
  });
}

hipError_t launch_dist_pieces(int kt, const DistPlan &d, int level, char *w, hipStream_t s) {
  Level L = level_args(kt, d, level, w);
  // a workgroup a bucket for one array; segments are shorter
  hipLaunchKernelGGL(dist_pieces_kernel, dim3(d.max_nodes[level], d.max_nodes[level] > 1 ? 16 : kDistSlots),
                     dim3(kPiecesThreads), 0, s, L);
  return hipGetLastError();
}

hipError_t launch_dist_leaves(int kt, bool kv, const DistPlan &d, const DistBufs &b, char *w,
                              hipStream_t s) {
  Level L = level_args(kt, d, d.levels, w);
  if (const hipError_t e = level_error_word(&L.err); e != hipSuccess) return e;
  const dim3 grid(d.leaf_grid);
  return with_type(kt, [&](auto c) {
    constexpr int KT = decltype(c)::value;
    using U = typename Key<KT>::U;
    if (kv)
      // (8 keys a thread: LDS holds three workgroups a CU, which with 256
      // threads of 16 keys left it 12 waves; 1069 against 1001 us at 2^27 u64.
      // Keys-only leaves fill two workgroups' LDS, and 1024 threads of 8 keys
      // measured slower there, 1632 against 1487 us at 2^28 int64.)
      hipLaunchKernelGGL((dist_leaf_kernel<KT, true, 512, 8, 6>), grid, dim3(512), 0, s, (const U *)b.ws,
                         b.vws, (U *)b.out, b.vout, L);
    else
      hipLaunchKernelGGL((dist_leaf_kernel<KT, false, 512, 16, 4>), grid, dim3(512), 0, s, (const U *)b.ws,
                         b.vws, (U *)b.out, b.vout, L);
    return hipGetLastError();
  });
}

hipError_t launch_dist_rest(int kt, bool kv, const DistPlan &d, const DistBufs &b, char *w,
                            hipStream_t s) {
  Level L = level_args(kt, d, d.levels, w);
  // workgroups claim tasks as long as there are any: usually none
  const dim3 grid(std::min<uint32_t>(d.max_rest, 768));
  return with_type(kt, [&](auto c) {
    constexpr int KT = decltype(c)::value;
    using U = typename Key<KT>::U;
    if (kv)
      hipLaunchKernelGGL((dist_rest_kernel<KT, true, 512, 8, 6>), grid, dim3(512), 0, s, (U *)b.ws, b.vws,
                         (U *)b.out, b.vout, L);
    else
      hipLaunchKernelGGL((dist_rest_kernel<KT, false, 512, 16, 4>), grid, dim3(512), 0, s, (U *)b.ws, b.vws,
                         (U *)b.out, b.vout, L);
    return hipGetLastError();
  });
}

}  // namespace pss
