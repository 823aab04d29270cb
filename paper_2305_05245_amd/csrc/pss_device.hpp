// Device code shared by the kernel files: the order-preserving key maps,
// register sorting networks, chunk merges and the LDS sort of one tile.
#pragma once
#include "pss_dist.hpp"
#include "pss_internal.hpp"

namespace pss {
namespace {

// ------------------------------------------------------------------ K0 ----
template <int KT> struct Key;
template <> struct Key<0> {  // uint32
  using U = uint32_t;
  static __device__ __forceinline__ U map(U x) { return x; }
  static __device__ __forceinline__ U unmap(U x) { return x; }
};
template <> struct Key<1> {  // int32: flip the sign bit
  using U = uint32_t;
  static __device__ __forceinline__ U map(U x) { return x ^ 0x80000000u; }
  static __device__ __forceinline__ U unmap(U x) { return x ^ 0x80000000u; }
};
template <> struct Key<2> {  // uint64
  using U = uint64_t;
  static __device__ __forceinline__ U map(U x) { return x; }
  static __device__ __forceinline__ U unmap(U x) { return x; }
};
template <> struct Key<3> {  // int64
  using U = uint64_t;
  static __device__ __forceinline__ U map(U x) { return x ^ 0x8000000000000000ull; }
  static __device__ __forceinline__ U unmap(U x) { return x ^ 0x8000000000000000ull; }
};
template <> struct Key<4> {  // float32, IEEE totalOrder: negative -> all bits
  using U = uint32_t;        // inverted, otherwise the sign bit set
  static __device__ __forceinline__ U map(U x) {
    return (x & 0x80000000u) ? ~x : (x | 0x80000000u);
  }
  static __device__ __forceinline__ U unmap(U x) {
    return (x & 0x80000000u) ? (x & 0x7fffffffu) : ~x;
  }
};
template <> struct Key<5> {  // float64, IEEE totalOrder
  using U = uint64_t;
  static __device__ __forceinline__ U map(U x) {
    return (x & 0x8000000000000000ull) ? ~x : (x | 0x8000000000000000ull);
  }
  static __device__ __forceinline__ U unmap(U x) {
    return (x & 0x8000000000000000ull) ? (x & 0x7fffffffffffffffull) : ~x;
  }
};

template <typename U>
__device__ __forceinline__ U unmap_runtime(U x, int kt) {
  if constexpr (sizeof(U) == 4) {
    switch (kt) {
      case 1: return Key<1>::unmap(x);
      case 4: return Key<4>::unmap(x);
      default: return x;
    }
  } else {
    switch (kt) {
      case 3: return Key<3>::unmap(x);
      case 5: return Key<5>::unmap(x);
      default: return x;
    }
  }
}

template <typename U> __device__ __forceinline__ constexpr U key_max() { return ~U(0); }

// The same value, hidden from the optimiser (an empty asm that "changes" its
// register).  A compare-exchange written as two selects on one comparison
// would otherwise be rewritten as a minimum and a maximum, which the 64-bit
// lowering computes with one comparison each; selecting between opaque
// copies keeps one comparison for both selects.
template <typename U> __device__ __forceinline__ U opaque(U x) {
  asm("" : "+v"(x));
  return x;
}

// LDS index with one pad slot after every 16 keys, so that a thread reading or
// writing its 16 consecutive keys does not hit the same bank as its neighbours.
__device__ __forceinline__ uint32_t pad16(uint32_t i) { return i + (i >> 4); }

// Order LDS accesses within one wave: everything this wave wrote before is
// visible to everything it reads after (no other wave takes part).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ----------------------------------------------------- sorting networks ----
// Index pairs of Batcher's odd-even merge sort on N registers (unstable,
// keys only) and of odd-even transposition sort (stable: only neighbours are
// compared and equal keys are never swapped), generated at compile time.
template <int N> constexpr int batcher_pairs() {
  int c = 0;
  for (int p = 1; p < N; p <<= 1)
    for (int k = p; k >= 1; k >>= 1)
      for (int j = k % p; j + k < N; j += 2 * k)
        for (int i = 0; i < k && i + j + k < N; ++i)
          if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) ++c;
  return c;
}
template <int N> struct BatcherNet {
  int a[batcher_pairs<N>()];
  int b[batcher_pairs<N>()];
  constexpr BatcherNet() : a(), b() {
    int c = 0;
    for (int p = 1; p < N; p <<= 1)
      for (int k = p; k >= 1; k >>= 1)
        for (int j = k % p; j + k < N; j += 2 * k)
          for (int i = 0; i < k && i + j + k < N; ++i)
            if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) {
              a[c] = i + j;
              b[c] = i + j + k;
              ++c;
            }
  }
};
template <int N> constexpr int transposition_pairs() { return (N / 2) * ((N + 1) / 2) + ((N - 1) / 2) * (N / 2); }
template <int N> struct TranspositionNet {
  int a[transposition_pairs<N>()];
  constexpr TranspositionNet() : a() {
    int c = 0;
    for (int phase = 0; phase < N; ++phase)
      for (int i = phase & 1; i + 1 < N; i += 2) a[c++] = i;
  }
};

template <typename U, bool KV, int N>
__device__ __forceinline__ void register_sort(U (&k)[N], uint32_t (&v)[KV ? N : 1]) {
  if constexpr (!KV) {
    constexpr BatcherNet<N> net{};
#pragma unroll
    for (int c = 0; c < batcher_pairs<N>(); ++c) {
      const U x = k[net.a[c]], y = k[net.b[c]];
      const bool lt = x < y;
      const U ox = opaque(x), oy = opaque(y);
      k[net.a[c]] = lt ? ox : oy;
      k[net.b[c]] = lt ? oy : ox;
    }
  } else {
    constexpr TranspositionNet<N> net{};
#pragma unroll
    for (int c = 0; c < transposition_pairs<N>(); ++c) {
      const int i = net.a[c];
      const bool s = k[i + 1] < k[i];
      const U x = k[i], y = k[i + 1];
      const uint32_t vx = v[i], vy = v[i + 1];
      k[i] = s ? y : x;
      k[i + 1] = s ? x : y;
      v[i] = s ? vy : vx;
      v[i + 1] = s ? vx : vy;
    }
  }
}

// Largest s in [0, n_segs) with prefix[s] <= idx (prefix[0] = 0): the segment
// whose range of a prefix-summed count contains idx.
__device__ __forceinline__ uint32_t seg_find(const uint64_t *prefix, uint32_t n_segs, uint64_t idx) {
  uint32_t lo = 0, hi = n_segs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (prefix[mid] <= idx) lo = mid;
    else hi = mid;
  }
  return lo;
}

// LDS slot of index i: the padded layout (one spare slot after every 16, for
// phases where each thread reads or writes 16 consecutive slots) or flat.
template <bool PAD> __device__ __forceinline__ uint32_t lds_at(uint32_t i) {
  return PAD ? pad16(i) : i;
}

// One chunk of a stable pairwise merge in LDS: the CI outputs from `start` on
// of merging A = [A0, A1) and B = [A1, B1) (ties to A), into registers.  The
// merge-path search finds how many of the first start-A0 outputs come from A;
// then one output per step.  Outputs at or past B1 (only in a pair's last
// chunk) are meaningless and must not be stored; computing them reads at
// most CI slots past B1, which every LDS array using this leaves as slack.
template <typename U, bool KV, int CI, bool PAD>
__device__ __forceinline__ void merge_chunk(const U *sk, const uint32_t *sv, uint32_t A0,
                                            uint32_t A1, uint32_t B1, uint32_t start,
                                            U (&rk)[CI], uint32_t (&rv)[KV ? CI : 1]) {
  const uint32_t la = A1 - A0, lb = B1 - A1, d = start - A0;
  uint32_t lo = d > lb ? d - lb : 0, hi = d < la ? d : la;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (sk[lds_at<PAD>(A0 + mid)] <= sk[lds_at<PAD>(A1 + d - 1 - mid)]) lo = mid + 1;
    else hi = mid;
  }
  uint32_t pa = A0 + lo, pb = A1 + (d - lo);
  U ka = sk[lds_at<PAD>(pa)], kb = sk[lds_at<PAD>(pb)];
  uint32_t va = 0, vb = 0;
  if constexpr (KV) {
    va = sv[lds_at<PAD>(pa)];
    vb = sv[lds_at<PAD>(pb)];
  }
#pragma unroll
  for (int i = 0; i < CI; ++i) {
    const bool takeA = pa < A1 && (pb >= B1 || ka <= kb);
    rk[i] = takeA ? ka : kb;
    if constexpr (KV) rv[i] = takeA ? va : vb;
    const uint32_t nxt = (takeA ? pa : pb) + 1;
    const U nk = sk[lds_at<PAD>(nxt)];
    ka = takeA ? nk : ka;
    kb = takeA ? kb : nk;
    if constexpr (KV) {
      const uint32_t nv = sv[lds_at<PAD>(nxt)];
      va = takeA ? nv : va;
      vb = takeA ? vb : nv;
    }
    pa += takeA ? 1u : 0u;
    pb += takeA ? 0u : 1u;
  }
}

// Keys-only chunk merge of two runs that are each followed in LDS by at least
// CI copies of the largest key: A = sk[a0, a0 + la), B = sk[b0, b0 + lb).  It
// produces outputs d .. d+CI-1 of their merged order.  After the merge-path
// search, every step outputs the smaller of the two heads and replaces it with
// the next key of its run.  Equal keys are bit-identical, so which run
// supplies a tie does not change the output; a used-up run shows the largest
// key from its gap, so no bound checks are needed, and a chunk reads at most
// CI slots past the end of a run.
template <typename U, int CI>
__device__ __forceinline__ void merge_chunk_keys(const U *sk, uint32_t a0, uint32_t la,
                                                 uint32_t b0, uint32_t lb, uint32_t d,
                                                 U (&rk)[CI]) {
  uint32_t lo = d > lb ? d - lb : 0, hi = d < la ? d : la;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (sk[a0 + mid] <= sk[b0 + d - 1 - mid]) lo = mid + 1;
    else hi = mid;
  }
  // positions as LDS byte offsets, so a step needs no index arithmetic
  const uint32_t pa = (a0 + lo) * (uint32_t)sizeof(U), pb = (b0 + (d - lo)) * (uint32_t)sizeof(U);
  const char *base = reinterpret_cast<const char *>(sk);
  const U ka = *reinterpret_cast<const U *>(base + pa);
  const U kb = *reinterpret_cast<const U *>(base + pb);
  const bool af = ka <= kb;
  U x = af ? ka : kb, y = af ? kb : ka;  // x: the next output, y: the other head
  uint32_t px = af ? pa : pb, py = af ? pb : pa;
#pragma unroll
  for (int i = 0; i < CI; ++i) {
    rk[i] = x;
    const uint32_t pn = px + (uint32_t)sizeof(U);
    const U nk = *reinterpret_cast<const U *>(base + pn);
    const bool keep = nk <= y;
    const U onk = opaque(nk), oy = opaque(y);
    const U nx = keep ? onk : oy, ny = keep ? oy : onk;
    const uint32_t npx = keep ? pn : py, npy = keep ? py : pn;
    x = nx;
    y = ny;
    px = npx;
    py = npy;
  }
}

// Keys only: merge the sorted 16-key runs held by single lanes into sorted
// 128-key runs held by groups of eight lanes (lane j of a group then holds the
// run's keys 16j..16j+15), with bitonic merge networks: a "flip" stage pairs
// key i of the lower run with key n-1-i of the upper one across lanes, then
// half-cleaners at falling distances, the last four inside each lane.  Lane
// exchanges use DPP moves (quad permutations and the half-row mirror).
template <typename U>
__device__ __forceinline__ void inlane_half_cleaners(U (&k)[kTileItems]) {
#pragma unroll
  for (int d = kTileItems / 2; d >= 1; d >>= 1) {
#pragma unroll
    for (int i = 0; i < kTileItems; ++i) {
      if ((i & d) == 0) {
        const U a = k[i], b = k[i + d];
        const bool sw = b < a;
        const U oa = opaque(a), ob = opaque(b);
        k[i] = sw ? ob : oa;
        k[i + d] = sw ? oa : ob;
      }
    }
  }
}

// x from the lane given by the DPP control CTRL (all lanes active)
template <int CTRL, typename U>
__device__ __forceinline__ U dpp_from(U x) {
  if constexpr (sizeof(U) == 8) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, 0xF, 0xF, false);
    return ((U)(uint32_t)hi << 32) | (U)(uint32_t)lo;
  } else {
    return (U)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
  }
}

constexpr int kDppXor1 = 0xB1;  // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;  // quad_perm [2,3,0,1]
constexpr int kDppXor3 = 0x1B;  // quad_perm [3,2,1,0]
constexpr int kDppXor7 = 0x141; // row_half_mirror: lane i of 8 reads lane 7-i
constexpr int kDppRor8 = 0x128; // row_ror:8: lane i of 16 reads lane i xor 8

// x from lane (lane xor 16) within each half of the wave (swizzle unit)
template <typename T>
__device__ __forceinline__ T swizzle_xor16(T x) {
  constexpr int kPattern = (0x10 << 10) | 0x1F;  // bit mode: and 0x1f, or 0, xor 0x10
  if constexpr (sizeof(T) == 8) {
    const int lo = __builtin_amdgcn_ds_swizzle((int)(uint32_t)x, kPattern);
    const int hi = __builtin_amdgcn_ds_swizzle((int)(uint32_t)((uint64_t)x >> 32), kPattern);
    return (T)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
  } else {
    return (T)__builtin_amdgcn_ds_swizzle((int)x, kPattern);
  }
}

// x from lane (lane xor D): DPP moves for D <= 8 (xor 4 is the half-row
// mirror followed by the quad reversal), the swizzle unit for 16, a full
// cross-lane permute beyond
template <int D, typename T>
__device__ __forceinline__ T shfl_xor_c(T x) {
  if constexpr (D == 1) return dpp_from<kDppXor1>(x);
  else if constexpr (D == 2) return dpp_from<kDppXor2>(x);
  else if constexpr (D == 4) return dpp_from<kDppXor3>(dpp_from<kDppXor7>(x));
  else if constexpr (D == 8) return dpp_from<kDppRor8>(x);
  else if constexpr (D == 16) return swizzle_xor16(x);
  else return __shfl_xor(x, D, 64);
}

template <int CTRL, bool FLIP, typename U>
__device__ __forceinline__ void cross_lane_stage(U (&k)[kTileItems], bool upper) {
  U o[kTileItems];
#pragma unroll
  for (int i = 0; i < kTileItems; ++i) o[i] = dpp_from<CTRL>(k[FLIP ? kTileItems - 1 - i : i]);
#pragma unroll
  for (int i = 0; i < kTileItems; ++i) {
    const bool lt = o[i] < k[i];
    k[i] = (lt != upper) ? o[i] : k[i];  // lower lane keeps the minimum, upper the maximum
  }
}

template <typename U>
__device__ __forceinline__ void lane_runs_to_128(U (&k)[kTileItems], uint32_t lane) {
  cross_lane_stage<kDppXor1, true>(k, (lane & 1) != 0);  // runs of 16 -> 32
  inlane_half_cleaners(k);
  cross_lane_stage<kDppXor3, true>(k, (lane & 2) != 0);  // runs of 32 -> 64
  cross_lane_stage<kDppXor1, false>(k, (lane & 1) != 0);
  inlane_half_cleaners(k);
  cross_lane_stage<kDppXor7, true>(k, (lane & 4) != 0);  // runs of 64 -> 128
  cross_lane_stage<kDppXor2, false>(k, (lane & 2) != 0);
  cross_lane_stage<kDppXor1, false>(k, (lane & 1) != 0);
  inlane_half_cleaners(k);
}

// ------------------------------------------------- LDS sort of one tile ---
// LDS slots of a tile of THREADS * 16 keys.  Key-value tiles: the padded
// layout.  Keys-only tiles: also every wave's region of RW slots, in which
// its 1024 keys sit padded at first and later as runs followed by gaps of
// the largest key.  Both plus the slack a merge chunk may read.
template <bool KV, int THREADS> struct TileLds {
  static constexpr uint32_t TILE = THREADS * kTileItems;
  static constexpr uint32_t RW = 64 * kTileItems + (64 * kTileItems / 256) * kGap;
  static constexpr uint32_t PADDED = TILE + TILE / 16;
  static constexpr uint32_t GAPPED = (THREADS / 64) * RW;
  static constexpr uint32_t SLOTS = (KV || PADDED > GAPPED ? PADDED : GAPPED) + 2 * kRoundItems + 2;
};

// Padded slot of tile position idx (one spare slot per 16 keys); keys-only
// tiles place each wave's 1024 keys at the start of that wave's region.
template <bool KV> __device__ __forceinline__ uint32_t tile_slot(uint32_t idx) {
  return KV ? pad16(idx) : (idx >> 10) * TileLds<KV, 64>::RW + pad16(idx & 1023u);
}

// Stable sort of a key-value tile of ITEMS (16 or 8) keys a thread.  Thread t holds
// the tile's consecutive positions from ITEMS t on, which it read from its own
// padded LDS slots; the sorted tile is left in sk / sv at flat slots 0 .. TILE-1
// (all threads past a barrier).
//
// SHORT (here and below): the tile holds len keys only, and waves whose 64 ITEMS
// positions all lie past them do nothing but wait; the tile is left sorted up to
// the last position of the last wave that has keys.  tid: the thread's index, for
// a caller that hides it from the optimiser (see dist_rest_kernel).
template <typename U, int THREADS, bool SHORT = false, int ITEMS = kTileItems>
__device__ __forceinline__ void lds_sort_pairs(U (&rk)[ITEMS], uint32_t (&rv)[ITEMS], U *sk,
                                               uint32_t *sv, uint32_t len = THREADS * ITEMS,
                                               uint32_t tid = threadIdx.x) {
  constexpr uint32_t TILE = THREADS * ITEMS;
  constexpr uint32_t WKEYS = 64 * ITEMS;  // keys per wave
  const uint32_t end = SHORT ? (len + WKEYS - 1) / WKEYS * WKEYS : TILE;
  const bool on = !SHORT || (tid >> 6) * WKEYS < end;
  if (on) {
    register_sort<U, true, ITEMS>(rk, rv);
    // every wave writes back the keys it read (its own positions)
    wave_sync();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint32_t idx = tid * ITEMS + i;
      sk[pad16(idx)] = rk[i];
      sv[pad16(idx)] = rv[i];
    }
    wave_sync();
  }

  // Rounds of pairwise merges of runs of L keys.  Each pair's output is cut
  // into chunks of CI keys (never crossing into the next pair), one chunk per
  // thread: at most THREADS chunks per round.  The first round reads the
  // padded layout; every round writes the flat one (CI is odd, so the
  // threads' chunk stores do not collide in LDS banks).  While a pair fits in
  // the keys that one wave's threads sorted, each wave merges only its
  // own keys and, after the first round, synchronises only with itself.
  constexpr int CI = ITEMS + 1;
  U mk[CI];
  uint32_t mv[CI];
  const uint32_t lane = tid & 63, wbase = (tid >> 6) * WKEYS;
  uint32_t L = ITEMS;
  for (; L < TILE && 2 * L <= WKEYS; L *= 2) {
    const uint32_t cpp = (2 * L + CI - 1) / CI;  // chunks per pair
    const uint32_t q = lane / cpp, c = lane - q * cpp;
    const bool active = on && q < WKEYS / (2 * L);
    const uint32_t A0 = wbase + q * 2 * L;
    const uint32_t cs = A0 + c * CI;  // this thread's first output
    const uint32_t count = active ? (A0 + 2 * L - cs < (uint32_t)CI ? A0 + 2 * L - cs : CI) : 0;
    if (active) {
      if (L == ITEMS)
        merge_chunk<U, true, CI, true>(sk, sv, A0, A0 + L, A0 + 2 * L, cs, mk, mv);
      else
        merge_chunk<U, true, CI, false>(sk, sv, A0, A0 + L, A0 + 2 * L, cs, mk, mv);
    }
    // The first round moves every wave's keys from the padded layout to the
    // flat one, whose slots overlap the previous wave's padded ones: all
    // waves must finish reading first.  Later rounds stay in the wave's own
    // flat slots.
    if (L == ITEMS) __syncthreads();
    else wave_sync();
#pragma unroll
    for (int i = 0; i < CI; ++i) {
      if ((uint32_t)i < count) {
        sk[cs + i] = mk[i];
        sv[cs + i] = mv[i];
      }
    }
    wave_sync();
  }
  __syncthreads();
  for (; L < end; L *= 2) {
    const uint32_t cpp = (2 * L + CI - 1) / CI;  // chunks per pair
    const uint32_t q = tid / cpp, c = tid - q * cpp;
    const uint32_t A0 = q * 2 * L;
    const uint32_t cs = A0 + c * CI;  // this thread's first output
    // (SHORT: a run with no other one to merge with stays where it is)
    const uint32_t B1 = SHORT && end < A0 + 2 * L ? end : A0 + 2 * L;
    const bool active = SHORT ? A0 + L < end && cs < B1 : A0 < TILE;
    const uint32_t count = active ? (B1 - cs < (uint32_t)CI ? B1 - cs : CI) : 0;
    if (active) merge_chunk<U, true, CI, false>(sk, sv, A0, A0 + L, B1, cs, mk, mv);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CI; ++i) {
      if ((uint32_t)i < count) {
        sk[cs + i] = mk[i];
        sv[cs + i] = mv[i];
      }
    }
    __syncthreads();
  }
}

// Sort of a keys-only tile: any 16 keys of the tile per thread in rk; the
// sorted tile is left in sk at flat slots 0 .. TILE-1 (all threads past a
// barrier).
template <typename U, int THREADS, bool SHORT = false>
__device__ __forceinline__ void lds_sort_keys(U (&rk)[kTileItems], U *sk,
                                              uint32_t len = THREADS * kTileItems,
                                              uint32_t tid = threadIdx.x) {
  using T = TileLds<false, THREADS>;
  constexpr uint32_t TILE = T::TILE;
  constexpr uint32_t WKEYS = 64 * kTileItems;  // keys per wave
  const uint32_t end = SHORT ? (len + WKEYS - 1) / WKEYS * WKEYS : TILE;
  const bool on = !SHORT || (tid >> 6) * WKEYS < end;
  if (on) {
    uint32_t none[1];
    register_sort<U, false, kTileItems>(rk, none);
    // Keys only.  Runs of 128 are formed in registers (bitonic merges across
    // lanes), written to the padded layout of each thread's own 16 slots.
    lane_runs_to_128(rk, tid & 63);
    wave_sync();
#pragma unroll
    for (int i = 0; i < kTileItems; ++i) sk[tile_slot<false>(tid * kTileItems + i)] = rk[i];
    wave_sync();
  }
  // Then rounds of merge-path merges.  Round 128 reads the padded layout and
  // writes the gapped one, where every run is followed by kGap slots of the
  // largest key, so the later rounds use merge_chunk_keys (no bound
  // checks).  While a pair fits in one wave's 1024 keys, runs of length L
  // sit at q (L + G) in the wave's own region of RW slots and the wave
  // synchronises only with itself; larger rounds use runs at j (L + G)
  // across the tile.
  constexpr int CI = kRoundItems;
  constexpr uint32_t G = kGap;
  const uint32_t lane = tid & 63, wv = tid >> 6;
  U mk[CI];
  uint32_t dummy_v[1];
  uint32_t L = 128;
  for (; L < TILE && 2 * L <= WKEYS; L *= 2) {
    const uint32_t cpp = (2 * L + CI - 1) / CI;  // chunks per pair
    const uint32_t q = lane / cpp, c = lane - q * cpp;
    const bool active = on && q < WKEYS / (2 * L);
    const uint32_t o = c * CI;  // this chunk's first output within the pair
    const uint32_t count = active ? (2 * L - o < (uint32_t)CI ? 2 * L - o : CI) : 0u;
    const bool to_tile = 4 * L > WKEYS;  // the next round's pairs span waves
    const uint32_t dst = to_tile ? (wv * (WKEYS / (2 * L)) + q) * (2 * L + G)
                                 : wv * T::RW + q * (2 * L + G);
    if (active) {
      if (L == 128) {
        // padded layout of the wave's keys at the start of its region
        const uint32_t A0 = q * 2 * L;
        merge_chunk<U, false, CI, true>(sk + wv * T::RW, (const uint32_t *)nullptr, A0, A0 + L, A0 + 2 * L, A0 + o, mk,
                                        dummy_v);
      } else {
        const uint32_t A0 = wv * T::RW + 2 * q * (L + G);
        merge_chunk_keys<U, CI>(sk, A0, L, A0 + L + G, L, o, mk);
      }
    }
    // a round writing tile-wide runs leaves the wave's region
    if (to_tile) __syncthreads();
    else wave_sync();
    // every active chunk stores all CI keys: a pair's last chunk spills
    // into the run's new gap, which it then fills with the largest key
    if (active) {
#pragma unroll
      for (int i = 0; i < CI; ++i) sk[dst + o + i] = mk[i];
      if (o + count == 2 * L)
        for (uint32_t j = 0; j < G; ++j) sk[dst + 2 * L + j] = key_max<U>();
    }
    if (to_tile) __syncthreads();
    else wave_sync();
  }
  for (; L < end; L *= 2) {
    const uint32_t cpp = (2 * L + CI - 1) / CI;  // chunks per pair
    const uint32_t q = tid / cpp, c = tid - q * cpp;
    const uint32_t o = c * CI;
    // keys of the pair and of its second run (SHORT: of the last pair, and none
    // if it has no second run, which then reads the largest keys after the first)
    uint32_t pair = 2 * L, lb = L;
    if constexpr (SHORT) {
      const uint32_t left = 2 * q * L < end ? end - 2 * q * L : 0u;
      pair = left < 2 * L ? left : 2 * L;
      lb = pair > L ? pair - L : 0u;
    }
    const bool active = SHORT ? o < pair : q < TILE / (2 * L);
    const uint32_t count = active ? (pair - o < (uint32_t)CI ? pair - o : CI) : 0u;
    const uint32_t A0 = 2 * q * (L + G), dst = q * (2 * L + G);
    if (active) merge_chunk_keys<U, CI>(sk, A0, pair - lb, lb ? A0 + L + G : A0 + pair, lb, o, mk);
    __syncthreads();
    if (active) {
#pragma unroll
      for (int i = 0; i < CI; ++i) sk[dst + o + i] = mk[i];
      if (o + count == pair && (SHORT || 2 * L < TILE))
        for (uint32_t j = 0; j < G; ++j) sk[dst + pair + j] = key_max<U>();
    }
    __syncthreads();
  }
}

// ------------------------------------------- nodes of the distribution ---
// p of a node: its share of the buckets the remaining levels have to reach.
__device__ __forceinline__ uint32_t node_picks(uint32_t len, uint32_t target, int remaining) {
  const uint32_t units = (len + target - 1) / target;
  uint32_t p = units;
  if (remaining == 2) p = (uint32_t)ceilf(sqrtf((float)units));
  else if (remaining >= 3) p = (uint32_t)ceilf(cbrtf((float)units));
  return p < 2 ? 2 : (p > kDistMaxPicks ? kDistMaxPicks : p);
}

__device__ __forceinline__ uint32_t node_cols(uint32_t p) {
  return 2 * p < kDistSlots ? 2 * p : kDistSlots;
}

// Table entries per bucket: one a range, or (tiles in place) one a tile, padded so
// that every bucket's entries start on 16 bytes.
__device__ __forceinline__ uint32_t node_stride(uint32_t len, uint32_t nr, bool tiled) {
  return tiled ? ((len + kDistTile - 1) / kDistTile + 7) / 8 * 8 : nr;
}

}  // namespace
}  // namespace pss
