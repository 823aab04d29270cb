// A CPU stand-in for the HIP runtime: the library's sources compile against it
// with g++ and run their kernels on the host, where the address and
// undefined-behaviour sanitizers check every access.
//
// One workgroup runs at a time.  Each of its threads is a fiber that runs to
// its next wave operation (ballot, shuffle, DPP move, wave barrier) or workgroup
// barrier; a wave's 64 threads go through their operations together, and the
// waves of a workgroup run one after the other from barrier to barrier, in an
// order that emu::seed chooses.  A barrier missing between two waves' accesses
// therefore shows as one wave seeing all or nothing of what another did.
// __shared__ variables are static; threads that return early take no part in
// later operations, as on the device.  Streams are synchronous.
#pragma once
#include <sys/mman.h>

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
  uint32_t x, y, z;
  dim3(uint32_t a = 1, uint32_t b = 1, uint32_t c = 1) : x(a), y(b), z(c) {}
};
struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

extern "C" void emu_switch(void **save, void *to);
asm(R"(
.text
.globl emu_switch
.weak emu_switch
emu_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");

namespace emu {
inline uint32_t seed = 0;  // 0: waves and workgroups in ascending order

enum State { kRun, kWave, kBlock, kDone };
struct Lane {
  void *sp;
  State state;
  uint32_t ops;  // wave operations so far
};
struct Wave {
  uint64_t val[2][64];
};
constexpr size_t kStack = 256 << 10;
inline char *stacks = nullptr;
inline Lane lanes[1024];
inline Wave waves[16];
inline void *scheduler_sp;
inline uint32_t cur, or_value;
inline void (*body_fn)(void *);
inline void *body_arg;

[[noreturn]] inline void fail(const char *what) {
  std::fprintf(stderr, "emulation: %s (workgroup %u, thread %u)\n", what, blockIdx.x, cur);
  std::abort();
}
inline void yield(State s) {
  lanes[cur].state = s;
  emu_switch(&lanes[cur].sp, scheduler_sp);
}
inline void entry() {
  body_fn(body_arg);
  yield(kDone);
  fail("a finished thread ran on");
}
inline uint32_t mix(uint32_t x) {
  x = (x ^ seed) * 0x9E3779B1u;
  x = (x ^ x >> 15) * 0x85EBCA6Bu;
  return x ^ x >> 13;
}
// i-th of n in the chosen order: a rotation, possibly reversed
inline uint32_t order(uint32_t i, uint32_t n, uint32_t salt) {
  if (!seed) return i;
  const uint32_t r = mix(salt), at = (uint32_t)(((uint64_t)i + r) % n);
  return r & 0x10000u ? n - 1 - at : at;
}

inline void run_lane(uint32_t t) {
  cur = t;
  threadIdx = dim3(t % blockDim.x, t / blockDim.x);
  lanes[t].state = kRun;
  emu_switch(&scheduler_sp, lanes[t].sp);
}
// Runs a wave until its threads wait at the workgroup's barrier or are done.
inline bool run_wave(uint32_t w, uint32_t threads) {
  const uint32_t lo = w * 64, hi = lo + 64 < threads ? lo + 64 : threads;
  for (;;) {
    uint32_t n[4] = {};
    for (uint32_t t = lo; t < hi; ++t) {
      if (lanes[t].state != kDone) run_lane(t);
      ++n[lanes[t].state];
    }
    if (n[kWave] && n[kBlock]) fail("threads of one wave at different operations");
    if (!n[kWave]) return n[kBlock] != 0;
  }
}
inline void run_block(uint32_t threads) {
  if (!stacks) {
    stacks = (char *)mmap(nullptr, kStack * 1024, PROT_READ | PROT_WRITE,
                          MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (stacks == MAP_FAILED) std::abort();
  }
  if (threads > 1024 || threads == 0) fail("workgroup size");
  for (uint32_t t = 0; t < threads; ++t) {
    void **top = (void **)(stacks + kStack * (t + 1) - 64);
    top[0] = (void *)&entry;  // returned to with the stack as after a call
    lanes[t] = Lane{(void *)(top - 6), kRun, 0};
    for (int i = 1; i <= 6; ++i) top[-i] = nullptr;
  }
  const uint32_t nw = (threads + 63) / 64;
  for (uint32_t phase = 0;; ++phase) {
    bool more = false;
    for (uint32_t i = 0; i < nw; ++i) more |= run_wave(order(i, nw, blockIdx.x * 977u + phase), threads);
    if (!more) return;
  }
}
template <typename F> void launch(dim3 grid, dim3 block, F body) {
  gridDim = grid;
  blockDim = block;
  body_fn = [](void *p) { (*(F *)p)(); };
  body_arg = &body;
  const uint64_t n = (uint64_t)grid.x * grid.y;
  for (uint64_t i = 0; i < n; ++i) {
    const uint32_t b = order((uint32_t)i, (uint32_t)n, 1u);
    blockIdx = dim3(b % grid.x, b / grid.x);
    run_block(block.x * block.y);
  }
}

// Leaves this thread's value for its wave; returns all 64 after every thread of
// the wave came here.
inline const uint64_t *exchange(uint64_t v) {
  const uint32_t t = cur;
  uint64_t *buf = waves[t / 64].val[lanes[t].ops & 1];
  buf[t % 64] = v;
  yield(kWave);
  ++lanes[t].ops;
  return buf;
}
inline bool live(uint32_t lane) {
  const uint32_t t = cur / 64 * 64 + lane;
  return t < blockDim.x * blockDim.y && lanes[t].state != kDone;
}
template <typename T> uint64_t bits(T v) {
  uint64_t b = 0;
  std::memcpy(&b, &v, sizeof v);
  return b;
}
template <typename T> T value(uint64_t b) {
  T v;
  std::memcpy(&v, &b, sizeof v);
  return v;
}
template <typename T> T from_lane(T v, uint32_t lane) {
  const uint64_t *a = exchange(bits(v));
  return live(lane) ? value<T>(a[lane]) : v;
}
}  // namespace emu

#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
  emu::launch(grid, block, [&] { (kernel)(__VA_ARGS__); })

inline void __syncthreads() { emu::yield(emu::kBlock); }
inline int __syncthreads_or(int x) {
  static int any;
  any |= x != 0;
  __syncthreads();
  const int r = any;
  __syncthreads();
  any = 0;  // (all have read it, and none sets it again before the next barrier)
  __syncthreads();
  return r;
}
inline uint32_t __lane() { return emu::cur % 64; }
inline uint64_t __ballot(int p) {
  const uint64_t *a = emu::exchange(p != 0);
  uint64_t m = 0;
  for (uint32_t l = 0; l < 64; ++l)
    if (emu::live(l) && a[l]) m |= (uint64_t)1 << l;
  return m;
}
inline int __any(int p) { return __ballot(p) != 0; }
inline int __all(int p) { return __ballot(!p) == 0; }
template <typename T> T __shfl(T v, int lane, int = 64) { return emu::from_lane(v, (uint32_t)lane & 63); }
template <typename T> T __shfl_xor(T v, int d, int = 64) { return emu::from_lane(v, __lane() ^ (uint32_t)d); }
template <typename T> T __shfl_up(T v, int d, int = 64) {
  const uint32_t l = __lane();
  return emu::from_lane(v, l >= (uint32_t)d ? l - (uint32_t)d : l);
}
template <typename T> T __shfl_down(T v, int d, int = 64) {
  const uint32_t l = __lane();
  return emu::from_lane(v, l + (uint32_t)d < 64 ? l + (uint32_t)d : l);
}
inline uint32_t __builtin_amdgcn_readfirstlane(uint32_t v) {
  const uint64_t *a = emu::exchange(v);
  for (uint32_t l = 0; l < 64; ++l)
    if (emu::live(l)) return (uint32_t)a[l];
  return v;
}
// DPP moves with all banks enabled and no bound control: `old` where the source
// lane does not exist or the row is masked off
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int rows, int, bool) {
  const uint64_t *a = emu::exchange((uint32_t)v);
  const uint32_t l = __lane(), row = l / 16, i = l % 16;
  if (!(rows >> row & 1)) return old;
  int s = -1;
  if (ctrl <= 0xFF) s = (int)(l / 4 * 4 + (ctrl >> 2 * (l % 4) & 3));          // quad_perm
  else if (ctrl > 0x110 && ctrl < 0x120) s = (int)i - (ctrl & 15) >= 0 ? (int)l - (ctrl & 15) : -1;  // row_shr
  else if (ctrl > 0x120 && ctrl < 0x130) s = (int)(row * 16 + (i + 16 - (ctrl & 15)) % 16);  // row_ror
  else if (ctrl == 0x140) s = (int)(row * 16 + 15 - i);                        // row_mirror
  else if (ctrl == 0x141) s = (int)(l / 8 * 8 + 7 - l % 8);                    // row_half_mirror
  else if (ctrl == 0x142) s = row > 0 ? (int)(row * 16 - 1) : -1;              // row_bcast15
  else if (ctrl == 0x143) s = row > 1 ? 31 : -1;                               // row_bcast31
  else emu::fail("DPP control");
  return s < 0 || !emu::live((uint32_t)s) ? old : (int)(uint32_t)a[s];
}
inline int __builtin_amdgcn_ds_swizzle(int v, int pattern) {
  const uint32_t l = __lane(), in = l & 31;
  const uint32_t s = ((in & (pattern & 31)) | (pattern >> 5 & 31)) ^ (pattern >> 10 & 31);
  return emu::from_lane(v, (l & 32) | s);
}
inline void __builtin_amdgcn_wave_barrier() { (void)emu::exchange(0); }
inline void __builtin_amdgcn_fence(int, const char *) {}
inline void __threadfence() {}
inline void __builtin_amdgcn_s_sleep(int) {}
inline uint32_t __builtin_amdgcn_sad_u8(uint32_t a, uint32_t b, uint32_t c) {
  for (int i = 0; i < 32; i += 8) {
    const int x = (int)(a >> i & 255), y = (int)(b >> i & 255);
    c += (uint32_t)(x > y ? x - y : y - x);
  }
  return c;
}
template <typename T> T __builtin_nontemporal_load(const T *p) { return *p; }
template <typename T, typename V> void __builtin_nontemporal_store(V v, T *p) { *p = (T)v; }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __clz(uint32_t x) { return x ? __builtin_clz(x) : 32; }
inline int __clzll(long long x) { return x ? __builtin_clzll((unsigned long long)x) : 64; }
inline int __ffsll(unsigned long long x) { return __builtin_ffsll((long long)x); }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }
template <typename T, typename V> T atomicAdd(T *p, V v) { T o = *p; *p = o + (T)v; return o; }
template <typename T, typename V> T atomicOr(T *p, V v) { T o = *p; *p = o | (T)v; return o; }
template <typename T, typename V> T atomicMax(T *p, V v) { T o = *p; if ((T)v > o) *p = (T)v; return o; }
#define __HIP_MEMORY_SCOPE_AGENT 4
template <typename T> T __hip_atomic_load(const T *p, int, int) { return *p; }

// ---------------------------------------------------------- host runtime ---
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidDevice = 101,
                  hipErrorInvalidSymbol = 13, hipErrorNotSupported = 801, hipErrorLaunchFailure = 719 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocDefault = 0 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal };
typedef struct emu_stream *hipStream_t;
typedef struct emu_event *hipEvent_t;
typedef struct emu_graph *hipGraph_t;
typedef struct emu_graph_exec *hipGraphExec_t;
#define HIP_SYMBOL(x) (&(x))
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char *hipGetErrorName(hipError_t) { return "hipError"; }
inline const char *hipGetErrorString(hipError_t) { return "emulated"; }
inline hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
template <typename T> hipError_t hipGetSymbolAddress(void **p, T *s) { *p = (void *)s; return hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
inline hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
template <typename T> hipError_t hipMemcpyFromSymbol(void *d, T *s, size_t n, size_t, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
template <typename T> hipError_t hipMemcpyToSymbol(T *d, const void *s, size_t n, size_t, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
template <typename T> hipError_t hipMemcpyFromSymbolAsync(void *d, T *s, size_t n, size_t, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipErrorNotSupported; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorNotSupported; }
inline hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, void *, char *, size_t) { return hipErrorNotSupported; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
inline hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
