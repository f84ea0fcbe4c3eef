// Internal helpers shared by the HIP sources of libdsmpnn (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <mutex>
#include <string>
#include <vector>
#include <algorithm>
#include <cstdio>
#include <cstdarg>

#include "../../include/dsmpnn.h"

struct dsmp_handle {
  int device = 0;
  hipStream_t stream = nullptr;
  int edge_algo = 0;   // DSMP_EDGE_AUTO / PER_EDGE / AGGREGATE
  int n_cu = 256;      // compute units of the device (sizes persistent grids)
  void* sample_scratch = nullptr;   // device address of the allocation-free sampling scratch
  // READBACK_BYTES of pinned host memory (allocated at creation) that kernels
  // write small results to for the calls that synchronise, and its device
  // address.  A call holds readback_mu from the launch of the kernel that writes
  // there until it has read the values: calls of other threads on the handle
  // would otherwise leave their totals, which are used as sizes, in its place.
  void* readback = nullptr;
  void* readback_dev = nullptr;
  std::mutex readback_mu;
  std::string err;
  std::mutex err_mu;   // two threads' calls may fail at once
  // kernel timing (opt-in)
  struct Mark {
    int cls;
    hipEvent_t a, b;
  };
  bool prof = false;
  std::vector<Mark> pending;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
  double tot_ms[DSMP_K_COUNT] = {};
  int64_t launches[DSMP_K_COUNT] = {};
};

namespace dsmp {

// Brackets the launches issued in its scope with a pair of events when the
// handle's timing is on.
struct ProfScope {
  dsmp_handle* h;
  int idx = -1;
  ProfScope(dsmp_handle* hh, int cls) : h(hh) {
    if (!h || !h->prof) return;
    std::pair<hipEvent_t, hipEvent_t> ev;
    if (!h->pool.empty()) {
      ev = h->pool.back();
      h->pool.pop_back();
    } else if (hipEventCreate(&ev.first) != hipSuccess || hipEventCreate(&ev.second) != hipSuccess) {
      return;
    }
    if (hipEventRecord(ev.first, h->stream) != hipSuccess) {
      h->pool.push_back(ev);
      return;
    }
    h->pending.push_back({cls, ev.first, ev.second});
    idx = (int)h->pending.size() - 1;
  }
  void end() {
    if (idx >= 0) (void)hipEventRecord(h->pending[idx].b, h->stream);
    idx = -1;
  }
  ~ProfScope() { end(); }
};

inline dsmp_status fail(dsmp_handle* h, dsmp_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  if (h) {
    std::lock_guard<std::mutex> lock(h->err_mu);
    h->err = buf;
  }
  return st;
}

#define DSMP_HIP(h, call)                                                              \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess)                                                              \
      return ::dsmp::fail((h), DSMP_HIP_ERROR, "%s failed: %s", #call,                 \
                          hipGetErrorString(e_));                                      \
  } while (0)

#define DSMP_LAUNCHED(h, what)                                                         \
  do {                                                                                 \
    hipError_t e_ = hipGetLastError();                                                 \
    if (e_ != hipSuccess)                                                              \
      return ::dsmp::fail((h), DSMP_HIP_ERROR, "launch of %s failed: %s", (what),      \
                          hipGetErrorString(e_));                                      \
  } while (0)

#define DSMP_CHECK(h, cond, st, ...)                                                   \
  do {                                                                                 \
    if (!(cond)) return ::dsmp::fail((h), (st), __VA_ARGS__);                          \
  } while (0)

// Bump allocator over a caller workspace; every sub-buffer is 256-byte aligned.
struct Carve {
  uintptr_t base;
  size_t off = 0;
  explicit Carve(void* p) : base(reinterpret_cast<uintptr_t>(p)) {}
  template <typename T>
  T* take(size_t count) {
    off = (off + 255) & ~size_t(255);
    T* p = reinterpret_cast<T*>(base + off);
    off += count * sizeof(T);
    return p;
  }
  size_t used() const { return (off + 255) & ~size_t(255); }
};

inline unsigned ceil_div(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

constexpr size_t READBACK_BYTES = 64;

// Exclusive scan over a workgroup of 1,024 threads (sh: 32 words of LDS, free
// again when it returns).
__device__ __forceinline__ uint32_t block_exclusive_scan_1024(uint32_t v, uint32_t* sh,
                                                             uint32_t* total) {
  // 1024 threads = 16 waves; wave scans by shuffles, then a scan of wave sums.
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  if (wid == 0) {
    uint32_t s = lane < 16 ? sh[lane] : 0u;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      uint32_t y = __shfl_up(s, o, 64);
      if (lane >= o) s += y;
    }
    if (lane < 16) sh[16 + lane] = s;
  }
  __syncthreads();
  uint32_t wave_off = wid > 0 ? sh[16 + wid - 1] : 0u;
  *total = sh[31];
  uint32_t r = wave_off + x - v;
  __syncthreads();
  return r;
}

// Device-wide exclusive scan of n uint32 counts into out[0..n] (out[n] = total),
// in one launch (up to 16,384), two (per-block sums, then per-block scans that
// add up the sums ahead of them) or, above 4 M, three (a scan of the sums
// between).  tmp needs scan_tmp_elems(n) uint32.
constexpr int SCAN_BLOCK = 1024;
inline size_t scan_tmp_elems(int64_t n) { return (size_t)ceil_div(n, SCAN_BLOCK) + 1; }
dsmp_status exclusive_scan_u32(dsmp_handle* h, const uint32_t* in, int32_t* out, int64_t n,
                               uint32_t* tmp);

// Fill n uint32 words with a value (a kernel, not a memset node).
// p[0..n) = v, and q[0..n) = v in the same launch when q is given
dsmp_status fill_u32(dsmp_handle* h, uint32_t* p, int64_t n, uint32_t v, uint32_t* q = nullptr);

// SplitMix64 output number c+1 after seeding the state with `seed`
// (Steele, Lea, Flood, OOPSLA 2014; Stafford's Mix13 finaliser).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t c) {
  uint64_t z = seed + (c + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// The counter c of splitmix64(seed, c) == z, step by step backwards (the
// multipliers are the inverses of those above modulo 2^64).
__device__ __forceinline__ uint64_t splitmix64_counter(uint64_t seed, uint64_t z) {
  z ^= (z >> 31) ^ (z >> 62);
  z *= 0x319642B2D24D8EC3ull;
  z ^= (z >> 27) ^ (z >> 54);
  z *= 0x96DE1B173F119089ull;
  z ^= (z >> 30) ^ (z >> 60);
  return (z - seed) * 0xF1DE83E19937733Dull - 1ull;
}

}  // namespace dsmp
