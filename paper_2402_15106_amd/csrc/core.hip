// Handle management, scan and fill utilities, node sampling and row gather.
#include "common.hpp"

#include <map>
#include <mutex>
#include <new>

using namespace dsmp;

// ------------------------------------------------------------------ scan

namespace {

__global__ __launch_bounds__(1024) void k_scan_blocksums(const uint32_t* __restrict__ in,
                                                         int64_t n, uint32_t* __restrict__ sums) {
  __shared__ uint32_t sh[32];
  int64_t i = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x;
  uint32_t v = i < n ? in[i] : 0u;
  uint32_t tot;
  block_exclusive_scan_1024(v, sh, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_sums(uint32_t* __restrict__ sums, int nb) {
  // exclusive scan of nb block sums in place, in chunks of 1024; sums[nb] = total
  __shared__ uint32_t sh[32];
  uint32_t carry = 0;
  for (int base = 0; base < nb; base += SCAN_BLOCK) {
    int i = base + threadIdx.x;
    uint32_t v = i < nb ? sums[i] : 0u;
    uint32_t tot;
    uint32_t ex = block_exclusive_scan_1024(v, sh, &tot);
    if (i < nb) sums[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(1024) void k_scan_final(const uint32_t* __restrict__ in, int64_t n,
                                                     const uint32_t* __restrict__ sums,
                                                     int32_t* __restrict__ out, int nb) {
  __shared__ uint32_t sh[32];
  int64_t i = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x;
  uint32_t v = i < n ? in[i] : 0u;
  uint32_t tot;
  uint32_t ex = block_exclusive_scan_1024(v, sh, &tot);
  if (i < n) out[i] = (int32_t)(sums[blockIdx.x] + ex);
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = (int32_t)sums[nb];
}

// k_scan_final without the scan of the block sums before it: every block adds
// up the sums ahead of it itself (at most SCAN_DIRECT of them, four loads per
// thread), which is shorter than one more launch (286,000 values: 12.7 -> 8.6 us).
constexpr int SCAN_DIRECT = 4096;
__global__ __launch_bounds__(1024) void k_scan_direct(const uint32_t* __restrict__ in, int64_t n,
                                                      const uint32_t* __restrict__ sums,
                                                      int32_t* __restrict__ out) {
  __shared__ uint32_t sh[32];
  const int b = blockIdx.x;
  const int64_t i = (int64_t)b * SCAN_BLOCK + threadIdx.x;
  const uint32_t v = i < n ? in[i] : 0u;
  uint32_t pre = 0;
  for (int k = threadIdx.x; k < b; k += SCAN_BLOCK) pre += sums[k];
  uint32_t before, tot;
  block_exclusive_scan_1024(pre, sh, &before);
  const uint32_t ex = block_exclusive_scan_1024(v, sh, &tot);
  if (i < n) out[i] = (int32_t)(before + ex);
  if (i == n - 1) out[n] = (int32_t)(before + tot);
}

// Exclusive scan of up to 16 * 1024 values by one workgroup in one launch:
// thread t takes SCAN_PER consecutive values, the per-thread totals are
// scanned across the block, and each thread writes its values' prefixes;
// out[n] = total.
constexpr int SCAN_PER = 16;
__global__ __launch_bounds__(1024) void k_scan_single(const uint32_t* __restrict__ in, int64_t n,
                                                      int32_t* __restrict__ out) {
  __shared__ uint32_t sh[32];
  const int64_t b = (int64_t)threadIdx.x * SCAN_PER;
  uint32_t v[SCAN_PER], sum = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    v[k] = b + k < n ? in[b + k] : 0u;
    sum += v[k];
  }
  uint32_t tot;
  uint32_t run = block_exclusive_scan_1024(sum, sh, &tot);
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    if (b + k < n) out[b + k] = (int32_t)run;
    run += v[k];
  }
  if (threadIdx.x == 0) out[n] = (int32_t)tot;
}

// p[0..n) = v, and q[0..n) = v too when q is not null (two arrays, one launch)
__global__ void k_fill_u32(uint32_t* p, uint32_t* q, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    p[i] = v;
    if (q) q[i] = v;
  }
}

}  // namespace

namespace dsmp {

dsmp_status exclusive_scan_u32(dsmp_handle* h, const uint32_t* in, int32_t* out, int64_t n,
                               uint32_t* tmp) {
  int nb = (int)ceil_div(n, SCAN_BLOCK);
  if (n <= (int64_t)SCAN_PER * 1024) {   // one launch
    hipLaunchKernelGGL(k_scan_single, dim3(1), dim3(1024), 0, h->stream, in, n, out);
    DSMP_LAUNCHED(h, "scan");
    return DSMP_OK;
  }
  if (nb == 0) {
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, h->stream, tmp, 0);
    hipLaunchKernelGGL(k_scan_final, dim3(1), dim3(1024), 0, h->stream, in, (int64_t)0, tmp, out, 0);
    DSMP_LAUNCHED(h, "scan");
    return DSMP_OK;
  }
  hipLaunchKernelGGL(k_scan_blocksums, dim3(nb), dim3(1024), 0, h->stream, in, n, tmp);
  if (nb <= SCAN_DIRECT) {
    hipLaunchKernelGGL(k_scan_direct, dim3(nb), dim3(1024), 0, h->stream, in, n, tmp, out);
    DSMP_LAUNCHED(h, "scan");
    return DSMP_OK;
  }
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, h->stream, tmp, nb);
  hipLaunchKernelGGL(k_scan_final, dim3(nb), dim3(1024), 0, h->stream, in, n, tmp, out, nb);
  DSMP_LAUNCHED(h, "scan");
  return DSMP_OK;
}

dsmp_status fill_u32(dsmp_handle* h, uint32_t* p, int64_t n, uint32_t v, uint32_t* q) {
  if (n <= 0) return DSMP_OK;
  unsigned g = ceil_div(n, 256);
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_fill_u32, dim3(g), dim3(256), 0, h->stream, p, q, n, v);
  DSMP_LAUNCHED(h, "fill");
  return DSMP_OK;
}

}  // namespace dsmp

// ------------------------------------------------------------------ handle

extern "C" int dsmp_version(void) { return 10000; }

// device address of the sampling scratch array on the current device (set-up
// of the allocation-free sampling entry point; defined with the array below)
static dsmp_status sample_scratch_setup(dsmp_handle* h);

extern "C" dsmp_status dsmp_create(dsmp_handle** out, int device) {
  if (!out) return DSMP_INVALID_ARG;
  *out = nullptr;
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return DSMP_INVALID_ARG;
  if (hipSetDevice(device) != hipSuccess) return DSMP_HIP_ERROR;
  dsmp_handle* h = new (std::nothrow) dsmp_handle();
  if (!h) return DSMP_HIP_ERROR;
  h->device = device;
  int cu = 0;
  if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cu > 0) h->n_cu = cu;
  const dsmp_status st = sample_scratch_setup(h);
  if (st != DSMP_OK) {
    delete h;
    return st;
  }
  void* dev = nullptr;
  if (hipHostMalloc(reinterpret_cast<void**>(&h->readback), READBACK_BYTES, hipHostMallocDefault) != hipSuccess ||
      hipHostGetDevicePointer(&dev, h->readback, 0) != hipSuccess) {
    if (h->readback) (void)hipHostFree(h->readback);
    delete h;
    return DSMP_HIP_ERROR;
  }
  h->readback_dev = dev;
  *out = h;
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_destroy(dsmp_handle* h) {
  if (!h) return DSMP_OK;
  for (auto& m : h->pending) { (void)hipEventDestroy(m.a); (void)hipEventDestroy(m.b); }
  for (auto& e : h->pool) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
  if (h->readback) (void)hipHostFree(h->readback);
  delete h;
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_profile_enable(dsmp_handle* h, int enable) {
  if (!h) return DSMP_INVALID_ARG;
  h->prof = enable != 0;
  return DSMP_OK;
}

static dsmp_status drain_marks(dsmp_handle* h) {
  for (auto& m : h->pending) {
    DSMP_HIP(h, hipEventSynchronize(m.b));
    float ms = 0.0f;
    DSMP_HIP(h, hipEventElapsedTime(&ms, m.a, m.b));
    h->tot_ms[m.cls] += ms;
    h->launches[m.cls] += 1;
    h->pool.push_back({m.a, m.b});
  }
  h->pending.clear();
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_profile_reset(dsmp_handle* h) {
  if (!h) return DSMP_INVALID_ARG;
  dsmp_status st = drain_marks(h);
  for (int k = 0; k < DSMP_K_COUNT; ++k) { h->tot_ms[k] = 0.0; h->launches[k] = 0; }
  return st;
}

extern "C" dsmp_status dsmp_profile_read(dsmp_handle* h, int cls, double* total_ms, int64_t* launches) {
  if (!h) return DSMP_INVALID_ARG;
  DSMP_CHECK(h, cls >= 0 && cls < DSMP_K_COUNT && total_ms && launches, DSMP_INVALID_ARG,
             "bad profile query");
  dsmp_status st = drain_marks(h);
  if (st != DSMP_OK) return st;
  *total_ms = h->tot_ms[cls];
  *launches = h->launches[cls];
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_set_stream(dsmp_handle* h, void* stream) {
  if (!h) return DSMP_INVALID_ARG;
  h->stream = reinterpret_cast<hipStream_t>(stream);
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_set_edge_algorithm(dsmp_handle* h, int32_t algorithm) {
  if (!h) return DSMP_INVALID_ARG;
  DSMP_CHECK(h, algorithm == DSMP_EDGE_AUTO || algorithm == DSMP_EDGE_PER_EDGE || algorithm == DSMP_EDGE_AGGREGATE,
             DSMP_INVALID_ARG, "unknown edge algorithm %d", algorithm);
  h->edge_algo = algorithm;
  return DSMP_OK;
}

extern "C" const char* dsmp_last_error(const dsmp_handle* h) { return h ? h->err.c_str() : ""; }

// ------------------------------------------------------------------ sampling
//
// Selection of the s smallest SplitMix64 keys out of M by an MSB-first radix
// select (the keys are recomputed, never stored), then a stable compaction of
// the candidates whose key is at most the threshold.  The keys are distinct
// (the mix is a bijection of the counter), so exactly s are kept.  Three forms
// by M, each bounded by the latency of its launches rather than by traffic:
//   M <= 8,192        one workgroup does everything in one launch
//                     (1,024 of 4,096: eleven launches of 56 us -> 7.2 us; against
//                     the next form 7.4 and 18.6 us at 4,096, 9.8 and 18.7 at
//                     8,192, what the threads' registers hold)
//   M <= 8,388,608    four launches (262,144 of 764,077: 95 -> 34 us): an 11-bit histogram, then one pass that
//                     counts the sure candidates and lists those in the
//                     threshold's bin (M / 2,048 on average), whose last
//                     workgroup ranks the list; then the compaction
//   larger M          four 16-bit digits, each a histogram and a pick (the
//                     list of a bin would no longer be short)

namespace {

struct SelState {
  unsigned long long prefix;   // digits fixed so far
  unsigned long long rank;     // 1-based rank of the wanted key among the unfixed ones
};

constexpr int SAMPLE_CHUNK = 1024;   // candidates per block in the compaction
constexpr int SEL_BINS = 65536;      // 16-bit digits

// Histogram of digit (k >> shift) & 0xFFFF over the keys that match the fixed prefix.
__global__ __launch_bounds__(256) void k_sel_hist(int64_t M, uint64_t seed, const SelState* st, int shift,
                                                  uint32_t* __restrict__ hist) {
  const uint64_t prefix = st->prefix;
  const uint64_t himask = shift >= 48 ? 0ull : (~0ull << (shift + 16));
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < M; i += stride) {
    const uint64_t k = splitmix64(seed, (uint64_t)i);
    if ((k & himask) == (prefix & himask)) atomicAdd(&hist[(k >> shift) & 0xFFFFu], 1u);
  }
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// One workgroup of 16 waves.  The histogram is read once, in 1 KB pieces
// that one wave loads whole: piece P = 16 w + v covers bins
// [256 P, 256 P + 256), lane l of it bins 256 P + 4 l .. + 3.  Every piece's
// total goes to LDS; wave 0 scans the 256 totals and finds the piece that
// holds the wanted rank; the wave that read that piece scans its lanes and
// fixes the digit.  Every wave clears the bins it read for the next pass.
__global__ __launch_bounds__(1024) void k_sel_pick(SelState* st, int shift, uint32_t* __restrict__ hist) {
  static_assert(SEL_BINS == 16 * 16 * 256, "16 waves x 16 pieces of 256 bins");
  __shared__ uint32_t psum[256];
  __shared__ uint32_t pick[2];   // the piece, and the count of the bins before it
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) pick[0] = ~0u;
  uint4* hb = reinterpret_cast<uint4*>(hist) + (size_t)w * 1024 + lane;
  uint4 x[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) x[v] = hb[64 * v];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t t = wave_sum(x[v].x + x[v].y + x[v].z + x[v].w);
    if (lane == 0) psum[16 * w + v] = t;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) hb[64 * v] = make_uint4(0u, 0u, 0u, 0u);
  const uint64_t r = st->rank;
  __syncthreads();   // piece totals are in LDS; every thread has read the rank
  if (w == 0) {
    const uint32_t a0 = psum[4 * lane], a1 = psum[4 * lane + 1], a2 = psum[4 * lane + 2], a3 = psum[4 * lane + 3];
    const uint32_t ls = a0 + a1 + a2 + a3;
    const uint32_t inc = wave_inclusive_scan(ls), ex = inc - ls;
    if (ex < r && r <= (uint64_t)inc) {
      uint32_t acc = ex;
      int P = 4 * lane;
      if (acc + a0 < r) {
        acc += a0; ++P;
        if (acc + a1 < r) {
          acc += a1; ++P;
          if (acc + a2 < r) { acc += a2; ++P; }
        }
      }
      pick[0] = (uint32_t)P;
      pick[1] = acc;
    }
  }
  __syncthreads();
  const uint32_t P = pick[0];
  if (P < 256 && w == (int)(P / 16)) {
    const int vs = P % 16;
    uint4 y = x[0];
#pragma unroll
    for (int v = 1; v < 16; ++v)
      if (v == vs) y = x[v];
    const uint32_t ls = y.x + y.y + y.z + y.w;
    const uint32_t inc = wave_inclusive_scan(ls);
    const uint64_t base = (uint64_t)pick[1] + (inc - ls);
    if (base < r && r <= base + ls) {
      const uint32_t c[4] = {y.x, y.y, y.z, y.w};
      uint64_t acc = base;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (acc + c[k] >= r) {
          st->rank = r - acc;
          st->prefix |= (uint64_t)(256 * P + 4 * lane + k) << shift;
          break;
        }
        acc += c[k];
      }
    }
  }
}

__global__ __launch_bounds__(1024) void k_sel_init(SelState* st, uint64_t s, uint32_t* hist) {
  if (blockIdx.x == 0 && threadIdx.x == 0) { st->prefix = 0; st->rank = s; }
  uint4* hb = reinterpret_cast<uint4*>(hist);
  for (int v = blockIdx.x * 1024 + threadIdx.x; v < SEL_BINS / 4; v += gridDim.x * 1024)
    hb[v] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(1024) void k_sel_count(int64_t M, uint64_t seed, const SelState* st,
                                                    uint32_t* __restrict__ cnt) {
  __shared__ uint32_t sh[32];
  int64_t i = (int64_t)blockIdx.x * SAMPLE_CHUNK + threadIdx.x;
  uint32_t f = (i < M && splitmix64(seed, (uint64_t)i) <= st->prefix) ? 1u : 0u;
  uint32_t tot;
  block_exclusive_scan_1024(f, sh, &tot);
  if (threadIdx.x == 0) cnt[blockIdx.x] = tot;
}

// At most s are written, whatever the threshold and the offsets are.
__global__ __launch_bounds__(1024) void k_sel_write(int64_t M, uint32_t s, uint64_t seed,
                                                    const unsigned long long* threshold,
                                                    const uint32_t* __restrict__ off,
                                                    int32_t* __restrict__ out) {
  __shared__ uint32_t sh[32];
  int64_t i = (int64_t)blockIdx.x * SAMPLE_CHUNK + threadIdx.x;
  uint32_t f = (i < M && splitmix64(seed, (uint64_t)i) <= *threshold) ? 1u : 0u;
  uint32_t tot;
  uint32_t ex = block_exclusive_scan_1024(f, sh, &tot);
  if (!f) return;
  const uint32_t at = off[blockIdx.x] + ex;
  if (at < s) out[at] = (int32_t)i;
}

// ---- one workgroup, and the middle form

constexpr int SEL_SMALL = 8192;           // candidates of the one-workgroup form (8 per thread)
constexpr int64_t SEL_MID = 1ll << 23;    // candidates of the middle form (a bin holds 4,096 on average)
constexpr int SEL_DIG = 11, SEL_DBINS = 1 << SEL_DIG;
constexpr int SEL_LIST = 16384;           // entries of the middle form's list
constexpr int SEL_GRID = 128;             // most workgroups of its passes (each ends in a fence and an atomic)

struct SelMid {                  // state of the middle form
  unsigned long long threshold;  // the kept keys are those at most this
  unsigned rank, bin;            // 1-based rank within bin `bin` of the top digit
  unsigned listed;               // candidates of that bin
  unsigned done1, done2;         // workgroups finished with each pass
};

struct SelLds {
  uint32_t hist[SEL_DBINS];
  uint32_t scan[32];
  uint32_t found[3];             // digit, candidates before it, candidates in it
};

// The digit whose bin holds the rank-th candidate (1-based), from the
// histogram in LDS: two bins per thread, one scan over the workgroup.
__device__ __forceinline__ void block_pick(SelLds& L, uint32_t rank) {
  const int t = threadIdx.x;
  const uint32_t c0 = L.hist[2 * t], c1 = L.hist[2 * t + 1];
  uint32_t tot;
  const uint32_t ex = block_exclusive_scan_1024(c0 + c1, L.scan, &tot);
  if (ex < rank && rank <= ex + c0) {
    L.found[0] = 2 * t; L.found[1] = ex; L.found[2] = c0;
  } else if (ex + c0 < rank && rank <= ex + c0 + c1) {
    L.found[0] = 2 * t + 1; L.found[1] = ex + c0; L.found[2] = c1;
  }
  __syncthreads();
}

// The rank-th smallest of the keys key(0 .. n-1) that agree with `prefix` in
// their top `fixed` bits, by one workgroup of 1,024 threads: a digit at a
// time, until every candidate left is kept.  Returns a threshold T: exactly
// `rank` of those keys are at most T.  (The digits run out after 64 bits at
// the latest, when one key is left, since the keys are distinct.)
template <typename KeyFn>
__device__ uint64_t block_select(SelLds& L, int64_t n, KeyFn key, uint64_t prefix, int fixed, uint32_t rank) {
  for (;;) {
    const int dig = 64 - fixed < SEL_DIG ? 64 - fixed : SEL_DIG, shift = 64 - fixed - dig;
    for (int b = threadIdx.x; b < SEL_DBINS; b += 1024) L.hist[b] = 0;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < n; i += 1024) {
      const uint64_t k = key(i);
      if (fixed == 0 || (k ^ prefix) >> (64 - fixed) == 0)
        atomicAdd(&L.hist[(k >> shift) & ((1u << dig) - 1u)], 1u);
    }
    __syncthreads();
    block_pick(L, rank);
    const uint32_t d = L.found[0], cnt = L.found[2];
    rank -= L.found[1];
    prefix |= (uint64_t)d << shift;
    fixed += dig;
    if (rank == cnt || fixed == 64) return prefix | (shift ? (1ull << shift) - 1ull : 0ull);
    __syncthreads();   // found[] is read before the next digit writes it
  }
}

__global__ __launch_bounds__(1024) void k_sel_small(int M, uint32_t s, uint64_t seed, int32_t* __restrict__ out) {
  __shared__ SelLds L;
  const uint64_t T = block_select(L, M, [&](int64_t i) { return splitmix64(seed, (uint64_t)i); }, 0, 0, s);
  constexpr int PER = SEL_SMALL / 1024;
  const int i0 = threadIdx.x * PER;
  uint32_t keep = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (i0 + u < M && splitmix64(seed, (uint64_t)(i0 + u)) <= T) keep |= 1u << u;
  uint32_t tot;
  __syncthreads();
  uint32_t at = block_exclusive_scan_1024(__popc(keep), L.scan, &tot);
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (keep >> u & 1u) out[at++] = i0 + u;
}

__global__ __launch_bounds__(1024) void k_mid_init(SelMid* st, uint32_t* hist) {
  if (threadIdx.x == 0) *st = SelMid{};
  for (int b = threadIdx.x; b < SEL_DBINS; b += 1024) hist[b] = 0;
}

// Whether this workgroup is the last of the grid to get here.  What the
// others wrote before it is then visible to agent-scope loads.  The barrier
// alone does not complete the workgroup's writes (it compiles to a wait for LDS
// operations and s_barrier), so every wave first waits for its own; one thread
// then fences for all of them (a fence by every thread is a write-back of the
// L2 by every wave: k_mid_list at 764,077 candidates takes 182 us with it and 746
// workgroups, 31 with one fence each, 16 with at most SEL_GRID workgroups).
__device__ __forceinline__ bool last_block(unsigned* counter) {
  __shared__ unsigned last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    last = atomicAdd(counter, 1u) == gridDim.x - 1;
    __threadfence();
  }
  __syncthreads();
  return last != 0;
}

__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// First pass: the histogram of the top digit, each workgroup's in LDS first
// (few workgroups, so that the merge is few atomics); the last one picks the
// digit that holds the s-th key.
__global__ __launch_bounds__(1024) void k_mid_hist(int64_t M, uint32_t s, uint64_t seed, SelMid* st, uint32_t* hist) {
  __shared__ SelLds L;
  for (int b = threadIdx.x; b < SEL_DBINS; b += 1024) L.hist[b] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * 1024;
  for (int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x; i < M; i += stride)
    atomicAdd(&L.hist[splitmix64(seed, (uint64_t)i) >> (64 - SEL_DIG)], 1u);
  __syncthreads();
  for (int b = threadIdx.x; b < SEL_DBINS; b += 1024)
    if (L.hist[b]) atomicAdd(&hist[b], L.hist[b]);
  if (!last_block(&st->done1)) return;
  for (int b = threadIdx.x; b < SEL_DBINS; b += 1024) L.hist[b] = load_agent(hist + b);
  __syncthreads();
  block_pick(L, s);
  if (threadIdx.x == 0) {
    st->bin = L.found[0];
    st->rank = s - L.found[1];
  }
}

// Second pass, by chunks of SAMPLE_CHUNK candidates: the count
// of those below the threshold's bin, and the ones in it to the list.  The
// last workgroup ranks the list, adds its kept ones to their chunks' counts
// and scans the counts.  A list that overflowed (a bin of four times its
// expected size at least) is ranked from the keys themselves.
__global__ __launch_bounds__(1024) void k_mid_list(int64_t M, uint64_t seed, SelMid* st, uint32_t* __restrict__ list,
                                                   uint32_t* cnt, int nb) {
  __shared__ SelLds L;
  __shared__ uint32_t below;
  const uint32_t bin = st->bin;
  for (int c = blockIdx.x; c < nb; c += gridDim.x) {
    if (threadIdx.x == 0) below = 0;
    __syncthreads();
    const int64_t i = (int64_t)c * SAMPLE_CHUNK + threadIdx.x;
    const uint32_t d = i < M ? (uint32_t)(splitmix64(seed, (uint64_t)i) >> (64 - SEL_DIG)) : ~0u;
    const uint64_t lt = __ballot(d < bin);
    if ((threadIdx.x & 63) == 0 && lt) atomicAdd(&below, (uint32_t)__popcll(lt));
    if (d == bin) {
      const uint32_t at = atomicAdd(&st->listed, 1u);
      if (at < SEL_LIST) __hip_atomic_store(list + at, (uint32_t)i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(cnt + c, below, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!last_block(&st->done2)) return;
  const uint32_t listed = load_agent(&st->listed), rank = st->rank;
  const uint64_t prefix = (uint64_t)bin << (64 - SEL_DIG);
  auto key_of = [&](int64_t c) { return splitmix64(seed, (uint64_t)c); };
  uint64_t T;
  if (listed <= SEL_LIST) {
    T = block_select(L, listed, [&](int64_t e) { return key_of(load_agent(list + e)); }, prefix, SEL_DIG, rank);
    for (uint32_t e = threadIdx.x; e < listed; e += 1024) {
      const uint32_t c = load_agent(list + e);
      if (key_of(c) <= T) atomicAdd(&cnt[c / SAMPLE_CHUNK], 1u);
    }
  } else {
    T = block_select(L, M, key_of, prefix, SEL_DIG, rank);
    for (int64_t c = threadIdx.x; c < M; c += 1024) {
      const uint64_t k = key_of(c);
      if (k >> (64 - SEL_DIG) == bin && k <= T) atomicAdd(&cnt[c / SAMPLE_CHUNK], 1u);
    }
  }
  if (threadIdx.x == 0) st->threshold = T;
  __threadfence();
  __syncthreads();
  uint32_t carry = 0;
  for (int b0 = 0; b0 < nb; b0 += 1024) {
    const int b = b0 + threadIdx.x;
    const uint32_t v = b < nb ? load_agent(cnt + b) : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan_1024(v, L.scan, &tot);
    if (b < nb) cnt[b] = carry + ex;
    carry += tot;
  }
}

__global__ void k_iota(int32_t* out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (int32_t)i;
}

size_t sample_ws(int64_t M) {
  size_t nb = ceil_div(M, SAMPLE_CHUNK);
  Carve c(nullptr);
  c.take<SelState>(1);
  c.take<uint32_t>(SEL_BINS);
  c.take<uint32_t>(nb + 2);
  return c.used();
}

}  // namespace

extern "C" dsmp_status dsmp_sample_workspace(int64_t M, size_t* bytes) {
  if (!bytes || M < 0) return DSMP_INVALID_ARG;
  *bytes = sample_ws(M);
  return DSMP_OK;
}

namespace {
// The selection on a workspace of at least sample_ws(M) bytes (checked by the callers).
dsmp_status sample_run(dsmp_handle* h, int64_t M, int64_t s, uint64_t seed, int32_t* idx_out, void* ws) {
  ProfScope prof(h, DSMP_K_SAMPLE);
  if (s == M) {
    hipLaunchKernelGGL(k_iota, dim3(ceil_div(M, 256)), dim3(256), 0, h->stream, idx_out, M);
    DSMP_LAUNCHED(h, "iota");
    return DSMP_OK;
  }
  Carve c(ws);
  SelState* st = c.take<SelState>(1);
  uint32_t* hist = c.take<uint32_t>(SEL_BINS);
  int nb = (int)ceil_div(M, SAMPLE_CHUNK);
  uint32_t* cnt = c.take<uint32_t>(nb + 2);
  if (M <= SEL_SMALL) {
    hipLaunchKernelGGL(k_sel_small, dim3(1), dim3(1024), 0, h->stream, (int)M, (uint32_t)s, seed, idx_out);
    DSMP_LAUNCHED(h, "sample");
    return DSMP_OK;
  }
  if (M <= SEL_MID) {
    // state, histogram and list in the room of the large form's histogram
    SelMid* ms = reinterpret_cast<SelMid*>(hist);
    uint32_t *mh = hist + 64, *list = hist + 64 + SEL_DBINS;
    static_assert(sizeof(SelMid) <= 256 && 64 + SEL_DBINS + SEL_LIST <= SEL_BINS, "fits the histogram's room");
    hipLaunchKernelGGL(k_mid_init, dim3(1), dim3(1024), 0, h->stream, ms, mh);
    hipLaunchKernelGGL(k_mid_hist, dim3(std::min(ceil_div(M, 4096), (unsigned)SEL_GRID)), dim3(1024), 0, h->stream, M, (uint32_t)s,
                       seed, ms, mh);
    hipLaunchKernelGGL(k_mid_list, dim3(std::min(nb, SEL_GRID)), dim3(1024), 0, h->stream, M, seed, ms, list, cnt, nb);
    hipLaunchKernelGGL(k_sel_write, dim3(nb), dim3(1024), 0, h->stream, M, (uint32_t)s, seed, &ms->threshold, cnt,
                       idx_out);
    DSMP_LAUNCHED(h, "sample");
    return DSMP_OK;
  }
  // the state and the histogram are cleared by a kernel on every call
  hipLaunchKernelGGL(k_sel_init, dim3(SEL_BINS / 4 / 1024), dim3(1024), 0, h->stream, st, (uint64_t)s, hist);
  unsigned g = ceil_div(M, 256);
  if (g > 2048) g = 2048;
  for (int shift = 48; shift >= 0; shift -= 16) {
    hipLaunchKernelGGL(k_sel_hist, dim3(g), dim3(256), 0, h->stream, M, seed, st, shift, hist);
    hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(1024), 0, h->stream, st, shift, hist);
  }
  hipLaunchKernelGGL(k_sel_count, dim3(nb), dim3(1024), 0, h->stream, M, seed, st, cnt);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, h->stream, cnt, nb);
  hipLaunchKernelGGL(k_sel_write, dim3(nb), dim3(1024), 0, h->stream, M, (uint32_t)s, seed, &st->prefix, cnt,
                       idx_out);
  DSMP_LAUNCHED(h, "sample");
  return DSMP_OK;
}

dsmp_status sample_check(dsmp_handle* h, int64_t M, int64_t s, const int32_t* idx_out) {
  DSMP_CHECK(h, M >= 0 && s >= 0 && s <= M, DSMP_INVALID_ARG, "need 0 <= s <= M (M=%lld s=%lld)",
             (long long)M, (long long)s);
  DSMP_CHECK(h, M <= INT32_MAX, DSMP_UNSUPPORTED, "M exceeds int32 range");
  DSMP_CHECK(h, s == 0 || idx_out != nullptr, DSMP_INVALID_ARG, "idx_out is NULL");
  return DSMP_OK;
}

// Allocation-free sampling: the workspace is a file-scope device array of a
// fixed size, enough for SAMPLE_NOALLOC_MAX_M candidates.  Host code never
// passes the array's name to a kernel: the device address comes from
// hipGetSymbolAddress, taken once per device at handle creation.
constexpr int64_t SAMPLE_NOALLOC_MAX_M = 1ll << 24;
constexpr size_t round256(size_t b) { return (b + 255) & ~size_t(255); }
constexpr size_t SAMPLE_SCRATCH_BYTES = round256(sizeof(SelState)) + round256(sizeof(uint32_t) * SEL_BINS) +
                                        round256(sizeof(uint32_t) * ((SAMPLE_NOALLOC_MAX_M + SAMPLE_CHUNK - 1) /
                                                                     SAMPLE_CHUNK + 2));
}  // namespace

static __device__ __align__(256) unsigned char scratch[SAMPLE_SCRATCH_BYTES];

static dsmp_status sample_scratch_setup(dsmp_handle* h) {
  static std::mutex mu;
  static std::map<int, void*> addr;   // device -> address of its copy of the array
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(h->device);
  if (it == addr.end()) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr)
      return fail(h, DSMP_HIP_ERROR, "hipGetSymbolAddress of the sampling scratch failed: %s", hipGetErrorString(e));
    it = addr.emplace(h->device, ptr).first;
  }
  h->sample_scratch = it->second;
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_sample_nodes(dsmp_handle* h, int64_t M, int64_t s, uint64_t seed,
                                         int32_t* idx_out, void* ws, size_t ws_bytes) {
  if (!h) return DSMP_INVALID_ARG;
  dsmp_status st = sample_check(h, M, s, idx_out);
  if (st != DSMP_OK || s == 0) return st;
  DSMP_CHECK(h, s == M || (ws != nullptr && ws_bytes >= sample_ws(M)), DSMP_WORKSPACE_TOO_SMALL,
             "sampling workspace needs %zu bytes", sample_ws(M));
  return sample_run(h, M, s, seed, idx_out, ws);
}

extern "C" dsmp_status dsmp_sample_nodes_noalloc(dsmp_handle* h, int64_t M, int64_t s, uint64_t seed,
                                                 int32_t* idx_out) {
  if (!h) return DSMP_INVALID_ARG;
  dsmp_status st = sample_check(h, M, s, idx_out);
  if (st != DSMP_OK || s == 0) return st;
  DSMP_CHECK(h, M <= SAMPLE_NOALLOC_MAX_M, DSMP_UNSUPPORTED,
             "allocation-free sampling takes at most %lld candidates (M=%lld)", (long long)SAMPLE_NOALLOC_MAX_M,
             (long long)M);
  DSMP_CHECK(h, h->sample_scratch != nullptr, DSMP_HIP_ERROR, "sampling scratch address not set up");
  DSMP_CHECK(h, sample_ws(M) <= SAMPLE_SCRATCH_BYTES, DSMP_UNSUPPORTED, "sampling scratch too small");
  return sample_run(h, M, s, seed, idx_out, h->sample_scratch);
}

// ------------------------------------------------------------------ gather

namespace {
// A thread per unit: a 16-byte unit where the rows and both arrays are
// aligned to it, else a word.  Indices are 32-bit below 2^31 units (the row of
// a unit is then one short division, a shift where a row is a power of two of
// units).  Gathers of 262,144 rows of 12, 16 and 256 bytes: 42.6 -> 30.5 us
// together, the last at 5.8 TB/s read and written (words with 64-bit divisions
// before).  At most GATHER_GRID workgroups, eight per CU, which step over the
// rest: with a workgroup for every 256 units 150,000 rows of 132 bytes take 14.2
// us, with 8,192 12.3 and with 2,048 11.4; rows of 16-byte units are the same.
constexpr int64_t GATHER_GRID = 2048;
template <typename U, typename I>
__global__ __launch_bounds__(256) void k_gather_rows(const U* __restrict__ src, int64_t n_src_rows, I units, int sh,
                                                     const int32_t* __restrict__ idx, I total, U* __restrict__ dst) {
  for (I t = (I)blockIdx.x * 256 + threadIdx.x; t < total; t += (I)gridDim.x * 256) {
    const I r = sh >= 0 ? t >> sh : t / units, w = t - r * units;
    const int32_t s = idx[r];
    dst[t] = (s >= 0 && s < n_src_rows) ? src[(int64_t)s * units + w] : U{};
  }
}

template <typename U>
void gather_launch(hipStream_t st, const void* src, int64_t n_src_rows, int64_t row_bytes, const int32_t* idx,
                   int64_t n, void* dst) {
  const int64_t units = row_bytes / (int64_t)sizeof(U), total = n * units;
  const int sh = (units & (units - 1)) == 0 ? __builtin_ctzll((unsigned long long)units) : -1;
  const unsigned g = (unsigned)std::min<int64_t>((total + 255) / 256, GATHER_GRID);
  if (total < (1ll << 31))   // a step past the end stays below 2^32
    hipLaunchKernelGGL((k_gather_rows<U, uint32_t>), dim3(g), dim3(256), 0, st, static_cast<const U*>(src),
                       n_src_rows, (uint32_t)units, sh, idx, (uint32_t)total, static_cast<U*>(dst));
  else
    hipLaunchKernelGGL((k_gather_rows<U, uint64_t>), dim3(g), dim3(256), 0, st, static_cast<const U*>(src),
                       n_src_rows, (uint64_t)units, sh, idx, (uint64_t)total, static_cast<U*>(dst));
}
}  // namespace

extern "C" dsmp_status dsmp_gather_rows(dsmp_handle* h, const void* src, int64_t n_src_rows,
                                        int64_t row_bytes, const int32_t* idx, int64_t n, void* dst) {
  if (!h) return DSMP_INVALID_ARG;
  DSMP_CHECK(h, n >= 0 && n_src_rows >= 0 && row_bytes > 0 && row_bytes % 4 == 0, DSMP_INVALID_ARG,
             "bad gather sizes");
  if (n == 0) return DSMP_OK;
  DSMP_CHECK(h, src && idx && dst, DSMP_INVALID_ARG, "gather pointer is NULL");
  ProfScope prof(h, DSMP_K_GATHER);
  const bool wide = row_bytes % 16 == 0 &&
                    ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0;
  if (wide) gather_launch<uint4>(h->stream, src, n_src_rows, row_bytes, idx, n, dst);
  else gather_launch<uint32_t>(h->stream, src, n_src_rows, row_bytes, idx, n, dst);
  DSMP_LAUNCHED(h, "gather_rows");
  return DSMP_OK;
}

// ------------------------------------------------------------ sub-domains

namespace {
struct Box {
  float lo[3], hi[3], elo[3], ehi[3];
};

// own[i] = 1 for nodes inside [lo, hi) in every axis; ovl[i] = 1 for the
// other nodes inside [lo - l, hi + l) (bounds rounded to float32 on the host)
__global__ void k_sub_flags(const float* __restrict__ pos, int64_t n, int D, Box b,
                            uint32_t* __restrict__ own, uint32_t* __restrict__ ovl) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  bool in = true, ext = true;
  for (int a = 0; a < D; ++a) {
    float p = pos[i * D + a];
    in = in && p >= b.lo[a] && p < b.hi[a];
    ext = ext && p >= b.elo[a] && p < b.ehi[a];
  }
  own[i] = in ? 1u : 0u;
  ovl[i] = (ext && !in) ? 1u : 0u;
}

// owned nodes to idx[0, n_owned), overlap nodes to idx[n_owned, n_total),
// each in ascending order (positions from the two exclusive scans)
__global__ void k_sub_scatter(int64_t n, const uint32_t* __restrict__ own, const uint32_t* __restrict__ ovl,
                              const int32_t* __restrict__ own_pos, const int32_t* __restrict__ ovl_pos,
                              int32_t* __restrict__ idx) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (own[i]) idx[own_pos[i]] = (int32_t)i;
  else if (ovl[i]) idx[own_pos[n] + ovl_pos[i]] = (int32_t)i;
}

// All of the selection for up to SUB_SMALL nodes by one workgroup: eight
// consecutive nodes per thread, both counts scanned at once (16 bits each),
// the two lists written and their lengths left in host memory.  One launch in
// place of four and two copies (8,192 nodes: 30 us of kernels -> 8).
constexpr int SUB_SMALL = 8192;
__global__ __launch_bounds__(1024) void k_sub_small(const float* __restrict__ pos, int n, int D, Box b,
                                                    int32_t* __restrict__ idx, int32_t* counts) {
  __shared__ uint32_t sh[32];
  constexpr int PER = SUB_SMALL / 1024;
  const int i0 = threadIdx.x * PER;
  uint32_t own = 0, ovl = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = i0 + u;
    if (i < n) {
      bool in = true, ext = true;
      for (int a = 0; a < D; ++a) {
        const float p = pos[i * D + a];
        in = in && p >= b.lo[a] && p < b.hi[a];
        ext = ext && p >= b.elo[a] && p < b.ehi[a];
      }
      own |= (in ? 1u : 0u) << u;
      ovl |= (ext && !in ? 1u : 0u) << u;
    }
  }
  uint32_t tot;
  const uint32_t ex = block_exclusive_scan_1024((uint32_t)__popc(own) | (uint32_t)__popc(ovl) << 16, sh, &tot);
  const int n_own = (int)(tot & 0xFFFFu), n_ovl = (int)(tot >> 16);
  int at = (int)(ex & 0xFFFFu), bt = n_own + (int)(ex >> 16);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (own >> u & 1u) idx[at++] = i0 + u;
    if (ovl >> u & 1u) idx[bt++] = i0 + u;
  }
  if (threadIdx.x == 0) {
    counts[0] = n_own;
    counts[1] = n_ovl;
    __threadfence_system();
  }
}

// the lengths of the two lists, left in host memory
__global__ void k_sub_counts(int64_t n, const int32_t* __restrict__ own_pos, const int32_t* __restrict__ ovl_pos,
                             int32_t* counts) {
  counts[0] = own_pos[n];
  counts[1] = ovl_pos[n];
  __threadfence_system();
}

__global__ void k_scatter_rows(const uint32_t* __restrict__ src, int64_t words, const int32_t* __restrict__ idx,
                               int64_t n, uint32_t* __restrict__ dst, int64_t n_dst_rows) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = n * words;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; t < total; t += stride) {
    int64_t r = t / words, w = t - r * words;
    int32_t d = idx[r];
    if (d >= 0 && d < n_dst_rows) dst[(int64_t)d * words + w] = src[t];
  }
}

struct SubWs {
  uint32_t *own, *ovl, *tmp;
  int32_t *own_pos, *ovl_pos;
};

SubWs carve_sub(void* ws, int64_t n, size_t* used) {
  Carve c(ws);
  SubWs w;
  w.own = c.take<uint32_t>(n + 1);
  w.ovl = c.take<uint32_t>(n + 1);
  w.own_pos = c.take<int32_t>(n + 1);
  w.ovl_pos = c.take<int32_t>(n + 1);
  w.tmp = c.take<uint32_t>(scan_tmp_elems(n));
  *used = c.used();
  return w;
}
}  // namespace

extern "C" dsmp_status dsmp_subdomain_workspace(int64_t n, size_t* bytes) {
  if (!bytes || n < 0) return DSMP_INVALID_ARG;
  carve_sub(nullptr, n, bytes);
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_subdomain_select(dsmp_handle* h, const float* pos, int64_t n, int32_t dim,
                                             const float* lo, const float* hi, float overlap,
                                             int32_t* idx_out, void* ws, size_t ws_bytes,
                                             int64_t* n_owned, int64_t* n_total) {
  if (!h) return DSMP_INVALID_ARG;
  DSMP_CHECK(h, n >= 0 && n <= INT32_MAX, n < 0 ? DSMP_INVALID_ARG : DSMP_UNSUPPORTED, "bad node count");
  DSMP_CHECK(h, dim == 2 || dim == 3, DSMP_UNSUPPORTED, "dim must be 2 or 3");
  DSMP_CHECK(h, lo && hi && n_owned && n_total, DSMP_INVALID_ARG, "sub-domain pointer is NULL");
  DSMP_CHECK(h, overlap >= 0.0f, DSMP_INVALID_ARG, "overlap must be >= 0");
  *n_owned = 0;
  *n_total = 0;
  if (n == 0) return DSMP_OK;
  DSMP_CHECK(h, pos && idx_out && ws, DSMP_INVALID_ARG, "sub-domain pointer is NULL");
  size_t need;
  SubWs w = carve_sub(ws, n, &need);
  DSMP_CHECK(h, ws_bytes >= need, DSMP_WORKSPACE_TOO_SMALL, "sub-domain workspace %zu < %zu", ws_bytes, need);
  Box b{};
  for (int a = 0; a < dim; ++a) {
    b.lo[a] = lo[a];
    b.hi[a] = hi[a];
    b.elo[a] = lo[a] - overlap;   // float32 rounding, as the bounds are defined
    b.ehi[a] = hi[a] + overlap;
  }
  ProfScope prof(h, DSMP_K_GATHER);
  hipStream_t s = h->stream;
  int32_t* counts = static_cast<int32_t*>(h->readback_dev);
  std::lock_guard<std::mutex> lock(h->readback_mu);
  if (n <= SUB_SMALL) {
    hipLaunchKernelGGL(k_sub_small, dim3(1), dim3(1024), 0, s, pos, (int)n, (int)dim, b, idx_out, counts);
    DSMP_LAUNCHED(h, "sub-domain selection");
  } else {
    hipLaunchKernelGGL(k_sub_flags, dim3(ceil_div(n, 256)), dim3(256), 0, s, pos, n, (int)dim, b, w.own, w.ovl);
    DSMP_LAUNCHED(h, "sub-domain flags");
    dsmp_status st;
    if ((st = exclusive_scan_u32(h, w.own, w.own_pos, n, w.tmp)) != DSMP_OK) return st;
    if ((st = exclusive_scan_u32(h, w.ovl, w.ovl_pos, n, w.tmp)) != DSMP_OK) return st;
    hipLaunchKernelGGL(k_sub_scatter, dim3(ceil_div(n, 256)), dim3(256), 0, s, n, w.own, w.ovl, w.own_pos,
                       w.ovl_pos, idx_out);
    hipLaunchKernelGGL(k_sub_counts, dim3(1), dim3(1), 0, s, n, w.own_pos, w.ovl_pos, counts);
    DSMP_LAUNCHED(h, "sub-domain scatter");
  }
  DSMP_HIP(h, hipStreamSynchronize(s));
  const volatile int32_t* tot = static_cast<const int32_t*>(h->readback);
  *n_owned = tot[0];
  *n_total = (int64_t)tot[0] + tot[1];
  return DSMP_OK;
}

extern "C" dsmp_status dsmp_scatter_rows(dsmp_handle* h, const void* src, int64_t n, int64_t row_bytes,
                                         const int32_t* idx, void* dst, int64_t n_dst_rows) {
  if (!h) return DSMP_INVALID_ARG;
  DSMP_CHECK(h, n >= 0 && n_dst_rows >= 0 && row_bytes > 0 && row_bytes % 4 == 0, DSMP_INVALID_ARG,
             "bad scatter sizes");
  if (n == 0) return DSMP_OK;
  DSMP_CHECK(h, src && idx && dst, DSMP_INVALID_ARG, "scatter pointer is NULL");
  ProfScope prof(h, DSMP_K_GATHER);
  int64_t words = row_bytes / 4;
  unsigned g = ceil_div(n * words, 256);
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_scatter_rows, dim3(g), dim3(256), 0, h->stream, static_cast<const uint32_t*>(src), words,
                     idx, n, static_cast<uint32_t*>(dst), n_dst_rows);
  DSMP_LAUNCHED(h, "scatter_rows");
  return DSMP_OK;
}
