// Aggregate-first evaluation of the NNConv edge contraction (eq. (1)).
//
// The message of edge e = (i <- j) is bilinear in the kernel-MLP output z_e
// and the source row h_j:
//     m_e[q] = sum_{k,p} W3[p*d+q][k] z_e[k] h_j[p] + sum_p b3[p*d+q] h_j[p].
// The mean over the edges of i is linear, so with z~ = [z; 1]
//     agg_i[q] = (1/deg_i) sum_{k,p} W3~[p*d+q][k] S_i[k][p],
//     S_i[k][p] = sum_{e in in(i)} z~_e[k] h_j(e)[p],
// one GEMM over the per-destination sums S (n_dst x (h2+1)d) in place of one
// product per edge.  The feature gradient has the same form over the edges
// leaving a source j, with T_j[k][q] = sum_{e in out(j)} z~_e[k] g_e[q] and
// dh_j[p] = sum_{k,q} W3~[p*d+q][k] T_j[k][q]; the weight gradient is
// dW3[p*d+q][k] = sum_i g_i[q] S_i[k][p] (g_e = g_i for every edge into i).
// Neither form writes anything of size E x d x d.
//
// K order of a sum row.  The (h2/32) x (d/32) tiles of 32 x 32 are stored in
// MFMA accumulator order: tile t = kt*(d/32) + ct, lane l, register r at
// K = 1024 t + 16 l + r holds k = 32 kt + 8 (r/4) + 4 (l/32) + r%4 (the
// stored, permuted z order) and c = 32 ct + l%32; the d values of the z~ = 1
// row follow at K = h2*d + c.  The packed W3 matrices (WgT, WhT) use the same
// K order, so neither side is ever transposed in memory.
#include "nnconv.hpp"

using namespace dsmp;

namespace {

template <typename T>
__device__ __forceinline__ typename MT<T>::frag ldf(const void* p) {
  return *reinterpret_cast<const typename MT<T>::frag*>(p);
}

// Unit kg (16 bytes) of four rows into LDS transposed: row (element) kg*KPU + w,
// columns c0..c0+3.  The rows come as values, loaded by the caller without
// conditions (rows past the end re-read the last one) and zeroed there: a load
// under a condition is waited for before the next is issued.
template <typename T, int ROWB>
__device__ __forceinline__ void put4_transposed(const uint4 (&v)[4], int kg, int c0, unsigned char* __restrict__ dstl) {
  constexpr int ESZ = sizeof(T);
  const uint32_t* d0 = reinterpret_cast<const uint32_t*>(&v[0]);
  const uint32_t* d1 = reinterpret_cast<const uint32_t*>(&v[1]);
  const uint32_t* d2 = reinterpret_cast<const uint32_t*>(&v[2]);
  const uint32_t* d3 = reinterpret_cast<const uint32_t*>(&v[3]);
  if constexpr (ESZ == 2) {
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const int sh = (w & 1) * 16, dw = w >> 1;
      const uint32_t lo = ((d0[dw] >> sh) & 0xFFFFu) | (((d1[dw] >> sh) & 0xFFFFu) << 16);
      const uint32_t hi = ((d2[dw] >> sh) & 0xFFFFu) | (((d3[dw] >> sh) & 0xFFFFu) << 16);
      *reinterpret_cast<uint2*>(dstl + (kg * 8 + w) * ROWB + c0 * ESZ) = make_uint2(lo, hi);
    }
  } else {
#pragma unroll
    for (int w = 0; w < 4; ++w)
      *reinterpret_cast<uint4*>(dstl + (kg * 4 + w) * ROWB + c0 * ESZ) = make_uint4(d0[w], d1[w], d2[w], d3[w]);
  }
}

// ------------------------------------------------------------ segment sums

struct OuterArgs {
  int64_t n_seg;               // segments: destinations (S) or sources (T)
  const int32_t* seg_ptr;      // [n_seg + 1] positions of each segment's edges
  const int32_t* pos_eid;      // NULL: edge id = position; else edge id = pos_eid[position] (k_outer_sum_tr: NULL)
  const int32_t* row_of;       // gathered row of edge e
  const unsigned char* zE;     // [E][h2] layer dtype, stored order
  const unsigned char* u;      // gathered rows [*][d] layer dtype
  unsigned char* out;          // [n_seg][ktot] layer dtype
  int64_t n_edges;             // edges of all segments
  int stream;                  // store the sums with the non-temporal hint
};

template <typename T, int DL, int H2>
struct OuterShape {
  static constexpr int KS = MT<T>::KS, EPL = MT<T>::EPL, ESZ = sizeof(T);
  static constexpr int ECH = 64;                          // edges per staged chunk
  static constexpr int NKT = H2 / 32, NCT = DL / 32, NTILE = NKT * NCT, TPW = (NTILE + 3) / 4;
  static constexpr int ROWB = (ECH + 16 / ESZ) * ESZ;     // LDS row pitch (bytes)
  static constexpr int ZU = (ECH / 4) * (H2 * ESZ / 16);  // transposed staging units
  static constexpr int UU = (ECH / 4) * (DL * ESZ / 16);
  static constexpr int LDS = (H2 + DL) * ROWB;
  static constexpr int64_t KTOT = (int64_t)H2 * DL + DL;
};

// One workgroup per segment: stage up to 64 of its edges at a time, z~ and
// the gathered rows both transposed to [element][edge], and accumulate the
// outer-product sum tile by tile on MFMA (edges are the contraction index).
// fp32 layers.  A chain of loads bounds small ones (edge ids, sources, rows):
// each step's go out together; 1,024 segments of 20 edges, d = 32: 15.0 -> 12.9
// us, 14.4 -> 11.4 by source, with a condition and a wait at every load before.
template <typename T, int DL, int H2>
__global__ __launch_bounds__(256) void k_outer_sum(OuterArgs a) {
  using S = OuterShape<T, DL, H2>;
  using M = MT<T>;
  constexpr int KS = S::KS, EPL = S::EPL, ESZ = S::ESZ, ECH = S::ECH;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* zt = smem;
  unsigned char* ut = smem + H2 * S::ROWB;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int64_t n = blockIdx.x;
  const int64_t pa = a.seg_ptr[n], pb = a.seg_ptr[n + 1];

  f32x16 acc[S::TPW];
#pragma unroll
  for (int j = 0; j < S::TPW; ++j) acc[j] = f32x16{};
  float hs = 0.0f;   // z~ = 1 row: sum of the gathered rows (threads tid < DL)

  for (int64_t c0 = pa; c0 < pb; c0 += ECH) {
    const int cnt = (int)(pb - c0 < ECH ? pb - c0 : ECH);
    __syncthreads();   // previous chunk fully consumed
    // a thread's four edges are the same in every round of the copy
    constexpr int EQ = ECH / 4, NIT = (S::ZU + S::UU + 255) / 256;
    static_assert(S::ZU % 256 == 0 && 256 % EQ == 0, "whole rounds of z units");
    const int eq = tid % EQ;
    int32_t e[4], ur[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t pos = c0 + (4 * eq + i < cnt ? 4 * eq + i : cnt - 1);
      e[i] = a.pos_eid ? a.pos_eid[pos] : (int32_t)pos;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) ur[i] = a.row_of[e[i]];
    uint4 v[NIT][4];
    auto unit = [&](int it) {   // of a z row, or of a gathered row (the last round may be part-filled)
      const int x = it * 256 + tid - (it * 256 < S::ZU ? 0 : S::ZU), n = it * 256 < S::ZU ? S::ZU : S::UU;
      return (x < n ? x : n - 1) / EQ;
    };
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned char* r = it * 256 < S::ZU ? a.zE + (size_t)e[i] * H2 * ESZ : a.u + (size_t)ur[i] * DL * ESZ;
        v[it][i] = *reinterpret_cast<const uint4*>(r + unit(it) * 16);
      }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * eq + i >= cnt) v[it][i] = make_uint4(0, 0, 0, 0);
      if (it * 256 + tid < S::ZU + S::UU)
        put4_transposed<T, S::ROWB>(v[it], unit(it), 4 * eq, it * 256 < S::ZU ? zt : ut);
    }
    __syncthreads();
    const int nks = (cnt + KS - 1) / KS;
    for (int ks = 0; ks < nks; ++ks) {
      const int col = (ks * KS + hh * EPL) * ESZ;
#pragma unroll
      for (int j = 0; j < S::TPW; ++j) {
        const int ti = wv + 4 * j;
        if (ti < S::NTILE) {
          const int kt = ti / S::NCT, ct = ti % S::NCT;
          const auto A = ldf<T>(zt + (kt * 32 + l32) * S::ROWB + col);
          const auto B = ldf<T>(ut + (ct * 32 + l32) * S::ROWB + col);
          acc[j] = M::mma(A, B, acc[j]);
        }
      }
    }
    if (tid < DL) {
      const T* row = reinterpret_cast<const T*>(ut + tid * S::ROWB);
      for (int s = 0; s < cnt; s += 8) {   // in order, eight reads at a time (zeros past cnt)
        float x[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = (float)row[s + t];
#pragma unroll
        for (int t = 0; t < 8; ++t) hs += x[t];
      }
    }
  }

  unsigned char* o = a.out + (size_t)n * S::KTOT * ESZ;
#pragma unroll
  for (int j = 0; j < S::TPW; ++j) {
    const int ti = wv + 4 * j;
    if (ti < S::NTILE) {
      unsigned char* dst = o + ((size_t)ti * 1024 + lane * 16) * ESZ;
      if constexpr (ESZ == 2) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = acc[j][r];
        *reinterpret_cast<bf16x8*>(dst) = pack_frag<__bf16>(v);
        *reinterpret_cast<bf16x8*>(dst + 16) = pack_frag<__bf16>(v + 8);
      } else {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *reinterpret_cast<f32x4*>(dst + r4 * 16) =
              f32x4{acc[j][4 * r4], acc[j][4 * r4 + 1], acc[j][4 * r4 + 2], acc[j][4 * r4 + 3]};
      }
    }
  }
  if (tid < DL) reinterpret_cast<T*>(o)[(size_t)H2 * DL + tid] = (T)hs;
}

// bf16 (sums over the edges of a destination, CSR order): the chunk's rows of z
// and of the gathered rows are copied to LDS as they are (each wave-wide load
// covers four whole z rows or eight gathered rows), and the fragments, whose
// contraction index is the edge, come from transposing LDS reads.  Slots past
// the segment's last edge re-read its last edge and are zeroed in the A
// fragment.
template <int DL, int H2, int ECH_ = 64>
struct OuterTrShape {
  static constexpr int ECH = ECH_;                             // edges per staged chunk
  static constexpr int ZPAD = tr_pad_units(H2 * 2), UPAD = tr_pad_units(DL * 2);
  static constexpr int ZP = H2 * 2 + 16 * ZPAD, UP = DL * 2 + 16 * UPAD;   // LDS row pitches
  static constexpr int ZNU = H2 * 2 / 16, UNU = DL * 2 / 16;   // 16-byte units per row
  static constexpr int ZU = ECH * (ZNU + ZPAD), UU = ECH * (UNU + UPAD);
  static constexpr int NKT = H2 / 32, NCT = DL / 32, NTILE = NKT * NCT, TPW = (NTILE + 3) / 4;
  static constexpr int LDS = ECH * (ZP + UP);
  static constexpr int64_t KTOT = (int64_t)H2 * DL + DL;
};

// One 32x32 tile of sums to the 2 KB at o in the K order (lane l's sixteen
// values at 32 l).  A store instruction of 16 bytes per lane would cover half
// of every line; lanes l and l ^ 7 trade halves, so that the first instruction
// writes the lines of the lanes with bit 2 clear whole and the second the
// others.  STREAM: with the non-temporal hint (as a template argument: the
// compiler folds the two stores of a run-time choice into plain ones).
template <bool STREAM>
__device__ __forceinline__ void store_tile_lines(unsigned char* o, const f32x16& acc) {
  const int lane = threadIdx.x & 63;
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = acc[r];
  const f32x4 lo = __builtin_bit_cast(f32x4, pack_frag<__bf16>(v));
  const f32x4 hi = __builtin_bit_cast(f32x4, pack_frag<__bf16>(v + 8));
  const bool up = lane & 4;
  f32x4 other;   // the partner's half: its upper one for the first line, its lower one for the second
#pragma unroll
  for (int x = 0; x < 4; ++x)   // DPP row_half_mirror: lane l reads lane l ^ 7
    other[x] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(up ? lo[x] : hi[x]), 0x141, 0xf, 0xf, true));
  const int p = lane ^ 7;
  f32x4* o1 = reinterpret_cast<f32x4*>(o + (up ? 2 * p + 1 : 2 * lane) * 16);
  f32x4* o2 = reinterpret_cast<f32x4*>(o + (up ? 2 * lane + 1 : 2 * p) * 16);
  const f32x4 v1 = up ? other : lo, v2 = up ? hi : other;
  if constexpr (STREAM) {
    __builtin_nontemporal_store(v1, o1);
    __builtin_nontemporal_store(v2, o2);
  } else {
    *o1 = v1;
    *o2 = v2;
  }
}

// One segment per workgroup of four waves: the dispatcher balances segments of
// uneven length, and as many workgroups as fit hide each other's chain of
// loads (bounds, source ids, rows).  So a chunk takes little LDS (32 slots
// where the mean segment is no longer than that: 16 KB at d = 64, eight
// workgroups per CU) and only the rows of its 16-edge products are copied; the
// source ids go straight from memory into the copies' addresses.
// 100,000 segments of 10.8 edges (d = 64): 597 -> 397 us (4.2 TB/s written);
// 30,011 of 21: 175 -> 107 us; 8,192 of 40: 55 -> 51 us.
template <int DL, int H2, int ECH, bool STREAM>
__global__ __launch_bounds__(256, 6) void k_outer_sum_tr(OuterArgs a) {
  using S = OuterTrShape<DL, H2, ECH>;
  using M = MT<__bf16>;
  constexpr int TPW = S::TPW, ZR = S::ZNU + S::ZPAD, UR = S::UNU + S::UPAD;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* zl = smem;
  unsigned char* ul = smem + ECH * S::ZP;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, hh = lane >> 5, wbase = tid & ~63;
  typedef __attribute__((address_space(4))) const int32_t cint32_t;
  cint32_t* sp = (cint32_t*)(a.seg_ptr);
  const int64_t n = blockIdx.x;
  const int64_t pa = sp[n], pb = sp[n + 1];
  f32x16 acc[TPW];
#pragma unroll
  for (int j = 0; j < TPW; ++j) acc[j] = f32x16{};
  float hs = 0.0f;   // z~ = 1 row: sum of the gathered rows (threads tid < DL)
  for (int64_t c0 = pa; c0 < pb; c0 += ECH) {
    const int cnt = (int)(pb - c0 < ECH ? pb - c0 : ECH), nks = (cnt + 15) / 16, rows = nks * 16;
    if (c0 > pa) __syncthreads();   // previous chunk fully consumed
    // the gathered rows' ids first: their copies wait for them
    constexpr int UI = (S::UU + 255) / 256;
    int id[UI];
#pragma unroll
    for (int k = 0; k < UI; ++k) {
      const int r = (k * 256 + tid) / UR;
      id[k] = k * 256 < rows * UR ? a.row_of[c0 + (r < cnt ? r : cnt - 1)] : 0;
    }
    for (int U0 = 0; U0 < rows * ZR; U0 += 256) {
      const int U = U0 + tid, r = U / ZR, u = U % ZR;
      if (U < rows * ZR)
        __builtin_amdgcn_global_load_lds(
            (gbl_void_t*)(a.zE + (size_t)(c0 + (r < cnt ? r : cnt - 1)) * H2 * 2 + (u < S::ZNU ? u : 0) * 16),
            (lds_void_t*)(zl + (size_t)(U0 + wbase) * 16), 16, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < UI; ++k) {
      const int U = k * 256 + tid, u = U % UR;
      if (U < rows * UR)
        __builtin_amdgcn_global_load_lds((gbl_void_t*)(a.u + (size_t)id[k] * DL * 2 + (u < S::UNU ? u : 0) * 16),
                                         (lds_void_t*)(ul + (size_t)(k * 256 + wbase) * 16), 16, 0, 0);
    }
    stage_wait();
    __syncthreads();
    for (int ks = 0; ks < nks; ++ks) {
#pragma unroll
      for (int j = 0; j < TPW; ++j) {
        const int ti = wv + 4 * j;
        if (ti < S::NTILE) {
          const int kt = ti / S::NCT, ct = ti % S::NCT;
          bf16x8 A = lds_frag_rows(zl, S::ZP, ks * 16, kt * 32);
          if (ks * 16 + 16 > cnt) {   // slots past the last edge
#pragma unroll
            for (int t = 0; t < 8; ++t)
              if (ks * 16 + 8 * hh + t >= cnt) A[t] = (__bf16)0.0f;
          }
          acc[j] = M::mma(A, lds_frag_rows(ul, S::UP, ks * 16, ct * 32), acc[j]);
        }
      }
    }
    if (tid < DL)
      for (int e = 0; e < cnt; ++e) hs += (float)*reinterpret_cast<const __bf16*>(ul + e * S::UP + tid * 2);
  }

  unsigned char* o = a.out + (size_t)n * S::KTOT * 2;
#pragma unroll
  for (int j = 0; j < TPW; ++j) {
    const int ti = wv + 4 * j;
    if (ti < S::NTILE) {
      store_tile_lines<STREAM>(o + (size_t)ti * 2048, acc[j]);
    }
  }
  if (tid < DL) reinterpret_cast<__bf16*>(o)[(size_t)H2 * DL + tid] = (__bf16)hs;
}

// ------------------------------------------------------------ GEMM with W3~

struct GemmArgs {
  int64_t n_rows, ktot;
  const unsigned char* A;    // [n_rows][ktot] layer dtype (segment sums)
  const unsigned char* BT;   // [DL][ktot] layer dtype (packed W3~ in the sum order)
  int nsl;                   // K slices
  int64_t csl;               // K chunks per slice
  float* part;               // [nsl][n_rows][DL] partial products
};

template <typename T, int DL>
struct GemmShape {
  static constexpr int ESZ = sizeof(T), KS = MT<T>::KS;
  static constexpr int CB = 128, SPC = CB / (KS * ESZ);   // bytes of a row per chunk, K steps per chunk
  static constexpr int AB = 128 * RowStage<128>::PITCH, BB = DL * RowStage<DL>::PITCH;
  static constexpr int BUF = AB + BB, LDS = 2 * BUF;
};

// part[s][n][c] = sum over slice s of K:  A[n][K] * BT[c][K].  A workgroup
// owns 128 rows (32 per wave) and all d columns of one K slice.  K advances
// in chunks of 128 bytes per row: the chunk of the 128 A rows and the d BT
// rows is copied to LDS by whole cache lines while the previous chunk is
// multiplied (two buffers).
template <typename T, int DL>
__global__ __launch_bounds__(256) void k_w3_gemm(GemmArgs a) {
  using M = MT<T>;
  using G = GemmShape<T, DL>;
  constexpr int KS = M::KS, EPL = M::EPL, ESZ = sizeof(T), NCT = DL / 32, SPC = G::SPC;
  constexpr int PITCH = RowStage<128>::PITCH;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int64_t r0 = (int64_t)blockIdx.x * 128;
  const int s = blockIdx.y;
  const int64_t nstep = a.ktot / KS, nchunk = (nstep + SPC - 1) / SPC;
  const int64_t c0 = s * a.csl, c1 = c0 + a.csl < nchunk ? c0 + a.csl : nchunk;
  f32x16 acc[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) acc[ct] = f32x16{};
  if (c0 < c1) {   // uniform over the workgroup; an empty slice writes zeros
  const int nvalid = (int)(a.n_rows - r0 < 128 ? a.n_rows - r0 : 128);
  RowStage<128> sa;
  RowStage<DL> sb;
  sa.init(a.ktot * ESZ, nvalid);
  sb.init(a.ktot * ESZ, DL);
  const unsigned char* ga = a.A + (size_t)r0 * a.ktot * ESZ;
  sa.issue(ga + c0 * G::CB, smem);
  sb.issue(a.BT + c0 * G::CB, smem + G::AB);
  stage_wait();
  __syncthreads();
  for (int64_t c = c0; c < c1; ++c) {
    unsigned char* cur = smem + ((c - c0) & 1) * G::BUF;
    if (c + 1 < c1) {
      unsigned char* nxt = smem + ((c + 1 - c0) & 1) * G::BUF;
      sa.issue(ga + (c + 1) * G::CB, nxt);
      sb.issue(a.BT + (c + 1) * G::CB, nxt + G::AB);
    }
    const int nst = (int)(nstep - c * SPC < SPC ? nstep - c * SPC : SPC);
    const unsigned char* la = cur + (wv * 32 + l32) * PITCH + hh * EPL * ESZ;
    const unsigned char* lb = cur + G::AB + l32 * PITCH + hh * EPL * ESZ;
#pragma unroll
    for (int st = 0; st < SPC; ++st) {
      if (st < nst) {
        const auto A = ldf<T>(la + st * KS * ESZ);
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          acc[ct] = M::mma(A, ldf<T>(lb + ct * 32 * PITCH + st * KS * ESZ), acc[ct]);
      }
    }
    stage_wait();
    __syncthreads();
  }
  }
  float* out = a.part + (size_t)s * a.n_rows * DL;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t rr = r0 + wv * 32 + 8 * (r / 4) + 4 * hh + (r % 4);
      if (rr < a.n_rows) out[rr * DL + ct * 32 + l32] = acc[ct][r];
    }
}

// ------------------------------------------------------------ dW3 from S

struct DW3AggArgs {
  int64_t n_rows, ktot, kcols;
  const unsigned char* OS;   // [n_rows][ktot] layer dtype
  const unsigned char* G;    // [n_rows][DL] layer dtype (g_i)
  int nsl;
  int64_t rows_per_sl;       // multiple of 64
  float* part;               // [nsl][DL][kcols]
};

template <typename T, int DL>
struct DW3AggShape {
  static constexpr int KS = MT<T>::KS, EPL = MT<T>::EPL, ESZ = sizeof(T);
  static constexpr int NCH = 64, KR = 256;              // rows per chunk, K columns per workgroup
  static constexpr int NQT = DL / 32, NKT = KR / 32, NTILE = NQT * NKT, TPW = NTILE / 4;
  static constexpr int ROWB = (NCH + 16 / ESZ) * ESZ;
  static constexpr int OU = (NCH / 4) * (KR * ESZ / 16), GU = (NCH / 4) * (DL * ESZ / 16);
  static constexpr int LDS = (KR + DL) * ROWB;
  static_assert(NTILE % 4 == 0, "tiles split over four waves");
};

// part[s][q][K] = sum over the rows of slice s of g[i][q] * S[i][K]: rows of
// S and g staged transposed to [column][row], rows are the contraction index.
// fp32 layers; a chunk's loads go out together (1,024 rows, d = 32: 19.3 -> 14.0
// us with the final sum).
template <typename T, int DL>
__global__ __launch_bounds__(256) void k_dw3_agg(DW3AggArgs a) {
  using S = DW3AggShape<T, DL>;
  using M = MT<T>;
  constexpr int KS = S::KS, EPL = S::EPL, ESZ = S::ESZ, NCH = S::NCH;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* ot = smem;
  unsigned char* gt = smem + S::KR * S::ROWB;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int64_t kc0 = (int64_t)blockIdx.x * S::KR;
  const int s = blockIdx.y;
  const int64_t rb = s * a.rows_per_sl;
  const int64_t re = rb + a.rows_per_sl < a.n_rows ? rb + a.rows_per_sl : a.n_rows;
  f32x16 acc[S::TPW];
#pragma unroll
  for (int j = 0; j < S::TPW; ++j) acc[j] = f32x16{};
  for (int64_t c0 = rb; c0 < re; c0 += NCH) {
    const int cnt = (int)(re - c0 < NCH ? re - c0 : NCH);
    __syncthreads();
    constexpr int EQ = NCH / 4, NIT = (S::OU + S::GU + 255) / 256;
    static_assert(S::OU % 256 == 0 && 256 % EQ == 0, "whole rounds of S units");
    const int eq = tid % EQ;
    uint4 v[NIT][4];
    auto unit = [&](int it) {   // of a row of S, or of g (the last round may be part-filled)
      const int x = it * 256 + tid - (it * 256 < S::OU ? 0 : S::OU), n = it * 256 < S::OU ? S::OU : S::GU;
      return (x < n ? x : n - 1) / EQ;
    };
    // columns past the end of a row of S (last K block) read as zeros
    auto inrow = [&](int it) { return it * 256 >= S::OU || kc0 + (int64_t)unit(it) * (16 / ESZ) < a.kcols; };
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = c0 + (4 * eq + i < cnt ? 4 * eq + i : cnt - 1);
        const unsigned char* r = it * 256 < S::OU ? a.OS + ((size_t)row * a.ktot + kc0) * ESZ + (inrow(it) ? unit(it) * 16 : 0)
                                                  : a.G + (size_t)row * DL * ESZ + unit(it) * 16;
        v[it][i] = *reinterpret_cast<const uint4*>(r);
      }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * eq + i >= cnt || !inrow(it)) v[it][i] = make_uint4(0, 0, 0, 0);
      if (it * 256 + tid < S::OU + S::GU)
        put4_transposed<T, S::ROWB>(v[it], unit(it), 4 * eq, it * 256 < S::OU ? ot : gt);
    }
    __syncthreads();
    const int nks = (cnt + KS - 1) / KS;
    for (int ks = 0; ks < nks; ++ks) {
      const int col = (ks * KS + hh * EPL) * ESZ;
#pragma unroll
      for (int j = 0; j < S::TPW; ++j) {
        const int ti = wv * S::TPW + j, qt = ti / S::NKT, kt = ti % S::NKT;
        acc[j] = M::mma(ldf<T>(gt + (qt * 32 + l32) * S::ROWB + col), ldf<T>(ot + (kt * 32 + l32) * S::ROWB + col),
                        acc[j]);
      }
    }
  }
  float* out = a.part + (size_t)s * DL * a.kcols;
#pragma unroll
  for (int j = 0; j < S::TPW; ++j) {
    const int ti = wv * S::TPW + j, qt = ti / S::NKT, kt = ti % S::NKT;
    const int64_t kc = kc0 + kt * 32 + l32;
    if (kc < a.kcols)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[(size_t)(qt * 32 + 8 * (r / 4) + 4 * hh + (r % 4)) * a.kcols + kc] = acc[j][r];
  }
}

// bf16 layers: the same sums with chunks of 32 rows of S (a piece of KR K
// columns: 256, or 128 at d = 128, which halves the accumulators per wave and
// measured 1.5x faster there) and of g copied to LDS by whole cache lines,
// two buffers, and the fragments read by transposing LDS reads (rows are the
// contraction index).  Wave w owns TPW consecutive K tiles of one q tile, so
// one g fragment feeds TPW products.  Rows past the slice re-read its last
// row and are zeroed in the g fragment; columns past the end of a row (last
// K block) are read from the next row (or the buffer's tail padding) and
// never stored.
template <int DL>
struct DW3TrShape {
  static constexpr int ECH = 32, KR = DL == 128 ? 128 : 256;
  using SS = RowStage<ECH, KR * 2, tr_pad_units(KR * 2)>;
  using GS = RowStage<ECH, DL * 2, tr_pad_units(DL * 2)>;
  static constexpr int SB = ECH * SS::PITCH, BUF = SB + ECH * GS::PITCH, LDS = 2 * BUF;
  static constexpr int NQT = DL / 32, NKT = KR / 32, TPW = NQT * NKT / 4;
  static_assert(TPW % 4 == 0 || TPW == 2, "K tiles per wave");
};

template <int DL>
__global__ __launch_bounds__(256) void k_dw3_agg_tr(DW3AggArgs a) {
  using S = DW3TrShape<DL>;
  using M = MT<__bf16>;
  constexpr int ECH = S::ECH, TPW = S::TPW;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int64_t kc0 = (int64_t)blockIdx.x * S::KR;
  const int s = blockIdx.y;
  const int64_t rb = s * a.rows_per_sl;
  const int64_t re = rb + a.rows_per_sl < a.n_rows ? rb + a.rows_per_sl : a.n_rows;
  // the wave's tiles: ti = wv*TPW + j  ->  qt = ti / NKT, kt = ti % NKT (one qt per wave)
  const int qt = (wv * TPW) / S::NKT, kt0 = (wv * TPW) % S::NKT;
  f32x16 acc[TPW];
#pragma unroll
  for (int j = 0; j < TPW; ++j) acc[j] = f32x16{};
  if (rb < re) {   // uniform over the workgroup
    const int nch = (int)((re - rb + ECH - 1) / ECH);
    typename S::SS ss;
    typename S::GS sg;
    auto issue = [&](int c, unsigned char* buf) {
      const int64_t r0 = rb + (int64_t)c * ECH;
      const int nv = (int)(re - r0 < ECH ? re - r0 : ECH);
      ss.init(a.ktot * 2, nv);
      sg.init(DL * 2, nv);
      ss.issue(a.OS + ((size_t)r0 * a.ktot + kc0) * 2, buf);
      sg.issue(a.G + (size_t)r0 * DL * 2, buf + S::SB);
    };
    issue(0, smem);
    stage_wait();
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
      const unsigned char* cur = smem + (c & 1) * S::BUF;
      if (c + 1 < nch) issue(c + 1, smem + ((c + 1) & 1) * S::BUF);
      const int64_t r0 = rb + (int64_t)c * ECH;
      const int cnt = (int)(re - r0 < ECH ? re - r0 : ECH);
      for (int ks = 0; ks * 16 < cnt; ++ks) {
        bf16x8 A = lds_frag_rows(cur + S::SB, S::GS::PITCH, ks * 16, qt * 32);
        if (ks * 16 + 16 > cnt) {
#pragma unroll
          for (int t = 0; t < 8; ++t)
            if (ks * 16 + 8 * hh + t >= cnt) A[t] = (__bf16)0.0f;
        }
#pragma unroll
        for (int j = 0; j < TPW; ++j)
          acc[j] = M::mma(A, lds_frag_rows(cur, S::SS::PITCH, ks * 16, (kt0 + j) * 32), acc[j]);
      }
      stage_wait();
      __syncthreads();
    }
  }
  float* out = a.part + (size_t)s * DL * a.kcols;
#pragma unroll
  for (int j = 0; j < TPW; ++j) {
    const int64_t kc = kc0 + (kt0 + j) * 32 + l32;
    if (kc < a.kcols)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[(size_t)(qt * 32 + 8 * (r / 4) + 4 * hh + (r % 4)) * a.kcols + kc] = acc[j][r];
  }
}

// dW3[p*d+q][k] (+)= sum_s part[s][q][K(k, p)], K in the sum order above;
// the bias rows K = h2*d + p give db3[p*d+q].
template <typename T>
__global__ __launch_bounds__(256) void k_dw3_agg_final(int d, int h2, int nsl, const float* __restrict__ part,
                                                       float* __restrict__ dW3, float* __restrict__ db3,
                                                       int accumulate) {
  const int64_t kcols = (int64_t)h2 * d + d, total = (int64_t)d * kcols;
  const int nct = d / 32;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total; x += (int64_t)gridDim.x * blockDim.x) {
    // x enumerates (q, K) with K fastest, so the reads of part are contiguous
    const int q = (int)(x / kcols);
    const int64_t K = x % kcols;
    const float v = ordered_sum(part + (int64_t)q * kcols + K, (int64_t)d * kcols, nsl);
    float* o;
    if (K < (int64_t)h2 * d) {
      const int ti = K / 1024, rem = K % 1024, l = rem / 16, r = rem % 16;
      const int kt = ti / nct, ct = ti % nct;
      const int kpos = kt * 32 + 8 * (r / 4) + 4 * (l / 32) + (r % 4), p = ct * 32 + (l % 32);
      o = dW3 + ((int64_t)p * d + q) * h2 + kperm<T>(kpos);
    } else {
      o = db3 + (K - (int64_t)h2 * d) * d + q;
    }
    *o = accumulate ? *o + v : v;
  }
}

// Persistent form of the outer-product sums for few workgroups per CU, with
// the first chunk of the next segment copied while this segment's sums are
// stored.  Loads and stores retire through one in-order counter, so a copy
// issued after a segment's stores would wait for them; here the copy goes out
// first, and the wait at the top of a segment leaves the previous segment's
// stores in flight.  The index chain runs ahead: edge ids two segments ahead,
// gathered-row ids one segment ahead, bounds by scalar loads.  Chunks after a
// segment's first (segments of more than ECH edges) are copied and multiplied
// in turn.  Barriers wait for LDS instructions only (lds_sync: a full
// barrier would wait for the stores).  The products, their order and the stored layout are those of
// k_outer_sum_tr.
template <int DL, int H2, int NW>
__global__ __launch_bounds__(64 * NW) void k_outer_sum_pf(OuterArgs a) {
  using S = OuterTrShape<DL, H2>;
  using M = MT<__bf16>;
  constexpr int ECH = S::ECH, NT = 64 * NW, TPW = (S::NTILE + NW - 1) / NW;
  static_assert(S::NTILE % NW == 0, "every wave holds TPW tiles");
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int rz[ECH], ru[ECH];   // source rows of the chunk's z and gathered rows
  unsigned char* zl = smem;
  unsigned char* ul = smem + ECH * S::ZP;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, hh = lane >> 5;
  const int64_t G = gridDim.x;
  typedef __attribute__((address_space(4))) const int32_t cint32_t;
  cint32_t* sp = (cint32_t*)(a.seg_ptr);
  auto bounds = [&](int64_t n, int64_t& p0, int64_t& p1) {   // empty past the last segment
    const int64_t nc = n < a.n_seg ? n : a.n_seg;
    p0 = sp[nc];
    p1 = n < a.n_seg ? (int64_t)sp[nc + 1] : p0;
  };
  // slot tid < ECH of a chunk takes the chunk's edge min(tid, cnt - 1)
  auto slot_pos = [&](int64_t c0, int64_t end) {
    const int cnt = (int)(end - c0 < ECH ? end - c0 : ECH);
    return c0 + (tid < cnt ? tid : cnt - 1);
  };
  auto edge_of = [&](int64_t pos) -> int { return a.pos_eid ? a.pos_eid[pos] : (int)pos; };
  auto copy_chunk = [&]() {
    const int wbase = tid & ~63;
    for (int U0 = 0; U0 < S::ZU; U0 += NT) {
      const int U = U0 + tid, r = U / (S::ZNU + S::ZPAD), u = U % (S::ZNU + S::ZPAD);
      if (U < S::ZU)
        __builtin_amdgcn_global_load_lds(
            (gbl_void_t*)(a.zE + (size_t)rz[r < ECH ? r : ECH - 1] * H2 * 2 + (u < S::ZNU ? u : 0) * 16),
            (lds_void_t*)(zl + (size_t)(U0 + wbase) * 16), 16, 0, 0);
    }
    for (int U0 = 0; U0 < S::UU; U0 += NT) {
      const int U = U0 + tid, r = U / (S::UNU + S::UPAD), u = U % (S::UNU + S::UPAD);
      if (U < S::UU)
        __builtin_amdgcn_global_load_lds(
            (gbl_void_t*)(a.u + (size_t)ru[r < ECH ? r : ECH - 1] * DL * 2 + (u < S::UNU ? u : 0) * 16),
            (lds_void_t*)(ul + (size_t)(U0 + wbase) * 16), 16, 0, 0);
    }
  };
  f32x16 acc[TPW];
  float hs = 0.0f;   // z~ = 1 row: sum of the gathered rows (threads tid < DL)
  auto multiply = [&](int cnt) {
    const int nks = (cnt + 15) / 16;
    for (int ks = 0; ks < nks; ++ks) {
#pragma unroll
      for (int j = 0; j < TPW; ++j) {
        const int ti = wv + NW * j;
        const int kt = ti / S::NCT, ct = ti % S::NCT;
        bf16x8 A = lds_frag_rows(zl, S::ZP, ks * 16, kt * 32);
        if (ks * 16 + 16 > cnt) {   // slots past the last edge
#pragma unroll
          for (int t = 0; t < 8; ++t)
            if (ks * 16 + 8 * hh + t >= cnt) A[t] = (__bf16)0.0f;
        }
        acc[j] = M::mma(A, lds_frag_rows(ul, S::UP, ks * 16, ct * 32), acc[j]);
      }
    }
    if (tid < DL)
      for (int e = 0; e < cnt; ++e) hs += (float)*reinterpret_cast<const __bf16*>(ul + e * S::UP + tid * 2);
  };

  int64_t n = blockIdx.x;
  if (n >= a.n_seg) return;
  int64_t pa, pb, pa1, pb1, pa2, pb2;
  bounds(n, pa, pb);
  bounds(n + G, pa1, pb1);
  bounds(n + 2 * G, pa2, pb2);
  // the first chunk of segment n, and the ids of segment n + G (and the edge
  // ids of n + 2G) ahead
  int pz1 = 0, pu1 = 0, pz2 = 0;
  if (tid < ECH && pb > pa) {
    const int z = edge_of(slot_pos(pa, pb));
    rz[tid] = z;
    ru[tid] = a.row_of[z];
  }
  if (tid < ECH && pb1 > pa1) pz1 = edge_of(slot_pos(pa1, pb1));
  lds_sync();
  if (pb > pa) copy_chunk();
  if (tid < ECH && pb1 > pa1) pu1 = a.row_of[pz1];
  bool first_iter = true;
  for (; n < a.n_seg; n += G) {
    // the copy of this segment's first chunk; after it only the previous
    // segment's stores (2 TPW per thread) went out
    if (first_iter) stage_wait();
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * TPW));
    first_iter = false;
    lds_sync();
    if (tid < ECH && pb2 > pa2) pz2 = edge_of(slot_pos(pa2, pb2));   // two segments ahead
#pragma unroll
    for (int j = 0; j < TPW; ++j) acc[j] = f32x16{};
    hs = 0.0f;
    if (pb > pa) multiply((int)(pb - pa < ECH ? pb - pa : ECH));
    for (int64_t c0 = pa + ECH; c0 < pb; c0 += ECH) {   // segments of more than ECH edges
      lds_sync();
      if (tid < ECH) {
        const int z = edge_of(slot_pos(c0, pb));
        rz[tid] = z;
        ru[tid] = a.row_of[z];
      }
      lds_sync();
      copy_chunk();
      stage_wait();
      lds_sync();
      multiply((int)(pb - c0 < ECH ? pb - c0 : ECH));
    }
    unsigned char* o = a.out + (size_t)n * S::KTOT * 2;
    // the z~ = 1 row before the next copy, so that exactly 2 TPW stores follow it
    if (tid < DL) reinterpret_cast<__bf16*>(o)[(size_t)H2 * DL + tid] = (__bf16)hs;
    lds_sync();   // every wave is done with the chunk buffers and ids
    if (tid < ECH && pb1 > pa1) {
      rz[tid] = pz1;
      ru[tid] = pu1;
    }
    lds_sync();
    if (pb1 > pa1) copy_chunk();   // segment n + G's first chunk, ahead of this segment's stores
    if (tid < ECH && pb2 > pa2) pu1 = a.row_of[pz2];
    pz1 = pz2;
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
      const int ti = wv + NW * j;
      unsigned char* dst = o + ((size_t)ti * 1024 + lane * 16) * 2;
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = acc[j][r];
      *reinterpret_cast<bf16x8*>(dst) = pack_frag<__bf16>(v);
      *reinterpret_cast<bf16x8*>(dst + 16) = pack_frag<__bf16>(v + 8);
    }
    pa = pa1; pb = pb1;
    pa1 = pa2; pb1 = pb2;
    bounds(n + 3 * G, pa2, pb2);
  }
}

template <typename K>
dsmp_status set_lds_bytes(dsmp_handle* h, K kernel, int bytes) {
  DSMP_HIP(h, hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  return DSMP_OK;
}

template <typename T, int DL, int H2>
dsmp_status outer_shape(dsmp_handle* h, const OuterArgs& a) {
  if constexpr (sizeof(T) == 2) {
    using S = OuterTrShape<DL, H2>;
    if constexpr (DL <= 64) {
      DSMP_CHECK(h, a.pos_eid == nullptr, DSMP_UNSUPPORTED,
                 "bf16 outer-product sums of d <= 64 take the edges in their stored order only");
      // chunks of 32 slots where the mean segment has no more edges
      const bool few = a.n_edges <= 32 * a.n_seg;
      auto kern = few ? (a.stream ? k_outer_sum_tr<DL, H2, 32, true> : k_outer_sum_tr<DL, H2, 32, false>)
                      : (a.stream ? k_outer_sum_tr<DL, H2, 64, true> : k_outer_sum_tr<DL, H2, 64, false>);
      constexpr int lds32 = OuterTrShape<DL, H2, 32>::LDS;
      static_assert(S::LDS <= 65536, "no attribute needed");
      hipLaunchKernelGGL(kern, dim3((unsigned)a.n_seg), dim3(256), few ? lds32 : S::LDS, h->stream, a);
    } else {
      // two workgroups fit on a CU: eight waves each, the next segment's first
      // chunk copied ahead of this segment's stores
      auto kern = k_outer_sum_pf<DL, H2, 8>;
      dsmp_status st = set_lds_bytes(h, kern, S::LDS);
      if (st != DSMP_OK) return st;
      int per_cu = 0;
      DSMP_HIP(h, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 512, S::LDS));
      hipLaunchKernelGGL(kern, dim3((unsigned)std::min<int64_t>(a.n_seg, (int64_t)h->n_cu * std::max(per_cu, 1))),
                         dim3(512), S::LDS, h->stream, a);
    }
  } else {
    using S = OuterShape<T, DL, H2>;
    auto kern = k_outer_sum<T, DL, H2>;
    dsmp_status st = set_lds_bytes(h, kern, S::LDS);
    if (st != DSMP_OK) return st;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.n_seg), dim3(256), S::LDS, h->stream, a);
  }
  DSMP_LAUNCHED(h, "segment outer-product sums");
  return DSMP_OK;
}

template <typename T, int DL>
dsmp_status gemm_shape(dsmp_handle* h, const GemmArgs& a) {
  using G = GemmShape<T, DL>;
  auto kern = k_w3_gemm<T, DL>;
  dsmp_status st = set_lds_bytes(h, kern, G::LDS);
  if (st != DSMP_OK) return st;
  hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(a.n_rows, 128), (unsigned)a.nsl), dim3(256), G::LDS, h->stream, a);
  DSMP_LAUNCHED(h, "W3 GEMM over segment sums");
  return DSMP_OK;
}

template <typename T, int DL>
dsmp_status dw3_shape(dsmp_handle* h, const DW3AggArgs& a) {
  if constexpr (sizeof(T) == 2) {
    using S = DW3TrShape<DL>;
    auto kern = k_dw3_agg_tr<DL>;
    dsmp_status st = set_lds_bytes(h, kern, S::LDS);
    if (st != DSMP_OK) return st;
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(a.kcols, S::KR), (unsigned)a.nsl), dim3(256), S::LDS,
                       h->stream, a);
  } else {
    using S = DW3AggShape<T, DL>;
    auto kern = k_dw3_agg<T, DL>;
    dsmp_status st = set_lds_bytes(h, kern, S::LDS);
    if (st != DSMP_OK) return st;
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(a.kcols, S::KR), (unsigned)a.nsl), dim3(256), S::LDS, h->stream,
                       a);
  }
  DSMP_LAUNCHED(h, "dW3 from segment sums");
  return DSMP_OK;
}

}  // namespace

namespace dsmp {

int64_t agg_ktot(const dsmp_layer_desc& d) { return (int64_t)d.h2 * d.d + d.d; }

bool use_aggregate(const dsmp_handle* h, const dsmp_layer_desc& d, int64_t n_dst, int64_t E) {
  if (h->edge_algo == DSMP_EDGE_PER_EDGE) return false;
  if (h->edge_algo == DSMP_EDGE_AGGREGATE) return true;
  return n_dst > 0 && E * d.d >= 512 * n_dst;
}

int agg_gemm_slices(int64_t n_rows, const dsmp_layer_desc& d) {
  const int64_t waves = ceil_div(n_rows, 32);
  int nsl = (int)(2048 / (waves > 0 ? waves : 1));
  if (nsl < 1) nsl = 1;
  if (nsl > 16) nsl = 16;
  return nsl;
}

dsmp_status launch_outer_sum(dsmp_handle* h, const dsmp_layer_desc& d, int64_t n_seg, int64_t n_edges,
                             const int32_t* seg_ptr, const int32_t* pos_eid, const int32_t* row_of, const unsigned char* zE,
                             const unsigned char* u, unsigned char* out) {
  if (n_seg == 0) return DSMP_OK;
  // sums larger than the 256 MB last-level cache are not in it when they are
  // next read (100,000 segments at d = 64, 1.65 GB: the sums 388 -> 397 us,
  // the product after them 475 -> 430; 30,011, 495 MB: 115 -> 107 and 160 -> 150; 8,192
  // segments, 135 MB: 34 -> 39 us)
  const int stream = n_seg * agg_ktot(d) * (d.dtype == DSMP_BF16 ? 2 : 4) > (256ll << 20);
  OuterArgs a{n_seg, seg_ptr, pos_eid, row_of, zE, u, out, n_edges, stream};
  if (d.dtype == DSMP_F32) {
    if (d.d == 32) return outer_shape<float, 32, 64>(h, a);
    if (d.d == 64) return outer_shape<float, 64, 128>(h, a);
  } else {
    if (d.d == 32) return outer_shape<__bf16, 32, 64>(h, a);
    if (d.d == 64) return outer_shape<__bf16, 64, 128>(h, a);
    if (d.d == 128) return outer_shape<__bf16, 128, 256>(h, a);
  }
  return fail(h, DSMP_UNSUPPORTED, "unsupported layer shape");
}

dsmp_status launch_w3_gemm(dsmp_handle* h, const dsmp_layer_desc& d, int64_t n_rows, const unsigned char* A,
                           const unsigned char* BT, int nsl, float* part) {
  if (n_rows == 0) return DSMP_OK;
  const int64_t ktot = agg_ktot(d);
  const int esz = d.dtype == DSMP_F32 ? 4 : 2;
  const int64_t nchunk = ceil_div(ktot * esz, 128);
  GemmArgs a{n_rows, ktot, A, BT, nsl, ceil_div(nchunk, nsl), part};
  if (d.dtype == DSMP_F32) {
    if (d.d == 32) return gemm_shape<float, 32>(h, a);
    if (d.d == 64) return gemm_shape<float, 64>(h, a);
  } else {
    if (d.d == 32) return gemm_shape<__bf16, 32>(h, a);
    if (d.d == 64) return gemm_shape<__bf16, 64>(h, a);
    if (d.d == 128) return gemm_shape<__bf16, 128>(h, a);
  }
  return fail(h, DSMP_UNSUPPORTED, "unsupported layer shape");
}

// Row slices of the dW3 product: 16 (at least 64 rows each).  Measured at
// the five workloads, 16 slices were as fast as or faster than 4, 8, 24 and
// 32 (fewer slices cut the partial sums' traffic but leave CUs idle; more add
// partials without speed).
int agg_dw3_slices(int64_t n_rows) {
  int64_t nsl = ceil_div(n_rows, 64);
  if (nsl < 1) nsl = 1;
  if (nsl > 16) nsl = 16;
  return (int)nsl;
}

dsmp_status launch_dw3_agg(dsmp_handle* h, const dsmp_layer_desc& d, int64_t n_rows, const unsigned char* OS,
                           const unsigned char* G, float* part, float* dW3, float* db3, int accumulate) {
  const int nsl = agg_dw3_slices(n_rows);
  const int64_t kcols = agg_ktot(d);
  if (n_rows > 0) {
    DW3AggArgs a{n_rows, agg_ktot(d), kcols, OS, G, nsl, ceil_div(ceil_div(n_rows, nsl), 64) * 64, part};
    dsmp_status st = DSMP_UNSUPPORTED;
    if (d.dtype == DSMP_F32) {
      if (d.d == 32) st = dw3_shape<float, 32>(h, a);
      if (d.d == 64) st = dw3_shape<float, 64>(h, a);
    } else {
      if (d.d == 32) st = dw3_shape<__bf16, 32>(h, a);
      if (d.d == 64) st = dw3_shape<__bf16, 64>(h, a);
      if (d.d == 128) st = dw3_shape<__bf16, 128>(h, a);
    }
    if (st != DSMP_OK) return st;
  }
  const int nuse = n_rows > 0 ? nsl : 0;
  const int64_t total = (int64_t)d.d * kcols;
  unsigned grid = (unsigned)ceil_div(total, 256);
  if (grid > 8192) grid = 8192;
  if (d.dtype == DSMP_F32)
    hipLaunchKernelGGL(k_dw3_agg_final<float>, dim3(grid), dim3(256), 0, h->stream, d.d, d.h2, nuse, part, dW3, db3,
                       accumulate);
  else
    hipLaunchKernelGGL(k_dw3_agg_final<__bf16>, dim3(grid), dim3(256), 0, h->stream, d.d, d.h2, nuse, part, dW3, db3,
                       accumulate);
  DSMP_LAUNCHED(h, "dW3 assembly");
  return DSMP_OK;
}

}  // namespace dsmp
