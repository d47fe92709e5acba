// Stage 1 of the pruned RNN-T loss: the trivial joiner of Sec. 3.1.
//
//   L_trivial(t,u,v) = am[t,v] + lm[u,v] - Z(t,u)               (Eq. (5))
//   Z(t,u) = log sum_v exp(am[t,v] + lm[u,v])                    (Eq. (6))
//
// Z is evaluated as the paper suggests, as an ordinary matrix product after
// applying offsets: with m_a[t] = max_v am[t,v] and m_l[u] = max_v lm[u,v],
//   Z(t,u) = m_a[t] + m_l[u] + log( sum_v e^{am[t,v]-m_a[t]} e^{lm[u,v]-m_l[u]} ),
// every factor is <= 1 so the product cannot overflow. The contraction over v
// runs on fp32 MFMA (short vocabularies) or three bf16 planes; the exponentials are formed while staging tiles to LDS
// and the px/py lookups (Eqs. (1)-(2)) are fused into the epilogue.
//
// The gradient w.r.t. am and lm (the simple loss is trained, Sec. 3.3) is two
// more contractions of the same shape:
//   d am[t,v] = sc (e^{am-m_a}[t,v] * sum_u W(t,u) e^{lm-m_l}[u,v]
//                   - sum_u gx(t,u) [v = y_{u+1}] - sum_u gy(t,u) [v = blank])
//   d lm[u,v] = sc (e^{lm-m_l}[u,v] * sum_t W(t,u) e^{am-m_a}[t,v]
//                   - sum_t gx(t,u) [v = y_{u+1}] - sum_t gy(t,u) [v = blank])
// with W(t,u) = (gx + gy)(t,u) e^{m_a + m_l - Z}: the log-softmax backward
// (gradient of the target/blank entries minus softmax times their sum).
//
// Smoothed joiner (Sec. 3.3.1), with weights a = a_lm, b = a_ac, c = 1-a-b:
//   L = c L_trivial + a L_lm + b L_acoustic,   L_lm(u,v) = lm[u,v] - Zlm[u],
//   L_acoustic(t,v) = am[t,v] + lavg[v] - Zac[t],
//   lavg[v] = log (1/(U+1)) sum_u e^{lm[u,v] - Zlm[u]},  Zlm, Zac row log-sum-exps.
// With Gx(u), Gy(u) the column sums and R(t) the row sums of gx + gy, and
// P_ac, P_lm the softmaxes of those joiners, the gradients gain
//   d am += b (R(t) P_ac[t,v] - sparse)       (sparse: the target/blank terms)
//   d lm += a ((Gx+Gy)(u) P_lm[u,v] - sparse) + b P_lm[u,v] (q[v] - s_u)
// where q[v] = g[v] / ((U+1) e^{lavg[v]}), g[v] = sum_t R(t) P_ac[t,v] - Sy(v)
// is the gradient w.r.t. lavg / b (Sy: target/blank column sums) and
// s_u = sum_v q[v] P_lm[u,v] (the chain rule through the average of softmaxes).
#include <float.h>

#include <cmath>

#include "gemm.h"
#include "kernels.h"
#include "prof.h"

namespace {

DEV float keep_nan_max(float m, float x) { return (x > m || x != x) ? x : m; }

// A workgroup barrier after this thread's LDS writes have completed. Unlike
// __syncthreads() it does not wait for outstanding global loads, so that the
// next step's loads stay in flight across it.
DEV void sg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

DEV float4 buf_load_f4(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}


// Length of each of `splits` contiguous K ranges over [0, K), a multiple of bk.
DEV int split_chunk(int K, int splits, int bk) { return ((K + splits - 1) / splits + bk - 1) / bk * bk; }

// ---------------------------------------------------------------------------
// Row maxima of am (rows t < T_n) and lm (rows u <= U_n): one wave per row.
// ---------------------------------------------------------------------------
// One wave per row: rows [0, N*T) of am, then rows [0, N*(U+1)) of lm.
__global__ __launch_bounds__(256) void rowmax_kernel(const float* __restrict__ am, const float* __restrict__ lm,
                                                     int N, int T, int U1, int V, BatchDev b,
                                                     float* __restrict__ m_a, float* __restrict__ m_l) {
  const int gr = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (gr >= N * (T + U1)) return;
  const int is_lm = gr >= N * T;
  const int row = is_lm ? gr - N * T : gr;
  const int R = is_lm ? U1 : T;
  const float* x = is_lm ? lm : am;
  float* out = is_lm ? m_l : m_a;
  const int n = row / R, i = row % R;
  int Tn, Un;
  utt_dims(b, n, Tn, Un);
  const int lim = is_lm ? Un + 1 : Tn;
  if (i >= lim) {
    if (lane == 0) out[row] = 0.f;
    return;
  }
  const float* r = x + (size_t)row * V;
  float m = kNegInfF;
  if ((V & 3) == 0) {
    const float4* r4 = reinterpret_cast<const float4*>(r);
#pragma unroll 4
    for (int v = lane; v < V / 4; v += 64) {
      float4 q = r4[v];
      m = keep_nan_max(m, q.x);
      m = keep_nan_max(m, q.y);
      m = keep_nan_max(m, q.z);
      m = keep_nan_max(m, q.w);
    }
  } else {
#pragma unroll 4
    for (int v = lane; v < V; v += 64) m = keep_nan_max(m, r[v]);
  }
  // within each 16-lane row by DPP rotations, then across the rows
  m = keep_nan_max(m, dpp_row_ror<8>(m));
  m = keep_nan_max(m, dpp_row_ror<4>(m));
  m = keep_nan_max(m, dpp_row_ror<2>(m));
  m = keep_nan_max(m, dpp_row_ror<1>(m));
  m = keep_nan_max(m, __shfl_xor(m, 16, 64));
  m = keep_nan_max(m, __shfl_xor(m, 32, 64));
  if (lane == 0) out[row] = m;
}

// ---------------------------------------------------------------------------
// Smoothing statistics (Sec. 3.3.1), one utterance's rows at a time.
// ---------------------------------------------------------------------------
// Zlm[n,u] = m_l + log sum_v e^{lm[u,v] - m_l}: one wave per row u <= U_n.
__global__ __launch_bounds__(256) void lm_lse_kernel(SimpleArgs a) {
  const int U1 = a.b.U + 1, V = a.V;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= a.b.N * U1) return;
  const int n = row / U1, u = row - n * U1;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  if (u > Un) {
    if (lane == 0) a.Zlm[row] = 0.f;
    return;
  }
  const float* x = a.lm + (size_t)row * V;
  const float m = a.m_l[row];
  float sum = 0.f;
  for (int v = lane; v < V; v += 64) sum += expf(x[v] - m);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (lane == 0) a.Zlm[row] = m + logf(sum);
}

// lavg[n,v] = log (1/(U_n+1)) sum_{u <= U_n} e^{lm[u,v] - Zlm[u]}: threads over v.
__global__ __launch_bounds__(256) void lm_avg_kernel(SimpleArgs a) {
  const int n = blockIdx.y, V = a.V, U1 = a.b.U + 1;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  const float* lmn = a.lm + (size_t)n * U1 * V;
  const float* z = a.Zlm + (size_t)n * U1;
  float s = 0.f;
#pragma unroll 8
  for (int u = 0; u <= Un; ++u) s += expf(lmn[(size_t)u * V + v] - z[u]);
  a.lavg[(size_t)n * V + v] = logf(s / (float)(Un + 1));
}

// Zac[n,t] = log sum_v e^{am[t,v] + lavg[v]}: one wave per frame t < T_n.
__global__ __launch_bounds__(256) void ac_lse_kernel(SimpleArgs a) {
  const int T = a.b.T, V = a.V;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= a.b.N * T) return;
  const int n = row / T, t = row - n * T;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  if (t >= Tn) {
    if (lane == 0) a.Zac[row] = 0.f;
    return;
  }
  const float* x = a.am + (size_t)row * V;
  const float* la = a.lavg + (size_t)n * V;
  float m = kNegInfF;
  for (int v = lane; v < V; v += 64) m = fmaxf(m, x[v] + la[v]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  float sum = 0.f;
  for (int v = lane; v < V; v += 64) sum += expf(x[v] + la[v] - m);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (lane == 0) a.Zac[row] = m + logf(sum);
}

// Gx[n,u], Gy[n,u]: column sums of the occupations over frames, from the
// per-16-frame partials in fixed order (fp64).
__global__ __launch_bounds__(256) void colsum_kernel(SimpleArgs a) {
  const int U1 = a.b.U + 1;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.b.N * U1) return;
  const int n = i / U1, u = i - n * U1;
  const double* px_ = a.cpx + (size_t)n * a.ncolblk * U1 + u;
  const double* py_ = a.cpy + (size_t)n * a.ncolblk * U1 + u;
  double cx = 0.0, cy = 0.0;
  // unrolled so that eight blocks' loads are in flight before the first add
  // (the adds keep their order)
#pragma unroll 8
  for (int q = 0; q < a.ncolblk; ++q) {
    cx += px_[(size_t)q * U1];
    cy += py_[(size_t)q * U1];
  }
  a.Gx[i] = cx;
  a.Gy[i] = cy;
}

// q[n,v] = (sum_t R(t) P_ac[t,v] - Sy(v)) / ((U_n+1) e^{lavg[v]}): kAcCols
// columns a block, its thread groups over the frames and the targets, their
// fp64 sums added in order. (One thread per column, every frame in turn, was
// a chain of dependent loads on a twentieth of the chip: 130 us at N = 13,
// T = 333, V = 1031.)
constexpr int kAcCols = 32, kAcGroups = 256 / kAcCols;
__global__ __launch_bounds__(256) void ac_colsum_kernel(SimpleArgs a) {
  __shared__ double part[kAcGroups][kAcCols];
  const int n = blockIdx.y, V = a.V, T = a.b.T, U1 = a.b.U + 1;
  const int c = threadIdx.x % kAcCols, grp = threadIdx.x / kAcCols;
  const int v = blockIdx.x * kAcCols + c;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  const float la = v < V ? a.lavg[(size_t)n * V + v] : 0.f;
  double g = 0.0;
  if (v < V) {
    const float* amn = a.am + (size_t)n * T * V;
#pragma unroll 8
    for (int t = grp; t < Tn; t += kAcGroups) {
      const double R = a.rx[(size_t)n * T + t] + a.ry[(size_t)n * T + t];
      g += R * (double)expf(amn[(size_t)t * V + v] + la - a.Zac[(size_t)n * T + t]);
    }
    for (int u = grp; u < Un; u += kAcGroups) {
      bool ok = true;
      if (symbol_at(a.b, n, u, V, ok) == v) g -= a.Gx[(size_t)n * U1 + u];
    }
    if (v == a.b.blank)
      for (int u = grp; u <= Un; u += kAcGroups) g -= a.Gy[(size_t)n * U1 + u];
  }
  part[grp][c] = g;
  __syncthreads();
  if (grp == 0 && v < V) {
    for (int k = 1; k < kAcGroups; ++k) g += part[k][c];
    a.q[(size_t)n * V + v] = (float)(g / ((double)(Un + 1) * (double)expf(la)));
  }
}

// su[n,u] = sum_v q[v] e^{lm[u,v] - Zlm[u]}: one wave per row u <= U_n.
__global__ __launch_bounds__(256) void lm_s_kernel(SimpleArgs a) {
  const int U1 = a.b.U + 1, V = a.V;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= a.b.N * U1) return;
  const int n = row / U1, u = row - n * U1;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  if (u > Un) return;
  const float* x = a.lm + (size_t)row * V;
  const float* qn = a.q + (size_t)n * V;
  const float z = a.Zlm[row];
  float sum = 0.f;
  for (int v = lane; v < V; v += 64) sum += qn[v] * expf(x[v] - z);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (lane == 0) a.su[row] = sum;
}

// Loads x[row][k..k+3] and the row max for exp(x - max); positions beyond the
// row end or of an invalid row load -inf, whose exponential is 0.
DEV void load_exp4(const float* x, const float* mx, int row, int k, int V, bool valid, RawExp<4>& r) {
  r.m = valid ? mx[row] : 0.f;
  const float* rowp = x + (size_t)(valid ? row : 0) * V;
  if (valid && ((V & 3) == 0) && (k + 4 <= V)) {
    float4 q = *reinterpret_cast<const float4*>(rowp + k);
    r.x[0] = q.x;
    r.x[1] = q.y;
    r.x[2] = q.z;
    r.x[3] = q.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) r.x[i] = (valid && k + i < V) ? rowp[k + i] : kNegInfF;
  }
}
// exp(x - max) of a staged operand (x <= max: the value lies in [0, 1]) with
// the hardware exp2: a few ulp, far below the contractions' fp32 rounding,
// and a fraction of the full-precision expf's instructions on the staging
// path that runs between the MFMAs.
DEV void finish_exp4(const RawExp<4>& r, float (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __expf(r.x[i] - r.m);
}
DEV void load_plain4(const float* p, bool valid, RawF<4>& r) {
  if (valid) {
    float4 q = *reinterpret_cast<const float4*>(p);
    r.v[0] = q.x;
    r.v[1] = q.y;
    r.v[2] = q.z;
    r.v[3] = q.w;
  } else {
    r.v[0] = r.v[1] = r.v[2] = r.v[3] = 0.f;
  }
}
DEV void finish_plain4(const RawF<4>& r, float (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = r.v[i];
}

// From this vocabulary on, the split gradient contractions take the 128 x 128
// tiles of 8 waves: enough tiles remain to fill the chip, and a 32 x 32 or
// 16 x 32 wave tile spends most of its time staging operands.
constexpr int kSimpleBigV = 2048;
using BigCfg = GemmCfg<128, 128, 32, 4, 2>;

// ---------------------------------------------------------------------------
// fp32 operands as three bf16 planes, x = p0 + p1 + p2 (8 significant bits
// each, rounded to nearest: together x to 2^-25 of it, over fp32's whole
// exponent range, which exponentials of misaligned rows and the occupation
// weights use; two fp16 planes would run out of range there). A product takes
// the six v_mfma_f32_16x16x32_bf16 whose planes' indices sum to at most 2 (the
// others are below 2^-24 of it) where fp32 MFMA takes eight 16x16x4, each as
// long as two of them.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any 4-byte address

DEV void split3(const float (&x)[8], uint4& p0, uint4& p1, uint4& p2) {
  uint32_t w[3][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float r[2] = {x[2 * q], x[2 * q + 1]};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const bf16x2 h = {(__bf16)r[0], (__bf16)r[1]};
      w[p][q] = __builtin_bit_cast(uint32_t, h);
      r[0] -= (float)h[0];
      r[1] -= (float)h[1];
    }
  }
  p0 = make_uint4(w[0][0], w[0][1], w[0][2], w[0][3]);
  p1 = make_uint4(w[1][0], w[1][1], w[1][2], w[1][3]);
  p2 = make_uint4(w[2][0], w[2][1], w[2][2], w[2][3]);
}

// acc += a b over one 32-long slice. The small products are summed by
// themselves, so that the running sum takes two roundings a slice: chained onto
// it (six roundings) the normaliser's mean error tripled (V = 8000: 6.3e-8
// against 2.3e-8 in the log-probs, 2.3e-8 with fp32 MFMA), for 17 us of 290.
DEV floatx4 mfma_split3(const bf16x8 (&a)[3], const bf16x8 (&b)[3], floatx4 acc) {
  floatx4 lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2], b[0], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[2], lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[0], lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[1], lo, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], acc + lo, 0, 0, 0);
}

// two at once, product by product
DEV void mfma_split3_pair(const bf16x8 (&a)[3], const bf16x8 (&b)[3], floatx4& acc, const bf16x8 (&c)[3],
                          const bf16x8 (&d)[3], floatx4& acc2) {
  constexpr int kA[5] = {2, 0, 1, 1, 0}, kB[5] = {0, 2, 1, 0, 1};
  floatx4 lo = {0.f, 0.f, 0.f, 0.f}, lo2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kA[p]], b[kB[p]], lo, 0, 0, 0);
    lo2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c[kA[p]], d[kB[p]], lo2, 0, 0, 0);
  }
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], acc + lo, 0, 0, 0);
  acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c[0], d[0], acc2 + lo2, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// Normaliser contraction, per utterance: C[t][u] = sum_v Ea[t][v] El[u][v],
// Ea = e^{am - m_a}, El = e^{lm - m_l}. One workgroup of 8 waves (4 x 2) per
// 128 frames, BN tokens and range of v: per step of 32 columns every thread
// loads 8 consecutive values of a row of am and of lm (a step ahead, held in
// registers across the barrier), forms their exponentials' planes once and
// stages them through one LDS stage of 24-48 KiB, so that two workgroups share
// a CU and one stages while the other computes. LDS rows are 64 bytes a plane,
// their four 16-byte chunks XOR-swizzled by the row, so that the fragment
// reads of 8 consecutive rows fall in distinct banks.
// Split over v into nsplit ranges (the contraction alone has too few tiles
// per batch to fill the chip); each writes its partial sums, and the epilogue
// kernel adds them in split order.
// ---------------------------------------------------------------------------
constexpr int kNsT = 128, kNsV = 32, kNsThreads = 512;
constexpr float kLog2eF = 1.44269504f;

struct NsRow {  // a staging thread's row of am or lm: its values from column v on, its maximum
  const float* p;
  float m;
  bool on;
};
DEV void ns_load(const NsRow& r, int v, int V, float (&x)[8]) {
  if (r.on && v + 8 <= V) {
    const f32x4u lo = *reinterpret_cast<const f32x4u*>(r.p + v), hi = *reinterpret_cast<const f32x4u*>(r.p + v + 4);
    x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
    x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = r.on && v + q < V ? r.p[v + q] : kNegInfF;  // its exponential is 0
  }
}
// chunk c of row r of a plane of 64-byte rows
DEV int ns_pos(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }
template <int ROWS>
DEV void ns_store(unsigned char* planes, int r, int c, const float (&x)[8], float m) {
  float e[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) e[q] = __builtin_amdgcn_exp2f((x[q] - m) * kLog2eF);
  uint4 p0, p1, p2;
  split3(e, p0, p1, p2);
  unsigned char* d = planes + ns_pos(r, c);
  *reinterpret_cast<uint4*>(d) = p0;
  *reinterpret_cast<uint4*>(d + ROWS * 64) = p1;
  *reinterpret_cast<uint4*>(d + 2 * ROWS * 64) = p2;
}
template <int ROWS>
DEV void ns_frag(const unsigned char* planes, int r, int c, bf16x8 (&f)[3]) {
  const unsigned char* s = planes + ns_pos(r, c);
#pragma unroll
  for (int p = 0; p < 3; ++p) f[p] = *reinterpret_cast<const bf16x8*>(s + p * ROWS * 64);
}

__host__ __device__ inline int ns_cols(int U1) { return U1 <= 64 ? 64 : U1 <= 96 || (U1 > 128 && U1 <= 192) ? 96 : 128; }

template <int BN>
__global__ __launch_bounds__(kNsThreads, 4) void normalizer_kernel(SimpleArgs a, int ntt, int ntu) {
  constexpr int FM = 2, FN = BN / 32;
  __shared__ __align__(16) unsigned char pa[3 * kNsT * 64], pb[3 * BN * 64];
  int b = blockIdx.x;
  const int tt = b % ntt; b /= ntt;
  const int tu = b % ntu; b /= ntu;
  const int sk = b % a.nsplit, n = b / a.nsplit;
  const int t0 = tt * kNsT, u0 = tu * BN;
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  if (t0 >= Tn || u0 > Un) return;
  const int kc = split_chunk(V, a.nsplit, kNsV);
  const int k0 = min(V, sk * kc), k1 = min(V, k0 + kc);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sr = tid >> 2, scol = (tid & 3) * 8;  // staging: row and first column of the step
  NsRow ra, rb;
  ra.on = t0 + sr < Tn;
  ra.p = a.am + ((size_t)n * T + (ra.on ? t0 + sr : 0)) * V;
  ra.m = ra.on ? a.m_a[(size_t)n * T + t0 + sr] : 0.f;
  rb.on = sr < BN && u0 + sr <= Un;
  rb.p = a.lm + ((size_t)n * U1 + (rb.on ? u0 + sr : 0)) * V;
  rb.m = rb.on ? a.m_l[(size_t)n * U1 + u0 + sr] : 0.f;
  const int wm = wave >> 1, wn = wave & 1, lr = lane & 15, lq = lane >> 4;
  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  float xa[8], xb[8];
  ns_load(ra, k0 + scol, k1, xa);
  ns_load(rb, k0 + scol, k1, xb);
  for (int k = k0; k < k1; k += kNsV) {
    ns_store<kNsT>(pa, sr, tid & 3, xa, ra.m);
    if (sr < BN) ns_store<BN>(pb, sr, tid & 3, xb, rb.m);
    sg_barrier();
    if (k + kNsV < k1) {
      ns_load(ra, k + kNsV + scol, k1, xa);
      ns_load(rb, k + kNsV + scol, k1, xb);
    }
    bf16x8 fa[FM][3];
#pragma unroll
    for (int i = 0; i < FM; ++i) ns_frag<kNsT>(pa, wm * 32 + i * 16 + lr, lq, fa[i]);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      bf16x8 fb[3];
      ns_frag<BN>(pb, wn * (BN / 2) + j * 16 + lr, lq, fb);
#pragma unroll
      for (int i = 0; i < FM; ++i) acc[i][j] = mfma_split3(fa[i], fb, acc[i][j]);
    }
    sg_barrier();
  }
  float* part = a.npart + ((size_t)sk * a.b.N + n) * T * U1;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + wm * 32 + i * 16 + 4 * lq + r;
      if (t >= Tn) continue;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int u = u0 + wn * (BN / 2) + j * 16 + lr;
        if (u <= Un) part[(size_t)t * U1 + u] = acc[i][j][r];
      }
    }
}

// Z = m_a + m_l + log(sum of the partials), px and py (Eqs. (1)-(2), (5)).
// A block takes a tile of kEpiTileCells cells: FT = kEpiTileCells / (64 R)
// frames of one utterance times the 64 R slots of a row of the lattice
// layout, kEpiNodes per thread with all their loads issued together (the
// kernel is a chain of two dependent load rounds: partial sums, offsets and
// symbols, then the am / lm values at the symbols). The nodes are formed in
// row-major order (coalesced reads of the partials and writes of Z, px,
// py), their diagonal-major copies go to LDS, and are then written diagonal
// by diagonal, so that the cells of one diagonal in the tile (consecutive
// slots) are written together. The blocks after the tiles fill the cells of
// the copies that no node of the rectangle maps to, kEpiNodes cells per
// thread. Small lattices take one node per thread (enough blocks to fill the
// chip), those of more than kEpiWideNodes nodes four.
constexpr int kEpiThreads = 512;
constexpr long long kEpiWideNodes = 1 << 20;
__host__ __device__ inline int epi_tile_frames(int R, int nodes) {
  const int f = kEpiThreads * nodes / (64 * R);
  return f > 1 ? f : 1;
}
static int epi_nodes(int N, int T, int U1) { return (long long)N * T * U1 > kEpiWideNodes ? 4 : 1; }

template <int kEpiNodes>
__global__ __launch_bounds__(kEpiThreads) void normalizer_epi_kernel(SimpleArgs a) {
  constexpr int kEpiTileCells = kEpiThreads * kEpiNodes < 64 * 16 ? 64 * 16 : kEpiThreads * kEpiNodes;
  __shared__ float tx[kEpiTileCells], ty[kEpiTileCells];  // [frame of the tile][slot]
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V;
  const int R = lattice_row_blocks(U1), W = 64 * R, FT = epi_tile_frames(R, kEpiNodes);
  const int tiles_per_utt = (T + FT - 1) / FT;
  const int tile_blocks = a.b.N * tiles_per_utt;
  if ((int)blockIdx.x >= tile_blocks) {
#pragma unroll
    for (int k = 0; k < kEpiNodes; ++k)
      lattice_fill_outside(a.pxd, a.pyd, (int)blockIdx.x - tile_blocks, threadIdx.x + k * kEpiThreads,
                           kEpiThreads * kEpiNodes, T, U1, R);
    return;
  }
  const int n = blockIdx.x / tiles_per_utt, t0 = (blockIdx.x - n * tiles_per_utt) * FT;
  const size_t L = (size_t)a.b.N * T * U1;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  const int blank = a.b.blank;
  const bool smooth = a.lm_only != 0.f || a.am_only != 0.f;
  // round 1: partial sums, row offsets and symbols of the thread's nodes
  static_assert(kEpiNodes == 1 || kEpiThreads * kEpiNodes >= 64 * 16, "a tile holds at least one frame");
  for (int c0 = 0; c0 < FT * W; c0 += kEpiThreads * kEpiNodes) {
  int tl[kEpiNodes], uu[kEpiNodes], yy[kEpiNodes];
  bool cell[kEpiNodes], node[kEpiNodes];
  size_t idx[kEpiNodes];
  float sm[kEpiNodes], ma[kEpiNodes], ml[kEpiNodes];
#pragma unroll
  for (int k = 0; k < kEpiNodes; ++k) {
    const int c = c0 + threadIdx.x + k * kEpiThreads;
    tl[k] = c / W;
    uu[k] = c - tl[k] * W;
    const int t = t0 + tl[k], u = uu[k];
    cell[k] = tl[k] < FT && u < U1 && t < T;  // FT * W may fall short of the tile's cells
    node[k] = cell[k] && t < Tn && u <= Un;
    idx[k] = cell[k] ? ((size_t)n * T + t) * U1 + u : 0;
    sm[k] = 0.f;
    ma[k] = node[k] ? a.m_a[(size_t)n * T + t] : 0.f;
    ml[k] = node[k] ? a.m_l[(size_t)n * U1 + u] : 0.f;
    bool ok = true;
    yy[k] = (node[k] && u < Un) ? symbol_at(a.b, n, u, V, ok) : 0;
  }
  for (int q0 = 0; q0 < a.nsplit; q0 += 4) {  // the split partials in order, loads of 4 per node issued together
    float pv[kEpiNodes][4];
#pragma unroll
    for (int k = 0; k < kEpiNodes; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) pv[k][j] = (node[k] && q0 + j < a.nsplit) ? a.npart[(size_t)(q0 + j) * L + idx[k]] : 0.f;
#pragma unroll
    for (int k = 0; k < kEpiNodes; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) sm[k] += pv[k][j];
  }
  // round 2: the am and lm values at blank and at the symbol
  float ab[kEpiNodes], lb[kEpiNodes], ay[kEpiNodes], ly[kEpiNodes];
#pragma unroll
  for (int k = 0; k < kEpiNodes; ++k) {
    const float* amt = a.am + ((size_t)n * T + (node[k] ? t0 + tl[k] : 0)) * V;
    const float* lmu = a.lm + ((size_t)n * U1 + (node[k] ? uu[k] : 0)) * V;
    ab[k] = node[k] ? amt[blank] : 0.f;
    lb[k] = node[k] ? lmu[blank] : 0.f;
    ay[k] = node[k] ? amt[yy[k]] : 0.f;
    ly[k] = node[k] ? lmu[yy[k]] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < kEpiNodes; ++k) {
    const int t = t0 + tl[k], u = uu[k];
    float dx = kNegInfF, dy = kNegInfF;
    if (cell[k]) {
      if (!node[k]) {
        a.Z[idx[k]] = 0.f;
        a.px[idx[k]] = kNegInfF;
        a.py[idx[k]] = kNegInfF;
      } else {
        const float s1 = (sm[k] > FLT_MIN || sm[k] != sm[k]) ? sm[k] : FLT_MIN;
        const float z = ma[k] + ml[k] + logf(s1);
        a.Z[idx[k]] = z;
        float py = ab[k] + lb[k] - z;
        float px = ay[k] + ly[k] - z;
        if (smooth) {
          // smoothed joiner: c L_trivial + a L_lm + b L_acoustic (Sec. 3.3.1)
          const float cw = 1.f - a.lm_only - a.am_only;
          const float zl = a.Zlm[(size_t)n * U1 + u];
          py = cw * py + a.lm_only * (lb[k] - zl);
          px = cw * px + a.lm_only * (ly[k] - zl);
          if (a.am_only != 0.f) {
            const float za = a.Zac[(size_t)n * T + t];
            const float* la = a.lavg + (size_t)n * V;
            py += a.am_only * (ab[k] + la[blank] - za);
            px += a.am_only * (ay[k] + la[yy[k]] - za);
          }
        }
        a.py[idx[k]] = py;
        a.px[idx[k]] = (u < Un) ? px : kNegInfF;
        dy = py;
        dx = (u < Un) ? px : kNegInfF;
      }
    }
    if (tl[k] < FT) {
      tx[tl[k] * W + u] = dx;
      ty[tl[k] * W + u] = dy;
    }
  }
  }
  __syncthreads();
  // diagonal d = t0 + k holds the tile's nodes (t0 + FT-1-j', u = d - t) for
  // the FT frames; item (k, j): u = k - (FT-1) + j, so that consecutive j are
  // consecutive u on one diagonal
  const int ft = min(FT, T - t0), nd = FT - 1 + U1;
  const size_t base = (size_t)n * (T + U1 - 1) * W;
  for (int it = threadIdx.x; it < nd * FT; it += blockDim.x) {
    const int k = it / FT, j = it - k * FT;
    const int u = k - (FT - 1) + j, tl = k - u;
    if (u < 0 || u >= U1 || tl < 0 || tl >= ft) continue;
    const size_t o = base + (size_t)(t0 + k) * W + u;
    a.pxd[o] = tx[tl * W + u];
    a.pyd[o] = ty[tl * W + u];
  }
}

// ---------------------------------------------------------------------------
// Normaliser and its epilogue in one kernel (U + 1 <= 128, V <= 1024). One workgroup
// of 8 waves per (utterance, 32 frames) holds C[t][u] for every u of its
// frames: C = sum over chunks of v of e^{am - m_a} [32 x CV] .
// e^{lm - m_l}^T [CV x U+1], both exponentials staged through two LDS
// stages: the MFMAs of chunk c read one stage, then the exponentials of
// chunk c+1 (loaded two chunks before) go to the other and chunk c+3's loads
// are issued; one barrier per chunk. Then Z, px and py of its nodes (Eqs.
// (1)-(2), (5)) go to the rectangle, and through LDS (the stages reused) to
// the diagonal-major copies, diagonal by diagonal. No split over v: no
// partial sums and no second launch. Wave w holds the C blocks of rows
// 16 (w & 1) .. +15 whose u block is (w >> 1) + 4 i. The blocks after the
// tiles fill the cells of the copies that no node of the rectangle maps to.
// ---------------------------------------------------------------------------
constexpr int kNfT = 32;         // frames per workgroup
constexpr int kNfV = 64;         // v per chunk at U + 1 <= 64 (32 above: two stages of 64 would halve the workgroups per CU)
constexpr int kNfThreads = 512;
constexpr int kNfMaxU1 = 128;
constexpr int kNfMaxV = 1024;
constexpr int kNfFill = 4;       // cells per thread of a fill block

template <int KP>
struct alignas(16) NfSmem {
  static constexpr int CV = KP > 64 ? 32 : kNfV;  // v per chunk
  static constexpr int S = CV + 4;                // row stride of a stage (conflict-free fragment reads)
  union {
    struct {
      float ea[2][kNfT * S];  // e^{am - m_a}, [stage][t][v]
      float el[2][KP * S];    // e^{lm - m_l}, [stage][u][v]
    } g;
    struct {
      float px[kNfT * KP];    // px, py of the tile's cells, [frame][slot of the lattice row]
      float py[kNfT * KP];
    } d;
  };
  float ma[kNfT], ab[kNfT], za[kNfT];  // per frame: m_a, am[t, blank], Zac
  float ml[KP], lb[KP], lyv[KP], zl[KP], lay[KP];  // per u: m_l, lm[u, blank], lm[u, y], Zlm, lavg[y]
  int yy[KP];                          // y_{u+1}
};

// One chunk's loads in registers: a thread takes float4 number tid of the
// am rows (if any) and tid + 512 i of the lm rows, the same rows in every
// chunk (their maxima stay in registers).
template <int KP>
struct NfPrefetch {
  static constexpr int Q = NfSmem<KP>::CV / 4;   // float4 per staged row
  static constexpr int AQ = kNfT * Q;            // float4 of the am rows
  static constexpr int NL = KP * Q / kNfThreads; // float4 of the lm rows per thread
  static_assert(AQ <= kNfThreads && NL * kNfThreads == KP * Q, "staging split");
  float4 x;
  float4 l[NL];
};

template <int KP, bool V4>
DEV void nf_load(Rsrc am, Rsrc lm, int t0, int v0, int Tn, int Un, int V, NfPrefetch<KP>& f) {
  using P = NfPrefetch<KP>;
  const int tid = threadIdx.x;
  {
    const int t = t0 + tid / P::Q, v = v0 + 4 * (tid % P::Q);
    const bool in = tid < P::AQ && t < Tn && v < V;
    const uint32_t o = (uint32_t)(t * V + v) * 4u;
    if (V4) {
      f.x = buf_load_f4(am, in ? o : kOob);
    } else {
      f.x.x = buf_load_f32(am, in ? o : kOob);
      f.x.y = buf_load_f32(am, in && v + 1 < V ? o + 4u : kOob);
      f.x.z = buf_load_f32(am, in && v + 2 < V ? o + 8u : kOob);
      f.x.w = buf_load_f32(am, in && v + 3 < V ? o + 12u : kOob);
    }
  }
#pragma unroll
  for (int i = 0; i < P::NL; ++i) {
    const int q = tid + i * kNfThreads, u = q / P::Q, v = v0 + 4 * (q % P::Q);
    const bool in = u <= Un && v < V;
    const uint32_t o = (uint32_t)(u * V + v) * 4u;
    if (V4) {
      f.l[i] = buf_load_f4(lm, in ? o : kOob);
    } else {
      f.l[i].x = buf_load_f32(lm, in ? o : kOob);
      f.l[i].y = buf_load_f32(lm, in && v + 1 < V ? o + 4u : kOob);
      f.l[i].z = buf_load_f32(lm, in && v + 2 < V ? o + 8u : kOob);
      f.l[i].w = buf_load_f32(lm, in && v + 3 < V ? o + 12u : kOob);
    }
  }
}

// e^{x - m} = 2^{(x - m) log2(e)} of one chunk into stage st (m per staged
// row; x - m first, so that a row's maximum gives exactly 1 and no rounding
// of m log2(e) biases a whole row). Rows past the utterance (loaded as
// zeros) only feed C entries of absent nodes, which nothing reads; the
// columns past V (the last chunk only, TAIL) are zeroed.
template <int KP, bool TAIL>
DEV void nf_store(NfSmem<KP>& sm, int st, const NfPrefetch<KP>& f, float mA, const float (&mL)[NfPrefetch<KP>::NL],
                  int v0, int V) {
  using P = NfPrefetch<KP>;
  constexpr int S = NfSmem<KP>::S;
  const int tid = threadIdx.x;
  auto ex = [&](float4 x, float m, int c) {
    const float xv[4] = {x.x, x.y, x.z, x.w};
    float e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      e[j] = __builtin_amdgcn_exp2f((xv[j] - m) * kLog2eF);
      if (TAIL && v0 + c + j >= V) e[j] = 0.f;
    }
    return make_float4(e[0], e[1], e[2], e[3]);
  };
  if (tid < P::AQ) {
    const int t = tid / P::Q, c = 4 * (tid % P::Q);
    *reinterpret_cast<float4*>(&sm.g.ea[st][t * S + c]) = ex(f.x, mA, c);
  }
#pragma unroll
  for (int i = 0; i < P::NL; ++i) {
    const int q = tid + i * kNfThreads, u = q / P::Q, c = 4 * (q % P::Q);
    *reinterpret_cast<float4*>(&sm.g.el[st][u * S + c]) = ex(f.l[i], mL[i], c);
  }
}

template <int KP>
DEV void nf_store_chunk(NfSmem<KP>& sm, int st, const NfPrefetch<KP>& f, float mA,
                        const float (&mL)[NfPrefetch<KP>::NL], int v0, int V) {
  if (v0 + NfSmem<KP>::CV <= V) nf_store<KP, false>(sm, st, f, mA, mL, v0, V);
  else nf_store<KP, true>(sm, st, f, mA, mL, v0, V);
}

template <int KP, bool V4>
__global__ __launch_bounds__(kNfThreads) void normalizer_fused_kernel(SimpleArgs a) {
  __shared__ NfSmem<KP> sm;
  using P = NfPrefetch<KP>;
  constexpr int CV = NfSmem<KP>::CV, S = NfSmem<KP>::S;
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V, blank = a.b.blank;
  const int ntt = (T + kNfT - 1) / kNfT, tiles = a.b.N * ntt;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int R = lattice_row_blocks(U1), W = 64 * R;  // W <= KP
  if ((int)blockIdx.x >= tiles) {
#pragma unroll
    for (int k = 0; k < kNfFill; ++k)
      lattice_fill_outside(a.pxd, a.pyd, (int)blockIdx.x - tiles, tid + k * kNfThreads, kNfFill * kNfThreads, T,
                           U1, R);
    return;
  }
  const int n = blockIdx.x / ntt, t0 = (blockIdx.x - n * ntt) * kNfT;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  const bool smooth = a.lm_only != 0.f || a.am_only != 0.f, acou = a.am_only != 0.f;
  const float* amn = a.am + (size_t)n * T * V;
  const float* lmn = a.lm + (size_t)n * U1 * V;
  // per-frame and per-u values of the epilogue (and the maxima of the staging)
  if (tid < kNfT) {
    const int t = t0 + tid;
    const bool node = t < Tn;
    sm.ma[tid] = node ? a.m_a[(size_t)n * T + t] : 0.f;
    sm.ab[tid] = node ? amn[(size_t)t * V + blank] : 0.f;
    sm.za[tid] = (node && acou) ? a.Zac[(size_t)n * T + t] : 0.f;
  }
  for (int u = tid; u < KP; u += kNfThreads) {
    const bool row = u <= Un;
    bool ok = true;
    const int y = (u < Un) ? symbol_at(a.b, n, u, V, ok) : 0;
    sm.yy[u] = y;
    sm.ml[u] = row ? a.m_l[(size_t)n * U1 + u] : 0.f;
    sm.lb[u] = row ? lmn[(size_t)u * V + blank] : 0.f;
    sm.lyv[u] = row ? lmn[(size_t)u * V + y] : 0.f;
    sm.zl[u] = (row && smooth) ? a.Zlm[(size_t)n * U1 + u] : 0.f;
    sm.lay[u] = (row && acou) ? a.lavg[(size_t)n * V + y] : 0.f;
  }
  __syncthreads();
  const int kn = (Un + 1 + 15) / 16 * 16;
  const int tb = wave & 1, ubw = __builtin_amdgcn_readfirstlane(wave >> 1);
  constexpr int NB = KP / 64;  // C blocks per wave: u block (w >> 1) + 4 i
  floatx4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (t0 < Tn) {
    const Rsrc amr = make_rsrc(amn, (size_t)T * V * 4), lmr = make_rsrc(lmn, (size_t)U1 * V * 4);
    const float mA = tid < P::AQ ? sm.ma[tid / P::Q] : 0.f;
    float mL[P::NL];
#pragma unroll
    for (int i = 0; i < P::NL; ++i) mL[i] = sm.ml[(tid + i * kNfThreads) / P::Q];
    const int nc = (V + CV - 1) / CV;
    // chunk c (> 0) in f[c % 2]; chunks past V load zeros (kOob): the loads
    // stay unconditional, so that each store waits only for its own chunk
    P f[2];
    nf_load<KP, V4>(amr, lmr, t0, 0, Tn, Un, V, f[0]);
    nf_store_chunk<KP>(sm, 0, f[0], mA, mL, 0, V);
    nf_load<KP, V4>(amr, lmr, t0, CV, Tn, Un, V, f[1]);
    nf_load<KP, V4>(amr, lmr, t0, 2 * CV, Tn, Un, V, f[0]);
    sg_barrier();
    auto step = [&](int c, P& fn) {
      const int st = c & 1;
      // chunk c: every fragment of the stage first, then the MFMAs of the
      // wave's u blocks that hold rows of the utterance
      floatx4 fa[CV / 16], fb[CV / 16][NB];
#pragma unroll
      for (int k = 0; k < CV / 16; ++k) {
        fa[k] = *reinterpret_cast<const floatx4*>(&sm.g.ea[st][(16 * tb + l16) * S + 16 * k + 4 * g4]);
#pragma unroll
        for (int i = 0; i < NB; ++i)
          fb[k][i] = *reinterpret_cast<const floatx4*>(&sm.g.el[st][(16 * (ubw + 4 * i) + l16) * S + 16 * k + 4 * g4]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < CV / 16; ++k)
#pragma unroll
        for (int i = 0; i < NB; ++i)
          if (16 * (ubw + 4 * i) < kn) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[k][q], fb[k][i][q], acc[i], 0, 0, 0);
          }
      // chunk c+1 into the other stage (last read by chunk c-1, before the
      // previous barrier), then chunk c+3's loads
      if (c + 1 < nc) nf_store_chunk<KP>(sm, st ^ 1, fn, mA, mL, (c + 1) * CV, V);
      nf_load<KP, V4>(amr, lmr, t0, (c + 3) * CV, Tn, Un, V, fn);
      sg_barrier();
    };
    for (int c = 0; c < nc; c += 2) {
      step(c, f[1]);
      if (c + 1 < nc) step(c + 1, f[0]);
    }
  }
  // epilogue: the target logits am[t, y_u] of the lane's nodes first (one gather round)
  const Rsrc amr = make_rsrc(amn, (size_t)T * V * 4);
  float ay[NB][4];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int u = 16 * (ubw + 4 * i) + l16;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 16 * tb + 4 * g4 + r;
      const bool node = t < Tn && u < Un;
      ay[i][r] = buf_load_f32(amr, node ? (uint32_t)(t * V + sm.yy[u]) * 4u : kOob);
    }
  }
  sg_barrier();  // every wave's MFMAs are done with the stages
  const float cw = 1.f - a.lm_only - a.am_only;
  const float* la = a.lavg + (size_t)n * V;
  const float lab = acou ? la[blank] : 0.f;
  const size_t L0 = ((size_t)n * T) * U1;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int u = 16 * (ubw + 4 * i) + l16;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int tl = 16 * tb + 4 * g4 + r, t = t0 + tl;
      const bool cell = t < T && u < U1, node = t < Tn && u <= Un;
      float z = 0.f, px = kNegInfF, py = kNegInfF;
      if (node) {
        const float sv = acc[i][r];
        const float s1 = (sv > FLT_MIN || sv != sv) ? sv : FLT_MIN;
        z = sm.ma[tl] + sm.ml[u] + logf(s1);
        py = sm.ab[tl] + sm.lb[u] - z;
        float pxv = ay[i][r] + sm.lyv[u] - z;
        if (smooth) {
          // smoothed joiner: c L_trivial + a L_lm + b L_acoustic (Sec. 3.3.1)
          py = cw * py + a.lm_only * (sm.lb[u] - sm.zl[u]) + a.am_only * (sm.ab[tl] + lab - sm.za[tl]);
          pxv = cw * pxv + a.lm_only * (sm.lyv[u] - sm.zl[u]) + a.am_only * (ay[i][r] + sm.lay[u] - sm.za[tl]);
        }
        px = (u < Un) ? pxv : kNegInfF;
      }
      if (cell) {
        const size_t idx = L0 + (size_t)t * U1 + u;
        a.Z[idx] = z;
        a.px[idx] = px;
        a.py[idx] = py;
      }
      if (u < U1) {
        sm.d.px[tl * KP + u] = px;
        sm.d.py[tl * KP + u] = py;
      }
    }
  }
  __syncthreads();
  // diagonal d = t0 + k holds the tile's nodes (t0 + tl, u = k - tl); item
  // (k, j): u = k - (kNfT - 1) + j, so that consecutive j are consecutive u
  // on one diagonal
  const int ft = min(kNfT, T - t0), nd = kNfT - 1 + U1;
  const size_t base = (size_t)n * (T + U1 - 1) * W;
  for (int it = tid; it < nd * kNfT; it += kNfThreads) {
    const int k = it / kNfT, j = it - k * kNfT;
    const int u = k - (kNfT - 1) + j, tl = k - u;
    if (u < 0 || u >= U1 || tl < 0 || tl >= ft) continue;
    const size_t o = base + (size_t)(t0 + k) * W + u;
    a.pxd[o] = sm.d.px[tl * KP + u];
    a.pyd[o] = sm.d.py[tl * KP + u];
  }
}

// ---------------------------------------------------------------------------
// d am: per utterance C[t][v] = sum_u Wt[t][u] El[u][v]  (K = U_n + 1)
// ---------------------------------------------------------------------------
using DamCfg = GemmCfg<32, 64, 32>;
constexpr int kDamSymChunk = 128;  // symbols per pass of the d am kernel's target columns

struct WtSrcKC {  // A(t, u) = Wt[t][u], rows padded to ldw (multiple of 4, zero-filled)
  using Raw = RawF<4>;
  const float* Wt;
  int t0, Tn, ldw;
  DEV void kc_load(int row, int k, Raw& r) const {
    const int t = t0 + row;
    const bool ok = t < Tn && k < ldw;
    load_plain4(Wt + (ok ? (size_t)t * ldw + k : 0), ok, r);
  }
  DEV void kc_finish(const Raw& r, float (&v)[4]) const { finish_plain4(r, v); }
};
struct ExpSrcMNC {  // B(k, col) = exp(x[k][c0+col] - mx[k]) for rows k < klim, cols < V
  using Raw = RawExp<4>;
  const float* x;  // [rows][V]
  const float* mx;
  int c0, klim, V;
  DEV void mnc_load(int k, int col, Raw& r) const { load_exp4(x, mx, k, c0 + col, V, k < klim, r); }
  DEV void mnc_finish(const Raw& r, float (&v)[4]) const { finish_exp4(r, v); }
};

template <class Cfg>
__global__ __launch_bounds__(Cfg::NT) void dam_kernel(SimpleArgs a) {
  __shared__ __align__(16) float smem[Cfg::SMEM_BYTES / sizeof(float)];
  const int n = blockIdx.z;
  const int t0 = blockIdx.x * Cfg::BM, v0 = blockIdx.y * Cfg::BN;
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  const bool active = t0 < Tn;
  floatx4 acc[Cfg::FM][Cfg::FN];
  if (active) {
    WtSrcKC sa{a.Wt + (size_t)n * T * a.ldw, t0, Tn, a.ldw};
    ExpSrcMNC sb{a.lm + (size_t)n * U1 * V, a.m_l + (size_t)n * U1, v0, Un + 1, V};
    KCLoader<Cfg, Cfg::BM, WtSrcKC> la(sa);
    MNCLoader<Cfg, Cfg::BN, ExpSrcMNC> lb(sb);
    gemm_mainloop<Cfg>(la, lb, 0, Un + 1, smem, acc);
  }
  const float* amn = a.am + (size_t)n * T * V;
  const float* ma = a.m_a + (size_t)n * T;
  const float* gxn = a.gx + (size_t)n * T * U1;
  float* out = a.am_grad + (size_t)n * T * V;
  const bool acou = a.am_only != 0.f;
  const float c = 1.f - a.lm_only - a.am_only;  // weight of the trivial joiner
  const float ks = 1.f - a.lm_only;             // weight of the target/blank terms
  // dense part: c e^{am - m_a} * acc (+ b R(t) P_ac[t,v] when smoothed)
  float res[Cfg::FM][Cfg::FN][4];
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + tile_row<Cfg>(i, r);
      const bool tv = active && t < Tn;
      const float mx = tv ? ma[t] : 0.f;
      const float bR = (tv && acou) ? a.am_only * (float)(a.rx[(size_t)n * T + t] + a.ry[(size_t)n * T + t]) : 0.f;
      const float za = (tv && acou) ? a.Zac[(size_t)n * T + t] : 0.f;
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) {
        const int v = v0 + tile_col<Cfg>(j);
        float d = 0.f;
        if (tv && v < V) {
          const float x = amn[(size_t)t * V + v];
          d = c * expf(x - mx) * acc[i][j][r];
          if (acou) d += bR * expf(x + a.lavg[(size_t)n * V + v] - za);
        }
        res[i][j][r] = d;
      }
    }
  if (active) {
    // sparse part: the target columns. Per chunk of kDamSymChunk symbols the
    // u whose symbol falls in the tile's columns are listed in ascending
    // order (ballot compaction), their gx values for the tile's frames are
    // gathered by all threads at once, and each lane subtracts them in the
    // list's order (ascending u: deterministic).
    constexpr int kChunk = kDamSymChunk;
    int* mu = reinterpret_cast<int*>(smem);  // [kChunk] listed u
    int* my = mu + kChunk;                   // [kChunk] their symbols
    constexpr int kWaves = Cfg::NT / 64;
    int* wcnt = my + kChunk;                 // [kWaves] per-wave counts
    float* g = reinterpret_cast<float*>(wcnt + kWaves);  // [kChunk][BM] gathered gx
    static_assert((2 * kChunk + kWaves) * 4 + kChunk * Cfg::BM * 4 <= Cfg::SMEM_BYTES, "sparse chunk fits");
    static_assert(Cfg::NT >= kChunk, "one thread per symbol of a chunk");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int c0 = 0; c0 < Un; c0 += kChunk) {
      __syncthreads();  // the previous user of smem is done
      const int u = c0 + threadIdx.x;
      int y = -1;
      if (threadIdx.x < kChunk && u < Un) {
        bool ok = true;
        y = symbol_at(a.b, n, u, V, ok);
      }
      const bool hit = y >= v0 && y < v0 + Cfg::BN;
      const uint64_t bal = __ballot(hit);
      if (lane == 0) wcnt[wv] = __popcll(bal);
      __syncthreads();
      int base = 0, nm = 0;
      for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
        base += (w < wv) ? wcnt[w] : 0;
        nm += wcnt[w];
      }
      if (hit) {
        const int k = base + __popcll(bal & ((1ull << lane) - 1));
        mu[k] = u;
        my[k] = y;
      }
      __syncthreads();
      for (int it = threadIdx.x; it < nm * Cfg::BM; it += blockDim.x) {
        const int k = it / Cfg::BM, tr = it - k * Cfg::BM, t = t0 + tr;
        g[it] = (t < Tn) ? gxn[(size_t)t * U1 + mu[k]] : 0.f;
      }
      __syncthreads();
      for (int k = 0; k < nm; ++k) {
        const int yk = my[k];
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j) {
          if (v0 + tile_col<Cfg>(j) != yk) continue;
#pragma unroll
          for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) res[i][j][r] -= ks * g[k * Cfg::BM + tile_row<Cfg>(i, r)];
        }
      }
    }
    const int blank = a.b.blank;
    if (blank >= v0 && blank < v0 + Cfg::BN) {
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) {
        if (v0 + tile_col<Cfg>(j) != blank) continue;
#pragma unroll
        for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int t = t0 + tile_row<Cfg>(i, r);
            if (t < Tn) res[i][j][r] = (float)((double)res[i][j][r] - (double)ks * a.ry[(size_t)n * T + t]);
          }
      }
    }
  }
  const float sc = a.scale ? a.scale[n] : 1.f;
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + tile_row<Cfg>(i, r);
      if (t >= T) continue;
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) {
        const int v = v0 + tile_col<Cfg>(j);
        if (v < V) out[(size_t)t * V + v] = (active && t < Tn) ? sc * res[i][j][r] : 0.f;
      }
    }
}

// ---------------------------------------------------------------------------
// d lm: per utterance C[u][v] = sum_t Wt[t][u] Ea[t][v]  (K = T_n)
// ---------------------------------------------------------------------------
using DlmCfg = GemmCfg<32, 64, 32>;

struct WtSrcMNC {  // A(u, t) = Wt[t][u]: global is [t][u], u-contiguous
  using Raw = RawF<4>;
  const float* Wt;
  int u0, Tn, ldw;
  DEV void mnc_load(int k, int col, Raw& r) const {
    const int u = u0 + col;
    const bool ok = k < Tn && u < ldw;
    load_plain4(Wt + (ok ? (size_t)k * ldw + u : 0), ok, r);
  }
  DEV void mnc_finish(const Raw& r, float (&v)[4]) const { finish_plain4(r, v); }
};

// Split over frames into lsplit K ranges; partial sums C[u][v] per split,
// finished by dlm_epi_kernel.
template <class Cfg>
__global__ __launch_bounds__(Cfg::NT) void dlm_kernel(SimpleArgs a) {
  __shared__ __align__(16) float smem[Cfg::SMEM_BYTES / sizeof(float)];
  const int n = blockIdx.z / a.lsplit, sk = blockIdx.z - n * a.lsplit;
  const int u0 = blockIdx.x * Cfg::BM, v0 = blockIdx.y * Cfg::BN;
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  if (u0 > Un) return;
  const int kc = split_chunk(Tn, a.lsplit, Cfg::BK);
  const int k0 = min(Tn, sk * kc), k1 = min(Tn, k0 + kc);
  floatx4 acc[Cfg::FM][Cfg::FN];
  WtSrcMNC sa{a.Wt + (size_t)n * T * a.ldw, u0, Tn, a.ldw};
  ExpSrcMNC sb{a.am + (size_t)n * T * V, a.m_a + (size_t)n * T, v0, Tn, V};
  MNCLoader<Cfg, Cfg::BM, WtSrcMNC> la(sa);
  MNCLoader<Cfg, Cfg::BN, ExpSrcMNC, decltype(la)::NBLK> lb(sb);  // threads after A's blocks
  gemm_mainloop<Cfg>(la, lb, k0, k1, smem, acc);
  float* part = a.lpart + ((size_t)sk * a.b.N + n) * U1 * V;
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = u0 + tile_row<Cfg>(i, r);
      if (u > Un) continue;
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) {
        const int v = v0 + tile_col<Cfg>(j);
        if (v < V) part[(size_t)u * V + v] = acc[i][j][r];
      }
    }
}

// d lm[u,v] = sc (e^{lm - m_l} sum_splits C - [v = y_{u+1}] sum_t gx - [v = blank] sum_t gy);
// one thread per 4 consecutive v of a row.
__global__ __launch_bounds__(256) void dlm_epi_kernel(SimpleArgs a) {
  const int U1 = a.b.U + 1, V = a.V;
  const int nvg = (V + 3) / 4;
  const size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (size_t)a.b.N * U1 * nvg) return;
  const int row = (int)(g / nvg);  // n * U1 + u
  const int v0 = (int)(g - (size_t)row * nvg) * 4;
  const int n = row / U1, u = row - n * U1;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  float* out = a.lm_grad + (size_t)row * V;
  if (u > Un) {
    for (int v = v0; v < min(V, v0 + 4); ++v) out[v] = 0.f;
    return;
  }
  const float sc = a.scale ? a.scale[n] : 1.f;
  const int blank = a.b.blank;
  bool ok = true;
  const int y = (u < Un) ? symbol_at(a.b, n, u, V, ok) : -1;
  const float ml = a.m_l[row];
  const float* lmr = a.lm + (size_t)row * V;
  const size_t stride = (size_t)a.b.N * U1 * V;
  const size_t base = (size_t)row * V;
  const bool smooth = a.lm_only != 0.f || a.am_only != 0.f;
  const float cw = 1.f - a.lm_only - a.am_only;  // weight of the trivial joiner
  const double ks = 1.0 - (double)a.am_only;      // weight of the target/blank terms
  // the target and blank columns collect Gx(u) = sum_t gx(t,u) and Gy(u) (fp64)
  const double gx = a.Gx[row], gy = a.Gy[row];
  const float zl = smooth ? a.Zlm[row] : 0.f;
  const float aG = smooth ? a.lm_only * (float)(gx + gy) : 0.f;
  const float su = a.am_only != 0.f ? a.su[row] : 0.f;
  for (int v = v0; v < min(V, v0 + 4); ++v) {
    float c = 0.f;
    for (int q = 0; q < a.lsplit; ++q) c += a.lpart[(size_t)q * stride + base + v];
    float d = cw * expf(lmr[v] - ml) * c;
    if (smooth) {
      const float p = expf(lmr[v] - zl);
      d += aG * p;
      if (a.am_only != 0.f) d += a.am_only * p * (a.q[(size_t)n * V + v] - su);
    }
    double gd = (double)d;
    if (v == y) gd -= ks * gx;
    if (v == blank) gd -= ks * gy;
    out[v] = (float)(sc * gd);
  }
}

// ---------------------------------------------------------------------------
// d am and d lm in one pass (U + 1 <= 320).
//
// One workgroup per (utterance, 64 columns of v, range of frames): one or two
// groups (sg_groups) of eight waves that take the range's steps of 32 frames in
// turn.
// Wave w of a group holds the 16 columns of block w >> 1, and of a step computes
//   d am [16 x 16] = W [16 x U+1] . e^{lm - m_l} [U+1 x 16], the frames whose
//     bit 2 is w & 1, finished at once (times e^{am - m_a}, minus the target
//     and blank terms) and stored;
//   d lm [u blocks of parity w & 1 x 16] += W^T [. x 32] . e^{am - m_a}
//     [32 x 16], kept in registers, added over the groups at the end and
//     finished (a single range) or stored as the range's partial sums for
//     dlm_epi_kernel.
// Both contractions run on three bf16 planes per operand. W's planes go
// through LDS: rows for d am, the same rows read transposed
// (ds_read_b64_tr_b16) for d lm. e^{lm - m_l} is formed once, into LDS at
// U + 1 <= 128 and above into the fragments that a wave keeps (whose registers
// then allow two waves a SIMD), and e^{am - m_a} by the lanes that use it, as
// d lm's fragment (column l16, frames 8 g4 .. + 7), whose frames
// 8 g4 + 4 (w & 1) .. + 3 are also those of the lane's d am results: d am's
// tile takes its rows in that order. A step's loads are in flight during the
// step before; W's planes have two stages a group, one barrier a step, but one
// stage and two barriers for one group at 64 < U + 1 <= 128, where two
// workgroups then fit a CU's LDS.
// (The step is bound by its waves' chains: fragment reads, exponentials and
// splits, MFMAs. Against fp32 MFMA with both operands in LDS, us with the column
// sums: N = 32, T = 500, U = 100, V = 500 46 for 66; N = 6, T = 287, U = 77,
// V = 4999 46 for 51; N = 16, T = 300, U = 80, V = 5000 96 for 120; N = 32,
// T = 100, U = 30, V = 8000 93 for 101; U = 300, V = 8000, N = 8, T = 1000 1,030
// for 1,360; but N = 8, T = 500, U = 100, V = 8000 156 for 143. Smoothed, N = 13,
// T = 333, U = 71, V = 1031: 44 for 180 with the two kernels it replaces and the
// acoustic statistics that they always formed.)
// ---------------------------------------------------------------------------
constexpr int kSgT = 32;        // frames per step
constexpr int kSgMaxU1 = 320;   // the fused kernel takes U + 1 up to this
constexpr int kSgV = 64;        // columns per workgroup
constexpr int kSgThreads = 512; // of a group
constexpr int kSgList = 24;     // listed targets whose gx one gather round stages (at KP = 128 the LDS is full)

template <int KP, int GRP_>  // u extent staged: U + 1 <= KP (a multiple of 64); groups of eight waves
struct alignas(16) SgSmem {
  static constexpr int ROWB = KP * 2;         // bytes per row of a plane
  static constexpr int PLANE = kSgT * ROWB;
  static constexpr int GRP = GRP_, WAVES = GRP * kSgThreads / 64;
  struct Stage {
    unsigned char w[3 * PLANE];     // planes of W(t, u) of the step's frames, [t][u] (zero past ldw)
    float g[kSgList * kSgT];        // gx(t, u_k) of listed targets, [k][t]
    double ry[kSgT];                // row sums of gy
    float ma[kSgT];                 // m_a, +inf past T_n (zero exponentials)
    float br[kSgT], za[kSgT];       // smoothed: weight and lse of the acoustic joiner
  };
  static constexpr int NST = GRP == 1 && KP == 128 ? 1 : 2;  // two workgroups' LDS on a CU
  Stage st[GRP][NST];
  static constexpr bool EL = KP <= 128;  // e^{lm - m_l} staged here, not in registers
  static constexpr int EPLANE = kSgV * ROWB;
  unsigned char el[EL ? 3 * EPLANE : 16];
  uint16_t lu[KP];                  // targets in the columns (ascending u)
  int sym[KP];                      // y_{u+1}
  float ml[KP];                     // m_l, +inf past U_n
  int cnt[WAVES];
  // Byte position of 16-byte chunk c of row r: swizzled by the row, so that
  // neither the rows 8i + j (i, j < 4) of a d am fragment nor the 32 bytes of
  // the rows 8i + j (i < 2, j < 4) of a transposed read share banks.
  // The swizzle stays within G groups of four chunks.
  static constexpr int G = KP % 128 == 0 ? 4 : 2;
  static DEV int pos(int r, int c) {
    const int key = G == 4 ? ((r & 3) << 1) | (r & 8) | ((r >> 4) & 1) : (r & 2) | ((r & 8) >> 1) | ((r >> 4) & 1);
    return r * ROWB + ((c ^ key) << 4);
  }
};

// The utterance's arrays as buffer resources of its T_n frames: rows past them
// read zeros and every load is issued unconditionally, so that the step's code
// is straight-line and the wait counts stay exact. A lane whose columns lie
// past V computes on what it reads there and stores nothing.
struct SgSrc {
  Rsrc wt, am, ma, gx, rx, ry, za;
  int ldw, V, U1, Tn;
  float am_only;
};

template <int KP>
struct SgPrefetch {  // one step's global loads, held until the step's LDS writes
  static constexpr int NW = (kSgT * KP / 8 + kSgThreads - 1) / kSgThreads;
  float4 w[NW][2];  // 8 values of W each
  static constexpr int NG = (kSgT * kSgList + kSgThreads - 1) / kSgThreads;
  float gx[NG];
  float ma, za;
  double rx, ry;
};

template <int KP, bool SM>
DEV void sg_load(const SgSrc& c, int t0, const uint16_t* lu, SgPrefetch<KP>& f) {
  const int tid = threadIdx.x % kSgThreads;
#pragma unroll
  for (int i = 0; i < SgPrefetch<KP>::NW; ++i) {
    const int q = tid + i * kSgThreads, r = q / (KP / 8), u = q % (KP / 8) * 8;
    const uint32_t o = (uint32_t)((t0 + r) * c.ldw + u) * 4u;
    f.w[i][0] = buf_load_f4(c.wt, r < kSgT && u < c.ldw ? o : kOob);
    f.w[i][1] = buf_load_f4(c.wt, r < kSgT && u + 4 < c.ldw ? o + 16u : kOob);
  }
#pragma unroll
  for (int i = 0; i < SgPrefetch<KP>::NG; ++i) {
    const int q = tid + i * kSgThreads, k = q / kSgT, t = t0 + q % kSgT;
    f.gx[i] = buf_load_f32(c.gx, (uint32_t)(t * c.U1 + lu[k]) * 4u);
  }
  const uint32_t t = (uint32_t)(t0 + tid);
  f.ma = buf_load_f32(c.ma, t * 4u);
  f.ry = buf_load_f64(c.ry, t * 8u);
  if constexpr (SM) {
    f.rx = buf_load_f64(c.rx, t * 8u);
    f.za = buf_load_f32(c.za, t * 4u);
  }
}

template <int KP, bool SM, int GRP>
DEV void sg_store(const SgSrc& c, typename SgSmem<KP, GRP>::Stage& st, const SgPrefetch<KP>& f, int t0) {
  using Smem = SgSmem<KP, GRP>;
  const int tid = threadIdx.x % kSgThreads;
#pragma unroll
  for (int i = 0; i < SgPrefetch<KP>::NW; ++i) {
    const int q = tid + i * kSgThreads, r = q / (KP / 8);
    const float x[8] = {f.w[i][0].x, f.w[i][0].y, f.w[i][0].z, f.w[i][0].w,
                        f.w[i][1].x, f.w[i][1].y, f.w[i][1].z, f.w[i][1].w};
    uint4 p0, p1, p2;
    split3(x, p0, p1, p2);
    if (r < kSgT) {
      unsigned char* d = st.w + Smem::pos(r, q % (KP / 8));
      *reinterpret_cast<uint4*>(d) = p0;
      *reinterpret_cast<uint4*>(d + Smem::PLANE) = p1;
      *reinterpret_cast<uint4*>(d + 2 * Smem::PLANE) = p2;
    }
  }
#pragma unroll
  for (int i = 0; i < SgPrefetch<KP>::NG; ++i)
    if (tid + i * kSgThreads < kSgT * kSgList) st.g[tid + i * kSgThreads] = f.gx[i];
  if (tid < kSgT) {
    st.ry[tid] = f.ry;
    st.ma[tid] = t0 + tid < c.Tn ? f.ma : INFINITY;
    if constexpr (SM) {
      st.br[tid] = c.am_only * (float)(f.rx + f.ry);
      st.za[tid] = f.za;
    }
  }
}

// rows r .. r + 7 of column v of am or lm
DEV void sg_load8(Rsrc m, int V, int r, int v, float (&x)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = buf_load_f32(m, (uint32_t)((r + j) * V + v) * 4u);
}

DEV void sg_planes(const float (&x)[8], bf16x8 (&f)[3]) {
  uint4 p0, p1, p2;
  split3(x, p0, p1, p2);
  f[0] = __builtin_bit_cast(bf16x8, p0);
  f[1] = __builtin_bit_cast(bf16x8, p1);
  f[2] = __builtin_bit_cast(bf16x8, p2);
}

template <int KP, bool SM, int GRP>  // SM: smoothed
__global__ __launch_bounds__(kSgThreads * GRP, KP <= 128 ? 4 : 1) void simple_grad_kernel(SimpleArgs a, int splits, int items) {
  using Smem = SgSmem<KP, GRP>;
  constexpr int NS = KP / 32, NUB = KP / 32, NT = GRP * kSgThreads;
  __shared__ Smem sm;
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V, blank = a.b.blank;
  // an eighth of the items, in order, to each XCD: the column tiles of a frame
  // range read the same rows of W from its L2
  const int nvt = (V + kSgV - 1) / kSgV;
  const int it = (blockIdx.x & 7) * (gridDim.x / 8) + (blockIdx.x >> 3);
  if (it >= items) return;
  const int v0 = it % nvt * kSgV, rest = it / nvt, sk = rest % splits, n = rest / splits;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform: the block guards below are scalar)
  const int grp = wave / (kSgThreads / 64), h = wave & 1;
  const int vw0 = v0 + ((wave >> 1) & 3) * 16, vw = vw0 + l16;  // the wave's and the lane's columns
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  const int kn = Un + 1;  // contraction length of d am, rows of d lm
  const float sc = a.scale ? a.scale[n] : 1.f;
  const bool acou = SM && a.am_only != 0.f;
  const float cw = SM ? 1.f - a.lm_only - a.am_only : 1.f;  // weight of the trivial joiner
  const float ks = SM ? 1.f - a.lm_only : 1.f;              // weight of d am's target and blank terms
  for (int u = tid; u < KP; u += NT) {
    bool ok = true;
    sm.sym[u] = (u < Un) ? symbol_at(a.b, n, u, V, ok) : -1;
    sm.ml[u] = (u <= Un) ? a.m_l[(size_t)n * U1 + u] : INFINITY;
    sm.lu[u] = 0;
  }
  __syncthreads();
  // e^{lm - m_l} of the lane's columns, in d am's fragments (rows 32 s + 8 g4 .. + 7)
  // (LDS: column 16 b + l at the row of the bits l3 l2 b0 l1 l0 and b1, where the
  // 16 columns of a fragment lie like the rows of a d am fragment of W)
  const Rsrc lmn = make_rsrc(a.lm + (size_t)n * U1 * V, (size_t)(Un + 1) * V * 4);
  bf16x8 el[Smem::EL ? 1 : NS][3];
  const int vb = (wave >> 1) & 3;
  const int erow = (l16 & 3) | ((l16 >> 2) << 3) | ((vb & 1) << 2) | ((vb >> 1) << 5);
  if constexpr (Smem::EL) {
#pragma unroll
    for (int b = wave & 3, c = (wave >> 2) * 4 + g4; c < KP / 8; c += NT / 64) {
      float e[8];
      sg_load8(lmn, V, 8 * c, v0 + 16 * b + l16, e);
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = __expf(e[j] - sm.ml[8 * c + j]);
      bf16x8 f[3];
      sg_planes(e, f);
      unsigned char* d = sm.el + Smem::pos((l16 & 3) | ((l16 >> 2) << 3) | ((b & 1) << 2) | ((b >> 1) << 5), c);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8*>(d + p * Smem::EPLANE) = f[p];
    }
  } else {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float e[8];
      sg_load8(lmn, V, 32 * s + 8 * g4, vw, e);
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = __expf(e[j] - sm.ml[32 * s + 8 * g4 + j]);
      sg_planes(e, el[s]);
    }
  }
  const float lavg = acou && vw < V ? a.lavg[(size_t)n * V + vw] : 0.f;
  // the targets that fall in the columns, ascending u (ballot compaction)
  {
    const int y = (tid < Un) ? sm.sym[tid] : -1;  // U_n < KP <= kSgThreads
    const bool hit = y >= v0 && y < v0 + kSgV;
    const uint64_t bal = __ballot(hit);
    if (lane == 0) sm.cnt[wave] = __popcll(bal);
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += sm.cnt[w];
    if (hit) {
      const int k = base + __popcll(bal & ((1ull << lane) - 1));
      sm.lu[k] = (uint16_t)tid;
    }
    __syncthreads();
  }
  int nm = 0;
#pragma unroll
  for (int w = 0; w < Smem::WAVES; ++w) nm += sm.cnt[w];
  // of a round of listed targets, those in the wave's columns (lane k holds target k)
  auto round_mask = [&](int k0, int& y) {
    y = lane < kSgList && k0 + lane < nm ? sm.sym[sm.lu[k0 + lane]] : -1;
    return (uint32_t)__ballot(y >= vw0 && y < vw0 + 16);
  };
  int ly0;
  const uint32_t mask0 = round_mask(0, ly0);
  // the range's steps, and its end: frames past it read and add zeros
  const int nlive = (Tn + kSgT - 1) / kSgT;
  const int s0 = sk * nlive / splits, s1 = (sk + 1) * nlive / splits, Te = min(Tn, s1 * kSgT);
  SgSrc src;
  src.wt = make_rsrc(a.Wt + (size_t)n * T * a.ldw, (size_t)Te * a.ldw * 4);
  src.am = make_rsrc(a.am + (size_t)n * T * V, (size_t)Te * V * 4);
  src.ma = make_rsrc(a.m_a + (size_t)n * T, (size_t)Te * 4);
  src.gx = make_rsrc(a.gx + (size_t)n * T * U1, (size_t)Te * U1 * 4);
  src.ry = make_rsrc(a.ry + (size_t)n * T, (size_t)Te * 8);
  if (SM) {
    src.rx = make_rsrc(a.rx + (size_t)n * T, (size_t)Te * 8);
    src.za = make_rsrc(a.Zac + (size_t)n * T, acou ? (size_t)Te * 4 : 0);
  }
  src.ldw = a.ldw;
  src.V = V;
  src.U1 = U1;
  src.Tn = Te;
  src.am_only = a.am_only;
  const Rsrc gout = make_rsrc(a.am_grad + (size_t)n * T * V, (size_t)T * V * 4);
  const uint32_t ov = vw < V ? (uint32_t)vw * 4u : kOob;  // the lane's column in a row of d am
  if (sk + 1 == splits)  // frames past T_n
    for (int t = Tn + (lane >> 4) + 4 * (wave & 1) + 8 * grp; t < T; t += 8 * GRP)
      __builtin_amdgcn_raw_buffer_store_b32(0u, gout, (int)((uint32_t)(t * V) * 4u + ov), 0, 0);
  floatx4 accl[NUB];
#pragma unroll
  for (int i = 0; i < NUB; ++i) accl[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  SgPrefetch<KP> f;
  float x[8];
  if (s0 < s1) {
    const int t0 = (s0 + grp) * kSgT;
    sg_load8(src.am, V, t0 + 8 * g4, vw, x);
    sg_load<KP, SM>(src, t0, sm.lu, f);
    sg_store<KP, SM, GRP>(src, sm.st[grp][0], f, t0);
    // (x is waited for here: otherwise the loop's first use of it also waits, each
    // step, for the stores of the step before)
#pragma unroll
    for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(x[j]));
  }
  // the lane's parts of the fragment addresses: d am rows, transposed rows
  // (chunk 4 q + c of a row lies at the position of chunk c, its bits 6 and up
  // XORed with q: the swizzle and the rows leave them alone)
  int pd = Smem::pos(8 * (l16 >> 2) + 4 * h + (l16 & 3), g4), pe = Smem::pos(erow, g4);
  int pt = Smem::pos(8 * g4 + (l16 >> 2), 2 * h + ((l16 & 3) >> 1)) + (l16 & 1) * 8;
  for (int st = s0; st < s1; st += GRP) {
    const int t0 = (st + grp) * kSgT, tn = t0 + GRP * kSgT;
    typename Smem::Stage& cur = sm.st[grp][((st - s0) / GRP) & (Smem::NST - 1)];
    typename Smem::Stage& nxt = sm.st[grp][((st - s0) / GRP + 1) & (Smem::NST - 1)];
    sg_barrier();  // the step's stage is written, the other one's reads are done
    floatx4 accd = floatx4{0.f, 0.f, 0.f, 0.f};
    float ed[4], xd[4];  // e^{am - m_a} and am of the lane's d am results
    asm volatile("" : "+v"(pd), "+v"(pt), "+v"(pe));  // (the XORs are cheaper than the registers of their results)
    bf16x8 ea[3];
    {
      const floatx4 m0 = *reinterpret_cast<const floatx4*>(&cur.ma[8 * g4]);
      const floatx4 m1 = *reinterpret_cast<const floatx4*>(&cur.ma[8 * g4 + 4]);
      float e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = __expf(x[j] - (j < 4 ? m0[j & 3] : m1[j & 3]));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e0 = e[r], e1 = e[4 + r], x0 = x[r], x1 = x[4 + r];
        ed[r] = h ? e1 : e0;
        if (SM) xd[r] = h ? x1 : x0;
      }
      sg_planes(e, ea);
    }
    // the next step's loads, in flight during this step's MFMAs and stores
    sg_load8(src.am, V, tn + 8 * g4, vw, x);
    sg_load<KP, SM>(src, tn, sm.lu, f);
    // a slice of d am and a block of d lm at a time: two chains of MFMAs in flight
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (32 * s < kn) {
        bf16x8 fd[3], fl[3], fe[3];
        const int o = s / Smem::G * (64 * Smem::G), q = s % Smem::G << 6;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const unsigned char* wt = cur.w + (pt ^ q) + o + p * Smem::PLANE;
          fd[p] = *reinterpret_cast<const bf16x8*>(cur.w + (pd ^ q) + o + p * Smem::PLANE);
          fl[p] = tr_frag2<bf16x8>(wt, wt + 4 * Smem::ROWB);  // (rows 4 apart share their swizzle)
          if constexpr (Smem::EL) fe[p] = *reinterpret_cast<const bf16x8*>(sm.el + (pe ^ q) + o + p * Smem::EPLANE);
        }
        if constexpr (Smem::EL) mfma_split3_pair(fd, fe, accd, fl, ea, accl[s]);
        else mfma_split3_pair(fd, el[s], accd, fl, ea, accl[s]);
      }
    // d am epilogue: e^{am - m_a} * acc (+ the acoustic joiner's part), minus gx
    // at the targets (ascending u) and the blank column's row sum of gy
    const int tl = 8 * g4 + 4 * h;
    float res[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (SM) {
        res[r] = cw * ed[r] * accd[r];
        if (acou) res[r] += cur.br[tl + r] * expf(xd[r] + lavg - cur.za[tl + r]);
      } else {
        res[r] = ed[r] * accd[r];
      }
    }
    for (int k0 = 0; k0 < nm; k0 += kSgList) {
      int ly = ly0;
      uint32_t bits = mask0;
      if (k0 > 0) {  // more targets than one gather round holds: the next ones, synchronously
        sg_barrier();
        for (int q = tid % kSgThreads; q < kSgT * kSgList; q += kSgThreads) {
          const int k = k0 + q / kSgT, t = t0 + q % kSgT;
          cur.g[q] = (k < nm && t < Te) ? a.gx[((size_t)n * T + t) * U1 + sm.lu[k]] : 0.f;
        }
        sg_barrier();
        bits = round_mask(k0, ly);
      }
      while (bits) {  // ascending u
        const int k = __builtin_ctz(bits), y = __builtin_amdgcn_readlane(ly, k);
        bits &= bits - 1;
        const floatx4 gk = *reinterpret_cast<const floatx4*>(&cur.g[k * kSgT + tl]);
#pragma unroll
        for (int r = 0; r < 4; ++r) res[r] -= vw == y ? ks * gk[r] : 0.f;
      }
    }
    if (vw == blank) {
#pragma unroll
      for (int r = 0; r < 4; ++r) res[r] = (float)((double)res[r] - (double)ks * cur.ry[tl + r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sc * res[r]), gout,
                                            (int)(t0 + tl + r < Te ? (uint32_t)((t0 + tl + r) * V) * 4u + ov : kOob), 0, 0);
    if constexpr (Smem::NST == 1) sg_barrier();  // every read of the stage is done
    sg_store<KP, SM, GRP>(src, nxt, f, tn);
  }
  // the groups' d lm sums: group g finishes the blocks i of parity g (all of
  // them where there is one group), the other's come through LDS
  if constexpr (GRP == 2) {
    static_assert(sizeof(sm.st) >= 2 * kSgThreads * (NUB / 2) * sizeof(floatx4), "one group's blocks");
    floatx4* ex = reinterpret_cast<floatx4*>(sm.st);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NUB; ++i)
      if (i % 2 != grp) ex[(i / 2) * NT + tid] = accl[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NUB; ++i)
      if (i % 2 == grp) {
        const floatx4 o = ex[(i / 2) * NT + (tid ^ kSgThreads)];
        accl[i] = grp == 0 ? accl[i] + o : o + accl[i];
      }
  }
  if (vw >= V) return;
#pragma unroll
  for (int i = 0; i < NUB; ++i) {
    if (GRP == 2 && i % 2 != grp) continue;
    const int u0 = 16 * (h + 2 * i) + 4 * g4;
    float e[4];
    if (splits == 1 && !SM) {
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __expf(buf_load_f32(lmn, (uint32_t)((u0 + r) * V + vw) * 4u) - sm.ml[u0 + r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = u0 + r;
      if (u >= U1) continue;
      if (splits > 1 || SM) {
        if (u <= Un) a.lpart[(((size_t)sk * a.b.N + n) * U1 + u) * V + vw] = accl[i][r];
        continue;
      }
      float out = 0.f;
      if (u <= Un) {
        double gd = (double)(e[r] * accl[i][r]);
        if (vw == sm.sym[u]) gd -= a.Gx[(size_t)n * U1 + u];
        if (vw == blank) gd -= a.Gy[(size_t)n * U1 + u];
        out = (float)(sc * gd);
      }
      a.lm_grad[((size_t)n * U1 + u) * V + vw] = out;
    }
  }
}

__global__ void fill_f32_kernel(float* p, size_t n, float v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

}  // namespace

hipError_t launch_rowmax(const SimpleArgs& a, hipStream_t s) {
  const int N = a.b.N, T = a.b.T, U1 = a.b.U + 1;
  {
    RNNT_PROF(s, "rowmax");
    hipLaunchKernelGGL(rowmax_kernel, dim3((N * (T + U1) + 3) / 4), dim3(256), 0, s, a.am, a.lm, N, T, U1, a.V, a.b,
                       a.m_a, a.m_l);
  }
  return hipGetLastError();
}

// Split counts: enough K ranges for about 1024 workgroups, each range at
// least two K-steps long.
static int split_count(long long tiles, int K, int bk) {
  long long sk = (1024 + tiles - 1) / tiles;
  const long long most = (K + 2 * bk - 1) / (2 * bk);
  if (sk > most) sk = most;
  if (sk > 16) sk = 16;
  return sk < 1 ? 1 : (int)sk;
}

// Whether the fused normaliser takes the call (see launch_normalizer; its
// offsets within an utterance's am and lm are 32-bit).
static bool normalizer_fused(int T, int U, int V) {
  return U + 1 <= kNfMaxU1 && V <= kNfMaxV && (long long)T * V * 4 < (1ll << 31) && (long long)(U + 1) * V * 4 < (1ll << 31);
}

// K ranges of the split normaliser (0 where the fused one runs, without partial sums): those of the least estimated time. The
// chip holds 512 workgroups at a time, two on a CU, whose steps then take
// about 1.75 us each (1.25 us alone on a CU), and every range's partial sums
// are written and read once (about 5 TB/s); a range is at least four steps.
int normalizer_splits(int N, int T, int U, int V) {
  if (normalizer_fused(T, U, V)) return 0;
  const int bn = ns_cols(U + 1);
  const double tiles = (double)N * ((T + kNsT - 1) / kNsT) * ((U + 1 + bn - 1) / bn);
  const int steps = (V + kNsV - 1) / kNsV;
  int best = 1;
  double least = 0.0;
  for (int sk = 1; sk <= 32 && (sk == 1 || sk * 4 <= steps); ++sk) {
    const double wgs = tiles * sk;
    const double us = std::ceil(wgs / 512) * ((steps + sk - 1) / sk) * (wgs > 256 ? 1.75 : 1.25) +
                      sk * (double)N * T * (U + 1) * 8 / 5e6;
    if (sk == 1 || us < least) {
      best = sk;
      least = us;
    }
  }
  return best;
}

template <class Cfg>
static int dlm_splits_cfg(int N, int T, int U, int V) {
  const long long tiles = (long long)N * ((U + 1 + Cfg::BM - 1) / Cfg::BM) * ((V + Cfg::BN - 1) / Cfg::BN);
  return split_count(tiles, T, Cfg::BK);
}
int dlm_splits(int N, int T, int U, int V) {
  return V >= kSimpleBigV ? dlm_splits_cfg<BigCfg>(N, T, U, V) : dlm_splits_cfg<DlmCfg>(N, T, U, V);
}

// Frame ranges of the one-pass d am / d lm kernel: enough for about
// kSgBlocks groups of eight waves, one per CU; 0 where the kernel does not
// apply. Of two groups a workgroup halves the ranges, and with them the partial
// sums: where one range is left, dlm_epi_kernel falls away (N = 16, T = 250,
// U = 60, V = 500: the step 314 -> 306 us; smoothed, N = 13, T = 333, U = 71,
// V = 1031: 521 -> 511 us).
constexpr int kSgBlocks = 256;

// Groups of a workgroup for U + 1 <= 128. Two share e^{lm - m_l} and halve an
// item's steps, but fill a CU; of one, two workgroups share a CU, so that one
// works while the other starts or ends. Where one group a workgroup would leave
// half of the chip's waves empty (up to 256 items), two win: N = 32, T = 500,
// U = 100, V = 500 46 us with the column sums against 60, N = 2, T = 300, U = 80,
// V = 5000 30 against 38. Beyond, one wins at U + 1 <= 64 (N = 8, T = 300,
// U = 50, V = 5000, 632 items: 56 against 64; N = 32, T = 100, U = 30, V = 8000,
// 4,000 items: 93 against 157). At 64 < U + 1 <= 128, with one stage of W, an
// item of two takes about 0.6 of the time of one, and the chip takes 256 or 512
// items at a time: one wins unless it leaves its last round half empty (N = 6,
// T = 287, U = 77, V = 4999, 474 items: 46 against 53; N = 16, T = 300, U = 80,
// V = 5000, 1,264 items: 97 against 112; but N = 24, T = 400, U = 90, V = 2000,
// 768 items: 89 against 85).
static int sg_groups(int N, int U, int V) {
  if (U + 1 > 128) return 1;
  const long long items = (long long)N * ((V + kSgV - 1) / kSgV);
  if (U + 1 <= 64) return items > 256 ? 1 : 2;
  return 5 * ((items + 511) / 512) <= 3 * ((items + 255) / 256) ? 1 : 2;
}
int simple_grad_splits(int N, int T, int U, int V) {
  // one utterance's am and lm must stay below 2^31 bytes, the rows that a tile reaches past them included (32-bit offsets)
  if (U + 1 > kSgMaxU1 || (long long)(T + kSgMaxU1) * V * 4 >= (1ll << 31)) return 0;
  const long long base = (long long)N * ((V + kSgV - 1) / kSgV);
  const int steps = (T + kSgT - 1) / kSgT;
  const int want = kSgBlocks / sg_groups(N, U, V);
  long long s = (want + base - 1) / base;
  if (s > steps) s = steps;
  return s < 1 ? 1 : (int)s;
}

template <int KP>
static void launch_normalizer_fused(const SimpleArgs& a, bool v4, unsigned blocks, hipStream_t s) {
  if (v4) hipLaunchKernelGGL((normalizer_fused_kernel<KP, true>), dim3(blocks), dim3(kNfThreads), 0, s, a);
  else hipLaunchKernelGGL((normalizer_fused_kernel<KP, false>), dim3(blocks), dim3(kNfThreads), 0, s, a);
}

hipError_t launch_normalizer(const SimpleArgs& a, hipStream_t s) {
  const int T = a.b.T, U1 = a.b.U + 1;
  if (normalizer_fused(T, a.b.U, a.V)) {
    // every u of 32 frames per workgroup, the epilogue in the same kernel: the
    // faster one where V is short, so that the epilogue's gathers weigh as much
    // as the contraction (N = 32, T = 500, U = 100, V = 500: 36 us against 22 +
    // 26 of the split kernels, N = 16, T = 250, U = 60: 14.6 against 10 + 7). Its
    // 32-frame tiles form the exponentials of every lm row anew, and run the
    // whole of V in sequence: at V = 2000 (N = 24, T = 400, U = 90) it took 87 us
    // against 76, with V = 2047 (unaligned rows) 139 against 76, at V = 8000
    // (N = 8, T = 1000, U = 300) 530 against 360.
    const size_t blocks = (size_t)a.b.N * ((T + kNfT - 1) / kNfT) +
                          (size_t)a.b.N * lattice_fill_blocks(T, a.b.U, kNfFill * kNfThreads);
    const bool v4 = (a.V & 3) == 0;
    RNNT_PROF(s, "normalizer");
    if (U1 <= 64) launch_normalizer_fused<64>(a, v4, (unsigned)blocks, s);
    else launch_normalizer_fused<kNfMaxU1>(a, v4, (unsigned)blocks, s);
    return hipGetLastError();
  }
  {
    RNNT_PROF(s, "normalizer");
    const int bn = ns_cols(U1), ntt = (T + kNsT - 1) / kNsT, ntu = (U1 + bn - 1) / bn;
    const dim3 grid((unsigned)((size_t)a.b.N * a.nsplit * ntt * ntu));
    if (bn == 64) hipLaunchKernelGGL(normalizer_kernel<64>, grid, dim3(kNsThreads), 0, s, a, ntt, ntu);
    else if (bn == 96) hipLaunchKernelGGL(normalizer_kernel<96>, grid, dim3(kNsThreads), 0, s, a, ntt, ntu);
    else hipLaunchKernelGGL(normalizer_kernel<128>, grid, dim3(kNsThreads), 0, s, a, ntt, ntu);
  }
  // tiles of the rectangle's nodes, then the cells of the diagonal-major copies
  const int nodes = epi_nodes(a.b.N, T, U1);
  const int FT = epi_tile_frames(lattice_row_blocks(U1), nodes);
  const size_t blocks =
      (size_t)a.b.N * ((T + FT - 1) / FT) + (size_t)a.b.N * lattice_fill_blocks(T, a.b.U, kEpiThreads * nodes);
  {
    RNNT_PROF(s, "normalizer_epi");
    if (nodes == 4) hipLaunchKernelGGL(normalizer_epi_kernel<4>, dim3((unsigned)blocks), dim3(kEpiThreads), 0, s, a);
    else hipLaunchKernelGGL(normalizer_epi_kernel<1>, dim3((unsigned)blocks), dim3(kEpiThreads), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_smoothing_stats(const SimpleArgs& a, hipStream_t s) {
  if (a.lm_only == 0.f && a.am_only == 0.f) return hipSuccess;
  const int N = a.b.N, T = a.b.T, U1 = a.b.U + 1;
  {
    RNNT_PROF(s, "smooth_stats");
    hipLaunchKernelGGL(lm_lse_kernel, dim3((N * U1 + 3) / 4), dim3(256), 0, s, a);
    // the acoustic joiner's statistics only where it has a weight
    if (a.am_only != 0.f) {
      hipLaunchKernelGGL(lm_avg_kernel, dim3((a.V + 255) / 256, N), dim3(256), 0, s, a);
      hipLaunchKernelGGL(ac_lse_kernel, dim3((N * T + 3) / 4), dim3(256), 0, s, a);
    }
  }
  return hipGetLastError();
}

// u extent KP: the smallest of 64, 128, 192, 320 that holds U + 1 (LDS and
// the d lm accumulators scale with it); GRP: sg_groups
template <int KP, int GRP>
static void launch_simple_grad(const SimpleArgs& a, int gs, hipStream_t s) {
  const int items = a.b.N * gs * ((a.V + kSgV - 1) / kSgV);
  const dim3 grid((items + 7) / 8 * 8), block(kSgThreads * GRP);
  if (a.lm_only != 0.f || a.am_only != 0.f) hipLaunchKernelGGL((simple_grad_kernel<KP, true, GRP>), grid, block, 0, s, a, gs, items);
  else hipLaunchKernelGGL((simple_grad_kernel<KP, false, GRP>), grid, block, 0, s, a, gs, items);
}

hipError_t launch_simple_grads(const SimpleArgs& a, hipStream_t s) {
  const int T = a.b.T, U1 = a.b.U + 1, V = a.V;
  {
    RNNT_PROF(s, "simple_colsum");
    hipLaunchKernelGGL(colsum_kernel, dim3((a.b.N * U1 + 255) / 256), dim3(256), 0, s, a);
  }
  if (a.am_only != 0.f) {
    RNNT_PROF(s, "smooth_grad_stats");
    hipLaunchKernelGGL(ac_colsum_kernel, dim3((V + kAcCols - 1) / kAcCols, a.b.N), dim3(256), 0, s, a);
    hipLaunchKernelGGL(lm_s_kernel, dim3((a.b.N * U1 + 3) / 4), dim3(256), 0, s, a);
  }
  const bool big = V >= kSimpleBigV;
  const int gs = simple_grad_splits(a.b.N, T, a.b.U, V);
  const bool smooth = a.lm_only != 0.f || a.am_only != 0.f;
  if (gs > 0 && a.am_grad && a.lm_grad) {
    {
      RNNT_PROF(s, "simple_grad");
      const bool two = sg_groups(a.b.N, a.b.U, V) == 2;
      if (U1 <= 64) two ? launch_simple_grad<64, 2>(a, gs, s) : launch_simple_grad<64, 1>(a, gs, s);
      else if (U1 <= 128) two ? launch_simple_grad<128, 2>(a, gs, s) : launch_simple_grad<128, 1>(a, gs, s);
      else if (U1 <= 192) launch_simple_grad<192, 1>(a, gs, s);
      else launch_simple_grad<kSgMaxU1, 1>(a, gs, s);
    }
    if (gs > 1 || smooth) {
      SimpleArgs e = a;
      e.lsplit = gs;  // the workspace holds max(dlm_splits, simple_grad_splits) partial sets
      const size_t groups = (size_t)a.b.N * U1 * ((V + 3) / 4);
      RNNT_PROF(s, "simple_dlm_epi");
      hipLaunchKernelGGL(dlm_epi_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, e);
    }
    return hipGetLastError();
  }
  if (a.am_grad) {
    RNNT_PROF(s, "simple_dam");
    if (big) {
      const dim3 grid((T + BigCfg::BM - 1) / BigCfg::BM, (V + BigCfg::BN - 1) / BigCfg::BN, a.b.N);
      hipLaunchKernelGGL(dam_kernel<BigCfg>, grid, dim3(BigCfg::NT), 0, s, a);
    } else {
      const dim3 grid((T + DamCfg::BM - 1) / DamCfg::BM, (V + DamCfg::BN - 1) / DamCfg::BN, a.b.N);
      hipLaunchKernelGGL(dam_kernel<DamCfg>, grid, dim3(DamCfg::NT), 0, s, a);
    }
  }
  if (a.lm_grad) {
    {
      RNNT_PROF(s, "simple_dlm");
      if (big) {
        const dim3 grid((U1 + BigCfg::BM - 1) / BigCfg::BM, (V + BigCfg::BN - 1) / BigCfg::BN, a.b.N * a.lsplit);
        hipLaunchKernelGGL(dlm_kernel<BigCfg>, grid, dim3(BigCfg::NT), 0, s, a);
      } else {
        const dim3 grid((U1 + DlmCfg::BM - 1) / DlmCfg::BM, (V + DlmCfg::BN - 1) / DlmCfg::BN, a.b.N * a.lsplit);
        hipLaunchKernelGGL(dlm_kernel<DlmCfg>, grid, dim3(DlmCfg::NT), 0, s, a);
      }
    }
    const size_t groups = (size_t)a.b.N * U1 * ((V + 3) / 4);
    {
      RNNT_PROF(s, "simple_dlm_epi");
      hipLaunchKernelGGL(dlm_epi_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, a);
    }
  }
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  {
    RNNT_PROF(s, "fill");
    hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  }
  return hipGetLastError();
}
