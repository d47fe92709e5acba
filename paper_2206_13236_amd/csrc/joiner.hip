// Stage 4a/4c: the full joiner evaluated only on the pruned (t, u) pairs
// (Sec. 3.2, Fig. 1(b)) and its backward pass.
//
// Rows. Every valid frame of the batch contributes S consecutive rows
// m = (frame_off[n] + t) * S + s (padding frames take no rows), so the GEMMs
// see one dense M = S * sum_n T_n dimension. A prep kernel writes, per row,
// the offsets of enc[n,t] and dec[n,u] (u = ranges[n,t,s]), the target symbol
// y_{u+1} (-1 at u = U_n, -2 when it lies outside [0, V)) and the output index
// n*T*S + t*S + s (-1 when the slot is absent, u > U_n).
//
// Operands. Every contraction runs on 16-bit MFMA with fp32 accumulation, its
// operands stored as rows of 16-bit words (gemm.h): bf16 inputs as they are,
// fp32 inputs as two fp16 planes whose products carry fp32's precision
// ("split"). h = tanh(enc + dec) and d(logits) are written in that form by
// the passes that produce them, W and its transpose by the prep kernel.
//
// Forward (per chunk of rows): an h pass, then logits = h W + bias. The
// epilogue reduces every (row, 64-column slice) to (max, sum exp) and
// captures the target and blank logits; a combine kernel turns them into
// lse, px = logit[y_{u+1}] - lse and py = logit[blank] - lse. The logits
// reach memory only when the caller asks for them ([N, T, S, V], the size
// the method's memory scales with).
//
// Backward (per chunk of at most a fixed number of rows, independent of the
// batch, so that d(logits), h and the d dec pieces are held for one chunk
// only and no [N, T, S, V] array exists):
//   1. dl = sc * ((gx+gy) softmax - gx [v=y] - gy [v=blank]) (log-softmax
//      backward) by recomputing h and the logits GEMM (or, when the caller
//      kept the forward's logits, by a streaming kernel over them); write the
//      chunk and column sums (db);
//   2. dh = dl W^T, dpre = dh (1 - h^2)  (tanh backward), kept in LDS: the
//      epilogue sums it into d enc[n,t] = sum_s dpre(row(t,s)) for the frames
//      inside the 128-row tile, and into per-tile pieces of the frames the
//      tile cuts and of d dec[n,u] = sum over the (t,s) with p_t + s = u;
//   3. dW += h^T dl with split-K partial sums;
//   4. the d dec pieces of the chunk are added to d dec in tile order;
// then a tail kernel adds the d enc pieces in tile order and sums dW and db
// over their partials, all in a fixed order.
#include <algorithm>

#include "gemm.h"
#include "kernels.h"
#include "prof.h"

namespace {

// 8 waves in a 4 x 2 grid (32 x 64 wave tiles): at most 128 registers per
// lane, so two workgroups (four waves per SIMD) share a CU.
constexpr int kGemmThreads = 512;
constexpr int kTileRows = 128;  // rows of every joiner GEMM tile but the wide forward's
constexpr int kTileCols = 128;
constexpr int kSlots = 512;      // joiner GEMM workgroups in flight: two on each of 256 CUs
constexpr int kDbRows = 32;     // rows summed into one db partial (a wave row of a tile)
// SP: fp32 inputs, split operands; otherwise bf16
template <bool SP>
using CfgN = LdsCfg<kTileRows, kTileCols, 4, 2, SP>;  // k-contiguous operands: logits and dh
template <bool SP>
using CfgT = TrCfg<kTileRows, kTileCols, 4, 2, SP>;   // dW: contraction over rows
// the forward at wide vocabularies: 256 x 256 tiles of 16 waves (64 x 64
// wave tiles, one workgroup per CU) read a third fewer operand bytes from
// LDS per MFMA than the 32 x 64 wave tiles: main loop alone, 6,941 x 8,000 x
// 768 in bf16 124 against 152 us, 20,020 x 5,000 x 512 split 362 against
// 391 us; slower where V gives few column tiles (16,040 x 500 x 512: 21.5
// against 16.0 us, split 41 against 28)
template <bool SP>
using CfgWide = LdsCfg<256, 256, 4, 4, SP>;
constexpr int kFwdWideV = 2048;
static_assert(CfgWide<false>::WN == 64 && CfgN<false>::WN == 64, "the forward's partial log-sum-exp slices are 64 columns");
static_assert(CfgN<false>::NT == kGemmThreads && CfgT<false>::NT == kGemmThreads, "joiner GEMM block size");
static_assert(CfgN<false>::WM == kDbRows, "db partial rows per wave row");

template <bool SP>
struct In { using T = float; };
template <>
struct In<false> { using T = uint16_t; };

// h lies in [-1, 1]: split operands hold 2^14 h.
constexpr float kHScale = 16384.f, kHInv = 1.f / 16384.f;

// ---------------------------------------------------------------------------
// Loads through buffer resources (make_rsrc, kOob: see common.h). A
// masked-out lane (row past the end, absent slot, column beyond J) loads from
// kOob and reads zeros instead of taking a divergent branch, so the loads of
// a pass issue back to back. Every input array is below 2^31 bytes (checked
// by the entry points).
// ---------------------------------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int W>
DEV void buf_words(Rsrc r, uint32_t off, uint32_t* w) {
  if constexpr (W == 8) {
    buf_words<4>(r, off, w);
    buf_words<4>(r, off + 16, w + 4);
  } else if constexpr (W == 4) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else {
    static_assert(W == 2, "8, 16 or 32 bytes");
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
    w[0] = v.x; w[1] = v.y;
  }
}

// N elements of TIn kept as 32-bit words until they are used, so that no
// conversion waits on an in-flight load.
template <typename TIn, int N>
struct RawVec {
  static constexpr int W = N * (int)sizeof(TIn) / 4;
  uint32_t w[W];
};

// The N elements at byte offset `off` (zeros unless `on`).
template <typename TIn, int N>
DEV void raw_load(Rsrc r, uint32_t off, bool on, RawVec<TIn, N>& out) {
  buf_words<RawVec<TIn, N>::W>(r, on ? off : kOob, out.w);
}

template <typename TIn, int N>
DEV void raw_to_float(const RawVec<TIn, N>& r, float (&v)[N]) {
  if constexpr (sizeof(TIn) == 4) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __uint_as_float(r.w[i]);
  } else {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      v[2 * i] = __uint_as_float(r.w[i] << 16);
      v[2 * i + 1] = __uint_as_float(r.w[i] & 0xffff0000u);
    }
  }
}

DEV float4 f4add(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// enc / dec resources of a launch (row offsets from rowinfo are element offsets).
template <typename TIn>
struct EncDec {
  Rsrc enc, dec;
  DEV EncDec(const JoinerArgs& a)
      : enc(make_rsrc(a.enc, (size_t)a.b.N * a.b.T * a.J * sizeof(TIn))),
        dec(make_rsrc(a.dec, (size_t)a.b.N * (a.b.U + 1) * a.J * sizeof(TIn))) {}
};

// The bias of this lane's output columns v0 + out_col(j) + r (`past` from
// column V on, 0 without a bias), with branch-free buffer loads issued ahead
// of the main loop and waited for once with wait_vmem() before the epilogue.
// A load inside a per-column branch would instead make the compiler wait
// again at every later branch, and with it for every store issued in between.
template <class Cfg>
DEV void bias_cols(const JoinerArgs& a, int v0, float past, float (&bj)[Cfg::FN][4]) {
  constexpr uint32_t esz = Cfg::SPLIT ? 4 : 2;
  const Rsrc rb = make_rsrc(a.bias, a.bias ? (size_t)a.V * esz : 0);
#pragma unroll
  for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = v0 + out_col<Cfg>(j) + r;
      const uint32_t off = col < a.V ? (uint32_t)col * esz : kOob;
      float v;
      if constexpr (Cfg::SPLIT) v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (int)off, 0, 0));
      else v = bf2f(__builtin_amdgcn_raw_buffer_load_b16(rb, (int)off, 0, 0));
      bj[j][r] = col < a.V ? v : past;
    }
}
// The factors that undo the scales of this lane's logits columns (split).
template <class Cfg>
DEV void unscale_cols(const JoinerArgs& a, int v0, float (&sj)[Cfg::FN][4]) {
  const Rsrc rs = make_rsrc(a.wt_inv, (size_t)a.V * 4);
#pragma unroll
  for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = v0 + out_col<Cfg>(j) + r;
      sj[j][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(col < a.V ? 4 * col : kOob), 0, 0));
    }
}

// ---------------------------------------------------------------------------
// Prep: per-utterance frame offsets and per-row info, W in the operand form,
// and the bound that scales d(logits).
// ---------------------------------------------------------------------------
constexpr int kPrepThreads = 256;

// bf16: W [J, V] copied into wn [J, row_words(V)] with zeros after column V:
// one 8-element group per thread.
DEV void prep_wpad(const JoinerArgs& a, int b) {
  const int gpr = a.ldd / 8;
  const int g = b * kPrepThreads + threadIdx.x;
  if (g >= a.J * gpr) return;
  const int j = g / gpr, c = (g - j * gpr) * 8;
  const uint16_t* src = reinterpret_cast<const uint16_t*>(a.W) + (size_t)j * a.V;
  uint32_t w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = (c + 2 * q < a.V) ? src[c + 2 * q] : 0u;
    const uint32_t hi = (c + 2 * q + 1 < a.V) ? src[c + 2 * q + 1] : 0u;
    w[q] = lo | (hi << 16);
  }
  *reinterpret_cast<uint4*>(a.wn + (size_t)j * a.ldd + c) = make_uint4(w[0], w[1], w[2], w[3]);
}

// bf16: W [J, V] transposed into wt [V, row_words(J)], one 64 x 64 tile per
// block through LDS: W read along v (consecutive threads, consecutive v), wt
// written in 16-byte groups of 8 consecutive j, zeros past J.
constexpr int kWtTile = 64;
DEV void prep_wt(const JoinerArgs& a, int b) {
  __shared__ uint16_t tile[kWtTile][kWtTile + 2];
  const int nvt = (a.V + kWtTile - 1) / kWtTile;
  const int j0 = (b / nvt) * kWtTile, v0 = (b % nvt) * kWtTile;
  const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
  const int c = threadIdx.x % kWtTile;
  for (int r = threadIdx.x / kWtTile; r < kWtTile; r += kPrepThreads / kWtTile) {
    const int j = j0 + r, v = v0 + c;
    tile[r][c] = (j < a.J && v < a.V) ? W[(size_t)j * a.V + v] : (uint16_t)0;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < kWtTile * (kWtTile / 8); q += kPrepThreads) {
    const int vr = q / (kWtTile / 8), jg = (q % (kWtTile / 8)) * 8;
    const int v = v0 + vr, j = j0 + jg;
    if (v >= a.V) continue;
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = (uint32_t)tile[jg + 2 * k][vr] | ((uint32_t)tile[jg + 2 * k + 1][vr] << 16);
    *reinterpret_cast<uint4*>(a.wt + (size_t)v * a.ldh + j) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// Eight scaled elements as a 16-byte chunk of each plane, at element k of a row.
DEV void store_split8(uint16_t* row, int k, const float (&x)[8], float s) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) split_f16x2(x[2 * q] * s, x[2 * q + 1] * s, h[q], l[q]);
  uint16_t* dst = row + split_word(k);
  *reinterpret_cast<uint4*>(dst) = make_uint4(h[0], h[1], h[2], h[3]);
  *reinterpret_cast<uint4*>(dst + 32) = make_uint4(l[0], l[1], l[2], l[3]);
}

template <bool SP>
constexpr int kHItems = SP ? 2 : 4;
template <bool SP>
constexpr __host__ __device__ int h_groups(int J) { return row_words<SP>(J) / (SP ? 16 : 8); }

// h = tanh(enc + dec) of 8 columns from j on into a row of h in operand form
// (zeros unless `on`).
template <bool SP>
DEV void store_h8(uint16_t* row, int j, const RawVec<typename In<SP>::T, 8>& e, const RawVec<typename In<SP>::T, 8>& d, bool on) {
  float fe[8], fd[8], h[8];
  raw_to_float(e, fe);
  raw_to_float(d, fd);
#pragma unroll
  for (int q = 0; q < 8; ++q) h[q] = on ? fast_tanh(fe[q] + fd[q]) : 0.f;
  if constexpr (SP) {
    store_split8(row, j, h, kHScale);
  } else {
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = (uint32_t)f2bf(h[2 * q]) | ((uint32_t)f2bf(h[2 * q + 1]) << 16);
    *reinterpret_cast<uint4*>(row + j) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

DEV float wave_max_f(float m) {
  m = row16_max(m);
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  return fmaxf(m, __shfl_xor(m, 32, 64));
}

// fp32: row j of W as planes in wn [J, row_words(V)] for dh, scaled by the
// row's largest element (undone per output column j by wn_inv). One block a
// row; the second pass reads the row from cache.
DEV void prep_wn_split(const JoinerArgs& a, int j) {
  __shared__ float s_max[kPrepThreads / 64];
  const float* src = reinterpret_cast<const float*>(a.W) + (size_t)j * a.V;
  float m = 0.f;
  for (int v = threadIdx.x; v < a.V; v += kPrepThreads) m = fmaxf(m, finite_abs(src[v]));
  m = wave_max_f(m);
  if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = m;
  __syncthreads();
  const float s = split_scale(fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3])));
  if (threadIdx.x == 0) a.wn_inv[j] = pow2_inv(s);
  for (int c = threadIdx.x * 8; c < a.ldd / 2; c += kPrepThreads * 8) {
    float x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = c + q < a.V ? src[c + q] : 0.f;
    store_split8(a.wn + (size_t)j * a.ldd, c, x, s);
  }
}

// fp32: kWtCols columns of W as rows of planes in wt [V, row_words(J)] for
// the logits, each scaled by its largest element (undone, with h's scale, per
// output column v by wt_inv).
constexpr int kWtCols = 8;
DEV void prep_wt_split(const JoinerArgs& a, int b) {
  __shared__ float s_max[kPrepThreads];
  const float* W = reinterpret_cast<const float*>(a.W);
  const int c = threadIdx.x % kWtCols, v = b * kWtCols + c;
  float m = 0.f;
  if (v < a.V) {
#pragma unroll 8
    for (int j = threadIdx.x / kWtCols; j < a.J; j += kPrepThreads / kWtCols) m = fmaxf(m, finite_abs(W[(size_t)j * a.V + v]));
  }
  s_max[threadIdx.x] = m;
  __syncthreads();
  for (int st = kPrepThreads / 2; st >= kWtCols; st >>= 1) {
    if ((int)threadIdx.x < st) s_max[threadIdx.x] = fmaxf(s_max[threadIdx.x], s_max[threadIdx.x + st]);
    __syncthreads();
  }
  if ((int)threadIdx.x < kWtCols && v < a.V) a.wt_inv[v] = pow2_inv(split_scale(s_max[c])) * kHInv;
  const int ng = a.ldh / 16;  // 8-element groups of a row
  for (int q = threadIdx.x; q < ng * kWtCols; q += kPrepThreads) {
    const int cc = q % kWtCols, j = q / kWtCols * 8, vv = b * kWtCols + cc;
    if (vv >= a.V) continue;
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = j < a.J ? W[(size_t)(j + k) * a.V + vv] : 0.f;  // J is a multiple of 8
    store_split8(a.wt + (size_t)vv * a.ldh, j, x, split_scale(s_max[cc]));
  }
}

// fp32 backward: the scale of a row's d(logits) planes, from the bound
// |scale| (|gx| + |gy|) (softmax <= 1), so that every row keeps fp32's
// relative precision whatever its utterance's scale and its occupations.
DEV float row_scale(const JoinerArgs& a, int n, size_t nts) {
  const float g = finite_abs(a.gxo[nts]) + finite_abs(a.gyo[nts]);
  return split_scale(finite_abs(g * (a.scale ? a.scale[n] : 1.f)));
}

// Blocks of the prep kernel after those of the utterances, and the column
// parts of h: with hj > 0 every 256 rows of an utterance have hj blocks, each
// of which also writes its share of the columns of those rows' h (the forward,
// rows below hrows: its first chunk), so that the h pass takes no launch of
// its own.
struct PrepBlocks {
  int wn, wt;
  int hj, hrows;
};
constexpr int kPrepHGroups = 8;  // 8-column groups of a row per block

template <bool SP>
__global__ __launch_bounds__(kPrepThreads) void joiner_prep_kernel(JoinerArgs a, PrepBlocks pb) {
  __shared__ int s_part[4];
  __shared__ int4 s_info[kPrepThreads];
  const int parts = pb.hj > 0 ? pb.hj : 1;
  const int per = (a.b.T * a.S + 255) / 256 * parts;  // blocks per utterance: one (t, s) slot per thread
  if ((int)blockIdx.x >= a.b.N * per) {
    int b = blockIdx.x - a.b.N * per;
    if (b < pb.wt) {
      if constexpr (SP) prep_wt_split(a, b);
      else prep_wt(a, b);
      return;
    }
    b -= pb.wt;
    if constexpr (SP) prep_wn_split(a, b);
    else prep_wpad(a, b);
    return;
  }
  const int n = blockIdx.x / per, rest = blockIdx.x - n * per, part = rest % parts;
  const int i0 = rest / parts * 256, i = i0 + threadIdx.x;
  const int T = a.b.T, U1 = a.b.U + 1, S = a.S, J = a.J;
  // frame offset of utterance n: sum of T_q over q < n, the lengths loaded
  // in parallel and summed by a block reduction
  int before = 0;
  for (int q = threadIdx.x; q < n; q += blockDim.x) {
    int Tq, Uq;
    utt_dims(a.b, q, Tq, Uq);
    before += Tq;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = before;
  __syncthreads();
  const int off = s_part[0] + s_part[1] + s_part[2] + s_part[3];
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  if (i == 0 && part == 0) {
    a.frame_off[n] = off;
    if (n == a.b.N - 1) a.frame_off[a.b.N] = off + Tn;
  }
  int4 r = make_int4(0, 0, -1, -1);
  float rs = 1.f;
  if (i < Tn * S) {
    const int t = i / S, s = i - t * S;
    const size_t nts = ((size_t)n * T + t) * S + s;
    const int u = a.ranges[nts];
    if (s == 0 && part == 0 && a.frame_nt) {
      a.frame_nt[off + t] = n * T + t;
      a.frame_p[off + t] = u;
    }
    if (u >= 0 && u <= Un) {
      bool ok = true;
      r.x = (int)(((size_t)n * T + t) * J);
      r.y = (int)(((size_t)n * U1 + u) * J);
      r.z = (u < Un) ? symbol_at(a.b, n, u, a.V, ok) : -1;
      if (!ok) r.z = -2;  // symbol outside [0, V): px is NaN, so the utterance's loss is NaN
      r.w = (int)nts;
      if (SP && a.rsc) rs = row_scale(a, n, nts);
    }
    if (part == 0) {
      a.rowinfo[(size_t)(off + t) * S + s] = r;
      if (SP && a.rsc) a.rsc[(size_t)(off + t) * S + s] = rs;
    }
  }
  // h of the block's rows, kPrepHGroups groups of 8 columns from its part on
  const int m0 = off * S + i0, rows = min(min(256, Tn * S - i0), pb.hrows - m0);
  if (pb.hj == 0 || rows <= 0) return;
  s_info[threadIdx.x] = r;
  __syncthreads();
  const int ng = h_groups<SP>(J), g0 = part * kPrepHGroups;
  const EncDec<typename In<SP>::T> ed(a);
  constexpr int NI = kHItems<SP>;
#pragma unroll 1
  for (int it = 0; it < kPrepHGroups; it += NI) {
    RawVec<typename In<SP>::T, 8> e[NI], d[NI];
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int q = (it + k) * kPrepThreads + threadIdx.x, row = q / kPrepHGroups, j = (g0 + q % kPrepHGroups) * 8;
      const int4 info = s_info[row];
      const bool on = row < rows && info.w >= 0 && j < J;
      raw_load(ed.enc, (uint32_t)(info.x + j) * (uint32_t)sizeof(typename In<SP>::T), on, e[k]);
      raw_load(ed.dec, (uint32_t)(info.y + j) * (uint32_t)sizeof(typename In<SP>::T), on, d[k]);
    }
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int q = (it + k) * kPrepThreads + threadIdx.x, row = q / kPrepHGroups, g = g0 + q % kPrepHGroups;
      if (row < rows && g < ng)
        store_h8<SP>(a.hbuf + (size_t)(m0 + row) * a.ldh, g * 8, e[k], d[k], s_info[row].w >= 0 && g * 8 < J);
    }
  }
}

// ---------------------------------------------------------------------------
// h = tanh(enc + dec) of the rows [cm0, min(cm1, M)) into the chunk buffer
// h [rows, row_words(J)] in operand form (zero rows for absent slots, zeros
// past column J): kHItems groups of 8 columns per thread (consecutive
// threads, consecutive groups), whose row info, then enc and dec loads, are
// issued together; the batch's row count M is loaded beside the row info
// (rows past it hold no row info and are skipped).
// ---------------------------------------------------------------------------
// Block blk of NT threads of an h pass into hdst (the chunk's rows from cm0).
template <bool SP, int NT>
DEV void h_rows_block(const JoinerArgs& a, uint16_t* hdst, int cm0, int cm1, int blk) {
  using TIn = typename In<SP>::T;
  constexpr int NI = kHItems<SP>;
  const int cpr = h_groups<SP>(a.J);
  const size_t base = (size_t)blk * (NT * NI) + threadIdx.x;
  int rr[NI], jj[NI];
  int4 info[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const size_t i = base + (size_t)k * NT;
    rr[k] = (int)(i / cpr);
    jj[k] = (int)(i - (size_t)rr[k] * cpr) * 8;
    // within the row info array (cm1 <= N*T*S); rows past M are masked below
    info[k] = cm0 + rr[k] < cm1 ? a.rowinfo[cm0 + rr[k]] : make_int4(0, 0, -1, -1);
  }
  const int M = a.frame_off[a.b.N] * a.S;
  const int mend = min(cm1, M);
  const EncDec<TIn> ed(a);
  RawVec<TIn, 8> e[NI], d[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const bool on = cm0 + rr[k] < mend && info[k].w >= 0 && jj[k] < a.J;
    raw_load(ed.enc, (uint32_t)(info[k].x + jj[k]) * sizeof(TIn), on, e[k]);
    raw_load(ed.dec, (uint32_t)(info[k].y + jj[k]) * sizeof(TIn), on, d[k]);
  }
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    if (cm0 + rr[k] >= mend) continue;
    store_h8<SP>(hdst + (size_t)rr[k] * a.ldh, jj[k], e[k], d[k], info[k].w >= 0 && jj[k] < a.J);
  }
}

// An h pass: rows [cm0, cm1) into h, `blocks` blocks.
struct HPass {
  int blocks, cm0, cm1;
  uint16_t* h;
};
static HPass h_pass(const JoinerArgs& slot, int cm0, int cm1, int threads) {
  const size_t groups = (size_t)(cm1 - cm0) * (slot.bf16 ? h_groups<false>(slot.J) : h_groups<true>(slot.J));
  const size_t per = (size_t)threads * (slot.bf16 ? kHItems<false> : kHItems<true>);
  return HPass{(int)((groups + per - 1) / per), cm0, cm1, slot.hbuf};
}

// ---------------------------------------------------------------------------
// Forward GEMM + partial log-sum-exp over the rows [cm0, cm1) (h in hbuf).
// The blocks past the ngemm tile blocks run the h pass of the next chunk.
// ---------------------------------------------------------------------------
template <bool SP, bool WIDE>
__global__ __launch_bounds__(WIDE ? CfgWide<SP>::NT : kGemmThreads, 4) void joiner_fwd_kernel(JoinerArgs a, int cm0, int cm1,
                                                                                              int ncol, int ngemm,
                                                                                              HPass hn) {
  using Cfg = typename std::conditional<WIDE, CfgWide<SP>, CfgN<SP>>::type;
  __shared__ __align__(16) unsigned char smem[Cfg::SMEM_BYTES];
  if ((int)blockIdx.x >= ngemm) {
    h_rows_block<SP, Cfg::NT>(a, hn.h, hn.cm0, hn.cm1, blockIdx.x - ngemm);
    return;
  }
  const int M = a.frame_off[a.b.N] * a.S;
  const int mend = min(cm1, M);
  // the column tiles of one row tile are consecutive tile ids (one XCD, shared A panel)
  const int tile = xcd_tile_id(mend > cm0 ? (mend - cm0 + Cfg::BM - 1) / Cfg::BM * ncol : 0);
  if (tile < 0) return;
  const int mt = tile / ncol, nt = tile - mt * ncol;
  const int m0 = cm0 + mt * Cfg::BM;
  const int v0 = nt * Cfg::BN;
  const int V = a.V;
  int4 info[Cfg::FM];
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int m = m0 + out_row<Cfg>(i);
    info[i] = m < mend ? a.rowinfo[m] : make_int4(0, 0, -1, -1);
  }
  float bj[Cfg::FN][4], sj[SP ? Cfg::FN : 1][4];
  auto loads = [&]() {
    bias_cols<Cfg>(a, v0, kNegInfF, bj);
    if constexpr (SP) unscale_cols<Cfg>(a, v0, sj);
  };
  floatx4 acc[Cfg::FM][Cfg::FN];
  // h of the chunk and W^T, both k = j contiguous
  const LdsSrc sa(a.hbuf + (size_t)(m0 - cm0) * a.ldh, min(Cfg::BM, mend - m0), a.ldh);
  const LdsSrc sb(a.wt + (size_t)v0 * a.ldh, min(Cfg::BN, V - v0), a.ldh);
  gemm_mainloop_lds<Cfg>(sa, sb, smem, acc);
  loads();
  wait_vmem();

  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) % Cfg::WGN, lq = lane >> 4;
  const int slice = nt * Cfg::WGN + wn;
  const int vs = v0 + wn * Cfg::WN;             // the slice's first column
  const unsigned brel = (unsigned)(a.b.blank - vs);  // the blank's column in the slice
  const bool vec_l = (V & 3) == 0;
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int m = m0 + out_row<Cfg>(i);
    float lg[Cfg::FN][4];
    float mx = kNegInfF;
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lg[j][r] = SP ? fmaf(acc[i][j][r], sj[SP ? j : 0][r], bj[j][r]) : acc[i][j][r] + bj[j][r];  // -inf from column V on
        mx = fmaxf(mx, lg[j][r]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mref = mx == kNegInfF ? 0.f : mx;  // a slice of -inf logits sums to 0
    float se = 0.f;
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) se += __expf(lg[j][r] - mref);
    se += __shfl_xor(se, 16, 64);
    se += __shfl_xor(se, 32, 64);
    if (info[i].w >= 0) {
      if (lq == 0 && slice < a.nparts) a.part[(size_t)m * a.nparts + slice] = make_float2(mx, se);
      const unsigned trel = (unsigned)(info[i].z - vs);
      if (trel < 64u && (int)(trel >> 2 & 3) == lq) {
        float x = 0.f;
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) x = (trel >> 4) == (unsigned)j && (trel & 3) == (unsigned)r ? lg[j][r] : x;
        a.tgt[m] = x;
      }
      if (brel < 64u && (int)(brel >> 2 & 3) == lq) {
        float x = 0.f;
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) x = (brel >> 4) == (unsigned)j && (brel & 3) == (unsigned)r ? lg[j][r] : x;
        a.blk[m] = x;
      }
      if (a.logits) {
        float* dst = a.logits + (size_t)info[i].w * V;
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j) {
          const int c = v0 + out_col<Cfg>(j);
          if (vec_l) {
            if (c < V) *reinterpret_cast<float4*>(dst + c) = make_float4(lg[j][0], lg[j][1], lg[j][2], lg[j][3]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (c + r < V) dst[c + r] = lg[j][r];
          }
        }
      }
      if (m < a.head_rows) {  // whole 4-column groups (the head's rows are padded to 8)
        float* dst = a.head + (size_t)m * a.ldl;
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j) {
          const int c = v0 + out_col<Cfg>(j);
          if (c < a.ldl) *reinterpret_cast<float4*>(dst + c) = make_float4(lg[j][0], lg[j][1], lg[j][2], lg[j][3]);
        }
      }
    }
  }
}

__global__ __launch_bounds__(256) void joiner_combine_kernel(JoinerArgs a) {
  const int T = a.b.T, S = a.S;
  const size_t total = (size_t)a.b.N * T * S;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int n = (int)(i / ((size_t)T * S));
  const int rem = (int)(i - (size_t)n * T * S);
  const int t = rem / S, s = rem - t * S;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  float px = kNegInfF, py = kNegInfF, l = 0.f;
  if (t < Tn) {
    const int m = (a.frame_off[n] + t) * S + s;
    const int4 info = a.rowinfo[m];
    if (info.w >= 0) {
      const float2* pp = a.part + (size_t)m * a.nparts;
      float M = kNegInfF;
      for (int p = 0; p < a.nparts; ++p) M = fmaxf(M, pp[p].x);
      float sum = 0.f;
      for (int p = 0; p < a.nparts; ++p) sum += pp[p].y * __expf(pp[p].x - M);
      l = M + __logf(sum);
      py = a.blk[m] - l;
      px = (info.z >= 0) ? a.tgt[m] - l : (info.z == -2 ? __builtin_nanf("") : kNegInfF);
    }
  }
  a.px[i] = px;
  a.py[i] = py;
  a.lse[i] = l;
}

// The same for wide vocabularies (more than kCombineSerialParts slices of 64
// columns): one wave per output, lanes over the slices (coalesced reads), the
// max and the sum each by a lane-ordered pass and a fixed reduction across
// the lanes, so the result does not depend on scheduling.
constexpr int kCombineSerialParts = 16;
__global__ __launch_bounds__(256) void joiner_combine_wide_kernel(JoinerArgs a) {
  const int T = a.b.T, S = a.S, lane = threadIdx.x & 63;
  const size_t total = (size_t)a.b.N * T * S;
  const size_t i = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= total) return;
  const int n = (int)(i / ((size_t)T * S));
  const int rem = (int)(i - (size_t)n * T * S);
  const int t = rem / S, s = rem - t * S;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  float px = kNegInfF, py = kNegInfF, l = 0.f;
  if (t < Tn) {
    const int m = (a.frame_off[n] + t) * S + s;
    const int4 info = a.rowinfo[m];
    if (info.w >= 0) {
      const float2* pp = a.part + (size_t)m * a.nparts;
      float M = kNegInfF;
      for (int p = lane; p < a.nparts; p += 64) M = fmaxf(M, pp[p].x);
      M = row16_max(M);  // within each 16-lane row, then across the rows
      M = fmaxf(M, __shfl_xor(M, 16, 64));
      M = fmaxf(M, __shfl_xor(M, 32, 64));
      float sum = 0.f;
      for (int p = lane; p < a.nparts; p += 64) sum += pp[p].y * __expf(pp[p].x - M);
      sum = row16_sum(sum);
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      l = M + __logf(sum);
      py = a.blk[m] - l;
      px = (info.z >= 0) ? a.tgt[m] - l : (info.z == -2 ? __builtin_nanf("") : kNegInfF);
    }
  }
  if (lane == 0) {
    a.px[i] = px;
    a.py[i] = py;
    a.lse[i] = l;
  }
}

// ---------------------------------------------------------------------------
// LDS of the backward's GEMM tiles: the operand stages (also dh's tile of
// dpre), then per-row info and per-row scalars of the row tile. One size for
// all of them, so that tiles of different kinds share one launch.
// ---------------------------------------------------------------------------
constexpr int kDpreLd = kTileCols + 4;  // row stride of the dpre tile (floats)
constexpr int kBwdStageBytes = kTileRows * kDpreLd * 4;
static_assert(CfgN<true>::SMEM_BYTES <= kBwdStageBytes && CfgT<true>::SMEM_BYTES <= kBwdStageBytes, "operand stages fit");
static_assert(CfgN<false>::SMEM_BYTES <= kBwdStageBytes && CfgT<false>::SMEM_BYTES <= kBwdStageBytes, "operand stages fit");
constexpr int kBwdLdsBytes = kBwdStageBytes + kTileRows * (int)(sizeof(int4) + sizeof(float));
DEV int4* lds_rowinfo(unsigned char* lds) { return reinterpret_cast<int4*>(lds + kBwdStageBytes); }
DEV float* lds_rowinv(unsigned char* lds) { return reinterpret_cast<float*>(lds_rowinfo(lds) + kTileRows); }

// Tile `tile` (row tile tile / ncol, column tile tile % ncol) of the rows
// [cm0, cm1) whose count of active tiles (rows present) is computed here: -1
// for blocks beyond it. The XCD-aware order of xcd_tile_id over a part of a
// launch: v is the block's index within its part of nblocks blocks.
DEV int part_tile(int v, int nblocks, int n_active) {
  const int n = min(n_active, nblocks);
  if (v >= n) return -1;
  const int per = n / kNumXcd, rem = n % kNumXcd;
  const int x = v % kNumXcd, loc = v / kNumXcd;
  return __builtin_amdgcn_readfirstlane((x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + loc);
}
DEV int chunk_row_tiles(const JoinerArgs& a, int cm0, int cm1) {
  const int mend = min(cm1, a.frame_off[a.b.N] * a.S);
  return mend > cm0 ? (mend - cm0 + kTileRows - 1) / kTileRows : 0;
}

// d(logits) of 4 neighbouring columns from column c on (a multiple of 4) into
// a row of the chunk buffer, in operand form (s: the planes' scales).
// Split d(logits) are stored twice, since the two contractions sum over
// different directions and two fp16 planes hold an element to 2^-39 of the
// largest one under its scale: dl with a scale per row for dh, which sums
// over a row, dc with a scale per column and 32 rows for dW, which sums over
// a column (a token of probability 1e-12 is 0 under a row's scale, an
// utterance of scale 1e-12 under a batch's). The second copy takes joiner and
// backward at N = 16, T = 300, V = 5000, S = 5, J = 512 from 1,420 to 1,630 us.
template <bool SP>
DEV void store_dl4(uint16_t* row, int c, const float (&d)[4], const float (&s)[4]) {
  if constexpr (SP) {
    uint32_t h[2], l[2];
    split_f16x2(d[0] * s[0], d[1] * s[1], h[0], l[0]);
    split_f16x2(d[2] * s[2], d[3] * s[3], h[1], l[1]);
    uint16_t* dst = row + split_word(c);
    *reinterpret_cast<uint2*>(dst) = make_uint2(h[0], h[1]);
    *reinterpret_cast<uint2*>(dst + 32) = make_uint2(l[0], l[1]);
  } else {
    *reinterpret_cast<uint2*>(row + c) = make_uint2((uint32_t)f2bf(d[0]) | ((uint32_t)f2bf(d[1]) << 16),
                                                    (uint32_t)f2bf(d[2]) | ((uint32_t)f2bf(d[3]) << 16));
  }
}
// What undoes the scales of 4 columns of dc and of h.
DEV float4 dc_factors(const float (&s)[4]) {
  return make_float4(pow2_inv(s[0]) * kHInv, pow2_inv(s[1]) * kHInv, pow2_inv(s[2]) * kHInv, pow2_inv(s[3]) * kHInv);
}
// Elements of a row of d(logits) in the chunk buffer (zeros from column V on).
template <bool SP>
constexpr __host__ __device__ int dl_cols(int V) { return row_words<SP>(V) / (SP ? 2 : 1); }

// ---------------------------------------------------------------------------
// Backward 1: recompute logits from h (hbuf, rows of the chunk), d(logits)
// of one 128 x 128 tile into the chunk buffer dl, db partials (one row per
// wave row of each row tile of the chunk; the first chunk writes them, later
// chunks add to them).
// ---------------------------------------------------------------------------
template <bool SP>
DEV void dlogits_tile(const JoinerArgs& a, int cm0, int cm1, int v, int nblocks, int ncol, unsigned char* lds) {
  using Cfg = CfgN<SP>;
  const int M = a.frame_off[a.b.N] * a.S;
  const int mend = min(cm1, M);
  const int tile = part_tile(v, nblocks, chunk_row_tiles(a, cm0, cm1) * ncol);
  if (tile < 0) return;
  const int mt = tile / ncol, nt = tile - mt * ncol;
  const int m0 = cm0 + mt * Cfg::BM;
  const int v0 = nt * Cfg::BN;
  const int V = a.V, TS = a.b.T * a.S;
  int4 info[Cfg::FM];
  float4 x[Cfg::FM];  // lse, gx, gy, scale of this lane's rows
  float rs[Cfg::FM];  // the scales of their planes (split)
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int m = m0 + out_row<Cfg>(i);
    info[i] = m < mend ? a.rowinfo[m] : make_int4(0, 0, -1, -1);
    x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    rs[i] = SP && m < mend ? a.rsc[m] : 1.f;
    if (info[i].w >= 0) {
      const int n = info[i].w / TS;
      x[i] = make_float4(a.lse_in[info[i].w], a.gxo[info[i].w], a.gyo[info[i].w], a.scale ? a.scale[n] : 1.f);
    }
  }
  const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) / Cfg::WGN;
  floatx4 acc[Cfg::FM][Cfg::FN];
  const LdsSrc sa(a.hbuf + (size_t)(m0 - cm0) * a.ldh, min(Cfg::BM, mend - m0), a.ldh);
  const LdsSrc sb(a.wt + (size_t)v0 * a.ldh, min(Cfg::BN, V - v0), a.ldh);
  gemm_mainloop_lds<Cfg>(sa, sb, lds, acc);
  // bias, scales and this lane's db_part entries (a later chunk adds to what
  // the earlier ones left), loaded before the epilogue's stores: see bias_cols
  float bj[Cfg::FN][4], sj[SP ? Cfg::FN : 1][4];
  bias_cols<Cfg>(a, v0, kNegInfF, bj);
  if constexpr (SP) unscale_cols<Cfg>(a, v0, sj);
  float* dbq = a.db_part + ((size_t)mt * Cfg::WGM + wm) * V;
  const int dcol = v0 + out_col<Cfg>(lane & 3) + (lane >> 2 & 3);  // the column whose sum this lane ends up with
  const float dbold = (cm0 != 0 && dcol < V) ? dbq[dcol] : 0.f;
  wait_vmem();

  float cs[Cfg::FN][4];
#pragma unroll
  for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) cs[j][r] = 0.f;
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int m = m0 + out_row<Cfg>(i);
    const float g = x[i].y + x[i].z;
    const bool on = info[i].w >= 0;
    uint16_t* row = a.dl + (size_t)(m - cm0) * a.ldd;
    const float ds[4] = {rs[i], rs[i], rs[i], rs[i]};
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      const int c = v0 + out_col<Cfg>(j);
      float d[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float lg = SP ? fmaf(acc[i][j][r], sj[SP ? j : 0][r], bj[j][r]) : acc[i][j][r] + bj[j][r];
        float gd = g * __expf(lg - x[i].x);
        if (c + r == info[i].z) gd -= x[i].y;
        if (c + r == a.b.blank) gd -= x[i].z;
        d[r] = on && c + r < V ? x[i].w * gd : 0.f;
        cs[j][r] += d[r];
        if (SP) acc[i][j][r] = d[r];
      }
      if (a.logits_grad && on) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (c + r < V) a.logits_grad[(size_t)info[i].w * V + c + r] = d[r];
      }
      if (m < mend && c < dl_cols<SP>(V)) store_dl4<SP>(row, c, d, ds);
    }
  }
  // dc: the scale of each column within the wave's 32 rows
  if constexpr (SP) {
    float* inv = a.dc_inv + ((size_t)mt * Cfg::WGM + wm) * a.ldl;
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      const int c = v0 + out_col<Cfg>(j);
      float s[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < Cfg::FM; ++i) mx = fmaxf(mx, __builtin_fabsf(acc[i][j][r]));
        s[r] = split_scale(row16_max(mx));
      }
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) {
        const int m = m0 + out_row<Cfg>(i);
        const float d[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
        if (m < mend && c < dl_cols<SP>(V)) store_dl4<SP>(a.dc + (size_t)(m - cm0) * a.ldd, c, d, s);
      }
      if ((lane & 15) == j && c < a.ldl) *reinterpret_cast<float4*>(inv + c) = dc_factors(s);
    }
  }
  // db partial: each column summed over the wave's 32 rows, 16 lanes x FM
  // each. Halving: the lanes of a pair keep half of the columns each and add
  // the partner's share, so 16 columns take 8 + 4 + 2 + 1 exchanges; lane l
  // ends with column (j, r) = (l & 3, l >> 2 & 3).
  const bool k1 = lane & 1, k2 = lane & 2, k4 = lane & 4, k8 = lane & 8;
  float c2[2][4], c1[4], h2[2];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float mine = k1 ? cs[2 * q + 1][r] : cs[2 * q][r], give = k1 ? cs[2 * q][r] : cs[2 * q + 1][r];
      c2[q][r] = mine + __shfl_xor(give, 1, 64);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float mine = k2 ? c2[1][r] : c2[0][r], give = k2 ? c2[0][r] : c2[1][r];
    c1[r] = mine + __shfl_xor(give, 2, 64);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float mine = k4 ? c1[2 * q + 1] : c1[2 * q], give = k4 ? c1[2 * q] : c1[2 * q + 1];
    h2[q] = mine + __shfl_xor(give, 4, 64);
  }
  const float mine = k8 ? h2[1] : h2[0], give = k8 ? h2[0] : h2[1];
  const float s = mine + __shfl_xor(give, 8, 64);
  if (dcol < V) dbq[dcol] = dbold + s;
}

// ---------------------------------------------------------------------------
// Backward 1, stored logits: the same d(logits) streamed from the logits the
// forward kept, either all of them ([N, T, S, V], logits_in) or those of the
// first chunk (head, rows in joiner-row order, for chunk 0 only). One block
// per kDlRows rows of the chunk, threads over groups of 4 columns (padding
// columns get zeros), several rows per thread with their loads issued
// together; the block's column sums are one db_part row.
// ---------------------------------------------------------------------------
constexpr int kDlRows = kDbRows;
constexpr int kDlThreads = 256;
constexpr int kDlInFlight = 16;  // rows per thread whose loads are issued together

// Threads per row of a block (over the ng 4-column groups of a row); a block
// takes tpr groups of kDlRows rows, and grid.y the ceil(ng / tpr) column
// ranges, so that wide rows spread over many blocks. Split: at most half of
// the block, so that a thread's rows are all in flight at once and their
// values stay in registers until the column's scale is known.
template <bool SP>
__host__ __device__ inline int dl_threads_per_row(int ng) {
  return ng <= 64 ? 64 : (SP || ng <= 128 ? 128 : kDlThreads);
}
static_assert(kDlRows / (kDlThreads / 128) <= kDlInFlight, "a split block's rows in one pass");
template <bool SP>
static dim3 dl_grid(const JoinerArgs& a, int rows) {
  const int ng = dl_cols<SP>(a.V) / 4, tpr = dl_threads_per_row<SP>(ng);
  return dim3((unsigned)((rows + kDlRows - 1) / kDlRows), (unsigned)((ng + tpr - 1) / tpr));
}

struct DlSmem {
  int4 ri[kDlRows];
  float4 rx[kDlRows];  // lse, gx, gy, scale
  float rs[kDlRows];   // the planes' scale (split)
  float4 red[kDlThreads];
};

// Block (bx, by) of the d(logits) stream: rows cm0 + 32 bx .., column groups of by.
template <bool SP>
DEV void dl_block(const JoinerArgs& a, int cm0, int cm1, int bx, int by, DlSmem& sm) {
  int4* ri = sm.ri;
  float4* rx = sm.rx;
  float4* red = sm.red;
  const int M = a.frame_off[a.b.N] * a.S;
  const int mend = min(cm1, M);
  const int m0 = cm0 + bx * kDlRows;
  if (m0 >= mend) return;
  const int V = a.V, TS = a.b.T * a.S, ldl = a.ldl, blank = a.b.blank;
  const int nrows = min(kDlRows, mend - m0);
  if (threadIdx.x < kDlRows) {
    const int r = threadIdx.x;
    int4 info = (r < nrows) ? a.rowinfo[m0 + r] : make_int4(0, 0, -1, -1);
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (info.w >= 0) {
      const int n = info.w / TS;
      x = make_float4(a.lse_in[info.w], a.gxo[info.w], a.gyo[info.w], a.scale ? a.scale[n] : 1.f);
    }
    ri[r] = info;
    rx[r] = x;
    if constexpr (SP) sm.rs[r] = r < nrows ? a.rsc[m0 + r] : 1.f;
  }
  __syncthreads();
  const bool from_head = a.logits_in == nullptr;  // chunk 0 from the head rows
  const float* __restrict__ lg = from_head ? a.head : a.logits_in;
  const int ng = dl_cols<SP>(V) / 4;
  const int tpr = dl_threads_per_row<SP>(ng);
  const int nrg = kDlThreads / tpr, rg = threadIdx.x / tpr, ct = threadIdx.x - rg * tpr;
  const bool vec = from_head || (V & 3) == 0;
  const int c = 4 * (by * tpr + ct);  // this thread's columns
  const bool gok = by * tpr + ct < ng;
  float cs[4] = {0.f, 0.f, 0.f, 0.f};
  float cm[4] = {0.f, 0.f, 0.f, 0.f};       // split: the columns' largest |d(logits)| of this thread's rows
  float l[kDlInFlight][4];                  // the rows in flight: their logits, then (split) their d(logits)
  if (gok) {
    for (int p0 = rg; p0 < nrows; p0 += nrg * kDlInFlight) {
#pragma unroll
      for (int k = 0; k < kDlInFlight; ++k) {
        const int r = p0 + k * nrg;
        const int4 info = ri[min(r, kDlRows - 1)];
        const bool ok = r < nrows && info.w >= 0 && c < V;
        const float* src = lg + (ok ? (from_head ? (size_t)(m0 + r) * ldl : (size_t)info.w * V) + c : 0);
        if (ok && vec) {
          const float4 q = *reinterpret_cast<const float4*>(src);
          l[k][0] = q.x; l[k][1] = q.y; l[k][2] = q.z; l[k][3] = q.w;
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) l[k][q] = (ok && c + q < V) ? src[q] : 0.f;
        }
      }
#pragma unroll
      for (int k = 0; k < kDlInFlight; ++k) {
        const int r = p0 + k * nrg;
        if (r >= nrows) break;
        const int4 info = ri[r];
        const float4 x = rx[r];
        const float g = x.y + x.z;
        float d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = c + q;
          d[q] = 0.f;
          if (info.w >= 0 && col < V) {
            float gd = g * __expf(l[k][q] - x.x);
            if (col == info.z) gd -= x.y;
            if (col == blank) gd -= x.z;
            d[q] = x.w * gd;
            if (a.logits_grad) a.logits_grad[(size_t)info.w * V + col] = d[q];
          }
          cs[q] += d[q];
          if constexpr (SP) {
            cm[q] = fmaxf(cm[q], __builtin_fabsf(d[q]));
            l[k][q] = d[q];
          }
        }
        const float ds[4] = {sm.rs[r], sm.rs[r], sm.rs[r], sm.rs[r]};
        store_dl4<SP>(a.dl + (size_t)(m0 + r - cm0) * a.ldd, c, d, ds);
      }
    }
  }
  if constexpr (SP) {
    red[threadIdx.x] = make_float4(cm[0], cm[1], cm[2], cm[3]);
    __syncthreads();
    for (int k = 0; k < nrg; ++k) {
      const float4 o = red[k * tpr + ct];
      cm[0] = fmaxf(cm[0], o.x); cm[1] = fmaxf(cm[1], o.y); cm[2] = fmaxf(cm[2], o.z); cm[3] = fmaxf(cm[3], o.w);
    }
    __syncthreads();  // red is used again below
    const float s[4] = {split_scale(cm[0]), split_scale(cm[1]), split_scale(cm[2]), split_scale(cm[3])};
    if (gok) {
#pragma unroll
      for (int k = 0; k < kDlInFlight; ++k) {
        const int r = rg + k * nrg;
        if (r < nrows) store_dl4<SP>(a.dc + (size_t)(m0 + r - cm0) * a.ldd, c, l[k], s);
      }
      if (rg == 0 && c < ldl) *reinterpret_cast<float4*>(a.dc_inv + (size_t)((m0 - cm0) / kDlRows) * ldl + c) = dc_factors(s);
    }
  }
  if (nrg > 1) {
    red[threadIdx.x] = make_float4(cs[0], cs[1], cs[2], cs[3]);
    __syncthreads();
    if (rg == 0) {
      for (int k = 1; k < nrg; ++k) {
        const float4 o = red[k * tpr + ct];
        cs[0] += o.x; cs[1] += o.y; cs[2] += o.z; cs[3] += o.w;
      }
    }
  }
  if (rg == 0 && gok) {
    float* db = a.db_part + (size_t)((m0 - cm0) / kDlRows) * V;  // the chunk's row; later chunks add
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (c + q < V) db[c + q] = cm0 == 0 ? cs[q] : db[c + q] + cs[q];
  }
}

// ---------------------------------------------------------------------------
// d enc and d dec pieces of one row tile of dpre, formed from the tile in
// LDS so that dpre never goes to HBM. Rows are (frame, slot)
// pairs, S per frame, frames of the batch in order; slot s of frame (n, t)
// is node u = p_t + s.
//   d enc: a frame whose S rows all lie in the tile is summed (ascending s)
//          straight into enc_grad; a frame cut by the tile's first or last
//          row leaves its piece in enc_part[tile][0 (cut at the start) or
//          1], for the tail to add the pieces in tile order.
//   d dec: the rows of one u in the tile (one per frame, slot decreasing as
//          p_t grows) are summed in ascending t into the chunk's row of dpre
//          of the first of them; the chunk's d dec pass adds those pieces of
//          u to d dec in tile order.
// ---------------------------------------------------------------------------
constexpr int kTileFrames = 130;  // frames a 128-row tile can touch (S = 1: 128; plus cut ends)

// Frames [fa, fa + nf) touched by rows [m0, mt_end) of a tile.
DEV void tile_frames(int m0, int mt_end, int S, int& fa, int& nf) {
  fa = m0 / S;
  nf = (mt_end - 1) / S - fa + 1;
}

// Thread k < nf: frame_nt and frame_p of frame fa + k, loaded before the
// main loop so that their latency hides under it.
struct TileFrameRegs {
  int nt, p;
};
DEV TileFrameRegs tile_frames_fetch(const JoinerArgs& a, int m0, int mend, int bm) {
  int fa, nf;
  tile_frames(m0, min(m0 + bm, mend), a.S, fa, nf);
  TileFrameRegs r{0, 0};
  if ((int)threadIdx.x < nf) {
    r.nt = a.frame_nt[fa + threadIdx.x];
    r.p = a.frame_p[fa + threadIdx.x];
  }
  return r;
}

template <class Cfg>
DEV void tile_enc_dec(const JoinerArgs& a, const float* C, int LDC, int cm0, int m0, int mend, int j0,
                      const int4* ri, TileFrameRegs fr) {
  static_assert(Cfg::NT >= kTileFrames && Cfg::NT >= Cfg::BM, "one thread per frame and per row of the tile");
  __shared__ int fr_nt[kTileFrames], fr_n[kTileFrames], fr_p[kTileFrames];
  __shared__ int16_t next_row[Cfg::BM];  // tile row of the next frame's row of the same u, or -1
  __shared__ int16_t first_row[Cfg::BM];  // rows that start a d dec piece (any order)
  __shared__ int n_first;
  const int S = a.S, J = a.J, T = a.b.T;
  const int mt_end = min(m0 + Cfg::BM, mend);  // rows [m0, mt_end) of the tile
  const int rows = mt_end - m0;
  int fa, nf;
  tile_frames(m0, mt_end, S, fa, nf);
  if ((int)threadIdx.x < nf) {
    fr_nt[threadIdx.x] = fr.nt;
    fr_n[threadIdx.x] = fr.nt / T;
    fr_p[threadIdx.x] = fr.p;
  }
  if (threadIdx.x == 0) n_first = 0;
  __syncthreads();
  // one thread per row: is it the first row of its u in the tile (the
  // previous frame's row of u, slot u - p_{t-1}, is absent, of another
  // utterance or before the tile), and which row of the tile comes next
  if ((int)threadIdx.x < rows && ri[threadIdx.x].w >= 0) {
    const int r = threadIdx.x, m = m0 + r, f = m / S, s = m - f * S, k = f - fa;
    const int n = fr_n[k], u = fr_p[k] + s;
    bool first = true;
    if (k > 0 && fr_n[k - 1] == n) {
      const int sp = u - fr_p[k - 1];
      first = !(sp < S && r - s - S + sp >= 0);
    }
    int nx = -1;
    if (k + 1 < nf && fr_n[k + 1] == n) {
      const int s2 = u - fr_p[k + 1], r2 = r - s + S + s2;
      if (s2 >= 0 && r2 < rows) nx = r2;
    }
    next_row[r] = (int16_t)nx;
    if (first) first_row[atomicAdd(&n_first, 1)] = (int16_t)r;
  }
  __syncthreads();
  constexpr int CG = Cfg::BN / 4;  // 4-column groups
  const int tile = m0 / Cfg::BM;
  // d enc
  for (int it = threadIdx.x; it < nf * CG; it += Cfg::NT) {
    const int k = it / CG, cg = it - k * CG, jj = j0 + 4 * cg;
    if (jj >= J) continue;
    const int fs = (fa + k) * S, r0 = max(fs, m0), r1 = min(fs + S, mt_end);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int m = r0; m < r1; ++m) acc = f4add(acc, *reinterpret_cast<const float4*>(C + (m - m0) * LDC + 4 * cg));
    float* dst;
    if (fs >= m0 && fs + S <= mt_end) dst = a.enc_grad + (size_t)fr_nt[k] * J + jj;
    else dst = a.enc_part + ((size_t)tile * 2 + (fs <= m0 ? 0 : 1)) * J + jj;
    *reinterpret_cast<float4*>(dst) = acc;
  }
  // d dec: each piece's rows in ascending t, into the row of its first one
  const int nfirst = n_first;
  for (int it = threadIdx.x; it < nfirst * CG; it += Cfg::NT) {
    const int i = it / CG, cg = it - i * CG, jj = j0 + 4 * cg;
    if (jj >= J) continue;
    const int r = first_row[i];
    float4 acc = *reinterpret_cast<const float4*>(C + r * LDC + 4 * cg);
    for (int r2 = next_row[r]; r2 >= 0; r2 = next_row[r2])
      acc = f4add(acc, *reinterpret_cast<const float4*>(C + r2 * LDC + 4 * cg));
    *reinterpret_cast<float4*>(a.dpre + (size_t)(m0 - cm0 + r) * J + jj) = acc;  // the chunk's row
  }
}

// ---------------------------------------------------------------------------
// Backward 2: dh = dl W^T, dpre = dh (1 - h^2), summed into the d enc / d dec
// pieces in LDS.
// ---------------------------------------------------------------------------
template <bool SP>
DEV void dh_tile(const JoinerArgs& a, int cm0, int cm1, int v, int nblocks, int ncol, unsigned char* lds) {
  using Cfg = CfgN<SP>;
  int4* ri = lds_rowinfo(lds);
  const int M = a.frame_off[a.b.N] * a.S;
  const int mend = min(cm1, M);
  const int tile = part_tile(v, nblocks, chunk_row_tiles(a, cm0, cm1) * ncol);
  if (tile < 0) return;
  const int mt = tile / ncol, nt = tile - mt * ncol;
  const int m0 = cm0 + mt * Cfg::BM;
  const int j0 = nt * Cfg::BN;
  const int J = a.J;
  float* rinv = lds_rowinv(lds);
  for (int r = threadIdx.x; r < Cfg::BM; r += Cfg::NT) {
    ri[r] = (m0 + r < mend) ? a.rowinfo[m0 + r] : make_int4(0, 0, -1, -1);
    if constexpr (SP) rinv[r] = (m0 + r < mend) ? pow2_inv(a.rsc[m0 + r]) : 0.f;
  }
  __syncthreads();
  const TileFrameRegs fr = tile_frames_fetch(a, m0, mend, Cfg::BM);
  // What the epilogue needs of this thread's 4-column groups of the tile for
  // h: bf16: enc and dec (h = tanh(enc + dec), unrounded), ahead of the main
  // loop; split: the planes of h, after it (whose registers they would take),
  // all issued together and waited for once.
  constexpr int NIT = Cfg::BM * Cfg::BN / 4 / Cfg::NT;  // 4-column groups per thread
  static_assert(Cfg::BM * Cfg::BN / 4 % Cfg::NT == 0, "whole groups per thread");
  RawVec<uint16_t, 4> pe[NIT], pd[NIT];
  auto fetch_h = [&]() {
    const EncDec<uint16_t> ed(a);
    const Rsrc rh = make_rsrc(a.hbuf + (size_t)(m0 - cm0) * a.ldh, (size_t)min(Cfg::BM, mend - m0) * a.ldh * 2);
#pragma unroll
    for (int q8 = 0; q8 < NIT; ++q8) {
      const int it = threadIdx.x + q8 * Cfg::NT;
      const int row = it / (Cfg::BN / 4), jj = j0 + (it - row * (Cfg::BN / 4)) * 4;
      const int4 info = ri[row];  // absent (w < 0) for rows past mend
      const bool on = info.w >= 0 && jj < J;  // J is a multiple of 8: a group is all in or out
      if constexpr (SP) {
        const uint32_t o = (uint32_t)(row * a.ldh + split_word(jj)) * 2;
        raw_load(rh, o, on, pe[q8]);
        raw_load(rh, o + 64, on, pd[q8]);
      } else {
        raw_load(ed.enc, (uint32_t)(info.x + jj) * 2, on, pe[q8]);
        raw_load(ed.dec, (uint32_t)(info.y + jj) * 2, on, pd[q8]);
      }
    }
  };
  if constexpr (!SP) fetch_h();
  floatx4 acc[Cfg::FM][Cfg::FN];
  // d(logits) of the chunk and W, both k = v contiguous
  const LdsSrc sa(a.dl + (size_t)(m0 - cm0) * a.ldd, min(Cfg::BM, mend - m0), a.ldd);
  const LdsSrc sb(a.wn + (size_t)j0 * a.ldd, min(Cfg::BN, J - j0), a.ldd);
  gemm_mainloop_lds<Cfg>(sa, sb, lds, acc);
  if constexpr (SP) fetch_h();
  float4 sj[SP ? Cfg::FN : 1];  // the factors that undo the scales, per column j
  if constexpr (SP) {
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      const int jj = j0 + out_col<Cfg>(j);
      sj[j] = jj < J ? *reinterpret_cast<const float4*>(a.wn_inv + jj) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  wait_vmem();

  // Epilogue through LDS (the operand stages are free after the main loop's
  // last barrier): the tile goes to LDS in the MFMA layout and comes back row
  // by row, 16-byte accesses both ways.
  constexpr int LDC = kDpreLd;
  float* C = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const float dinv = SP ? rinv[out_row<Cfg>(i)] : 1.f;
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      float4 o = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
      if constexpr (SP) {
        o.x *= sj[j].x * dinv;
        o.y *= sj[j].y * dinv;
        o.z *= sj[j].z * dinv;
        o.w *= sj[j].w * dinv;
      }
      *reinterpret_cast<float4*>(C + out_row<Cfg>(i) * LDC + out_col<Cfg>(j)) = o;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q8 = 0; q8 < NIT; ++q8) {
    const int it = threadIdx.x + q8 * Cfg::NT;
    const int row = it / (Cfg::BN / 4), cg = it - row * (Cfg::BN / 4);
    if (j0 + cg * 4 >= J) continue;  // J is a multiple of 8: the group is all in or all out
    float4* cr = reinterpret_cast<float4*>(C + row * LDC + cg * 4);
    const bool on = ri[row].w >= 0;  // absent (w < 0) for rows past mend
    float h[4], dp[4];
    if constexpr (SP) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint16_t hi = (uint16_t)(pe[q8].w[q >> 1] >> (16 * (q & 1))), lo = (uint16_t)(pd[q8].w[q >> 1] >> (16 * (q & 1)));
        h[q] = ((float)__builtin_bit_cast(_Float16, hi) + (float)__builtin_bit_cast(_Float16, lo)) * kHInv;
      }
    } else {
      float fe[4], fd[4];
      raw_to_float(pe[q8], fe);
      raw_to_float(pd[q8], fd);
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = on ? fast_tanh(fe[q] + fd[q]) : 0.f;
    }
    const float4 c = *cr;
    dp[0] = c.x; dp[1] = c.y; dp[2] = c.z; dp[3] = c.w;
#pragma unroll
    for (int q = 0; q < 4; ++q) dp[q] = on ? dp[q] * (1.f - h[q] * h[q]) : 0.f;
    *cr = make_float4(dp[0], dp[1], dp[2], dp[3]);  // dpre stays in the tile for the d enc / d dec pieces
  }
  __syncthreads();
  tile_enc_dec<Cfg>(a, C, LDC, cm0, m0, mend, j0, ri, fr);
}

// ---------------------------------------------------------------------------
// Backward 3: dW partial += h^T dl over one split of the chunk's rows (the
// first chunk writes the partials, later chunks add to them). Tiles: the
// (j, v) tiles of one split are consecutive tile ids, so one XCD reads that
// split's rows. Both operands are the chunk's rows as the other contractions
// read them (gemm_mainloop_tr transposes on the way out of LDS).
// ---------------------------------------------------------------------------
template <bool SP>
DEV void dw_tile(const JoinerArgs& a, int cm0, int cm1, int first, int v, int nj, int nv, unsigned char* lds) {
  using Cfg = CfgT<SP>;
  const int M = a.frame_off[a.b.N] * a.S;
  const int mend = min(cm1, M);
  const int per_split = nj * nv;
  const int tile = part_tile(v, per_split * a.splits, per_split * a.splits);
  const int z = tile / per_split, jv = tile - z * per_split;
  const int jt = jv / nv, vt = jv - jt * nv;
  const int j0 = jt * Cfg::BM, v0 = vt * Cfg::BN;
  const int rows = cm1 - cm0;
  const int per = ((rows + a.splits - 1) / a.splits + Cfg::BK - 1) / Cfg::BK * Cfg::BK;
  const int kb = cm0 + z * per;
  const int ke = min(kb + per, mend);
  const int V = a.V, J = a.J;
  float* part = a.dw_part + (size_t)z * J * V;
  if (kb >= ke) {
    // no rows for this split: the first chunk still defines the partial
    if (first) {
      for (int e = threadIdx.x; e < Cfg::BM * Cfg::BN; e += Cfg::NT) {
        const int j = j0 + e / Cfg::BN, vv = v0 + e % Cfg::BN;
        if (j < J && vv < V) part[(size_t)j * V + vv] = 0.f;
      }
    }
    return;
  }
  floatx4 acc[Cfg::FM][Cfg::FN];
  const int krows = __builtin_amdgcn_readfirstlane(ke - kb);
  const TrSrc sa{reinterpret_cast<const unsigned char*>(a.hbuf + (size_t)(kb - cm0) * a.ldh), krows, a.ldh, j0 * Cfg::XP};
  const TrSrc sb{reinterpret_cast<const unsigned char*>((SP ? a.dc : a.dl) + (size_t)(kb - cm0) * a.ldd), krows, a.ldd,
                 v0 * Cfg::XP};
  static_assert(!SP || Cfg::BK == kDbRows, "a K-step's rows share dc's scales");
  const TrFactors sf{SP ? a.dc_inv + (size_t)((kb - cm0) / kDbRows) * a.ldl : nullptr, a.ldl, v0};
  gemm_mainloop_tr<Cfg>(sa, sb, sf, lds, acc);
  const bool vec = (V & 3) == 0;  // rows of partials at 16-byte offsets
  // the partials the earlier chunks left for this thread's elements, loaded
  // together before any store rather than one load-add-store round trip per
  // element
  float old[Cfg::FM][Cfg::FN][4];
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int jj = 0; jj < Cfg::FN; ++jj) {
      const int j = j0 + out_row<Cfg>(i), vv = v0 + out_col<Cfg>(jj);
      const float* src = part + (size_t)j * V + vv;
      if (vec) {
        const float4 q = !first && j < J && vv < V ? *reinterpret_cast<const float4*>(src) : make_float4(0.f, 0.f, 0.f, 0.f);
        old[i][jj][0] = q.x; old[i][jj][1] = q.y; old[i][jj][2] = q.z; old[i][jj][3] = q.w;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) old[i][jj][r] = !first && j < J && vv + r < V ? src[r] : 0.f;
      }
    }
  wait_vmem();
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int j = j0 + out_row<Cfg>(i);
    if (j >= J) continue;
#pragma unroll
    for (int jj = 0; jj < Cfg::FN; ++jj) {
      const int vv = v0 + out_col<Cfg>(jj);
      float* dst = part + (size_t)j * V + vv;
      float o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        o[r] = first ? acc[i][jj][r] : old[i][jj][r] + acc[i][jj][r];
      }
      if (vec) {
        if (vv < V) *reinterpret_cast<float4*>(dst) = make_float4(o[0], o[1], o[2], o[3]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (vv + r < V) dst[r] = o[r];
      }
    }
  }
}

// The tail of the backward: dW and db summed from their partials, d enc and
// d dec from their pieces. Four independent, latency-bound reductions, run as
// one launch whose block ranges take one part each (d dec, d enc, dW, db), so
// that their memory latencies overlap.
constexpr int kTailThreads = 256;

// dW = sum of the split partials, in split order: four consecutive elements
// per thread (16-byte loads, 16 partials in flight) where J*V and dW's
// address allow, else one.
constexpr int kWsumVec = 4;

DEV bool tail_wsum_vec(const JoinerArgs& a) {
  return (((size_t)a.J * a.V) % kWsumVec) == 0 && (reinterpret_cast<uintptr_t>(a.W_grad) & 15) == 0;
}

DEV void tail_wsum(const JoinerArgs& a, int b) {
  const size_t JV = (size_t)a.J * a.V;
  const size_t i = (size_t)b * kTailThreads + threadIdx.x;
  if (tail_wsum_vec(a)) {
    if (i * kWsumVec >= JV) return;
    const float4* src = reinterpret_cast<const float4*>(a.dw_part) + i;
    const size_t stride = JV / kWsumVec;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 16
    for (int z = 0; z < a.splits; ++z) {
      const float4 v = src[(size_t)z * stride];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    reinterpret_cast<float4*>(a.W_grad)[i] = s;
    return;
  }
  if (i >= JV) return;
  float s = 0.f;
#pragma unroll 8
  for (int z = 0; z < a.splits; ++z) s += a.dw_part[(size_t)z * JV + i];
  a.W_grad[i] = s;
}

// db = sum of the column partials written by the d(logits) kernel (one per
// 32 rows of a chunk streamed, one per wave row of a GEMM tile recomputed,
// each summed over the chunks): a block takes 16 columns; each of its 16
// thread groups sums a contiguous sixteenth of the rows in ascending order,
// 8 loads in flight, then the sixteenths are added in order.
constexpr int kDbCols = 16;

DEV void tail_dbsum(const JoinerArgs& a, int b, float (*red)[kDbCols]) {
  const int c = threadIdx.x % kDbCols, part = threadIdx.x / kDbCols;  // 16 parts
  constexpr int kParts = kTailThreads / kDbCols;
  const int v = b * kDbCols + c;
  const int M = min(a.frame_off[a.b.N] * a.S, a.chunk_rows);  // rows of the first (largest) chunk
  // the rows the first chunk wrote: one per 32 rows streamed (stored logits
  // or the head), one per wave row of each recomputed tile (the same 32-row
  // groups, whole tiles); a later chunk only adds to a prefix of them
  const bool streamed = a.logits_in || (a.head && a.head_rows == a.chunk_rows);
  const int rows = streamed ? (M + kDlRows - 1) / kDlRows : (M + kTileRows - 1) / kTileRows * (kTileRows / kDbRows);
  const int q = (rows + kParts - 1) / kParts, r0 = min(rows, part * q), r1 = min(rows, r0 + q);
  float s = 0.f;
  if (v < a.V) {
    const float* col = a.db_part + v;
    for (int r = r0; r < r1; r += 8) {
      float x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = (r + k < r1) ? col[(size_t)(r + k) * a.V] : 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s += x[k];
    }
  }
  red[part][c] = s;
  __syncthreads();
  if (part == 0 && v < a.V) {
    float t = red[0][c];
    for (int k = 1; k < kParts; ++k) t += red[k][c];
    a.bias_grad[v] = t;
  }
}

// d enc rows per block: threads over float4 column groups of J.
DEV int encdec_rows_per_block(int J) {
  const int tpr = J / 4;
  return tpr >= kTailThreads ? 1 : kTailThreads / tpr;
}


// d enc and d dec from the pieces the dh kernel left (see tile_enc_dec).
// d enc: frames cut by a row tile add their pieces in tile order (the others
// are already written); zero rows past T_n.
DEV void tail_enc_pieces(const JoinerArgs& a, int b) {
  const int T = a.b.T, S = a.S, J = a.J, tpr = J / 4;
  const int R = encdec_rows_per_block(J);
  const int rr = threadIdx.x / tpr, c = threadIdx.x - rr * tpr;
  const int row = b * R + rr;  // n * T + t
  if (rr >= R || row >= a.b.N * T) return;
  const int n = row / T, t = row - n * T;
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  float4* out = reinterpret_cast<float4*>(a.enc_grad + (size_t)row * J);
  if (t >= Tn) {
    for (int g = c; g < tpr; g += kTailThreads) out[g] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const int fs = (a.frame_off[n] + t) * S, ia = fs / kTileRows, ib = (fs + S - 1) / kTileRows;
  if (ia == ib) return;  // the frame lies in one tile: written by the dh kernel
  for (int g = c; g < tpr; g += kTailThreads) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = ia; i <= ib; ++i)
      acc = f4add(acc, reinterpret_cast<const float4*>(a.enc_part + ((size_t)i * 2 + (fs <= i * kTileRows ? 0 : 1)) * J)[g]);
    out[g] = acc;
  }
}

// d dec[n, u] from the pieces of u in one chunk of rows [cm0, cm1): one
// piece per row tile that holds rows of u, each in the chunk's row of dpre
// of its first row (ascending t). The row of u in frame t,
// m_t = (frame_off[n] + t) S + u - p_t, grows with t (p_{t+1} - p_t < S
// while u stays in the band), so the chunk's frames of u and the first frame
// of each tile are found by binary searches; the pieces are loaded 8 at a
// time and added in tile order, onto d dec as the earlier chunks left it
// (0 in the chunk that holds the first row of u), so that the sum's order is
// that of one pass over all tiles. The first chunk also writes the zero rows
// (u > U_n, or u in no frame's band).
// u rows of one utterance per d dec block: the block loads the utterance's
// band starts once and its row groups (J / 4 threads each) take the rows.
// Four rows are one pass of the GEMM launch's 512-thread blocks at J = 512;
// longer groups serialise the latency-bound searches of several passes in
// one block and measured slower (16 rows: +5% per step at BPE, +7% long).
constexpr int kDecGroup = 4;
__host__ __device__ inline int dec_blocks(int N, int U1) { return N * ((U1 + kDecGroup - 1) / kDecGroup); }

DEV void tail_dec_pieces(const JoinerArgs& a, int b, int* sp, int cm0, int cm1, const float* dpre) {
  const int nt = blockDim.x;
  const int T = a.b.T, U1 = a.b.U + 1, S = a.S, J = a.J, tpr = J / 4;
  const int ng = (U1 + kDecGroup - 1) / kDecGroup;
  const int n = b / ng, u0 = (b - n * ng) * kDecGroup, u1 = min(U1, u0 + kDecGroup);
  int Tn, Un;
  utt_dims(a.b, n, Tn, Un);
  // row groups: tpr threads per u row (all threads, looping, when a row is wider)
  const int rgw = tpr < nt ? tpr : nt, nrg = nt / rgw;
  const int rg = threadIdx.x / rgw, ct = threadIdx.x - rg * rgw;
  auto zero_row = [&](int u) {
    float4* out = reinterpret_cast<float4*>(a.dec_grad + ((size_t)n * U1 + u) * J);
    for (int g = ct; g < tpr; g += rgw) out[g] = make_float4(0.f, 0.f, 0.f, 0.f);
  };
  // No row of utterance n in the chunk (most blocks: an utterance spans one
  // or two chunks): the first chunk zeroes the rows, which the chunk holding
  // the first row of each u overwrites; later chunks have nothing to add.
  const int off = a.frame_off[n];
  if (u0 > Un || (size_t)a.frame_off[n + 1] * S <= (size_t)cm0 || (size_t)off * S >= (size_t)cm1) {
    if (cm0 == 0 && rg < nrg)
      for (int u = u0 + rg; u < u1; u += nrg) zero_row(u);
    return;
  }
  for (int t = threadIdx.x; t < Tn; t += nt) sp[t] = a.ranges[((size_t)n * T + t) * S];
  __syncthreads();
  if (rg >= nrg) return;
  const int mend = min(cm1, a.frame_off[a.b.N] * S);
  const int rows = __builtin_amdgcn_readfirstlane(a.chunk_rows);  // keeps the resource scalar
  const Rsrc dr = make_rsrc(dpre, (size_t)rows * J * sizeof(float));
  for (int u = u0 + rg; u < u1; u += nrg) {
    if (u > Un) {
      if (cm0 == 0) zero_row(u);
      continue;
    }
    // frames [t0, t1) whose band holds u
    int lo = 0, hi = Tn;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sp[mid] > u - S) hi = mid;
      else lo = mid + 1;
    }
    const int t0 = lo;
    hi = Tn;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sp[mid] > u) hi = mid;
      else lo = mid + 1;
    }
    const int t1 = lo;
    auto row_of = [&](int t) { return (off + t) * S + u - sp[t]; };
    // the first frame in [l, h] whose row of u is at least r (h + 1: none)
    auto first_at = [&](int l, int h, int r) {
      int e = h + 1;
      while (l < e) {
        const int mid = (l + e) >> 1;
        if (row_of(mid) >= r) e = mid;
        else l = mid + 1;
      }
      return l;
    };
    if (t1 <= t0) {
      if (cm0 == 0) zero_row(u);
      continue;
    }
    const int ta = first_at(t0, t1 - 1, cm0), tb = first_at(ta, t1 - 1, mend);  // frames of u in the chunk
    if (ta >= tb) continue;
    const bool starts = row_of(t0) >= cm0;  // the chunk holds the first row of u
    const int ia = row_of(ta) / kTileRows, ib = row_of(tb - 1) / kTileRows;
    float4* out = reinterpret_cast<float4*>(a.dec_grad + ((size_t)n * U1 + u) * J);
    for (int g = ct; g < tpr; g += rgw) {
      float4 acc = starts ? make_float4(0.f, 0.f, 0.f, 0.f) : out[g];
      for (int i0 = ia; i0 <= ib; i0 += 8) {
        float4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int i = i0 + k;
          const int t = (i > ia && i <= ib) ? first_at(ta, tb - 1, i * kTileRows) : ta;  // first frame of u in tile i
          const uint32_t o = (uint32_t)(((size_t)(row_of(t) - cm0) * J + 4 * g) * sizeof(float));
          const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(dr, (int)(i <= ib ? o : kOob), 0, 0);
          v[k] = make_float4(__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w));
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) acc = f4add(acc, v[k]);
      }
      out[g] = acc;
    }
  }
}

struct TailRanges {
  int dec, enc, wsum, dbsum;  // block counts, in launch order
  int cm0, cm1;               // the chunk whose d dec pieces the dec blocks add
  HPass h0, h1;               // h passes of later chunks (recomputed path), run after them
};

// One launch per chunk of rows: its d dec pieces and the h passes of later
// chunks; the last chunk's launch also runs the d enc, dW and db reductions.
template <bool SP>
__global__ __launch_bounds__(kTailThreads) void joiner_tail_kernel(JoinerArgs a, TailRanges r) {
  extern __shared__ int sp[];  // p_t of one utterance (d dec blocks)
  __shared__ float red[kTailThreads / kDbCols][kDbCols];  // db blocks
  int b = blockIdx.x;
  if (b < r.dec) { tail_dec_pieces(a, b, sp, r.cm0, r.cm1, a.dpre); return; }
  b -= r.dec;
  if (b < r.enc) { tail_enc_pieces(a, b); return; }
  b -= r.enc;
  if (b < r.wsum) { tail_wsum(a, b); return; }
  b -= r.wsum;
  if (b < r.dbsum) { tail_dbsum(a, b, red); return; }
  b -= r.dbsum;
  const HPass& hp = b < r.h0.blocks ? r.h0 : r.h1;
  if (b >= r.h0.blocks) b -= r.h0.blocks;
  h_rows_block<SP, kTailThreads>(a, hp.h, hp.cm0, hp.cm1, b);
}

// d(logits) of a chunk streamed from stored logits or the head (the first
// dlx * dly blocks) and h passes (the rest) as block kinds of one launch.
// Both are memory-bound and independent, so that they run side by side
// instead of one after the other.
template <bool SP>
__global__ __launch_bounds__(kTailThreads) void joiner_head_kernel(JoinerArgs a, HPass h0, HPass h1, int cm0, int cm1,
                                                                   int dlx, int dly) {
  __shared__ DlSmem dsm;
  static_assert(kTailThreads == kDlThreads, "one block size for both kinds");
  int b = blockIdx.x;
  if (b < dlx * dly) {
    dl_block<SP>(a, cm0, cm1, b % dlx, b / dlx, dsm);
    return;
  }
  b -= dlx * dly;
  const HPass& hp = b < h0.blocks ? h0 : h1;
  if (b >= h0.blocks) b -= h0.blocks;
  h_rows_block<SP, kTailThreads>(a, hp.h, hp.cm0, hp.cm1, b);
}

// The backward's GEMM kernel. Every block kind runs in one kernel, each on
// its own range of blocks, so that the recomputed logits of the next chunk
// (L), dh of the current chunk (D) and its dW (W) share a launch (a chunk's
// dh alone puts only one workgroup on each CU), and so that the memory- and
// latency-bound passes of the pipeline run in the slots the GEMM tiles leave
// free at the end of the launch instead of as launches of their own: the h
// pass of a later chunk (H) and the d dec pass of the previous chunk (E).
struct BwdParts {
  int nL, nLcol;   // blocks and column tiles of L (chunk [lm0, lm1) of `nxt`)
  int nD, nDcol;   // blocks and column tiles of D (chunk [cm0, cm1) of `cur`)
  int nW, nWj, nWv;  // blocks and (j, v) tiles per split of W (same chunk)
  int lm0, lm1, cm0, cm1, first;
  int d_first;     // D's tiles (K = V) are longer than W's (K = a split's rows): dispatched before them
  HPass h;         // H
  int nE;          // blocks of E: one per (n, u) row of d dec, adding the pieces of chunk [ecm0, ecm1) in edpre
  int ecm0, ecm1;
  const float* edpre;
};

// Blocks in the order E, then W and D (the kind with the longer K loop
// first), L, H: the d dec blocks first (short and latency-bound; dispatched
// last they would run after the GEMM tiles and lengthen the launch's tail),
// then the longest GEMM tiles, so that the shorter ones fill in around them.
template <bool SP>
__global__ __launch_bounds__(kGemmThreads, 4) void joiner_bwd_gemm_kernel(JoinerArgs cur, JoinerArgs nxt, BwdParts p) {
  __shared__ __align__(16) unsigned char lds[kBwdLdsBytes];
  int b = blockIdx.x;
  if (b < p.nE) {
    static_assert(kBwdLdsBytes >= 16384 * (int)sizeof(int), "p_t of one utterance (T <= 16384) in LDS");
    tail_dec_pieces(cur, b, reinterpret_cast<int*>(lds), p.ecm0, p.ecm1, p.edpre);
    return;
  }
  b -= p.nE;
  if (b < p.nW + p.nD) {
    const int bd = p.d_first ? b : b - p.nW;  // index among the D blocks (negative: a W block)
    if (bd >= 0 && bd < p.nD) dh_tile<SP>(cur, p.cm0, p.cm1, bd, p.nD, p.nDcol, lds);
    else dw_tile<SP>(cur, p.cm0, p.cm1, p.first, p.d_first ? b - p.nD : b, p.nWj, p.nWv, lds);
    return;
  }
  b -= p.nW + p.nD;
  if (b < p.nL) {
    dlogits_tile<SP>(nxt, p.lm0, p.lm1, b, p.nL, p.nLcol, lds);
    return;
  }
  b -= p.nL;
  if (b < p.h.blocks) h_rows_block<SP, kGemmThreads>(cur, p.h.h, p.h.cm0, p.h.cm1, b);
}

// ranges[n,t,s] = s: every (t, u) of the lattice as a "band" of width U+1.
__global__ __launch_bounds__(256) void full_ranges_kernel(int* ranges, size_t total, int S) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) ranges[i] = (int)(i % (size_t)S);
}

}  // namespace

hipError_t launch_full_ranges(int* ranges, int N, int T, int S, hipStream_t s) {
  const size_t total = (size_t)N * T * S;
  {
    RNNT_PROF(s, "full_ranges");
    hipLaunchKernelGGL(full_ranges_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, ranges, total, S);
  }
  return hipGetLastError();
}

int joiner_nparts(int V) { return (V + 63) / 64; }
int joiner_ldl(int V) { return (V + 7) / 8 * 8; }
int joiner_words(int n, int bf16) { return bf16 ? row_words<false>(n) : row_words<true>(n); }
bool joiner_w_copy(int V, int bf16) { return !bf16 || V % 64 != 0; }

// Rows of a chunk buffer whose rows of `row_elems` fp32 words stay below
// 2^31 bytes (offsets within a tile are 32-bit), as a multiple of the
// 128-row tile; 0 when not even one tile fits.
static long long joiner_rsrc_rows(long long row_elems) {
  return ((0x7fffffffll / (row_elems * 4)) / 128) * 128;
}

int joiner_bwd_chunk_max_rows(int J, int V) {
  const long long w = (long long)(J > joiner_ldl(V) ? J : joiner_ldl(V));
  const long long r = joiner_rsrc_rows(w);
  return (int)(r < (1ll << 30) ? r : (1ll << 30));
}

// The padded row count mmax in chunks of at most `cap` rows, split evenly
// (so that no chunk is left nearly empty), as a multiple of the 128-row tile.
static long long even_chunk(long long mmax, long long cap) {
  const long long n = (mmax + cap - 1) / cap;
  return ((mmax + n - 1) / n + 127) / 128 * 128;
}

// The backward's chunk: d(logits) of about 16 MiB, but 8,192 to 16,384 rows
// (64 to 128 row tiles, so that each launch of the pipelined backward puts
// one or two workgroups of every kind on each CU), within the 32-bit limit.
// The head the forward keeps is one chunk: the bound keeps it well below the
// whole [N, T, S, V] logits at the benchmark shapes (a 32 MiB bound would
// hold every row of the BPE batch in it).
// The bound depends on J, V and the dtype only, not on N or T. Chunks are
// taken whole from the start of the padded rows: rows past the last frame of
// the batch (padding frames take none) are absent, so a trailing chunk that
// holds only those costs a few empty launches, while splitting the present
// rows evenly would leave both chunks under-filled. `request` (a multiple of
// 128, or 0) overrides the size.
int joiner_bwd_chunk_rows(int N, int T, int S, int J, int V, int bf16, int request) {
  const long long mmax = (long long)N * T * S;
  const long long all = (mmax + 127) / 128 * 128;
  if (request > 0) return (int)(request < all ? request : all);
  const long long bytes_per_row = (long long)joiner_ldl(V) * (bf16 ? 2 : 4);
  long long cap = ((16ll << 20) / bytes_per_row) / 128 * 128;
  cap = cap < 8192 ? 8192 : cap > 16384 ? 16384 : cap;
  const long long lim = joiner_bwd_chunk_max_rows(J, V);
  if (cap > lim) cap = lim;
  return (int)(cap < all ? cap : all);
}

int joiner_fwd_chunk_rows(int N, int T, int S, int J, int bf16) {
  const long long mmax = (long long)N * T * S;
  // h of one chunk: at most 32,768 rows (48 MiB at J = 768 in bf16), half of that split
  long long cap = bf16 ? 32768 : 16384;
  const long long lim = joiner_rsrc_rows(J);
  if (cap > lim) cap = lim;
  return (int)even_chunk(mmax, cap);
}

// dW splits a chunk's rows into ranges so that one of its tiles takes about
// 1.5 times the K-steps that a CU's slot (two workgroups) gets of the launch's
// dh and dW tiles together: with fewer splits a few long dW tiles outlast the
// launch (a K-step takes 0.8 us on an otherwise idle CU: at J = 512, V = 2000
// in bf16 one split's 128 steps were the whole 104 us of a launch, and three
// splits took the step from 857 to 620 us), with more each writes and re-reads
// another [J, V] of partials (the long step: 626 us with 8 splits, 631 with
// 11, 636 with 16, 648 with 24). At least 8 steps a tile.
int joiner_bwd_splits(int J, int V, int chunk_rows, int bf16) {
  auto tiles = [](long long n, int t) { return (n + t - 1) / t; };
  const long long dh = tiles(chunk_rows, kTileRows) * tiles(J, kTileCols) * (joiner_words(V, bf16) / 64);
  const long long steps = tiles(chunk_rows, bf16 ? CfgT<false>::BK : CfgT<true>::BK);  // of one unsplit dW tile
  const long long dw = tiles(J, kTileRows) * tiles(V, kTileCols) * steps;
  const long long want = std::max<long long>(8, (dh + dw) * 3 / (2 * kSlots));
  const long long s = (steps + want / 2) / want;
  return (int)std::min<long long>(std::max<long long>(s, 1), 32);
}

int joiner_db_rows(int chunk_rows) { return (chunk_rows + kTileRows - 1) / kTileRows * (kTileRows / kDbRows); }

// Whether the forward's first h pass runs in the prep kernel's blocks: these
// cover every padded row, so it does while the first chunk is at least a
// quarter of them (a launch less: step at N = 32, T = 500 643 -> 633 us, three
// chunks); beyond, most would have no rows of it, and their number times J / 64
// would pass what a launch can hold.
constexpr int kPrepHChunks = 4;
static bool fwd_h_in_prep(const JoinerArgs& a) {
  return (long long)a.b.N * a.b.T * a.S <= (long long)kPrepHChunks * a.chunk_rows;
}
static hipError_t launch_tail(const JoinerArgs& a, const TailRanges& tr, hipStream_t s, const char* name);

hipError_t launch_joiner_prep(const JoinerArgs& a, hipStream_t s) {
  {
    RNNT_PROF(s, "joiner_prep");
    PrepBlocks pb{};
    if (a.bf16) {
      if (a.wt) pb.wt = ((a.J + kWtTile - 1) / kWtTile) * ((a.V + kWtTile - 1) / kWtTile);
      if (a.wn && a.wn != a.W) pb.wn = (a.J * (a.ldd / 8) + kPrepThreads - 1) / kPrepThreads;
    } else {
      if (a.wt) pb.wt = (a.V + kWtCols - 1) / kWtCols;
      if (a.wn) pb.wn = a.J;
    }
    if (a.px && fwd_h_in_prep(a)) {
      pb.hj = ((a.bf16 ? h_groups<false>(a.J) : h_groups<true>(a.J)) + kPrepHGroups - 1) / kPrepHGroups;
      pb.hrows = a.chunk_rows;
    }
    const dim3 grid(a.b.N * ((a.b.T * a.S + 255) / 256) * std::max(1, pb.hj) + pb.wt + pb.wn);
    if (a.bf16) hipLaunchKernelGGL(joiner_prep_kernel<false>, grid, dim3(kPrepThreads), 0, s, a, pb);
    else hipLaunchKernelGGL(joiner_prep_kernel<true>, grid, dim3(kPrepThreads), 0, s, a, pb);
  }
  return hipGetLastError();
}

hipError_t launch_joiner_fwd(const JoinerArgs& a, hipStream_t s) {
  const int mmax = a.b.N * a.b.T * a.S;
  const int C = a.chunk_rows;
  const int nch = (mmax + C - 1) / C;
  auto lo = [&](int k) { return k * C; };
  auto hi = [&](int k) { return (k + 1) * C < mmax ? (k + 1) * C : mmax; };
  // h of chunk k in slot k % 2; chunk 0's was written by the prep kernel (or is
  // by a launch of its own), that of chunk k + 1 comes from the trailing blocks of chunk k's GEMM launch
  // (they write the slot chunk k - 1's launch read)
  auto slot = [&](int k) {
    JoinerArgs c = a;
    c.hbuf = a.hring[k % 2];
    return c;
  };
  // offsets within a 256-row tile stay below 2^31 (ldh words of 2 bytes a row)
  const bool wide = a.V >= kFwdWideV && a.ldh <= (1 << 20);
  const int bm = wide ? CfgWide<false>::BM : kTileRows, bn = wide ? CfgWide<false>::BN : kTileCols;
  const int nt = wide ? CfgWide<false>::NT : kGemmThreads;
  if (!fwd_h_in_prep(a)) {
    TailRanges tr{};
    tr.h0 = h_pass(slot(0), lo(0), hi(0), kTailThreads);
    const hipError_t e = launch_tail(a, tr, s, "joiner_h");
    if (e != hipSuccess) return e;
  }
  for (int k = 0; k < nch; ++k) {
    const int cm0 = lo(k), cm1 = hi(k);
    const JoinerArgs c = slot(k);
    HPass hn{};
    if (k + 1 < nch) hn = h_pass(slot(k + 1), lo(k + 1), hi(k + 1), nt);
    const int ncol = (a.V + bn - 1) / bn;
    const int ngemm = (cm1 - cm0 + bm - 1) / bm * ncol;
    const dim3 grid((unsigned)(ngemm + hn.blocks));
    RNNT_PROF(s, "joiner_fwd");
    if (a.bf16) {
      if (wide) hipLaunchKernelGGL((joiner_fwd_kernel<false, true>), grid, dim3(nt), 0, s, c, cm0, cm1, ncol, ngemm, hn);
      else hipLaunchKernelGGL((joiner_fwd_kernel<false, false>), grid, dim3(nt), 0, s, c, cm0, cm1, ncol, ngemm, hn);
    } else {
      if (wide) hipLaunchKernelGGL((joiner_fwd_kernel<true, true>), grid, dim3(nt), 0, s, c, cm0, cm1, ncol, ngemm, hn);
      else hipLaunchKernelGGL((joiner_fwd_kernel<true, false>), grid, dim3(nt), 0, s, c, cm0, cm1, ncol, ngemm, hn);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const size_t total = (size_t)a.b.N * a.b.T * a.S;
  {
    RNNT_PROF(s, "joiner_combine");
    if (a.nparts > kCombineSerialParts)
      hipLaunchKernelGGL(joiner_combine_wide_kernel, dim3((unsigned)((total + 3) / 4)), dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL(joiner_combine_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// Joiner args of chunk k's buffers in the recomputed path's rings: h in slot
// k % 3, d(logits) and the d dec pieces in slot k % 2.
static JoinerArgs ring_slot(const JoinerArgs& a, int k) {
  JoinerArgs c = a;
  c.hbuf = a.hring[k % 3];
  c.dl = a.dlring[k % 2];
  c.dc = a.dcring[k % 2];
  c.dc_inv = a.dcinvring[k % 2];
  c.dpre = a.dpring[k % 2];
  return c;
}

static TailRanges tail_ranges(const JoinerArgs& a, int cm0, int cm1, bool last) {
  const size_t JV = (size_t)a.J * a.V;
  const int R = (a.J / 4 >= kTailThreads) ? 1 : kTailThreads / (a.J / 4);
  TailRanges tr{};
  tr.cm0 = cm0;
  tr.cm1 = cm1;
  tr.dec = (cm1 > cm0) ? dec_blocks(a.b.N, a.b.U + 1) : 0;
  tr.enc = last ? (a.b.N * a.b.T + R - 1) / R : 0;
  const bool wvec = JV % kWsumVec == 0 && (reinterpret_cast<uintptr_t>(a.W_grad) & 15) == 0;
  const size_t wthreads = wvec ? JV / kWsumVec : JV;
  tr.wsum = (last && a.W_grad) ? (int)((wthreads + kTailThreads - 1) / kTailThreads) : 0;
  tr.dbsum = (last && a.bias_grad) ? (a.V + kDbCols - 1) / kDbCols : 0;
  return tr;
}

static hipError_t launch_tail(const JoinerArgs& a, const TailRanges& tr, hipStream_t s, const char* name) {
  const int blocks = tr.dec + tr.enc + tr.wsum + tr.dbsum + tr.h0.blocks + tr.h1.blocks;
  if (blocks == 0) return hipSuccess;
  RNNT_PROF(s, name);
  const size_t sh = (size_t)a.b.T * sizeof(int);
  if (a.bf16) hipLaunchKernelGGL(joiner_tail_kernel<false>, dim3(blocks), dim3(kTailThreads), sh, s, a, tr);
  else hipLaunchKernelGGL(joiner_tail_kernel<true>, dim3(blocks), dim3(kTailThreads), sh, s, a, tr);
  return hipGetLastError();
}

// d(logits) of chunk [cm0, cm1) from stored logits or the head, beside the h
// passes h0 and h1.
static hipError_t launch_head(const JoinerArgs& a, int cm0, int cm1, const HPass& h0, const HPass& h1, hipStream_t s) {
  const dim3 g = a.bf16 ? dl_grid<false>(a, cm1 - cm0) : dl_grid<true>(a, cm1 - cm0);
  const dim3 blocks(g.x * g.y + h0.blocks + h1.blocks);
  RNNT_PROF(s, "joiner_dl");
  if (a.bf16)
    hipLaunchKernelGGL(joiner_head_kernel<false>, blocks, dim3(kTailThreads), 0, s, a, h0, h1, cm0, cm1, (int)g.x, (int)g.y);
  else
    hipLaunchKernelGGL(joiner_head_kernel<true>, blocks, dim3(kTailThreads), 0, s, a, h0, h1, cm0, cm1, (int)g.x, (int)g.y);
  return hipGetLastError();
}

// A GEMM launch of the backward: L of chunk [lm0, lm1) (ring slot of
// `nxt`), D and W of chunk [cm0, cm1) (slot of `cur`); an empty range skips
// its part.
// The other block kinds a pipeline launch may carry: the h pass of a later
// chunk (H) and the d dec pass of the previous one (E).
struct BwdExtras {
  HPass h{};
  const JoinerArgs* dec = nullptr;  // the previous chunk's args (its d dec pieces, in its dpre)
  int dcm0 = 0, dcm1 = 0;
};

static hipError_t launch_bwd_gemms(const JoinerArgs& cur, const JoinerArgs& nxt, int lm0, int lm1, int cm0,
                                   int cm1, hipStream_t s, const BwdExtras& x = BwdExtras()) {
  const int V = cur.V, J = cur.J;
  BwdParts p{};
  p.lm0 = lm0;
  p.lm1 = lm1;
  p.cm0 = cm0;
  p.cm1 = cm1;
  p.first = cm0 == 0;
  auto tiles = [](int n, int t) { return (n + t - 1) / t; };
  p.nLcol = tiles(V, kTileCols);
  p.nL = lm1 > lm0 ? tiles(lm1 - lm0, kTileRows) * p.nLcol : 0;
  p.nDcol = tiles(J, kTileCols);
  p.nD = cm1 > cm0 ? tiles(cm1 - cm0, kTileRows) * p.nDcol : 0;
  p.nWj = tiles(J, kTileRows);
  p.nWv = tiles(V, kTileCols);
  p.nW = cm1 > cm0 ? p.nWj * p.nWv * cur.splits : 0;
  {
    const int bk = cur.bf16 ? CfgT<false>::BK : CfgT<true>::BK;
    const int per = tiles(tiles(cm1 - cm0, cur.splits), bk) * bk;  // a split's rows (dw_tile)
    p.d_first = V > per;
  }
  p.h = x.h;
  if (x.dec && x.dcm1 > x.dcm0) {
    p.nE = dec_blocks(cur.b.N, cur.b.U + 1);
    p.ecm0 = x.dcm0;
    p.ecm1 = x.dcm1;
    p.edpre = x.dec->dpre;
  }
  const int blocks = p.nL + p.nD + p.nW + p.h.blocks + p.nE;
  if (blocks == 0) return hipSuccess;
  RNNT_PROF(s, "joiner_bwd");
  const dim3 g(blocks), t(kGemmThreads);
  if (cur.bf16) hipLaunchKernelGGL(joiner_bwd_gemm_kernel<false>, g, t, 0, s, cur, nxt, p);
  else hipLaunchKernelGGL(joiner_bwd_gemm_kernel<true>, g, t, 0, s, cur, nxt, p);
  return hipGetLastError();
}

// One slot of every chunk buffer (stored logits, or the unpruned loss's
// workspace): the pipeline below would write the next chunk's h and
// d(logits) where the current chunk's are still read, so the chunks run one
// by one: d(logits) streamed beside the h pass (or the h pass, then the
// recomputed logits), then dh and dW, then the chunk's d dec pass.
static hipError_t launch_joiner_bwd_one_slot(const JoinerArgs& a, hipStream_t s) {
  const int mmax = a.b.N * a.b.T * a.S;
  hipError_t e = hipSuccess;
  for (int cm0 = 0; cm0 < mmax && e == hipSuccess; cm0 += a.chunk_rows) {
    const int cm1 = (cm0 + a.chunk_rows < mmax) ? cm0 + a.chunk_rows : mmax;
    const HPass hp = h_pass(a, cm0, cm1, kTailThreads);
    if (a.logits_in) {
      e = launch_head(a, cm0, cm1, hp, HPass{}, s);
    } else {
      TailRanges tr{};
      tr.h0 = hp;
      e = launch_tail(a, tr, s, "joiner_h");
      if (e == hipSuccess) e = launch_bwd_gemms(a, a, cm0, cm1, 0, 0, s);
    }
    if (e == hipSuccess) e = launch_bwd_gemms(a, a, 0, 0, cm0, cm1, s);
    if (e == hipSuccess) e = launch_tail(a, tail_ranges(a, cm0, cm1, cm1 >= mmax), s, cm1 >= mmax ? "joiner_tail" : "joiner_dec");
  }
  return e;
}

hipError_t launch_joiner_bwd(const JoinerArgs& a, hipStream_t s) {
  const int mmax = a.b.N * a.b.T * a.S;
  const int C = a.chunk_rows;
  hipError_t e = hipSuccess;
  if (a.logits_grad) {
    e = launch_fill_f32(a.logits_grad, (size_t)mmax * a.V, 0.f, s);
    if (e != hipSuccess) return e;
  }
  const int nch = (mmax + C - 1) / C;
  if (a.logits_in || (nch > 1 && a.dlring[0] == a.dlring[1])) return launch_joiner_bwd_one_slot(a, s);
  // Recomputed logits, software-pipelined over the chunks with rings of
  // chunk buffers (h: 3 slots; d(logits) and the d dec pieces: 2 slots):
  //   tail{H(0), H(1)}; gemm{L(0)} (or chunk 0 streamed from the head beside
  //   the h passes);
  //   for each chunk k: gemm{W(k), D(k), L(k+1), H(k+2), E(k-1)};
  //   tail{E(last), d enc, dW and db sums}
  // (H: h pass, L: recomputed logits and d(logits), D: dh and the d enc /
  // d dec pieces, W: dW, E: a chunk's d dec pass). Every launch's reads were
  // written by earlier launches on the stream; within a launch, H writes the
  // h slot of chunk k+2 while W, D and L read those of chunks k and k+1, L
  // writes the d(logits) slot of chunk k+1 while D and W read chunk k's, and
  // E reads chunk k-1's pieces while D writes chunk k's.
  auto lo = [&](int k) { return k * C; };
  auto hi = [&](int k) { return (k + 1) * C < mmax ? (k + 1) * C : mmax; };
  TailRanges tr{};
  tr.h0 = h_pass(ring_slot(a, 0), lo(0), hi(0), kTailThreads);
  if (nch > 1) tr.h1 = h_pass(ring_slot(a, 1), lo(1), hi(1), kTailThreads);
  if (a.head && a.head_rows == C) {
    // chunk 0's logits were kept by the forward: stream them instead of the
    // one recomputation launch the pipeline cannot fill
    e = launch_head(ring_slot(a, 0), lo(0), hi(0), tr.h0, tr.h1, s);
  } else {
    e = launch_tail(a, tr, s, "joiner_h");
    if (e == hipSuccess) e = launch_bwd_gemms(ring_slot(a, 0), ring_slot(a, 0), lo(0), hi(0), 0, 0, s);
  }
  for (int k = 0; k < nch && e == hipSuccess; ++k) {
    const JoinerArgs cur = ring_slot(a, k), nxt = ring_slot(a, k + 1), prev = ring_slot(a, k > 0 ? k - 1 : 0);
    const bool more = k + 1 < nch;
    BwdExtras x;
    if (k + 2 < nch) x.h = h_pass(ring_slot(a, k + 2), lo(k + 2), hi(k + 2), kGemmThreads);
    if (k >= 1) {
      x.dec = &prev;
      x.dcm0 = lo(k - 1);
      x.dcm1 = hi(k - 1);
    }
    e = launch_bwd_gemms(cur, nxt, more ? lo(k + 1) : 0, more ? hi(k + 1) : 0, lo(k), hi(k), s, x);
  }
  if (e == hipSuccess) {
    const JoinerArgs last = ring_slot(a, nch - 1);
    e = launch_tail(last, tail_ranges(last, lo(nch - 1), hi(nch - 1), true), s, "joiner_tail");
  }
  return e;
}
