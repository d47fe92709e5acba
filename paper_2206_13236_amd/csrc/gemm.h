// MFMA GEMM main loops for gfx950: the register-staged fp32 engine of the
// separate d am and d lm kernels (generated operands), then the engine whose
// operands go straight to LDS (the joiner).
//
// A workgroup of WGM x WGN wave64s (NT threads) computes a BM x BN
// tile of C = A * B with K-steps of BK. Operand tiles are staged through LDS
// in a k-contiguous layout ([row][k], rows padded by 16 bytes) so that every
// lane fetches one 16-byte fragment per 16x16 output block per k-slice; with
// v_mfma_f32_16x16x4_f32 a fragment holds 4 consecutive k and feeds 4 MFMAs
// (the k order inside a slice is permuted identically for A and B, which
// leaves the sum unchanged). Global -> register fetches of the next K-step are
// issued before the MFMAs of the current one; LDS is double buffered, so there
// is one barrier per K-step.
//
// Operand sources are supplied by each kernel, in two halves so that global
// loads for the next K-step stay in flight while the current one computes:
//   KC  source (global is k-contiguous):
//     kc_load(row, k, Raw&)            issue the loads only
//     kc_finish(const Raw&, v[4])      turn them into 4 values
//   MNC source (global is row-contiguous): mnc_load(k, row, Raw&) and
//     mnc_finish(const Raw&, v[4]).
// Generated operands (exp(x - max)) are formed in *_finish, which runs after
// the MFMAs of the current K-step.
//
// Output element (i, j, r) of a lane: row = wm*WM + i*16 + 4*(lane>>4) + r,
// col = wn*WN + j*16 + (lane & 15).
#pragma once

#include <type_traits>

#include "common.h"

template <int BM_, int BN_, int BK_, int WGM_ = 2, int WGN_ = 2>
struct GemmCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_;
  static constexpr int KV = 4;                // k values per 16-byte fragment
  static constexpr int KSLICE = 4 * KV;       // k covered by one fragment across 4 lane groups
  static constexpr int LDK = BK + KV;         // padded LDS row stride (elements)
  static constexpr int WGM = WGM_, WGN = WGN_;       // wave grid
  static constexpr int NT = 64 * WGM * WGN;          // threads per workgroup
  static constexpr int WM = BM / WGM, WN = BN / WGN;  // wave tile
  static constexpr int FM = WM / 16, FN = WN / 16;
  static constexpr int A_ELEMS = BM * LDK, B_ELEMS = BN * LDK;
  static constexpr int STAGE_ELEMS = A_ELEMS + B_ELEMS;
  static constexpr int SMEM_BYTES = 2 * STAGE_ELEMS * 4;
  static_assert(BK % KSLICE == 0, "BK must be a multiple of the fragment k-slice");
  static_assert(FM >= 1 && FN >= 1, "tile too small");
};

// Raw operand registers of a source whose values need no transform.
template <int N>
struct RawF {
  float v[N];
};

// Raw registers of an exp(x - m) source: the loaded values and the row max.
template <int N>
struct RawExp {
  float x[N];
  float m;
};

DEV void store4(float* dst, const float* v) { *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]); }

// Operand tile whose global source is k-contiguous.
template <class Cfg, int ROWS, class Src>
struct KCLoader {
  static constexpr int KV = Cfg::KV;
  static constexpr int CPR = Cfg::BK / KV;               // 16-byte chunks per row
  static constexpr int NCH = (ROWS * CPR + Cfg::NT - 1) / Cfg::NT;  // chunks per thread
  struct Reg { typename Src::Raw v[NCH]; };
  const Src& src;
  DEV explicit KCLoader(const Src& s) : src(s) {}
  DEV void fetch(int k0, Reg& r) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int c = threadIdx.x + Cfg::NT * i;
      if (ROWS * CPR % Cfg::NT == 0 || c < ROWS * CPR) src.kc_load(c / CPR, k0 + (c % CPR) * KV, r.v[i]);
    }
  }
  DEV void put(const Reg& r, float* lds) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int c = threadIdx.x + Cfg::NT * i;
      if (ROWS * CPR % Cfg::NT == 0 || c < ROWS * CPR) {
        float v[KV];
        src.kc_finish(r.v[i], v);
        store4(lds + (c / CPR) * Cfg::LDK + (c % CPR) * KV, v);
      }
    }
  }
};

// Operand tile whose global source is row-contiguous ([k][row]); the loader
// transposes 4 x 4 blocks in registers so LDS stays k-contiguous.
// Blocks go to threads from TOFF on (modulo NT): when both operands of a
// contraction have fewer blocks than threads, giving them disjoint threads
// spreads the staging over all waves.
template <class Cfg, int ROWS, class Src, int TOFF = 0>
struct MNCLoader {
  static constexpr int KV = Cfg::KV;
  static constexpr int NV = 4;                             // rows per block
  static constexpr int NBR = ROWS / NV;                    // blocks along rows
  static constexpr int NKB = Cfg::BK / KV;                 // blocks along k
  static constexpr int NBLK = NKB * NBR;
  // Consecutive lanes take consecutive k-blocks of the same rows: a transposed
  // LDS store of NKB lanes then fills one padded row contiguously (fewer bank
  // conflicts than lanes 4 rows apart), and each global load still reads
  // NKB x 16 contiguous bytes per row.
  static constexpr int NPT = (NBLK + Cfg::NT - 1) / Cfg::NT;
  struct Reg { typename Src::Raw v[NPT][KV]; };
  const Src& src;
  DEV explicit MNCLoader(const Src& s) : src(s) {}
  DEV void fetch(int k0, Reg& r) const {
#pragma unroll
    for (int b = 0; b < NPT; ++b) {
      int blk = (threadIdx.x + TOFF) % Cfg::NT + Cfg::NT * b;
      if (NBLK % Cfg::NT == 0 || blk < NBLK) {
        const int kb = blk % NKB, nb = blk / NKB;
#pragma unroll
        for (int i = 0; i < KV; ++i) src.mnc_load(k0 + kb * KV + i, nb * NV, r.v[b][i]);
      }
    }
  }
  DEV void put(const Reg& r, float* lds) const {
#pragma unroll
    for (int b = 0; b < NPT; ++b) {
      int blk = (threadIdx.x + TOFF) % Cfg::NT + Cfg::NT * b;
      if (NBLK % Cfg::NT == 0 || blk < NBLK) {
        const int kb = blk % NKB, nb = blk / NKB;
        float m[KV][NV];
#pragma unroll
        for (int i = 0; i < KV; ++i) src.mnc_finish(r.v[b][i], m[i]);
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          float col[KV];
#pragma unroll
          for (int i = 0; i < KV; ++i) col[i] = m[i][c];
          store4(lds + (nb * NV + c) * Cfg::LDK + kb * KV, col);
        }
      }
    }
  }
};

// MFMAs of the k-slices [K0, K1) of one LDS stage.
template <class Cfg, int K0 = 0, int K1 = Cfg::BK>
DEV void gemm_compute_stage(const float* As, const float* Bs,
                            floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
  const float* a_base = As + (wm * Cfg::WM + (lane & 15)) * Cfg::LDK + (lane >> 4) * Cfg::KV;
  const float* b_base = Bs + (wn * Cfg::WN + (lane & 15)) * Cfg::LDK + (lane >> 4) * Cfg::KV;
#pragma unroll
  for (int kk = K0; kk < K1; kk += Cfg::KSLICE) {
    floatx4 fa[Cfg::FM], fb[Cfg::FN];
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) fa[i] = *reinterpret_cast<const floatx4*>(a_base + i * 16 * Cfg::LDK + kk);
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) fb[j] = *reinterpret_cast<const floatx4*>(b_base + j * 16 * Cfg::LDK + kk);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][s], fb[j][s], acc[i][j], 0, 0, 0);
  }
}

// Runs the K loop over [k_begin, k_end) and leaves the tile in `acc`.
// Must be called by all NT threads of the workgroup (it contains barriers).
template <class Cfg, class LA, class LB>
DEV void gemm_mainloop(const LA& la, const LB& lb, int k_begin, int k_end,
                       float* smem, floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int nk = (k_end - k_begin + Cfg::BK - 1) / Cfg::BK;
  if (nk <= 0) return;
  float* As0 = smem;
  float* Bs0 = smem + Cfg::A_ELEMS;
  float* As1 = smem + Cfg::STAGE_ELEMS;
  float* Bs1 = smem + Cfg::STAGE_ELEMS + Cfg::A_ELEMS;
  constexpr int KH = (Cfg::BK / Cfg::KSLICE) / 2 * Cfg::KSLICE;
  typename LA::Reg ra;
  typename LB::Reg rb;
  la.fetch(k_begin, ra);
  lb.fetch(k_begin, rb);
  la.put(ra, As0);
  lb.put(rb, Bs0);
  __syncthreads();
  // The next stage is staged between the two halves of the current stage's
  // MFMAs: its global loads have the first half to land, and its transforms
  // and LDS stores can issue while the second half's MFMAs execute.
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    if (more) {
      la.fetch(k_begin + (kt + 1) * Cfg::BK, ra);
      lb.fetch(k_begin + (kt + 1) * Cfg::BK, rb);
    }
    const bool odd = kt & 1;
    const float* Ac = odd ? As1 : As0;
    const float* Bc = odd ? Bs1 : Bs0;
    gemm_compute_stage<Cfg, 0, KH>(Ac, Bc, acc);
    if (more) {
      la.put(ra, odd ? As0 : As1);
      lb.put(rb, odd ? Bs0 : Bs1);
    }
    gemm_compute_stage<Cfg, KH, Cfg::BK>(Ac, Bc, acc);
    __syncthreads();
  }
}

// XCD-aware tile order. Workgroup w of a launch (x fastest, then y, then z)
// is dispatched to XCD w % 8, and every XCD has its own L2. Tile ids are
// renumbered so that each XCD receives one contiguous run of them: tiles
// that are neighbours in tile-id order (and share an operand panel) then run
// on the same XCD at about the same time and share its L2.
// Only the first n_active workgroups get a tile (-1 for the rest), so that a
// grid sized for the padded maximum spreads its real tiles over all XCDs.
constexpr int kNumXcd = 8;
DEV int xcd_tile_id(int n_active) {
  const int w = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const int n = min(n_active, (int)(gridDim.x * gridDim.y * gridDim.z));
  if (w >= n) return -1;
  const int per = n / kNumXcd, rem = n % kNumXcd;
  const int x = w % kNumXcd, loc = w / kNumXcd;
  return __builtin_amdgcn_readfirstlane((x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + loc);
}

// Row/column of output element (i, j, r) of this lane within the tile.
template <class Cfg>
DEV int tile_row(int i, int r) {
  const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) / Cfg::WGN;
  return wm * Cfg::WM + i * 16 + 4 * (lane >> 4) + r;
}
template <class Cfg>
DEV int tile_col(int j) {
  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) % Cfg::WGN;
  return wn * Cfg::WN + j * 16 + (lane & 15);
}

// ---------------------------------------------------------------------------
// Main loops with both operands loaded straight from global memory into LDS
// (buffer_load_dwordx4 ... lds: the 16 bytes of lane i land at the
// instruction's LDS base + 16 i). Nothing is staged through registers, and two
// workgroups share a CU (64 KiB of LDS each at 128 x 128, two stages). A
// K-step's loads are issued before the previous K-step's fragments are read,
// but the compiler takes any LDS read for one of the bytes in flight and waits
// for them (s_waitcnt vmcnt(0)) before the first of those reads: they overlap
// the other workgroup's work, not their own workgroup's MFMAs.
//
// Two 16-bit operand formats:
//   bf16   one 16-bit word per element;
//   split  an fp32 element x as two fp16 planes of s x (s a power of two that
//          brings the largest element under it, of a row or column, to
//          [2^13, 2^14)): hi = fp16(s x), lo = fp16(s x - hi). After hi's 11
//          bits up to 12 of the 24 remain, with a sign, of which lo holds 11:
//          hi + lo differs from s x by up to 2^-23 of it, an fp32 ulp. That
//          holds down to 2^-16 of the largest element; below, the difference
//          is up to 2^-25, 2^-38 of the largest. A product takes three
//          v_mfma_f32_16x16x32_f16 (lo hi, hi lo, hi hi, accumulated in fp32;
//          lo lo, up to 2^-22 of it, is left out) where fp32 MFMA would take
//          eight 16x16x4, each as long as two of them: a fifth of the matrix
//          time, for the same 4 bytes per element. So one product is off by up
//          to 2^-21 (2^-24 in fp32), a sum by less than with fp32 MFMA, whose
//          error its K / 4 accumulations make: norm of all outputs' error
//          against 64 bits 1.0e-6 for 1.5e-6 at J = 512, V = 5000, 3.7e-7 for
//          5.5e-7 in the unpruned loss at V = 500. Rows hold groups of 32
//          elements, 32 hi then 32 lo (128 bytes).
// ---------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// 16-bit words of a row of n elements: whole K-steps of 64 words (128 bytes),
// zero past the last element.
template <bool SPLIT>
constexpr __host__ __device__ int row_words(int n) { return SPLIT ? (n + 31) / 32 * 64 : (n + 63) / 64 * 64; }
// Word of element k's hi plane within its row (its lo plane: 32 words on).
DEV int split_word(int k) { return (k >> 5) * 64 + (k & 31); }

// The planes of an (already scaled) element. A value beyond fp16 (infinity) or
// a NaN is the lo plane, beside a zero hi plane: of the other operand it meets
// the hi plane alone, whose sign is the element's (its lo plane may have the
// other sign, or be zero), so that a product with infinity is what it is in fp32.
DEV void split_f16(float x, uint16_t& hi, uint16_t& lo) {
  const _Float16 h = (_Float16)(__builtin_fabsf(x) < 65520.f ? x : 0.f);
  const _Float16 l = (_Float16)(x - (float)h);
  hi = __builtin_bit_cast(uint16_t, h);
  lo = __builtin_bit_cast(uint16_t, l);
}
// Two neighbouring elements: words of the hi and of the lo plane.
DEV void split_f16x2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  uint16_t h0, l0, h1, l1;
  split_f16(x0, h0, l0);
  split_f16(x1, h1, l1);
  hi = (uint32_t)h0 | ((uint32_t)h1 << 16);
  lo = (uint32_t)l0 | ((uint32_t)l1 << 16);
}

// The power of two that brings |x| <= mx to [2^13, 2^14), at most 2^100, so
// that it and its inverse are normal numbers (elements below 2^-100 of 1 lose
// their low bits). mx >= 0, infinity included, no NaN.
DEV float split_scale(float mx) {
  const uint32_t e = max(__float_as_uint(mx) >> 23, 40u);  // biased
  return __uint_as_float((13u + 2 * 127u - e) << 23);
}
DEV float finite_abs(float x) {
  const float a = __builtin_fabsf(x);
  return a <= 3.4028234663852886e38f ? a : 0.f;  // inf and NaN do not set the scale
}

// The inverse of a power of two.
DEV float pow2_inv(float s) { return __uint_as_float(0x7f000000u - __float_as_uint(s)); }

// Both main loops compute the tile transposed within each MFMA (B's fragment
// first): output element (i, j, r) of a lane is row wm*WM + i*16 + (lane & 15),
// column wn*WN + j*16 + 4*(lane >> 4) + r, so that a lane holds 4 neighbouring
// columns of FM rows: row-wise epilogues reduce most of a row in registers
// and store 4 columns at a time.
template <class Cfg>
DEV int out_row(int i) {
  const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) / Cfg::WGN;
  return wm * Cfg::WM + i * 16 + (lane & 15);
}
template <class Cfg>
DEV int out_col(int j) {
  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) % Cfg::WGN;
  return wn * Cfg::WN + j * 16 + 4 * (lane >> 4);
}

// Operands k-contiguous in global memory: rows of whole K-steps (row_words),
// 128-byte aligned. An LDS row holds one K-step, 128 bytes (64 bf16 elements,
// or one split group of 32), unpadded; the 16-byte chunks of row r are stored
// XOR-swizzled (chunk c at position c ^ (r & 7)), so that the fragment reads
// of 8 consecutive rows fall in distinct banks.
template <int BM_, int BN_, int WGM_, int WGN_, bool SPLIT_>
struct LdsCfg {
  static constexpr int BM = BM_, BN = BN_;
  static constexpr bool SPLIT = SPLIT_;
  static constexpr int KW = 64;                // words of a row per K-step
  static constexpr int WGM = WGM_, WGN = WGN_;
  static constexpr int NW = WGM * WGN, NT = 64 * NW;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int FM = WM / 16, FN = WN / 16;
  static constexpr int CH = KW / 8;            // 16-byte chunks per row
  static constexpr int ROWB = KW * 2;          // bytes per LDS row
  static constexpr int RPI = 64 / CH;          // rows filled by one wave-wide load
  static constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int SMEM_BYTES = 2 * STAGE_BYTES;
  static constexpr int A_IPW = BM / RPI / NW, B_IPW = BN / RPI / NW;  // loads per wave per stage
  static_assert((BM / RPI) % NW == 0 && (BN / RPI) % NW == 0, "whole loads per wave");
  static_assert(FM >= 1 && FN >= 1, "tile too small");
};

// `rows` rows of a k-contiguous array of 16-bit words from `base` on, row
// stride ld words (a multiple of a K-step); rows past the last one read zeros
// (through the resource's size).
struct LdsSrc {
  Rsrc rsrc;
  int ld;
  DEV LdsSrc(const void* base, int rows, int ld_) : rsrc(make_rsrc(base, (size_t)__builtin_amdgcn_readfirstlane(rows) * ld_ * 2)), ld(ld_) {}
};

typedef __attribute__((address_space(3))) void* LdsPtr;

// One operand tile for the K-step at byte k0 of the rows into `lds`: wave w
// issues loads w*IPW .. w*IPW+IPW-1, load q filling tile rows
// [q*RPI, (q+1)*RPI).
template <class Cfg, int IPW>
DEV void lds_fetch(const LdsSrc& s, int k0, unsigned char* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int q = wave * IPW + i;
    const int r = q * Cfg::RPI + lane / Cfg::CH;
    const int c = (lane % Cfg::CH) ^ (r & 7);  // the chunk stored at this lane's position
    __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rsrc, (LdsPtr)(lds + q * 1024), 16, (uint32_t)r * (uint32_t)(s.ld * 2) + c * 16,
                                             k0, 0, 0);
  }
}

template <class Cfg>
DEV void mfma_bf16(const bf16x8 (&fa)[Cfg::FM], const bf16x8 (&fb)[Cfg::FN], floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
}
template <class Cfg>
DEV void mfma_f16(const f16x8 (&fa)[Cfg::FM], const f16x8 (&fb)[Cfg::FN], floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[j], fa[i], acc[i][j], 0, 0, 0);
}

template <class Cfg>
DEV void lds_compute_stage(const unsigned char* As, const unsigned char* Bs, floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
  const int lr = lane & 15, lq = lane >> 4;
  // fragment rows are 16-aligned plus lr, so their swizzle key is lr & 7
  const unsigned char* a_row = As + (wm * Cfg::WM + lr) * Cfg::ROWB;
  const unsigned char* b_row = Bs + (wn * Cfg::WN + lr) * Cfg::ROWB;
  const int p0 = (lq ^ (lr & 7)) * 16, p1 = ((4 + lq) ^ (lr & 7)) * 16;
  if constexpr (Cfg::SPLIT) {
    f16x8 ah[Cfg::FM], al[Cfg::FM], bh[Cfg::FN], bl[Cfg::FN];
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) al[i] = *reinterpret_cast<const f16x8*>(a_row + i * 16 * Cfg::ROWB + p1);
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) bh[j] = *reinterpret_cast<const f16x8*>(b_row + j * 16 * Cfg::ROWB + p0);
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) ah[i] = *reinterpret_cast<const f16x8*>(a_row + i * 16 * Cfg::ROWB + p0);
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) bl[j] = *reinterpret_cast<const f16x8*>(b_row + j * 16 * Cfg::ROWB + p1);
    mfma_f16<Cfg>(al, bh, acc);
    mfma_f16<Cfg>(ah, bl, acc);
    mfma_f16<Cfg>(ah, bh, acc);
  } else {
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const int pos = kc ? p1 : p0;
      bf16x8 fa[Cfg::FM], fb[Cfg::FN];
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(a_row + i * 16 * Cfg::ROWB + pos);
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(b_row + j * 16 * Cfg::ROWB + pos);
      mfma_bf16<Cfg>(fa, fb, acc);
    }
  }
}

// Waits for this wave's outstanding loads, then meets the other waves.
DEV void lds_stage_barrier() { asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory"); }

template <class Cfg>
DEV void zero_acc(floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
}

// K loop over all words of the rows with two LDS stages: at step kt the loads
// of step kt+1 go to the other stage; one barrier per step. Leaves the
// tile in `acc` and LDS free for the caller (it ends with a barrier). Must be
// called by all NT threads of the workgroup.
template <class Cfg>
DEV void gemm_mainloop_lds(const LdsSrc& sa, const LdsSrc& sb, unsigned char* smem, floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
  zero_acc<Cfg>(acc);
  const int nk = sa.ld / Cfg::KW;
  lds_fetch<Cfg, Cfg::A_IPW>(sa, 0, smem);
  lds_fetch<Cfg, Cfg::B_IPW>(sb, 0, smem + Cfg::A_BYTES);
  for (int kt = 0; kt < nk; ++kt) {
    lds_stage_barrier();  // step kt landed everywhere; step kt-1's slot is free
    if (kt + 1 < nk) {
      unsigned char* st = smem + ((kt + 1) & 1) * Cfg::STAGE_BYTES;
      lds_fetch<Cfg, Cfg::A_IPW>(sa, (kt + 1) * Cfg::ROWB, st);
      lds_fetch<Cfg, Cfg::B_IPW>(sb, (kt + 1) * Cfg::ROWB, st + Cfg::A_BYTES);
    }
    const unsigned char* cs = smem + (kt & 1) * Cfg::STAGE_BYTES;
    lds_compute_stage<Cfg>(cs, cs + Cfg::A_BYTES, acc);
  }
  __syncthreads();
}

// The same for a contraction over rows, C[i][j] = sum_m A[m][i] B[m][j] with
// both operands stored row by row (m): a K-step's rows go to LDS as they are
// and the fragments are read transposed (ds_read_b64_tr_b16: of each 16
// lanes, lane l gives the address of 4 columns of row l / 4 and receives the
// 4 rows of column l), so that no transposed copy of an operand exists in
// memory. A fragment's k order (rows 4q..4q+3 and 16+4q..16+4q+3 for lane
// group q) is the same for A and B.
// An LDS row holds the tile's columns, 256 bytes in bf16 and 512 when split
// (at 128 columns); its 32-byte pairs of chunks are stored XOR-swizzled by
// the row (pair p at position p ^ (r & 7)), so that the 32 bytes read from
// each of 8 consecutive rows fall in distinct banks.
template <int BM_, int BN_, int WGM_, int WGN_, bool SPLIT_>
struct TrCfg {
  static constexpr int BM = BM_, BN = BN_;
  static constexpr bool SPLIT = SPLIT_;
  static constexpr int XP = SPLIT ? 2 : 1;     // words per element
  static constexpr int BK = SPLIT ? 32 : 64;   // rows (k) per K-step
  static constexpr int WGM = WGM_, WGN = WGN_;
  static constexpr int NW = WGM * WGN, NT = 64 * NW;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int FM = WM / 16, FN = WN / 16;
  static constexpr int A_ROWB = BM * XP * 2, B_ROWB = BN * XP * 2;  // bytes per LDS row
  static constexpr int A_BYTES = BK * A_ROWB, B_BYTES = BK * B_ROWB;
  // split: the factors of B's columns in this K-step (one wave-wide load, whose last half is past the columns)
  static constexpr int F_BYTES = SPLIT ? 1024 : 0;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES + F_BYTES;
  static constexpr int SMEM_BYTES = 2 * STAGE_BYTES;
  static constexpr int A_IPW = A_BYTES / 1024 / NW, B_IPW = B_BYTES / 1024 / NW;  // loads per wave per stage
  static_assert(A_ROWB % 256 == 0 && B_ROWB % 256 == 0, "whole swizzle blocks per row");
  static_assert(!SPLIT || BN * 4 <= F_BYTES, "the factors are one load");
  static_assert(A_BYTES / 1024 % NW == 0 && B_BYTES / 1024 % NW == 0, "whole loads per wave");
};

// Rows [0, rows) of an array of 16-bit words from `base` on (row stride ld
// words), words [c0, ld) of each; words past ld and rows past the last one
// read zeros.
struct TrSrc {
  const unsigned char* base;
  int rows, ld, c0;
};

// The factors of a split B operand's columns, [K-step][ld] from `base` on, for
// columns [c0, ld) (zeros past ld): B's planes are scaled by a power of two of
// their own in every column of a K-step's rows, undone as the K-step's products
// join the sum, so that neither a small column nor a small group of rows runs
// out of fp16's range beside large ones.
struct TrFactors {
  const float* base;
  int ld, c0;
};

// An operand tile's rows from r0 on: the resource starts there, so that 32-bit
// offsets only span one K-step.
template <int IPW, int ROWB>
DEV void tr_fetch(const TrSrc& s, int r0, unsigned char* lds) {
  constexpr int CPR = ROWB / 16, RPI = 64 / CPR;  // chunks per row, rows per load
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Rsrc rs = make_rsrc(s.base + (size_t)r0 * s.ld * 2, (size_t)min(s.rows - r0, 64) * s.ld * 2);
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int q = wave * IPW + i;
    const int r = q * RPI + lane / CPR;
    const int c = s.c0 + ((lane % CPR) ^ ((r & 7) << 1)) * 8;  // the chunk stored at this lane's position
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LdsPtr)(lds + q * 1024), 16,
                                             c < s.ld ? (uint32_t)r * (uint32_t)(s.ld * 2) + c * 2 : kOob, 0, 0, 0);
  }
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* LdsTrPtr;

// A 16-column fragment of two times 16 rows; `p` and `q` are this lane's
// addresses in the first and second.
template <class F>
DEV F tr_frag2(const unsigned char* p, const unsigned char* q) {
  struct { s16x4 a, b; } v;
  v.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTrPtr)(p));
  v.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTrPtr)(q));
  return __builtin_bit_cast(F, v);
}
template <class F, int ROWB>
DEV F tr_frag(const unsigned char* p) {
  return tr_frag2<F>(p, p + 16 * ROWB);
}

template <class Cfg>
DEV void tr_compute_stage(const unsigned char* As, const unsigned char* Bs, const float* fac,
                          floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
  const int row = lane >> 2, key = row & 7;  // rows 0..15 of a fragment, 4 lanes a row
  const unsigned char* a = As + row * Cfg::A_ROWB + (lane & 3) * 8;
  const unsigned char* b = Bs + row * Cfg::B_ROWB + (lane & 3) * 8;
  // pair of 16-column block c: its 32 bytes in bf16; its hi plane when split
  // (the lo plane two pairs on)
  auto pair = [](int c) { return Cfg::SPLIT ? (c >> 1) * 4 + (c & 1) : c; };
  if constexpr (Cfg::SPLIT) {
    static_assert(Cfg::BK == 32, "one factor per column and K-step");
    f16x8 ah[Cfg::FM], al[Cfg::FM];
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) {
      al[i] = tr_frag<f16x8, Cfg::A_ROWB>(a + (((pair(wm * Cfg::FM + i) + 2) ^ key) << 5));
      ah[i] = tr_frag<f16x8, Cfg::A_ROWB>(a + ((pair(wm * Cfg::FM + i) ^ key) << 5));
    }
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      const f16x8 bh = tr_frag<f16x8, Cfg::B_ROWB>(b + ((pair(wn * Cfg::FN + j) ^ key) << 5));
      const f16x8 bl = tr_frag<f16x8, Cfg::B_ROWB>(b + (((pair(wn * Cfg::FN + j) + 2) ^ key) << 5));
      const floatx4 f = *reinterpret_cast<const floatx4*>(fac + out_col<Cfg>(j));
      floatx4 t[Cfg::FM];
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) t[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bh, al[i], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) t[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bl, ah[i], t[i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) t[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bh, ah[i], t[i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = fmaf(t[i][r], f[r], acc[i][j][r]);
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < Cfg::BK; ks += 32) {
      bf16x8 fa[Cfg::FM], fb[Cfg::FN];
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
        fa[i] = tr_frag<bf16x8, Cfg::A_ROWB>(a + ks * Cfg::A_ROWB + ((pair(wm * Cfg::FM + i) ^ key) << 5));
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j)
        fb[j] = tr_frag<bf16x8, Cfg::B_ROWB>(b + ks * Cfg::B_ROWB + ((pair(wn * Cfg::FN + j) ^ key) << 5));
      mfma_bf16<Cfg>(fa, fb, acc);
    }
  }
}

// One K-step's rows of both operands, and its factors, into a stage.
template <class Cfg>
DEV void tr_fetch_stage(const TrSrc& sa, const TrSrc& sb, const TrFactors& f, int kt, unsigned char* st) {
  tr_fetch<Cfg::A_IPW, Cfg::A_ROWB>(sa, kt * Cfg::BK, st);
  tr_fetch<Cfg::B_IPW, Cfg::B_ROWB>(sb, kt * Cfg::BK, st + Cfg::A_BYTES);
  if constexpr (Cfg::SPLIT) {
    if (threadIdx.x < 64) {
      const Rsrc rs = make_rsrc(f.base + (size_t)kt * f.ld, (size_t)f.ld * 4);
      const int c = 4 * (int)threadIdx.x;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LdsPtr)(st + Cfg::A_BYTES + Cfg::B_BYTES), 16,
                                               c < Cfg::BN ? (uint32_t)(f.c0 + c) * 4u : kOob, 0, 0, 0);
    }
  }
}

// K loop over all rows of the sources: as gemm_mainloop_lds.
template <class Cfg>
DEV void gemm_mainloop_tr(const TrSrc& sa, const TrSrc& sb, const TrFactors& f, unsigned char* smem,
                          floatx4 (&acc)[Cfg::FM][Cfg::FN]) {
  zero_acc<Cfg>(acc);
  const int nk = (sa.rows + Cfg::BK - 1) / Cfg::BK;
  if (nk <= 0) return;
  tr_fetch_stage<Cfg>(sa, sb, f, 0, smem);
  for (int kt = 0; kt < nk; ++kt) {
    lds_stage_barrier();
    if (kt + 1 < nk) tr_fetch_stage<Cfg>(sa, sb, f, kt + 1, smem + ((kt + 1) & 1) * Cfg::STAGE_BYTES);
    const unsigned char* cs = smem + (kt & 1) * Cfg::STAGE_BYTES;
    tr_compute_stage<Cfg>(cs, cs + Cfg::A_BYTES, reinterpret_cast<const float*>(cs + Cfg::A_BYTES + Cfg::B_BYTES), acc);
  }
  __syncthreads();
}
