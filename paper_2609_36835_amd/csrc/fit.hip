// Mass-bias and compact-value fits (Appendix A.9, eq. mass_fit, eq. value_lstsq).
//
// Both fits solve ridge-regularised normal equations (M + lam I) x = rhs with
// M a float32 Gram matrix of size tp (padded; the padding is an identity
// block with zero right-hand side, so padded unknowns solve to 0):
//   k_ridge_init     lam = delta * tr(M)/t, write M + lam I into the work copy
//   Cholesky         float32, left-looking over 256-wide outer panels:
//                      k_chol_scales  per-row power-of-two shifts s_r from the
//                                     diagonal (sqrt(A_rr) s_r in [2^13, 2^14))
//                      (contraction)  before a panel is factored, the big
//                                     contraction on fp16 MFMA applies every
//                                     earlier panel to it (hi / lo planes of
//                                     L s_r, three products, about 2^-22
//                                     relative)
//                      k_chol_diag256 factor the panel's 256 x 256 diagonal
//                                     block in LDS (16-column steps, fp32
//                                     MFMA) and invert its 64 x 64 diagonal
//                                     blocks
//                      k_chol_strip16 the rows below it: the same panel steps
//                                     and updates on a 128 x 256 strip held in
//                                     LDS as hi / lo planes (fp16 MFMA), then
//                                     L and its planes written back
//                    a failed pivot records info = column + 1 for that pair
//   escalation       pairs that failed are refactored by the same kernels with
//                    delta raised tenfold (from 1e-7 when zero), at most
//                    max_escalations times (launch_cholesky)
//   solves           TRSV (one rhs, float64 accumulation, by the 64 x 64 diagonal
//                    inverses, right-looking) / TRSM (128 rhs, fp32 MFMA, by the
//                    inverses of the 256 x 256 diagonal blocks, k_chol_inv256,
//                    right-looking for few pairs and left-looking for many), both
//                    in 256-row blocks
//   residuals        rhs - (M + lam I) x, float64 (mass fit) or float32 MFMA
//                    (value fit), for iterative refinement
#include "common.hpp"
#include "gemm.hpp"
#include "gemm_big.hpp"
#include "fit.hpp"

namespace arckv {

constexpr int kNB = 64;          // Cholesky block
constexpr int kSD = kNB + 1;     // LDS stride of a 64x64 fp32 tile

// --------------------------------------------------------------- ridge
// info starts at -1 for pairs flagged with non-finite inputs (bad, may be
// null), which every later kernel then skips, and 0 otherwise.
__global__ void __launch_bounds__(256) k_ridge_init(float *__restrict__ Gw, const float *__restrict__ Gc, int t,
                                                    int64_t ld, float delta0, FitState st,
                                                    const int32_t *__restrict__ bad) {
  __shared__ double red[4];
  const int b = blockIdx.x, tid = threadIdx.x;
  const size_t base = (size_t)b * ld * ld;
  double tr = 0.0;
  for (int r = tid; r < t; r += 256) tr += (double)Gc[base + (size_t)r * ld + r];
  tr = wave_sum(tr);
  if ((tid & 63) == 0) red[tid >> 6] = tr;
  __syncthreads();
  tr = red[0] + red[1] + red[2] + red[3];
  const float lam = (float)((double)delta0 * tr / (double)t);
  for (int64_t r = tid; r < ld; r += 256) Gw[base + (size_t)r * ld + r] = r < t ? Gc[base + (size_t)r * ld + r] + lam : 1.0f;
  if (tid == 0) {
    st.trace[b] = tr;
    st.lam[b] = lam;
    st.delta[b] = delta0;
    st.nesc[b] = 0;
    st.info[b] = bad && bad[b] ? -1 : 0;
  }
}

// ---------------------------------------------------------------- ridge escalation
// A pair whose factorisation failed (info > 0) is refactored with the ridge
// raised tenfold, from kDeltaFloor when it was zero, by the same batched
// blocked factorisation, while it has escalations left (nesc < max_esc); pairs
// that are settled carry kEscSkip meanwhile (every factorisation kernel skips
// info != 0), non-finite ones keep -1.
constexpr int32_t kEscSkip = -0x30000000;
constexpr float kDeltaFloor = 1e-7f;

__global__ void k_esc_state(int B, int t, FitState st, int max_esc) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= B) return;
  const int32_t f = st.info[b];
  if (f > 0 && st.nesc[b] < max_esc) {
    const float delta = fmaxf(10.0f * st.delta[b], kDeltaFloor);
    st.delta[b] = delta;
    st.lam[b] = (float)((double)delta * st.trace[b] / (double)t);
    st.nesc[b] += 1;
    st.info[b] = 0;
  } else if (f == 0) {
    st.info[b] = kEscSkip;
  }
}

// Gw = Gc + lam I (lower triangle and diagonal; padding diagonal 1) for the
// pairs being refactored (info == 0).  One row per thread-block row.
__global__ void __launch_bounds__(256) k_esc_copy(float *__restrict__ Gw, const float *__restrict__ Gc, int t,
                                                  int64_t ld, FitState st) {
  const int b = blockIdx.y;
  const int64_t r = blockIdx.x;
  if (st.info[b] != 0) return;
  const float lam = st.lam[b];
  const size_t base = (size_t)b * ld * ld + (size_t)r * ld;
  for (int64_t c = threadIdx.x; c <= r; c += 256)
    Gw[base + c] = c == r ? (r < t ? Gc[base + c] + lam : 1.0f) : Gc[base + c];
}

__global__ void k_esc_restore(int B, int32_t *__restrict__ info) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < B && info[b] == kEscSkip) info[b] = 0;
}

// cnt[0] = number of pairs whose factorisation failed (info > 0) and that
// have escalations left.
__global__ void __launch_bounds__(256) k_count_failed(int B, const FitState st, int max_esc, int32_t *cnt) {
  __shared__ int red[4];
  int c = 0;
  for (int b = threadIdx.x; b < B; b += 256) c += st.info[b] > 0 && st.nesc[b] < max_esc;
  for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) cnt[0] = red[0] + red[1] + red[2] + red[3];
}

// ---------------------------------------------------------------- refinement guard
// Each refinement step recomputes the residual from the data, so it converges
// at a rate set by how far the float32 factor is from those normal equations.
// Where the ridge is small next to the Gram's float32 rounding (a
// rank-deficient Gram, t > n, with a ridge near 1e-6 of its mean diagonal) the
// steps instead grow the solution along the Gram's near-null directions.  After
// every step but the first the correction is compared with the previous one:
// a correction above 1e-10 |w| that is not at most half the previous one is
// undone and ends the pair's refinement (kRefStop); while it has escalations
// left the pair is then refactored with the ridge raised tenfold and solved
// again (div).  Pairs not being refactored meanwhile carry kDoneSkip.
constexpr int32_t kRefStop = -0x20000000;
constexpr int32_t kDoneSkip = -0x10000000;

// One workgroup per pair, after step it (w already holds w + x); it = 0 records
// the first correction's norm.
__global__ void __launch_bounds__(256) k_refine_watch(double *__restrict__ w, const double *__restrict__ x,
                                                      int64_t tp, int it, double *__restrict__ xprev,
                                                      int32_t *__restrict__ div, FitState st, int max_esc) {
  __shared__ double red[2][4];
  const int b = blockIdx.x, tid = threadIdx.x;
  if (st.info[b] != 0) return;
  const double xp = xprev[b];   // read by every thread before thread 0 rewrites it
  const size_t o = (size_t)b * tp;
  double x2 = 0.0, w2 = 0.0;
  for (int64_t r = tid; r < tp; r += 256) {
    const double a = x[o + r], c = w[o + r];
    x2 = fma(a, a, x2);
    w2 = fma(c, c, w2);
  }
  x2 = wave_sum(x2);
  w2 = wave_sum(w2);
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = x2;
    red[1][tid >> 6] = w2;
  }
  __syncthreads();
  const double xn = sqrt(red[0][0] + red[0][1] + red[0][2] + red[0][3]);
  const double wn = sqrt(red[1][0] + red[1][1] + red[1][2] + red[1][3]);
  if (it == 0 || !(xn > 0.5 * xp && xn > 1e-10 * wn)) {
    if (tid == 0) xprev[b] = xn;
    return;
  }
  for (int64_t r = tid; r < tp; r += 256) w[o + r] -= x[o + r];
  if (tid == 0) {
    st.info[b] = kRefStop;
    div[b] = st.nesc[b] < max_esc;
  }
}

// cnt[0] = number of nonzero flags.
__global__ void __launch_bounds__(256) k_count_flags(int B, const int32_t *__restrict__ flag, int32_t *cnt) {
  __shared__ int red[4];
  int c = 0;
  for (int b = threadIdx.x; b < B; b += 256) c += flag[b] != 0;
  for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) cnt[0] = red[0] + red[1] + red[2] + red[3];
}

// Pairs to refactor get info = 1 (picked up by k_esc_state); the settled rest kDoneSkip.
__global__ void k_div_mark(int B, int32_t *__restrict__ div, int32_t *__restrict__ info) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= B) return;
  const int32_t f = info[b];
  if (div[b]) {
    info[b] = 1;
    div[b] = 0;
  } else if (f == 0 || f == kRefStop) {
    info[b] = kDoneSkip;
  }
}

__global__ void k_refine_restore(int B, int32_t *__restrict__ info) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < B && (info[b] == kRefStop || info[b] == kDoneSkip)) info[b] = 0;
}

// ---------------------------------------------------------------- non-finite inputs
// bad[b] |= 1 when any value of pair b in the arrays is not finite (bad is
// cleared by the caller); blockIdx.z is the array, a grid-stride pass over its
// [B][per], 16 bytes at a time where each pair's values start on a 16-byte
// boundary.  One launch for all inputs of a fit: one each took 3 to 10 us.
__global__ void __launch_bounds__(256) k_nonfinite(FiniteCheck f, int32_t *__restrict__ bad) {
  const int b = blockIdx.y;
  const float *a = f.a[blockIdx.z];
  const int64_t per = f.per[blockIdx.z];
  if (!a) return;
  const float *ab = a + (size_t)b * per;
  bool any = false;
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  const bool wide = ((uintptr_t)a & 15) == 0 && (per & 3) == 0;
  if (wide) {
    for (int64_t i = i0; i < per / 4; i += step) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(ab + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) any |= !isfinite(v[e]);
    }
  } else {
    for (int64_t i = i0; i < per; i += step) any |= !isfinite(ab[i]);
  }
  if (__any(any) && (threadIdx.x & 63) == 0) atomicOr(&bad[b], 1);
}

// ------------------------------------------------- the panel's diagonal block
// 16 x 16 fp32 tiles in LDS: element (r, c) at float 64 (c % 4) + 4 r + c / 4, so
// lane 16 g + r reads columns g, 4 + g, 8 + g, 12 + g of row r with one
// conflict-free 16-byte access.  fp32 MFMA adds its products one by one, each with
// one rounding, so the four instructions of diag_mac(acc, X, Y) add X Y^T in
// column order, exactly as fused multiply-adds would.  With Y read by
// diag_get_perm (row 4 (r % 4) + r / 4) the result is in the same layout; with Y
// read by diag_get lane 16 g + r gets columns 4 g .. 4 g + 3 of row r.
__device__ __forceinline__ f32x4 diag_get(const float *tile, int lane) {
  return *reinterpret_cast<const f32x4 *>(tile + 4 * lane);
}
__device__ __forceinline__ f32x4 diag_get_perm(const float *tile, int lane) {
  return *reinterpret_cast<const f32x4 *>(tile + 4 * ((lane & 0x30) + 4 * (lane & 3) + ((lane >> 2) & 3)));
}
__device__ __forceinline__ f32x4 diag_mac(f32x4 acc, f32x4 x, f32x4 y) {
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(y[s], x[s], acc, 0, 0, 0);
  return acc;
}
// The same for N accumulators with one Y, side by side: a product that waits for the
// one before it takes longer than its issue.
template <int N>
__device__ __forceinline__ void diag_mac_n(f32x4 *acc, const f32x4 *x, f32x4 y) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[s], x[u][s], acc[u], 0, 0, 0);
}
// Row r of a tile into (or from) one lane's 16 registers.
__device__ __forceinline__ void diag_row(const float *tile, int r, float (&a)[16]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 v = *reinterpret_cast<const f32x4 *>(tile + 64 * g + 4 * r);
#pragma unroll
    for (int s = 0; s < 4; ++s) a[4 * s + g] = v[s];
  }
}
__device__ __forceinline__ void diag_put_row(float *tile, int r, const float (&a)[16]) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<f32x4 *>(tile + 64 * g + 4 * r) = f32x4{a[g], a[4 + g], a[8 + g], a[12 + g]};
}

// Workgroup barrier for LDS alone: the stores to global memory, which the kernel
// does not read back, stay in flight.
__device__ __forceinline__ void diag_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// v with lane LANE replaced by the wave-uniform x.
template <int LANE>
__device__ __forceinline__ float lane_put(float v, float x) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(x), "n"(LANE));
  return v;
}

// a[q] -= l col_q for q = C + 1 .. 15, col_q lane q's col.  The lanes are read
// first: a vector instruction has to wait two cycles for a scalar just read.
template <int C>
__device__ __forceinline__ void sub_column(float (&a)[16], float col, float l) {
  float v[16];
#pragma unroll
  for (int q = C + 1; q < 16; ++q) v[q] = lane_value(col, q);
#pragma unroll
  for (int q = C + 1; q < 16; ++q) a[q] = fmaf(-v[q], l, a[q]);
}

// sqrt(p) and the root's reciprocal from the hardware's estimate r0 of 1 / sqrt(p) with
// one residual each, both faithful: over every significand of two binades and every
// r0 within one unit of the rounded value (2^24 x 3), the root is one unit off the
// correctly rounded one 5 times and the reciprocal 64 times, never more.  TINY scales p below 2^-96 by 2^64 first, whose
// residuals would underflow.
constexpr float kTinyPivot = 0x1p-96f;
template <bool TINY>
__device__ __forceinline__ void pivot_root(float p, float &root, float &inv) {
  const bool small = TINY && p < kTinyPivot;
  const float q = small ? p * 0x1p64f : p;
  const float r0 = __builtin_amdgcn_rsqf(q);
  const float d0 = q * r0;
  const float d = fmaf(fmaf(-d0, d0, q), 0.5f * r0, d0);
  const float i = fmaf(fmaf(-d, r0, 1.0f), r0, r0);
  root = small ? d * 0x1p-32f : d;
  inv = small ? i * 0x1p32f : i;
}

// Columns C .. 15 of the factorisation of up to 64 rows in one wave, one row per
// lane, lanes 0 .. 15 the diagonal tile's.  a[c] becomes L_rc (of the diagonal
// tile for r > c only; entries above are never read by another lane); lane C
// of the first 16 keeps column C's pivot in piv.
template <int C, bool TINY>
__device__ __forceinline__ void factor_columns(float (&a)[16], float &piv) {
  if constexpr (C < 16) {
    float root, inv;
    const float p = lane_value(a[C], C);
    pivot_root<TINY>(p, root, inv);
    piv = lane_put<C>(piv, p);
    a[C] *= inv;
    sub_column<C>(a, a[C], a[C]);
    factor_columns<C + 1, TINY>(a, piv);
  }
}

// Rows C .. 15 of the substitution L X = Y, one column per lane: y[c] becomes
// X_c = Y_c inv_c, L and inv as factor_columns leaves them.
template <int C>
__device__ __forceinline__ void substitute_rows(float (&y)[16], const float (&a)[16], float inv) {
  if constexpr (C < 16) {
    y[C] *= lane_value(inv, C);
    sub_column<C>(y, a[C], y[C]);
    substitute_rows<C + 1>(y, a, inv);
  }
}

// The 256 x 256 diagonal block at K0 in one workgroup per pair: L in place and
// the inverses X of its four 64 x 64 diagonal blocks to dinv.  The block is held
// in LDS as its 136 lower 16 x 16 tiles.  For each 64-wide step K (tile columns
// 4 K .. 4 K + 3), with wave 4 K + s the owner of tile column 4 K + s inside the
// diagonal block and wave i that of tile row i below it:
//   phase p = 0 .. 3: wave p of the block factors tile column p (its rows down to
//     the block's end, one per lane), after the product of column p - 1 that just
//     became visible; wave p - 1 meanwhile forms X's tile row p - 1 by
//     substitution, one column per lane; phase 4: X's last tile row.  The waves of
//     the blocks below spend the phases on step K - 1's update of their tiles,
//     A -= L L^T over its 64 columns.
//   panel: the rows below, L_i = A_i X^T.
// Every entry sees the operations, in the order, of a column-by-column
// factorisation of each 64 x 64 block, a row-by-row substitution for its inverse
// and 64-wide products for the rest.  nb = ceil((t - K0) / 64) steps, at most 4:
// the padding is an identity already.  A failed pivot records info = column + 1.
//
// Bound by the chain of its 256 pivots (16 tile columns of about 1.6 us, 0.7 us of
// them the pivots).  One launch in place of ten (64-column factorisations of 35 us
// and three panel and three update launches on single blocks): 197 -> 48 us per
// block at 8 pairs.  Keeping the operations' order costs 4 us against a form with
// explicit 16 x 16 inverses, whose roundings, of the same size, moved the fitted
// biases of nearly square systems (t = 3277, n = 4096) by up to 0.56 of their scale.
constexpr int kDiagXn = 260;   // floats of a tile of X: its column-wise stores hit 16 banks
constexpr size_t kDiag256Lds = (size_t)(136 * 256 + 6 * 256 + 10 * kDiagXn + 16) * sizeof(float);

__global__ void __launch_bounds__(1024) k_chol_diag256(float *__restrict__ Gw, int64_t ld, int K0, int nb,
                                                       int32_t *__restrict__ info, float *__restrict__ dinv) {
  extern __shared__ __attribute__((aligned(16))) float diag_smem[];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (info[b] != 0) return;   // uniform over the workgroup
  float *const sXt = diag_smem + 136 * 256, *const sXn = sXt + 6 * 256;
  int32_t *fail = reinterpret_cast<int32_t *>(sXn + 10 * kDiagXn);   // of every tile column: a slot is written in one phase only
  auto tile = [&](int i, int m) { return diag_smem + (i * (i + 1) / 2 + m) * 256; };
  auto xt = [&](int i, int m) { return sXt + (i * (i + 1) / 2 + m) * 256; };        // X_im^T, i <= 2
  auto xn = [&](int i, int m) { return sXn + (i * (i + 1) / 2 + m) * kDiagXn; };   // X_im
  float *D = Gw + (size_t)b * ld * ld + (size_t)K0 * ld + K0;
  float *grow = D + (size_t)(16 * wave + r) * ld + 4 * g;   // this lane's part of tile row `wave`
  float *Xb = dinv + ((size_t)b * (ld / kNB) + K0 / kNB) * kNB * kNB;
  // columns 4 g .. 4 g + 3 of row r into a tile
  auto put_quad = [&](float *to, f32x4 v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) to[64 * e + 4 * r + g] = v[e];
  };
  {
    f32x4 v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m)
      if (m <= wave) v[m] = *reinterpret_cast<const f32x4 *>(grow + 16 * m);
#pragma unroll
    for (int m = 0; m < 16; ++m)
      if (m <= wave) put_quad(tile(wave, m), v[m]);
  }
  if (tid < 16) fail[tid] = 0;
  const int blk = wave >> 2, s = wave & 3;
  if (blk >= nb) {   // a block of padding: identity
#pragma unroll
    for (int c = 0; c < 16; ++c) Xb[(size_t)blk * kNB * kNB + (16 * s + c) * kNB + lane] = 16 * s + c == lane ? 1.0f : 0.0f;
  }
  __syncthreads();
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  int32_t failed = 0;
  for (int K = 0; K < nb; ++K) {   // uniform over the workgroup, as the phases
    const int k0 = 4 * K, j = k0 + s;
    f32x4 cc[4], yt[3];   // the column's tiles; X's tile row s (transposed) before its substitution
    float a[16], inv;
    const bool mine = blk == K, below = blk > K && blk < nb;
    const int todo = below && K > 0 ? wave - k0 + 1 : 0;   // tiles of this row that step K - 1 updates
    if (mine) {
      // step K - 1's product (a wave with fewer tiles repeats its last one: the four
      // chains then run side by side without branches)
#pragma unroll
      for (int u = 0; u < 4; ++u) cc[u] = zero;
      if (K > 0) {
#pragma unroll 1
        for (int m = k0 - 4; m < k0; ++m) {
          const f32x4 y = diag_get_perm(tile(j, m), lane);
          f32x4 x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = diag_get(tile(min(j + u, k0 + 3), m), lane);
          __builtin_amdgcn_sched_barrier(0);
          diag_mac_n<4>(cc, x, y);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) cc[u] = diag_get(tile(min(j + u, k0 + 3), j), lane) - cc[u];
#pragma unroll
      for (int u = 0; u < 3; ++u) yt[u] = zero;
    }
#pragma unroll 1
    for (int p = 0; p < 5; ++p) {
      if (mine) {
        if (p > 0 && p < 4 && s >= p) {   // column p - 1's product, just visible
          const f32x4 y = diag_get_perm(tile(j, k0 + p - 1), lane);
          f32x4 x[3];   // (a wave with fewer tiles repeats its last one)
#pragma unroll
          for (int u = 0; u < 3; ++u) x[u] = -diag_get(tile(min(j + u, k0 + 3), k0 + p - 1), lane);
          __builtin_amdgcn_sched_barrier(0);
          diag_mac_n<3>(cc, x, y);
        }
        if (s == p) {
          __builtin_amdgcn_s_setprio(3);   // the critical chain
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (s + u < 4) *reinterpret_cast<f32x4 *>(tile(j + u, j) + 4 * lane) = cc[u];
          __builtin_amdgcn_wave_barrier();
          float *own = tile(j + (s + g < 4 ? g : 0), j);   // lanes past the block's end repeat the diagonal tile
          float piv = 0.0f, root;
          diag_row(own, r, a);
          factor_columns<0, false>(a, piv);
          pivot_root<false>(piv, root, inv);
          if (__ballot(g == 0 && !(piv >= kTinyPivot && piv < INFINITY))) {   // a failed or tiny pivot: again, scaled
            diag_row(own, r, a);
            factor_columns<0, true>(a, piv);
            pivot_root<true>(piv, root, inv);
            const uint64_t bad = __ballot(g == 0 && !(piv > 0.0f && piv < INFINITY));
            if (bad != 0 && lane == 0) fail[j] = K0 + 16 * j + __ffsll((unsigned long long)bad);
          }
          __builtin_amdgcn_wave_barrier();
          if (s + g < 4) diag_put_row(own, r, a);
          if (g == 0) own[64 * (r & 3) + 4 * r + (r >> 2)] = root;
          __builtin_amdgcn_s_setprio(0);
        }
        if (p > 1 && s >= p - 1) {   // X's tile row p - 2 is visible
#pragma unroll
          for (int u = 0; u < 3; ++u)
            if (u <= p - 2)
              yt[u] = diag_mac(yt[u], -diag_get(xt(p - 2, u), lane), diag_get_perm(tile(j, k0 + p - 2), lane));
        }
        if (s == p - 1) {   // X's tile row s
#pragma unroll
          for (int u = 0; u < 3; ++u)
            if (u < s) *reinterpret_cast<f32x4 *>(xn(s, u) + 4 * lane) = yt[u];
          __builtin_amdgcn_wave_barrier();
          float y[16];
          diag_row(xn(s, min(g, s)), r, y);
#pragma unroll
          for (int c = 0; c < 16; ++c) y[c] = g < s ? y[c] : g == s && c == r ? 1.0f : 0.0f;
          __builtin_amdgcn_wave_barrier();
          substitute_rows<0>(y, a, inv);
          if (g <= s) {
            if (s < 3) diag_put_row(xt(s, g), r, y);
            float *to = xn(s, g) + 64 * (r & 3) + (r >> 2);
#pragma unroll
            for (int c = 0; c < 16; ++c) to[4 * c] = y[c];
          }
          float *to = Xb + (size_t)K * kNB * kNB + 16 * s * kNB + lane;
#pragma unroll
          for (int c = 0; c < 16; ++c) to[c * kNB] = y[c];
        }
      } else if (todo > 0) {
        for (int m = k0 + p * todo / 5; m < k0 + (p + 1) * todo / 5; ++m) {
          f32x4 acc = zero;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            acc = diag_mac(acc, diag_get(tile(wave, k0 - 4 + q), lane), diag_get_perm(tile(m, k0 - 4 + q), lane));
          float *t = tile(wave, m) + 4 * lane;
          *reinterpret_cast<f32x4 *>(t) = *reinterpret_cast<const f32x4 *>(t) - acc;
        }
      }
      diag_barrier();
    }
#pragma unroll
    for (int p = 3; p >= 0; --p) failed = fail[k0 + p] ? fail[k0 + p] : failed;
    if (failed) break;   // uniform
    if (mine) {   // tile row j of the block's L
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (m <= s) {
          const float *t = tile(j, k0 + m) + 4 * r + g;
          const f32x4 v = {t[0], t[64], t[128], t[192]};
          if (m < s) {
            *reinterpret_cast<f32x4 *>(grow + 16 * (k0 + m)) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (4 * g + e <= r) grow[16 * (k0 + m) + e] = v[e];
          }
        }
    } else if (below) {
      f32x4 x[4], l[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) x[m] = diag_get(tile(wave, k0 + m), lane);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        l[u] = zero;
#pragma unroll
        for (int m = 0; m <= u; ++m) l[u] = diag_mac(l[u], x[m], diag_get(xn(u, m), lane));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        put_quad(tile(wave, k0 + u), l[u]);
        *reinterpret_cast<f32x4 *>(grow + 16 * (k0 + u)) = l[u];
      }
    }
    diag_barrier();
  }
  if (failed && tid == 0) info[b] = failed;
}

// Left-looking update of the column panel K0 .. K0 + 255:
// G[K0 + r][K0 + c] -= acc s_r s_c for the tile's entries with c <= r + 63
// (the lower triangle, up to whole diagonal 64-blocks), s the rows' inverse
// scales 2^-shift (k_chol_scales; BM x BN tiles); per row block of the wave,
// every old value is loaded before any store so the loads pipeline.
template <int TM, int TN, int BM, int BN>
struct EpiCholUpd {
  float *G;
  int64_t ld;
  int K0;
  const int32_t *info;
  const float *rs;        // inverse scales of pair 0, rows from K0
  int64_t rs_pair;        // floats between pairs
  __device__ __forceinline__ bool skip(int p) const { return info[p] != 0; }
  __device__ __forceinline__ void operator()(f32x16 (&acc)[TM][TN], int p, int row0, int col0, int mt, int nt,
                                             int lane, int, int) const {
    if (info[p] != 0) return;   // uniform over the workgroup
    // the tile's row and column scales, staged in LDS (the operand stages are
    // free: the caller synchronised the workgroup before the epilogue)
    extern __shared__ __attribute__((aligned(1024))) char big_smem[];
    float *ssc = reinterpret_cast<float *>(big_smem);
    const float *sp = rs + (size_t)p * rs_pair;
    for (int x = threadIdx.x; x < BM + BN; x += blockDim.x) ssc[x] = sp[x < BM ? mt * BM + x : nt * BN + x - BM];
    __syncthreads();
    float *Gp = G + (size_t)p * ld * ld + (size_t)K0 * ld + K0;
    const int col = lane & 31, rl = row0 - mt * BM, cl = col0 - nt * BN;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float old[TN][16];
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = row0 + 32 * i + acc_row(v, lane), c = col0 + 32 * j + col;
          old[j][v] = __builtin_nontemporal_load(&Gp[(size_t)r * ld + c]);
        }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const float scj = ssc[BM + cl + 32 * j + col];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = row0 + 32 * i + acc_row(v, lane), c = col0 + 32 * j + col;
          const float sr = ssc[rl + 32 * i + acc_row(v, lane)];
          if (c <= r + 63) Gp[(size_t)r * ld + c] = old[j][v] - acc[i][j][v] * (sr * scj);
        }
      }
    }
  }
};

// Rows K1 .. ld of the outer panel (columns K0 .. K1 = K0 + 256), once its
// 256 x 256 diagonal block is factored: for each 64-column block k in order,
// the panel step L_rk = A_rk L_kk^-T (with the stored inverse), then the
// update of the panel's later blocks j, A_rj -= L_rk L_jk^T; then the rows' L
// is written back with the fp16 hi / lo planes of the left-looking updates'
// operand.  A workgroup keeps ROWS rows x 256 columns in LDS, so the strip is
// read and written once instead of once per step; each ROWS x 64 product is
// ROWS / 32 x 2 waves of 32 x 32.
// Bound by each wave's chain of ten steps.  At 8 pairs of ld = 1792: 29.1 us with
// the products' elements going to LDS one at a time (64 operations per wave and
// update) and B split between the barriers; 25.0 us with four at a time and the
// next B split under the products; 22.3 us with strips of 64 rows, one wave per
// SIMD, which is taken while every such strip has a CU of its own (kStripFew).
//
// k_chol_strip16: the strip on fp16 MFMA (32x32x16), every product as hi.hi + hi.lo +
// lo.hi of fp16 planes (about 2^-22 relative, as in the trailing
// contraction).  With s_x = 2^shift[x] (sqrt(A_xx) s_x in [2^13, 2^14)):
//  - an entry of a block not yet factored, |A'_rc| <= sqrt(A_rr A_cc), is held
//    as A'_rc s_r s_c 2^-14, a factored one, |L_rc| <= sqrt(A_rr), as L_rc s_r,
//    both below 2^14, as hi / lo planes in LDS;
//  - the B operand rows (D_k with its columns m scaled by 2^14 / s_m, or L_jk)
//    are split after scaling each row by the power of two that brings its
//    largest magnitude into [2^13, 2^14);
//  - an update recombines hi + lo in fp32, subtracts and splits again.
// The planes left in LDS are the split the left-looking contractions read,
// and G gets (hi + lo) / s_r.  LDS rows are unpadded with their 16-byte chunks XOR-swizzled by
// row, so each quarter-wave's fragment reads touch 16 distinct bank groups.
constexpr int kStripFew = 256;   // strips of 64 rows that still have a CU each
constexpr size_t strip16_lds(int rows) {
  return ((size_t)2 * rows * 256 + (size_t)2 * kNB * kNB) * sizeof(f16) + (size_t)(kNB + rows + 256) * sizeof(int32_t);
}

// max(v, the lane that the DPP control CTRL names).
template <int CTRL>
__device__ __forceinline__ float row_max(float v) {
  return fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true)));
}

template <int ROWS>
__global__ void __launch_bounds__(4 * ROWS) __attribute__((amdgpu_waves_per_eu(1, 2)))
k_chol_strip16(float *__restrict__ Gw, int64_t ld, int K0, const float *__restrict__ dinv, f16 *__restrict__ Lp,
               const int32_t *__restrict__ shift, const int32_t *__restrict__ info) {
  extern __shared__ __attribute__((aligned(16))) char strip16_smem[];
  f16 *sTh = reinterpret_cast<f16 *>(strip16_smem);        // [ROWS][256] hi
  f16 *sTl = sTh + ROWS * 256;                               // [ROWS][256] lo
  f16 *sBh = sTl + ROWS * 256;                               // [64][64] hi
  f16 *sBl = sBh + kNB * kNB;                                // [64][64] lo
  float *sBs = reinterpret_cast<float *>(sBl + kNB * kNB);   // [64] scales that take a product with B's rows to its units
  int32_t *sSh = reinterpret_cast<int32_t *>(sBs + kNB);     // [ROWS] row shifts of the strip
  int32_t *sShC = sSh + ROWS;                                // [256] shifts of the panel's columns
  constexpr int kThreads = 4 * ROWS, kB = kNB * kNB / 4 / kThreads;   // quads of B per thread
  const int b = blockIdx.y;
  if (info[b] != 0) return;   // uniform over the workgroup
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5, col = lane & 31;
  const int K1 = K0 + 256;
  const int64_t R = K1 + (int64_t)blockIdx.x * ROWS;
  float *G = Gw + (size_t)b * ld * ld;
  const int nb = (int)(ld / kNB);
  // element (r, c) of a plane: T rows of 32 chunks, B rows of 8 chunks
  auto tix = [](int r, int c) { return r * 256 + 8 * ((c >> 3) ^ (r & 15)) + (c & 7); };
  auto bix = [](int i, int m) { return i * kNB + 8 * ((m >> 3) ^ ((i >> 1) & 7)) + (m & 7); };
  auto split4 = [](f32x4 x, f16x4 &hi, f16x4 &lo) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      hi[q] = (f16)x[q];
      lo[q] = (f16)(x[q] - (float)hi[q]);
    }
  };
  if (tid < ROWS) sSh[tid] = shift[(size_t)b * ld + R + tid];
  if (tid < 256) sShC[tid] = shift[(size_t)b * ld + K0 + tid];
  constexpr int kSteps = 10;
  constexpr int8_t step_k[kSteps] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3};
  constexpr int8_t step_j[kSteps] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};
  f32x4 pre[2][kB];   // of steps st + 1 and st + 2
  auto load_b = [&](int st) {
    const int k = step_k[st], j = step_j[st];
    const float *src = j == k ? dinv + ((size_t)b * nb + K0 / kNB + k) * kNB * kNB
                              : G + (size_t)(K0 + kNB * j) * ld + K0 + kNB * k;
    const int64_t lds = j == k ? kNB : ld;
#pragma unroll
    for (int c = 0; c < kB; ++c) {
      const int e = tid + kThreads * c, i = e >> 4, c4 = (e & 15) * 4;
      pre[st & 1][c] = *reinterpret_cast<const f32x4 *>(src + (size_t)i * lds + c4);
    }
  };
  // B rows scaled by their own power of two (16 consecutive lanes hold a row);
  // for D_k its columns first take 2^14 / s_m
  f16x4 bhi[kB], blo[kB];
  float bsc[kB];
  auto split_b = [&](int st) {
    const int k = step_k[st], j = step_j[st];
    const bool panel = j == k;
#pragma unroll
    for (int c = 0; c < kB; ++c) {
      const int e = tid + kThreads * c, i = e >> 4, c4 = (e & 15) * 4;
      f32x4 x = pre[st & 1][c];
      if (panel) {
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = ldexpf(x[q], 14 - sShC[64 * k + c4 + q]);
      }
      float m = fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3])));
      m = row_max<0xB1>(m);    // lanes 1 apart, 2 apart,
      m = row_max<0x4E>(m);
      m = row_max<0x141>(m);   // the other half of 8, the other half of 16
      m = row_max<0x140>(m);
      int ex = 0;
      if (m > 0.0f) frexpf(m, &ex);
      const int sc = max(min(14 - ex, 126), -126);
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = ldexpf(x[q], sc);
      split4(x, bhi[c], blo[c]);
      bsc[c] = ldexpf(1.0f, panel ? -sc : sShC[64 * j + i] - 14 - sc);
    }
  };
  auto stash_b = [&]() {
#pragma unroll
    for (int c = 0; c < kB; ++c) {
      const int e = tid + kThreads * c, i = e >> 4, c4 = (e & 15) * 4;
      *reinterpret_cast<f16x4 *>(&sBh[bix(i, c4)]) = bhi[c];
      *reinterpret_cast<f16x4 *>(&sBl[bix(i, c4)]) = blo[c];
      if ((e & 15) == 0) sBs[i] = bsc[c];
    }
  };
  // this wave's 32 x 32 block of T[:, 64 ka ..] x B^T, in the scaled units: with B as
  // the first operand a lane holds row arow, its columns 32 wn + 8 q + 4 h .. + 3 in
  // accumulators 4 q .. 4 q + 3, which go to LDS four at a time
  const int arow = 32 * wm + col, brow = 32 * wn + col;
  auto product = [&](int ka) {
    f32x16 acc = zero16();
#pragma unroll
    for (int ks = 0; ks < kNB / 16; ++ks) {
      const int ca = 64 * ka + 16 * ks + 8 * h, cb = 16 * ks + 8 * h;
      const bf16x8 ah = *reinterpret_cast<const bf16x8 *>(&sTh[tix(arow, ca)]);
      const bf16x8 al = *reinterpret_cast<const bf16x8 *>(&sTl[tix(arow, ca)]);
      const bf16x8 bh = *reinterpret_cast<const bf16x8 *>(&sBh[bix(brow, cb)]);
      const bf16x8 bl = *reinterpret_cast<const bf16x8 *>(&sBl[bix(brow, cb)]);
      acc = mma16<f16>(bh, ah, acc);
      acc = mma16<f16>(bl, ah, acc);
      acc = mma16<f16>(bh, al, acc);
    }
    return acc;
  };
  {  // the strip, ROWS rows x 64 groups of 4, scaled by s_r s_c 2^-14 and split
    f32x4 v[ROWS * 64 / kThreads];
#pragma unroll
    for (int i = 0; i < ROWS * 64 / kThreads; ++i) {
      const int e = tid + kThreads * i, r = e >> 6, c4 = (e & 63) * 4;
      v[i] = *reinterpret_cast<const f32x4 *>(G + (size_t)(R + r) * ld + K0 + c4);
    }
    load_b(0);
    load_b(1);
    __syncthreads();   // sSh, sShC
#pragma unroll
    for (int i = 0; i < ROWS * 64 / kThreads; ++i) {
      const int e = tid + kThreads * i, r = e >> 6, c4 = (e & 63) * 4;
      const int sh = sSh[r] - 14;
      f32x4 x;
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = ldexpf(v[i][q], sh + sShC[c4 + q]);
      f16x4 hi, lo;
      split4(x, hi, lo);
      *reinterpret_cast<f16x4 *>(&sTh[tix(r, c4)]) = hi;
      *reinterpret_cast<f16x4 *>(&sTl[tix(r, c4)]) = lo;
    }
  }
  split_b(0);
  // block kb (final after its panel step): planes and L = (hi + lo) / s_r of
  // all ROWS rows, four columns per thread-group, issued while later steps run
  f16 *hib = Lp + (size_t)b * 2 * ld * ld, *lob = hib + (size_t)ld * ld;
  auto write_block = [&](int kb) {
#pragma unroll
    for (int q = 0; q < ROWS * 16 / kThreads; ++q) {
      const int g = tid + kThreads * q, rr = g >> 4, c = 64 * kb + (g & 15) * 4;
      const int64_t r = R + rr;
      const f16x4 hi = *reinterpret_cast<const f16x4 *>(&sTh[tix(rr, c)]);
      const f16x4 lo = *reinterpret_cast<const f16x4 *>(&sTl[tix(rr, c)]);
      const float us = ldexpf(1.0f, -sSh[rr]);
      f32x4 x;
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = ((float)hi[u] + (float)lo[u]) * us;
      *reinterpret_cast<f32x4 *>(G + (size_t)r * ld + K0 + c) = x;
      *reinterpret_cast<f16x4 *>(hib + (size_t)r * ld + K0 + c) = hi;
      *reinterpret_cast<f16x4 *>(lob + (size_t)r * ld + K0 + c) = lo;
    }
  };
#pragma unroll
  for (int st = 0; st < kSteps; ++st) {
    const int k = step_k[st], j = step_j[st];
    __syncthreads();   // the strip is up to date and every wave is done with sB
    if (st > 0 && step_j[st - 1] == step_k[st - 1]) write_block(step_k[st - 1]);
    stash_b();
    if (st + 2 < kSteps) load_b(st + 2);
    __syncthreads();
    const f32x16 acc = product(k);
    if (st + 1 < kSteps) split_b(st + 1);   // under the products
    // panel step: L_k s_r replaces block k, once every wave has read it; update of
    // block j (this wave's own entries), in its units s_r s_c 2^-14
    if (j == k) __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cl = 32 * wn + 8 * q + 4 * h;
      const f32x4 sc = *reinterpret_cast<const f32x4 *>(&sBs[cl]);
      f16x4 &th = *reinterpret_cast<f16x4 *>(&sTh[tix(arow, 64 * j + cl)]);
      f16x4 &tl = *reinterpret_cast<f16x4 *>(&sTl[tix(arow, 64 * j + cl)]);
      f32x4 x;
      if (j == k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = acc[4 * q + e] * sc[e];
      } else {
        const f16x4 hi = th, lo = tl;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = ((float)hi[e] + (float)lo[e]) - acc[4 * q + e] * sc[e];
      }
      f16x4 hi, lo;
      split4(x, hi, lo);
      th = hi;
      tl = lo;
    }
  }
  __syncthreads();
  write_block(step_k[kSteps - 1]);   // the last panel step's block
}

// Per-row shifts of the left-looking updates' operand.  |L_rk| <= sqrt(A_rr)
// for every k (row r of L L^T = A), so 2^sh with sqrt(A_rr) 2^sh in
// [2^13, 2^14) keeps every scaled entry of the row below 2^14, inside fp16's
// range with the lo part carrying the next 11 bits; one shift per row for the
// whole factorisation lets a contraction run over all earlier panels at once.
// shift[r] = sh, inv[r] = 2^-sh (rows of a non-positive diagonal get 0: their
// factorisation fails at that pivot).
__global__ void __launch_bounds__(256) k_chol_scales(const float *__restrict__ Gw, int64_t ld,
                                                     int32_t *__restrict__ shift, float *__restrict__ inv,
                                                     const int32_t *__restrict__ info) {
  const int b = blockIdx.y;
  if (info[b] != 0) return;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= ld) return;
  const float d = Gw[(size_t)b * ld * ld + (size_t)r * ld + r];
  int sh = 0;
  if (d > 0.0f && isfinite(d)) {
    int ex = 0;
    frexpf(sqrtf(d), &ex);   // sqrt(d) = f 2^ex, f in [0.5, 1)
    sh = max(min(14 - ex, 126), -126);
  }
  shift[(size_t)b * ld + r] = sh;
  inv[(size_t)b * ld + r] = ldexpf(1.0f, -sh);
}

// ------------------------------------------------- inverses of the 256-wide diagonal blocks
// D_K = L_KK^-1, 256 x 256 lower triangular in fp32, for the value fit's solves,
// which then take ld / 256 steps.  It is kept in the unused diagonal block of
// the planes of L (the contractions read rows below a panel only): of row r,
// columns 0 .. 127 in the hi plane's 512 bytes at (K0 + r, K0) and columns
// 128 .. 255 in the lo plane's.  The four 64 x 64 diagonal blocks are stored
// with their zeros above the diagonal, the other upper entries are not stored.
struct DiagInv {
  const float *hi, *lo;   // row 0 of either half
  int64_t ldf;            // floats between rows
  __device__ __forceinline__ const float *at(int r, int c) const {   // four columns from c, c a multiple of 4
    return (c < 128 ? hi + c : lo + (c - 128)) + (size_t)r * ldf;
  }
};

__device__ inline DiagInv diag_inv(const void *lsplit, int64_t ld, int b, int64_t K0) {
  const f16 *p = reinterpret_cast<const f16 *>(lsplit) + (size_t)b * 2 * ld * ld + (size_t)K0 * ld + K0;
  return {reinterpret_cast<const float *>(p), reinterpret_cast<const float *>(p + (size_t)ld * ld), ld / 2};
}

// 16 x 16 fp32 tiles in LDS and in registers share one layout: element (r, c)
// at float 64 (c / 4) + 4 r + c % 4, so lane l = 16 g + r holds columns
// 4 g .. 4 g + 3 of row r as four consecutive floats (one conflict-free 16-byte
// access per lane).  tile_mac(acc, X, Y) adds X Y^T: with the MFMA's operands
// given as (Y, X) its output lands in this layout again, so a result feeds the
// next product without leaving the registers.
__device__ inline f32x4 tile_mac(f32x4 acc, f32x4 x, f32x4 y) {
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(y[s], x[s], acc, 0, 0, 0);
  return acc;
}

// After the factorisation, the lower 16 x 16 tiles of L and the inverses of its
// diagonal tiles (from dinv) in LDS; a wave solves one tile column j of X = L^-1
// by substitution, X_ij = -X_ii sum_m L_im X_mj, its tiles transposed in registers.
// Columns are independent, so no barrier.  One workgroup of 16 waves per (block,
// pair) is bound by the CU's fp32 MFMA rate; while there are few of them, four
// workgroups of four waves and four columns each (z, 7 - z, 8 + z, 15 - z) share
// a block, with the registers to read a whole tile row of L ahead of its products:
// 26 -> 18 us at 8 pairs of ld = 1024, 28 -> 19 us at ld = 1792.
constexpr size_t kInv256Lds = (size_t)136 * 256 * sizeof(float);

template <int NW>
__global__ void __launch_bounds__(64 * NW) k_chol_inv256(const float *__restrict__ Gw, int64_t ld, int t,
                                                         const float *__restrict__ dinv, void *__restrict__ lsplit,
                                                         const int32_t *__restrict__ info) {
  extern __shared__ __attribute__((aligned(16))) float diag_smem[];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  if (info[b] != 0) return;   // uniform over the workgroup
  const int64_t K0 = (int64_t)blockIdx.x * 256;
  const int nk = (int)((t - K0 + 15) / 16);   // tile rows that are not padding
  auto tile = [&](int i, int m) { return diag_smem + (i * (i + 1) / 2 + m) * 256; };
  auto get = [&](int i, int m) { return *reinterpret_cast<const f32x4 *>(tile(i, m) + 4 * lane); };
  for (int i = wave; i < 16; i += NW) {   // tile row i
    const float *grow = Gw + (size_t)b * ld * ld + (size_t)(K0 + 16 * i + r) * ld + K0 + 4 * g;
    const float *drow = dinv + ((size_t)b * (ld / kNB) + K0 / kNB + (i >> 2)) * kNB * kNB +
                        (16 * (i & 3) + r) * kNB + 16 * (i & 3) + 4 * g;
    f32x4 v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m)
      if (m <= i) v[m] = *reinterpret_cast<const f32x4 *>(m < i ? grow + 16 * m : drow);
#pragma unroll
    for (int m = 0; m < 16; ++m)
      if (m <= i) *reinterpret_cast<f32x4 *>(tile(i, m) + 4 * lane) = v[m];
  }
  __syncthreads();
  const int z = blockIdx.z;
  const int j = NW == 16 ? wave : wave == 0 ? z : wave == 1 ? 7 - z : wave == 2 ? 8 + z : 15 - z;
  float *out = const_cast<float *>(diag_inv(lsplit, ld, b, K0).at(0, j < 8 ? 0 : 128)) + 16 * (j & 7) + r;
  const int64_t ldf = ld / 2;
  f32x4 xt[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (i == j) {
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = tile(j, j)[64 * (r >> 2) + 4 * (4 * g + v) + (r & 3)];
    } else if (i > j && i < nk) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
      if constexpr (NW == 4) {   // the row's tiles of L first, and no branches between the products
        f32x4 l[16];
#pragma unroll
        for (int m = 0; m <= i; ++m) l[m] = get(i, m);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < i; ++m) {   // (xt[m] is zero for m < j)
          if (m & 1) s1 = tile_mac(s1, xt[m], l[m]);
          else s0 = tile_mac(s0, xt[m], l[m]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) s0[v] = -(s0[v] + s1[v]);
        x = tile_mac(x, s0, l[i]);
      } else {
#pragma unroll
        for (int m = 0; m < i; ++m)
          if (m >= j) {
            if (m & 1) s1 = tile_mac(s1, xt[m], get(i, m));
            else s0 = tile_mac(s0, xt[m], get(i, m));
          }
#pragma unroll
        for (int v = 0; v < 4; ++v) s0[v] = -(s0[v] + s1[v]);
        x = tile_mac(x, s0, get(i, i));
      }
    }
    xt[i] = x;
    if (i >= (j & ~3)) {   // with the zero tiles above the diagonal inside the 64 x 64 block
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(size_t)(16 * i + 4 * g + v) * ldf] = x[v];
    }
  }
}

// --------------------------------------------------------------- one right-hand side
// The sum over each 16 consecutive lanes, in every one of them.
template <int CTRL>
__device__ __forceinline__ double row16_add(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return v + __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
__device__ __forceinline__ double row16_sum(double v) {   // rotations by 8, 4, 2 and 1 lanes
  return row16_add<0x121>(row16_add<0x122>(row16_add<0x124>(row16_add<0x128>(v))));
}

// One-rhs triangular solves, float64 vectors, right-looking over 256-row
// blocks K with one launch per block:
//   forward  L y = rhs:   L_KK y_K = s_K,     s_i -= L_iK y_K      (rows i below)
//   backward L^T x = y:   L_KK^T x_K = y_K,   y_i -= L_Ki^T x_K    (columns i before)
// Every workgroup forms the block solution in four steps of 64 rows with the
// inverses D_k of the 64 x 64 diagonal blocks (dinv), and updates `per` chunks
// of 64 targets; workgroup 0 also writes the solution (and adds it to `acc` on
// the backward pass when given).  Forward step 0 reads the rhs, later steps the
// work vector s; the backward pass updates y in place.  The steps of 64 are part of
// the result: with fp32 inverses of whole 256 x 256 blocks the refinement of
// nearly square systems ends elsewhere (t = 3277, n = 4096: biases 1.7e-4 apart in
// norm).  Bound by the launches, the two dependent reads and the four steps of
// one: 8 pairs at t = 1638, 8.0 and 8.4 us forward and backward (7.4 and 7.5 with the
// inverse of the whole block, which takes 19 us per factorisation to form; 64-row
// blocks with a launch each, four launches of 4.3 us); 256 pairs at t = 3277: 18.5 -> 18.0
// ms for the mass fit's solve stage with its residuals.
template <bool FWD>
__global__ void __launch_bounds__(1024) k_trsv256(const float *__restrict__ Gw, const float *__restrict__ dinv,
                                                  int64_t ld, int K, int per, const double *__restrict__ rhs,
                                                  double *__restrict__ work, double *__restrict__ out,
                                                  double *__restrict__ acc, const int32_t *__restrict__ info) {
  constexpr int SR = 68;   // stride of red: 16 rows of one column in different banks
  __shared__ __attribute__((aligned(16))) double sv[256], sol[256];
  __shared__ double red[FWD ? 1 : 3 * 16 * SR];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t skip = info[b];   // looked at after the loads: they need not wait for it
  const int64_t K0 = (int64_t)K * 256;
  const int nch = (int)(FWD ? (ld - K0 - 256) / 64 : K0 / 64);   // chunks of 64 targets
  const int ch0 = blockIdx.x * per, ch1 = min(ch0 + per, nch);
  const float *L = Gw + (size_t)b * ld * ld;
  const float *LK = L + (size_t)K0 * ld + K0;                          // the diagonal block
  const float *D = dinv + ((size_t)b * (ld / kNB) + K0 / kNB) * kNB * kNB;   // its four inverses
  const double *src = (FWD && K == 0 ? rhs : work) + (size_t)b * ld;
  const double own = src[K0 + (tid & 255)];
  // the chunk's part of L, loaded ahead of its use: forward 16 lanes per
  // target row, backward 16 lanes per row of the block
  const int q = tid & 15, rg = tid >> 4;
  f32x4 lv[4];
  double old = 0.0;   // the target's value before the update
  const double *prev = (FWD && K == 0 ? rhs : work) + (size_t)b * ld;
  auto load_l = [&](int ch) {
    old = prev[FWD ? K0 + 256 + 64 * ch + rg : (int64_t)64 * ch + lane];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      lv[u] = *reinterpret_cast<const f32x4 *>(FWD ? L + (size_t)(K0 + 256 + 64 * ch + rg) * ld + K0 + 4 * (q + 16 * u)
                                                   : L + (size_t)(K0 + rg + 64 * u) * ld + 64 * ch + 4 * q);
  };
  // d[k]: the thread's part of D_k; l[j (j - 1) / 2 + k]: of block (j, k) of L, j > k.
  // Forward: row rg, columns 4 q .. + 3; backward: rows 4 wave .. + 3, column lane.
  f32x4 d[4], l[6];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (FWD) {
      d[k] = *reinterpret_cast<const f32x4 *>(D + (kNB * k + rg) * kNB + 4 * q);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) d[k][e] = D[(kNB * k + 4 * wave + e) * kNB + lane];
    }
  }
#pragma unroll
  for (int j = 1; j < 4; ++j)
#pragma unroll
    for (int k = 0; k < j; ++k) {
      f32x4 &v = l[j * (j - 1) / 2 + k];
      if constexpr (FWD) {
        v = *reinterpret_cast<const f32x4 *>(LK + (size_t)(kNB * j + rg) * ld + kNB * k + 4 * q);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = LK[(size_t)(kNB * j + 4 * wave + e) * ld + kNB * k + lane];
      }
    }
  if (ch0 < ch1) load_l(ch0);
  if (tid < 256) sv[tid] = own;
  __syncthreads();
  if (skip != 0) return;   // uniform over the workgroup
  auto dot4 = [](f32x4 x, const double *v) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fma((double)x[e], v[e], s);
    return s;
  };
  if constexpr (FWD) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double s = row16_sum(dot4(d[k], sv + kNB * k + 4 * q));
      if (q == 0) sol[kNB * k + rg] = s;
      __syncthreads();
      if (k == 3) break;
#pragma unroll
      for (int j = k + 1; j < 4; ++j) {
        const double u = row16_sum(dot4(l[j * (j - 1) / 2 + k], sol + kNB * k + 4 * q));
        if (q == 0) sv[kNB * j + rg] -= u;
      }
      __syncthreads();
    }
  } else {
#pragma unroll
    for (int k = 3; k >= 0; --k) {
      red[wave * SR + lane] = dot4(d[k], sv + kNB * k + 4 * wave);
      __syncthreads();
      const double s = row16_sum(red[q * SR + rg]);
      if (q == 0) sol[kNB * k + rg] = s;
      __syncthreads();
      if (k == 0) break;
#pragma unroll
      for (int j = 0; j < k; ++j)
        red[(16 * j + wave) * SR + lane] = dot4(l[k * (k - 1) / 2 + j], sol + kNB * k + 4 * wave);
      __syncthreads();
#pragma unroll
      for (int j = 0; j < k; ++j) {
        const double u = row16_sum(red[(16 * j + q) * SR + rg]);
        if (q == 0) sv[kNB * j + rg] -= u;
      }
      __syncthreads();
    }
  }
  if (blockIdx.x == 0 && tid < 256) {
    out[(size_t)b * ld + K0 + tid] = sol[tid];
    if (!FWD && acc) acc[(size_t)b * ld + K0 + tid] += sol[tid];
  }
  for (int ch = ch0; ch < ch1; ++ch) {   // uniform over the workgroup
    if constexpr (FWD) {
      double s = 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) s = fma((double)lv[u][e], sol[4 * (q + 16 * u) + e], s);
      const double base = old;
      if (ch + 1 < ch1) load_l(ch + 1);
#pragma unroll
      for (int m = 8; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
      if (q == 0) work[(size_t)b * ld + K0 + 256 + 64 * ch + rg] = base - s;
    } else {
      double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double v = sol[rg + 64 * u];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = fma((double)lv[u][e], v, s[e]);
      }
      const double base = old;
      if (ch + 1 < ch1) load_l(ch + 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[e] += __shfl_xor(s[e], 16, 64);
        s[e] += __shfl_xor(s[e], 32, 64);
      }
      __syncthreads();   // the previous use of red is over
      if (lane < 16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave * SR + 4 * lane + e] = s[e];
      }
      __syncthreads();
      if (tid < 64) {
        double x = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) x += red[w * SR + tid];
        work[(size_t)b * ld + 64 * ch + tid] = base - x;
      }
    }
  }
}

// Refinement residual of the mass fit computed from the data, not from the
// float32 Gram: res = Phi_C^T (m - Phi_C w) - lam w with Phi_C = exp(L^T - z)
// re-evaluated in fp32 and every sum in float64.
// Optional key lists restrict either stage to a subset of the compact keys
// (list [P][tp], count [P]): the exact non-negative fit sums only over its free
// keys (w = 0 elsewhere) and needs each residual only on one side of its
// partition.  Without a list every key r < t takes part.
// Stage 1: u_i = m_i - sum_{r<t} Phi[i][r] w_r.  64 queries per workgroup, four
// per lane (16-byte loads of the L^T rows, 256-byte runs); the 32 groups of 16
// lanes take the compact keys r = group (mod 32), four of them in flight, and
// their partial sums meet in LDS.  256 queries per workgroup of four waves left
// a call over few pairs with long serial sums on half of the CUs:
// 143 -> 48 us a call for 8
// pairs at n = 4096, t = 1638.
__global__ void __launch_bounds__(512) k_mass_resid_rows(const float *__restrict__ LT, const float *__restrict__ z,
                                                         const float *__restrict__ m, const double *__restrict__ w,
                                                         int n, int t, int64_t tp, int64_t np_,
                                                         double *__restrict__ u, const int32_t *__restrict__ info,
                                                         const int32_t *__restrict__ list,
                                                         const int32_t *__restrict__ count) {
  constexpr int NG = 32;
  __shared__ double red[8][64];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = tid & 15, grp = tid >> 4;
  if (info[b] != 0) return;
  const int i0 = blockIdx.x * 64 + 4 * q;
  const float *L = LT + (size_t)b * tp * np_ + i0;   // L^T rows are zero beyond n
  const double *wb = w + (size_t)b * tp;
  const int32_t *lb = list ? list + (size_t)b * tp : nullptr;
  const int c = list ? count[b] : t;
  float zi[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) zi[k] = i0 + k < n ? z[(size_t)b * n + i0 + k] : 0.0f;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  auto term = [&](f32x4 v, double wr) {
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] += (double)expf(v[k] - zi[k]) * wr;
  };
  int k = grp;
  for (; k + 3 * NG < c; k += 4 * NG) {
    f32x4 v[4];
    double wr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = lb ? lb[k + e * NG] : k + e * NG;
      v[e] = *reinterpret_cast<const f32x4 *>(L + (size_t)r * np_);
      wr[e] = wb[r];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) term(v[e], wr[e]);
  }
  for (; k < c; k += NG) {
    const int r = lb ? lb[k] : k;
    term(*reinterpret_cast<const f32x4 *>(L + (size_t)r * np_), wb[r]);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {   // the wave's four groups
    a[e] += __shfl_xor(a[e], 16, 64);
    a[e] += __shfl_xor(a[e], 32, 64);
    if (lane < 16) red[wave][4 * lane + e] = a[e];
  }
  __syncthreads();
  if (tid < 64) {
    const int i = blockIdx.x * 64 + tid;
    double acc = 0.0;
#pragma unroll
    for (int wv = 0; wv < 8; ++wv) acc += red[wv][tid];
    u[(size_t)b * np_ + i] = i < n ? (double)m[(size_t)b * n + i] - acc : 0.0;
  }
}

// Stage 2: res_r = sum_i Phi[i][r] u_i - lam w_r.  A workgroup takes four
// compact keys, so that the z and u loads are shared by them, and each of its four
// waves every fourth run of 256 queries, four per lane (16-byte loads of the L^T
// rows and of u); the waves' sums meet in LDS.  Bound by the reads of L^T; a wave
// that swept all queries of its keys alone was bound by their latency: 36 -> 21 us
// at 8 pairs of n = 4096, t = 819, 56 -> 41 us at t = 1638; 64 pairs at t = 3277,
// 615 -> 598 us.
// With a list, slot k handles key list[k] (k < count) and writes only there.
constexpr int kResKeys = 4;   // compact keys per workgroup
__global__ void __launch_bounds__(256) k_mass_resid_cols(const float *__restrict__ LT, const float *__restrict__ z,
                                                         const double *__restrict__ u, const double *__restrict__ w,
                                                         const float *__restrict__ lam, int n, int t, int64_t tp,
                                                         int64_t np_, double *__restrict__ res,
                                                         const int32_t *__restrict__ info,
                                                         const int32_t *__restrict__ list,
                                                         const int32_t *__restrict__ count) {
  typedef __attribute__((__vector_size__(2 * sizeof(double)))) double f64x2;
  __shared__ double red[4][kResKeys];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k0 = blockIdx.x * kResKeys;   // first slot of this workgroup
  if (info[b] != 0) return;
  const int lim = list ? count[b] : t;   // slots k < lim are live keys
  if (k0 >= lim) {   // uniform over the workgroup
    if (!list && tid < kResKeys) res[(size_t)b * tp + k0 + tid] = 0.0;   // padding keys r >= t
    return;
  }
  int r[kResKeys];
  const float *row[kResKeys];
#pragma unroll
  for (int q = 0; q < kResKeys; ++q) {
    const int k = k0 + q < lim ? k0 + q : lim - 1;   // dead slots repeat a live key, unstored
    r[q] = list ? list[(size_t)b * tp + k] : k;
    row[q] = LT + ((size_t)b * tp + r[q]) * np_;
  }
  const float *zb = z + (size_t)b * n;
  const double *ub = u + (size_t)b * np_;   // zero beyond n
  double acc[kResKeys] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int i0 = 256 * wave + 4 * lane; i0 < n; i0 += 1024) {
    const f64x2 u01 = *reinterpret_cast<const f64x2 *>(ub + i0);
    const f64x2 u23 = *reinterpret_cast<const f64x2 *>(ub + i0 + 2);
    const double uu[4] = {u01[0], u01[1], u23[0], u23[1]};
    float zz[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) zz[e] = zb[i0 + e < n ? i0 + e : n - 1];
#pragma unroll
    for (int q = 0; q < kResKeys; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(row[q] + i0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double term = (double)expf(v[e] - zz[e]) * uu[e];
        acc[q] += i0 + e < n ? term : 0.0;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kResKeys; ++q) {
    const double sum = wave_sum(acc[q]);
    if (lane == 0) red[wave][q] = sum;
  }
  __syncthreads();
  if (tid < kResKeys) {
    const int k = k0 + tid;
    if (k < lim) {
      const int rk = list ? list[(size_t)b * tp + k] : k;
      const double sum = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
      res[(size_t)b * tp + rk] = sum - (double)lam[b] * w[(size_t)b * tp + rk];
    } else if (!list) {
      res[(size_t)b * tp + k] = 0.0;   // padding keys r >= t
    }
  }
}

// beta = clip(log(max(max(w, 0), eps)), bmin, bmax); NaN for failed pairs.
__global__ void __launch_bounds__(256) k_bias_finalize(const double *__restrict__ w, int64_t ld, int t, float eps,
                                                       float bmin, float bmax, const int32_t *__restrict__ info,
                                                       float *__restrict__ beta, float *__restrict__ beta_ws) {
  const int b = blockIdx.y;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= ld) return;
  float v = 0.0f;
  if (r < t) {
    if (info[b] != 0) {
      v = NAN;
    } else {
      const double wv = w[(size_t)b * ld + r];
      const double ws = wv > 0.0 ? wv : 0.0;
      v = (float)log(ws > (double)eps ? ws : (double)eps);
      v = fminf(fmaxf(v, bmin), bmax);
    }
    beta[(size_t)b * t + r] = v;
  }
  if (beta_ws) beta_ws[(size_t)b * ld + r] = v;
}

// --------------------------------------------------------------- value-fit operands
// P^T[r][i] = softmax_r(L^T[r][i] + beta_r) for r < t, i < n (own column max),
// split into bf16 hi/lo planes (or fp32), written in both layouts the value fit
// contracts over: PT [planes][tp][np] and, if Pm is given, Pm [planes][np][tp].
// A workgroup takes 64 queries: each wave first runs an online max/sum over the
// compact keys r = wave (mod 4) and the four partial (max, sum) pairs are
// merged in LDS; then the 64 x 64 (r, i) tiles are formed, stored row-wise into
// PT and, through an LDS transpose, into Pm.
template <typename T>
__global__ void __launch_bounds__(256) k_phat(const float *__restrict__ LT, const float *__restrict__ beta, int n,
                                              int t, int64_t tp, int64_t np_, void *__restrict__ out,
                                              void *__restrict__ outm) {
  constexpr int PL = sizeof(T) == 2 ? 2 : 1;
  __shared__ float smx[4][64], ssum[4][64];
  __shared__ __attribute__((aligned(16))) T sp[PL][64][64 + 8];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.x * 64, i = i0 + lane;
  const float *L = LT + (size_t)b * tp * np_ + i;
  const float *bb = beta + (size_t)b * tp;
  // exp(d) for d = x - max <= 0 as the hardware 2^(d log2(e)); the online max
  // advances eight keys at a time and rescales the running sum only when the
  // lane's maximum grew.
  constexpr float kLog2e = 1.4426950408889634f;
  float mx = -INFINITY, sum = 0.0f;
  if (i < n) {
    int r = wave;
    for (; r + 28 < t; r += 32) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = L[(size_t)(r + 4 * u) * np_] + bb[r + 4 * u];
      float cm = x[0];
#pragma unroll
      for (int u = 1; u < 8; ++u) cm = fmaxf(cm, x[u]);
      if (cm > mx) {
        sum *= __builtin_amdgcn_exp2f((mx - cm) * kLog2e);
        mx = cm;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += __builtin_amdgcn_exp2f((x[u] - mx) * kLog2e);
    }
    for (; r < t; r += 4) {
      const float x = L[(size_t)r * np_] + bb[r];
      if (x > mx) {
        sum *= __builtin_amdgcn_exp2f((mx - x) * kLog2e);
        mx = x;
      }
      sum += __builtin_amdgcn_exp2f((x - mx) * kLog2e);
    }
  }
  smx[wave][lane] = mx;
  ssum[wave][lane] = sum;
  __syncthreads();
  const float M = fmaxf(fmaxf(smx[0][lane], smx[1][lane]), fmaxf(smx[2][lane], smx[3][lane]));
  float S = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    S += smx[q][lane] == -INFINITY ? 0.0f : ssum[q][lane] * __builtin_amdgcn_exp2f((smx[q][lane] - M) * kLog2e);
  const float inv = (i < n && S > 0.0f) ? 1.0f / S : 0.0f;
  T *PT = reinterpret_cast<T *>(out) + (size_t)b * PL * tp * np_;
  T *Pm = reinterpret_cast<T *>(outm) + (size_t)b * PL * tp * np_;
  constexpr int EPV = 16 / sizeof(T);                     // elements per 16-byte store
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  // this wave's 16 keys of the next tile: logits and biases loaded while the
  // current tile is stored
  float ln[16], bn[16];
  auto fetch_l = [&](int64_t q0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int64_t r = q0 + 16 * wave + e;
      const bool ok = i < n && r < t;
      ln[e] = ok ? L[(size_t)r * np_] : 0.0f;
      bn[e] = ok ? bb[r] : 0.0f;
    }
  };
  fetch_l(0);
  for (int64_t r0 = 0; r0 < tp; r0 += 64) {
    __syncthreads();   // the previous tile's stores have read sp
    float lc[16], bc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      lc[e] = ln[e];
      bc[e] = bn[e];
    }
    if (r0 + 64 < tp) fetch_l(r0 + 64);
#pragma unroll
    for (int e4 = 0; e4 < 16; e4 += 4) {   // four consecutive keys per LDS write
      float pv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t r = r0 + 16 * wave + e4 + e;
        pv[e] = (i < n && r < t) ? __builtin_amdgcn_exp2f((lc[e4 + e] + bc[e4 + e] - M) * kLog2e) * inv : 0.0f;
      }
      const int rr = 16 * wave + e4;
      if constexpr (PL == 2) {
        bf16x4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          hi[e] = (bf16)pv[e];
          lo[e] = (bf16)(pv[e] - (float)hi[e]);
        }
        *reinterpret_cast<bf16x4 *>(&sp[0][lane][rr]) = hi;
        *reinterpret_cast<bf16x4 *>(&sp[1][lane][rr]) = lo;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) sp[0][lane][rr + e] = pv[e];
      }
    }
    __syncthreads();
    // P^T rows r0 + rr, columns i0 .. i0 + 63 (gathered down the tile)
    for (int e = tid; e < PL * 64 * (64 / EPV); e += 256) {
      const int q = e / (64 * (64 / EPV)), rr = (e / (64 / EPV)) % 64, c = (e % (64 / EPV)) * EPV;
      T v[EPV];
#pragma unroll
      for (int k = 0; k < EPV; ++k) v[k] = sp[q][c + k][rr];
      *reinterpret_cast<u32x4 *>(&PT[(size_t)q * tp * np_ + (size_t)(r0 + rr) * np_ + i0 + c]) =
          *reinterpret_cast<const u32x4 *>(v);
    }
    if (outm)   // P rows i0 + row, columns r0 .. r0 + 63
      for (int e = tid; e < PL * 64 * (64 / EPV); e += 256) {
        const int q = e / (64 * (64 / EPV)), row = (e / (64 / EPV)) % 64, c = (e % (64 / EPV)) * EPV;
        *reinterpret_cast<u32x4 *>(&Pm[(size_t)q * np_ * tp + (size_t)(i0 + row) * tp + r0 + c]) =
            *reinterpret_cast<const u32x4 *>(&sp[q][row][c]);
      }
  }
}

// out[c][i] = in[i][c] for a [rows][128] fp32 matrix, zero-padded to rows_pad
// columns; bf16 hi/lo planes or fp32.
template <typename T>
__global__ void __launch_bounds__(256) k_transpose128(const float *__restrict__ in, int rows, int64_t in_pair,
                                                      int64_t rows_pad, void *__restrict__ out, int64_t out_pair) {
  __shared__ float s[64][kHeadDim + 1];
  const int b = blockIdx.y, tid = threadIdx.x;
  const int i0 = blockIdx.x * 64;
  // every row's read is issued before the first is used: under the row test a workgroup
  // waited for them in turn, 11.6 us a call at 1 pair of 256 rows (value fit of 8 pairs,
  // t = 1638, with its two calls 2056 -> 2042 us)
  float x[64 * kHeadDim / 256];
#pragma unroll
  for (int k = 0; k < 64 * kHeadDim / 256; ++k) {
    const int e = tid + 256 * k, r = e / kHeadDim, c = e % kHeadDim;
    x[k] = in[(size_t)b * in_pair + (size_t)min(i0 + r, rows - 1) * kHeadDim + c];
  }
#pragma unroll
  for (int k = 0; k < 64 * kHeadDim / 256; ++k) {
    const int e = tid + 256 * k, r = e / kHeadDim, c = e % kHeadDim;
    s[r][c] = i0 + r < rows ? x[k] : 0.0f;
  }
  __syncthreads();
#pragma unroll 8
  for (int e = tid; e < 64 * kHeadDim; e += 256) {
    const int c = e / 64, r = e % 64;
    const float v = s[r][c];
    const size_t o = (size_t)b * out_pair + (size_t)c * rows_pad + i0 + r;
    if constexpr (sizeof(T) == 2) {
      bf16 *ob = reinterpret_cast<bf16 *>(out);
      split_bf16(v, ob[o], ob[o + (size_t)kHeadDim * rows_pad]);
    } else {
      reinterpret_cast<float *>(out)[o] = v;
    }
  }
}

// --------------------------------------------------------------- 128 right-hand sides
// L Y = R (forward) and L^T X = Y (backward) for 128 right-hand sides, fp32
// MFMA throughout, in 256-row blocks K:
//   k_trsm_diag       X_K = D_K R_K (or D_K^T R_K), written to X and, as 16 x 16 tiles
//   k_trsm_diag_left  of X^T in the fragments' layout, to xt [B][ld / 16][8][256]
//   k_trsm_upd        R_i -= L_iK X_K (or L_Ki^T X_K) on the remaining rows
//   k_trsm_left       R_K -= L_Ki X_i (or L_iK^T X_i) for the solved blocks i in order
// Few pairs are right-looking (diag, upd): the remaining rows are updated by
// their own workgroups, so a call fills the chip.  Many are left-looking (left,
// diag_left): a block's rows stay in registers while every solved block is applied,
// so R is read and written once and not once per block, and the operands are staged
// in LDS, whose tiles several waves read.  Both forms apply the blocks in the same
// order with the same sums, so a pair's solution is the same bits however many are
// solved together.
// Four solves and the refinement's products, right- and left-looking, in ms: t = 3277,
// 64 pairs 8.5 and 9.0, 96: 12.3 and 10.5, 128: 16.2 and 11.9, 256: 31.3 and 22.9; t =
// 1638, 64 pairs 3.39 and 3.42, 128: 6.5 and 5.0, 256: 12.3 and 9.4; t = 819, 64 pairs
// 1.26 and 1.19, 256: 5.7 and 4.5.  (One workgroup per pair for the whole solve: 24.8,
// 9.0 and 3.9 at 256 pairs with 64-wide inverses, other sums; 24.9, 9.8 and 4.6 with these.)
// k_trsm_left takes 36 us per applied block of 256 pairs, 0.76 of the fp32 MFMA rate,
// and k_trsm_diag_left 44 us, most of it the reads and writes of R, X and xt.
// R is overwritten; X must not alias it.

// acc[i][j] += the product of 16 columns of L's row tiles i and 16 rows of X's column
// tiles j: fragments l and x.
template <int RT, int CT>
__device__ __forceinline__ void trsm_mac(f32x4 (&acc)[RT][CT], const f32x4 (&l)[RT], const f32x4 (&x)[CT]) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][e], l[i][e], acc[i][j], 0, 0, 0);
}

// Tile (rt, ct) of X_K: the sum of its even and odd k tiles' products, column r and
// rows 4 g .. 4 g + 3 in lane 16 g + r.
__device__ __forceinline__ void trsm_put(float *X, float *xt, int64_t ld, int b, int K, int rt, int ct, int lane,
                                         f32x4 even, f32x4 odd) {
  const int r = lane & 15, g = lane >> 4;
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = even[e] + odd[e];
  *reinterpret_cast<f32x4 *>(xt + (((size_t)b * (ld / 16) + 16 * K + rt) * 8 + ct) * 256 + 4 * lane) = o;
#pragma unroll
  for (int e = 0; e < 4; ++e) X[((size_t)b * ld + 256 * (int64_t)K + 16 * rt + 4 * g + e) * kHeadDim + 16 * ct + r] = o[e];
}

// The parts of L_iK (forward; of L_Ki^T) and of X_K^T that one wave's products over
// rows row0 .. + 31 and column tiles ct0 .. + CT - 1 read: a 16-byte load per lane
// and tile (the backward rows of L: four 4-byte loads).
template <bool FWD, int CT>
struct TrsmOperands {
  const float *L, *x;
  int64_t ld;
  __device__ __forceinline__ TrsmOperands(const float *Gw, const float *xt, int64_t ld, int b, int K, int64_t row0,
                                          int ct0, int lane)
      : ld(ld) {
    const int r = lane & 15, g = lane >> 4;
    const int64_t K0 = (int64_t)K * 256;
    L = Gw + (size_t)b * ld * ld + (FWD ? (size_t)(row0 + r) * ld + K0 + 4 * g : (size_t)(K0 + 4 * g) * ld + row0 + r);
    x = xt + (((size_t)b * (ld / 16) + 16 * K) * 8 + ct0) * 256 + 4 * lane;
  }
  __device__ __forceinline__ void load(int kt, f32x4 (&l)[2], f32x4 (&xv)[CT]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (FWD) {
        l[i] = *reinterpret_cast<const f32x4 *>(L + (size_t)(16 * i) * ld + 16 * kt);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) l[i][e] = L[(size_t)(16 * kt + e) * ld + 16 * i];
      }
    }
#pragma unroll
    for (int j = 0; j < CT; ++j) xv[j] = *reinterpret_cast<const f32x4 *>(x + (size_t)(8 * kt + j) * 256);
  }
};

// One 16 x 16 tile per wave, 16 rows x 64 columns per workgroup.  A tile is the sum
// of its even and of its odd k tiles, over the k tiles where D has entries (or
// stored zeros): up to the diagonal tile, or from it.  Every tile is loaded, so that
// all loads are in flight at once; the others' values are replaced by zeros.
template <bool FWD>
__global__ void __launch_bounds__(256) k_trsm_diag(const void *__restrict__ lsplit, int64_t ld, int K,
                                                   const float *__restrict__ R, float *__restrict__ X,
                                                   float *__restrict__ xt, const int32_t *__restrict__ info) {
  const int b = blockIdx.y;
  if (info[b] != 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int64_t K0 = (int64_t)K * 256;
  const DiagInv D = diag_inv(lsplit, ld, b, K0);
  const int rt = blockIdx.x >> 1, ct = 4 * (blockIdx.x & 1) + wave;
  const float *Rb = R + ((size_t)b * ld + K0) * kHeadDim + 16 * ct + r;
  const int k0 = FWD ? 0 : rt, k1 = FWD ? rt + 1 : 16;
  f32x4 d[16], v[16];
#pragma unroll
  for (int kt = 0; kt < 16; ++kt) {
    if constexpr (FWD) {
      d[kt] = *reinterpret_cast<const f32x4 *>(D.at(16 * rt + r, 16 * kt + 4 * g));
    } else {
      const float *dp = D.at(16 * kt + 4 * g, 16 * rt) + r;
#pragma unroll
      for (int e = 0; e < 4; ++e) d[kt][e] = dp[(size_t)e * D.ldf];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[kt][e] = Rb[(size_t)(16 * kt + 4 * g + e) * kHeadDim];
  }
  __builtin_amdgcn_sched_barrier(0);   // loads first
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int kt = 0; kt < 16; ++kt) {   // adds (R_kt^T) (D_rt,kt)^T: the tile of X^T
    const bool in = kt >= k0 && kt < k1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      d[kt][e] = in ? d[kt][e] : 0.0f;
      v[kt][e] = in ? v[kt][e] : 0.0f;
    }
    if (kt & 1) s1 = tile_mac(s1, v[kt], d[kt]);
    else s0 = tile_mac(s0, v[kt], d[kt]);
  }
  trsm_put(X, xt, ld, b, K, rt, ct, lane, s0, s1);
}

// 64 rows x 32 TN columns per workgroup, 32 x 16 TN per wave (2 x 2 waves);
// fragments straight from global memory.
template <bool FWD, int TN>
__global__ void __launch_bounds__(256) k_trsm_upd(const float *__restrict__ Gw, int64_t ld, int K,
                                                  float *__restrict__ R, const float *__restrict__ xt,
                                                  const int32_t *__restrict__ info) {
  constexpr int NCG = kHeadDim / (32 * TN);
  const int b = blockIdx.y;
  if (info[b] != 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int cg = blockIdx.x % NCG, rc = blockIdx.x / NCG;
  const int64_t row0 = (FWD ? (int64_t)K * 256 + 256 : 0) + 64 * (int64_t)rc + 32 * (wave & 1);
  const int ct0 = 2 * TN * cg + TN * (wave >> 1);
  const TrsmOperands<FWD, TN> op(Gw, xt, ld, b, K, row0, ct0, lane);
  f32x4 acc[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (TN == 2) {   // few workgroups: a wave's whole operands in flight at once
    f32x4 l[16][2], x[16][TN];
#pragma unroll
    for (int kt = 0; kt < 16; ++kt) op.load(kt, l[kt], x[kt]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kt = 0; kt < 16; ++kt) trsm_mac(acc, l[kt], x[kt]);
  } else {
#pragma unroll 4
    for (int kt = 0; kt < 16; ++kt) {
      f32x4 l[2], x[TN];
      op.load(kt, l, x);
      trsm_mac(acc, l, x);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      f32x4 *p = reinterpret_cast<f32x4 *>(R + ((size_t)b * ld + row0 + 16 * i + r) * kHeadDim + 16 * (ct0 + j) + 4 * g);
      f32x4 o = *p;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] -= acc[i][j][e];
      *p = o;
    }
}

// The left-looking kernels stage their operands in LDS as 16 x 16 tiles, each by one
// 16-byte direct-to-LDS load per lane (lane l fills floats 4 l .. 4 l + 3), in the order
// that a wave's fragments are read without bank conflicts:
//   rows   lane 16 g + r's fragment is row r, columns 4 g .. 4 g + 3, one 16-byte read
//   cols   it is column r, rows 4 g .. 4 g + 3: row 4 g + e lies at float 16 (4 e + g)
typedef __attribute__((address_space(3))) void trsm_lds_t;

__device__ __forceinline__ int64_t stage_rows(int lane, int64_t ld) { return (lane & 15) * ld + 4 * (lane >> 4); }
__device__ __forceinline__ int64_t stage_cols(int lane, int64_t ld) {
  return (4 * ((lane >> 2) & 3) + (lane >> 4)) * ld + 4 * (lane & 3);
}
__device__ __forceinline__ void stage_tile(const float *src, float *tile) {
  __builtin_amdgcn_global_load_lds((const void *)src, (trsm_lds_t *)tile, 16, 0, 0);
}
__device__ __forceinline__ f32x4 tile_rows(const float *tile, int lane) {
  return *reinterpret_cast<const f32x4 *>(tile + 4 * lane);
}
__device__ __forceinline__ f32x4 tile_cols(const float *tile, int lane) {
  const float *p = tile + 16 * (lane >> 4) + (lane & 15);
  return f32x4{p[0], p[64], p[128], p[192]};
}

// Block K's rows, 128 per workgroup over all 128 columns, 32 x 64 per wave: every
// solved block's product with its own sum, subtracted in the solve's order, as
// k_trsm_upd subtracts them one launch at a time.  Two k tiles per stage, two stages.
// A pair's two workgroups share an XCD, whose L2 they read the solution from.
constexpr int kTrsmLeftRows = 128;
template <bool FWD>
__global__ void __launch_bounds__(512, 4) k_trsm_left(const float *__restrict__ Gw, int64_t ld, int K,
                                                      float *__restrict__ R, const float *__restrict__ xt,
                                                      const int32_t *__restrict__ info) {
  constexpr int NS = 4;
  __shared__ __attribute__((aligned(1024))) float stage[NS][16][256];   // 8 row tiles, 8 column tiles of a k tile
  const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const int b = (int)(tile >> 1), rc = (int)(tile & 1);
  if (info[b] != 0) return;   // uniform over the workgroup
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wr = wave & 3, wc = wave >> 2;
  const int64_t row0 = (int64_t)K * 256 + kTrsmLeftRows * rc;
  const int nblk = (int)(ld / 256), stages = 16 * (FWD ? K : nblk - 1 - K);
  const float *Lb = Gw + (size_t)b * ld * ld + (FWD ? row0 * ld + stage_rows(lane, ld) : row0 + stage_cols(lane, ld));
  const float *xb = xt + (size_t)b * ld * kHeadDim + 4 * lane;
  auto issue = [&](int q) {   // wave w loads tiles 2 w and 2 w + 1
    const int64_t kt = 16 * (int64_t)(FWD ? q >> 4 : nblk - 1 - (q >> 4)) + (q & 15);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int m = 2 * wave + u;
      const float *src = m < 8 ? Lb + (FWD ? 16 * m * ld + 16 * kt : 16 * kt * ld + 16 * m) : xb + (8 * kt + m - 8) * 256;
      stage_tile(src, stage[q % NS][m]);
    }
  };
  float *Rw = R + ((size_t)b * ld + row0 + 32 * wr + r) * kHeadDim + 64 * wc + 4 * g;
  f32x4 o[2][4], acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      o[i][j] = *reinterpret_cast<const f32x4 *>(Rw + (size_t)(16 * i) * kHeadDim + 16 * j);
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
  for (int q = 0; q < NS - 1; ++q) issue(q);
  for (int q = 0; q < stages; ++q) {   // uniform over the launch
    // stage q has landed, the younger ones may be in flight; after the barrier every
    // wave's has, and stage q - 1, which is refilled next, has been read
    if (q + NS - 2 < stages) wait_vmcnt<2 * (NS - 2)>();
    else wait_vmcnt<0>();
    wait_lgkmcnt0();
    lds_barrier();
    if (q + NS - 1 < stages) issue(q + NS - 1);
    f32x4 l[2], x[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float *t = stage[q % NS][2 * wr + i];
      l[i] = FWD ? tile_rows(t, lane) : tile_cols(t, lane);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = tile_rows(stage[q % NS][8 + 4 * wc + j], lane);
    trsm_mac(acc, l, x);
    asm volatile("" ::: "memory");   // the reads stay above the next wait
    if ((q & 15) == 15) {   // a block is complete
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
          for (int e = 0; e < 4; ++e) o[i][j][e] -= acc[i][j][e];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4 *>(Rw + (size_t)(16 * i) * kHeadDim + 16 * j) = o[i][j];
}

// k_trsm_diag's sums, 32 columns per workgroup and four workgroups per pair: R_K's
// columns are staged in LDS at once, and wave w streams the tiles of D of row tiles
// w, 7 - w, 8 + w and 15 - w, 18 pairs of k tiles in all for every wave, straight
// into its fragments, three pairs ahead.  No barrier but the one after R.
template <bool FWD>
__global__ void __launch_bounds__(256, 4) k_trsm_diag_left(const void *__restrict__ lsplit, int64_t ld, int K,
                                                           const float *__restrict__ R, float *__restrict__ X,
                                                           float *__restrict__ xt, const int32_t *__restrict__ info) {
  __shared__ __attribute__((aligned(1024))) float sR[16][2][256];   // [k tile][column tile], cols order
  const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const int b = (int)(tile >> 2), cg = (int)(tile & 3);
  if (info[b] != 0) return;   // uniform over the workgroup
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t K0 = (int64_t)K * 256;
  const DiagInv D = diag_inv(lsplit, ld, b, K0);
  const float *Rb = R + ((size_t)b * ld + K0) * kHeadDim + 32 * cg + stage_cols(lane, kHeadDim);
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int kt = 4 * wave + (u >> 1), j = u & 1;
    stage_tile(Rb + (size_t)(16 * kt) * kHeadDim + 16 * j, sR[kt][j]);
  }
  // the wave's row tile i and its pairs of k tiles: up to the diagonal tile, or from it
  auto row_tile = [&](int i) { return (i & 1 ? 8 * (i >> 1) + 7 - wave : 8 * (i >> 1) + wave); };
  auto first_pair = [&](int i) { return FWD ? 0 : row_tile(i) >> 1; };
  auto last_pair = [&](int i) { return FWD ? row_tile(i) >> 1 : 7; };
  auto load_d = [&](int rt, int kt) {   // a tile past the range reads the diagonal one
    const int k = FWD ? min(kt, rt) : max(kt, rt);
    f32x4 d;
    if constexpr (FWD) {
      d = *reinterpret_cast<const f32x4 *>(D.at(16 * rt + r, 16 * k + 4 * g));
    } else {
      const float *dp = D.at(16 * k + 4 * g, 16 * rt) + r;
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] = dp[(size_t)e * D.ldf];
    }
    return d;
  };
  f32x4 d[3][2];
  int li = 0, lp = first_pair(0);   // the next pair to load
  auto load_next = [&](f32x4 (&to)[2]) {
    const int rt = row_tile(li);
    to[0] = load_d(rt, 2 * lp);
    to[1] = load_d(rt, 2 * lp + 1);
    if (lp < last_pair(li)) ++lp;
    else if (li < 3) lp = first_pair(++li);   // past the last pair: that one again
  };
#pragma unroll
  for (int u = 0; u < 3; ++u) load_next(d[u]);
  wait_vmcnt<0>();
  __syncthreads();
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 s[2][2] = {{zero, zero}, {zero, zero}};   // [kt & 1][column tile]
  int i = 0, kp = first_pair(0);
  for (int f = 0; f < 18; f += 3) {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int rt = row_tile(i);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int kt = 2 * kp + p;
        if (FWD ? kt > rt : kt < rt) continue;   // uniform over the wave
        const f32x4 v0 = tile_cols(sR[kt][0], lane), v1 = tile_cols(sR[kt][1], lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[p][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[u][p][e], v0[e], s[p][0], 0, 0, 0);
          s[p][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[u][p][e], v1[e], s[p][1], 0, 0, 0);
        }
      }
      load_next(d[u]);
      if (kp < last_pair(i)) {
        ++kp;
      } else {   // the row tile is complete
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          trsm_put(X, xt, ld, b, K, rt, 2 * cg + j, lane, s[0][j], s[1][j]);
          s[0][j] = s[1][j] = zero;
        }
        if (i < 3) kp = first_pair(++i);
      }
    }
  }
}

__global__ void __launch_bounds__(256) k_add_copy(float *__restrict__ x, const float *__restrict__ dx, int64_t n_per,
                                                  const int32_t *__restrict__ info) {
  const int b = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n_per || info[b] != 0) return;
  x[(size_t)b * n_per + e] += dx[(size_t)b * n_per + e];
}

// Copy the first t rows of the padded [tp][128] solution to the output, NaN
// for pairs whose factorisation failed.
__global__ void __launch_bounds__(256) k_values_out(const float *__restrict__ Xp, int64_t tp, int t,
                                                    const int32_t *__restrict__ info, float *__restrict__ Cv) {
  const int b = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)t * kHeadDim) return;
  Cv[(size_t)b * t * kHeadDim + e] = info[b] != 0 ? NAN : Xp[(size_t)b * tp * kHeadDim + e];
}

// --------------------------------------------------------------- exact NNLS (bias_mode 1)
// Block principal pivoting (Judice & Pires 1994, in the single-right-hand-side
// form of Kim & Park 2011) for min ||Phi_C w - m||^2 + lam ||w||^2, w >= 0, the
// ridged system of the projected fit.  Per pair: F (passive set, 1 = free), x,
// y = (G + lam I) x - h from the data residual, and the state
// {best infeasible count N, backup budget p, done, spare}.  The iteration starts
// from the unconstrained solution (F = every key), which the projected fit has
// already computed; each later iteration solves the free-set system compressed
// to its |F| x |F| block.
constexpr int32_t kNnlsSkip = -0x40000000;   // info marker of a pair that has converged

__global__ void __launch_bounds__(256) k_nnls_init(int t, int64_t tp, const int32_t *__restrict__ info,
                                                   int32_t *__restrict__ F, double *__restrict__ y,
                                                   int32_t *__restrict__ state) {
  const int b = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < tp) {
    F[(size_t)b * tp + r] = r < t;
    y[(size_t)b * tp + r] = 0.0;
  }
  if (r == 0) {
    state[4 * b] = t + 1;
    state[4 * b + 1] = 3;
    state[4 * b + 2] = info[b] != 0;   // a failed projected fit is not iterated
    state[4 * b + 3] = 0;
  }
}

// One workgroup per pair: the infeasible set V = {free x < -tol} u {bound y < -tol},
// then the exchange rule: all of V while |V| improves on the best count (or the
// backup budget lasts), otherwise only its largest index.  Marks the pair done
// (and skipped by the factor and solve kernels) when V is empty.
__global__ void __launch_bounds__(256) k_nnls_update(const double *__restrict__ x, const double *__restrict__ y,
                                                     const double *__restrict__ h, int t, int64_t tp,
                                                     int32_t *__restrict__ F, int32_t *__restrict__ state,
                                                     int32_t *__restrict__ info) {
  __shared__ double sx[4], sh[4];
  __shared__ int32_t scnt[4], smax[4];
  __shared__ int32_t s_mode;   // 0 none, 1 all of V, 2 the largest index only
  __shared__ int32_t s_j;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (state[4 * b + 2] || info[b] != 0) return;   // settled, or a factorisation failed
  const double *xb = x + (size_t)b * tp, *yb = y + (size_t)b * tp, *hb = h + (size_t)b * tp;
  int32_t *Fb = F + (size_t)b * tp;
  double mx = 0.0, mh = 0.0;
  for (int r = tid; r < t; r += 256) {
    mx = fmax(mx, fabs(xb[r]));
    mh = fmax(mh, fabs(hb[r]));
  }
  for (int o = 32; o >= 1; o >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    mh = fmax(mh, __shfl_xor(mh, o, 64));
  }
  if (lane == 0) {
    sx[wave] = mx;
    sh[wave] = mh;
  }
  __syncthreads();
  // tolerances: float32-level relative to the solution and right-hand side scales
  const double tx = 1e-6 * fmax(fmax(sx[0], sx[1]), fmax(sx[2], sx[3]));
  const double ty = 1e-6 * fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
  auto infeasible = [&](int r) { return Fb[r] ? xb[r] < -tx : yb[r] < -ty; };
  int32_t cnt = 0, jmax = -1;
  for (int r = tid; r < t; r += 256)
    if (infeasible(r)) {
      ++cnt;
      jmax = r;
    }
  for (int o = 32; o >= 1; o >>= 1) {
    cnt += __shfl_xor(cnt, o, 64);
    jmax = max(jmax, __shfl_xor(jmax, o, 64));
  }
  if (lane == 0) {
    scnt[wave] = cnt;
    smax[wave] = jmax;
  }
  __syncthreads();
  if (tid == 0) {
    const int32_t V = scnt[0] + scnt[1] + scnt[2] + scnt[3];
    s_j = max(max(smax[0], smax[1]), max(smax[2], smax[3]));
    int32_t mode = 0;
    if (V == 0) {
      state[4 * b + 2] = 1;
      info[b] = kNnlsSkip;
    } else if (V < state[4 * b]) {
      state[4 * b] = V;
      state[4 * b + 1] = 3;
      mode = 1;
    } else if (state[4 * b + 1] >= 1) {
      state[4 * b + 1] -= 1;
      mode = 1;
    } else {
      mode = 2;
    }
    state[4 * b + 3] += mode != 0;   // iterations taken
    s_mode = mode;
  }
  __syncthreads();
  if (s_mode == 1) {
    // infeasible(r) reads only F[r], which this thread alone owns
    for (int r = tid; r < t; r += 256)
      if (infeasible(r)) Fb[r] ^= 1;
  } else if (s_mode == 2 && tid == 0) {
    Fb[s_j] ^= 1;
  }
}

__global__ void k_nnls_zero(int32_t *__restrict__ red) {
  if (threadIdx.x < 2) red[threadIdx.x] = 0;
}

// Free and bound lists of every unsettled pair: idx[k] = the k-th free key,
// bidx[k] = the k-th bound key (both ascending), pos[r] = the free slot of r or
// -1; nf = |F|, nb = t - |F|; red = {max nf, unsettled pairs}.
__global__ void __launch_bounds__(256) k_nnls_index(const int32_t *__restrict__ F, int t, int64_t tp,
                                                    const int32_t *__restrict__ info, int32_t *__restrict__ idx,
                                                    int32_t *__restrict__ bidx, int32_t *__restrict__ pos,
                                                    int32_t *__restrict__ nf, int32_t *__restrict__ nb,
                                                    int32_t *__restrict__ red) {
  __shared__ int32_t wsum[4];
  __shared__ int32_t base;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (info[b] != 0) return;   // settled or failed
  if (tid == 0) base = 0;
  __syncthreads();
  const int32_t *Fb = F + (size_t)b * tp;
  int32_t *ib = idx + (size_t)b * tp, *bb = bidx + (size_t)b * tp, *pb = pos + (size_t)b * tp;
  for (int64_t r0 = 0; r0 < tp; r0 += 256) {
    const int64_t r = r0 + tid;
    const bool f = r < t && Fb[r] != 0;
    const uint64_t m = __ballot(f);
    if (lane == 0) wsum[wave] = __popcll(m);
    __syncthreads();
    int32_t before = base + __popcll(m & ((1ull << lane) - 1ull));   // free keys below r
    for (int w = 0; w < wave; ++w) before += wsum[w];
    if (f) ib[before] = (int32_t)r;
    else if (r < t) bb[r - before] = (int32_t)r;
    if (r < tp) pb[r] = f ? before : -1;
    __syncthreads();
    if (tid == 0) base += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
  if (tid == 0) {
    nf[b] = base;
    nb[b] = t - base;
    atomicMax(&red[0], base);
    atomicAdd(&red[1], 1);
  }
}

// Compressed free-set system [ldf][ldf]: G_{idx_i idx_j} + lam [i = j] for
// i, j < nf, identity beyond.
__global__ void __launch_bounds__(256) k_nnls_gather_gram(const float *__restrict__ Gc, int64_t tp,
                                                          const int32_t *__restrict__ idx,
                                                          const int32_t *__restrict__ nf, const FitState st,
                                                          int64_t ldf, float *__restrict__ Gw) {
  const int b = blockIdx.y;
  if (st.info[b] != 0) return;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= ldf * ldf) return;
  const int64_t i = e / ldf, j = e % ldf;
  // the factorisation reads the lower triangle only
  if (j > i) return;
  const int32_t n = nf[b];
  float v = i == j ? 1.0f : 0.0f;
  if (i < n) {   // then j <= i < n; the free list ascends, so (idx_i, idx_j) is in the stored lower triangle
    const int32_t *ib = idx + (size_t)b * tp;
    v = Gc[(size_t)b * tp * tp + (size_t)ib[i] * tp + ib[j]] + (i == j ? st.lam[b] : 0.0f);
  }
  Gw[(size_t)b * ldf * ldf + e] = v;
}

// out[k] = in[idx_k] for k < nf, 0 beyond (a compressed right-hand side).
__global__ void __launch_bounds__(256) k_nnls_gather_vec(const double *__restrict__ in, int64_t tp,
                                                         const int32_t *__restrict__ idx,
                                                         const int32_t *__restrict__ nf,
                                                         const int32_t *__restrict__ info, int64_t ldf,
                                                         double *__restrict__ out) {
  const int b = blockIdx.y;
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= ldf || info[b] != 0) return;
  out[(size_t)b * ldf + k] = k < nf[b] ? in[(size_t)b * tp + idx[(size_t)b * tp + k]] : 0.0;
}

// x[r] = xf[pos_r] on free keys and 0 on bound ones (acc: x[r] += ...).
__global__ void __launch_bounds__(256) k_nnls_scatter(const double *__restrict__ xf, int64_t ldf,
                                                      const int32_t *__restrict__ pos, int64_t tp,
                                                      const int32_t *__restrict__ info, int acc,
                                                      double *__restrict__ x) {
  const int b = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= tp || info[b] != 0) return;
  const int32_t p = pos[(size_t)b * tp + r];
  const double v = p >= 0 ? xf[(size_t)b * ldf + p] : 0.0;
  double *o = x + (size_t)b * tp + r;
  *o = acc ? *o + v : v;
}

// y = -(data residual) on bound keys, 0 on free ones.
__global__ void __launch_bounds__(256) k_nnls_dual(const double *__restrict__ res, const int32_t *__restrict__ F,
                                                   int64_t tp, const int32_t *__restrict__ info,
                                                   double *__restrict__ y) {
  const int b = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= tp || info[b] != 0) return;
  const size_t o = (size_t)b * tp + r;
  y[o] = F[o] ? 0.0 : -res[o];
}

// After the iterations: converged pairs are ok again; pairs still iterating get -2.
__global__ void k_nnls_finish(const int32_t *__restrict__ state, int B, int32_t *__restrict__ info) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= B) return;
  if (info[b] == kNnlsSkip) info[b] = 0;
  else if (info[b] == 0 && !state[4 * b + 2]) info[b] = -2;
}

// ------------------------------------------------------------------ launchers
hipError_t launch_fill_i32(int32_t *p, int64_t count, int32_t v, hipStream_t s);
hipError_t launch_trsv(const float *Gw, const float *dinv, int B, int64_t ld, const double *rhs, double *sw,
                       double *y, double *x, double *acc, const int32_t *info, hipStream_t s);
hipError_t launch_cholesky_factor(float *Gw, const float *Gc, int B, int t, int64_t ld, float delta0, int max_esc,
                                  FitState st, float *dinv, void *lsplit, hipStream_t s);

// Escalation rounds over the pairs whose factorisation failed and that have
// escalations left.  Before each round the number of such pairs is read back
// to the host (cnt: one device int32), so rounds run only when a pair needs
// one; with max_esc = 0 nothing is read back.
static hipError_t launch_esc_rounds(float *Gw, const float *Gc, int B, int t, int64_t ld, int max_esc, FitState st,
                                    float *dinv, void *lsplit, int32_t *cnt, hipStream_t s) {
  hipError_t e = hipSuccess;
  for (int round = 0; round < max_esc; ++round) {
    hipLaunchKernelGGL(k_count_failed, dim3(1), dim3(256), 0, s, B, st, max_esc, cnt);
    int32_t failed = 0;
    if ((e = hipMemcpyAsync(&failed, cnt, sizeof(failed), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    if (failed == 0) break;
    hipLaunchKernelGGL(k_esc_state, dim3((B + 255) / 256), dim3(256), 0, s, B, t, st, max_esc);
    hipLaunchKernelGGL(k_esc_copy, dim3((unsigned)ld, B), dim3(256), 0, s, Gw, Gc, t, ld, st);
    if ((e = launch_cholesky_factor(Gw, Gc, B, t, ld, 0.0f, 0, st, dinv, lsplit, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_esc_restore, dim3((B + 255) / 256), dim3(256), 0, s, B, st.info);
  }
  return hipGetLastError();
}

// Ridge + factorisation of the work copy Gw of Gc, then the escalation rounds.
hipError_t launch_cholesky(float *Gw, const float *Gc, int B, int t, int64_t ld, float delta0, int max_esc,
                           FitState st, float *dinv, void *lsplit, const int32_t *bad, int32_t *cnt,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_ridge_init, dim3(B), dim3(256), 0, s, Gw, Gc, t, ld, delta0, st, bad);
  hipError_t e = launch_cholesky_factor(Gw, Gc, B, t, ld, delta0, 0, st, dinv, lsplit, s);
  if (e != hipSuccess) return e;
  return launch_esc_rounds(Gw, Gc, B, t, ld, max_esc, st, dinv, lsplit, cnt, s);
}

// Clears bad [B], then marks the pairs with a non-finite value in f's arrays.
hipError_t launch_nonfinite(const FiniteCheck &f, int B, int32_t *bad, hipStream_t s) {
  const hipError_t e = launch_fill_i32(bad, B, 0, s);
  if (e != hipSuccess) return e;
  int64_t most = 0;
  for (int q = 0; q < FiniteCheck::kMax; ++q)
    if (f.a[q] && f.per[q] > most) most = f.per[q];
  if (most == 0) return hipSuccess;
  const int64_t blocks = (most + 1023) / 1024;
  hipLaunchKernelGGL(k_nonfinite, dim3((unsigned)(blocks < 64 ? blocks : 64), B, FiniteCheck::kMax), dim3(256), 0, s,
                     f, bad);
  return hipGetLastError();
}

// Factor the prepared work copy Gw in place (no ridge set-up, no escalation).
hipError_t launch_cholesky_factor(float *Gw, const float *Gc, int B, int t, int64_t ld, float delta0, int max_esc,
                                  FitState st, float *dinv, void *lsplit, hipStream_t s) {
  // 256-wide outer panels, left-looking: before a panel is factored, one
  // contraction applies every earlier panel to it (rows K0 .. ld, K = 3 K0 over
  // the fp16 hi / lo planes of L), so each trailing entry is read and written
  // once per factorisation instead of once per outer panel.  Inside the panel,
  // its 256 x 256 diagonal block in one workgroup per pair, then the fused
  // strip kernel on the rows below, which also writes their planes for the
  // later panels' contractions.
  // lsplit layout (B (4 ld^2 + 8 ld) bytes): planes [B][2][ld][ld] fp16 (hi,
  // lo), then shifts [B][ld] int32, then inverse scales [B][ld] fp32.
  constexpr int kOuter = 256;
  f16 *Lp = reinterpret_cast<f16 *>(lsplit);
  int32_t *shift = reinterpret_cast<int32_t *>(Lp + (size_t)B * 2 * ld * ld);
  float *sinv = reinterpret_cast<float *>(shift + (size_t)B * ld);
  hipLaunchKernelGGL(k_chol_scales, dim3((unsigned)((ld + 255) / 256), B), dim3(256), 0, s, Gw, ld, shift, sinv,
                     st.info);
  auto strip = [&](auto kern, int rows, int K0) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((ld - K0 - kOuter) / rows), B), dim3(4 * rows), strip16_lds(rows), s, Gw,
                       ld, K0, dinv, Lp, shift, st.info);
    return hipGetLastError();
  };
  auto set_lds = [](const void *kern, size_t bytes) {
    return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  };
  hipError_t ea = set_lds((const void *)k_chol_diag256, kDiag256Lds);
  if (ea == hipSuccess) ea = set_lds((const void *)k_chol_strip16<64>, strip16_lds(64));
  if (ea == hipSuccess) ea = set_lds((const void *)k_chol_strip16<128>, strip16_lds(128));
  if (ea != hipSuccess) return ea;
  for (int K0 = 0; K0 < ld; K0 += kOuter) {
    const int K1 = (int)(K0 + kOuter < ld ? K0 + kOuter : ld);
    if (K0 > 0) {
      // A[K0.., K0..K1) -= L[K0.., 0..K0) L[K0..K1, 0..K0)^T: the three products
      // hi.hi, hi.lo, lo.hi per k-step from both planes of each operand (each
      // plane is read once), 256 x 256 tiles down the panel
      const f16 *Ar = Lp + (size_t)K0 * ld;
      BigShape g{B, (int)(ld - K0), kOuter, K0, 2 * ld * ld, ld * ld, ld, 2 * ld * ld, ld * ld, ld, false, 4};
      const bf16 *Ab = reinterpret_cast<const bf16 *>(Ar);
      hipError_t err;
      // 64 x 64 tiles while 256 x 256 ones would leave most CUs without any:
      // then each slab of a tile waits for its loads, and a tile's time is its
      // number of slabs, so many small tiles finish sooner (67 -> 19 us a
      // call at 8 pairs, ld = 1792)
      if ((int64_t)B * (ld - K0) / 256 < kFewTiles) {
        EpiCholUpd<1, 1, 64, 64> e{Gw, ld, K0, st.info, sinv + K0, ld};
        err = launch_gemm_big<2, 2, 1, 1, 32, 2, 2, 4, f16>(g, Ab, Ab, e, s);
      } else {
        EpiCholUpd<2, 4, 256, 256> e{Gw, ld, K0, st.info, sinv + K0, ld};
        err = launch_gemm_big<4, 2, 2, 4, 32, 2, 2, 2, f16>(g, Ab, Ab, e, s);
      }
      if (err != hipSuccess) return err;
    }
    // the 256 x 256 diagonal block
    const int nb = t - K0 < kOuter ? (t - K0 + kNB - 1) / kNB : kOuter / kNB;
    hipLaunchKernelGGL(k_chol_diag256, dim3(B), dim3(1024), kDiag256Lds, s, Gw, ld, K0, nb > 0 ? nb : 0, st.info, dinv);
    // the rows below: all four steps, written back once, with their planes
    if (K1 < ld) {
      const bool few = (ld - K1) / 64 * B <= kStripFew;
      const hipError_t e = few ? strip(k_chol_strip16<64>, 64, K0) : strip(k_chol_strip16<128>, 128, K0);
      if (e != hipSuccess) return e;
    }
  }
  (void)Gc;
  (void)delta0;
  (void)max_esc;
  return hipGetLastError();
}

// The inverses of the factored pairs' 256 x 256 diagonal blocks, for launch_trsm.
hipError_t launch_inv256(const float *Gw, int B, int t, int64_t ld, const float *dinv, void *lsplit,
                         const int32_t *info, hipStream_t s) {
  const int nblk = (int)(ld / 256);
  auto inv = [&](auto kern, int nw) {
    const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kInv256Lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk, B, 16 / nw), dim3(64 * nw), kInv256Lds, s, Gw, ld, t, dinv, lsplit,
                       info);
    return hipGetLastError();
  };
  // four workgroups per block as long as each has a CU
  return (int64_t)nblk * B <= 64 ? inv(k_chol_inv256<4>, 4) : inv(k_chol_inv256<16>, 16);
}

// Forward L y = rhs then backward L^T x = y; sw and y are work vectors
// [B][ld]; x receives the solution, acc (optional) accumulates it.  A
// workgroup takes one chunk of 64 targets while few pairs leave CUs idle, and
// up to four (256 rows, as much of L as of D_K) once the launch holds more
// than kTrsvGroups of them, so that D_K is not re-read for every 64 rows.
constexpr int kTrsvGroups = 512;
hipError_t launch_trsv(const float *Gw, const float *dinv, int B, int64_t ld, const double *rhs, double *sw,
                       double *y, double *x, double *acc, const int32_t *info, hipStream_t s) {
  const int nblk = (int)(ld / 256);
  auto groups = [&](int nch, int &per) {
    per = (int)((int64_t)nch * B / kTrsvGroups);
    per = per < 1 ? 1 : per > 4 ? 4 : per;
    return nch > 0 ? (nch + per - 1) / per : 1;
  };
  int per = 1;
  for (int K = 0; K < nblk; ++K) {
    const int ng = groups(4 * (nblk - 1 - K), per);
    hipLaunchKernelGGL(k_trsv256<true>, dim3(ng, B), dim3(1024), 0, s, Gw, dinv, ld, K, per, rhs, sw, y,
                       (double *)nullptr, info);
  }
  for (int K = nblk - 1; K >= 0; --K) {
    const int ng = groups(4 * K, per);
    hipLaunchKernelGGL(k_trsv256<false>, dim3(ng, B), dim3(1024), 0, s, Gw, dinv, ld, K, per,
                       (const double *)nullptr, y, x, acc, info);
  }
  return hipGetLastError();
}

hipError_t launch_mass_residual(const float *LT, const float *z, const float *m, const double *w, const float *lam,
                                int B, int n, int t, int64_t tp, int64_t np_, double *u, double *res,
                                const int32_t *info, hipStream_t s, const int32_t *row_list,
                                const int32_t *row_count, const int32_t *col_list, const int32_t *col_count) {
  hipLaunchKernelGGL(k_mass_resid_rows, dim3((unsigned)(np_ / 64), B), dim3(512), 0, s, LT, z, m, w, n, t, tp, np_,
                     u, info, row_list, row_count);
  hipLaunchKernelGGL(k_mass_resid_cols, dim3((unsigned)(tp / kResKeys), B), dim3(256), 0, s, LT, z, u, w, lam,
                     n, t, tp, np_, res, info, col_list, col_count);
  return hipGetLastError();
}

// Mass-fit solve for the factored pairs (info == 0): w = (G + lam I)^-1 h by
// the float32 factor, then refine_steps refinement steps against the data
// under the refinement guard above (which needs two steps to compare); pairs the guard cuts off are refactored
// with the ridge raised tenfold and solved again, while escalations remain.
// Each such round reads back one integer (the number of pairs to refactor).
hipError_t launch_mass_solve(float *Gw, const float *Gc, float *dinv, void *lsplit, const MassSolve &ms, int B, int n,
                             int t, int64_t tp, int64_t np_, int refine_steps, int max_esc, FitState st, int32_t *cnt,
                             hipStream_t s) {
  hipError_t e;
  const dim3 gb((B + 255) / 256);
  if ((e = launch_fill_i32(ms.div, B, 0, s)) != hipSuccess) return e;
  for (int round = 0;; ++round) {
    if ((e = launch_trsv(Gw, dinv, B, tp, ms.h, ms.sw, ms.y, ms.w, nullptr, st.info, s)) != hipSuccess) return e;
    for (int it = 0; it < refine_steps; ++it) {
      if ((e = launch_mass_residual(ms.LT, ms.z, ms.m, ms.w, st.lam, B, n, t, tp, np_, ms.u, ms.res, st.info, s,
                                      nullptr, nullptr, nullptr, nullptr)) != hipSuccess)
        return e;
      if ((e = launch_trsv(Gw, dinv, B, tp, ms.res, ms.sw, ms.y, ms.x, ms.w, st.info, s)) != hipSuccess) return e;
      hipLaunchKernelGGL(k_refine_watch, dim3(B), dim3(256), 0, s, ms.w, ms.x, tp, it, ms.rprev, ms.div, st,
                         max_esc);
    }
    if (refine_steps < 2 || round == max_esc) break;
    hipLaunchKernelGGL(k_count_flags, dim3(1), dim3(256), 0, s, B, (const int32_t *)ms.div, cnt);
    int32_t flagged = 0;
    if ((e = hipMemcpyAsync(&flagged, cnt, sizeof(flagged), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    if (flagged == 0) break;
    hipLaunchKernelGGL(k_div_mark, gb, dim3(256), 0, s, B, ms.div, st.info);
    if ((e = launch_esc_rounds(Gw, Gc, B, t, tp, max_esc, st, dinv, lsplit, cnt, s)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_refine_restore, gb, dim3(256), 0, s, B, st.info);
  return hipGetLastError();
}

// Pivoting iterations on the projected fit's refined solution x (in place).
// Each iteration reads back {largest free set, unsettled pairs} to size the
// compressed system and to stop once every pair has settled, so this
// synchronises the stream once per iteration.
hipError_t launch_nnls(const float *Gc, float *Gw, const double *h, const float *LT, const float *z, const float *m,
                       int B, int n, int t, int64_t tp, int64_t np_, int max_iter, int refine_steps, FitState st,
                       float *dinv, void *lsplit, NnlsWork nw, double *x, double *sw, double *yw, double *u,
                       double *res, hipStream_t s) {
  const dim3 gv((unsigned)((tp + 255) / 256), (unsigned)B);
  hipLaunchKernelGGL(k_nnls_init, gv, dim3(256), 0, s, t, tp, st.info, nw.F, nw.y, nw.state);
  hipError_t e;
  for (int it = 0;; ++it) {
    // the update after the last solve only checks feasibility (and marks done)
    hipLaunchKernelGGL(k_nnls_update, dim3(B), dim3(256), 0, s, x, nw.y, h, t, tp, nw.F, nw.state, st.info);
    if (it == max_iter) break;
    hipLaunchKernelGGL(k_nnls_zero, dim3(1), dim3(64), 0, s, nw.red);
    hipLaunchKernelGGL(k_nnls_index, dim3(B), dim3(256), 0, s, nw.F, t, tp, st.info, nw.idx, nw.bidx, nw.pos,
                       nw.nf, nw.nb, nw.red);
    int32_t red[2] = {0, 0};
    if ((e = hipMemcpyAsync(red, nw.red, sizeof(red), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    if (red[1] == 0) break;   // every pair has settled (or failed)
    const int64_t ldf = red[0] > 256 ? (red[0] + 255) / 256 * 256 : 256;
    const dim3 gf((unsigned)((ldf + 255) / 256), (unsigned)B);
    hipLaunchKernelGGL(k_nnls_gather_gram, dim3((unsigned)((ldf * ldf + 255) / 256), (unsigned)B), dim3(256), 0, s,
                       Gc, tp, nw.idx, nw.nf, st, ldf, Gw);
    if ((e = launch_cholesky_factor(Gw, Gc, B, t, ldf, 0.0f, 0, st, dinv, lsplit, s)) != hipSuccess) return e;
    for (int rs = 0; rs <= refine_steps; ++rs) {
      // rs = 0 solves for x from h; later steps solve for a correction from the
      // residual of the full ridged system against the data, h - (G + lam I) x
      hipLaunchKernelGGL(k_nnls_gather_vec, gf, dim3(256), 0, s, rs == 0 ? h : res, tp, nw.idx, nw.nf, st.info, ldf,
                         nw.rf);
      if ((e = launch_trsv(Gw, dinv, B, ldf, nw.rf, sw, yw, nw.xf, nullptr, st.info, s)) != hipSuccess) return e;
      hipLaunchKernelGGL(k_nnls_scatter, gv, dim3(256), 0, s, nw.xf, ldf, nw.pos, tp, st.info, rs > 0 ? 1 : 0, x);
      // x vanishes off F, so Phi_C x sums over the free keys; the residual is
      // needed on the free keys for a correction, on the bound keys (the dual)
      // after the last one
      const bool last = rs == refine_steps;
      if ((e = launch_mass_residual(LT, z, m, x, st.lam, B, n, t, tp, np_, u, res, st.info, s, nw.idx, nw.nf,
                                    last ? nw.bidx : nw.idx, last ? nw.nb : nw.nf)) != hipSuccess)
        return e;
    }
    hipLaunchKernelGGL(k_nnls_dual, gv, dim3(256), 0, s, res, nw.F, tp, st.info, nw.y);
  }
  hipLaunchKernelGGL(k_nnls_finish, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, nw.state, B, st.info);
  return hipGetLastError();
}

hipError_t launch_bias_finalize(const double *w, int B, int64_t ld, int t, float eps, float bmin, float bmax,
                                const int32_t *info, float *beta, float *beta_ws, hipStream_t s) {
  hipLaunchKernelGGL(k_bias_finalize, dim3((unsigned)((ld + 255) / 256), B), dim3(256), 0, s, w, ld, t, eps, bmin,
                     bmax, info, beta, beta_ws);
  return hipGetLastError();
}

hipError_t launch_phat(int dtype, const float *LT, const float *beta_ws, int B, int n, int t, int64_t tp,
                       int64_t np_, void *out, void *outm, hipStream_t s) {
  dim3 grid((unsigned)(np_ / 64), B);
  if (dtype == ARCKV_BF16)
    hipLaunchKernelGGL(k_phat<bf16>, grid, dim3(256), 0, s, LT, beta_ws, n, t, tp, np_, out, outm);
  else
    hipLaunchKernelGGL(k_phat<float>, grid, dim3(256), 0, s, LT, beta_ws, n, t, tp, np_, out, outm);
  return hipGetLastError();
}

hipError_t launch_transpose128(int dtype, const float *in, int B, int rows, int64_t in_pair, int64_t rows_pad,
                               void *out, int64_t out_pair, hipStream_t s) {
  dim3 grid((unsigned)(rows_pad / 64), B);
  if (dtype == ARCKV_BF16)
    hipLaunchKernelGGL(k_transpose128<bf16>, grid, dim3(256), 0, s, in, rows, in_pair, rows_pad, out, out_pair);
  else
    hipLaunchKernelGGL(k_transpose128<float>, grid, dim3(256), 0, s, in, rows, in_pair, rows_pad, out, out_pair);
  return hipGetLastError();
}

// L X = R (fwd) or L^T X = R for 128 right-hand sides; R is overwritten, xt is
// scratch [B][ld][128].  From kTrsmLeftPairs pairs on left-looking (the figures above).
// Right-looking updates take 64 columns per workgroup while that leaves CUs idle, else
// all 128, which reads L once instead of twice.
constexpr int kTrsmLeftPairs = 65;
template <bool FWD>
static hipError_t trsm(const float *Gw, const void *lsplit, int B, int64_t ld, float *R, float *X, float *xt,
                       const int32_t *info, hipStream_t s) {
  const int nblk = (int)(ld / 256);
  const bool many = B >= kTrsmLeftPairs;
  for (int st = 0; st < nblk; ++st) {
    const int K = FWD ? st : nblk - 1 - st;
    if (many) {
      if (st > 0)
        hipLaunchKernelGGL(k_trsm_left<FWD>, dim3(256 / kTrsmLeftRows * (unsigned)B), dim3(512), 0, s, Gw, ld, K, R,
                           xt, info);
      hipLaunchKernelGGL(k_trsm_diag_left<FWD>, dim3(4 * (unsigned)B), dim3(256), 0, s, lsplit, ld, K, R, X, xt, info);
      continue;
    }
    hipLaunchKernelGGL(k_trsm_diag<FWD>, dim3(32, B), dim3(256), 0, s, lsplit, ld, K, R, X, xt, info);
    const int chunks = 4 * (nblk - 1 - st);
    if (chunks == 0) break;
    if ((int64_t)chunks * B < 512)
      hipLaunchKernelGGL((k_trsm_upd<FWD, 2>), dim3(2 * chunks, B), dim3(256), 0, s, Gw, ld, K, R, xt, info);
    else
      hipLaunchKernelGGL((k_trsm_upd<FWD, 4>), dim3(chunks, B), dim3(256), 0, s, Gw, ld, K, R, xt, info);
  }
  return hipGetLastError();
}

hipError_t launch_trsm(bool fwd, const float *Gw, const void *lsplit, int B, int64_t ld, float *R, float *X, float *xt,
                       const int32_t *info, hipStream_t s) {
  return fwd ? trsm<true>(Gw, lsplit, B, ld, R, X, xt, info, s) : trsm<false>(Gw, lsplit, B, ld, R, X, xt, info, s);
}

hipError_t launch_add(float *x, const float *dx, int B, int64_t n_per, const int32_t *info, hipStream_t s) {
  hipLaunchKernelGGL(k_add_copy, dim3((unsigned)((n_per + 255) / 256), B), dim3(256), 0, s, x, dx, n_per, info);
  return hipGetLastError();
}

hipError_t launch_values_out(const float *Xp, int B, int64_t tp, int t, const int32_t *info, float *Cv,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_values_out, dim3((unsigned)(((int64_t)t * kHeadDim + 255) / 256), B), dim3(256), 0, s, Xp, tp,
                     t, info, Cv);
  return hipGetLastError();
}

}  // namespace arckv
