// Key-to-anchor assignment with a certified argmax (Section 3.4,
// eq. anchor_assignment; ties to the lowest r).
//
// The bulk similarity contraction S[r][j] = sum_i U_S[i][r] E[i][j] runs on
// fp16 (bf16 inputs) or fp32 (fp32 inputs) operands; rounding the operands can
// reorder two anchors whose similarities to a key are close.  Every key is
// therefore decided in up to three passes, each a certified filter for the next:
//
//  A  the contraction keeps, per (anchor tile, key), the two best similarities
//     and the third value (EpiArgmax*).  With eta the relative and alpha the
//     absolute error bound of one similarity, no anchor r with
//     S_A(r) < (S_A(best) - alpha)(1 - eta)/(1 + eta) - alpha can be the argmax.
//     A key with exactly one anchor above that threshold is decided; the others
//     are flagged, with the best two of each tile above the threshold, or the
//     whole tile where its third value reaches it, as candidates
//     (k_assign_finalize).
//  C  flagged keys are re-scored against their candidates' fp32 profiles
//     (k_prof_anchor_*): for bf16 inputs the key's logits come from MFMA with
//     one fp32 accumulator per 16-wide slice of the head dimension, the eight
//     slices summed in fp32 (logit error at most gamma_23 s ||q|| ||k||), the
//     exponentials from v_exp_f32 (exp32_err), and each dot product from fp32
//     products summed four at a time, then in float64 (for fp32 inputs, float64
//     logits).  Keys that still have more than one survivor go on
//     (k_assign_refine).
//  D  float64 throughout: logits, exponentials, norms and dot products
//     (k_assign_exact).  Equal float64 similarities go to the lower r.
//
// The bounds are stated on the functions that use them.
#include <type_traits>

#include "assign.hpp"
#include "common.hpp"

namespace arckv {
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

constexpr double kU32 = 5.9604644775390625e-08;   // 2^-24, unit roundoff of fp32
constexpr double kU16 = 4.8828125e-04;            // 2^-11, unit roundoff of fp16

__device__ inline double gamma_m(double m) { return m * kU32 / (1.0 - m * kU32); }

// Per-pair constants of the error bounds.
struct AssignPair {
  double qmax;   // max_i ||q_i||_2
  double amax;   // max_r ||k_{s_r}||_2
};

// A fixed grid of nx workgroups per pair, remapped so that each XCD receives a
// contiguous range of (pair, x): all workgroups of a pair share one L2 (the
// pair's queries and anchor profiles are read by each of them).
__device__ inline void pair_block(int nx, int P, int &x, int &b) {
  const int64_t lin = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t tile = xcd_remap(lin, (int64_t)nx * P);
  b = (int)(tile / nx);
  x = (int)(tile % nx);
}

// ---------------------------------------------------------------- counters and norms
// Clears the work-list counters, the statistics and pn of P pairs.
__global__ void __launch_bounds__(256) k_assign_clear(AssignLists L, AssignPair *__restrict__ pn, int P) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < P * kAssignStats) L.stats[i] = 0;
  if (i >= P) return;
  L.fcnt[i] = L.dcnt[i] = 0;
  L.pcnt[i] = 0;
  pn[i] = {0.0, 0.0};
}

// Sum of squares of a 128-element row, in float64, loaded 16 bytes at a time.
template <typename E>
__device__ inline double row_sumsq(const E *x) {
  typedef __attribute__((__vector_size__(16))) E EV;
  constexpr int N = 16 / sizeof(E);
  double ss = 0.0;
#pragma unroll 4
  for (int k = 0; k < kHeadDim; k += N) {
    const EV w = *reinterpret_cast<const EV *>(x + k);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const double v = (double)(float)w[u];
      ss = fma(v, v, ss);
    }
  }
  return ss;
}

// pn[b] = {max_i ||q_i||, max_r ||k_{s_r}||}, in float64, rounded up by one part
// in 1e12 so that the bounds built on them stay upper bounds.  A row per
// thread over the n queries and the t anchors; the workgroups' maxima meet in
// an integer maximum of the (non-negative) doubles' bits.
template <typename E>
__global__ void __launch_bounds__(256) k_pair_norms(const E *__restrict__ Q, const E *__restrict__ K,
                                                    const int32_t *__restrict__ anchors, int n, int T, int t,
                                                    AssignPair *__restrict__ pn) {
  const int b = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  const bool isq = i < n;
  double v = 0.0;
  if (isq) v = row_sumsq(Q + ((size_t)b * n + i) * kHeadDim);
  else if (i - n < t) v = row_sumsq(K + ((size_t)b * T + anchors[(size_t)b * t + i - n]) * kHeadDim);
  double mq = isq ? v : 0.0, ma = isq ? 0.0 : v;
  for (int m = 32; m >= 1; m >>= 1) {
    mq = fmax(mq, __shfl_xor(mq, m, 64));
    ma = fmax(ma, __shfl_xor(ma, m, 64));
  }
  if ((threadIdx.x & 63) != 0) return;
  auto top = [](double *p, double ss) {
    if (ss > 0.0)
      atomicMax(reinterpret_cast<unsigned long long *>(p),
                (unsigned long long)__double_as_longlong(sqrt(ss) * (1.0 + 1e-12)));
  };
  top(&pn[b].qmax, mq);
  top(&pn[b].amax, ma);
}

// Logit of one (query, key) element from the eight 16-wide slices of the head
// dimension: each slice is one MFMA into a zero accumulator (products of bf16
// values are exact in fp32, so a slice sum is within gamma_16 of the sum of its
// |products|), and the eight slice sums are added in fp32 in a fixed order, so
// the logit is within gamma_23 s sum_k |q_k k_k| <= gamma_23 s ||q|| ||k|| of exact.
constexpr double kSliceTerms = 23.0;

// Relative error bound of exp(s l - z) evaluated as 2^(l c2 - z2) with c2 = s
// log2(e) and z2 = z log2(e) rounded to fp32, one fp32 fma and v_exp_f32 (1 ulp):
// the exponent's absolute error is at most u (2 |l c2| + 2 |z2| + |result|)
// and |result| <= |l c2| + |z2|.  A bounds |l c2|, Z bounds |z2|.
__device__ inline double exp32_err(double A, double Z) {
  return 0.6931471805599453 * kU32 * (3.0 * A + 3.0 * Z) + 2.0 * kU32;
}

// ---------------------------------------------------------------- anchor profiles
// Precise anchor profiles e_ir = exp(s q_i.k_{s_r} - z_merge) for bf16 inputs:
// logits from eight MFMA slices added in a fixed order (kSliceTerms), the
// exponential in fp32 (exp32_err).  Ua [P][tp][np] float32 (zero for i >= n);
// npart [ranges][P][tp] the squared norms' parts, accumulated in float64.  A
// workgroup owns 128 anchors (32 per wave, kept as MFMA B fragments) and one
// range of the queries, swept in tiles of 64.
__global__ void __launch_bounds__(256) k_prof_anchor_bf16(const bf16 *__restrict__ Q, const bf16 *__restrict__ K,
                                                          const int32_t *__restrict__ anchors,
                                                          const float *__restrict__ zmerge, int n, int T, int t,
                                                          int64_t tp, int64_t np_, int tiles_per, double scale,
                                                          float *__restrict__ Ua, double *__restrict__ npart) {
  constexpr int SQ = kHeadDim + 8;
  __shared__ __attribute__((aligned(16))) bf16 sQ[64 * SQ];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = lane >> 5, col = lane & 31;
  const int r = blockIdx.x * 128 + wave * 32 + col;
  const bool rvalid = r < t;
  bf16x8 bfr[8];
  const bf16 *kr = K + ((size_t)b * T + (rvalid ? anchors[(size_t)b * t + r] : 0)) * kHeadDim;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    bfr[ks] = rvalid ? *reinterpret_cast<const bf16x8 *>(kr + ks * 16 + 8 * h) : Mfma<bf16>::zero();
  const float c2 = (float)(scale * 1.4426950408889634), zs2 = zmerge[b] * 1.4426950408889634f;
  const bf16 *Qb = Q + (size_t)b * n * kHeadDim;
  float *urow = Ua + ((size_t)b * tp + (rvalid ? r : 0)) * np_;
  double ss = 0.0;
  // the next 64-query tile is loaded into registers while this one is processed
  f32x4 qn[4];
  auto fetch_q = [&](int j0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = tid + 256 * u, rr = c / 16, cc = (c % 16) * 8;
      qn[u] = j0 + rr < n ? *reinterpret_cast<const f32x4 *>(Qb + (size_t)(j0 + rr) * kHeadDim + cc)
                          : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  const int i_lo = 64 * tiles_per * blockIdx.z, i_hi = (int)min(np_, (int64_t)i_lo + 64 * tiles_per);
  fetch_q(i_lo);
  for (int i0 = i_lo; i0 < i_hi; i0 += 64) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = tid + 256 * u, rr = c / 16, cc = (c % 16) * 8;
      *reinterpret_cast<f32x4 *>(&sQ[rr * SQ + cc]) = qn[u];
    }
    if (i0 + 64 < i_hi) fetch_q(i0 + 64);
    __syncthreads();
#pragma unroll
    for (int ms = 0; ms < 2; ++ms) {
      const bf16 *arow = &sQ[(32 * ms + col) * SQ + 8 * h];
      f32x16 lsum = Mfma<bf16>::mma(*reinterpret_cast<const bf16x8 *>(arow), bfr[0], zero16());
#pragma unroll
      for (int ks = 1; ks < 8; ++ks) {
        const f32x16 part = Mfma<bf16>::mma(*reinterpret_cast<const bf16x8 *>(arow + ks * 16), bfr[ks], zero16());
#pragma unroll
        for (int v = 0; v < 16; ++v) lsum[v] += part[v];
      }
      float e[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = i0 + 32 * ms + acc_row(v, lane);
        const float ev = i < n ? __builtin_amdgcn_exp2f(fmaf(lsum[v], c2, -zs2)) : 0.0f;
        ss = fma((double)ev, (double)ev, ss);
        e[v] = ev;
      }
      if (rvalid) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4 *>(urow + i0 + 32 * ms + 8 * g + 4 * h) =
              f32x4{e[4 * g], e[4 * g + 1], e[4 * g + 2], e[4 * g + 3]};
      }
    }
  }
  ss += __shfl_xor(ss, 32, 64);
  if (rvalid && h == 0) npart[((size_t)blockIdx.z * gridDim.y + b) * tp + r] = ss;
}

// fp32 inputs: the same profiles with float64 logits and exponentials (one
// workgroup per anchor, one thread per query).
__global__ void __launch_bounds__(256) k_prof_anchor_f32(const float *__restrict__ Q, const float *__restrict__ K,
                                                         const int32_t *__restrict__ anchors,
                                                         const float *__restrict__ zmerge, int n, int T, int t,
                                                         int64_t tp, int64_t np_, double scale,
                                                         float *__restrict__ Ua, double *__restrict__ npart) {
  __shared__ double kr[kHeadDim];
  __shared__ double red[4];
  const int b = blockIdx.y, r = blockIdx.x, tid = threadIdx.x;
  if (tid < kHeadDim) kr[tid] = (double)K[((size_t)b * T + anchors[(size_t)b * t + r]) * kHeadDim + tid];
  __syncthreads();
  const double zm = (double)zmerge[b];
  float *urow = Ua + ((size_t)b * tp + r) * np_;
  double ss = 0.0;
  for (int64_t i = tid; i < np_; i += 256) {
    double ev = 0.0;
    if (i < n) {
      const float *q = Q + ((size_t)b * n + i) * kHeadDim;
      double l = 0.0;
      for (int k = 0; k < kHeadDim; ++k) l = fma((double)q[k], kr[k], l);
      ev = exp(scale * l - zm);
    }
    ss = fma(ev, ev, ss);
    urow[i] = (float)ev;
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) npart[(size_t)b * tp + r] = red[0] + red[1] + red[2] + red[3];
}

// anorm [P][tp] = ||e_r||_2 from the parts of its square, and the
// contraction's anchor operand U [P][tp][np]: Ua / anorm, stored in fp16
// scaled by 2^15 for bf16 inputs (one rounding of the fp32 product) or in
// fp32; rows r >= t and columns i >= n are zero.  One wave per row, four
// consecutive columns per lane (np_ is a multiple of 256).
template <typename T>
__global__ void __launch_bounds__(256) k_anchor_u(const float *__restrict__ Ua, const double *__restrict__ npart,
                                                  int ranges, int n, int t, int64_t tp, int64_t np_, float uscale,
                                                  double *__restrict__ anorm, T *__restrict__ U) {
  typedef __attribute__((__vector_size__(4 * sizeof(T)))) T T4;
  const int b = blockIdx.y, lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= tp) return;
  T *urow = U + ((size_t)b * tp + r) * np_;
  const float *arow = Ua + ((size_t)b * tp + r) * np_;
  double nr = 0.0;
  if (r < t) {
    for (int z = 0; z < ranges; ++z) nr += npart[((size_t)z * gridDim.y + b) * tp + r];
    nr = sqrt(nr);
    if (lane == 0) anorm[(size_t)b * tp + r] = nr;
  }
  const float inv = nr > 0.0 ? (float)((double)uscale / nr) : 0.0f;
  for (int64_t i = 4 * lane; i < np_; i += 256) {
    f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
    if (r < t && i < n) a = *reinterpret_cast<const f32x4 *>(arow + i);
    T4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (T)(i + e < n ? a[e] * inv : 0.0f);
    *reinterpret_cast<T4 *>(urow + i) = o;
  }
}

// ---------------------------------------------------------------- pass A bounds
// Relative (eta) and absolute (alpha, in the units of the stored similarity)
// error bound of one pass-A similarity of key j, whose key has norm kn and mass
// weight phi.  Every term of S(j, r) = sum_i E_ij U_ir is >= 0, so a relative
// bound on each term bounds the sum.
//  bf16 inputs, fp16 operands scaled by 2^15 (S_A = 2^30 S):
//   E'  logit on MFMA, fp32 accumulation over d: gamma_128 s ||q|| ||k_j||;
//       exponent argument formed in fp32 and v_exp_f32 (1 ulp); fp16 rounding.
//   U'  the precise profile (gamma_23 s ||q|| ||k_r|| + exp32_err, fp32),
//       divided by its float64 norm (same bound), a fp32 product and one fp16
//       rounding.
//   fp16 x fp16 products are exact in fp32; the fp32 accumulation of n >= 0
//   terms adds gamma_n; the epilogue truncates the stored value by < 2^-18.  Operands below the fp16 normal range (E' or U' < 2^-14)
//   carry an absolute error <= 2^-25 instead: alpha = 2^-25 (||U'_r||_1 + ||E'_j||_1)
//   <= 2^-10 (sqrt(n) + n phi_j), with ||U_r||_2 = 1.
//  fp32 inputs: fp32 products are rounded (u each, d + 2 terms in the logit and
//   one in every product of the contraction); the anchor operand is the float64
//   profile rounded to fp32 and normalised in fp32.
struct BoundA {
  double eta, alpha;
};

__device__ inline BoundA bound_a(bool bf16in, int n, double s, double zm, const AssignPair &pn, double kn,
                                 double phi) {
  const double A = s * pn.qmax * kn * 1.4426950408889634 * 1.001;   // |logit| log2(e) bound of the key
  BoundA o;
  if (bf16in) {
    const double Z = fabs(zm) * 1.4426950408889634 + (double)kProfLog2Scale;
    const double e_key = gamma_m(kHeadDim) * s * pn.qmax * kn + 0.6931471805599453 * kU32 * (3.0 * A + 4.0 * Z) +
                         2.0 * kU32;
    const double e_anc = gamma_m(kSliceTerms) * s * pn.qmax * pn.amax +
                         exp32_err(s * pn.qmax * pn.amax * 1.4426950408889634 * 1.001, fabs(zm) * 1.4426950408889634);
    const double eE = (1.0 + e_key) * (1.0 + kU16) - 1.0;
    const double eU = (1.0 + e_anc + kU32) / (1.0 - e_anc) * (1.0 + 2.0 * kU32) * (1.0 + kU16) - 1.0;
    // the contraction's epilogue stores similarities with the low 5 bits
    // cleared (relative truncation < 2^-18)
    o.eta = (1.0 + eE) * (1.0 + eU) * (1.0 + gamma_m(n)) * (1.0 + 3.814697265625e-06) - 1.0;
    o.alpha = 9.765625e-04 * 1.01 * (sqrt((double)n) + (double)n * phi * 1.001) + (double)n * 1e-18;
  } else {
    const double Z = fabs(zm) * 1.4426950408889634;
    const double e_key = gamma_m(kHeadDim + 2) * s * pn.qmax * kn +
                         0.6931471805599453 * kU32 * (3.0 * A + 4.0 * Z) + 2.0 * kU32;
    const double eU = 3.0 * kU32 + 1e-14;
    o.eta = (1.0 + e_key) * (1.0 + eU) * (1.0 + kU32) * (1.0 + gamma_m(n)) - 1.0;
    o.alpha = (double)n * 1e-36;
  }
  return o;
}

__device__ inline float threshold_a(float s1, const BoundA &bd) {
  const double th = ((double)s1 - bd.alpha) * (1.0 - bd.eta) / (1.0 + bd.eta) - bd.alpha;
  // round down so that a similarity equal to the exact threshold is kept
  return (float)th - fabsf((float)th) * 1.2e-7f - 1e-37f;
}

template <typename E>
__device__ inline double row_norm(const E *x) {
  return sqrt(row_sumsq(x)) * (1.0 + 1e-12);
}

// Candidate anchors of one key after pass A.  For each anchor tile the best
// two above the threshold are candidates; a tile whose third value reaches the
// threshold may hold more, and contributes all its anchors ("overflow").
struct CandA {
  int singles, overflow;
  int count;   // the candidates, with every anchor of an overflowing tile
  float th;
  uint64_t g1;
};

__device__ inline CandA cand_a(const uint64_t *p1, const uint64_t *p2, const uint32_t *p3, int64_t stride, int MT,
                               int t, int TR, float th_or_nan, uint64_t g1) {
  CandA c;
  c.g1 = g1;
  c.th = th_or_nan;
  c.singles = 0;
  c.overflow = 0;
  c.count = 0;
#pragma unroll 4
  for (int mt = 0; mt < MT; ++mt) {
    const uint64_t a = p1[(size_t)mt * stride], b2 = p2[(size_t)mt * stride];
    const float v3 = __uint_as_float(p3[(size_t)mt * stride]);
    const bool over = v3 >= c.th;
    const int one = (int)(a != 0ull && packed_r(a) < (uint32_t)t && packed_sim(a) >= c.th) +
                    (int)(b2 != 0ull && packed_r(b2) < (uint32_t)t && packed_sim(b2) >= c.th);
    c.overflow += over;
    c.singles += over ? 0 : one;
    c.count += over ? min(t, (mt + 1) * TR) - mt * TR : one;
  }
  return c;
}

// Queue key j for the float64 pass with k candidates starting at pool offset
// off (off < 0: all t anchors).  More than kPassDSplit pool candidates are
// split over consecutive entries; the capacity dcap covers the largest split
// the pool allows.
__device__ inline void push_d(const AssignLists &L, int b, int j, int off, int k) {
  const bool split = off >= 0 && k > kPassDSplit;
  const int ne = split ? (k + kPassDSplit - 1) / kPassDSplit : 1;
  const int slot = atomicAdd(&L.dcnt[b], ne);
  for (int e = 0; e < ne; ++e) {
    const size_t q = (size_t)b * L.dcap + slot + e;
    L.dkey[q] = j;
    L.doff[q] = split ? off + e * kPassDSplit : off;
    L.dn[q] = split ? min(kPassDSplit, k - e * kPassDSplit) : k;
    L.dgrp[q] = split ? slot : -1;
    L.dgn[q] = ne;
  }
  atomicAdd(&L.stats[b * kAssignStats + 1], 1);
}

// Pass A decision, one thread per position j: anchors map to themselves
// (eq. anchor_assignment); a key with one candidate takes it; the others take
// the pass-A best for now, and their candidates go to the pair's pool for
// pass C.  Anchor tiles have TR rows.
template <typename E>
__global__ void __launch_bounds__(256) k_assign_finalize(
    const uint64_t *__restrict__ part1, const uint64_t *__restrict__ part2, const uint32_t *__restrict__ part3,
    int MT, int64_t Np, const int32_t *__restrict__ anchors, const E *__restrict__ K, const float *__restrict__ phi,
    const float *__restrict__ zmerge, const AssignPair *__restrict__ pn, int T, int t, int n, int TR, double s,
    int32_t *__restrict__ kappa, AssignLists L) {
  const int b = blockIdx.y;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= T) return;
  const int32_t *S = anchors + (size_t)b * t;
  int lo = 0, hi = t;   // lo = #{anchors < j}
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (S[mid] < j) lo = mid + 1;
    else hi = mid;
  }
  if (lo < t && S[lo] == j) {
    kappa[(size_t)b * T + j] = lo;
    return;
  }
  const size_t c = (size_t)b * MT * Np + (size_t)(j - lo);
  const uint64_t *p1 = part1 + c, *p2 = part2 + c;
  const uint32_t *p3 = part3 + c;
  uint64_t g1 = 0;
#pragma unroll 4
  for (int mt = 0; mt < MT; ++mt) g1 = max(g1, p1[(size_t)mt * Np]);
  const uint32_t r1 = packed_r(g1);
  const double kn = row_norm(K + ((size_t)b * T + j) * kHeadDim);
  const BoundA bd = bound_a(sizeof(E) == 2, n, s, (double)zmerge[b], pn[b], kn, (double)phi[(size_t)b * T + j]);
  const float th = threshold_a(packed_sim(g1), bd);
  const CandA ca = cand_a(p1, p2, p3, Np, MT, t, TR, th, g1);
  kappa[(size_t)b * T + j] = (int32_t)(r1 < (uint32_t)t ? r1 : 0u);
  if (ca.overflow == 0 && ca.singles == 1) return;
  int32_t *st = L.stats + (size_t)b * kAssignStats;
  atomicAdd(&st[0], 1);
  if (ca.overflow) atomicAdd(&st[7], 1);
  // the key's candidates: the best two above the threshold of each tile, or
  // every anchor of a tile whose third value reaches it (four tiles' partials at a
  // time, as above: one after the other, each of three walks took a round trip per
  // tile; 692 -> 573 us at 64 pairs of T = 32768, t = 3277)
  auto listed = [&](uint64_t a) { return a != 0ull && packed_r(a) < (uint32_t)t && packed_sim(a) >= th; };
  const int nc = ca.count;
  atomicAdd(&st[2], nc);
  if (nc == 0) {   // no finite similarity reaches the threshold (non-finite input): the pass-A best stands
    atomicAdd(&st[3], 1);
    atomicAdd(&st[4], 1);
    return;
  }
  const int64_t off = (int64_t)atomicAdd(&L.pcnt[b], (unsigned long long)nc);
  if (off + nc > L.pcap) {   // pool full (near-equal profiles): decided in float64 over all t anchors
    push_d(L, b, j, -1, t);
    return;
  }
  int32_t *pl = L.pool + (size_t)b * L.pcap + off;
  int k = 0;
  for (int m0 = 0; m0 < MT; m0 += 4) {
    float v3[4];
    uint64_t a[4], a2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t at = (size_t)min(m0 + u, MT - 1) * Np;
      v3[u] = __uint_as_float(p3[at]);
      a[u] = p1[at];
      a2[u] = p2[at];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int mt = m0 + u;
      if (mt >= MT) break;
      if (v3[u] >= th) {
        for (int r = mt * TR; r < min(t, (mt + 1) * TR); ++r) pl[k++] = r;
        continue;
      }
      if (listed(a[u])) pl[k++] = (int32_t)packed_r(a[u]);
      if (listed(a2[u])) pl[k++] = (int32_t)packed_r(a2[u]);
    }
  }
  const int slot = atomicAdd(&L.fcnt[b], 1);
  L.fkey[(size_t)b * L.cap + slot] = j;
  L.foff[(size_t)b * L.cap + slot] = (int32_t)off;
  L.fn[(size_t)b * L.cap + slot] = nc;
  atomicAdd(&st[6], 1);
}

// Workgroup barrier that waits for this wave's LDS operations only: global
// loads issued before it stay in flight across it.
__device__ __forceinline__ void lds_only_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0); vmcnt and expcnt unconstrained
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------- pass C
// Refine the keys queued by pass A.  The queued keys of a pair form groups of
// 64 (in queue order) and a group's candidates in the pool form chunks of CAP;
// each (group, chunk) is one work item.  The keys' profiles are formed in
// fp32 and each candidate pair accumulates sum_i e_ij e_ir (fp32 products
// summed four at a time, then in float64) against the anchor's stored
// profile; the similarity e_j . e_r / ||e_r|| goes back to the pool, and
// k_assign_decide takes the decisions once every item is done.
//  bf16 inputs: logits from eight MFMA slices as in k_prof_anchor_bf16
//   (kSliceTerms), exponentials within exp32_err.  Bound of one similarity:
//   (1 + eps_k)(1 + eps_a)/(1 - eps_a)(1 + gamma_4) - 1 with eps_k = gamma_23 s
//   ||q|| ||k_j|| + exp32_err and eps_a the same with max ||k_r|| (profile and norm).
//  fp32 inputs: float64 logits and exponentials; the bound is the fp32
//   rounding of the two profiles and of the partial products.
// A key whose best similarity exceeds every other candidate's by more than the
// bound on both is decided; the survivors of the others go to pass D.
// Work distribution: k_refine_plan lays out each pair's (group, chunk) pieces
// (goff), and every piece is cut into nspl query ranges, each an item of its own
// that leaves a part of the similarities (summed in order by k_assign_decide);
// a fixed grid of kRefineBlocks workgroups per pair takes consecutive runs of
// items, so few pieces still use many CUs, the chunks of one group with many
// candidates (keys whose candidates include whole anchor tiles) spread over
// workgroups, and a workgroup with several ranges of one piece sets it up once.
// One range: 154 us at 8 pairs, T = 8192 (n = 4096); in ranges 95 us (fp32, 2 pairs
// of T = 1024, n = 256: 100 and 17 us).
// The queries are swept in tiles of 128.  Per tile the eight waves form the 64 keys' profiles (one
// 32 x 32 MFMA tile each: a key half by a quarter of the queries) into a
// shared LDS tile; each wave takes 32 candidates, two per load instruction: a
// half-wave covers one candidate's 128 queries, four per lane, so every load
// reads two contiguous 512-byte runs of anchor profile rows.  The candidates'
// partial sums stay in registers (float64) across the tiles and are reduced
// over the half-waves once per item.
constexpr int kRefineBlocks = 128;
constexpr int kRefineCpw = 32;   // candidates per wave

template <typename E>
__global__ void __launch_bounds__(512, 2) k_assign_refine(const E *__restrict__ Q, const E *__restrict__ K,
                                                       const float *__restrict__ zmerge,
                                                       const float *__restrict__ Ua, const double *__restrict__ anorm,
                                                       int T, int n, int64_t tp, int64_t np_, double s,
                                                       AssignLists L) {
  constexpr bool BF = sizeof(E) == 2;
  constexpr int NK = 64, NW = 8, CPW = kRefineCpw, CAP = NW * CPW, QT = 128, SE = QT + 4;
  constexpr int SKB = BF ? kHeadDim + 8 : kHeadDim + 4;   // key-row stride (elements)
  __shared__ int32_t kpos[NK], koff[NK], kbase[NK + 1], khalf, item_g, item_c0, item_sp;
  __shared__ int32_t cr[CAP];
  __shared__ int32_t ck[CAP];
  __shared__ __attribute__((aligned(16))) E sK[NK * SKB];
  __shared__ __attribute__((aligned(16))) float eS[NK * SE];   // the keys' profiles on one query tile
  // pair-major over the whole grid (no XCD remap): the anchor profiles do not
  // fit an L2 anyway, and a pair with many candidates spreads over every XCD
  const int bx = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = lane >> 5, col = lane & 31;
  const int F = L.fcnt[b];
  const double zm = (double)zmerge[b];
  const float c2 = (float)(s * 1.4426950408889634), zs2 = zmerge[b] * 1.4426950408889634f;
  const E *Qb = Q + (size_t)b * n * kHeadDim;
  const float *Uab = Ua + (size_t)b * tp * np_;
  int32_t *pool = L.pool + (size_t)b * L.pcap;
  const int nspl = L.nspl;
  double *psim = L.psim + (size_t)b * 2 * nspl * L.pcap;
  const int tiles_per = ((n + QT - 1) / QT + nspl - 1) / nspl;   // query tiles per range
  const int kt = wave >> 2, qsub = wave & 3;   // this wave's key half and query quarter in the profile phase
  const int G = (F + NK - 1) / NK;
  const int32_t *goff = L.goff + (size_t)b * L.gcap;
  const int items = F > 0 ? goff[G] * nspl : 0;
  const int run = (items + kRefineBlocks - 1) / kRefineBlocks;
  int cur = -1, cur_c0 = -1;   // the group and the chunk in the shared arrays
  for (int it = bx * run; it < min(items, (bx + 1) * run); ++it) {   // uniform over the workgroup
    __syncthreads();   // the previous item is done with the shared arrays
    if (tid == 0) {   // the group g with goff[g] <= piece < goff[g + 1]
      const int piece = it / nspl;
      int lo = 0, hi = G;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (goff[mid] <= piece) lo = mid;
        else hi = mid;
      }
      item_g = lo;
      item_c0 = (piece - goff[lo]) * CAP;
      item_sp = it - piece * nspl;
    }
    __syncthreads();
    const int g = item_g, c0 = item_c0, sp = item_sp;
    const bool same = g == cur && c0 == cur_c0;   // another range of the piece set up before
    cur_c0 = c0;
    if (g != cur) {   // load the group's keys (uniform)
      cur = g;
      const int f0 = g * NK, nk = min(NK, F - f0);
      if (tid < NK) {
        kpos[tid] = -1;
        koff[tid] = 0;
        if (tid < nk) {
          const size_t q = (size_t)b * L.cap + f0 + tid;
          kpos[tid] = L.fkey[q];
          koff[tid] = L.foff[q];
        }
      }
      __syncthreads();
      if (wave == 0) {   // first candidate slot of each key: a prefix sum over the wave
        const int m = lane < nk ? L.fn[(size_t)b * L.cap + f0 + lane] : 0;
        int x = m;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const int y = __shfl_up(x, d, 64);
          if (lane >= d) x += y;
        }
        kbase[lane] = x - m;
        if (lane == 63) kbase[NK] = x;
      }
      for (int x = tid; x < NK * kHeadDim; x += NW * 64) {   // the keys' rows (zero for empty slots)
        const int k = x / kHeadDim, c = x % kHeadDim;
        sK[k * SKB + c] = kpos[k] >= 0 ? K[((size_t)b * T + kpos[k]) * kHeadDim + c] : (E)0.0f;
      }
      __syncthreads();
    }
    const int total = kbase[NK];
    {
      const int cn = min(CAP, total - c0);
      if (!same) {
      __syncthreads();   // the previous chunk is done with cr / ck / khalf
      if (tid == 0) khalf = 0;
      __syncthreads();
      for (int c = tid; c < CAP; c += NW * 64) {
        int lo = -1, r = 0;
        if (c < cn) {
          const int gi = c0 + c;
          int lo2 = 0, hi = NK;   // the key k with kbase[k] <= gi < kbase[k + 1]
          while (hi - lo2 > 1) {
            const int mid = (lo2 + hi) >> 1;
            if (kbase[mid] <= gi) lo2 = mid;
            else hi = mid;
          }
          lo = lo2;
          r = pool[koff[lo] + gi - kbase[lo]];
          atomicOr(&khalf, 1 << (lo >> 5));   // which 32-key halves this chunk's candidates belong to
        }
        ck[c] = lo;
        cr[c] = r;
      }
      __syncthreads();
      }
      const int need = khalf;
      const int i_lo = QT * tiles_per * sp, i_hi = min(n, i_lo + QT * tiles_per);   // this item's queries
      double acc[CPW / 2];
#pragma unroll
      for (int u = 0; u < CPW / 2; ++u) acc[u] = 0.0;
      const int cw0 = wave * CPW;   // this wave's candidates cw0 + 2u + h
      const int qo = 4 * col;        // half-wave lane col covers queries i0 + 4 col .. + 3
      // Loads are unconditional so that the compiler can count them exactly
      // across the tile loop (a load under a branch may not have been issued,
      // which forces a full drain at the next use): an empty candidate slot
      // holds anchor 0 and is skipped when used; query rows past n are
      // clamped, and their profiles are zeroed below.
      auto load_w = [&](int i0, int u) -> f32x4 {
        const int c = cw0 + 2 * u + h;
        return *reinterpret_cast<const f32x4 *>(Uab + (size_t)cr[c] * np_ + i0 + qo);
      };
      // bf16 inputs: the loads run one query tile ahead.  The query fragments
      // of tile i0 + 128 are issued as soon as the MFMAs of tile i0 have read
      // theirs, and each anchor-profile value of tile i0 + 128 as soon as its
      // tile-i0 value is used; the tile barriers wait for LDS only.  Vector
      // loads complete in issue order, so the profile phase waits for its
      // query fragments alone while the anchor values stay in flight.
      // fp32 inputs: one tile at a time.
      bf16x8 qa[BF ? 8 : 1];
      auto load_q = [&](int i0) {
        if constexpr (BF) {
          const int iq = i0 + 32 * qsub + col;   // this lane's query row of the MFMA A operand
          const bf16 *qrow = reinterpret_cast<const bf16 *>(Qb) + (size_t)(iq < n ? iq : n - 1) * kHeadDim + 8 * h;
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) qa[ks] = *reinterpret_cast<const bf16x8 *>(qrow + ks * 16);
        }
      };
      auto tile_barrier = [&]() {
        if constexpr (BF) lds_only_barrier();
        else __syncthreads();
      };
      f32x4 w[CPW / 2];
      if constexpr (BF) {
        load_q(min(i_lo, n - 1));
        // the same issue order as at the end of each tile (query fragments,
        // then anchor values), so that the counts agree at the loop head
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < CPW / 2; ++u) w[u] = load_w(i_lo < n ? i_lo : 0, u);
      }
      for (int i0 = i_lo; i0 < i_hi; i0 += QT) {   // none in a range past the last query
        const int nxt = i0 + QT < i_hi ? i0 + QT : i0;   // the last tile reloads itself
        if constexpr (!BF) {
#pragma unroll
          for (int u = 0; u < CPW / 2; ++u) w[u] = load_w(i0, u);
        }
        // ---- the 64 keys' profiles on queries [i0, i0 + 128) (bf16: always, so
        // that no load or MFMA of the tile loop sits under a branch)
        if constexpr (BF) {
          f32x16 lsum;
          const bf16 *krow = reinterpret_cast<const bf16 *>(sK) + (kt * 32 + col) * SKB + 8 * h;
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 bk = *reinterpret_cast<const bf16x8 *>(krow + ks * 16);
            const f32x16 part = Mfma<bf16>::mma(qa[ks], bk, zero16());
            if (ks == 0) lsum = part;
            else {
#pragma unroll
              for (int v = 0; v < 16; ++v) lsum[v] += part[v];
            }
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int qi = 32 * qsub + acc_row(v, lane);
            const float ev = i0 + qi < n ? __builtin_amdgcn_exp2f(fmaf(lsum[v], c2, -zs2)) : 0.0f;
            eS[(kt * 32 + col) * SE + qi] = ev;
          }
        } else {
          // float64 logits on fp64 MFMA (16 x 16 x 4; fp32 values are exact in
          // fp64): wave w forms queries 16 w .. + 15 of the tile against the four
          // 16-key groups, each lane supplying k = 16 g + 4 lk + u to product u of
          // group g
          const int lr = lane & 15, lk = lane >> 4;
          const float *qrow = reinterpret_cast<const float *>(Qb) + (size_t)min(i0 + 16 * wave + lr, n - 1) * kHeadDim + 4 * lk;
          f32x4 bq[8];
#pragma unroll
          for (int gg = 0; gg < 8; ++gg) bq[gg] = *reinterpret_cast<const f32x4 *>(qrow + 16 * gg);
          const int qi = 16 * wave + lr;
#pragma unroll
          for (int k4 = 0; k4 < 4; ++k4) {
            if (!((need >> (k4 >> 1)) & 1)) continue;   // no candidate of this key half in the chunk
            const float *krow = reinterpret_cast<const float *>(sK) + (16 * k4 + lr) * SKB + 4 * lk;
            f64x4 l0 = {0.0, 0.0, 0.0, 0.0}, l1 = l0;
#pragma unroll
            for (int gg = 0; gg < 8; gg += 2) {
              const f32x4 a0 = *reinterpret_cast<const f32x4 *>(krow + 16 * gg);
              const f32x4 a1 = *reinterpret_cast<const f32x4 *>(krow + 16 * gg + 16);
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                l0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a0[u], (double)bq[gg][u], l0, 0, 0, 0);
                l1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a1[u], (double)bq[gg + 1][u], l1, 0, 0, 0);
              }
            }
            // lane holds keys 16 k4 + 4 r + lk for query 16 w + lr
#pragma unroll
            for (int r = 0; r < 4; ++r)
              eS[(16 * k4 + 4 * r + lk) * SE + qi] = i0 + qi < n ? (float)exp(s * (l0[r] + l1[r]) - zm) : 0.0f;
          }
        }
        if constexpr (BF) load_q(nxt);   // the MFMAs above have read qa
        tile_barrier();   // the tile's profiles are complete
        // ---- CPW candidates per wave: half-wave h takes candidate cw0 + 2u + h
        // Branch-free: an empty slot reads key 0's profile and adds an exact zero.
#pragma unroll
        for (int u = 0; u < CPW / 2; ++u) {
          const int k = ck[cw0 + 2 * u + h];
          const f32x4 e4 = *reinterpret_cast<const f32x4 *>(&eS[(k >= 0 ? k : 0) * SE + qo]);
          float p4 = e4[0] * w[u][0];   // four non-negative products in fp32 (within gamma_4), then float64
#pragma unroll
          for (int e = 1; e < 4; ++e) p4 = fmaf(e4[e], w[u][e], p4);
          acc[u] += k >= 0 ? (double)p4 : 0.0;
          if constexpr (BF) w[u] = load_w(nxt, u);
        }
        tile_barrier();   // reads of the tile done before the next one overwrites it
      }
      // ---- reduce each candidate's partial sums over its half-wave
#pragma unroll
      for (int u = 0; u < CPW / 2; ++u) {
        double d = acc[u];
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) d += __shfl_xor(d, m, 64);
        const int c = cw0 + 2 * u + h;
        if (col == 0 && c < cn) {
          const int k = ck[c];
          psim[(size_t)sp * L.pcap + koff[k] + c0 + c - kbase[k]] = d / anorm[(size_t)b * tp + cr[c]];
        }
      }
    }
  }
}

// Pass C work items: each group of 64 queued keys (in queue order) has
// ceil(candidates / cap_c) chunks; goff[g] is the first item of group g (an
// exclusive prefix) and goff[G] the pair's item count.  One workgroup per
// pair, 256 groups per scan step.
__global__ void __launch_bounds__(256) k_refine_plan(AssignLists L, int cap_c) {
  __shared__ int32_t sc[256];
  __shared__ int32_t carry;
  const int b = blockIdx.x, tid = threadIdx.x;
  const int F = L.fcnt[b], G = (F + 63) / 64;
  int32_t *goff = L.goff + (size_t)b * L.gcap;
  const int32_t *fn = L.fn + (size_t)b * L.cap;
  if (tid == 0) carry = 0;
  for (int g0 = 0; g0 < G; g0 += 256) {   // uniform over the workgroup
    const int g = g0 + tid;
    int nit = 0;
    if (g < G) {
      int tot = 0;
      for (int k = g * 64; k < min(F, g * 64 + 64); ++k) tot += fn[k];
      nit = (tot + cap_c - 1) / cap_c;
    }
    __syncthreads();   // carry holds the previous steps' total
    sc[tid] = nit;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {   // inclusive scan
      const int v = tid >= d ? sc[tid - d] : 0;
      __syncthreads();
      sc[tid] += v;
      __syncthreads();
    }
    if (g < G) goff[g] = carry + sc[tid] - nit;
    __syncthreads();
    if (tid == 0) carry += sc[255];
  }
  __syncthreads();
  if (tid == 0) goff[G] = carry;
}

// The largest similarity of N consecutive lanes and its anchor, equal ones to the lower r.
template <int N>
__device__ __forceinline__ void best_of(double &sim, int &r) {
#pragma unroll
  for (int w = N / 2; w >= 1; w >>= 1) {
    const double os = __shfl_xor(sim, w, 64);
    const int orr = __shfl_xor(r, w, 64);
    if (os > sim || (os == sim && orr < r)) {
      sim = os;
      r = orr;
    }
  }
}

// Pass C decision, one wave per queued key, once every chunk of its
// candidates has its similarity: the best one (equal ones to the lower r)
// becomes the key's anchor for now, the candidates within the bound of it
// survive, compacted in place and in order at the front of the key's pool
// segment, and a key with more than one survivor goes to pass D.  A wave and
// not a thread: a key with whole anchor tiles has up to t candidates, which
// one thread read one dependent load at a time (77 us against 8 for 8 pairs of
// T = 15,001, t = 1500).
template <typename E>
__global__ void __launch_bounds__(256) k_assign_decide(const E *__restrict__ K, const float *__restrict__ zmerge,
                                                       const AssignPair *__restrict__ pn, int T, double s,
                                                       int32_t *__restrict__ kappa, AssignLists L) {
  constexpr bool BF = sizeof(E) == 2;
  const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int F = L.fcnt[b];
  const AssignPair pp = pn[b];
  const double zm = (double)zmerge[b];
  int32_t *pool = L.pool + (size_t)b * L.pcap;
  const double *psim = L.psim + (size_t)b * 2 * L.nspl * L.pcap;
  auto sim = [&](int c) {   // the query ranges' parts, in order
    double v = psim[c];
    for (int sp = 1; sp < L.nspl; ++sp) v += psim[(size_t)sp * L.pcap + c];
    return v;
  };
  for (int f = blockIdx.x * 4 + wave; f < F; f += gridDim.x * 4) {   // uniform over the wave
    const size_t q = (size_t)b * L.cap + f;
    const int j = L.fkey[q], o = L.foff[q], m = L.fn[q];
    if (m <= 0) continue;
    double bs = -INFINITY;
    int br = 0x7FFFFFFF;
    for (int c = lane; c < m; c += 64) {
      const double v = sim(o + c);
      const int r = pool[o + c];
      if (v > bs || (v == bs && r < br)) {
        bs = v;
        br = r;
      }
    }
    best_of<64>(bs, br);
    if (br == 0x7FFFFFFF) {   // no comparable similarity (non-finite input): the first candidate stands
      if (lane == 0) kappa[(size_t)b * T + j] = pool[o];
      continue;
    }
    double eta;
    if constexpr (BF) {
      const E *kr = K + ((size_t)b * T + j) * kHeadDim + 2 * lane;   // the row's norm, two elements per lane
      const double k0 = (double)(float)kr[0], k1 = (double)(float)kr[1];
      const double kn = sqrt(wave_sum(fma(k0, k0, k1 * k1))) * (1.0 + 1e-12);
      const double g = gamma_m(kSliceTerms) * s * pp.qmax, Z = fabs(zm) * 1.4426950408889634;
      const double ek = g * kn + exp32_err(s * pp.qmax * kn * 1.4426950408889634 * 1.001, Z);
      const double ea = g * pp.amax + exp32_err(s * pp.qmax * pp.amax * 1.4426950408889634 * 1.001, Z);
      eta = (1.0 + ek) * (1.0 + ea) / (1.0 - ea) * (1.0 + gamma_m(4)) * (1.0 + 1e-12) - 1.0;
    } else {
      eta = 3.0 * kU32 + gamma_m(4) + 1e-12;
    }
    const double thc = bs * (1.0 - eta) / (1.0 + eta) - 1e-300;
    if (lane == 0) kappa[(size_t)b * T + j] = br;
    // writes trail reads: this wave alone owns the key's pool segment, and a
    // round's 64 candidates are read before its survivors are written
    int ns = 0;
    for (int c0 = 0; c0 < m; c0 += 64) {
      const int c = c0 + lane;
      const bool keep = c < m && sim(o + c) >= thc;
      const int r = keep ? pool[o + c] : 0;
      const uint64_t mask = __ballot(keep);
      if (keep) pool[o + ns + __popcll(mask & ((1ull << lane) - 1ull))] = r;
      ns += __popcll(mask);
    }
    if (ns > 1 && lane == 0) push_d(L, b, j, o, ns);
  }
}

// ---------------------------------------------------------------- pass D
// Float64 decision for the remaining keys: logits as float64 sums of exact
// products, exp in float64, norms and dot products in float64; the largest
// similarity wins and equal ones go to the lower r.  A key's entries are the
// anchors that survived pass C.  k_exact_plan packs consecutive queued
// entries into items of up to 32 vectors (an entry is its key and its
// candidates); a fixed grid of kExactBlocks workgroups per pair takes items
// it = blockIdx.x, blockIdx.x + kExactBlocks, ...  An item's keys and
// candidate anchors share one sweep over the queries in tiles of 64, and an
// entry with more candidates than fit (all t anchors) continues in the next
// sweep.
// The queries of an item are cut into nspl ranges, each a work item of its own;
// a candidate's parts of the dot product and of the squared norm take the place
// of its refined similarities, which are read by then, and k_exact_merge adds
// them in order and decides.  An entry over all t anchors runs over all queries
// and decides by itself.  Whole sweeps took 288 us at 8 pairs of T = 8192,
// n = 4096, with some ten items per pair; in ranges 75 us.
constexpr int kExactBlocks = 128;

// Pass D work items: greedy packing of consecutive entries into items of at
// most 32 vectors (an entry needs 1 + its candidates; a larger one forms an
// item of its own).  ditem = {count, first entry of each item, dcnt}.  One
// workgroup per pair; entry sizes staged in LDS, packed by one thread.
__global__ void __launch_bounds__(256) k_exact_plan(AssignLists L) {
  constexpr int W = 2048;
  __shared__ int32_t sdn[W];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int D = L.dcnt[b];
  const int32_t *dn = L.dn + (size_t)b * L.dcap, *doff = L.doff + (size_t)b * L.dcap;
  int32_t *items = L.ditem + (size_t)b * (L.dcap + 2);
  int nit = 0, nv = 0;   // thread 0 only
  for (int w0 = 0; w0 < D; w0 += W) {   // uniform over the workgroup
    const int nw = min(W, D - w0);
    __syncthreads();   // thread 0 is done with the previous window
    // an entry over all t anchors has an item of its own however few they are
    for (int x = tid; x < nw; x += 256) sdn[x] = doff[w0 + x] < 0 ? 32 : dn[w0 + x];
    __syncthreads();
    if (tid == 0) {
      for (int x = 0; x < nw; ++x) {
        const int need = 1 + sdn[x];
        if (w0 + x == 0 || nv + need > 32) {
          items[1 + nit++] = w0 + x;
          nv = 0;
        }
        nv += need;
      }
    }
  }
  if (tid == 0) {
    items[0] = nit;
    items[1 + nit] = D;
  }
}

// Decisions, 16 lanes per entry: the largest similarity of its candidates and, for
// the first entry of a split key, of all the key's entries (which are consecutive, as
// are their candidates), equal ones to the lower r.  One thread per entry read up to
// t candidates of a tied key in turn, each 2 nspl float64 values: 50 us at 64 pairs of
// T = 32768 (a wave per entry 21, 16 lanes 8).
__global__ void __launch_bounds__(256) k_exact_merge(int T, int32_t *__restrict__ kappa, AssignLists L) {
  const int b = blockIdx.y, lane = threadIdx.x & 15;
  const int D = L.dcnt[b];
  const double *part = L.psim + (size_t)b * 2 * L.nspl * L.pcap;
  const int32_t *pool = L.pool + (size_t)b * L.pcap;
  for (int di = blockIdx.x * 16 + (threadIdx.x >> 4); di < D; di += gridDim.x * 16) {   // uniform over the 16 lanes
    const size_t q = (size_t)b * L.dcap + di;
    const int o = L.doff[q], grp = L.dgrp[q];
    if (o < 0 || (grp >= 0 && grp != di)) continue;   // decided in its item, or with the key's first entry
    int m = L.dn[q];
    if (grp >= 0) {
      int more = 0;
      for (int e = 1 + lane; e < L.dgn[q]; e += 16) more += L.dn[q + e];
#pragma unroll
      for (int w = 8; w >= 1; w >>= 1) more += __shfl_xor(more, w, 64);
      m += more;
    }
    double bs = -1.0;
    int br = 0x7FFFFFFF;
    for (int c = lane; c < m; c += 16) {
      double dot = 0.0, nn = 0.0;
      for (int sp = 0; sp < L.nspl; ++sp) {
        dot += part[(size_t)(2 * sp) * L.pcap + o + c];
        nn += part[(size_t)(2 * sp + 1) * L.pcap + o + c];
      }
      const double sim = nn > 0.0 ? dot / sqrt(nn) : 0.0;
      const int r = pool[o + c];
      if (sim > bs || (sim == bs && r < br)) {
        bs = sim;
        br = r;
      }
    }
    best_of<16>(bs, br);
    if (lane == 0 && br != 0x7FFFFFFF) kappa[(size_t)b * T + L.dkey[q]] = br;
  }
}

template <typename E>
__global__ void __launch_bounds__(256) k_assign_exact(const E *__restrict__ Q, const E *__restrict__ K,
                                                      const int32_t *__restrict__ anchors,
                                                      const float *__restrict__ zmerge, int T, int t, int n, double s,
                                                      int32_t *__restrict__ kappa, AssignLists L) {
  constexpr int NV = 32, NQ = 64, SK = kHeadDim + 4;
  __shared__ __attribute__((aligned(16))) float sK[NV * SK];
  __shared__ __attribute__((aligned(16))) float sQ[NQ * SK];
  __shared__ double sE[NV * (NQ + 1)];
  __shared__ int32_t vpos[NV], vown[NV], vr[NV], vpool[NV];
  __shared__ double vdot[NV], vnn[NV];
  // batch segments: first and one-past-last vector, continues, final
  __shared__ int32_t sg_v0[NV], sg_v1[NV], sg_cont[NV], sg_final[NV];
  __shared__ int32_t nv_s, nseg_s, di_s, ci_s, done_s;
  __shared__ double run_sim;
  __shared__ int32_t run_r;
  int bx, b;
  pair_block(kExactBlocks, gridDim.y, bx, b);
  const int tid = threadIdx.x;
  const int D = L.dcnt[b];
  const int32_t *S = anchors + (size_t)b * t;
  const double zm = (double)zmerge[b];
  const E *Qb = Q + (size_t)b * n * kHeadDim;
  // rows of 128 elements of E as 4 floats per thread-step (bf16: 4 values = 8 bytes)
  auto load4 = [](const E *p) -> f32x4 {
    if constexpr (sizeof(E) == 2) {
      const bf16x4 v = *reinterpret_cast<const bf16x4 *>(p);
      return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
    } else {
      return *reinterpret_cast<const f32x4 *>(p);
    }
  };
  const int32_t *items = L.ditem + (size_t)b * (L.dcap + 2);
  const int nspl = L.nspl, nitems = D > 0 ? items[0] * nspl : 0;
  const int run = (nitems + kExactBlocks - 1) / kExactBlocks;
  const int tiles_per = ((n + NQ - 1) / NQ + nspl - 1) / nspl;
  double *part = L.psim + (size_t)b * 2 * nspl * L.pcap;
  for (int it = bx * run; it < min(nitems, (bx + 1) * run); ++it) {   // uniform over the workgroup
    const int item = it / nspl, sp = it - item * nspl;
    const int g0 = items[1 + item], g1 = items[2 + item];
    const bool direct = L.doff[(size_t)b * L.dcap + g0] < 0;   // all t anchors: all queries, decided here
    if (direct && sp != 0) continue;
    const int i_lo = direct ? 0 : NQ * tiles_per * sp, i_hi = direct ? n : min(n, i_lo + NQ * tiles_per);
    __syncthreads();   // every thread has left the previous item's loop
    if (tid == 0) {
      di_s = g0;
      ci_s = 0;
      done_s = 0;
    }
    __syncthreads();
    while (!done_s) {
      // the next batch, built by the first wave: lane e holds entry di_s + e (an
      // item has at most 16 that fit a batch), a prefix sum gives its first vector,
      // and lane v then looks up vector v
      if (tid < 64) {
        const int di0 = di_s, ci0 = ci_s, e = tid;
        const size_t q = (size_t)b * L.dcap + di0 + e;
        const bool have = e < 16 && di0 + e < g1;
        const int left = have ? L.dn[q] - (e == 0 ? ci0 : 0) : 0;   // candidates of the entry not yet taken
        const int key = have ? L.dkey[q] : 0, off = have ? L.doff[q] : 0;
        int x = have ? 1 + left : 0;
        const int need = x;
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
          const int y = __shfl_up(x, d, 64);
          if (tid >= d) x += y;
        }
        const int v0 = x - need;
        // an entry takes part if its key and one candidate fit; the last one may be cut off
        const bool in = have && v0 + 2 <= NV;
        const int v1 = min(v0 + need, NV);
        const uint64_t im = __ballot(in);
        const int ns = __popcll(im);   // entries 0 .. ns - 1
        if (in) {
          sg_cont[e] = e == 0 && ci0 > 0;
          sg_v0[e] = v0;
          sg_v1[e] = v1;
          sg_final[e] = v1 == v0 + need;
        }
        const int nv = __shfl(v1, ns - 1, 64);
        int en = 0;   // this lane's vector: its entry is the last with v0 <= tid
        for (int k = 1; k < ns; ++k) en += __shfl(v0, k, 64) <= tid;
        const int ev0 = __shfl(v0, en, 64), ekey = __shfl(key, en, 64), eoff = __shfl(off, en, 64);
        if (tid < nv) {
          const int ci = tid - ev0 - 1 + (en == 0 ? ci0 : 0);
          if (tid == ev0) {
            vpos[tid] = ekey;
            vown[tid] = -1;
            vr[tid] = -1;
            vpool[tid] = -1;
          } else {
            const int r = eoff < 0 ? ci : L.pool[(size_t)b * L.pcap + eoff + ci];   // every anchor is a candidate
            vpos[tid] = S[r];
            vown[tid] = ev0;
            vr[tid] = r;
            vpool[tid] = eoff + ci;
          }
        }
        const int lv0 = __shfl(v0, ns - 1, 64), lneed = __shfl(need, ns - 1, 64);
        if (tid == 0) {
          const bool cut = nv < lv0 + lneed;   // the last entry goes on in the next batch
          nv_s = nv;
          nseg_s = ns;
          di_s = di0 + ns - (cut ? 1 : 0);
          ci_s = cut ? (ns == 1 ? ci0 : 0) + nv - lv0 - 1 : 0;
        }
      }
      __syncthreads();
      const int nv = nv_s;
      for (int x = tid; x < NV * kHeadDim / 4; x += 256) {
        const int v = x / (kHeadDim / 4), k = 4 * (x % (kHeadDim / 4));
        const f32x4 w = v < nv ? load4(K + ((size_t)b * T + vpos[v]) * kHeadDim + k) : f32x4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4 *>(&sK[v * SK + k]) = w;
      }
      __syncthreads();   // sK and the batch's vectors are published
      // Running sums of vector rv: eight lanes per vector (queries 8 rq .. 8 rq + 7
      // of each tile), combined in a fixed tree and kept by the first lane.
      const int rv = tid >> 3, rq = tid & 7;
      const int vo = rv < nv ? vown[rv] : -1;
      double acc_d = 0.0, acc_n = 0.0;
      const int lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = lane >> 4;
      // the next query tile is loaded into registers while this one's products run
      constexpr int QCH = NQ * kHeadDim / 4 / 256;   // groups of 4 values per thread
      using Raw = std::conditional_t<sizeof(E) == 2, bf16x4, f32x4>;
      Raw qn[QCH];
      auto fetch_q = [&](int j0) {
#pragma unroll
        for (int c = 0; c < QCH; ++c) {
          const int x = tid + 256 * c, q = x / (kHeadDim / 4), k = 4 * (x % (kHeadDim / 4));
          qn[c] = j0 + q < n ? *reinterpret_cast<const Raw *>(Qb + (size_t)(j0 + q) * kHeadDim + k) : Raw{};
        }
      };
      fetch_q(i_lo);
      for (int i0 = i_lo; i0 < i_hi; i0 += NQ) {   // none in a range past the last query
        __syncthreads();   // every wave is done with the previous tile
#pragma unroll
        for (int c = 0; c < QCH; ++c) {
          const int x = tid + 256 * c, q = x / (kHeadDim / 4), k = 4 * (x % (kHeadDim / 4));
          f32x4 w;
#pragma unroll
          for (int u = 0; u < 4; ++u) w[u] = (float)qn[c][u];
          *reinterpret_cast<f32x4 *>(&sQ[q * SK + k]) = w;
        }
        if (i0 + NQ < i_hi) fetch_q(i0 + NQ);
        __syncthreads();
        // logits on fp64 MFMA (16 x 16 x 4): wave w owns queries 16 w .. 16 w + 15
        // of the tile and both 16-vector halves; each lane supplies k = 16 g + 4 lk + u
        // to the four products of group g (bf16 / fp32 values are exact in fp64)
        f64x4 c0 = {0.0, 0.0, 0.0, 0.0}, c1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
        for (int g = 0; g < kHeadDim / 16; ++g) {
          const f32x4 a0 = *reinterpret_cast<const f32x4 *>(&sK[lr * SK + 16 * g + 4 * lk]);
          const f32x4 a1 = *reinterpret_cast<const f32x4 *>(&sK[(16 + lr) * SK + 16 * g + 4 * lk]);
          const f32x4 bq = *reinterpret_cast<const f32x4 *>(&sQ[(16 * wave + lr) * SK + 16 * g + 4 * lk]);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            c0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a0[u], (double)bq[u], c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a1[u], (double)bq[u], c1, 0, 0, 0);
          }
        }
        // lane holds vectors 4 r + lk (and + 16) for query 16 w + lr
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int v = 4 * r + lk, q = 16 * wave + lr;
          const bool qv = i0 + q < n;
          sE[v * (NQ + 1) + q] = v < nv && qv ? exp(s * c0[r] - zm) : 0.0;
          sE[(v + 16) * (NQ + 1) + q] = v + 16 < nv && qv ? exp(s * c1[r] - zm) : 0.0;
        }
        __syncthreads();
        double d = 0.0, nn = 0.0;
        if (vo >= 0) {
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const int q = 8 * rq + x;
            const double ev = sE[rv * (NQ + 1) + q];
            d = fma(sE[vo * (NQ + 1) + q], ev, d);
            nn = fma(ev, ev, nn);
          }
        }
        d += __shfl_xor(d, 1, 64);
        nn += __shfl_xor(nn, 1, 64);
        d += __shfl_xor(d, 2, 64);
        nn += __shfl_xor(nn, 2, 64);
        d += __shfl_xor(d, 4, 64);
        nn += __shfl_xor(nn, 4, 64);
        acc_d += d;
        acc_n += nn;
      }
      if (rq == 0) {
        if (direct) {
          vdot[rv] = acc_d;
          vnn[rv] = acc_n;
        } else if (vo >= 0) {
          part[(size_t)(2 * sp) * L.pcap + vpool[rv]] = acc_d;
          part[(size_t)(2 * sp + 1) * L.pcap + vpool[rv]] = acc_n;
        }
      }
      __syncthreads();
      if (tid == 0) {
        for (int g = 0; direct && g < nseg_s; ++g) {
          double bs = sg_cont[g] ? run_sim : -1.0;
          int br = sg_cont[g] ? run_r : 0x7FFFFFFF;
          for (int v = sg_v0[g] + 1; v < sg_v1[g]; ++v) {
            const double sim = vnn[v] > 0.0 ? vdot[v] / sqrt(vnn[v]) : 0.0;
            if (sim > bs || (sim == bs && vr[v] < br)) {
              bs = sim;
              br = vr[v];
            }
          }
          if (sg_final[g]) {
            if (br != 0x7FFFFFFF) kappa[(size_t)b * T + vpos[sg_v0[g]]] = br;
          } else {
            run_sim = bs;
            run_r = br;
          }
        }
        done_s = di_s >= g1;
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------- launchers
// Clears the work lists' counters and the statistics, then pn.
hipError_t launch_pair_norms(int dtype, const void *Q, const void *K, const int32_t *anchors, int P, int n, int T,
                             int t, void *pn, const AssignLists &L, hipStream_t s) {
  hipLaunchKernelGGL(k_assign_clear, dim3((unsigned)((P * kAssignStats + 255) / 256)), dim3(256), 0, s, L,
                     (AssignPair *)pn, P);
  const dim3 g((unsigned)(((int64_t)n + t + 255) / 256), P);
  if (dtype == ARCKV_BF16)
    hipLaunchKernelGGL(k_pair_norms<bf16>, g, dim3(256), 0, s, (const bf16 *)Q, (const bf16 *)K, anchors, n, T, t,
                       (AssignPair *)pn);
  else
    hipLaunchKernelGGL(k_pair_norms<float>, g, dim3(256), 0, s, (const float *)Q, (const float *)K, anchors, n, T, t,
                       (AssignPair *)pn);
  return hipGetLastError();
}

// npart: scratch for npart_blocks [P][tp] blocks of doubles (at least one).
// While the 128-anchor groups of the call's `all` pairs are fewer than kAnchorGroups
// workgroups (four per CU), each one's query sweep is cut into up to eight ranges:
// 8 pairs with n = 4096, t = 819 took 155 us whole, 36 us in ranges; n = 3000, t =
// 1500: 130 and 44 us.  The pairs of the call, not the P of this chunk: the ranges
// group the norms' sums, and a pair's result must not depend on its chunk.
constexpr int kAnchorGroups = 1024;
hipError_t launch_anchor_profiles(int dtype, const void *Q, const void *K, const int32_t *anchors,
                                  const float *zmerge, int P, int all, int n, int T, int t, int64_t tp, int64_t np_,
                                  float scale, float *Ua, double *anorm, double *npart, int64_t npart_blocks, void *U,
                                  hipStream_t s) {
  if (dtype == ARCKV_BF16) {
    const int64_t groups = (int64_t)((t + 127) / 128) * all, tiles = np_ / 64;
    int64_t ranges = kAnchorGroups / groups;
    for (int64_t lim : {(int64_t)8, npart_blocks, tiles}) ranges = ranges < lim ? ranges : lim;
    if (ranges < 1) ranges = 1;
    const int per = (int)((tiles + ranges - 1) / ranges);
    ranges = (tiles + per - 1) / per;
    hipLaunchKernelGGL(k_prof_anchor_bf16, dim3((unsigned)((t + 127) / 128), P, (unsigned)ranges), dim3(256), 0, s,
                       (const bf16 *)Q, (const bf16 *)K, anchors, zmerge, n, T, t, tp, np_, per, (double)scale, Ua,
                       npart);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_anchor_u<f16>, dim3((unsigned)(tp / 4), P), dim3(256), 0, s, (const float *)Ua,
                       (const double *)npart, (int)ranges, n, t, tp, np_, kProfScale, anorm, (f16 *)U);
  } else {
    hipLaunchKernelGGL(k_prof_anchor_f32, dim3((unsigned)t, P), dim3(256), 0, s, (const float *)Q, (const float *)K,
                       anchors, zmerge, n, T, t, tp, np_, (double)scale, Ua, npart);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_anchor_u<float>, dim3((unsigned)(tp / 4), P), dim3(256), 0, s, (const float *)Ua,
                       (const double *)npart, 1, n, t, tp, np_, 1.0f, anorm, (float *)U);
  }
  return hipGetLastError();
}

__global__ void k_fill_i32(int32_t *p, int64_t count, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = v;
}

hipError_t launch_fill_i32(int32_t *p, int64_t count, int32_t v, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count, v);
  return hipGetLastError();
}

// Pass A decision.  MT anchor tiles of TR rows;
// Np = the partials' row stride (compacted key columns).
hipError_t launch_assign_finalize(int dtype, const void *K, const uint64_t *part1, const uint64_t *part2,
                                  const uint32_t *part3, int MT, int TR, int64_t Np, const int32_t *anchors,
                                  const float *phi, const float *zmerge, const void *pn, int P, int T, int t, int n,
                                  float scale, int32_t *kappa, const AssignLists &L, hipStream_t s) {
  const dim3 gf((unsigned)((T + 255) / 256), P);
  if (dtype == ARCKV_BF16)
    hipLaunchKernelGGL(k_assign_finalize<bf16>, gf, dim3(256), 0, s, part1, part2, part3, MT, Np, anchors,
                       (const bf16 *)K, phi, zmerge, (const AssignPair *)pn, T, t, n, TR, (double)scale, kappa, L);
  else
    hipLaunchKernelGGL(k_assign_finalize<float>, gf, dim3(256), 0, s, part1, part2, part3, MT, Np, anchors,
                       (const float *)K, phi, zmerge, (const AssignPair *)pn, T, t, n, TR, (double)scale, kappa, L);
  return hipGetLastError();
}

// Pass C (a grid of early exits where nothing is queued).
hipError_t launch_assign_refine(int dtype, const void *Q, const void *K, const float *zmerge, const void *pn,
                                const float *Ua, const double *anorm, int P, int T, int t, int n, int64_t tp,
                                int64_t np_, float scale, int32_t *kappa, const AssignLists &L, hipStream_t s) {
  if (T - t <= 0) return hipSuccess;
  const bool bf = dtype == ARCKV_BF16;
  hipLaunchKernelGGL(k_refine_plan, dim3(P), dim3(256), 0, s, L, 8 * kRefineCpw);
  const dim3 g(kRefineBlocks, P), gd(64, P);
  if (bf) {
    hipLaunchKernelGGL(k_assign_refine<bf16>, g, dim3(512), 0, s, (const bf16 *)Q, (const bf16 *)K, zmerge, Ua,
                       anorm, T, n, tp, np_, (double)scale, L);
    hipLaunchKernelGGL(k_assign_decide<bf16>, gd, dim3(256), 0, s, (const bf16 *)K, zmerge, (const AssignPair *)pn,
                       T, (double)scale, kappa, L);
  } else {
    hipLaunchKernelGGL(k_assign_refine<float>, g, dim3(512), 0, s, (const float *)Q, (const float *)K, zmerge, Ua,
                       anorm, T, n, tp, np_, (double)scale, L);
    hipLaunchKernelGGL(k_assign_decide<float>, gd, dim3(256), 0, s, (const float *)K, zmerge,
                       (const AssignPair *)pn, T, (double)scale, kappa, L);
  }
  return hipGetLastError();
}

// Pass D.
hipError_t launch_assign_exact(int dtype, const void *Q, const void *K, const int32_t *anchors, const float *zmerge,
                               int P, int T, int t, int n, float scale, int32_t *kappa, const AssignLists &L,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_exact_plan, dim3(P), dim3(256), 0, s, L);
  if (dtype == ARCKV_BF16)
    hipLaunchKernelGGL(k_assign_exact<bf16>, dim3(kExactBlocks, P), dim3(256), 0, s, (const bf16 *)Q,
                       (const bf16 *)K, anchors, zmerge, T, t, n, (double)scale, kappa, L);
  else
    hipLaunchKernelGGL(k_assign_exact<float>, dim3(kExactBlocks, P), dim3(256), 0, s, (const float *)Q,
                       (const float *)K, anchors, zmerge, T, t, n, (double)scale, kappa, L);
  hipLaunchKernelGGL(k_exact_merge, dim3(32, P), dim3(256), 0, s, T, kappa, L);
  return hipGetLastError();
}

}  // namespace arckv
