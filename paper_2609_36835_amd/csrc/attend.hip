// Decode-time attention over a compacted block, optionally followed by an
// uncompressed block (eq. compact_attention; joint form of Appendix A.7,
// eq. concatenated_attention_preservation).  For pair p (one sequence and
// KV head) and each of its G query rows q:
//   o = softmax([s q C_k^T + beta, s q K_f^T]) [C_v; V_f]
// i.e. the fitted bias beta is added to the compact block's logits and the
// uncompressed block gets zero bias.  beta = NULL (zero bias) with C_k = K,
// C_v = V and F = 0 is plain full-cache attention.
//
// HBM-bound: every key and value row is read once.  Split-key ("flash
// decoding") in two kernels:
//   k_attend_partial  a workgroup of 8 waves takes 256 consecutive keys of
//                     the concatenated block; each wave scores its 32 keys
//                     against the G queries on MFMA 16x16x32 (keys as rows,
//                     queries as columns), takes the softmax of its chunk, and
//                     forms P V on MFMA too: the lane that holds a query's
//                     probabilities is the one that feeds them, so they pass
//                     through no LDS.  The eight waves' (max, sum, o) are
//                     merged in LDS into one partial per workgroup.  All of
//                     the chunk's K and V loads are issued up front, without
//                     branches.  Small calls are bound by the launches and one
//                     round trip to memory: 8 pairs of 856 keys take 9.1 us
//                     (11.1 us with P V on the VALU and loads under branches);
//                     512 pairs of 3533 keys, 160 us (197), 5.8 TB/s.
//   k_attend_combine  merges the partials of a pair with the usual
//                     max-rescaling and writes o.
#include <mutex>

#include "common.hpp"

namespace arckv {

namespace {
constexpr int kAttKPW = 32;                 // keys per wave
constexpr int kAttW = 8;                    // waves per workgroup
constexpr int kAttChunk = kAttW * kAttKPW;  // keys per workgroup

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

__device__ inline f32x4_t mfma16(bf16x8 a, bf16x8 b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The upper halves of two 32-bit words, one after the other.
__device__ inline uint32_t upper_halves(uint32_t first, uint32_t second) {
  return __builtin_amdgcn_perm(second, first, 0x07060302u);
}
__device__ inline uint32_t lower_halves(uint32_t first, uint32_t second) {
  return __builtin_amdgcn_perm(second, first, 0x05040100u);
}

// Row `key` of the concatenated block [compact (t rows); fixed (F rows)], the last
// row past the end.  By selection only: with branches the compiler waits for some
// loads inside them, a memory round trip each.
__device__ inline const bf16 *att_row(const bf16 *C, const bf16 *Fx, int p, int t, int F, int key) {
  key = min(key, t + F - 1);
  const bool c = key < t;
  return (c ? C : Fx) + ((int64_t)p * (c ? t : F) + (c ? key : key - t)) * kHeadDim;
}
}  // namespace

template <int G, bool STREAM>
__global__ void __launch_bounds__(64 * kAttW) k_attend_partial(int t, int F, float scale, const bf16 *__restrict__ Q,
                                                         const bf16 *__restrict__ Ck, const float *__restrict__ beta,
                                                         const bf16 *__restrict__ Cv, const bf16 *__restrict__ Kf,
                                                         const bf16 *__restrict__ Vf, float *__restrict__ part_o,
                                                         float *__restrict__ part_ml, int nch) {
  static_assert(G >= 1 && G <= 8, "query rows per pair");
  __shared__ __align__(16) float sO[kAttW][G][kHeadDim];   // per-wave partial outputs
  __shared__ float sM[kAttW][G], sL[kAttW][G];
  const int p = blockIdx.y, ch = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int L = t + F;
  const int key0 = ch * kAttChunk + wave * kAttKPW;
  const int g = lane >> 4, r = lane & 15;        // MFMA lane coordinates

  // ---- issue every load of the chunk: K as MFMA A fragments (key rows), V rows
  // for the PV pass (lane = the keys of its logits below x dims 8 r .. 8 r + 7)
  constexpr int KT = kAttKPW / 16, VI = kAttKPW / 4;
  bf16x8 kf[KT][4];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    const bf16 *row = att_row(Ck, Kf, p, t, F, key0 + 16 * kt + r);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[kt][ks] = *reinterpret_cast<const bf16x8 *>(row + 32 * ks + 8 * g);
  }
  // queries as the B operand: column r = query row r (the last one again for r >= G)
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8 *>(Q + ((size_t)p * G + min(r, G - 1)) * kHeadDim + 32 * ks + 8 * g);
  // the biases of this lane's keys, with the other loads: after the products
  // they would cost a memory round trip of their own
  float bv[VI];
#pragma unroll
  for (int i = 0; i < VI; ++i) bv[i] = 0.0f;
  if (beta && key0 < t) {
#pragma unroll
    for (int i = 0; i < VI; ++i) bv[i] = beta[(size_t)p * t + min(key0 + 16 * (i / 4) + 4 * g + i % 4, t - 1)];
  }
  union Frag {
    uint32_t w[4];
    bf16x8 v;
  };
  Frag vf[VI];
#pragma unroll
  for (int i = 0; i < VI; ++i) {
    const bf16x8 *v = reinterpret_cast<const bf16x8 *>(att_row(Cv, Vf, p, t, F, key0 + 16 * (i / 4) + 4 * g + i % 4) + 8 * r);
    vf[i].v = STREAM ? __builtin_nontemporal_load(v) : *v;
  }
  __builtin_amdgcn_sched_barrier(0);   // the loads stay above the products

  // ---- logits: lane (g, r) holds keys key0 + 16 kt + 4 g + j (j < 4) for query r
  float sv[VI];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = mfma16(kf[kt][ks], qf[ks], acc);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int key = key0 + 16 * kt + 4 * g + j;
      sv[4 * kt + j] = key < L ? fmaf(scale, acc[j], key < t ? bv[4 * kt + j] : 0.0f) : -INFINITY;
    }
  }
  // ---- softmax of the wave's keys per query (reduce the lane's VI, then over g)
  float m = sv[0];
#pragma unroll
  for (int i = 1; i < VI; ++i) m = fmaxf(m, sv[i]);
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  const float mref = m == -INFINITY ? 0.0f : m;   // a wave past the end keeps zero mass
  float l = 0.0f;
#pragma unroll
  for (int i = 0; i < VI; ++i) {
    sv[i] = __expf(sv[i] - mref);
    l += sv[i];
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (g == 0 && r < G) {
    sM[wave][r] = m;
    sL[wave][r] = l;
  }
  // ---- P V on MFMA over the wave's 32 keys: lane (g, r) holds query r's
  // probabilities of keys 16 (i / 4) + 4 g + i % 4, which is an A operand's row r
  // with those keys as its contraction slots 8 g + i, and V's same keys at dims
  // 8 r + e, which is column r of eight B operands, one per e.  Each probability
  // goes in as three bf16 terms (truncated, so all of one sign) that sum to it
  // exactly; the first has products of its own, which alone carry an infinite value
  // (0 times it in the other terms would be NaN).
  Frag ph, pm, pl;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t h[2], mi[2], lo[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float x = sv[2 * k + c];
      h[c] = __float_as_uint(x) & 0xffff0000u;
      const float x1 = x - __uint_as_float(h[c]);
      mi[c] = __float_as_uint(x1) & 0xffff0000u;
      lo[c] = __float_as_uint(x1 - __uint_as_float(mi[c]));
    }
    ph.w[k] = upper_halves(h[0], h[1]);
    pm.w[k] = upper_halves(mi[0], mi[1]);
    pl.w[k] = upper_halves(lo[0], lo[1]);
  }
  // a row past the end stands for zeros (its probability is zero, but zero times
  // an infinite value is not)
#pragma unroll
  for (int i = 0; i < VI; ++i)
    if (key0 + 16 * (i / 4) + 4 * g + i % 4 >= L) vf[i] = Frag{};
  float o[4][8];   // row 4 g + j = query, column 8 r + e
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    Frag b;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      b.w[k] = e & 1 ? upper_halves(vf[2 * k].w[e / 2], vf[2 * k + 1].w[e / 2])
                     : lower_halves(vf[2 * k].w[e / 2], vf[2 * k + 1].w[e / 2]);
    const f32x4_t first = mfma16(ph.v, b.v, f32x4_t{0.0f, 0.0f, 0.0f, 0.0f});
    const f32x4_t rest = mfma16(pm.v, b.v, mfma16(pl.v, b.v, f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}));
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j][e] = fabsf(first[j]) < INFINITY ? first[j] + rest[j] : first[j];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (4 * g + j < G) {
      float *to = &sO[wave][4 * g + j][8 * r];
      *reinterpret_cast<float4 *>(to) = make_float4(o[j][0], o[j][1], o[j][2], o[j][3]);
      *reinterpret_cast<float4 *>(to + 4) = make_float4(o[j][4], o[j][5], o[j][6], o[j][7]);
    }
  __syncthreads();
  // ---- merge the waves: one partial (max, sum, o) per query for the chunk
  float *po = part_o + (((size_t)p * nch + ch) * G) * kHeadDim;
  float *pml = part_ml + (((size_t)p * nch + ch) * G) * 2;
  for (int idx = tid; idx < G * kHeadDim; idx += 64 * kAttW) {
    const int q = idx / kHeadDim, dim = idx % kHeadDim;
    float M = sM[0][q];
#pragma unroll
    for (int w = 1; w < kAttW; ++w) M = fmaxf(M, sM[w][q]);
    const float Mref = M == -INFINITY ? 0.0f : M;
    float acc = 0.0f, lsum = 0.0f;
#pragma unroll
    for (int w = 0; w < kAttW; ++w) {
      const float f = sM[w][q] == -INFINITY ? 0.0f : __expf(sM[w][q] - Mref);
      acc = fmaf(f, sO[w][q][dim], acc);
      lsum = fmaf(f, sL[w][q], lsum);
    }
    po[(size_t)q * kHeadDim + dim] = acc;
    if (dim == 0) {
      pml[2 * q] = M;
      pml[2 * q + 1] = lsum;
    }
  }
}

// One workgroup per pair: thread (q, dim) merges the pair's nch partials.
__global__ void __launch_bounds__(1024) k_attend_combine(int G, const float *__restrict__ part_o,
                                                          const float *__restrict__ part_ml, int nch,
                                                          float *__restrict__ out) {
  const int p = blockIdx.x, idx = threadIdx.x;
  if (idx >= G * kHeadDim) return;
  const int q = idx / kHeadDim, dim = idx % kHeadDim;
  const float *ml = part_ml + (size_t)p * nch * G * 2;
  // Both sweeps are unrolled so that eight chunks' loads are in flight at once
  // (one dependent load per chunk left the long contexts latency-bound).
  float M = -INFINITY;
#pragma unroll 8
  for (int c = 0; c < nch; ++c) M = fmaxf(M, ml[((size_t)c * G + q) * 2]);
  const float Mref = M == -INFINITY ? 0.0f : M;
  float acc = 0.0f, lsum = 0.0f;
  const float *po = part_o + (size_t)p * nch * G * kHeadDim;
#pragma unroll 8
  for (int c = 0; c < nch; ++c) {
    const float mc = ml[((size_t)c * G + q) * 2];
    const float f = mc == -INFINITY ? 0.0f : __expf(mc - Mref);
    acc = fmaf(f, po[((size_t)c * G + q) * kHeadDim + dim], acc);
    lsum = fmaf(f, ml[((size_t)c * G + q) * 2 + 1], lsum);
  }
  out[((size_t)p * G + q) * kHeadDim + dim] = acc / lsum;
}

int attend_chunks(int t, int F) { return (t + F + kAttChunk - 1) / kAttChunk; }

// ---------------------------------------------------------------- static scratch
// The split-key partials of arckv_attend_noalloc live in this file-scope
// device array instead of a caller workspace: one copy per GPU, held until the
// process ends.  On the host the array's name is only a stand-in, never a
// device address; the address is taken once per device with
// hipGetSymbolAddress (with that device current) and kept here.
constexpr size_t kAttendScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kAttendScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

size_t attend_scratch_bytes() { return kAttendScratchBytes; }

// Device address of the current device's scratch array.
hipError_t attend_scratch(void **ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

// Keys and values of a call, in bytes, above which the values are read as a
// stream that the caches do not keep: what the 256 MB last-level cache holds.  Two
// streams that both pass through it slow each other down: 512 pairs of 32768, 16384,
// 8192 and 3533 keys take 1581, 756, 414 and 173 us with both kept (VALU products with
// loads under branches: 1557, 754, 403 and 197), 1451, 704, 371 and 160 us so; with
// both streamed 1601, 786, 390 and 178, with the keys alone 1556, 758, 385 and 182.  A
// call that fits may find its values there again: 8 pairs of 8192 keys 11.9 us kept, 12.5
// streamed.
constexpr int64_t kAttendKept = (int64_t)256 << 20;

hipError_t launch_attend(int P, int G, int t, int F, float scale, const void *Q, const void *Ck, const float *beta,
                         const void *Cv, const void *Kf, const void *Vf, float *part_o, float *part_ml, float *out,
                         hipStream_t s) {
  const int nch = attend_chunks(t, F);
  dim3 grid((unsigned)nch, (unsigned)P);
  const bool stream_v = (int64_t)P * (t + F) * 4 * kHeadDim > kAttendKept;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(64 * kAttW), 0, s, t, F, scale, (const bf16 *)Q, (const bf16 *)Ck, beta,
                       (const bf16 *)Cv, (const bf16 *)Kf, (const bf16 *)Vf, part_o, part_ml, nch);
  };
  switch (G) {
    case 1: stream_v ? go(k_attend_partial<1, true>) : go(k_attend_partial<1, false>); break;
    case 2: stream_v ? go(k_attend_partial<2, true>) : go(k_attend_partial<2, false>); break;
    case 4: stream_v ? go(k_attend_partial<4, true>) : go(k_attend_partial<4, false>); break;
    case 8: stream_v ? go(k_attend_partial<8, true>) : go(k_attend_partial<8, false>); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_attend_combine, dim3((unsigned)P), dim3((unsigned)(G * kHeadDim)), 0, s, G, part_o, part_ml,
                     nch, out);
  return hipGetLastError();
}

}  // namespace arckv
