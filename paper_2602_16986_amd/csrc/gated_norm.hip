// U-gated layer normalisation after the attention (paper Eq. 4 without the f2 projection):
//   Y = (LayerNorm_D(A) * gamma + beta) * U          over the D = H*d features of each token
// and its backward (gated_norm_backward of the paper's appendix pseudocode, which recomputes the
// normalised activations instead of saving them).  Both passes are HBM-bound streaming kernels:
// one wavefront per token row, 16-byte loads per lane, wave-level reductions through DPP
// shuffles, everything between the load and the store in registers.
#include "hstu_common.h"
#include "hstu_kernels.h"
#include "partial_sums.h"

namespace hstu {

constexpr int kRowsPerBlock = 4;        // forward: one wave per row, 4 waves per workgroup
constexpr int kBwdWaves = 8;            // backward: 8 waves per workgroup, each walking over rows
constexpr int kMaxBwdBlocks = 512;      // two workgroups per CU; also the number of partial column-sum rows

// op over the 64 lanes of a wave, in every lane: neighbours, pairs, quads (mirrored in 8), octets (mirrored in 16), then rows in
// pairs and halves
template <typename Op> __device__ __forceinline__ float wave_all(float v, Op op) {
  v = op(v, dpp<0xB1>(v));                                 // quad_perm 1 0 3 2
  v = op(v, dpp<0x4E>(v));                                 // quad_perm 2 3 0 1
  v = op(v, dpp<0x141>(v));                                // row_half_mirror
  v = op(v, dpp<0x140>(v));                                // row_mirror
  const uint32_t a = __builtin_bit_cast(uint32_t, v);
  const auto p = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  v = op(__builtin_bit_cast(float, (uint32_t)p[0]), __builtin_bit_cast(float, (uint32_t)p[1]));
  const uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto q = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (uint32_t)q[0]), __builtin_bit_cast(float, (uint32_t)q[1]));
}
__device__ __forceinline__ float wave_sum(float v) { return wave_all(v, [](float x, float y) { return x + y; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_all(v, [](float x, float y) { return fmaxf(x, y); }); }

// 8 consecutive elements starting at element index e0 of a row, widened to fp32
template <typename E>
__device__ __forceinline__ void load8(const E* row, int e0, float (&v)[8]) {
  if constexpr (sizeof(E) == 2) {
    const u32x4 raw = *(const u32x4*)(row + e0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(raw[i] << 16);
      v[2 * i + 1] = __uint_as_float(raw[i] & 0xFFFF0000u);
    }
  } else {
    const f32x4 a = *(const f32x4*)(row + e0), b = *(const f32x4*)(row + e0 + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
  }
}

template <typename E>
__device__ __forceinline__ void store8(E* row, int e0, const float (&v)[8]) {
  if constexpr (sizeof(E) == 2) {
    *(u32x4*)(row + e0) = (u32x4){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                                  pack_bf16x2(v[6], v[7])};
  } else {
    *(f32x4*)(row + e0) = (f32x4){v[0], v[1], v[2], v[3]};
    *(f32x4*)(row + e0 + 4) = (f32x4){v[4], v[5], v[6], v[7]};
  }
}
// 8 consecutive elements as loaded (one 16-byte chunk of bf16, two of fp32), widened when they are used
template <typename E> struct Raw8;
template <> struct Raw8<__bf16> { u32x4 w; };
template <> struct Raw8<float> { f32x4 lo, hi; };
__device__ __forceinline__ Raw8<__bf16> load8raw(const __bf16* row, int e0) { return {*(const u32x4*)(row + e0)}; }
__device__ __forceinline__ Raw8<float> load8raw(const float* row, int e0) { return {*(const f32x4*)(row + e0), *(const f32x4*)(row + e0 + 4)}; }
__device__ __forceinline__ void widen8(const Raw8<__bf16>& r, float (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(r.w[i] << 16);
    v[2 * i + 1] = __uint_as_float(r.w[i] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ void widen8(const Raw8<float>& r, float (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[i] = r.lo[i]; v[4 + i] = r.hi[i]; }
}

// v[i] *= d/dt [t sigmoid(t)] at t = pre[i]: the gradient passes back through a SiLU whose input is `pre`
template <typename E>
__device__ __forceinline__ void dsilu8(const Raw8<E>& pre, float (&v)[8]) {
  float t[8];
  widen8(pre, t);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * t[i]));
    v[i] *= sg * (1.0f + t[i] * (1.0f - sg));
  }
}

// mean and reciprocal standard deviation of one row held as NCH chunks of 8 per lane
template <int NCH>
__device__ __forceinline__ void row_stats(const float (&a)[NCH][8], int lane, int D, float eps, float& mu, float& rs) {
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c)
    if ((lane + 64 * c) * 8 < D)
#pragma unroll
      for (int i = 0; i < 8; ++i) s += a[c][i];
  mu = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c)
    if ((lane + 64 * c) * 8 < D)
#pragma unroll
      for (int i = 0; i < 8; ++i) { const float dlt = a[c][i] - mu; q += dlt * dlt; }
  const float var = wave_sum(q) / (float)D;
  rs = 1.0f / sqrtf(var + eps);
}

template <typename E, int NCH>
__global__ __launch_bounds__(64 * kRowsPerBlock) void gated_norm_fwd_kernel(const NormFwdArgs p) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + wave;
  const int D = p.D;
  if (row >= p.T) return;
  const E* arow = (const E*)p.a + row * p.sa;
  const E* urow = p.u ? (const E*)p.u + row * p.su : nullptr;       // no gate: plain layer norm
  E* yrow = (E*)p.y + row * p.sy;
  float a[NCH][8];
  // Narrow bf16 rows: the gate's rows travel with the first loads, not after the reductions.  us, late -> early: 256 features,
  // 300 rows 2.44 -> 2.36, 87,000 rows 29.5 -> 27.4, 512 features 43.6 -> 40.9; more registers of them cost occupancy: 2,048
  // features, 10,000 rows 19.7 -> 21.4, fp32, 3,000 rows 12.1 -> 13.6.
  constexpr bool kEarly = NCH == 1 && sizeof(E) == 2;
  Raw8<E> ur;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int e0 = (lane + 64 * c) * 8;
    if (e0 < D) {
      load8(arow, e0, a[c]);
      if (kEarly && urow) ur = load8raw(urow, e0);
    }
  }
  float mu, rs;
  if (p.stats_in) { mu = p.mean[row]; rs = p.rstd[row]; }           // statistics saved by an earlier pass
  else row_stats<NCH>(a, lane, D, p.eps, mu, rs);
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int e0 = (lane + 64 * c) * 8;
    if (e0 < D) {
      float uv[8], gv[8], bv[8], out[8];
      if (!kEarly && urow) ur = load8raw(urow, e0);
      if (urow) widen8(ur, uv);
      load8(p.gamma, e0, gv);
      if (p.beta) load8(p.beta, e0, bv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        out[i] = (a[c][i] - mu) * rs * gv[i] + (p.beta ? bv[i] : 0.f);
        if (urow) out[i] *= uv[i];
      }
      store8(yrow, e0, out);
    }
  }
  if (lane == 0 && !p.stats_in) {
    if (p.mean) p.mean[row] = mu;
    if (p.rstd) p.rstd[row] = rs;
  }
}

// Forward with row-wise FP8 output (paper Section 4.2.2: the scaling and quantisation that the FP8 projections need are
// fused into the norm kernel that precedes them, Eq. 1 and Eq. 4, so that the normalised rows never make a round trip
// through memory in 16 bits).  Per row: y as in the kernel above (or, without gamma, the input rows themselves, times the
// gate if there is one: plain row-wise quantisation, used for the weights), amax = max |y|, scale = amax / 448,
// code = E4M3(y * (448 / amax)), ties to even.  All of it in fp32, one division per row and one multiplication per element.
template <typename E, int NCH>
__global__ __launch_bounds__(64 * kRowsPerBlock) void norm_quant_fwd_kernel(const NormFwdArgs p, unsigned char* __restrict__ q,
                                                                            int64_t sq, float* __restrict__ qscale) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + wave;
  const int D = p.D;
  if (row >= p.T) return;
  const E* arow = (const E*)p.a + row * p.sa;
  const E* urow = p.u ? (const E*)p.u + row * p.su : nullptr;
  float a[NCH][8];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int e0 = (lane + 64 * c) * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[c][i] = 0.f;
    if (e0 < D) load8(arow, e0, a[c]);
  }
  float mu = 0.f, rs = 1.f;
  if (p.gamma) row_stats<NCH>(a, lane, D, p.eps, mu, rs);
  float amax = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int e0 = (lane + 64 * c) * 8;
    if (e0 < D) {
      float uv[8], gv[8], bv[8];
      if (urow) load8(urow, e0, uv);
      if (p.gamma) load8(p.gamma, e0, gv);
      if (p.beta) load8(p.beta, e0, bv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float y = a[c][i];
        if (p.gamma) y = (y - mu) * rs * gv[i] + (p.beta ? bv[i] : 0.f);
        if (urow) y *= uv[i];
        a[c][i] = y;
        amax = fmaxf(amax, fabsf(y));
      }
    }
  }
  amax = wave_max(amax);
  const float safe = amax > 0.f ? amax : 448.0f;
  const float scale = safe / 448.0f;
  const float inv = 448.0f / safe;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int e0 = (lane + 64 * c) * 8;
    if (e0 < D) {
      int w0 = 0, w1 = 0;
      w0 = __builtin_amdgcn_cvt_pk_fp8_f32(a[c][0] * inv, a[c][1] * inv, w0, false);
      w0 = __builtin_amdgcn_cvt_pk_fp8_f32(a[c][2] * inv, a[c][3] * inv, w0, true);
      w1 = __builtin_amdgcn_cvt_pk_fp8_f32(a[c][4] * inv, a[c][5] * inv, w1, false);
      w1 = __builtin_amdgcn_cvt_pk_fp8_f32(a[c][6] * inv, a[c][7] * inv, w1, true);
      *(int2*)(q + row * sq + e0) = make_int2(w0, w1);
    }
  }
  if (lane == 0) {
    qscale[row] = scale;
    if (p.gamma && p.mean) p.mean[row] = mu;
    if (p.gamma && p.rstd) p.rstd[row] = rs;
  }
}

// Backward.  Per row: ahat = (a - mu) rstd, dn = dy u, dU = dy (ahat gamma + beta), dahat = dn gamma, dA = rstd (dahat -
// mean(dahat) - ahat mean(dahat ahat)).  Column sums dgamma = sum dn ahat and dbeta = sum dn (if wanted) are kept per lane over
// the rows a wave visits, combined across the workgroup's waves in a fixed order through LDS and written as one partial row per
// workgroup.  Few rows are a chain of latencies: the chunks of a row are fetched together, the reductions are DPP, and the waves'
// column sums meet in one step.  With the gradient's rows fetched behind the first reductions, lane permutations through LDS and
// the waves' sums added in turn, bf16, us with the column-sum launch, before -> now: 384 features, 6,418 rows 16.7 -> 12.5,
// 20,000 rows 25.2 -> 19.1, 87,728 rows 80.9 -> 69.2; 512 features 17.4 -> 12.6, 27.5 -> 21.2, 90.6 -> 89.9 (memory).
template <typename E> struct BwdRow { Raw8<E> a, dy, u; };          // what the reductions need
template <typename E> struct BwdTail { Raw8<E> pre, res; };         // and what the results need
template <typename E> constexpr bool kAhead = sizeof(E) == 2;      // a chunk of fp32 is 8 registers: fetched where it is used, nothing ahead

template <typename E>
__device__ __forceinline__ void fetch_row(const NormBwdArgs& p, int64_t row, int e0, BwdRow<E>& r) {
  r.a = load8raw((const E*)p.a + row * p.sa, e0);
  r.dy = load8raw((const E*)p.dy + row * p.sdy, e0);
  if (p.u) r.u = load8raw((const E*)p.u + row * p.su, e0);
}
template <typename E>
__device__ __forceinline__ void fetch_tail(const NormBwdArgs& p, int64_t row, int e0, BwdTail<E>& r) {
  if (p.du_pre) r.pre = load8raw((const E*)p.du_pre + row * p.sdu_pre, e0);
  if (p.residual) r.res = load8raw((const E*)p.residual + row * p.sres, e0);
}

// BETA: a bias, or its gradient, is there.
template <typename E, bool BETA>
__global__ __launch_bounds__(64 * kBwdWaves, 4) void gated_norm_bwd_kernel(const NormBwdArgs p, float* __restrict__ partial) {
  extern __shared__ __attribute__((aligned(16))) float red[];         // [waves][dgamma, with BETA dbeta][D]
  constexpr int kSums = BETA ? 2 : 1;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int D = p.D, e0 = lane * 8;
  const bool on = e0 < D;
  float gsum[8], bsum[8], gv[8], bv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) { gsum[i] = 0.f; bsum[i] = 0.f; gv[i] = 0.f; bv[i] = 0.f; }
  if (on) {
    load8(p.gamma, e0, gv);
    if (BETA && p.beta) load8(p.beta, e0, bv);
  }
  const int64_t stride = (int64_t)gridDim.x * kBwdWaves;
  for (int64_t row = (int64_t)blockIdx.x * kBwdWaves + wave; row < p.T; row += stride) {
    BwdRow<E> r;
    BwdTail<E> tail;
    if (on) {
      fetch_row(p, row, e0, r);
      if (kAhead<E>) fetch_tail(p, row, e0, tail);
    }
    float a[1][8], dah[8];
    if (on) widen8(r.a, a[0]);
    float mu, rs;
    row_stats<1>(a, lane, D, p.eps, mu, rs);
    float m1 = 0.f, m2 = 0.f;
    if (on) {
      float dyv[8], uv[8], duv[8], yv[8];
      widen8(r.dy, dyv);
      if (p.u) widen8(r.u, uv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float ah = (a[0][i] - mu) * rs;
        const float dn = p.u ? dyv[i] * uv[i] : dyv[i];
        const float nv = ah * gv[i] + bv[i];
        duv[i] = dyv[i] * nv;
        yv[i] = p.u ? nv * uv[i] : nv;
        gsum[i] += dn * ah;
        if (BETA) bsum[i] += dn;
        dah[i] = dn * gv[i];
        m1 += dah[i];
        m2 += dah[i] * ah;
        a[0][i] = ah;
      }
      if (p.u) {                                       // (no gate: plain layer norm, no dU)
        if (!kAhead<E> && p.du_pre) tail.pre = load8raw((const E*)p.du_pre + row * p.sdu_pre, e0);
        if (p.du_pre) dsilu8(tail.pre, duv);
        store8((E*)p.du + row * p.sdu, e0, duv);
        if (p.y_out) store8((E*)p.y_out + row * p.sy_out, e0, yv);
      }
    }
    m1 = wave_sum(m1) / (float)D;
    m2 = wave_sum(m2) / (float)D;
    if (on) {
      float dav[8], rv[8];
      if (!kAhead<E> && p.residual) tail.res = load8raw((const E*)p.residual + row * p.sres, e0);
      if (p.residual) widen8(tail.res, rv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        dav[i] = rs * (dah[i] - m1 - a[0][i] * m2);
        if (p.residual) dav[i] += rv[i];               // gradient that bypasses the norm (residual connection)
      }
      store8((E*)p.da + row * p.sda, e0, dav);
    }
  }
  // fixed-order combination of the waves' column sums
  if (on) {
    float* mine = red + wave * kSums * D + e0;
    *(f32x4*)mine = (f32x4){gsum[0], gsum[1], gsum[2], gsum[3]};
    *(f32x4*)(mine + 4) = (f32x4){gsum[4], gsum[5], gsum[6], gsum[7]};
    if (BETA) {
      *(f32x4*)(mine + D) = (f32x4){bsum[0], bsum[1], bsum[2], bsum[3]};
      *(f32x4*)(mine + D + 4) = (f32x4){bsum[4], bsum[5], bsum[6], bsum[7]};
    }
  }
  __syncthreads();
  float* prow = partial + (int64_t)blockIdx.x * 2 * D;
  for (int i = threadIdx.x * 4; i < kSums * D; i += blockDim.x * 4) {
    f32x4 t = *(const f32x4*)(red + i);
#pragma unroll
    for (int w = 1; w < kBwdWaves; ++w) t += *(const f32x4*)(red + w * kSums * D + i);
    *(f32x4*)(prow + i) = t;
  }
}

// Backward for rows wider than 512 features: a workgroup of W waves shares one row, every thread owns one 16-byte chunk of it
// (and the column sums of those 8 features over all the rows its workgroup visits, so the waves need no combination at the end).
// The row statistics cross the waves through LDS with two barriers per row: the sum of a first, then sum (a - mu)^2, sum dahat
// and sum dahat (a - mu) together (mean(dahat ahat) = rstd times the last one / D).  The slots alternate with the row parity, so
// a wave that runs ahead never overwrites what a slower one still reads.  One wave per row needed 48 registers per 512 features
// (and spilled from 2048 features on).  What the reductions of the next row need is fetched a row ahead (bf16), 128 registers
// keep 16 waves on a compute unit, and a wave sums eight and more slots a lane each (48 values in flight spilled at 16 waves).
// bf16 without a bias, us with the column-sum launch, before -> now: 1024 features, 6,418 rows 31.8 -> 20.7, 87,728 rows 217 ->
// 179; 2048 features, 6,418 rows 43.0 -> 29.7; 4096 features, 20,000 rows 227 -> 158; 8192 features 2,017 -> 324; fp32 at 8192
// features, 6,418 rows 285 -> 208.
//
// The sum of W (up to 16) values in LDS, in every lane: eight and more a value per lane of a row of 16 (48 values in flight spill
// at W = 16).
template <int W> __device__ __forceinline__ float sum_slots(const float* slots, int lane) {
  if constexpr (W <= 4) {
    float v = slots[0];
#pragma unroll
    for (int w = 1; w < W; ++w) v += slots[w];
    return v;
  } else {
    float v = slots[lane & (W - 1)];
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    if (W > 8) v += dpp<0x140>(v);
    return v;
  }
}

template <typename E, int W, bool BETA>
__global__ __launch_bounds__(64 * W, W < 16 && (BETA || !kAhead<E>) ? 3 : 4) void gated_norm_bwd_wide_kernel(const NormBwdArgs p, float* __restrict__ partial) {
  __shared__ float red1[2][W];
  __shared__ float red2[2][3][W];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int D = p.D, e0 = threadIdx.x * 8;
  const bool on = e0 < D;
  // Where registers are short, dahat is formed again instead of kept over the barrier, and at 16 waves of fp32 the bias read
  // again.  us, kept -> again: bf16, 1,024 features, 30,000 rows 65 -> 61, 8,192 features, 3,000 rows 59.8 -> 52.4; fp32, 8,192
  // features with a bias, 1 row 18.7 -> 15.7 (before the rows were fetched ahead 16.4), without, 3,000 rows 121 -> 106; but fp32,
  // 520 features, 30,000 rows 82 -> 89.
  constexpr bool kHoldDah = !kAhead<E> && W < 16, kHoldBias = BETA && (kAhead<E> || W < 16);
  float gv[8], bv[8], gsum[8], bsum[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) { gv[i] = 0.f; bv[i] = 0.f; gsum[i] = 0.f; bsum[i] = 0.f; }
  if (on) {
    load8(p.gamma, e0, gv);
    if (kHoldBias && p.beta) load8(p.beta, e0, bv);
  }
  const float inv_d = 1.0f / (float)D;
  int par = 0;
  BwdRow<E> r, next;                                   // the next row's chunks are fetched while this one's sums cross the waves
  if (kAhead<E> && on && blockIdx.x < p.T) fetch_row(p, blockIdx.x, e0, r);
  for (int64_t row = blockIdx.x; row < p.T; row += gridDim.x, par ^= 1) {
    BwdTail<E> tail;
    if (on && kAhead<E>) {
      fetch_tail(p, row, e0, tail);
      if (row + gridDim.x < p.T) fetch_row(p, row + gridDim.x, e0, next);
    } else if (on) {
      fetch_row(p, row, e0, r);
    }
    float a[8], dyv[8], dah[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { a[i] = 0.f; dyv[i] = 0.f; }
    if (on) {
      widen8(r.a, a);
      widen8(r.dy, dyv);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += a[i];
    s = wave_sum(s);
    if (lane == 0) red1[par][wave] = s;
    __syncthreads();
    const float mu = sum_slots<W>(red1[par], lane) * inv_d;
    float q = 0.f, s1 = 0.f, s2 = 0.f;
    if (on) {
      float uv[8];
      if (p.u) widen8(r.u, uv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float c = a[i] - mu;
        dah[i] = (p.u ? dyv[i] * uv[i] : dyv[i]) * gv[i];
        q += c * c;
        s1 += dah[i];
        s2 += dah[i] * c;
        a[i] = c;
      }
    }
    q = wave_sum(q); s1 = wave_sum(s1); s2 = wave_sum(s2);
    if (lane == 0) { red2[par][0][wave] = q; red2[par][1][wave] = s1; red2[par][2][wave] = s2; }
    __syncthreads();
    const float tq = sum_slots<W>(red2[par][0], lane), t1 = sum_slots<W>(red2[par][1], lane), t2 = sum_slots<W>(red2[par][2], lane);
    const float rs = 1.0f / sqrtf(tq * inv_d + p.eps);
    const float m1 = t1 * inv_d, m2 = rs * t2 * inv_d;
    if (on) {
      float duv[8], dav[8], yv[8], uv[8], rv[8];
      if (p.u) widen8(r.u, uv);
      if (!kAhead<E> && p.residual) tail.res = load8raw((const E*)p.residual + row * p.sres, e0);
      if (p.residual) widen8(tail.res, rv);
      if (BETA && !kHoldBias && p.beta) load8(p.beta, e0, bv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float ah = a[i] * rs;
        const float nv = ah * gv[i] + bv[i];
        const float dn = p.u ? dyv[i] * uv[i] : dyv[i];
        duv[i] = dyv[i] * nv;
        yv[i] = p.u ? nv * uv[i] : nv;
        gsum[i] += dn * ah;
        if (BETA) bsum[i] += dn;
        dav[i] = rs * ((kHoldDah ? dah[i] : dn * gv[i]) - m1 - ah * m2);
        if (p.residual) dav[i] += rv[i];               // gradient that bypasses the norm (residual connection)
      }
      if (p.u) {                                       // (no gate: plain layer norm, no dU)
        if (!kAhead<E> && p.du_pre) tail.pre = load8raw((const E*)p.du_pre + row * p.sdu_pre, e0);
        if (p.du_pre) dsilu8(tail.pre, duv);
        store8((E*)p.du + row * p.sdu, e0, duv);
        if (p.y_out) store8((E*)p.y_out + row * p.sy_out, e0, yv);
      }
      store8((E*)p.da + row * p.sda, e0, dav);
    }
    if (kAhead<E>) r = next;
  }
  if (on) {
    float* prow = partial + (int64_t)blockIdx.x * 2 * D;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      prow[e0 + i] = gsum[i];
      if (BETA) prow[D + e0 + i] = bsum[i];
    }
  }
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void gated_norm_colsum_kernel(const ColsumJob job) {
  __shared__ f32x4 red[kThreads / 64][4];
  column_sums<kThreads>(job, blockIdx.x, red);
}

// No more threads than there are rows to add need, and 256 where the columns alone fill the chip with workgroups.  The whole
// backward, us with 1,024 threads everywhere -> this way (64 columns x 16 row groups before): 100 rows x 512 features 10.95 ->
// 10.5 (10.4); 1 row x 4,096 with dbeta 10.8 -> 9.3 (9.2); 100 rows 13.1 -> 12.2 (12.0); 1,000 rows x 512 and more unchanged
// (11.4; 12.9 before), where 256 threads take 0.1-0.4 longer.
static hipError_t launch_colsum(int nblk, const NormBwdArgs& p, const float* partial, hipStream_t stream) {
  const ColsumJob job = {nblk, p.D, partial, p.dgamma, p.dbeta};
  const dim3 grid(job.blocks());
  if (nblk <= 16) hipLaunchKernelGGL(gated_norm_colsum_kernel<64>, grid, dim3(64), 0, stream, job);
  else if (nblk <= 64 || grid.x > 256) hipLaunchKernelGGL(gated_norm_colsum_kernel<256>, grid, dim3(256), 0, stream, job);
  else hipLaunchKernelGGL(gated_norm_colsum_kernel<1024>, grid, dim3(1024), 0, stream, job);
  return hipGetLastError();
}

// waves that share a row in the backward: 1 up to 512 features, else the power of two that gives every thread one chunk
static int bwd_row_waves(int D) {
  int w = 1;
  while (w * 512 < D) w <<= 1;
  return w;                                               // 1, 2, 4, 8, 16 (D <= 8192)
}

// workgroups of the backward = rows of partial column sums
int gated_norm_bwd_blocks(int64_t T, int D) {
  const int w = bwd_row_waves(D);
  if (w == 1) {
    const int64_t need = (T + kBwdWaves - 1) / kBwdWaves;
    return (int)(need < kMaxBwdBlocks ? need : kMaxBwdBlocks);
  }
  const int64_t cap = 256 * (16 / w);                     // 16 waves per compute unit
  return (int)(T < cap ? T : cap);
}

template <typename E, int NCH>
static hipError_t fwd_one(const NormFwdArgs& p, hipStream_t stream) {
  const unsigned grid = (unsigned)((p.T + kRowsPerBlock - 1) / kRowsPerBlock);
  hipLaunchKernelGGL((gated_norm_fwd_kernel<E, NCH>), dim3(grid), dim3(64 * kRowsPerBlock), 0, stream, p);
  return hipGetLastError();
}

template <typename E, int W>
static hipError_t bwd_wide(const NormBwdArgs& p, float* partial, hipStream_t stream, bool sums) {
  const int nblk = gated_norm_bwd_blocks(p.T, p.D);
  if (p.beta || p.dbeta) hipLaunchKernelGGL((gated_norm_bwd_wide_kernel<E, W, true>), dim3(nblk), dim3(64 * W), 0, stream, p, partial);
  else hipLaunchKernelGGL((gated_norm_bwd_wide_kernel<E, W, false>), dim3(nblk), dim3(64 * W), 0, stream, p, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !sums) return e;
  return launch_colsum(nblk, p, partial, stream);
}

template <typename E>
static hipError_t bwd_one(const NormBwdArgs& p, float* partial, hipStream_t stream, bool sums) {
  const int nblk = gated_norm_bwd_blocks(p.T, p.D);
  const size_t smem = (size_t)kBwdWaves * p.D * sizeof(float);                           // (32 KB at most)
  if (p.beta || p.dbeta) hipLaunchKernelGGL((gated_norm_bwd_kernel<E, true>), dim3(nblk), dim3(64 * kBwdWaves), 2 * smem, stream, p, partial);
  else hipLaunchKernelGGL((gated_norm_bwd_kernel<E, false>), dim3(nblk), dim3(64 * kBwdWaves), smem, stream, p, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !sums) return e;
  return launch_colsum(nblk, p, partial, stream);
}

template <typename E, int NCH>
static hipError_t quant_one(const NormFwdArgs& p, void* q, int64_t sq, float* qscale, hipStream_t stream) {
  const unsigned grid = (unsigned)((p.T + kRowsPerBlock - 1) / kRowsPerBlock);
  hipLaunchKernelGGL((norm_quant_fwd_kernel<E, NCH>), dim3(grid), dim3(64 * kRowsPerBlock), 0, stream, p, (unsigned char*)q, sq, qscale);
  return hipGetLastError();
}

static int chunks_per_lane(int D) {
  const int chunks = (D / 8 + 63) / 64;
  int nch = 1;
  while (nch < chunks) nch <<= 1;
  return nch;
}

hipError_t launch_norm_fwd(const NormFwdArgs& p, hipStream_t stream) {
  const int nch = chunks_per_lane(p.D);
#define FWD_CALL(E, N) fwd_one<E, N>(p, stream)
  if (p.dtype == 0) {
    switch (nch) {
      case 1: return FWD_CALL(__bf16, 1);
      case 2: return FWD_CALL(__bf16, 2);
      case 4: return FWD_CALL(__bf16, 4);
      case 8: return FWD_CALL(__bf16, 8);
      default: return FWD_CALL(__bf16, 16);
    }
  }
  switch (nch) {
    case 1: return FWD_CALL(float, 1);
    case 2: return FWD_CALL(float, 2);
    case 4: return FWD_CALL(float, 4);
    case 8: return FWD_CALL(float, 8);
    default: return FWD_CALL(float, 16);
  }
#undef FWD_CALL
}

hipError_t launch_norm_quant_fwd(const NormFwdArgs& p, void* q, int64_t sq, float* qscale, hipStream_t stream) {
  const int nch = chunks_per_lane(p.D);
#define Q_CALL(E, N) quant_one<E, N>(p, q, sq, qscale, stream)
  if (p.dtype == 0) {
    switch (nch) {
      case 1: return Q_CALL(__bf16, 1);
      case 2: return Q_CALL(__bf16, 2);
      case 4: return Q_CALL(__bf16, 4);
      case 8: return Q_CALL(__bf16, 8);
      default: return Q_CALL(__bf16, 16);
    }
  }
  switch (nch) {
    case 1: return Q_CALL(float, 1);
    case 2: return Q_CALL(float, 2);
    case 4: return Q_CALL(float, 4);
    case 8: return Q_CALL(float, 8);
    default: return Q_CALL(float, 16);
  }
#undef Q_CALL
}

hipError_t launch_norm_bwd(const NormBwdArgs& p, float* partial, hipStream_t stream, bool sums) {
  if (p.T <= 0 && !sums) return hipSuccess;
  if (p.T <= 0) return launch_colsum(0, p, partial, stream);   // no rows: the column sums are zero
  const int w = bwd_row_waves(p.D);
#define BWD_WIDE(E)                                        \
  switch (w) {                                             \
    case 1: return bwd_one<E>(p, partial, stream, sums);         \
    case 2: return bwd_wide<E, 2>(p, partial, stream, sums);     \
    case 4: return bwd_wide<E, 4>(p, partial, stream, sums);     \
    case 8: return bwd_wide<E, 8>(p, partial, stream, sums);     \
    default: return bwd_wide<E, 16>(p, partial, stream, sums);   \
  }
  if (p.dtype == 0) { BWD_WIDE(__bf16) }
  BWD_WIDE(float)
#undef BWD_WIDE
}

// contiguous [T, D] tensors, statistics computed: the form behind the C entry points
hipError_t launch_gated_norm_fwd(int64_t T, int D, int dtype, const void* attn, const void* u, const float* gamma,
                                 const float* beta, float eps, void* y, float* mean, float* rstd, hipStream_t stream) {
  NormFwdArgs p = {};
  p.T = T; p.D = D; p.dtype = dtype; p.a = attn; p.sa = D; p.u = u; p.su = D; p.gamma = gamma; p.beta = beta; p.eps = eps;
  p.y = y; p.sy = D; p.mean = mean; p.rstd = rstd; p.stats_in = 0;
  return launch_norm_fwd(p, stream);
}

hipError_t launch_gated_norm_bwd(int64_t T, int D, int dtype, const void* dy, const void* attn, const void* u,
                                 const float* gamma, const float* beta, float eps, void* dattn, void* du, float* dgamma,
                                 float* dbeta, float* partial, hipStream_t stream) {
  NormBwdArgs p = {};
  p.T = T; p.D = D; p.dtype = dtype; p.dy = dy; p.sdy = D; p.a = attn; p.sa = D; p.u = u; p.su = D; p.gamma = gamma;
  p.beta = beta; p.eps = eps; p.da = dattn; p.sda = D; p.du = du; p.sdu = D; p.residual = nullptr; p.sres = D;
  p.dgamma = dgamma; p.dbeta = dbeta;
  return launch_norm_bwd(p, partial, stream);
}

}  // namespace hstu
