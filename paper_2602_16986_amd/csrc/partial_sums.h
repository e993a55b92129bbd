// Sums of partial results in a fixed order: the column sums that the norms' backward leaves per workgroup, and the slabs of a
// weight gradient.
#pragma once
#include "hstu_common.h"
#include "hstu_kernels.h"

namespace hstu {

// A value from another lane of the same row of 16, by DPP (a lane permutation through LDS, which __shfl_xor is, takes some 100
// cycles where this takes 8).
template <int kCtrl> __device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xF, 0xF, true));
}

// the sum over the lanes of a wave that are equal mod 4: two rotations inside a row of 16 lanes, then the rows in pairs
__device__ __forceinline__ float sum_every_4th_lane(float v) {
  v += dpp<0x124>(v);                                      // row_ror:4
  v += dpp<0x128>(v);                                      // row_ror:8
  const uint32_t a = __builtin_bit_cast(uint32_t, v);
  const auto p = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, (uint32_t)p[0]) + __builtin_bit_cast(float, (uint32_t)p[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return __builtin_bit_cast(float, (uint32_t)q[0]) + __builtin_bit_cast(float, (uint32_t)q[1]);
}

// dgamma[c] = sum over workgroups of partial[blk][0][c]; dbeta likewise from partial[blk][1][c] (not read unless wanted).
// A few MB at most, so what counts is how many loads are in flight: a workgroup owns 16 columns (a 64-byte segment of every
// partial row) and walks the rows kThreads / 4 at a time; a column's sums meet in a fixed tree (lanes, then waves).  With 64 columns
// and 16 row groups per workgroup every thread walked 32 (512 features) or 128 (1024) rows one after the other:
// 512 features 11.2 us, now 4.8; 1024 features 45.3 us, now 8.1.
template <int kThreads>
__device__ __forceinline__ void column_sums(const ColsumJob& job, int block, f32x4 (&red)[kThreads / 64][4]) {
  const int nblk = job.nblk, D = job.D;
  const float* __restrict__ partial = job.partial;
  float* const dgamma = job.dgamma; float* const dbeta = job.dbeta;
  const int tid = threadIdx.x, c4 = tid & 3, lane = tid & 63, wave = tid >> 6;
  const int c = block * 16 + 4 * c4;                  // D is a multiple of 8: 4 columns are all in or all out
  const int cols = dbeta ? 2 * D : D;                 // (of every partial row; the others may never have been written)
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (c < cols) {
#pragma unroll 4
    for (int b = tid >> 2; b < nblk; b += kThreads / 4) s += *(const f32x4*)(partial + (int64_t)b * 2 * D + c);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = sum_every_4th_lane(s[i]);
  if (lane < 4) red[wave][c4] = s;
  __syncthreads();
  if (tid < 4 && c < cols) {
    f32x4 t = red[0][c4];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) t += red[w][c4];
    float* const dst = c < D ? dgamma + c : dbeta + (c - D);
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[i] = t[i];
  }
}

constexpr int kSlabsAhead = 8;             // loads that a thread has in flight
// C = sum over slabs of partial, in slab order; 4 elements a thread
__device__ __forceinline__ void slab_sums(const SlabJob& job, int64_t i) {
  if (i >= job.elems4) return;
  const f32x4* __restrict__ partial = (const f32x4*)job.partial;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  int k = 0;
  for (; k + kSlabsAhead <= job.nslab; k += kSlabsAhead) {
    f32x4 p[kSlabsAhead];
#pragma unroll
    for (int e = 0; e < kSlabsAhead; ++e) p[e] = partial[(int64_t)(k + e) * job.elems4 + i];
#pragma unroll
    for (int e = 0; e < kSlabsAhead; ++e) s += p[e];
  }
  for (; k < job.nslab; ++k) s += partial[(int64_t)k * job.elems4 + i];
  ((f32x4*)job.C)[i] = s;
}

}  // namespace hstu
