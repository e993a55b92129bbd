// Sums of dS per distance for the gradient of the relative-bias table, kept in registers by a wave of a backward pass.
#pragma once
#include <type_traits>
#include <utility>

#include "hstu_common.h"
#include "hstu_kernels.h"

namespace hstu {

// Diagonal sums of a 32 x 32 block of dS, shared out over the wave.  Lane l32 of half-wave hf holds, in register R, the streamed row
// 8 (R / 4) + 4 hf + R % 4 of the block; the sum over the pairs with (streamed row - lane row) = o lands at lane -o mod 64: part 0 of it,
// plus part 1 of the lane 4 further (the upper half-wave's rows are 4 further).  The rotations shift zeros in, so that a value and what
// comes around the end of a 16-lane row go to their sums without a select: two adds per register.
template <int CTRL>
__device__ __forceinline__ float dpp0(float v) {                         // the value DPP control CTRL brings, 0 where it brings none
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int R>
__device__ __forceinline__ void key_diag_step(float v, float& x0, float& x1, float& x2) {
  constexpr int q = R >> 2, rho = 8 * (q & 1) + (R & 3);
  float& lo = (q >> 1) == 0 ? x0 : x1;
  float& hi = (q >> 1) == 0 ? x1 : x2;
  if constexpr (rho == 0) {
    lo += v;
  } else {
    lo += dpp0<0x100 + rho>(v);                                          // row_shl: lane b of a row reads lane b + rho
    hi += dpp0<0x110 + 16 - rho>(v);                                     // row_shr: ... lane b + rho - 16
  }
}
// Sums of 16 registers over the 16 lanes of a row, handed out: lane i of a row leaves with the sum of register i.
template <int CTRL, int HALF>
__device__ __forceinline__ void row_fold(float (&v)[16], bool upper) {
#pragma unroll
  for (int r = 0; r < HALF; ++r) {
    const float keep = upper ? v[r + HALF] : v[r], give = upper ? v[r] : v[r + HALF];
    v[r] = keep + dpp0<CTRL>(give);
  }
}
__device__ __forceinline__ float row_sums(float (&v)[16], int i16) {
  row_fold<0x140, 8>(v, i16 & 8);                                        // row_mirror: lane ^ 15
  row_fold<0x141, 4>(v, i16 & 4);                                        // row_half_mirror: lane ^ 7
  row_fold<0x1B, 2>(v, i16 & 2);                                         // quad_perm: lane ^ 3
  row_fold<0xB1, 1>(v, i16 & 1);                                         // quad_perm: lane ^ 1
  return v[0];
}
template <int... R, typename V>
__device__ __forceinline__ void key_diag_all(std::integer_sequence<int, R...>, const V& vals, float& part0, float& part1) {
  float x0 = 0.f, x1 = 0.f, x2 = 0.f;
  (key_diag_step<R>(vals[R], x0, x1, x2), ...);
  // row g of a half-wave is 16 keys further: its class j meets class j - g of row 0
  const uint32_t m = __builtin_bit_cast(uint32_t, x1);
  x0 += __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_permlane16_swap(m, 0u, false, false)[1]);
  x2 += __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_permlane16_swap(0u, m, false, false)[0]);
  const auto parts = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x0), __builtin_bit_cast(uint32_t, x2), false, false);
  part0 = __builtin_bit_cast(float, (uint32_t)parts[0]);                 // queries of the lower half-wave ...
  part1 = __builtin_bit_cast(float, (uint32_t)parts[1]);                 // ... and of the upper one
}

// A 32 x 32 block of this wave, w0 = the distance of its first pair, holds the 63 distances around w0.
// Far from the diagonal they lie in one bucket of the table (the buckets of a log-spaced one are hundreds of distances wide there) and
// which distance of a bucket receives a sum does not matter: the block adds the plain sum of its dS, kept per lane until the
// bucket is left.  Any other block adds along its diagonals: lane l of `win` collects distance win_w0 + SGN * (l, or l - 64 for the upper
// half); the next block is 32 further, so the lower half of the window is complete then and leaves for the table of sums per
// distance, and the upper half becomes the lower one.  All of it stays in registers: strips in LDS with one read-add-write per class and
// half-wave, and a flush per tile by the workgroup, cost the dQ pass as much again as its products (64 features, 1024 + 256 semi-local,
// 8k-16k tokens: 0.31 ms without the gradient, 0.66 with it, 0.43 this way; 0.53 with one copy of the table for all dies).
// SGN: distance = SGN * (lane row - streamed row).  NLATE > 0: sums that leave do so at late_out(), for kernels that wait for a tile's
// loads at its end (that wait would wait for them).
constexpr int kNoWindow = -(1 << 30);
template <int SGN, int NLATE>
struct DistSums {
  static constexpr int kLate = NLATE > 0 ? NLATE : 1;
  float win, run_sum, late[kLate];
  int win_w0, run_end, run_w0, late_w0[kLate];
  float* dist_h;
  const int32_t* bucket_end;
  uint32_t stride;

  __device__ __forceinline__ void init(const AttnArgs& a, int xcd, int h) {
    win = run_sum = 0.f;
    win_w0 = kNoWindow;
    run_end = run_w0 = 0;
#pragma unroll
    for (int u = 0; u < kLate; ++u) { late[u] = 0.f; late_w0[u] = kNoWindow; }
    dist_h = a.dbias_dist + (int64_t)(xcd % a.dbias_copies * a.H + h) * a.dbias_pitch + a.dbias_lead;
    bucket_end = a.bucket_end;
    stride = (uint32_t)a.bias_stride;
  }
  // (the lane's number is made where it is needed: as a value that lives through the tile loop it would be spilled, and its reload wait for the tile's loads)
  static __device__ __forceinline__ int lane_id() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
  }
  __device__ __forceinline__ void win_out(int w0, float v) {
    const uint32_t off = (uint32_t)(32 + SGN * ((int)((uint32_t)lane_id() << 26) >> 26));
    if (v != 0.f && (uint32_t)(w0 - 32) + off < stride) atomicAdd(dist_h + (w0 - 32) + off, v);
  }
  __device__ __forceinline__ void win_flush() {
    if (win_w0 != kNoWindow) win_out(win_w0, win);
    win = 0.f;
    win_w0 = kNoWindow;
  }
  __device__ __forceinline__ void run_flush() {
    if (run_end != 0) {
      float v = run_sum;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      if (lane_id() == 0 && v != 0.f) atomicAdd(dist_h + run_w0, v);
    }
    run_sum = 0.f;
    run_end = 0;
  }
  __device__ __forceinline__ void late_out() {
#pragma unroll
    for (int u = 0; u < NLATE; ++u) {
      if (late_w0[u] != kNoWindow) win_out(late_w0[u], late[u]);
      late_w0[u] = kNoWindow;
    }
  }
  __device__ __forceinline__ void flush() { late_out(); win_flush(); run_flush(); }
  // the end of the bucket that holds all distances of a block without negative ones, 0: they lie in several
  __device__ __forceinline__ int one_bucket(int w0) const {
    const int end = ((const __attribute__((address_space(4))) int32_t*)(uintptr_t)bucket_end)[w0 - 31];
    return end > w0 + 31 ? end : 0;
  }
  // adds the 16 dS of this lane in sub-block `sub` of the tile; end: of one_bucket()
  template <typename V>
  __device__ __forceinline__ void add(const V& vals, int sub, int w0, int end) {
    if (end != 0) {
      if (end != run_end) {                                // (distances are walked in order: a bucket that is left rarely comes back)
        run_flush();
        run_end = end;
        run_w0 = w0 - 31;
      }
      float t0 = vals[0], t1 = vals[1];
#pragma unroll
      for (int r = 2; r < 16; r += 2) { t0 += vals[r]; t1 += vals[r + 1]; }
      run_sum += t0 + t1;
      return;
    }
    if (w0 == win_w0 - 32 * SGN) {
      const auto halves = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, win), 0u, false, false);
      const float done = __builtin_bit_cast(float, (uint32_t)halves[0]);
      if constexpr (NLATE > 0) { late[sub] = done; late_w0[sub] = win_w0; } else win_out(win_w0, done);
      win = __builtin_bit_cast(float, (uint32_t)halves[1]);
    } else {
      win_flush();
    }
    win_w0 = w0;
    float part0, part1;
    key_diag_all(std::make_integer_sequence<int, 16>{}, vals, part0, part1);
    win += part0;
    win += __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * lane_id() + 16, __builtin_bit_cast(int, part1)));      // (of lane l + 4 mod 64)
  }
};

}  // namespace hstu
