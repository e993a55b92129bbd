// Attention truncation on a jagged batch (paper Section 4.3): the layers after the first group run on the
// most recent `keep` history tokens of every sequence (plus its candidates).  Three HBM-bound kernels: the
// offsets of the truncated batch, the row gather, and its backward (row scatter with zero fill).
#include "hstu_kernels.h"

namespace hstu {
namespace {

constexpr int kScanThreads = 1024;
constexpr int kCopyThreads = 256;            // 4 waves
constexpr int kRowsPerWave = 8;              // consecutive rows handled by one wave per step
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// out[b + 1] = sum over b' <= b of the kept rows of sequence b'; one workgroup walks the batch in chunks.
__global__ __launch_bounds__(kScanThreads) void truncate_offsets_kernel(int B, int keep, const int32_t* __restrict__ offsets,
                                                                        const int32_t* __restrict__ num_targets,
                                                                        int32_t* __restrict__ out) {
  __shared__ int32_t wave_sum[kScanThreads / 64];
  __shared__ int32_t carry_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) { carry_s = 0; out[0] = 0; }
  __syncthreads();
  for (int base = 0; base < B; base += kScanThreads) {
    const int b = base + tid;
    int kept = 0;
    if (b < B) {
      const int len = max(offsets[b + 1] - offsets[b], 0);
      const int m = num_targets ? min(max(num_targets[b], 0), len) : 0;
      kept = min(len - m, keep) + m;
    }
    int incl = kept;                         // inclusive scan inside the wave
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(incl, d, 64);
      if (lane >= d) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = carry_s;
    for (int w = 0; w < wave; ++w) before += wave_sum[w];
    if (b < B) out[b + 1] = before + incl;
    __syncthreads();
    if (tid == kScanThreads - 1) carry_s = before + incl;
    __syncthreads();
  }
}

// largest s with off[s] <= r (off non-decreasing, off[0] = 0 <= r < off[B]); lands on a non-empty sequence
__device__ __forceinline__ int find_sequence(const int32_t* __restrict__ off, int B, int r) {
  int lo = 0, hi = B;                        // off[lo] <= r < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= r) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ void copy_rows(const char* const src[kRowsPerWave], char* const dst[kRowsPerWave], int64_t row_bytes,
                                          int lane) {
  for (int64_t c = (int64_t)lane * 16; c < row_bytes; c += 64 * 16) {
    i32x4_t v[kRowsPerWave];
#pragma unroll
    for (int i = 0; i < kRowsPerWave; ++i)
      v[i] = src[i] ? __builtin_nontemporal_load((const i32x4_t*)(src[i] + c)) : i32x4_t{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kRowsPerWave; ++i)
      if (dst[i]) __builtin_nontemporal_store(v[i], (i32x4_t*)(dst[i] + c));
  }
}

// Wide rows, and middling numbers of narrow ones (in_steps), one per instruction of a wave.
// y row r of truncated sequence b is x row  offsets[b+1] - (out_offsets[b+1] - r).
__global__ __launch_bounds__(kCopyThreads) void truncate_gather_kernel(int B, const int32_t* __restrict__ offsets,
                                                                       const int32_t* __restrict__ out_offsets, int64_t row_bytes,
                                                                       const char* __restrict__ x, int64_t x_stride,
                                                                       char* __restrict__ y, int64_t y_stride, int64_t y_rows) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * (kCopyThreads / 64) + (threadIdx.x >> 6);
  const int64_t waves = (int64_t)gridDim.x * (kCopyThreads / 64);
  const int64_t rows = min((int64_t)out_offsets[B], y_rows);
  for (int64_t r0 = wave * kRowsPerWave; r0 < rows; r0 += waves * kRowsPerWave) {
    int b = find_sequence(out_offsets, B, (int)r0);
    const char* src[kRowsPerWave];
    char* dst[kRowsPerWave];
#pragma unroll
    for (int i = 0; i < kRowsPerWave; ++i) {
      const int64_t r = r0 + i;
      src[i] = nullptr; dst[i] = nullptr;
      if (r < rows) {
        while (b + 1 < B && r >= out_offsets[b + 1]) ++b;
        const int from = offsets[b + 1] - (out_offsets[b + 1] - (int)r);
        if (from >= offsets[b] && from < offsets[b + 1]) src[i] = x + (int64_t)from * x_stride;   // else: offsets that do not belong together
        dst[i] = y + r * y_stride;
      }
    }
    copy_rows(src, dst, row_bytes, lane);
  }
}

// dx row t of sequence b (position i, `drop` = rows of b that were cut) is dy row out_offsets[b] + i - drop, or zero for i < drop.
__global__ __launch_bounds__(kCopyThreads) void truncate_scatter_kernel(int B, int64_t T, const int32_t* __restrict__ offsets,
                                                                        const int32_t* __restrict__ out_offsets, int64_t row_bytes,
                                                                        const char* __restrict__ dy, int64_t dy_stride,
                                                                        char* __restrict__ dx, int64_t dx_stride) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * (kCopyThreads / 64) + (threadIdx.x >> 6);
  const int64_t waves = (int64_t)gridDim.x * (kCopyThreads / 64);
  const int64_t rows = min((int64_t)offsets[B], T);
  for (int64_t r0 = wave * kRowsPerWave; r0 < rows; r0 += waves * kRowsPerWave) {
    int b = find_sequence(offsets, B, (int)r0);
    const char* src[kRowsPerWave];
    char* dst[kRowsPerWave];
#pragma unroll
    for (int i = 0; i < kRowsPerWave; ++i) {
      const int64_t r = r0 + i;
      src[i] = nullptr; dst[i] = nullptr;
      if (r < rows) {
        while (b + 1 < B && r >= offsets[b + 1]) ++b;
        const int drop = (offsets[b + 1] - offsets[b]) - (out_offsets[b + 1] - out_offsets[b]);
        const int pos = (int)r - offsets[b];
        if (pos >= drop && drop >= 0) src[i] = dy + (int64_t)(out_offsets[b] + pos - drop) * dy_stride;
        dst[i] = dx + r * dx_stride;
      }
    }
    copy_rows(src, dst, row_bytes, lane);
  }
}

// The same, by a whole wave: 64 places at a time
__device__ __forceinline__ int find_with_wave(const int32_t* __restrict__ off, int B, int r, int lane) {
  int lo = 0, n = B;                         // it is one of the n from lo on
  while (n > 1) {
    const int step = (n + 63) >> 6, at = lane * step;
    const uint64_t le = __ballot(at < n && off[lo + min(at, n - 1)] <= r);
    const int k = max(63 - __clzll((long long)le), 0);
    lo += k * step;
    n = min(step, n - k * step);
  }
  return lo;
}

// Rows of up to 512 bytes.  A step of a wave copies kUnroll groups of rows, a group as many consecutive rows as 16 bytes a lane
// of one instruction cover.  The sequences around the step's first row sit in the lanes (a: the offsets that the rows are counted
// in, b: the others), so that finding a group's sequence takes comparisons and no further trip to memory.
constexpr int kUnroll = 8;
struct Window { int32_t a, b; int first; bool covers; };
struct Place { int32_t a0, a1, b0, b1; };    // a sequence in both offsets

__device__ __forceinline__ Window look(const int32_t* __restrict__ oa, const int32_t* __restrict__ ob, int B, int r0, int last, int lane) {
  Window w;
  w.first = find_with_wave(oa, B, r0, lane);
  w.a = oa[min(w.first + lane, B)];
  w.b = ob[min(w.first + lane, B)];
  w.covers = last < __builtin_amdgcn_readlane(w.a, 63) || w.first + 63 >= B;
  return w;
}
// The sequence of row r: the same for the group's rows [g0, g1] (all lanes), or the lane's own.
__device__ __forceinline__ Place place(const Window& w, const int32_t* __restrict__ oa, const int32_t* __restrict__ ob, int B, int g0, int g1, int r,
                                       int lane) {
  if (w.covers) {
    const bool some = w.first + lane < B;    // (sequences without rows share their start with the next one: the last that starts at or before r holds it)
    const int k0 = max(63 - __clzll((long long)__ballot(some && w.a <= g0)), 0), k1 = max(63 - __clzll((long long)__ballot(some && w.a <= g1)), 0);
    if (k0 == k1 && k0 < 63)
      return {__builtin_amdgcn_readlane(w.a, k0), __builtin_amdgcn_readlane(w.a, k0 + 1), __builtin_amdgcn_readlane(w.b, k0), __builtin_amdgcn_readlane(w.b, k0 + 1)};
    if (k1 < 63) {
      int k = k0;
      for (;;) {
        const int next = __shfl(w.a, k + 1, 64);
        const bool on = k < k1 && next <= r;
        if (__ballot(on) == 0) break;
        k += on;
      }
      return {__shfl(w.a, k, 64), __shfl(w.a, k + 1, 64), __shfl(w.b, k, 64), __shfl(w.b, k + 1, 64)};
    }
  }
  int lo = 0, hi = B;                        // off[lo] <= r < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (oa[mid] <= r) lo = mid; else hi = mid;
  }
  return {oa[lo], oa[lo + 1], ob[lo], ob[lo + 1]};
}

// GATHER as truncate_gather_kernel, rows counted in out_offsets; else as truncate_scatter_kernel, rows counted in offsets.
// What bounds it: memory, once every lane has 16 bytes to move.  us, forward / backward, with the kernels above -> here: 439,000
// rows of 256 bytes cut to 120,000 28.9 / 77.5 -> 13.9 / 31.7 (4.4 TB/s), of 128 bytes 23 / 72 -> 12 / 20, 779,000 rows of 400
// bytes 96 / 169 -> 62 / 96; rows of 1 KiB, which stay with the kernels above, 134 -> 147 backward.
template <bool GATHER>
__global__ __launch_bounds__(kCopyThreads) void truncate_copy_kernel(int B, const int32_t* __restrict__ offsets, const int32_t* __restrict__ out_offsets,
                                                                     int lanes_per_row, const char* __restrict__ src,
                                                                     int64_t src_stride, char* __restrict__ dst, int64_t dst_stride, int64_t dst_rows) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * (kCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t waves = (int64_t)gridDim.x * (kCopyThreads / 64);
  const int32_t* const oa = GATHER ? out_offsets : offsets;
  const int32_t* const ob = GATHER ? offsets : out_offsets;
  const int64_t rows = min((int64_t)oa[B], dst_rows);
  const int per = 64 / lanes_per_row, sub = lane / lanes_per_row, c = (lane - sub * lanes_per_row) * 16;   // rows of a group, this lane's, its bytes
  for (int64_t r0 = wave * (kUnroll * per); r0 < rows; r0 += waves * (kUnroll * per)) {
    const Window w = look(oa, ob, B, (int)r0, (int)min(r0 + kUnroll * per, rows) - 1, lane);
    const char* from[kUnroll];
    char* to[kUnroll];
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      from[i] = nullptr; to[i] = nullptr;
      const int64_t g0 = r0 + i * per, g1 = min(g0 + per, rows) - 1, r = g0 + sub;
      if (g0 >= rows) continue;
      const Place p = place(w, oa, ob, B, (int)g0, (int)g1, (int)min(r, g1), lane);
      if (sub >= per || r > g1) continue;
      if (GATHER) {
        const int row = p.b1 - (p.a1 - (int)r);
        if (row >= p.b0 && row < p.b1) from[i] = src + (int64_t)row * src_stride;        // else: offsets that do not belong together
      } else {
        const int drop = (p.a1 - p.a0) - (p.b1 - p.b0), pos = (int)r - p.a0;
        if (pos >= drop && drop >= 0) from[i] = src + (int64_t)(p.b0 + pos - drop) * src_stride;
      }
      to[i] = dst + r * dst_stride;
    }
    i32x4_t v[kUnroll];
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) v[i] = from[i] ? __builtin_nontemporal_load((const i32x4_t*)(from[i] + c)) : i32x4_t{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kUnroll; ++i)
      if (to[i]) __builtin_nontemporal_store(v[i], (i32x4_t*)(to[i] + c));
  }
}

int copy_grid(int64_t rows, int rows_per_step) {
  const int64_t steps = (rows + rows_per_step - 1) / rows_per_step;
  const int64_t wgs = (steps + kCopyThreads / 64 - 1) / (kCopyThreads / 64);
  return (int)max((int64_t)1, min(wgs, (int64_t)256 * 32));
}

// Rows of up to 512 bytes, at least two to an instruction, where a step's chain of trips to memory is all there is to wait for
// (one step), or the steps fill the chip.  In between a row an instruction spreads over more waves; and with few rows a sequence,
// which a step walks through, it takes more rows to pay.  us, row an instruction -> steps: 64 sequences, 27,000 rows of 48 bytes
// 7.9 -> 5.8, 20,000 sequences, 200,000 rows 45 -> 10, one sequence, 51 rows of 16 bytes 4.7 -> 2.5;  but one sequence, 2,400
// rows of 128 bytes 5.1 -> 5.9, 512 sequences, 400 rows of 16 bytes 7.1 -> 10.4, 1,300 rows 6.9 -> 11.5, 5,000 sequences, 7,500
// rows 8.0 -> 15.7.
constexpr int64_t kNarrowRow = 512;
bool in_steps(int B, int64_t rows, int64_t row_bytes) {
  if (row_bytes > kNarrowRow) return false;
  return (rows <= kUnroll * (64 / (row_bytes / 16)) || rows >= 8192) && (rows >= 8 * (int64_t)B || rows >= 65536);
}

template <bool GATHER>
hipError_t launch_copy(int B, int64_t rows, const int32_t* offsets, const int32_t* out_offsets, int64_t row_bytes, const void* src, int64_t src_stride,
                       void* dst, int64_t dst_stride, hipStream_t stream) {
  const int lanes = (int)(row_bytes / 16), grid = copy_grid(rows, kUnroll * (64 / lanes));
  hipLaunchKernelGGL(truncate_copy_kernel<GATHER>, dim3(grid), dim3(kCopyThreads), 0, stream, B, offsets, out_offsets, lanes, (const char*)src, src_stride,
                     (char*)dst, dst_stride, rows);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_truncate_offsets(int B, int keep, const int32_t* offsets, const int32_t* num_targets, int32_t* out,
                                   hipStream_t stream) {
  hipLaunchKernelGGL(truncate_offsets_kernel, dim3(1), dim3(kScanThreads), 0, stream, B, keep, offsets, num_targets, out);
  return hipGetLastError();
}

hipError_t launch_truncate_gather(int B, const int32_t* offsets, const int32_t* out_offsets, int64_t row_bytes, const void* x,
                                  int64_t x_stride, void* y, int64_t y_stride, int64_t y_rows, hipStream_t stream) {
  if (!in_steps(B, y_rows, row_bytes)) {
    hipLaunchKernelGGL(truncate_gather_kernel, dim3(copy_grid(y_rows, kRowsPerWave)), dim3(kCopyThreads), 0, stream, B, offsets, out_offsets,
                       row_bytes, (const char*)x, x_stride, (char*)y, y_stride, y_rows);
    return hipGetLastError();
  }
  return launch_copy<true>(B, y_rows, offsets, out_offsets, row_bytes, x, x_stride, y, y_stride, stream);
}

hipError_t launch_truncate_scatter(int B, int64_t T, const int32_t* offsets, const int32_t* out_offsets, int64_t row_bytes,
                                   const void* dy, int64_t dy_stride, void* dx, int64_t dx_stride, hipStream_t stream) {
  if (!in_steps(B, T, row_bytes)) {
    hipLaunchKernelGGL(truncate_scatter_kernel, dim3(copy_grid(T, kRowsPerWave)), dim3(kCopyThreads), 0, stream, B, T, offsets, out_offsets,
                       row_bytes, (const char*)dy, dy_stride, (char*)dx, dx_stride);
    return hipGetLastError();
  }
  return launch_copy<false>(B, T, offsets, out_offsets, row_bytes, dy, dy_stride, dx, dx_stride, stream);
}

}  // namespace hstu
