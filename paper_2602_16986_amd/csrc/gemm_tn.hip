// Weight gradients of the layer's two projections (layer pseudocode of the paper's appendix: d_linear_w = X^T dY):
//   C[n1, n2] = sum over token rows t of A[t, n1] * B[t, n2],   A [T, N1], B [T, N2] bf16 row-major, C fp32.
// The reduction runs over the jagged token axis (10^5 rows) and the output is small (512 x 512 .. 2048 x 512), so the work is cut
// along t: gemm_rows.hip multiplies 128 x 128 output tiles of slabs of token rows (both fragments through the LDS transpose
// loads), and launch_layer_sums adds the fp32 sums of the slabs in a fixed order (deterministic, no atomics).  One slab writes C
// itself.
#include <algorithm>

#include "hstu_common.h"
#include "hstu_kernels.h"
#include "partial_sums.h"

namespace hstu {
namespace {
constexpr int kTile = 128;                 // output tile edge
constexpr int kBK = 64;                    // token rows of a k-tile
}  // namespace

bool gemm_tn_supported(int N1, int N2) { return N1 >= kTile && N2 >= kTile && N1 % kTile == 0 && N2 % kTile == 0; }

namespace {
constexpr double kTileUs = 0.72, kSumsUs = 3.5;                    // 64 token rows of a tile; the launch that adds slabs up
double slab_us(int N1, int N2) { return (double)N1 * N2 * 8 / 5e6; }
int tiles_of(int N1, int N2) { return (N1 / kTile) * (N2 / kTile); }

// No more slabs than k-tiles, nor than give every compute unit two workgroups; and slabs that take longer to write and read than
// the whole product never pay.  None of the three falls as T grows: the room for the partial sums is sized by this, so that a
// workspace for T rows serves fewer rows too.
int64_t most_slabs(int64_t T, int N1, int N2) {
  const int tiles = tiles_of(N1, N2);
  const int64_t k_tiles = (T + kBK - 1) / kBK;
  const double whole = kTileUs * (double)((tiles + 255) / 256 * k_tiles);
  const int64_t pay = (int64_t)std::max(1.0, (whole - kSumsUs) / slab_us(N1, N2));
  return std::min(std::min(k_tiles, pay), (int64_t)std::max(1, 512 / tiles));
}
}  // namespace

// The number of slabs with the least time: a compute unit works through its tiles at 0.72 us per 64 token rows, and slabs cost a
// launch that adds them up and a copy of the output each to write and read.  us of both launches, with a kernel of its own (64 x
// 64 per wave, tiles staged through registers, 512 workgroups) -> here:
//   T          2048 x 512          512 x 512
//   87,728     298  -> 260         73   -> 62
//   20,000      70  ->  58
//    6,418      32  ->  29         20   -> 16
//    1,000      18  ->  14         11   -> 11
int gemm_tn_slabs(int64_t T, int N1, int N2) {
  const int tiles = tiles_of(N1, N2);
  const int64_t most = most_slabs(T, N1, N2);
  int64_t best = 1;
  double least = 0;
  for (int64_t n = 1; n <= most; ++n) {
    const int64_t rows = ((T + n - 1) / n + kBK - 1) / kBK;
    double us = kTileUs * (double)((tiles * n + 255) / 256 * rows);
    if (n > 1) us += kSumsUs + (double)n * slab_us(N1, N2);
    if (n == 1 || us < least) { least = us; best = n; }
  }
  return (int)best;
}

namespace {
int64_t slab_rows(int64_t T, int nslab) { return ((T + nslab - 1) / nslab + kBK - 1) / kBK * kBK; }
}  // namespace

size_t gemm_tn_workspace_bytes(int64_t T, int N1, int N2) {
  const int64_t most = most_slabs(T, N1, N2);
  return most <= 1 ? 0 : (size_t)most * (size_t)N1 * (size_t)N2 * sizeof(float);
}

hipError_t launch_gemm_tn(int64_t T, int N1, int N2, const void* A, int64_t lda, const void* B, int64_t ldb, float* C, float* partial,
                          SlabJob& sums, hipStream_t stream) {
  GemmRowsArgs g = {};
  g.M = N1; g.N = N2; g.K = T; g.A = A; g.lda = lda; g.W = B; g.ldw = ldb; g.ldd = N2;
  g.slab = slab_rows(T, gemm_tn_slabs(T, N1, N2));
  const int nslab = (int)((T + g.slab - 1) / g.slab);              // (of which rounding may leave fewer than planned, none of them empty)
  g.D = nslab == 1 ? C : partial;
  sums = {(int64_t)N1 * N2 / 4, nslab == 1 ? 0 : nslab, partial, C};
  return launch_gemm_rows(g, kGemmTN, kEpiSums, stream);
}

namespace {
constexpr int kSumThreads = 256;
struct SumJobs { SlabJob slabs[2]; ColsumJob cols[2]; int end[4]; };      // end: workgroups up to and with the job
__global__ __launch_bounds__(kSumThreads) void layer_sums_kernel(const SumJobs j) {
  __shared__ f32x4 red[kSumThreads / 64][4];
  const int b = blockIdx.x;
  if (b < j.end[0]) slab_sums(j.slabs[0], (int64_t)b * kSumThreads + threadIdx.x);
  else if (b < j.end[1]) slab_sums(j.slabs[1], (int64_t)(b - j.end[0]) * kSumThreads + threadIdx.x);
  else if (b < j.end[2]) column_sums<kSumThreads>(j.cols[0], b - j.end[1], red);
  else column_sums<kSumThreads>(j.cols[1], b - j.end[2], red);
}
}  // namespace

// The partial sums of a layer's backward in one launch instead of four of 4-7 us: a training step of 6,418 rows 330 -> 324 us, of
// 14,000 rows (widths 256, 128) 248 -> 235.
hipError_t launch_layer_sums(const SlabJob (&slabs)[2], const ColsumJob (&cols)[2], hipStream_t stream) {
  SumJobs j = {{slabs[0], slabs[1]}, {cols[0], cols[1]}, {}};
  int end = 0;
  for (int i = 0; i < 2; ++i) j.end[i] = end += slabs[i].nslab > 0 ? (int)((slabs[i].elems4 + kSumThreads - 1) / kSumThreads) : 0;
  for (int i = 0; i < 2; ++i) j.end[2 + i] = end += cols[i].blocks();
  hipLaunchKernelGGL(layer_sums_kernel, dim3(end), dim3(kSumThreads), 0, stream, j);
  return hipGetLastError();
}

}  // namespace hstu
