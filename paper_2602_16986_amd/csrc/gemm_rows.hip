// Products over token rows (the layer's two projections, the gradients of their inputs and of their weights; paper Eq. 2 and f2 of
// Eq. 5), bf16 operands, fp32 accumulation, one rounding:
//   D[m, n] = epilogue( sum_k A[m, k] W[n, k] )     W [N, K] row-major (kGemmNT) or [K, N] row-major (kGemmNN)
//   D[m, n] = sum_k A[k, m] W[k, n]                 kGemmTN: k are the token rows, cut into slabs whose fp32 sums leave one by one (gemm_tn.hip)
// with the layer's pointwise work in the epilogue: SiLU with the gate's columns sent to a tensor of their own, the pre-activations
// beside their SiLU, or the residual rows added.
//
// A workgroup owns tiles of WM 32 MI token rows x WN 64 columns, one of its WM WN multiplying waves 32 MI x 64 of it; the token
// rows sit on the accumulators' lane axis, the columns on the register axis.  Both operands arrive in LDS by direct-to-LDS loads,
// 64 k at a time, one barrier per k-tile.
// What bounds it, and what follows (87,728 rows, 2048 columns, K = 512, SiLU; the library's two products with it in their
// epilogue: 294 us):
// 1.  The L2's request rate.  Every load covers whole 128-byte lines: with 32 k at a time, 64-byte halves of lines whose other
//    halves have left the first-level cache when they are wanted, 303 us.
// 2.  The stores of the output, which a burst of every compute unit at the end of its tile leaves to the memory (without them
//    185 us).  Memory operations of a wave complete in order, so a wave that stores cannot wait for a later load without waiting
//    for the stores: four further waves only load, across tiles (the workgroups are persistent), and run on while the others
//    store.  288 us without them.  Stores are non-temporal (282 without) and leave in whole lines: the accumulators go through
//    LDS as fp32, 16 rows x 64 columns at a time and wave by wave (no barrier).  252 us with both.
// 3. Power, then: products and LDS reads alone run at 1.1-1.2 PFLOP/s.
// A wave's last products of a k-tile follow the barrier that publishes the next one, whose first operands are read in between:
// 250 us, and 346 instead of 362 for 40,000 x 1024 x K = 4096.
// Rows of 128 bytes (operands with k contiguous) keep 16-byte chunk c of row r at c ^ (r / 2) % 8; rows of W [K, N], read through
// the LDS transpose loads, at c ^ (4 (r % 4) + (r / 4) % 4): every read is free of bank conflicts, and the swizzle costs nothing
// because it is applied to the loads' source addresses.
#include <algorithm>
#include <type_traits>

#include "gemm_tiles.h"
#include "hstu_common.h"
#include "hstu_kernels.h"

namespace hstu {
namespace {

typedef __attribute__((address_space(3))) void* lds_void;
typedef __attribute__((address_space(3))) short4v* lds_s4;
typedef __attribute__((address_space(3))) const bf16x8* lds_b8;
typedef __attribute__((address_space(3))) f32x4* lds_f4;
typedef __attribute__((address_space(3))) const i32x4* lds_i4;
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kBK = 64;                                  // of a k-tile: 128 bytes
constexpr uint32_t kOutside = 0x80000000u;               // a lane offset beyond every range: the load returns zeros

// WM x WN waves multiply, kLoaders more only load.
constexpr int kLoaders = 4;
template <int WM, int WN, int MI, int STAGES>
struct Tile {
  static constexpr int kWaves = WM * WN, kThreads = 64 * (kWaves + kLoaders);
  static constexpr int kRows = 32 * MI * WM, kCols = 64 * WN;
  static constexpr int kA = kRows * kBK * 2, kW = kCols * kBK * 2, kStage = kA + kW;
  static constexpr int kLoadsA = kRows / 8 / kLoaders, kLoadsW = kCols / 8 / kLoaders, kLoads = kLoadsA + kLoadsW;   // wave-level loads (1 KB) of a loader per stage
  static constexpr int kArea = 32 * 32 * 4;                                                                          // a wave's part of the epilogue's staging
  static constexpr int kSmem = STAGES * kStage + kWaves * kArea;
  static constexpr int kWgPerCu = (160 << 10) / kSmem < 2 ? 1 : 2;
  static constexpr int kWavesPerSimd = (kWaves + kLoaders) / 4 * kWgPerCu;
  static_assert(kRows % (8 * kLoaders) == 0 && kCols % (8 * kLoaders) == 0, "every loader loads the same number of rows");
};

__device__ __forceinline__ float silu(float t) { return t * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * t)); }

__device__ __forceinline__ void store8(__bf16* at, const float (&v)[8]) {
  const u32x4 o = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
  __builtin_nontemporal_store(o, (u32x4*)at);
}

template <int WM, int WN, int MI, int STAGES, int OP, int EPI>
__global__ __launch_bounds__((Tile<WM, WN, MI, STAGES>::kThreads), (Tile<WM, WN, MI, STAGES>::kWavesPerSimd)) void gemm_rows_kernel(const GemmRowsArgs p, int tiles) {
  using S = Tile<WM, WN, MI, STAGES>;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5, l32 = lane & 31, i16 = lane & 15, grp16 = lane >> 4;
  constexpr bool kAT = OP == kGemmTN, kWT = OP == kGemmTN || OP == kGemmNN, kFp8 = OP == kGemmFp8;   // operands with k as their slow axis; E4M3 codes
  constexpr int kElem = kFp8 ? 1 : 2, kTileK = 128 / kElem;
  // Workgroups go to the 8 dies round-robin; a die takes a contiguous range of tiles, columns first: the tiles of one range of
  // token rows run beside each other and the rows come from memory once.
  const int tiles_n = (p.N + S::kCols - 1) / S::kCols;
  const int tiles_slab = kAT ? (int)((p.M + S::kRows - 1) / S::kRows) * tiles_n : 1;               // (kGemmTN: of a slab of the reduction)
  // k of a tile: all, or the tile's slab
  auto k_first = [&](int t) -> int64_t { return kAT ? (int64_t)(t / tiles_slab) * p.slab : 0; };
  auto k_count = [&](int t) -> int64_t { return kAT ? min(p.slab, p.K - k_first(t)) : p.K; };
  auto k_tiles = [&](int t) -> int { return (int)((k_count(t) + kTileK - 1) / kTileK); };
  const int xcd = blockIdx.x % kNumXcd, per_die = (gridDim.x - xcd + kNumXcd - 1) / kNumXcd;
  int tile = xcd * (tiles / kNumXcd) + min(xcd, tiles % kNumXcd);
  const int tile_end = tile + tiles / kNumXcd + (xcd < tiles % kNumXcd ? 1 : 0);
  tile += blockIdx.x / kNumXcd;
  if (tile >= tile_end) return;

  constexpr int kPitchW = S::kCols * 2, kPitchA = S::kRows * 2;                   // of operands with k as their slow axis
  const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void)smem;
  if (wave >= S::kWaves) {
    // ---- global -> LDS.  Load c of a loader: rows 8 (lw + kLoaders c) .. + 7 of an operand with k contiguous.  Of W [K, N]: 1
    // KB of whole rows.
    const int lw = wave - S::kWaves;
    const uint32_t rowa = (uint32_t)(p.lda * kElem), roww = (uint32_t)(p.ldw * kElem);
    const uint32_t chunk = (uint32_t)((lane & 7) ^ ((4 * lw + (lane >> 4)) & 7));
    const uint32_t va = (uint32_t)(8 * lw + (lane >> 3)) * rowa + 16 * chunk;
    const int tail = kAT ? 0 : (int)(p.K % kTileK) * kElem;                     // bytes
    const bool in_tail = (int)(16 * chunk) < tail;                             // (of the last k-tile, where that is not whole)
    const uint32_t vw = (uint32_t)(8 * lw + (lane >> 3)) * roww + 16 * chunk;
    // A descriptor holds the rows of the tile (rows past it read as zero); k advances in the scalar offset (for W [K, N] the
    // descriptor advances).
    auto rsrc = [&](uint64_t addr, int left, int most, uint32_t row) -> i32x4 {
      return (i32x4){(int)(uint32_t)addr, (int)(uint32_t)(addr >> 32), (int)(left > 0 ? (uint32_t)min(left, most) * row : 0u), 0x00020000};
    };
    auto dma16 = [&](const i32x4& rs, uint32_t voff, uint32_t soff, uint32_t dst) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "s"(dst), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
    };
    i32x4 ra, rw;
    // An operand with k as its slow axis: load c brings 1 KB of whole rows of the tile's columns, a descriptor holds the 64 rows
    // of a k-tile.  A row's swizzle depends on c through its parity at most.  (A loader's own instructions are what a k-tile of a
    // small tile waits for: nothing is computed per load but a sum.)
    struct Rows { uint64_t addr; uint32_t voff[2], stride; };
    auto aim_rows = [&](auto pitch, const void* base, int64_t k0, uint32_t row_bytes, int first_col, int cols, Rows& o) {
      constexpr int kPitch = decltype(pitch)::value, kPer = 1024 / kPitch, kChunks = kPitch / 16;
      static_assert(kPer == 2 || kPer == 4, "256 or 512 bytes");
      o.addr = (uint64_t)(uintptr_t)base + (uint64_t)k0 * row_bytes + (uint64_t)first_col * 2;
      o.stride = kPer * kLoaders * row_bytes;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int r = kPer * (lw + kLoaders * c) + lane / kChunks, ch = (lane % kChunks) ^ (4 * (r & 3) + ((r >> 2) & 3));
        o.voff[c] = first_col + 8 * ch < cols ? (uint32_t)(kPer * lw + lane / kChunks) * row_bytes + 16 * (uint32_t)ch : kOutside;
      }
    };
    Rows oa, ow;
    int nk = 0;
    int64_t load_k = 0;
    auto aim = [&](int t) {                                                       // the loads at tile t
      const int in_slab = kAT ? t % tiles_slab : t, tm = in_slab / tiles_n;
      const int64_t m0 = (int64_t)tm * S::kRows;
      const int n0 = (in_slab - tm * tiles_n) * S::kCols;
      nk = k_tiles(t);
      load_k = k_count(t);
      if constexpr (kAT) aim_rows(std::integral_constant<int, kPitchA>{}, p.A, k_first(t), rowa, (int)m0, (int)p.M, oa);
      else ra = rsrc((uint64_t)(uintptr_t)p.A + (uint64_t)m0 * rowa, (int)min((int64_t)S::kRows, p.M - m0), S::kRows, rowa);
      if constexpr (kWT) aim_rows(std::integral_constant<int, kPitchW>{}, p.W, k_first(t), roww, n0, p.N, ow);
      else rw = rsrc((uint64_t)(uintptr_t)p.W + (uint64_t)n0 * roww, p.N - n0, S::kCols, roww);
    };
    // k-tile `step` into stage s
    auto issue = [&](int step, int s) {
      const bool outside = tail != 0 && step == nk - 1 && !in_tail;
      const uint32_t dst = smem_base + (uint32_t)(s * S::kStage + lw * 1024), k_off = (uint32_t)step * 128;
      const int left = (int)min(load_k - (int64_t)step * kBK, (int64_t)kBK);
      const i32x4 da = kAT ? rsrc(oa.addr + (uint64_t)step * (kBK * rowa), left, kBK, rowa) : ra;
      const i32x4 dw = kWT ? rsrc(ow.addr + (uint64_t)step * (kBK * roww), left, kBK, roww) : rw;
      const uint32_t a0 = outside ? kOutside : va, w0 = outside ? kOutside : vw;
#pragma unroll
      for (int c = 0; c < S::kLoadsA; ++c)
        dma16(da, kAT ? oa.voff[c & 1] + (uint32_t)c * oa.stride : a0 + (uint32_t)(8 * kLoaders * c) * rowa, kAT ? 0u : k_off, dst + (uint32_t)(kLoaders * 1024 * c));
#pragma unroll
      for (int c = 0; c < S::kLoadsW; ++c)
        dma16(dw, kWT ? ow.voff[c & 1] + (uint32_t)c * ow.stride : w0 + (uint32_t)(8 * kLoaders * c) * roww, kWT ? 0u : k_off, dst + (uint32_t)(S::kA + kLoaders * 1024 * c));
    };
    // Loads run STAGES - 1 k-tiles ahead of the products, across tiles.  A loader waits for its loads alone: in a wave that
    // stores as well, waiting for a load means waiting for every store in front of it.
    int t = tile, step = 0, s = 0, flying = 0;
    aim(t);
    auto next = [&]() {
      issue(step, s);
      ++flying;
      s = s == STAGES - 1 ? 0 : s + 1;
      if (++step == nk) {
        step = 0;
        t += per_die;
        if (t < tile_end) aim(t);
      }
    };
#pragma unroll
    for (int i = 0; i < STAGES - 1; ++i)
      if (t < tile_end) next();
    while (flying > 0) {
      if (flying == STAGES - 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(S::kLoads * (STAGES - 2)) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      --flying;
      if (t < tile_end) next();
    }
    return;
  }

  // ---- LDS -> operands
  const int wm = wave / WN, wn = wave % WN;
  const uint32_t row128 = (uint32_t)(l32 * 128 + 16 * ((kFp8 ? 2 * hf : hf) ^ ((l32 >> 1) & 7)));   // k-step ks of a tile: chunk ^ 2 ks (E4M3: 4 ks)
  const uint32_t ta = smem_base + (uint32_t)(wm * 32 * MI * 128) + row128;
  const uint32_t tw = smem_base + S::kA + (uint32_t)(wn * 64 * 128) + row128;
  // Transposed: lanes of a half-wave take rows 8 hf + 0..3 (then + 4) of 16 k; lane l32 ends up with column l32's 8 values of k.
  const int vchunk = 2 * (grp16 & 1) + ((i16 & 3) >> 1), vbyte = 8 * (i16 & 1), vrow = i16 >> 2;
  const uint32_t tr_lo = (uint32_t)(16 * (vchunk ^ (2 * hf) ^ (4 * vrow))), tr_hi = (uint32_t)(16 * (vchunk ^ (2 * hf + 1) ^ (4 * vrow)));
  const uint32_t tra = smem_base + (uint32_t)((8 * hf + vrow) * kPitchA + vbyte), trw = smem_base + S::kA + (uint32_t)((8 * hf + vrow) * kPitchW + vbyte);
  auto transposed = [&](uint32_t at, uint32_t columns, int pitch) -> bf16x8 {     // columns: byte of the fragment's first one in its row
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(at + (tr_lo ^ columns)));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(at + (tr_hi ^ columns) + (uint32_t)(4 * pitch)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // (E4M3: a lane's 32 codes of 64 k are two neighbouring 16-byte chunks of its row, as in fp8_gemm_bias2d_kernel: which codes
  // meet in a lane changes the last bits of the matrix instruction's sums, and a row's results should not depend on the kernel)
  typedef typename std::conditional<kFp8, i32x8, bf16x8>::type Operand;
  auto contiguous = [&](uint32_t base, uint32_t at, int ks) -> Operand {
    if constexpr (kFp8) {
      const i32x4 lo = *(lds_i4)(uintptr_t)((base ^ (uint32_t)(64 * ks)) + at), hi = *(lds_i4)(uintptr_t)((base ^ (uint32_t)(64 * ks + 16)) + at);
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      return *(lds_b8)(uintptr_t)((base ^ (uint32_t)(32 * ks)) + at);
    }
  };
  auto wfrag = [&](uint32_t stage_off, int ks, int ni) -> Operand {
    if constexpr (kWT) return transposed(trw + stage_off + (uint32_t)(ks * 16 * kPitchW), (uint32_t)(16 * (8 * wn + 4 * ni)), kPitchW);
    else return contiguous(tw, stage_off + (uint32_t)(ni * 32 * 128), ks);
  };
  auto afrag = [&](uint32_t stage_off, int ks, int mi) -> Operand {
    if constexpr (kAT) return transposed(tra + stage_off + (uint32_t)(ks * 16 * kPitchA), (uint32_t)(64 * (MI * wm + mi)), kPitchA);
    else return contiguous(ta, stage_off + (uint32_t)(mi * 32 * 128), ks);
  };

  auto product = [&](const Operand& w, const Operand& x, const f32x16& acc) -> f32x16 {
    if constexpr (kFp8) return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, x, acc, 0, 0, 0, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, acc, 0, 0, 0);
  };
  constexpr int kSteps = kFp8 ? 2 : 4, kTotal = kSteps * MI;                       // k-steps of a k-tile
  Operand wf[2][2], af[2];
  uint32_t off = 0;                                                                // of the k-tile's stage
  auto first_operands = [&]() {
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) wf[0][ni] = wfrag(off, 0, ni);
    af[0] = afrag(off, 0, 0);
  };
  // this wave's reads of its k-tile are done and the loaders' loads of the next one have landed: the barrier frees the one and
  // publishes the other
  auto turn = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  turn();
  for (;;) {
    const int in_slab = kAT ? tile % tiles_slab : tile, tm = in_slab / tiles_n;
    const int64_t m0 = (int64_t)tm * S::kRows;
    const int n0 = (in_slab - tm * tiles_n) * S::kCols;
    const int next = tile + per_die, nk = k_tiles(tile);
    f32x16 acc[2][MI];
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ni][mi][r] = 0.f;
    first_operands();
    for (int step = 0; step < nk; ++step) {
      const uint32_t at = off;
#pragma unroll
      for (int n = 0; n < kTotal; ++n) {                                           // two products each; the operands of the next one are read first
        const int ks = n / MI, mi = n % MI;
        if (n + 1 < kTotal) {
          af[(n + 1) & 1] = afrag(at, (n + 1) / MI, (n + 1) % MI);
          if (mi == 0 && ks + 1 < kSteps) {
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) wf[(ks + 1) & 1][ni] = wfrag(at, ks + 1, ni);
          }
        } else if (step + 1 < nk || next < tile_end) {
          turn();
          off = off == (uint32_t)((STAGES - 1) * S::kStage) ? 0u : off + S::kStage;
          if (step + 1 < nk) first_operands();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) acc[ni][mi] = product(wf[ks & 1][ni], af[n & 1], acc[ni][mi]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    // ---- epilogue: 16 token rows x 64 columns at a time through the wave's own part of the staging (chunk c of row r at c ^ r)
    const int rows = (int)min((int64_t)S::kRows, p.M - m0) - 32 * MI * wm;         // of the wave's part of the tile
    const uint32_t area = smem_base + (uint32_t)(STAGES * S::kStage + wave * S::kArea);
    const uint32_t put = area + (uint32_t)((l32 & 15) * 256 + 16 * (hf ^ (l32 & 15)));
    const uint32_t get = area + (uint32_t)((lane >> 3) * 256 + 16 * ((2 * (lane & 7)) ^ (lane >> 3)));     // and 8 rows further: chunk ^ 8
    const int col = n0 + 64 * wn + 8 * (lane & 7);
    const bool col_ok = col < p.N;
    const bool first = (EPI == kEpiSiluSplit || EPI == kEpiPreAndSilu) && col < p.split;   // of the gate
    const int64_t w0 = m0 + 32 * MI * wm + (lane >> 3);
    const int64_t ldd = EPI == kEpiSiluSplit && first ? p.ldd0 : p.ldd;
    __bf16* const d = (EPI == kEpiSiluSplit && first ? (__bf16*)p.D0 : (__bf16*)p.D) + w0 * ldd + col;
    float* const sums = (float*)p.D + (kAT ? (int64_t)(tile / tiles_slab) * p.M * p.N : 0) + w0 * ldd + col;          // (kEpiSums)
    f32x4 sb[2];                                                                   // E4M3: the columns' scales, and the rows'
    constexpr bool kRes = EPI == kEpiResidual;
    float sa[kRes ? MI : 2];
    if (kFp8 && col_ok) {
      sb[0] = *(const f32x4*)(p.scale_w + col);
      sb[1] = *(const f32x4*)(p.scale_w + col + 4);
    }
    if (kFp8 && kRes) {                                                            // (of the accumulators' rows)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
        if (32 * mi + l32 < rows) sa[mi] = p.scale_a[m0 + 32 * (MI * wm + mi) + l32];
    }
    // Residual rows come kAhead parts early: memory operations complete in order, so waiting for a load waits for the stores
    // before it, and 16 rows in flight per wave do not cover the latency.  Descriptors drop what lies outside (the row is in the
    // lane's offset, which the range check covers): a branch would keep the compiler from counting the stores in between.  As
    // many parts as the registers hold.  us, one part -> these: E4M3, K = 1024, 262,144 x 1024 444 -> 430, 100,000 x 1024 176 ->
    // 171;  a bf16 layer's forward, widths 512, 6,400 rows 74.1 -> 72.8, 87,000 rows 643 -> 633.  Without a residual the rows'
    // scales stay one part early: all of them at once 851 -> 876 (the forward of 100,000 rows, E = 1024, H D = 512: the stores
    // come in one burst).
    constexpr int kAhead = !kRes ? 1 : MI == 1 || MI == 4 ? 2 : MI == 2 && S::kWavesPerSimd == 4 ? 3 : 4;
    u32x4 res[kAhead][2];
    __amdgpu_buffer_rsrc_t rc, rd;
    const uint32_t vc = col_ok ? (uint32_t)((lane >> 3) * p.ldc + col) * 2 : kOutside, vd = col_ok ? (uint32_t)((lane >> 3) * p.ldd + col) * 2 : kOutside;
    if (kRes) {
      const int64_t r0 = m0 + 32 * MI * wm;
      const int there = max(0, min(rows, 32 * MI));
      rc = __builtin_amdgcn_make_buffer_rsrc((void*)((const __bf16*)p.C + (there ? r0 * p.ldc : 0)), 0, (int)(there * p.ldc * 2), 0x00020000);
      rd = __builtin_amdgcn_make_buffer_rsrc((void*)((__bf16*)p.D + (there ? r0 * p.ldd : 0)), 0, (int)(there * p.ldd * 2), 0x00020000);
    }
    auto fetch = [&](int part) {
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int row = 16 * part + 8 * it;
        if (kRes) res[part % kAhead][it] = __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(vc + (uint32_t)(row * p.ldc * 2)), 0, 0);
        else if (kFp8 && col_ok && row + (lane >> 3) < rows) sa[it] = p.scale_a[w0 + row];
      }
    };
    if (kRes || kFp8) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i) fetch(i);
    }
#pragma unroll
    for (int part = 0; part < 2 * MI; ++part) {
      const int mi = part / 2;
      if (kFp8 && kRes && part % 2 == 0) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[ni][mi][r] *= sa[mi];
      }
      if ((l32 >> 4) == part % 2) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *(lds_f4)(uintptr_t)(put ^ (uint32_t)(128 * ni + 32 * q)) =
                (f32x4){acc[ni][mi][4 * q], acc[ni][mi][4 * q + 1], acc[ni][mi][4 * q + 2], acc[ni][mi][4 * q + 3]};
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                           // (the wave's own writes: no other wave touches its part)
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const uint32_t at = (get ^ (uint32_t)(128 * it)) + (uint32_t)(8 * 256 * it);
        const f32x4 lo = *(lds_f4)(uintptr_t)at, hi = *(lds_f4)(uintptr_t)(at ^ 16);
        const int row = 16 * part + 8 * it;
        float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        if (!kRes && (!col_ok || row + (lane >> 3) >= rows)) continue;
        if (EPI == kEpiSums) {
          *(f32x4*)(sums + row * ldd) = lo;
          *(f32x4*)(sums + row * ldd + 4) = hi;
          continue;
        }
        if (kFp8) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = (kRes ? v[e] : v[e] * sa[it]) * sb[e / 4][e % 4];
        }
        if (kRes) {
          // (E4M3: the scaled product is rounded before the residual is added, as in fp8_gemm_bias2d_kernel: a row's results do
          // not depend on how many rows are beside it)
#pragma clang fp contract(off)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[2 * e] += __uint_as_float(res[part % kAhead][it][e] << 16);
            v[2 * e + 1] += __uint_as_float(res[part % kAhead][it][e] & 0xFFFF0000u);
          }
          const u32x4 o = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
          __builtin_amdgcn_raw_buffer_store_b128(o, rd, (int)(vd + (uint32_t)(row * p.ldd * 2)), 0, 2);     // (non-temporal)
          continue;
        }
        if (EPI == kEpiSiluSplit) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = silu(v[e]);
        }
        store8(d + row * ldd, v);
        if (EPI == kEpiPreAndSilu && !first) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = silu(v[e]);
          store8((__bf16*)p.D0 + (w0 + row) * p.ldd0 + col, v);
        }
      }
      if ((kRes || kFp8) && part + kAhead < 2 * MI) fetch(part + kAhead);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    tile = next;
    if (tile >= tile_end) return;
  }
}

template <int WM, int WN, int MI, int STAGES, int OP, int EPI>
hipError_t launch_tile(const GemmRowsArgs& p, hipStream_t stream) {
  using S = Tile<WM, WN, MI, STAGES>;
  static bool attr_set[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {
    const hipError_t e = hipFuncSetAttribute((const void*)gemm_rows_kernel<WM, WN, MI, STAGES, OP, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, S::kSmem);
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  const int64_t slabs = OP == kGemmTN ? (p.K + p.slab - 1) / p.slab : 1;
  const int64_t tiles = ((p.M + S::kRows - 1) / S::kRows) * ((p.N + S::kCols - 1) / S::kCols) * slabs;
  if (tiles > INT32_MAX / 2) return hipErrorInvalidValue;
  const int grid = (int)std::min<int64_t>(tiles, 256 * S::kWgPerCu);
  hipLaunchKernelGGL((gemm_rows_kernel<WM, WN, MI, STAGES, OP, EPI>), dim3(grid), dim3(S::kThreads), S::kSmem, stream, p, (int)tiles);
  return hipGetLastError();
}
template <int OP, int EPI>
hipError_t launch_epi(const GemmRowsArgs& p, int tile, hipStream_t stream) {
  if constexpr (OP == kGemmTN) {
    return tile == kTile128Deep ? launch_tile<2, 2, 2, 4, OP, EPI>(p, stream) : launch_tile<2, 2, 2, 2, OP, EPI>(p, stream);
  } else if constexpr (OP == kGemmFp8) {
    if constexpr (EPI != kEpiResidual)
      if (tile == kTile192) return launch_tile<2, 4, 3, 2, OP, EPI>(p, stream);
    return tile == kTile64Deep ? launch_tile<2, 2, 1, 5, OP, EPI>(p, stream)
         : tile == kTile64 ? launch_tile<2, 2, 1, 2, OP, EPI>(p, stream) : launch_tile<2, 4, 2, 2, OP, EPI>(p, stream);
  } else {
    switch (tile) {
      case kTile64Deep: return launch_tile<2, 2, 1, 5, OP, EPI>(p, stream);
      case kTile64: return launch_tile<2, 2, 1, 2, OP, EPI>(p, stream);
      case kTile128Deep: return launch_tile<2, 2, 2, 4, OP, EPI>(p, stream);
      case kTile128: return launch_tile<2, 2, 2, 2, OP, EPI>(p, stream);
      case kTile192: return launch_tile<2, 4, 3, 2, OP, EPI>(p, stream);
      default: return launch_tile<2, 4, 4, 2, OP, EPI>(p, stream);
    }
  }
}

}  // namespace

// With long rows and much work the library's kernels are the faster ones, once they have been chosen for the size.  They are
// chosen by timing on a class's first call, which blocks, and then serve every count of the class, some of them badly.  So a
// class goes to the library as a whole, and only if its smallest count is beyond the line: one call leaves nothing to choose for
// another of its class.  A layer's step with widths of 1024, us, library (chosen for this count) -> here: 30,000 rows 1,939 ->
// 1,910, 60,000 rows 3,678 -> 3,602, 120,000 rows 7,232 -> 7,205 (forward 1,715 -> 1,746); 26,000 rows, chosen for 24,000, the
// forward 482 -> 408.  Widths of 2048: 15,000 rows 2,854 -> 2,921, 50,000 rows 9,192 -> 9,689; 8,000 rows, chosen for 6,000,
// 1,739 -> 1,598, but 7,500 rows, chosen for them, 1,489 -> 1,532.  Below the line a forward is up to 11 % slower than with the
// library's kernels chosen for the very count (16,000 rows, widths of 1024 231 -> 247, 5,000 rows, widths of 2048 227 -> 251), a
// step as fast or faster, and neither waits for a choice.
bool gemm_rows_preferred(int64_t M, int64_t N, int64_t K) { return K < 1024 || (double)(token_class(M) / 2) * (double)N * (double)K < 1e11; }

hipError_t launch_gemm_rows(const GemmRowsArgs& p, int op, int epilogue, hipStream_t stream) {
  if (p.M <= 0 || p.N <= 0 || p.K <= 0 || p.N % 8 != 0 || (op != kGemmTN && p.K % 8 != 0)) return hipErrorInvalidValue;
  const bool residual = epilogue == kEpiResidual;
  const int tile = op == kGemmTN ? (p.M + 127) / 128 * ((p.N + 127) / 128) * ((p.K + p.slab - 1) / p.slab) <= 256 ? kTile128Deep : kTile128
                 : op == kGemmFp8 ? fp8_tile(p.M, p.N, residual) : gemm_rows_tile(p.M, p.N, p.K, residual);
  if (op == kGemmNT && epilogue == kEpiSiluSplit) return launch_epi<kGemmNT, kEpiSiluSplit>(p, tile, stream);
  if (op == kGemmNT && epilogue == kEpiPreAndSilu) return launch_epi<kGemmNT, kEpiPreAndSilu>(p, tile, stream);
  if (op == kGemmNT && epilogue == kEpiResidual) return launch_epi<kGemmNT, kEpiResidual>(p, tile, stream);
  if (op == kGemmNN && epilogue == kEpiPlain) return launch_epi<kGemmNN, kEpiPlain>(p, tile, stream);
  if (op == kGemmFp8 && epilogue == kEpiPlain) return launch_epi<kGemmFp8, kEpiPlain>(p, tile, stream);
  if (op == kGemmFp8 && epilogue == kEpiResidual) return launch_epi<kGemmFp8, kEpiResidual>(p, tile, stream);
  if (op == kGemmFp8 && epilogue == kEpiSiluSplit) return launch_epi<kGemmFp8, kEpiSiluSplit>(p, tile, stream);
  if (op == kGemmTN && epilogue == kEpiSums) return launch_epi<kGemmTN, kEpiSums>(p, tile, stream);
  return hipErrorInvalidValue;
}

}  // namespace hstu
