// Attention backward for bf16 with 32 or 64 features per head: the dQ pass and the dK/dV pass as software pipelines inside every wave.
//
// Both passes recompute scores (handing dS on would move as many bytes as for 128 features and save a half or a quarter of the matrix work).
// With this few features the pointwise work (two transcendentals and five plain instructions per score) takes longer than the matrix
// instructions, and a matrix instruction hides vector instructions only when they follow it in the same wave.  So a wave walks its tiles
// of 32 streamed rows in steps that hold two of them:
//   step s, first half:   S(s) = Y1(s) R1^T, dP(s) = Y2(s) R2^T        |  pointwise work of streamed rows 16..31 of tile s - 1
//   step s, second half:  output products of tile s - 1                |  pointwise work of streamed rows 0..15 of tile s
// (dQ pass: R = Q, dO, Y = K, V, output dQ += K^T dS; dK/dV pass: R = K, V, Y = Q, dO, outputs dV += dO^T P, dK += Q^T dS.)
// Scores are seeded with the bias as a function of the distance, the dK/dV pass takes the seeds in ascending order; candidates, which stand
// at one position, are seeded element by element in a second copy of the loop.  A tile that holds only pairs that the wave's rows may see
// goes through as it is; in any other the score and dP of masked pairs are replaced between the halves (-1e30 leaves P = -0 and
// dS / dP = 0), whatever their rows held, and the output products of a tile with no visible pair read zeros instead of its rows: rows that
// are not finite stay with the tokens that may see them.  (Against a mask in the seeds, which needs finite rows: 8 x 8k-16k, 64 features, semi-local
// 586 -> 604 us, dense 2,413 -> 2,430; 24 x 1-3,000 semi-local 196 -> 201; 2 x 396, K1 = 168, where hardly a tile is full, 32.6 -> 36.9.)
//
// Tiles and seed strips are loaded straight to LDS three steps ahead: those of step s + 3 are issued in step s, have landed and are published
// at the end of step s + 1, and the first fragments are read at the end of step s + 2; the output products read tile s - 1: five stages.
#include <type_traits>
#include <utility>

#include "dist_sums.h"
#include "hstu_common.h"
#include "hstu_kernels.h"

namespace hstu {
namespace {

enum { kDQ = 0, kDKDV = 1 };
constexpr int kBX = 128, kBN = 32, kWaves = 4, kThreads = 64 * kWaves;
constexpr int kStages = 5, kStripStages = 4;
constexpr int kStripCopy = 1088, kStripBytes = 4 * kStripCopy;         // as in attn_fwd_pipe.hip
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
constexpr float kMasked = -1e30f;
constexpr int kNoTile = 1 << 25;                                        // (beyond any tile, and its first row still an int)

template <int D, int MODE>
struct Narrow {
  static constexpr int kRow = 2 * D, kTile = kBN * kRow, kStage = 2 * kTile;
  static constexpr int kSteps = D / 16, kBlocks = D / 32, kOut = MODE == kDKDV ? 2 : 1;
  static constexpr int kSlots1 = 2 * kSteps, kSlots2 = 2 * kBlocks * kOut;               // matrix instructions of the two halves
  static constexpr int kScores1 = 8 / kSlots1, kScores2 = 8 / kSlots2;                    // scores per slot
  static constexpr int kRowsPer = 1024 / kRow;                                            // rows that one wave-level load brings
  static constexpr bool kSplit = D == 32;              // waves 0 and 1 load Y1, 2 and 3 load Y2 (else every wave 8 rows of each)
  static constexpr int kLoads = kSplit ? 2 : 3;        // per wave and step
  static constexpr int kZero = kStages * kStage, kStripBase = kZero + kOut * kTile, kSmemBytes = kStripBase + kStripStages * kStripBytes;
  static __device__ __forceinline__ int swizzle(int r) { return D == 64 ? 4 * ((r >> 1) & 1) + ((r >> 2) & 3) : (r >> 2) & 3; }   // as Pipe::swizzle
};

typedef __attribute__((address_space(3))) void* lds_void;
typedef __attribute__((address_space(3))) short4v* lds_s4;
typedef __attribute__((address_space(3))) const bf16x8* lds_b8;
typedef __attribute__((address_space(3))) const f32x4* lds_f4;
template <int N> using IC = std::integral_constant<int, N>;
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

template <int D, int MODE, bool CAND, bool DBIAS>
__global__ __launch_bounds__(kThreads, 2) void attn_bwd_narrow_kernel(const AttnArgs a) {
  using W = Narrow<D, MODE>;
  constexpr int kSteps = W::kSteps, kBlocks = W::kBlocks, kOut = W::kOut, kSlots1 = W::kSlots1, kSlots2 = W::kSlots2;
  static_assert(!DBIAS || MODE == kDQ, "the bias gradient rides with the dQ pass");
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  const int wg = blockIdx.x;
  const int xcd = wg % kNumXcd, slot_id = wg / kNumXcd;
  const int pos = ((slot_id / kXcdGroup) * kNumXcd + xcd) * kXcdGroup + slot_id % kXcdGroup;
  const int count = a.header->count;                                   // (fetched together with the entry, which is dropped if beyond)
  const WorkItem item = a.items[min(pos, a.max_items - 1)];
  if (pos >= count) return;
  const int xb = item.rb_h >> 8, h = item.rb_h & 255, seq0 = item.seq0, L = item.len;
  const SeqGeom g = {L, item.hist, a.K1, a.K2};
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5, l32 = lane & 31, grp16 = lane >> 4, i16 = lane & 15;
  const int x0 = xb * kBX, xw0 = x0 + wave * 32, x = xw0 + l32;
  const bool x_ok = x < L;

  const int64_t hoff = (int64_t)h * D;
  const int64_t sr1 = MODE == kDQ ? a.sq : a.sk, sr2 = MODE == kDQ ? a.so : a.sv, sy1 = MODE == kDQ ? a.sk : a.sq, sy2 = MODE == kDQ ? a.sv : a.so;
  const __bf16* R1 = (const __bf16*)(MODE == kDQ ? a.q : a.k) + seq0 * sr1 + hoff;
  const __bf16* R2 = (const __bf16*)(MODE == kDQ ? a.dout : a.v) + seq0 * sr2 + hoff;
  const __bf16* Y1 = (const __bf16*)(MODE == kDQ ? a.k : a.q) + seq0 * sy1 + hoff;
  const __bf16* Y2 = (const __bf16*)(MODE == kDQ ? a.v : a.dout) + seq0 * sy2 + hoff;

  // ---- stationary rows as B operands; that of the score product times alpha log2 e (scores in units of ln 2)
  bf16x8 r1[kSteps], r2[kSteps];
#pragma unroll
  for (int ks = 0; ks < kSteps; ++ks) {
    u32x4 raw1 = {0u, 0u, 0u, 0u}, raw2 = {0u, 0u, 0u, 0u};
    if (x_ok) {
      raw1 = *(const u32x4*)(R1 + (int64_t)x * sr1 + ks * 16 + hf * 8);
      raw2 = *(const u32x4*)(R2 + (int64_t)x * sr2 + ks * 16 + hf * 8);
    }
    r1[ks] = __builtin_bit_cast(bf16x8, raw1);
    r2[ks] = __builtin_bit_cast(bf16x8, raw2);
  }
  auto finish_rows = [&]() {                                           // (first use behind the first tiles' loads)
    const float score_scale = kLog2e * a.alpha;
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) {
      u32x4 raw = __builtin_bit_cast(u32x4, r1[ks]);
#pragma unroll
      for (int w = 0; w < 4; ++w)
        raw[w] = pack_bf16x2(__builtin_bit_cast(float, raw[w] << 16) * score_scale, __builtin_bit_cast(float, raw[w] & 0xFFFF0000u) * score_scale);
      r1[ks] = __builtin_bit_cast(bf16x8, raw);
    }
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) asm volatile("" : "+v"(r1[ks]), "+v"(r2[ks]));
  };

  f32x16 out[kOut][kBlocks];
#pragma unroll
  for (int o = 0; o < kOut; ++o)
#pragma unroll
    for (int ob = 0; ob < kBlocks; ++ob)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[o][ob][r] = 0.f;

  // ---- the item's tiles; those with a candidate's row are the last ones
  const int xlast = min(x0 + kBX, L) - 1;
  const TileRanges tr = MODE == kDQ ? tile_ranges(g, x0, xlast, kBN) : row_tile_ranges(g, x0, xlast, kBN);
  const int t_begin = item.t0, t_end = max(min(tr.count(), item.t1), item.t0), n = t_end - t_begin;
  const int na = tr.a1 - tr.a0, nb = tr.b1 - tr.b0, nc = tr.c1 - tr.c0;
  const int cand_t0 = (CAND && g.n < L) ? g.n / kBN : kNoTile;         // first tile with a candidate's row
  const int pc = min(max(cand_t0 - tr.a0, 0), na) + min(max(cand_t0 - tr.b0, 0), nb) + min(max(cand_t0 - tr.c0, 0), nc);
  const int nfast = min(max(pc, t_begin), t_end) - t_begin;
  auto tile_of = [&](int idx) -> int { return tr.at(t_begin + idx); };
  const WaveTiles tiles = MODE == kDQ ? key_tiles_of(g, xw0) : query_tiles_of(g, xw0);
  const bool band = g.K1 >= 0;

  // ---- seeds
  const int px = (MODE == kDQ && CAND) ? min(x, g.n) : x, x0v = (MODE == kDQ && CAND) ? min(x0, g.n) : x0;
  const int strip_s0 = kBX - 1 - (px - x0v) + 4 * hf;
  const float* seed_h = (MODE == kDQ ? a.seed : a.seed_up) + (int64_t)h * a.seed_len;
  const int seed0 = MODE == kDQ ? a.seed_dmax : kSeedUpZero;            // index of distance 0
  const float bias0 = CAND ? seed_h[seed0] : 0.f;                       // a candidate's own pair
  const float cand_seed = CAND && MODE == kDKDV && x < g.n ? seed_h[seed0 + g.n - x] : 0.f;      // of this lane's key for the candidates, all at position n

  // ---- global -> LDS
  const bool second = W::kSplit && wave >= 2;
  const uint32_t rowb1 = (uint32_t)((second ? sy2 : sy1) * 2), rowb2 = (uint32_t)(sy2 * 2);
  const uint64_t base1 = (uint64_t)(uintptr_t)(second ? Y2 : Y1), base2 = (uint64_t)(uintptr_t)Y2;
  const int wrow = W::kRowsPer * (W::kSplit ? wave & 1 : wave);         // first row of a tile that this wave loads
  const int dma_row = lane / (64 / W::kRowsPer);
  const int dma_chunk = (lane % (64 / W::kRowsPer)) ^ W::swizzle(wrow + dma_row);
  uint32_t voff1 = __umul24((uint32_t)dma_row, rowb1) + (uint32_t)(dma_chunk * 16);
  uint32_t voff2 = __umul24((uint32_t)dma_row, rowb2) + (uint32_t)(dma_chunk * 16);
  uint32_t voffS = 16u * (uint32_t)lane + 4u * (uint32_t)wave;
  asm volatile("" : "+v"(voff1), "+v"(voff2), "+v"(voffS));
  auto make_rsrc = [&](uint64_t addr, uint32_t bytes) -> i32x4 {
    return (i32x4){__builtin_amdgcn_readfirstlane((int)(uint32_t)addr), __builtin_amdgcn_readfirstlane((int)(uint32_t)(addr >> 32)),
                   __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
  };
  const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void)smem;
  const uint32_t m0_rows = smem_base + (uint32_t)(wave & (W::kSplit ? 1 : 3)) * 1024u + (second ? (uint32_t)W::kTile : 0u);
  const uint32_t m0_strip = smem_base + (uint32_t)W::kStripBase + (uint32_t)wave * (uint32_t)kStripCopy;
  auto dma16 = [&](i32x4 rs, uint32_t voff, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(voff), "s"(rs) : "memory", "m0");
  };
  // where a tile sits; one beyond the list has empty ranges (its loads are still issued: the waits count loads)
  struct Src { uint64_t a1, a2; int left; uint32_t s_off; int yt; };
  auto src_of = [&](int idx) -> Src {
    const bool valid = idx < n;
    const int yt = valid ? tile_of(idx) : 0;
    const int yrow = yt * kBN + wrow;
    Src r;
    r.a1 = base1 + (uint64_t)(uint32_t)yrow * rowb1;
    r.a2 = base2 + (uint64_t)(uint32_t)yrow * rowb2;
    r.left = valid ? L - yrow : -kNoTile;
    // strip index s: distance x0v + kBX - 1 - y0 - s (dQ pass), y0 - x0 - (kBX - 1) + s (dK/dV pass)
    r.s_off = 4u * (uint32_t)(MODE == kDQ ? seed0 - (x0v + (kBX - 1) - yt * kBN) : seed0 + yt * kBN - x0 - (kBX - 1));
    r.yt = valid ? yt : kNoTile;
    return r;
  };
  auto next_src = [&](const Src& prev, int idx) -> Src {                // nearly always the next tile of the sequence
    const int yt = idx < n ? tile_of(idx) : kNoTile;
    if (__builtin_expect(yt != prev.yt + 1, 0)) return src_of(idx);
    Src r = prev;
    r.a1 = prev.a1 + kBN * rowb1;
    r.a2 = prev.a2 + kBN * rowb2;
    r.left = prev.left - kBN;
    r.s_off = prev.s_off + 4u * kBN;
    r.yt = yt;
    return r;
  };
  auto load = [&](const Src& sr, int what, uint32_t stage_off, int strip_stage) {      // what: 0 .. kLoads - 1
    const uint32_t left = (uint32_t)max(sr.left, 0);
    if (what == 0) dma16(make_rsrc(sr.a1, left * rowb1), voff1, m0_rows + stage_off);
    else if (what == 1 && !W::kSplit) dma16(make_rsrc(sr.a2, left * rowb2), voff2, m0_rows + stage_off + W::kTile);
    else dma16(make_rsrc((uint64_t)(uintptr_t)seed_h, sr.yt == kNoTile ? 0u : (uint32_t)a.seed_len * 4u), voffS + sr.s_off, m0_strip + (uint32_t)(strip_stage * kStripBytes));
  };

  // ---- LDS fragment addresses, moved from stage to stage by an addition per step
  const int zl = W::swizzle(l32);
  const int kb = (int)smem_base + l32 * W::kRow + ((hf ^ (zl & 1)) << 4) + ((zl >> 1) << 5);
  const int vchunk = 2 * (grp16 & 1) + ((i16 & 3) >> 1), vbyte = 8 * (i16 & 1);
  const int tb = (int)smem_base + (4 * hf + (i16 >> 2)) * W::kRow + ((W::swizzle(i16 >> 2) >> 2) << 6) + ((vchunk ^ hf) << 4) + vbyte;
  int kaddr[kSteps], taddr[2 * kBlocks];
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    kaddr[i] = kb ^ (i << 5);
    taddr[i] = (tb ^ (((i >> 1) << 6) | ((i & 1) << 5))) + W::kZero;      // "tile -1"
    asm volatile("" : "+v"(kaddr[i]), "+v"(taddr[i]));
  }
  const int saddr = (int)smem_base + W::kStripBase + (strip_s0 & 3) * kStripCopy + (strip_s0 & ~3) * 4;
  auto rowfrag = [&](int i) -> bf16x8 {                                 // slot i of the first half
    return *(lds_b8)(uintptr_t)(uint32_t)(kaddr[i % kSteps] + (i / kSteps) * W::kTile);
  };
  // slot j of the second half: k-step (16 streamed rows), output, feature block.  dK/dV pass: dV (from dO) first
  auto ks2_of = [](int j) { return j / (kOut * kBlocks); };
  auto out_of = [](int j) { return MODE == kDQ ? 0 : 1 - (j / kBlocks) % 2; };           // 0: dQ / dK, 1: dV
  auto trfrag = [&](int j) -> bf16x8 {
    const int ob = j % kBlocks, at = ks2_of(j) * 16 * W::kRow + (out_of(j) == 1 ? W::kTile : 0);
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(uint32_t)(taddr[2 * ob] + at));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(uint32_t)(taddr[2 * ob + 1] + at + 8 * W::kRow));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // Below, c is a compile-time constant per score register: streamed row y0 + c with y0 = first row of the tile + 4 hf.
  // Seeds of a tile with candidates' rows.
  auto seed_candidates = [&](f32x16& acc, int yt) {
    const int y0 = yt * kBN + 4 * hf, hist = g.n - y0, selfc = x >= g.n ? x - y0 : -1000;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int c = 8 * (r >> 2) + (r & 3);
      if (MODE == kDKDV) acc[r] = c < hist ? acc[r] : cand_seed;
      acc[r] = c == selfc ? bias0 : acc[r];
    }
  };
  // Masked pairs of a tile that is not full; returns whether none is visible.
  auto mask = [&](f32x16& sc, f32x16& dp, int yt) -> bool {
    const int t0 = yt * kBN;
    if (tiles.empty(yt)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { sc[r] = kMasked; dp[r] = 0.f; }
      return true;
    }
    int x = xw0 + l32;
    asm volatile("" : "+v"(x));                                          // (nothing of this is kept in registers through the loop)
    const bool x_ok = x < L;
    const int px = (MODE == kDQ && CAND) ? min(x, g.n) : x, y0 = t0 + 4 * hf;
    const int selfc = CAND && x >= g.n ? x - y0 : -1;                    // a candidate sees itself
    uint32_t vis;                                                        // bit c: this lane's row sees, or is seen by, streamed row y0 + c
    if constexpr (MODE == kDQ) {
      const int last = min(px, g.n - 1) - y0;                           // history keys up to the row's position, inside the window or the prefix
      vis = ~bits_from(last + 1) & (band ? bits_from(px - g.K1 + 1 - y0) | ~bits_from(g.K2 - y0) : ~0u);
    } else {
      const int last = (band && x >= g.K2 ? min(x + g.K1, g.n) : g.n) - 1 - y0;
      vis = bits_from(x - y0) & ~bits_from(last + 1);
      if (CAND && x < g.n && (!band || g.n - x < g.K1 || x < g.K2)) vis |= bits_from(g.n - y0) & ~bits_from(L - y0);
    }
    if (CAND) vis |= selfc >= 0 && selfc < 32 ? 1u << selfc : 0u;
    if (!x_ok) vis = 0u;
    mask_scores<true>(vis, sc, kMasked, dp);
    return false;
  };
  auto seed = [&](f32x16& acc, int strip_stage) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 bv = *(lds_f4)(uintptr_t)(uint32_t)(saddr + strip_stage * kStripBytes + 32 * q4);
      acc[4 * q4 + 0] = bv[0]; acc[4 * q4 + 1] = bv[1]; acc[4 * q4 + 2] = bv[2]; acc[4 * q4 + 3] = bv[3];
    }
  };

  // ---- bias gradient
  DistSums<1, 1> dist;
  if constexpr (DBIAS) dist.init(a, xcd, h);
  auto dist_tile = [&](const auto& ds, int yt) {                        // ds: this lane's 16 values of tile yt, masked ones zero
    const int y0 = yt * kBN, w0 = xw0 - y0;
    if (CAND && xw0 + 31 >= g.n) {
      // candidate rows stand at position n: one distance per key (their own key: distance 0), summed over the rows
      float cv[16], hv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) { cv[r] = x < g.n ? 0.f : ds[r]; hv[r] = x < g.n ? ds[r] : 0.f; }
      const float v = row_sums(cv, i16);
      const int y = y0 + 8 * (i16 >> 2) + 4 * hf + (i16 & 3);
      if (v != 0.f) atomicAdd(dist.dist_h + max(g.n - y, 0), v);
      if (xw0 < g.n) dist.add(hv, 0, w0, 0);
    } else if (xw0 < L && w0 > -32) {
      dist.add(ds, 0, w0, w0 >= 31 ? dist.one_bucket(w0) : 0);
    }
  };

  // ---- prologue
  Src cur = src_of(0);
  int yt0 = cur.yt, yt1 = kNoTile, yt2 = kNoTile;                       // of tiles s, s + 1, s + 2; cur: s + 3 once step s has issued it
  const int yt_first = cur.yt;
#pragma unroll
  for (int what = 0; what < W::kLoads; ++what) load(cur, what, 0, 0);
  cur = next_src(cur, 1); yt1 = cur.yt;
#pragma unroll
  for (int what = 0; what < W::kLoads; ++what) load(cur, what, W::kStage, 1);
  cur = next_src(cur, 2); yt2 = cur.yt;
#pragma unroll
  for (int what = 0; what < W::kLoads; ++what) load(cur, what, 2 * W::kStage, 2);
  {                                                                     // the zeros that are read in place of a tile with no visible pair, and of "tile -1" in step 0
    Src none = src_of(n);
    if (kOut == 2 || !second) load(none, 0, W::kZero, 3);
    if (kOut == 2 && !W::kSplit) load(none, 1, W::kZero, 3);
  }
  finish_rows();
  wait_loads<0>();
  __syncthreads();

  f32x16 sacc[2], pacc[2];
  uint32_t pk[kOut][2][8];                                              // packed dS, and P (dK/dV pass)
  constexpr int kPF = 2;                                                // slots between a fragment's LDS read and its product
  bf16x8 fr[kPF + 1];
#pragma unroll
  for (int i = 0; i < kPF; ++i) fr[i] = rowfrag(i);
  seed(sacc[0], 0);
  if (CAND && nfast == 0 && n > 0) seed_candidates(sacc[0], yt_first);
#pragma unroll
  for (int r = 0; r < 16; ++r) { sacc[1][r] = 0.f; pacc[1][r] = 0.f; }
#pragma unroll
  for (int o = 0; o < kOut; ++o)
#pragma unroll
    for (int i = 0; i < 8; ++i) pk[o][0][i] = pk[o][1][i] = 0u;

  // The pointwise work as a rolling chain: a score's exp2, a slot's share later its reciprocal, another share later P and dS.
  float c_t1 = 0.f, c_d1 = 0.f, c_e1 = 0.f, c_t2 = 0.f, c_d2 = 0.f, c_g2 = 0.f, c_p = 0.f, c_s = 0.f;
  float dsv[2][DBIAS ? 16 : 1];
  // feeds one score; q, r: the score that comes out, register r of the tile of parity q
  auto feed = [&](float t, float d, int q, int r) {
    const float e = __builtin_amdgcn_exp2f(-t);
    const float gg = __builtin_amdgcn_rcpf(1.0f + c_e1);
    const float p = c_t2 * c_g2;
    const float s = c_d2 * fmaf(p, fmaf(-kLn2, c_g2, kLn2), c_g2);
    c_t2 = c_t1; c_d2 = c_d1; c_g2 = gg;
    c_t1 = t; c_d1 = d; c_e1 = e;
    asm volatile("" : "+v"(c_g2), "+v"(c_e1));                           // the work stays in its slot
    if constexpr (DBIAS) dsv[q][r] = s;
    if (r & 1) {
      pk[0][q][r >> 1] = pack_bf16x2(c_s, s);
      asm volatile("" : "+v"(pk[0][q][r >> 1]));
      if constexpr (MODE == kDKDV) { pk[kOut - 1][q][r >> 1] = pack_bf16x2(c_p, p); asm volatile("" : "+v"(pk[kOut - 1][q][r >> 1])); }
    } else {
      c_s = s; c_p = p;
    }
  };

  // Stages of tiles s + 3 and s, which go round, and where the output products of tile s - 1 read.
  int load_stage = 3, row_stage = 0, tr_off = W::kZero;
  int full_end = 0;                                                     // up to here tiles hold only visible pairs of this wave's rows
  int yt_m1 = kNoTile;                                                  // tile s - 1
  auto step = [&](int s, auto par_c, auto cand_c) {
    constexpr int P = decltype(par_c)::value;
    constexpr bool CAND_TILES = decltype(cand_c)::value;
    if constexpr (DBIAS) dist.late_out();
    cur = next_src(cur, s + 3);
    const uint32_t load_off = (uint32_t)(load_stage * W::kStage);
    const int load_strip = (s + 3) & (kStripStages - 1);
    bf16x8 nfr[kPF];
#pragma unroll
    for (int r = 0; r < 16; ++r) pacc[P][r] = 0.f;
    // ---------------- first half
#pragma unroll
    for (int i = 0; i < kSlots1; ++i) {
      if (i < W::kLoads) load(cur, i, load_off, load_strip);
      if (i + kPF < kSlots1) fr[(i + kPF) % (kPF + 1)] = rowfrag(i + kPF);
      else fr[(i + kPF) % (kPF + 1)] = trfrag(i + kPF - kSlots1);
      __builtin_amdgcn_sched_barrier(0);
      if (i < kSteps) sacc[P] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % (kPF + 1)], r1[i % kSteps], sacc[P], 0, 0, 0);
      else pacc[P] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % (kPF + 1)], r2[i % kSteps], pacc[P], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = i * W::kScores1; e < (i + 1) * W::kScores1; ++e) feed(sacc[P ^ 1][8 + e], pacc[P ^ 1][8 + e], P ^ 1, 6 + e);
      __builtin_amdgcn_sched_barrier(0);
    }
    int tr_next = row_stage * W::kStage;
    if (yt0 >= full_end) {                                              // (tiles ascend)
      full_end = tiles.full_end(yt0);
      if (yt0 >= full_end && yt0 != kNoTile && mask(sacc[P], pacc[P], yt0)) tr_next = W::kZero;
    }
    {
      const int next = row_stage == kStages - 1 ? 0 : row_stage + 1, delta = (next - row_stage) * W::kStage;
      row_stage = next;
#pragma unroll
      for (int i = 0; i < kSteps; ++i) kaddr[i] += delta;
    }
    // ---------------- second half
#pragma unroll
    for (int j = 0; j < kSlots2; ++j) {
      if (j == kSlots2 / 2) {
        seed(sacc[P ^ 1], (s + 1) & (kStripStages - 1));
        if (CAND_TILES) { if (s + 1 >= nfast && s + 1 < n) seed_candidates(sacc[P ^ 1], yt1); }
      }
      constexpr int N = kSlots1 + kSlots2;
      const int f = kSlots1 + j;                                        // slot of the step
      if (f + kPF < N) fr[(f + kPF) % (kPF + 1)] = trfrag(j + kPF);
      else if (f + kPF - N < kPF) nfr[f + kPF - N] = rowfrag(f + kPF - N);
      __builtin_amdgcn_sched_barrier(0);
      {
        const int o = out_of(j), ks2 = ks2_of(j), ob = j % kBlocks;
        const uint32_t* w = pk[o][P ^ 1];
        const bf16x8 pb = __builtin_bit_cast(bf16x8, (u32x4){w[4 * ks2], w[4 * ks2 + 1], w[4 * ks2 + 2], w[4 * ks2 + 3]});
        out[o][ob] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[f % (kPF + 1)], pb, out[o][ob], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = j * W::kScores2; e < (j + 1) * W::kScores2; ++e) feed(sacc[P][e], pacc[P][e], e < 2 ? P ^ 1 : P, e < 2 ? 14 + e : e - 2);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < kPF; ++i) fr[i] = nfr[i];
    {
      const int delta = tr_next - tr_off;
      tr_off = tr_next;
#pragma unroll
      for (int i = 0; i < 2 * kBlocks; ++i) taddr[i] += delta;
      load_stage = load_stage == kStages - 1 ? 0 : load_stage + 1;
    }
    if constexpr (DBIAS) {
      if (yt_m1 != kNoTile) dist_tile(dsv[P ^ 1], yt_m1);
    }
    yt_m1 = yt0; yt0 = yt1; yt1 = yt2; yt2 = cur.yt;
    wait_loads<W::kLoads>();                                            // the loads of the step before have landed
    __syncthreads();
  };
  // A wave past the end of the sequence only does its share of the loads, step for step with the others (wave-uniform).  64 sequences of 129-150 tokens,
  // 8 heads of 32: backward 41.3 -> 39.3 us; of 1-400, 4 heads of 64: 49.3 -> 47.8; nothing on long ones.
  if (xw0 >= L) {
#pragma unroll 1
    for (int s = 0; s <= n; ++s) {
      cur = next_src(cur, s + 3);
#pragma unroll
      for (int what = 0; what < W::kLoads; ++what) load(cur, what, (uint32_t)(load_stage * W::kStage), (s + 3) & (kStripStages - 1));
      load_stage = load_stage == kStages - 1 ? 0 : load_stage + 1;
      wait_loads<W::kLoads>();
      __syncthreads();
    }
    wait_loads<0>();
    return;
  }
  // steps whose seeded tile has no candidate, in pairs; then the rest (tiles with candidates and the step that drains the last one)
  int s = 0;
  for (; s + 2 < nfast; s += 2) {
    step(s, IC<0>{}, std::false_type{});
    step(s + 1, IC<1>{}, std::false_type{});
  }
  for (; s <= n; s += 2) {
    step(s, IC<0>{}, std::bool_constant<CAND>{});
    if (s + 1 > n) break;
    step(s + 1, IC<1>{}, std::bool_constant<CAND>{});
  }
  if constexpr (DBIAS) dist.flush();
  wait_loads<0>();                                                      // nothing may still be landing in LDS when the wave ends

  // ---- epilogue.  Lane x holds features 32 ob + 8 (r / 4) + 4 hf + r % 4.
  if (item.slot >= 0) {                                                 // a piece of a cut block: raw sums, finish_kernel adds them up
    float* dst = a.partial + ((int64_t)item.slot * kOut * kBX + (wave * 32 + l32)) * D;
#pragma unroll
    for (int o = 0; o < kOut; ++o)
#pragma unroll
      for (int ob = 0; ob < kBlocks; ++ob)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *(f32x4*)(dst + (int64_t)o * kBX * D + ob * 32 + 8 * q4 + 4 * hf) =
              (f32x4){out[o][ob][4 * q4 + 0], out[o][ob][4 * q4 + 1], out[o][ob][4 * q4 + 2], out[o][ob][4 * q4 + 3]};
    return;
  }
  if (!x_ok) return;
#pragma unroll
  for (int o = 0; o < kOut; ++o) {
    const float scale = a.inv_n * (o == 0 ? a.alpha : kLn2);
    const int64_t sd = MODE == kDQ ? a.sq : (o == 0 ? a.sk : a.sv);
    __bf16* dst = (__bf16*)(MODE == kDQ ? a.dq : (o == 0 ? a.dk : a.dv)) + (int64_t)(seq0 + x) * sd + hoff;
    const __bf16* pre = (const __bf16*)(MODE == kDQ ? a.pre_q : (o == 0 ? a.pre_k : a.pre_v));      // the operand was SiLU(pre): hand back the gradient of pre
    if (pre) pre += (int64_t)(seq0 + x) * a.s_pre + hoff;
#pragma unroll
    for (int ob = 0; ob < kBlocks; ++ob)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int f = ob * 32 + 8 * q4 + 4 * hf;
        float v0 = out[o][ob][4 * q4 + 0] * scale, v1 = out[o][ob][4 * q4 + 1] * scale;
        float v2 = out[o][ob][4 * q4 + 2] * scale, v3 = out[o][ob][4 * q4 + 3] * scale;
        if (pre) {
          const u32x2 t = *(const u32x2*)(pre + f);
          v0 *= dsilu(__uint_as_float(t[0] << 16)); v1 *= dsilu(__uint_as_float(t[0] & 0xFFFF0000u));
          v2 *= dsilu(__uint_as_float(t[1] << 16)); v3 *= dsilu(__uint_as_float(t[1] & 0xFFFF0000u));
        }
        *(u32x2*)(dst + f) = (u32x2){pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
      }
  }
}

template <int D, int MODE, bool CAND, bool DBIAS>
hipError_t launch_one(const AttnArgs& a, hipStream_t stream) {
  auto kern = attn_bwd_narrow_kernel<D, MODE, CAND, DBIAS>;
  constexpr int smem_bytes = Narrow<D, MODE>::kSmemBytes;
  static_assert(smem_bytes <= 80 * 1024, "two workgroups share a compute unit");
  if constexpr (smem_bytes > 64 * 1024) {                                // beyond the default limit
    static bool attr_set[64] = {};                                       // per instantiation and device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    if (dev < 0 || dev >= 64 || !attr_set[dev]) {
      const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes);
      if (e != hipSuccess) return e;
      if (dev >= 0 && dev < 64) attr_set[dev] = true;
    }
  }
  const int per = kNumXcd * kXcdGroup;
  const int grid = (a.max_items + per - 1) / per * per;
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), smem_bytes, stream, a);
  return hipGetLastError();
}

template <int D>
hipError_t launch_width(const AttnArgs& a, bool key_blocks, hipStream_t stream) {
  if (key_blocks) return a.num_targets ? launch_one<D, kDKDV, true, false>(a, stream) : launch_one<D, kDKDV, false, false>(a, stream);
  if (a.dbias_dist) return a.num_targets ? launch_one<D, kDQ, true, true>(a, stream) : launch_one<D, kDQ, false, true>(a, stream);
  return a.num_targets ? launch_one<D, kDQ, true, false>(a, stream) : launch_one<D, kDQ, false, false>(a, stream);
}

}  // namespace

hipError_t launch_attn_bwd_narrow(const AttnArgs& a, bool key_blocks, hipStream_t stream) {
  if (!a.seed || !a.seed_up) return hipErrorInvalidValue;
  switch (a.D) {
    case 32: return launch_width<32>(a, key_blocks, stream);
    case 64: return launch_width<64>(a, key_blocks, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace hstu
