// dQ of the attention backward as one matrix product over the dS that the dK/dV pass has left in memory (bf16, 128 features):
//   dQ^T[feature][query] += K^T[feature][key] dS^T[key][query]
// over the tile lists of the dQ pass (128-query blocks, 64-key tiles, pieces of cut blocks as there).  A backward whose two passes are
// independent executes seven products per tile, S and dP twice, and the pointwise work twice; with dS handed on it is five and one.
//
// dS comes in tiles of 32 queries x 128 keys (8 KB), those of one key block consecutive by query (AttnArgs::ds_table).  A tile is four 2 KB
// parts, one per wave of the dK/dV pass (32 keys), a part two 1 KB halves (16 queries each) of 64 16-byte slots: slot
// 32 hi + (key ^ 8 hi ^ 4 half) holds queries 16 half + 4 hi + {0..3} and 8 further, as that pass has them in registers.  The transpose
// loads here turn them into a B operand with keys on the k-slots; the XOR keeps the 16 slots that half a wave reads in different banks.
// Every pair of a tile that the dK/dV pass visits is written (masked ones as zero); a query tile outside a key block's list is skipped.
//
// What bounds it: reading dS once (2 bytes a pair).  8 sequences of 8k-16k tokens, 4 heads, dense (4.2 GB): 0.86 ms, 4.8 TB/s, where the dQ
// pass that recomputes S and dP takes 1.52; 1024 + 256 semi-local 0.24 against 0.39.  Storing dS costs the dK/dV pass 8 % (1.95 -> 2.12 ms),
// a fifth of that the traffic.  Both sides bypass the caches' replacement (nt): K stays in the L2 (0.97 ms without).  Three to five stages of
// 32 keys with 80-96 KB in flight per compute unit measure the same as two of 64 keys.
#include "hstu_common.h"
#include "hstu_kernels.h"

namespace hstu {
namespace {

constexpr int kBX = 128, kBN = 64, kD = 128, kWaves = 4;
constexpr int kTileK = kBN * kD * 2, kTileDs = kBX * kBN * 2, kStage = kTileK + kTileDs;
constexpr int kSmem = 2 * kStage;

__global__ __launch_bounds__(64 * kWaves, 2) void attn_dq_kernel(const AttnArgs a) {
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  typedef __attribute__((address_space(3))) void* lds_void;
  typedef __attribute__((address_space(3))) short4v* lds_s4;
  typedef const __attribute__((address_space(4))) i32x4* const_i4;
  const int wg = blockIdx.x;
  const int xcd = wg % kNumXcd, slot = wg / kNumXcd;
  const int pos = ((slot / kXcdGroup) * kNumXcd + xcd) * kXcdGroup + slot % kXcdGroup;
  const int count = a.header->count;
  const WorkItem item = a.items[min(pos, a.max_items - 1)];
  if (!ds_fits(a.ds_lists[1], a.ds_cap)) {                 // the dK/dV pass has left nothing: neither list has anything to finish
    if (wg == 0 && threadIdx.x == 0) {
      for (SchedHeader* const list : {a.ds_lists[0], a.ds_lists[1]}) {
        list->count = 0;
        list->splits = 0;
        list->bad_batch = 1;
      }
    }
    return;
  }
  if (pos >= count) return;
  const int xb = item.rb_h >> 8, h = item.rb_h & 255, seq0 = item.seq0, L = item.len;
  const SeqGeom g = {L, item.hist, a.K1, a.K2};
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5, l32 = lane & 31, grp16 = lane >> 4, i16 = lane & 15;
  const int x0 = xb * kBX, x = x0 + wave * 32 + l32, qt = (x0 >> 5) + wave;

  const TileRanges tr = tile_ranges(g, x0, min(x0 + kBX, L) - 1, kBN);
  const int t_begin = item.t0, ntiles = min(tr.count(), item.t1);
  const int last_pair = __builtin_amdgcn_readfirstlane(a.ds_pair0[item.b]) + (L - 1) / kBX;            // of key block 0
  const_i4 table = (const_i4)(uintptr_t)a.ds_table;
  const __bf16* K = (const __bf16*)a.k + (int64_t)seq0 * a.sk + (int64_t)h * kD;
  const uint32_t rowb = (uint32_t)(a.sk * 2);
  const uint32_t k_voff = __umul24((uint32_t)grp16, rowb) + (uint32_t)(16 * (i16 ^ (4 * grp16 + wave)));
  const uint32_t ds_voff = (uint32_t)lane * 16;
  auto dma16 = [&](uint64_t addr, uint32_t bytes, uint32_t voff, uint32_t dst) {
    const i32x4 rs = {(int)(uint32_t)addr, (int)(uint32_t)(addr >> 32), (int)bytes, 0x00020000};
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(voff), "s"(rs) : "memory", "m0");
  };
  auto dma16_nt = [&](uint64_t addr, uint32_t bytes, uint32_t voff, uint32_t dst) {
    const i32x4 rs = {(int)(uint32_t)addr, (int)(uint32_t)(addr >> 32), (int)bytes, 0x00020000};
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" :: "s"(dst), "v"(voff), "s"(rs) : "memory", "m0");
  };
  auto entry_of = [&](int yt) -> i32x4 { return table[last_pair - (yt >> 1)]; };
  // (a 32 x 64 block without a visible pair holds zeros, where it was written: neither read nor multiplied)
  auto has_ds = [&](int yt, const i32x4& e) {
    return qt >= e[1] && qt < e[1] + e[2] && classify_tile(g, 32 * qt, 32 * qt + 31, yt * kBN, yt * kBN + kBN - 1) != kTileEmpty;
  };
  // loads of key tile yt (its table entry: e) into LDS stage s; some: has_ds()
  auto issue = [&](int yt, const i32x4& e, bool some, int s) {
    const uint32_t dst0 = (uint32_t)(uintptr_t)(lds_void)(smem + s * kStage);
    const uint64_t ds = (uint64_t)(uintptr_t)a.ds + (uint64_t)(uint32_t)(e[0] + h * e[2] + qt - e[1]) * kDsTileBytes + (yt & 1) * (kDsTileBytes / 2);
    const uint32_t ds_bytes = some ? kDsTileBytes / 2 : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) dma16_nt(ds, ds_bytes, ds_voff + 1024 * j, dst0 + kTileK + wave * (kTileDs / 4) + 1024 * j);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int row = yt * kBN + 4 * (4 * c + wave);
      dma16((uint64_t)(uintptr_t)K + (uint64_t)(uint32_t)row * rowb, (uint32_t)max(L - row, 0) * rowb, k_voff, dst0 + (4 * c + wave) * 1024);
    }
  };

  f32x16 out[4];
#pragma unroll
  for (int ob = 0; ob < 4; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) out[ob][r] = 0.f;

  const int vchunk = 2 * (grp16 & 1) + ((i16 & 3) >> 1), vbyte = 8 * (i16 & 1);
  const int tb0 = (int)(uint32_t)(uintptr_t)(lds_void)smem + (4 * hf + (i16 >> 2)) * 256 + ((i16 >> 2) << 6) + ((vchunk ^ hf) << 4) + vbyte;
  const int q1 = grp16 & 1, c4 = i16 & 3;
  const int db0 = (int)(uint32_t)(uintptr_t)(lds_void)smem + kTileK + wave * (kTileDs / 4) + q1 * 1024 + (c4 & 1) * 640 + ((hf ^ q1) << 6) + (i16 >> 2) * 16 + (c4 >> 1) * 8;

  i32x4 e = {0, 0, 0, 0}, e_next = {0, 0, 0, 0};
  int yt_next = 0;
  bool some = false;
  if (t_begin < ntiles) {
    const int yt = tr.at(t_begin);
    e = entry_of(yt);
    some = has_ds(yt, e);
    issue(yt, e, some, 0);
    yt_next = tr.at(min(t_begin + 1, ntiles - 1));
    e_next = entry_of(yt_next);
  }
  for (int t = t_begin; t < ntiles; ++t) {
    const int s = (t - t_begin) & 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's loads of tile t have landed; the barrier publishes them
    __syncthreads();
    const bool mine = some;
    e = e_next;
    if (t + 1 < ntiles) {
      some = has_ds(yt_next, e);
      issue(yt_next, e, some, s ^ 1);
      yt_next = tr.at(min(t + 2, ntiles - 1));
      e_next = entry_of(yt_next);
    }
    if (!mine) continue;
    int tb = tb0 + s * kStage, db = db0 + s * kStage;
    asm volatile("" : "+v"(tb), "+v"(db));
    auto pair = [&](int lo_at, int hi_at) -> bf16x8 {
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(uint32_t)lo_at);
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(uint32_t)hi_at);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto dsfrag = [&](int k) -> bf16x8 {                    // keys [16 k, 16 k + 16) of the tile
      const int at = (k >> 1) * 2048 + (k & 1) * 256;
      return pair(db + at, (db ^ 128) + at);
    };
    auto kfrag = [&](int k, int ob) -> bf16x8 { return pair((tb ^ (ob << 6)) + k * 4096, (tb ^ ((ob << 6) | 32)) + k * 4096 + 2048); };
    constexpr int PF = 4;                                  // fragments are fetched PF products ahead
    bf16x8 fr[PF], fd[2];
    fd[0] = dsfrag(0);
#pragma unroll
    for (int i = 0; i < PF; ++i) fr[i] = kfrag(i >> 2, i & 3);
#pragma unroll
    for (int n = 0; n < 16; ++n) {
      const bf16x8 fa = fr[n % PF];
      if (n % 4 == 0 && n + 4 < 16) fd[((n >> 2) + 1) & 1] = dsfrag((n >> 2) + 1);
      if (n + PF < 16) fr[n % PF] = kfrag((n + PF) >> 2, (n + PF) & 3);
      __builtin_amdgcn_sched_barrier(0);
      out[n & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fd[(n >> 2) & 1], out[n & 3], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  if (item.slot >= 0) {                                    // a piece: raw sums to its slot, finish_kernel adds them up
    float* dst = a.partial + ((int64_t)item.slot * kBX + (wave * 32 + l32)) * kD;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *(f32x4*)(dst + ob * 32 + 8 * q4 + 4 * hf) = (f32x4){out[ob][4 * q4], out[ob][4 * q4 + 1], out[ob][4 * q4 + 2], out[ob][4 * q4 + 3]};
    return;
  }
  if (x >= L) return;
  const float scale = a.inv_n * a.alpha;
  __bf16* dst = (__bf16*)a.dq + (int64_t)(seq0 + x) * a.sq + (int64_t)h * kD;
  const __bf16* pre = (const __bf16*)a.pre_q;              // the operand was SiLU(pre): hand back the gradient of pre
  if (pre) pre += (int64_t)(seq0 + x) * a.s_pre + (int64_t)h * kD;
#pragma unroll
  for (int ob = 0; ob < 4; ++ob)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int f = ob * 32 + 8 * q4 + 4 * hf;
      float v0 = out[ob][4 * q4] * scale, v1 = out[ob][4 * q4 + 1] * scale, v2 = out[ob][4 * q4 + 2] * scale, v3 = out[ob][4 * q4 + 3] * scale;
      if (pre) {
        const u32x2 t = *(const u32x2*)(pre + f);
        v0 *= dsilu(__uint_as_float(t[0] << 16)); v1 *= dsilu(__uint_as_float(t[0] & 0xFFFF0000u));
        v2 *= dsilu(__uint_as_float(t[1] << 16)); v3 *= dsilu(__uint_as_float(t[1] & 0xFFFF0000u));
      }
      *(u32x2*)(dst + f) = (u32x2){pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
    }
}

}  // namespace

hipError_t launch_attn_dq_from_ds(const AttnArgs& a, hipStream_t stream) {
  static bool attr_set[64] = {};                                         // per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
  if (dev < 0 || dev >= 64 || !attr_set[dev]) {
    const hipError_t e = hipFuncSetAttribute((const void*)attn_dq_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kSmem);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) attr_set[dev] = true;
  }
  const int per = kNumXcd * kXcdGroup;
  const int grid = (a.max_items + per - 1) / per * per;
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(attn_dq_kernel, dim3(grid), dim3(64 * kWaves), kSmem, stream, a);
  return hipGetLastError();
}

}  // namespace hstu
