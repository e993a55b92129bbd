// Host arithmetic that a launch is planned with before the device has seen the offsets: bounds on what the scheduler will make of a batch.
// Plain C++ on plain values, so that the host-side check of the tiling logic compiles the same header.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "hstu_geometry.h"

namespace hstu {

// How a list is cut: blocks of more than 2 x chunk tiles are, into equal pieces of at most that (fp32 key blocks and the forward over a query tail:
// into pieces of chunk); chunk = 1 / target of all tiles, at least min_chunk, and as much more as the partial-sum slots ask for.  A list is cut only
// if its longest block has more than 2 x chunk + launch + slots / slots_per_tile tiles.  which: 0 forward, 1 dQ list, 2 dK/dV list.
//
// It is the work of a compute unit, not of a workgroup slot on it, that a long block has to exceed before cutting gains anything: the other workgroups
// there end, and it goes on at nearly the full rate of the unit.  Cutting costs the launch that adds pieces up, 5 us, and the traffic of the slots.
// Timed with and without cuts on 1,560 batches (64 to 70,000 rows, all widths, types and masks), cut - uncut is within a few percent of the time
//   5 us + b x slots - t x (longest block - max(longest piece, f x all tiles / 256)),  in us
//     bf16, 128 features: b .024 t .55 (forward), .039 .81 (dQ, 64-key tiles), .050 1.13 (dK/dV);  64: .013 .54, .015 .56, .032 .76;
//     32: .005 .47, .001 .48, .017 .64;  f .6-.8
//     fp32, 128: .031 4.7, .034 6.5, .072 8.8;  64: .012 2.7, .010 3.5, .055 4.6;  32: .010 1.7, .000 2.1, .033 2.8;  f .7-1.5
// launch and slots_per_tile follow from these; bf16 targets put a piece at .46 (forward) or .7 of a unit's share, fp32 ones at one share (a workgroup or two fill a
// unit).  The rule before (a slot's share; bf16 lists of many blocks uncut up to 60, 20 or 24 tiles more; fp32 from a few tiles on) did not ask how many slots there
// would be: 32 x 1,000 tokens, one head of 128, 256 + 64 semi-local, backward 68 -> 60 us; the forward of 2 x 1,365-3,018, 8 heads of 64, 41 -> 33; of 4 x 900, 8 heads of 64
// in fp32 69 -> 55.  Over those batches, geometric mean: bf16 forward 1.02-1.03, backward 1.01-1.02, fp32 1.00-1.03 times as fast; single ones from 9 % slower (forward
// of 10 x 1,894-4,048 129 -> 141) to 25 % faster.
struct CutRule { int target_chunks, min_chunk, launch, slots_per_tile; };
// (in fp32 with a quarter more than 2 x chunk)
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int worth_cutting(int chunk, bool fp32) { return 2 * chunk + (fp32 ? chunk / 2 : 0); }
// With candidates the host cannot tell whether a list will be cut, and the launch that adds pieces up follows it in vain: lists of kManyBlocks and more, most of
// which are not, are cut, and named by schedule_may_cut(), for kUnsure times as much.
constexpr int kManyBlocks = 512, kUnsure = 7;
inline CutRule cut_rule_for(bool fp32, int head_dim, int which, bool query_tail) {
  if (fp32) {
    const int launch = which == 0 ? (head_dim == 32 ? 2 : 1) : which == 1 ? (head_dim == 32 ? 2 : 0) : head_dim == 32 ? 1 : 0;
    return {head_dim == 32 ? 1024 : 512, head_dim == 32 ? 2 : 1, launch, which == 2 ? 256 : 128};
  }
  if (query_tail) return {2048, 8, 0, 1 << 30};
  constexpr int launch[3][3] = {{8, 8, 7}, {8, 8, 7}, {9, 5, 5}}, per[3][3] = {{28, 32, 32}, {24, 32, 24}, {20, 24, 22}};
  const int width = head_dim == 32 ? 0 : head_dim == 64 ? 1 : 2;
  return {which == 0 ? 1104 : 732, which == 1 && width == 2 ? 4 : 8, launch[width][which], per[width][which]};
}
// Partial-sum slots of a list of at most `blocks` blocks, under every mask: what the pieces of its cut blocks may take.
inline int slot_cap_for(int64_t blocks, bool fp32) { return (int)std::min((fp32 ? 8 : 2) * blocks, (int64_t)768); }

struct PlanBatch {
  int batch, heads, total_tokens, max_seqlen;
  int K1, K2;                        // of SeqGeom, both below 2^28
  bool candidates;                   // their counts are known on the device only
  const int32_t* host_offsets;       // or nullptr
};

// dS tiles (32 queries x 128 keys) that the dK/dV pass can leave for the dQ product: an upper bound over all heads.  From the host
// copy of the lengths where there is one, else from the longest sequence; candidates can add whole columns for the key blocks that the
// window in front of position n reaches.
inline int64_t ds_tiles_bound(const PlanBatch& p) {
  const int64_t K1 = p.K1, K2 = p.K2;
  const int64_t wide = K1 >= 0 ? (K1 + 158) / 32 : 0, cand_blocks = p.candidates && K1 >= 0 ? K1 / 128 + 2 : 0;
  auto of = [&](int64_t L) -> int64_t {
    const int64_t nq = (L + 31) / 32, nk = (L + 127) / 128;
    const int64_t dense = nk * nq - 2 * nk * (nk - 1);
    if (K1 < 0) return dense;
    const int64_t pre = std::min(nk, (K2 + 127) / 128);
    return std::min(dense, pre * nq - 2 * pre * (pre - 1) + (nk - pre) * wide + std::min(nk, cand_blocks) * nq);
  };
  int64_t tiles = 0;
  if (p.host_offsets) {
    for (int b = 0; b < p.batch; ++b) tiles += of((int64_t)p.host_offsets[b + 1] - p.host_offsets[b]);
  } else {
    const int64_t most = std::min(p.max_seqlen, p.total_tokens), blocks = (int64_t)p.total_tokens / 128 + p.batch;
    const int64_t nq = (most + 31) / 32, nk = (most + 127) / 128;
    tiles = blocks * (2 * nk + 2);
    if (K1 >= 0) tiles = std::min(tiles, p.batch * (std::min(nk, (K2 + 127) / 128) + std::min(nk, cand_blocks)) * nq + blocks * wide);
  }
  return tiles * p.heads;
}

// Most batches are cut nowhere, and a launch that would add up pieces costs 5 us for finding that out.  false: no list that the scheduler can
// build for this problem has a cut block (it stays so for a later call that reuses the list and describes the batch in another way).  First the longest block is
// bounded by the longest sequence and the mask, and the tiles from below by the visible pairs, which takes the lengths: without a host copy of
// the offsets only min_chunk counts, and so it does with candidates (their counts are known on the device only) or a query tail.  Where the
// lengths say it all, the blocks are priced as the scheduler does (10 ns each, on the host; more than 1,024 of them are not worth it).
inline bool schedule_may_cut(const PlanBatch& p, int query_tail, int which, int block_rows, int tile_cols, bool fp32 = false, int head_dim = 128) {
  const bool key_major = which == 2, by_position = !p.candidates && query_tail == 0;
  const CutRule rule = cut_rule_for(fp32, head_dim, which, query_tail > 0);
  const double share = 1.0 / rule.target_chunks;
  double longest = p.max_seqlen, pairs = 0.0;
  long long blocks = 0;
  if (p.host_offsets) {
    longest = 0.0;
    for (int b = 0; b < p.batch; ++b) {
      const double L = p.host_offsets[b + 1] - p.host_offsets[b];
      blocks += (p.host_offsets[b + 1] - p.host_offsets[b] + block_rows - 1) / block_rows;
      longest = L > longest ? L : longest;
      pairs += p.K1 < 0 || L <= p.K1 ? 0.5 * L * L : p.K1 * (L - 0.5 * p.K1);       // (those of a global prefix left out)
    }
  }
  double most = std::ceil(longest / tile_cols);          // tiles of the longest block
  if (p.K1 >= 0 && by_position && !(key_major && p.K2 > 0)) {
    const double band = std::floor((double)(block_rows + p.K1) / tile_cols) + 2, prefix = key_major ? 0 : std::ceil((double)p.K2 / tile_cols);
    if (band + prefix < most) most = band + prefix;
  }
  double chunk = rule.min_chunk;
  if (by_position) {
    const double tiles = std::ceil(share * pairs * p.heads / ((double)block_rows * tile_cols) * (1 - 1e-9));
    if (tiles > chunk) chunk = tiles;
  }
  if (most <= 2 * chunk + rule.launch * (p.candidates && query_tail == 0 && blocks * p.heads >= kManyBlocks ? kUnsure : 1)) return false;      // (a tail has fewer blocks)
  if (!by_position || !p.host_offsets || blocks > 1024) return true;
  const TileShift tile = {31 - __builtin_clz((unsigned)tile_cols)};
  int cost[1024], count = 0, max_cost = 0;
  long long all = 0;
  for (int b = 0; b < p.batch; ++b) {
    const int L = p.host_offsets[b + 1] - p.host_offsets[b];
    const SeqGeom g = {L, L, p.K1, p.K2};
    for (int r0 = 0; r0 < L; r0 += block_rows) {
      const int r1 = imin(r0 + block_rows, L) - 1;
      const int c = (key_major ? row_tile_ranges_of(g, r0, r1, tile) : tile_ranges_of(g, r0, r1, tile)).count();
      cost[count++] = c;
      all += c;
      max_cost = imax(max_cost, c);
    }
  }
  int piece = (int)std::max((double)rule.min_chunk, std::ceil((double)(all * p.heads) * share));
  const long long cap = slot_cap_for(((int64_t)p.total_tokens / block_rows + p.batch) * p.heads, fp32);
  while (max_cost > worth_cutting(piece, fp32) + rule.launch) {            // as the scheduler does: pieces grow until the slots fit
    const int most_tiles = fp32 && key_major ? piece : 2 * piece;
    long long slots = 0;
    for (int i = 0; i < count; ++i)
      if (cost[i] > 2 * piece) slots += (cost[i] + most_tiles - 1) / most_tiles;
    slots *= p.heads;
    if (slots <= cap) return max_cost > worth_cutting(piece, fp32) + rule.launch + slots / rule.slots_per_tile;
    piece += 2 * slots <= 3 * cap ? std::max(piece >> 2, 1) : piece;
  }
  return false;
}

}  // namespace hstu
