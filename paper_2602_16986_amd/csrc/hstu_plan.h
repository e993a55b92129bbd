// Host arithmetic that a launch is planned with before the device has seen the offsets: bounds on what the scheduler will make of a batch.
// Plain C++ on plain values, so that the host-side check of the tiling logic compiles the same header.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace hstu {

constexpr int kMinChunk = 8;         // a long block is cut into pieces of at least this many tiles ...
constexpr int kTailTargetChunks = 2048;  // forward over a query tail: ... and of about 1/2048 of all scheduled tiles
constexpr int kFwdTargetChunks = 1536;   // forward: 2 x chunk = one slot's share when 768 workgroups are resident
constexpr int kBwdTargetChunks = 1024;   // backward: the same with 512 resident workgroups

// How a list is cut: blocks of more than 2 x chunk tiles (one slot's share) are, into pieces of at most that (chunk = 1 / target of all tiles, at
// least min_chunk; fp32 key blocks and the forward over a query tail into pieces of chunk).  A list whose longest block has no more than
// longest_uncut tiles, or no more than a share and slack, is not.  which: 0 forward, 1 dQ list, 2 dK/dV list.
// The slack is what cutting costs, 10 us and more for the partial sums of many blocks and the launch that adds them up, in tiles of a
// block that others leave the compute unit to; it counts for lists with a block for every second workgroup slot or more.  Before, lists of nearly equal blocks were cut in two for nothing, and key blocks into pieces of half a
// share.  us before and with it: forward of 8 x 1,024-4,096 semi-local with candidates 72 -> 57, C2 102 -> 97; whole step of 16 x 1,024
// dense 189 -> 177, 10 x 2,048 dense 374 -> 305, one of 6,000 355 -> 298, 24 x 1,024-2,048 semi-local 365 -> 349; with 40 / 12 / 16 and
// 90 / 32 / 40 instead of 60 / 20 / 24 10 x 2,048 takes 342 and 309, 4 x 1,500-4,000 299 and 315 (296).
// In fp32 a tile of 32 rows takes the matrix pipe 1-8 us (64 cycles an instruction, D / 2 of them for a 32 x 32 block of scores), up to
// twice as long as the launch that adds pieces up, and such batches are small, so a block is worth cutting from a few tiles on; 256 workgroups
// are resident (two per compute unit with 32 features).  Whole step, bf16's rule against this one: one sequence of 487 tokens, 7 heads of 128
// features 500 -> 234 us, 4 heads of 64 238 -> 101; 900 tokens, 4 heads of 32 159 -> 86; 8 sequences of 400-1,000, 8 heads: 1-4 % less.  Up to 8 tiles of 32
// features the extra launch costs what the pieces save.
struct CutRule {
  int target_chunks, min_chunk, longest_uncut, slack;
#if defined(__HIPCC__)
  __host__ __device__
#endif
  int slack_of(long long blocks) const { return 4 * blocks >= target_chunks ? slack : 0; }      // target_chunks: twice the slots
};
inline CutRule cut_rule_for(bool fp32, int head_dim, int which, bool query_tail) {
  if (fp32) return head_dim == 32 ? CutRule{1024, 2, 8, 0} : CutRule{512, 1, 2, 0};
  if (query_tail) return {kTailTargetChunks, kMinChunk, 0, 0};
  return which == 0 ? CutRule{kFwdTargetChunks, kMinChunk, 0, 60} : CutRule{kBwdTargetChunks, kMinChunk, 0, which == 1 ? 20 : 24};
}

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

// Most batches are cut nowhere, and a launch that would add up pieces costs 4.5 us for finding that out.  A block is cut
// when it is longer than 2 x chunk, chunk >= min_chunk and >= share x (all tiles).  The longest block is bounded by the longest
// sequence and the mask, the tiles from below by the visible pairs, which takes the lengths: without a host copy of the offsets
// only min_chunk counts, and so it does with candidates (their counts are known on the device only) or a query tail.
// which: 0 forward, 1 dQ list, 2 dK/dV list.  false: no list that the scheduler can build for this problem has a cut block.
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
      blocks += (p.host_offsets[b + 1] - p.host_offsets[b] + block_rows - 1) / block_rows * p.heads;
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
  return most > 2 * chunk + rule.slack_of(blocks) && most > rule.longest_uncut;
}

}  // namespace hstu
