// Host-side brute-force check of the tile enumeration and classification in hstu_geometry.h
// (the very header the kernels compile).  Built with the host compiler by the CPU test suite.
//   geometry_check(L, M, K1, K2, block_rows, BN) returns 0 when, for one sequence,
//   - every visible (query, key) pair falls in a tile enumerated for its row block (forward / dQ
//     orientation) and for its key block (dK/dV orientation), the ranges are ascending and disjoint,
//   - every enumerated tile holds at least one visible pair (no fully masked tile is scheduled),
//   - classify_tile says Full only if all pairs of the 32x32 block are visible history pairs with
//     distance i - j, and Empty only if none is visible;
//   - the tiles of 32 that key_tiles_of() and query_tiles_of() call full hold only visible pairs with history keys (of existing rows), run by run, and
//     classify_tile()'s full ones are among them; those that they call empty hold none, and classify_tile()'s empty ones of history rows are among them;
//   otherwise a non-zero code naming the violated property.
//   plan_check(...) does the same for the bounds of hstu_plan.h on one batch: the room for dS holds the tiles of the dK/dV list, with the
//   host copy of the offsets and without it; the query tiles of a key block are consecutive (the dQ product addresses dS by that); and a
//   list in which the scheduler cuts a block is one that schedule_may_cut() names, and where the lengths say it all no other list is.
#include <vector>

#include "hstu_geometry.h"
#include "gemm_tiles.h"
#include "hstu_plan.h"

using namespace hstu;

static int check_ranges(const TileRanges& t) {
  if (t.a0 > t.a1 || t.b0 > t.b1 || t.c0 > t.c1) return 1;
  if (t.a1 > t.b0 && t.b1 > t.b0) return 1;
  if ((t.b1 > t.c0 || t.a1 > t.c0) && t.c1 > t.c0) return 1;
  return 0;
}

extern "C" int geometry_check(int L, int M, int K1, int K2, int block_rows, int BN) {
  const SeqGeom g = {L, L - M, K1, K2};
  const int ntile = (L + BN - 1) / BN;
  for (int orient = 0; orient < 2; ++orient) {
    for (int r0 = 0; r0 < L; r0 += block_rows) {
      const int r1 = imin(r0 + block_rows, L) - 1;
      const TileRanges t = orient == 0 ? tile_ranges(g, r0, r1, BN) : row_tile_ranges(g, r0, r1, BN);
      if (check_ranges(t)) return 10 + orient;
      std::vector<int> listed(ntile + 2, 0), needed(ntile + 2, 0);
      for (int idx = 0; idx < t.count(); ++idx) {
        const int yt = t.at(idx);
        if (yt < 0 || yt >= ntile) return 20 + orient;
        if (listed[yt]) return 30 + orient;
        listed[yt] = 1;
        if (idx > 0 && yt <= t.at(idx - 1)) return 40 + orient;
      }
      for (int x = r0; x <= r1; ++x)
        for (int y = 0; y < L; ++y) {
          int delta;
          const bool vis = orient == 0 ? visible(g, x, y, delta) : visible(g, y, x, delta);
          if (vis) needed[y / BN] = 1;
        }
      for (int yt = 0; yt < ntile; ++yt) {
        if (needed[yt] && !listed[yt]) return 50 + orient;     // a visible pair would be skipped
        if (listed[yt] && !needed[yt]) return 60 + orient;     // a fully masked tile is scheduled
      }
    }
  }
  // classification of 32 x 32 blocks (rows beyond L included, as the kernels see them)
  const int lim = (L + 63) / 32 * 32;
  for (int q0 = 0; q0 < lim; q0 += 32)
    for (int k0 = 0; k0 < lim; k0 += 32) {
      const int kind = classify_tile(g, q0, q0 + 31, k0, k0 + 31);
      int nvis = 0, nbad = 0;
      for (int i = q0; i < q0 + 32; ++i)
        for (int j = k0; j < k0 + 32; ++j) {
          int delta = 0;
          const bool vis = visible(g, i, j, delta);
          nvis += vis;
          const int p = i < g.n ? i : g.n;                       // a candidate row stands at position n
          if (!vis || delta != p - j || i >= L || j >= L) ++nbad;
        }
      if (kind == kTileFull && nbad) return 70;
      if (kind == kTileEmpty && nvis) return 80;
    }
  for (int w0 = 0; w0 < L; w0 += 32)
    for (int keys = 0; keys < 2; ++keys) {                   // tiles of keys for query rows w0 .., or of queries for keys w0 ..
      const WaveTiles t = keys ? key_tiles_of(g, w0) : query_tiles_of(g, w0);
      std::vector<int> full(lim / 32 + 1, 0);
      for (int yt = 0; yt < lim / 32; ++yt) {
        const int y0 = 32 * yt;
        bool any = false;
        full[yt] = 1;
        for (int x = w0; x < w0 + 32 && x < L; ++x)
          for (int y = y0; y < y0 + 32; ++y) {
            int delta;
            const int i = keys ? x : y, j = keys ? y : x;
            const bool vis = visible(g, i, j, delta);
            any |= vis;
            if (j >= g.n || (!keys && i >= g.n) || !vis) full[yt] = 0;
          }
        const int kind = keys ? classify_tile(g, w0, w0 + 31, y0, y0 + 31) : classify_tile(g, y0, y0 + 31, w0, w0 + 31, false);
        if (kind == kTileFull && t.full_end(yt) <= yt) return 90 + keys;
        if (t.empty(yt) && any) return 92 + keys;
        const bool history = keys ? imin(w0 + 31, L - 1) < g.n : y0 + 31 < g.n && w0 + 31 < g.n;
        if (history && kind == kTileEmpty && !t.empty(yt)) return 94 + keys;
      }
      for (int yt = 0; yt < lim / 32; ++yt)
        for (int f = yt; f < t.full_end(yt); ++f)
          if (f >= lim / 32 || !full[f]) return 96 + keys;
    }
  return 0;
}

// What the scheduler makes of one list (which: 0 forward, 1 dQ, 2 dK/dV): the blocks' costs in natural order (first sequence first, a sequence's last block first), and in
// out[]: whether blocks are cut, the first and the last piece size, the partial-sum slots, the blocks of all heads that are cut.  Returns the number of blocks of one head.
struct PlannedList { bool cut; int64_t first, chunk, slots, split; };
static PlannedList planned(const std::vector<int>& costs, int64_t rows_over_128_and_batch, int H, int which, bool tail, bool candidates, bool fp32, int D) {
  const CutRule rule = cut_rule_for(fp32, D, which, tail);
  int64_t all = 0;
  int most = 0;
  for (int c : costs) { all += (int64_t)c * H; most = imax(most, c); }
  const bool many = candidates && (int64_t)costs.size() * H >= kManyBlocks;
  const int launch = candidates && !many ? 0 : rule.launch, least = 2 * rule.min_chunk + rule.launch * (many ? kUnsure : 1);
  const int64_t first = std::max((int64_t)rule.min_chunk, (int64_t)std::ceil((double)all * (1.0 / rule.target_chunks)));
  const int64_t cap = slot_cap_for(rows_over_128_and_batch * H, fp32);
  PlannedList l = {false, first, first, 0, 0};
  while (most > worth_cutting((int)l.chunk, fp32) + launch && most > least) {              // the piece size grows until the slots fit
    const int64_t piece = tail || (fp32 && which == 2) ? l.chunk : 2 * l.chunk;
    l.slots = l.split = 0;
    for (int c : costs)
      if (c > 2 * l.chunk) { l.slots += (c + piece - 1) / piece * H; l.split += H; }
    if (l.slots <= cap) {
      l.cut = most > worth_cutting((int)l.chunk, fp32) + launch + l.slots / rule.slots_per_tile;
      break;
    }
    l.chunk += 4 * l.slots <= (tail ? 5 : 6) * cap ? std::max(l.chunk / 4, (int64_t)1) : l.chunk;
  }
  return l;
}
extern "C" int planned_list(int B, const int32_t* lengths, const int32_t* targets, int H, int K1, int K2, int which, int tile, int fp32, int D, int32_t* costs_out, int64_t* out) {
  std::vector<int> costs;
  int64_t rows = 0;
  for (int b = 0; b < B; ++b) {
    const SeqGeom g = {lengths[b], lengths[b] - (targets ? targets[b] : 0), K1, K2};
    rows += g.L;
    for (int r0 = (g.L - 1) / 128 * 128; g.L > 0 && r0 >= 0; r0 -= 128) {
      const int r1 = imin(r0 + 128, g.L) - 1;
      costs.push_back((which == 2 ? row_tile_ranges(g, r0, r1, tile) : tile_ranges(g, r0, r1, tile)).count());
    }
  }
  const PlannedList l = planned(costs, rows / 128 + B, H, which, false, targets != nullptr, fp32 != 0, D);
  for (size_t i = 0; costs_out && i < costs.size(); ++i) costs_out[i] = costs[i];
  out[0] = l.cut; out[1] = l.first; out[2] = l.chunk; out[3] = l.slots; out[4] = l.split;
  return (int)costs.size();
}

// targets: nullptr or the candidates of every sequence; slack: by how much max_seqlen exceeds the longest one
extern "C" int plan_check(int B, const int32_t* lengths, const int32_t* targets, int H, int K1, int K2, int query_tail, int slack) {
  std::vector<int32_t> offsets(B + 1, 0);
  int longest = 0;
  for (int b = 0; b < B; ++b) {
    offsets[b + 1] = offsets[b] + lengths[b];
    longest = imax(longest, lengths[b]);
  }
  const PlanBatch with = {B, H, offsets[B], longest + slack, K1, K2, targets != nullptr, offsets.data()};
  PlanBatch without = with;
  without.host_offsets = nullptr;
  auto geom = [&](int b) { return SeqGeom{lengths[b], lengths[b] - (targets ? targets[b] : 0), K1, K2}; };

  int64_t ds = 0;
  for (int b = 0; b < B; ++b)
    for (int k0 = 0; k0 < lengths[b]; k0 += 128) {
      const TileRanges t = row_tile_ranges(geom(b), k0, imin(k0 + 128, lengths[b]) - 1, 32);
      for (int i = 1; i < t.count(); ++i)
        if (t.at(i) != t.at(0) + i) return 1;
      ds += (int64_t)t.count() * H;
    }
  if (ds > ds_tiles_bound(with)) return 2;
  if (ds > ds_tiles_bound(without)) return 3;

  for (int which = 0; which < 3; ++which)
    for (int tile = 32; tile <= 64; tile += 32) {
      const int tail = which == 0 ? query_tail : 0;
      std::vector<int> costs;
      for (int b = 0; b < B; ++b) {
        const SeqGeom g = geom(b);
        for (int r0 = tail_origin(g.n, tail); r0 < g.L; r0 += 128) {
          const int r1 = imin(r0 + 128, g.L) - 1;
          costs.push_back((which == 2 ? row_tile_ranges(g, r0, r1, tile) : tile_ranges(g, r0, r1, tile)).count());
        }
      }
      for (int rule_of = 0; rule_of < 6; ++rule_of) {      // bf16 and fp32 with 32, 64 and 128 features
        const bool fp32 = rule_of >= 3;
        const int D = 32 << rule_of % 3;
        const bool cut = planned(costs, (int64_t)offsets[B] / 128 + B, H, which, tail > 0, targets != nullptr, fp32, D).cut;
        if (cut && !schedule_may_cut(with, tail, which, 128, tile, fp32, D)) return 10 + which;
        if (cut && !schedule_may_cut(without, tail, which, 128, tile, fp32, D)) return 20 + which;
        if (!cut && !targets && tail == 0 && costs.size() <= 1024 && schedule_may_cut(with, tail, which, 128, tile, fp32, D))
          return 30 + which;                               // the launch that adds pieces up, for a list that is not cut
      }
    }
  return 0;
}

// The tile of a product over token rows, by gemm_rows.hip's own rule: kTile64Deep .. kTile256 (fp8: kTile64, kTile128, kTile192)
extern "C" int product_tile(long long M, int N, long long K, int residual, int fp8) {
  return fp8 ? fp8_tile(M, N, residual != 0) : gemm_rows_tile(M, N, K, residual != 0);
}
