// Integer geometry of the HSTU attention mask: visibility predicate, enumeration of the tiles
// that hold a visible pair, and tile classification.  Plain C++ with no device intrinsics, so
// the same header serves the HIP kernels and a host-side check of the tiling logic.
#pragma once

#if defined(__HIPCC__)
#define HSTU_HD __host__ __device__ __forceinline__
#else
#define HSTU_HD inline
#endif

namespace hstu {

HSTU_HD int imin(int a, int b) { return a < b ? a : b; }
HSTU_HD int imax(int a, int b) { return a > b ? a : b; }

// Geometry of one sequence under the mask of paper Section 4.2.1 (ordinary 0-based
// orientation: query row i sees key j <= i) extended with trailing candidate rows.
struct SeqGeom {
  int L;    // tokens
  int n;    // history tokens, L - num_targets
  int K1;   // local window (< 0: dense causal)
  int K2;   // global prefix
};

// visible(i, j) and the relative-position distance fed to the bias table.
HSTU_HD bool visible(const SeqGeom& g, int i, int j, int& delta) {
  const bool self = (i >= g.n) && (j == i);
  const int p = i < g.n ? i : g.n;
  const bool hist = (j < g.n) && (j <= p) && (g.K1 < 0 || p - j < g.K1 || j < g.K2);
  delta = self ? 0 : p - j;
  return (i < g.L) && (self || hist);
}

// First row of the query blocks of a sequence of which only the last `tail` history rows and the candidates are wanted (tail > 0): the
// blocks start at the 32 rows (a wave's) that hold the first of them.  0: every row is wanted, blocks start at the first one.
HSTU_HD int tail_origin(int hist, int tail) { return tail > 0 ? imax(hist - tail, 0) & ~31 : 0; }

// Column tiles (width BN) that hold at least one visible key for the query rows
// [r0, r1] (inclusive, r1 < L) of one sequence: up to three disjoint ascending
// half-open ranges: the global prefix, the local band, the candidates' own diagonal.
struct TileRanges {
  int a0, a1, b0, b1, c0, c1;
  HSTU_HD int count() const { return (a1 - a0) + (b1 - b0) + (c1 - c0); }
  HSTU_HD int at(int idx) const {
    if (idx < a1 - a0) return a0 + idx;
    idx -= a1 - a0;
    if (idx < b1 - b0) return b0 + idx;
    return c0 + idx - (b1 - b0);
  }
};

// The column tile that holds a column, for a tile width known to the compiler or one that is a power of two (device code that
// takes the width as an argument: a shift instead of the twenty-odd instructions of an integer division).
struct TileWidth {
  int bn;
  HSTU_HD int index(int col) const { return col / bn; }
  HSTU_HD int width() const { return bn; }
};
struct TileShift {
  int shift;
  HSTU_HD int index(int col) const { return col >> shift; }
  HSTU_HD int width() const { return 1 << shift; }
};

template <class W>
HSTU_HD TileRanges tile_ranges_of(const SeqGeom& g, int r0, int r1, const W tile) {
  TileRanges t = {0, 0, 0, 0, 0, 0};
  const bool has_hist = r0 < g.n;
  const bool has_cand = r1 >= g.n;
  const int p_lo = has_hist ? r0 : g.n;                      // smallest effective position
  const int p_hi = has_cand ? g.n : r1;                      // largest effective position
  const int maxkey = imin(p_hi, g.n - 1);                     // last history key any row may see
  int end = 0;
  if (maxkey >= 0) {
    if (g.K1 < 0) {
      t.a1 = tile.index(maxkey) + 1;
      end = t.a1;
    } else {
      const int pre = imin(g.K2, maxkey + 1);                 // prefix keys [0, pre)
      t.a1 = tile.index(pre + tile.width() - 1);
      end = t.a1;
      const int lo = imax(0, p_lo - g.K1 + 1);                // band keys [lo, maxkey]
      if (g.K1 > 0 && lo <= maxkey) {
        t.b0 = imax(tile.index(lo), end);
        t.b1 = imax(tile.index(maxkey) + 1, t.b0);
        end = t.b1;
      }
    }
  }
  if (t.b1 == 0) { t.b0 = t.b1 = end; }
  if (has_cand) {                                            // self pairs of candidate rows
    const int c_lo = imax(r0, g.n);
    t.c0 = imax(tile.index(c_lo), end);
    t.c1 = imax(tile.index(r1) + 1, t.c0);
  } else {
    t.c0 = t.c1 = end;
  }
  return t;
}
HSTU_HD TileRanges tile_ranges(const SeqGeom& g, int r0, int r1, int BN) { return tile_ranges_of(g, r0, r1, TileWidth{BN}); }

// Query-row tiles (height BN) that see at least one key of [k0, k1] (k1 < L): the mirror image of
// tile_ranges(), used by the key-stationary backward pass.
template <class W>
HSTU_HD TileRanges row_tile_ranges_of(const SeqGeom& g, int k0, int k1, const W tile) {
  TileRanges t = {0, 0, 0, 0, 0, 0};
  int end = 0;
  bool cands_see_block = false;
  if (k0 < g.n) {
    const int kh1 = imin(k1, g.n - 1);
    int hi = -1;
    if (g.K1 < 0 || k0 < g.K2) hi = g.n - 1;
    else if (g.K1 > 0) hi = imin(kh1 + g.K1 - 1, g.n - 1);
    if (hi >= k0) {
      t.a0 = tile.index(k0);
      t.a1 = tile.index(hi) + 1;
      end = t.a1;
    }
    cands_see_block = (g.K1 < 0) || (k0 < g.K2) || (g.n - kh1 < g.K1);
  }
  t.b0 = t.b1 = end;
  int c_lo = -1, c_hi = -2;
  if (g.n < g.L && cands_see_block) { c_lo = g.n; c_hi = g.L - 1; }
  else if (k1 >= g.n) { c_lo = imax(k0, g.n); c_hi = k1; }
  if (c_hi >= c_lo) {
    t.c0 = imax(tile.index(c_lo), end);
    t.c1 = imax(tile.index(c_hi) + 1, t.c0);
  } else {
    t.c0 = t.c1 = end;
  }
  return t;
}
HSTU_HD TileRanges row_tile_ranges(const SeqGeom& g, int k0, int k1, int BN) { return row_tile_ranges_of(g, k0, k1, TileWidth{BN}); }

// How a block of query rows [w0, w1] relates to a key tile [j0, j1] (j1 may exceed L-1).
enum TileKind { kTileEmpty = 0, kTileFull = 1, kTilePartial = 2 };

// cand_rows: also recognise blocks of candidate rows (all at position n) against history keys as empty or full; without
// it they are reported as partial (for callers whose fast paths assume the distance i - j).
HSTU_HD int classify_tile(const SeqGeom& g, int w0, int w1, int j0, int j1, bool cand_rows = true) {
  if (w0 >= g.L) return kTileEmpty;
  if (w1 < g.n) {                                            // history rows only, all valid
    if (j0 > w1) return kTileEmpty;
    if (g.K1 >= 0 && w0 - j1 >= g.K1 && j0 >= g.K2) return kTileEmpty;
    if (j1 <= w0 && (g.K1 < 0 || w1 - j0 < g.K1 || j1 < g.K2)) return kTileFull;
  } else if (cand_rows && w0 >= g.n && j1 < g.n) {           // candidate rows only (all at position n), history keys only
    if (g.K1 >= 0 && g.n - j1 >= g.K1 && j0 >= g.K2) return kTileEmpty;
    if (w1 < g.L && (g.K1 < 0 || g.n - j0 < g.K1 || j1 < g.K2)) return kTileFull;
  }
  return kTilePartial;
}

// Of the tiles of 32 that a wave's 32 rows meet: the full ones (all their pairs are visible) and those that may hold a visible pair at all, by number.
struct WaveTiles {
  int full_pre, full_lo, full_hi;                            // full: [0, full_pre) and [full_lo, full_hi)
  int live_pre, live_lo, live_hi, live_end;                  // may be visible: [0, live_pre), [live_lo, live_hi) and from live_end on
  HSTU_HD int full_end(int yt) const { return yt < full_pre ? full_pre : (yt >= full_lo && yt < full_hi ? full_hi : yt); }     // of the run of full tiles yt is in, or yt
  HSTU_HD bool empty(int yt) const { return yt >= live_pre && (yt < live_lo || yt >= live_hi) && yt < live_end; }
};
// Key tiles for the query rows w0 .. w0 + 31 (w0 a multiple of 32; those of them that exist; a candidate stands at position n, and waves with candidates
// leave out no later tile).
HSTU_HD WaveTiles key_tiles_of(const SeqGeom& g, int w0) {
  const bool band = g.K1 >= 0;
  const int first = imin(w0, g.n), last = imin(imin(w0 + 31, g.L - 1), g.n), far = 1 << 30;
  WaveTiles t;
  t.full_hi = first >> 5;
  t.full_lo = band ? imax((last - g.K1) >> 5, -1) + 1 : 0;
  t.full_pre = band ? imin(g.K2 >> 5, t.full_hi) : 0;
  t.live_pre = band ? (g.K2 + 31) >> 5 : 0;
  t.live_lo = band ? (first - g.K1 + 1) >> 5 : 0;
  t.live_hi = imin(w0 + 31, g.L - 1) < g.n ? (w0 >> 5) + 1 : far;
  if (t.live_pre > t.live_hi) t.live_pre = t.live_hi;
  t.live_end = far;
  return t;
}
// Query tiles for the keys k0 .. k0 + 31; full ones hold history rows only, and any tile with a candidate may be visible.
HSTU_HD WaveTiles query_tiles_of(const SeqGeom& g, int k0) {
  const bool window = g.K1 >= 0 && k0 + 31 >= g.K2, all_window = g.K1 >= 0 && k0 >= g.K2;
  WaveTiles t;
  t.full_pre = t.live_pre = 0;
  t.full_lo = (k0 >> 5) + 1;
  t.full_hi = window ? imin((k0 + g.K1) >> 5, g.n >> 5) : g.n >> 5;
  t.live_lo = k0 >> 5;
  t.live_hi = all_window ? (k0 + g.K1 + 62) >> 5 : 1 << 30;
  t.live_end = g.n >> 5;
  return t;
}

}  // namespace hstu
