// Jagged-offset tile scheduler and relative-bias expansion (gfx950), one launch in front of an attention pass.
//
// The scheduler turns seq_offsets (+ num_targets and the mask parameters K1, K2) into an
// ordered list of work items (sequence, block of rows, head).  Fully masked column tiles
// are never visited: every kernel enumerates the visible tiles of its block with
// tile_ranges()/row_tile_ranges(), and the scheduler uses the same functions to price
// each block so that expensive blocks start first (longest-processing-time order).  In the
// key-major list of the dK/dV pass a block far longer than the average (the key blocks of a
// global prefix, which every query of the sequence sees) is cut into pieces along the query
// axis; the pieces write partial sums that a small kernel adds up in a fixed order.
// The cost of a block does not depend on the head, so pricing, cutting and sorting work on (sequence, block) pairs
// and every entry of the sorted list is written once per head (heads adjacent): a single workgroup does all of this.
// Semi-local attention costs O((K1+K2) L) only because of the skipping (paper Section 4.2.1).
//
// What bounds it: nothing but latency (a launch, a few dependent trips to memory, barriers), so the work is arranged to have few
// of each: one workgroup per list, scans and reductions in DPP adds with one trip through LDS, a stable radix sort of 6 bits per
// pass (two passes for costs up to 4,095 tiles) instead of a comparison sort, and the expansion of the bias table (and the
// clearing of the bias gradient's sums) in further workgroups of the same launch.  The instruction cache is cold on every launch
// (the attention kernels fill it), so code that is walked once costs its fetches: loops stay rolled, what a thread would keep in
// registers across them sits in LDS, and block and tile sizes are shifts.  Measured on the launch, with the expansion in it: 10
// blocks 4.9 us (11.3 with a comparison sort and 49 KB of unrolled code), 346 blocks of 512-2048-token sequences 8.7 us (18.4 +
// 5.2 for the expansion's own launch), 690 blocks of 8k-16k tokens 9.4 us (27 + 5); of the last, 1.0 us go to the offsets and
// their scan, 1.1 to pricing, 1.1 to each pass of the sort, 1.2 to writing the list.  Few blocks with many pieces (a query tail)
// spent their time on rounds of scans for the piece size and on one thread writing all pieces of its block, and every call on the
// expansion's searches through the bucket bounds in global memory.  A forward, us, without -> with waves that share the pieces,
// staged bounds and scans without barriers: tail of one 65,536-token history (1 head) 49.5 -> 37.4, of a 20,000-token one (4
// heads) 34.7 -> 31.4, of eight 8k-16k ones 81.5 -> 80.3;  short lists with few pieces: fp32, 426 tokens, 32.3 -> 31.9, 2,733
// tokens (32 features) 30.6 -> 30.2.
#include <cmath>

#include "hstu_common.h"
#include "hstu_kernels.h"
#include "hstu_plan.h"

namespace hstu {
namespace {

constexpr int kSchedThreads = 1024;
constexpr int kSchedWaves = kSchedThreads / 64;
constexpr int kSortMax = 8192;       // lists of up to this many (sequence, block) pairs are sorted by cost in LDS
constexpr int kSeqCache = 1024;      // batches up to this size keep their block prefix sums and lengths in LDS
constexpr int kDigitBits = 6, kDigits = 1 << kDigitBits;   // radix sort: one digit per pass, one counter per lane of a wave
constexpr int kKeyBits = 12;         // costs are sorted exactly up to 4,095 tiles, by 4,096 equal classes beyond
constexpr int kCountPitch = kSchedWaves + 1;
constexpr int kMaxExpandBlocks = 192;

// One workgroup builds one list; the backward pass has two (dQ blocks and dK/dV blocks) side by side.
struct SchedJob {
  int block_shift, tile_shift;        // rows of a block and of a tile: powers of two
  bool key_major, fp32;
  bool even;                          // cut blocks into equal pieces of at most 2 x chunk tiles (else: pieces of chunk tiles)
  int query_tail;                     // > 0 (query-major lists only): only the blocks that hold the last query_tail history rows or candidates
  int slot_cap;            // > 0: blocks much longer than the average may be cut along the streamed axis
  CutRule rule;            // how they are
  SchedHeader* header;
  WorkItem* items;
  int32_t* seq_base;
  SplitItem* splits;
  int32_t* ds_table;       // key-major list, optional: AttnArgs::ds_table
};

struct SchedShared {
  uint32_t keys[2][kSortMax];            // (inverted cost << 13) | entry, from pass to pass; [1] holds the pairs' costs until the first pass
  uint16_t rank[kSortMax];               // of a key among those of its wave with the same digit
  uint32_t entry_item[kSortMax];         // entry -> pair | (piece << 13); unused when nothing is cut (entry = pair)
  uint16_t slot_c[kSortMax];             // pair -> its first slot (x H: slot of head 0), 0xFFFF = not cut
  int32_t base_c[kSeqCache + 1], len_c[kSeqCache], hist_c[kSeqCache], row_c[kSeqCache];
  uint32_t count[kDigits * kCountPitch]; // [digit][wave]
  int32_t wave_total[8][kSchedWaves];    // scratch of scans and reductions
  unsigned long long tiles, dense;       // of a list that is not sorted
  int32_t bad;
};

// v plus (or max with) the value that DPP control CTRL brings from another lane, 0 where it brings none
template <int CTRL, int ROWS>
__device__ __forceinline__ int from_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
__device__ __forceinline__ int row_scan(int v) {            // inclusive sums inside each row of 16 lanes
  v += from_lane<0x111, 0xF>(v);                            // row_shr:1, 2, 4, 8
  v += from_lane<0x112, 0xF>(v);
  v += from_lane<0x114, 0xF>(v);
  return v + from_lane<0x118, 0xF>(v);
}
__device__ __forceinline__ int wave_scan(int v) {           // inclusive sums over the wave
  v = row_scan(v);
  v += from_lane<0x142, 0xA>(v);                            // row_bcast:15 into rows 1 and 3
  return v + from_lane<0x143, 0xC>(v);                      // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ int row_max(int v) {             // lane 15 of a row: its maximum (values >= 0)
  v = max(v, from_lane<0x111, 0xF>(v));
  v = max(v, from_lane<0x112, 0xF>(v));
  v = max(v, from_lane<0x114, 0xF>(v));
  return max(v, from_lane<0x118, 0xF>(v));
}
__device__ __forceinline__ int wave_max(int v) {            // lane 63: the maximum (values >= 0)
  v = row_max(v);
  v = max(v, from_lane<0x142, 0xA>(v));
  return max(v, from_lane<0x143, 0xC>(v));
}

// Exclusive scan of one value per thread over the workgroup; also returns the grand total.  One barrier: consecutive
// calls must use different scratch (a call's barrier protects the scratch of the call before it).
__device__ __forceinline__ int block_scan(int v, int32_t* wave_total, int& total) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int incl = wave_scan(v);
  if (lane == 63) wave_total[wave] = incl;
  __syncthreads();
  const int sums = row_scan(wave_total[lane & (kSchedWaves - 1)]);
  total = __builtin_amdgcn_readlane(sums, kSchedWaves - 1);
  const int before = wave > 0 ? __builtin_amdgcn_readlane(sums, wave - 1) : 0;
  return before + incl - v;
}

__device__ void schedule_list(const SchedJob& job, SchedShared& sh, const int32_t* __restrict__ offsets,
                              const int32_t* __restrict__ num_targets, int B, int H, int K1, int K2, int T, int max_seqlen) {
  const int block_shift = job.block_shift, block_rows = 1 << block_shift, tail = job.query_tail;
  const TileShift tile = {job.tile_shift};
  auto blocks_in = [&](int rows) { return (rows + block_rows - 1) >> block_shift; };
  SchedHeader* header = job.header;
  WorkItem* items = job.items;
  int32_t* seq_base = job.seq_base;
  const bool cached = B <= kSeqCache;                    // else the searches below read seq_base / offsets from global memory
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) { sh.bad = 0; sh.tiles = 0; sh.dense = 0; }
  __syncthreads();

  // 1.  Exclusive scan of blocks-per-sequence (per head).  The offsets live on the device and the host may never have seen
  // them: a batch whose offsets are not a non-decreasing walk from 0 to at most T in steps of at most max_seqlen, or whose
  // candidate counts leave [0, L], gets an empty list (every kernel that follows then returns at once) instead of rows
  // addressed outside the tensors.
  int bad = 0, blocks_per_head = 0;
#pragma unroll 1
  for (int c0 = 0; c0 < B; c0 += kSchedThreads) {
    const int b = c0 + tid;
    int nb = 0, o0 = 0, L = 0, m = 0;
    if (b < B) {
      o0 = offsets[b];
      const int o1 = offsets[b + 1];
      m = num_targets ? num_targets[b] : 0;
      bad |= (o0 < 0) | (o1 < o0) | (o1 > T) | (m < 0) | (b == 0 && o0 != 0);
      L = bad ? 0 : o1 - o0;
      bad |= (L > max_seqlen) | (m > L);
      nb = blocks_in(L - tail_origin(L - m, tail));
    }
    if (__ballot(bad) != 0 && lane == 0) sh.bad = 1;
    int total;
    const int excl = blocks_per_head + block_scan(nb, sh.wave_total[(c0 / kSchedThreads) & 1], total);
    if (b < B) {
      if (cached) { sh.base_c[b] = excl; sh.len_c[b] = L; sh.hist_c[b] = L - m; sh.row_c[b] = o0; }
      if (!cached || job.ds_table) seq_base[b] = excl;
    }
    blocks_per_head += total;
  }
  if (tid == 0) {
    if (cached) sh.base_c[B] = blocks_per_head;
    else seq_base[B] = blocks_per_head;
  }
  __threadfence_block();
  __syncthreads();
  if (sh.bad) {
    if (tid == 0) *header = SchedHeader{0, 0, 0, 0, 0, 1, 0};
    return;
  }
  const int total = blocks_per_head * H;                 // <= max_items by construction of the bound
  const int pairs = blocks_per_head;                     // (sequence, block) pairs: what is priced, cut and sorted
  auto base_of = [&](int b) { return cached ? sh.base_c[b] : seq_base[b]; };

  // Item idx of `heads` heads in natural order (sequence-major, then head, then block index descending; with a query
  // tail the blocks start at tail_origin()) -> its work item (whole) and, if wanted, its cost in tiles.  heads = 1 enumerates the pairs.
  int first_tile = 0;                                    // out of locate(): the first tile of a priced item
  auto locate = [&](int idx, int heads, bool priced, int& cost) {
    int lo = 0, hi = B;                                  // invariant: base[lo]*heads <= idx < base[hi]*heads
#pragma unroll 1
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if ((long long)base_of(mid) * heads <= idx) lo = mid; else hi = mid;
    }
    WorkItem it;
    it.b = lo;
    if (cached) { it.seq0 = sh.row_c[lo]; it.len = sh.len_c[lo]; it.hist = sh.hist_c[lo]; }
    else {
      it.seq0 = offsets[lo];
      it.len = offsets[lo + 1] - it.seq0;
      it.hist = it.len - (num_targets ? num_targets[lo] : 0);
    }
    int rank = idx - base_of(lo) * heads, h = 0;
    if (heads > 1) {
      const int nb = base_of(lo + 1) - base_of(lo);
      h = rank / nb;
      rank -= h * nb;
    }
    const int row0 = tail_origin(it.hist, tail);
    const int rb = blocks_in(it.len - row0) - 1 - rank;
    it.rb_h = (rb << 8) | h;
    it.t0 = 0; it.t1 = 0x7FFFFFFF; it.slot = -1;
    if (priced) {
      const SeqGeom g = {it.len, it.hist, K1, K2};
      const int r0 = row0 + (rb << block_shift), r1 = min(r0 + block_rows, it.len) - 1;
      const TileRanges tr = job.key_major ? row_tile_ranges_of(g, r0, r1, tile) : tile_ranges_of(g, r0, r1, tile);
      cost = tr.count();
      first_tile = tr.at(0);
    }
    return it;
  };

  // 2. price the pairs (of a list that is not sorted: the items, which are written as they come)
  const bool sorted = pairs <= kSortMax;
  uint32_t* costs = sh.keys[1];
  // (sums of a sorted list's costs stay below 2^31: 8,192 blocks are a million rows, at most 32,768 tiles each)
  unsigned long long my_tiles = 0, my_dense = 0;
  int my_max = 0;
#pragma unroll 1
  for (int idx = tid; idx < (sorted ? pairs : total); idx += kSchedThreads) {
    int cost = 0;
    const WorkItem it = locate(idx, sorted ? 1 : H, true, cost);
    my_tiles += cost;
    my_dense += tile.index(it.len + tile.width() - 1);
    my_max = max(my_max, cost);
    if (sorted && job.ds_table) { job.ds_table[4 * idx + 1] = first_tile; job.ds_table[4 * idx + 2] = cost; }
    if (sorted) costs[idx] = cost;
    else items[idx] = it;
  }
  if (!sorted) {
    atomicAdd(&sh.tiles, my_tiles);
    atomicAdd(&sh.dense, my_dense);
    __syncthreads();
    if (tid == 0) *header = SchedHeader{total, 0, (int64_t)sh.tiles, (int64_t)sh.dense, 0, 0, -1};
    return;
  }
  {
    const int t = wave_scan((int)my_tiles), d = wave_scan((int)my_dense), m = wave_max(my_max);
    if (lane == 63) { sh.wave_total[0][wave] = t; sh.wave_total[1][wave] = d; sh.wave_total[2][wave] = m; }
  }
  __syncthreads();
  const int col = lane & (kSchedWaves - 1);
  const int pair_tiles = __builtin_amdgcn_readlane(row_scan(sh.wave_total[0][col]), kSchedWaves - 1);
  const int pair_dense = __builtin_amdgcn_readlane(row_scan(sh.wave_total[1][col]), kSchedWaves - 1);
  const int max_cost = __builtin_amdgcn_readlane(row_max(sh.wave_total[2][col]), kSchedWaves - 1);
  const int64_t all_tiles = (int64_t)pair_tiles * H, all_dense = (int64_t)pair_dense * H;

  // 3.  Cut blocks that are much longer than the rest (CutRule; the few key blocks of a global prefix are seen by every query of
  // their sequence).  Each piece becomes an entry of the list and accumulates into a partial-sum slot of its own (one per head).
  // The piece size doubles until the slots and the list fit, and grows by a quarter once the slots are short by a quarter (with a
  // query tail) or a half: doubled there, most blocks are no longer than twice a piece and stay whole (16 sequences of
  // 2,000-4,000 tokens, 4 heads of 32 features, tail 500: 91 us, 69 this way; n tiles in pieces of n / (slots - blocks), which
  // always fit, 86).
  int chunk = (int)fmin((double)0x3FFFFFFF, fmax((double)job.rule.min_chunk, ceil((double)all_tiles * (1.0 / job.rule.target_chunks))));
  // pieces of a block of `cost` tiles and their length: the fewest equal pieces of at most 2 x chunk tiles (every piece costs a
  // partial-sum slot and its traffic), or pieces of `chunk` tiles
  auto pieces_of = [&](int cost, int& len) {
    len = cost;
    if (cost <= 2 * chunk) return 1;
    const int most = job.even ? 2 * chunk : chunk;
    const int pieces = (cost + most - 1) / most;
    len = job.even ? (cost + pieces - 1) / pieces : chunk;
    return pieces;
  };
  const int ipt = (pairs + kSchedThreads - 1) / kSchedThreads;
  const int own0 = min(tid * ipt, pairs), own1 = min(own0 + ipt, pairs);   // the scans below give every thread consecutive pairs
  int64_t ds_tiles = -1;
  if (job.ds_table) {                                      // where the dS tiles of a pair's heads start
    int sum = 0, all;
#pragma unroll 1
    for (int idx = own0; idx < own1; ++idx) sum += (int)costs[idx];
    sum = block_scan(sum, sh.wave_total[7], all);
    ds_tiles = (int64_t)all * H;
#pragma unroll 1
    for (int idx = own0; idx < own1; ++idx) { job.ds_table[4 * idx] = (int)((uint32_t)sum * (uint32_t)H); sum += (int)costs[idx]; }
  }
  int slot0 = 0, rank0 = 0, slots = 0, nsplit = 0, entries = pairs;        // first slot and rank of this thread's pairs among the cut ones; totals
  bool cuts = false;                                       // uniform: some block is cut
  const bool many = num_targets && (long long)pairs * H >= kManyBlocks;
  const int launch = num_targets && !many ? 0 : job.rule.launch;      // (with candidates it is there in any case)
  const bool wanted = job.slot_cap > 0 && max_cost > worth_cutting(chunk, job.fp32) + launch &&
                      max_cost > 2 * job.rule.min_chunk + job.rule.launch * (many ? kUnsure : 1);
  const bool few = pairs <= 64;                            // every wave adds all of them up for itself, a pair a lane: no barriers
  const int at = few ? min(lane, pairs) : own0, to = few ? min(lane + 1, pairs) : own1;
#pragma unroll 1
  for (int round = 0; wanted && max_cost > 2 * chunk; round ^= 1) {
    int my_slots = 0, my_cuts = 0;
#pragma unroll 1
    for (int idx = at; idx < to; ++idx) {
      int len;
      const int pieces = pieces_of((int)costs[idx], len);
      my_slots += pieces > 1 ? pieces : 0;
      my_cuts += pieces > 1 ? 1 : 0;
    }
    if (few) {
      slot0 = wave_scan(my_slots);
      rank0 = wave_scan(my_cuts);
      slots = __builtin_amdgcn_readlane(slot0, 63);
      nsplit = __builtin_amdgcn_readlane(rank0, 63);
      slot0 -= my_slots;
      rank0 -= my_cuts;
    } else {
      slot0 = block_scan(my_slots, sh.wave_total[3 + 2 * round], slots);
      rank0 = block_scan(my_cuts, sh.wave_total[4 + 2 * round], nsplit);
    }
    entries = pairs - nsplit + slots;
    if (entries <= kSortMax && (long long)slots * H <= job.slot_cap) {       // uniform: every thread sees the same totals
      cuts = max_cost > worth_cutting(chunk, job.fp32) + launch + slots * H / job.rule.slots_per_tile;
      break;
    }
    const bool nearly = 4 * (long long)slots * H <= (tail > 0 ? 5 : 6) * (long long)job.slot_cap;
    chunk += nearly ? max(chunk >> 2, 1) : chunk;              // ends: with no pair cut, entries = pairs <= kSortMax
  }
  if (!cuts) { entries = pairs; nsplit = 0; }
  if (tid == 0) *header = SchedHeader{entries * H, nsplit * H, all_tiles, all_dense, chunk, 0, ds_tiles};
  const int key_max = cuts ? min(max_cost, 2 * chunk) : max_cost;            // no entry is longer than this
  const int key_bits = max(32 - __clz(key_max), 1);
  const int shift = max(key_bits - kKeyBits, 0);
  // (ties keep the natural order of the entries: sequence-major, last block first; entry < 8192 = 2^13)
  auto key_of = [&](int cost, int entry) { return ((uint32_t)((key_max >> shift) - (cost >> shift)) << 13) | (uint32_t)entry; };
  if (!cuts) {
#pragma unroll 1
    for (int idx = tid; idx < pairs; idx += kSchedThreads) sh.keys[0][idx] = key_of((int)costs[idx], idx);
  } else {
    int slot = slot0, rank = rank0, e = at - rank0 + slot0;
    // A pair's pieces and heads are its thread's; with many pieces the waves share those of few pairs (all of them for a few
    // pieces: 0.9 us, the instructions of 16 waves on 4 SIMDs)
    const bool share = few && (max_cost >> 5) > chunk;
    const int first = share ? wave : 0, step = share ? kSchedWaves : 1;
#pragma unroll 1
    for (int idx = few && !share && wave > 0 ? to : at; idx < to; ++idx) {
      const int cost = (int)costs[idx];
      int plen;
      const int pieces = pieces_of(cost, plen);
      sh.slot_c[idx] = pieces > 1 ? (uint16_t)slot : (uint16_t)0xFFFF;
#pragma unroll 1
      for (int c = first; c < pieces; c += step) {
        sh.keys[0][e + c] = key_of(min(plen, cost - c * plen), e + c);
        sh.entry_item[e + c] = (uint32_t)idx | ((uint32_t)c << 13);
      }
      if (pieces > 1) {                                  // the pieces of head h own the slots [(slot * H + h * pieces), + pieces)
        int unused;
        const WorkItem it = locate(idx, 1, false, unused);
#pragma unroll 1
        for (int h = first; h < H; h += step) job.splits[rank * H + h] = SplitItem{it.b, it.rb_h | h, slot * H + h * pieces, pieces, it.seq0, it.len, it.hist, 0};
        slot += pieces;
        ++rank;
      }
      e += pieces;
    }
  }
  __syncthreads();

  // 4. stable radix sort of the keys, ascending = most expensive first.  Wave w owns the positions [w * per, (w + 1) * per) of
  // the list as it stands; a key's place is the number of keys with smaller digits, plus those of the same digit in earlier
  // waves, plus those ahead of it in its own wave (which the wave counts 64 keys at a time, equal digits found with ballots).
  const int per = ((entries + kSchedWaves - 1) / kSchedWaves + 63) & ~63;     // at most 512
  const int first = wave * per + lane, last = min(wave * per + per, entries);
  int src = 0;
#pragma unroll 1
  for (int bit = 13; bit < 13 + min(key_bits, kKeyBits); bit += kDigitBits, src ^= 1) {
    volatile uint32_t* mine = sh.count + wave;                                 // this wave's counter of digit d: mine[d * kCountPitch]
    mine[lane * kCountPitch] = 0u;
#pragma unroll 1
    for (int i = first; i - lane < last; i += 64) {
      const bool on = i < last;
      const uint32_t d = on ? (sh.keys[src][i] >> bit) & (kDigits - 1) : 0u;
      uint64_t peers = __ballot(on);
#pragma unroll
      for (int q = 0; q < kDigitBits; ++q) {
        const uint64_t ones = __ballot((d >> q) & 1u);
        peers &= ((d >> q) & 1u) ? ones : ~ones;
      }
      const uint32_t ahead = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
      const uint32_t seen = mine[d * kCountPitch];                             // (LDS operations of a wave complete in order)
      if (on) {
        sh.rank[i] = (uint16_t)(seen + ahead);
        if (ahead == 0) mine[d * kCountPitch] = seen + (uint32_t)__popcll(peers);
      }
    }
    __syncthreads();
    uint32_t& counter = sh.count[(tid / kSchedWaves) * kCountPitch + tid % kSchedWaves];    // digit-major, then wave
    int all;
    counter = (uint32_t)block_scan((int)counter, sh.wave_total[src], all);
    __syncthreads();
#pragma unroll 1
    for (int i = first; i < last; i += 64) {
      const uint32_t key = sh.keys[src][i];
      sh.keys[src ^ 1][sh.count[((key >> bit) & (kDigits - 1)) * kCountPitch + wave] + sh.rank[i]] = key;
    }
    __syncthreads();
  }

  // 5. the list.  The attention kernels keep runs of kXcdGroup consecutive items on one die; a run is made of consecutive
  // entries of one head (for equal costs these are neighbouring blocks of one sequence, which share most of the rows
  // they stream), so a group of kXcdGroup sorted entries becomes H runs, one per head.
#pragma unroll 1
  for (int pos = tid; pos < entries; pos += kSchedThreads) {
    const uint32_t entry = sh.keys[src][pos] & 0x1FFF;
    const uint32_t ei = cuts ? sh.entry_item[entry] : entry;
    const int idx = (int)(ei & 0x1FFF), c = (int)(ei >> 13);
    int cost = 0, pieces = 0;
    const bool cut = cuts && sh.slot_c[idx] != 0xFFFF;
    WorkItem it = locate(idx, 1, cut, cost);
    if (cut) {
      int plen;
      pieces = pieces_of(cost, plen);
      it.t0 = c * plen;
      it.t1 = min(it.t0 + plen, cost);
      it.slot = (int)sh.slot_c[idx] * H + c;
    }
    const int grp0 = pos & ~(kXcdGroup - 1), gsize = min(kXcdGroup, entries - grp0);
    WorkItem* dst = items + (size_t)grp0 * H + (pos - grp0);
#pragma unroll 1
    for (int h = 0; h < H; ++h, dst += gsize, it.rb_h += 1, it.slot += pieces) *dst = it;
  }
}

// Thread `id` of `n` threads fills its share of the tables:
//   bias[h, x] = log2(e) * table[h, bucket(x)], bucket(x) = max{c : bounds[c] <= x}, for x in [0, bias_len): the attention kernels
//   keep their scores in units of ln 2; bucket_end[x]: where the next bucket starts;
//   and the zeros around every head's row;
//   seed[v][h][i] (AttnArgs::seed), d = seed_dmax - i, and seed_up[h][i], d = i - kSeedUpZero;
//   and clears the per-distance sums of the bias gradient.
// The bounds (where they fit) wait in LDS: a search is seven dependent loads, from the caches 3 us.
__device__ void expand_tables(const ExpandJob& j, int H, int K1, int max_seqlen, int id, int n, int32_t* lds_bounds, int lds_most) {
  const bool staged = j.num_buckets <= lds_most;
  for (int c = threadIdx.x; staged && c < j.num_buckets; c += kSchedThreads) lds_bounds[c] = j.bounds[c];
  __syncthreads();
  auto bucket = [&](int x) {
    int lo = 0, hi = j.num_buckets;                       // bounds[lo] <= x < bounds[hi] (bounds[num_buckets] = +inf)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if ((staged ? lds_bounds[mid] : j.bounds[mid]) <= x) lo = mid; else hi = mid;
    }
    return lo;
  };
  for (int x = id; (j.bias || j.bucket_end) && x < j.bias_len; x += n) {
    const int c = bucket(x);
    for (int h = 0; j.bias && h < H; ++h) j.bias[(size_t)h * j.bias_pitch + x] = j.table[(size_t)h * j.num_buckets + c] * 1.4426950408889634f;
    if (j.bucket_end) j.bucket_end[x] = c + 1 < j.num_buckets ? j.bounds[c + 1] : 0x7FFFFFFF;
  }
  for (int i = id; j.bias && i < (H + 1) * kBiasPad; i += n) j.bias[(int64_t)(i / kBiasPad) * j.bias_pitch - kBiasPad + i % kBiasPad] = 0.f;
  for (int i = id; j.seed && i < j.seed_len; i += n) {
    const int d = j.seed_dmax - i;
    const int c = j.table ? bucket(d < 0 ? 0 : (d > max_seqlen ? max_seqlen : d)) : 0;    // distances beyond any real pair take the last real one's bias
    for (int h = 0; h < H; ++h) {
      const float b = j.table ? j.table[(size_t)h * j.num_buckets + c] * 1.4426950408889634f : 0.f;
      j.seed[(size_t)h * j.seed_len + i] = d < 0 ? -1e30f : b;
      j.seed[((size_t)H + h) * j.seed_len + i] = (d < 0 || (K1 >= 0 && d >= K1)) ? -1e30f : b;
    }
  }
  for (int i = id; j.seed_up && i < j.seed_len; i += n) {
    const int d = i - kSeedUpZero;
    const int c = j.table ? bucket(d < 0 ? 0 : (d > max_seqlen ? max_seqlen : d)) : 0;
    for (int h = 0; h < H; ++h) {
      const float b = j.table ? j.table[(size_t)h * j.num_buckets + c] * 1.4426950408889634f : 0.f;
      j.seed_up[(size_t)h * j.seed_len + i] = d < 0 ? -1e30f : b;
    }
  }
  for (int64_t i = id; i < j.zero_count; i += n) j.zero[i] = 0.f;
}

__global__ __launch_bounds__(kSchedThreads) void schedule_kernel(const int32_t* __restrict__ offsets,
                                                                 const int32_t* __restrict__ num_targets, int B, int H,
                                                                 int K1, int K2, int T, int max_seqlen, int njobs, SchedJob job0,
                                                                 SchedJob job1, ExpandJob ex) {
  __shared__ SchedShared sh;
  const int blk = blockIdx.x;
  if (blk < njobs) schedule_list(blk == 0 ? job0 : job1, sh, offsets, num_targets, B, H, K1, K2, T, max_seqlen);
  else expand_tables(ex, H, K1, max_seqlen, (blk - njobs) * kSchedThreads + threadIdx.x, ((int)gridDim.x - njobs) * kSchedThreads,
                     (int32_t*)sh.keys[0], kSortMax);
}

int log2_of(int n) { return 31 - __builtin_clz((unsigned)n); }

hipError_t launch(const AttnArgs& a, int njobs, const SchedJob& j0, const SchedJob& j1, const ExpandJob& ex, hipStream_t stream) {
  int64_t most = ex.bias || ex.bucket_end ? ex.bias_len : 0;
  if (ex.seed && ex.seed_len > most) most = ex.seed_len;
  if (ex.zero_count / 4 > most) most = ex.zero_count / 4;
  int64_t blocks = (most + kSchedThreads - 1) / kSchedThreads;
  if (blocks > kMaxExpandBlocks) blocks = kMaxExpandBlocks;
  if (njobs + blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(schedule_kernel, dim3(njobs + (unsigned)blocks), dim3(kSchedThreads), 0, stream, a.offsets, a.num_targets, a.B, a.H,
                     a.K1, a.K2, a.T, a.max_seqlen, njobs, j0, j1, ex);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_schedule(const AttnArgs& a, bool lists, int block_rows, int tile_cols, SchedHeader* header, WorkItem* items,
                           int32_t* seq_base, SplitItem* splits, int slot_cap, bool fp32, const ExpandJob& ex, hipStream_t stream) {
  // (the forward over a query tail takes finer pieces: few blocks, each against a whole history)
  const bool even = a.query_tail == 0;
  const SchedJob job = {log2_of(block_rows), log2_of(tile_cols), false, fp32, even, a.query_tail, slot_cap, cut_rule_for(fp32, a.D, 0, !even), header, items, seq_base, splits, nullptr};
  return launch(a, lists ? 1 : 0, job, job, ex, stream);
}

hipError_t launch_schedule_pair(const AttnArgs& a, bool lists, const int block_rows[2], const int tile_cols[2], SchedHeader* const header[2],
                                WorkItem* const items[2], int32_t* const seq_base[2], SplitItem* const splits[2],
                                const int slot_cap[2], bool fp32, int32_t* ds_table, const ExpandJob& ex, hipStream_t stream) {
  const SchedJob j0 = {log2_of(block_rows[0]), log2_of(tile_cols[0]), false, fp32, true, 0, slot_cap[0], cut_rule_for(fp32, a.D, 1, false), header[0], items[0], seq_base[0], splits[0], nullptr};
  const SchedJob j1 = {log2_of(block_rows[1]), log2_of(tile_cols[1]), true, fp32, !fp32, 0, slot_cap[1], cut_rule_for(fp32, a.D, 2, false), header[1], items[1], seq_base[1], splits[1], ds_table};
  return launch(a, lists ? 2 : 0, j0, j1, ex, stream);
}

int schedule_sorted_pairs() { return kSortMax; }

}  // namespace hstu
