// C-ABI entry points of the jagged HSTU attention library: argument validation, workspace
// layout and kernel launches.  Declarations and the meaning of every argument: include/hstu_attn.h.
#include "../../include/hstu_attn.h"
#include "hstu_common.h"
#include "hstu_kernels.h"
#include "hstu_plan.h"
#include "profile.h"

#include <algorithm>
#include <mutex>

using namespace hstu;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Upper bound of the schedule length: every sequence adds at most one ragged block.
inline int64_t max_items_for(const hstu_attn_params* p, int block_rows) {
  return ((int64_t)p->total_tokens / block_rows + p->batch) * p->num_heads;
}

// Copies of the sums per distance: one per die while they stay small (16 MB, up to 62 distances a row of padding apart: clearing and adding them up takes a few
// microseconds).
inline int dbias_copies_for(const hstu_attn_params* p) {
  return (int64_t)kDbiasCopies * p->num_heads * ((int64_t)p->max_seqlen + 1) <= (int64_t)4 << 20 ? kDbiasCopies : 1;
}

struct Layout {           // byte offsets inside a workspace
  size_t header[2], items[2], seq_base[2], bias, seed, seed_up, splits, partial, splits_dq, partial_dq, dbias, ds_table, total;
  size_t ds_bytes;        // room for dS that the backward can use behind `total`, or elsewhere; 0: none
  int max_items[2];
  int slot_cap;           // partial-sum slots of the dK/dV pass (key blocks cut along the query axis) or of the forward
  int slot_cap_dq;        // ... of the dQ pass (query blocks of a small batch cut along the key axis)
};

// Sequences are shorter than 2^24 tokens: windows beyond 2^28 mean the same and keep the kernels' index sums inside int32.
inline int window_of(int32_t w) { return w < 0 ? -1 : (w < (1 << 28) ? w : (1 << 28)); }

PlanBatch plan_of(const hstu_attn_params* p) {
  return {p->batch, p->num_heads, p->total_tokens, p->max_seqlen, window_of(p->local_window), window_of(p->global_prefix), p->num_targets != nullptr,
          p->seq_offsets_host};
}
// 1/18 of the card's memory: seven sequences of 16,384 tokens with eight heads under the dense mask (14.1 GiB; eight need 16.1); beyond it
// the two passes stay independent of each other (dQ recomputes S and dP).
constexpr int64_t kDsMaxBytes = (int64_t)16 << 30;

// The pipelined kernels take bias and mask from seed tables, the others the bias from a table of its own.
inline bool seeded(const hstu_attn_params* p, bool for_backward) { return p->dtype == HSTU_BF16 && (!for_backward || p->head_dim != 128); }

// One schedule for the forward; two (dQ pass, dK/dV pass) for the backward.
Layout make_layout(const hstu_attn_params* p, int for_backward) {
  Layout l = {};
  size_t off = 0;
  const int nsched = for_backward ? 2 : 1;
  for (int s = 0; s < nsched; ++s) {
    const int rows = !for_backward ? fwd_block_rows(p->dtype, p->head_dim)
                                   : (s == 0 ? dq_block_rows(p->dtype, p->head_dim) : dkv_block_rows(p->dtype, p->head_dim));
    l.max_items[s] = (int)max_items_for(p, rows);
    // a list also holds the pieces of its cut blocks (hstu_plan.h)
    if ((for_backward && s == 1) || !for_backward) {
      l.slot_cap = slot_cap_for(l.max_items[s], p->dtype == HSTU_FP32);
      l.max_items[s] += l.slot_cap;
    } else {
      l.slot_cap_dq = slot_cap_for(l.max_items[s], p->dtype == HSTU_FP32);
      l.max_items[s] += l.slot_cap_dq;
    }
    l.header[s] = off; off += kAlign;
    l.items[s] = off; off += align_up((size_t)l.max_items[s] * sizeof(WorkItem));
    l.seq_base[s] = off; off += align_up(((size_t)p->batch + 1) * sizeof(int32_t));
  }
  // All that a later call with reuse_schedule takes from this one comes first, at places that follow from the sizes such calls share (not
  // from max_seqlen, the host copy of the offsets or the room for dS).
  l.splits = off; off += align_up((size_t)(l.slot_cap / 2 + 1) * sizeof(SplitItem));
  // (dS for 32 and 64 features: its product would move as many bytes as for 128 and save a half or a quarter of the matrix work)
  const bool ds = for_backward && p->dtype == HSTU_BF16 && p->head_dim == 128 &&
                  (int64_t)p->total_tokens / 128 + p->batch <= schedule_sorted_pairs();
  if (for_backward) { l.splits_dq = off; off += align_up((size_t)(l.slot_cap_dq / 2 + 1) * sizeof(SplitItem)); }
  if (ds) { l.ds_table = off; off += align_up(((size_t)p->total_tokens / 128 + p->batch) * 16); }
  if (seeded(p, for_backward)) {                       // score seeds by distance (bias + mask) ...
    const size_t table = (size_t)p->num_heads * (size_t)seed_len_for(p->max_seqlen) * sizeof(float);
    l.seed = off; off += align_up(kSeedVariants * table);
    if (for_backward) { l.seed_up = off; off += align_up(table); }
  } else {                                             // ... or the bias by distance
    l.bias = off + kBiasPad * sizeof(float);
    off += align_up(((size_t)p->num_heads * ((size_t)p->max_seqlen + 1 + kBiasPad) + kBiasPad) * sizeof(float));
  }
  if (!for_backward) {
    l.partial = off;
    off += align_up((size_t)l.slot_cap * fwd_block_rows(p->dtype, p->head_dim) * p->head_dim * sizeof(float));
  }
  if (for_backward) {
    l.partial = off;
    off += align_up((size_t)l.slot_cap * 2 * dkv_block_rows(p->dtype, p->head_dim) * p->head_dim * sizeof(float));
    l.partial_dq = off;
    off += align_up((size_t)l.slot_cap_dq * dq_block_rows(p->dtype, p->head_dim) * p->head_dim * sizeof(float));
    l.dbias = off;                                     // per-distance sums of dS for the bias-table gradient, then the bucket ends per distance
    off += align_up(((size_t)dbias_copies_for(p) * p->num_heads * dbias_pitch_for(p->max_seqlen) + p->max_seqlen + 1) * sizeof(float));
    const int64_t bytes = ds ? ds_tiles_bound(plan_of(p)) * kDsTileBytes : 0;
    if (bytes <= kDsMaxBytes) l.ds_bytes = (size_t)bytes;
  }
  l.total = off;
  return l;
}

int validate(const hstu_attn_params* p) {
  if (!p) return HSTU_ERR_NULL;
  if (p->batch < 0 || p->total_tokens < 0 || p->max_seqlen < 0 || p->num_heads < 1 || p->num_heads > 256) return HSTU_ERR_SHAPE;
  if (p->dtype != HSTU_BF16 && p->dtype != HSTU_FP32) return HSTU_ERR_UNSUPPORTED;
  if (p->head_dim != 32 && p->head_dim != 64 && p->head_dim != 128) return HSTU_ERR_UNSUPPORTED;
  const int64_t hd = (int64_t)p->num_heads * p->head_dim;
  const int64_t quantum = p->dtype == HSTU_BF16 ? 8 : 4;     // rows must start on 16-byte boundaries
  const int64_t strides[4] = {p->row_stride_q, p->row_stride_k, p->row_stride_v, p->row_stride_o};
  for (int i = 0; i < 4; ++i)
    if (strides[i] < hd || strides[i] % quantum != 0) return HSTU_ERR_SHAPE;
  // the kernels address a tile row as (sequence base) + 32-bit byte offset = 24-bit row * 24-bit stride
  const int64_t esize = p->dtype == HSTU_BF16 ? 2 : 4;
  if (p->max_seqlen >= 1 << 24) return HSTU_ERR_UNSUPPORTED;
  for (int i = 0; i < 4; ++i)
    if (strides[i] * esize >= 1 << 24 || strides[i] * esize * ((int64_t)p->max_seqlen + 1) >= (int64_t)1 << 32)
      return HSTU_ERR_UNSUPPORTED;
  if (p->batch > 0 && !p->seq_offsets) return HSTU_ERR_NULL;
  if (p->global_prefix < 0) return HSTU_ERR_SHAPE;
  if ((p->rab_table == nullptr) != (p->rab_bounds == nullptr)) return HSTU_ERR_NULL;
  if (p->rab_table && (p->num_buckets < 1 || p->num_buckets > 4096)) return HSTU_ERR_SHAPE;
  if (p->d_rab_table && !p->rab_table) return HSTU_ERR_NULL;
  if (p->query_tail < 0) return HSTU_ERR_SHAPE;
  if (p->reuse_schedule != 0 && p->reuse_schedule != 1) return HSTU_ERR_SHAPE;
  if ((int64_t)p->total_tokens * p->num_heads / 32 + (int64_t)p->batch * p->num_heads > 0x7FFFFF00) return HSTU_ERR_SHAPE;
  if (p->seq_offsets_host) {
    const int32_t* o = p->seq_offsets_host;
    if (o[0] != 0) return HSTU_ERR_SHAPE;
    for (int b = 0; b < p->batch; ++b) {
      const int64_t len = (int64_t)o[b + 1] - o[b];
      if (len < 0 || len > p->max_seqlen) return HSTU_ERR_SHAPE;
    }
    if (o[p->batch] != p->total_tokens) return HSTU_ERR_SHAPE;
  }
  return HSTU_OK;
}

inline bool misaligned(const void* ptr) { return ((uintptr_t)ptr & 15u) != 0; }

AttnArgs make_args(const hstu_attn_params* p, const void* q, const void* k, const void* v) {
  AttnArgs a = {};
  a.q = q; a.k = k; a.v = v;
  a.sq = p->row_stride_q; a.sk = p->row_stride_k; a.sv = p->row_stride_v; a.so = p->row_stride_o;
  a.offsets = p->seq_offsets; a.num_targets = p->num_targets;
  a.B = p->batch; a.H = p->num_heads; a.D = p->head_dim; a.T = p->total_tokens; a.max_seqlen = p->max_seqlen;
  a.K1 = window_of(p->local_window);
  a.K2 = window_of(p->global_prefix);
  a.alpha = p->alpha; a.inv_n = p->inv_n;
  a.query_tail = p->query_tail > 0 ? p->query_tail : 0;
  return a;
}

// Fills the bias fields of the kernel arguments and describes the tables behind them (lead: AttnArgs::dbias_lead).
ExpandJob prepare_bias(const hstu_attn_params* p, AttnArgs& a, unsigned char* ws, const Layout& l, bool for_forward, int lead) {
  ExpandJob ex = {};
  a.bias = nullptr;
  a.bias_stride = p->max_seqlen + 1;
  a.bias_pitch = a.bias_stride + kBiasPad;
  a.seed = nullptr;
  ex.table = p->rab_table; ex.bounds = p->rab_bounds;
  ex.num_buckets = p->rab_table ? p->num_buckets : 0;      // (any number is accepted without a table; the kernel reads that many bounds)
  if (seeded(p, !for_forward)) {
    ex.seed = (float*)(ws + l.seed);
    ex.seed_len = seed_len_for(p->max_seqlen);
    ex.seed_dmax = seed_dmax_for(p->max_seqlen);
    if (!for_forward) ex.seed_up = (float*)(ws + l.seed_up);
    a.seed = ex.seed; a.seed_up = ex.seed_up; a.seed_len = ex.seed_len; a.seed_dmax = ex.seed_dmax;
  }
  if (!p->rab_table) return ex;
  ex.bias_len = a.bias_stride;
  if (!seeded(p, !for_forward)) {
    a.bias = ex.bias = (float*)(ws + l.bias);
    ex.bias_pitch = a.bias_pitch;
  }
  if (!for_forward && p->d_rab_table) {               // only the bias-table gradient needs the bucket ends and the sums per distance
    a.dbias_copies = dbias_copies_for(p);
    a.dbias_pitch = dbias_pitch_for(p->max_seqlen);
    a.dbias_lead = lead;
    const int64_t n = (int64_t)a.dbias_copies * p->num_heads * a.dbias_pitch;
    a.dbias_dist = ex.zero = (float*)(ws + l.dbias);
    ex.zero_count = n;
    a.bucket_end = ex.bucket_end = (int32_t*)(ws + l.dbias) + n;
  }
  return ex;
}

}  // namespace

// ---- optional per-kernel timing (for benchmarks): HIP events around every launch, on the launch stream
namespace hstu {
constexpr int kProfSlots = 64;
struct ProfSlot { const char* name; hipEvent_t e0, e1; bool used; };
static ProfSlot g_prof[kProfSlots];
static bool g_prof_on = false, g_prof_init = false;
static int g_prof_n = 0;

ProfScope::ProfScope(const char* name, hipStream_t st) : s(nullptr), stream(st) {
  if (!g_prof_on || g_prof_n >= kProfSlots) return;
  s = &g_prof[g_prof_n++];
  s->name = name;
  s->used = hipEventRecord(s->e0, stream) == hipSuccess;
}
ProfScope::~ProfScope() {
  if (s && s->used) s->used = hipEventRecord(s->e1, stream) == hipSuccess;
}
}  // namespace hstu

extern "C" {

int hstu_profile_enable(int on) {
  if (on && !g_prof_init) {
    for (int i = 0; i < kProfSlots; ++i) {
      if (hipEventCreate(&g_prof[i].e0) != hipSuccess || hipEventCreate(&g_prof[i].e1) != hipSuccess) return HSTU_ERR_LAUNCH;
      g_prof[i].used = false;
    }
    g_prof_init = true;
  }
  g_prof_on = on != 0;
  g_prof_n = 0;
  return HSTU_OK;
}

int hstu_profile_read(int max_entries, const char** names, float* ms) {
  int n = 0;
  for (int i = 0; i < g_prof_n && n < max_entries; ++i) {
    if (!g_prof[i].used) continue;
    if (hipEventSynchronize(g_prof[i].e1) != hipSuccess) return HSTU_ERR_LAUNCH;
    float t = 0.f;
    if (hipEventElapsedTime(&t, g_prof[i].e0, g_prof[i].e1) != hipSuccess) return HSTU_ERR_LAUNCH;
    names[n] = g_prof[i].name;
    ms[n] = t;
    ++n;
  }
  g_prof_n = 0;
  return n;
}

const char* hstu_status_string(int status) {
  switch (status) {
    case HSTU_OK: return "HSTU_OK";
    case HSTU_ERR_NULL: return "HSTU_ERR_NULL: required pointer is NULL";
    case HSTU_ERR_SHAPE: return "HSTU_ERR_SHAPE: invalid sizes, strides, alignment or offsets";
    case HSTU_ERR_UNSUPPORTED: return "HSTU_ERR_UNSUPPORTED: head_dim, dtype or feature count not supported";
    case HSTU_ERR_WORKSPACE: return "HSTU_ERR_WORKSPACE: workspace missing, misaligned or too small";
    case HSTU_ERR_LAUNCH: return "HSTU_ERR_LAUNCH: HIP runtime refused a launch";
    default: return "unknown hstu_status";
  }
}

size_t hstu_attn_workspace_bytes(const hstu_attn_params* p, int for_backward) {
  if (validate(p) != HSTU_OK) return 0;
  const Layout l = make_layout(p, for_backward);
  return l.total + l.ds_bytes;
}

size_t hstu_attn_workspace_least_bytes(const hstu_attn_params* p, int for_backward) {
  return validate(p) != HSTU_OK ? 0 : make_layout(p, for_backward).total;
}

int hstu_attn_fwd(const hstu_attn_params* p, const void* q, const void* k, const void* v, void* out, void* workspace,
                  size_t workspace_bytes, void* stream_) {
  const int st = validate(p);
  if (st != HSTU_OK) return st;
  if (p->total_tokens == 0 || p->batch == 0) return HSTU_OK;
  if (!q || !k || !v || !out) return HSTU_ERR_NULL;
  if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out)) return HSTU_ERR_SHAPE;
  const Layout l = make_layout(p, 0);
  if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < l.total) return HSTU_ERR_WORKSPACE;
  hipStream_t stream = (hipStream_t)stream_;
  unsigned char* ws = (unsigned char*)workspace;

  AttnArgs a = make_args(p, q, k, v);
  a.out = out;
  a.max_items = l.max_items[0];
  a.header = (const SchedHeader*)(ws + l.header[0]);
  a.items = (const WorkItem*)(ws + l.items[0]);
  a.splits = (const SplitItem*)(ws + l.splits);
  a.partial = (float*)(ws + l.partial);
  // (a list is cut only where the launch that finishes cut blocks follows: lengths on the device may be longer than the host's copy says)
  const bool fp32 = p->dtype == HSTU_FP32;
  const bool may_cut = schedule_may_cut(plan_of(p), a.query_tail, 0, fwd_block_rows(p->dtype, p->head_dim), fwd_tile_rows(p->dtype, p->head_dim), fp32,
                                        p->head_dim);
  {
    const ExpandJob ex = prepare_bias(p, a, ws, l, true, 0);
    ProfScope ps(p->reuse_schedule ? "bias_expand_fwd" : "schedule_fwd", stream);
    if (launch_schedule(a, !p->reuse_schedule, fwd_block_rows(p->dtype, p->head_dim), fwd_tile_rows(p->dtype, p->head_dim),
                        (SchedHeader*)(ws + l.header[0]), (WorkItem*)(ws + l.items[0]), (int32_t*)(ws + l.seq_base[0]),
                        (SplitItem*)(ws + l.splits), may_cut ? l.slot_cap : 0, fp32, ex, stream) != hipSuccess)
      return HSTU_ERR_LAUNCH;
  }
  {
    ProfScope ps("attn_fwd", stream);                      // includes the kernel that adds up the pieces of cut blocks
    if (launch_attn_fwd(a, p->dtype, stream) != hipSuccess) return HSTU_ERR_LAUNCH;
    if (may_cut && launch_fwd_finish(a, p->dtype, a.header, a.splits, a.partial, stream) != hipSuccess) return HSTU_ERR_LAUNCH;
  }
  return HSTU_OK;
}

int hstu_attn_bwd(const hstu_attn_params* p, const void* q, const void* k, const void* v, const void* dout, void* dq,
                  void* dk, void* dv, void* workspace, size_t workspace_bytes, void* stream_) {
  return hstu::attn_bwd_through_silu(p, q, k, v, nullptr, nullptr, nullptr, 0, dout, dq, dk, dv, workspace, workspace_bytes, nullptr, 0, stream_);
}

}  // extern "C"

int hstu::attn_bwd_through_silu(const hstu_attn_params* p, const void* q, const void* k, const void* v, const void* pre_q,
                                const void* pre_k, const void* pre_v, int64_t s_pre, const void* dout, void* dq, void* dk,
                                void* dv, void* workspace, size_t workspace_bytes, void* ds, size_t ds_bytes, void* stream_) {
  const int st = validate(p);
  if (st != HSTU_OK) return st;
  if (pre_q || pre_k || pre_v) {
    if (p->dtype != HSTU_BF16) return HSTU_ERR_UNSUPPORTED;
    if (!pre_q || !pre_k || !pre_v) return HSTU_ERR_NULL;
    if (misaligned(pre_q) || misaligned(pre_k) || misaligned(pre_v) || s_pre % 8 != 0 ||
        s_pre < (int64_t)p->num_heads * p->head_dim)
      return HSTU_ERR_SHAPE;
  }
  if (p->query_tail > 0) return HSTU_ERR_UNSUPPORTED;    // the query tail is a forward (inference) feature
  if (p->total_tokens == 0 || p->batch == 0) {           // no pairs: the only output that still exists is a zero table gradient
    if (p->d_rab_table &&
        launch_fill_zero(p->d_rab_table, (size_t)p->num_heads * p->num_buckets, (hipStream_t)stream_) != hipSuccess)
      return HSTU_ERR_LAUNCH;
    return HSTU_OK;
  }
  if (!q || !k || !v || !dout || !dq || !dk || !dv) return HSTU_ERR_NULL;
  if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(dout) || misaligned(dq) || misaligned(dk) ||
      misaligned(dv))
    return HSTU_ERR_SHAPE;
  const Layout l = make_layout(p, 1);
  if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < l.total) return HSTU_ERR_WORKSPACE;
  hipStream_t stream = (hipStream_t)stream_;
  unsigned char* ws = (unsigned char*)workspace;

  AttnArgs a = make_args(p, q, k, v);
  a.dout = dout; a.dq = dq; a.dk = dk; a.dv = dv;
  a.pre_q = pre_q; a.pre_k = pre_k; a.pre_v = pre_v; a.s_pre = s_pre;
  if (!ds) {                                             // behind everything else: a workspace without that room is accepted
    ds = ws + l.total;
    ds_bytes = workspace_bytes - l.total;
  }
  const bool through_ds = l.ds_bytes != 0 && ds_bytes >= l.ds_bytes;
  const int rows[2] = {dq_block_rows(p->dtype, p->head_dim), dkv_block_rows(p->dtype, p->head_dim)};
  const int cols[2] = {stream_tile_rows(p->dtype, p->head_dim), dkv_tile_rows(p->dtype, p->head_dim)};
  bool may_cut[2];                                       // as in the forward
  const bool fp32 = p->dtype == HSTU_FP32;
  for (int s = 0; s < 2; ++s) may_cut[s] = schedule_may_cut(plan_of(p), 0, 1 + s, rows[s], cols[s], fp32, p->head_dim);
  {
    const ExpandJob ex = prepare_bias(p, a, ws, l, false, through_ds ? kDbiasLead : 0);
    ProfScope ps(p->reuse_schedule ? "bias_expand_bwd" : "schedule_bwd", stream);
    SchedHeader* const hd[2] = {(SchedHeader*)(ws + l.header[0]), (SchedHeader*)(ws + l.header[1])};
    WorkItem* const it[2] = {(WorkItem*)(ws + l.items[0]), (WorkItem*)(ws + l.items[1])};
    int32_t* const sb[2] = {(int32_t*)(ws + l.seq_base[0]), (int32_t*)(ws + l.seq_base[1])};
    SplitItem* const sp[2] = {(SplitItem*)(ws + l.splits_dq), (SplitItem*)(ws + l.splits)};
    const int caps[2] = {may_cut[0] ? l.slot_cap_dq : 0, may_cut[1] ? l.slot_cap : 0};
    // (the table of dS tiles goes with the lists, whether this call has room for dS or not: a later one that reuses them decides for itself)
    if (launch_schedule_pair(a, !p->reuse_schedule, rows, cols, hd, it, sb, sp, caps, fp32, l.ds_table ? (int32_t*)(ws + l.ds_table) : nullptr, ex,
                             stream) != hipSuccess)
      return HSTU_ERR_LAUNCH;
  }
  const SchedHeader* headers[2];
  const SplitItem* const splits[2] = {(const SplitItem*)(ws + l.splits_dq), (const SplitItem*)(ws + l.splits)};
  const float* const partial[2] = {(const float*)(ws + l.partial_dq), (const float*)(ws + l.partial)};
  if (through_ds) {
    a.ds = ds;
    a.ds_table = (const int32_t*)(ws + l.ds_table);
    a.ds_pair0 = (const int32_t*)(ws + l.seq_base[1]);
    a.ds_cap = std::min((int64_t)(ds_bytes / kDsTileBytes), (int64_t)0x7FFFFFFF);
    for (int s = 0; s < 2; ++s) a.ds_lists[s] = (SchedHeader*)(ws + l.header[s]);
  }
  for (int i = 0; i < 2; ++i) {
    const int s = through_ds ? 1 - i : i;                // s = 0: dQ pass (query blocks), s = 1: dK/dV pass (key blocks)
    a.max_items = l.max_items[s];
    a.header = headers[s] = (const SchedHeader*)(ws + l.header[s]);
    a.items = (const WorkItem*)(ws + l.items[s]);
    a.partial = const_cast<float*>(partial[s]);
    a.splits = splits[s];
    ProfScope ps(s == 0 ? "attn_bwd_dq" : "attn_bwd_dkdv", stream);
    const hipError_t e = s == 1 ? launch_attn_bwd_dkdv(a, p->dtype, stream)
                                : (through_ds ? launch_attn_dq_from_ds(a, stream) : launch_attn_bwd_dq(a, p->dtype, stream));
    if (e != hipSuccess) return HSTU_ERR_LAUNCH;
  }
  for (int s = 0; s < 2; ++s)
    if (!may_cut[s]) headers[s] = nullptr;
  DbiasJob db = {};
  if (p->d_rab_table) db = {p->rab_bounds, p->num_buckets, p->d_rab_table};
  {
    ProfScope ps("attn_bwd_finish", stream);             // the pieces of cut blocks, the bias-table gradient
    if (launch_bwd_finish(a, p->dtype, headers, splits, partial, db, stream) != hipSuccess) return HSTU_ERR_LAUNCH;
  }
  return HSTU_OK;
}

extern "C" {

int hstu_attn_schedule_stats(const hstu_attn_params* p, const void* workspace, int for_backward, int64_t out[3]) {
  const int st = validate(p);
  if (st != HSTU_OK) return st;
  if (!workspace || !out) return HSTU_ERR_NULL;
  const Layout l = make_layout(p, for_backward);
  SchedHeader h;
  if (hipMemcpy(&h, (const unsigned char*)workspace + l.header[0], sizeof(h), hipMemcpyDeviceToHost) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  out[0] = h.count; out[1] = h.tiles; out[2] = h.dense_tiles;
  return h.bad_batch ? HSTU_ERR_SHAPE : HSTU_OK;          // the scheduler found the device-side offsets inconsistent
}

static int validate_norm(int64_t T, int32_t D, int32_t dtype) {
  if (T < 0 || D < 1) return HSTU_ERR_SHAPE;
  if (dtype != HSTU_BF16 && dtype != HSTU_FP32) return HSTU_ERR_UNSUPPORTED;
  if (D % 8 != 0 || D > 8192) return HSTU_ERR_UNSUPPORTED;
  return HSTU_OK;
}

int hstu_gated_norm_fwd(int64_t T, int32_t D, int32_t dtype, const void* attn, const void* u, const float* gamma,
                        const float* beta, float eps, void* y, float* mean, float* rstd, void* stream) {
  const int st = validate_norm(T, D, dtype);
  if (st != HSTU_OK) return st;
  if (T == 0) return HSTU_OK;
  if (!attn || !u || !gamma || !y) return HSTU_ERR_NULL;
  if (misaligned(attn) || misaligned(u) || misaligned(gamma) || misaligned(y) || (beta && misaligned(beta))) return HSTU_ERR_SHAPE;
  ProfScope ps("gated_norm_fwd", (hipStream_t)stream);
  if (launch_gated_norm_fwd(T, D, dtype, attn, u, gamma, beta, eps, y, mean, rstd, (hipStream_t)stream) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

size_t hstu_gated_norm_bwd_workspace_bytes(int64_t T, int32_t D) {
  if (T < 0 || D < 1) return 0;
  const size_t blocks = (size_t)gated_norm_bwd_blocks(T, D);
  return align_up((blocks > 0 ? blocks : 1) * 2 * (size_t)D * sizeof(float));
}

int hstu_gated_norm_bwd(int64_t T, int32_t D, int32_t dtype, const void* dy, const void* attn, const void* u,
                        const float* gamma, const float* beta, float eps, void* dattn, void* du, float* dgamma,
                        float* dbeta, void* workspace, size_t workspace_bytes, void* stream) {
  const int st = validate_norm(T, D, dtype);
  if (st != HSTU_OK) return st;
  if (!gamma || !dgamma) return HSTU_ERR_NULL;
  if (T > 0 && (!dy || !attn || !u || !dattn || !du)) return HSTU_ERR_NULL;
  if (misaligned(dy) || misaligned(attn) || misaligned(u) || misaligned(gamma) || misaligned(dattn) || misaligned(du) ||
      (beta && misaligned(beta)))
    return HSTU_ERR_SHAPE;
  if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < hstu_gated_norm_bwd_workspace_bytes(T, D))
    return HSTU_ERR_WORKSPACE;
  ProfScope ps("gated_norm_bwd", (hipStream_t)stream);
  if (launch_gated_norm_bwd(T, D, dtype, dy, attn, u, gamma, beta, eps, dattn, du, dgamma, dbeta, (float*)workspace,
                            (hipStream_t)stream) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

// ---- the gated-norm backward for callers that cannot allocate -------------------------------------------------
// Same kernels as hstu_gated_norm_bwd; the partial column sums live in a file-scope device array instead of a
// caller-provided workspace.  In host code the array's name is only a stand-in: the address the kernels get is the one
// hipGetSymbolAddress reports for the current device (every GPU holds its own copy), looked up once per device.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxScratchDevices = 64;
static void* g_scratch_ptr[kMaxScratchDevices];
static std::mutex g_scratch_mutex;

static int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return HSTU_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return HSTU_ERR_LAUNCH;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return HSTU_OK;
}

size_t hstu_gated_norm_bwd_static_max_bytes(void) { return kStaticScratchBytes; }

int hstu_gated_norm_bwd_static(int64_t T, int32_t D, int32_t dtype, const void* dy, const void* attn, const void* u,
                               const float* gamma, const float* beta, float eps, void* dattn, void* du, float* dgamma,
                               float* dbeta, void* stream) {
  const int st = validate_norm(T, D, dtype);
  if (st != HSTU_OK) return st;
  if (!gamma || !dgamma) return HSTU_ERR_NULL;
  if (T > 0 && (!dy || !attn || !u || !dattn || !du)) return HSTU_ERR_NULL;
  if (misaligned(dy) || misaligned(attn) || misaligned(u) || misaligned(gamma) || misaligned(dattn) || misaligned(du) ||
      (beta && misaligned(beta)))
    return HSTU_ERR_SHAPE;
  if (hstu_gated_norm_bwd_workspace_bytes(T, D) > kStaticScratchBytes) return HSTU_ERR_WORKSPACE;
  void* partial = nullptr;
  const int sp = static_scratch(&partial);
  if (sp != HSTU_OK) return sp;
  // every workgroup overwrites the columns that are wanted of its row of partial sums (dgamma's, with a bias or its gradient also
  // dbeta's) and the column-sum kernel reads only those, of the rows of this launch: nothing left by an earlier call is
  // ever read and nothing needs clearing
  if (launch_gated_norm_bwd(T, D, dtype, dy, attn, u, gamma, beta, eps, dattn, du, dgamma, dbeta, (float*)partial,
                            (hipStream_t)stream) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

// ---- attention truncation (Section 4.3) ------------------------------------------------------------------------
static bool bad16(const void* ptr) { return ((uintptr_t)ptr & 15) != 0; }
static int validate_rows(int64_t row_bytes, int64_t stride_a, int64_t stride_b) {
  if (row_bytes < 0 || (row_bytes & 15) || (stride_a & 15) || (stride_b & 15) || stride_a < row_bytes || stride_b < row_bytes)
    return HSTU_ERR_SHAPE;
  return HSTU_OK;
}

int hstu_truncate_offsets(int32_t batch, int32_t keep, const int32_t* seq_offsets, const int32_t* num_targets,
                          int32_t* out_offsets, void* stream) {
  if (batch < 0 || keep < 0) return HSTU_ERR_SHAPE;
  if (!seq_offsets || !out_offsets) return HSTU_ERR_NULL;
  ProfScope ps("truncate_offsets", (hipStream_t)stream);
  if (launch_truncate_offsets(batch, keep, seq_offsets, num_targets, out_offsets, (hipStream_t)stream) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

int hstu_truncate_fwd(int32_t batch, const int32_t* seq_offsets, const int32_t* out_offsets, int64_t row_bytes,
                      const void* x, int64_t x_stride_bytes, void* y, int64_t y_stride_bytes, int64_t y_rows,
                      void* stream) {
  if (batch < 0 || y_rows < 0) return HSTU_ERR_SHAPE;
  const int st = validate_rows(row_bytes, x_stride_bytes, y_stride_bytes);
  if (st != HSTU_OK) return st;
  if (batch == 0 || y_rows == 0 || row_bytes == 0) return HSTU_OK;
  if (!seq_offsets || !out_offsets || !x || !y) return HSTU_ERR_NULL;
  if (bad16(x) || bad16(y)) return HSTU_ERR_SHAPE;
  ProfScope ps("truncate_fwd", (hipStream_t)stream);
  if (launch_truncate_gather(batch, seq_offsets, out_offsets, row_bytes, x, x_stride_bytes, y, y_stride_bytes, y_rows,
                             (hipStream_t)stream) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

int hstu_truncate_bwd(int32_t batch, int64_t total_tokens, const int32_t* seq_offsets, const int32_t* out_offsets,
                      int64_t row_bytes, const void* dy, int64_t dy_stride_bytes, void* dx, int64_t dx_stride_bytes,
                      void* stream) {
  if (batch < 0 || total_tokens < 0 || total_tokens > 0x7fffffff) return HSTU_ERR_SHAPE;
  const int st = validate_rows(row_bytes, dy_stride_bytes, dx_stride_bytes);
  if (st != HSTU_OK) return st;
  if (batch == 0 || total_tokens == 0 || row_bytes == 0) return HSTU_OK;
  if (!seq_offsets || !out_offsets || !dx) return HSTU_ERR_NULL;   // dy may be NULL when no row survives (never read then)
  if (bad16(dy) || bad16(dx)) return HSTU_ERR_SHAPE;
  ProfScope ps("truncate_bwd", (hipStream_t)stream);
  if (launch_truncate_scatter(batch, total_tokens, seq_offsets, out_offsets, row_bytes, dy, dy_stride_bytes, dx,
                              dx_stride_bytes, (hipStream_t)stream) != hipSuccess)
    return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

// ---- FP8 around the projections (Section 4.2.2) ------------------------------------------------------------------
int hstu_norm_quant_fp8(int64_t T, int32_t D, int32_t dtype, const void* a, const void* u, const float* gamma,
                        const float* beta, float eps, void* q, float* q_scale, float* mean, float* rstd, void* stream) {
  const int st = validate_norm(T, D, dtype);
  if (st != HSTU_OK) return st;
  if (T == 0) return HSTU_OK;
  if (!a || !q || !q_scale) return HSTU_ERR_NULL;
  if (beta && !gamma) return HSTU_ERR_NULL;
  if (misaligned(a) || (u && misaligned(u)) || (gamma && misaligned(gamma)) || (beta && misaligned(beta)) ||
      ((uintptr_t)q & 7u))
    return HSTU_ERR_SHAPE;
  NormFwdArgs p = {};
  p.T = T; p.D = D; p.dtype = dtype; p.a = a; p.sa = D; p.u = u; p.su = D; p.gamma = gamma; p.beta = beta; p.eps = eps;
  p.y = nullptr; p.sy = D; p.mean = mean; p.rstd = rstd; p.stats_in = 0;
  ProfScope ps("norm_quant_fp8", (hipStream_t)stream);
  if (launch_norm_quant_fwd(p, q, D, q_scale, (hipStream_t)stream) != hipSuccess) return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

int hstu_fp8_gemm_bias2d(int64_t M, int32_t N, int32_t K, const void* a_q, const float* a_scale, const void* b_q,
                         const float* b_scale, const void* c, void* d, void* stream) {
  if (M < 0 || N < 1 || K < 1) return HSTU_ERR_SHAPE;
  if (!fp8_gemm_supported(N, K)) return HSTU_ERR_UNSUPPORTED;
  if (M == 0) return HSTU_OK;
  if (!a_q || !a_scale || !b_q || !b_scale || !d) return HSTU_ERR_NULL;
  if (misaligned(a_q) || misaligned(b_q) || misaligned(b_scale) || (c && misaligned(c)) || misaligned(d)) return HSTU_ERR_SHAPE;
  if ((M + 127) / 128 > 0x7fffffff) return HSTU_ERR_SHAPE;
  ProfScope ps("fp8_gemm_bias2d", (hipStream_t)stream);
  if (launch_fp8_gemm_bias2d(M, N, K, a_q, a_scale, b_q, b_scale, c, d, (hipStream_t)stream) != hipSuccess) return HSTU_ERR_LAUNCH;
  return HSTU_OK;
}

}  // extern "C"
