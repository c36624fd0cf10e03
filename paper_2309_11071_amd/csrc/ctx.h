// Internal context of the library: device-resident graph store, cached per-layer tables and
// the work buffers of the per-layer event pipeline.  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "../../include/ink.h"
#include "prim.h"

namespace ink {

#ifndef INK_BIG_DEG
#define INK_BIG_DEG 256
#endif
// Neighbour rows in flight per lane group while gathering, by aggregator family and, for max / min, lanes per row.  8 where they
// gain anything: for max / min over rows of 64 floats they cost 3 % (200k nodes, inference: .549 -> .566 ms; 109 instead of 94
// registers), over 128 floats nothing is gained (625k nodes 4.00 and 4.01 ms), over 256 floats 4 instead of 8 cost 1 % (100k
// nodes .929 -> .940).
#ifndef INK_U_SEL8
#define INK_U_SEL8 4
#endif
#ifndef INK_U_SEL16
#define INK_U_SEL16 4
#endif
#ifndef INK_U_SEL32
#define INK_U_SEL32 4
#endif
#ifndef INK_U_SEL64
#define INK_U_SEL64 8
#endif
#ifndef INK_U_SUM
#define INK_U_SUM 8         // sums are cheap in registers: 8 loads in flight measured 3.5 % faster than 4 on narrow rows
#endif
#ifndef INK_BIG_CHUNK
#define INK_BIG_CHUNK 1024
#endif
constexpr int kBigChunk = INK_BIG_CHUNK;  // neighbours per chunk of such a row
#ifndef INK_BIG_CHUNK_SUM
#define INK_BIG_CHUNK_SUM 2048
#endif
// ... in long launches of sums that go by slices, whose lane groups add 64 rows in a chain.  1024 / 2048 / 4096, inference: GCN of
// 256 columns on 29k nodes, 490 neighbours each, 1.25 / 1.22 / 1.22 ms, on 100k nodes, 200 each, 2.30 / 2.27 / 2.22; GIN of 128 on
// 400k, 20 each, 1.33 / 1.31 / 1.32, on 20k, 50 each, .204 / .202 / .213.  Whole rows keep 1024: with 2048 their chains are twice as
// long, and the error of a long row against 64 bits grew by a fifth to two fifths (41 columns 1.34e-7 -> 1.61e-7, 256 columns of a table
// beyond 2 GB 2.9e-7 -> 4.0e-7; slices 1.6e-7).  Max / min at 2048 lose: 60k nodes, 50 each, .480 -> .506.
constexpr int kBigChunkSum = INK_BIG_CHUNK_SUM;
static_assert(kBigChunk <= kBigChunkSum, "buffer bounds of the long-row path use the smaller chunk");
#ifndef INK_BIG_DEG_SUM
#define INK_BIG_DEG_SUM 1024
#endif
// rows with more in-neighbours are re-gathered cooperatively (bigrows.h): kBigDeg for max / min,
// whose per-neighbour work is heavier, kBigDegSum for the sum-type aggregators (both measured)
constexpr int kBigDeg = INK_BIG_DEG;
constexpr int kBigDegSum = INK_BIG_DEG_SUM;
static_assert(kBigDeg <= kBigDegSum, "buffer bounds of the long-row path use the smaller threshold");
constexpr uint32_t kEvKindShift = 30;
constexpr uint32_t kEvIdMask = (1u << kEvKindShift) - 1;
enum : uint32_t { EV_DEL = 0, EV_ADD = 1, EV_CHG = 2 };   // removed edge / inserted edge / changed source

// One direction of the graph store: per-node edge blocks with slack inside one id pool.
struct GraphSide {
  int64_t *off = nullptr;    // [n] first slot of the node's block
  int32_t *deg = nullptr;    // [n] used slots
  int32_t *cap = nullptr;    // [n] block capacity
  uint8_t *asc = nullptr;    // [n] 1 while the block's ids are ascending (true until the node's first applied op)
  int32_t *ids = nullptr;    // pool
  int64_t pool_cap = 0;      // slots in the pool
  int64_t pool_top = 0;      // first free slot (host mirror, exact)
};

struct Table {               // N x d float (or int) table with row stride ld (multiple of 4)
  void *p = nullptr;
  int d = 0, ld = 0;
  float *f() const { return (float *)p; }
  int32_t *i() const { return (int32_t *)p; }
};

struct DevLayer {
  int in_dim = 0, out_dim = 0, hidden = 0, act = 0;
  // first (or only) linear map: rows = K (padded to a multiple of 32), cols = ldw (multiple of 32)
  float *W1 = nullptr; int K1 = 0, K1p = 0, N1 = 0, N1p = 0; float *b1 = nullptr;
  float *W2 = nullptr; int K2 = 0, K2p = 0, N2 = 0, N2p = 0; float *b2 = nullptr;   // GIN second linear
};

constexpr int64_t kShortBatch = 16384;     // largest batch of the short form of the graph stage
constexpr int64_t kPinnedBatch = 1024;     // host batches up to this size are read by the device from pinned memory

// A layer of at most this many events can run in one workgroup (layer_one.hip), which leaves in slot C_ONE how far it came.
constexpr int kOneEvents = 32;
enum { kOneNothing = 0, kOneEventsDone, kOneDone };

constexpr int kStripes = 64;
enum { ST_EXPOSED = 0, ST_REGATHER, ST_ACHG, ST_NODEL, ST_NOEFFECT, ST_COVERED, ST_REGATHER_LONG, ST_PAD7, ST_N };
struct Counters {            // device-written, host-read through pinned memory
  int32_t v[32];
  // statistics that many waves bump: striped by workgroup so that no single address is contended
  unsigned long long stripe[kStripes][ST_N];
  unsigned long long sum(int which) const {
    unsigned long long t = 0;
    for (int i = 0; i < kStripes; i++) t += stripe[i][which];
    return t;
  }
};
// what the host sees of them: the slots and the stripe totals (192 bytes through pinned memory)
struct HostCounters {
  int32_t v[32];
  unsigned long long total[ST_N];
  unsigned long long sum(int which) const { return total[which]; }
};
// slots of Counters::v: event count of the next layer, unique targets, long rows listed, rows to
// transform, rows changed, chunks of long rows, distinct ops of a batch, scratch of the graph stage,
// (C_NEXP: exposed rows of moderate length listed for the recompute, next to the long ones in C_NBIG)
// touched nodes and block chunks of the out side (single-workgroup graph stage), and two 64-bit
// slots (pool tops handed to the apply kernels).  Slot 0 flags a malformed update batch.
// (C_NEVL, C_NEVCH: targets with a long event segment and the chunks of those segments)
// The graph stage of short batches has a block of its own (ink_ctx::d_gcnt): next to the slots above it holds
// the pool space each side needs (stripe 0, words 0 and 1), the effective ops as the out side sees them, the effective ops
// of the in side whether or not the apply kernel may run (C_GINS, C_GDEL) and whether it may (C_OK).
enum { C_ERR = 0, C_NEV = 1, C_NT, C_NEXP, C_NCHUNK, C_NBIG, C_NEVL, C_NEVCH, C_NC, C_NEXT, C_NOPS, C_TMP0, C_TMP1,
       C_TMP2, C_TMP3, C_OT, C_OCH, C_TOP64 = 18, C_TOP64B = 20,
       C_OINS = 22, C_ODEL, C_GINS, C_GDEL, C_OK, C_ONE = 31 };

// The counters reach the host through pinned host memory: one wave writes the slots and the
// stripe totals, then a sequence number that the host polls.  A blocking stream synchronisation
// costs an interrupt round trip per read-back, and a short batch has four of them.  The loads
// bypass the L1 so that a workgroup may publish what its own threads stored before a barrier.
static_assert(kStripes == kWave, "one stripe per lane");
__device__ __forceinline__ void publish_wave(const Counters *d, HostCounters *h, uint32_t *h_seq, uint32_t seq) {
  const int l = lane_id();
  if (l < 32) h->v[l] = __hip_atomic_load(&d->v[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // lane l adds counter l % 8 of every eighth stripe: eight coalesced loads and three exchanges (a tree of exchanges per
  // counter made the record 2 us longer)
  static_assert(ST_N == 8, "eight counters a stripe");
  const unsigned long long *p = &d->stripe[0][0];
  unsigned long long t = 0;
#pragma unroll
  for (int k = 0; k < kStripes * ST_N; k += kWave) t += __hip_atomic_load(p + k + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int o = ST_N; o < kWave; o <<= 1) t += __shfl_xor(t, o, kWave);
  if (l < ST_N) h->total[l] = t;
  __threadfence_system();
  if (l == 0) __hip_atomic_store(h_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace ink

struct ink_ctx {
  int n = 0;
  int64_t n_edges = 0, n_edges_now = 0;
  int64_t pool_reserve = 0;
  int64_t n_cap = 0;          // node capacity: every per-node array has this many entries (>= n)
  int64_t big_hint[INK_MAX_LAYERS + 1] = {0};   // chunks of long rows seen by the last update at each layer
  double dense_frac = 0;             // events / edges above which a layer re-aggregates every node; 0: by aggregator and width
  int id_bits = 1;
  int kind = 0, agg = 0, n_layers = 0, mem = 0, profile = 0;
  float eps = 0.f, slack = 0.25f;
  bool batch_dev = false;
  bool affected_mode = false;        // current call is the affected-area recompute baseline
  bool is_select = true, is_min = false, inferred = false, own_stream = false;
  bool drained = false;              // the last record read back covers everything the call launched
  bool broken = false;               // an updating call failed on the device side: state may be half-written
  hipStream_t stream = nullptr;
  int device = 0;                    // HIP device the context lives on
  void *scratch = nullptr;           // that device's copy of the static work array of ink_full_infer_noalloc
  std::string err;

  ink::GraphSide gin, gout;
  int32_t *new_out = nullptr;        // [n] out-edges appended by the current batch (tail of the block)
  std::vector<ink::DevLayer> layers;
  // tables: H[0..k]; A[1..k] aggregated (sum-type: plain sums); ARG[1..k]
  std::vector<ink::Table> H, A, ARG, UB, ARG2;   // UB / ARG2: max/min only, bound on the runner-up value and its holder when known
  // GCN only: XW[l] = unscaled transformed messages h_{l-1} W_l, H-like scaled copies live in Msc[l]
  std::vector<ink::Table> XW, Msc;
  float *cnorm = nullptr;            // GCN: (indeg + 1)^(-1/2) per node
  std::vector<ink::Table> USER;      // per layer: the term of user-defined events (allocated by the first event of the layer)
  ink::DevBuf u_ev, u_rows, u_key, u_val, u_uniq, u_seg, u_flag, u_idx, u_list;   // work buffers of ink_apply_user_events

  ink::PrimWorkspace ws;
  ink::Counters *d_cnt = nullptr;    // device counters
  ink::HostCounters *h_cnt = nullptr;   // pinned host mirror, written by the publish kernel
  uint32_t *h_seq = nullptr;         // (same allocation) sequence number of the last published copy
  uint32_t pub_seq = 0;
  ink::Counters *d_gcnt = nullptr;   // the graph stage's own block, its pinned mirror and sequence number
  ink::HostCounters *h_gcnt = nullptr;
  uint32_t *h_gseq = nullptr;
  ink::HostCounters *h_one[INK_MAX_LAYERS + 1] = {nullptr};   // records of the layers that ran in one workgroup, and
  uint32_t *h_oseq[INK_MAX_LAYERS + 1] = {nullptr};           // their sequence numbers (pinned)
  uint32_t one_seq[INK_MAX_LAYERS + 1] = {0};                 // what to wait for
  ink_edge_update *h_batch = nullptr;   // pinned staging of short host batches
  int64_t small_batch = 16384;       // batches up to this size take the short form of the graph stage
  uint64_t *bm_a = nullptr;          // node bitmaps (n bits each)

  // batch buffers (grown on demand)
  int64_t n_touched_src = 0;         // sources whose out-block got new ids in the current batch
  ink::DevBuf b_raw, b_uniq, b_misc;
  int32_t *del_src = nullptr, *del_dst = nullptr, *ins_src = nullptr, *ins_dst = nullptr;  // Delta E lists
  ink::DevBuf b_del_s, b_del_d, b_ins_s, b_ins_d;
  int64_t n_del = 0, n_ins = 0;

  // per-layer pipeline buffers
  ink::DevBuf f_list[2];             // F_l (ascending node ids), ping-pong between layers
  ink::DevBuf f_old[2];              // old message rows of F_l (sum-type aggregators)
  ink::DevBuf f_pref;                // prefix of out-degrees over F_l
  ink::DevBuf f_delta;               // new - old message rows of F_l (sum-type aggregators)
  ink::DevBuf ev_key, ev_val;        // events
  ink::DevBuf t_list, t_seg;         // unique targets, segment offsets
  ink::DevBuf c_list, c_flag, c_idx; // rows to transform, per-row changed flag, compacted positions
  ink::DevBuf c_old;                 // previous table rows of the transformed rows (sum-type)
  ink::DevBuf b_touch_in;            // destinations touched by the current batch
  int64_t n_touched_in = 0;
  ink::DevBuf exp_list;              // exposed rows of moderate length, listed by the event kernel
  ink::DevBuf evl_list, evl_owner;   // targets with long event segments, and the owner of each chunk of them
  int32_t *arrived = nullptr;        // [kLatencyTargets] parts of a row or segment that are there, in a launch that combines them itself; 0 between launches (behind d_gcnt)
  ink::DevBuf big_list, big_part_v, big_part_i, big_part_s, big_part_j, big_pref;   // cooperative re-gather of long rows
  ink::DevBuf stage0, stage1;        // transform staging
  ink::DevBuf res_ids, res_emb;      // result of the last batch

  // the last result (n < 0: none), and its copy in pinned memory: where the kernel that gathers a result writes it, too
  struct Result { const int32_t *ids = nullptr; const float *rows = nullptr; int64_t n = -1; } last;
  char *h_res = nullptr;             // INK_RESULT_HOST_BYTES, allocated with a context for batches in host memory, otherwise by the first ink_copy_result
  bool mirror = false;               // results are asked for on the host
  bool mirrored = false;             // the last one was written there if it fits
  bool fetched = true;               // ... and has been asked for
  int64_t mirror_rows() const { return INK_RESULT_HOST_BYTES / (4 + 4 * (int64_t)H[n_layers].d) / 4 * 4; }
  int32_t *mirror_ids() const { return reinterpret_cast<int32_t *>(h_res); }
  float *mirror_emb() const { return reinterpret_cast<float *>(h_res) + mirror_rows(); }

  ink_stats stats;
  struct Pending { int cls, layer, kern; hipEvent_t a, b; };
  std::vector<hipEvent_t> ev_free;
  std::vector<Pending> ev_pending;
};

namespace ink {

// Times what is launched during its life with a pair of HIP events on the context's stream (only
// while profiling is on): into the class total `cls` (>= 0) and / or into kernel slot `kern` of
// layer `layer` (1-based).  Launch counts per class are always kept.
struct Prof {
  ink_ctx *c; int cls, layer, kern; hipEvent_t a = nullptr, b = nullptr;
  Prof(ink_ctx *c_, int cls_, int layer_ = 0, int kern_ = -1) : c(c_), cls(cls_), layer(layer_), kern(kern_) {
    if (cls >= 0) c->stats.launches[cls]++;
    if (!c->profile) return;
    while (c->ev_free.size() < 2) { hipEvent_t e; if (hipEventCreate(&e) != hipSuccess) return; c->ev_free.push_back(e); }
    a = c->ev_free.back(); c->ev_free.pop_back();
    b = c->ev_free.back(); c->ev_free.pop_back();
    (void)hipEventRecord(a, c->stream);
  }
  ~Prof() {
    if (!a) return;
    (void)hipEventRecord(b, c->stream);
    c->ev_pending.push_back({cls, layer, kern, a, b});
  }
};
struct KernelTimer : Prof {
  KernelTimer(ink_ctx *c_, int layer_, int kern_) : Prof(c_, -1, layer_, kern_) {}
};

// ---- graph store (graph.hip)
hipError_t graph_build(ink_ctx *c, const int64_t *rowptr_h, const int32_t *col_h);
// applies a batch in memory the device can read (ink_edge_update records); fills Delta E lists and counts
// `queued`, if given, launches the one-workgroup form of the stage with the layers behind it (layer_one.hip); its record has the number it gets
struct RawUpdate { uint8_t op; uint8_t pad[3]; int32_t src, dst; };
struct OneSide { int64_t *off; int32_t *deg, *cap, *ids; uint8_t *asc; int32_t *new_cnt, *uniq; long long pool_base, room; };
struct OneGraph {
  const RawUpdate *raw; int n, n_nodes;
  OneSide in, out;
  int32_t *ins_s, *ins_d, *del_s, *del_d;          // applied edge changes
  float slack;
};
ink_status graph_apply_batch(ink_ctx *c, const void *raw, int64_t n, int64_t *n_ins, int64_t *n_del,
                             hipError_t (*queued)(ink_ctx *, const OneGraph &, uint32_t) = nullptr);
hipError_t graph_reserve(ink_ctx *c, int64_t max_batch);   // batch buffers for that many entries
ink_status graph_add_nodes(ink_ctx *c, int64_t n_new);   // empty edge blocks for nodes n .. n + n_new - 1 (before n grows)
hipError_t read_counters(ink_ctx *c, bool end_batch = false);   // device counters -> c->h_cnt, waits for them; with end_batch as graph_end_batch on the way
hipError_t wait_published(ink_ctx *c, const uint32_t *h_seq, uint32_t seq);   // until that record has arrived
hipError_t graph_end_batch(ink_ctx *c);     // clears per-batch marks (new_out)
hipError_t graph_export(ink_ctx *c, int64_t *rowptr_h, int32_t *col_h);

// ---- aggregation (agg.hip)
// Rows that are re-gathered in chunks (bigrows.h): node and first chunk of each, in ascending order of both; the counters
// C_NCHUNK and C_NBIG are one 64-bit word, so that one atomic takes a row's place and its chunks'.
struct BigRows { int32_t *list, *base; int chunk; };
static_assert(C_NCHUNK % 2 == 0 && C_NBIG == C_NCHUNK + 1, "chunks in the lower half, rows in the upper");
struct AggArgs {
  int n;
  const int64_t *in_off; const int32_t *in_deg; const int32_t *in_ids;
  const float *M; int ldm;          // message table
  float *A; int32_t *ARG; int ld;   // aggregated table and argument table (row stride ld)
  float *UB;                        // max/min: bound on the best value among the non-holders (same layout)
  const uint8_t *in_asc;            // per node: in-list ascending by id (asked only for rows with infinities or NaN: equal values leave the first its place)
  int32_t *ARG2;                    // max/min: the non-holder that has exactly that value (lowest id), or -1 if not known
  bool keep_empty;                  // recompute of every row: those without neighbours keep what they have unless their bit is set
  int d;                            // columns handled by this launch (<= 256; wider rows go block by block)
  int wd;                           // d rounded up to 4
  bool is_min;
  bool nonneg;                      // no message has its sign bit set (the layer before ends in ReLU, which gives +0 for every other value)
  int big_deg;                      // rows with more in-neighbours go to the chunked cooperative path
  BigRows big;                      // its list
  int64_t big_chunks;               // its chunks, about: what the chunk kernel is launched for (it strides if there are more)
  int layer;                        // 1-based layer the launch belongs to (per-kernel timing)
  int count_cond;                   // tally the per-target condition counters (only the first 256-column block of a wide row does)
};
// full re-aggregation of every node (targets == nullptr) or of a target list; flags rows whose
// alpha changed in bitmap `chg` (may be null); big rows go through the cooperative path
hipError_t agg_select_full(ink_ctx *c, const AggArgs &a, const int32_t *targets, int64_t n_targets,
                           uint64_t *chg);
struct EventBounds { int64_t n_events, max_seg; };    // events of the layer; most events one target can have
// n_targets may be an upper bound of the device-side count *n_targets_dev
hipError_t agg_select_events(ink_ctx *c, const AggArgs &a, const int32_t *targets, const int32_t *seg,
                             int64_t n_targets, const int32_t *n_targets_dev, const uint32_t *ev_val, const EventBounds &eb,
                             uint64_t *chg);
// the long exposed rows that the event stage of a layer listed (at most n_targets), as agg_select_events ends
hipError_t agg_select_long_rows(ink_ctx *c, const AggArgs &a, int64_t n_targets, uint64_t *chg);
hipError_t agg_select_reserve(ink_ctx *c, AggArgs &a);      // its buffers, before the list is filled (and the list's place in a)
int agg_select_long_degree(const AggArgs &a, int64_t n_targets);   // rows with more neighbours are listed
// sum-type aggregators (agg_sum.hip): A holds the plain sum of message rows.  F (ascending ids)
// and f_old (their previous message rows, row stride ld_old) describe the changed sources.
hipError_t agg_sum_full(ink_ctx *c, const AggArgs &a, const int32_t *targets, int64_t n_targets, uint64_t *chg);
hipError_t agg_sum_events(ink_ctx *c, const AggArgs &a, const int32_t *targets, const int32_t *seg,
                          int64_t n_targets, const int32_t *n_targets_dev, const uint32_t *ev_val, const EventBounds &eb,
                          const int32_t *F, int nF, const float *f_old, const float *f_delta, int ld_old, uint64_t *chg);
// f_delta[i] = M[F[i]] - f_old[i] (row stride ld_old): what a kept edge of changed source i adds
hipError_t agg_sum_delta_rows(ink_ctx *c, const AggArgs &a, const int32_t *F, int nF, const float *f_old,
                              float *f_delta, int ld_old);

// ---- dense transform (xform.hip)
struct XformArgs {
  int mode;                 // 0 SAGE concat [A | Hprev], 1 GIN (1+eps) Hprev + A, 2 dense rows,
                            // 3 GCN: x = act(c_v (A + Hp) + in_bias), with A = neighbour sums, Hp = own scaled message
  const int32_t *rows;      // row ids (null: identity)
  int64_t n_rows;           // rows to transform; an upper bound when n_rows_dev is set
  const int32_t *n_rows_dev;   // optional device-side row count (<= n_rows)
  const float *A; int lda;  // aggregated table
  const float *Hp; int ldh; // previous-layer table (or dense input for mode 2)
  int d_in;
  float eps;
  const float *W; int Kp; int Np; const float *bias; int n_out; int relu;
  // output: either staging (dense [n_rows][ld_out]) or table rows with compare-and-emit
  float *out; int ld_out; int to_table;
  uint8_t *row_changed;     // [n_rows] set to 1 if the table row changed bitwise (to_table)
  float *old_rows; int ld_old;   // optional copy of the previous table rows ([n_rows][ld_old])
  const int32_t *out_rows;  // table row ids for to_table when the input is dense (mode 2); null: identity
  const int32_t *mean_deg;  // modes 0/1 with mean aggregation: A is divided by max(deg, 1)
  const float *cnorm;       // mode 3: per-node c_v
  const float *in_bias; int in_relu;   // mode 3
  const float *in_user; int ld_in_user;   // mode 3: per-node term added after in_bias, before the activation; null: none
  float *h_store; int ld_hs;           // mode 3: where x (= h_l) is written, one row per node
  const float *out_scale;   // per-node factor applied to the output row (after bias), null: none
  const float *user; int ld_user;      // per-node term added after the bias, before the activation (to_table only), null: none
};
hipError_t xform_run(ink_ctx *c, const XformArgs &x);
// SAGE: row of the padded weight matrix where W_self starts (both halves of the input at multiples of 4)
__host__ __device__ inline int xform_self_row(int in_dim) { return (in_dim + 3) & ~3; }
// ---- the layers of a small update in one workgroup (layer_one.hip)
constexpr int kRecordBytes = 256;                  // a layer's record: HostCounters and its sequence number behind them
struct OneLayer {
  AggArgs a;                                       // with big_deg of a short launch
  int lanes;                                       // lanes per row
  const float *Hp; int ldh; int d_in;              // SAGE transform
  const float *W; int Kp, Np; const float *bias; int n_out, relu;
  const float *user; int ld_user;
  float *out; int ld_out;
};
struct OneUpdate {
  OneGraph graph;
  Counters *g, *cnt;                               // graph stage's counters; where a layer that is not finished leaves its own
  int32_t *f_list[2], *pref;                       // changed sources that layer l leaves: [l & 1]; prefix of their kept out-edges
  const int64_t *out_off; const int32_t *out_ids, *out_deg; int32_t *new_out; const int32_t *touched_src;
  int32_t *t_list; uint64_t *bm;
  float *res;                                      // the changed rows of the last layer, packed
  int32_t *h_ids; float *h_emb;                    // ... and ids and rows in pinned memory (null: not wanted there)
  char *h; uint32_t seq;                           // record of layer 1, the others behind it; its sequence number, those of the others follow
  char *h_graph; uint32_t graph_seq;               // record of the graph stage
  int n_layers;
  OneLayer layer[INK_MAX_LAYERS];
};
static_assert(sizeof(OneUpdate) <= 4096, "fits a launch's arguments");
hipError_t layers_one(ink_ctx *c, OneUpdate &p);
// position of W[k][col] in the padded device copy: k-chunks of 32, in a chunk one tile per 32 columns, in the order
// in which a wave loads its operands of the tile's 16 two-k steps: lane (k % 2) * 32 + col % 32 needs k % 32 / 2 = 0 .. 15,
// four of them per 16-byte load, and the 64 lanes of a load are contiguous
inline size_t xform_weight_index(int k, int col, int Np) {
  const int lane = (k & 1) * 32 + col % 32, step = (k % 32) >> 1;
  return (size_t)(k / 32) * 32 * Np + (size_t)(col / 32) * 1024 + (size_t)(step / 4) * 256 + (size_t)lane * 4 + (size_t)(step % 4);
}

}  // namespace ink
