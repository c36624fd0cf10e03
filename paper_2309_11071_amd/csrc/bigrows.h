// Work list for rows with more than kBigDeg in-neighbours: each such row is cut into chunks of
// kBigChunk neighbours (kBigChunkSum for long launches of sums), one workgroup per chunk, then one wave per row combines its chunks in
// order; in short launches of few chunks the wave that finishes a row's last chunk does.  A row takes its chunks when it is listed, so the plan stands when the list does (a scan of the list for it was one or
// two launches more), and the chunk / row kernels run a fixed grid that strides over it, so no host round trip is
// needed; with no long rows they return at once.
#pragma once
#include "ctx.h"

namespace ink {

constexpr int kBigGrid = 4096;             // workgroups of the per-row combine kernel

// Few targets (small batches): latency matters more than throughput, so rows are handed to the
// cooperative path much earlier and each chunk is shared by 16 waves instead of 4.
constexpr int kLatencyTargets = 8192;

// upper bound of the long rows one launch can list: with at most kLatencyTargets targets every
// target may be one, otherwise a long row has more than kBigDeg in-neighbours; never more than nodes
inline int64_t big_rows_capacity(const ink_ctx *c) {
  int64_t e = c->n_edges_now > c->n_edges ? c->n_edges_now : c->n_edges;
  int64_t r = e / kBigDeg > kLatencyTargets ? e / kBigDeg : kLatencyTargets;
  return (r < c->n_cap ? r : c->n_cap) + 1;
}
// ... and of their chunks: a row of deg neighbours has at most deg / chunk + 1
inline int64_t big_chunk_capacity(const ink_ctx *c) {
  int64_t e = c->n_edges_now > c->n_edges ? c->n_edges_now : c->n_edges;
  return e / kBigChunk + big_rows_capacity(c);
}

// Workgroups of a chunk kernel: one per expected chunk and slice (the hardware balances them; in a short launch one per chunk, whose
// slices are kSlicedItems at most or strided over), no more than there can be,
// and otherwise at least what fills the chip (1024 threads each in a short launch, 256 in a long one).  Most updates have no long
// row, and empty workgroups cost their start: 8192 of 1024 threads, rows of 256 floats, 8.6 us, 1024 of them 2.7 (200 updates on
// 100k nodes with 10 neighbours each 204 -> 192 us).  A kernel strides over the chunks that are there, so kBigGridMax only keeps the launch below the 2^32 threads that HIP takes: a graph of 2M nodes and 440M
// edges has 2.1M chunks at most, 17M workgroups of 256 threads in slices of 256 columns.  Multiples of 8, so that b % 8
// survives the stride.
constexpr int64_t kBigGridMax = 1 << 20;
static_assert(kBigGridMax % 8 == 0 && kBigGridMax * 1024 < 1ll << 32, "threads of a launch");
inline unsigned big_grid(const ink_ctx *c, int64_t chunks, int slices, bool latency) {
  int64_t n = latency ? chunks : chunks * slices, least = latency ? 1024 : 2048, most = big_chunk_capacity(c) * slices;
  if (n < least) n = least;
  if (n > most) n = most;
  if (n > kBigGridMax) n = kBigGridMax;
  return (unsigned)((n + 7) & ~7ll);
}

// buffers of the long-row path; call before the kernel that fills the list (growing drops contents)
inline hipError_t ensure_big_buffers(ink_ctx *c, int ld, bool with_ids) {
  INK_TRY(c->big_list.reserve((size_t)big_rows_capacity(c) * 4));
  INK_TRY(c->big_pref.reserve((size_t)(c->big_list.cap / 4 + 1) * 4));
  int64_t cap = big_chunk_capacity(c);
  INK_TRY(c->big_part_v.reserve((size_t)cap * ld * sizeof(float)));
  if (with_ids) {
    INK_TRY(c->big_part_i.reserve((size_t)cap * ld * sizeof(int32_t)));
    INK_TRY(c->big_part_s.reserve((size_t)cap * ld * sizeof(float)));
    INK_TRY(c->big_part_j.reserve((size_t)cap * ld * sizeof(int32_t)));
  }
  return hipSuccess;
}

inline bool latency_mode(int64_t n_targets) { return n_targets <= kLatencyTargets; }
inline int big_threshold(int64_t n_targets, int lanes_per_row, int throughput_deg) {
  return latency_mode(n_targets) ? 32 * (kWave / lanes_per_row) : throughput_deg;
}

inline BigRows big_rows_of(ink_ctx *c, int chunk) { return BigRows{c->big_list.as<int32_t>(), c->big_pref.as<int32_t>(), chunk}; }
inline hipError_t clear_big_rows(ink_ctx *c) { return hipMemsetAsync(&c->d_cnt->v[C_NCHUNK], 0, 2 * sizeof(int32_t), c->stream); }

__device__ __forceinline__ int big_row_chunks(int deg, int chunk) { return (int)((unsigned)(deg + chunk - 1) / (unsigned)chunk); }
// places for `rows` rows of `chunks` chunks together: the first of each
__device__ __forceinline__ void reserve_big(Counters *cnt, int rows, int chunks, int &i, int &base) {
  const unsigned long long t = atomicAdd((unsigned long long *)&cnt->v[C_NCHUNK], ((unsigned long long)rows << 32) + (unsigned)chunks);
  i = (int)(t >> 32);
  base = (int)(uint32_t)t;
}
// lists row v (one lane)
__device__ __forceinline__ void list_big_row(const BigRows &b, Counters *cnt, int v, int deg) {
  int i, base;
  reserve_big(cnt, 1, big_row_chunks(deg, b.chunk), i, base);
  b.list[i] = v;
  b.base[i] = base;
}

// Short launches of few chunks have no kernel that combines a row's parts: the wave that stores the last of them does.  The parts are then stored
// and read past the L2s of the XCDs (COHERENT), a store is waited for before it is counted, and the count is 0 again afterwards.
// True for the last of `units`.  (A launch of at most kLatencyTargets targets lists at most as many rows: ink_ctx::arrived.  With
// fences instead, which write back and invalidate, the last part took 1.5 us longer.)
__device__ __forceinline__ bool last_to_arrive(int32_t *at, int units) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (units == 1) return true;
  int n = 0;
  if (lane_id() == 0) n = __hip_atomic_fetch_add(at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  n = __builtin_amdgcn_readfirstlane(n);
  asm volatile("" ::: "memory");
  if (n != units - 1) return false;
  if (lane_id() == 0) __hip_atomic_store(at, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}
// That pays while there are few of them: a launch saved is 2 to 6 us, but every part is stored and read past the caches and waited for
// while the rest of its workgroup stands.  Inferences of 1500 to 8000 nodes, two layers, at the expected chunks in brackets (of an R-MAT graph
// half to one and a half times as many are there), us, with a kernel that combines / by the last to arrive: max of 128 columns 120 / 114 (219),
// 176 / 176 (391), 294 / 315 (1172), 687 / 753 (5859); of 64 88 / 86 (219), 107 / 113 (366), 144 / 160 (782), 475 / 650 (5859); min of 250
// 182 / 174 (98), 205 / 210 (366), 383 / 397 (977); GCN of 250 118 / 116 (98), 153 / 157 (586), 371 / 405 (5859).  Sums of at most 128
// columns, a quarter of the stores and fewer rows above the limit, longer: GIN of 128 110 / 105 (391), 152 / 149 (1953), 206 / 207 (3126),
// 261 / 265 (5859), mean of 64 123 / 120 (1953), 190 / 192 (5859).  Behind the events of an update, at twice the chunks of the last
// one: 100 updates of max on 8000 nodes with 20 neighbours each 334 / 326, 500 with 150 each, some 600 chunks, 556 / 561.
constexpr int64_t kArriveChunks = 256, kArriveChunksSum = 2048, kArriveChunksEvents = 1024;
inline bool combine_on_arrival(const AggArgs &a, bool sums) { return a.big_chunks <= (sums && a.wd <= 128 ? kArriveChunksSum : kArriveChunks); }
template <bool COHERENT, class T> __device__ __forceinline__ void put_part(T *p, T x) {
  if constexpr (COHERENT) __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = x;
}
template <bool COHERENT, class V> __device__ __forceinline__ V get_part(const void *p) {      // 16 bytes
  static_assert(sizeof(V) == 16, "four values");
  if constexpr (COHERENT) {
    union { uint64_t u[2]; V v; } x;
    x.u[0] = __hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x.u[1] = __hip_atomic_load((const uint64_t *)p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return x.v;
  } else return *reinterpret_cast<const V *>(p);
}

// row (index in the list), node id and neighbour range of global chunk cg
__device__ __forceinline__ void big_chunk(const BigRows &b, int n_big, int cg, const int32_t *in_deg, int &i, int &v, int64_t &j0, int64_t &j1) {
  i = wave_last_le(b.base, n_big, cg);      // called by whole waves with wave-uniform arguments
  v = b.list[i];
  int64_t deg = in_deg[v];
  j0 = (int64_t)(cg - b.base[i]) * b.chunk;
  j1 = j0 + b.chunk < deg ? j0 + b.chunk : deg;
}

// Slices: the columns of a chunk are shared out in groups of kSliceCols, one 128-byte line of every row.  Workgroups go
// round the 8 XCDs, so item b runs on XCD b % 8; with S slices, XCD x takes the S parts x S .. x S + S - 1 of the 8 S
// parts (slice u / 8, every eighth chunk) one after the other.  An XCD then reads one slice of the message table, or two
// in turn, instead of all of it, and its L2 holds as many times more rows of it.
constexpr int kSliceLanes = 8, kSliceCols = 4 * kSliceLanes;
// Tables up to which long launches of sums go by slices.  Beyond, hardly a row is read twice while it is in an L2, and a
// row in four or eight parts is as many address translations.  Inferences, slices against whole rows: GIN of 128 columns,
// 20 edges a node, 1M / 2.5M nodes (1.3 GB) 4.03 / 10.5 ms against 4.11 / 10.6, 5M (2.6 GB) / 10M 22.5 / 46.5 against
// 22.2 / 45.2; GCN of 256 on 1M (1 GB) 9.45 against 9.55, on 4M (4.1 GB) 21.95 against 21.3.
constexpr int64_t kSlicedTableBytes = 2ll << 30;
// Items (chunks times slices) up to which short launches go by slices: what the chip holds of their workgroups of 1024 threads, where
// the launch's time is one chunk's.  Beyond, an item's fixed costs are paid once for every slice, and whole rows are faster.  Inferences
// of 8000 nodes with 8 to 4000 rows of 150 to 1000 neighbours, whole / in slices, us, at 512 items, 1024 items and 4000 rows: GCN of 250
// columns 89 / 85, 87 / 89, 315 / 432; mean of 128 47 / 45.5, 49.5 / 51, 148 / 208; max of 128 67.5 / 65, 70 / 82, 398 / 602; min of 250 86.5 / 84,
// 88 / 102, 469 / 1131.  (Max / min of at most two slices, 64 floats, stay with them: 60 / 59, 122 / 117, 368 / 345; sums of 64 39 / 38.5, 58 / 60,
// 132.5 / 141.5.)
constexpr int kSlicedItems = 512;
inline int big_slices(int wd) { return (wd + kSliceCols - 1) / kSliceCols; }
__device__ __forceinline__ int slice_items(int total, int slices) { return ((total + 7) >> 3) * 8 * slices; }
__device__ __forceinline__ bool slice_item(int b, int total, int slices, int &chunk, int &slice) {
  const int per = (total + 7) >> 3, i = b >> 3, j = i / per, u = (b & 7) * slices + j;
  slice = u >> 3;
  chunk = (i - j * per) * 8 + (u & 7);
  return chunk < total;
}

}  // namespace ink
