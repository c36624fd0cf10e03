// C ABI entry points and the per-layer driver of the incremental update (Sec. 2.3 workflow):
// for every aggregation layer  seed events from the changed edges -> expand events from the
// changed sources -> group by target -> incremental aggregation / recompute -> dense combination
// on the changed rows -> compare-and-emit the next layer's sources.
#include <algorithm>
#include <chrono>
#include <cstring>
#include <cstdio>
#include <mutex>
#include <new>
#include <vector>

#include "bigrows.h"
#include "events.h"

using namespace ink;

#define API_TRY(x)                                                                         \
  do {                                                                                     \
    hipError_t e_ = (x);                                                                   \
    if (e_ != hipSuccess) {                                                                \
      c->err = std::string("HIP error: ") + hipGetErrorString(e_) + " at " #x;             \
      return e_ == hipErrorOutOfMemory ? INK_E_OOM : INK_E_DEVICE;                         \
    }                                                                                      \
  } while (0)

static thread_local std::string g_create_err;

static inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
static inline dim3 grid1(int64_t n, int per = 256) { return dim3((unsigned)std::max<int64_t>(1, (n + per - 1) / per)); }

// ------------------------------------------------------------------------------------ kernels
// Changed edges and changed sources of a layer: what its events are made from.
struct EventInputs {
  const int32_t *del_s, *del_d, *ins_s, *ins_d; int n_del, n_ins;
  const int32_t *F; int nF; const int32_t *pref; int n_chg;      // changed sources, prefix and total of their kept out-edges
  const int64_t *off; const int32_t *ids; int payload_index;
};

// All events of a layer, one tile of the sort per workgroup, which also counts the tile's digits for the
// first sort pass (the keys are not read again for it).  A wave creates ITEMS * 64 consecutive events: it
// finds the sources of its first and last propagated event with two wave-wide searches (64 probes per
// round) and brings the sources between those two into LDS, their prefixes and where their targets stand.  A lane then
// looks for the source of each of its events there, four events together, and only the targets come from memory.  With
// search, source and offset a chain of loads per event: 313k events 30 -> 15 us, 1500 12 -> 6.6, 1.56M 27 -> 15.
// More sources than the wave's share of LDS holds (fewer than three events each) are searched where they are.
constexpr int kStagedSources = 256;
template <int D, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_make_events(EventInputs in, uint32_t *key, uint32_t *val, int32_t *hist, int nb, Counters *cnt) {
  __shared__ int h[1 << D];
  __shared__ int s_u[kSortWaves][kStagedSources], s_pref[kSortWaves][kStagedSources];
  __shared__ int64_t s_at[kSortWaves][kStagedSources];       // where event c of the source stands in ids: s_at + c
  if (blockIdx.x == 0)                 // the layer's counters start here
    for (int i = threadIdx.x; i < (int)(sizeof(Counters) / sizeof(int32_t)); i += kSortThreads) ((int32_t *)cnt)[i] = 0;
  tile_hist_clear<D>(h);
  const int l = lane_id(), w = threadIdx.x / kWave;
  const int64_t n = (int64_t)in.n_del + in.n_chg + in.n_ins;
  const int64_t e_base = ((int64_t)blockIdx.x * kSortWaves + w) * (ITEMS * kWave);
  const int64_t e_end = e_base + ITEMS * kWave < n ? e_base + ITEMS * kWave : n;
  // the wave's propagated events [c0, c1)
  const int64_t c0 = (e_base > in.n_del ? e_base : in.n_del) - in.n_del;
  const int64_t c1 = (e_end < in.n_del + (int64_t)in.n_chg ? e_end : in.n_del + (int64_t)in.n_chg) - in.n_del;
  int lo = 0, hi = 0;
  if (c0 < c1) {
    lo = wave_last_le(in.pref, in.nF, (int)c0);                                   // pref[0] = 0 <= every event
    hi = lo + wave_last_le(in.pref + lo, in.nF - lo, (int)(c1 - 1));              // pref[lo] <= c0 <= c1 - 1
  }
  const bool staged = hi - lo < kStagedSources;
  if (staged && c0 < c1) {             // read by this wave alone
    for (int i = lo + l; i <= hi; i += kWave) {
      const int u = in.F[i], p = in.pref[i];
      s_u[w][i - lo] = u; s_pref[w][i - lo] = p; s_at[w][i - lo] = in.off[u] - p;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  constexpr int U = 4;                 // a lane's targets under way together
  static_assert(ITEMS % U == 0, "whole batches");
  for (int k0 = 0; k0 < ITEMS; k0 += U) {
    uint32_t kk[U], vv[U];
    int64_t at[U];
#pragma unroll
    for (int j = 0; j < U; j++) {
      const int64_t e = e_base + (k0 + j) * kWave + l;
      at[j] = -1;
      if (e >= e_end) continue;
      if (e < in.n_del) seed_event((int)e, in.del_s, in.del_d, in.ins_s, in.ins_d, in.n_del, &kk[j], &vv[j]);
      else if (e < in.n_del + (int64_t)in.n_chg) {
        const int c = (int)(e - in.n_del);
        int a, u;
        if (staged) {
          const int i = source_of_event(s_pref[w], hi - lo + 1, c);
          a = lo + i; u = s_u[w][i]; at[j] = s_at[w][i] + c;
        } else {
          a = lo + source_of_event(in.pref + lo, hi - lo + 1, c);
          u = in.F[a]; at[j] = in.off[u] + (c - in.pref[a]);
        }
        vv[j] = (EV_CHG << kEvKindShift) | (uint32_t)(in.payload_index ? a : u);
      } else seed_event((int)(e - in.n_chg), in.del_s, in.del_d, in.ins_s, in.ins_d, in.n_del, &kk[j], &vv[j]);
    }
#pragma unroll
    for (int j = 0; j < U; j++)
      if (at[j] >= 0) kk[j] = (uint32_t)in.ids[at[j]];
#pragma unroll
    for (int j = 0; j < U; j++) {
      const int64_t e = e_base + (k0 + j) * kWave + l;
      if (e >= e_end) continue;
      key[e] = kk[j];
      val[e] = vv[j];
      atomicAdd(&h[kk[j] & ((1 << D) - 1)], 1);
    }
  }
  tile_hist_store<D>(h, hist, nb);
}

static void make_events(const SortPlan &p, const EventInputs &in, uint32_t *key, uint32_t *val, int32_t *hist, Counters *cnt, hipStream_t s) {
#define INK_MAKE(D, I) hipLaunchKernelGGL((k_make_events<D, I>), dim3(p.tiles), dim3(kSortThreads), 0, s, in, key, val, hist, p.tiles, cnt)
  if (p.digit_bits == 8) { if (p.items == 4) INK_MAKE(8, 4); else INK_MAKE(8, 12); }
  else if (p.digit_bits == 9) { if (p.items == 4) INK_MAKE(9, 4); else INK_MAKE(9, 12); }
  else { if (p.items == 4) INK_MAKE(11, 4); else INK_MAKE(11, 12); }
#undef INK_MAKE
}

// The record; on the way the marks of a batch that ends with it are cleared: zero_at[0 .. n_zero) of `zero`.  That is one
// workgroup's chain, .7 us per 1000 marks, and a launch of k_zero_at in front of the record instead takes 2.3 us and a gap: from
// some 5000 marks on it is the shorter (10000 / 50000 / 1M marks 10 / 26 / 295 us in the record).
constexpr int kPublishThreads = 512;
constexpr int64_t kPublishMarks = 4096;
__global__ __launch_bounds__(kPublishThreads) void k_publish(const Counters *d, HostCounters *h, uint32_t *h_seq, uint32_t seq,
                                                             const int32_t *zero_at, int n_zero, int32_t *zero) {
  if (n_zero > 0) {                     // nothing is written after the record
    for (int i = threadIdx.x; i < n_zero; i += kPublishThreads) zero[zero_at[i]] = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  if (threadIdx.x < kWave) publish_wave(d, h, h_seq, seq);
}

// A layer with few events (at most THREADS * ITEMS): clearing the counters, creating the events,
// grouping them by target (stable, so deletions stay ahead of changes ahead of insertions) and
// the segment heads in one workgroup.  Output as from the separate kernels: val in grouped
// order, the distinct targets, the start of each target's events plus the closing offset, and
// the target count in the counter block.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_small_group(const int32_t *del_s, const int32_t *del_d, const int32_t *ins_s,
                                                         const int32_t *ins_d, int n_del, int n_ins, const int32_t *F,
                                                         int nF, const int32_t *pref, int n_chg, const int64_t *off,
                                                         const int32_t *ids, int payload_index, int passes,
                                                         uint32_t *key_out, uint32_t *val_out, int32_t *t_list,
                                                         int32_t *t_seg, Counters *cnt) {
  __shared__ SmallSortLds<THREADS, ITEMS> S;
  __shared__ int sm[THREADS / kWave + 1];
  {
    int32_t *z = (int32_t *)cnt;
    for (int i = threadIdx.x; i < (int)(sizeof(Counters) / sizeof(int32_t)); i += THREADS)
      if (i != C_NT) z[i] = 0;
  }
  const int n_seed = n_del + n_ins, nE = n_seed + n_chg;
  for (int e = threadIdx.x; e < nE; e += THREADS) {
    uint32_t k, v;
    if (e < n_del) seed_event(e, del_s, del_d, ins_s, ins_d, n_del, &k, &v);
    else if (e < n_del + n_chg) expand_event(e - n_del, F, nF, pref, off, ids, payload_index, &k, &v);
    else seed_event(e - n_chg, del_s, del_d, ins_s, ins_d, n_del, &k, &v);
    S.sk[e] = k; S.sv[e] = v;
  }
  small_sort_lds<THREADS, ITEMS>(S, nE, passes);
  const int t0 = threadIdx.x * ITEMS;
  int h[ITEMS], c = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int i = t0 + k;
    h[k] = i < nE && (i == 0 || S.sk[i] != S.sk[i - 1]);
    c += h[k];
    if (i < nE) { key_out[i] = S.sk[i]; val_out[i] = S.sv[i]; }
  }
  int nT;
  int ex = block_excl_scan<THREADS>(c, sm, &nT);
#pragma unroll
  for (int k = 0; k < ITEMS; k++)
    if (h[k]) { t_list[ex] = (int32_t)S.sk[t0 + k]; t_seg[ex] = t0 + k; ex++; }
  if (threadIdx.x == 0) { t_seg[nT] = nE; cnt->v[C_NT] = nT; }
}

// The rows a layer with few events has to transform, in one workgroup: the targets whose bit the
// aggregation set in the bitmap (the bits are cleared on the way), the sources F (self term) and
// the nodes D whose in-degree changed, sorted and made unique -> rows[], their number -> C_NC.
// Also clears the first n_flags bytes of flag (the transform sets the flags of changed rows).
// n_t_bound + nF + nD is at most THREADS * ITEMS.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_small_collect(const int32_t *t_list, const int32_t *n_t_dev, int n_t_bound,
                                                           unsigned long long *bm, const int32_t *F, int nF,
                                                           const int32_t *D, int nD, int passes, int32_t *rows,
                                                           uint8_t *flag, int n_flags, Counters *cnt) {
  __shared__ SmallSortLds<THREADS, ITEMS> S;
  __shared__ int sm[THREADS / kWave + 1];
  for (int i = threadIdx.x; i < n_flags; i += THREADS) flag[i] = 0;
  const int nT = n_t_bound > 0 ? min(*n_t_dev, n_t_bound) : 0;
  const int M = n_t_bound + nF + nD;
  const int t0 = threadIdx.x * ITEMS;
  int id[ITEMS], c = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int i = t0 + k;
    id[k] = -1;
    if (i < n_t_bound) {
      if (i < nT) {
        int v = t_list[i];
        unsigned long long bit = 1ull << (v & 63);
        if (atomicAnd(&bm[v >> 6], ~bit) & bit) id[k] = v;
      }
    } else if (i < n_t_bound + nF) id[k] = F[i - n_t_bound];
    else if (i < M) id[k] = D[i - n_t_bound - nF];
    c += id[k] >= 0;
  }
  int m;
  int ex = block_excl_scan<THREADS>(c, sm, &m);
#pragma unroll
  for (int k = 0; k < ITEMS; k++)
    if (id[k] >= 0) { S.sk[ex] = (uint32_t)id[k]; S.sv[ex] = 0; ex++; }
  small_sort_lds<THREADS, ITEMS>(S, m, passes);
  int h[ITEMS];
  c = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int i = t0 + k;
    h[k] = i < m && (i == 0 || S.sk[i] != S.sk[i - 1]);
    c += h[k];
  }
  int nC;
  ex = block_excl_scan<THREADS>(c, sm, &nC);
#pragma unroll
  for (int k = 0; k < ITEMS; k++)
    if (h[k]) rows[ex++] = (int32_t)S.sk[t0 + k];
  if (threadIdx.x == 0) cnt->v[C_NC] = nC;
}

// The emission of a layer with few transformed rows (at most THREADS * ITEMS) in one workgroup:
// rows whose flag is set -> their positions (idx) and ids (f_list), the count, the exclusive prefix of
// their kept out-degrees and its total.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_small_emit(const uint8_t *flag, const int32_t *rows, int nC, const int32_t *nC_dev, int32_t *idx,
                                                        int32_t *f_list, const int32_t *deg,
                                                        const int32_t *new_out, int32_t *f_pref, Counters *cnt,
                                                        HostCounters *h, uint32_t *h_seq, uint32_t seq) {
  __shared__ int s_f[THREADS * ITEMS];
  __shared__ int sm[THREADS / kWave + 1];
  const int t0 = threadIdx.x * ITEMS;
  if (nC_dev) nC = min(nC, *nC_dev);
  int f[ITEMS], c = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int i = t0 + k;
    f[k] = i < nC && flag[i] != 0;
    c += f[k];
  }
  int nF;
  int ex = block_excl_scan<THREADS>(c, sm, &nF);
#pragma unroll
  for (int k = 0; k < ITEMS; k++)
    if (f[k]) { int u = rows[t0 + k]; idx[ex] = t0 + k; f_list[ex] = u; s_f[ex] = u; ex++; }
  if (threadIdx.x == 0) cnt->v[C_NEXT] = nF;
  __syncthreads();
  int kd[ITEMS];
  c = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int i = t0 + k;
    kd[k] = i < nF ? deg[s_f[i]] - new_out[s_f[i]] : 0;
    c += kd[k];
  }
  int n_ev;
  ex = block_excl_scan<THREADS>(c, sm, &n_ev);
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    if (t0 + k < nC) f_pref[t0 + k] = ex;
    ex += kd[k];
  }
  if (threadIdx.x == 0) cnt->v[C_NEV] = n_ev;
  __threadfence();
  __syncthreads();
  if (threadIdx.x < kWave) publish_wave(cnt, h, h_seq, seq);
}

// Sets the bits of the listed nodes; with deg only of those that have no edge left.
__global__ void k_mark_nodes(const int32_t *list, int n, const int32_t *list2, int n2, uint64_t *bm, const int32_t *deg) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n + n2) return;
  const int v = i < n ? list[i] : list2[i - n];
  if (!deg || deg[v] == 0) atomicOr((unsigned long long *)&bm[v >> 6], 1ull << (v & 63));
}

// The changed rows of a long layer: their positions, their ids and the prefix of the events they propagate, in one scan
// over the row flags (two launches).  A tile's sum packs both counts: rows in the upper, events in the lower 32 bits
// (a layer has less than 2^31 events).  Compaction, gather of the ids and prefix were five launches; the six scans of a
// batch of 10000 on 1.25M nodes took 140 us that way and take 112, a batch of 100 passes in 1.63 instead of 1.67 ms.
struct EmitRows {
  const uint8_t *flag; const int32_t *rows;      // flags are read 8 at a time: room for 7 past n
  const int32_t *deg, *new_out;                  // deg null: no events wanted
  int64_t bound; const int32_t *n_dev;           // rows: bound, or fewer as *n_dev says
  __device__ __forceinline__ int64_t count() const { return n_dev && *n_dev < bound ? *n_dev : bound; }
  __device__ __forceinline__ unsigned long long flags8(int64_t base) const {
    const int64_t n = count();
    if (base >= n) return 0;
    const unsigned long long f = *reinterpret_cast<const unsigned long long *>(flag + base);
    return n - base >= 8 ? f : f & ((1ull << (8 * (n - base))) - 1);
  }
  __device__ __forceinline__ int events(int u) const { return deg ? kept_out_degree(deg, new_out, u) : 0; }
};
// Rows per thread.  Every load of a row's degrees is a miss, and 8 rows a thread left the layers in the middle to a handful of
// workgroups: count and write, 8 rows a thread against 1, 6k rows 21 / 9 us, 150k 23 / 10.  Beyond the line the sums of the tiles
// before its own, which every workgroup adds up, count more; the last layer of 700k rows, which asks for no degree, takes 15 us with 8.
constexpr int kEmitThreads = 256;
constexpr int64_t kEmitFew = 1 << 18;
inline int emit_per_thread(int64_t n) { return n <= kEmitFew ? 1 : 8; }

__device__ __forceinline__ unsigned long long block_excl_scan64(unsigned long long x, unsigned long long *sm, unsigned long long *total) {
  const int l = lane_id(), w = threadIdx.x / kWave;
  unsigned long long inc = x;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const unsigned long long y = __shfl_up(inc, o, kWave);
    if (l >= o) inc += y;
  }
  __syncthreads();                 // sm may still be read by the scan before
  if (l == kWave - 1) sm[w] = inc;
  __syncthreads();
  unsigned long long before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kEmitThreads / kWave; i++) { if (i < w) before += sm[i]; all += sm[i]; }
  *total = all;
  return before + inc - x;
}

// u[k]: id of row base + k, v[k]: its packed count (0 if its flag is not set).  The count, the flags and the ids are asked for
// together and the degrees of all rows behind them, whether or not they are wanted (past the count the list may hold anything:
// node 0 stands in).
template <int I>
__device__ __forceinline__ unsigned long long emit_items(const EmitRows &e, int64_t base, int u[I], unsigned long long v[I]) {
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < I; k++) { u[k] = 0; v[k] = 0; }
  if (base >= e.bound) return 0;
  static_assert(I == 1 || I == 8, "one load of flags");
  const unsigned long long f = I == 8 ? *reinterpret_cast<const unsigned long long *>(e.flag + base) : e.flag[base];
#pragma unroll
  for (int k = 0; k < I; k++) u[k] = e.rows[base + k < e.bound ? base + k : e.bound - 1];
  const int64_t n = e.count();
  int ev[I];
#pragma unroll
  for (int k = 0; k < I; k++) u[k] = base + k < n ? u[k] : 0;
#pragma unroll
  for (int k = 0; k < I; k++) ev[k] = e.events(u[k]);
#pragma unroll
  for (int k = 0; k < I; k++) {
    if (base + k < n && ((f >> (8 * k)) & 0xFF)) v[k] = (1ull << 32) + (unsigned)ev[k];
    s += v[k];
  }
  return s;
}

template <int I>
__global__ __launch_bounds__(kEmitThreads) void k_emit_count(EmitRows e, unsigned long long *tile) {
  __shared__ unsigned long long sm[kEmitThreads / kWave];
  int u[I]; unsigned long long v[I], tot;
  (void)block_excl_scan64(emit_items<I>(e, ((int64_t)blockIdx.x * kEmitThreads + threadIdx.x) * I, u, v), sm, &tot);
  if (threadIdx.x == 0) tile[blockIdx.x] = tot;
}

template <int I>
__global__ __launch_bounds__(kEmitThreads) void k_emit_write(EmitRows e, const unsigned long long *tile, int32_t *idx, int32_t *ids,
                                                             int32_t *pref, Counters *cnt, HostCounters *h, uint32_t *h_seq, uint32_t seq) {
  __shared__ unsigned long long sm[kEmitThreads / kWave];
  unsigned long long part = 0, before, tot;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += kEmitThreads) part += tile[i];
  const int64_t base = ((int64_t)blockIdx.x * kEmitThreads + threadIdx.x) * I;
  int u[I]; unsigned long long v[I];
  const unsigned long long mine = emit_items<I>(e, base, u, v);
  (void)block_excl_scan64(part, sm, &before);
  unsigned long long at = before + block_excl_scan64(mine, sm, &tot);
#pragma unroll
  for (int k = 0; k < I; k++) {
    if (!v[k]) continue;
    const int p = (int)(at >> 32);
    idx[p] = (int32_t)(base + k);
    ids[p] = u[k];
    if (e.deg) pref[p] = (int32_t)(uint32_t)at;
    at += v[k];
  }
  if (blockIdx.x != gridDim.x - 1) return;
  if (threadIdx.x == 0) {
    cnt->v[C_NEXT] = (int32_t)((before + tot) >> 32);
    if (e.deg) cnt->v[C_NEV] = (int32_t)(uint32_t)(before + tot);
    __threadfence();
  }
  __syncthreads();
  if (threadIdx.x < kWave) publish_wave(cnt, h, h_seq, seq);      // the counts are all the host waits for; the lists are for kernels behind this one
}

__global__ void k_gather_i32(const int32_t *table, const int32_t *idx, int n, const int32_t *n_dev, int32_t *out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n_dev) n = *n_dev;
  if (i < n) out[i] = table[idx[i]];
}

// Where a result goes besides the library's own buffer: pinned host memory, ids and rows, the first `rows` of them.
// The stores have left the chip when a wave ends, before the record that the host waits for is written.
struct HostMirror { int32_t *ids; float *emb; int64_t rows; };

__global__ void k_gather_rows(const float *table, int ld, int d, const int32_t *rows, int64_t n,
                              float *out) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t r = t / d;
  int k = (int)(t % d);
  if (r < n) out[r * d + k] = table[(int64_t)rows[r] * ld + k];
}

// the same, 16 bytes per thread, for d a multiple of 4
__global__ void k_gather_rows4(const float *table, int ld, int d4, const int32_t *rows, int64_t n,
                               float *out) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t r = t / d4;
  int k = (int)(t - r * d4);
  if (r < n)
    reinterpret_cast<float4 *>(out)[r * d4 + k] = *reinterpret_cast<const float4 *>(table + (int64_t)rows[r] * ld + 4 * k);
}

// The last layer's changed rows: their ids and the rows themselves, in one launch.  A workgroup has `per` (a multiple of 64)
// of the transformed rows; what stands before them it counts itself, in the tile sums of k_emit_count and the flags of its
// own tile, or, without tile sums (at most kSmallLayer rows), in all flags.  Emission of a short layer in one workgroup and a
// gather behind it took 12 and 7 us; 100 updates on 10k nodes .357 -> .342 ms a pass of two.
__global__ __launch_bounds__(256) void k_emit_result(EmitRows e, const unsigned long long *tile, int tile_rows, int per, const float *table, int ld, int d,
                                                     int32_t *ids, float *out, HostMirror m, Counters *cnt) {
  __shared__ int sm[256 / kWave];
  __shared__ int row[256], n_here;
  const int l = lane_id(), t = threadIdx.x, w = t / kWave;
  const int64_t n = e.n_dev && *e.n_dev < e.bound ? *e.n_dev : e.bound;
  const int64_t r0 = (int64_t)blockIdx.x * per;
  if (r0 >= n && !(n == 0 && blockIdx.x == 0)) return;
  const int64_t t0 = tile ? r0 / tile_rows : 0;
  int before = 0;
  for (int64_t i = t; i < t0; i += 256) before += (int)(tile[i] >> 32);
  for (int64_t p = t0 * tile_rows + 8 * t; p < r0; p += 8 * 256) before += __popcll(e.flags8(p) & 0x0101010101010101ull);
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, kWave);
  if (l == 0) sm[w] = before;
  // this workgroup's rows, in order (per <= 256: a wave per 64 of them)
  const int64_t r = r0 + t;
  const bool on = t < per && r < n && e.flag[r] != 0;
  const uint64_t mask = __ballot(on);
  __shared__ int wn[256 / kWave];
  if (l == 0) wn[w] = __popcll(mask);
  __syncthreads();
  int at = __popcll(mask & ((1ull << l) - 1)), all = 0;
  before = 0;
#pragma unroll
  for (int i = 0; i < 256 / kWave; i++) { at += i < w ? wn[i] : 0; all += wn[i]; before += sm[i]; }
  if (on) { row[at] = e.rows[r]; ids[before + at] = row[at]; }
  if (on && before + at < m.rows) m.ids[before + at] = row[at];
  if (t == 0) {
    n_here = all;
    if (r0 + per >= n) cnt->v[C_NEXT] = before + all;
  }
  __syncthreads();
  const int k = n_here;
  if (d % 4 == 0) {
    const int d4 = d / 4;
    for (unsigned i = t; i < (unsigned)(k * d4); i += 256) {
      const unsigned j = i / (unsigned)d4, c = i - j * (unsigned)d4;
      const float4 x = *reinterpret_cast<const float4 *>(table + (int64_t)row[j] * ld + 4 * c);
      reinterpret_cast<float4 *>(out)[(int64_t)(before + (int)j) * d4 + c] = x;
      if (before + (int)j < m.rows) reinterpret_cast<float4 *>(m.emb)[(int64_t)(before + (int)j) * d4 + c] = x;
    }
  } else {
    for (unsigned i = t; i < (unsigned)(k * d); i += 256) {
      const unsigned j = i / (unsigned)d, c = i - j * (unsigned)d;
      const float x = table[(int64_t)row[j] * ld + c];
      out[(int64_t)(before + (int)j) * d + c] = x;
      if (before + (int)j < m.rows) m.emb[(int64_t)(before + (int)j) * d + c] = x;
    }
  }
  if (m.rows > 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

static void gather_rows(hipStream_t s, const float *table, int ld, int d, const int32_t *rows, int64_t n, float *out) {
  if (n <= 0) return;
  if (d % 4 == 0) hipLaunchKernelGGL(k_gather_rows4, grid1(n * (d / 4)), dim3(256), 0, s, table, ld, d / 4, rows, n, out);
  else hipLaunchKernelGGL(k_gather_rows, grid1(n * d), dim3(256), 0, s, table, ld, d, rows, n, out);
}

__global__ void k_pack_rows(const void *table, int ld, int d, int64_t row0, int64_t nrows, void *out) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t r = t / d;
  int k = (int)(t % d);
  if (r < nrows) ((uint32_t *)out)[r * d + k] = ((const uint32_t *)table)[(row0 + r) * ld + k];
}

// the same for widths of whole 16-byte groups: a workgroup takes `per` rows
__global__ __launch_bounds__(256) void k_pack_rows4(const float4 *table, int ld4, int d4, int64_t row0, int64_t nrows, int per, float4 *out) {
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int rows = nrows - r0 < per ? (int)(nrows - r0) : per;
  for (unsigned t = threadIdx.x; t < (unsigned)(rows * d4); t += 256) {
    const unsigned r = t / (unsigned)d4, k = t - r * (unsigned)d4;
    out[(r0 + r) * d4 + k] = table[(row0 + r0 + r) * ld4 + k];
  }
}

__global__ void k_unpack_rows(const float *in, int d, int ld, int64_t n, float *table) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t r = t / d;
  int k = (int)(t % d);
  if (r < n) table[r * ld + k] = in[r * d + k];
}

__global__ void k_iota_u32(uint32_t *out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (uint32_t)i;
}

// adjacent equal keys in a sorted list -> *flag = 1
__global__ void k_any_adjacent_equal(const uint32_t *keys, int64_t n, int32_t *flag) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i + 1 < n && keys[i] == keys[i + 1]) *flag = 1;
}

// any id outside [0, n_nodes) (a negative id is a huge unsigned one) -> *flag = 1
__global__ void k_any_out_of_range(const uint32_t *ids, int64_t n, uint32_t n_nodes, int32_t *flag) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && ids[i] >= n_nodes) *flag = 1;
}

// The ids of at most THREADS * ITEMS feature rows in one workgroup: order, distinctness (C_TMP0) and range (C_TMP1); the
// counters start here, and the rows' flags.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_feature_ids(const int32_t *in, int n, uint32_t n_nodes, int passes, uint32_t *ids, uint32_t *perm,
                                                         uint8_t *flag, Counters *cnt) {
  __shared__ SmallSortLds<THREADS, ITEMS> S;
  bool far = false, twice = false;
  for (int i = threadIdx.x; i < n; i += THREADS) {
    const uint32_t id = (uint32_t)in[i];
    far |= id >= n_nodes;
    S.sk[i] = id; S.sv[i] = (uint32_t)i;
  }
  for (int i = threadIdx.x; i < (int)(sizeof(Counters) / sizeof(int32_t)); i += THREADS)
    if (i != C_TMP0 && i != C_TMP1) ((int32_t *)cnt)[i] = 0;
  small_sort_lds<THREADS, ITEMS>(S, n, passes);
  for (int i = threadIdx.x; i < n; i += THREADS) {
    ids[i] = S.sk[i]; perm[i] = S.sv[i]; flag[i] = 0;
    twice |= i + 1 < n && S.sk[i] == S.sk[i + 1];
  }
  const bool any_far = __syncthreads_or(far) != 0, any_twice = __syncthreads_or(twice) != 0;
  if (threadIdx.x == 0) { cnt->v[C_TMP0] = any_twice; cnt->v[C_TMP1] = any_far; }
}

// New input features for the nodes ids[i] (ascending); the caller's row of ids[i] is rows[perm[i]].
// Writes the feature table with compare-and-emit: flag[i] = 1 if the row changed bitwise,
// old_rows[i] = the previous row (optional), dense[i] = the new row padded to ld (optional).
// A batch that the counters call bad changes nothing.
__global__ void k_set_features(const uint32_t *ids, const uint32_t *perm, int64_t n, const float *rows, int d, float *X,
                               int ld, float *old_rows, float *dense, uint8_t *flag, int32_t *list, const Counters *cnt) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t i = t / ld;
  int k = (int)(t % ld);
  if (i >= n || (cnt->v[C_TMP0] | cnt->v[C_TMP1]) != 0) return;
  int64_t v = ids[i];
  if (k == 0) list[i] = (int32_t)v;
  float nv = k < d ? rows[(int64_t)perm[i] * d + k] : 0.f;
  float o = X[v * ld + k];
  if (old_rows) old_rows[i * ld + k] = o;
  if (dense) dense[i * ld + k] = nv;
  if (__float_as_uint(o) != __float_as_uint(nv)) {
    X[v * ld + k] = nv;
    flag[i] = 1;
  }
}

__global__ void k_gather_rows_ld(const float *in, int ld, const int32_t *idx, int64_t n, const int32_t *n_dev,
                                 float *out) {
  // out[i][:] = in[idx[i]][:], both with row stride ld (a multiple of 4): 16 bytes per thread
  const int ld4 = ld >> 2;
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t r = t / ld4;
  int k = (int)(t - r * ld4);
  if (n_dev) n = *n_dev;
  if (r < n)
    reinterpret_cast<float4 *>(out)[r * ld4 + k] = *reinterpret_cast<const float4 *>(in + (int64_t)idx[r] * ld + 4 * k);
}

__device__ __forceinline__ float gcn_coef(int indeg) {      // (indeg + 1)^(-1/2)
  return __fdiv_rn(1.0f, __fsqrt_rn((float)(indeg + 1)));
}

__global__ void k_gcn_coef_all(const int32_t *deg, int n, float *cnorm) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cnorm[i] = gcn_coef(deg[i]);
}

// scaled = c_v * raw for the nodes in `nodes` (null: all); optionally keeps the old scaled rows
// and flags rows that changed bitwise (flag must be pre-zeroed)
__global__ void k_gcn_rescale(const int32_t *nodes, int64_t n, const int32_t *deg, float *cnorm, const float *raw,
                              float *scaled, int ld, int d, float *old_rows, uint8_t *flag) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t i = t / ld;
  int k = (int)(t % ld);
  if (i >= n) return;
  int v = nodes ? nodes[i] : (int)i;
  float cv = gcn_coef(deg[v]);
  if (k == 0) cnorm[v] = cv;
  float o = scaled[(int64_t)v * ld + k];
  float nv = k < d ? __fmul_rn(cv, raw[(int64_t)v * ld + k]) : 0.f;
  if (old_rows) old_rows[i * ld + k] = o;
  if (__float_as_uint(o) != __float_as_uint(nv)) {
    scaled[(int64_t)v * ld + k] = nv;
    if (flag) flag[i] = 1;
  }
}

// last GCN layer: h = act(c_v (S + own scaled message) + b) for the listed rows, compare-and-emit
__global__ void k_gcn_final(const int32_t *rows, int64_t n, const float *S, const float *Msc, const float *cnorm,
                            const float *bias, const float *user, int ld_user, int relu, float *H, int ld, int d,
                            uint8_t *flag) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t i = t / ld;
  int k = (int)(t % ld);
  if (i >= n || k >= d) return;
  int64_t v = rows ? rows[i] : i;
  float x = __fmul_rn(cnorm[v], __fadd_rn(S[v * ld + k], Msc[v * ld + k]));
  if (bias) x = __fadd_rn(x, bias[k]);
  if (user) x = __fadd_rn(x, user[v * ld_user + k]);
  if (relu) x = x > 0.f ? x : 0.f;
  float o = H[v * ld + k];
  if (__float_as_uint(o) != __float_as_uint(x)) {
    H[v * ld + k] = x;
    if (flag) flag[i] = 1;
  }
}

// ------------------------------------------------------------------------------------ helpers
static ink_status fail(ink_ctx *c, ink_status st, const std::string &msg) {
  if (c) c->err = msg; else g_create_err = msg;
  return st;
}

// What a failing call had enqueued by then may read the caller's arrays: it has ended before the call returns.
static ink_status drain(ink_ctx *c, ink_status st) {
  (void)hipStreamSynchronize(c->stream);
  return st;
}

// An updating call that fails on the device side (allocation or HIP error) may have rewritten part of
// the graph store or of the cache: the context is then marked unusable and every later call but
// ink_last_error / ink_destroy returns INK_E_STATE.
static ink_status seal(ink_ctx *c, ink_status st) {
  if (st != INK_E_OOM && st != INK_E_DEVICE) return st;
  c->broken = true;
  return drain(c, st);
}
// Around a call with a result: the last one is gone when it starts, and results stop going to the host once one was not fetched.
static void begin_result(ink_ctx *c) {
  if (c->mirrored && !c->fetched && c->last.n > 0) c->mirror = false;
  c->last.n = -1;
  c->mirrored = c->fetched = false;
}
static void want_host_results(ink_ctx *c) {      // without the pinned memory results are copied
  if (!c->h_res && hipHostMalloc((void **)&c->h_res, INK_RESULT_HOST_BYTES, hipHostMallocCoherent) != hipSuccess) { c->h_res = nullptr; (void)hipGetLastError(); }
  c->mirror = c->h_res != nullptr;
}
static ink_status end_result(ink_ctx *c, ink_status st, const ink_update_result *out) {
  if (st == INK_OK) { c->last.ids = out->changed_ids; c->last.rows = out->embeddings; c->last.n = out->n_changed; }
  return seal(c, st);
}
static const char *kBrokenMsg = "the context is unusable after a failed update (INK_E_OOM / INK_E_DEVICE): destroy it";

static hipError_t alloc_table(Table &t, int64_t n, int d) {
  // rows start on 64-byte boundaries: a gathered row then touches the fewest cache lines (rows of 41
  // floats, 233k nodes / 114M edges: 176 -> 192 bytes per row and 5 % less aggregation time; 128-byte
  // alignment loses that again to the larger table)
  t.d = d;
  t.ld = round_up(d, 16);
  size_t bytes = (size_t)n * t.ld * 4;
  hipError_t e = hipMalloc(&t.p, bytes);
  if (e != hipSuccess) return e;
  return hipMemset(t.p, 0, bytes);
}

// uploads rows [row_off, row_off + K) of a weight matrix W ([K][N], host or device) into the
// zero-initialised padded device matrix `dst` ([Kp][Np] elements) in the order the transform
// kernel stages it (xform_weight_index)
static hipError_t upload_padded(const float *src, int K, int N, int Kp, int Np, int row_off, float *dst, bool src_dev) {
  std::vector<float> h((size_t)K * N);
  hipError_t e = hipMemcpy(h.data(), src, h.size() * 4, src_dev ? hipMemcpyDeviceToHost : hipMemcpyHostToHost);
  if (e != hipSuccess) return e;
  std::vector<float> p((size_t)Kp * Np);
  e = hipMemcpy(p.data(), dst, p.size() * 4, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return e;
  for (int k = 0; k < K; k++)
    for (int j = 0; j < N; j++) p[xform_weight_index(row_off + k, j, Np)] = h[(size_t)k * N + j];
  return hipMemcpy(dst, p.data(), p.size() * 4, hipMemcpyHostToDevice);
}

static hipError_t upload_vec(const float *src, int n, float **dst, bool src_dev) {
  if (!src) { *dst = nullptr; return hipSuccess; }
  hipError_t e = hipMalloc((void **)dst, (size_t)round_up(n, 32) * 4);
  if (e != hipSuccess) return e;
  e = hipMemset(*dst, 0, (size_t)round_up(n, 32) * 4);
  if (e != hipSuccess) return e;
  return hipMemcpy(*dst, src, (size_t)n * 4, src_dev ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice);
}

static void prof_collect(ink_ctx *c) {
  for (auto &p : c->ev_pending) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
      if (p.cls >= 0) c->stats.ms[p.cls] += ms;
      if (p.kern >= 0 && p.layer >= 1 && p.layer <= INK_MAX_LAYERS) c->stats.layer[p.layer - 1].ms_kernel[p.kern] += ms;
    }
    c->ev_free.push_back(p.a); c->ev_free.push_back(p.b);
  }
  c->ev_pending.clear();
}

hipError_t ink::read_counters(ink_ctx *c, bool end_batch) {
  if (end_batch && c->n_touched_src > kPublishMarks) {
    const hipError_t e = graph_end_batch(c);
    if (e != hipSuccess) return e;
  }
  const uint32_t seq = ++c->pub_seq;
  const int n_zero = end_batch ? (int)c->n_touched_src : 0;
  if (end_batch) c->n_touched_src = 0;
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(n_zero > 0 ? kPublishThreads : kWave), 0, c->stream, (const Counters *)c->d_cnt, c->h_cnt, c->h_seq, seq,
                     (const int32_t *)c->b_uniq.as<int32_t>(), n_zero, c->new_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return wait_published(c, c->h_seq, seq);
}

// Waits until the record with this sequence number has arrived: a spin of up to a millisecond, as long as all but the largest layers
// take and a host core's time until then (ink.h), then the blocking wait, whose wake-up is 15 to 20 us.  Spins of .15 and 1 ms, us a pass: 10000 updates at hubs of 612k nodes 2107 / 2076,
// 1000 feature rows on 200k nodes 1461 / 1430, GCN of 57M edges 2797 / 2758.
hipError_t ink::wait_published(ink_ctx *c, const uint32_t *h_seq, uint32_t seq) {
  hipError_t e;
  const auto t0 = std::chrono::steady_clock::now();
  for (int spin = 0;; spin++) {
    if (__atomic_load_n(h_seq, __ATOMIC_ACQUIRE) == seq) return hipSuccess;
    if ((spin & 63) == 63 &&
        std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() > 1000.0)
      break;
  }
  e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return e;
  return __atomic_load_n(h_seq, __ATOMIC_ACQUIRE) == seq ? hipSuccess : hipErrorUnknown;
}

static const Table &msg_table(ink_ctx *c, int l) {   // m_l: h_{l-1} (aggregate first) or GCN's scaled h_{l-1} W_l
  return c->kind == INK_MODEL_GCN ? c->Msc[l] : c->H[l - 1];
}

static AggArgs agg_args(ink_ctx *c, int l) {       // layer l in 1..k
  AggArgs a;
  a.n = c->n;
  a.in_off = c->gin.off; a.in_deg = c->gin.deg; a.in_ids = c->gin.ids; a.in_asc = c->gin.asc;
  const Table &M = msg_table(c, l);
  a.M = M.f(); a.ldm = M.ld;
  a.A = c->A[l].f(); a.ARG = c->is_select ? c->ARG[l].i() : nullptr; a.ld = c->A[l].ld; a.d = c->A[l].d;
  a.UB = c->is_select ? c->UB[l].f() : nullptr;
  a.ARG2 = c->is_select ? c->ARG2[l].i() : nullptr;
  a.wd = round_up(a.d, 4);
  a.is_min = c->is_min;
  a.nonneg = l > 1 && c->kind != INK_MODEL_GCN && c->layers[l - 2].act == INK_ACT_RELU;
  a.big_deg = kBigDeg;
  a.big_chunks = 2 * c->big_hint[l];
  a.count_cond = 1;
  a.keep_empty = false;
  a.layer = l;
  return a;
}

// dense combination of layer l for the rows in `rows` (null: all nodes).  With flags != null the
// layer's table is updated with compare-and-emit.
static hipError_t run_transform(ink_ctx *c, int l, const int32_t *rows, int64_t n_rows, uint8_t *flags,
                                float *old_rows = nullptr, const int32_t *n_rows_dev = nullptr) {
  const DevLayer &L = c->layers[l - 1];
  XformArgs x;
  memset(&x, 0, sizeof(x));
  x.rows = rows; x.n_rows = n_rows; x.n_rows_dev = n_rows_dev;
  x.old_rows = old_rows; x.ld_old = c->H[l].ld;
  if (c->agg == INK_AGG_MEAN) x.mean_deg = c->gin.deg;
  x.A = c->A[l].f(); x.lda = c->A[l].ld;
  x.Hp = c->H[l - 1].f(); x.ldh = c->H[l - 1].ld;
  x.d_in = L.in_dim; x.eps = c->eps;
  if (c->kind == INK_MODEL_SAGE) {
    x.mode = 0;
    x.W = L.W1; x.Kp = L.K1p; x.Np = L.N1p; x.bias = L.b1; x.n_out = L.out_dim; x.relu = L.act == INK_ACT_RELU;
    x.out = c->H[l].f(); x.ld_out = c->H[l].ld; x.to_table = 1; x.row_changed = flags;
    x.user = c->USER[l].f(); x.ld_user = c->USER[l].ld;
    return xform_run(c, x);
  }
  // GIN: two linear maps through a staging buffer
  hipError_t e = c->stage0.reserve((size_t)n_rows * L.N1p * 4);
  if (e != hipSuccess) return e;
  x.mode = 1;
  x.W = L.W1; x.Kp = L.K1p; x.Np = L.N1p; x.bias = L.b1; x.n_out = L.hidden; x.relu = 1;
  x.out = c->stage0.as<float>(); x.ld_out = L.N1p; x.to_table = 0; x.old_rows = nullptr;
  e = xform_run(c, x);
  if (e != hipSuccess) return e;
  XformArgs y;
  memset(&y, 0, sizeof(y));
  y.mode = 2; y.rows = rows; y.n_rows = n_rows; y.n_rows_dev = n_rows_dev;
  y.Hp = c->stage0.as<float>(); y.ldh = L.N1p; y.d_in = L.hidden;
  y.W = L.W2; y.Kp = L.K2p; y.Np = L.N2p; y.bias = L.b2; y.n_out = L.out_dim; y.relu = L.act == INK_ACT_RELU;
  y.out = c->H[l].f(); y.ld_out = c->H[l].ld; y.to_table = 1; y.row_changed = flags; y.out_rows = rows;
  y.old_rows = old_rows; y.ld_old = c->H[l].ld;
  y.user = c->USER[l].f(); y.ld_user = c->USER[l].ld;
  return xform_run(c, y);
}

// ------------------------------------------------------------------------------------ static work memory
// Work memory of ink_full_infer_noalloc: the list of long rows, the first chunk of each, the partial
// rows of the chunks and GIN's staging rows.  One array per
// GPU for the life of the process, shared by every call on that GPU.  Nothing in it has to start
// from zero: every part is written by the launch that reads it afterwards.
static __device__ __align__(256) unsigned char scratch[INK_NOALLOC_SCRATCH_BYTES];

// device address of `scratch` per GPU, looked up once with that GPU current (ink_create does it);
// host code uses these pointers, never the array's name
constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mu;

static hipError_t scratch_lookup(int *dev_out, void **ptr_out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  if (dev_out) *dev_out = dev;
  if (ptr_out) *ptr_out = g_scratch_ptr[dev];
  return hipSuccess;
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ------------------------------------------------------------------------------------ create
// Event records of a layer are addressed with 32-bit offsets: at most one per edge plus one per
// list entry of the batch (below 2^30), so the edge count is held below 2^31 - 2^30.
constexpr int64_t kMaxEdges = (1ll << 31) - (1ll << 30) - 1;

static ink_status validate_model(const ink_model *m, int feat_dim, std::string &why) {
  if (m->n_layers < 1 || m->n_layers > INK_MAX_LAYERS || !m->layers) { why = "n_layers out of range or layers NULL"; return INK_E_ARG; }
  if (m->kind != INK_MODEL_SAGE && m->kind != INK_MODEL_GIN && m->kind != INK_MODEL_GCN) { why = "unknown model kind"; return INK_E_ARG; }
  if (m->agg < INK_AGG_MAX || m->agg > INK_AGG_GCN_SYM) { why = "unknown aggregator"; return INK_E_ARG; }
  if ((m->kind == INK_MODEL_GCN) != (m->agg == INK_AGG_GCN_SYM)) { why = "GCN needs INK_AGG_GCN_SYM (and only GCN takes it)"; return INK_E_ARG; }
  int d = feat_dim;
  for (int l = 0; l < m->n_layers; l++) {
    const ink_layer &L = m->layers[l];
    if (L.in_dim != d) { why = "layer in_dim does not match the previous width"; return INK_E_ARG; }
    int agg_w = m->kind == INK_MODEL_GCN ? L.out_dim : L.in_dim;      // GCN aggregates after the linear map
    (void)agg_w;
    if (L.in_dim < 1 || L.out_dim < 1 || L.out_dim > INK_MAX_OUT_DIM || L.in_dim > INK_MAX_IN_DIM) { why = "layer width out of range"; return INK_E_ARG; }
    if (!L.W_neigh) { why = "W_neigh is NULL"; return INK_E_ARG; }
    if (m->kind == INK_MODEL_SAGE && !L.W_self) { why = "GraphSAGE needs W_self"; return INK_E_ARG; }
    if (m->kind == INK_MODEL_GIN && (!L.W_mlp2 || L.mlp_hidden < 1 || L.mlp_hidden > 256)) { why = "GIN needs W_mlp2 and 1 <= mlp_hidden <= 256"; return INK_E_ARG; }
    if (L.act != INK_ACT_NONE && L.act != INK_ACT_RELU) { why = "unknown activation"; return INK_E_ARG; }
    d = L.out_dim;
  }
  return INK_OK;
}

extern "C" ink_status ink_create(const ink_csr *g, const float *features, int32_t feat_dim, const ink_model *model,
                                 const ink_options *opts, ink_ctx **out) {
  if (out) *out = nullptr;
  if (!g || !features || !model || !out || !g->rowptr || (g->n_edges > 0 && !g->col))
    return fail(nullptr, INK_E_ARG, "ink_create: NULL argument");
  if (g->n_nodes < 1 || g->n_edges < 0 || feat_dim < 1 || g->n_nodes >= (1 << 30))
    return fail(nullptr, INK_E_ARG, "ink_create: bad n_nodes / n_edges / feat_dim");
  std::string why;
  ink_status st = validate_model(model, feat_dim, why);
  if (st != INK_OK) return fail(nullptr, st, "ink_create: " + why);
  const bool dev = opts && opts->mem == INK_MEM_DEVICE;
  const int n = g->n_nodes;
  const int64_t E = g->n_edges;
  if (E > kMaxEdges) return fail(nullptr, INK_E_ARG, "ink_create: more than 2^31 - 2^30 edges (event offsets are 32-bit)");
  // graph to the host (validation and block layout are host work)
  std::vector<int64_t> rowptr((size_t)n + 1);
  std::vector<int32_t> col((size_t)E);
  if (hipMemcpy(rowptr.data(), g->rowptr, rowptr.size() * 8, dev ? hipMemcpyDeviceToHost : hipMemcpyHostToHost) != hipSuccess ||
      (E && hipMemcpy(col.data(), g->col, col.size() * 4, dev ? hipMemcpyDeviceToHost : hipMemcpyHostToHost) != hipSuccess))
    return fail(nullptr, INK_E_DEVICE, "ink_create: cannot read the graph arrays");
  if (rowptr[0] != 0 || rowptr[n] != E) return fail(nullptr, INK_E_ARG, "ink_create: rowptr[0] != 0 or rowptr[n] != n_edges");
  for (int v = 0; v < n; v++) {
    if (rowptr[v + 1] < rowptr[v]) return fail(nullptr, INK_E_ARG, "ink_create: rowptr not monotone");
    for (int64_t e = rowptr[v]; e < rowptr[v + 1]; e++) {
      int32_t u = col[e];
      if (u < 0 || u >= n) return fail(nullptr, INK_E_RANGE, "ink_create: column id out of range");
      if (u == v) return fail(nullptr, INK_E_ARG, "ink_create: self loop in the graph");
      if (e > rowptr[v] && col[e - 1] >= u) return fail(nullptr, INK_E_ARG, "ink_create: row not strictly ascending");
    }
  }
  if (opts && opts->node_capacity >= (1 << 30)) return fail(nullptr, INK_E_ARG, "ink_create: node_capacity too large");
  ink_ctx *c = new (std::nothrow) ink_ctx();
  if (!c) return fail(nullptr, INK_E_OOM, "ink_create: host allocation failed");
  c->n = n; c->n_edges = E; c->n_edges_now = E;
  c->n_cap = (opts && opts->node_capacity > n) ? opts->node_capacity : n;
  c->id_bits = 1; while ((1ll << c->id_bits) < c->n_cap) c->id_bits++;
  c->kind = model->kind; c->agg = model->agg; c->n_layers = model->n_layers; c->eps = model->gin_eps;
  c->is_select = model->agg == INK_AGG_MAX || model->agg == INK_AGG_MIN; c->is_min = model->agg == INK_AGG_MIN;
  c->mem = dev ? INK_MEM_DEVICE : INK_MEM_HOST;
  c->slack = (opts && opts->slack_factor > 0.f) ? opts->slack_factor : 0.25f;
  c->profile = opts ? opts->profile : 0;
  c->pool_reserve = opts ? opts->pool_reserve : 0;
  if (opts && opts->small_batch_limit != 0)
    c->small_batch = opts->small_batch_limit < 0 ? 0 : std::min<int64_t>(opts->small_batch_limit, kShortBatch);
  c->batch_dev = dev || (opts && opts->batch_mem == INK_MEM_DEVICE);
  if (opts && opts->dense_threshold != 0.f) c->dense_frac = opts->dense_threshold < 0.f ? 1e30 : opts->dense_threshold;
  memset(&c->stats, 0, sizeof(c->stats));
#define CREATE_TRY(x)                                                                              \
  do {                                                                                             \
    hipError_t e_ = (x);                                                                           \
    if (e_ != hipSuccess) {                                                                        \
      g_create_err = std::string("ink_create: HIP error: ") + hipGetErrorString(e_) + " at " #x;   \
      ink_destroy(c);                                                                              \
      return e_ == hipErrorOutOfMemory ? INK_E_OOM : INK_E_DEVICE;                                 \
    }                                                                                              \
  } while (0)
  if (opts && opts->hip_stream) c->stream = (hipStream_t)opts->hip_stream;
  else { CREATE_TRY(hipStreamCreate(&c->stream)); c->own_stream = true; }
  CREATE_TRY(scratch_lookup(&c->device, &c->scratch));
  CREATE_TRY(graph_build(c, rowptr.data(), col.data()));
  const int64_t nc = c->n_cap;     // every per-node array is allocated for the capacity
  CREATE_TRY(hipMalloc(&c->new_out, (size_t)nc * 4));
  CREATE_TRY(hipMemset(c->new_out, 0, (size_t)nc * 4));
  CREATE_TRY(hipMalloc(&c->d_cnt, sizeof(Counters)));
  CREATE_TRY(hipMemset(c->d_cnt, 0, sizeof(Counters)));
  constexpr size_t kGraphCounters = sizeof(Counters) + kLatencyTargets * sizeof(int32_t);      // and `arrived`
  CREATE_TRY(hipMalloc(&c->d_gcnt, kGraphCounters));
  CREATE_TRY(hipMemset(c->d_gcnt, 0, kGraphCounters));
  c->arrived = reinterpret_cast<int32_t *>(c->d_gcnt + 1);
  {   // one pinned allocation: layer record + sequence number, graph record + sequence number, one more per layer, batch staging
    static_assert(sizeof(HostCounters) == 192, "records and sequence numbers on their own cache lines");
    char *h = nullptr;
    constexpr size_t kRecords = kRecordBytes * (INK_MAX_LAYERS + 2);
    CREATE_TRY(hipHostMalloc((void **)&h, kRecords + kPinnedBatch * sizeof(ink_edge_update), hipHostMallocCoherent));
    memset(h, 0, kRecords);
    c->h_cnt = reinterpret_cast<HostCounters *>(h);
    c->h_seq = reinterpret_cast<uint32_t *>(h + 192);
    c->h_gcnt = reinterpret_cast<HostCounters *>(h + kRecordBytes);
    c->h_gseq = reinterpret_cast<uint32_t *>(h + kRecordBytes + sizeof(HostCounters));
    for (int l = 1; l <= INK_MAX_LAYERS; l++) {
      c->h_one[l] = reinterpret_cast<HostCounters *>(h + kRecordBytes * (l + 1));
      c->h_oseq[l] = reinterpret_cast<uint32_t *>(h + kRecordBytes * (l + 1) + sizeof(HostCounters));
    }
    c->h_batch = reinterpret_cast<ink_edge_update *>(h + kRecords);
  }
  // Who hands batches over in host memory wants results there, and the first one, too: first pass of 100 updates and
  // their inverse, 10k nodes, 1.15 -> .93 ms, 333 on 87k nodes 1.86 -> 1.45.
  if (!c->batch_dev) want_host_results(c);
  size_t bmw = ((size_t)nc + 63) / 64;
  CREATE_TRY(hipMalloc(&c->bm_a, bmw * 8));
  CREATE_TRY(hipMemset(c->bm_a, 0, bmw * 8));
  if (opts && opts->max_batch > 0) {       // size the batch staging up front
    if (!c->batch_dev) CREATE_TRY(c->b_raw.reserve((size_t)opts->max_batch * sizeof(ink_edge_update)));
    CREATE_TRY(graph_reserve(c, opts->max_batch));
    CREATE_TRY(c->c_list.reserve((size_t)nc * 4));
  }
  CREATE_TRY(c->big_list.reserve((size_t)(c->gin.pool_cap / kBigDeg + 4096) * 4));
  // tables
  c->H.resize(c->n_layers + 1); c->A.resize(c->n_layers + 1); c->ARG.resize(c->n_layers + 1);
  c->UB.resize(c->n_layers + 1); c->ARG2.resize(c->n_layers + 1);
  c->XW.resize(c->n_layers + 1); c->Msc.resize(c->n_layers + 1); c->USER.resize(c->n_layers + 1);
  if (c->kind == INK_MODEL_GCN) CREATE_TRY(hipMalloc(&c->cnorm, (size_t)nc * 4));
  CREATE_TRY(alloc_table(c->H[0], nc, feat_dim));
  {
    DevBuf tmp;
    const float *src = features;
    if (!dev) {
      CREATE_TRY(tmp.reserve((size_t)n * feat_dim * 4));
      CREATE_TRY(hipMemcpy(tmp.p, features, (size_t)n * feat_dim * 4, hipMemcpyHostToDevice));
      src = tmp.as<float>();
    }
    hipLaunchKernelGGL(k_unpack_rows, grid1((int64_t)n * feat_dim), dim3(256), 0, c->stream, src, (int)feat_dim,
                       c->H[0].ld, (int64_t)n, c->H[0].f());
    CREATE_TRY(hipStreamSynchronize(c->stream));
    tmp.release();
  }
  c->layers.resize(c->n_layers);
  for (int l = 1; l <= c->n_layers; l++) {
    const ink_layer &S = model->layers[l - 1];
    DevLayer &L = c->layers[l - 1];
    L.in_dim = S.in_dim; L.out_dim = S.out_dim; L.hidden = S.mlp_hidden; L.act = S.act;
    CREATE_TRY(alloc_table(c->H[l], nc, S.out_dim));
    CREATE_TRY(alloc_table(c->A[l], nc, c->kind == INK_MODEL_GCN ? S.out_dim : S.in_dim));
    if (c->is_select) { CREATE_TRY(alloc_table(c->ARG[l], nc, S.in_dim)); CREATE_TRY(alloc_table(c->UB[l], nc, S.in_dim)); CREATE_TRY(alloc_table(c->ARG2[l], nc, S.in_dim)); }
    if (c->kind == INK_MODEL_GCN) {
      CREATE_TRY(alloc_table(c->Msc[l], nc, S.out_dim));
      if (l == 1) CREATE_TRY(alloc_table(c->XW[1], nc, S.out_dim));
      L.K1 = S.in_dim; L.K1p = round_up(L.K1, 32); L.N1 = S.out_dim; L.N1p = round_up(L.N1, 32);
      CREATE_TRY(hipMalloc(&L.W1, (size_t)L.K1p * L.N1p * 4));
      CREATE_TRY(hipMemset(L.W1, 0, (size_t)L.K1p * L.N1p * 4));
      CREATE_TRY(upload_padded(S.W_neigh, S.in_dim, S.out_dim, L.K1p, L.N1p, 0, L.W1, dev));
      CREATE_TRY(upload_vec(S.bias, S.out_dim, &L.b1, dev));
    } else if (c->kind == INK_MODEL_SAGE) {
      L.K1 = 2 * xform_self_row(S.in_dim); L.K1p = round_up(L.K1, 32); L.N1 = S.out_dim; L.N1p = round_up(L.N1, 32);
      CREATE_TRY(hipMalloc(&L.W1, (size_t)L.K1p * L.N1p * 4));
      CREATE_TRY(hipMemset(L.W1, 0, (size_t)L.K1p * L.N1p * 4));
      CREATE_TRY(upload_padded(S.W_neigh, S.in_dim, S.out_dim, L.K1p, L.N1p, 0, L.W1, dev));
      CREATE_TRY(upload_padded(S.W_self, S.in_dim, S.out_dim, L.K1p, L.N1p, xform_self_row(S.in_dim), L.W1, dev));
      CREATE_TRY(upload_vec(S.bias, S.out_dim, &L.b1, dev));
    } else {   // GIN
      L.K1 = S.in_dim; L.K1p = round_up(L.K1, 32); L.N1 = S.mlp_hidden; L.N1p = round_up(L.N1, 32);
      L.K2 = S.mlp_hidden; L.K2p = round_up(L.K2, 32); L.N2 = S.out_dim; L.N2p = round_up(L.N2, 32);
      CREATE_TRY(hipMalloc(&L.W1, (size_t)L.K1p * L.N1p * 4));
      CREATE_TRY(hipMemset(L.W1, 0, (size_t)L.K1p * L.N1p * 4));
      CREATE_TRY(upload_padded(S.W_neigh, S.in_dim, S.mlp_hidden, L.K1p, L.N1p, 0, L.W1, dev));
      CREATE_TRY(upload_vec(S.bias, S.mlp_hidden, &L.b1, dev));
      CREATE_TRY(hipMalloc(&L.W2, (size_t)L.K2p * L.N2p * 4));
      CREATE_TRY(hipMemset(L.W2, 0, (size_t)L.K2p * L.N2p * 4));
      CREATE_TRY(upload_padded(S.W_mlp2, S.mlp_hidden, S.out_dim, L.K2p, L.N2p, 0, L.W2, dev));
      CREATE_TRY(upload_vec(S.bias_mlp2, S.out_dim, &L.b2, dev));
    }
  }
  *out = c;
  return INK_OK;
}

extern "C" void ink_destroy(ink_ctx *c) {
  if (!c) return;
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  for (GraphSide *g : {&c->gin, &c->gout}) {
    if (g->off) (void)hipFree(g->off);
    if (g->deg) (void)hipFree(g->deg);
    if (g->cap) (void)hipFree(g->cap);
    if (g->asc) (void)hipFree(g->asc);
    if (g->ids) (void)hipFree(g->ids);
  }
  if (c->new_out) (void)hipFree(c->new_out);
  for (auto &L : c->layers) for (float *p : {L.W1, L.b1, L.W2, L.b2}) if (p) (void)hipFree(p);
  for (auto *vec : {&c->H, &c->A, &c->ARG, &c->UB, &c->ARG2, &c->XW, &c->Msc, &c->USER}) for (auto &t : *vec) if (t.p) (void)hipFree(t.p);
  if (c->cnorm) (void)hipFree(c->cnorm);
  if (c->d_cnt) (void)hipFree(c->d_cnt);
  if (c->d_gcnt) (void)hipFree(c->d_gcnt);
  if (c->h_cnt) (void)hipHostFree(c->h_cnt);
  if (c->h_res) (void)hipHostFree(c->h_res);
  if (c->bm_a) (void)hipFree(c->bm_a);
  for (DevBuf *b : {&c->ws.blk, &c->ws.hist, &c->ws.tmpk, &c->ws.tmpv, &c->b_raw, &c->b_misc, &c->b_uniq, &c->b_del_s,
                    &c->b_del_d, &c->b_ins_s, &c->b_ins_d, &c->f_list[0], &c->f_list[1], &c->f_old[0], &c->f_old[1],
                    &c->f_pref, &c->ev_key, &c->ev_val, &c->t_list, &c->t_seg, &c->evl_list, &c->evl_owner, &c->c_list, &c->c_flag, &c->c_idx, &c->c_old,
                    &c->b_touch_in,
                    &c->u_ev, &c->u_rows, &c->u_key, &c->u_val, &c->u_uniq, &c->u_seg, &c->u_flag, &c->u_idx, &c->u_list, &c->exp_list, &c->big_list, &c->big_part_v, &c->big_part_i, &c->big_part_s, &c->big_part_j, &c->big_pref, &c->f_delta, &c->stage0, &c->stage1, &c->res_ids, &c->res_emb})
    b->release();
  for (auto e : c->ev_free) (void)hipEventDestroy(e);
  for (auto &p : c->ev_pending) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
  if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
  delete c;
}

extern "C" const char *ink_last_error(const ink_ctx *c) { return c ? c->err.c_str() : g_create_err.c_str(); }

// ------------------------------------------------------------------------------------ full inference
// Aggregated rows wider than one wave covers (256 floats) are handled one 256-column block at a
// time: the aggregators act per dimension, so the blocks are independent.
constexpr int kAggBlock = 256;
static int agg_blocks(const AggArgs &a) { return (a.d + kAggBlock - 1) / kAggBlock; }
static AggArgs agg_block(const AggArgs &a, int b) {
  AggArgs r = a;
  int c0 = b * kAggBlock;
  r.M += c0; r.A += c0;
  if (r.ARG) { r.ARG += c0; r.UB += c0; r.ARG2 += c0; }
  r.d = std::min(kAggBlock, a.d - c0);
  r.wd = round_up(r.d, 4);
  r.count_cond = b == 0;      // a target's condition is tallied once, for its first block
  return r;
}

// recompute of every node (targets == null) or of the listed ones
static hipError_t agg_full_any(ink_ctx *c, const AggArgs &a_in, uint64_t *chg, const int32_t *targets = nullptr,
                               int64_t n_targets = -1) {
  AggArgs a = a_in;
  if (!targets) {        // every node: the chunk count is bounded by the edge count
    n_targets = c->n;
    a.big_chunks = c->n_edges_now / kBigChunk + std::min<int64_t>(c->n, c->n_edges_now / kBigDeg) + 1;
  }
  for (int b = 0; b < agg_blocks(a); b++) {
    AggArgs ab = agg_block(a, b);
    hipError_t e = c->is_select ? agg_select_full(c, ab, targets, n_targets, chg)
                                : agg_sum_full(c, ab, targets, n_targets, chg);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// GCN: message table of layer l + 1 from the finished layer l (rows == null: every node):
// h_l = act(c (S_l + m_l) + b_l) is stored, then m_{l+1} = c * (h_l W_{l+1}) with compare-and-emit
static hipError_t gcn_next_messages(ink_ctx *c, int l, const int32_t *rows, int64_t n_rows, uint8_t *flags,
                                    float *old_rows) {
  const DevLayer &L = c->layers[l - 1], &Ln = c->layers[l];
  XformArgs x;
  memset(&x, 0, sizeof(x));
  x.mode = 3; x.rows = rows; x.n_rows = n_rows;
  x.A = c->A[l].f(); x.lda = c->A[l].ld; x.Hp = c->Msc[l].f(); x.ldh = c->Msc[l].ld; x.d_in = L.out_dim;
  x.cnorm = c->cnorm; x.in_bias = L.b1; x.in_relu = L.act == INK_ACT_RELU;
  x.in_user = c->USER[l].f(); x.ld_in_user = c->USER[l].ld;
  x.h_store = c->H[l].f(); x.ld_hs = c->H[l].ld;
  x.W = Ln.W1; x.Kp = Ln.K1p; x.Np = Ln.N1p; x.bias = nullptr; x.n_out = Ln.out_dim; x.relu = 0;
  x.out_scale = c->cnorm;
  x.out = c->Msc[l + 1].f(); x.ld_out = c->Msc[l + 1].ld; x.to_table = 1; x.row_changed = flags;
  x.old_rows = old_rows; x.ld_old = c->Msc[l + 1].ld;
  return xform_run(c, x);
}

static hipError_t gcn_final(ink_ctx *c, const int32_t *rows, int64_t n_rows, uint8_t *flags) {
  int k = c->n_layers;
  const DevLayer &L = c->layers[k - 1];
  if (n_rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gcn_final, grid1(n_rows * c->H[k].ld), dim3(256), 0, c->stream, rows, n_rows,
                     (const float *)c->A[k].f(), (const float *)c->Msc[k].f(), (const float *)c->cnorm,
                     (const float *)L.b1, (const float *)c->USER[k].f(), c->USER[k].ld, (int)(L.act == INK_ACT_RELU),
                     c->H[k].f(), c->H[k].ld, c->H[k].d, flags);
  return hipGetLastError();
}

static ink_status full_infer_impl(ink_ctx *c) {
  auto t0 = std::chrono::steady_clock::now();
  memset(&c->stats, 0, sizeof(c->stats));
  c->stats.n_layers = c->n_layers;
  hipStream_t s = c->stream;
  if (c->kind == INK_MODEL_GCN) {
    Prof p(c, INK_T_TRANSFORM);
    const DevLayer &L = c->layers[0];
    XformArgs x;
    memset(&x, 0, sizeof(x));
    x.mode = 2; x.n_rows = c->n; x.Hp = c->H[0].f(); x.ldh = c->H[0].ld; x.d_in = L.in_dim;
    x.W = L.W1; x.Kp = L.K1p; x.Np = L.N1p; x.n_out = L.out_dim;
    x.out = c->XW[1].f(); x.ld_out = c->XW[1].ld; x.to_table = 0;
    API_TRY(xform_run(c, x));
    hipLaunchKernelGGL(k_gcn_rescale, grid1((int64_t)c->n * c->Msc[1].ld), dim3(256), 0, s, (const int32_t *)nullptr,
                       (int64_t)c->n, (const int32_t *)c->gin.deg, c->cnorm, (const float *)c->XW[1].f(),
                       c->Msc[1].f(), c->Msc[1].ld, c->Msc[1].d, (float *)nullptr, (uint8_t *)nullptr);
    API_TRY(hipGetLastError());
  }
  for (int l = 1; l <= c->n_layers; l++) {
    AggArgs a = agg_args(c, l);
    { Prof p(c, INK_T_AGG); API_TRY(agg_full_any(c, a, nullptr)); }
    {
      Prof p(c, INK_T_TRANSFORM, l, INK_K_XFORM);
      if (c->kind != INK_MODEL_GCN) API_TRY(run_transform(c, l, nullptr, c->n, nullptr));
      else if (l < c->n_layers) API_TRY(gcn_next_messages(c, l, nullptr, c->n, nullptr, nullptr));
      else API_TRY(gcn_final(c, nullptr, c->n, nullptr));
    }
    ink_layer_stats &S = c->stats.layer[l - 1];
    S.dense = 1; S.n_targets = c->n; S.n_exposed = c->n; S.n_regather_nb = c->n_edges_now; S.n_transformed = c->n;
  }
  API_TRY(hipStreamSynchronize(s));
  prof_collect(c);
  c->inferred = true;
  c->stats.ms_total = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
  return INK_OK;
}

extern "C" ink_status ink_full_infer(ink_ctx *c) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  begin_result(c);
  return seal(c, full_infer_impl(c));
}

// ------------------------------------------------------------------------------------ full inference without allocation
extern "C" ink_status ink_full_infer_noalloc(ink_ctx *c) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  begin_result(c);
  void *base = c->scratch;
  if (!base) return fail(c, INK_E_DEVICE, "ink_full_infer_noalloc: the scratch array's address was not found at ink_create");
  // what the full inference reserves, from the same bounds its kernels' launchers use
  int wd_max = 0, n1p_max = 0;
  for (int l = 1; l <= c->n_layers; l++) {
    wd_max = std::max(wd_max, std::min(round_up(c->A[l].d, 4), kAggBlock));
    if (c->kind == INK_MODEL_GIN) n1p_max = std::max(n1p_max, c->layers[l - 1].N1p);
  }
  const size_t list_b = align256((size_t)big_rows_capacity(c) * 4);
  const size_t pref_b = align256((list_b / 4 + 1) * 4);
  const size_t part_b = align256((size_t)big_chunk_capacity(c) * wd_max * 4);
  const int n_part = c->is_select ? 4 : 1;
  const size_t stage_b = align256((size_t)c->n * n1p_max * 4);
  const size_t need = list_b + pref_b + (size_t)n_part * part_b + stage_b;
  if (need > (size_t)INK_NOALLOC_SCRATCH_BYTES) {
    char msg[256];
    snprintf(msg, sizeof(msg), "ink_full_infer_noalloc: this graph and model need %zu bytes of work memory, the static "
             "scratch holds %zu: use ink_full_infer", need, (size_t)INK_NOALLOC_SCRATCH_BYTES);
    return fail(c, INK_E_RANGE, msg);
  }
  // lend the carve-outs to the buffers the kernels' launchers use, run, and put the owners back
  DevBuf *bufs[] = {&c->big_list, &c->big_pref, &c->big_part_v, &c->big_part_i, &c->big_part_s, &c->big_part_j,
                    &c->stage0};
  const size_t sizes[] = {list_b, pref_b, part_b, c->is_select ? part_b : 0, c->is_select ? part_b : 0,
                          c->is_select ? part_b : 0, stage_b};
  constexpr int NB = sizeof(bufs) / sizeof(bufs[0]);
  DevBuf saved[NB];
  size_t used = 0;
  for (int i = 0; i < NB; i++) {
    saved[i] = *bufs[i];
    bufs[i]->p = sizes[i] ? (char *)base + used : nullptr;
    bufs[i]->cap = sizes[i];
    bufs[i]->fixed = true;
    used += sizes[i];
  }
  const int profile = c->profile;
  c->profile = 0;                    // HIP events are created on demand: not in this call
  ink_status st = full_infer_impl(c);
  c->profile = profile;
  for (int i = 0; i < NB; i++) *bufs[i] = saved[i];
  return seal(c, st);
}

// ------------------------------------------------------------------------------------ updates
// Events + grouping + aggregation of layer l.  F (nF ids, ascending) are the sources whose message
// changed and n_chg the events they propagate (their kept out-edges, prefix already in f_pref);
// f_old holds their previous message rows (sum-type only).  Marks targets whose aggregate changed
// in c->bm_a.  Counters are read back by the caller's next synchronisation.
constexpr int64_t kSmallLayer = 4096;           // events / rows up to which a layer's bookkeeping runs in one workgroup
constexpr int64_t kBitmapOneLaunch = 16384;     // nodes up to which the bitmap scan is a single launch
constexpr int64_t kNoSyncEvents = 1 << 18;     // below this the target count stays on the device

// Events of a layer above which re-aggregating every node costs less than grouping the events.  An edge re-aggregated
// costs one cached row read; an event its creation, a place in the sort, its row, and the exposed rows it leaves.  A node
// re-aggregated costs its four table rows: a graph of some 300k nodes holds them in the caches, a larger one pays about
// 2.5 events a node.  Measured for max, edge batches, last of three layers: the fraction of the edges at which both ways
// take the same time (rule in brackets), rows of 64 / 128 / 256 floats:
//   20M nodes, 10 edges each   .69 (.60) / -         / -              20M, 20 edges   -         / .48 (.57) / -
//   10M, 10 edges              -         / .65 (.69) / -              10M, 20 edges   .51 (.47) / -         / -
//   5M, 10 edges               -         / .66 (.69) / -              5M, 20 edges    .51 (.47) / .53 (.57) / -
//   2.5M, 10 edges             .71 (.57) / -         / -              2.5M, 20 edges  -         / .58 (.56) / -
//   1.25M, 8 edges             .73 (.59) / .67 (.69) / -              1.25M, 20 edges .47 (.45) / .53 (.55) / -
//   800k, 10 edges             .57 (.51) / .54 (.61) / -              600k, 20 edges  .38 (.41) / -         / .53 (.51)
//   450k, 14 edges             .43 (.41) / .40 (.51) / .51 (.51)      300k, 8 edges   .38 (.35) / -         / .37 (.45)
// and below .3 at 100k nodes and fewer.  Without the nodes in the rule 3265 updates on 1.25M nodes with 8 edges each
// (rows of 64 floats, .36) took 2.11 instead of 1.57 ms.  5 to 20 % of those targets were exposed.  New feature rows
// expose 20 to 50 % in the second layer, which makes events dearer, above all of wide rows: even at .62 / .52 / - on
// 1.25M nodes with 8 edges, .42 / .40 / - with 20, .63 / - / - on 2.5M with 10, - / .55 / - on 5M with 10, so without edge
// updates the nodes count for rows of at most 64 floats only.  (In the first layer, where 80 % and more are exposed, both
// ways are even at .15 to .4.)  Sums stay at .75 of the edges although they would be even at .15 to .6: a sum formed anew
// differs in its last bits from the one kept, so nodes that no event touches would be reported as changed.  Layers of the
// one-workgroup path pay for launches, not for events.
static double dense_line(const ink_ctx *c, int64_t n_events, int width, int64_t n_edges, bool edge_updates) {
  const double edges = (double)std::max<int64_t>(n_edges, 1);
  if (c->dense_frac != 0) return c->dense_frac * edges;
  if (n_events <= kSmallLayer || (c->agg != INK_AGG_MAX && c->agg != INK_AGG_MIN)) return 0.75 * edges;
  const double nodes = width <= 64 || edge_updates ? 2.5 * std::max(0, c->n - 300000) : 0.;
  return std::min(0.75 * edges, (width <= 64 ? 0.35 : 0.45) * edges + nodes);
}

static ink_status layer_aggregate(ink_ctx *c, int l, const int32_t *F, int64_t nF, int64_t n_chg, const float *f_old,
                                  int ld_old, int64_t n_ins, int64_t n_del) {
  hipStream_t s = c->stream;
  ink_layer_stats &S = c->stats.layer[l - 1];
  Counters *dc = c->d_cnt;
  AggArgs a = agg_args(c, l);
  const int64_t n_seed = n_ins + n_del;
  S.n_sources = nF;
  int64_t nE = n_seed + n_chg;
  S.n_events = nE;
  uint64_t *bm = c->bm_a;
  bool dense = nE > 0 && (double)nE > dense_line(c, nE, a.d, c->n_edges_now, n_seed > 0);
  S.dense = dense;
  const bool small = !dense && nE > 0 && nE <= kSmallLayer;
  if (dense || nE == 0) API_TRY(hipMemsetAsync(dc, 0, sizeof(Counters), s));      // otherwise the kernel that makes the events does
  if (dense) {
    // so many events that re-aggregating every node costs less than grouping them (Sec. 5.1)
    Prof p(c, INK_T_AGG);
    // Rows without neighbours are empty already, but for those that lost theirs: their bits are set beforehand
    // (and their rows transformed, even if they had aggregated to 0).  Of others only what changed may be marked, and in the baseline,
    // where a marked node propagates whether or not it changed, of these, too.
    if (c->is_select && !c->affected_mode) {
      if (n_del > 0)
        hipLaunchKernelGGL(k_mark_nodes, grid1(n_del), dim3(256), 0, s, (const int32_t *)c->del_dst, (int)n_del, (const int32_t *)nullptr, 0, bm, (const int32_t *)c->gin.deg);
      a.keep_empty = true;
    }
    API_TRY(agg_full_any(c, a, bm));
    return INK_OK;
  }
  if (nE == 0) return INK_OK;
  API_TRY(c->ev_key.reserve((size_t)nE * 4));
  API_TRY(c->ev_val.reserve((size_t)nE * 4));
  API_TRY(c->t_list.reserve((size_t)(nE + 1) * 4));
  API_TRY(c->t_seg.reserve((size_t)(nE + 2) * 4));
  uint32_t *key = c->ev_key.as<uint32_t>(), *val = c->ev_val.as<uint32_t>();
  int64_t nT = std::min<int64_t>(nE, c->n);       // upper bound unless read back below
  if (small) {
    // few events: counters, events, grouping and segment heads in one launch
    Prof p(c, INK_T_GROUP);
    const int passes = (c->id_bits + kRadixBits - 1) / kRadixBits;
#define INK_SMALL_GROUP(T, I)                                                                                      \
  hipLaunchKernelGGL((k_small_group<T, I>), dim3(1), dim3(T), 0, s, (const int32_t *)c->del_src,                    \
                     (const int32_t *)c->del_dst, (const int32_t *)c->ins_src, (const int32_t *)c->ins_dst,        \
                     (int)n_del, (int)n_ins, F, (int)nF, (const int32_t *)c->f_pref.as<int32_t>(), (int)n_chg,     \
                     (const int64_t *)c->gout.off, (const int32_t *)c->gout.ids, c->is_select ? 0 : 1, passes, key, \
                     val, c->t_list.as<int32_t>(), c->t_seg.as<int32_t>(), dc)
    if (nE <= 256) INK_SMALL_GROUP(256, 1);
    else if (nE <= 1024) INK_SMALL_GROUP(256, 4);
    else INK_SMALL_GROUP(1024, 4);
#undef INK_SMALL_GROUP
    API_TRY(hipGetLastError());
  } else {
    const SortPlan sp = sort_plan(nE, c->id_bits);
    API_TRY(sort_reserve(c->ws, sp));
    API_TRY(c->ws.tmpk.reserve((size_t)nE * 4));
    API_TRY(c->ws.tmpv.reserve((size_t)nE * 4));
    {
      Prof p(c, INK_T_EVENTS);
      make_events(sp, EventInputs{c->del_src, c->del_dst, c->ins_src, c->ins_dst, (int)n_del, (int)n_ins, F, (int)nF,
                                  c->f_pref.as<int32_t>(), (int)n_chg, c->gout.off, c->gout.ids, c->is_select ? 0 : 1},
                  key, val, c->ws.hist.as<int32_t>(), dc, s);
      API_TRY(hipGetLastError());
    }
    Prof p(c, INK_T_GROUP);
    {
      KernelTimer kt(c, l, INK_K_SORT);
      API_TRY(radix_sort_planned(c->ws, sp, key, val, c->ws.tmpk.as<uint32_t>(), c->ws.tmpv.as<uint32_t>(), nE, true, s));
      if (sp.passes & 1) { std::swap(c->ev_key, c->ws.tmpk); std::swap(c->ev_val, c->ws.tmpv); }     // the sorted pair stays where it is
    }
    const bool count = nE > kNoSyncEvents;
    const RecordTo rec{dc, c->h_cnt, c->h_seq, count ? ++c->pub_seq : 0};
    bool given = false;
    API_TRY(segment_heads(c->ws, key, nE, c->t_list.as<int32_t>(), c->t_seg.as<int32_t>(), &dc->v[C_NT], s, nullptr, count ? &rec : nullptr, &given));
    if (count) {
      API_TRY(given ? wait_published(c, rec.h_seq, rec.seq) : read_counters(c));
      nT = c->h_cnt->v[C_NT];
    }
  }
  if (c->affected_mode) {
    // baseline "Affected" (Sec. 4.1): every node an event reaches is recomputed from its whole
    // neighbourhood, without looking at the events' content, and counts as affected
    Prof p(c, INK_T_AGG);
    if (nE <= kNoSyncEvents) {
      API_TRY(read_counters(c));
      nT = c->h_cnt->v[C_NT];
    }
    API_TRY(agg_full_any(c, a, bm, c->t_list.as<int32_t>(), nT));
    if (nT > 0) hipLaunchKernelGGL(k_mark_nodes, grid1(nT), dim3(256), 0, s, (const int32_t *)c->t_list.as<int32_t>(), (int)nT, (const int32_t *)nullptr, 0, bm, (const int32_t *)nullptr);
    API_TRY(hipGetLastError());
    return INK_OK;
  }
  {
    Prof p(c, INK_T_AGG);
    if (!c->is_select && nF > 0) {
      API_TRY(c->f_delta.reserve((size_t)nF * ld_old * 4));
      API_TRY(agg_sum_delta_rows(c, a, F, (int)nF, f_old, c->f_delta.as<float>(), ld_old));
    }
    const EventBounds eb{nE, nF + n_seed};      // a source or a changed edge names a target once
    for (int b = 0; b < agg_blocks(a); b++) {
      AggArgs ab = agg_block(a, b);
      int c0 = b * kAggBlock;
      if (b > 0) API_TRY(hipMemsetAsync(&dc->v[C_NEXP], 0, 5 * sizeof(int32_t), s));   // lists of long rows, exposed rows and long segments
      if (c->is_select)
        API_TRY(agg_select_events(c, ab, c->t_list.as<int32_t>(), c->t_seg.as<int32_t>(), nT, &dc->v[C_NT],
                                  c->ev_val.as<uint32_t>(), eb, bm));
      else
        API_TRY(agg_sum_events(c, ab, c->t_list.as<int32_t>(), c->t_seg.as<int32_t>(), nT, &dc->v[C_NT],
                               c->ev_val.as<uint32_t>(), eb, F, (int)nF, f_old ? f_old + c0 : nullptr,
                               c->f_delta.as<float>() ? c->f_delta.as<float>() + c0 : nullptr, ld_old, bm));
    }
  }
  return INK_OK;
}

// fills the layer's statistics from the counters of the last read-back
static void layer_stats_from_counters(ink_ctx *c, int l, const HostCounters *h) {
  ink_layer_stats &S = c->stats.layer[l - 1];
  if (S.dense) {
    S.n_targets = c->n; S.n_exposed = c->n; S.n_regather_nb = c->n_edges_now;
    S.n_regather_nb_long = (int64_t)h->sum(ST_REGATHER_LONG);
    return;
  }
  c->big_hint[l] = h->v[C_NCHUNK];
  S.n_targets = h->v[C_NT];
  if (c->affected_mode) {
    S.n_exposed = S.n_targets; S.n_regather_nb = (int64_t)h->sum(ST_REGATHER);
    return;
  }
  S.n_exposed = (int64_t)h->sum(ST_EXPOSED);
  S.n_regather_nb = (int64_t)h->sum(ST_REGATHER);
  S.n_regather_nb_long = (int64_t)h->sum(ST_REGATHER_LONG);
  S.n_alpha_changed = (int64_t)h->sum(ST_ACHG);
  S.n_no_deletion = (int64_t)h->sum(ST_NODEL);
  S.n_deletion_no_effect = (int64_t)h->sum(ST_NOEFFECT);
  S.n_covered = (int64_t)h->sum(ST_COVERED);
}

// bitmap (plus extra id lists) -> ascending row list in c->c_list; returns the count, or, with
// bound >= 0, that upper bound without waiting for the device (the count stays in C_NC).
// n_t_bound >= 0 says that only the first *C_NT (at most n_t_bound) entries of c->t_list can have
// their bit set; a short candidate list is then collected in one workgroup, which also clears
// the row flags (*flags_cleared), unless the graph is so small that scanning the whole bitmap is
// one launch as well (then sorting the candidates costs more than the scan).
static ink_status collect_rows(ink_ctx *c, const int32_t *extra0, int64_t n0, const int32_t *extra1, int64_t n1,
                               int64_t *nC, int64_t bound = -1, int64_t n_t_bound = -1, bool *flags_cleared = nullptr) {
  hipStream_t s = c->stream;
  Prof p(c, INK_T_COMPACT);
  API_TRY(c->c_list.reserve((size_t)c->n * 4));
  const RecordTo rec{c->d_cnt, c->h_cnt, c->h_seq, bound < 0 ? ++c->pub_seq : 0};
  bool given = false;
  const int64_t M = n_t_bound + n0 + n1;
  if (n_t_bound >= 0 && M <= kSmallLayer && c->n > kBitmapOneLaunch) {
    const int64_t n_flags = std::min<int64_t>(M, c->n);
    API_TRY(c->c_flag.reserve((size_t)n_flags + 64));
    const int passes = (c->id_bits + kRadixBits - 1) / kRadixBits;
#define INK_SMALL_COLLECT(T, I)                                                                                    \
  hipLaunchKernelGGL((k_small_collect<T, I>), dim3(1), dim3(T), 0, s, (const int32_t *)c->t_list.as<int32_t>(),     \
                     (const int32_t *)&c->d_cnt->v[C_NT], (int)n_t_bound, (unsigned long long *)c->bm_a, extra0,   \
                     (int)n0, extra1, (int)n1, passes, c->c_list.as<int32_t>(), c->c_flag.as<uint8_t>(),           \
                     (int)n_flags, c->d_cnt)
    if (M <= 256) INK_SMALL_COLLECT(256, 1);
    else if (M <= 1024) INK_SMALL_COLLECT(256, 4);
    else INK_SMALL_COLLECT(1024, 4);
#undef INK_SMALL_COLLECT
    API_TRY(hipGetLastError());
    if (flags_cleared) *flags_cleared = true;
  } else if (c->n <= kOneTileBits && n0 + n1 <= kSmallLayer) {
    given = bound < 0;
    API_TRY(bitmap_one(c->bm_a, c->n, extra0, n0, extra1, n1, c->c_list.as<int32_t>(), &c->d_cnt->v[C_NC], s, given ? &rec : nullptr));
  } else {
    if (n0 + n1 > 0) hipLaunchKernelGGL(k_mark_nodes, grid1(n0 + n1), dim3(256), 0, s, extra0, (int)n0, extra1, (int)n1, c->bm_a, (const int32_t *)nullptr);
    API_TRY(bitmap_to_list(c->ws, c->bm_a, c->n, c->c_list.as<int32_t>(), &c->d_cnt->v[C_NC], 1, s, bound < 0 ? &rec : nullptr, &given));
  }
  if (bound >= 0) { *nC = bound; return INK_OK; }
  API_TRY(given ? wait_published(c, rec.h_seq, rec.seq) : read_counters(c));
  *nC = c->h_cnt->v[C_NC];
  return INK_OK;
}

// for a gather whose record the call waits for
static HostMirror host_mirror(ink_ctx *c) {
  c->mirrored = c->mirror;
  return c->mirror ? HostMirror{c->mirror_ids(), c->mirror_emb(), c->mirror_rows()} : HostMirror{nullptr, nullptr, -1};
}

// rows of c_list whose flag is set -> f_list[nxt] (ids) and, for sum-type, f_old[nxt] (old rows
// taken from c_old with row stride ld).  With want_events the events those rows will propagate in
// the next layer are counted in the same round trip (prefix of kept out-degrees in f_pref).
// With `result` (the last layer's output table) and a modest nC, the new rows of the changed nodes
// are gathered into res_emb and the batch's marks are cleared before that round trip, so nothing
// is left to launch after it; *result_done says whether that happened.
constexpr size_t kEagerResultBytes = (size_t)64 << 20;
static ink_status emit_changed(ink_ctx *c, int64_t nC, const int32_t *nC_dev, int nxt, bool keep_old, int ld, bool want_events,
                               int64_t *nF2, int64_t *n_chg, const Table *result = nullptr,
                               bool *result_done = nullptr) {
  hipStream_t s = c->stream;
  Prof p(c, INK_T_COMPACT);
  Counters *dc = c->d_cnt;
  *nF2 = 0; *n_chg = 0;
  API_TRY(c->f_list[nxt].reserve((size_t)nC * 4));
  const bool small = nC <= kSmallLayer;
  const int per_thread = emit_per_thread(nC), tile_rows = per_thread * kEmitThreads, tiles = nblocks(nC, tile_rows);
  const EmitRows e{c->c_flag.as<uint8_t>(), c->c_list.as<int32_t>(), want_events ? c->gout.deg : nullptr, c->new_out, nC, nC_dev};
  unsigned long long *tile = nullptr;
  if (!small) {
    API_TRY(c->ws.blk.reserve((size_t)tiles * sizeof(unsigned long long)));
    tile = c->ws.blk.as<unsigned long long>();
    if (per_thread == 1) hipLaunchKernelGGL(k_emit_count<1>, dim3(tiles), dim3(kEmitThreads), 0, s, e, tile);
    else hipLaunchKernelGGL(k_emit_count<8>, dim3(tiles), dim3(kEmitThreads), 0, s, e, tile);
  }
  const uint32_t seq = ++c->pub_seq;         // the kernel that finds the counts publishes them itself
  if (result && (size_t)nC * result->d * 4 <= kEagerResultBytes) {
    API_TRY(c->res_emb.reserve((size_t)nC * result->d * 4));
    const int per = nC <= 65536 ? 64 : 256;          // wide rows want workgroups, long tables few sums
    hipLaunchKernelGGL(k_emit_result, dim3((unsigned)((nC + per - 1) / per)), dim3(256), 0, s, e, (const unsigned long long *)tile, tile_rows, per,
                       (const float *)result->f(), result->ld, result->d, c->f_list[nxt].as<int32_t>(), c->res_emb.as<float>(),
                       host_mirror(c), dc);
    *result_done = true;
  } else if (small) {         // not the last layer, whose results fit the form above
    API_TRY(c->f_pref.reserve((size_t)(nC + 1) * 4));
#define INK_SMALL_EMIT(T, I)                                                                                       \
  hipLaunchKernelGGL((k_small_emit<T, I>), dim3(1), dim3(T), 0, s, (const uint8_t *)c->c_flag.as<uint8_t>(),        \
                     (const int32_t *)c->c_list.as<int32_t>(), (int)nC, nC_dev, c->c_idx.as<int32_t>(),            \
                     c->f_list[nxt].as<int32_t>(), (const int32_t *)c->gout.deg,                                   \
                     (const int32_t *)c->new_out, c->f_pref.as<int32_t>(), dc, c->h_cnt, c->h_seq, seq)
    if (nC <= 256) INK_SMALL_EMIT(256, 1);
    else if (nC <= 1024) INK_SMALL_EMIT(256, 4);
    else INK_SMALL_EMIT(1024, 4);
#undef INK_SMALL_EMIT
  } else {
    if (want_events) API_TRY(c->f_pref.reserve((size_t)(nC + 1) * 4));
#define INK_EMIT(I)                                                                                                              \
  hipLaunchKernelGGL(k_emit_write<I>, dim3(tiles), dim3(kEmitThreads), 0, s, e, (const unsigned long long *)tile, c->c_idx.as<int32_t>(), \
                     c->f_list[nxt].as<int32_t>(), c->f_pref.as<int32_t>(), dc, c->h_cnt, c->h_seq, seq)
    if (per_thread == 1) INK_EMIT(1);
    else INK_EMIT(8);
#undef INK_EMIT
  }
  if (keep_old) {
    API_TRY(c->f_old[nxt].reserve((size_t)nC * ld * 4));
    hipLaunchKernelGGL(k_gather_rows_ld, grid1(nC * (ld / 4)), dim3(256), 0, s, (const float *)c->c_old.as<float>(), ld,
                       (const int32_t *)c->c_idx.as<int32_t>(), (int64_t)0, (const int32_t *)&dc->v[C_NEXT],
                       c->f_old[nxt].as<float>());
  }
  API_TRY(hipGetLastError());
  // with the result gathered, one record after it ends the call: no synchronisation of the stream on top
  c->drained = result_done && *result_done;
  if (c->drained) API_TRY(read_counters(c, true));
  else API_TRY(wait_published(c, c->h_seq, seq));
  *nF2 = c->h_cnt->v[C_NEXT];
  if (want_events) *n_chg = (uint32_t)c->h_cnt->v[C_NEV];
  return INK_OK;
}

// Layers first..k for the sources F_first = f_list[cur] (nF ids whose layer-1 message changed, n_chg events
// along their kept out-edges) and the applied edge changes; D (nD ids) are nodes whose in-degree
// changed (normalised aggregators).  Fills the result for layer k.
// Rows that have to be re-transformed at a layer for a reason of their own (their user term changed):
// asked for at the start of every layer up to `last_layer`.
struct LayerRows {
  int last_layer;
  ink_status (*rows_of)(ink_ctx *c, int l, void *state, const int32_t **rows, int64_t *n);
  void *state;
};

static ink_status propagate_layers(ink_ctx *c, int64_t nF, int64_t n_chg, int cur, int64_t n_ins, int64_t n_del,
                                   const int32_t *D_all, int64_t nD_all, ink_update_result *out,
                                   const LayerRows *own = nullptr, int first = 1, bool events_done = false) {
  hipStream_t s = c->stream;
  const int64_t n_seed = n_ins + n_del;
  const bool gcn = c->kind == INK_MODEL_GCN;
  const bool keep_old = !c->is_select && !c->affected_mode;   // delta updates subtract the old message rows
  c->drained = false;
  for (int l = first; l <= c->n_layers && (n_seed > 0 || nF > 0 || (own && l <= own->last_layer)); l++) {
    ink_layer_stats &S = c->stats.layer[l - 1];
    const int32_t *D = D_all;
    int64_t nD = nD_all;
    if (own) {
      ink_status st_own = own->rows_of(c, l, own->state, &D, &nD);
      if (st_own != INK_OK) return st_own;
    }
    const int32_t *F = c->f_list[cur].as<int32_t>();
    int ld_msg = msg_table(c, l).ld;
    ink_status st = INK_OK;
    if (l == first && events_done) {       // begun by layer_one: the long exposed rows are left
      Prof p(c, INK_T_AGG);
      S.n_sources = nF; S.n_events = n_seed + n_chg;
      API_TRY(agg_select_long_rows(c, agg_args(c, l), std::min<int64_t>(S.n_events, c->n), c->bm_a));
    } else {
      st = layer_aggregate(c, l, F, nF, n_chg, keep_old ? c->f_old[cur].as<float>() : nullptr, ld_msg, n_ins, n_del);
    }
    if (st != INK_OK) return st;
    // rows to transform: aggregate changed; own message changed (self term); degree changed.
    // A layer with few events keeps the row count on the device: the transform and the emission
    // are launched for an upper bound and stop at the count, which saves one host round trip.
    int64_t nC = 0;
    const bool lazy = !gcn && !S.dense && !c->affected_mode && S.n_events <= kNoSyncEvents;
    const int64_t bound = lazy ? std::min<int64_t>(std::min<int64_t>(S.n_events, c->n) + nF + nD, c->n) : -1;
    // without the dense fallback and the baseline only grouped targets can have changed aggregates
    const int64_t n_t_bound = (S.dense || c->affected_mode) ? -1 : (S.n_events > 0 ? std::min<int64_t>(S.n_events, c->n) : 0);
    bool flags_cleared = false;
    st = collect_rows(c, F, nF, D, nD, &nC, bound, n_t_bound, &flags_cleared);
    if (st != INK_OK) return st;
    const int32_t *nC_dev = lazy ? &c->d_cnt->v[C_NC] : nullptr;
    if (!lazy) { S.n_transformed = nC; layer_stats_from_counters(c, l, c->h_cnt); }
    int nxt = cur ^ 1;
    int64_t nF2 = 0, n_chg2 = 0;
    bool result_done = false;
    if (nC > 0) {
      const bool last = l == c->n_layers;
      int ld_next = gcn ? (last ? c->H[l].ld : c->Msc[l + 1].ld) : c->H[l].ld;
      API_TRY(c->c_flag.reserve((size_t)nC + 64));
      API_TRY(c->c_idx.reserve((size_t)nC * 4));
      bool want_old = keep_old && !last;
      if (want_old) API_TRY(c->c_old.reserve((size_t)nC * ld_next * 4));
      {
        Prof p(c, INK_T_TRANSFORM, l, INK_K_XFORM);
        const int32_t *rows = c->c_list.as<int32_t>();
        float *old_rows = want_old ? c->c_old.as<float>() : nullptr;
        if (!gcn) {
          API_TRY(run_transform(c, l, rows, nC, c->c_flag.as<uint8_t>(), old_rows, nC_dev));
        } else {
          if (!flags_cleared) API_TRY(hipMemsetAsync(c->c_flag.p, 0, (size_t)nC, s));
          if (!last) API_TRY(gcn_next_messages(c, l, rows, nC, c->c_flag.as<uint8_t>(), old_rows));
          else API_TRY(gcn_final(c, rows, nC, c->c_flag.as<uint8_t>()));
        }
        // the baseline propagates from every node of the affected area, changed or not
        if (c->affected_mode && !last) API_TRY(hipMemsetAsync(c->c_flag.p, 1, (size_t)nC, s));
      }
      st = emit_changed(c, nC, nC_dev, nxt, want_old, ld_next, !last, &nF2, &n_chg2, last ? &c->H[l] : nullptr, &result_done);
      if (st != INK_OK) return st;
    } else if (lazy) {
      API_TRY(read_counters(c));
    }
    if (lazy) { S.n_transformed = c->h_cnt->v[C_NC]; layer_stats_from_counters(c, l, c->h_cnt); }
    S.n_changed = nF2;
    nF = nF2;
    n_chg = n_chg2;
    cur = nxt;
    if (l == c->n_layers) {
      out->n_changed = nF;
      if (nF > 0) {
        int d = c->H[l].d;
        out->changed_ids = c->f_list[cur].as<int32_t>();    // stays untouched until the next call
        if (!result_done) {
          API_TRY(c->res_emb.reserve((size_t)nF * d * 4));
          gather_rows(s, (const float *)c->H[l].f(), c->H[l].ld, d, out->changed_ids, nF, c->res_emb.as<float>());
        }
        out->embeddings = c->res_emb.as<float>();
      }
    }
  }
  return INK_OK;
}

// The end of a call: what propagate_layers left running, if anything (profiling reads events recorded after the record).
static hipError_t finish_stream(ink_ctx *c) {
  return c->drained && !c->profile ? hipSuccess : hipStreamSynchronize(c->stream);
}

// Whether layers of this context can run in one workgroup (layer_one.hip): SAGE with max or min, rows of at most 256
// floats, and a graph whose dense fallback starts above the layer's event limit.  Profiling times the separate stages.
static bool layer_one_possible(const ink_ctx *c, int64_t n_batch) {
  if (c->kind != INK_MODEL_SAGE || !c->is_select || c->affected_mode || c->profile || c->n_edges_now <= n_batch) return false;
  for (int l = 1; l <= c->n_layers; l++)
    if (c->A[l].d > kAggBlock || kOneEvents > dense_line(c, kOneEvents, c->A[l].d, c->n_edges_now - n_batch, true)) return false;
  return true;
}

// The graph stage and the layers, before the stage's record is awaited.
static hipError_t layers_one_begin(ink_ctx *c, const OneGraph &graph, uint32_t graph_seq) {
  const size_t rows = 2 * kOneEvents;
  for (DevBuf *b : {&c->f_list[0], &c->f_list[1], &c->t_list, &c->f_pref}) INK_TRY(b->reserve((rows + 2) * 4));
  INK_TRY(c->res_emb.reserve(rows * c->H[c->n_layers].d * 4));
  OneUpdate p;
  memset(&p, 0, sizeof(p));
  AggArgs a[INK_MAX_LAYERS];
  for (int l = 1; l <= c->n_layers; l++) {       // all layers before the first pointer is taken: they share the buffers
    a[l - 1] = agg_args(c, l);
    INK_TRY(agg_select_reserve(c, a[l - 1]));
  }
  for (int l = 1; l <= c->n_layers; l++) {
    const DevLayer &L = c->layers[l - 1];
    OneLayer &q = p.layer[l - 1];
    q.a = a[l - 1];
    q.a.big = a[c->n_layers - 1].big;
    q.a.big_deg = agg_select_long_degree(q.a, kOneEvents);
    q.Hp = c->H[l - 1].f(); q.ldh = c->H[l - 1].ld; q.d_in = L.in_dim;
    q.W = L.W1; q.Kp = L.K1p; q.Np = L.N1p; q.bias = L.b1; q.n_out = L.out_dim; q.relu = L.act == INK_ACT_RELU;
    q.user = c->USER[l].f(); q.ld_user = c->USER[l].ld;
    q.out = c->H[l].f(); q.ld_out = c->H[l].ld;
    c->one_seq[l] = ++c->pub_seq;
  }
  p.graph = graph; p.h_graph = reinterpret_cast<char *>(c->h_gcnt); p.graph_seq = graph_seq;
  p.g = c->d_gcnt; p.cnt = c->d_cnt;
  p.f_list[0] = c->f_list[0].as<int32_t>(); p.f_list[1] = c->f_list[1].as<int32_t>(); p.pref = c->f_pref.as<int32_t>();
  p.out_off = c->gout.off; p.out_ids = c->gout.ids; p.out_deg = c->gout.deg; p.new_out = c->new_out;
  p.touched_src = c->b_uniq.as<int32_t>();
  p.t_list = c->t_list.as<int32_t>(); p.bm = c->bm_a;
  p.res = c->res_emb.as<float>();
  static_assert(2 * kOneEvents * (4 + 4 * INK_MAX_OUT_DIM) <= INK_RESULT_HOST_BYTES, "its result fits there");
  if (c->mirror) { p.h_ids = c->mirror_ids(); p.h_emb = c->mirror_emb(); }
  p.h = reinterpret_cast<char *>(c->h_one[1]); p.seq = c->one_seq[1];
  p.n_layers = c->n_layers;
  return layers_one(c, p);
}

// Their records.  *l_next: first layer not done, with its sources in f_list[(*l_next - 1) & 1]; *events_done: its events are.
static ink_status layers_one_finish(ink_ctx *c, int64_t n_seed, int *l_next, bool *events_done, int64_t *nF, int64_t *n_chg,
                                    ink_update_result *out) {
  int l = 1;
  for (; l <= c->n_layers && n_seed > 0; l++) {
    API_TRY(wait_published(c, c->h_oseq[l], c->one_seq[l]));
    const HostCounters *h = c->h_one[l];
    if (h->v[C_ONE] != kOneDone) { *events_done = h->v[C_ONE] == kOneEventsDone; break; }
    ink_layer_stats &S = c->stats.layer[l - 1];
    S.n_sources = *nF; S.n_events = n_seed + *n_chg;
    layer_stats_from_counters(c, l, h);
    S.n_transformed = h->v[C_NC];
    S.n_changed = *nF = h->v[C_NEXT];
    *n_chg = (uint32_t)h->v[C_NEV];
  }
  *l_next = l;
  if (l > c->n_layers) {
    c->n_touched_src = 0;                                 // the last layer has cleared the marks
    out->n_changed = *nF;
    c->mirrored = c->mirror;
    if (*nF > 0) { out->changed_ids = c->f_list[c->n_layers & 1].as<int32_t>(); out->embeddings = c->res_emb.as<float>(); }
  }
  return INK_OK;
}

static ink_status apply_updates_impl(ink_ctx *c, const ink_edge_update *upd, int64_t n, ink_update_result *out);

extern "C" ink_status ink_apply_updates(ink_ctx *c, const ink_edge_update *upd, int64_t n, ink_update_result *out) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  c->affected_mode = false;
  begin_result(c);
  return end_result(c, apply_updates_impl(c, upd, n, out), out);
}

extern "C" ink_status ink_apply_updates_affected(ink_ctx *c, const ink_edge_update *upd, int64_t n,
                                                 ink_update_result *out) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  c->affected_mode = true;
  begin_result(c);
  ink_status st = apply_updates_impl(c, upd, n, out);
  c->affected_mode = false;
  return end_result(c, st, out);
}

static ink_status apply_updates_impl(ink_ctx *c, const ink_edge_update *upd, int64_t n, ink_update_result *out) {
  if (!out || n < 0 || (n > 0 && !upd)) return fail(c, INK_E_ARG, "ink_apply_updates: NULL argument or negative n");
  if (!c->inferred) return fail(c, INK_E_STATE, "ink_apply_updates: call ink_full_infer first");
  if (n >= (1ll << 30)) return fail(c, INK_E_ARG, "ink_apply_updates: batch too large");
  if (c->n_edges_now + n > kMaxEdges) return fail(c, INK_E_ARG, "ink_apply_updates: the graph would exceed the edge limit");
  auto t0 = std::chrono::steady_clock::now();
  memset(out, 0, sizeof(*out));
  hipStream_t s = c->stream;
  // Validation before anything is touched: a host-resident batch is checked here; a device-resident
  // one by the first kernel of the graph stage, which drops the whole batch on a bad entry (the
  // graph stage reports it after its first read-back, before any block is modified).
  if (!c->batch_dev) {
    for (int64_t i = 0; i < n; i++) {
      if (upd[i].op > 1) return fail(c, INK_E_ARG, "ink_apply_updates: op must be 0 (insert) or 1 (delete)");
      if (upd[i].src < 0 || upd[i].src >= c->n || upd[i].dst < 0 || upd[i].dst >= c->n)
        return fail(c, INK_E_RANGE, "ink_apply_updates: node id out of range");
    }
  }
  memset(&c->stats, 0, sizeof(c->stats));
  c->stats.n_layers = c->n_layers;
  int64_t n_ins = 0, n_del = 0;
  bool one = false;            // graph stage and first layers may have run in one launch (layers_one_begin)
  if (n > 0) {
    Prof p(c, INK_T_GRAPH);
    // a device batch is read where it is; a short host batch from pinned memory, by the one kernel that reads it
    const void *raw = upd;
    if (!c->batch_dev) {
      if (n <= kPinnedBatch) { memcpy(c->h_batch, upd, (size_t)n * sizeof(ink_edge_update)); raw = c->h_batch; }
      else {
        API_TRY(c->b_raw.reserve((size_t)n * sizeof(ink_edge_update)));
        API_TRY(hipMemcpyAsync(c->b_raw.p, upd, (size_t)n * sizeof(ink_edge_update), hipMemcpyHostToDevice, s));
        raw = c->b_raw.p;
      }
    }
    one = n <= kOneEvents && n <= c->small_batch && layer_one_possible(c, n);
    ink_status st = graph_apply_batch(c, raw, n, &n_ins, &n_del, one ? layers_one_begin : nullptr);
    if (st != INK_OK) return drain(c, st);       // behind the record that tells of a bad entry stand launches that do nothing for it
  }
  out->n_applied_ins = n_ins; out->n_applied_del = n_del; out->n_noop = n - n_ins - n_del;
  c->n_edges_now += n_ins - n_del;
  const int64_t n_seed = n_ins + n_del;
  const bool gcn = c->kind == INK_MODEL_GCN;
  // nodes whose in-degree may have changed: their normalisation (GCN, mean) changes row-locally
  const int32_t *D = (const int32_t *)c->b_touch_in.p;
  const int64_t nD = (n_seed > 0 && (gcn || c->agg == INK_AGG_MEAN)) ? c->n_touched_in : 0;

  int64_t nF = 0;            // |F_l|: sources whose message m_l changed
  int64_t n_chg = 0;         // events F_l propagates along its kept out-edges
  int cur = 0;               // f_list[cur] / f_old[cur] describe F_l
  if (gcn && nD > 0) {
    // layer-1 messages are c_u * (x_u W_1): a degree change rescales the row
    Prof p(c, INK_T_TRANSFORM);
    int ld = c->Msc[1].ld;
    API_TRY(c->c_flag.reserve((size_t)nD + 64));
    API_TRY(c->c_idx.reserve((size_t)nD * 4));
    API_TRY(c->c_old.reserve((size_t)nD * ld * 4));
    API_TRY(c->c_list.reserve((size_t)c->n * 4));
    API_TRY(hipMemsetAsync(c->c_flag.p, 0, (size_t)nD, s));
    API_TRY(hipMemcpyAsync(c->c_list.p, D, (size_t)nD * 4, hipMemcpyDeviceToDevice, s));
    hipLaunchKernelGGL(k_gcn_rescale, grid1(nD * ld), dim3(256), 0, s, D, nD, (const int32_t *)c->gin.deg, c->cnorm,
                       (const float *)c->XW[1].f(), c->Msc[1].f(), ld, c->Msc[1].d, c->c_old.as<float>(),
                       c->c_flag.as<uint8_t>());
    API_TRY(hipGetLastError());
    ink_status st = emit_changed(c, nD, nullptr, cur, true, ld, true, &nF, &n_chg);
    if (st != INK_OK) return st;
  }
  int first = 1;
  bool events_done = false;
  if (one) {
    ink_status st = layers_one_finish(c, n_seed, &first, &events_done, &nF, &n_chg, out);
    if (st != INK_OK) return st;
    cur = (first - 1) & 1;
  }
  if (first <= c->n_layers) {
    ink_status st = propagate_layers(c, nF, n_chg, cur, n_ins, n_del, D, nD, out, nullptr, first, events_done);
    if (st != INK_OK) return st;
  }
  API_TRY(graph_end_batch(c));
  if (first <= c->n_layers) API_TRY(finish_stream(c));     // otherwise the last record covers everything
  prof_collect(c);
  c->stats.ms_total = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
  return INK_OK;
}

// ------------------------------------------------------------------------------------ feature updates
static ink_status update_features_impl(ink_ctx *c, const int32_t *node_ids, const float *rows, int64_t n,
                                       ink_update_result *out);
extern "C" ink_status ink_update_features(ink_ctx *c, const int32_t *node_ids, const float *rows, int64_t n,
                                          ink_update_result *out) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  begin_result(c);
  return end_result(c, update_features_impl(c, node_ids, rows, n, out), out);
}

static ink_status update_features_impl(ink_ctx *c, const int32_t *node_ids, const float *rows, int64_t n,
                                       ink_update_result *out) {
  if (!out || n < 0 || (n > 0 && (!node_ids || !rows))) return fail(c, INK_E_ARG, "ink_update_features: NULL argument or negative n");
  if (!c->inferred) return fail(c, INK_E_STATE, "ink_update_features: call ink_full_infer first");
  if (n > c->n) return fail(c, INK_E_ARG, "ink_update_features: more rows than nodes (ids must be distinct)");
  auto t0 = std::chrono::steady_clock::now();
  memset(out, 0, sizeof(*out));
  hipStream_t s = c->stream;
  c->affected_mode = false;
  const int d0 = c->H[0].d, ld0 = c->H[0].ld;
  // validation before anything is touched: host-resident ids are range-checked here, device-resident
  // ones by a kernel; distinctness is checked on the sorted device copy (one read-back for both)
  if (!c->batch_dev)
    for (int64_t i = 0; i < n; i++)
      if (node_ids[i] < 0 || node_ids[i] >= c->n) return fail(c, INK_E_RANGE, "ink_update_features: node id out of range");
  memset(&c->stats, 0, sizeof(c->stats));
  c->stats.n_layers = c->n_layers;
  if (n == 0) return INK_OK;
  const bool gcn = c->kind == INK_MODEL_GCN;
  const bool keep_old = !c->is_select;
  Counters *dc = c->d_cnt;
  int64_t nF = 0, n_chg = 0;
  int cur = 0;
  bool later = false;          // the ids' verdict comes with the emission's record
  auto bad_ids = [&]() {
    if (c->h_cnt->v[C_TMP1]) return drain(c, fail(c, INK_E_RANGE, "ink_update_features: node id out of range"));
    if (c->h_cnt->v[C_TMP0]) return drain(c, fail(c, INK_E_ARG, "ink_update_features: a node id appears more than once"));
    return INK_OK;
  };
  {
    Prof p(c, INK_T_GRAPH);
    const hipMemcpyKind kind = c->batch_dev ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    size_t per = ((size_t)n * 4 + 255) & ~(size_t)255;
    API_TRY(c->b_misc.reserve(per * 2));
    uint32_t *ids = c->b_misc.as<uint32_t>(), *perm = (uint32_t *)((char *)c->b_misc.p + per);
    const float *drows = rows;
    if (!c->batch_dev) {
      API_TRY(c->stage1.reserve((size_t)n * d0 * 4));
      API_TRY(hipMemcpyAsync(c->stage1.p, rows, (size_t)n * d0 * 4, hipMemcpyHostToDevice, s));
      drows = c->stage1.as<float>();
    }
    // Few ids: order and checks in one launch, and, but for GCN, which has a product to do first, no round trip before the
    // rows: the record that the emission ends with tells of a bad batch, for which nothing was changed.  1000 rows of
    // 100 floats: eleven launches and two round trips until then, now three and one, 25 us of an update of 810.
    const bool few = n <= kSmallLayer;
    API_TRY(c->c_flag.reserve((size_t)n + 64));
    if (few) {
      const int32_t *in = node_ids;
      if (!c->batch_dev) {
        if (n * 4 <= kPinnedBatch * (int64_t)sizeof(ink_edge_update)) { memcpy(c->h_batch, node_ids, (size_t)n * 4); in = reinterpret_cast<const int32_t *>(c->h_batch); }
        else { API_TRY(hipMemcpyAsync(perm, node_ids, (size_t)n * 4, kind, s)); in = (const int32_t *)perm; }
      }
      const int passes = (c->id_bits + kRadixBits - 1) / kRadixBits;
#define INK_FEATURE_IDS(T, I) hipLaunchKernelGGL((k_feature_ids<T, I>), dim3(1), dim3(T), 0, s, in, (int)n, (uint32_t)c->n, passes, ids, perm, c->c_flag.as<uint8_t>(), dc)
      if (n <= 256) INK_FEATURE_IDS(256, 1);
      else if (n <= 1024) INK_FEATURE_IDS(256, 4);
      else INK_FEATURE_IDS(1024, 4);
#undef INK_FEATURE_IDS
    } else {
      API_TRY(hipMemcpyAsync(ids, node_ids, (size_t)n * 4, kind, s));
      hipLaunchKernelGGL(k_iota_u32, grid1(n), dim3(256), 0, s, perm, n);
      API_TRY(radix_sort_pairs(c->ws, ids, perm, n, c->id_bits, s));
      API_TRY(hipMemsetAsync(dc, 0, sizeof(Counters), s));
      API_TRY(hipMemsetAsync(c->c_flag.p, 0, (size_t)n, s));
      hipLaunchKernelGGL(k_any_adjacent_equal, grid1(n), dim3(256), 0, s, (const uint32_t *)ids, n, &dc->v[C_TMP0]);
      if (c->batch_dev)
        hipLaunchKernelGGL(k_any_out_of_range, grid1(n), dim3(256), 0, s, (const uint32_t *)ids, n, (uint32_t)c->n, &dc->v[C_TMP1]);
    }
    API_TRY(hipGetLastError());
    later = few && !gcn;
    if (!later) {
      API_TRY(read_counters(c));
      const ink_status st = bad_ids();
      if (st != INK_OK) return st;
    }
    API_TRY(c->c_idx.reserve((size_t)n * 4));
    API_TRY(c->c_list.reserve((size_t)c->n * 4));
    float *old0 = nullptr, *dense = nullptr;
    if (keep_old && !gcn) { API_TRY(c->c_old.reserve((size_t)n * ld0 * 4)); old0 = c->c_old.as<float>(); }
    if (gcn) { API_TRY(c->stage0.reserve((size_t)n * ld0 * 4)); dense = c->stage0.as<float>(); }
    hipLaunchKernelGGL(k_set_features, grid1(n * ld0), dim3(256), 0, s, (const uint32_t *)ids, (const uint32_t *)perm, n,
                       drows, d0, c->H[0].f(), ld0, old0, dense, c->c_flag.as<uint8_t>(), c->c_list.as<int32_t>(), (const Counters *)dc);
    API_TRY(hipGetLastError());
  }
  int ld_msg = ld0;
  if (gcn) {
    // layer-1 messages are c_u (x_u W_1): redo the product for the listed rows, then rescale
    Prof p(c, INK_T_TRANSFORM);
    const DevLayer &L = c->layers[0];
    ld_msg = c->Msc[1].ld;
    XformArgs x;
    memset(&x, 0, sizeof(x));
    x.mode = 2; x.n_rows = n; x.Hp = c->stage0.as<float>(); x.ldh = ld0; x.d_in = L.in_dim;
    x.W = L.W1; x.Kp = L.K1p; x.Np = L.N1p; x.n_out = L.out_dim;
    x.out = c->XW[1].f(); x.ld_out = c->XW[1].ld; x.to_table = 1; x.out_rows = c->c_list.as<int32_t>();
    API_TRY(xform_run(c, x));
    API_TRY(c->c_old.reserve((size_t)n * ld_msg * 4));
    API_TRY(hipMemsetAsync(c->c_flag.p, 0, (size_t)n, s));
    hipLaunchKernelGGL(k_gcn_rescale, grid1(n * ld_msg), dim3(256), 0, s, (const int32_t *)c->c_list.as<int32_t>(), n,
                       (const int32_t *)c->gin.deg, c->cnorm, (const float *)c->XW[1].f(), c->Msc[1].f(), ld_msg,
                       c->Msc[1].d, c->c_old.as<float>(), c->c_flag.as<uint8_t>());
    API_TRY(hipGetLastError());
  }
  ink_status st = emit_changed(c, n, nullptr, cur, keep_old, ld_msg, true, &nF, &n_chg);
  if (st == INK_OK && later) st = bad_ids();
  if (st != INK_OK) return st;
  st = propagate_layers(c, nF, n_chg, cur, 0, 0, nullptr, 0, out);
  if (st != INK_OK) return st;
  API_TRY(finish_stream(c));
  prof_collect(c);
  c->stats.ms_total = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
  return INK_OK;
}

// ------------------------------------------------------------------------------------ user-defined events
// key of event i for the pass over layer l: its target, or n_nodes (sorts behind every node) if it
// belongs to another layer; value = its position in the list
__global__ void k_user_keys(const ink_user_event *ev, int64_t n, int layer, uint32_t n_nodes, uint32_t *key, uint32_t *val) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  key[i] = ev[i].layer == layer ? (uint32_t)ev[i].target : n_nodes;
  val[i] = (uint32_t)i;
}

// One wave per target: its events (positions pos[seg[j] .. seg[j + 1]) of the list, in list order)
// are applied to the node's term; flag[j] = 1 if the term changed bitwise.
__global__ __launch_bounds__(256) void k_user_apply(const int32_t *uniq, const int32_t *seg, const int32_t *n_uniq,
                                                    const uint32_t *pos, const ink_user_event *ev, const float *rows,
                                                    int stride, float *U, int ld, int d, uint8_t *flag) {
  const int l = lane_id();
  int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  if (j >= *n_uniq) return;
  const int64_t v = uniq[j];
  const int e0 = seg[j], e1 = seg[j + 1];
  bool chg = false;
  for (int k = l; k < d; k += kWave) {
    const float old = U[v * ld + k];
    float u = old;
    for (int e = e0; e < e1; e++) {
      const uint32_t i = pos[e];
      const int op = ev[i].op;
      const float r = rows[(int64_t)i * stride + k];
      u = op == INK_USER_SET ? r : (op == INK_USER_ADD ? __fadd_rn(u, r) : 0.f);
    }
    if (__float_as_uint(u) != __float_as_uint(old)) { U[v * ld + k] = u; chg = true; }
  }
  const bool any = __ballot(chg) != 0ull;
  if (l == 0) flag[j] = any ? 1 : 0;
}

struct UserState {
  int64_t n;                       // events in the list
  int row_stride;                  // floats between the rows of two events
  int64_t per_layer[INK_MAX_LAYERS + 1];   // events that name each layer
};

// the nodes whose term of layer l changed -> ascending list (the rows this layer re-transforms for its own reasons)
static ink_status user_rows_of(ink_ctx *c, int l, void *state, const int32_t **rows, int64_t *n_rows) {
  const UserState *u = (const UserState *)state;
  *rows = nullptr; *n_rows = 0;
  const int64_t m = u->per_layer[l];
  if (m == 0) return INK_OK;
  hipStream_t s = c->stream;
  Prof p(c, INK_T_EVENTS);
  uint32_t *key = c->u_key.as<uint32_t>(), *val = c->u_val.as<uint32_t>();
  hipLaunchKernelGGL(k_user_keys, grid1(u->n), dim3(256), 0, s, (const ink_user_event *)c->u_ev.p, u->n, l, (uint32_t)c->n, key, val);
  API_TRY(hipGetLastError());
  // stable: the layer's events come first, grouped by target, each group in list order
  API_TRY(radix_sort_pairs(c->ws, key, val, u->n, c->id_bits + 1, s));
  int32_t *n_uniq = &c->d_cnt->v[C_TMP0], *n_chg = &c->d_cnt->v[C_TMP1];
  API_TRY(segment_heads(c->ws, key, m, c->u_uniq.as<int32_t>(), c->u_seg.as<int32_t>(), n_uniq, s));
  hipLaunchKernelGGL(k_user_apply, grid1(m * kWave), dim3(256), 0, s, (const int32_t *)c->u_uniq.as<int32_t>(),
                     (const int32_t *)c->u_seg.as<int32_t>(), (const int32_t *)n_uniq, (const uint32_t *)val,
                     (const ink_user_event *)c->u_ev.p, (const float *)c->u_rows.p, u->row_stride,
                     c->USER[l].f(), c->USER[l].ld, c->USER[l].d, c->u_flag.as<uint8_t>());
  API_TRY(hipGetLastError());
  API_TRY(read_counters(c));
  const int64_t nu = c->h_cnt->v[C_TMP0];
  API_TRY(compact_flags_u8(c->ws, c->u_flag.as<uint8_t>(), nu, c->u_idx.as<int32_t>(), n_chg, s));
  hipLaunchKernelGGL(k_gather_i32, grid1(nu), dim3(256), 0, s, (const int32_t *)c->u_uniq.as<int32_t>(),
                     (const int32_t *)c->u_idx.as<int32_t>(), 0, (const int32_t *)n_chg, c->u_list.as<int32_t>());
  API_TRY(hipGetLastError());
  API_TRY(read_counters(c));
  *rows = c->u_list.as<int32_t>();
  *n_rows = c->h_cnt->v[C_TMP1];
  return INK_OK;
}

static ink_status apply_user_events_impl(ink_ctx *c, const ink_user_event *events, const float *rows, int32_t row_stride,
                                         int64_t n, ink_update_result *out) {
  if (!out || n < 0 || (n > 0 && (!events || !rows))) return fail(c, INK_E_ARG, "ink_apply_user_events: NULL argument or negative n");
  if (!c->inferred) return fail(c, INK_E_STATE, "ink_apply_user_events: call ink_full_infer first");
  if (n >= (1ll << 30)) return fail(c, INK_E_ARG, "ink_apply_user_events: too many events");
  UserState u;
  memset(&u, 0, sizeof(u));
  u.n = n;
  u.row_stride = row_stride;
  int last = 0;
  for (int64_t i = 0; i < n; i++) {
    const ink_user_event &e = events[i];
    if (e.layer < 1 || e.layer > c->n_layers) return fail(c, INK_E_RANGE, "ink_apply_user_events: layer out of range");
    if (e.target < 0 || e.target >= c->n) return fail(c, INK_E_RANGE, "ink_apply_user_events: node id out of range");
    if (e.op < INK_USER_SET || e.op > INK_USER_CLEAR) return fail(c, INK_E_ARG, "ink_apply_user_events: unknown op");
    if (row_stride < c->H[e.layer].d) return fail(c, INK_E_ARG, "ink_apply_user_events: row_stride below the layer's width");
    u.per_layer[e.layer]++;
    last = std::max(last, (int)e.layer);
  }
  auto t0 = std::chrono::steady_clock::now();
  memset(out, 0, sizeof(*out));
  memset(&c->stats, 0, sizeof(c->stats));
  c->stats.n_layers = c->n_layers;
  if (n == 0) return INK_OK;
  c->affected_mode = false;
  hipStream_t s = c->stream;
  // everything that can fail for lack of memory comes before the first term is touched
  for (int l = 1; l <= last; l++)
    if (u.per_layer[l] > 0 && !c->USER[l].p) API_TRY(alloc_table(c->USER[l], c->n_cap, c->H[l].d));
  API_TRY(c->u_ev.reserve((size_t)n * sizeof(ink_user_event)));
  API_TRY(c->u_rows.reserve((size_t)n * row_stride * 4));
  for (DevBuf *b : {&c->u_key, &c->u_val, &c->u_uniq, &c->u_seg, &c->u_idx, &c->u_list}) API_TRY(b->reserve((size_t)(n + 2) * 4));
  API_TRY(c->u_flag.reserve((size_t)n + 64));
  API_TRY(c->c_list.reserve((size_t)c->n * 4));
  API_TRY(hipMemcpyAsync(c->u_ev.p, events, (size_t)n * sizeof(ink_user_event), hipMemcpyHostToDevice, s));
  API_TRY(hipMemcpyAsync(c->u_rows.p, rows, (size_t)n * row_stride * 4, hipMemcpyHostToDevice, s));
  LayerRows own{last, user_rows_of, &u};
  ink_status st = propagate_layers(c, 0, 0, 0, 0, 0, nullptr, 0, out, &own);
  if (st != INK_OK) return st;
  API_TRY(finish_stream(c));
  prof_collect(c);
  c->stats.ms_total = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
  return INK_OK;
}

extern "C" ink_status ink_apply_user_events(ink_ctx *c, const ink_user_event *events, const float *rows,
                                            int32_t row_stride, int64_t n, ink_update_result *out) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  begin_result(c);
  return end_result(c, apply_user_events_impl(c, events, rows, row_stride, n, out), out);
}

// ------------------------------------------------------------------------------------ node arrival
__global__ void k_iota_i32(int32_t *out, int64_t n, int32_t first) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = first + (int32_t)i;
}

__global__ void k_unpack_rows_at(const float *in, int d, int ld, int64_t row0, int64_t n, float *table) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t i = t / ld;
  int k = (int)(t % ld);
  if (i >= n) return;
  table[(row0 + i) * ld + k] = k < d ? in[i * d + k] : 0.f;
}

static ink_status add_nodes_impl(ink_ctx *c, const float *features, int64_t n_new, ink_update_result *out);
extern "C" ink_status ink_add_nodes(ink_ctx *c, const float *features, int64_t n_new, ink_update_result *out) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  begin_result(c);
  return end_result(c, add_nodes_impl(c, features, n_new, out), out);
}

static ink_status add_nodes_impl(ink_ctx *c, const float *features, int64_t n_new, ink_update_result *out) {
  if (!out || n_new < 0 || (n_new > 0 && !features)) return fail(c, INK_E_ARG, "ink_add_nodes: NULL argument or negative n_new");
  if (!c->inferred) return fail(c, INK_E_STATE, "ink_add_nodes: call ink_full_infer first");
  if ((int64_t)c->n + n_new > c->n_cap) return fail(c, INK_E_RANGE, "ink_add_nodes: beyond ink_options.node_capacity");
  auto t0 = std::chrono::steady_clock::now();
  memset(out, 0, sizeof(*out));
  memset(&c->stats, 0, sizeof(c->stats));
  c->stats.n_layers = c->n_layers;
  if (n_new == 0) return INK_OK;
  hipStream_t s = c->stream;
  c->affected_mode = false;
  const int n0 = c->n;
  const int d0 = c->H[0].d, ld0 = c->H[0].ld;
  const bool gcn = c->kind == INK_MODEL_GCN;
  {
    Prof p(c, INK_T_GRAPH);
    ink_status st = graph_add_nodes(c, n_new);
    if (st != INK_OK) return st;
    const float *drows = features;
    if (!c->batch_dev) {
      API_TRY(c->stage1.reserve((size_t)n_new * d0 * 4));
      API_TRY(hipMemcpyAsync(c->stage1.p, features, (size_t)n_new * d0 * 4, hipMemcpyHostToDevice, s));
      drows = c->stage1.as<float>();
    }
    hipLaunchKernelGGL(k_unpack_rows_at, grid1(n_new * ld0), dim3(256), 0, s, drows, d0, ld0, (int64_t)n0, n_new, c->H[0].f());
    API_TRY(c->res_ids.reserve((size_t)n_new * 4));
    hipLaunchKernelGGL(k_iota_i32, grid1(n_new), dim3(256), 0, s, c->res_ids.as<int32_t>(), n_new, (int32_t)n0);
    API_TRY(hipGetLastError());
  }
  c->n = n0 + (int)n_new;          // from here on the new ids are valid rows
  const int32_t *rows = c->res_ids.as<int32_t>();
  if (gcn) {
    // layer-1 message of a node without in-edges: d-hat = 1, so c_v = 1 and m_1 = x W_1
    Prof p(c, INK_T_TRANSFORM);
    const DevLayer &L = c->layers[0];
    XformArgs x;
    memset(&x, 0, sizeof(x));
    x.mode = 2; x.n_rows = n_new; x.Hp = c->H[0].f() + (int64_t)n0 * ld0; x.ldh = ld0; x.d_in = L.in_dim;
    x.W = L.W1; x.Kp = L.K1p; x.Np = L.N1p; x.n_out = L.out_dim;
    x.out = c->XW[1].f(); x.ld_out = c->XW[1].ld; x.to_table = 1; x.out_rows = rows;
    API_TRY(xform_run(c, x));
    hipLaunchKernelGGL(k_gcn_rescale, grid1(n_new * c->Msc[1].ld), dim3(256), 0, s, rows, n_new, (const int32_t *)c->gin.deg,
                       c->cnorm, (const float *)c->XW[1].f(), c->Msc[1].f(), c->Msc[1].ld, c->Msc[1].d, (float *)nullptr,
                       (uint8_t *)nullptr);
    API_TRY(hipGetLastError());
  }
  for (int l = 1; l <= c->n_layers; l++) {
    API_TRY(hipMemsetAsync(c->d_cnt, 0, sizeof(Counters), s));
    AggArgs a = agg_args(c, l);
    { Prof p(c, INK_T_AGG); API_TRY(agg_full_any(c, a, nullptr, rows, n_new)); }
    {
      Prof p(c, INK_T_TRANSFORM);
      if (!gcn) API_TRY(run_transform(c, l, rows, n_new, nullptr));
      else if (l < c->n_layers) API_TRY(gcn_next_messages(c, l, rows, n_new, nullptr, nullptr));
      else API_TRY(gcn_final(c, rows, n_new, nullptr));
    }
    ink_layer_stats &S = c->stats.layer[l - 1];
    S.n_targets = n_new; S.n_exposed = n_new; S.n_transformed = n_new; S.n_changed = n_new;
  }
  {
    int k = c->n_layers, d = c->H[k].d;
    API_TRY(c->res_emb.reserve((size_t)n_new * d * 4));
    gather_rows(s, (const float *)c->H[k].f(), c->H[k].ld, d, rows, n_new, c->res_emb.as<float>());
    API_TRY(hipGetLastError());
    out->n_changed = n_new;
    out->changed_ids = c->res_ids.as<int32_t>();
    out->embeddings = c->res_emb.as<float>();
  }
  API_TRY(hipStreamSynchronize(s));
  prof_collect(c);
  c->stats.ms_total = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
  return INK_OK;
}

// ------------------------------------------------------------------------------------ inspection
extern "C" ink_status ink_get_layer(ink_ctx *c, int32_t layer, int32_t which, int64_t row0, int64_t nrows, void *dst,
                                    int32_t dst_mem, int32_t *width_out) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  if (!c->inferred) return fail(c, INK_E_STATE, "ink_get_layer: call ink_full_infer first");
  if (layer < 0 || layer > c->n_layers || which < 0 || which > 5 || (which > 0 && layer == 0))
    return fail(c, INK_E_RANGE, "ink_get_layer: layer / which out of range");
  if (row0 < 0 || nrows < 0 || row0 + nrows > c->n) return fail(c, INK_E_RANGE, "ink_get_layer: rows out of range");
  if (which >= 2 && which <= 4 && !c->is_select) return fail(c, INK_E_ARG, "ink_get_layer: no argument table for sum-type aggregators");
  const Table &t = which == 0 ? c->H[layer] : (which == 1 ? c->A[layer] : (which == 2 ? c->ARG[layer] : (which == 3 ? c->UB[layer] : (which == 4 ? c->ARG2[layer] : c->USER[layer]))));
  if (!t.p) return fail(c, INK_E_ARG, "ink_get_layer: table not kept for this model");
  if (width_out) *width_out = t.d;
  if (nrows == 0) return INK_OK;
  if (!dst) return fail(c, INK_E_ARG, "ink_get_layer: dst is NULL");
  size_t bytes = (size_t)nrows * t.d * 4;
  void *dev_dst = dst;
  if (dst_mem != INK_MEM_DEVICE) { API_TRY(c->stage1.reserve(bytes)); dev_dst = c->stage1.p; }
  if (t.d % 4 == 0 && ((uintptr_t)dev_dst & 15) == 0) {
    // 16 bytes per lane and the division by the width in 32 bits: 625k rows of 128 floats 193 -> 102 us (6.2 TB/s)
    const int per = std::max(1, 2048 / (t.d / 4));
    hipLaunchKernelGGL(k_pack_rows4, grid1(nrows, per), dim3(256), 0, c->stream, (const float4 *)t.p, t.ld / 4, t.d / 4, row0,
                       nrows, per, (float4 *)dev_dst);
  } else
    hipLaunchKernelGGL(k_pack_rows, grid1(nrows * t.d), dim3(256), 0, c->stream, (const void *)t.p, t.ld, t.d, row0, nrows,
                       dev_dst);
  API_TRY(hipGetLastError());
  if (dst_mem != INK_MEM_DEVICE) API_TRY(hipMemcpyAsync(dst, dev_dst, bytes, hipMemcpyDeviceToHost, c->stream));
  API_TRY(hipStreamSynchronize(c->stream));
  return INK_OK;
}

extern "C" ink_status ink_copy_result(ink_ctx *c, int32_t *ids, float *embeddings, int64_t n) {
  if (!c) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  if (c->last.n < 0) return fail(c, INK_E_STATE, "ink_copy_result: the last call left no result");
  if (n != c->last.n || (n > 0 && (!ids || !embeddings))) return fail(c, INK_E_ARG, "ink_copy_result: NULL argument or not the result's size");
  c->fetched = true;
  want_host_results(c);
  if (n == 0) return INK_OK;
  const size_t row = (size_t)c->H[c->n_layers].d * 4;
  if (c->mirrored && n <= c->mirror_rows()) {
    memcpy(ids, c->mirror_ids(), (size_t)n * 4);
    memcpy(embeddings, c->mirror_emb(), (size_t)n * row);
    return INK_OK;
  }
  API_TRY(hipMemcpyAsync(ids, c->last.ids, (size_t)n * 4, hipMemcpyDeviceToHost, c->stream));
  API_TRY(hipMemcpyAsync(embeddings, c->last.rows, (size_t)n * row, hipMemcpyDeviceToHost, c->stream));
  API_TRY(hipStreamSynchronize(c->stream));
  return INK_OK;
}

extern "C" ink_status ink_get_graph(ink_ctx *c, int64_t *rowptr, int32_t *col) {
  if (!c || !rowptr) return INK_E_ARG;
  if (c->broken) return fail(c, INK_E_STATE, kBrokenMsg);
  API_TRY(hipStreamSynchronize(c->stream));
  API_TRY(graph_export(c, rowptr, col));
  return INK_OK;
}

extern "C" ink_status ink_set_profiling(ink_ctx *c, int32_t on) {
  if (!c) return INK_E_ARG;
  c->profile = on != 0;
  return INK_OK;
}

extern "C" ink_status ink_get_stats(ink_ctx *c, void *dst, size_t bytes) {
  if (!c || !dst) return INK_E_ARG;
  memcpy(dst, &c->stats, std::min(bytes, sizeof(ink_stats)));
  return INK_OK;
}
