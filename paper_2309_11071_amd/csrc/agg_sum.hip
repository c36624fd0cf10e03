// Aggregation kernels for the accumulative aggregators (sum, mean, degree-normalised sum):
// the cached state is the plain sum S_v of the (possibly pre-scaled) message rows of the
// in-neighbours, updated by adding deltas (the extension sketched in Sec. 7): for a removed edge
// the old message is subtracted, for an inserted edge the new one is added, and for a kept edge
// whose source changed the difference new - old is added.  The three edge sets are disjoint, so
// no message is counted twice.  Events of a target are consumed in their stored order and lane
// groups are combined in a fixed pattern: results are reproducible run to run.
#include <algorithm>

#include "longev.h"
#include "rowload.h"

namespace ink {

struct S4 { float v[4]; };

__device__ __forceinline__ float4 ldf4(const float *p) { return *reinterpret_cast<const float4 *>(p); }

// Lanes per row: 16 / 32 / 64 (64 / LPR groups fill the wave) or 12 (five groups, lanes 60-63 idle:
// rows of at most 48 floats, five of them per load instead of four).
template <int LPR> __device__ __forceinline__ void sum_groups(S4 &a) {
  if constexpr ((LPR & (LPR - 1)) == 0) {
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1)
#pragma unroll
      for (int c = 0; c < 4; c++) a.v[c] = __fadd_rn(a.v[c], __shfl_xor(a.v[c], off, kWave));
  } else {       // group 0 + group 1 + ... in that order; valid in the lanes of group 0
    constexpr int G = kWave / LPR;
    const int q = lane_id() % LPR;
    S4 r = a;
#pragma unroll
    for (int g = 1; g < G; g++)
#pragma unroll
      for (int c = 0; c < 4; c++) r.v[c] = __fadd_rn(r.v[c], __shfl(a.v[c], q + g * LPR, kWave));
    a = r;
  }
}
template <int LPR> __device__ __forceinline__ bool lane_in_groups() { return lane_id() < (kWave / LPR) * LPR; }

// U rows per lane group added in order; FULL: every slot is a row, otherwise empty ones add +0 (a sum that starts at
// +0 is never -0, so that is the identity)
template <int LPR, int U, bool FULL>
__device__ __forceinline__ void add_batch(const RowTable<LPR> &tab, int win, int it, int cnt, S4 &acc) {
  constexpr int G = kWave / LPR;
  int id[U];
  float4 row[U];
  tab.template load_batch<U>(win, it, FULL ? kWave - 1 : cnt - 1, id, row);
#pragma unroll
  for (int u = 0; u < U; u++) {
    const float x[4] = {row[u].x, row[u].y, row[u].z, row[u].w};
    const bool on = FULL || it + u * G + tab.g < cnt;
#pragma unroll
    for (int c = 0; c < 4; c++) acc.v[c] = __fadd_rn(acc.v[c], on ? x[c] : 0.f);
  }
}

// sum of rows M[ids[j]] for j in [j0, j1): group g takes j0 + g, j0 + g + G, ... in order
template <int LPR>
__device__ __forceinline__ void sum_range(const int32_t *ids, int64_t j0, int64_t j1, const float *M, int ldm,
                                          bool lane_on, int q, S4 &acc) {
  constexpr int G = kWave / LPR, W = G * LPR == kWave ? kWave : G * (kWave / G);    // ids per window, a multiple of G
  constexpr int U = INK_U_SUM;
  const int l = lane_id();
  const RowTable<LPR> tab(M, ldm, lane_on, q);
#pragma unroll
  for (int c = 0; c < 4; c++) acc.v[c] = 0.f;
  const int32_t *p = ids + j0;
  const int n = __builtin_amdgcn_readfirstlane((int)(j1 - j0));
  int win = n > 0 ? p[l < n ? l : n - 1] : 0;
  for (int jb = 0; jb < n; jb += W) {
    const int cnt = n - jb < W ? n - jb : W, ahead = jb + W + l;
    const int next = jb + W < n ? p[ahead < n ? ahead : n - 1] : 0;
    for (int it = 0; it < cnt;) {
      const int left = cnt - it;
      if (left >= G * U) { add_batch<LPR, U, true>(tab, win, it, cnt, acc); it += G * U; }
      else if (left > G * U / 4) { add_batch<LPR, U / 2, false>(tab, win, it, cnt, acc); it += G * U / 2; }
      else { add_batch<LPR, U / 4, false>(tab, win, it, cnt, acc); it += G * U / 4; }
    }
    win = next;
  }
  sum_groups<LPR>(acc);
}

__device__ __forceinline__ void mark_bit_s(uint64_t *bm, int v) {
  atomicOr((unsigned long long *)&bm[v >> 6], 1ull << (v & 63));
}

// stores the row; returns wave-uniform "some value of the first d dimensions changed"
template <int LPR>
__device__ __forceinline__ bool store_sum(float *A, int ld, int d, int v, bool lane_on, int q, const S4 &nv,
                                          bool compare) {
  const int l = lane_id();
  bool writer = lane_on && l < LPR;
  bool chg = false;
  if (writer) {
    float *p = A + (int64_t)v * ld + 4 * q;
    if (compare) {
      float4 o = ldf4(p);
      float ov[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int c = 0; c < 4; c++)
        if (4 * q + c < d) chg |= __float_as_uint(ov[c]) != __float_as_uint(nv.v[c]);
    }
    if (!compare || chg) *reinterpret_cast<float4 *>(p) = make_float4(nv.v[0], nv.v[1], nv.v[2], nv.v[3]);
  }
  return __ballot(chg) != 0ull;
}

template <int LPR>
__global__ __launch_bounds__(256) void k_sum_full(AggArgs a, const int32_t *targets, int64_t n_targets, uint64_t *chg,
                                                  int compare, Counters *cnt) {
  const int l = lane_id();
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd && lane_in_groups<LPR>();
  // wave-uniform, so that the row's place and length are scalar loads that are under way together
  const int64_t wid = (int64_t)blockIdx.x * (blockDim.x / kWave) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  if (wid >= n_targets) return;
  const int v = targets ? targets[wid] : (int)wid;
  const int deg = a.in_deg[v];
  const int64_t off = a.in_off[v];
  if (targets && l == 0) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_REGATHER], (unsigned long long)deg);
  if (deg > a.big_deg && l == 0)      // few rows: also tallied when every row is recomputed
    atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_REGATHER_LONG], (unsigned long long)deg);
  if (deg > a.big_deg) {
    if (l == 0) list_big_row(a.big, cnt, v, deg);
    return;
  }
  S4 acc;
  sum_range<LPR>(a.in_ids + off, 0, deg, a.M, a.ldm, lane_on, q, acc);
  bool ch = store_sum<LPR>(a.A, a.ld, a.d, v, lane_on, q, acc, compare != 0);
  if (ch && chg && l == 0) mark_bit_s(chg, v);
}

// Chunks of long rows of at most 48 floats, of a table too large for slices to pay (kSlicedTableBytes), or of a short launch with many
// (kSlicedItems), as they are: the NW waves of a workgroup take a part of a chunk each; the wave that has stored a part calls
// stored(place of its row in the list, node)
template <int LPR, int NW, bool COHERENT, class Stored>
__device__ __forceinline__ void whole_sum_chunks(const AggArgs &a, int total, int n_big, float (*sv)[kWave * 4], float *part, const Stored &stored) {
  const int l = lane_id(), w = threadIdx.x / kWave;
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd && lane_in_groups<LPR>();
  for (int cg = blockIdx.x; cg < total; cg += gridDim.x) {
    int i, v;
    int64_t j0, j1;
    big_chunk(a.big, n_big, cg, a.in_deg, i, v, j0, j1);
    int64_t off = a.in_off[v];
    int64_t len = j1 - j0;
    int64_t w0 = j0 + len * w / NW, w1 = j0 + len * (w + 1) / NW;
    S4 acc;
    sum_range<LPR>(a.in_ids + off, w0, w1, a.M, a.ldm, lane_on, q, acc);
#pragma unroll
    for (int c = 0; c < 4; c++) sv[w][l * 4 + c] = acc.v[c];
    __syncthreads();
    if (w == 0) {
      for (int ww = 1; ww < NW; ww++)
#pragma unroll
        for (int c = 0; c < 4; c++) acc.v[c] = __fadd_rn(acc.v[c], sv[ww][l * 4 + c]);
      if (lane_on && l < LPR) {
        int64_t o = (int64_t)cg * a.wd + 4 * q;
#pragma unroll
        for (int c = 0; c < 4; c++) put_part<COHERENT>(part + o + c, acc.v[c]);
      }
      stored(i, v);
    }
    __syncthreads();
  }
}

template <int LPR>
__global__ __launch_bounds__(256) void k_sum_big_partial(AggArgs a, const Counters *cnt, float *part) {
  constexpr int NW = 4;
  __shared__ float sv[NW][kWave * 4];
  whole_sum_chunks<LPR, NW, false>(a, cnt->v[C_NCHUNK], cnt->v[C_NBIG], sv, part, [](int, int) {});
}

// Chunks of the other rows, in slices (bigrows.h).  Whole rows came from beyond the L2 as often as not (GCN of 256 columns
// on 29k nodes with 490 neighbours each, a table of 30 MB: 45M of 89M lines, 7 TB/s, 795 us); a slice of 32 columns stays
// in an XCD's L2 (4.4M of 97M lines, 661 us, 18.8 TB/s out of the L2s, of which the narrow rows above reach 17 to 24).
// Inferences: that one 1.43 -> 1.22 ms, 100k nodes with 200 neighbours each and 256 columns 2.50 -> 2.27, GIN of 128
// columns on 20k, 100k, 400k and 1M nodes 1.02, 1.0, 1.04 and 1.01 times as fast.
template <int NW, bool COHERENT, class Stored>
__device__ __forceinline__ void sum_slices(const AggArgs &a, int total, int n_big, int slices, float (*sv)[kSliceCols], float *part, const Stored &stored) {
  constexpr int LPR = kSliceLanes;
  const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int q = l % LPR, items = slice_items(total, slices);
  for (int b = blockIdx.x; b < items; b += gridDim.x) {
    int cg, slice, i, v;
    int64_t j0, j1;
    if (!slice_item(b, total, slices, cg, slice)) continue;
    big_chunk(a.big, n_big, cg, a.in_deg, i, v, j0, j1);
    const int64_t off = a.in_off[v], len = j1 - j0;
    const int64_t w0 = j0 + len * w / NW, w1 = j0 + len * (w + 1) / NW;
    const int c0 = slice * kSliceCols;
    S4 acc;
    sum_range<LPR>(a.in_ids + off, w0, w1, a.M + c0, a.ldm, c0 + 4 * q < a.wd, q, acc);
    if (l < LPR)
#pragma unroll
      for (int c = 0; c < 4; c++) sv[w][l * 4 + c] = acc.v[c];
    __syncthreads();
    const int col = threadIdx.x;
    if (col < kSliceCols && c0 + col < a.wd) {
      float x = sv[0][col];
      for (int ww = 1; ww < NW; ww++) x = __fadd_rn(x, sv[ww][col]);
      put_part<COHERENT>(part + (int64_t)cg * a.wd + c0 + col, x);
    }
    if (w == 0) stored(i, v);
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_sum_big_slices(AggArgs a, const Counters *cnt, int slices, float *part) {
  __shared__ float sv[4][kSliceCols];
  sum_slices<4, false>(a, cnt->v[C_NCHUNK], cnt->v[C_NBIG], slices, sv, part, [](int, int) {});
}

// One wave combines the parts [p0, p1) of row v: its lane groups take them in turn, U of them in flight.
template <int LPR, int U, bool COHERENT>
__device__ __forceinline__ void combine_sum_row(const AggArgs &a, int v, int p0, int p1, const float *part, uint64_t *chg, int compare) {
  const int l = lane_id();
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd && lane_in_groups<LPR>();
  constexpr int G = kWave / LPR;
  const int g = l / LPR < G ? l / LPR : G - 1, qo = lane_on ? 4 * q : 0;
  S4 acc;
#pragma unroll
  for (int c = 0; c < 4; c++) acc.v[c] = 0.f;
  for (int pb = p0; pb < p1; pb += G * U) {
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int p = pb + u * G + g;
      x[u] = get_part<COHERENT, float4>(part + (int64_t)(p < p1 ? p : p1 - 1) * a.wd + qo);
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const bool on = pb + u * G + g < p1;
      const float y[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
      for (int c = 0; c < 4; c++) acc.v[c] = __fadd_rn(acc.v[c], on ? y[c] : 0.f);
    }
  }
  sum_groups<LPR>(acc);
  const bool ch = store_sum<LPR>(a.A, a.ld, a.d, v, lane_on, q, acc, compare != 0);
  if (ch && chg && l == 0) mark_bit_s(chg, v);
}

// Launches of few targets: 16 waves a chunk, and its slices in workgroups of their own unless they are many (kSlicedItems); a row's
// last part combines it if there are few (combine_on_arrival).  64 registers, so that a CU holds two, which leaves 12 or 20
// bytes a lane of half of the forms to scratch.
template <int LPR, bool ARRIVE>
__global__ __launch_bounds__(1024, 8) void k_sum_big_short(AggArgs a, const Counters *cnt, int slices, float *part, uint64_t *chg, int compare,
                                                           int32_t *arrived) {
  constexpr int NW = 16;
  __shared__ float whole[NW][kWave * 4], sliced[NW][kSliceCols];
  const int total = cnt->v[C_NCHUNK], n_big = cnt->v[C_NBIG];
  const bool whole_rows = total > kSlicedItems / slices;
  auto stored = [&](int i, int v) {
    if constexpr (ARRIVE) {
      const int chunks = big_row_chunks(a.in_deg[v], a.big.chunk), p0 = a.big.base[i];
      if (last_to_arrive(arrived + i, whole_rows ? chunks : chunks * slices)) combine_sum_row<LPR, 4, true>(a, v, p0, p0 + chunks, part, chg, compare);
    }
  };
  if (whole_rows) whole_sum_chunks<LPR, NW, ARRIVE>(a, total, n_big, whole, part, stored);
  else sum_slices<NW, ARRIVE>(a, total, n_big, slices, sliced, part, stored);
}

template <int LPR>
__global__ __launch_bounds__(64) void k_sum_big_final(AggArgs a, const float *part, uint64_t *chg, int compare,
                                                      const Counters *cnt) {
  const int n_big = cnt->v[C_NBIG];
  for (int i = blockIdx.x; i < n_big; i += gridDim.x) {
    const int v = a.big.list[i], p0 = a.big.base[i];
    combine_sum_row<LPR, 8, false>(a, v, p0, p0 + big_row_chunks(a.in_deg[v], a.big.chunk), part, chg, compare);
  }
}

__device__ __forceinline__ int find_in(const int32_t *F, int nF, int u) {   // position of u in ascending F, or -1
  int lo = 0, hi = nF - 1;
  while (lo <= hi) {
    int m = (lo + hi) >> 1;
    int x = F[m];
    if (x == u) return m;
    if (x < u) lo = m + 1; else hi = m - 1;
  }
  return -1;
}

__global__ void k_delta_rows(const float *M, int ldm, const int32_t *F, int nF, const float *f_old, float *f_delta,
                             int ld_old) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t i = t / ld_old;
  int k = (int)(t % ld_old);
  if (i < nF) f_delta[i * ld_old + k] = __fsub_rn(M[(int64_t)F[i] * ldm + k], f_old[i * ld_old + k]);
}

struct SumSources {             // the changed sources of the layer and their rows
  const int32_t *F; int nF;
  const float *f_old, *f_delta; int ld_old;
};

// What an event adds, in its word: a row of f_delta (changed source), a row of M (inserted edge), or the negative of a
// row of f_old or M (removed edge: what the source contributed before).
enum : uint32_t { ADD_DELTA = 0, ADD_NEW = 1, SUB_OLD = 2, SUB_SAME = 3 };
static_assert(EV_CHG == 2 && EV_ADD == ADD_NEW, "kinds");

// device memory, named so: from an integer the compiler knows no more than a flat address
typedef __attribute__((address_space(1))) const char GlobalChar;
typedef float F4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const F4v GlobalF4;

// U events of a window in order, a row to the wave: their addresses and signs are scalars, so an event is three
// v_readlane, one load and four multiply-adds (y * 1 and y * -1 are exact: the sums are those of additions).  With the
// address worked out for each event and the last batch padded to eight it was 21 vector and 26 scalar instructions, and
// the waves waited for issue more than for memory: 1.56M events of 256 columns for 87k targets 134 -> 113 us.
template <int U>
__device__ __forceinline__ void add_event_rows(uint32_t lo, uint32_t hi, float sign, int it, uint32_t lane_bytes, S4 &acc) {
  F4v r[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const uint64_t row = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, it + u) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)lo, it + u);
    r[u] = *reinterpret_cast<const GlobalF4 *>(reinterpret_cast<const GlobalChar *>(row) + lane_bytes);
  }
#pragma unroll
  for (int u = 0; u < U; u++) {
    const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sign), it + u));
    const float y[4] = {r[u].x, r[u].y, r[u].z, r[u].w};
#pragma unroll
    for (int c = 0; c < 4; c++) acc.v[c] = __fmaf_rn(y[c], s, acc.v[c]);
  }
}

// Each lane finds the row of its own event once per window (a removed edge is a search of F), and the loads stand under no
// condition: 116k-node GCN of 256 columns, 500 updates, 3.34 -> 3.16 ms a pass against a search per lane group and a masked
// load per event.
// adds the events [e0, e1) of one target to acc: lane group g takes e0 + g, e0 + g + G, ... in order
template <int LPR>
__device__ __forceinline__ void sum_event_range(const AggArgs &a, const uint32_t *ev, int e0, int e1, const SumSources &src,
                                                bool lane_on, int q, S4 &acc) {
  constexpr int G = kWave / LPR;
  constexpr int U = LPR == kWave ? 8 : 4;    // events in flight per lane group (8 for one group: GCN of 256 columns 3.08 -> 3.03 ms a pass; for two: GIN 7.28 -> 7.36)
  const int l = lane_id();
  const RowTable<LPR> tab(a.M, a.ldm, lane_on, q);
  const uint32_t old_bytes = (uint32_t)src.ld_old * 4u;
  for (int eb = e0; eb < e1; eb += kWave) {
    const int ee = eb + l;
    uint32_t mine = ev[ee < e1 ? ee : e1 - 1];
    const int cntw = (e1 - eb) < kWave ? (e1 - eb) : kWave;
    // each lane finds the row of its own event
    const uint32_t kind = mine >> kEvKindShift;
    if (kind == EV_CHG) mine &= kEvIdMask;          // ADD_DELTA, position of the source in F
    if (kind == EV_DEL) {
      const int pos = src.nF > 0 ? find_in(src.F, src.nF, (int)(mine & kEvIdMask)) : -1;
      mine = pos >= 0 ? (SUB_OLD << kEvKindShift) | (uint32_t)pos : (SUB_SAME << kEvKindShift) | mine;
    }
    auto row_of = [&](uint32_t x) {                  // tables picked by selects: every load is unconditional
      const uint32_t k = x >> kEvKindShift;
      const char *t = reinterpret_cast<const char *>(k & 1u ? a.M : (k == ADD_DELTA ? src.f_delta : src.f_old));
      return t + (uint64_t)(x & kEvIdMask) * (k & 1u ? tab.row_bytes : old_bytes);
    };
    if constexpr (G == 1) {
      const uint64_t at = reinterpret_cast<uint64_t>(row_of(mine));
      const uint32_t lo = (uint32_t)at, hi = (uint32_t)(at >> 32);
      const float sign = mine & 0x80000000u ? -1.f : 1.f;
      int it = 0;
      for (; it + U <= cntw; it += U) add_event_rows<U>(lo, hi, sign, it, tab.lane_bytes, acc);
      if (cntw - it >= 4) { add_event_rows<4>(lo, hi, sign, it, tab.lane_bytes, acc); it += 4; }
      if (cntw - it >= 2) { add_event_rows<2>(lo, hi, sign, it, tab.lane_bytes, acc); it += 2; }
      if (cntw - it >= 1) add_event_rows<1>(lo, hi, sign, it, tab.lane_bytes, acc);
    } else {
      for (int it = 0; it < cntw; it += G * U) {
        uint32_t x[U];
        float4 r[U];
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = (uint32_t)tab.template pick<U>((int)mine, it, u, cntw - 1);
#pragma unroll
        for (int u = 0; u < U; u++) r[u] = *reinterpret_cast<const float4 *>(row_of(x[u]) + tab.lane_bytes);
#pragma unroll
        for (int u = 0; u < U; u++) {
          const bool on = it + u * G + tab.g < cntw;
          const uint32_t neg = x[u] & 0x80000000u;          // SUB_*: a - b is a + (-b)
          const float y[4] = {r[u].x, r[u].y, r[u].z, r[u].w};
#pragma unroll
          for (int c = 0; c < 4; c++) acc.v[c] = __fadd_rn(acc.v[c], on ? __uint_as_float(__float_as_uint(y[c]) ^ neg) : 0.f);
        }
      }
    }
  }
}

// cached row of v plus acc, stored if it changed
template <int LPR>
__device__ __forceinline__ void add_to_row(const AggArgs &a, int v, bool lane_on, int q, const S4 &acc, uint64_t *chg, Counters *cnt) {
  S4 nv;
#pragma unroll
  for (int c = 0; c < 4; c++) nv.v[c] = 0.f;
  if (lane_on) {
    float4 o = ldf4(a.A + (int64_t)v * a.ld + 4 * q);
    nv.v[0] = __fadd_rn(o.x, acc.v[0]); nv.v[1] = __fadd_rn(o.y, acc.v[1]);
    nv.v[2] = __fadd_rn(o.z, acc.v[2]); nv.v[3] = __fadd_rn(o.w, acc.v[3]);
  }
  bool ch = store_sum<LPR>(a.A, a.ld, a.d, v, lane_on, q, nv, true);
  if (ch && lane_id() == 0) { mark_bit_s(chg, v); if (a.count_cond) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_ACHG], 1ull); }
}

template <int LPR>
__global__ __launch_bounds__(256) void k_sum_events(AggArgs a, const int32_t *targets, const int32_t *seg,
                                                    const int32_t *n_targets_p, const uint32_t *ev, SumSources src,
                                                    uint64_t *chg, Counters *cnt, LongEvents lng) {
  const int q = lane_id() % LPR;
  const bool lane_on = 4 * q < a.wd;
  // wave-uniform: target and bounds are scalar loads (GIN, 1.25M nodes: 7.37 -> 7.28 ms a pass)
  const int wid = (int)blockIdx.x * (int)(blockDim.x / kWave) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  if (wid >= *n_targets_p) return;
  const int e0 = seg[wid], e1 = seg[wid + 1];
  if (e1 - e0 > lng.limit) { list_long_segment(lng, wid, e1 - e0, cnt); return; }
  S4 acc;
#pragma unroll
  for (int c = 0; c < 4; c++) acc.v[c] = 0.f;
  sum_event_range<LPR>(a, ev, e0, e1, src, lane_on, q, acc);
  sum_groups<LPR>(acc);
  add_to_row<LPR>(a, targets[wid], lane_on, q, acc, chg, cnt);
}

// one wave per long segment: its lane groups take the chunks in turn
template <int LPR, bool COHERENT>
__device__ __forceinline__ void combine_sum_segment(const AggArgs &a, const int32_t *targets, const LongEvents &lng, const LongSeg &L, int n_ev,
                                                    const float *part, uint64_t *chg, Counters *cnt) {
  constexpr int G = kWave / LPR;
  const int l = lane_id(), q = l % LPR, g = l / LPR;
  const bool lane_on = 4 * q < a.wd;
  const int nch = long_seg_chunks(lng, n_ev);
  S4 acc;
#pragma unroll
  for (int c = 0; c < 4; c++) acc.v[c] = 0.f;
  if (lane_on)
    for (int p = g; p < nch; p += G) {
      const float4 x = get_part<COHERENT, float4>(part + (int64_t)(L.base + p) * a.wd + 4 * q);
      acc.v[0] = __fadd_rn(acc.v[0], x.x); acc.v[1] = __fadd_rn(acc.v[1], x.y);
      acc.v[2] = __fadd_rn(acc.v[2], x.z); acc.v[3] = __fadd_rn(acc.v[3], x.w);
    }
  sum_groups<LPR>(acc);
  add_to_row<LPR>(a, targets[L.target], lane_on, q, acc, chg, cnt);
}

// one workgroup per chunk of a long segment, its waves take a quarter of the events each; ARRIVE (short launches): the segment's last chunk combines it
template <int LPR, bool ARRIVE>
__global__ __launch_bounds__(256) void k_sum_ev_partial(AggArgs a, const int32_t *targets, const int32_t *seg, const uint32_t *ev, SumSources src,
                                                        LongEvents lng, float *part, uint64_t *chg, Counters *cnt, int32_t *arrived) {
  constexpr int NW = 4;
  __shared__ float sv[NW][kWave * 4];
  const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  const int total = cnt->v[C_NEVCH];
  for (int ch = blockIdx.x; ch < total; ch += gridDim.x) {
    int e0, e1;
    long_chunk(lng, ch, seg, e0, e1);
    const int len = e1 - e0;
    S4 acc;
#pragma unroll
    for (int c = 0; c < 4; c++) acc.v[c] = 0.f;
    sum_event_range<LPR>(a, ev, e0 + len * w / NW, e0 + len * (w + 1) / NW, src, lane_on, q, acc);
    sum_groups<LPR>(acc);
#pragma unroll
    for (int c = 0; c < 4; c++) sv[w][l * 4 + c] = acc.v[c];
    __syncthreads();
    if (w == 0) {
      if (lane_on && l < LPR) {
        for (int ww = 1; ww < NW; ww++)
#pragma unroll
          for (int c = 0; c < 4; c++) acc.v[c] = __fadd_rn(acc.v[c], sv[ww][l * 4 + c]);
#pragma unroll
        for (int c = 0; c < 4; c++) put_part<ARRIVE>(part + (int64_t)ch * a.wd + 4 * q + c, acc.v[c]);
      }
      if constexpr (ARRIVE) {
        const int i = lng.owner[ch];
        const LongSeg L = lng.list[i];
        const int n_ev = seg[L.target + 1] - seg[L.target];
        if (last_to_arrive(arrived + i, long_seg_chunks(lng, n_ev))) combine_sum_segment<LPR, true>(a, targets, lng, L, n_ev, part, chg, cnt);
      }
    }
    __syncthreads();
  }
}

template <int LPR>
__global__ __launch_bounds__(64) void k_sum_ev_final(AggArgs a, const int32_t *targets, const int32_t *seg, LongEvents lng,
                                                     const float *part, uint64_t *chg, Counters *cnt) {
  const int n = cnt->v[C_NEVL];
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const LongSeg L = lng.list[i];
    combine_sum_segment<LPR, false>(a, targets, lng, L, seg[L.target + 1] - seg[L.target], part, chg, cnt);
  }
}

static int lanes_per_row(int ld) { return ld <= 64 ? 16 : (ld <= 128 ? 32 : 64); }
// full re-aggregation only: narrow rows take 12 lanes (rows of 41 floats, 233k nodes / 114M edges: 4.5 % less aggregation time)
static int lanes_per_row_full(int ld) { return ld <= 48 ? 12 : lanes_per_row(ld); }

template <int LPR>
static hipError_t sum_full_t(ink_ctx *c, const AggArgs &a_in, const int32_t *targets, int64_t n_targets,
                             uint64_t *chg) {
  if (n_targets <= 0) return hipSuccess;
  AggArgs a = a_in;
  a.big_deg = big_threshold(n_targets, LPR, kBigDegSum);
  int compare = chg != nullptr;
  INK_TRY(ensure_big_buffers(c, a.wd, false));
  const bool latency = latency_mode(n_targets), whole = LPR == 12 || (int64_t)a.n * a.ldm * 4 > kSlicedTableBytes;
  a.big = big_rows_of(c, latency || whole ? kBigChunk : kBigChunkSum);
  INK_TRY(clear_big_rows(c));
  {
    KernelTimer kt(c, a.layer, INK_K_AGG_FULL);
    hipLaunchKernelGGL((k_sum_full<LPR>), dim3((unsigned)((n_targets + 3) / 4)), dim3(256), 0, c->stream, a, targets,
                       n_targets, chg, compare, c->d_cnt);
    INK_TRY(hipGetLastError());
  }
  KernelTimer kt(c, a.layer, INK_K_AGG_LONG);
  const int slices = big_slices(a.wd);
  const Counters *cnt = c->d_cnt;
  float *part = c->big_part_v.as<float>();
  const bool arrive = latency && combine_on_arrival(a, true);
  if (arrive)
    hipLaunchKernelGGL((k_sum_big_short<LPR, true>), dim3(big_grid(c, a.big_chunks, slices, true)), dim3(1024), 0, c->stream, a, cnt, slices, part, chg,
                       compare, c->arrived);
  else if (latency)
    hipLaunchKernelGGL((k_sum_big_short<LPR, false>), dim3(big_grid(c, a.big_chunks, slices, true)), dim3(1024), 0, c->stream, a, cnt, slices, part, chg,
                       compare, c->arrived);
  else if (whole)
    hipLaunchKernelGGL((k_sum_big_partial<LPR>), dim3(big_grid(c, a.big_chunks, 1, false)), dim3(256), 0, c->stream, a, cnt, part);
  else
    hipLaunchKernelGGL(k_sum_big_slices, dim3(big_grid(c, a.big_chunks, slices, false)), dim3(256), 0, c->stream, a, cnt, slices, part);
  if (!arrive) hipLaunchKernelGGL((k_sum_big_final<LPR>), dim3(kBigGrid), dim3(64), 0, c->stream, a, (const float *)part, chg, compare, cnt);
  return hipGetLastError();
}

template <int LPR>
static hipError_t sum_events_t(ink_ctx *c, const AggArgs &a, const int32_t *targets, const int32_t *seg,
                               int64_t n_targets, const int32_t *n_targets_dev, const uint32_t *ev, const EventBounds &eb,
                               const SumSources &src, uint64_t *chg) {
  if (n_targets <= 0) return hipSuccess;
  KernelTimer kt(c, a.layer, INK_K_AGG_EVENTS);
  LongEvents lng = long_events(eb, n_targets);
  INK_TRY(ensure_long_events(c, eb, a.wd, false, &lng));
  hipLaunchKernelGGL((k_sum_events<LPR>), dim3((unsigned)((n_targets + 3) / 4)), dim3(256), 0, c->stream, a, targets,
                     seg, n_targets_dev, ev, src, chg, c->d_cnt, lng);
  if (eb.max_seg > lng.limit) {      // otherwise no segment can be long
    float *part = c->big_part_v.as<float>();
    const dim3 chunks((unsigned)std::min<int64_t>(long_ev_chunks(lng, eb.n_events), 8192)), rows((unsigned)std::min<int64_t>(long_ev_rows(lng, eb.n_events), 8192));
    if (latency_mode(n_targets)) {
      hipLaunchKernelGGL((k_sum_ev_partial<LPR, true>), chunks, dim3(256), 0, c->stream, a, targets, seg, ev, src, lng, part, chg, c->d_cnt, c->arrived);
    } else {
      hipLaunchKernelGGL((k_sum_ev_partial<LPR, false>), chunks, dim3(256), 0, c->stream, a, targets, seg, ev, src, lng, part, chg, c->d_cnt, c->arrived);
      hipLaunchKernelGGL((k_sum_ev_final<LPR>), rows, dim3(64), 0, c->stream, a, targets, seg, lng, (const float *)part, chg, c->d_cnt);
    }
  }
  return hipGetLastError();
}

hipError_t agg_sum_full(ink_ctx *c, const AggArgs &a, const int32_t *targets, int64_t n_targets, uint64_t *chg) {
  switch (lanes_per_row_full(a.wd)) {
    case 12: return sum_full_t<12>(c, a, targets, n_targets, chg);
    case 16: return sum_full_t<16>(c, a, targets, n_targets, chg);
    case 32: return sum_full_t<32>(c, a, targets, n_targets, chg);
    default: return sum_full_t<64>(c, a, targets, n_targets, chg);
  }
}

hipError_t agg_sum_events(ink_ctx *c, const AggArgs &a, const int32_t *targets, const int32_t *seg,
                          int64_t n_targets, const int32_t *n_targets_dev, const uint32_t *ev_val, const EventBounds &eb,
                          const int32_t *F, int nF, const float *f_old, const float *f_delta, int ld_old, uint64_t *chg) {
  const SumSources src{F, nF, f_old, f_delta, ld_old};
  switch (lanes_per_row(a.wd)) {
    case 16: return sum_events_t<16>(c, a, targets, seg, n_targets, n_targets_dev, ev_val, eb, src, chg);
    case 32: return sum_events_t<32>(c, a, targets, seg, n_targets, n_targets_dev, ev_val, eb, src, chg);
    default: return sum_events_t<64>(c, a, targets, seg, n_targets, n_targets_dev, ev_val, eb, src, chg);
  }
}

hipError_t agg_sum_delta_rows(ink_ctx *c, const AggArgs &a, const int32_t *F, int nF, const float *f_old,
                              float *f_delta, int ld_old) {
  if (nF <= 0) return hipSuccess;
  int64_t n = (int64_t)nF * ld_old;
  hipLaunchKernelGGL(k_delta_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, a.M, a.ldm, F, nF, f_old,
                     f_delta, ld_old);
  return hipGetLastError();
}

}  // namespace ink
