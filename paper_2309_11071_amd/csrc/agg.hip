// Aggregation kernels for the selection aggregators (max / min) with per-dimension argument
// tracking: full re-aggregation ("recompute", Sec. 2.5.2) and the event-driven incremental
// update with reset detection (Sec. 2.5.1).  One wave64 owns one target row; a lane holds four
// consecutive dimensions, so a row of d floats occupies LPR = 16/32/64 lanes and a wave works on
// 64 / LPR neighbour rows at a time.  Rows are read as coalesced 16-byte lane loads.
//
// Next to the selected value and its holder the cache keeps, per dimension, a bound on the best
// value among the OTHER neighbours (exact after a recompute, afterwards only ever loosened).  A
// holder that got worse but still strictly beats that bound stays the holder, and a candidate that
// strictly beats it covers a reset even if it is worse than the old value: both save the
// recompute that the value-only rule of Sec. 2.5.1 would need.
#include <algorithm>

#include "rowblock.h"
#include "select.h"

#ifndef INK_EV_INLINE_WIDE
#define INK_EV_INLINE_WIDE 1       // inline recompute of exposed rows: 0 never, 1 rows of 64 lanes and short launches, 2 also 32 lanes, 3 always
#endif
#ifndef INK_EVENT_GRID
#define INK_EVENT_GRID 8192        // workgroups of the event kernel (measured: 4096-8192 best, fewer leave a tail)
#endif

namespace ink {



// ------------------------------------------------------------------ full re-aggregation
// what a recompute launch does besides storing the rows
enum { FULL_COMPARE = 1,        // compare with the cached row: store and mark only what changed
       FULL_TALLY = 2,          // count the rows and the neighbour rows fetched
       FULL_COUNT_CHANGED = 4 };   // count the rows whose value changed

// A wave takes blocks of rows (rowblock.h), the grid strides over them; n_targets_dev (optional) is the device-side
// row count, n_targets then only bounds it.
template <bool IS_MIN, int LPR>
__global__ __launch_bounds__(256) void k_agg_full(AggArgs a, const int32_t *targets, int64_t n_targets,
                                                  const int32_t *n_targets_dev, uint64_t *chg, int flags, Counters *cnt) {
  const int l = lane_id();
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  if (n_targets_dev) { int64_t nd = *n_targets_dev; n_targets = nd < n_targets ? nd : n_targets; }
  const int64_t n_waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  const int per = ieee_mode_off(row_block(n_targets, n_waves));
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  int64_t nb = 0, nb_long = 0;
  for (int64_t r0 = ((int64_t)blockIdx.x * (blockDim.x / kWave) + wave) * per; r0 < n_targets; r0 += n_waves * per) {
    RowBlock B;
    B.load(a, targets, r0, n_targets - r0 < per ? (int)(n_targets - r0) : per, chg, cnt, nb, nb_long);
    int win = 0;
    if (B.todo) win = B.first_ids(a.in_ids, __builtin_ctzll(B.todo));
    while (B.todo) {
      const int j = __builtin_ctzll(B.todo), v = B.row(j);
      B.todo &= B.todo - 1;
      const int next = B.todo ? B.first_ids(a.in_ids, __builtin_ctzll(B.todo)) : 0;
      F4 bv; I4 bi; F4 sv; I4 si;
      gather_row<IS_MIN, LPR>(a.in_ids + B.place(j), B.length(j), win, a.M, a.ldm, lane_on, q, a.nonneg, B.ascending(j), bv, bi, sv, si);
      win = next;
      finish_empty<IS_MIN>(bv, bi, sv, si);
      RowOut o{a.A, a.ARG, a.UB, a.ARG2, a.ld, a.d};
      F4 dum; I4 dumi;
      bool ch;
      if (flags & FULL_COMPARE) ch = store_row<LPR>(o, v, lane_on, q, bv, bi, sv, si, false, dum, dumi);
      else {
        const int64_t o4 = (int64_t)v * a.ld + 4 * q;       // every lane group has the row: the first two store half of the tables each
        if (lane_on && l < LPR) {
          store_past(a.A + o4, bv.v);
          store_past(a.ARG + o4, bi.v);
        }
        if (lane_on && (LPR == kWave || l / LPR == 1)) {
          store_past(a.UB + o4, sv.v);
          store_past(a.ARG2 + o4, si.v);
        }
        ch = false;
      }
      if (ch && chg && l == 0) {
        mark_bit(chg, v);
        if ((flags & FULL_COUNT_CHANGED) && a.count_cond) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_ACHG], 1ull);
      }
    }
  }
  if (flags & FULL_TALLY) tally_rows(cnt, nb, nb_long);
}

// cooperative path for rows with more than kBigDeg in-neighbours: a workgroup per chunk of
// kBigChunk neighbours, partial rows to scratch
struct BigParts { float *v; int32_t *i; float *s; int32_t *j; };     // best, its id, runner-up, its id: a row per chunk

// whole rows: the NW waves of a workgroup take a part of a chunk each; the wave that has stored a part calls stored(place of its row in the list, node)
template <bool IS_MIN, int LPR, int NW, bool COHERENT, class Stored>
__device__ __forceinline__ void whole_chunks(const AggArgs &a, int total, int n_big, float (*sv)[kWave * 4], int (*si)[kWave * 4], float (*ss)[kWave * 4],
                                             int (*sj)[kWave * 4], const BigParts &part, const Stored &stored) {
  const int l = lane_id(), w = threadIdx.x / kWave;
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  for (int cg = blockIdx.x; cg < total; cg += gridDim.x) {
    int i, v;
    int64_t j0, j1;
    big_chunk(a.big, n_big, cg, a.in_deg, i, v, j0, j1);
    int64_t off = a.in_off[v];
    int64_t len = j1 - j0;
    int64_t w0 = j0 + len * w / NW, w1 = j0 + len * (w + 1) / NW;
    F4 bv; I4 bi; F4 s2; I4 j2;
    gather_range<IS_MIN, LPR>(a.in_ids + off, w0, w1, a.M, a.ldm, lane_on, q, a.nonneg, a.in_asc[v] != 0, bv, bi, s2, j2);
#pragma unroll
    for (int c = 0; c < 4; c++) {
      sv[w][l * 4 + c] = bv.v[c]; si[w][l * 4 + c] = bi.v[c]; ss[w][l * 4 + c] = s2.v[c]; sj[w][l * 4 + c] = j2.v[c];
    }
    __syncthreads();
    if (w == 0) {
      for (int ww = 1; ww < NW; ww++)
#pragma unroll
        for (int c = 0; c < 4; c++)
          merge2i<IS_MIN>(sv[ww][l * 4 + c], si[ww][l * 4 + c], ss[ww][l * 4 + c], sj[ww][l * 4 + c], bv.v[c], bi.v[c],
                          s2.v[c], j2.v[c]);
      if (lane_on && l < LPR) {
        int64_t o = (int64_t)cg * a.wd + 4 * q;
#pragma unroll
        for (int c = 0; c < 4; c++) {
          put_part<COHERENT>(part.v + o + c, bv.v[c]); put_part<COHERENT>(part.i + o + c, bi.v[c]);
          put_part<COHERENT>(part.s + o + c, s2.v[c]); put_part<COHERENT>(part.j + o + c, j2.v[c]);
        }
      }
      stored(i, v);
    }
    __syncthreads();
  }
}

template <bool IS_MIN, int LPR>
__global__ __launch_bounds__(256) void k_big_partial(AggArgs a, const Counters *cnt, BigParts part) {
  constexpr int NW = 4;
  __shared__ float sv[NW][kWave * 4], ss[NW][kWave * 4];
  __shared__ int si[NW][kWave * 4], sj[NW][kWave * 4];
  const int total = ieee_mode_off(cnt->v[C_NCHUNK]);
  whole_chunks<IS_MIN, LPR, NW, false>(a, total, cnt->v[C_NBIG], sv, si, ss, sj, part, [](int, int) {});
}

// One wave combines the parts [p0, p1) of row v: its lane groups take them in turn, U of them in flight, then the row is stored.  (One
// row after the other made a hub's chain the launch's time: 45 us on 12.5M edges and rows of 128 floats, now 21.)
template <bool IS_MIN, int LPR, int U, bool COHERENT>
__device__ __forceinline__ void combine_row(const AggArgs &a, int v, int p0, int p1, const BigParts &part, uint64_t *chg, int compare, Counters *cnt) {
  const int l = lane_id();
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  constexpr int G = kWave / LPR;
  const int g = l / LPR, qo = lane_on ? 4 * q : 0;
  F4 bv; I4 bi; F4 s2; I4 j2;
#pragma unroll
  for (int c = 0; c < 4; c++) {
    bv.v[c] = worst<IS_MIN>(); bi.v[c] = 0x7fffffff; s2.v[c] = worst<IS_MIN>(); j2.v[c] = 0x7fffffff;
  }
  for (int pb = p0; pb < p1; pb += G * U) {
    float4 xv[U], xs[U];
    int4 xi[U], xj[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int p = pb + u * G + g;
      const int64_t o = (int64_t)(p < p1 ? p : p1 - 1) * a.wd + qo;
      xv[u] = get_part<COHERENT, float4>(part.v + o); xi[u] = get_part<COHERENT, int4>(part.i + o);
      xs[u] = get_part<COHERENT, float4>(part.s + o); xj[u] = get_part<COHERENT, int4>(part.j + o);
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const bool on = pb + u * G + g < p1;        // a partial row past the end is empty: it takes no place
      const float yv[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w}, ys[4] = {xs[u].x, xs[u].y, xs[u].z, xs[u].w};
      const int yi[4] = {xi[u].x, xi[u].y, xi[u].z, xi[u].w}, yj[4] = {xj[u].x, xj[u].y, xj[u].z, xj[u].w};
#pragma unroll
      for (int c = 0; c < 4; c++)
        merge2i<IS_MIN>(on ? yv[c] : worst<IS_MIN>(), on ? yi[c] : 0x7fffffff, on ? ys[c] : worst<IS_MIN>(),
                        on ? yj[c] : 0x7fffffff, bv.v[c], bi.v[c], s2.v[c], j2.v[c]);
    }
  }
  reduce_groups_i<IS_MIN, LPR>(bv, bi, s2, j2);
  finish_empty<IS_MIN>(bv, bi, s2, j2);
  RowOut o{a.A, a.ARG, a.UB, a.ARG2, a.ld, a.d};
  F4 dum; I4 dumi;
  bool ch = store_row<LPR>(o, v, lane_on, q, bv, bi, s2, j2, false, dum, dumi);
  if (compare && ch && chg && l == 0) {
    mark_bit(chg, v);
    if (a.count_cond) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_ACHG], 1ull);
  }
}

// The same for launches of few targets, where one chunk's time is the launch's: 16 waves take a slice of kSliceCols
// columns of a chunk, so that a row of 128 floats is spread over four workgroups, and a load brings eight rows; many
// chunks (kSlicedItems) are whole rows again, 16 waves each.
// Updates of 100 edges: 10k nodes, rows of 64 floats, 1.13 -> 1.06 ms for four, 1.25M nodes, rows of 128, 1.58 -> 1.53 ms a pass.
// Long launches stay with whole rows: the slices leave a third of the reads beyond the L2 out (16.6M -> 10.8M of 128
// bytes, 625k nodes and rows of 128 floats), but the chunks' fixed costs four times over take as much (10 to 600k nodes,
// rows of 128 and 256 floats: 0.94 to 1.0 of the speed).
template <bool IS_MIN, int ROW, bool ARRIVE>
__global__ __launch_bounds__(1024) void k_big_short(AggArgs a, Counters *cnt, int slices, BigParts part, uint64_t *chg, int compare, int32_t *arrived) {
  constexpr int LPR = kSliceLanes, NW = 16;
  __shared__ float sv[NW][kWave * 4], ss[NW][kWave * 4];
  __shared__ int si[NW][kWave * 4], sj[NW][kWave * 4];
  const int total = ieee_mode_off(cnt->v[C_NCHUNK]), n_big = cnt->v[C_NBIG];
  const bool whole = slices > 2 && total > kSlicedItems / slices;
  // ARRIVE (few chunks): a row's last part combines it; a launch of its own took 6 to 7 us, this 4 to 5 (100 updates on 10k nodes 338 -> 324 us a pass)
  auto stored = [&](int i, int v) {
    if constexpr (ARRIVE) {
      const int chunks = big_row_chunks(a.in_deg[v], a.big.chunk), p0 = a.big.base[i];
      if (last_to_arrive(arrived + i, whole ? chunks : chunks * slices)) combine_row<IS_MIN, ROW, 2, true>(a, v, p0, p0 + chunks, part, chg, compare, cnt);
    }
  };
  if (whole) { whole_chunks<IS_MIN, ROW, NW, ARRIVE>(a, total, n_big, sv, si, ss, sj, part, stored); return; }
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
    F4 bv; I4 bi; F4 s2; I4 j2;
    gather_range<IS_MIN, LPR>(a.in_ids + off, w0, w1, a.M + c0, a.ldm, c0 + 4 * q < a.wd, q, a.nonneg, a.in_asc[v] != 0, bv, bi, s2, j2);
    if (l < LPR)
#pragma unroll
      for (int c = 0; c < 4; c++) {
        sv[w][l * 4 + c] = bv.v[c]; si[w][l * 4 + c] = bi.v[c]; ss[w][l * 4 + c] = s2.v[c]; sj[w][l * 4 + c] = j2.v[c];
      }
    __syncthreads();
    const int col = threadIdx.x;
    if (col < kSliceCols && c0 + col < a.wd) {
      float xv = sv[0][col], xs = ss[0][col];
      int xi = si[0][col], xj = sj[0][col];
      for (int ww = 1; ww < NW; ww++) merge2i<IS_MIN>(sv[ww][col], si[ww][col], ss[ww][col], sj[ww][col], xv, xi, xs, xj);
      const int64_t o = (int64_t)cg * a.wd + c0 + col;
      put_part<ARRIVE>(part.v + o, xv); put_part<ARRIVE>(part.i + o, xi); put_part<ARRIVE>(part.s + o, xs); put_part<ARRIVE>(part.j + o, xj);
    }
    if (w == 0) stored(i, v);
    __syncthreads();
  }
}

// A kernel for launches whose rows are many.  (In theirs the chunk kernel's registers would suffer from the combination: 80 -> 126.)
template <bool IS_MIN, int LPR>
__global__ __launch_bounds__(64) void k_big_final(AggArgs a, BigParts part, uint64_t *chg, int compare, Counters *cnt) {
  const int n_big = cnt->v[C_NBIG];
  for (int i = blockIdx.x; i < n_big; i += gridDim.x) {
    const int v = a.big.list[i], p0 = a.big.base[i];
    combine_row<IS_MIN, LPR, 4, false>(a, v, p0, p0 + big_row_chunks(a.in_deg[v], a.big.chunk), part, chg, compare, cnt);
  }
}

#ifndef INK_EV_BLOCK
#define INK_EV_BLOCK 8             // consecutive targets per wave visit (at most 62)
#endif
constexpr int kEvBlock = INK_EV_BLOCK;
// The grid is sized to what the chip holds at once; every wave walks blocks of kEvBlock consecutive
// targets with the grid's wave count as stride.  One load per block brings the targets' ids and
// segment bounds (lane j holds those of target j), so a target's own chain is: cached row and event
// words (issued together), then the source rows.
// INLINE: exposed rows of moderate length are recomputed by the wave that finds them instead of
// being listed for a follow-up launch.  Measured: on large launches over 128-float rows the listing
// form is 3 % faster (waves that recompute leave their neighbours in the block waiting), on rows of
// 256 floats the inline form saves 0.1 of 0.9 ms of aggregation, and on short launches it saves a
// launch.  The launcher picks per call.
template <bool IS_MIN, int LPR, bool INLINE>
__global__ __launch_bounds__(256) void k_agg_events(AggArgs a, const int32_t *targets, const int32_t *seg,
                                                    const int32_t *n_targets_p, const uint32_t *ev, uint64_t *chg,
                                                    int32_t *exp_list, Counters *cnt, int ev_block,
                                                    LongEvents lng) {
  static_assert(kEvBlock + 2 <= kWave, "a lane per target and bound of the block");
  RowSink exp;
  const int l = lane_id();
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  const int n = INLINE ? ieee_mode_off(*n_targets_p) : *n_targets_p;      // exposed rows are gathered here
  const int n_blk = (n + ev_block - 1) / ev_block;      // ev_block <= kEvBlock: 1 for short launches, whose targets should not queue behind each other in one wave
  const int n_waves = (int)gridDim.x * (int)(blockDim.x / kWave);
  const int wave0 = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave));
  for (int blk = wave0; blk < n_blk; blk += n_waves) {
    const int w0 = blk * ev_block;
    const int kt = n - w0 < ev_block ? n - w0 : ev_block;
    const int my_t = targets[w0 + (l < kt ? l : kt - 1)];
    const int my_s = seg[w0 + (l <= kt ? l : kt)];
    for (int t = 0; t < kt; t++) {
      const int v = __builtin_amdgcn_readlane(my_t, t);
      const int e0 = __builtin_amdgcn_readlane(my_s, t), e1 = __builtin_amdgcn_readlane(my_s, t + 1);
      if (e1 - e0 > lng.limit) { list_long_segment(lng, w0 + t, e1 - e0, cnt); continue; }
      Cached<IS_MIN> c;
      EvAcc<IS_MIN> s;
      reduce_events<IS_MIN, LPR>(a, v, ev, e0, e1, lane_on, q, c, s);
      finish_target<IS_MIN, LPR, INLINE>(a, v, c, s, lane_on, q, BitMark{chg}, exp_list, exp, cnt);
    }
  }
  if constexpr (!INLINE) exp.flush(exp_list, &cnt->v[C_NEXP]);
}

// What the waves of a long segment's chunk hand on, per dimension: best candidate, its source, the
// runner-up candidate value, and the flags (bit 0 reset, bit 1 runner-up invalid, bit 2 any_del).
struct EvPart { float *v; int32_t *i; float *s; int32_t *f; };

// One wave per long segment: its lane groups take the chunks in turn, then the target is decided.
template <bool IS_MIN, int LPR, bool INLINE, bool COHERENT>
__device__ __forceinline__ void combine_segment(const AggArgs &a, const int32_t *targets, const LongEvents &lng, const LongSeg &L, int n_ev,
                                                const EvPart &part, uint64_t *chg, int32_t *exp_list, RowSink &exp, Counters *cnt) {
  constexpr int G = kWave / LPR;
  const int l = lane_id(), q = l % LPR, g = l / LPR;
  const bool lane_on = 4 * q < a.wd;
  const int v = targets[L.target];
  const int nch = long_seg_chunks(lng, n_ev);
  Cached<IS_MIN> c;
  load_cached<IS_MIN>(a, v, lane_on, q, c);
  EvAcc<IS_MIN> s;
  s.init();
  int fl = 0;
  if (lane_on)
    for (int p = g; p < nch; p += G) {
      const int64_t o = (int64_t)(L.base + p) * a.wd + 4 * q;
      const float4 pv = get_part<COHERENT, float4>(part.v + o), ps = get_part<COHERENT, float4>(part.s + o);
      const int4 pi = get_part<COHERENT, int4>(part.i + o), pf = get_part<COHERENT, int4>(part.f + o);
      const float xv[4] = {pv.x, pv.y, pv.z, pv.w}, xs[4] = {ps.x, ps.y, ps.z, ps.w};
      const int xi[4] = {pi.x, pi.y, pi.z, pi.w}, xf[4] = {pf.x, pf.y, pf.z, pf.w};
#pragma unroll
      for (int k = 0; k < 4; k++) {
        merge2<IS_MIN>(xv[k], xi[k], xs[k], s.cv.v[k], s.ci.v[k], s.cs.v[k]);
        s.reset[k] |= (xf[k] & 1) != 0;
        s.inv2[k] |= (xf[k] & 2) != 0;
        fl |= xf[k];
      }
    }
  s.any_del = __ballot((fl & 4) != 0) != 0ull;
  finish_target<IS_MIN, LPR, INLINE>(a, v, c, s, lane_on, q, BitMark{chg}, exp_list, exp, cnt);
}

// One workgroup per chunk of a long segment: its waves take a quarter of the events each.  ARRIVE (short launches): the segment's last chunk
// combines it; a launch of its own took 4 to 5 us, most often for nothing.  (With the decision of a target in it the kernel has 105 registers
// instead of 79, four waves a SIMD instead of six; a short launch has a wave or two.)
template <bool IS_MIN, int LPR, bool ARRIVE>
__global__ __launch_bounds__(256) void k_ev_partial(AggArgs a, const int32_t *targets, const int32_t *seg, const uint32_t *ev,
                                                    LongEvents lng, EvPart part, uint64_t *chg, Counters *cnt, int32_t *arrived) {
  constexpr int NW = 4;
  __shared__ float sv[NW][kWave * 4], ss[NW][kWave * 4];
  __shared__ int si[NW][kWave * 4], sf[NW][kWave * 4];
  const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  const int total = ARRIVE ? ieee_mode_off(cnt->v[C_NEVCH]) : cnt->v[C_NEVCH];      // exposed rows are gathered where the target is decided
  for (int ch = blockIdx.x; ch < total; ch += gridDim.x) {
    int e0, e1;
    const int v = targets[long_chunk(lng, ch, seg, e0, e1)];
    const int len = e1 - e0;
    Cached<IS_MIN> c;
    EvAcc<IS_MIN> s;
    reduce_events<IS_MIN, LPR>(a, v, ev, e0 + len * w / NW, e0 + len * (w + 1) / NW, lane_on, q, c, s);
    reduce_groups<IS_MIN, LPR>(s.cv, s.ci, s.cs);
    int fl[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
      fl[k] = reduce_flags<LPR>((int)s.reset[k] | ((int)s.inv2[k] << 1) | ((int)s.any_del << 2));
      sv[w][l * 4 + k] = s.cv.v[k]; si[w][l * 4 + k] = s.ci.v[k]; ss[w][l * 4 + k] = s.cs.v[k]; sf[w][l * 4 + k] = fl[k];
    }
    __syncthreads();
    if (w == 0) {
      if (lane_on && l < LPR) {
        for (int ww = 1; ww < NW; ww++)
#pragma unroll
          for (int k = 0; k < 4; k++) {
            merge2<IS_MIN>(sv[ww][l * 4 + k], si[ww][l * 4 + k], ss[ww][l * 4 + k], s.cv.v[k], s.ci.v[k], s.cs.v[k]);
            fl[k] |= sf[ww][l * 4 + k];
          }
        const int64_t o = (int64_t)ch * a.wd + 4 * q;
#pragma unroll
        for (int k = 0; k < 4; k++) {
          put_part<ARRIVE>(part.v + o + k, s.cv.v[k]); put_part<ARRIVE>(part.i + o + k, s.ci.v[k]);
          put_part<ARRIVE>(part.s + o + k, s.cs.v[k]); put_part<ARRIVE>(part.f + o + k, fl[k]);
        }
      }
      if constexpr (ARRIVE) {
        const int i = lng.owner[ch];
        const LongSeg L = lng.list[i];
        const int n_ev = seg[L.target + 1] - seg[L.target];
        RowSink exp;
        if (last_to_arrive(arrived + i, long_seg_chunks(lng, n_ev)))
          combine_segment<IS_MIN, LPR, true, true>(a, targets, lng, L, n_ev, part, chg, nullptr, exp, cnt);
      }
    }
    __syncthreads();
  }
}

template <bool IS_MIN, int LPR, bool INLINE>
__global__ __launch_bounds__(64) void k_ev_final(AggArgs a, const int32_t *targets, const int32_t *seg, LongEvents lng,
                                                 EvPart part, uint64_t *chg, int32_t *exp_list,
                                                 Counters *cnt) {
  RowSink exp;
  const int n = INLINE ? ieee_mode_off(cnt->v[C_NEVL]) : cnt->v[C_NEVL];
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const LongSeg L = lng.list[i];
    combine_segment<IS_MIN, LPR, INLINE, false>(a, targets, lng, L, seg[L.target + 1] - seg[L.target], part, chg, exp_list, exp, cnt);
  }
  if constexpr (!INLINE) exp.flush(exp_list, &cnt->v[C_NEXP]);
}

// ------------------------------------------------------------------ host side
static int lanes_per_row(int ld) { return ld <= 64 ? 16 : (ld <= 128 ? 32 : 64); }

template <bool IS_MIN, int LPR>
static hipError_t run_big(ink_ctx *c, const AggArgs &a, uint64_t *chg, int compare, int64_t n_rows_max, bool few) {
  const BigParts part{c->big_part_v.as<float>(), c->big_part_i.as<int32_t>(), c->big_part_s.as<float>(), c->big_part_j.as<int32_t>()};
  const bool latency = latency_mode(n_rows_max), arrive = latency && few;
  if (latency) {
    const int slices = big_slices(a.wd);
    const dim3 grid(big_grid(c, a.big_chunks, slices, true));
    if (arrive) hipLaunchKernelGGL((k_big_short<IS_MIN, LPR, true>), grid, dim3(1024), 0, c->stream, a, c->d_cnt, slices, part, chg, compare, c->arrived);
    else hipLaunchKernelGGL((k_big_short<IS_MIN, LPR, false>), grid, dim3(1024), 0, c->stream, a, c->d_cnt, slices, part, chg, compare, c->arrived);
  } else
    hipLaunchKernelGGL((k_big_partial<IS_MIN, LPR>), dim3(big_grid(c, a.big_chunks, 1, false)), dim3(256), 0, c->stream, a, (const Counters *)c->d_cnt, part);
  if (!arrive) hipLaunchKernelGGL((k_big_final<IS_MIN, LPR>), dim3(kBigGrid), dim3(64), 0, c->stream, a, part, chg, compare, c->d_cnt);
  return hipGetLastError();
}

// Workgroups of a recompute launch, whose waves stride over the rows in blocks of up to 16.  The kernel has 94 to 105
// registers, 4 or 5 waves per SIMD: 2048 workgroups at most are on the chip together.  As many as that leave the last long rows as a
// tail, and many more have a row or three a wave and nothing from the blocks.  2048 / 4096 / 8192 / 16384 / 65536 workgroups / a
// wave per row, inference: 625k nodes, 3 layers of 128 floats, 4.16 / 4.07 / 4.00 / 4.00 / 4.11 / 4.54 ms, 200k nodes of 64
// floats .562 / .563 / .543 / .549 / .638 / .641, 100k of 256 .963 / .939 / .931 / .929 / .967 / .963.
constexpr int64_t kFullGrid = 16384;

template <bool IS_MIN, int LPR>
static hipError_t full_t(ink_ctx *c, const AggArgs &a_in, const int32_t *targets, int64_t n_targets, uint64_t *chg) {
  if (n_targets <= 0) return hipSuccess;
  AggArgs a = a_in;
  a.big_deg = big_threshold(n_targets, LPR, kBigDeg);
  int compare = chg != nullptr;
  INK_TRY(ensure_big_buffers(c, a.wd, true));
  a.big = big_rows_of(c, kBigChunk);
  INK_TRY(clear_big_rows(c));
  int64_t blocks = std::min<int64_t>((n_targets + 3) / 4, kFullGrid);
  {
    KernelTimer kt(c, a.layer, INK_K_AGG_FULL);
    hipLaunchKernelGGL((k_agg_full<IS_MIN, LPR>), dim3((unsigned)blocks), dim3(256), 0, c->stream, a, targets, n_targets,
                       (const int32_t *)nullptr, chg, (compare ? FULL_COMPARE | FULL_TALLY : 0), c->d_cnt);
    INK_TRY(hipGetLastError());
  }
  KernelTimer kt(c, a.layer, INK_K_AGG_LONG);
  return run_big<IS_MIN, LPR>(c, a, chg, compare, n_targets, combine_on_arrival(a, false));
}

template <bool IS_MIN, int LPR, bool INLINE>
static hipError_t launch_events(ink_ctx *c, const AggArgs &a, const int32_t *targets, const int32_t *seg, int64_t n_targets,
                                const int32_t *n_targets_dev, const uint32_t *ev, const EventBounds &eb, uint64_t *chg) {
  KernelTimer kt(c, a.layer, INK_K_AGG_EVENTS);
  const bool latency = latency_mode(n_targets);
  // few targets per wave visit while the launch has fewer blocks than the chip has waves to spread them over
  const int ev_block = (int)std::max<int64_t>(1, std::min<int64_t>(kEvBlock, n_targets / 32768));
  int64_t blocks = std::min<int64_t>(((n_targets + ev_block - 1) / ev_block + 3) / 4, INK_EVENT_GRID);
  LongEvents lng = long_events(eb, n_targets);
  INK_TRY(ensure_long_events(c, eb, a.wd, true, &lng));
  int32_t *exp_list = c->exp_list.as<int32_t>();
  hipLaunchKernelGGL((k_agg_events<IS_MIN, LPR, INLINE>), dim3((unsigned)blocks), dim3(256), 0, c->stream, a, targets, seg,
                     n_targets_dev, ev, chg, exp_list, c->d_cnt, ev_block, lng);
  if (eb.max_seg > lng.limit) {      // otherwise no segment can be long
    EvPart part{c->big_part_v.as<float>(), c->big_part_i.as<int32_t>(), c->big_part_s.as<float>(), c->big_part_j.as<int32_t>()};
    const dim3 chunks((unsigned)std::min<int64_t>(long_ev_chunks(lng, eb.n_events), 8192)), rows((unsigned)std::min<int64_t>(long_ev_rows(lng, eb.n_events), 8192));
    if (latency) {                   // its exposed rows are recomputed on the spot (events_t)
      hipLaunchKernelGGL((k_ev_partial<IS_MIN, LPR, true>), chunks, dim3(256), 0, c->stream, a, targets, seg, ev, lng, part, chg, c->d_cnt, c->arrived);
    } else {
      hipLaunchKernelGGL((k_ev_partial<IS_MIN, LPR, false>), chunks, dim3(256), 0, c->stream, a, targets, seg, ev, lng, part, chg, c->d_cnt, c->arrived);
      hipLaunchKernelGGL((k_ev_final<IS_MIN, LPR, INLINE>), rows, dim3(64), 0, c->stream, a, targets, seg, lng, part, chg, exp_list, c->d_cnt);
    }
  }
  return hipGetLastError();
}

// n_targets may be an upper bound: the kernel stops at the device-side count n_targets_dev.
// Exposed rows are listed by the event kernels and recomputed by the two launches after them.
template <bool IS_MIN, int LPR>
static hipError_t events_t(ink_ctx *c, const AggArgs &a_in, const int32_t *targets, const int32_t *seg,
                           int64_t n_targets, const int32_t *n_targets_dev, const uint32_t *ev, const EventBounds &eb,
                           uint64_t *chg) {
  if (n_targets <= 0) return hipSuccess;
  AggArgs a = a_in;
  a.big_deg = big_threshold(n_targets, LPR, kBigDeg);
  INK_TRY(ensure_big_buffers(c, a.wd, true));
  a.big = big_rows_of(c, kBigChunk);
  INK_TRY(c->exp_list.reserve((size_t)n_targets * 4));
  const bool inline_exposed = INK_EV_INLINE_WIDE == 0 ? false : (LPR >= (INK_EV_INLINE_WIDE == 1 ? 64 : (INK_EV_INLINE_WIDE == 2 ? 32 : 16)) || latency_mode(n_targets));
  if (inline_exposed) INK_TRY((launch_events<IS_MIN, LPR, true>(c, a, targets, seg, n_targets, n_targets_dev, ev, eb, chg)));
  else INK_TRY((launch_events<IS_MIN, LPR, false>(c, a, targets, seg, n_targets, n_targets_dev, ev, eb, chg)));
  if (!inline_exposed) {
    KernelTimer kt(c, a.layer, INK_K_AGG_EXPOSED);
    int64_t rb = std::min<int64_t>((n_targets + 3) / 4, latency_mode(n_targets) ? 2048 : 16384);
    hipLaunchKernelGGL((k_agg_full<IS_MIN, LPR>), dim3((unsigned)rb), dim3(256), 0, c->stream, a,
                       (const int32_t *)c->exp_list.as<int32_t>(), n_targets, (const int32_t *)&c->d_cnt->v[C_NEXP], chg,
                       FULL_COMPARE | FULL_COUNT_CHANGED, c->d_cnt);
    INK_TRY(hipGetLastError());
  }
  KernelTimer kt(c, a.layer, INK_K_AGG_LONG);
  return run_big<IS_MIN, LPR>(c, a, chg, 1, n_targets, a.big_chunks <= kArriveChunksEvents);
}

#define DISPATCH(fn, ...)                                                         \
  do {                                                                            \
    int lpr_ = lanes_per_row(a.wd);                                               \
    if (a.is_min) {                                                               \
      if (lpr_ == 16) return fn<true, 16>(__VA_ARGS__);                           \
      if (lpr_ == 32) return fn<true, 32>(__VA_ARGS__);                           \
      return fn<true, 64>(__VA_ARGS__);                                           \
    } else {                                                                      \
      if (lpr_ == 16) return fn<false, 16>(__VA_ARGS__);                          \
      if (lpr_ == 32) return fn<false, 32>(__VA_ARGS__);                          \
      return fn<false, 64>(__VA_ARGS__);                                          \
    }                                                                             \
  } while (0)

hipError_t agg_select_full(ink_ctx *c, const AggArgs &a, const int32_t *targets, int64_t n_targets, uint64_t *chg) {
  DISPATCH(full_t, c, a, targets, n_targets, chg);
}

template <bool IS_MIN, int LPR>
static hipError_t long_rows_t(ink_ctx *c, const AggArgs &a_in, int64_t n_targets, uint64_t *chg) {
  AggArgs a = a_in;
  a.big = big_rows_of(c, kBigChunk);
  KernelTimer kt(c, a.layer, INK_K_AGG_LONG);
  return run_big<IS_MIN, LPR>(c, a, chg, 1, n_targets, a.big_chunks <= kArriveChunksEvents);
}

hipError_t agg_select_long_rows(ink_ctx *c, const AggArgs &a, int64_t n_targets, uint64_t *chg) {
  DISPATCH(long_rows_t, c, a, n_targets, chg);
}

hipError_t agg_select_reserve(ink_ctx *c, AggArgs &a) {
  INK_TRY(ensure_big_buffers(c, a.wd, true));
  a.big = big_rows_of(c, kBigChunk);
  return hipSuccess;
}
int agg_select_long_degree(const AggArgs &a, int64_t n_targets) { return big_threshold(n_targets, lanes_per_row(a.wd), kBigDeg); }

hipError_t agg_select_events(ink_ctx *c, const AggArgs &a, const int32_t *targets, const int32_t *seg,
                             int64_t n_targets, const int32_t *n_targets_dev, const uint32_t *ev_val, const EventBounds &eb,
                             uint64_t *chg) {
  DISPATCH(events_t, c, a, targets, seg, n_targets, n_targets_dev, ev_val, eb, chg);
}

}  // namespace ink
