// Device code of the selection aggregators (max / min) that more than one kernel uses: the order of values, the
// gather of a row's neighbours, the reduction of a target's events and the decision what they change.
#pragma once
#include "longev.h"
#include "rowload.h"

namespace ink {

struct F4 { float v[4]; };
struct I4 { int v[4]; };

template <bool IS_MIN> __device__ __forceinline__ bool better(float x, float y) {
  return IS_MIN ? (x < y) : (x > y);
}
template <bool IS_MIN> __device__ __forceinline__ float worst() {
  return IS_MIN ? __builtin_huge_valf() : -__builtin_huge_valf();
}
template <bool IS_MIN> __device__ __forceinline__ float best_of(float x, float y) { return better<IS_MIN>(x, y) ? x : y; }
// merge of two disjoint sets, each with its best value, that one's id and its runner-up value sv (best among the others);
// better value first, lower id on equal value
template <bool IS_MIN> __device__ __forceinline__ void merge2(float ov, int oi, float os, float &bv, int &bi, float &sv) {
  float loser;
  if (better<IS_MIN>(ov, bv) || (ov == bv && oi < bi)) { loser = bv; bv = ov; bi = oi; }
  else loser = ov;
  sv = best_of<IS_MIN>(loser, best_of<IS_MIN>(sv, os));
}
// ... and with the runner-up's id si (lowest id among the non-holders that have the value sv)
// asc: the caller feeds ids in ascending order, and equal values leave the entry seen first its place
template <bool IS_MIN>
__device__ __forceinline__ void take2i(float x, int id, bool asc, float &bv, int &bi, float &sv, int &si) {
  const bool first = better<IS_MIN>(x, bv) || (!asc && x == bv && id < bi);
  const bool second = better<IS_MIN>(x, sv) || (!asc && x == sv && id < si);
  const float nsv = first ? bv : (second ? x : sv);
  const int nsi = first ? bi : (second ? id : si);
  bv = first ? x : bv;
  bi = first ? id : bi;
  sv = nsv;
  si = nsi;
}
// merge of the (best, runner-up) pairs of two disjoint sets
template <bool IS_MIN>
__device__ __forceinline__ void merge2i(float ov, int oi, float os, int osi, float &bv, int &bi, float &sv, int &si) {
  float lv; int li;
  if (better<IS_MIN>(ov, bv) || (ov == bv && oi < bi)) { lv = bv; li = bi; bv = ov; bi = oi; }
  else { lv = ov; li = oi; }
  if (better<IS_MIN>(lv, sv) || (lv == sv && li < si)) { sv = lv; si = li; }
  if (better<IS_MIN>(os, sv) || (os == sv && osi < si)) { sv = os; si = osi; }
}

__device__ __forceinline__ float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }


// Reduce (bv, bi) over the lane groups of a wave (groups are LPR lanes wide); every lane ends
// with the result for its 4 dimensions.
template <bool IS_MIN, int LPR> __device__ __forceinline__ void reduce_groups(F4 &bv, I4 &bi, F4 &sv) {
#pragma unroll
  for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
    for (int c = 0; c < 4; c++) {
      float ov = __shfl_xor(bv.v[c], off, kWave);
      int oi = __shfl_xor(bi.v[c], off, kWave);
      float os = __shfl_xor(sv.v[c], off, kWave);
      merge2<IS_MIN>(ov, oi, os, bv.v[c], bi.v[c], sv.v[c]);
    }
  }
}
template <bool IS_MIN, int LPR> __device__ __forceinline__ void reduce_groups_i(F4 &bv, I4 &bi, F4 &sv, I4 &si) {
#pragma unroll
  for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
    for (int c = 0; c < 4; c++) {
      float ov = __shfl_xor(bv.v[c], off, kWave);
      int oi = __shfl_xor(bi.v[c], off, kWave);
      float os = __shfl_xor(sv.v[c], off, kWave);
      int oj = __shfl_xor(si.v[c], off, kWave);
      merge2i<IS_MIN>(ov, oi, os, oj, bv.v[c], bi.v[c], sv.v[c], si.v[c]);
    }
  }
}
template <int LPR> __device__ __forceinline__ int reduce_flags(int fl) {
#pragma unroll
  for (int off = LPR; off < kWave; off <<= 1) fl |= __shfl_xor(fl, off, kWave);
  return fl;
}

// ---- the gather of a recompute: best and runner-up of every dimension, each with its id
// An entry (value x, id) is one double: the bits of x on top, below them the id, coded so that among equal values the
// lower id is the better double.  Doubles are then ordered as entries are selected, and an entry takes three
// instructions (best, the worse of it and the old best, runner-up) next to the one or two to three that make the double;
// value and id compared apart took 12, or 8 where the ids are known to ascend.  The vector instructions were half of the
// time of a recompute (SQ_ACTIVE_INST_VALU: 51 % for short rows, 57 % for long ones) and more where lists no longer
// ascend: 10000 updates on 1.25M nodes and rows of 128 floats 4.42 -> 4.19 ms, on 612k nodes, hubs and rows of 256
// 1.49 -> 1.28, inference of 625k nodes 4.51 -> 4.38.
template <bool IS_MIN> __device__ __forceinline__ double first_of(double x, double y) {
  double r;
  if constexpr (IS_MIN) asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  else asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}
template <bool IS_MIN> __device__ __forceinline__ double last_of(double x, double y) { return first_of<!IS_MIN>(x, y); }
// no entry: worse than any (a finite double beyond those of the infinities)
template <bool IS_MIN> __device__ __forceinline__ constexpr int no_entry() { return IS_MIN ? 0x7fe00000 : (int)0xffe00000; }

// A float NaN from 0x7ff00000 (or 0xfff00000) on is a NaN as a double, too.  It is never best: a kernel that gathers turns
// its IEEE mode off, in which v_max_f64 / v_min_f64 answer a signalling NaN with a quiet one (and the next entry would
// replace that, the best so far gone) instead of the other operand.  But the worse of it and the best is the best, which
// stands as its own runner-up from then on, unless a better entry makes that true: gather_row looks for it in the end.
// The statement passes on a value that the kernel's loop over rows needs and touches nothing else: as a builtin it was a
// write to memory, after which no load was a scalar one (k_agg_events 151 -> 344 us), as a volatile statement it cost k_big_partial
// five registers and a wave per SIMD.
__device__ __forceinline__ int ieee_mode_off(int x) {
  asm("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 9, 1), 0" : "+s"(x));
  return x;
}

template <bool IS_MIN> struct Top2 {
  double b[4], s[4];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int c = 0; c < 4; c++) b[c] = s[c] = __hiloint2double(no_entry<IS_MIN>(), 0);
  }
  __device__ __forceinline__ void take(int c, double e) {
    s[c] = first_of<IS_MIN>(s[c], last_of<IS_MIN>(b[c], e));
    b[c] = first_of<IS_MIN>(b[c], e);
  }
};
// NONNEG: no value has its sign bit set.  Otherwise -0 counts as +0 (which of them an entry has is looked up in the end).
template <bool IS_MIN, bool NONNEG> __device__ __forceinline__ double entry(float x, int id, bool on) {
  int hi, lo;
  if constexpr (NONNEG) { hi = __float_as_int(x); lo = IS_MIN ? id : ~id; }
  else {
    hi = __float_as_int(__fadd_rn(x, 0.f));
    const int sign = hi >> 31;
    lo = IS_MIN ? id ^ sign : ~(id ^ sign);
  }
  return __hiloint2double(on ? hi : no_entry<IS_MIN>(), lo);
}
template <bool IS_MIN> __device__ __forceinline__ int entry_id(double e) {
  const int lo = __double2loint(e), sign = __double2hiint(e) >> 31;
  return IS_MIN ? lo ^ sign : ~(lo ^ sign);
}
template <bool IS_MIN> __device__ __forceinline__ bool is_entry(double e) { return __double2hiint(e) != no_entry<IS_MIN>(); }

// x of this lane and of the lane OFF away, in any order
template <int OFF> __device__ __forceinline__ void both(uint32_t x, uint32_t &p, uint32_t &r) {
  if constexpr (OFF == 32) { const auto t = __builtin_amdgcn_permlane32_swap(x, x, false, false); p = t[0]; r = t[1]; }
  else if constexpr (OFF == 16) { const auto t = __builtin_amdgcn_permlane16_swap(x, x, false, false); p = t[0]; r = t[1]; }
  else { static_assert(OFF == 8, "half a row of 16 lanes"); p = x; r = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false); }
}
template <int OFF> __device__ __forceinline__ void both(double x, double &p, double &r) {
  uint32_t pl, rl, ph, rh;
  both<OFF>((uint32_t)__double2loint(x), pl, rl);
  both<OFF>((uint32_t)__double2hiint(x), ph, rh);
  p = __hiloint2double((int)ph, (int)pl);
  r = __hiloint2double((int)rh, (int)rl);
}
template <bool IS_MIN, int OFF> __device__ __forceinline__ void merge_lanes(Top2<IS_MIN> &t) {
#pragma unroll
  for (int c = 0; c < 4; c++) {
    double b0, b1, s0, s1;
    both<OFF>(t.b[c], b0, b1);
    both<OFF>(t.s[c], s0, s1);
    t.b[c] = first_of<IS_MIN>(b0, b1);
    t.s[c] = first_of<IS_MIN>(first_of<IS_MIN>(s0, s1), last_of<IS_MIN>(b0, b1));
  }
}
// over the lane groups of a wave: every lane ends with the result for its 4 dimensions
template <bool IS_MIN, int LPR> __device__ __forceinline__ void merge_groups(Top2<IS_MIN> &t) {
  if constexpr (LPR <= 8) merge_lanes<IS_MIN, 8>(t);
  if constexpr (LPR <= 16) merge_lanes<IS_MIN, 16>(t);
  if constexpr (LPR <= 32) merge_lanes<IS_MIN, 32>(t);
}

// U rows per lane group; FULL: every slot is a row
template <bool IS_MIN, int LPR, bool NONNEG, int U, bool FULL>
__device__ __forceinline__ void take_batch(const RowTable<LPR> &tab, int win, int it, int cnt, Top2<IS_MIN> &t) {
  constexpr int G = kWave / LPR;
  int id[U];
  float4 row[U];
  tab.template load_batch<U>(win, it, FULL ? kWave - 1 : cnt - 1, id, row);
#pragma unroll
  for (int u = 0; u < U; u++) {
    const float x[4] = {row[u].x, row[u].y, row[u].z, row[u].w};
    const bool on = FULL || it + u * G + tab.g < cnt;
#pragma unroll
    for (int c = 0; c < 4; c++) t.take(c, entry<IS_MIN, NONNEG>(x[c], id[u], on));
  }
}

// Best and runner-up of the n rows ids[..] by the whole wave, per lane group; win: the first ids, one per lane
template <bool IS_MIN, int LPR, bool NONNEG>
__device__ __forceinline__ void gather_top2(const int32_t *ids, int n, int win, const RowTable<LPR> &tab, Top2<IS_MIN> &t) {
  constexpr int G = kWave / LPR;
  constexpr int U = LPR == 8 ? INK_U_SEL8 : LPR == 16 ? INK_U_SEL16 : (LPR == 32 ? INK_U_SEL32 : INK_U_SEL64);
  t.init();
  for (int jb = 0; jb < n; jb += kWave) {
    const int cnt = n - jb < kWave ? n - jb : kWave;
    const int next = ids_ahead(ids, jb + kWave, n);
    for (int it = 0; it < cnt;) {
      const int left = cnt - it;
      if (left >= G * U) { take_batch<IS_MIN, LPR, NONNEG, U, true>(tab, win, it, cnt, t); it += G * U; }
      else if (left > G * U / 4) { take_batch<IS_MIN, LPR, NONNEG, U / 2, false>(tab, win, it, cnt, t); it += G * U / 2; }
      else { take_batch<IS_MIN, LPR, NONNEG, U / 4, false>(tab, win, it, cnt, t); it += G * U / 4; }
    }
    win = next;
  }
}

// The same entry by entry, for rows in whose result an infinity or a NaN stands that the doubles do not order as values
// are: a NaN takes no place, the worst infinity takes one only in lists not known to be ascending (asc).
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void gather_slow(const int32_t *ids, int n, const RowTable<LPR> &tab, bool asc,
                                            F4 &bv, I4 &bi, F4 &sv, I4 &si) {
#pragma unroll
  for (int c = 0; c < 4; c++) { bv.v[c] = worst<IS_MIN>(); bi.v[c] = 0x7fffffff; sv.v[c] = worst<IS_MIN>(); si.v[c] = 0x7fffffff; }
#pragma unroll 1
  for (int j = tab.g; j < n; j += kWave / LPR) {
    const int id = ids[j];
    const float4 r = tab.load(id);
    const float x[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int c = 0; c < 4; c++) take2i<IS_MIN>(x[c], id, asc, bv.v[c], bi.v[c], sv.v[c], si.v[c]);
  }
  reduce_groups_i<IS_MIN, LPR>(bv, bi, sv, si);
}

// Selection over the n neighbours ids[..] of one row, by the whole wave; win: ids_ahead(ids, 0, n).  On return every lane
// holds the best and the runner-up (value, id) of its 4 dimensions; (worst, INT_MAX) where there is none.  n, nonneg and
// asc are wave-uniform: the table has no value with its sign bit set; the ids are ascending.
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void gather_row(const int32_t *ids, int n, int win, const float *M, int ldm, bool lane_on, int q,
                                           bool nonneg, bool asc, F4 &bv, I4 &bi, F4 &sv, I4 &si) {
  const RowTable<LPR> tab(M, ldm, lane_on, q);
  Top2<IS_MIN> t;
  if (nonneg) gather_top2<IS_MIN, LPR, true>(ids, n, win, tab, t);
  else gather_top2<IS_MIN, LPR, false>(ids, n, win, tab, t);
  merge_groups<IS_MIN, LPR>(t);
  bool odd = false, zero = false;
#pragma unroll
  for (int c = 0; c < 4; c++) {
    const double e[2] = {t.b[c], t.s[c]};
    float v[2]; int id[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const int hi = __double2hiint(e[k]);
      const bool has = is_entry<IS_MIN>(e[k]);
      v[k] = has ? __int_as_float(hi) : worst<IS_MIN>();
      id[k] = has ? entry_id<IS_MIN>(e[k]) : 0x7fffffff;
      odd |= has && !better<IS_MIN>(v[k], worst<IS_MIN>());
      zero |= hi == 0;
    }
    bv.v[c] = v[0]; bi.v[c] = id[0]; sv.v[c] = v[1]; si.v[c] = id[1];
  }
  if (!nonneg) {
    // An entry as its own runner-up: there is a NaN (ReLU leaves none).  Here and without a look whether there is an entry, which more
    // than one neighbour makes true but for NaNs: in the loop above it was 3 % of k_agg_full (200k nodes, rows of 100 floats, 169 -> 174 us).
#pragma unroll
    for (int c = 0; c < 4; c++) odd |= n > 1 && __double2loint(t.s[c]) == __double2loint(t.b[c]);
    // The sign of a zero, from the row it came from, which is in the L2 still.  Features with many zeros pay for it, inference
    // against features without: 625k nodes and rows of 128 floats 1.24 ms against 1.22, 200k and 64 floats .298 against .285.
    if (__ballot(zero && lane_on) != 0ull) {
      const float *m = M + 4 * q;
#pragma unroll
      for (int c = 0; c < 4; c++)
        if (lane_on) {
          if (bv.v[c] == 0.f) bv.v[c] = m[(int64_t)bi.v[c] * ldm + c];
          if (sv.v[c] == 0.f) sv.v[c] = m[(int64_t)si.v[c] * ldm + c];
        }
    }
  }
  if (__ballot(odd && lane_on) != 0ull) gather_slow<IS_MIN, LPR>(ids, n, tab, asc, bv, bi, sv, si);
}
// ... over ids[j0 .. j1)
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void gather_range(const int32_t *ids, int64_t j0, int64_t j1, const float *M, int ldm, bool lane_on,
                                             int q, bool nonneg, bool asc, F4 &bv, I4 &bi, F4 &sv, I4 &si) {
  const int n = __builtin_amdgcn_readfirstlane((int)(j1 - j0));
  gather_row<IS_MIN, LPR>(ids + j0, n, ids_ahead(ids + j0, 0, n), M, ldm, lane_on, q, nonneg, asc, bv, bi, sv, si);
}

// 16 bytes of a table row that nothing reads again before it has left the caches: past them, so that they keep the
// gathered rows.
template <typename T> __device__ __forceinline__ void store_past(T *p, const T v[4]) {
  typedef T t4 __attribute__((ext_vector_type(4)));
  const t4 x = {v[0], v[1], v[2], v[3]};
  __builtin_nontemporal_store(x, reinterpret_cast<t4 *>(p));
}

struct RowOut {
  float *A; int32_t *ARG; float *UB; int32_t *ARG2; int ld; int d;
};

// Writes (bv, bi) as the new aggregated row of v if it differs from what is stored; returns
// (wave-uniform) whether any VALUE of the first d dimensions changed bitwise.
template <int LPR>
__device__ __forceinline__ bool store_row(const RowOut &o, int v, bool lane_on, int q, const F4 &bv,
                                          const I4 &bi, const F4 &sv, const I4 &si, bool have_old, const F4 &ov,
                                          const I4 &oi) {
  const int l = lane_id();
  bool writer = lane_on && l < LPR;
  bool vchg = false, ichg = false;
  if (writer) {    // bound and runner-up are rewritten unconditionally (they never decide whether a row "changed")
    store_past(o.UB + (int64_t)v * o.ld + 4 * q, sv.v);
    store_past(o.ARG2 + (int64_t)v * o.ld + 4 * q, si.v);
  }
  if (writer) {
    F4 cv = ov; I4 ci = oi;
    if (!have_old) {
      float4 a = ld4(o.A + (int64_t)v * o.ld + 4 * q);
      int4 b = *reinterpret_cast<const int4 *>(o.ARG + (int64_t)v * o.ld + 4 * q);
      cv.v[0] = a.x; cv.v[1] = a.y; cv.v[2] = a.z; cv.v[3] = a.w;
      ci.v[0] = b.x; ci.v[1] = b.y; ci.v[2] = b.z; ci.v[3] = b.w;
    }
#pragma unroll
    for (int c = 0; c < 4; c++) {
      if (4 * q + c < o.d) vchg |= __float_as_uint(cv.v[c]) != __float_as_uint(bv.v[c]);
      ichg |= ci.v[c] != bi.v[c];
    }
    if (vchg || ichg) {
      *reinterpret_cast<float4 *>(o.A + (int64_t)v * o.ld + 4 * q) = make_float4(bv.v[0], bv.v[1], bv.v[2], bv.v[3]);
      *reinterpret_cast<int4 *>(o.ARG + (int64_t)v * o.ld + 4 * q) = make_int4(bi.v[0], bi.v[1], bi.v[2], bi.v[3]);
    }
  }
  return __ballot(vchg) != 0ull;
}

// no in-neighbours: alpha = 0, arg = -1; fewer than two: no runner-up
template <bool IS_MIN>
__device__ __forceinline__ void finish_empty(F4 &bv, I4 &bi, F4 &sv, I4 &si) {
#pragma unroll
  for (int c = 0; c < 4; c++) {
    if (bi.v[c] == 0x7fffffff) { bv.v[c] = 0.f; bi.v[c] = -1; sv.v[c] = worst<IS_MIN>(); }
    if (si.v[c] == 0x7fffffff) si.v[c] = -1;
  }
}

__device__ __forceinline__ void mark_bit(uint64_t *bm, int v) {
  atomicOr((unsigned long long *)&bm[v >> 6], 1ull << (v & 63));
}
struct BitMark {
  uint64_t *bm;
  __device__ __forceinline__ void operator()(int v) const { mark_bit(bm, v); }
};

// ------------------------------------------------------------------ event-driven incremental update
// Events of a target arrive as one contiguous segment of ev_val (kind << 30 | source id).
//   DEL  (edge u -> v removed):    dimension i needs a reset iff arg[v][i] == u
//   ADD  (edge s -> v inserted):   (m_s[i], s) is a candidate
//   CHG  (message of u changed, edge kept): (m_u[i], u) is a candidate; if u held dimension i and
//        its value got worse the dimension needs a reset, if equal nothing happened there
// A reset dimension is covered when the best candidate strictly beats the old value, otherwise
// the row is exposed and recomputed from its whole current neighbourhood.
//
// A target has a handful of events, and what bounds the kernel is the traffic of its random row
// accesses (one source row per event, four cached rows per target, up to four written back), not
// the latency of one target's chain: keeping the next targets' rows in flight across targets
// (register double-buffering, event words staged in LDS) was measured and bought nothing, so the
// loop is the plain one.

#ifndef INK_EV_U
#define INK_EV_U 2                 // source rows in flight per lane group and batch
#endif
constexpr uint32_t kEvNone = 0xFFFFFFFFu;     // no event: its kind bits name no kind

template <bool IS_MIN> struct Cached {        // this lane's four dimensions of a target's cached row
  F4 ov; I4 oi; F4 ou; I4 o2;                 // value, holder, bound on the other neighbours, runner-up id or -1
};
template <bool IS_MIN>
__device__ __forceinline__ void load_cached(const AggArgs &a, int v, bool lane_on, int q, Cached<IS_MIN> &k) {
#pragma unroll
  for (int c = 0; c < 4; c++) { k.ov.v[c] = 0.f; k.oi.v[c] = -1; k.ou.v[c] = worst<IS_MIN>(); k.o2.v[c] = -1; }
  if (lane_on) {
    const int64_t o = (int64_t)v * a.ld + 4 * q;
    const float4 x = ld4(a.A + o);
    const int4 y = *reinterpret_cast<const int4 *>(a.ARG + o);
    const float4 z = ld4(a.UB + o);
    const int4 y2 = *reinterpret_cast<const int4 *>(a.ARG2 + o);
    k.ov.v[0] = x.x; k.ov.v[1] = x.y; k.ov.v[2] = x.z; k.ov.v[3] = x.w;
    k.oi.v[0] = y.x; k.oi.v[1] = y.y; k.oi.v[2] = y.z; k.oi.v[3] = y.w;
    k.ou.v[0] = z.x; k.ou.v[1] = z.y; k.ou.v[2] = z.z; k.ou.v[3] = z.w;
    k.o2.v[0] = y2.x; k.o2.v[1] = y2.y; k.o2.v[2] = y2.z; k.o2.v[3] = y2.w;
  }
}

// U events per lane group: their words and, unless they are deletions, their sources' message rows
template <int U> struct EvBatch { uint32_t code[U]; float4 row[U]; };

// events it + u G + g (u < U) of the window `mine` (lane j holds event j, cntw of them are real)
template <bool IS_MIN, int LPR, int U>
__device__ __forceinline__ void issue_batch(const AggArgs &a, uint32_t mine, int it, int cntw, bool lane_on, int q,
                                            EvBatch<U> &b) {
  constexpr int G = kWave / LPR;
  const float W = worst<IS_MIN>();
  const int g = lane_id() / LPR;
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int k = it + u * G + g;
    const uint32_t x = __shfl(mine, k < kWave ? k : 0, kWave);
    const bool valid = k < cntw && lane_on;
    b.code[u] = valid ? x : kEvNone;
    b.row[u] = make_float4(W, W, W, W);        // an event without a row offers the worst value: it never wins
    if (valid && (x >> kEvKindShift) != EV_DEL) b.row[u] = ld4(a.M + (int64_t)(x & kEvIdMask) * a.ldm + 4 * q);
  }
}

template <bool IS_MIN> struct EvAcc {
  F4 cv; I4 ci; F4 cs;       // best candidate, its source, runner-up candidate value
  bool reset[4];             // per dimension: the holder left or got worse
  bool inv2[4];              // per dimension: the recorded runner-up left or changed its message
  bool any_del;              // wave-uniform: the segment cancels something (a removed edge or a changed source)
  __device__ __forceinline__ void init() {
    any_del = false;
#pragma unroll
    for (int c = 0; c < 4; c++) {
      cv.v[c] = worst<IS_MIN>(); ci.v[c] = 0x7fffffff; cs.v[c] = worst<IS_MIN>();
      reset[c] = false; inv2[c] = false;
    }
  }
};

// Written without branches: the per-lane conditions become wave masks in scalar registers and the
// updates selects and min / max (this loop runs once per event and lane group and is half of the
// kernel's vector instructions, and the kernel's time follows their number).  What keeps it short:
//  * an event without a row (a removed edge, an empty slot) carries the worst value, so it needs no
//    mask of its own: it never becomes a candidate, and as "new value of the holder" it is a reset;
//  * an inserted edge cannot name the old holder or runner-up (it was no neighbour), so the id
//    tests need no kind;
//  * the runner-up among the candidates is the middle one of (r, cv, cs), whichever of the first two
//    wins, because cs never beats cv;
//  * TIES false (wave-uniform): the candidates so far are changed sources in ascending id order (the order the
//    events are created in), so on equal values the earlier one keeps the dimension and the id
//    comparison is skipped.  The caller sets TIES from a target's first inserted edge on.
// v_med3_f32 as it is: no NaN reaches it (inputs are finite, the sentinels are infinities).
__device__ __forceinline__ float vmed3(float a, float b, float c) {
  float d;
  asm("v_med3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

template <bool IS_MIN, int U>
__device__ __forceinline__ void consume_batch(const EvBatch<U> &b, const Cached<IS_MIN> &k, EvAcc<IS_MIN> &s, bool TIES) {
#pragma unroll
  for (int u = 0; u < U; u++) {
    const uint32_t x = b.code[u];
    const int id = (int)(x & kEvIdMask);               // "no event": an id no node has
    const float r[4] = {b.row[u].x, b.row[u].y, b.row[u].z, b.row[u].w};
    bool first[4];
#pragma unroll
    for (int c = 0; c < 4; c++) {      // & and | on purpose: no short-circuit, no branch
      s.inv2[c] |= k.o2.v[c] == id;
      s.reset[c] |= (k.oi.v[c] == id) & better<IS_MIN>(k.ov.v[c], r[c]);
      first[c] = better<IS_MIN>(r[c], s.cv.v[c]);
    }
    if (TIES) {
      asm volatile("");                // keeps this a (wave-uniform) branch: only targets with an inserted edge pay for it
      const uint32_t kind = x >> kEvKindShift;
      const bool has_row = (kind == EV_ADD) | (kind == EV_CHG);
#pragma unroll
      for (int c = 0; c < 4; c++) first[c] |= has_row & (r[c] == s.cv.v[c]) & (id < s.ci.v[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; c++) {
      s.cs.v[c] = vmed3(r[c], s.cv.v[c], s.cs.v[c]);
      s.cv.v[c] = first[c] ? r[c] : s.cv.v[c];
      s.ci.v[c] = first[c] ? id : s.ci.v[c];
    }
  }
}

// Rows that a launch lists for the kernels after it.  A list has one global counter, and a wave that
// takes a slot waits for its answer: 131 k exposed rows took 0.4 of 2.4 ms (655 k targets) that way.
// So a wave keeps its rows in a register, one per lane, and takes their slots together at its end or
// when the register is full.
struct RowSink {
  int n = 0, id = 0;
  __device__ __forceinline__ void flush(int32_t *list, int32_t *n_list) {
    if (n == 0) return;
    int base = 0;
    if (lane_id() == 0) base = atomicAdd(n_list, n);
    base = __builtin_amdgcn_readfirstlane(base);
    if (lane_id() < n) list[base + lane_id()] = id;
    n = 0;
  }
  __device__ __forceinline__ void push(int v, int32_t *list, int32_t *n_list) {     // whole wave, wave-uniform arguments
    if (lane_id() == n) id = v;
    if (++n == kWave) flush(list, n_list);
  }
};

// The decision for target v once its events are reduced (the lane groups still hold partial
// results), the recompute of an exposed row of moderate length, and the store.  `mark` notes a change of its value.
template <bool IS_MIN, int LPR, bool INLINE, class Mark>
__device__ __forceinline__ void finish_target(const AggArgs &a, int v, const Cached<IS_MIN> &k, EvAcc<IS_MIN> &s,
                                              bool lane_on, int q, const Mark &mark, int32_t *exp_list,
                                              RowSink &exp, Counters *cnt) {
  const int l = lane_id();
  const F4 &ov = k.ov; const I4 &oi = k.oi; const F4 &ou = k.ou; const I4 &o2 = k.o2;
  F4 &cv = s.cv; I4 &ci = s.ci; F4 &cs = s.cs;
  // combine the lane groups: the flags travel packed in one register
  unsigned fl = 0u;
#pragma unroll
  for (int c = 0; c < 4; c++) fl |= ((unsigned)s.reset[c] << c) | ((unsigned)s.inv2[c] << (4 + c));
  fl = (unsigned)reduce_flags<LPR>((int)fl);
  bool reset[4], inv2[4];
#pragma unroll
  for (int c = 0; c < 4; c++) { reset[c] = (fl >> c) & 1u; inv2[c] = (fl >> (4 + c)) & 1u; }
  reduce_groups<IS_MIN, LPR>(cv, ci, cs);
  // Per dimension: (nv, ni) new value and holder, nu new bound on the others, n2 the other neighbour
  // that has exactly the value nu (lowest such id) where that is certain, else -1.  A recorded
  // runner-up is trusted only while it neither left nor changed; it lets a reset that no candidate
  // covers be settled by promotion instead of a recompute, once per dimension between recomputes.
  F4 nv = ov; I4 ni = oi; F4 nu = ou; I4 n2;
  bool exposed = false;
  bool vchg = false, ichg = false, uchg = false;      // what of the cached row changes (short live ranges: per dimension)
#pragma unroll
  for (int c = 0; c < 4; c++) {
    const bool has_cand = ci.v[c] != 0x7fffffff;
    const int r2 = inv2[c] ? -1 : o2.v[c];               // runner-up still known to hold ou
    const bool ou_beats_cs = better<IS_MIN>(ou.v[c], cs.v[c]);
    n2.v[c] = r2;
    if (oi.v[c] < 0) {                       // no neighbours before this batch
      n2.v[c] = -1;
      if (has_cand) { nv.v[c] = cv.v[c]; ni.v[c] = ci.v[c]; nu.v[c] = cs.v[c]; }
    } else if (reset[c]) {
      // the holder left or got worse (then its new value is one of the candidates); every other
      // old neighbour is bounded by ou, and those that reach ou have ids above r2
      if (has_cand && better<IS_MIN>(cv.v[c], ou.v[c])) {
        nv.v[c] = cv.v[c]; ni.v[c] = ci.v[c]; nu.v[c] = best_of<IS_MIN>(ou.v[c], cs.v[c]);
        n2.v[c] = ou_beats_cs ? r2 : -1;
      } else if (r2 >= 0 && has_cand && cv.v[c] == ou.v[c] && ci.v[c] < r2) {
        nv.v[c] = cv.v[c]; ni.v[c] = ci.v[c];            // candidate and runner-up tie: the lower id holds
        n2.v[c] = ou_beats_cs ? r2 : -1;                 // nu stays ou, held by r2
      } else if (r2 >= 0) {
        nv.v[c] = ou.v[c]; ni.v[c] = r2;                 // the runner-up takes over; who follows is not known
        n2.v[c] = -1;                                    // nu stays ou: it bounds the old others and every candidate
      } else exposed = true;
    } else if (has_cand) {
      if (ci.v[c] == oi.v[c]) {              // the holder itself, unchanged or better at this dimension
        nv.v[c] = cv.v[c]; nu.v[c] = best_of<IS_MIN>(ou.v[c], cs.v[c]);
        n2.v[c] = ou_beats_cs ? r2 : -1;
      } else if (better<IS_MIN>(cv.v[c], ov.v[c]) || (cv.v[c] == ov.v[c] && ci.v[c] < oi.v[c])) {
        nv.v[c] = cv.v[c]; ni.v[c] = ci.v[c];          // the old holder joins the others
        nu.v[c] = best_of<IS_MIN>(best_of<IS_MIN>(ou.v[c], ov.v[c]), cs.v[c]);
        n2.v[c] = -1;
        if (better<IS_MIN>(ov.v[c], cs.v[c])) {        // it is their best unless the old runner-up ties with it
          if (better<IS_MIN>(ov.v[c], ou.v[c])) n2.v[c] = oi.v[c];
          else if (r2 >= 0) n2.v[c] = oi.v[c] < r2 ? oi.v[c] : r2;
        }
      } else {
        nu.v[c] = best_of<IS_MIN>(ou.v[c], cv.v[c]);
        n2.v[c] = better<IS_MIN>(ou.v[c], cv.v[c]) ? r2 : -1;
      }
    }
    vchg |= (4 * q + c < a.d) & (__float_as_uint(ov.v[c]) != __float_as_uint(nv.v[c]));
    ichg |= oi.v[c] != ni.v[c];
    uchg |= (__float_as_uint(ou.v[c]) != __float_as_uint(nu.v[c])) | (o2.v[c] != n2.v[c]);
  }
  exposed = __ballot(exposed && lane_on) != 0ull;
  if (a.count_cond) {   // condition of this target (Sec. 2.5.1; the distribution shown in Sec. 5.2)
    bool rs = (reset[0] || reset[1] || reset[2] || reset[3]) && lane_on;
    bool any_reset = __ballot(rs) != 0ull;
    bool dl = s.any_del;
    if (l == 0 && !exposed) {
      int which = !dl ? ST_NODEL : (!any_reset ? ST_NOEFFECT : ST_COVERED);
      atomicAdd(&cnt->stripe[blockIdx.x % kStripes][which], 1ull);
    }
  }
  if (exposed) {
    const int deg = __builtin_amdgcn_readfirstlane(a.in_deg[v]);
    if (l == 0) {
      if (a.count_cond) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_EXPOSED], 1ull);
      atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_REGATHER], (unsigned long long)deg);
    }
    if constexpr (INLINE) {      // rows of moderate length are recomputed on the spot
      if (deg <= a.big_deg) {
        F4 bv; I4 bi; F4 sv; I4 si;
        gather_range<IS_MIN, LPR>(a.in_ids + a.in_off[v], 0, deg, a.M, a.ldm, lane_on, q, a.nonneg, a.in_asc[v] != 0, bv, bi, sv, si);
        finish_empty<IS_MIN>(bv, bi, sv, si);
        RowOut o{a.A, a.ARG, a.UB, a.ARG2, a.ld, a.d};
        const bool ch = store_row<LPR>(o, v, lane_on, q, bv, bi, sv, si, true, ov, oi);
        if (ch && l == 0) { mark(v); if (a.count_cond) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_ACHG], 1ull); }
        return;
      }
    }
    // recomputed by the kernels that follow: long rows chunk by chunk, the others one wave per row
    if (l == 0) {
      if (deg > a.big_deg) {
        list_big_row(a.big, cnt, v, deg);
        atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_REGATHER_LONG], (unsigned long long)deg);
      }
    }
    if (!INLINE && deg <= a.big_deg) exp.push(v, exp_list, &cnt->v[C_NEXP]);
    return;
  }
  // each half of the cached row is rewritten only if it changed: most targets keep their bound and
  // runner-up, many keep value and holder
  const bool writer = lane_on && l < LPR;
  vchg &= writer;
  if (writer) {
    if (vchg || ichg) {
      *reinterpret_cast<float4 *>(a.A + (int64_t)v * a.ld + 4 * q) = make_float4(nv.v[0], nv.v[1], nv.v[2], nv.v[3]);
      *reinterpret_cast<int4 *>(a.ARG + (int64_t)v * a.ld + 4 * q) = make_int4(ni.v[0], ni.v[1], ni.v[2], ni.v[3]);
    }
    if (uchg) {
      *reinterpret_cast<float4 *>(a.UB + (int64_t)v * a.ld + 4 * q) = make_float4(nu.v[0], nu.v[1], nu.v[2], nu.v[3]);
      *reinterpret_cast<int4 *>(a.ARG2 + (int64_t)v * a.ld + 4 * q) = make_int4(n2.v[0], n2.v[1], n2.v[2], n2.v[3]);
    }
  }
  const bool ch = __ballot(vchg) != 0ull;
  if (ch && l == 0) { mark(v); if (a.count_cond) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][ST_ACHG], 1ull); }
}

// The events [e0, e1) of target v into s and the target's cached row into c; every lane group keeps
// its own partial result.
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void reduce_events(const AggArgs &a, int v, const uint32_t *ev, int e0, int e1, bool lane_on, int q,
                                              Cached<IS_MIN> &c, EvAcc<IS_MIN> &s) {
  constexpr int G = kWave / LPR;
  constexpr int U = INK_EV_U;
  const int l = lane_id();
  load_cached<IS_MIN>(a, v, lane_on, q, c);
  s.init();
  bool ties = false;
  for (int eb = e0; eb < e1; eb += kWave) {
    const int ee = eb + l;
    const uint32_t mine = ee < e1 ? ev[ee] : kEvNone;
    const int cntw = e1 - eb < kWave ? e1 - eb : kWave;
    // wave-uniform: from the first inserted edge of the window on, equal values are settled by id
    const uint64_t adds = __ballot(ee < e1 && (mine >> kEvKindShift) == EV_ADD);
    s.any_del |= __ballot(ee < e1 && (mine >> kEvKindShift) != EV_ADD) != 0ull;
    const int first_add = adds ? __builtin_ctzll(adds) : kWave;
    for (int it = 0; it < cntw; it += G * U) {
      EvBatch<U> bx;
      issue_batch<IS_MIN, LPR, U>(a, mine, it, cntw, lane_on, q, bx);
      ties |= it + G * U > first_add;
      consume_batch<IS_MIN, U>(bx, c, s, ties);
    }
  }
}

}  // namespace ink
