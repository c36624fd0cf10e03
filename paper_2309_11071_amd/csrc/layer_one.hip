// A small update in one launch of one workgroup: the graph stage (graph_one.h), then layer by layer events, grouping, aggregation, row
// collection, transform and emission, the stages that otherwise take eight to ten launches and a host round trip a layer.  For SAGE layers with
// max or min aggregation.
//
// A single inserted edge has a handful of events a layer; a launch costs about 5 us and a round trip 10 to 15, whatever
// they do.  One workgroup of 16 waves has every stage's result in LDS or in its own CU's cache when the next stage starts.
// What bounds it is the chain of dependent memory accesses and barriers, so
//   * what at most 64 lanes have to do (events and their order, the rows to transform, the emission) is done by one wave
//     with lane exchanges, no barrier inside; counters, sources and records of the layers stand in LDS to the end
//   * the weights of the transform are asked for before the rows that go through it are known, the old rows and the
//     degrees of the emission together with the rows' inputs
//   * all layers are in one launch, so that the code is in the instruction cache from the second on: a layer of its own launch
//     cost 2.2 us between the launches and 1.6 until its first event.
// One edge on 1.25M vertices, three layers of one event each, rows of 128 floats: 18.4 us a layer as launches of workgroup-wide
// stages (transform 6.3, order 1.6, row collection 1.8, emission 1.6, the event 2.3 to 3.7), now 10.8 by the clock in here (event
// 3.0, weights asked for 2.0, rows known .5, inputs, products and stores 3.8, emission .7, order .5, from the layer before .5; rows of 64 floats
// 8.0: 3.5, 1.0, .4, 1.6, .7, .5, .5; graph stage 4.7, records 1.7); a pass of two updates 208 -> 174 us, on 10k vertices, rows of 64, 126 -> 100; of
// 200 distinct updates the median call 96 -> 72 and 48 -> 33.
// Nothing waits for the host: a layer finds its size on the device, and the first one that is too large ends the launch, as does a
// batch that the graph stage leaves to its longer forms.  (The graph stage as a launch in front: 2 us more an update, a pass of two
// 129 -> 125 us on 1.25M vertices, 99.4 -> 97.2 on 10k.)
//   * at most kOneEvents events: 16 waves take 4 us for 16 targets, most of it instructions that the CU's four SIMDs
//     share, so 100 targets (28 us, and 18 to transform them) are no faster than the launches of the general path
//   * exposed rows with many neighbours are recomputed here while they are at most kOneGather floats (2 MB, about
//     20 us at what one CU reads); beyond, the layer stops after its events (kOneEventsDone) and the host continues
//     it with the launches of the general path, which finds the targets, the bitmap and the list of long rows
//     where its own event kernel leaves them
#include <stddef.h>
#include "events.h"
#include "graph_one.h"
#include "select.h"

namespace ink {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kOneThreads = 1024, kOneWaves = kOneThreads / kWave;
constexpr int kOneRows = 2 * kOneEvents;          // rows to transform: targets and sources
constexpr int kSerialWave = kOneWaves - 1;        // does what one wave does: the one with the fewest targets, and weights needed last
constexpr int64_t kOneGather = 512 * 1024;
constexpr int kTileK = 128;                       // part of the input staged in LDS at a time (more than kFewRows rows)
constexpr int kFewRows = 16;                      // up to as many, one tile of 16 rows: all of the input at once
constexpr int kMaxK = 512;                        // (two halves of at most 256)
constexpr int kMergeFloats = 2048;                // columns of partial results held at a time
constexpr int kTileStride = 36;                   // LDS row of a 32-k chunk: even k, odd k, padding (as in xform.hip)
constexpr int kFewStride = kFewRows * kTileStride + 8;   // a chunk of few rows: eight chunks on different banks

struct OneLds {
  uint32_t seed_k[kOneEvents], seed_v[kOneEvents], sk[kOneEvents], sv[kOneEvents];
  int t_list[kOneEvents], t_seg[kOneEvents + 1], t_chg[kOneEvents];
  int rows[kOneRows], flag[kOneRows];
  int F[kOneRows], pref[kOneRows];                // changed sources, prefix of their kept out-edges, start of their blocks
  int64_t off[kOneRows];
  int kept[kOneRows];                             // of the rows to transform: kept out-edges,
  int64_t start[kOneRows];                        // start of the block
  int n_t, n_c, n_f, n_ev, n_del, n_seed;
  Counters cnt;                                   // this layer's; all it bumps are the slots and stripe 0
  HostCounters rec[INK_MAX_LAYERS];
  union {
    float x[kTileK / 32][kOneRows][kTileStride];
    float xf[kMaxK / 32 * kFewStride];
    struct { float v[kMergeFloats]; int i[kMergeFloats]; float s[kMergeFloats]; int j[kMergeFloats]; } m;
    OneGraphLds graph;
  };
  HostCounters graph_rec;
  f4v acc[kOneWaves / 2][kWave];                  // tiles of a product on their way from one wave to the next
};

template <bool IS_MIN> static __shared__ OneLds one_lds;

// A lane's number found anew at every use, and the place in LDS likewise (one_layer, below).
__device__ __forceinline__ int lane_anew() {
  int l = lane_id();
  asm volatile("" : "+v"(l));
  return l;
}
__device__ __forceinline__ OneLds *lds_anew(OneLds *p) {
  typedef __attribute__((address_space(3))) OneLds Lds;
  uint32_t at = (uint32_t)(uint64_t)(Lds *)p;
  asm volatile("" : "+s"(at));
  return (OneLds *)(Lds *)(uint64_t)at;
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x / kWave); }

// The event phase marks a target here.
struct OneMark {
  int *flag;
  __device__ __forceinline__ void operator()(int) const { *flag = 1; }
};

__device__ __forceinline__ int lanes_before(uint64_t mask) { return __popcll(mask & ((1ull << lane_anew()) - 1)); }

// One wave: the layer's nE events in the order of their targets (equal targets in creation order), the distinct targets and
// where each one's events start.
__device__ __forceinline__ void order_events(OneLds &S, const OneUpdate *K, int nE, int n_del, int n_chg, int nF) {
  const int l = lane_anew();
  uint32_t k = 0, v = 0;
  if (l < nE) {
    if (l >= n_del && l < n_del + n_chg) {
      const int c = l - n_del, a = source_of_event(S.pref, nF, c);
      k = (uint32_t)K->out_ids[S.off[a] + (c - S.pref[a])];
      v = (EV_CHG << kEvKindShift) | (uint32_t)S.F[a];
    } else {
      const int i = l < n_del ? l : l - n_chg;
      k = S.seed_k[i]; v = S.seed_v[i];
    }
  }
  int rank = 0;
  for (int j = 0; j < nE; j++) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)k, j);
    rank += (o < k) | ((o == k) & (j < l));
  }
  if (l < nE) { S.sk[rank] = k; S.sv[rank] = v; }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const uint32_t mine = l < nE ? S.sk[l] : 0;
  const bool head = l < nE && (l == 0 || S.sk[l - 1] != mine);
  const uint64_t heads = __ballot(head);
  if (head) { const int at = lanes_before(heads); S.t_list[at] = (int)mine; S.t_seg[at] = l; }
  if (l < kOneEvents) S.t_chg[l] = 0;
  if (l == 0) { const int nT = __popcll(heads); S.t_seg[nT] = nE; S.n_t = nT; S.cnt.v[C_NT] = nT; }
}

// One wave: the rows to transform, ascending: targets whose aggregate changed and sources (their own message changed).
// Lane i < kOneEvents has target i, the other half the sources; both are ascending and distinct.
__device__ __forceinline__ void collect_rows_one(OneLds &S, int nT, int nF) {
  static_assert(2 * kOneEvents == kWave, "a lane per candidate");
  const int l = lane_anew(), f = l - kOneEvents;
  const bool target = l < nT && S.t_chg[l] != 0, source = f >= 0 && f < nF;
  const int id = f < 0 ? (l < nT ? S.t_list[l] : 0) : (source ? S.F[f] : 0);
  const uint64_t targets = __ballot(target);
  int rank = 0;
  bool dup = false;
  for (uint64_t m = targets; m; m &= m - 1) {
    const int o = __builtin_amdgcn_readlane(id, __builtin_ctzll(m));
    rank += o < id;
    dup |= source && o == id;
  }
  const uint64_t sources = __ballot(source && !dup);
  for (uint64_t m = sources; m; m &= m - 1) rank += __builtin_amdgcn_readlane(id, __builtin_ctzll(m)) < id;
  if (target || (source && !dup)) S.rows[rank] = id;
  S.flag[l] = 0;
  if (l == 0) S.n_c = __popcll(targets) + __popcll(sources);
}

// A listed row, recomputed by the whole workgroup: every wave takes a part of the neighbours, then every thread
// merges the waves' results of one column.
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void recompute_long_row(OneLds &S, const AggArgs &a, int v, int nT) {
  constexpr int SLOTS = kMergeFloats / (LPR * 4) < kOneWaves ? kMergeFloats / (LPR * 4) : kOneWaves;
  const int l = lane_anew(), w = wave_id(), t = w * kWave + l, q = l % LPR;
  const bool lane_on = 4 * q < a.wd;
  const int64_t deg = a.in_deg[v];
  F4 bv; I4 bi; F4 sv; I4 si;
  gather_range<IS_MIN, LPR>(a.in_ids + a.in_off[v], deg * w / kOneWaves, deg * (w + 1) / kOneWaves, a.M, a.ldm, lane_on, q,
                            a.nonneg, a.in_asc[v] != 0, bv, bi, sv, si);
  auto put = [&](int slot) {
    if (l < LPR)
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const int i = slot * LPR * 4 + 4 * l + c;
        S.m.v[i] = bv.v[c]; S.m.i[i] = bi.v[c]; S.m.s[i] = sv.v[c]; S.m.j[i] = si.v[c];
      }
  };
  __syncthreads();
  if constexpr (SLOTS < kOneWaves) {
    static_assert(SLOTS >= kOneWaves / 2, "two rounds");
    if (w >= SLOTS) put(w - SLOTS);
    __syncthreads();
    if (w < kOneWaves - SLOTS)
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const int i = w * LPR * 4 + 4 * q + c;
        merge2i<IS_MIN>(S.m.v[i], S.m.i[i], S.m.s[i], S.m.j[i], bv.v[c], bi.v[c], sv.v[c], si.v[c]);
      }
    __syncthreads();
  }
  if (w < SLOTS) put(w);
  __syncthreads();
  bool vchg = false;
  if (t < a.wd) {
    float xv = S.m.v[t], xs = S.m.s[t]; int xi = S.m.i[t], xj = S.m.j[t];
#pragma unroll
    for (int k = 1; k < SLOTS; k++) {
      const int i = k * LPR * 4 + t;
      merge2i<IS_MIN>(S.m.v[i], S.m.i[i], S.m.s[i], S.m.j[i], xv, xi, xs, xj);
    }
    if (xi == 0x7fffffff) { xv = 0.f; xi = -1; xs = worst<IS_MIN>(); }
    if (xj == 0x7fffffff) xj = -1;
    const int64_t o = (int64_t)v * a.ld + t;
    a.UB[o] = xs; a.ARG2[o] = xj;
    vchg = t < a.d && __float_as_uint(a.A[o]) != __float_as_uint(xv);
    a.A[o] = xv; a.ARG[o] = xi;
  }
  const bool any = __syncthreads_or(vchg) != 0;
  if (any && t < nT && S.t_list[t] == v) S.t_chg[t] = 1;
  if (any && t == 0) S.cnt.stripe[0][ST_ACHG]++;
}

// What a row of the transform's output becomes: bias, user term, activation; the row's flag if it changes.
__device__ __forceinline__ void put_output(OneLds &S, const OneLayer &p, int i, int col, float v, float bias, float old) {
  if (p.bias) v = __fadd_rn(v, bias);
  if (p.user) v = __fadd_rn(v, p.user[(int64_t)S.rows[i] * p.ld_user + col]);
  if (p.relu) v = v > 0.f ? v : 0.f;
  if (__float_as_uint(old) != __float_as_uint(v)) { p.out[(int64_t)S.rows[i] * p.ld_out + col] = v; S.flag[i] = 1; }
}

// The SAGE transform of at most kFewRows rows: 16 x 16 tiles of the output with four-k steps, the chain of a tile's products over
// k in order.  A tile of up to 8 that there are has two or more waves: they take blocks of four chunks of 32 k in turn and
// hand the tile on through LDS, so that twice to eight times the weights are under way at once.  load() asks for a wave's
// first block, before the rows are known.
struct FewRows {
  int ct, g, G, n_blk, n_ch;
  bool mine;
  f4v b[4][4];
  __device__ __forceinline__ void issue(const OneLayer &p, int c, int ch) {
    const int l = lane_anew(), kq = l >> 4;                            // kq: which of a step's four k
    const int wl = (kq & 1) * 32 + (ct & 1) * 16 + (l & 15);         // the lane of a weight tile that holds this lane's operands
    const f4v *wp = reinterpret_cast<const f4v *>(p.W) + (int64_t)(ch < n_ch ? ch : n_ch - 1) * 8 * p.Np + (ct / 2) * 256 + wl;
#pragma unroll
    for (int u = 0; u < 4; u++) b[c][u] = wp[u * 64];
  }
  __device__ __forceinline__ void load(const OneLayer &p, int w) {
    const int tiles = p.Np / 16;
    n_ch = p.Kp / 32; n_blk = (n_ch + 3) / 4;
    G = kOneWaves / tiles < n_blk ? kOneWaves / tiles : n_blk;
    g = w / tiles; ct = w - g * tiles; mine = g < G;
    if (mine)
#pragma unroll
      for (int c = 0; c < 4; c++) issue(p, c, 4 * g + c);
  }
  __device__ __forceinline__ void run(OneLds &S, const OneLayer &p, int w, int n_c) {
    const int l = lane_anew(), kq = l >> 4, col = ct * 16 + (l & 15), d4 = xform_self_row(p.d_in);
    const bool ends = mine && g == (n_blk - 1) % G && col < p.n_out;
    // wave w stages row w
    const int64_t row = w < n_c ? S.rows[w] : 0;
    constexpr int XP = kMaxK / (4 * kWave);
    f4v x[XP];
#pragma unroll
    for (int u = 0; u < XP; u++) {
      const int k = 4 * (l + u * kWave);
      if (w < n_c && k < 2 * d4) x[u] = *reinterpret_cast<const f4v *>(k < d4 ? p.a.A + row * p.a.ld + k : p.Hp + row * p.ldh + (k - d4));
    }
    float old[4], bias = 0.f;
    if (ends) {
      if (p.bias) bias = p.bias[col];
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (4 * kq + r < n_c) old[r] = p.out[(int64_t)S.rows[4 * kq + r] * p.ld_out + col];
    }
    if (w < n_c)
#pragma unroll
      for (int u = 0; u < XP; u++) {
        const int k = 4 * (l + u * kWave);
        if (k >= n_ch * 32) continue;
        const int left = k < 2 * d4 ? p.d_in - (k < d4 ? k : k - d4) : 0;    // past it and in the padding of an aggregated row anything may stand
        float *xp = S.xf + k / 32 * kFewStride + w * kTileStride + k % 32 / 4;      // the four k of a step in four groups of 8
        xp[0] = left > 0 ? x[u].x : 0.f; xp[8] = left > 1 ? x[u].y : 0.f; xp[16] = left > 2 ? x[u].z : 0.f; xp[24] = left > 3 ? x[u].w : 0.f;
      }
    __syncthreads();
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    for (int blk = 0; blk < n_blk; blk++) {
      if (mine && blk % G == g) {
        if (blk > 0 && G > 1) acc = S.acc[ct][l];
#pragma unroll
        for (int c = 0; c < 4; c++) {
          if (4 * blk + c >= n_ch) continue;
          const float4 *ap = reinterpret_cast<const float4 *>(S.xf + (4 * blk + c) * kFewStride + (l & 15) * kTileStride + kq * 8);
          const float4 lo = ap[0], hi = ap[1];
          const float a[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          const bool second = kq >> 1;
#pragma unroll
          for (int s = 0; s < 8; s++) {
            const f4v q = b[c][s >> 1];
            const float bw = s & 1 ? (second ? q.w : q.z) : (second ? q.y : q.x);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bw, acc, 0, 0, 0);
          }
          if (blk + G < n_blk) issue(p, c, 4 * (blk + G) + c);
        }
        if (blk + 1 < n_blk && G > 1) S.acc[ct][l] = acc;
      }
      if (blk + 1 < n_blk && G > 1) __syncthreads();
    }
    if (ends)
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (4 * kq + r < n_c) put_output(S, p, 4 * kq + r, col, acc[r], bias, old[r]);
  }
};

// The same of up to kOneRows rows: a wave owns one 32 x 32 tile with two-k steps.  The input passes through LDS 128 k at a
// time, the weights come straight from the L2; both are loaded a block ahead, a chunk's weights into the registers that its
// products have just released.
__device__ __forceinline__ void transform_rows(OneLds &S, const OneLayer &p, int n_c) {
  constexpr int NCH = kTileK / 32, XPT = kOneRows * kTileK / 4 / kOneThreads, NR = 16;
  const int l = lane_anew(), w = wave_id(), t = w * kWave + l;
  const int rt = w / 8, ct = w % 8;                                  // waves w, w + 4, .. share a SIMD: neighbours in ct do not
  const int d4 = xform_self_row(p.d_in), n_ch = p.Kp / 32;
  const int col = ct * 32 + (l & 31);
  const bool mine = ct < p.Np / 32 && rt * 32 < n_c;
  const int kl = (t % (kTileK / 4)) * 4, rl0 = t / (kTileK / 4);     // this thread stages k kl .. kl + 3 of rows rl0, rl0 + 32
  const f4v *wp = reinterpret_cast<const f4v *>(p.W) + (mine ? ct : 0) * 256 + l;
  int64_t row[XPT];
#pragma unroll
  for (int u = 0; u < XPT; u++) row[u] = n_c > 0 ? S.rows[rl0 + u * 32 < n_c ? rl0 + u * 32 : n_c - 1] : 0;
  f4v x[XPT], b[NCH][4];
  auto issue_x = [&](int c0) {
    const int k = c0 * 32 + kl, kk = k < d4 ? k : (k < 2 * d4 ? k - d4 : 0);
#pragma unroll
    for (int u = 0; u < XPT; u++)
      x[u] = *reinterpret_cast<const f4v *>(k < d4 ? p.a.A + row[u] * p.a.ld + kk : p.Hp + row[u] * p.ldh + kk);
  };
  auto issue_w = [&](int c, int ch) {
    const int64_t o = (int64_t)(ch < n_ch ? ch : n_ch - 1) * 8 * p.Np;
#pragma unroll
    for (int u = 0; u < 4; u++) b[c][u] = wp[o + u * 64];
  };
  issue_x(0);
  if (mine)
#pragma unroll
    for (int c = 0; c < NCH; c++) issue_w(c, c);
  typedef float acc_t __attribute__((ext_vector_type(NR)));
  acc_t acc;
#pragma unroll
  for (int r = 0; r < NR; r++) acc[r] = 0.f;
  for (int c0 = 0; c0 < n_ch; c0 += NCH) {
    const int k = c0 * 32 + kl;
    const int left = k < 2 * d4 ? p.d_in - (k < d4 ? k : k - d4) : 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < XPT; u++) {
      const float v0 = left > 0 ? x[u].x : 0.f, v1 = left > 1 ? x[u].y : 0.f, v2 = left > 2 ? x[u].z : 0.f, v3 = left > 3 ? x[u].w : 0.f;
      float *xp = S.x[kl / 32][rl0 + u * 32] + (kl % 32) / 2;        // even k, odd k
      *reinterpret_cast<float2 *>(xp) = make_float2(v0, v2);
      *reinterpret_cast<float2 *>(xp + 16) = make_float2(v1, v3);
    }
    __syncthreads();
    issue_x(c0 + NCH);
    if (mine)
#pragma unroll
      for (int c = 0; c < NCH; c++) {           // chunks past the last: zeros of the input
        const float4 *ap = reinterpret_cast<const float4 *>(&S.x[c][rt * 32 + (l & 31)][(l >> 5) * 16]);
        float4 a4[4];
#pragma unroll
        for (int u = 0; u < 4; u++) a4[u] = ap[u];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[u].x, b[c][u].x, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[u].y, b[c][u].y, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[u].z, b[c][u].z, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[u].w, b[c][u].w, acc, 0, 0, 0);
        }
        if (c0 + NCH < n_ch) issue_w(c, c0 + NCH + c);
      }
  }
  if (!mine || col >= p.n_out) return;
  const float bias = p.bias ? p.bias[col] : 0.f;
  auto slot = [&](int r) { return rt * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); };
  float old[NR];
#pragma unroll
  for (int r = 0; r < NR; r++) {
    const int i = slot(r);
    old[r] = i < n_c ? p.out[(int64_t)S.rows[i] * p.ld_out + col] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < NR; r++)
    if (slot(r) < n_c) put_output(S, p, slot(r), col, acc[r], bias, old[r]);
}

// The targets, one per wave at a time; exposed rows of moderate length on the spot.
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void aggregate_targets(OneLds &S, const AggArgs &a, int w, int nT) {
  const int q = lane_anew() % LPR;
  const bool lane_on = 4 * q < a.wd;
  RowSink exp;
  for (int i = w; i < nT; i += kOneWaves) {
    const int v = __builtin_amdgcn_readfirstlane(S.t_list[i]);
    const int e0 = __builtin_amdgcn_readfirstlane(S.t_seg[i]), e1 = __builtin_amdgcn_readfirstlane(S.t_seg[i + 1]);
    Cached<IS_MIN> c;
    EvAcc<IS_MIN> s;
    reduce_events<IS_MIN, LPR>(a, v, S.sv, e0, e1, lane_on, q, c, s);
    finish_target<IS_MIN, LPR, true>(a, v, c, s, lane_on, q, OneMark{&S.t_chg[i]}, nullptr, exp, &S.cnt);
  }
}

// One layer.  As the body of a loop it would lose everything that is computed from a lane's number or an address in LDS to the
// front of the loop and then to memory, more registers than there are (460 bytes a lane): both are made to look new here.
template <bool IS_MIN>
__device__ __forceinline__ int one_layer(const OneUpdate *K, int layer) {
  OneLds &S = *lds_anew(&one_lds<IS_MIN>);
  const OneLayer p = K->layer[layer - 1];
  const int l = lane_anew(), w = wave_id(), t = w * kWave + l;
  const int n_del = __builtin_amdgcn_readfirstlane(S.n_del), n_seed = __builtin_amdgcn_readfirstlane(S.n_seed);
  const int nF = __builtin_amdgcn_readfirstlane(S.n_f), n_chg = __builtin_amdgcn_readfirstlane(S.n_ev);
  const int nE = ieee_mode_off(__builtin_amdgcn_readfirstlane(n_seed + n_chg));
  if (n_seed == 0 || n_chg > kOneEvents || nE > kOneEvents || nF > kOneEvents) return kOneNothing;
  if (w == kSerialWave) order_events(S, K, nE, n_del, n_chg, nF);
  __syncthreads();
  const int nT = __builtin_amdgcn_readfirstlane(S.n_t);
  if (p.lanes == 16) aggregate_targets<IS_MIN, 16>(S, p.a, w, nT);
  else if (p.lanes == 32) aggregate_targets<IS_MIN, 32>(S, p.a, w, nT);
  else aggregate_targets<IS_MIN, 64>(S, p.a, w, nT);
  __threadfence_block();
  __syncthreads();
  // long exposed rows
  const int n_big = __builtin_amdgcn_readfirstlane(S.cnt.v[C_NBIG]);
  if (n_big > 0) {
    int64_t nb = 0;
    for (int i = 0; i < n_big; i++) nb += p.a.in_deg[p.a.big.list[i]];
    if (nb * p.a.wd > kOneGather) return kOneEventsDone;
    for (int i = 0; i < n_big; i++) {
      const int v = __builtin_amdgcn_readfirstlane(p.a.big.list[i]);
      if (p.lanes == 16) recompute_long_row<IS_MIN, 16>(S, p.a, v, nT);
      else if (p.lanes == 32) recompute_long_row<IS_MIN, 32>(S, p.a, v, nT);
      else recompute_long_row<IS_MIN, 64>(S, p.a, v, nT);
    }
    __threadfence_block();
    __syncthreads();
  }
  // rows to transform; one wave fetches what the emission wants of them while the others have the inputs under way (in a
  // register until then it would have that wave wait for its own stores: .4 us)
  int nC;
  auto await_rows = [&]() {
    __syncthreads();
    nC = __builtin_amdgcn_readfirstlane(S.n_c);
    if (w == kSerialWave && l < nC) { const int u = S.rows[l]; S.kept[l] = kept_out_degree(K->out_deg, K->new_out, u); S.start[l] = K->out_off[u]; }
  };
  if (nT + nF <= kFewRows) {
    FewRows fr;
    if (w == kSerialWave) collect_rows_one(S, nT, nF);       // before its weights, which go into the queue behind all others'
    fr.load(p, w);
    await_rows();
    fr.run(S, p, w, nC);
  } else {
    if (w == kSerialWave) collect_rows_one(S, nT, nF);
    await_rows();
    transform_rows(S, p, nC);
  }
  __syncthreads();
  // changed rows in order, and the events they propagate; the layer's record
  const bool last = layer == K->n_layers;
  HostCounters &R = S.rec[layer - 1];
  if (w == kSerialWave) {
    const bool f = l < nC && S.flag[l] != 0;
    const uint64_t mask = __ballot(f);
    const int at = lanes_before(mask), nF2 = __popcll(mask);
    const int u = f ? S.rows[l] : 0, kept = f ? S.kept[l] : 0;
    int inc = kept;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) { const int y = __shfl_up(inc, o, kWave); inc += l >= o ? y : 0; }
    const int n_ev = last ? 0 : __builtin_amdgcn_readlane(inc, kWave - 1);
    if (f) {
      S.F[at] = u; S.pref[at] = inc - kept; S.off[at] = S.start[l];
      K->f_list[layer & 1][at] = u; K->pref[at] = inc - kept;
    }
    if (l == 0) {
      S.n_f = nF2; S.n_ev = n_ev;
      R.v[C_NC] = nC; R.v[C_NEXT] = nF2; R.v[C_NEV] = n_ev; R.v[C_ONE] = kOneDone;
    }
  } else if (w == 0) {
    if (l < 32 && l != C_NC && l != C_NEXT && l != C_NEV && l != C_ONE) R.v[l] = S.cnt.v[l];
    else if (l >= 32 && l < 32 + ST_N) R.total[l - 32] = S.cnt.stripe[0][l - 32];
    if (l < 32) S.cnt.v[l] = 0;
    else if (l < 32 + ST_N) S.cnt.stripe[0][l - 32] = 0;
  }
  __threadfence_block();
  __syncthreads();
  return kOneDone;
}

template <bool IS_MIN>
__global__ __launch_bounds__(kOneThreads) void k_layers_one(OneUpdate) {
  OneLds &S = one_lds<IS_MIN>;
  // the arguments where the launch has put them: a layer's are found by a running index
  const OneUpdate *K = (const OneUpdate *)__builtin_amdgcn_kernarg_segment_ptr();
  const int l = lane_anew(), w = wave_id(), t = w * kWave + l;
  // which are in host memory: the waves bring a line of 64 bytes each; a stage whose first look there is its own takes .7 us longer
  const int n_layers = K->n_layers;
  for (int i = w * 16; i < (int)(offsetof(OneUpdate, layer) / 4) + n_layers * (int)(sizeof(OneLayer) / 4); i += kOneWaves * 16) {
    const int seen = reinterpret_cast<const int *>(K)[i];
    asm volatile("" : : "s"(seen));
  }
  for (int i = t; i < (int)(sizeof(Counters) / sizeof(int32_t)); i += kOneThreads) ((int32_t *)&S.cnt)[i] = 0;
  graph_one(S.graph, K->graph, S.graph_rec);
  const int n_ins = __builtin_amdgcn_readfirstlane(S.graph_rec.v[C_TMP2]), n_del = __builtin_amdgcn_readfirstlane(S.graph_rec.v[C_TMP3]);     // 0 unless the batch was applied
  if (t < 32) K->g->v[t] = S.graph_rec.v[t];
  if (t < n_ins + n_del) seed_event(t, K->graph.del_s, K->graph.del_d, K->graph.ins_s, K->graph.ins_d, n_del, &S.seed_k[t], &S.seed_v[t]);
  if (t == 0) { S.n_f = 0; S.n_ev = 0; S.n_del = n_del; S.n_seed = n_ins + n_del; }
  __syncthreads();
  int layer = 1, status;
  while ((status = one_layer<IS_MIN>(K, layer)) == kOneDone && layer < n_layers) layer++;
  if (status == kOneDone) {       // the result, and the batch's marks
    const int nF = __builtin_amdgcn_readfirstlane(S.n_f);
    const float *out = K->layer[n_layers - 1].out;
    const int d = K->layer[n_layers - 1].n_out, ld = K->layer[n_layers - 1].ld_out;
    for (int i = t; i < nF * d; i += kOneThreads) {
      const float x = out[(int64_t)S.F[i / d] * ld + i % d];
      K->res[i] = x;
      if (K->h_emb) K->h_emb[i] = x;
    }
    if (K->h_ids && t < nF) K->h_ids[t] = S.F[t];
    const int n_src = S.graph_rec.v[C_OT];
    for (int i = t; i < n_src; i += kOneThreads) K->new_out[K->touched_src[i]] = 0;
  } else {
    if (status == kOneEventsDone) {       // what the general path goes on from
      const int nT = S.n_t;
      if (t < nT) { const int v = S.t_list[t]; K->t_list[t] = v; if (S.t_chg[t]) mark_bit(K->bm, v); }
      for (int i = t; i < (int)(sizeof(Counters) / sizeof(int32_t)); i += kOneThreads) ((int32_t *)K->cnt)[i] = ((const int32_t *)&S.cnt)[i];
    }
    if (t < (int)(sizeof(HostCounters) / sizeof(int32_t))) ((int32_t *)&S.rec[layer - 1])[t] = t == C_ONE ? status : 0;
  }
  // The records end the call, and the result may then be read on any stream: every wave waits here until
  // its own stores have reached the L2 (a barrier alone lets them be under way), and wave 0 writes them back from there.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (w == 0) {
    constexpr int N = sizeof(HostCounters) / sizeof(int32_t);
    if (l < N) reinterpret_cast<int32_t *>(K->h_graph)[l] = reinterpret_cast<const int32_t *>(&S.graph_rec)[l];
    for (int i = l; i < layer * N; i += kWave) {
      const int r = i / N;
      reinterpret_cast<int32_t *>(K->h + r * kRecordBytes)[i - r * N] = reinterpret_cast<const int32_t *>(S.rec)[i];
    }
    __threadfence_system();
    if (l == 0) __hip_atomic_store(reinterpret_cast<uint32_t *>(K->h_graph + sizeof(HostCounters)), K->graph_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    if (l < layer) __hip_atomic_store(reinterpret_cast<uint32_t *>(K->h + l * kRecordBytes + sizeof(HostCounters)), K->seq + l, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

hipError_t layers_one(ink_ctx *c, OneUpdate &p) {
  for (int l = 0; l < p.n_layers; l++) p.layer[l].lanes = p.layer[l].a.wd <= 64 ? 16 : (p.layer[l].a.wd <= 128 ? 32 : 64);
  if (p.layer[0].a.is_min) hipLaunchKernelGGL(k_layers_one<true>, dim3(1), dim3(kOneThreads), 0, c->stream, p);
  else hipLaunchKernelGGL(k_layers_one<false>, dim3(1), dim3(kOneThreads), 0, c->stream, p);
  return hipGetLastError();
}

}  // namespace ink
