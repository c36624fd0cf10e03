// A whole layer of a small update in one workgroup: events, grouping, aggregation, row collection, transform and
// emission, the stages that otherwise take eight to ten launches and a host round trip.  For SAGE layers with max or
// min aggregation.
//
// A single inserted edge has a handful of events a layer; a launch costs about 5 us and a round trip 10 to 15, whatever
// they do, and the separate stages of such a layer took 55 us of little else.  One workgroup of 16 waves has every
// stage's result in LDS or in its own CU's cache when the next stage starts; it takes 14 us for one event on rows of
// 128 floats (of which the transform 6, the event 2 to 4) and 12 to 30 for five, bound by the chain of dependent memory
// accesses.  The layers of an update are enqueued behind each other and behind the graph stage without waiting
// for the host: a layer reads its size on the device and does nothing if the layer before did not finish or if it is
// too large itself.  One edge on 1.25M vertices, three layers of one event each: 255 -> 90 us an update.
//   * at most kOneEvents events: 16 waves take 4 us for 16 targets, most of it instructions that the CU's four SIMDs
//     share, so 100 targets (28 us, and 18 to transform them) are no faster than the launches of the general path
//   * exposed rows with many neighbours are recomputed here while they are at most kOneGather floats (2 MB, about
//     20 us at what one CU reads); beyond, the layer stops after its events (kOneEventsDone) and the host continues
//     it with the launches of the general path, which finds the targets, the bitmap and the list of long rows
//     where its own event kernel leaves them
#include "events.h"
#include "select.h"

namespace ink {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kOneThreads = 1024, kOneWaves = kOneThreads / kWave;
constexpr int kOneRows = 2 * kOneEvents;          // rows to transform: targets and sources
constexpr int64_t kOneGather = 512 * 1024;
constexpr int kTileK = 128;                       // part of the input staged in LDS at a time
constexpr int kMergeFloats = 2048;                // columns of partial results held at a time
constexpr int kTileStride = 36;                   // LDS row of a 32-k chunk: even k, odd k, padding (as in xform.hip)

struct OneLds {
  uint32_t ek[kOneEvents], ev[kOneEvents], sk[kOneEvents], sv[kOneEvents];
  int t_list[kOneEvents], t_seg[kOneEvents + 1];
  int cand[kOneRows], first[kOneRows], rows[kOneRows], flag[kOneRows];
  int sm[kOneWaves + 1];
  int n_c;
  union {
    float x[kTileK / 32][kOneRows][kTileStride];
    struct { float v[kMergeFloats]; int i[kMergeFloats]; float s[kMergeFloats]; int j[kMergeFloats]; } m;
  };
};

// Orders n (<= kOneEvents) events by target, equal targets in creation order: 32 threads count an event's rank.
__device__ __forceinline__ void sort_events(OneLds &S, int n) {
  constexpr int P = kOneThreads / kOneEvents;
  const int i = threadIdx.x / P, p = threadIdx.x % P;
  int rank = 0;
  if (i < n) {
    const uint32_t k = S.ek[i];
    for (int j = p; j < n; j += P) { const uint32_t o = S.ek[j]; rank += (o < k) | ((o == k) & (j < i)); }
  }
#pragma unroll
  for (int o = 1; o < P; o <<= 1) rank += __shfl_xor(rank, o, kWave);
  if (i < n && p == 0) { S.sk[rank] = S.ek[i]; S.sv[rank] = S.ev[i]; }
}

// A listed row, recomputed by the whole workgroup: every wave takes a part of the neighbours, then every thread
// merges the waves' results of one column.
template <bool IS_MIN, int LPR>
__device__ __forceinline__ void recompute_long_row(OneLds &S, const AggArgs &a, int v, uint64_t *chg, Counters *cnt) {
  constexpr int SLOTS = kMergeFloats / (LPR * 4) < kOneWaves ? kMergeFloats / (LPR * 4) : kOneWaves;
  const int t = threadIdx.x, l = lane_id(), w = t / kWave, q = l % LPR;
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
  if (__syncthreads_or(vchg) && t == 0) { mark_bit(chg, v); atomicAdd(&cnt->stripe[0][ST_ACHG], 1ull); }
}

// Distinct ascending ids of cand[0 .. n) -> rows, their number -> n_c (n <= kOneRows, 16 threads a candidate).
__device__ __forceinline__ void sort_rows(OneLds &S, int n) {
  constexpr int P = kOneThreads / kOneRows;
  const int i = threadIdx.x / P, p = threadIdx.x % P;
  const int id = i < n ? S.cand[i] : 0;
  int dup = 0;
  for (int j = p; j < i && i < n; j += P) dup |= S.cand[j] == id;
#pragma unroll
  for (int o = 1; o < P; o <<= 1) dup |= __shfl_xor(dup, o, kWave);
  if (p == 0) S.first[i] = i < n && !dup;
  __syncthreads();
  int rank = 0;
  for (int j = p; j < n && i < n; j += P) rank += S.first[j] & (S.cand[j] < id);
#pragma unroll
  for (int o = 1; o < P; o <<= 1) rank += __shfl_xor(rank, o, kWave);
  if (i < n && p == 0 && S.first[i]) { S.rows[rank] = id; atomicAdd(&S.n_c, 1); }
}

// The SAGE transform of rows [0, n_c), n_c <= 64: a wave owns one tile of the output and the chain of its products over
// k, 32 x 32 with two-k steps or, for up to 16 rows (TINY), 16 x 16 with four-k steps, which take half the time per k.
// The input passes through LDS 128 k at a time, the weights come straight from the L2; both are loaded a block
// ahead, a chunk's weights into the registers that its products have just released.
template <bool TINY>
__device__ __forceinline__ void transform_rows(OneLds &S, const OneLayer &p, int n_c) {
  constexpr int NCH = kTileK / 32, XPT = TINY ? 1 : kOneRows * kTileK / 4 / kOneThreads, NR = TINY ? 4 : 16;
  const int t = threadIdx.x, l = lane_id(), w = t / kWave;
  const int rt = TINY ? 0 : w / 8, ct = TINY ? w : w % 8;           // waves w, w + 4, .. share a SIMD: neighbours in ct do not
  const int d4 = xform_self_row(p.d_in), n_ch = p.Kp / 32;
  const int kq = l >> 4;                                             // TINY: which of a step's four k
  const int col = TINY ? ct * 16 + (l & 15) : ct * 32 + (l & 31);
  const bool mine = TINY ? ct < p.Np / 16 : ct < p.Np / 32 && rt * 32 < n_c;
  const int kl = (t % (kTileK / 4)) * 4, rl0 = t / (kTileK / 4);     // this thread stages k kl .. kl + 3 of rows rl0, rl0 + 32
  const int wl = TINY ? (kq & 1) * 32 + (ct & 1) * 16 + (l & 15) : l; // the lane of a weight tile that holds this lane's operands
  const f4v *wp = reinterpret_cast<const f4v *>(p.W) + (mine ? (TINY ? ct / 2 : ct) : 0) * 256 + wl;
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
    const int left = k < 2 * d4 ? p.d_in - (k < d4 ? k : k - d4) : 0;    // past it and in the padding of an aggregated row anything may stand
    __syncthreads();
#pragma unroll
    for (int u = 0; u < XPT; u++) {
      const float v0 = left > 0 ? x[u].x : 0.f, v1 = left > 1 ? x[u].y : 0.f, v2 = left > 2 ? x[u].z : 0.f, v3 = left > 3 ? x[u].w : 0.f;
      float *xr = S.x[kl / 32][rl0 + u * 32];
      if (TINY) {                               // in a row of a chunk: the four k of a step in four groups of 8
        float *xp = xr + (kl % 32) / 4;
        xp[0] = v0; xp[8] = v1; xp[16] = v2; xp[24] = v3;
      } else {                                  // even k, odd k
        float *xp = xr + (kl % 32) / 2;
        *reinterpret_cast<float2 *>(xp) = make_float2(v0, v2);
        *reinterpret_cast<float2 *>(xp + 16) = make_float2(v1, v3);
      }
    }
    __syncthreads();
    issue_x(c0 + NCH);
    if (mine)
#pragma unroll
      for (int c = 0; c < NCH; c++) {           // chunks past the last: zeros of the input
        if constexpr (TINY) {
          const float4 *ap = reinterpret_cast<const float4 *>(&S.x[c][l & 15][kq * 8]);
          const float4 lo = ap[0], hi = ap[1];
          const float a[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          const bool second = kq >> 1;
#pragma unroll
          for (int s = 0; s < 8; s++) {
            const f4v q = b[c][s >> 1];
            const float bw = s & 1 ? (second ? q.w : q.z) : (second ? q.y : q.x);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bw, acc, 0, 0, 0);
          }
        } else {
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
        }
        if (c0 + NCH < n_ch) issue_w(c, c0 + NCH + c);
      }
  }
  if (!mine || col >= p.n_out) return;
  const float bias = p.bias ? p.bias[col] : 0.f;
  auto slot = [&](int r) { return TINY ? 4 * kq + r : rt * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); };
  float old[NR];
#pragma unroll
  for (int r = 0; r < NR; r++) {
    const int i = slot(r);
    old[r] = i < n_c ? p.out[(int64_t)S.rows[i] * p.ld_out + col] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < NR; r++) {
    const int i = slot(r);
    if (i >= n_c) continue;
    float v = acc[r];
    if (p.bias) v = __fadd_rn(v, bias);
    if (p.user) v = __fadd_rn(v, p.user[(int64_t)S.rows[i] * p.ld_user + col]);
    if (p.relu) v = v > 0.f ? v : 0.f;
    if (__float_as_uint(old[r]) != __float_as_uint(v)) { p.out[(int64_t)S.rows[i] * p.ld_out + col] = v; S.flag[i] = 1; }
  }
}

template <bool IS_MIN, int LPR>
__global__ __launch_bounds__(kOneThreads) void k_layer_one(OneLayer p) {
  __shared__ OneLds S;
  const int t = threadIdx.x, l = lane_id(), w = __builtin_amdgcn_readfirstlane(t / kWave);
  Counters *cnt = p.cnt;
  // sizes of this layer: the applied edge changes, and the changed sources the layer before left behind
  const int n_ins = p.g->v[C_TMP2], n_del = p.g->v[C_TMP3];     // 0 unless the batch was applied
  bool go = p.g->v[C_OK] != 0;
  int nF = 0, n_chg = 0;
  if (p.layer > 1) { go = go && p.chain->done == p.layer - 1; nF = p.chain->n_f; n_chg = p.chain->n_ev; }
  const int nE = ieee_mode_off(n_ins + n_del + n_chg);
  go = go && n_chg <= kOneEvents && nE <= kOneEvents && nF <= kOneEvents;
  __syncthreads();                              // all have read the chain record before it is rewritten
  if (go) {                                     // otherwise the counters may be those of a layer that the host continues
    int32_t *z = (int32_t *)cnt;
    for (int i = t; i < (int)(sizeof(Counters) / sizeof(int32_t)); i += kOneThreads) z[i] = 0;
  }
  if (t == 0) { S.n_c = 0; if (p.layer == 1) p.chain->done = 0; }
  __threadfence_block();
  __syncthreads();
  int status = kOneNothing;
  if (go) {
    // events and their order
    if (t < nE) {
      uint32_t k, v;
      if (t < n_del) seed_event(t, p.del_s, p.del_d, p.ins_s, p.ins_d, n_del, &k, &v);
      else if (t < n_del + n_chg) expand_event(t - n_del, p.F, nF, p.pref, p.out_off, p.out_ids, 0, &k, &v);
      else seed_event(t - n_chg, p.del_s, p.del_d, p.ins_s, p.ins_d, n_del, &k, &v);
      S.ek[t] = k; S.ev[t] = v;
    }
    __syncthreads();
    sort_events(S, nE);
    __syncthreads();
    int nT;
    {
      const int h = t < nE && (t == 0 || S.sk[t] != S.sk[t - 1]);
      const int ex = block_excl_scan<kOneThreads>(h, S.sm, &nT);
      if (h) { S.t_list[ex] = (int)S.sk[t]; S.t_seg[ex] = t; p.t_list[ex] = (int)S.sk[t]; }
      if (t == 0) { S.t_seg[nT] = nE; cnt->v[C_NT] = nT; }
    }
    __syncthreads();
    // the targets, one per wave at a time; exposed rows of moderate length on the spot
    {
      const int q = l % LPR;
      const bool lane_on = 4 * q < p.a.wd;
      RowSink exp;
      for (int i = w; i < nT; i += kOneWaves) {
        const int v = __builtin_amdgcn_readfirstlane(S.t_list[i]);
        const int e0 = __builtin_amdgcn_readfirstlane(S.t_seg[i]), e1 = __builtin_amdgcn_readfirstlane(S.t_seg[i + 1]);
        Cached<IS_MIN> c;
        EvAcc<IS_MIN> s;
        reduce_events<IS_MIN, LPR>(p.a, v, S.sv, e0, e1, lane_on, q, c, s);
        finish_target<IS_MIN, LPR, true>(p.a, v, c, s, lane_on, q, p.bm, nullptr, exp, cnt);
      }
    }
    __threadfence_block();
    __syncthreads();
    // long exposed rows
    const int n_big = __hip_atomic_load(&cnt->v[C_NBIG], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int64_t nb = 0;
    for (int i = 0; i < n_big; i++) nb += p.a.in_deg[p.a.big.list[i]];
    status = nb * p.a.wd <= kOneGather ? kOneDone : kOneEventsDone;
    if (status == kOneDone) {
      for (int i = 0; i < n_big; i++) recompute_long_row<IS_MIN, LPR>(S, p.a, p.a.big.list[i], p.bm, cnt);
      __threadfence_block();
      __syncthreads();
      // rows to transform: targets whose aggregate changed, sources (their own message changed)
      int n_cand;
      {
        int id = -1;
        if (t < nT) {
          const int v = S.t_list[t];
          const unsigned long long bit = 1ull << (v & 63);
          if (atomicAnd((unsigned long long *)&p.bm[v >> 6], ~bit) & bit) id = v;
        } else if (t >= kOneEvents && t - kOneEvents < nF) id = p.F[t - kOneEvents];
        const int ex = block_excl_scan<kOneThreads>(id >= 0, S.sm, &n_cand);
        if (id >= 0) S.cand[ex] = id;
        if (t < kOneRows) S.flag[t] = 0;
      }
      __syncthreads();
      sort_rows(S, n_cand);
      __syncthreads();
      const int nC = S.n_c;
      if (nC <= 16) transform_rows<true>(S, p, nC); else transform_rows<false>(S, p, nC);
      __syncthreads();
      // changed rows in order, and the events they propagate
      int nF2, n_ev;
      const int u = t < nC ? S.rows[t] : -1;
      const int f = t < nC && S.flag[t];
      const int kd = f ? p.out_deg[u] - p.new_out[u] : 0;
      const int ex = block_excl_scan<kOneThreads>(f, S.sm, &nF2);
      const int ep = block_excl_scan<kOneThreads>(kd, S.sm, &n_ev);
      if (f) { p.F_next[ex] = u; p.pref[ex] = ep; S.cand[ex] = u; }
      if (t == 0) {
        cnt->v[C_NC] = nC; cnt->v[C_NEXT] = nF2; cnt->v[C_NEV] = p.last ? 0 : n_ev;
        p.chain->done = p.layer; p.chain->n_f = nF2; p.chain->n_ev = n_ev;
      }
      if (p.last) {     // the result, and the batch's marks
        __threadfence_block();
        __syncthreads();
        const int d = p.n_out;
        for (int i = t; i < nF2 * d; i += kOneThreads) {
          const float x = p.out[(int64_t)S.cand[i / d] * p.ld_out + i % d];
          p.res[i] = x;
          if (p.h_emb) p.h_emb[i] = x;
        }
        if (p.h_ids && t < nF2) p.h_ids[t] = S.cand[t];
        const int n_src = n_ins + n_del > 0 ? p.g->v[C_OT] : 0;
        for (int i = t; i < n_src; i += kOneThreads) p.new_out[p.touched_src[i]] = 0;
      }
    }
  }
  if (t == 0) cnt->v[C_ONE] = status;
  // The record of the last layer ends the call, and the result may then be read on any stream: every wave waits here until
  // its own stores have reached the L2 (a barrier alone lets them be under way), and wave 0 writes them back from there.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (w == 0) {                                 // publish_wave, for counters whose stripes but the first are 0
    if (l < 32) p.h->v[l] = __hip_atomic_load(&cnt->v[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else if (l < 32 + ST_N) p.h->total[l - 32] = __hip_atomic_load(&cnt->stripe[0][l - 32], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence_system();
    if (l == 0) __hip_atomic_store(p.h_seq, p.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

hipError_t layer_one(ink_ctx *c, const OneLayer &p) {
#define INK_ONE(M, L) hipLaunchKernelGGL((k_layer_one<M, L>), dim3(1), dim3(kOneThreads), 0, c->stream, p)
  const int lanes = p.a.wd <= 64 ? 16 : (p.a.wd <= 128 ? 32 : 64);
  if (p.a.is_min) { if (lanes == 16) INK_ONE(true, 16); else if (lanes == 32) INK_ONE(true, 32); else INK_ONE(true, 64); }
  else { if (lanes == 16) INK_ONE(false, 16); else if (lanes == 32) INK_ONE(false, 32); else INK_ONE(false, 64); }
#undef INK_ONE
  return hipGetLastError();
}

}  // namespace ink
