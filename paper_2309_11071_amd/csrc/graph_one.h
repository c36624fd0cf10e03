// The graph stage of a few entries in one workgroup, and what it shares with the other forms of the stage (graph.hip).
#pragma once
#include "ctx.h"

namespace ink {

// what is wrong with a list entry: bit 0 = op is neither insert nor delete, bit 1 = id out of range
__device__ __forceinline__ int entry_error(const RawUpdate &a, int n_nodes) {
  int e = a.op > 1 ? 1 : 0;
  if (a.src < 0 || a.src >= n_nodes || a.dst < 0 || a.dst >= n_nodes) e |= 2;
  return e;
}

constexpr int kChunk = 2048;           // slots of a touched node's block that are walked together
constexpr uint64_t kNoKey = ~0ull;     // sorts behind every (node, other) pair

__device__ __forceinline__ uint64_t update_key(const RawUpdate &a, int side) {
  return side ? ((uint64_t)(uint32_t)a.src << 32) | (uint32_t)a.dst : ((uint64_t)(uint32_t)a.dst << 32) | (uint32_t)a.src;
}

// 0 no-op, 1 insert, 2 delete, from the op (0 insert, 1 delete, 2 dead) and the slot where its edge was found
__device__ __forceinline__ int effect_of(int op, int pos) { return op == 0 ? (pos < 0 ? 1 : 0) : (op == 1 && pos >= 0 ? 2 : 0); }

__device__ __forceinline__ long long relocated_cap(int deg, int cap, float slack) {
  long long want = 2ll * cap;
  long long extra = (long long)(deg * (double)slack + 0.999);
  if (extra < 4) extra = 4;
  if (want < deg + extra) want = deg + extra;
  return (want + 3) & ~3ll;
}

// Deletes up to 64 slots of a block, one per lane (pos, if del), whole wave: [0, d1) survives, its holes take the
// survivors of the tail [d1, d1 + nd) in slot order, holes in op order.
__device__ __forceinline__ void fill_holes(int32_t *ids, int d1, int nd, int pos, bool del) {
  const int l = lane_id();
  const bool hole = del && pos < d1;
  // the tail has nd <= 64 slots; those that are deleted themselves do not survive
  uint64_t gone = del && pos >= d1 ? 1ull << (pos - d1) : 0ull;
  for (int o = 32; o > 0; o >>= 1) gone |= __shfl_xor((unsigned long long)gone, o, kWave);
  const uint64_t live = (nd < kWave ? (1ull << nd) - 1 : ~0ull) & ~gone;
  const uint64_t holes = __ballot(hole);
  const int rank = __popcll(holes & ((1ull << l) - 1));
  const int tail_id = l < nd ? ids[d1 + l] : 0;
  uint64_t m = live;
  int src = 0;
  for (int r = 0; r < __popcll(holes); r++) {       // slot of the r-th survivor, for the lane whose hole it fills
    const int b = __ffsll((unsigned long long)m) - 1;
    if (hole && rank == r) src = b;
    m &= m - 1;
  }
  const int id = __shfl(tail_id, src, kWave);
  if (hole) ids[pos] = id;
}

// ---- the whole graph stage of a few entries in one workgroup
// A wave sorts one side's entries in registers and finds their nodes; all waves walk the blocks of both sides' nodes;
// then, if the batch is valid, the pools have room and the sides agree, a wave per node applies its ops.  The four
// launches of the short form take 26 us for a single entry, nearly all of it launches and barriers; this one takes 9.
// Limits: kOneEvents entries (a wave holds a side's list), kOneGraphChunks chunks of ids to walk (256 = half a million
// ids, two rounds of the workgroup take about as long as the launches saved); a batch beyond them, or one
// that needs larger pools, is left untouched (C_ONE stays 0) and takes the short form.
constexpr int kOneGraphChunks = 256;
struct OneGraphLds {
  int node[2][kOneEvents], other[2][kOneEvents], op[2][kOneEvents], pos[2][kOneEvents];
  int uniq[2][kOneEvents], seg[2][kOneEvents + 1], n_uniq[2];
  int deg[2 * kOneEvents], cap[2 * kOneEvents], chunk[2 * kOneEvents + 1];     // touched nodes of both sides behind each other
  int64_t off[2 * kOneEvents];
  int n_ins[2 * kOneEvents], n_del[2 * kOneEvents], want[2 * kOneEvents];      // want: new capacity if the block moves, else 0
  int64_t new_off[2 * kOneEvents];
  int tot_ins[2], tot_del[2];
  long long need[2];
  int err;
};
static_assert(kOneEvents <= kWave, "a lane per entry");

// The record of the stage, slots and the pool space of both sides, is left in `record`, which the whole workgroup may read at once.
__device__ __forceinline__ void graph_one(OneGraphLds &S, const OneGraph &p, HostCounters &record) {
  constexpr int NW = 1024 / kWave;
  const RawUpdate *raw = p.raw;
  const int n = p.n;
  const OneSide &in = p.in, &out = p.out;
  const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), t = w * kWave + l;
  if (w < 2) {                        // wave s: the op list of side s in (node, other) order, equal pairs in batch order
    const int side = w;
    RawUpdate a{};
    int bad = 0;
    if (l < n) { a = raw[l]; bad = entry_error(a, p.n_nodes); }
    const int err = (__ballot(bad & 1) ? 1 : 0) | (__ballot(bad & 2) ? 2 : 0);
    if (t == 0) S.err = err;
    const OneSide &o = side ? out : in;
    const uint64_t key = l < n ? update_key(a, side) : kNoKey;
    int rank = 0;
    for (int j = 0; j < n; j++) {
      const uint64_t kj = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(key >> 32), j) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, j);
      rank += (kj < key) | ((kj == key) & (j < l));
    }
    if (l < n) { S.node[side][rank] = (int)(key >> 32); S.other[side][rank] = (int)(uint32_t)key; S.op[side][rank] = a.op; S.pos[side][rank] = -1; }
    __builtin_amdgcn_wave_barrier();
    const int v = l < n ? S.node[side][l] : -1, x = l < n ? S.other[side][l] : -1;
    const int pv = l > 0 && l < n ? S.node[side][l - 1] : -1;
    const int nv = l + 1 < n ? S.node[side][l + 1] : -1, nx = l + 1 < n ? S.other[side][l + 1] : -1;
    const bool head = l < n && v != pv;
    const uint64_t heads = __ballot(head);
    if (l < n && ((nv == v && nx == x) || v == x)) S.op[side][l] = 2;          // overridden by a later entry, or a self loop
    const int at = __popcll(heads & ((1ull << l) - 1));
    if (head) { S.uniq[side][at] = v; S.seg[side][at] = l; }
    if (l == 0) { S.n_uniq[side] = err ? 0 : __popcll(heads); S.seg[side][__popcll(heads)] = n; }
    if (!err && head) o.uniq[at] = v;
  }
  __syncthreads();
  const int n0 = S.n_uniq[0], n_all = n0 + S.n_uniq[1];
  if (t < n_all) {
    const OneSide &o = t < n0 ? in : out;
    const int v = t < n0 ? S.uniq[0][t] : S.uniq[1][t - n0];
    S.deg[t] = o.deg[v]; S.cap[t] = o.cap[v]; S.off[t] = o.off[v];
  }
  if (w == 0) {                       // prefix of the chunk counts (n_all <= kWave)
    const int ch = l < n_all ? (S.deg[l] + kChunk - 1) / kChunk : 0;
    const int inc = wave_incl_scan(ch);
    if (l < n_all) S.chunk[l] = inc - ch;
    if (l == kWave - 1) S.chunk[n_all] = inc;
  }
  __syncthreads();
  const int total = S.chunk[n_all];
  const bool walk = total <= kOneGraphChunks;
  if (walk)
    for (int c = w; c < total; c += NW) {
      int i = 0;
      for (int j = 1; j < n_all; j++) i = S.chunk[j] <= c ? j : i;      // empty blocks have no chunk: the last one that starts here owns it
      i = __builtin_amdgcn_readfirstlane(i);
      const int side = i >= n0, k = side ? i - n0 : i;
      const int s0 = S.seg[side][k], s1 = S.seg[side][k + 1], d = S.deg[i];
      const int32_t *ids = (side ? out.ids : in.ids) + S.off[i];
      const int p_begin = (c - S.chunk[i]) * kChunk, p_end = p_begin + kChunk < d ? p_begin + kChunk : d;
      for (int p = p_begin + 4 * l; p < p_end; p += 4 * kWave) {
        const int4 e4 = *reinterpret_cast<const int4 *>(ids + p);
        const int e[4] = {e4.x, e4.y, e4.z, e4.w};
        for (int m = s0; m < s1; m++)
#pragma unroll
          for (int j = 0; j < 4; j++)
            if (e[j] == S.other[side][m] && p + j < d) S.pos[side][m] = p + j;
      }
    }
  __syncthreads();
  if (w < 2) {                        // effective ops of side w, what they do to each node, and the pool space they need
    const int side = w;
    const int e = l < n && !S.err ? effect_of(S.op[side][l], S.pos[side][l]) : 0;
    const uint64_t mi = __ballot(e == 1), md = __ballot(e == 2);
    const uint64_t below = (1ull << l) - 1;
    if (side == 0 && e == 1) { p.ins_s[__popcll(mi & below)] = S.other[0][l]; p.ins_d[__popcll(mi & below)] = S.node[0][l]; }
    if (side == 0 && e == 2) { p.del_s[__popcll(md & below)] = S.other[0][l]; p.del_d[__popcll(md & below)] = S.node[0][l]; }
    int want = 0;
    if (l < S.n_uniq[side]) {
      const int i = side * n0 + l;
      const uint64_t seg = ((S.seg[side][l + 1] < kWave ? 1ull << S.seg[side][l + 1] : 0ull) - 1) & ~((1ull << S.seg[side][l]) - 1);
      const int ni = __popcll(mi & seg), nd = __popcll(md & seg);
      const int d2 = S.deg[i] - nd + ni;
      S.n_ins[i] = ni; S.n_del[i] = nd;
      if (d2 > S.cap[i]) want = (int)relocated_cap(d2, S.cap[i], p.slack);
      S.want[i] = want;
    }
    const int inc = wave_incl_scan(want);
    if (l < S.n_uniq[side]) S.new_off[side * n0 + l] = (side ? out : in).pool_base + inc - want;
    if (l == kWave - 1) S.need[side] = inc;
    if (l == 0) { S.tot_ins[side] = __popcll(mi); S.tot_del[side] = __popcll(md); }
  }
  __syncthreads();
  const bool agree = S.tot_ins[0] == S.tot_ins[1] && S.tot_del[0] == S.tot_del[1];
  const bool room = S.need[0] <= in.room && S.need[1] <= out.room;
  const bool ok = !S.err && walk && agree && room;
  if (ok) {
    // holes in the surviving part of a block are filled from its tail, in op order
    for (int i = w; i < n_all; i += NW) {
      const int nd = S.n_del[i];
      if (nd == 0) continue;
      const int side = i >= n0, k0 = S.seg[side][side ? i - n0 : i], k1 = S.seg[side][(side ? i - n0 : i) + 1];
      int32_t *ids = (side ? out.ids : in.ids) + S.off[i];
      const int d1 = S.deg[i] - nd, k = k0 + l;
      const int pos = k < k1 ? S.pos[side][k] : -1;
      fill_holes(ids, d1, nd, pos, k < k1 && effect_of(S.op[side][k], pos) == 2);
    }
    __threadfence_block();
    __syncthreads();
    for (int i = 0; i < n_all; i++) {               // blocks that outgrow their slots
      if (S.want[i] == 0) continue;
      int32_t *pool = i >= n0 ? out.ids : in.ids;
      const int d1 = S.deg[i] - S.n_del[i];
      for (int p = t; p < d1; p += 1024) pool[S.new_off[i] + p] = pool[S.off[i] + p];
    }
    for (int i = w; i < n_all; i += NW) {
      const int ni = S.n_ins[i], nd = S.n_del[i];
      if (ni == 0 && nd == 0) continue;
      const int side = i >= n0, j = side ? i - n0 : i, k = S.seg[side][j] + l;
      const OneSide &o = side ? out : in;
      const int d1 = S.deg[i] - nd, v = S.uniq[side][j];
      const bool move = S.want[i] > 0;
      int32_t *ids = o.ids + (move ? S.new_off[i] : S.off[i]);
      const bool ins = k < S.seg[side][j + 1] && effect_of(S.op[side][k], S.pos[side][k]) == 1;
      const uint64_t m = __ballot(ins);
      if (ins) ids[d1 + __popcll(m & ((1ull << l) - 1))] = S.other[side][k];
      if (l == 0) {
        if (move) { o.cap[v] = S.want[i]; o.off[v] = S.new_off[i]; }
        o.deg[v] = d1 + ni;
        o.asc[v] = 0;
        if (o.new_cnt) o.new_cnt[v] = ni;
      }
    }
  }
  __threadfence_block();
  __syncthreads();
  if (w == 0) {
    int x = 0;
    const int slot = l;
    if (slot == C_ERR) x = S.err;
    if (slot == C_TMP0) x = n0;
    if (slot == C_OT) x = n_all - n0;
    if (slot == C_GINS) x = S.tot_ins[0];
    if (slot == C_GDEL) x = S.tot_del[0];
    if (slot == C_OINS) x = S.tot_ins[1];
    if (slot == C_ODEL) x = S.tot_del[1];
    if (slot == C_OK) x = ok;
    if (slot == C_TMP2) x = ok ? S.tot_ins[0] : 0;
    if (slot == C_TMP3) x = ok ? S.tot_del[0] : 0;
    if (slot == C_ONE) x = S.err || !agree || ok;            // otherwise: walk the long way
    if (l < 32) record.v[l] = x;
    if (l < ST_N) record.total[l] = l < 2 ? (unsigned long long)S.need[l] : 0;
  }
  __syncthreads();
}

}  // namespace ink
