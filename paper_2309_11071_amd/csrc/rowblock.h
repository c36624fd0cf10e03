// Rows of a recompute launch, taken by a wave in blocks: one load per lane brings the place and length of up to
// kRowBlock rows, rows that need nothing are left out, and the ids of the next row are under way while one is gathered.
// What it is for is the rows left out: half of the nodes of a power-law graph have no in-neighbours, and a layer that
// re-aggregates every node need not touch their four table rows unless they lost their last edge.  10000 updates and their inverse on
// 1.25M nodes, rows of 128 floats, 8.14 -> 7.69 ms, 1000 feature rows on 200k nodes 1.53 -> 1.47.  Leaving out all
// rows without an event takes a byte per target from every event, 60 us per 10M, and saves another 0.3 % of the edges.  Where
// every row is gathered the blocks change nothing (inference of 625k nodes 4.23 against 4.22 ms).
#pragma once
#include "bigrows.h"
#include "rowload.h"

namespace ink {

constexpr int kRowBlock = 16;

struct RowBlock {
  int v, deg, asc, off_lo, off_hi;         // lane j: row j of the block
  uint64_t todo;                           // wave-uniform: rows of the block that are gathered by this wave
  // rows [r0, r0 + k) of the launch; those with more than big_deg neighbours go to the list (one place per block)
  __device__ __forceinline__ void load(const AggArgs &a, const int32_t *targets, int64_t r0, int k, const uint64_t *set, Counters *cnt,
                                       int64_t &nb, int64_t &nb_long) {
    const int l = lane_id();
    const int j = l < k ? l : k - 1;
    v = targets ? targets[r0 + j] : (int)(r0 + j);
    const int64_t off = a.in_off[v];
    deg = a.in_deg[v];
    asc = a.in_asc[v];
    const bool on = l < k && (!a.keep_empty || deg > 0 || (set[v >> 6] >> (v & 63) & 1));
    off_lo = (int)(uint32_t)off; off_hi = (int)(off >> 32);
    const bool big = on && deg > a.big_deg;
    nb += on ? deg : 0; nb_long += big ? deg : 0;
    const uint64_t bigs = __ballot(big);
    todo = __ballot(on) & ~bigs;
    if (bigs) {
      const int mine = big ? big_row_chunks(deg, a.big.chunk) : 0;
      int upto = mine;                     // chunks of the block's rows up to this one
#pragma unroll
      for (int o = 1; o < kRowBlock; o <<= 1) { const int y = __shfl_up(upto, o, kWave); if (l >= o) upto += y; }
      int i = 0, base = 0;
      if (l == kRowBlock - 1) reserve_big(cnt, __popcll(bigs), upto, i, base);
      i = __builtin_amdgcn_readlane(i, kRowBlock - 1) + __popcll(bigs & ((1ull << l) - 1));
      base = __builtin_amdgcn_readlane(base, kRowBlock - 1) + upto - mine;
      if (big) { a.big.list[i] = v; a.big.base[i] = base; }
    }
  }
  __device__ __forceinline__ int row(int j) const { return __builtin_amdgcn_readlane(v, j); }
  __device__ __forceinline__ int length(int j) const { return __builtin_amdgcn_readlane(deg, j); }
  __device__ __forceinline__ bool ascending(int j) const { return __builtin_amdgcn_readlane(asc, j) != 0; }
  __device__ __forceinline__ int64_t place(int j) const {
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(off_hi, j) << 32) | (uint32_t)__builtin_amdgcn_readlane(off_lo, j));
  }
  // the first ids of row j, one per lane
  __device__ __forceinline__ int first_ids(const int32_t *in_ids, int j) const { return ids_ahead(in_ids + place(j), 0, length(j)); }
};

// rows per visit: what the launch's waves have to take each, up to kRowBlock
__device__ __forceinline__ int row_block(int64_t n, int64_t n_waves) {
  const int64_t per = (n + n_waves - 1) / n_waves;
  return per < 1 ? 1 : per > kRowBlock ? kRowBlock : (int)per;
}

// what the lanes of a launch's waves tallied, to the counters
__device__ __forceinline__ void tally_rows(Counters *cnt, int64_t nb, int64_t nb_long) {
#pragma unroll
  for (int o = kRowBlock / 2; o > 0; o >>= 1) {
    nb += __shfl_xor(nb, o, kWave); nb_long += __shfl_xor(nb_long, o, kWave);
  }
  if (lane_id() != 0 || nb == 0) return;
  unsigned long long *s = cnt->stripe[blockIdx.x % kStripes];
  atomicAdd(&s[ST_REGATHER], (unsigned long long)nb);
  if (nb_long) atomicAdd(&s[ST_REGATHER_LONG], (unsigned long long)nb_long);
}

}  // namespace ink
