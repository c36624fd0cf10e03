// Loads of many rows of one table by a wave: a lane holds four floats of a row, LPR lanes hold a row, kWave / LPR lane
// groups take a row each, U rows per group are in flight.
//
// What counts here is that no load stands under a condition: a load whose execution depends on a lane's id costs a
// mask, a branch, its own wait for the id's shuffle and, because the compiler cannot count it, a wait for
// everything before the first use.  So a slot past the end repeats the last row (it is in the L1) and its value is
// dropped where it is used, and lanes past the row's end read its start.  Measured against conditional loads, whole
// passes: 116k-node GCN with 57M edges 3.53 -> 3.34 ms, 3-layer max on 1.25M nodes 9.81 -> 9.53, its inference on 625k
// nodes 5.18 -> 4.99.  There the short rows (6.7M of 12.5M edges, four tables written) now move 7.8 TB/s a layer and the long ones
// 9.4 TB/s, out of the caches in part, so what is left is the memory's.
#pragma once
#include "ctx.h"

namespace ink {

// ids [at, at + 64) of a list of n, one per lane; those past the end repeat the last
__device__ __forceinline__ int ids_ahead(const int32_t *ids, int at, int n) {
  const int k = at + lane_id();
  return at < n ? ids[k < n ? k : n - 1] : 0;
}

template <int LPR> struct RowTable {
  const char *base;         // LPR < 64: of this lane's four floats
  uint32_t row_bytes, lane_bytes;
  int g;                    // lane group
  __device__ __forceinline__ RowTable(const float *M, int ldm, bool lane_on, int q) {
    row_bytes = (uint32_t)ldm * 4u;
    lane_bytes = lane_on ? 16u * (uint32_t)q : 0u;
    base = reinterpret_cast<const char *>(M) + (LPR < kWave ? lane_bytes : 0u);
    constexpr int G = kWave / LPR;
    const int gg = lane_id() / LPR;
    g = gg < G ? gg : G - 1;
  }
  // lane's entry it + u G + g of the window held one per lane in `win`
  template <int U> __device__ __forceinline__ int pick(int win, int it, int u, int last) const {
    constexpr int G = kWave / LPR;
    if constexpr (LPR == kWave) {
      const int k = it + u;
      return __builtin_amdgcn_readlane(win, k < last ? k : last);
    } else {
      const int k = it + u * G + g;
      return __builtin_amdgcn_ds_bpermute((k < last ? k : last) * 4, win);
    }
  }
  __device__ __forceinline__ float4 load(int id) const {
    const char *p = base + (uint64_t)(uint32_t)id * row_bytes;
    if constexpr (LPR == kWave) p += lane_bytes;
    return *reinterpret_cast<const float4 *>(p);
  }
  template <int U> __device__ __forceinline__ void load_batch(int win, int it, int last, int id[U], float4 row[U]) const {
#pragma unroll
    for (int u = 0; u < U; u++) id[u] = pick<U>(win, it, u, last);
#pragma unroll
    for (int u = 0; u < U; u++) row[u] = load(id[u]);
  }
};

}  // namespace ink
