// How the events of a layer are made from the applied edge changes and the changed sources.
#pragma once
#include "ctx.h"

namespace ink {

// The events of a layer are created in this order: removed edges, changed sources (by ascending
// source, each over its kept out-edges), inserted edges.  The grouping is stable, so every target
// sees its events in that order: among the events that carry a row, the changed sources come first
// and in ascending id order, which is what lets the max / min kernel drop the id comparison of ties
// until the first inserted edge shows up (consume_batch in select.h).
// seed i of the applied edge changes: deletions first, then insertions; key = target
__device__ __forceinline__ void seed_event(int i, const int32_t *del_s, const int32_t *del_d, const int32_t *ins_s,
                                           const int32_t *ins_d, int n_del, uint32_t *key, uint32_t *val) {
  if (i < n_del) { *key = (uint32_t)del_d[i]; *val = (EV_DEL << kEvKindShift) | (uint32_t)del_s[i]; }
  else {
    int j = i - n_del;
    *key = (uint32_t)ins_d[j]; *val = (EV_ADD << kEvKindShift) | (uint32_t)ins_s[j];
  }
}

// out-edges of a changed source that exist in both snapshots: the block minus the ids appended by this batch
__device__ __forceinline__ int kept_out_degree(const int32_t *deg, const int32_t *new_out, int u) { return deg[u] - new_out[u]; }

// the changed source that owns propagated event e: the last of those whose prefix is not above it (pref[0] <= e)
__device__ __forceinline__ int source_of_event(const int32_t *pref, int nF, int e) {
  int lo = 0, hi = nF - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (pref[mid] <= e) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// propagated event e: source = the changed node owning it, target = its e-th kept out-neighbour.
// payload_index: store the position in F instead of the node id.
__device__ __forceinline__ void expand_event(int e, const int32_t *F, int nF, const int32_t *pref, const int64_t *off,
                                             const int32_t *ids, int payload_index, uint32_t *key, uint32_t *val) {
  const int lo = source_of_event(pref, nF, e);
  int u = F[lo];
  int p = e - pref[lo];
  *key = (uint32_t)ids[off[u] + p];
  *val = (EV_CHG << kEvKindShift) | (uint32_t)(payload_index ? lo : u);
}

}  // namespace ink
