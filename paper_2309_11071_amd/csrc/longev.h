// Work list for targets with many events.  One wave per target is a serial chain over its events
// (about 0.2 us per event), and on a power-law graph the hubs have tens of thousands of them: on
// 17 M events over 655 k targets (rows of 128 floats) the largest hub's wave alone ran for 6.7 ms;
// with this list the launch takes 1.75 ms, bound by its row traffic.  The event kernels list every segment above a
// threshold and reserve its chunks of kEvChunk events; one workgroup reduces each chunk and one wave
// per listed target combines the chunks in order.  The reservation also records each chunk's owner,
// so no plan has to be scanned and no chunk searches for its segment.
#pragma once
#include "bigrows.h"

namespace ink {

struct LongSeg { int32_t target, base; };      // position in the target list, first chunk

struct LongEvents {                            // device buffers of the list
  LongSeg *list; int32_t *owner;
  int limit;                                   // segments with more events are listed
};

inline int64_t long_ev_rows(int64_t n_events, int limit) { return n_events / limit + 1; }
inline int64_t long_ev_chunks(int64_t n_events, int limit) { return n_events / kEvChunk + long_ev_rows(n_events, limit); }

// room for every segment and chunk that n_events events can hold, and for the chunks' partial rows
// (with_ids: value, id, runner-up and flags; else one value); nothing if no segment can be long
inline hipError_t ensure_long_events(ink_ctx *c, const EventBounds &eb, int wd, bool with_ids, LongEvents *out) {
  const int64_t n_events = eb.n_events, chunks = long_ev_chunks(n_events, out->limit);
  if (eb.max_seg <= out->limit) return hipSuccess;
  INK_TRY(c->evl_list.reserve((size_t)long_ev_rows(n_events, out->limit) * sizeof(LongSeg)));
  INK_TRY(c->evl_owner.reserve((size_t)chunks * 4));
  INK_TRY(c->big_part_v.reserve((size_t)chunks * wd * 4));
  if (with_ids) {
    INK_TRY(c->big_part_i.reserve((size_t)chunks * wd * 4));
    INK_TRY(c->big_part_s.reserve((size_t)chunks * wd * 4));
    INK_TRY(c->big_part_j.reserve((size_t)chunks * wd * 4));
  }
  out->list = c->evl_list.as<LongSeg>();
  out->owner = c->evl_owner.as<int32_t>();
  return hipSuccess;
}

// lists target t (whole wave, wave-uniform arguments)
__device__ __forceinline__ void list_long_segment(const LongEvents &L, int t, int n_ev, Counters *cnt) {
  const int l = lane_id();
  const int nch = (n_ev + kEvChunk - 1) / kEvChunk;
  int i = 0, base = 0;
  if (l == 0) {
    i = atomicAdd(&cnt->v[C_NEVL], 1);
    base = atomicAdd(&cnt->v[C_NEVCH], nch);
    L.list[i] = LongSeg{t, base};
  }
  i = __builtin_amdgcn_readfirstlane(i);
  base = __builtin_amdgcn_readfirstlane(base);
  for (int j = l; j < nch; j += kWave) L.owner[base + j] = i;
}

// event range of chunk ch and the position of its target in the target list
__device__ __forceinline__ int long_chunk(const LongEvents &L, int ch, const int32_t *seg, int &e0, int &e1) {
  const LongSeg s = L.list[L.owner[ch]];
  e0 = seg[s.target] + (ch - s.base) * kEvChunk;
  const int end = seg[s.target + 1];
  e1 = e0 + kEvChunk < end ? e0 + kEvChunk : end;
  return s.target;
}

}  // namespace ink
