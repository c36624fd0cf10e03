// Work list for targets with many events.  One wave per target is a serial chain over its events
// (about 0.2 us per event), and on a power-law graph the hubs have tens of thousands of them: on
// 17 M events over 655 k targets (rows of 128 floats) the largest hub's wave alone ran for 6.7 ms;
// with this list the launch takes 1.75 ms, bound by its row traffic.  The event kernels list every segment above a
// threshold and reserve its chunks; one workgroup reduces each chunk and one wave
// per listed target combines the chunks in order.  The reservation also records each chunk's owner,
// so no plan has to be scanned and no chunk searches for its segment.
#pragma once
#include "bigrows.h"

namespace ink {

struct LongSeg { int32_t target, base; };      // position in the target list, first chunk

struct LongEvents {                            // device buffers of the list
  LongSeg *list; int32_t *owner;
  int limit;                                   // segments with more events are listed
  int chunk;                                   // events of such a segment per workgroup
};

// Where a segment is long.  Short lists and small chunks cut the chain of one wave, which is the time of a launch that has
// less than a wave's work for every wave the chip holds; a large launch pays for the partial rows instead, and one that
// does not wait for its target count pays two launches as soon as a segment may be long.  Event stage, us, limit and chunk
// 64, 128 / 128, 256 / 256, 256: max over rows of 128 floats, 37k events 48 / 37 / 37, 57k 64 / 52 / 52, 312k 140 / 154 / 166,
// 589k 212 / 215 / 236, 5.3M 826 / 751 / 786, 6.4M 1251 / 877 / 912, 17M - / 2000 / 1750; rows of 256 floats 56k 95 / 82 / 79,
// 495k 317 / 322 / 348; sums over rows of 128 floats 159k 68 / 65 / 63, 18M 2133 / 1262 / 1021.
inline LongEvents long_events(int64_t n_events, bool latency) {
  if (latency) return LongEvents{nullptr, nullptr, 128, 256};
  if (n_events <= (1 << 18) || n_events > (1 << 23)) return LongEvents{nullptr, nullptr, 256, 256};
  if (n_events <= (1 << 20)) return LongEvents{nullptr, nullptr, 64, 128};
  return LongEvents{nullptr, nullptr, 128, 256};
}

inline int64_t long_ev_rows(const LongEvents &L, int64_t n_events) { return n_events / L.limit + 1; }
inline int64_t long_ev_chunks(const LongEvents &L, int64_t n_events) { return n_events / L.chunk + long_ev_rows(L, n_events); }

// room for every segment and chunk that n_events events can hold, and for the chunks' partial rows
// (with_ids: value, id, runner-up and flags; else one value); nothing if no segment can be long
inline hipError_t ensure_long_events(ink_ctx *c, const EventBounds &eb, int wd, bool with_ids, LongEvents *out) {
  const int64_t n_events = eb.n_events, chunks = long_ev_chunks(*out, n_events);
  if (eb.max_seg <= out->limit) return hipSuccess;
  INK_TRY(c->evl_list.reserve((size_t)long_ev_rows(*out, n_events) * sizeof(LongSeg)));
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

__device__ __forceinline__ int long_seg_chunks(const LongEvents &L, int n_ev) { return (n_ev + L.chunk - 1) / L.chunk; }
// lists target t (whole wave, wave-uniform arguments)
__device__ __forceinline__ void list_long_segment(const LongEvents &L, int t, int n_ev, Counters *cnt) {
  const int l = lane_id();
  const int nch = long_seg_chunks(L, n_ev);
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
  e0 = seg[s.target] + (ch - s.base) * L.chunk;
  const int end = seg[s.target + 1];
  e1 = e0 + L.chunk < end ? e0 + L.chunk : end;
  return s.target;
}

}  // namespace ink
