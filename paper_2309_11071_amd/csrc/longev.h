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
// 605k 220 / 223 / 244, 3.7M 667 / 638 / 648, 17M - / 2000 / 1750; rows of 256 floats 56k 95 / 82 / 79, 537k 302 / 365 / 338; sums
// over 128 floats 159k 68 / 65 / 63, 296k 81 / 86 / 95, 725k 146 / 147 / 149, 2.05M 246 / 244 / 248, 18M 2133 / 1262 / 1021; over 256
// 494k 99 / 102 / 103, 1.6M 189 / 186 / 191, 5.8M 732 / 470 / 477; over 64 282k 70 / 72 / 75, 4.4M 278 / 273 / 273.
// Those have 2 to 5 events a target, up to 13 beyond 2M.  Where targets have many, nearly every event is in a segment above a low limit, and
// their lists and partial rows cost more than the chains (events a target in brackets): sums over 128 floats 301k
// (7) 47 / 50 / 54, 357k (8) 49 / 55 / 60, 525k (13) 77 / 57 / 61, 869k (13) 111 / 80 / 84, 1.34M (10) 154 / 112 / 120, 1.86M (23) 270 / 123 / 115, 3.5M (41)
// 309 / 253 / 154, 1.28M (67) 177 / 137 / 76; over 64 869k (13) 103 / 65 / 67, 1.23M (19) 108 / 77 / 73, 1.86M (23) 257 / 109 / 88; max over 128
// 1.23M (33) 510 / 459 / 444, 2.3M (30) 790 / 650 / 540.  And segments of at most 500 to 600 events have no chain worth cutting: sums over
// 256 floats 341k 46 / 48 / 43, 558k 73 / 74 / 67, 866k 101 / 92 / 87; of at most 1000, 526k 77 / 57 / 60, 1.31M 120 / 110 / 118.
inline LongEvents long_events(const EventBounds &eb, int64_t n_targets) {
  const int64_t n = eb.n_events;
  if (latency_mode(n_targets)) return LongEvents{nullptr, nullptr, 128, 256};
  if (n <= (1 << 18) || n > (1 << 23) || n > 16 * n_targets || eb.max_seg <= 768) return LongEvents{nullptr, nullptr, 256, 256};
  if (n <= (1 << 20) && n <= 8 * n_targets) return LongEvents{nullptr, nullptr, 64, 128};
  return LongEvents{nullptr, nullptr, 128, 256};
}

inline int64_t long_ev_rows(const LongEvents &L, int64_t n_events) { return n_events / L.limit + 1; }
// A segment of e > limit events has at most e / chunk + 1 chunks, and at most e / limit if a chunk is two limits or more.
inline int64_t long_ev_chunks(const LongEvents &L, int64_t n_events) {
  return (L.chunk >= 2 * L.limit ? 0 : n_events / L.chunk) + long_ev_rows(L, n_events);
}

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
