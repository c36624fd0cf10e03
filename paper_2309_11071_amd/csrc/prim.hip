// Scan, compaction and radix sort kernels (gfx950, wave64).
#include <algorithm>

#include "ctx.h"

namespace ink {


// ---------------------------------------------------------------- scan of an int array
struct LoadI32 { const int32_t *p; __device__ int operator()(int64_t i) const { return p[i]; } };
struct StoreExcl { int32_t *p; __device__ void operator()(int64_t i, int, int ex) const { p[i] = ex; } };

hipError_t scan_excl_i32(PrimWorkspace &ws, const int32_t *in, int32_t *out, int64_t n,
                         int32_t *total, hipStream_t s) {
  return tile_scan<LoadI32, StoreExcl, kScanItems, true>(ws, LoadI32{in}, StoreExcl{out}, n, total, s);
}

// ---------------------------------------------------------------- flag compaction
struct LoadFlag { const uint8_t *p; __device__ int operator()(int64_t i) const { return p[i] != 0; } };
struct StoreIdx {
  int32_t *p;
  __device__ void operator()(int64_t i, int v, int ex) const { if (v) p[ex] = (int32_t)i; }
};

hipError_t compact_flags_u8(PrimWorkspace &ws, const uint8_t *flags, int64_t n, int32_t *out_idx,
                            int32_t *count, hipStream_t s) {
  return tile_scan<LoadFlag, StoreIdx, kScanItems, true>(ws, LoadFlag{flags}, StoreIdx{out_idx}, n, count, s);
}

// ---------------------------------------------------------------- bitmap -> ascending id list
struct LoadPop { const uint64_t *p; __device__ int operator()(int64_t i) const { return __popcll(p[i]); } };
struct StoreBits {
  uint64_t *words; int32_t *out; int clear;
  __device__ void operator()(int64_t i, int v, int ex) const {
    if (!v) return;
    uint64_t w = words[i];
    while (w) {
      int b = __ffsll((unsigned long long)w) - 1;
      out[ex++] = (int32_t)(i * 64 + b);
      w &= w - 1;
    }
    if (clear) words[i] = 0;
  }
};

struct PublishThen {
  RecordTo r;
  __device__ __forceinline__ void operator()() const {
    if (threadIdx.x == 0) __threadfence();
    __syncthreads();
    if (threadIdx.x < kWave) publish_wave(r.d, r.h, r.h_seq, r.seq);
  }
};

// A bitmap of one tile, with the items of two short lists set in it first: 256 threads, a word each.  (A launch for the marks in front
// took 4 us: 100 updates on 10k nodes 316 -> 311 us a pass.)
__global__ __launch_bounds__(kScanThreads) void k_bitmap_one(uint64_t *words, int nw, const int32_t *a, int na, const int32_t *b, int nb, int32_t *out,
                                                             int32_t *count, RecordTo record) {
  __shared__ int sm[kScanThreads / kWave + 1];
  __shared__ unsigned long long set[kScanThreads];
  const int t = threadIdx.x;
  set[t] = t < nw ? words[t] : 0;
  __syncthreads();
  for (int i = t; i < na + nb; i += kScanThreads) {
    const int v = i < na ? a[i] : b[i - na];
    atomicOr(&set[v >> 6], 1ull << (v & 63));
  }
  __syncthreads();
  unsigned long long w = set[t];
  int tot;
  int at = block_excl_scan(__popcll(w), sm, &tot);
  if (t < nw) words[t] = 0;
  for (; w; w &= w - 1) out[at++] = t * 64 + __builtin_ctzll(w);
  if (t == 0) *count = tot;
  if (record.d) PublishThen{record}();
}
hipError_t bitmap_one(uint64_t *words, int64_t n_bits, const int32_t *a, int64_t na, const int32_t *b, int64_t nb, int32_t *out_idx, int32_t *count,
                      hipStream_t s, const RecordTo *record) {
  hipLaunchKernelGGL(k_bitmap_one, dim3(1), dim3(kScanThreads), 0, s, words, (int)((n_bits + 63) / 64), a, (int)na, b, (int)nb, out_idx, count,
                     record ? *record : RecordTo());
  return hipGetLastError();
}

hipError_t bitmap_to_list(PrimWorkspace &ws, uint64_t *words, int64_t n_bits, int32_t *out_idx,
                          int32_t *count, int clear, hipStream_t s, const RecordTo *record, bool *given) {
  int64_t nw = (n_bits + 63) / 64;
  const LoadPop f{words};
  const StoreBits w{words, out_idx, clear};
  if (record) return tile_scan<LoadPop, StoreBits, 1, false, PublishThen>(ws, f, w, nw, count, s, PublishThen{*record}, given);
  return tile_scan<LoadPop, StoreBits, 1>(ws, f, w, nw, count, s);
}

// ---------------------------------------------------------------- segment heads of sorted keys
struct LoadHead {
  const uint32_t *k; const int32_t *n_dev;
  __device__ int operator()(int64_t i) const {
    if (n_dev && i >= *n_dev) return 0;
    return i == 0 || k[i] != k[i - 1];
  }
};
struct StoreHead {
  const uint32_t *k; int32_t *uniq; int32_t *seg; int64_t n; const int32_t *n_dev;
  __device__ void operator()(int64_t i, int v, int ex) const {
    if (v) { uniq[ex] = (int32_t)k[i]; seg[ex] = (int32_t)i; }
    int64_t nn = n_dev ? (int64_t)*n_dev : n;
    if (i == nn - 1) seg[ex + v] = (int32_t)nn;    // closing offset after the last run
  }
};

hipError_t segment_heads(PrimWorkspace &ws, const uint32_t *keys, int64_t n, int32_t *uniq,
                         int32_t *seg, int32_t *count, hipStream_t s, const int32_t *n_dev, const RecordTo *record, bool *given) {
  const LoadHead f{keys, n_dev};
  const StoreHead w{keys, uniq, seg, n, n_dev};
  // a record is for lists whose count the host waits for, which are long
  if (record) return tile_scan<LoadHead, StoreHead, kScanItems, false, PublishThen, false>(ws, f, w, n, count, s, PublishThen{*record}, given);
  return tile_scan<LoadHead, StoreHead, kScanItems, true>(ws, f, w, n, count, s);
}

// ---------------------------------------------------------------- stable LSD radix sort
// Three launches a pass: digit counts per tile, one workgroup per digit turns them into exclusive
// prefixes over the tiles (and the digit's total), the scatter adds the prefix over the digits'
// totals itself.  Nothing waits for another workgroup.

// hist[d * nb + b] = number of keys of tile b with digit d
template <int D, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint32_t *keys, int64_t n, int shift, int32_t *hist, int nb) {
  __shared__ int h[1 << D];
  tile_hist_clear<D>(h);
  const int64_t base = (int64_t)blockIdx.x * (kSortThreads * ITEMS);
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int64_t i = base + k * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & ((1 << D) - 1)], 1);
  }
  tile_hist_store<D>(h, hist, nb);
}

// row d of hist (nb entries) -> its exclusive prefix; total[d] = its sum.  One workgroup per digit.
__global__ __launch_bounds__(kSortThreads) void k_digit_scan(int32_t *hist, int nb, int32_t *total) {
  __shared__ int sm[kSortWaves + 1];
  int32_t *row = hist + (int64_t)blockIdx.x * nb;
  int carry = 0;
  for (int b0 = 0; b0 < nb; b0 += kSortThreads * kScanItems) {
    const int b = b0 + threadIdx.x * kScanItems;
    int x[kScanItems], s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) { x[k] = b + k < nb ? row[b + k] : 0; s += x[k]; }
    int tot;
    int ex = carry + block_excl_scan<kSortThreads>(s, sm, &tot);
#pragma unroll
    for (int k = 0; k < kScanItems; k++) { if (b + k < nb) row[b + k] = ex; ex += x[k]; }
    carry += tot;
  }
  if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Each wave owns a contiguous run of ITEMS * 64 keys of the tile and walks it in rounds of
// 64 consecutive keys, so ranks follow the input order (stability).  The pairs are first put in
// digit order inside LDS and written out from there, so that neighbouring lanes store to
// neighbouring addresses (runs of one digit) instead of 64 unrelated ones per instruction.
template <int D, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const uint32_t *keys, const uint32_t *vals,
                                                                 uint32_t *okeys, uint32_t *ovals, int64_t n,
                                                                 int shift, const int32_t *hist_scanned,
                                                                 const int32_t *digit_total, int nb) {
  constexpr int ND = 1 << D, DPT = ND / kSortThreads, TILE = kSortThreads * ITEMS;
  static_assert(DPT >= 1 && TILE < 65536, "digits per thread; tile positions are 16-bit");
  __shared__ uint16_t cnt[kSortWaves][ND];     // per-wave digit counts, then the wave's first slot of the digit in the tile
  __shared__ int out_delta[ND];                // output position of a key minus its slot in the tile
  __shared__ uint32_t skey[TILE], sval[TILE];
  __shared__ int sm[kSortWaves + 1];
  const int w = threadIdx.x / kWave, l = lane_id();
  for (int i = threadIdx.x; i < kSortWaves * ND / 2; i += kSortThreads) reinterpret_cast<uint32_t *>(&cnt[0][0])[i] = 0;
  __syncthreads();
  const int64_t tbase = (int64_t)blockIdx.x * TILE;
  const int64_t wbase = tbase + (int64_t)w * (ITEMS * kWave);
  uint32_t key[ITEMS], val[ITEMS];
  int rank[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    int64_t i = wbase + k * kWave + l;
    bool ok = i < n;
    key[k] = ok ? keys[i] : 0xFFFFFFFFu;
    val[k] = ok ? vals[i] : 0;
  }
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    const bool ok = wbase + k * kWave + l < n;
    const int dg = (int)((key[k] >> shift) & (ND - 1));
    // lanes holding the same digit
    uint64_t same = __ballot(ok);
#pragma unroll
    for (int b = 0; b < D; b++) {
      uint64_t m = __ballot((dg >> b) & 1);
      same &= ((dg >> b) & 1) ? m : ~m;
    }
    const uint64_t lt = (l == 0) ? 0ull : (~0ull >> (kWave - l));
    const int before = __popcll(same & lt);
    int prev = 0;
    if (ok) prev = cnt[w][dg];                 // all lanes of a digit group read the same value
    rank[k] = prev + before;
    // the last lane of each group publishes the new count (after every lane has read)
    const bool leader = ok && ((same >> l) >> 1) == 0;
    if (leader) cnt[w][dg] = (uint16_t)(prev + before + 1);
  }
  __syncthreads();
  // thread t handles digits t DPT ...: their totals in the tile, the exclusive prefix over digits (of the
  // tile and of the whole input), the waves' first slots
  {
    const int d0 = threadIdx.x * DPT;
    int tot[DPT], all[DPT], st = 0, sa = 0;
#pragma unroll
    for (int j = 0; j < DPT; j++) {
      tot[j] = 0;
#pragma unroll
      for (int i = 0; i < kSortWaves; i++) tot[j] += cnt[i][d0 + j];
      all[j] = digit_total[d0 + j];
      st += tot[j]; sa += all[j];
    }
    int dummy;
    int first = block_excl_scan<kSortThreads>(st, sm, &dummy);
    int base = block_excl_scan<kSortThreads>(sa, sm, &dummy);
#pragma unroll
    for (int j = 0; j < DPT; j++) {
      out_delta[d0 + j] = base + hist_scanned[(int64_t)(d0 + j) * nb + blockIdx.x] - first;
      int run = first;
#pragma unroll
      for (int i = 0; i < kSortWaves; i++) {
        const int c = cnt[i][d0 + j];
        cnt[i][d0 + j] = (uint16_t)run;
        run += c;
      }
      first += tot[j];
      base += all[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; k++) {
    if (wbase + k * kWave + l < n) {
      const int dg = (key[k] >> shift) & (ND - 1);
      const int slot = cnt[w][dg] + rank[k];
      skey[slot] = key[k];
      sval[slot] = val[k];
    }
  }
  __syncthreads();
  const int in_tile = (int)(n - tbase < TILE ? n - tbase : TILE);
  for (int s = threadIdx.x; s < in_tile; s += kSortThreads) {
    const uint32_t kk = skey[s];
    const int64_t pos = (uint32_t)(out_delta[(kk >> shift) & (ND - 1)] + s);
    okeys[pos] = kk;
    ovals[pos] = sval[s];
  }
}

// Whole sort in one workgroup: the same stable digit ranking, all passes in LDS, one launch.
// Keys live in registers between the ranking and the scatter of a pass, so one LDS copy of the
// pairs is enough.  THREADS x ITEMS pairs at most; beyond kSmallSort one workgroup is slower than the
// device-wide passes (10 000 pairs: 38 us, against 19 us for two of them).
constexpr int kWideThreads = 1024;
constexpr int kSmallSort = 4096;

template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_small_sort(uint32_t *keys, uint32_t *vals, int n, int passes) {
  __shared__ SmallSortLds<THREADS, ITEMS> S;
  for (int i = threadIdx.x; i < n; i += THREADS) { S.sk[i] = keys[i]; S.sv[i] = vals[i]; }
  small_sort_lds<THREADS, ITEMS>(S, n, passes);
  for (int i = threadIdx.x; i < n; i += THREADS) { keys[i] = S.sk[i]; vals[i] = S.sv[i]; }
}

SortPlan sort_plan(int64_t n, int bits) {
  // Few pairs: their passes are launch-bound and stay in the caches, so wide digits; many pairs: digits
  // that leave runs long enough for whole cache lines in a tile of 3072.  Measured per sort: 312 k pairs of
  // 21 bits: three 8-bit passes 43 us, two 11-bit passes 27 us.
  SortPlan p;
  const int widest = n <= (1 << 20) ? 11 : 9;
  p.passes = (bits + widest - 1) / widest;
  const int d = (bits + p.passes - 1) / p.passes;
  p.digit_bits = d <= 8 ? 8 : (d <= 9 ? 9 : 11);
  p.items = n <= (1 << 18) ? 4 : 12;          // short sorts need the smaller tiles to fill the chip
  p.tiles = nblocks(n, kSortThreads * p.items);
  return p;
}

hipError_t sort_reserve(PrimWorkspace &ws, const SortPlan &p) {
  return ws.hist.reserve(((size_t)(1 << p.digit_bits) * (p.tiles + 1)) * sizeof(int32_t));
}

template <int D, int ITEMS>
static void radix_pass(const SortPlan &p, int pass, bool have_hist, const uint32_t *ka, const uint32_t *va, uint32_t *kb,
                       uint32_t *vb, int64_t n, int32_t *hist, hipStream_t s) {
  const int shift = pass * p.digit_bits;
  int32_t *total = hist + ((int64_t)p.tiles << D);
  if (!have_hist)
    hipLaunchKernelGGL((k_radix_hist<D, ITEMS>), dim3(p.tiles), dim3(kSortThreads), 0, s, ka, n, shift, hist, p.tiles);
  hipLaunchKernelGGL(k_digit_scan, dim3(1 << D), dim3(kSortThreads), 0, s, hist, p.tiles, total);
  hipLaunchKernelGGL((k_radix_scatter<D, ITEMS>), dim3(p.tiles), dim3(kSortThreads), 0, s, ka, va, kb, vb, n, shift,
                     (const int32_t *)hist, (const int32_t *)total, p.tiles);
}

hipError_t radix_sort_planned(PrimWorkspace &ws, const SortPlan &p, uint32_t *&keys, uint32_t *&vals, uint32_t *key_alt,
                              uint32_t *val_alt, int64_t n, bool have_first_hist, hipStream_t s) {
  INK_TRY(sort_reserve(ws, p));
  int32_t *hist = ws.hist.as<int32_t>();
  for (int pass = 0; pass < p.passes; pass++) {
    const bool hh = have_first_hist && pass == 0;
#define INK_PASS(D) \
  (p.items == 4 ? radix_pass<D, 4>(p, pass, hh, keys, vals, key_alt, val_alt, n, hist, s) \
                : radix_pass<D, 12>(p, pass, hh, keys, vals, key_alt, val_alt, n, hist, s))
    if (p.digit_bits == 8) INK_PASS(8);
    else if (p.digit_bits == 9) INK_PASS(9);
    else INK_PASS(11);
#undef INK_PASS
    std::swap(keys, key_alt);
    std::swap(vals, val_alt);
  }
  return hipGetLastError();
}

hipError_t radix_sort_pairs(PrimWorkspace &ws, uint32_t *keys, uint32_t *vals, int64_t n, int bits,
                            hipStream_t s) {
  if (n <= 1 || bits <= 0) return hipSuccess;
  int passes = (bits + kRadixBits - 1) / kRadixBits;
  if (n <= kSmallSort) {
    if (n <= 256)
      hipLaunchKernelGGL((k_small_sort<256, 1>), dim3(1), dim3(256), 0, s, keys, vals, (int)n, passes);
    else if (n <= 1024)
      hipLaunchKernelGGL((k_small_sort<256, 4>), dim3(1), dim3(256), 0, s, keys, vals, (int)n, passes);
    else
      hipLaunchKernelGGL((k_small_sort<kWideThreads, 4>), dim3(1), dim3(kWideThreads), 0, s, keys, vals, (int)n, passes);
    return hipGetLastError();
  }
  const SortPlan p = sort_plan(n, bits);
  INK_TRY(ws.tmpk.reserve((size_t)n * sizeof(uint32_t)));
  INK_TRY(ws.tmpv.reserve((size_t)n * sizeof(uint32_t)));
  uint32_t *k = keys, *v = vals;
  INK_TRY(radix_sort_planned(ws, p, k, v, ws.tmpk.as<uint32_t>(), ws.tmpv.as<uint32_t>(), n, false, s));
  if (k != keys) {
    INK_TRY(hipMemcpyAsync(keys, k, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
    INK_TRY(hipMemcpyAsync(vals, v, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
  }
  return hipSuccess;
}

}  // namespace ink
