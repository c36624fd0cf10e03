// Device graph store: for each direction (in-neighbours for aggregation / recompute, Sec. 2.5.2;
// out-neighbours for event propagation, Sec. 2.4.2) every node owns a block of ids with slack
// inside one pool.  A batch is normalised to its net effect on the edge set, then applied per
// touched node: deleted slots are refilled from the block's tail, inserted ids are appended, a
// full block moves to a larger one at the pool's end.  Every step is a deterministic function of
// the batch and the current store.
#include <algorithm>
#include <vector>

#include "graph_one.h"

namespace ink {


#define INK_TRYS(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) { c->err = std::string("HIP error: ") + hipGetErrorString(e_); return INK_E_DEVICE; } } while (0)

static inline int64_t align4(int64_t x) { return (x + 3) & ~(int64_t)3; }

static int32_t block_cap(int64_t deg, float slack) {
  int64_t extra = (int64_t)(deg * (double)slack + 0.999);
  if (extra < 4) extra = 4;
  return (int32_t)align4(deg + extra);
}

static hipError_t side_alloc(GraphSide &g, int n, const std::vector<int64_t> &off, const std::vector<int32_t> &deg,
                             const std::vector<int32_t> &cap, const std::vector<int32_t> &ids, int64_t top,
                             int64_t reserve_opt) {
  int64_t reserve = reserve_opt > 0 ? reserve_opt : std::max<int64_t>(top / 4, 1 << 20);
  g.pool_cap = top + reserve;
  g.pool_top = top;
  INK_TRY(hipMalloc(&g.off, sizeof(int64_t) * (size_t)n));
  INK_TRY(hipMalloc(&g.deg, sizeof(int32_t) * (size_t)n));
  INK_TRY(hipMalloc(&g.cap, sizeof(int32_t) * (size_t)n));
  INK_TRY(hipMalloc(&g.asc, (size_t)n));
  INK_TRY(hipMemset(g.asc, 1, (size_t)n));       // built from ascending CSR rows; empty blocks are ascending too
  INK_TRY(hipMalloc(&g.ids, sizeof(int32_t) * (size_t)g.pool_cap));
  INK_TRY(hipMemcpy(g.off, off.data(), sizeof(int64_t) * (size_t)n, hipMemcpyHostToDevice));
  INK_TRY(hipMemcpy(g.deg, deg.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice));
  INK_TRY(hipMemcpy(g.cap, cap.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice));
  INK_TRY(hipMemcpy(g.ids, ids.data(), sizeof(int32_t) * (size_t)top, hipMemcpyHostToDevice));
  return hipSuccess;
}

hipError_t graph_build(ink_ctx *c, const int64_t *rowptr, const int32_t *col) {
  const int n = c->n;
  const int nc = (int)c->n_cap;        // per-node arrays cover the capacity; nodes >= n own no block yet
  const int64_t E = rowptr[n];
  std::vector<int64_t> off(nc, 0);
  std::vector<int32_t> deg(nc, 0), cap(nc, 0);
  // in side straight from the CSR
  int64_t top = 0;
  for (int v = 0; v < n; v++) {
    int64_t d = rowptr[v + 1] - rowptr[v];
    off[v] = top; deg[v] = (int32_t)d; cap[v] = block_cap(d, c->slack);
    top += cap[v];
  }
  {
    std::vector<int32_t> ids((size_t)top, -1);
    for (int v = 0; v < n; v++) std::copy(col + rowptr[v], col + rowptr[v + 1], ids.begin() + off[v]);
    INK_TRY(side_alloc(c->gin, nc, off, deg, cap, ids, top, c->pool_reserve));
  }
  // out side: transpose
  std::vector<int32_t> odeg(n, 0);
  for (int64_t e = 0; e < E; e++) odeg[col[e]]++;
  top = 0;
  for (int v = 0; v < n; v++) {
    off[v] = top; deg[v] = odeg[v]; cap[v] = block_cap(odeg[v], c->slack);
    top += cap[v];
  }
  {
    std::vector<int32_t> ids((size_t)top, -1);
    std::vector<int64_t> cur(off);
    for (int v = 0; v < n; v++)
      for (int64_t e = rowptr[v]; e < rowptr[v + 1]; e++) ids[cur[col[e]]++] = v;
    INK_TRY(side_alloc(c->gout, nc, off, deg, cap, ids, top, c->pool_reserve));
  }
  return hipSuccess;
}

hipError_t graph_export(ink_ctx *c, int64_t *rowptr, int32_t *col) {
  const int n = c->n;
  std::vector<int64_t> off(n);
  std::vector<int32_t> deg(n);
  INK_TRY(hipMemcpy(off.data(), c->gin.off, sizeof(int64_t) * (size_t)n, hipMemcpyDeviceToHost));
  INK_TRY(hipMemcpy(deg.data(), c->gin.deg, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost));
  rowptr[0] = 0;
  for (int v = 0; v < n; v++) rowptr[v + 1] = rowptr[v] + deg[v];
  if (!col) return hipSuccess;
  std::vector<int32_t> pool((size_t)c->gin.pool_top);
  INK_TRY(hipMemcpy(pool.data(), c->gin.ids, sizeof(int32_t) * pool.size(), hipMemcpyDeviceToHost));
  for (int v = 0; v < n; v++) {
    std::copy(pool.begin() + off[v], pool.begin() + off[v] + deg[v], col + rowptr[v]);
    std::sort(col + rowptr[v], col + rowptr[v + 1]);
  }
  return hipSuccess;
}

// ------------------------------------------------------------------------------- batch kernels
// Also validates the batch: a bad entry sets *err, and no kernel uses an id as an index before
// k_mark_last has seen *err and dropped every entry.
__global__ void k_unpack(const RawUpdate *raw, int64_t n, int n_nodes, uint32_t *src, uint32_t *dst, uint32_t *pos,
                         int32_t *err) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  RawUpdate a = raw[i];
  int e = entry_error(a, n_nodes);
  if (e) atomicOr(err, e);
  src[i] = (uint32_t)a.src;
  dst[i] = (uint32_t)a.dst;
  pos[i] = (uint32_t)i;
}

__global__ void k_gather_u32(const uint32_t *table, const uint32_t *idx, int64_t n, uint32_t *out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = table[idx[i]];
}

// entry j (in (dst, src, position) order) is the final word on its edge if the next entry names
// another edge; self loops never count
__global__ void k_mark_last(const RawUpdate *raw, const uint32_t *perm, int64_t n, uint8_t *flag, const int32_t *err) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  if (*err) { flag[j] = 0; return; }
  RawUpdate a = raw[perm[j]];
  bool last = true;
  if (j + 1 < n) {
    RawUpdate b = raw[perm[j + 1]];
    last = (a.src != b.src) || (a.dst != b.dst);
  }
  flag[j] = last && a.src != a.dst;
}

// unique ops in (dst, src) order: node = dst, other = src, op = final op
__global__ void k_take_ops(const RawUpdate *raw, const uint32_t *perm, const int32_t *idx, const int32_t *count,
                           uint32_t *node, int32_t *other, uint8_t *op, int32_t *pos) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= *count) return;
  RawUpdate a = raw[perm[idx[k]]];
  node[k] = (uint32_t)a.dst;
  other[k] = a.src;
  op[k] = a.op;
  pos[k] = -1;
}


__global__ void k_chunk_counts(const int32_t *nodes, const int32_t *n_nodes, int64_t n_max, const int32_t *deg,
                               int32_t *chunks) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_max) return;
  chunks[i] = i < *n_nodes ? (deg[nodes[i]] + kChunk - 1) / kChunk : 0;
}

// Walk the blocks of the touched nodes; an id found in the node's op list records its slot.
__global__ __launch_bounds__(256) void k_classify(const int32_t *nodes, const int32_t *n_nodes, const int32_t *seg,
                                                  const int32_t *chunk_pref, const int32_t *n_chunks,
                                                  const int64_t *off, const int32_t *deg, const int32_t *ids,
                                                  const int32_t *other, int32_t *pos) {
  int total = *n_chunks, nn = *n_nodes;
  for (int ch = blockIdx.x; ch < total; ch += gridDim.x) {
    // node owning this chunk: last i with chunk_pref[i] <= ch
    int i = wave_last_le(chunk_pref, nn, ch);
    int v = nodes[i];
    int s0 = seg[i], s1 = seg[i + 1];
    int d = deg[v];
    int64_t base = off[v];
    int p0 = (ch - chunk_pref[i]) * kChunk;
    int p1 = p0 + kChunk < d ? p0 + kChunk : d;
    for (int p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
      int e = ids[base + p];
      int a = s0, b = s1 - 1;
      while (a <= b) {
        int m = (a + b) >> 1;
        int x = other[m];
        if (x == e) {
          pos[m] = p;
          break;
        }
        if (x < e) a = m + 1; else b = m - 1;
      }
    }
  }
}

// per touched node: effective op flags, counts and the pool space a relocation would need.
// eff: 0 no-op, 1 insert, 2 delete.  One wave per node.
__global__ __launch_bounds__(256) void k_effect(const int32_t *nodes, const int32_t *n_nodes, const int32_t *seg,
                                                const uint8_t *op, const int32_t *pos, uint8_t *eff,
                                                const int32_t *deg, const int32_t *cap, int32_t *nd_ins,
                                                int32_t *nd_del, float slack, Counters *cnt, int st_need,
                                                int st_ins, int st_del) {
  int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  int l = threadIdx.x & (kWave - 1);
  if (w >= *n_nodes) return;
  int s0 = seg[w], s1 = seg[w + 1];
  int ni = 0, nd = 0;
  for (int k = s0 + l; k < s1; k += kWave) {
    int e = 0;
    if (op[k] == 0) e = pos[k] < 0 ? 1 : 0;
    else e = pos[k] >= 0 ? 2 : 0;
    eff[k] = (uint8_t)e;
    ni += e == 1;
    nd += e == 2;
  }
  for (int o = 32; o > 0; o >>= 1) { ni += __shfl_xor(ni, o, kWave); nd += __shfl_xor(nd, o, kWave); }
  if (l == 0) {
    int v = nodes[w];
    nd_ins[w] = ni; nd_del[w] = nd;
    int nd2 = deg[v] - nd + ni;
    if (nd2 > cap[v])      // pool space needed
      atomicAdd(&cnt->stripe[blockIdx.x % kStripes][st_need], (unsigned long long)relocated_cap(nd2, cap[v], slack));
    if (ni) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][st_ins], (unsigned long long)ni);  // effective inserts
    if (nd) atomicAdd(&cnt->stripe[blockIdx.x % kStripes][st_del], (unsigned long long)nd);  // effective deletes
  }
}

// ---- apply: refill deleted slots from the tail, relocate if the block is too small, append inserted ids
struct ApplySide {              // op lists and store of one direction (device pointers)
  const int32_t *uniq, *seg, *other; const uint8_t *op; int32_t *pos;
  const int32_t *nd_ins, *nd_del;
  const int32_t *n_uniq;        // touched nodes
  int64_t *off; int32_t *deg, *cap, *ids; uint8_t *asc;
  unsigned long long *pool_used, pool_base;
  int32_t *fill;                // one slot per op
  int32_t *new_cnt;             // per node: ids appended by this batch (out side), or null
};
// One workgroup per touched node and side: workgroups [0, n_max) take the in side, the next n_max the out
// side; those past a side's device-side node count leave.  A node with at most 64 ops (nearly all) is
// handled by one wave without a barrier, the other waves only help to move its block.
__global__ __launch_bounds__(256) void k_apply(ApplySide in, ApplySide out, int n_max, float slack, const int32_t *ok) {
  __shared__ int sm[kScanThreads / kWave + 1];
  __shared__ long long s_newoff;
  const bool second = (int)blockIdx.x >= n_max;
  const ApplySide &g = second ? out : in;
  const int i = (int)blockIdx.x - (second ? n_max : 0);
  if ((ok && !*ok) || i >= *g.n_uniq) return;
  const int ni = g.nd_ins[i], nd = g.nd_del[i];
  if (ni == 0 && nd == 0) return;
  const int v = g.uniq[i];
  const int s0 = g.seg[i], s1 = g.seg[i + 1];
  // every thread reads the descriptor here; it is written back after the last barrier
  const int64_t base0 = g.off[v];
  const int d0 = g.deg[v], cap0 = g.cap[v];
  __syncthreads();
  const int d1 = d0 - nd, d2 = d1 + ni;   // survivors, new degree
  int32_t *ids = g.ids + base0;
  const bool one_wave = s1 - s0 <= kWave;
  const int l = lane_id(), w = threadIdx.x / kWave;
  if (nd > 0) {
    if (one_wave) {
      if (w == 0) {
        const int k = s0 + l;
        const int pos = k < s1 ? g.pos[k] : -1;
        fill_holes(ids, d1, nd, pos, k < s1 && effect_of(g.op[k], pos) == 2);
      }
    } else {
      for (int k = s0 + threadIdx.x; k < s1; k += blockDim.x)
        if (effect_of(g.op[k], g.pos[k]) == 2) ids[g.pos[k]] = -1;
      __threadfence_block();
      __syncthreads();
      // survivors in the tail [d1, d0), in slot order -> fill[s0 ...]
      int carry = 0;
      for (int p0 = d1; p0 < d0; p0 += kScanThreads) {
        int p = p0 + threadIdx.x;
        int e = p < d0 ? ids[p] : -1;
        int tot;
        int ex = block_excl_scan(e >= 0 ? 1 : 0, sm, &tot);
        if (e >= 0) g.fill[s0 + carry + ex] = e;
        carry += tot;
        __syncthreads();
      }
      __threadfence_block();
      __syncthreads();
      // holes in the head [0, d1), in op order, take them in turn
      carry = 0;
      for (int k0 = s0; k0 < s1; k0 += kScanThreads) {
        int k = k0 + threadIdx.x;
        bool hole = k < s1 && effect_of(g.op[k], g.pos[k]) == 2 && g.pos[k] < d1;
        int tot;
        int ex = block_excl_scan(hole ? 1 : 0, sm, &tot);
        if (hole) ids[g.pos[k]] = g.fill[s0 + carry + ex];
        carry += tot;
        __syncthreads();
      }
    }
  }
  const bool move = d2 > cap0;        // workgroup-uniform
  long long want = cap0;
  int64_t base = base0;
  if (move) {
    want = relocated_cap(d2, cap0, slack);
    if (threadIdx.x == 0) s_newoff = (long long)(g.pool_base + atomicAdd(g.pool_used, (unsigned long long)want));
    __threadfence_block();
    __syncthreads();
    base = s_newoff;
    int32_t *to = g.ids + base;
    for (int p = threadIdx.x; p < d1; p += blockDim.x) to[p] = ids[p];
    ids = to;
  }
  if (ni > 0) {
    if (one_wave) {
      if (w == 0) {
        const int k = s0 + l;
        const bool ins = k < s1 && effect_of(g.op[k], g.pos[k]) == 1;
        const uint64_t m = __ballot(ins);
        if (ins) ids[d1 + __popcll(m & ((1ull << l) - 1))] = g.other[k];
      }
    } else {
      int carry = 0;
      for (int k0 = s0; k0 < s1; k0 += kScanThreads) {
        int k = k0 + threadIdx.x;
        bool ins = k < s1 && effect_of(g.op[k], g.pos[k]) == 1;
        int tot;
        int ex = block_excl_scan(ins ? 1 : 0, sm, &tot);
        if (ins) ids[d1 + carry + ex] = g.other[k];
        carry += tot;
        __syncthreads();
      }
    }
  }
  if (threadIdx.x == 0) {
    if (move) { g.cap[v] = (int32_t)want; g.off[v] = base; }
    g.deg[v] = d2;
    g.asc[v] = 0;              // holes were refilled from the tail / ids appended: order no longer known
    if (g.new_cnt) g.new_cnt[v] = ni;
  }
}

// effective ops -> Delta E lists in (node, other) order
__global__ void k_split_ops(const uint32_t *node, const int32_t *other, const uint8_t *eff, const int32_t *n_ops,
                            const int32_t *idx_ins, const int32_t *idx_del, int32_t *ins_s, int32_t *ins_d,
                            int32_t *del_s, int32_t *del_d, const int32_t *n_ins, const int32_t *n_del) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < *n_ins) { int j = idx_ins[k]; ins_s[k] = other[j]; ins_d[k] = (int32_t)node[j]; }
  if (k < *n_del) { int j = idx_del[k]; del_s[k] = other[j]; del_d[k] = (int32_t)node[j]; }
}
__global__ void k_flag_eq(const uint8_t *eff, const int32_t *n_ops, int64_t n_max, uint8_t want, uint8_t *flag) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_max) flag[k] = k < *n_ops && eff[k] == want;
}

// out side: ops = [deletes | inserts] keyed by source
__global__ void k_out_ops(const int32_t *del_s, const int32_t *del_d, const int32_t *ins_s, const int32_t *ins_d,
                          int n_del, int n_ins, uint32_t *key, uint32_t *val) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_del) { key[k] = (uint32_t)del_s[k]; val[k] = (uint32_t)k; }
  else if (k < n_del + n_ins) { key[k] = (uint32_t)ins_s[k - n_del]; val[k] = (uint32_t)k; }
}
// after a stable sort by source of entries that were in (dst, src) order per kind, entries of one
// source are not yet ordered by destination across the two kinds; a second stable sort fixes the
// order: we sort by destination first, then by source (both stable)
__global__ void k_out_dst_key(const int32_t *del_d, const int32_t *ins_d, int n_del, int n_ins, uint32_t *key,
                              uint32_t *val) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_del) { key[k] = (uint32_t)del_d[k]; val[k] = (uint32_t)k; }
  else if (k < n_del + n_ins) { key[k] = (uint32_t)ins_d[k - n_del]; val[k] = (uint32_t)k; }
}
__global__ void k_out_take(const uint32_t *perm, const int32_t *del_s, const int32_t *del_d, const int32_t *ins_s,
                           const int32_t *ins_d, int n_del, int n_ins, uint32_t *node, int32_t *other, uint8_t *op,
                           int32_t *pos) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_del + n_ins) return;
  int j = (int)perm[k];
  if (j < n_del) { node[k] = (uint32_t)del_s[j]; other[k] = del_d[j]; op[k] = 1; }
  else { node[k] = (uint32_t)ins_s[j - n_del]; other[k] = ins_d[j - n_del]; op[k] = 0; }
  pos[k] = -1;
}

__global__ void k_zero_at(const int32_t *nodes, int n, int32_t *arr) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) arr[nodes[i]] = 0;
}

__global__ void k_copy_blocks(int n, const int64_t *off, const int32_t *deg, const int32_t *src, int32_t *dst) {
  // one wave per node; offsets are unchanged (same layout in a larger pool)
  int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  int l = threadIdx.x & (kWave - 1);
  if (w >= n) return;
  int64_t o = off[w];
  int d = deg[w];
  for (int p = l; p < d; p += kWave) dst[o + p] = src[o + p];
}

static inline dim3 grid1(int64_t n, int per = 256) { return dim3((unsigned)std::max<int64_t>(1, (n + per - 1) / per)); }

struct Arena {
  char *base; size_t used = 0, cap;
  Arena(DevBuf &b) : base((char *)b.p), cap(b.cap) {}
  template <class T> T *get(size_t n) {
    size_t bytes = (n * sizeof(T) + 255) & ~(size_t)255;
    T *p = (T *)(base + used);
    used += bytes;
    return p;
  }
};

static hipError_t grow_pool(ink_ctx *c, GraphSide &g, int64_t need_total) {
  int64_t new_cap = std::max<int64_t>(g.pool_cap * 2, g.pool_top + need_total + (1 << 20));
  int32_t *np = nullptr;
  INK_TRY(hipMalloc(&np, sizeof(int32_t) * (size_t)new_cap));
  hipLaunchKernelGGL(k_copy_blocks, grid1((int64_t)c->n * kWave), dim3(256), 0, c->stream, c->n,
                     (const int64_t *)g.off, (const int32_t *)g.deg, (const int32_t *)g.ids, np);
  INK_TRY(hipStreamSynchronize(c->stream));
  INK_TRY(hipFree(g.ids));
  g.ids = np;
  g.pool_cap = new_cap;
  return hipSuccess;
}

// empty blocks of kNewNodeCap slots for the nodes n0 .. n0 + n_new - 1 at the pool's top
constexpr int kNewNodeCap = 4;
__global__ void k_init_blocks(int64_t *off, int32_t *deg, int32_t *cap, int32_t *ids, int n0, int64_t n_new, int64_t top) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_new) return;
  int64_t o = top + i * kNewNodeCap;
  off[n0 + i] = o; deg[n0 + i] = 0; cap[n0 + i] = kNewNodeCap;
  for (int k = 0; k < kNewNodeCap; k++) ids[o + k] = -1;
}

ink_status graph_add_nodes(ink_ctx *c, int64_t n_new) {
  for (GraphSide *g : {&c->gin, &c->gout}) {
    int64_t need = n_new * kNewNodeCap;
    if (g->pool_top + need > g->pool_cap) {
      hipError_t e = grow_pool(c, *g, need);
      if (e == hipErrorOutOfMemory) { c->err = "out of device memory while growing the edge pool"; return INK_E_OOM; }
      INK_TRYS(e);
    }
    hipLaunchKernelGGL(k_init_blocks, grid1(n_new), dim3(256), 0, c->stream, g->off, g->deg, g->cap, g->ids, c->n, n_new,
                       g->pool_top);
    INK_TRYS(hipGetLastError());
    g->pool_top += need;
  }
  return INK_OK;
}

// A kernel found a malformed entry and dropped the whole batch before any block was touched:
// clear the flag and report.
static ink_status batch_error(ink_ctx *c) {
  int e = c->h_cnt->v[C_ERR];
  INK_TRYS(hipMemsetAsync(&c->d_cnt->v[C_ERR], 0, sizeof(int32_t), c->stream));
  INK_TRYS(hipStreamSynchronize(c->stream));
  if (e & 2) { c->err = "ink_apply_updates: node id out of range"; return INK_E_RANGE; }
  c->err = "ink_apply_updates: op must be 0 (insert) or 1 (delete)";
  return INK_E_ARG;
}

// One direction.  Ops (node, other, op, pos) are in (node, other) order on the device; n_ops is
// known on the host.  all_effective: presence was already established (out side).
struct SideBufs {
  uint32_t *node; int32_t *other; uint8_t *op; int32_t *pos; uint8_t *eff;
  int32_t *uniq, *seg, *chunks, *chunk_pref, *nd_ins, *nd_del, *fill;
};

// n_ops_max bounds the number of ops; the exact count sits on the device in *n_ops_dev.  One host
// round trip per direction: it returns the touched-node count, the totals and the pool space
// that relocations need.
static ink_status apply_side(ink_ctx *c, GraphSide &g, SideBufs &b, int64_t n_ops_max, const int32_t *n_ops_dev,
                             int32_t *new_cnt, int *n_touched_out, int64_t *tot_ins, int64_t *tot_del) {
  hipStream_t s = c->stream;
  Counters *dc = c->d_cnt;
  // scratch slots, the 64-bit slot and the stripes in one fill (the batch's op count sits before them)
  INK_TRYS(hipMemsetAsync(&dc->v[C_TMP0], 0, sizeof(Counters) - C_TMP0 * sizeof(int32_t), s));
  INK_TRYS(segment_heads(c->ws, b.node, n_ops_max, b.uniq, b.seg, &dc->v[C_TMP0], s, n_ops_dev));
  hipLaunchKernelGGL(k_chunk_counts, grid1(n_ops_max), dim3(256), 0, s, (const int32_t *)b.uniq,
                     (const int32_t *)&dc->v[C_TMP0], n_ops_max, (const int32_t *)g.deg, b.chunks);
  INK_TRYS(scan_excl_i32(c->ws, b.chunks, b.chunk_pref, n_ops_max, &dc->v[C_TMP1], s));
  hipLaunchKernelGGL(k_classify, dim3(2048), dim3(256), 0, s, (const int32_t *)b.uniq, (const int32_t *)&dc->v[C_TMP0],
                     (const int32_t *)b.seg, (const int32_t *)b.chunk_pref, (const int32_t *)&dc->v[C_TMP1],
                     (const int64_t *)g.off, (const int32_t *)g.deg, (const int32_t *)g.ids, (const int32_t *)b.other, b.pos);
  hipLaunchKernelGGL(k_effect, grid1(n_ops_max * kWave), dim3(256), 0, s, (const int32_t *)b.uniq,
                     (const int32_t *)&dc->v[C_TMP0], (const int32_t *)b.seg, (const uint8_t *)b.op,
                     (const int32_t *)b.pos, b.eff, (const int32_t *)g.deg, (const int32_t *)g.cap, b.nd_ins, b.nd_del,
                     c->slack, dc, (int)ST_REGATHER, (int)ST_EXPOSED, (int)ST_ACHG);
  INK_TRYS(read_counters(c));
  if (c->h_cnt->v[C_ERR]) return batch_error(c);
  int n_touched = c->h_cnt->v[C_TMP0];
  *n_touched_out = n_touched;
  int64_t need = (int64_t)c->h_cnt->sum(ST_REGATHER);
  *tot_ins = (int64_t)c->h_cnt->sum(ST_EXPOSED);
  *tot_del = (int64_t)c->h_cnt->sum(ST_ACHG);
  if (n_touched == 0) return INK_OK;
  if (g.pool_top + need > g.pool_cap) {
    hipError_t e = grow_pool(c, g, need);
    if (e == hipErrorOutOfMemory) { c->err = "out of device memory while growing the edge pool"; return INK_E_OOM; }
    INK_TRYS(e);
  }
  // blocks that move take their space at the pool's top: base by value, the amount handed out so
  // far in a 64-bit slot of the counter block (zero since the fill above)
  unsigned long long *d_used = (unsigned long long *)&dc->v[C_TOP64];
  const ApplySide a{b.uniq, b.seg, b.other, b.op, b.pos, b.nd_ins, b.nd_del, &dc->v[C_TMP0], g.off, g.deg, g.cap, g.ids, g.asc,
                    d_used, (unsigned long long)g.pool_top, b.fill, new_cnt};
  hipLaunchKernelGGL(k_apply, dim3(n_touched), dim3(256), 0, s, a, a, n_touched, c->slack, (const int32_t *)nullptr);
  INK_TRYS(hipGetLastError());
  g.pool_top += need;      // exact: the apply kernel allocates precisely what k_effect summed
  return INK_OK;
}

// ------------------------------------------------------------ short batches
// A batch of at most kShortBatch entries goes through the same steps in four launches (up to 1024 entries)
// or six: sort the entries by (node, other end, position) for both directions and build the op lists of
// the touched nodes; walk the touched blocks of both directions; effective ops, Delta E, what the blocks need;
// apply both directions.  One record goes to the host, and nothing is written to the store before
// the apply kernel, which the device itself allows (C_OK) if the batch is valid and the pools have room.
// An entry that a later one on the same edge overrides, or a self loop, stays in the lists as a dead op.
// Bound by the latency of its few launches and of one round trip; measured per update call with 10 000
// entries on 612 k nodes / 15.5 M edges: 0.15 ms less than two sequential sides with two round trips, with 1 to 500
// entries 0.03 - 0.06 ms less.  Its six launches for 10 000 entries take 84 us: sort 13, merge 12, heads 8, walk 24, finish 10, apply
// 18 (205 with a workgroup a side for heads and finish that took 1024 entries a turn, 149 when it took all at once).
constexpr int kOneChunk = 1024;        // entries that one workgroup sorts
constexpr int kMaxChunks = (int)(kShortBatch / kOneChunk);


struct ShortSide {           // op lists of one direction (device pointers), in (node, other) order
  int32_t *node, *other; uint8_t *op; int32_t *pos;
  int32_t *uniq, *seg, *chunk_pref;
  int32_t *nd_ins, *nd_del, *fill;
  int32_t *head;                       // per op: its node's place in uniq if it is the node's first, else -1
  const int64_t *off; const int32_t *deg, *cap, *ids;
  int64_t *uoff; int32_t *udeg, *ucap; // the touched nodes' blocks, one behind the other
  uint64_t *skey; int32_t *sidx;       // sorted chunks (batches of more than one)
  int64_t *eoff; int32_t *edeg, *ecap; // the blocks of the ops' nodes (batches of more than one chunk)
  int slot_n, slot_ch;                 // touched nodes, chunks of their blocks (slots of the graph counters)
};

// THREADS (key, index) pairs, one per thread in, sorted in A out: every wave sorts its 64 by rank, then
// runs are merged pairwise, an element's rank in the sibling run found by binary search in LDS.
template <int THREADS> struct SortLds { uint64_t k[2][THREADS]; int32_t i[2][THREADS]; };
template <int THREADS>
__device__ __forceinline__ int block_sort(SortLds<THREADS> &S, uint64_t key, int idx) {
  const int l = lane_id(), t = threadIdx.x;
  const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
  int rank = 0;
  for (int j = 0; j < kWave; j++) {
    const uint64_t kj = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, j) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)lo, j);
    rank += (kj < key) | ((kj == key) & (j < l));
  }
  int cur = 0, p = (t & ~(kWave - 1)) + rank;
  S.k[0][p] = key; S.i[0][p] = idx;
  __syncthreads();
  for (int len = kWave; len < THREADS; len <<= 1) {
    const uint64_t k = S.k[cur][t];
    const int id = S.i[cur][t];
    const int run = t & ~(len - 1), pair = t & ~(2 * len - 1);
    const bool left = run == pair;
    const uint64_t *sib = &S.k[cur][left ? pair + len : pair];
    int a = 0, b = len;        // sibling elements before mine: smaller ones; for the right run also equal ones
    while (a < b) {
      const int m = (a + b) >> 1;
      if (left ? sib[m] < k : sib[m] <= k) a = m + 1; else b = m;
    }
    const int q = pair + (t - run) + a;
    S.k[cur ^ 1][q] = k; S.i[cur ^ 1][q] = id;
    cur ^= 1;
    __syncthreads();
  }
  return cur;
}

// slots 0 .. 31 from zero, except the four that the two sides' workgroups set themselves
__device__ __forceinline__ void clear_graph_slots(Counters *g, int err) {
  const int i = threadIdx.x;
  if (i < 32 && i != C_TMP0 && i != C_TMP1 && i != C_OT && i != C_OCH) g->v[i] = i == C_ERR ? err : 0;
  if (i < 2) g->stripe[0][i] = 0;      // what the sides need of the pools
}

// Distinct nodes of the sorted op list (node of op i: node(i), n <= THREADS ops), the start of each node's ops plus the
// closing offset, the prefix of the chunk counts of their blocks, and both totals.  sm: LDS of the scans.
template <int THREADS, class NodeAt>
__device__ __forceinline__ void heads_and_chunks(NodeAt node, int n, const ShortSide &o, int *sm, Counters *g) {
  const int i = threadIdx.x;
  const int v = i < n ? node(i) : -1;
  const int h = i < n && (i == 0 || v != node(i - 1));
  int n_uniq, n_ch;
  const int ex = block_excl_scan<THREADS>(h, sm, &n_uniq);
  if (h) { o.uniq[ex] = v; o.seg[ex] = i; }
  if (i < n) o.head[i] = h ? ex : -1;
  if (i == 0) o.seg[n_uniq] = n;
  __threadfence_block();
  __syncthreads();
  int ch = 0;
  if (i < n_uniq) {
    const int u = o.uniq[i], d = o.deg[u];
    o.udeg[i] = d; o.ucap[i] = o.cap[u]; o.uoff[i] = o.off[u];
    ch = (d + kChunk - 1) / kChunk;
  }
  const int ec = block_excl_scan<THREADS>(ch, sm, &n_ch);
  if (i < n_uniq) o.chunk_pref[i] = ec;
  if (i == 0) { g->v[o.slot_n] = n_uniq; g->v[o.slot_ch] = n_ch; }
}

// Up to THREADS entries: one workgroup per side does everything up to the op lists.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_short_one(const RawUpdate *raw, int n, int n_nodes, ShortSide in, ShortSide out, Counters *g) {
  __shared__ SortLds<THREADS> S;
  __shared__ int sm[THREADS / kWave + 1];
  const int side = blockIdx.x, t = threadIdx.x;
  const ShortSide &o = side ? out : in;
  RawUpdate a{};
  int bad = 0;
  if (t < n) { a = raw[t]; bad = entry_error(a, n_nodes); }
  const int any_bad = __syncthreads_or(bad & 1) | (__syncthreads_or(bad & 2) ? 2 : 0);
  if (side == 0) clear_graph_slots(g, any_bad);
  if (any_bad) {              // drop the batch: nothing below uses an id as an index
    if (t == 0) { g->v[o.slot_n] = 0; g->v[o.slot_ch] = 0; o.seg[0] = 0; }
    return;
  }
  const int cur = block_sort<THREADS>(S, t < n ? update_key(a, side) : kNoKey, t | (a.op << 16));
  const uint64_t *sk = S.k[cur];
  if (t < n) {
    const uint64_t k = sk[t];
    const int node = (int)(k >> 32), other = (int)(uint32_t)k;
    const bool dead = (t + 1 < n && sk[t + 1] == k) || node == other;
    o.node[t] = node; o.other[t] = other; o.op[t] = (uint8_t)(dead ? 2 : S.i[cur][t] >> 16); o.pos[t] = -1;
  }
  heads_and_chunks<THREADS>([&](int i) { return (int)(sk[i] >> 32); }, n, o, sm, g);
}

// More entries: chunks of 1024 sorted by one workgroup each (grid: chunks of the in side, then of the out side) ...
__global__ __launch_bounds__(kOneChunk) void k_short_sort(const RawUpdate *raw, int n, int n_nodes, int n_chunks, ShortSide in,
                                                          ShortSide out, int32_t *chunk_err) {
  __shared__ SortLds<kOneChunk> S;
  const int side = (int)blockIdx.x >= n_chunks, ch = (int)blockIdx.x - (side ? n_chunks : 0), t = threadIdx.x;
  const ShortSide &o = side ? out : in;
  const int i = ch * kOneChunk + t;
  RawUpdate a{};
  int bad = 0;
  if (i < n) { a = raw[i]; bad = entry_error(a, n_nodes); }
  const int any_bad = __syncthreads_or(bad & 1) | (__syncthreads_or(bad & 2) ? 2 : 0);
  if (side == 0 && t == 0) chunk_err[ch] = any_bad;
  const int cur = block_sort<kOneChunk>(S, i < n ? update_key(a, side) : kNoKey, i | (a.op << 16));
  o.skey[i] = S.k[cur][t];
  o.sidx[i] = S.i[cur][t];
}
__device__ __forceinline__ int batch_bad(const int32_t *chunk_err, int n_chunks) {      // whole wave
  static_assert(kMaxChunks <= kWave, "a lane per chunk");
  const int e = lane_id() < n_chunks ? chunk_err[lane_id()] : 0;
  return (__ballot(e & 1) ? 1 : 0) | (__ballot(e & 2) ? 2 : 0);
}
// ... and merged by rank: an element's place is the sum of its ranks in all chunks (the searches of one thread
// advance in step, so their loads are in flight together).  A workgroup has all keys of its side in LDS (ten steps of dependent
// reads took 31 us out of the L2, 10 chunks) and finds the places of 256 of them: the searches are what takes the time, and with
// 1024 a workgroup four times as many of them share a CU's LDS (10000 entries 26 -> 12 us, with the reads of a step asked for together).
constexpr int kMergeThreads = 256, kMergeParts = kOneChunk / kMergeThreads;
// Chunks a kernel is built for: the searches of a thread advance through all of them, and a chunk is 8 KB of a CU's 160, so up to ten leave
// room for two workgroups.  3 chunks, us, built for 4 / 10 / 16: 5.8 / 8.6 / 11.0; 4 6.0 / 8.2 / 11.1; 5 - / 8.6 / 11.2; 10 - / 9.0 / 11.7; 16 12.2.
constexpr int kMergeFew = 4, kMergeTwoOnCu = 160 * 1024 / 2 / (kOneChunk * (int)sizeof(uint64_t));
template <int C>               // at least n_chunks: chunks past them repeat the first, and what is found there is not used
__global__ __launch_bounds__(kMergeThreads) void k_short_merge(int n, int n_chunks, ShortSide in, ShortSide out, const int32_t *chunk_err) {
  const int part = (int)blockIdx.x % kMergeParts, b = (int)blockIdx.x / kMergeParts;
  const int side = b >= n_chunks, ch = b - (side ? n_chunks : 0), t = part * kMergeThreads + threadIdx.x;
  const ShortSide &o = side ? out : in;
  if (batch_bad(chunk_err, n_chunks)) return;
  __shared__ __align__(16) uint64_t S[C * kOneChunk];
  {
    constexpr int U = kOneChunk / 2 / kMergeThreads;      // 16 bytes a load, all under way together
    const ulonglong2 *src = reinterpret_cast<const ulonglong2 *>(o.skey) + threadIdx.x;
    ulonglong2 x[C][U];
#pragma unroll
    for (int c = 0; c < C; c++)
#pragma unroll
      for (int u = 0; u < U; u++) x[c][u] = src[(c < n_chunks ? c : 0) * (kOneChunk / 2) + u * kMergeThreads];
#pragma unroll
    for (int c = 0; c < C; c++)
#pragma unroll
      for (int u = 0; u < U; u++) reinterpret_cast<ulonglong2 *>(S)[c * (kOneChunk / 2) + u * kMergeThreads + threadIdx.x] = x[c][u];
  }
  __syncthreads();
  const int me = ch * kOneChunk + t;
  const uint64_t k = S[me];
  if (k == kNoKey) return;
  int lo[C];
#pragma unroll
  for (int c = 0; c < C; c++) lo[c] = 0;
  for (int step = kOneChunk / 2; step > 0; step >>= 1) {
    uint64_t x[C];
#pragma unroll
    for (int c = 0; c < C; c++) x[c] = S[c * kOneChunk + lo[c] + step - 1];
#pragma unroll
    for (int c = 0; c < C; c++) lo[c] += (x[c] < k) | ((x[c] == k) & (c < ch)) ? step : 0;      // equal keys of earlier chunks stand before, of later ones behind
  }
  int rank = t;
  bool dead = t + 1 < kOneChunk && S[me + 1] == k;
#pragma unroll
  for (int c = 0; c < C; c++) {
    // the search above covers 1023 elements; the last step settles the chunk's last one
    const uint64_t x = S[c * kOneChunk + lo[c]], y = S[c * kOneChunk + (lo[c] + 1 < kOneChunk ? lo[c] + 1 : lo[c])];
    const bool before = (x < k) | ((x == k) & (c < ch)), other = c < n_chunks && c != ch;
    rank += other ? lo[c] + (before ? 1 : 0) : 0;
    dead |= other && c > ch && (before ? (lo[c] + 1 < kOneChunk && y == k) : x == k);
  }
  const int node = (int)(k >> 32), end = (int)(uint32_t)k;
  dead |= node == end;
  o.node[rank] = node; o.other[rank] = end; o.op[rank] = (uint8_t)(dead ? 2 : o.sidx[me] >> 16); o.pos[rank] = -1;
  o.edeg[rank] = o.deg[node]; o.ecap[rank] = o.cap[node]; o.eoff[rank] = o.off[node];       // here many workgroups share the random reads
}

// Exclusive prefix of x over a workgroup of 1024, and the total, of two counts packed into 64 bits (sm: a slot per wave).
__device__ __forceinline__ uint64_t chunk_prefix(uint64_t x, uint64_t *sm, uint64_t *total) {
  const int l = lane_id(), w = threadIdx.x / kWave;
  uint64_t inc = x;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint64_t y = __shfl_up((unsigned long long)inc, o, kWave);
    if (l >= o) inc += y;
  }
  __syncthreads();                 // sm may still be read by the scan before
  if (l == kWave - 1) sm[w] = inc;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kOneChunk / kWave; i++) { before += i < w ? sm[i] : 0; all += sm[i]; }
  *total = all;
  return before + inc - x;
}

// The touched nodes of the merged entries: a workgroup has 1024 of them and counts what stands before them itself, so that
// nothing waits for another workgroup.  (One workgroup a side for all entries took 26 us for 10000, this takes 8.)
__global__ __launch_bounds__(kOneChunk) void k_short_heads(int n, int n_chunks, ShortSide in, ShortSide out, const int32_t *chunk_err,
                                                           Counters *g) {
  __shared__ uint64_t sm[kOneChunk / kWave];
  const int side = (int)blockIdx.x >= n_chunks, b = (int)blockIdx.x - (side ? n_chunks : 0), t = threadIdx.x;
  const ShortSide &o = side ? out : in;
  const int err = batch_bad(chunk_err, n_chunks);
  if (blockIdx.x == 0) clear_graph_slots(g, err);
  if (err) n = 0;
  // heads in the upper half, chunks of their blocks in the lower
  auto count = [](int pv, int v, int d) __attribute__((always_inline)) {
    return v != pv ? (1ull << 32) + (unsigned)((d + kChunk - 1) / kChunk) : 0ull;      // node ids are not negative
  };
  uint64_t part = 0, before, tot;
  const int i = b * kOneChunk + t;
  const uint64_t mine = i < n ? count(i > 0 ? o.node[i - 1] : -1, o.node[i], o.edeg[i]) : 0;
  if (!err)
    for (int k = t; k < b * (kOneChunk / 4); k += kOneChunk) {       // four entries a load
      const int pv = k > 0 ? o.node[4 * k - 1] : -1;
      const int4 v = reinterpret_cast<const int4 *>(o.node)[k], d = reinterpret_cast<const int4 *>(o.edeg)[k];
      part += count(pv, v.x, d.x) + count(v.x, v.y, d.y) + count(v.y, v.z, d.z) + count(v.z, v.w, d.w);
    }
  (void)chunk_prefix(part, sm, &before);
  const uint64_t at = before + chunk_prefix(mine, sm, &tot);
  const int u = (int)(at >> 32);
  if (mine) {
    o.uniq[u] = o.node[i]; o.seg[u] = i;
    o.udeg[u] = o.edeg[i]; o.ucap[u] = o.ecap[i]; o.uoff[u] = o.eoff[i];
    o.chunk_pref[u] = (int)(uint32_t)at;
  }
  if (i < n) o.head[i] = mine ? u : -1;
  if (b == n_chunks - 1 && t == 0) {
    const int n_uniq = (int)((before + tot) >> 32);
    o.seg[n_uniq] = n;
    g->v[o.slot_n] = n_uniq; g->v[o.slot_ch] = (int)(uint32_t)(before + tot);
  }
}

// Walk the blocks of the touched nodes of both sides, one chunk of slots per wave visit (most blocks are short: a
// workgroup per visit left three of its waves without work in their chains of loads); an id found in
// the node's op list records its slot (of several ops on one edge the last one, which is the live one, may
// not be missed).  Reads only: the blocks are walked with 16-byte loads, a node's few ops sit in registers, those of a hub in
// LDS, where every id looks for itself: out of the L2 the searches of one hub's chunk were the launch's end (10000 entries 37 -> 24 us).
constexpr int kClassifyOps = 1024;
__global__ __launch_bounds__(256) void k_short_classify(ShortSide in, ShortSide out, const Counters *g) {
  const int nch_in = g->v[in.slot_ch], total = nch_in + g->v[out.slot_ch];
  __shared__ int s_ops[256 / kWave][kClassifyOps];
  const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), wave = (int)(blockIdx.x * (256 / kWave)) + w;
  for (int c = wave; c < total; c += gridDim.x * (256 / kWave)) {
    const bool second = c >= nch_in;
    const ShortSide &o = second ? out : in;
    const int ch = second ? c - nch_in : c;
    const int i = wave_last_le(o.chunk_pref, g->v[o.slot_n], ch);      // node owning this chunk
    const int s0 = o.seg[i], cnt = o.seg[i + 1] - s0;
    const int d = o.udeg[i];
    const int32_t *ids = o.ids + o.uoff[i];      // blocks start on 16-byte boundaries and hold a multiple of 4 slots
    const int mine = o.other[s0 + (l < cnt ? l : 0)];
    const bool staged = cnt > 8 && cnt <= kClassifyOps;
    if (staged) {                                // read by this wave alone
      for (int m = l; m < cnt; m += kWave) s_ops[w][m] = o.other[s0 + m];
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    const int p_begin = (ch - o.chunk_pref[i]) * kChunk, p_end = p_begin + kChunk < d ? p_begin + kChunk : d;
    constexpr int U = 4;                         // loads under way
    for (int p0 = p_begin; p0 < p_end; p0 += 4 * kWave * U) {
     int4 q[U];
#pragma unroll
     for (int u = 0; u < U; u++) {
       const int p = p0 + 4 * (u * kWave + l);
       q[u] = p0 + 4 * u * kWave < p_end ? *reinterpret_cast<const int4 *>(ids + (p < p_end ? p : p0)) : make_int4(-1, -1, -1, -1);
     }
#pragma unroll
     for (int u = 0; u < U; u++) {
      const int p = p0 + 4 * (u * kWave + l);
      if (p0 + 4 * u * kWave >= p_end) break;
      const int e[4] = {p < p_end ? q[u].x : -1, p < p_end ? q[u].y : -1, p < p_end ? q[u].z : -1, p < p_end ? q[u].w : -1};
      if (cnt <= 8) {
        for (int m = 0; m < cnt; m++) {
          const int x = __builtin_amdgcn_readlane(mine, m);
#pragma unroll
          for (int j = 0; j < 4; j++)
            if (e[j] == x && p + j < d) o.pos[s0 + m] = p + j;
        }
      } else if (staged) {
        int a[4] = {0, 0, 0, 0};                 // ops whose other end is not beyond e, the last of them left to the end
        for (int len = cnt; len > 1; len -= len >> 1) {
#pragma unroll
          for (int j = 0; j < 4; j++) a[j] += s_ops[w][a[j] + (len >> 1) - 1] <= e[j] ? len >> 1 : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
          a[j] += s_ops[w][a[j]] <= e[j];
          if (a[j] > 0 && s_ops[w][a[j] - 1] == e[j] && p + j < d) o.pos[s0 + a[j] - 1] = p + j;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; j++) {
          int a = s0, b = s0 + cnt;              // first op whose other end is beyond e
          while (a < b) {
            const int m = (a + b) >> 1;
            if (o.other[m] <= e[j]) a = m + 1; else b = m;
          }
          if (a > s0 && o.other[a - 1] == e[j] && p + j < d) o.pos[a - 1] = p + j;
        }
      }
     }
    }
  }
}

// Effective ops: Delta E in (dst, src) order (in side), insertions and deletions per touched node, the pool space that
// relocations need.  A workgroup has 1024 ops of a side and the nodes whose first op is among them; what stands before its ops, and
// the ops of its last node that lie beyond them, it counts itself.  The workgroup that ends last decides whether the batch may be
// applied and publishes the record.  (One workgroup a side took 29 us for 10000 ops, this takes 10.)
__global__ __launch_bounds__(kOneChunk) void k_short_finish(int n, int n_chunks, ShortSide in, ShortSide out, int32_t *ins_s, int32_t *ins_d,
                                                            int32_t *del_s, int32_t *del_d, float slack, long long room_in,
                                                            long long room_out, Counters *g, HostCounters *h, uint32_t *h_seq,
                                                            uint32_t seq) {
  static_assert(kShortBatch < 1 << 16, "insertions in the low half, deletions in the high half");
  __shared__ int sm[kOneChunk / kWave], sp[kOneChunk / kWave];
  __shared__ int P[kOneChunk + 1];               // effective ops among the workgroup's first t
  __shared__ unsigned long long s_need;
  __shared__ int s_tail, s_beyond, s_last;
  const int side = (int)blockIdx.x >= n_chunks, b = (int)blockIdx.x - (side ? n_chunks : 0), t = threadIdx.x;
  const int l = lane_id(), w = t / kWave;
  const ShortSide &o = side ? out : in;
  const int n_ops = g->v[o.slot_n] ? n : 0;      // none after a malformed entry
  auto count = [](int op, int pos) __attribute__((always_inline)) { const int e = effect_of(op, pos); return e == 1 ? 1 : e == 2 ? 1 << 16 : 0; };
  const int i = b * kOneChunk + t, end = (b + 1) * kOneChunk;
  const int mine = i < n_ops ? count(o.op[i], o.pos[i]) : 0;
  const int u = i < n_ops ? o.head[i] : -1;
  int part = 0;
  if (n_ops)
    for (int k = t; k < b * (kOneChunk / 4); k += kOneChunk) {       // four ops a load
      const uchar4 op = reinterpret_cast<const uchar4 *>(o.op)[k];
      const int4 pos = reinterpret_cast<const int4 *>(o.pos)[k];
      part += count(op.x, pos.x) + count(op.y, pos.y) + count(op.z, pos.z) + count(op.w, pos.w);
    }
  const int stop = u >= 0 ? o.seg[u + 1] : 0, dg = u >= 0 ? o.udeg[u] : 0, cap = u >= 0 ? o.ucap[u] : 0;
#pragma unroll
  for (int k = kWave / 2; k > 0; k >>= 1) part += __shfl_xor(part, k, kWave);
  const uint64_t below = (1ull << l) - 1, mi = __ballot(mine == 1), md = __ballot(mine > 1);
  if (l == 0) { sm[w] = __popcll(mi) + (__popcll(md) << 16); sp[w] = part; }
  if (t == 0) { s_tail = -1; s_beyond = 0; s_need = 0; }
  __syncthreads();
  int before = 0, here = __popcll(mi & below) + (__popcll(md & below) << 16), tot = 0;
#pragma unroll
  for (int k = 0; k < kOneChunk / kWave; k++) { before += sp[k]; here += k < w ? sm[k] : 0; tot += sm[k]; }
  const int at = before + here;
  P[t] = here;
  if (t == 0) P[kOneChunk] = tot;
  if (stop > end) s_tail = stop;                 // the last node's, if any
  if (side == 0 && mine == 1) { ins_s[at & 0xFFFF] = o.other[i]; ins_d[at & 0xFFFF] = o.node[i]; }
  else if (side == 0 && mine) { del_s[at >> 16] = o.other[i]; del_d[at >> 16] = o.node[i]; }
  __syncthreads();
  if (s_tail > 0) {
    int beyond = 0;
    for (int k = end + t; k < s_tail; k += kOneChunk) beyond += count(o.op[k], o.pos[k]);
    if (beyond) atomicAdd(&s_beyond, beyond);
    __syncthreads();
  }
  if (u >= 0) {
    const int x = P[stop < end ? stop - b * kOneChunk : kOneChunk] - P[t] + (stop > end ? s_beyond : 0);
    const int ni = x & 0xFFFF, nd = x >> 16;
    o.nd_ins[u] = ni; o.nd_del[u] = nd;
    const int d2 = dg - nd + ni;
    if (d2 > cap) atomicAdd(&s_need, (unsigned long long)relocated_cap(d2, cap, slack));
  }
  __syncthreads();
  if (t == 0) {
    if (b == n_chunks - 1) {
      const int total = before + tot;
      __hip_atomic_store(&g->v[side ? C_OINS : C_GINS], total & 0xFFFF, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&g->v[side ? C_ODEL : C_GDEL], total >> 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (s_need) atomicAdd(&g->stripe[0][side], s_need);      // cleared with the slots; the other stripes stay 0
    __threadfence();
    s_last = atomicAdd(&g->v[C_NC], 1) == (int)gridDim.x - 1;      // slot unused otherwise by the graph stage
    __threadfence();
    if (s_last) {
      auto rd = [&](int s) { return __hip_atomic_load(&g->v[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      auto needs = [&](int k) { return (long long)__hip_atomic_load(&g->stripe[0][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      const int ni = rd(C_GINS), nd = rd(C_GDEL);
      const bool ok = rd(C_ERR) == 0 && needs(0) <= room_in && needs(1) <= room_out && rd(C_OINS) == ni && rd(C_ODEL) == nd;
      __hip_atomic_store(&g->v[C_OK], ok ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&g->v[C_TMP2], ok ? ni : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&g->v[C_TMP3], ok ? nd : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __threadfence();
    }
  }
  __syncthreads();
  if (s_last && t < kWave) publish_wave(g, h, h_seq, seq);
}

// The stage by itself: batches of models whose layers do not take the one-workgroup form.
__global__ __launch_bounds__(1024) void k_graph_one(OneGraph p, Counters *g, HostCounters *h, uint32_t *h_seq, uint32_t seq) {
  __shared__ OneGraphLds S;
  __shared__ HostCounters record;
  graph_one(S, p, record);
  const int l = threadIdx.x;
  if (l >= kWave) return;
  if (l < 32) { g->v[l] = record.v[l]; h->v[l] = record.v[l]; }
  if (l < ST_N) h->total[l] = record.total[l];
  __threadfence_system();
  if (l == 0) __hip_atomic_store(h_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

static size_t short_bytes(int64_t n) {
  const size_t pad = (size_t)(n + kOneChunk - 1) / kOneChunk * kOneChunk;
  return 2 * (pad * 12 + 22 * ((size_t)(n + 64) * 4 + 256)) + 4096;
}

hipError_t graph_reserve(ink_ctx *c, int64_t max_batch) {
  const size_t per = (((size_t)max_batch + 64) * 4 + 255) / 256 * 256;
  INK_TRY(c->b_misc.reserve(std::max(per * 28, short_bytes(std::min(max_batch, kShortBatch)))));
  for (DevBuf *b : {&c->b_del_s, &c->b_del_d, &c->b_ins_s, &c->b_ins_d, &c->b_touch_in, &c->b_uniq}) INK_TRY(b->reserve(per));
  return hipSuccess;
}

static ApplySide apply_side_of(const ShortSide &b, GraphSide &g, Counters *gc, int slot_top, int32_t *new_cnt) {
  return ApplySide{b.uniq, b.seg, b.other, b.op, b.pos, b.nd_ins, b.nd_del, &gc->v[b.slot_n], g.off, g.deg, g.cap, g.ids, g.asc,
                   (unsigned long long *)&gc->v[slot_top], (unsigned long long)g.pool_top, b.fill, new_cnt};
}

static ink_status short_error(ink_ctx *c, const int32_t *v) {
  if (v[C_ERR]) {      // the whole batch was dropped before any block was touched
    if (v[C_ERR] & 2) { c->err = "ink_apply_updates: node id out of range"; return INK_E_RANGE; }
    c->err = "ink_apply_updates: op must be 0 (insert) or 1 (delete)";
    return INK_E_ARG;
  }
  if (v[C_OINS] != v[C_GINS] || v[C_ODEL] != v[C_GDEL]) {
    c->err = "graph store inconsistent: in- and out-adjacency disagree";
    return INK_E_DEVICE;
  }
  return INK_OK;
}

static void short_result(ink_ctx *c, const int64_t need[2], int64_t *n_ins_out, int64_t *n_del_out) {
  const int32_t *v = c->h_gcnt->v;
  c->gin.pool_top += need[0];
  c->gout.pool_top += need[1];
  c->n_ins = *n_ins_out = v[C_GINS];
  c->n_del = *n_del_out = v[C_GDEL];
  c->n_touched_in = v[C_TMP0];
  c->n_touched_src = c->n_ins + c->n_del > 0 ? v[C_OT] : 0;
}

// *done: the batch was within the limits of the one-workgroup form (or is in error)
static ink_status graph_apply_one(ink_ctx *c, const RawUpdate *raw, int64_t n, int64_t *n_ins_out, int64_t *n_del_out,
                                  hipError_t (*queued)(ink_ctx *, const OneGraph &, uint32_t), bool *done) {
  const size_t per = ((size_t)(n + 64) * 4 + 255) & ~(size_t)255;
  for (DevBuf *b : {&c->b_del_s, &c->b_del_d, &c->b_ins_s, &c->b_ins_d, &c->b_touch_in, &c->b_uniq}) INK_TRYS(b->reserve(per));
  c->del_src = c->b_del_s.as<int32_t>(); c->del_dst = c->b_del_d.as<int32_t>();
  c->ins_src = c->b_ins_s.as<int32_t>(); c->ins_dst = c->b_ins_d.as<int32_t>();
  auto side = [](GraphSide &g, int32_t *new_cnt, DevBuf &uniq) {
    return OneSide{g.off, g.deg, g.cap, g.ids, g.asc, new_cnt, uniq.as<int32_t>(), (long long)g.pool_top, (long long)(g.pool_cap - g.pool_top)};
  };
  const OneGraph p{raw, (int)n, c->n, side(c->gin, nullptr, c->b_touch_in), side(c->gout, c->new_out, c->b_uniq),
                   c->ins_src, c->ins_dst, c->del_src, c->del_dst, c->slack};
  const uint32_t seq = ++c->pub_seq;
  if (queued) INK_TRYS(queued(c, p, seq));
  else {
    hipLaunchKernelGGL(k_graph_one, dim3(1), dim3(1024), 0, c->stream, p, c->d_gcnt, c->h_gcnt, c->h_gseq, seq);
    INK_TRYS(hipGetLastError());
  }
  INK_TRYS(wait_published(c, c->h_gseq, seq));
  const int32_t *v = c->h_gcnt->v;
  *done = v[C_ONE] != 0;
  if (!*done) return INK_OK;
  ink_status st = short_error(c, v);
  if (st != INK_OK) return st;
  const int64_t need[2] = {(int64_t)c->h_gcnt->total[0], (int64_t)c->h_gcnt->total[1]};
  short_result(c, need, n_ins_out, n_del_out);
  return INK_OK;
}

static ink_status graph_apply_short(ink_ctx *c, const RawUpdate *raw, int64_t n64, int64_t *n_ins_out, int64_t *n_del_out) {
  hipStream_t s = c->stream;
  const int n = (int)n64;
  const size_t per = ((size_t)(n + 64) * 4 + 255) & ~(size_t)255;
  INK_TRYS(c->b_misc.reserve(short_bytes(n)));
  for (DevBuf *b : {&c->b_del_s, &c->b_del_d, &c->b_ins_s, &c->b_ins_d, &c->b_touch_in, &c->b_uniq}) INK_TRYS(b->reserve(per));
  Arena ar(c->b_misc);
  const int n_chunks = (n + kOneChunk - 1) / kOneChunk;
  ShortSide sd[2];
  GraphSide *gs[2] = {&c->gin, &c->gout};
  for (int k = 0; k < 2; k++) {
    ShortSide &b = sd[k];
    b.skey = ar.get<uint64_t>((size_t)n_chunks * kOneChunk); b.sidx = ar.get<int32_t>((size_t)n_chunks * kOneChunk);
    b.node = ar.get<int32_t>(n); b.other = ar.get<int32_t>(n); b.op = ar.get<uint8_t>(n); b.pos = ar.get<int32_t>(n);
    b.seg = ar.get<int32_t>(n + 2); b.chunk_pref = ar.get<int32_t>(n + 1);
    b.nd_ins = ar.get<int32_t>(n + 1); b.nd_del = ar.get<int32_t>(n + 1); b.fill = ar.get<int32_t>(n + 1); b.head = ar.get<int32_t>(n + 1);
    b.uoff = ar.get<int64_t>(n); b.udeg = ar.get<int32_t>(n); b.ucap = ar.get<int32_t>(n);
    b.eoff = ar.get<int64_t>(n); b.edeg = ar.get<int32_t>(n); b.ecap = ar.get<int32_t>(n);
    b.off = gs[k]->off; b.deg = gs[k]->deg; b.cap = gs[k]->cap; b.ids = gs[k]->ids;
    b.slot_n = k ? C_OT : C_TMP0; b.slot_ch = k ? C_OCH : C_TMP1;
  }
  int32_t *chunk_err = ar.get<int32_t>(kMaxChunks);
  sd[0].uniq = c->b_touch_in.as<int32_t>();     // the touched lists are written in place
  sd[1].uniq = c->b_uniq.as<int32_t>();
  Counters *g = c->d_gcnt;
  c->del_src = c->b_del_s.as<int32_t>(); c->del_dst = c->b_del_d.as<int32_t>();
  c->ins_src = c->b_ins_s.as<int32_t>(); c->ins_dst = c->b_ins_d.as<int32_t>();
  if (n <= 256) hipLaunchKernelGGL((k_short_one<256>), dim3(2), dim3(256), 0, s, raw, n, c->n, sd[0], sd[1], g);
  else if (n <= 512) hipLaunchKernelGGL((k_short_one<512>), dim3(2), dim3(512), 0, s, raw, n, c->n, sd[0], sd[1], g);
  else if (n <= kOneChunk) hipLaunchKernelGGL((k_short_one<kOneChunk>), dim3(2), dim3(kOneChunk), 0, s, raw, n, c->n, sd[0], sd[1], g);
  else {
    hipLaunchKernelGGL(k_short_sort, dim3(2 * n_chunks), dim3(kOneChunk), 0, s, raw, n, c->n, n_chunks, sd[0], sd[1], chunk_err);
#define INK_MERGE(C) \
  hipLaunchKernelGGL(k_short_merge<C>, dim3(2 * n_chunks * kMergeParts), dim3(kMergeThreads), 0, s, n, n_chunks, sd[0], sd[1], (const int32_t *)chunk_err)
    if (n_chunks <= kMergeFew) INK_MERGE(kMergeFew);
    else if (n_chunks <= kMergeTwoOnCu) INK_MERGE(kMergeTwoOnCu);
    else INK_MERGE(kMaxChunks);
#undef INK_MERGE
    hipLaunchKernelGGL(k_short_heads, dim3(2 * n_chunks), dim3(kOneChunk), 0, s, n, n_chunks, sd[0], sd[1], (const int32_t *)chunk_err, g);
  }
  hipLaunchKernelGGL(k_short_classify, dim3(n <= kOneChunk ? 256 : 2048), dim3(256), 0, s, sd[0], sd[1], (const Counters *)g);
  const uint32_t seq = ++c->pub_seq;
  hipLaunchKernelGGL(k_short_finish, dim3(2 * n_chunks), dim3(kOneChunk), 0, s, n, n_chunks, sd[0], sd[1], c->ins_src, c->ins_dst, c->del_src,
                     c->del_dst, c->slack, (long long)(c->gin.pool_cap - c->gin.pool_top), (long long)(c->gout.pool_cap - c->gout.pool_top), g,
                     c->h_gcnt, c->h_gseq, seq);
  auto apply = [&](const int32_t *ok) {
    hipLaunchKernelGGL(k_apply, dim3(2 * n), dim3(256), 0, s, apply_side_of(sd[0], c->gin, g, C_TOP64, nullptr),
                       apply_side_of(sd[1], c->gout, g, C_TOP64B, c->new_out), n, c->slack, ok);
    return hipGetLastError();
  };
  INK_TRYS(apply(&g->v[C_OK]));
  INK_TRYS(wait_published(c, c->h_gseq, seq));
  const int32_t *v = c->h_gcnt->v;
  ink_status st = short_error(c, v);
  if (st != INK_OK) return st;
  const int64_t need[2] = {(int64_t)c->h_gcnt->total[0], (int64_t)c->h_gcnt->total[1]};
  if (!v[C_OK]) {      // a pool is full: larger ones, then the apply kernel again
    for (int k = 0; k < 2; k++)
      if (gs[k]->pool_top + need[k] > gs[k]->pool_cap) {
        hipError_t e = grow_pool(c, *gs[k], need[k]);
        if (e == hipErrorOutOfMemory) { c->err = "out of device memory while growing the edge pool"; return INK_E_OOM; }
        INK_TRYS(e);
      }
    INK_TRYS(apply(nullptr));
  }
  short_result(c, need, n_ins_out, n_del_out);
  return INK_OK;
}

ink_status graph_apply_batch(ink_ctx *c, const void *raw_v, int64_t n, int64_t *n_ins_out, int64_t *n_del_out,
                             hipError_t (*queued)(ink_ctx *, const OneGraph &, uint32_t)) {
  hipStream_t s = c->stream;
  *n_ins_out = *n_del_out = 0;
  c->n_ins = c->n_del = 0;
  c->n_touched_in = 0;
  if (n == 0) return INK_OK;
  const RawUpdate *raw = (const RawUpdate *)raw_v;
  if (n <= kOneEvents && n <= c->small_batch) {
    bool done = false;
    ink_status st = graph_apply_one(c, raw, n, n_ins_out, n_del_out, queued, &done);
    if (st != INK_OK || done) return st;      // otherwise the layers behind it did nothing
  }
  if (n <= c->small_batch) return graph_apply_short(c, raw, n, n_ins_out, n_del_out);
  size_t per = ((size_t)(n + 64) * 4 + 255) & ~(size_t)255;
  INK_TRYS(c->b_misc.reserve(per * 28));
  INK_TRYS(c->b_del_s.reserve(per)); INK_TRYS(c->b_del_d.reserve(per));
  INK_TRYS(c->b_ins_s.reserve(per)); INK_TRYS(c->b_ins_d.reserve(per));
  Arena ar(c->b_misc);
  uint32_t *k0 = ar.get<uint32_t>(n), *v0 = ar.get<uint32_t>(n), *k1 = ar.get<uint32_t>(n);
  uint32_t *srcv = ar.get<uint32_t>(n), *dstv = ar.get<uint32_t>(n);
  uint8_t *flag = ar.get<uint8_t>(n + 64);
  int32_t *idx = ar.get<int32_t>(n), *idx2 = ar.get<int32_t>(n);
  SideBufs b;
  b.node = ar.get<uint32_t>(n); b.other = ar.get<int32_t>(n); b.op = ar.get<uint8_t>(n + 64);
  b.pos = ar.get<int32_t>(n); b.eff = ar.get<uint8_t>(n + 64);
  b.uniq = ar.get<int32_t>(n + 1); b.seg = ar.get<int32_t>(n + 2); b.chunks = ar.get<int32_t>(n + 1);
  b.chunk_pref = ar.get<int32_t>(n + 1); b.nd_ins = ar.get<int32_t>(n + 1); b.nd_del = ar.get<int32_t>(n + 1);
  b.fill = ar.get<int32_t>(n + 1);
  Counters *dc = c->d_cnt;
  int32_t *n_ops_d = &dc->v[C_NOPS];

  // (dst, src, position) order through two stable sorts
  hipLaunchKernelGGL(k_unpack, grid1(n), dim3(256), 0, s, raw, n, c->n, srcv, dstv, v0, &dc->v[C_ERR]);
  INK_TRYS(hipMemcpyAsync(k0, srcv, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
  INK_TRYS(radix_sort_pairs(c->ws, k0, v0, n, c->id_bits, s));
  hipLaunchKernelGGL(k_gather_u32, grid1(n), dim3(256), 0, s, (const uint32_t *)dstv, (const uint32_t *)v0, n, k1);
  INK_TRYS(radix_sort_pairs(c->ws, k1, v0, n, c->id_bits, s));
  // final op per distinct edge; their number stays on the device (n bounds it)
  hipLaunchKernelGGL(k_mark_last, grid1(n), dim3(256), 0, s, raw, (const uint32_t *)v0, n, flag,
                     (const int32_t *)&dc->v[C_ERR]);
  INK_TRYS(compact_flags_u8(c->ws, flag, n, idx, n_ops_d, s));
  hipLaunchKernelGGL(k_take_ops, grid1(n), dim3(256), 0, s, raw, (const uint32_t *)v0, (const int32_t *)idx,
                     (const int32_t *)n_ops_d, b.node, b.other, b.op, b.pos);

  int n_touched = 0;
  int64_t ti = 0, td = 0;
  ink_status st = apply_side(c, c->gin, b, n, n_ops_d, nullptr, &n_touched, &ti, &td);
  if (st != INK_OK) return st;
  c->n_ins = ti; c->n_del = td;
  *n_ins_out = ti; *n_del_out = td;
  c->n_touched_in = n_touched;
  if (ti + td == 0) return INK_OK;
  INK_TRYS(c->b_touch_in.reserve((size_t)(n_touched + 1) * 4));
  INK_TRYS(hipMemcpyAsync(c->b_touch_in.p, b.uniq, (size_t)n_touched * 4, hipMemcpyDeviceToDevice, s));

  // Delta E lists, (dst, src) order
  hipLaunchKernelGGL(k_flag_eq, grid1(n), dim3(256), 0, s, (const uint8_t *)b.eff, (const int32_t *)n_ops_d, n,
                     (uint8_t)1, flag);
  INK_TRYS(compact_flags_u8(c->ws, flag, n, idx, &dc->v[C_TMP2], s));
  hipLaunchKernelGGL(k_flag_eq, grid1(n), dim3(256), 0, s, (const uint8_t *)b.eff, (const int32_t *)n_ops_d, n,
                     (uint8_t)2, flag);
  INK_TRYS(compact_flags_u8(c->ws, flag, n, idx2, &dc->v[C_TMP3], s));
  c->del_src = c->b_del_s.as<int32_t>(); c->del_dst = c->b_del_d.as<int32_t>();
  c->ins_src = c->b_ins_s.as<int32_t>(); c->ins_dst = c->b_ins_d.as<int32_t>();
  hipLaunchKernelGGL(k_split_ops, grid1(n), dim3(256), 0, s, (const uint32_t *)b.node, (const int32_t *)b.other,
                     (const uint8_t *)b.eff, (const int32_t *)n_ops_d, (const int32_t *)idx, (const int32_t *)idx2,
                     c->ins_src, c->ins_dst, c->del_src, c->del_dst, (const int32_t *)&dc->v[C_TMP2],
                     (const int32_t *)&dc->v[C_TMP3]);

  // out side: the effective ops in (src, dst) order
  int64_t m = ti + td;
  hipLaunchKernelGGL(k_out_dst_key, grid1(m), dim3(256), 0, s, (const int32_t *)c->del_dst, (const int32_t *)c->ins_dst,
                     (int)td, (int)ti, k0, v0);
  INK_TRYS(radix_sort_pairs(c->ws, k0, v0, m, c->id_bits, s));
  // key <- source of the permuted entries
  hipLaunchKernelGGL(k_out_ops, grid1(m), dim3(256), 0, s, (const int32_t *)c->del_src, (const int32_t *)c->del_dst,
                     (const int32_t *)c->ins_src, (const int32_t *)c->ins_dst, (int)td, (int)ti, srcv, dstv);
  hipLaunchKernelGGL(k_gather_u32, grid1(m), dim3(256), 0, s, (const uint32_t *)srcv, (const uint32_t *)v0, m, k1);
  INK_TRYS(radix_sort_pairs(c->ws, k1, v0, m, c->id_bits, s));
  hipLaunchKernelGGL(k_out_take, grid1(m), dim3(256), 0, s, (const uint32_t *)v0, (const int32_t *)c->del_src,
                     (const int32_t *)c->del_dst, (const int32_t *)c->ins_src, (const int32_t *)c->ins_dst, (int)td,
                     (int)ti, b.node, b.other, b.op, b.pos);
  int64_t oi = 0, od = 0;
  st = apply_side(c, c->gout, b, m, nullptr, c->new_out, &n_touched, &oi, &od);
  if (st != INK_OK) return st;
  if (oi != ti || od != td) {
    c->err = "graph store inconsistent: in- and out-adjacency disagree";
    return INK_E_DEVICE;
  }
  // remember the touched sources so that the per-batch marks can be cleared
  INK_TRYS(c->b_uniq.reserve((size_t)(n_touched + 1) * 4));
  INK_TRYS(hipMemcpyAsync(c->b_uniq.p, b.uniq, (size_t)n_touched * 4, hipMemcpyDeviceToDevice, s));
  c->n_touched_src = n_touched;
  return INK_OK;
}

hipError_t graph_end_batch(ink_ctx *c) {
  if (c->n_touched_src > 0)
    hipLaunchKernelGGL(k_zero_at, grid1(c->n_touched_src), dim3(256), 0, c->stream, (const int32_t *)c->b_uniq.p,
                       (int)c->n_touched_src, c->new_out);
  c->n_touched_src = 0;
  return hipGetLastError();
}

}  // namespace ink
