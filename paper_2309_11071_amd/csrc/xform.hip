// Dense combination on compacted rows with fp32 MFMA (v_mfma_f32_32x32x2_f32), fused with the
// gather of the input rows, bias, activation and the compare-and-emit step (a row is reported
// as changed only if its new value differs bitwise from the cached one; Sec. 2.5.2).
//
// Every output element is one chain of fused multiply-adds over k = 0 .. K-1 in ascending order
// starting from +0 (the MFMA unit applies its two k-steps in that order), independent of the
// tile or row slot it is computed in, so a row's result never depends on which other rows share
// the launch.  Zero-padded k-steps leave the accumulator unchanged.
#include <algorithm>

#include "ctx.h"

namespace ink {

typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int KT = 32;       // k-chunk staged in LDS

__device__ __forceinline__ void ld4v(const float *p, float out[4]) {
  float4 v = *reinterpret_cast<const float4 *>(p);
  out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
}

// Four consecutive inputs k .. k + 3 (k a multiple of 4) of one row in two parts: issue_x4 loads what they
// are made of, finish_x4 combines it where the values are used, so that loads stay in flight across
// other work.  Always 16-byte loads: table rows are padded with zeros to 16 floats, SAGE's two halves
// start at multiples of 4 (xform_self_row), and a group past a row's end reads the row's start instead.
template <int MODE> struct RawX { float4 a; };
template <> struct RawX<1> { float4 a, b; };
template <> struct RawX<3> { float4 a, b; };

template <int MODE>
__device__ __forceinline__ void issue_x4(const XformArgs &x, int64_t row, int k, RawX<MODE> &r) {
  if constexpr (MODE == 0) {           // SAGE: [alpha | h_prev]
    const int d4 = xform_self_row(x.d_in);
    const int ks = k - d4 < d4 ? k - d4 : 0;
    const float *p = k < d4 ? x.A + row * x.lda + k : x.Hp + row * x.ldh + ks;
    r.a = *reinterpret_cast<const float4 *>(p);
  } else if constexpr (MODE == 2) {    // dense rows
    r.a = *reinterpret_cast<const float4 *>(x.Hp + row * x.ldh + (k < x.ldh ? k : 0));
  } else {                             // GIN: (1 + eps) h_prev + alpha; GCN: act(c_v (S + own scaled message) + b)
    r.a = *reinterpret_cast<const float4 *>(x.A + row * x.lda + (k < x.lda ? k : 0));
    r.b = *reinterpret_cast<const float4 *>(x.Hp + row * x.ldh + (k < x.ldh ? k : 0));
  }
}
// per-row scalar of the combination: degree (mean) or c_v (GCN)
template <int MODE> __device__ __forceinline__ float row_scalar(const XformArgs &x, int64_t row) {
  if (MODE == 3) return x.cnorm[row];
  if ((MODE == 0 || MODE == 1) && x.mean_deg) { const int dg = x.mean_deg[row]; return (float)(dg > 0 ? dg : 1); }
  return 1.f;
}
// GCN also writes the combined row as h_l
template <int MODE>
__device__ __forceinline__ void finish_x4(const XformArgs &x, int64_t row, int k, float sc, bool store_h, const RawX<MODE> &r, float v[4]) {
  v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w;
  if constexpr (MODE == 0) {
    const int d4 = xform_self_row(x.d_in);
    if (x.mean_deg && k < d4)
#pragma unroll
      for (int i = 0; i < 4; i++) v[i] = __fdiv_rn(v[i], sc);
    if (k >= 2 * d4 || d4 != x.d_in)       // past the input, or in the padding of an aggregated row (anything may stand there)
#pragma unroll
      for (int i = 0; i < 4; i++) v[i] = k < 2 * d4 && (k < d4 ? k : k - d4) + i < x.d_in ? v[i] : 0.f;
  } else if constexpr (MODE == 1) {
    const float h[4] = {r.b.x, r.b.y, r.b.z, r.b.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const float a = x.mean_deg ? __fdiv_rn(v[i], sc) : v[i];
      v[i] = k + i < x.d_in ? __fadd_rn(__fmul_rn(1.0f + x.eps, h[i]), a) : 0.f;
    }
  } else if constexpr (MODE == 2) {
#pragma unroll
    for (int i = 0; i < 4; i++) v[i] = k + i < x.d_in ? v[i] : 0.f;
  } else {
    const float h[4] = {r.b.x, r.b.y, r.b.z, r.b.w};
    float b[4], u[4];
    if (x.in_bias) ld4v(x.in_bias + k, b);
    if (x.in_user) ld4v(x.in_user + row * x.ld_in_user + (k < x.ld_in_user ? k : 0), u);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      float t = __fmul_rn(sc, __fadd_rn(v[i], h[i]));
      if (x.in_bias) t = __fadd_rn(t, b[i]);
      if (x.in_user) t = __fadd_rn(t, u[i]);
      if (x.in_relu) t = t > 0.f ? t : 0.f;
      v[i] = k + i < x.d_in ? t : 0.f;
    }
    if (store_h && x.h_store && k < x.ld_hs) *reinterpret_cast<float4 *>(x.h_store + row * x.ld_hs + k) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// LDS layouts (floats): X tile [BM][2][16] with row stride XS, W tile [Np][2][16] with row stride
// XS.  Index [.][p][s] holds k = k0 + 2 s + p, so the 16 values a lane feeds to the 16 MFMA steps
// of a chunk (lanes 0-31 take the even k, lanes 32-63 the odd k) are contiguous: four 16-byte LDS
// reads.  The stride of 36 floats spreads 16 lanes x 4 banks over all 64 banks.
constexpr int XS = 36;

// Compute phase of one k-chunk for the NTW column tiles ct0, ct0 + 2, ... of this wave: all LDS
// reads of a tile are issued before its 16 back-to-back MFMAs.
template <int NTW, int CS>
__device__ __forceinline__ void mfma_chunk(const float *Xs, const float *Ws, int rt, int ct0, int l, f16v *acc) {
  const float *ap = Xs + (rt * 32 + (l & 31)) * XS + (l >> 5) * 16;
  float a[16];
#pragma unroll
  for (int v = 0; v < 4; v++) {
    float4 t4 = *reinterpret_cast<const float4 *>(ap + 4 * v);
    a[4 * v] = t4.x; a[4 * v + 1] = t4.y; a[4 * v + 2] = t4.z; a[4 * v + 3] = t4.w;
  }
#pragma unroll
  for (int i = 0; i < NTW; i++) {
    const float *bp = Ws + ((ct0 + CS * i) * 32 + (l & 31)) * XS + (l >> 5) * 16;
    float b[16];
#pragma unroll
    for (int v = 0; v < 4; v++) {
      float4 t4 = *reinterpret_cast<const float4 *>(bp + 4 * v);
      b[4 * v] = t4.x; b[4 * v + 1] = t4.y; b[4 * v + 2] = t4.z; b[4 * v + 3] = t4.w;
    }
#pragma unroll
    for (int sidx = 0; sidx < 16; sidx++)
      acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[sidx], b[sidx], acc[i], 0, 0, 0);
  }
}

// Epilogue of a workgroup's tile: bias, user term, output scale, activation, then either a plain
// store or compare-and-emit against the cached table row.  A lane holds rows
// 8*(r/4) + 4*(l/32) + r%4 of its row tile, column l % 32 of each of its column tiles.
template <int TPW, int CS, int NT, int BM>
__device__ __forceinline__ void xform_epilogue(const XformArgs &x, const f16v *acc, const int64_t *srow, const int64_t *sout,
                                               int *schg, int rt, int ct0, int l, int t, int64_t r0) {
#pragma unroll
  for (int i = 0; i < TPW; i++) {
    int ct = ct0 + CS * i;
    if (ct >= NT) continue;
    int col = ct * 32 + (l & 31);
    if (col >= x.n_out) continue;
    float bias = x.bias ? x.bias[col] : 0.f;
    float oldv[16];
    const bool compare = x.to_table && (x.row_changed || x.old_rows);     // a whole inference only stores
    if (compare) {         // all loads of the cached values first, then compare and store
#pragma unroll
      for (int r = 0; r < 16; r++) {
        int rl = rt * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
        oldv[r] = srow[rl] >= 0 ? x.out[sout[rl] * x.ld_out + col] : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
      int rl = rt * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
      int64_t row = srow[rl];
      if (row < 0) continue;
      float v = acc[i][r];
      if (x.bias) v = __fadd_rn(v, bias);
      if (x.user) v = __fadd_rn(v, x.user[sout[rl] * x.ld_user + col]);
      if (x.out_scale) v = __fmul_rn(v, x.out_scale[sout[rl]]);
      if (x.relu) v = v > 0.f ? v : 0.f;
      int64_t j = r0 + rl;
      if (compare) {
        float old = oldv[r];
        if (x.old_rows) x.old_rows[j * x.ld_old + col] = old;
        if (__float_as_uint(old) != __float_as_uint(v)) { x.out[sout[rl] * x.ld_out + col] = v; schg[rl] = 1; }
      } else {
        x.out[(x.to_table ? sout[rl] : j) * x.ld_out + col] = v;
      }
    }
  }
  if (x.to_table && x.row_changed) {
    __syncthreads();
    if (t < BM && srow[t] >= 0) x.row_changed[r0 + t] = (uint8_t)schg[t];
  }
}

// Bound by memory as much as by the matrix cores: 655k SAGE rows 256 -> 121 are 1.3 GB and 41 GFLOP, .27 ms
// of either, and take .46 ms (.48 with a scalar path for rows of odd width and loads that waited where they
// were issued); the two products of 1.25M GIN rows 128 -> 128 -> 172 take .76 ms (.85) for 3.4 GB.  What keeps it
// there is the number of waves in flight: prefetching the weights as well, or 128 rows per workgroup, costs
// registers and LDS and measured .46 - .7 ms; keeping the weights in LDS for a persistent workgroup .52 ms.
// BM = rows per workgroup (64 or 128), NT = number of 32-column tiles (Np / 32), NW = waves per
// workgroup.  With RT = BM / 32 row tiles, wave w works on row tile w % RT and on the column tiles
// w / RT, w / RT + NW / RT, ...
template <int MODE, int NT, int NW, int BM>
__global__ __launch_bounds__(NW * 64) void k_xform(XformArgs x) {
  extern __shared__ float smem[];
  float *Xs = smem;                           // [BM][XS]
  float *Ws = smem + BM * XS;                 // [Np][XS]
  __shared__ int64_t srow[BM];     // input row (gather) of each tile row, -1 past the end
  __shared__ int64_t sout[BM];     // table row written by the epilogue
  __shared__ int schg[BM];
  constexpr int RT = BM / 32;
  constexpr int CS = NW / RT;                 // column-tile stride between the tiles of one wave
  constexpr int TPW = (NT + CS - 1) / CS;
  constexpr int Np = NT * 32;
  constexpr int NTHR = NW * 64;
  constexpr int KPT = KT * BM / NTHR >= 4 ? KT * BM / NTHR : 4;   // consecutive k of one row that a thread stages (8 or 4)
  constexpr int XTHR = KT * BM / KPT;         // threads that stage X (all of them up to 8 waves)
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const int rt = w % RT;                      // row tile of this wave
  const int ct0 = w / RT;                     // first column tile; then += CS
  const int64_t r0 = (int64_t)blockIdx.x * BM;
  int64_t n_rows = x.n_rows;
  if (x.n_rows_dev) {          // the launch covers an upper bound; workgroups past the count leave
    int64_t nd = *x.n_rows_dev;
    n_rows = nd < n_rows ? nd : n_rows;
    if (r0 >= n_rows) return;
  }
  if (t < BM) {
    int64_t j = r0 + t;
    int64_t row = -1;
    if (j < n_rows) row = (MODE == 2) ? j : (x.rows ? (int64_t)x.rows[j] : j);
    srow[t] = row;
    sout[t] = (row >= 0 && MODE == 2 && x.to_table && x.out_rows) ? (int64_t)x.out_rows[j] : row;
    schg[t] = 0;
  }
  f16v acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; i++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[i][r] = 0.f;
  __syncthreads();
  // thread -> row t / 4, 8 consecutive k of the X chunk
  const bool xstage = t < XTHR;
  const int xr = (t % XTHR) / (KT / KPT), xks = (t % (KT / KPT)) * KPT;
  const int64_t xrow = xstage ? srow[xr] : -1;
  // the loads of the next chunk are issued a whole iteration before their values are combined and
  // staged, so the gather latency overlaps the barriers, the weight staging and the MFMAs of the chunk between
  RawX<MODE> raw[KPT / 4];
  const float sc = xrow >= 0 ? row_scalar<MODE>(x, xrow) : 1.f;
  auto issue = [&](int k0) {
    if (xrow >= 0) {
#pragma unroll
      for (int kk = 0; kk < KPT; kk += 4) issue_x4<MODE>(x, xrow, k0 + xks + kk, raw[kk / 4]);
    }
  };
  issue(0);
  for (int k0 = 0; k0 < x.Kp; k0 += KT) {
    float xv[KPT];
#pragma unroll
    for (int kk = 0; kk < KPT; kk++) xv[kk] = 0.f;
    if (xrow >= 0) {
#pragma unroll
      for (int kk = 0; kk < KPT; kk += 4) finish_x4<MODE>(x, xrow, k0 + xks + kk, sc, true, raw[kk / 4], xv + kk);
    }
    if (xstage) {   // even k first, then odd k
      float *xp = Xs + xr * XS + (xks >> 1);
      if constexpr (KPT == 8) {
        *reinterpret_cast<float4 *>(xp) = make_float4(xv[0], xv[2], xv[4], xv[6]);
        *reinterpret_cast<float4 *>(xp + 16) = make_float4(xv[1], xv[3], xv[5], xv[7]);
      } else {
        *reinterpret_cast<float2 *>(xp) = make_float2(xv[0], xv[2]);
        *reinterpret_cast<float2 *>(xp + 16) = make_float2(xv[1], xv[3]);
      }
    }
    {   // stage the W chunk (xform_weight_index) -> rows of stride XS
      const float4 *src = reinterpret_cast<const float4 *>(x.W + (int64_t)k0 * Np);
      constexpr int n4 = KT * Np / 4;
#pragma unroll
      for (int i = t; i < n4; i += NTHR)
        *reinterpret_cast<float4 *>(Ws + ((i >> 8) * 32 + (i & 31)) * XS + ((i >> 5) & 1) * 16 + ((i >> 6) & 3) * 4) = src[i];
    }
    if (k0 + KT < x.Kp) issue(k0 + KT);
    __syncthreads();
    // this wave owns TPW column tiles, or one fewer when the last one would lie past NT
    if (ct0 + (TPW - 1) * CS < NT) mfma_chunk<TPW, CS>(Xs, Ws, rt, ct0, l, acc);
    else if (TPW > 1) mfma_chunk<(TPW > 1 ? TPW - 1 : 1), CS>(Xs, Ws, rt, ct0, l, acc);
    __syncthreads();
  }
  xform_epilogue<TPW, CS, NT, BM>(x, acc, srow, sout, schg, rt, ct0, l, t, r0);
}

// ---- few rows
// Few rows are a chain of latencies: the kernel above takes 17 us for any number up to some thousands (256 inputs, 128
// outputs), two barriers and a gather for each of its eight chunks.  Here a wave owns 16 rows and TPW tiles of 16 columns, has the inputs and weights of four chunks under
// way, and meets the others only to join the flags of its rows.  v_mfma_f32_16x16x4_f32 takes half the cycles of
// 32x32x2 for twice the k and adds its four products in ascending order like the two of the other (test_gpu_xform_few).
__device__ __forceinline__ void swap32(float &x, float &y) {     // upper lanes of x <-> lower lanes of y
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(t[0]); y = __uint_as_float(t[1]);
}
__device__ __forceinline__ void swap16(float &x, float &y) {     // odd rows of 16 lanes of x <-> even rows of y
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(t[0]); y = __uint_as_float(t[1]);
}

typedef float f4acc __attribute__((ext_vector_type(4)));
constexpr int kFewWaves = 8;

template <int MODE, int TPW>
__global__ __launch_bounds__(kFewWaves * kWave) void k_xform_few(XformArgs x) {
  constexpr int D = TPW == 2 || MODE == 3 ? 2 : 4;       // chunks of KT under way, as many as the registers hold
  __shared__ uint32_t part[kFewWaves];
  const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int kq = l >> 4;                          // which of a step's four k
  int64_t n_rows = x.n_rows;
  if (x.n_rows_dev) {          // the launch covers an upper bound; workgroups past the count leave
    int64_t nd = *x.n_rows_dev;
    n_rows = nd < n_rows ? nd : n_rows;
  }
  const int64_t r0 = (int64_t)blockIdx.x * 16;
  if (r0 >= n_rows) return;
  const int n_ch = x.Kp / KT;
  // the weights of tile ct: lane (k % 2) * 32 + col % 32 of the layout (xform_weight_index)
  float4 b[D][TPW][4];
  const float4 *wp[TPW];
#pragma unroll
  for (int i = 0; i < TPW; i++) {
    const int ct = w * TPW + i;
    wp[i] = reinterpret_cast<const float4 *>(x.W) + (ct >> 1) * 256 + (kq & 1) * 32 + (ct & 1) * 16 + (l & 15);
  }
  auto issue_w = [&](int d, int ch) {
    const int64_t o = (int64_t)(ch < n_ch ? ch : n_ch - 1) * 8 * x.Np;
#pragma unroll
    for (int i = 0; i < TPW; i++)
#pragma unroll
      for (int u = 0; u < 4; u++) b[d][i][u] = wp[i][o + u * 64];
  };
#pragma unroll
  for (int d = 0; d < D; d++) issue_w(d, d);
  // lanes past the last row repeat it: no load stands under a condition, and nothing of it is stored
  const int left = n_rows - r0 < 16 ? (int)(n_rows - r0) : 16;
  const int64_t j = r0 + ((l & 15) < left ? (l & 15) : left - 1);
  const int64_t row = (MODE == 2 || !x.rows) ? j : (int64_t)x.rows[j];
  const int orow = (int)(!x.to_table ? j : MODE == 2 && x.out_rows ? (int64_t)x.out_rows[j] : row);
  const bool store_h = w == 0 && (l & 15) < left;
  RawX<MODE> raw[D][2];
  auto issue = [&](int d, int ch) {
    const int k0 = (ch < n_ch ? ch : n_ch - 1) * KT + 4 * kq;
#pragma unroll
    for (int i = 0; i < 2; i++) issue_x4<MODE>(x, row, k0 + 16 * i, raw[d][i]);
  };
#pragma unroll
  for (int d = 0; d < D; d++) issue(d, d);
  const float sc = row_scalar<MODE>(x, row);
  // the rows that are replaced: a lane holds rows 4 kq + r, column l % 16 of each of its tiles
  const bool compare = x.to_table && (x.row_changed || x.old_rows);     // a whole inference only stores
  int o[4];
  float old[TPW][4];
#pragma unroll
  for (int r = 0; r < 4; r++) o[r] = __shfl(orow, 4 * kq + r, kWave);
#pragma unroll
  for (int i = 0; i < TPW; i++) {
    const int col = (w * TPW + i) * 16 + (l & 15);
#pragma unroll
    for (int r = 0; r < 4; r++) old[i][r] = compare && col < x.n_out ? x.out[(int64_t)o[r] * x.ld_out + col] : 0.f;
  }
  f4acc acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) acc[i][r] = 0.f;
  auto chunk = [&](const int d, const int ch) __attribute__((always_inline)) {     // d: constant
    float a[8];                                    // step s: k 4 s + kq
#pragma unroll
    for (int i = 0; i < 2; i++) {
      float *v = a + 4 * i;                        // lanes kq hold k 16 i + 4 kq ..: transposed over the four lane groups
      finish_x4<MODE>(x, row, ch * KT + 16 * i + 4 * kq, sc, store_h, raw[d][i], v);
      swap32(v[0], v[2]); swap32(v[1], v[3]);
      swap16(v[0], v[1]); swap16(v[2], v[3]);
    }
    issue(d, ch + D);
#pragma unroll
    for (int i = 0; i < TPW; i++)
#pragma unroll
      for (int s = 0; s < 8; s++) {
        const float4 q = b[d][i][s >> 1];
        const float bw = s & 1 ? (kq >> 1 ? q.w : q.z) : (kq >> 1 ? q.y : q.x);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bw, acc[i], 0, 0, 0);
      }
    issue_w(d, ch + D);
  };
  int ch = 0;
  for (; ch + D <= n_ch; ch += D)
#pragma unroll
    for (int d = 0; d < D; d++) chunk(d, ch + d);
#pragma unroll
  for (int d = 0; d < D - 1; d++)
    if (ch + d < n_ch) chunk(d, ch + d);
  unsigned changed = 0;                            // bit r: some value of this lane's row r
#pragma unroll
  for (int i = 0; i < TPW; i++) {
    const int col = (w * TPW + i) * 16 + (l & 15);
    if (col >= x.n_out) continue;
    const float bias = x.bias ? x.bias[col] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int rl = 4 * kq + r;
      if (rl >= left) continue;
      float v = acc[i][r];
      if (x.bias) v = __fadd_rn(v, bias);
      if (x.user) v = __fadd_rn(v, x.user[(int64_t)o[r] * x.ld_user + col]);
      if (x.out_scale) v = __fmul_rn(v, x.out_scale[o[r]]);
      if (x.relu) v = v > 0.f ? v : 0.f;
      float *p = x.out + (int64_t)o[r] * x.ld_out + col;
      if (compare) {
        if (x.old_rows) x.old_rows[(r0 + rl) * x.ld_old + col] = old[i][r];
        if (__float_as_uint(old[i][r]) != __float_as_uint(v)) { *p = v; changed |= 1u << r; }
      } else *p = v;
    }
  }
  if (!(x.to_table && x.row_changed)) return;
  uint32_t rows = 0;                               // bit of every row of the tile
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const uint64_t m = __ballot((changed >> r) & 1u);
#pragma unroll
    for (int q = 0; q < 4; q++) rows |= ((m >> (16 * q)) & 0xffffu ? 1u : 0u) << (4 * q + r);
  }
  if (l == 0) part[w] = rows;
  __syncthreads();
  if (w != 0) return;
  for (int i = 1; i < (int)(blockDim.x / kWave); i++) rows |= part[i];
  if (l < left) x.row_changed[r0 + l] = (uint8_t)((rows >> l) & 1u);
}

#ifndef INK_XF_WIDE_FROM
#define INK_XF_WIDE_FROM 3      // 8 waves per workgroup from this many column tiles on
#endif
#ifndef INK_XF_WIDER_FROM
#define INK_XF_WIDER_FROM 5     // 16 waves per workgroup from this many column tiles on
#endif

// 64 rows per workgroup: 128 rows (half the weight staging per row) measured the same or slower
template <int MODE, int NT>
static void launch_nt(ink_ctx *c, const XformArgs &x) {
  constexpr int BM = 64;
  size_t sh = (size_t)(BM + x.Np) * XS * sizeof(float);
  dim3 grid((unsigned)((x.n_rows + BM - 1) / BM));
  if constexpr (NT >= INK_XF_WIDER_FROM) hipLaunchKernelGGL((k_xform<MODE, NT, 16, BM>), grid, dim3(1024), sh, c->stream, x);
  else if constexpr (NT >= INK_XF_WIDE_FROM) hipLaunchKernelGGL((k_xform<MODE, NT, 8, BM>), grid, dim3(512), sh, c->stream, x);
  else hipLaunchKernelGGL((k_xform<MODE, NT, 4, BM>), grid, dim3(256), sh, c->stream, x);
}

template <int MODE>
static hipError_t launch(ink_ctx *c, const XformArgs &x) {
  switch (x.Np / 32) {
    case 1: launch_nt<MODE, 1>(c, x); break;
    case 2: launch_nt<MODE, 2>(c, x); break;
    case 3: launch_nt<MODE, 3>(c, x); break;
    case 4: launch_nt<MODE, 4>(c, x); break;
    case 5: launch_nt<MODE, 5>(c, x); break;
    case 6: launch_nt<MODE, 6>(c, x); break;
    case 7: launch_nt<MODE, 7>(c, x); break;
    case 8: launch_nt<MODE, 8>(c, x); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t xform_run(ink_ctx *c, const XformArgs &x) {
  if (x.n_rows <= 0) return hipSuccess;
  if (x.Np % 32 || x.Kp % KT || x.Np > 256) return hipErrorInvalidValue;
  // Rows up to which the time is the chain of one workgroup.  500 / 2000 / 6000 rows of 256 inputs and 128 outputs take 12 / 13 /
  // 22 us, in the other form 17 / 17 / 18; a bound that is found before its count is usually twice it.  Updates, the few-row form against
  // none: 50 edges on 100k nodes, widths 100, 256, 47, .43 -> .38 ms, 100 on 10k nodes .39 -> .375, 333 on 87k nodes .75 -> .73.
  if (x.n_rows <= (x.n_rows_dev ? 4096 : 2048)) {
    const dim3 grid((unsigned)((x.n_rows + 15) / 16));
    const int tiles = x.Np / 16;
#define INK_FEW(M)                                                                                             \
  if (tiles <= kFewWaves) hipLaunchKernelGGL((k_xform_few<M, 1>), grid, dim3(tiles * kWave), 0, c->stream, x);   \
  else hipLaunchKernelGGL((k_xform_few<M, 2>), grid, dim3(tiles / 2 * kWave), 0, c->stream, x)
    switch (x.mode) {
      case 0: INK_FEW(0); break;
      case 1: INK_FEW(1); break;
      case 2: INK_FEW(2); break;
      case 3: INK_FEW(3); break;
      default: return hipErrorInvalidValue;
    }
#undef INK_FEW
    return hipGetLastError();
  }
  switch (x.mode) {
    case 0: return launch<0>(c, x);
    case 1: return launch<1>(c, x);
    case 2: return launch<2>(c, x);
    case 3: return launch<3>(c, x);
  }
  return hipErrorInvalidValue;
}

}  // namespace ink
