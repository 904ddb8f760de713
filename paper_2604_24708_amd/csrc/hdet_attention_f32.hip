// Causal attention of the full-precision path, one launch forward and one (sequences of up to 32) or two backward, for head sizes of whole groups of 8 up to
// 64 and sequences up to 512 (other shapes: products and softmax kernels of their own).
//
// What bounds it: the sizes of this path (a few dozen to a few hundred rows) make it latency, one dependent launch after the other.  Three launches
// each way with the scores, probabilities and their gradients going through memory between them become one or two; the probabilities are kept for the
// backward.  us, three launches -> these, forward / backward, gaps between the launches not counted (heads over all replicas and sequences, S, head size):
//   64, 32, 16 11.8 -> 5.1 / 11.5 -> 5.9;  64, 128, 64 16.8 -> 8.6 / 20.3 -> 17.6;  288, 192, 32 57 -> 28 / 92 -> 51;  288, 192, 64 69 -> 45 / 101 -> 89;
//   64, 256, 64 30 -> 18 / 40 -> 34;  64, 512, 64 78 -> 46 / 136 -> 95;  256, 512, 64 312 -> 170 / 507 -> 365
// (A backward of one launch at any length, blocks of keys with a dp and a row dot of their own, takes as long in its kernels, 16.2, 54, 99, 35, 97 and 380, and
// saves a gap between launches; but a block of keys sees a row's dot only as da . a, see below.)
//
// fp32 products on the matrix cores (v_mfma_f32_32x32x2_f32), a block of four wavefronts to 32 queries (or keys) of a head:
//  * A wavefront takes every fourth tile of 32 x 32 of the other side, at and below the diagonal only, fragments straight from global memory.
//  * The first product is formed with the axis that the second contracts over as its rows: a lane's sixteen accumulators are then four groups of four
//    consecutive entries of that axis for one column, which is the second product's first operand as it stands.  Neither scores nor probabilities
//    touch LDS.
//  * Row maximum, row sum and row dot (both in 64 bits: sixteen terms in a lane's chain), then the four wavefronts' partial results, meet in LDS and are added in the order of the wavefronts.
//  * Every product is four sums at least, as the products through memory are: one chain puts the gradients 1.04 to 1.1 times as far from 64 bits.
//
// Distance from 64 bits of the qkv weights' gradients against three launches each way, geometric mean over 50 models (S 17 to 512, head sizes 16 to 64,
// queries, keys or values with an offset or none): queries 0.87, keys 0.93, values 0.97.

#include "hdet_elem.h"
#include "hdet_internal.h"

namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kThreads = 256, kWaves = 4;

__device__ __forceinline__ f16v zero16() {
  f16v z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}
// accumulator e of a lane belongs to this row of its tile (its column is lane % 32)
__device__ __forceinline__ int acc_row(int e, int half) { return (e >> 2) * 8 + half * 4 + (e & 3); }

// DH / 8 groups of a row's DH entries: the lane's four of each group of eight
template <int G>
__device__ __forceinline__ void load_row(float (&v)[G][4], const float* row, int half) {
#pragma unroll
  for (int c = 0; c < G; ++c) {
    const f4u x = *reinterpret_cast<const f4u*>(row + 8 * c + 4 * half);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[c][j] = x[j];
  }
}
// in four sums, as the products through memory form it
template <int G>
__device__ __forceinline__ f16v product(const float (&a)[G][4], const float (&b)[G][4]) {
  f16v acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = zero16();
#pragma unroll
  for (int c = 0; c < G; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][j], b[c][j], acc[j], 0, 0, 0);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
// the second product's other operand: rows r0 .. r0 + 31 (at most `last`) of an [S][DH] matrix, columns 32 n + lane % 32
template <int NB>
__device__ __forceinline__ void load_cols(float (&v)[16][NB], const float* m, int64_t ld, int r0, int last, int dh, int lane) {
  const int half = lane >> 5, c = lane & 31;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = r0 + acc_row(e, half);
    const float* row = m + (int64_t)(r < last ? r : last) * ld;
#pragma unroll
    for (int n = 0; n < NB; ++n) v[e][n] = row[32 * n + c < dh ? 32 * n + c : dh - 1];
  }
}
// C sums a wavefront: one where four wavefronts have a tile or more each, else more, so that a result is four sums at least
template <int C, int NB>
__device__ __forceinline__ void clear(f16v (&acc)[C][NB]) {
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[c][n] = zero16();
}
template <int C, int NB>
__device__ __forceinline__ void accumulate(f16v (&acc)[C][NB], const f16v& a, const float (&b)[16][NB]) {
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[e % C][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e][n], acc[e % C][n], 0, 0, 0);
}
template <int C, int NB>
__device__ __forceinline__ void add_up(f16v (&acc)[C][NB]) {
#pragma unroll
  for (int c = 1; c < C; ++c)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[0][n] += acc[c][n];
}
// the wavefronts' partial [32][DH] results added in their order and written: rows r0 .. (below S) of an [S][DH] matrix
template <int C, int NB>
__device__ __forceinline__ void write_sum(f16v (&acc)[C][NB], float* red, float* m, int64_t ld, int r0, int S, int dh, int lane, int w) {
  add_up<C, NB>(acc);
  float* mine = red + w * (NB * 16 * 64) + lane;
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int e = 0; e < 16; ++e) mine[(n * 16 + e) * 64] = acc[0][n][e];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NB * 4; ++u) {
    const int q = w * NB * 4 + u;
    float v = red[q * 64 + lane];
#pragma unroll
    for (int p = 1; p < kWaves; ++p) v += red[(p * NB * 16 + q) * 64 + lane];
    const int r = r0 + acc_row(q & 15, lane >> 5), c = 32 * (q >> 4) + (lane & 31);
    if (r < S && c < dh) m[(int64_t)r * ld + c] = v;
  }
}

// a lane's sixteen entries of row `row` of an [S][S] matrix, columns of tile kt
__device__ __forceinline__ void store_row(float* row, const f16v& x, int kt, int half, int S) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int j = kt * 32 + acc_row(4 * g, half);
    if (j + 3 < S) *reinterpret_cast<f4u*>(row + j) = f4u{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j + e < S) row[j + e] = x[4 * g + e];
    }
  }
}

struct head { const float* q; const float* k; const float* v; int64_t ld; float scale; int64_t hd, at_a; };
__device__ __forceinline__ head head_of(const hdet_attn_f32_desc& t, int hd) {
  const int h = hd % t.heads, b = hd / t.heads, dh = t.d_model / t.heads, r = b / t.batch;
  const float* q = t.qkv + (int64_t)b * t.seq_len * 3 * t.d_model + h * dh;
  float scale = t.scale;
  if (t.temp_channel >= 0) scale = scale / (float)hdet_channel_value(t.ctrl, t.temp_channel, r, 0.0);
  return {q, q + t.d_model, q + 2 * t.d_model, 3 * (int64_t)t.d_model, scale, hd, (int64_t)b * t.seq_len * t.d_model + h * dh};
}

// NT: 32-key tiles a wavefront holds; G = DH / 8; NB = ceil(DH / 32)
template <int G, int NT, int C>
__global__ __launch_bounds__(kThreads) void attn_f32_fwd_kernel(const hdet_attn_f32_desc t, int nblk) {
  constexpr int NB = (G + 3) / 4, DH = 8 * G, PRE = NT < 2 ? NT : 2;     // tiles of values in flight
  __shared__ float red[kWaves * NB * 16 * 64];
  __shared__ float rmax[kWaves][32];
  __shared__ double rsum[kWaves][32];
  const int qb = nblk - 1 - (int)blockIdx.y;                         // the longest rows first
  const head hd = head_of(t, (int)blockIdx.x);
  const int S = t.seq_len, last = S - 1, lane = threadIdx.x & 63, half = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = qb * 32 + (lane & 31);
  float qf[G][4];
  load_row<G>(qf, hd.q + (int64_t)(i < last ? i : last) * hd.ld, half);
  f16v s[NT];
  float vf[PRE][16][NB];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int kt = w + kWaves * u;
    if (kt > qb) continue;                                           // uniform over the wavefront
    float kf[G][4];
    const int j = kt * 32 + (lane & 31);
    load_row<G>(kf, hd.k + (int64_t)(j < last ? j : last) * hd.ld, half);
    if (u < PRE) load_cols<NB>(vf[u], hd.v, hd.ld, kt * 32, last, DH, lane);      // on their way under the softmax
    s[u] = product<G>(kf, qf);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[u][e] = kt * 32 + acc_row(e, half) <= i ? s[u][e] : -INFINITY;
      mx = fmaxf(mx, s[u][e] * hd.scale);
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (lane < 32) rmax[w][lane] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(rmax[0][lane & 31], rmax[1][lane & 31]), fmaxf(rmax[2][lane & 31], rmax[3][lane & 31]));
  double sum = 0.0;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    if (w + kWaves * u > qb) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) { s[u][e] = expf(__builtin_fmaf(s[u][e], hd.scale, -mx)); sum += s[u][e]; }
  }
  sum += __shfl_xor(sum, 32);
  if (lane < 32) rsum[w][lane] = sum;
  __syncthreads();
  const float inv = 1.f / (float)(((rsum[0][lane & 31] + rsum[1][lane & 31]) + rsum[2][lane & 31]) + rsum[3][lane & 31]);
  f16v acc[C][NB];
  clear<C, NB>(acc);
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int kt = w + kWaves * u;
    if (kt > qb) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[u][e] *= inv;
    if (i < S) store_row(t.p + (hd.hd * S + i) * S, s[u], kt, half, S);
    accumulate<C, NB>(acc, s[u], vf[u % PRE]);
    if (u + PRE < NT && kt + kWaves * PRE <= qb) load_cols<NB>(vf[u % PRE], hd.v, hd.ld, (kt + kWaves * PRE) * 32, last, DH, lane);
  }
  write_sum<C, NB>(acc, red, t.a + hd.at_a, t.d_model, qb * 32, S, DH, lane, w);
}

// Backward: dp = da v^T, ds = p (dp - sum over the row of dp p) scale, dq = ds k, dk = ds^T q, dv = p^T da.  The row's sum is taken of the very dp that it is
// subtracted from: what is wrong with all of a row's dp, or with the sum, then cancels in sum_j ds_j k_j.  (da . a is the same number without a walk over the
// row, but is wrong by what a was rounded to: gradients of queries and keys 1.0 to 1.1 times as far from 64 bits as this, 1.4 to 3 times where keys or values
// have a common offset.)
//
// a tile of the lane's row of p as (key, query)
__device__ __forceinline__ f16v row_of_p(const hdet_attn_f32_desc& t, const head& hd, int kt, int i, int half) {
  const int S = t.seq_len;
  const float* p = t.p + (hd.hd * S + i) * S;
  f16v pv;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int k0 = kt * 32 + acc_row(4 * g, half);
    if (i < S && k0 + 3 < S) {
      const f4u x = *reinterpret_cast<const f4u*>(p + k0);
#pragma unroll
      for (int e = 0; e < 4; ++e) pv[4 * g + e] = x[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) pv[4 * g + e] = i < S && k0 + e < S ? p[k0 + e] : 0.f;
    }
  }
  return pv;
}
// dp of the tile as (key, query)
template <int G>
__device__ __forceinline__ f16v keys_by_queries(const head& hd, const float (&df)[G][4], int kt, int last, int lane) {
  const int j = kt * 32 + (lane & 31);
  float vf[G][4];
  load_row<G>(vf, hd.v + (int64_t)(j < last ? j : last) * hd.ld, lane >> 5);
  return product<G>(vf, df);
}
// a tile of an [S][S] matrix of the head as (query, key), what lies above the diagonal zero
__device__ __forceinline__ f16v queries_by_keys(const float* m, int64_t hd, int qt, int j, int S, int half) {
  f16v x;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = qt * 32 + acc_row(e, half);
    x[e] = r < S && j < S && j <= r ? m[(hd * S + r) * S + j] : 0.f;
  }
  return x;
}
__device__ __forceinline__ void add_products(double& dot, const f16v& dp, const f16v& pv) {
#pragma unroll
  for (int e = 0; e < 16; ++e) dot += (double)dp[e] * (double)pv[e];
}

// Sequences of one tile: a wavefront each for dk, dv and dq; those of dk and dq form the row dots alike, that of dk forms dp once more in the order that its
// product wants (the same bits).
template <int G>
__global__ __launch_bounds__(192, 2) void attn_f32_bwd_tile_kernel(const hdet_attn_f32_desc t) {
  constexpr int NB = (G + 3) / 4, DH = 8 * G, C = 4;
  const head hd = head_of(t, (int)blockIdx.x);
  const int S = t.seq_len, last = S - 1, lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31, lc = l32 < last ? l32 : last;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* da = t.da + hd.at_a;
  float* out = t.dqkv + (hd.q - t.qkv);
  float cols[16][NB], df[G][4];
  f16v acc[C][NB], x;
  clear<C, NB>(acc);
  if (w == 1) {
    x = queries_by_keys(t.p, hd.hd, 0, l32, S, half);
    load_cols<NB>(cols, da, t.d_model, 0, last, DH, lane);
    out += 2 * t.d_model;
  } else {
    load_row<G>(df, da + (int64_t)lc * t.d_model, half);
    load_cols<NB>(cols, w == 0 ? hd.q : hd.k, hd.ld, 0, last, DH, lane);
    const f16v pv = row_of_p(t, hd, 0, l32, half), dp = keys_by_queries<G>(hd, df, 0, last, lane);
    double sum = 0.0;
    add_products(sum, dp, pv);
    const float dot = (float)(sum + __shfl_xor(sum, 32));
    if (w == 0) {
      float vf[G][4];
      load_row<G>(vf, hd.v + (int64_t)lc * hd.ld, half);
      const f16v pk = queries_by_keys(t.p, hd.hd, 0, l32, S, half), dk = product<G>(df, vf);
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e] = pk[e] * (dk[e] - __shfl(dot, acc_row(e, half))) * hd.scale;
      out += t.d_model;
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e] = pv[e] * (dp[e] - dot) * hd.scale;
    }
  }
  accumulate<C, NB>(acc, x, cols);
  add_up<C, NB>(acc);
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = acc_row(e, half), c = 32 * n + l32;
      if (r < S && c < DH) out[(int64_t)r * hd.ld + c] = acc[0][n][e];
    }
}

// Longer ones, first launch: blocks of queries hold their row's dp as the forward holds its scores, leave ds at and below the diagonal's tiles and form dq;
// blocks of keys form dv.
template <int G, int NT, int C>
__global__ __launch_bounds__(kThreads, 2) void attn_f32_bwd_dq_dv_kernel(const hdet_attn_f32_desc t, int nblk) {
  constexpr int NB = (G + 3) / 4, DH = 8 * G;
  __shared__ float red[kWaves * NB * 16 * 64];
  __shared__ double rdot[kWaves][32];
  const head hd = head_of(t, (int)blockIdx.x);
  const int rank = (int)blockIdx.y, S = t.seq_len, last = S - 1;
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* da = t.da + hd.at_a;
  float* out = t.dqkv + (hd.q - t.qkv);
  f16v acc[C][NB];
  clear<C, NB>(acc);
  if (rank & 1) {                                                    // blocks of queries and of keys in turn, the longest first
    const int kb = rank >> 1, j = kb * 32 + l32;
#pragma unroll 1
    for (int qt = kb + w; qt < nblk; qt += kWaves) {
      float cols[16][NB];
      load_cols<NB>(cols, da, t.d_model, qt * 32, last, DH, lane);
      accumulate<C, NB>(acc, queries_by_keys(t.p, hd.hd, qt, j, S, half), cols);
    }
    write_sum<C, NB>(acc, red, out + 2 * t.d_model, hd.ld, kb * 32, S, DH, lane, w);
    return;
  }
  const int qb = nblk - 1 - (rank >> 1), i = qb * 32 + l32;
  constexpr bool kHold = NT < 4;                                     // p and the first keys too; with four tiles of dp the registers end there
  f16v dp[NT], pv[kHold ? NT : 1];
  float cols[16][NB];
  double sum = 0.0;
  {
    float df[G][4];
    load_row<G>(df, da + (int64_t)(i < last ? i : last) * t.d_model, half);
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int kt = w + kWaves * u;
      if (kt > qb) continue;                                         // uniform over the wavefront
      f16v& pu = pv[kHold ? u : 0];
      pu = row_of_p(t, hd, kt, i, half);
      dp[u] = keys_by_queries<G>(hd, df, kt, last, lane);
      if (kHold && u == 0) load_cols<NB>(cols, hd.k, hd.ld, kt * 32, last, DH, lane);      // on their way while the wavefronts meet
      add_products(sum, dp[u], pu);
    }
  }
  sum += __shfl_xor(sum, 32);
  if (lane < 32) rdot[w][lane] = sum;
  __syncthreads();
  const float dot = (float)(((rdot[0][l32] + rdot[1][l32]) + rdot[2][l32]) + rdot[3][l32]);
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int kt = w + kWaves * u;
    if (kt > qb) continue;
    if (!kHold || u > 0) load_cols<NB>(cols, hd.k, hd.ld, kt * 32, last, DH, lane);
    f16v& pu = pv[kHold ? u : 0];
    if (!kHold) pu = row_of_p(t, hd, kt, i, half);
#pragma unroll
    for (int e = 0; e < 16; ++e) dp[u][e] = pu[e] * (dp[u][e] - dot) * hd.scale;
    if (i < S) store_row(t.ds + (hd.hd * S + i) * S, dp[u], kt, half, S);
    accumulate<C, NB>(acc, dp[u], cols);
  }
  write_sum<C, NB>(acc, red, out, hd.ld, qb * 32, S, DH, lane, w);
}

// second launch: dk
template <int G, int C>
__global__ __launch_bounds__(kThreads) void attn_f32_bwd_dk_kernel(const hdet_attn_f32_desc t, int nblk) {
  constexpr int NB = (G + 3) / 4, DH = 8 * G;
  __shared__ float red[kWaves * NB * 16 * 64];
  const head hd = head_of(t, (int)blockIdx.x);
  const int kb = (int)blockIdx.y, S = t.seq_len, lane = threadIdx.x & 63, half = lane >> 5, j = kb * 32 + (lane & 31);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f16v acc[C][NB];
  clear<C, NB>(acc);
#pragma unroll 1
  for (int qt = kb + w; qt < nblk; qt += kWaves) {
    float cols[16][NB];
    load_cols<NB>(cols, hd.q, hd.ld, qt * 32, S - 1, DH, lane);
    accumulate<C, NB>(acc, queries_by_keys(t.ds, hd.hd, qt, j, S, half), cols);
  }
  write_sum<C, NB>(acc, red, t.dqkv + (hd.q - t.qkv) + t.d_model, hd.ld, kb * 32, S, DH, lane, w);
}

}  // namespace

bool hdet_attn_f32_fusable(int seq_len, int d_model, int heads) {
  const int dh = d_model / heads;
  return dh % 8 == 0 && dh <= 64 && seq_len <= 512;
}

#define HDET_ATTN_HEAD(dh, CALL) \
  switch (dh) { case 8: CALL(1); break; case 16: CALL(2); break; case 24: CALL(3); break; case 32: CALL(4); break; \
                case 40: CALL(5); break; case 48: CALL(6); break; case 56: CALL(7); break; default: CALL(8); break; }

// Heads along the grid's x, which takes as many as the separate products take; row blocks along y, at most 32, so that all of a rank come before the next.
hipError_t hdet_launch_attn_f32_fwd(const hdet_attn_f32_desc& t, hipStream_t s) {
  if (!hdet_attn_f32_fusable(t.seq_len, t.d_model, t.heads)) return hipErrorInvalidValue;
  const int nblk = (t.seq_len + 31) / 32;
  const dim3 grid((unsigned)(t.n_replicas * t.batch * t.heads), nblk);
#define FWD(G)                                                                                                              \
  if (nblk == 1) hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 1, 4>), grid, dim3(kThreads), 0, s, t, nblk);                   \
  else if (nblk <= 4) hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 1, 2>), grid, dim3(kThreads), 0, s, t, nblk);              \
  else if (nblk <= 8) hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 2, 1>), grid, dim3(kThreads), 0, s, t, nblk);              \
  else hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 4, 1>), grid, dim3(kThreads), 0, s, t, nblk)
  HDET_ATTN_HEAD(t.d_model / t.heads, FWD)
#undef FWD
  return hipGetLastError();
}

hipError_t hdet_launch_attn_f32_bwd(const hdet_attn_f32_desc& t, hipStream_t s) {
  if (!hdet_attn_f32_fusable(t.seq_len, t.d_model, t.heads)) return hipErrorInvalidValue;
  const int nblk = (t.seq_len + 31) / 32;
  const unsigned heads = (unsigned)(t.n_replicas * t.batch * t.heads);
  const dim3 both(heads, 2 * nblk), keys(heads, nblk);
#define DQ_DV(G, NT, C) hipLaunchKernelGGL((attn_f32_bwd_dq_dv_kernel<G, NT, C>), both, dim3(kThreads), 0, s, t, nblk)
#define DK(G, C) hipLaunchKernelGGL((attn_f32_bwd_dk_kernel<G, C>), keys, dim3(kThreads), 0, s, t, nblk)
#define BWD(G)                                                                                                   \
  if (nblk == 1) hipLaunchKernelGGL((attn_f32_bwd_tile_kernel<G>), dim3(heads), dim3(192), 0, s, t);             \
  else if (nblk <= 4) { DQ_DV(G, 1, 2); DK(G, 2); }                                                              \
  else if (nblk <= 8) { DQ_DV(G, 2, 1); DK(G, 1); }                                                              \
  else { DQ_DV(G, 4, 1); DK(G, 1); }
  HDET_ATTN_HEAD(t.d_model / t.heads, BWD)
#undef BWD
#undef DK
#undef DQ_DV
  return hipGetLastError();
}
