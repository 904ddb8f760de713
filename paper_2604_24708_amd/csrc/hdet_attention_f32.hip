// Causal attention of the full-precision path, one launch forward and one backward, for head sizes of whole groups of 8 up to 64 and
// sequences up to 512 (other shapes: products and softmax kernels of their own).
//
// What bounds it: the sizes of this path (a few dozen to a few hundred rows) make it latency, one dependent launch after the other.  Three launches
// each way with the scores, probabilities and their gradients going through memory between them become one; only the probabilities are kept, for the
// backward.  us, three launches -> one, forward / backward, gaps between the launches not counted (heads over all replicas and sequences, S, head size):
//   64, 32, 16 11.8 -> 5.0 / 11.5 -> 5.7;  64, 128, 64 16.8 -> 9 / 20.3 -> 16.5;  288, 192, 32 57 -> 24 / 92 -> 50;  288, 192, 64 69 -> 44 / 101 -> 100;
//   64, 256, 64 30 -> 17 / 40 -> 35;  64, 512, 64 78 -> 45 / 136 -> 95;  256, 512, 64 312 -> 163 / 507 -> 384
// The backward is told to take registers for two wavefronts a SIMD: with 256 the loads of a whole tile are in flight (95 us at S = 512; 125 with the
// 180 that the compiler takes by itself, 134 with 168).
//
// fp32 products on the matrix cores (v_mfma_f32_32x32x2_f32), a block of four wavefronts to 32 queries (or keys) of a head:
//  * A wavefront takes every fourth tile of 32 x 32 of the other side, at and below the diagonal only, fragments straight from global memory.
//  * The first product is formed with the axis that the second contracts over as its rows: a lane's sixteen accumulators are then four groups of four
//    consecutive entries of that axis for one column, which is the second product's first operand as it stands.  Neither scores nor probabilities
//    touch LDS.
//  * Row maximum and sum, then the four wavefronts' partial results, meet in LDS and are added in the order of the wavefronts.
//  * sum_j dp_ij p_ij = da_i . a_i, so that the backward needs no row of dp at a time: blocks of queries form dq, blocks of keys dk and dv, each from
//    its own tiles of dp.

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
// NC: sums over the row, each half as long with two
template <int G, int NC = 1>
__device__ __forceinline__ f16v product(const float (&a)[G][4], const float (&b)[G][4]) {
  f16v acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = zero16();
#pragma unroll
  for (int c = 0; c < G; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[c % NC] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][j], b[c][j], acc[c % NC], 0, 0, 0);
  return NC > 1 && G > 1 ? acc[0] + acc[NC - 1] : acc[0];
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
template <int NB>
__device__ __forceinline__ void accumulate(f16v (&acc)[NB], const f16v& a, const float (&b)[16][NB]) {
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e][n], acc[n], 0, 0, 0);
}
// the wavefronts' partial [32][DH] results added in their order and written: rows r0 .. (below S) of an [S][DH] matrix
template <int NB>
__device__ __forceinline__ void write_sum(const f16v (&acc)[NB], float* red, float* m, int64_t ld, int r0, int S, int dh, int lane, int w) {
  float* mine = red + w * (NB * 16 * 64) + lane;
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int e = 0; e < 16; ++e) mine[(n * 16 + e) * 64] = acc[n][e];
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

struct head { const float* q; const float* k; const float* v; int64_t ld; float scale; int64_t hd, at_a; };
__device__ __forceinline__ head head_of(const hdet_attn_f32_desc& t, int hd) {
  const int h = hd % t.heads, b = hd / t.heads, dh = t.d_model / t.heads, r = b / t.batch;
  const float* q = t.qkv + (int64_t)b * t.seq_len * 3 * t.d_model + h * dh;
  float scale = t.scale;
  if (t.temp_channel >= 0) scale = scale / (float)hdet_channel_value(t.ctrl, t.temp_channel, r, 0.0);
  return {q, q + t.d_model, q + 2 * t.d_model, 3 * (int64_t)t.d_model, scale, hd, (int64_t)b * t.seq_len * t.d_model + h * dh};
}

// NT: 32-key tiles a wavefront holds; G = DH / 8; NB = ceil(DH / 32)
template <int G, int NT>
__global__ __launch_bounds__(kThreads) void attn_f32_fwd_kernel(const hdet_attn_f32_desc t, int nblk) {
  constexpr int NB = (G + 3) / 4, DH = 8 * G;
  __shared__ float red[kWaves * NB * 16 * 64];
  __shared__ float rmax[kWaves][32], rsum[kWaves][32];
  const int qb = nblk - 1 - (int)blockIdx.y;                         // the longest rows first
  const head hd = head_of(t, (int)blockIdx.x);
  const int S = t.seq_len, last = S - 1, lane = threadIdx.x & 63, half = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = qb * 32 + (lane & 31);
  float qf[G][4];
  load_row<G>(qf, hd.q + (int64_t)(i < last ? i : last) * hd.ld, half);
  f16v s[NT];
  float vf[NT][16][NB];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int kt = w + kWaves * u;
    if (kt > qb) continue;                                           // uniform over the wavefront
    float kf[G][4];
    const int j = kt * 32 + (lane & 31);
    load_row<G>(kf, hd.k + (int64_t)(j < last ? j : last) * hd.ld, half);
    load_cols<NB>(vf[u], hd.v, hd.ld, kt * 32, last, DH, lane);      // on their way under the softmax
    s[u] = product<G, 2>(kf, qf);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[u][e] = kt * 32 + acc_row(e, half) <= i ? s[u][e] * hd.scale : -INFINITY;
      mx = fmaxf(mx, s[u][e]);
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (lane < 32) rmax[w][lane] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(rmax[0][lane & 31], rmax[1][lane & 31]), fmaxf(rmax[2][lane & 31], rmax[3][lane & 31]));
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    if (w + kWaves * u > qb) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) { s[u][e] = expf(s[u][e] - mx); sum += s[u][e]; }
  }
  sum += __shfl_xor(sum, 32);
  if (lane < 32) rsum[w][lane] = sum;
  __syncthreads();
  const float inv = 1.f / (((rsum[0][lane & 31] + rsum[1][lane & 31]) + rsum[2][lane & 31]) + rsum[3][lane & 31]);
  f16v acc[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) acc[n] = zero16();
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int kt = w + kWaves * u;
    if (kt > qb) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[u][e] *= inv;
    if (i < S) {
      float* p = t.p + (hd.hd * S + i) * S;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int j = kt * 32 + acc_row(4 * g, half);
        if (j + 3 < S) *reinterpret_cast<f4u*>(p + j) = f4u{s[u][4 * g], s[u][4 * g + 1], s[u][4 * g + 2], s[u][4 * g + 3]};
        else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < S) p[j + e] = s[u][4 * g + e];
        }
      }
    }
    accumulate<NB>(acc, s[u], vf[u]);
  }
  write_sum<NB>(acc, red, t.a + hd.at_a, t.d_model, qb * 32, S, DH, lane, w);
}

// da . a of the lane's row (the same in both halves)
template <int G>
__device__ __forceinline__ float row_dot(const float (&da)[G][4], const float* a, int half) {
  float af[G][4];
  double d = 0.0;                                                    // what it is off by, every entry of the row's ds is off by
  load_row<G>(af, a, half);
#pragma unroll
  for (int c = 0; c < G; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) d += (double)da[c][j] * (double)af[c][j];
  return (float)(d + __shfl_xor(d, 32));
}

template <int G>
__global__ __launch_bounds__(kThreads, 2) void attn_f32_bwd_kernel(const hdet_attn_f32_desc t, int nblk) {
  constexpr int NB = (G + 3) / 4, DH = 8 * G;
  __shared__ float red[kWaves * NB * 16 * 64];
  const int rank = (int)blockIdx.y, S = t.seq_len, last = S - 1;
  const head hd = head_of(t, (int)blockIdx.x);
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* da = t.da + hd.at_a;
  const float* a = t.a + hd.at_a;
  const float* p = t.p + hd.hd * S * S;
  float* dq = t.dqkv + (hd.q - t.qkv);
  const bool keys = (rank & 1) == 0;                                 // blocks of keys and of queries in turn, the longest first
  if (keys) {
    const int kb = rank >> 1, j = kb * 32 + l32;
    float vf[G][4];
    load_row<G>(vf, hd.v + (int64_t)(j < last ? j : last) * hd.ld, half);
    f16v dk[NB], dv[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) { dk[n] = zero16(); dv[n] = zero16(); }
#pragma unroll 1
    for (int qt = kb + w; qt < nblk; qt += kWaves) {
      const int i = qt * 32 + l32, ic = i < last ? i : last;
      float df[G][4], cols[16][NB];
      load_row<G>(df, da + (int64_t)ic * t.d_model, half);
      f16v pv;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = qt * 32 + acc_row(e, half);
        pv[e] = r < S && j < S && j <= r ? p[(int64_t)r * S + j] : 0.f;
      }
      load_cols<NB>(cols, da, t.d_model, qt * 32, last, DH, lane);
      const float dot = row_dot<G>(df, a + (int64_t)ic * t.d_model, half);
      f16v ds = product<G>(df, vf);                                  // rows: queries, columns: keys
      accumulate<NB>(dv, pv, cols);
      load_cols<NB>(cols, hd.q, hd.ld, qt * 32, last, DH, lane);
#pragma unroll
      for (int e = 0; e < 16; ++e) ds[e] = pv[e] * (ds[e] - __shfl(dot, acc_row(e, half))) * hd.scale;
      accumulate<NB>(dk, ds, cols);
    }
    write_sum<NB>(dk, red, dq + t.d_model, hd.ld, kb * 32, S, DH, lane, w);
    __syncthreads();
    write_sum<NB>(dv, red, dq + 2 * t.d_model, hd.ld, kb * 32, S, DH, lane, w);
  } else {
    const int qb = nblk - 1 - (rank >> 1), i = qb * 32 + l32, ic = i < last ? i : last;
    float df[G][4];
    load_row<G>(df, da + (int64_t)ic * t.d_model, half);
    const float dot = row_dot<G>(df, a + (int64_t)ic * t.d_model, half);
    f16v acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = zero16();
#pragma unroll 1
    for (int kt = w; kt <= qb; kt += kWaves) {
      const int j = kt * 32 + l32;
      float vf[G][4], cols[16][NB];
      load_row<G>(vf, hd.v + (int64_t)(j < last ? j : last) * hd.ld, half);
      f16v pv;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int k0 = kt * 32 + acc_row(4 * g, half);
        if (i < S && k0 + 3 < S) {
          const f4u x = *reinterpret_cast<const f4u*>(p + (int64_t)i * S + k0);
#pragma unroll
          for (int e = 0; e < 4; ++e) pv[4 * g + e] = x[e];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) pv[4 * g + e] = i < S && k0 + e < S ? p[(int64_t)i * S + k0 + e] : 0.f;
        }
      }
      load_cols<NB>(cols, hd.k, hd.ld, kt * 32, last, DH, lane);
      f16v ds = product<G>(vf, df);                                  // rows: keys, columns: queries
#pragma unroll
      for (int e = 0; e < 16; ++e) ds[e] = pv[e] * (ds[e] - dot) * hd.scale;
      accumulate<NB>(acc, ds, cols);
    }
    write_sum<NB>(acc, red, dq, hd.ld, qb * 32, S, DH, lane, w);
  }
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
  if (nblk <= 4) hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 1>), grid, dim3(kThreads), 0, s, t, nblk);                      \
  else if (nblk <= 8) hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 2>), grid, dim3(kThreads), 0, s, t, nblk);                 \
  else hipLaunchKernelGGL((attn_f32_fwd_kernel<G, 4>), grid, dim3(kThreads), 0, s, t, nblk)
  HDET_ATTN_HEAD(t.d_model / t.heads, FWD)
#undef FWD
  return hipGetLastError();
}

hipError_t hdet_launch_attn_f32_bwd(const hdet_attn_f32_desc& t, hipStream_t s) {
  if (!hdet_attn_f32_fusable(t.seq_len, t.d_model, t.heads)) return hipErrorInvalidValue;
  const int nblk = (t.seq_len + 31) / 32;
  const dim3 grid((unsigned)(t.n_replicas * t.batch * t.heads), 2 * nblk);
#define BWD(G) hipLaunchKernelGGL((attn_f32_bwd_kernel<G>), grid, dim3(kThreads), 0, s, t, nblk)
  HDET_ATTN_HEAD(t.d_model / t.heads, BWD)
#undef BWD
  return hipGetLastError();
}
