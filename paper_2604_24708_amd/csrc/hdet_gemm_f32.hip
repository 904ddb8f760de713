// Replica-batched fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums) for the
// full-precision model path: element strides select which of forward / dgrad / wgrad it is, the batch index selects
// the replica (and, for attention, the sequence and head).
//
// What bounds it: the products of this path are small (a replica's batch of a few dozen to a few thousand rows), so
// it is the length of a block's serial K loop and the number of wavefronts in flight, not the matrix rate, that
// counts.  Hence:
//  * No LDS on the operand path and no barrier in the loop: a wavefront loads its MFMA fragments straight from
//    global memory (L1 / L2 serve the reuse) a few steps ahead.  A lane of an 8-k step holds k = 4 (lane / 32) + j
//    for MFMA j = 0..3 -- any assignment of k to MFMAs is right as long as A and B agree -- so that an operand
//    contiguous along k is one 16-byte load per lane and 32 x 8 block, and one contiguous along its output axis is
//    four loads of whole 128-byte lines.
//  * The wavefronts of a block may split K (WK > 1): each walks its own contiguous part, the partial tiles meet in
//    LDS and are added in ascending order of k, every wavefront finishing 1 / WK of the tile.  A 32 x 32 tile with
//    K = 1024 in 8 parts is 16 steps per wavefront instead of 128.
// Loads are dword aligned only (odd leading dimensions are common here); rows beyond the matrix are clamped to its
// last row (their results are not stored), the K mod 8 tail is a separate masked step.
// Measured against a 64 x 64 tile staged through LDS on the vector units (us per launch, 4 replicas, same box):
//   512 x 256, K = 1024 (NT)  152 -> 17;   512 x 256, K = 4000 (NN)  270 -> 46;   4000 x 256, K = 512 (TN)  104 -> 46 (91 TFLOP/s);
//   128 x 64, K = 64 (NT)     15 -> 4;     128 x 64, K = 512 (NN)    80 -> 6.

#include "hdet_internal.h"

namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// 32 rows x 8 k of an operand as the four MFMAs' fragments.  KFAST: element (row, k) at [row * ld + k], else [k * ld + row].
// `base` is uniform and points at (first row of the tile, k of the step); `lane_off` is the lane's own element offset.
template <bool KFAST>
__device__ __forceinline__ int64_t lane_offset(int row0, int rows, int64_t ld, int lane) {
  int row = lane & 31;
  if (row0 + row >= rows) row = rows - 1 - row0;                    // row0 < rows: the last row again
  const int kk = (lane >> 5) << 2;
  return KFAST ? row * ld + kk : kk * ld + row;
}
template <bool KFAST>
__device__ __forceinline__ void load_step(float (&v)[4], const float* base, int64_t lane_off, int64_t ld) {
  if (KFAST) {
    const f4u x = *reinterpret_cast<const f4u*>(base + lane_off);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = x[j];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (base + j * ld)[lane_off];
  }
}
// the K mod 8 tail: `kleft` valid k, zeros behind them
template <bool KFAST>
__device__ __forceinline__ void load_tail(float (&v)[4], const float* base, int64_t lane_off, int64_t ld, int kleft, int lane) {
  const int kk = (lane >> 5) << 2;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = 0.f;
    if (kk + j < kleft) v[j] = KFAST ? base[lane_off + j] : (base + j * ld)[lane_off];
  }
}

// Wave tile (32 WTM) x (32 WTN); WM x WN x WK wavefronts; U: 8-k steps loaded ahead.
template <bool AK, bool BK, int EPI, int WTM, int WTN, int WM, int WN, int WK, int U>
__global__ __launch_bounds__(64 * WM * WN * WK) void sgemm_kernel(const hdet_sgemm_args g) {
  constexpr int NW = WTM * WTN * 16;                                // accumulator registers
  static_assert(WK == 1 || NW % WK == 0, "the wavefronts of a K split share the tile's registers evenly");
  __shared__ float part[WK > 1 ? WM * WN * WK * NW * 64 : 1];
  // launch order -> tile: XCD x (own L2; launch index mod 8) takes the x-th of eight contiguous ranges of tiles
  unsigned bx, by, bz;
  {
    const unsigned total = gridDim.x * gridDim.y * gridDim.z;
    unsigned t = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned x = t & 7u, rem = total & 7u;
    t = x * (total >> 3) + (x < rem ? x : rem) + (t >> 3);
    bx = t % gridDim.x;
    by = (t / gridDim.x) % gridDim.y;
    bz = t / (gridDim.x * gridDim.y);
  }
  const hdet_batch_index bi = hdet_split_batch(bz, g.n1, g.n2);
  const int z = bi.z0;                                              // replica: bias and mask are per replica
  const float* A = g.a + hdet_batch_offset(bi, g.a_s);
  const float* B = g.b + hdet_batch_offset(bi, g.b_s);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = w % WK, wmn = w / WK;
  const int m0 = (by * WM + wmn / WN) * (32 * WTM), n0 = (bx * WN + wmn % WN) * (32 * WTN);
  const bool active = m0 < g.m && n0 < g.n;                         // uniform over the wavefront
  const int64_t lda = AK ? g.a_rs : g.a_cs, ldb = BK ? g.b_cs : g.b_rs;

  f16v acc[WTM][WTN];
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int j = 0; j < WTN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  if (active) {
    const float* abase[WTM];
    const float* bbase[WTN];
    int64_t aoff[WTM], boff[WTN];
#pragma unroll
    for (int i = 0; i < WTM; ++i) {
      const int r0 = m0 + 32 * i < g.m ? m0 + 32 * i : m0;          // a 32-row group beyond the matrix repeats the first one
      abase[i] = A + (AK ? r0 * lda : (int64_t)r0);
      aoff[i] = lane_offset<AK>(r0, g.m, lda, lane);
    }
#pragma unroll
    for (int j = 0; j < WTN; ++j) {
      const int r0 = n0 + 32 * j < g.n ? n0 + 32 * j : n0;
      bbase[j] = B + (BK ? r0 * ldb : (int64_t)r0);
      boff[j] = lane_offset<BK>(r0, g.n, ldb, lane);
    }
    const int64_t astep = AK ? 8 : 8 * lda, bstep = BK ? 8 : 8 * ldb;
    const int nfull = g.k >> 3, per = (nfull + WK - 1) / WK;
    const int c0 = wk * per < nfull ? wk * per : nfull, c1 = c0 + per < nfull ? c0 + per : nfull;

    float a[2][U][WTM][4], b[2][U][WTN][4];
    auto fetch = [&](int buf, int c) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int cc = c + u < c1 ? c + u : c1 - 1;                 // past the end: the last step again, not used
#pragma unroll
        for (int i = 0; i < WTM; ++i) load_step<AK>(a[buf][u][i], abase[i] + cc * astep, aoff[i], lda);
#pragma unroll
        for (int j = 0; j < WTN; ++j) load_step<BK>(b[buf][u][j], bbase[j] + cc * bstep, boff[j], ldb);
      }
    };
    auto step = [&](float (&av)[WTM][4], float (&bv)[WTN][4]) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
          for (int j = 0; j < WTN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][q], bv[j][q], acc[i][j], 0, 0, 0);
    };
    if (c0 < c1) {
      fetch(0, c0);
      for (int c = c0; c < c1; c += 2 * U) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int cur = c + half * U;
          if (cur < c1) {
            if (cur + U < c1) fetch(half ^ 1, cur + U);
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (u == 0 || cur + u < c1) step(a[half][u], b[half][u]);
          }
        }
      }
    }
    const int kleft = g.k & 7;
    if (kleft && wk == WK - 1) {
      float av[WTM][4], bv[WTN][4];
#pragma unroll
      for (int i = 0; i < WTM; ++i) load_tail<AK>(av[i], abase[i] + nfull * astep, aoff[i], lda, kleft, lane);
#pragma unroll
      for (int j = 0; j < WTN; ++j) load_tail<BK>(bv[j], bbase[j] + nfull * bstep, boff[j], ldb, kleft, lane);
      step(av, bv);
    }
  }

  float* C = g.c + hdet_batch_offset(bi, g.c_s);
  // accumulator register e of lane l is C(row, col) with row = (e / 4) * 8 + (l / 32) * 4 + e % 4, col = l % 32 in its block
  auto put = [&](int i, int j, int e, float v) {
    const int row = m0 + 32 * i + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = n0 + 32 * j + (lane & 31);
    if (row >= g.m || col >= g.n) return;
    if (EPI == HDET_SEPI_BIAS || EPI == HDET_SEPI_BIAS_RELU) v += g.bias[(int64_t)z * g.bias_bs + col];
    if (EPI == HDET_SEPI_BIAS_RELU) v = v > 0.f ? v : 0.f;
    if (EPI == HDET_SEPI_MASK) v = g.mask[(int64_t)z * g.mask_bs + (int64_t)row * g.mask_rs + col] > 0.f ? v : 0.f;
    C[(int64_t)row * g.c_rs + col] = v;
  };
  if (WK == 1) {
    if (!active) return;
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) put(i, j, e, acc[i][j][e]);
  } else {
    float* mine = part + (wmn * WK + wk) * (NW * 64) + lane;        // [register][lane] of this wavefront's partial tile
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) mine[((i * WTN + j) * 16 + e) * 64] = acc[i][j][e];
    __syncthreads();
    if (!active) return;
    const float* all = part + wmn * WK * (NW * 64) + lane;
#pragma unroll
    for (int t = 0; t < NW / WK; ++t) {
      const int q = wk * (NW / WK) + t;
      float v = all[q * 64];
#pragma unroll
      for (int p = 1; p < WK; ++p) v += all[(p * NW + q) * 64];
      put(q / (16 * WTN), (q / 16) % WTN, q % 16, v);
    }
  }
}

// operand orders: forward (NT: both contiguous along k), dgrad (NN: A along k), wgrad (TN: neither)
enum { kNT = 0, kNN = 1, kTN = 2 };

template <int FORM, int EPI, int WTM, int WTN, int WM, int WN, int WK, int U>
void launch_cfg(const hdet_sgemm_args& g, int batch, hipStream_t s) {
  const int tm = 32 * WTM * WM, tn = 32 * WTN * WN;
  const dim3 grid((g.n + tn - 1) / tn, (g.m + tm - 1) / tm, batch);
  hipLaunchKernelGGL((sgemm_kernel<FORM != kTN, FORM == kNT, EPI, WTM, WTN, WM, WN, WK, U>), grid, dim3(64 * WM * WN * WK), 0, s, g);
}

// Tile and K split by the number of blocks a launch would have, b(tm x tn) = tiles over the whole batch, on 256 CUs
// (microseconds over 8 replicas or as given, same box; chosen | other candidates):
//   few tiles: 32 x 32, K in 4.        128 x 64, K = 64, 4 items: 3.9 | 64 x 32 4.3 | 64 x 64 5.2 (K in 8: 4.3, in 16: 4.1)
//   up to one 64 x 32 block per CU (and at least 5/8 of them), K in 4:
//                                      512 x 256, K = 1024, 4 items: 15.4 | 32 x 32 22.4 | 64 x 64 22.8
//   up to one 64 x 64 block per CU, K in 4:
//                                      256 x 1024, K = 512, 4 items, wgrad: 14.9 | 64 x 32 23.4 | 64 x 128 24.5
//   more: 64 x 128, K in 2             512 x 1024, K = 256, 4 items: 18.0 | 64 x 64 24.6 | 64 x 32 27.2
//   many, an operand contiguous along k: 64 x 64 with two steps in flight instead of four, whose smaller register count lets a
//         CU hold more of them         4096 x 2048, K = 512, 8 items: 798 | 64 x 128 910 (wgrad: 914 | 64 x 128 588)
template <int FORM, int EPI>
void launch_form(const hdet_sgemm_args& g, int batch, hipStream_t s) {
  auto blocks = [&](int tm, int tn) { return (int64_t)((g.m + tm - 1) / tm) * ((g.n + tn - 1) / tn) * batch; };
  const int cus = hdet_compute_units();
  const int64_t b32 = blocks(64, 32), b128 = blocks(64, 128);
  if (b32 * 8 < (int64_t)cus * 5) launch_cfg<FORM, EPI, 1, 1, 1, 1, 4, 4>(g, batch, s);
  else if (b32 <= cus) launch_cfg<FORM, EPI, 2, 1, 1, 1, 4, 4>(g, batch, s);
  else if (blocks(64, 64) <= cus) launch_cfg<FORM, EPI, 2, 2, 1, 1, 4, 4>(g, batch, s);
  else if (FORM == kTN || b128 <= 2 * (int64_t)cus) launch_cfg<FORM, EPI, 2, 2, 1, 2, 2, 4>(g, batch, s);
  else launch_cfg<FORM, EPI, 2, 2, 1, 1, 4, 2>(g, batch, s);
}

}  // namespace

hipError_t hdet_launch_sgemm(const hdet_sgemm_args& g_in, int epi, int batch, hipStream_t s) {
  hdet_sgemm_args g = g_in;
  if (g.n1 < 1) g.n1 = 1;
  if (g.n2 < 1) g.n2 = 1;
  // which axis of an operand is contiguous (an operand of one row or column may be read either way)
  const bool ak = g.a_cs == 1, bk = g.b_rs == 1 && (ak || g.b_cs != 1);
  if ((!ak && g.a_rs != 1) || (!bk && g.b_cs != 1) || (!ak && bk)) return hipErrorInvalidValue;
  if (epi == HDET_SEPI_NONE) {
    if (ak && bk) launch_form<kNT, HDET_SEPI_NONE>(g, batch, s);
    else if (ak) launch_form<kNN, HDET_SEPI_NONE>(g, batch, s);
    else launch_form<kTN, HDET_SEPI_NONE>(g, batch, s);
  } else if (epi == HDET_SEPI_BIAS && ak && bk) {
    launch_form<kNT, HDET_SEPI_BIAS>(g, batch, s);
  } else if (epi == HDET_SEPI_BIAS_RELU && ak && bk) {
    launch_form<kNT, HDET_SEPI_BIAS_RELU>(g, batch, s);
  } else if (epi == HDET_SEPI_MASK && ak && g.b_cs == 1) {
    launch_form<kNN, HDET_SEPI_MASK>(g, batch, s);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
