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
//    K = 1024 in 4 parts is 32 steps per wavefront instead of 128.
// That is how small products and those of odd leading dimensions or addresses are formed (loads are dword aligned only); a product from about one tile
// a CU on whose operands are whole 16-byte chunks goes through LDS (sgemm_lds_tile).  Here rows beyond the matrix are clamped to its
// last row (their results are not stored), the K mod 8 tail is a separate masked step.
// Measured against a 64 x 64 tile staged through LDS on the vector units (us per launch, 4 replicas, same machine):
//   512 x 256, K = 1024 (NT)  152 -> 17;   512 x 256, K = 4000 (NN)  270 -> 46;   4000 x 256, K = 512 (TN)  104 -> 46 (91 TFLOP/s);
//   128 x 64, K = 64 (NT)     15 -> 4;     128 x 64, K = 512 (NN)    80 -> 6.

#include <algorithm>
#include <type_traits>

#include "hdet_elem.h"
#include "hdet_internal.h"
#include "hdet_lds.h"

namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f4a __attribute__((ext_vector_type(4)));

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

// operand orders: forward (NT: both contiguous along k), dgrad (NN: A along k), wgrad (TN: neither)
enum { kNT = 0, kNN = 1, kTN = 2 };

constexpr int kThreads = 256;      // every tile configuration is four wavefronts: they can share a launch

// One block's tile, tile index t of tx x ty x batch.  Wave tile (32 WTM) x (32 WTN); WM x WN x WK wavefronts; U: 8-k steps
// loaded ahead.  `part`: the block's LDS (lds_floats).
template <int WTM, int WTN, int WM, int WN, int WK> constexpr int lds_floats() { return WM * WN * WK * WTM * WTN * 16 * 64; }

template <bool AK, bool BK, int WTM, int WTN, int WM, int WN, int WK, int U>
__device__ __forceinline__ void sgemm_tile(const hdet_sgemm_args& g, int epi, unsigned t, unsigned tx, unsigned ty, unsigned total, float* part) {
  constexpr int NW = WTM * WTN * 16;                                // accumulator registers
  static_assert(WK > 1 && NW % WK == 0, "the wavefronts of a K split share the tile's registers evenly");
  static_assert(WM * WN * WK * 64 == kThreads, "four wavefronts");
  // launch order -> tile: XCD x (own L2; launch index mod 8) takes the x-th of eight contiguous ranges of tiles
  unsigned bx, by, bz;
  {
    const unsigned x = t & 7u, rem = total & 7u;
    t = x * (total >> 3) + (x < rem ? x : rem) + (t >> 3);
    bx = t % tx;
    by = (t / tx) % ty;
    bz = t / (tx * ty);
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
  const bool block_sums = !AK && g.rowsum && bx == 0;               // the wavefronts of the first tile column also add up A's rows
  const bool sums = block_sums && n0 == 0 && active;
  float rs[WTM];
#pragma unroll
  for (int i = 0; i < WTM; ++i) rs[i] = 0.f;
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
      if (!AK && sums) {
#pragma unroll
        for (int i = 0; i < WTM; ++i) rs[i] += (av[i][0] + av[i][1]) + (av[i][2] + av[i][3]);
      }
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
  float* mine = part + (wmn * WK + wk) * (NW * 64) + lane;          // [register][lane] of this wavefront's partial tile
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int j = 0; j < WTN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) mine[((i * WTN + j) * 16 + e) * 64] = acc[i][j][e];
  __syncthreads();
  const float* all = part + wmn * WK * (NW * 64) + lane;
  // accumulator register e of lane l is C(row, col) with row = (e / 4) * 8 + (l / 32) * 4 + e % 4, col = l % 32 in its block;
  // the epilogue is uniform over the launch
  auto finish = [&](auto kind) {
    constexpr int EPI = decltype(kind)::value;
    constexpr bool kBias = EPI == HDET_SEPI_BIAS || EPI == HDET_SEPI_BIAS_RELU || EPI == HDET_SEPI_BIAS_GELU || EPI == HDET_SEPI_BIAS_RESID;
    constexpr bool kMask = EPI == HDET_SEPI_MASK || EPI == HDET_SEPI_BIAS_RESID || EPI == HDET_SEPI_GELUGRAD;
    constexpr int CH = NW / WK < 8 ? NW / WK : 8;                   // elements whose second operand is requested together
#pragma unroll
    for (int t0 = 0; t0 < NW / WK; t0 += CH) {
      float x[CH], bias[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int q = wk * (NW / WK) + t0 + u, e = q % 16;
        const int row = m0 + 32 * (q / (16 * WTN)) + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = n0 + 32 * ((q / 16) % WTN) + (lane & 31);
        if (row < g.m && col < g.n) {
          if (kBias) bias[u] = g.bias[(int64_t)z * g.bias_bs + col];
          if (kMask) x[u] = g.mask[(int64_t)z * g.mask_bs + (int64_t)row * g.mask_rs + col];
        }
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int q = wk * (NW / WK) + t0 + u, e = q % 16;
        float v = all[q * 64];
#pragma unroll
        for (int p = 1; p < WK; ++p) v += all[(p * NW + q) * 64];
        const int row = m0 + 32 * (q / (16 * WTN)) + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = n0 + 32 * ((q / 16) % WTN) + (lane & 31);
        if (row >= g.m || col >= g.n) continue;
        const int64_t at = (int64_t)row * g.c_rs + col;
        if (kBias) v += bias[u];
        if (EPI == HDET_SEPI_BIAS_RELU) v = v > 0.f ? v : 0.f;
        if (EPI == HDET_SEPI_MASK) v = x[u] > 0.f ? v : 0.f;
        if (EPI == HDET_SEPI_BIAS_RESID) v += x[u];
        if (EPI == HDET_SEPI_GELUGRAD) v *= hdet_gelu_tanh_grad(x[u]);
        C[at] = v;
        if (EPI == HDET_SEPI_BIAS_GELU) (g.c2 + hdet_batch_offset(bi, g.c_s))[at] = hdet_gelu_tanh(v);
      }
    }
  };
  if (active) switch (epi) {
    case HDET_SEPI_NONE: finish(std::integral_constant<int, HDET_SEPI_NONE>{}); break;
    case HDET_SEPI_BIAS: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS>{}); break;
    case HDET_SEPI_BIAS_RELU: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS_RELU>{}); break;
    case HDET_SEPI_BIAS_GELU: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS_GELU>{}); break;
    case HDET_SEPI_BIAS_RESID: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS_RESID>{}); break;
    case HDET_SEPI_MASK: if (AK && !BK) finish(std::integral_constant<int, HDET_SEPI_MASK>{}); break;
    case HDET_SEPI_GELUGRAD: if (AK && !BK) finish(std::integral_constant<int, HDET_SEPI_GELUGRAD>{}); break;
  }
  if (block_sums) {
    float* rpart = part + wmn * WK * (WTM * 32);                    // [K part][row] of this wavefront's row sums
    __syncthreads();
    if (sums) {
#pragma unroll
      for (int i = 0; i < WTM; ++i) {
        const float v = rs[i] + __shfl_xor(rs[i], 32);              // the two halves of a step's k
        if (lane < 32) rpart[wk * (WTM * 32) + 32 * i + lane] = v;
      }
    }
    __syncthreads();
    if (sums)
      for (int r = wk * 64 + lane; r < WTM * 32; r += WK * 64) {
        if (m0 + r >= g.m) continue;
        float v = rpart[r];
#pragma unroll
        for (int p = 1; p < WK; ++p) v += rpart[p * (WTM * 32) + r];
        g.rowsum[(int64_t)z * g.rowsum_bs + m0 + r] = v;
      }
  }
}

template <int FORM, int WTM, int WTN, int WM, int WN, int WK, int U>
__global__ __launch_bounds__(kThreads) void sgemm_kernel(const hdet_sgemm_args g, int epi, unsigned tx, unsigned ty) {
  __shared__ float part[lds_floats<WTM, WTN, WM, WN, WK>()];
  sgemm_tile<FORM != kTN, FORM == kNT, WTM, WTN, WM, WN, WK, U>(g, epi, blockIdx.x, tx, ty, gridDim.x, part);
}

// ---- products of many tiles -----------------------------------------------------------------------------------------------------
// Operand tiles go straight into LDS (hdet_lds.h), NST stages of TK k, where the wavefronts share them.  What bounds such a product when
// wavefronts load their own fragments is the addresses: an operand contiguous along k costs a lane a row of its own, 32 lines a
// load, each of which is fetched again for every 8 k.  LDS holds
//  * an operand contiguous along k as [row][TK], the 16-byte chunks of a row XOR-permuted by the row: one 128-bit read a lane is four k of its row;
//  * one contiguous along its rows as [k][ROWS], odd groups of four k with the halves of 64 rows exchanged: four 32-bit reads.
// us, 4 replicas, fragments from global memory / through LDS:  512 x 4000, K = 256 85 / 50 (84 TFLOP/s);  512 x 1024, K = 256, both GELU outputs
// 27.9 / 19.5;  512 x 768, K = 256 21.6 / 15.1;  512 x 256, K = 256 and 1024 14.8 / 12;  weight gradients 4000 x 256, K = 512 53 / 45, 1024 x 256 15.9 / 14.9;
// 512 x 4096, K = 4096 428 / 321;  8 replicas, 1024 x 32000, K = 256 2459 / 1470.  Below two rounds of blocks some 6 us of each are launch, first
// loads and last stores.  Three or four stages instead of two, fragments read one group ahead, 32 x 32 tiles with K in 4 in place of 64 x 32: the
// same to 5 % slower; 128 x 64 tiles 2 to 60 % slower, for want of blocks.
constexpr uint32_t kAbsent = 0x80000000u;   // offset beyond every extent the host lets through
template <bool KMAJOR, int ROWS, int TK>
struct stage_tile {
  static constexpr int NI = ROWS * TK / (kThreads * 4), CPR = KMAJOR ? TK / 4 : ROWS / 4;     // loads a thread and stage, chunks a row
  uint32_t off[NI], kstep;
  int kofs[NI];
  __device__ __forceinline__ void init(int row0, int rows, int64_t ld, int tid) {
    kstep = KMAJOR ? TK * 4 : (uint32_t)(ld * TK * 4);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = tid + i * kThreads, hi = c / CPR, lo = c % CPR;
      if (KMAJOR) {
        kofs[i] = (lo ^ (hi & 7)) * 4;
        off[i] = row0 + hi < rows ? (uint32_t)(((row0 + hi) * ld + kofs[i]) * 4) : kAbsent;
      } else {
        const int row = row0 + (lo ^ (ROWS >= 64 ? (hi & 4) << 1 : 0)) * 4;
        kofs[i] = hi;
        off[i] = row < rows ? (uint32_t)((hi * ld + row) * 4) : kAbsent;
      }
    }
  }
  __device__ __forceinline__ void issue(hdet_rsrc rsrc, uint32_t addr, int kt, int kdim, int wave) const {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      lds_load16(rsrc, addr + (i * kThreads + wave * 64) * 16, kofs[i] + kt * TK < kdim ? off[i] + (uint32_t)kt * kstep : kAbsent);
  }
  // the four MFMAs' fragments of eight k (group q of the stage) and 32 rows from r0 on
  static __device__ __forceinline__ void fragment(float (&v)[4], const float* tile, int r0, int q, int lane) {
    if (KMAJOR) {
      const f4a x = *reinterpret_cast<const f4a*>(tile + (r0 + (lane & 31)) * TK + (((2 * q + (lane >> 5)) ^ (lane & 7)) << 2));
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = x[j];
    } else {
      const int h = lane >> 5, row = (r0 + (lane & 31)) ^ (ROWS >= 64 ? h << 5 : 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = tile[(8 * q + 4 * h + j) * ROWS + row];
    }
  }
};

// Block tile (32 WTM WM) x (32 WTN WN) by WM x WN x WK wavefronts of (32 WTM) x (32 WTN) each; with WK > 1 a stage's k are shared out.
template <int WTM, int WTN, int WM, int WN, int WK, int NST> constexpr int stage_floats() { return NST * 32 * (WTM * WM + WTN * WN) * 32 * WK; }
template <int FORM, int WTM, int WTN, int WM, int WN, int WK, int NST>
__device__ __forceinline__ void sgemm_lds_tile(const hdet_sgemm_args& g, int epi, unsigned t, unsigned tx, unsigned ty, unsigned total, float* S) {
  constexpr bool AK = FORM != kTN, BK = FORM == kNT;
  constexpr int BM = 32 * WTM * WM, BN = 32 * WTN * WN, TK = 32 * WK, STAGE = (BM + BN) * TK, NW = WTM * WTN * 16;
  static_assert(WM * WN * WK * 64 == kThreads, "four wavefronts");
  static_assert(WK == 1 || kThreads * NW <= NST * STAGE, "the parts of a K split meet in the stages");
  typedef stage_tile<AK, BM, TK> ta;
  typedef stage_tile<BK, BN, TK> tb;
  constexpr int LPT = ta::NI + tb::NI;
  {
    const unsigned x = t & 7u, rem = total & 7u;                      // as in sgemm_tile
    t = x * (total >> 3) + (x < rem ? x : rem) + (t >> 3);
  }
  const unsigned bx = t % tx, by = (t / tx) % ty, bz = t / (tx * ty);
  const hdet_batch_index bi = hdet_split_batch(bz, g.n1, g.n2);
  const int z = bi.z0, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = w % WK, wmn = w / WK, wm = (wmn / WN) * (32 * WTM), wn = (wmn % WN) * (32 * WTN);
  const int m0 = by * BM, n0 = bx * BN;
  const int64_t lda = AK ? g.a_rs : g.a_cs, ldb = BK ? g.b_cs : g.b_rs;
  const hdet_rsrc ra = make_rsrc(g.a + hdet_batch_offset(bi, g.a_s), (uint32_t)((((AK ? g.m : g.k) - 1) * lda + (AK ? g.k : g.m)) * 4));
  const hdet_rsrc rb = make_rsrc(g.b + hdet_batch_offset(bi, g.b_s), (uint32_t)((((BK ? g.n : g.k) - 1) * ldb + (BK ? g.k : g.n)) * 4));
  const uint32_t s_addr = lds_addr_of(reinterpret_cast<const uint16_t*>(S));
  ta la; tb lb;
  la.init(m0, g.m, lda, tid);
  lb.init(n0, g.n, ldb, tid);
  const bool block_sums = !AK && g.rowsum && bx == 0, sums = block_sums && wmn % WN == 0;
  // four sums over K, whichever wavefronts they are in: one long chain of additions is further from the exact sum (2-layer d = 256 transformer: 8.5e-7
  // of the gradients, 6e-7 with four)
  constexpr int NC = 4 / WK;
  float rs[WTM][NC];
  f16v chain[NC][WTM][WTN], (&acc)[WTM][WTN] = chain[0];
#pragma unroll
  for (int i = 0; i < WTM; ++i) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      rs[i][c] = 0.f;
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) chain[c][i][j][e] = 0.f;
    }
  }
  const int nk = (g.k + TK - 1) / TK;
  auto load = [&](int kt, int s) {
    la.issue(ra, s_addr + s * STAGE * 4, kt, g.k, w);
    lb.issue(rb, s_addr + (s * STAGE + BM * TK) * 4, kt, g.k, w);
  };
#pragma unroll
  for (int s = 0; s < NST - 1; ++s) load(s, s);
  for (int kt0 = 0; kt0 < nk; kt0 += NST) {
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      if (kt0 + s >= nk) break;
      wait_and_barrier<(NST - 2) * LPT>();                 // this stage has landed, and every wavefront has read the one before
      load(kt0 + s + NST - 1, (s + NST - 1) % NST);
      const float* at = S + s * STAGE;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float a[WTM][4], b[WTN][4];
#pragma unroll
        for (int i = 0; i < WTM; ++i) ta::fragment(a[i], at, wm + 32 * i, 4 * wk + q, lane);
#pragma unroll
        for (int j = 0; j < WTN; ++j) tb::fragment(b[j], at + BM * TK, wn + 32 * j, 4 * wk + q, lane);
        if (!AK && sums) {
#pragma unroll
          for (int i = 0; i < WTM; ++i) rs[i][q % NC] += (a[i][0] + a[i][1]) + (a[i][2] + a[i][3]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < WTN; ++j) chain[q % NC][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][u], b[j][u], chain[q % NC][i][j], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int c = 1; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int j = 0; j < WTN; ++j) acc[i][j] += chain[c][i][j];
  wait_and_barrier<0>();
  // rows of A summed: the two halves of a group's k, then the parts of the K split
  if (block_sums) {
    if (sums) {
#pragma unroll
      for (int i = 0; i < WTM; ++i) {
        float v = rs[i][0];
#pragma unroll
        for (int c = 1; c < NC; ++c) v += rs[i][c];
        v += __shfl_xor(v, 32);
        if (lane < 32) S[(wk * WM + wmn / WN) * (WTM * 32) + 32 * i + lane] = v;
      }
    }
    __syncthreads();
    if (tid < BM && m0 + tid < g.m) {
      float v = S[tid];
#pragma unroll
      for (int p = 1; p < WK; ++p) v += S[p * BM + tid];
      g.rowsum[(int64_t)z * g.rowsum_bs + m0 + tid] = v;
    }
    __syncthreads();
  }
  if (WK > 1) {
    float* mine = S + (wmn * WK + wk) * (NW * 64) + lane;
#pragma unroll
    for (int q = 0; q < NW; ++q) mine[q * 64] = acc[q / (16 * WTN)][(q / 16) % WTN][q % 16];
    __syncthreads();
  }
  const float* all = S + wmn * WK * (NW * 64) + lane;
  float* C = g.c + hdet_batch_offset(bi, g.c_s);
  float* C2 = g.c2 + hdet_batch_offset(bi, g.c_s);
  auto finish = [&](auto kind) {
    constexpr int EPI = decltype(kind)::value;
    constexpr bool kBias = EPI == HDET_SEPI_BIAS || EPI == HDET_SEPI_BIAS_RELU || EPI == HDET_SEPI_BIAS_GELU || EPI == HDET_SEPI_BIAS_RESID;
    constexpr bool kMask = EPI == HDET_SEPI_MASK || EPI == HDET_SEPI_BIAS_RESID || EPI == HDET_SEPI_GELUGRAD;
    constexpr int PER = NW / WK, CH = PER < 8 ? PER : 8;
    float bias[WTN];
#pragma unroll
    for (int j = 0; j < WTN; ++j) bias[j] = kBias && n0 + wn + 32 * j + (lane & 31) < g.n ? g.bias[(int64_t)z * g.bias_bs + n0 + wn + 32 * j + (lane & 31)] : 0.f;
#pragma unroll
    for (int t0 = 0; t0 < PER; t0 += CH) {
      float x[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int q = wk * PER + t0 + u, e = q % 16;
        const int row = m0 + wm + 32 * (q / (16 * WTN)) + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = n0 + wn + 32 * ((q / 16) % WTN) + (lane & 31);
        if (kMask && row < g.m && col < g.n) x[u] = g.mask[(int64_t)z * g.mask_bs + (int64_t)row * g.mask_rs + col];
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int q = wk * PER + t0 + u, e = q % 16;
        float v;
        if (WK > 1) {
          v = all[q * 64];
#pragma unroll
          for (int p = 1; p < WK; ++p) v += all[(p * NW + q) * 64];
        } else {
          const int r = t0 + u;
          v = acc[r / (16 * WTN)][(r / 16) % WTN][r % 16];
        }
        const int row = m0 + wm + 32 * (q / (16 * WTN)) + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = n0 + wn + 32 * ((q / 16) % WTN) + (lane & 31);
        if (row >= g.m || col >= g.n) continue;
        const int64_t to = (int64_t)row * g.c_rs + col;
        if (kBias) v += WK > 1 ? bias[(q / 16) % WTN] : bias[((t0 + u) / 16) % WTN];
        if (EPI == HDET_SEPI_BIAS_RELU) v = v > 0.f ? v : 0.f;
        if (EPI == HDET_SEPI_MASK) v = x[u] > 0.f ? v : 0.f;
        if (EPI == HDET_SEPI_BIAS_RESID) v += x[u];
        if (EPI == HDET_SEPI_GELUGRAD) v *= hdet_gelu_tanh_grad(x[u]);
        C[to] = v;
        if (EPI == HDET_SEPI_BIAS_GELU) C2[to] = hdet_gelu_tanh(v);
      }
    }
  };
  switch (epi) {
    case HDET_SEPI_NONE: finish(std::integral_constant<int, HDET_SEPI_NONE>{}); break;
    case HDET_SEPI_BIAS: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS>{}); break;
    case HDET_SEPI_BIAS_RELU: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS_RELU>{}); break;
    case HDET_SEPI_BIAS_GELU: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS_GELU>{}); break;
    case HDET_SEPI_BIAS_RESID: if (AK && BK) finish(std::integral_constant<int, HDET_SEPI_BIAS_RESID>{}); break;
    case HDET_SEPI_MASK: if (AK && !BK) finish(std::integral_constant<int, HDET_SEPI_MASK>{}); break;
    case HDET_SEPI_GELUGRAD: if (AK && !BK) finish(std::integral_constant<int, HDET_SEPI_GELUGRAD>{}); break;
  }
}

template <int FORM, int WTM, int WTN, int WM, int WN, int WK, int NST>
__global__ __launch_bounds__(kThreads) void sgemm_lds_kernel(const hdet_sgemm_args g, int epi, unsigned tx, unsigned ty) {
  __shared__ __attribute__((aligned(1024))) float S[stage_floats<WTM, WTN, WM, WN, WK, NST>()];
  sgemm_lds_tile<FORM, WTM, WTN, WM, WN, WK, NST>(g, epi, blockIdx.x, tx, ty, gridDim.x, S);
}
// The two tiles: 64 x 64, and 64 x 32 whose wavefronts share K
#define HDET_SGEMM_LDS(WIDE, CALL) \
  if (WIDE) { CALL(1, 1, 2, 2, 1, 2); } else { CALL(1, 1, 2, 1, 2, 2); }

// Whether an operand is made of whole 16-byte chunks, 16-byte aligned, within the 2 GiB that a descriptor's offsets reach (with a stage's step beyond)
bool chunked(const float* p, bool kmajor, int rows, int k, int64_t ld, const int64_t* bs) {
  const int64_t ext = ((kmajor ? rows : k) + 128) * ld + 256;
  return ((uintptr_t)p & 15) == 0 && (ld & 3) == 0 && ((bs[0] | bs[1] | bs[2]) & 3) == 0 && ((kmajor ? k : rows) & 3) == 0 && ld > 0 && ext < (int64_t)1 << 29;
}
template <int FORM>
bool lds_eligible(const hdet_sgemm_args& g) {
  return chunked(g.a, FORM != kTN, g.m, g.k, FORM != kTN ? g.a_rs : g.a_cs, g.a_s) && chunked(g.b, FORM == kNT, g.n, g.k, FORM == kNT ? g.b_cs : g.b_rs, g.b_s);
}

constexpr int64_t kMaxBlocks = 0xffffff;      // blocks of 256 threads in a grid of less than 2^32 threads
struct tiles { unsigned x, y, total; };
template <int WTM, int WTN, int WM, int WN>
tiles tile_grid(const hdet_sgemm_args& g, int batch) {
  const unsigned x = (g.n + 32 * WTN * WN - 1) / (32 * WTN * WN), y = (g.m + 32 * WTM * WM - 1) / (32 * WTM * WM);
  return {x, y, x * y * (unsigned)batch};
}

// Tile and K split by the number of blocks a launch would have, b(tm x tn) = tiles over the whole batch, on 256 CUs.  Through LDS there are two
// tiles, 64 x 32 where this says so and 64 x 64 for all larger ones; the figures are those of fragments from global memory
// (microseconds over 8 replicas or as given, same machine; chosen | other candidates):
//   few tiles: 32 x 32, K in 4.        128 x 64, K = 64, 4 items: 3.9 | 64 x 32 4.3 | 64 x 64 5.2 (K in 8: 4.3, in 16: 4.1)
//   up to one 64 x 32 block per CU (and at least 5/8 of them), K in 4:
//                                      512 x 256, K = 1024, 4 items: 15.4 | 32 x 32 22.4 | 64 x 64 22.8
//   up to one 64 x 64 block per CU, K in 4:
//                                      256 x 1024, K = 512, 4 items, wgrad: 14.9 | 64 x 32 23.4 | 64 x 128 24.5
//   more: 64 x 128, K in 2             512 x 1024, K = 256, 4 items: 18.0 | 64 x 64 24.6 | 64 x 32 27.2
//   many, an operand contiguous along k: 64 x 64 with two steps in flight instead of four, whose smaller register count lets a
//         CU hold more of them         4096 x 2048, K = 512, 8 items: 798 | 64 x 128 910 (wgrad: 914 | 64 x 128 588)
// The two tiles through LDS, 64 x 64 | 64 x 32, by tiles of 64 x 32 a CU (forward products; weight gradients alike).  K = 256: one 11.8 | 8.0, 1.5
// 12.4 | 12.0, 2.5 16.6 | 14.2, 3 16.9 | 14.9, 4 16.7 | 21.8, 8 31.4 | 32.0, 16 54 | 57, 128 397 | 451;  K = 1024: one 26.4 | 16.8, 1.5 26.8 | 24.2, 2.5
// 39.9 | 32.5, 3 40.3 | 33.2, 4 41.7 | 50.6, 8 92 | 86, 16 162 | 173, 128 1282 | 1320.  So the line at one tile a CU, drawn for fragments from global
// memory, lies too low for these by a factor of three: 3 to 20 % between them.
enum { kCfg32, kCfg64x32, kCfg64, kCfg64x128, kCfg64Light };
int64_t count_blocks(const hdet_sgemm_args& g, int batch, int tm, int tn) {
  return (int64_t)((g.m + tm - 1) / tm) * ((g.n + tn - 1) / tn) * batch;
}
template <typename F>
int choose_cfg(F blocks, bool k_contiguous) {
  const int64_t cus = hdet_compute_units();
  if (blocks(64, 32) * 8 < cus * 5) return kCfg32;
  if (blocks(64, 32) <= cus) return kCfg64x32;
  if (blocks(64, 64) <= cus) return kCfg64;
  if (!k_contiguous || blocks(64, 128) <= 2 * cus) return kCfg64x128;
  return kCfg64Light;
}
#define HDET_SGEMM_SMALL(CALL)                     \
  case kCfg32: CALL(1, 1, 1, 1, 4, 4); break;      \
  case kCfg64x32: CALL(2, 1, 1, 1, 4, 4); break;
#define HDET_SGEMM_LARGE(CALL)                     \
  case kCfg64: CALL(2, 2, 1, 1, 4, 4); break;      \
  case kCfg64x128: CALL(2, 2, 1, 2, 2, 4); break;  \
  case kCfg64Light: CALL(2, 2, 1, 1, 4, 2); break;

// Two products of few blocks and the loss reduction: blocks [0, wt) form the weight gradient, [wt, wt + ot) the other product
// (the one with the longer contraction comes first), the rest reduce a replica's loss each.  Small layers' backward is bound by
// launches and by CUs left idle, and its two products and the bias gradient need nothing of each other.  Each product keeps the
// tile it would have alone.  Only the two small tiles share this kernel: with the larger tiles of fragments from global memory it
// needs 284 registers, a wavefront per SIMD (2-layer d = 256 transformer 962 to 993 us a step with them in pairs, 830 without).
// Larger products share sgemm_lds_pair_kernel where they can go through LDS.
// Per training step: MLP 64-128-10, batch 32, 4 replicas 39 -> 34 us; 2-layer d = 64 transformer 350 -> 261,
// d = 256 890 -> 868 (bias gradients, GELU and residual sums without passes of their own).
struct pair_grid { unsigned wx, wy, wt, ox, oy, ot; int wgrad_first, wcfg, ocfg; };
template <bool NT>
__global__ __launch_bounds__(kThreads) void sgemm_pair_kernel(const hdet_sgemm_args w, const hdet_sgemm_args o, int epi, const pair_grid pg,
                                                             const hdet_loss_args loss) {
  extern __shared__ float part[];
  unsigned t = blockIdx.x;
  if (t >= pg.wt + pg.ot) {
    hdet_reduce_loss(loss.row_loss, loss.rows, loss.ctrl, (int)(t - pg.wt - pg.ot), reinterpret_cast<double*>(part));
    return;
  }
  const unsigned first = pg.wgrad_first ? pg.wt : pg.ot;
  const bool wgrad = (t < first) == (pg.wgrad_first != 0);
  if (t >= first) t -= first;
#define WGRAD(WTM, WTN, WM, WN, WK, U) sgemm_tile<false, false, WTM, WTN, WM, WN, WK, U>(w, HDET_SEPI_NONE, t, pg.wx, pg.wy, pg.wt, part)
#define OTHER(WTM, WTN, WM, WN, WK, U) sgemm_tile<true, NT, WTM, WTN, WM, WN, WK, U>(o, epi, t, pg.ox, pg.oy, pg.ot, part)
  if (wgrad) switch (pg.wcfg) { HDET_SGEMM_SMALL(WGRAD) }
  else switch (pg.ocfg) { HDET_SGEMM_SMALL(OTHER) }
#undef WGRAD
#undef OTHER
}

// The same for two products of many tiles (sgemm_lds_tile): what the launch, the first loads and the last stores take is paid once, and one product's
// blocks work while the other's wait.  wcfg, ocfg: 64 x 64 tiles or 64 x 32.  One after the other / together, us, 4 replicas: 4000 outputs of 256, 512 rows
// 93 / 85;  1024 of 256 27.7 / 25.7;  256 of 1024 through the GELU 35.3 / 30.8;  768 of 256 26.9 / 23.1.
// A product of few tiles beside a larger one: lds_pair_pays.
template <bool NT>
__global__ __launch_bounds__(kThreads) void sgemm_lds_pair_kernel(const hdet_sgemm_args w, const hdet_sgemm_args o, int epi, const pair_grid pg,
                                                                 const hdet_loss_args loss) {
  constexpr int kFloats = std::max(stage_floats<1, 1, 2, 2, 1, 2>(), stage_floats<1, 1, 2, 1, 2, 2>());
  __shared__ __attribute__((aligned(1024))) float S[kFloats];
  unsigned t = blockIdx.x;
  if (t >= pg.wt + pg.ot) {
    hdet_reduce_loss(loss.row_loss, loss.rows, loss.ctrl, (int)(t - pg.wt - pg.ot), reinterpret_cast<double*>(S));
    return;
  }
  const unsigned first = pg.wgrad_first ? pg.wt : pg.ot;
  const bool wgrad = (t < first) == (pg.wgrad_first != 0);
  if (t >= first) t -= first;
#define WGRAD(WTM, WTN, WM, WN, WK, NST) sgemm_lds_tile<kTN, WTM, WTN, WM, WN, WK, NST>(w, HDET_SEPI_NONE, t, pg.wx, pg.wy, pg.wt, S)
#define OTHER(WTM, WTN, WM, WN, WK, NST) sgemm_lds_tile<NT ? kNT : kNN, WTM, WTN, WM, WN, WK, NST>(o, epi, t, pg.ox, pg.oy, pg.ot, S)
  if (wgrad) { HDET_SGEMM_LDS(pg.wcfg, WGRAD) }
  else { HDET_SGEMM_LDS(pg.ocfg, OTHER) }
#undef WGRAD
#undef OTHER
}

template <int FORM>
hipError_t launch_form(const hdet_sgemm_args& g, int epi, int batch, hipStream_t s) {
  const int cfg = choose_cfg([&](int tm, int tn) { return count_blocks(g, batch, tm, tn); }, FORM != kTN);
  if (count_blocks(g, batch, 64, 64) > kMaxBlocks) return hipErrorInvalidValue;
#define CALL(WTM, WTN, WM, WN, WK, U)                                                                                            \
  {                                                                                                                              \
    const tiles t = tile_grid<WTM, WTN, WM, WN>(g, batch);                                                                       \
    hipLaunchKernelGGL((sgemm_kernel<FORM, WTM, WTN, WM, WN, WK, U>), dim3(t.total), dim3(kThreads), 0, s, g, epi, t.x, t.y);    \
  }
  if (cfg >= kCfg64x32 && lds_eligible<FORM>(g)) {
#define LDS(WTM, WTN, WM, WN, WK, NST)                                                                                           \
  {                                                                                                                              \
    const tiles t = tile_grid<WTM, WTN, WM, WN>(g, batch);                                                                       \
    hipLaunchKernelGGL((sgemm_lds_kernel<FORM, WTM, WTN, WM, WN, WK, NST>), dim3(t.total), dim3(kThreads), 0, s, g, epi, t.x, t.y); \
  }
    HDET_SGEMM_LDS(cfg >= kCfg64, LDS)
#undef LDS
    return hipGetLastError();
  }
  switch (cfg) { HDET_SGEMM_SMALL(CALL) HDET_SGEMM_LARGE(CALL) }
#undef CALL
  return hipGetLastError();
}

template <bool NT>
hipError_t launch_pair(const hdet_sgemm_args& w, int wb, int wcfg, const hdet_sgemm_args& o, int epi, int ob, int ocfg,
                       const hdet_loss_args& loss, hipStream_t s) {
  tiles tw = {}, to = {};                                           // ob = 0: no other product, to.total stays 0
  int lds = 64;                                                     // the loss reduction's
#define WGRAD(WTM, WTN, WM, WN, WK, U) { tw = tile_grid<WTM, WTN, WM, WN>(w, wb); lds = std::max(lds, 4 * lds_floats<WTM, WTN, WM, WN, WK>()); }
#define OTHER(WTM, WTN, WM, WN, WK, U) { to = tile_grid<WTM, WTN, WM, WN>(o, ob); lds = std::max(lds, 4 * lds_floats<WTM, WTN, WM, WN, WK>()); }
  switch (wcfg) { HDET_SGEMM_SMALL(WGRAD) }
  if (ob) switch (ocfg) { HDET_SGEMM_SMALL(OTHER) }
#undef WGRAD
#undef OTHER
  const pair_grid pg = {tw.x, tw.y, tw.total, to.x, to.y, to.total, w.k >= o.k, wcfg, ocfg};
  hipLaunchKernelGGL(sgemm_pair_kernel<NT>, dim3(tw.total + to.total + (unsigned)loss.n_replicas), dim3(kThreads), lds, s, w, o, epi, pg, loss);
  return hipGetLastError();
}

// Whether a product of few tiles (32 x 32, K in 4, if alone) goes beside a larger one, which costs it half its blocks and half its K split: a chain of 6.7 ns
// for each of its k, to be hidden by the larger product (at the 100 TFLOP/s of such tiles) and what a launch of its own would add (4 us).  A training
// step in us, apart / together (replicas, rows, layer):  4 512 128 -> 2000 221 / 214;  4 512 128 -> 1000 191 / 188;  8 512 64 -> 2000 219 / 212;  MLPs
// 64-1024-64, 4 256 52 / 46;  32-512-32, 4 512 47 / 42;  level 4 512 128 -> 4000 260 / 260, 4 512 64 -> 2000 178 / 179;
// 4 256 64 -> 4000 167 / 176;  4 512 32 -> 8000 240 / 261;  2 64 64 -> 32000 347 / 466;  MLP 4096-128-4096, 2 128 106 / 116.
bool lds_pair_pays(const hdet_sgemm_args& few, const hdet_sgemm_args& many, int many_batch) {
  return 6.7e-3 * few.k <= 2e-8 * many.m * many.n * (double)many.k * many_batch + 4.0;
}

template <bool NT>
hipError_t launch_lds_pair(const hdet_sgemm_args& w, int wb, bool wwide, const hdet_sgemm_args& o, int epi, int ob, bool owide,
                           const hdet_loss_args& loss, hipStream_t s) {
  const tiles tw = wwide ? tile_grid<1, 1, 2, 2>(w, wb) : tile_grid<1, 1, 2, 1>(w, wb), to = owide ? tile_grid<1, 1, 2, 2>(o, ob) : tile_grid<1, 1, 2, 1>(o, ob);
  const pair_grid pg = {tw.x, tw.y, tw.total, to.x, to.y, to.total, w.k >= o.k, wwide, owide};
  hipLaunchKernelGGL(sgemm_lds_pair_kernel<NT>, dim3(tw.total + to.total + (unsigned)loss.n_replicas), dim3(kThreads), 0, s, w, o, epi, pg, loss);
  return hipGetLastError();
}

hdet_sgemm_args with_batch(const hdet_sgemm_args& g_in) {
  hdet_sgemm_args g = g_in;
  if (g.n1 < 1) g.n1 = 1;
  if (g.n2 < 1) g.n2 = 1;
  return g;
}

}  // namespace

hipError_t hdet_launch_sgemm(const hdet_sgemm_args& g_in, int epi, int batch, hipStream_t s) {
  const hdet_sgemm_args g = with_batch(g_in);
  // which axis of an operand is contiguous (an operand of one row or column may be read either way)
  const bool ak = g.a_cs == 1, bk = g.b_rs == 1 && (ak || g.b_cs != 1);
  if ((!ak && g.a_rs != 1) || (!bk && g.b_cs != 1) || (!ak && bk)) return hipErrorInvalidValue;
  const bool nt = epi == HDET_SEPI_BIAS || epi == HDET_SEPI_BIAS_RELU || epi == HDET_SEPI_BIAS_GELU || epi == HDET_SEPI_BIAS_RESID;
  const bool nn = epi == HDET_SEPI_MASK || epi == HDET_SEPI_GELUGRAD;
  if (!nt && !nn && epi != HDET_SEPI_NONE) return hipErrorInvalidValue;
  if (nn) return ak && g.b_cs == 1 ? launch_form<kNN>(g, epi, batch, s) : hipErrorInvalidValue;
  if (ak && bk) return launch_form<kNT>(g, epi, batch, s);
  if (nt) return hipErrorInvalidValue;
  return ak ? launch_form<kNN>(g, epi, batch, s) : launch_form<kTN>(g, epi, batch, s);
}

hipError_t hdet_launch_sgemm_pair(const hdet_sgemm_args& wgrad, int wgrad_batch, const hdet_sgemm_args* other, bool other_nt, int epi,
                                  int other_batch, const hdet_loss_args* loss, hipStream_t s) {
  const hdet_sgemm_args w = with_batch(wgrad), o = other ? with_batch(*other) : hdet_sgemm_args{};
  const hdet_loss_args l = loss ? *loss : hdet_loss_args{nullptr, 0, nullptr, 0};
  if (w.a_rs != 1 || w.b_cs != 1) return hipErrorInvalidValue;
  if (other && (o.a_cs != 1 || (other_nt ? o.b_rs != 1 : o.b_cs != 1))) return hipErrorInvalidValue;
  const bool fits = epi == HDET_SEPI_NONE || (!other_nt && (epi == HDET_SEPI_MASK || epi == HDET_SEPI_GELUGRAD));
  if (!fits) return hipErrorInvalidValue;
  const int ob = other ? other_batch : 0;
  const int wcfg = choose_cfg([&](int tm, int tn) { return count_blocks(w, wgrad_batch, tm, tn); }, false);
  const int ocfg = ob ? choose_cfg([&](int tm, int tn) { return count_blocks(o, ob, tm, tn); }, true) : kCfg32;
  if (wcfg <= kCfg64x32 && ocfg <= kCfg64x32)
    return other_nt ? launch_pair<true>(w, wgrad_batch, wcfg, o, epi, ob, ocfg, l, s) : launch_pair<false>(w, wgrad_batch, wcfg, o, epi, ob, ocfg, l, s);
  if (ob && lds_eligible<kTN>(w) && (other_nt ? lds_eligible<kNT>(o) : lds_eligible<kNN>(o)) &&
      (wcfg != kCfg32 || lds_pair_pays(w, o, ob)) && (ocfg != kCfg32 || lds_pair_pays(o, w, wgrad_batch)) &&
      count_blocks(w, wgrad_batch, 64, 32) + count_blocks(o, ob, 64, 32) <= kMaxBlocks) {
    const bool ww = wcfg >= kCfg64, ow = ocfg >= kCfg64;
    return other_nt ? launch_lds_pair<true>(w, wgrad_batch, ww, o, epi, ob, ow, l, s) : launch_lds_pair<false>(w, wgrad_batch, ww, o, epi, ob, ow, l, s);
  }
  if (hipError_t e = launch_form<kTN>(w, HDET_SEPI_NONE, wgrad_batch, s)) return e;
  if (ob)
    if (hipError_t e = other_nt ? launch_form<kNT>(o, epi, ob, s) : launch_form<kNN>(o, epi, ob, s)) return e;
  return loss ? hdet_launch_loss_reduce(l.row_loss, l.rows, l.ctrl, l.n_replicas, s) : hipSuccess;
}
