// Replica-batched bf16 GEMM on the gfx950 matrix cores for the "Forward + backward" of
// Algorithm 1 in mixed precision: bf16 operands, fp32 accumulation, N independent weight
// sets with the replica on blockIdx.z.  This file holds the entry point and the general
// kernel, which takes any shape, leading dimension and alignment; products whose operands are
// made of whole, aligned 16-byte chunks are routed to the LDS-direct kernel
// (hdet_gemm_bf16_dma.hip).
//
//   C(m,n) = sum_k A(m,k) * B(k,n)          A, B bfloat16; C fp32 or bfloat16
//
// One kernel serves the three products of a Linear layer; which axis of an operand is
// contiguous in memory differs between them:
//   forward  Y  = X  W^T : A = X [b][k]  (k contiguous)   B(k,n) = W[n][k]  (k contiguous)
//   dgrad    dX = dY W   : A = dY[b][o]  (k=o contiguous) B(k,n) = W[k][n]  (n contiguous)
//   wgrad    dW = dY^T X : A(m,k) = dY[k][m] (m contiguous) B(k,n) = X[k][n] (n contiguous)
// Tiles are staged through LDS with 128-bit coalesced global loads and 128-bit LDS stores in
// the operand's own memory order, and read back as MFMA operands (8 consecutive contraction
// elements per lane):
//   * contraction-contiguous operand: LDS tile [128 rows][32 k], one ds_read_b128 per fragment;
//   * operand contiguous along the output axis: LDS tile [32 k][128 rows], read with the
//     transposing LDS load of gfx950 (ds_read_b64_tr_b16, two per fragment), so that no
//     transposed copy of weights or activations ever exists in HBM.
//
// Tiling: each wavefront owns a 64x64 (or 32x32) output tile (2x2 blocks or one of v_mfma_f32_32x32x16_bf16);
// a block is 2x2 wavefronts (128x128 or 64x64 tile).  K step 32, LDS double-buffered (one barrier per K
// step), the global loads of the next four steps (of the next one in grids of many blocks: one_step) in flight in registers; launch
// indices are remapped so that each XCD's L2 serves a contiguous range of tiles.  What bounds it is the latency of those loads: with one
// step in flight, and the funnel shift waiting for its data at once, 0.9 us a step of a block that is alone.  96 x 1500, K = 700 gradient, 6 items 20.1 -> 15.9 us, 1500 x 784, K = 576
// 13.4 -> 10.6, odd rows 96 x 1501, K = 703, 4 items 23.0 -> 14.1.
//
// Loads of operands that are not made of aligned chunks: memory is read in aligned dwords (16 bytes per
// lane; global loads need no more than dword alignment) and, where a chunk starts at an odd element, one
// dword more and a funnel shift by 16 bits.  Rows beyond the matrix read its last row or first chunk again
// (their results are not stored), so that only the last K step looks at the extent of anything.
//
// Measured against predicated 2-byte loads of such chunks: 96 x 700, K = 1500 (rows of 1500 elements, 6 replicas, 128 x 128
// tiles) 282 -> 28.6 us, 700 x 1500, K = 576 77 -> 14.8 us; 256 x 4095, K = 4095, 8 replicas: 337 us (204 TFLOP/s).
//
// Products with few output tiles take a second kernel (hdet_bgemm_frag_kernel below).

#include <type_traits>

#include "hdet_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));

constexpr int TK = 32;
constexpr int LDK = TK;          // pitch of a [row][k] tile: 64 B, no padding; the four 16-byte chunks of a
                                 // row are stored XOR-swizzled by (row / 4) % 4, which makes both the
                                 // staging stores (4 rows x 4 chunks per 16 lanes) and the fragment
                                 // loads (16 rows x 1 chunk per 16 lanes) free of bank conflicts
// pitch of a [k][row] tile of ROWS rows: ROWS + 32 elements, i.e. 16 banks past a multiple of 64, so
// the 4 k-rows that a 16-lane group of a transposing read touches fall on disjoint banks
__host__ __device__ constexpr int ldr(int rows) { return rows + 32; }
__host__ __device__ constexpr int tile_elems(int rows) { return TK * ldr(rows); }   // >= rows * LDK

__device__ __forceinline__ unsigned short f2bf(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x0040u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

typedef unsigned int u4a __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// 8 consecutive elements starting at src[idx], all of them readable.  src is 2-byte aligned; `odd_possible` (uniform) says
// whether &src[idx] may be no multiple of 4 bytes.  The fifth dword of an odd chunk holds its last element, that of an even one
// is its fourth again: nothing beyond the dword of the last element is touched.
__device__ __forceinline__ us8 load8_any(const uint16_t* src, int64_t idx, bool odd_possible) {
  const uint16_t* q = src + idx;
  if (!odd_possible) return __builtin_bit_cast(us8, (u4)*reinterpret_cast<const u4a*>(q));
  const unsigned odd = ((unsigned)(uintptr_t)q >> 1) & 1u;
  const unsigned int* p = reinterpret_cast<const unsigned int*>(q - odd);
  const u4a d = *reinterpret_cast<const u4a*>(p);
  const unsigned e = p[3 + odd], sh = odd << 4;
  const u4 r = {__builtin_amdgcn_alignbit(d[1], d[0], sh), __builtin_amdgcn_alignbit(d[2], d[1], sh), __builtin_amdgcn_alignbit(d[3], d[2], sh),
                __builtin_amdgcn_alignbit(e, d[3], sh)};
  return __builtin_bit_cast(us8, r);
}
// ... of which the first `valid` count (others 0), in an operand of `extent` elements
__device__ __forceinline__ us8 load8(const uint16_t* src, int64_t idx, int valid, int64_t extent, bool odd_possible) {
  us8 r = {0, 0, 0, 0, 0, 0, 0, 0};
  if (valid <= 0) return r;
  if (idx + 8 <= extent) {
    r = load8_any(src, idx, odd_possible);
#pragma unroll
    for (int j = 1; j < 8; ++j)
      if (j >= valid) r[j] = 0;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < valid) r[j] = src[idx + j];
  }
  return r;
}

// One operand tile: ROWS (64 or 128) rows of the output dimension x 32 of the contraction.
// KMAJOR: element (row, k) at src[row * ld + k], LDS tile[row][k];
// otherwise at src[k * ld + row], LDS tile[k][row].
template <bool KMAJOR, int ROWS, int THREADS>
struct operand {
  static constexpr int NCH = ROWS * 4 / THREADS;   // 8-element chunks per thread and K step
  static constexpr int RCH = ROWS / 8;         // chunks per k-row of a [k][row] tile
  us8 reg[NCH];
  // K step that lies inside the matrix and is not its last one: rows beyond `rows` repeat others
  __device__ __forceinline__ void fetch(const uint16_t* src, int64_t ld, int row0, int rows, int k0, bool odd, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * THREADS;
      if (KMAJOR) {
        const int row = row0 + (c >> 2);
        reg[i] = load8_any(src, (int64_t)(row < rows ? row : rows - 1) * ld + k0 + ((c & 3) << 3), odd);
      } else {
        const int row = row0 + ((c % RCH) << 3);
        reg[i] = load8_any(src, (int64_t)(k0 + c / RCH) * ld + (row < rows ? row : row0), odd);
      }
    }
  }
  // last K step: zeros beyond the contraction, nothing beyond the operand's extent is read
  __device__ __forceinline__ void fetch_last(const uint16_t* src, int64_t ld, int row0, int rows, int k0, int kdim, bool odd, int tid) {
    const int64_t extent = (int64_t)((KMAJOR ? rows : kdim) - 1) * ld + (KMAJOR ? kdim : rows);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * THREADS;
      if (KMAJOR) {
        const int row = row0 + (c >> 2), k = k0 + ((c & 3) << 3);
        reg[i] = load8(src, (int64_t)row * ld + k, row < rows ? kdim - k : 0, extent, odd);
      } else {
        const int k = k0 + c / RCH, row = row0 + ((c % RCH) << 3);
        reg[i] = load8(src, (int64_t)k * ld + row, k < kdim ? rows - row : 0, extent, odd);
      }
    }
  }
  __device__ __forceinline__ void commit(uint16_t* tile, int tid) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * THREADS;
      const us8 v = reg[i];
      if (KMAJOR) *reinterpret_cast<us8*>(tile + (c >> 2) * LDK + ((((c & 3) ^ (c >> 4)) & 3) << 3)) = v;
      else *reinterpret_cast<us8*>(tile + (c / RCH) * ldr(ROWS) + ((c % RCH) << 3)) = v;
    }
  }
  // MFMA 32x32x16 operand fragment: lane l gets (row = r0 + l % 32, k = ks + 8 * (l / 32) + 0..7).
  static __device__ __forceinline__ bf16x8 fragment(const uint16_t* tile, int r0, int ks, int lane) {
    if (KMAJOR) {
      const int row = r0 + (lane & 31);
      const int chunk = ((ks >> 3) + (lane >> 5)) ^ ((row >> 2) & 3);
      return *reinterpret_cast<const bf16x8*>(tile + row * LDK + (chunk << 3));
    }
    // Transposing read: within a 16-lane group, lane p points at the 4 elements
    // (k = kb + p / 4, rows rb + 4 * (p % 4) .. + 3) and lane i receives (k = kb .. kb + 3, row rb + i).
    const int p = lane & 15;
    const int rb = r0 + (((lane >> 4) & 1) << 4);
    const int kb = ks + ((lane >> 5) << 3);
    const uint16_t* q = tile + (kb + (p >> 2)) * ldr(ROWS) + rb + ((p & 3) << 2);
    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(q));
    const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(q + 4 * ldr(ROWS)));
    const s8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, both);
  }
};

// The chunks of an operand that one thread loads, in K steps that lie inside the matrix and are not its last one: rows beyond `rows`
// repeat others.  ODD: some chunk may start at an odd element; then a fifth dword is loaded, and the funnel shift waits until the chunk
// goes to LDS.
template <bool KMAJOR, int ROWS, int THREADS, bool ODD>
struct chunk_stream {
  typedef operand<KMAJOR, ROWS, THREADS> op;
  static constexpr int NCH = op::NCH;
  const char* p[NCH];           // dword at or before the chunk of K step 0
  unsigned odd[NCH];            // the same in every K step: TK is even
  int64_t step;                 // bytes between K steps
  struct stage { u4 d[NCH]; unsigned e[ODD ? NCH : 1]; };
  __device__ __forceinline__ void init(const uint16_t* src, int64_t ld, int row0, int rows, int tid) {
    step = (KMAJOR ? TK : TK * ld) * 2;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * THREADS;
      int64_t at;
      if (KMAJOR) {
        const int row = row0 + (c >> 2);
        at = (int64_t)(row < rows ? row : rows - 1) * ld + ((c & 3) << 3);
      } else {
        const int row = row0 + ((c % op::RCH) << 3);
        at = (int64_t)(c / op::RCH) * ld + (row < rows ? row : row0);
      }
      odd[i] = ODD ? ((unsigned)(uintptr_t)(src + at) >> 1) & 1u : 0u;
      p[i] = reinterpret_cast<const char*>(src + at - odd[i]);
    }
  }
  __device__ __forceinline__ void request(stage& x, int kt) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const unsigned int* q = reinterpret_cast<const unsigned int*>(p[i] + kt * step);
      x.d[i] = *reinterpret_cast<const u4a*>(q);
      if (ODD) x.e[ODD ? i : 0] = q[3 + odd[i]];
    }
  }
  __device__ __forceinline__ void commit(const stage& x, uint16_t* tile, int tid) const {
    op o;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      u4 r = x.d[i];
      if (ODD) {
        const unsigned sh = odd[i] << 4, e = x.e[ODD ? i : 0];
        r = u4{__builtin_amdgcn_alignbit(r[1], r[0], sh), __builtin_amdgcn_alignbit(r[2], r[1], sh), __builtin_amdgcn_alignbit(r[3], r[2], sh),
               __builtin_amdgcn_alignbit(e, r[3], sh)};
      }
      o.reg[i] = __builtin_bit_cast(us8, r);
    }
    o.commit(tile, tid);
  }
};

// one element of C with the epilogue EPI
template <int EPI>
__device__ __forceinline__ void put_element(const hdet_bgemm_args& g, int z, int64_t c_base, int row, int col, float v) {
  if (row >= g.m || col >= g.n) return;
  const int64_t off = c_base + (int64_t)row * g.ldc + col;
  if (EPI == HDET_EPI_BIAS_RELU_BF16 || EPI == HDET_EPI_BIAS_F32 || EPI == HDET_EPI_BIAS_BF16) v += g.bias[(int64_t)z * g.bias_bs + col];
  if (EPI == HDET_EPI_F32 || EPI == HDET_EPI_BIAS_F32) {
    reinterpret_cast<float*>(g.c)[off] = v;
    return;
  }
  if (EPI == HDET_EPI_BIAS_RELU_BF16) v = v > 0.f ? v : 0.f;
  if (EPI == HDET_EPI_MASK_BF16)         // gradient through the ReLU of the layer below
    v = bf2f(g.mask[(int64_t)z * g.mask_bs + (int64_t)row * g.mask_ld + col]) > 0.f ? v : 0.f;
  reinterpret_cast<uint16_t*>(g.c)[off] = f2bf(v);
}

}  // namespace

// Row sums of A beside a weight gradient (the bias gradient: A(o, b) = dZ[b][o]): one more MFMA per fragment, against a B of
// ones, in the wavefronts of the first tile column.  Measured against a launch of its own that reads dZ again (1500, 700 and
// 100 columns of 576 rows: 12.3, 11.8 and 10.5 us): free.
template <bool A_KMAJOR, bool B_KMAJOR, int EPI> constexpr bool has_rowsum() { return !A_KMAJOR && !B_KMAJOR && EPI == HDET_EPI_F32; }
__device__ __forceinline__ bf16x8 ones() {
  const us8 o = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  return __builtin_bit_cast(bf16x8, o);
}

// WT x WT: 32x32 MFMA blocks per wavefront; 2 x 2 wavefronts per block, block tile (64 WT) x (64 WT).
// DEPTH: K steps whose loads are in flight, 4 or 1 (one_step says when).  PIECES: the contraction is summed in that many pieces, each from
// zero, and the pieces are added in ascending order (launch_general).
template <bool A_KMAJOR, bool B_KMAJOR, int EPI, int WT, int DEPTH, int PIECES = 1>
__global__ __launch_bounds__(256, 2) void hdet_bgemm_kernel(const hdet_bgemm_args g) {
  constexpr int TM = 64 * WT, TN = TM, THREADS = 256;
  __shared__ __attribute__((aligned(16))) uint16_t As[2][tile_elems(TM)];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][tile_elems(TN)];
  // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2) in launch order.
  // Remap the launch index so that an XCD works on a contiguous range of tiles: the tiles that
  // share an A row-panel or a weight panel then meet in one L2 instead of eight.
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  {
    const unsigned total = gridDim.x * gridDim.y * gridDim.z;
    if ((total & 7u) == 0u) {
      const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
      const unsigned t = (lin & 7u) * (total >> 3) + (lin >> 3);
      bx = t % gridDim.x;
      by = (t / gridDim.x) % gridDim.y;
      bz = t / (gridDim.x * gridDim.y);
    }
  }
  const hdet_batch_index bi = hdet_split_batch(bz, g.n1, g.n2);
  const int z = bi.z0;            // replica: bias and mask are per replica
  const uint16_t* A = g.a + hdet_batch_offset(bi, g.a_s);
  const uint16_t* B = g.b + hdet_batch_offset(bi, g.b_s);
  const int64_t c_base = hdet_batch_offset(bi, g.c_s);
  const int m0 = by * TM, n0 = bx * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * (32 * WT), wn = (wave & 1) * (32 * WT);
  const bool a_odd = (g.lda & 1) != 0 || (reinterpret_cast<uintptr_t>(A) & 3) != 0;
  const bool b_odd = (g.ldb & 1) != 0 || (reinterpret_cast<uintptr_t>(B) & 3) != 0;

  f16v acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  constexpr bool SUMS = has_rowsum<A_KMAJOR, B_KMAJOR, EPI>();
  const bool sums = SUMS && g.rowsum && bx == 0 && wn == 0;         // uniform over the wavefront
  f16v rsum[SUMS ? WT : 1];
#pragma unroll
  for (int i = 0; i < (SUMS ? WT : 1); ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) rsum[i][e] = 0.f;

  typedef operand<A_KMAJOR, TM, THREADS> ta;
  typedef operand<B_KMAJOR, TN, THREADS> tb;
  const int nk = (g.k + TK - 1) / TK;
  // steps of 16 k a piece and left of this one; the last piece takes what is left over
  const int per_piece = ((g.k >> 4) + PIECES - 1) / PIECES;
  int left = per_piece, pieces_left = PIECES - 1;
  f16v tot[PIECES > 1 ? WT : 1][PIECES > 1 ? WT : 1], rtot[PIECES > 1 && SUMS ? WT : 1];
  auto close_piece = [&] {
    if constexpr (PIECES > 1) {
      const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < WT; ++i) {
#pragma unroll
        for (int j = 0; j < WT; ++j) { tot[i][j] += acc[i][j]; acc[i][j] = zero; }
        if constexpr (SUMS) { rtot[i] += rsum[i]; rsum[i] = zero; }
      }
    }
  };
  if constexpr (PIECES > 1) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
#pragma unroll
      for (int i = 0; i < WT; ++i) {
#pragma unroll
        for (int j = 0; j < WT; ++j) tot[i][j][e] = 0.f;
        if constexpr (SUMS) rtot[i][e] = 0.f;
      }
  }
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < TK; ks += 16) {
      if constexpr (PIECES > 1) {
        if (left == 0 && pieces_left > 0) {            // uniform
          close_piece();
          left = per_piece;
          --pieces_left;
        }
        --left;
      }
      bf16x8 af[WT], bfr[WT];
#pragma unroll
      for (int i = 0; i < WT; ++i) af[i] = ta::fragment(As[buf], wm + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < WT; ++j) bfr[j] = tb::fragment(Bs[buf], wn + j * 32, ks, lane);
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      if (SUMS && sums) {
#pragma unroll
        for (int i = 0; i < WT; ++i) rsum[SUMS ? i : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], ones(), rsum[SUMS ? i : 0], 0, 0, 0);
      }
    }
  };
  // a chunk at the end of a k-row reads on into the next one, which has to be long enough for that
  const bool roomy = (A_KMAJOR || g.lda >= 8) && (B_KMAJOR || g.ldb >= 8);
  if constexpr (DEPTH == 1) {
    // the loads of the next K step are in flight during the MFMAs of this one; other blocks on the CU cover the rest of their latency
    ta oa;
    tb ob;
    auto request = [&](int kt) {
      if (kt + 1 < nk && roomy) {
        oa.fetch(A, g.lda, m0, g.m, kt * TK, a_odd, tid);
        ob.fetch(B, g.ldb, n0, g.n, kt * TK, b_odd, tid);
      } else {
        oa.fetch_last(A, g.lda, m0, g.m, kt * TK, g.k, a_odd, tid);
        ob.fetch_last(B, g.ldb, n0, g.n, kt * TK, g.k, b_odd, tid);
      }
    };
    auto commit = [&](int buf) {
      oa.commit(As[buf], tid);
      ob.commit(Bs[buf], tid);
    };
    request(0);
    commit(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      if (kt + 1 < nk) request(kt + 1);
      __builtin_amdgcn_sched_barrier(0);     // keep the loads ahead of the MFMAs ...
      multiply(kt & 1);
      __builtin_amdgcn_sched_barrier(0);     // ... and every use of the loaded data behind them
      commit((kt & 1) ^ 1);                  // last read before the previous barrier
      __syncthreads();
    }
  } else {
    // The last K step, which alone looks at the extent of anything, is requested first and stays in registers until its turn.
    ta la;
    tb lb;
    la.fetch_last(A, g.lda, m0, g.m, (nk - 1) * TK, g.k, a_odd, tid);
    lb.fetch_last(B, g.ldb, n0, g.n, (nk - 1) * TK, g.k, b_odd, tid);
    // DEPTH register stages: the loads of a K step are requested DEPTH steps before it is written to LDS, one step before its
    // MFMAs; two LDS buffers, one barrier a step.
    auto pipelined = [&](auto odd_) {
      constexpr bool ODD = decltype(odd_)::value;
      const int nf = nk - 1;
      chunk_stream<A_KMAJOR, TM, THREADS, ODD> ca;
      chunk_stream<B_KMAJOR, TN, THREADS, ODD> cb;
      ca.init(A, g.lda, m0, g.m, tid);
      cb.init(B, g.ldb, n0, g.n, tid);
      typename decltype(ca)::stage ra[DEPTH];
      typename decltype(cb)::stage rb[DEPTH];
      auto request = [&](int s, int kt) {            // past the end: the last whole step again, not used
        const int k = kt < nf ? kt : nf - 1;
        ca.request(ra[s], k);
        cb.request(rb[s], k);
      };
      auto commit = [&](int s) {
        ca.commit(ra[s], As[s & 1], tid);
        cb.commit(rb[s], Bs[s & 1], tid);
      };
      auto commit_last = [&](int s) {
        la.commit(As[s & 1], tid);
        lb.commit(Bs[s & 1], tid);
      };
      if (nf > 0) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) request(s, s);
        commit(0);
        request(0, DEPTH);
      } else {
        commit_last(0);
      }
      __syncthreads();
      int kt0 = 0;
      for (; kt0 + DEPTH < nf; kt0 += DEPTH) {        // no branch inside: it would have the compiler wait for every load
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
          multiply(s & 1);
          commit((s + 1) % DEPTH);                    // last read before the previous barrier
          request((s + 1) % DEPTH, kt0 + s + 1 + DEPTH);
          __syncthreads();
        }
      }
#pragma unroll
      for (int s = 0; s < DEPTH; ++s) {
        if (kt0 + s >= nf) break;
        multiply(s & 1);
        if (kt0 + s + 1 < nf) commit((s + 1) % DEPTH);
        else commit_last((s + 1) % DEPTH);
        __syncthreads();
      }
      multiply(nf & 1);
    };
    if (roomy) {
      if (a_odd || b_odd) pipelined(std::true_type{});
      else pipelined(std::false_type{});
    } else {
      for (int kt = 0; kt < nk; ++kt) {
        ta xa;
        tb xb;
        xa.fetch_last(A, g.lda, m0, g.m, kt * TK, g.k, a_odd, tid);
        xb.fetch_last(B, g.ldb, n0, g.n, kt * TK, g.k, b_odd, tid);
        if (kt) __syncthreads();
        xa.commit(As[0], tid);
        xb.commit(Bs[0], tid);
        __syncthreads();
        multiply(0);
      }
    }
  }

  if constexpr (PIECES > 1) {
    close_piece();
#pragma unroll
    for (int i = 0; i < WT; ++i) {
#pragma unroll
      for (int j = 0; j < WT; ++j) acc[i][j] = tot[i][j];
      if constexpr (SUMS) rsum[i] = rtot[i];
    }
  }
  // epilogue: accumulator element e of lane l is C(row, col) with
  //   row = (e / 4) * 8 + (l / 32) * 4 + e % 4,  col = l % 32   inside its 32x32 block
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        put_element<EPI>(g, z, c_base, m0 + wm + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), n0 + wn + j * 32 + (lane & 31), acc[i][j][e]);
  if (SUMS && sums && (lane & 31) == 0) {                           // every column holds the sum
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + wm + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        if (row < g.m) g.rowsum[(int64_t)z * g.rowsum_bs + row] = rsum[SUMS ? i : 0][e];
      }
  }
}

// Products with few output tiles: what counts there is the length of a block's K loop and the wavefronts in flight, as for
// the fp32 products (hdet_gemm_f32.hip), and the kernel is built the same way.  A wavefront loads the fragments of the block's
// 32 x 32 tile straight from global memory, four steps of 16 k ahead, without LDS and without a barrier; WK wavefronts
// share the contraction and add their partial tiles through LDS in ascending order of k.  An operand contiguous along k is one
// 16-byte load per lane and fragment (with the funnel shift where chunks start at odd elements); one contiguous along its
// output axis is eight 2-byte loads, 32 consecutive elements at a time, so that no alignment is needed at all.
template <bool KMAJOR>
__device__ __forceinline__ us8 frag_load(const uint16_t* src, int64_t lane_off, int64_t ld, bool odd) {
  if (KMAJOR) return load8_any(src, lane_off, odd);
  us8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (src + j * ld)[lane_off];
  return r;
}
template <bool KMAJOR>
__device__ __forceinline__ us8 frag_load_tail(const uint16_t* src, int64_t lane_off, int64_t ld, int valid) {
  us8 r = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j < valid) r[j] = KMAJOR ? src[lane_off + j] : (src + j * ld)[lane_off];
  return r;
}

template <bool A_KMAJOR, bool B_KMAJOR, int EPI, int WK>
__global__ __launch_bounds__(64 * WK) void hdet_bgemm_frag_kernel(const hdet_bgemm_args g) {
  constexpr int U = 4;                                              // steps in flight
  static_assert(WK > 1 && 16 % WK == 0, "the wavefronts of a K split share the tile's 16 registers evenly");
  __shared__ float part[WK * 16 * 64];
  unsigned bx, by, bz;
  {   // launch order -> tile: XCD x (launch index mod 8) takes the x-th of eight contiguous ranges of tiles
    const unsigned total = gridDim.x * gridDim.y * gridDim.z;
    unsigned t = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned x = t & 7u, rem = total & 7u;
    t = x * (total >> 3) + (x < rem ? x : rem) + (t >> 3);
    bx = t % gridDim.x;
    by = (t / gridDim.x) % gridDim.y;
    bz = t / (gridDim.x * gridDim.y);
  }
  const hdet_batch_index bi = hdet_split_batch(bz, g.n1, g.n2);
  const int z = bi.z0;
  const uint16_t* A = g.a + hdet_batch_offset(bi, g.a_s);
  const uint16_t* B = g.b + hdet_batch_offset(bi, g.b_s);
  const int64_t c_base = hdet_batch_offset(bi, g.c_s);
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = by * 32, n0 = bx * 32;
  const bool a_odd = (g.lda & 1) != 0 || (reinterpret_cast<uintptr_t>(A) & 3) != 0;
  const bool b_odd = (g.ldb & 1) != 0 || (reinterpret_cast<uintptr_t>(B) & 3) != 0;

  constexpr bool SUMS = has_rowsum<A_KMAJOR, B_KMAJOR, EPI>();
  const bool sums = SUMS && g.rowsum && bx == 0;                    // uniform over the block
  f16v acc, rsum;
#pragma unroll
  for (int e = 0; e < 16; ++e) { acc[e] = 0.f; rsum[e] = 0.f; }

  // lane l: row r0 + l % 32 (the matrix's last row again beyond it), k = 8 (l / 32) + 0..7
  const int arow = m0 + (lane & 31) < g.m ? m0 + (lane & 31) : g.m - 1, brow = n0 + (lane & 31) < g.n ? n0 + (lane & 31) : g.n - 1;
  const int64_t aoff = A_KMAJOR ? arow * g.lda + half * 8 : half * 8 * g.lda + arow;
  const int64_t boff = B_KMAJOR ? brow * g.ldb + half * 8 : half * 8 * g.ldb + brow;
  const int64_t astep = A_KMAJOR ? 16 : 16 * g.lda, bstep = B_KMAJOR ? 16 : 16 * g.ldb;
  const int nfull = g.k >> 4, per = (nfull + WK - 1) / WK;
  const int c0 = wk * per < nfull ? wk * per : nfull, c1 = c0 + per < nfull ? c0 + per : nfull;

  us8 a[2][U], b[2][U];
  auto fetch = [&](int buf, int c) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = c + u < c1 ? c + u : c1 - 1;                   // past the end: the last step again, not used
      a[buf][u] = frag_load<A_KMAJOR>(A + cc * astep, aoff, g.lda, a_odd);
      b[buf][u] = frag_load<B_KMAJOR>(B + cc * bstep, boff, g.ldb, b_odd);
    }
  };
  auto step = [&](us8 av, us8 bv) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), acc, 0, 0, 0);
    if (SUMS && sums) rsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), ones(), rsum, 0, 0, 0);
  };
  if (c0 < c1) {
    fetch(0, c0);
    for (int c = c0; c < c1; c += 2 * U) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int cur = c + h * U;
        if (cur < c1) {
          if (cur + U < c1) fetch(h ^ 1, cur + U);
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u == 0 || cur + u < c1) step(a[h][u], b[h][u]);
        }
      }
    }
  }
  const int kleft = g.k & 15;
  if (kleft && wk == WK - 1)
    step(frag_load_tail<A_KMAJOR>(A + nfull * astep, aoff, g.lda, kleft - half * 8), frag_load_tail<B_KMAJOR>(B + nfull * bstep, boff, g.ldb, kleft - half * 8));

  float* mine = part + wk * (16 * 64) + lane;                       // [register][lane] of this wavefront's partial tile
#pragma unroll
  for (int e = 0; e < 16; ++e) mine[e * 64] = acc[e];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 16 / WK; ++t) {
    const int e = wk * (16 / WK) + t;
    float v = part[e * 64 + lane];
#pragma unroll
    for (int p = 1; p < WK; ++p) v += part[(p * 16 + e) * 64 + lane];
    put_element<EPI>(g, z, c_base, m0 + (e >> 2) * 8 + half * 4 + (e & 3), n0 + (lane & 31), v);
  }
  if (SUMS && sums) {
    __syncthreads();                                                // the tile's partial sums have been read
    if ((lane & 31) == 0) {                                         // every column holds the sum: [K part][row]
#pragma unroll
      for (int e = 0; e < 16; ++e) part[wk * 32 + (e >> 2) * 8 + half * 4 + (e & 3)] = rsum[e];
    }
    __syncthreads();
    const int r = threadIdx.x;
    if (r < 32) {
      float v = part[r];
#pragma unroll
      for (int p = 1; p < WK; ++p) v += part[p * 32 + r];
      if (m0 + r < g.m) g.rowsum[(int64_t)z * g.rowsum_bs + m0 + r] = v;
    }
  }
}

namespace {

// blocks of tm x tn a product would have over its batch
int64_t tiles(const hdet_bgemm_args& g, int batch, int tm, int tn) {
  return (int64_t)((g.m + tm - 1) / tm) * ((g.n + tn - 1) / tn) * batch;
}
// A product that leaves most of the chip idle in 64 x 64 tiles takes the fragment kernel with 32 x 32 tiles and K in 4, whatever its K.
// (K in 8 is 5 to 30 % faster from K = 512 on -- 96 x 703, K = 1501, 4 items 22.4 / 25.4 us, 100 x 300, K = 3001, 3 items 27.2 / 40.9 -- and not
// kept: sums in another order put stored activations on the other side of a rounding boundary, and units behind a ReLU on the other side of
// zero, which moves single entries of a small batch's gradients by more than their tensor's root mean square.)
bool few_tiles(const hdet_bgemm_args& g, int batch) { return tiles(g, batch, 64, 64) * 5 < 2 * (int64_t)hdet_compute_units(); }

// Whether the LDS kernel keeps one K step in flight instead of four, which need half again as many registers (4 blocks a CU in 64 x 64 tiles instead
// of 6, 2 instead of 3 in 128 x 128) and begin a block later.  By who else is there to cover the latency of the loads; chunks at odd elements, whose
// funnel shift would wait at once, have more of it.  (4 to 6 tiles a CU, 4 to 5 of even weight gradients, are one round of the one and two of the
// other.)  us, one / four in flight, items of one step:
//   128 x 128, rows of A: even 2184 x 2122, K = 830, 5 items 115 / 133;  3460 x 2682, K = 3238, 6 items 742 / 832;  7600 x 1280 gradient, K = 16,
//     5 items 104 / 140;  odd 3460 x 3238, K = 137, 6 items 138 / 177;  9326 x 570, K = 309, 6 items 116 / 132;  1508 x 2164, K = 1537, 6 items 235 / 210
//   128 x 128 weight gradients, even 2880 x 2468, K = 1661, 8 items 387 / 288, odd 2723 x 1277, K = 1599, 6 items 288 / 136
//   64 x 64 (tiles a CU): 623 x 350, K = 3320, 8 items (1.9) 84 / 56;  351 x 3124, K = 404, 5 items (5.7) 32.7 / 35.7;  1274 x 1949 gradient, K = 896,
//     odd, 2 items (4.8) 35 / 43;  3034 x 324, K = 1220, 6 items (6.8) 74 / 56;  2056 x 1540 gradient, K = 28, 4 items (12.9) 30 / 36;  weight
//     gradients, even 404 x 2152, K = 351, 5 items (4.6) 17.2 / 20.4, 1280 x 1812, K = 7600, 5 items (11.3) 532 / 778, odd 1277 x 650, K = 1599,
//     6 items (5.2) 90 / 62, 856 x 3437, K = 71, 4 items (11.8) 18.5 / 20.1;  even, 900 x 1284, K = 6000, 4 items (4.9) 160 / 263, 1028 x 1028,
//     K = 2600, 5 items (5.6) 109 / 108, 2872 x 196, K = 9657, 8 items (5.6) 517 / 356, 2100 x 452, K = 4000, 6 items (6.2) 205 / 149
// Of 467 products of 122 random networks none but 20 lose more than 6 % by this rule, most of them in 64 x 64 tiles at 9 a CU and more with K from 1800 on
// (666 x 2025, K = 6626, 8 items 550 / 666), where as many others gain as much.
bool one_step(const hdet_bgemm_args& g, bool wgrad, int wt, int64_t blocks) {
  const int64_t cus = hdet_compute_units();
  const bool odd = ((g.lda | g.ldb | g.a_s[0] | g.a_s[1] | g.a_s[2] | g.b_s[0] | g.b_s[1] | g.b_s[2]) & 1) != 0 ||
                   ((reinterpret_cast<uintptr_t>(g.a) | reinterpret_cast<uintptr_t>(g.b)) & 3) != 0;
  if (wt == 2) return !odd || g.k < 768;             // (weight gradients never: launch_general)
  if (blocks <= 3 * cus) return false;
  if (g.k < 256) return true;
  if (!wgrad) return blocks > 4 * cus && blocks <= 6 * cus;
  return !odd && (blocks <= 5 * cus || blocks > 7 * cus);
}

// `aligned`: the LDS-direct kernel could form the product as well, whose sums are not split.
template <bool AK, bool BK, int EPI>
hipError_t launch_general(const hdet_bgemm_args& g, int batch, bool aligned, hipStream_t s) {
#define HDET_LDS(WT, ...)                                                                             \
  hipLaunchKernelGGL((hdet_bgemm_kernel<AK, BK, EPI, WT, __VA_ARGS__>), dim3((g.n + 64 * WT - 1) / (64 * WT), (g.m + 64 * WT - 1) / (64 * WT), batch), dim3(256), 0, s, g)
  const int64_t cus = hdet_compute_units();
  if (few_tiles(g, batch)) hipLaunchKernelGGL((hdet_bgemm_frag_kernel<AK, BK, EPI, 4>), dim3((g.n + 31) / 32, (g.m + 31) / 32, batch), dim3(256), 0, s, g);
  // less than one 64 x 64 block per CU and a long contraction: the sums of K in 8, by one block that walks the eighths one after the
  // other.  (Eight wavefronts of the fragment kernel, an eighth each, give the same bits.  us, so / in this kernel: 96 x 700, K = 1500,
  // 6 items 24.4 / 19.7;  97 x 2111, K = 1501, 3 items 58.7 / 23.3;  64 x 1500, K = 2047, 5 items 46.7 / 35.6;  130 x 1001, K = 4095, 4 items
  // 119 / 45.8;  96 x 1500, K = 1500 gradient, 4 items 32.9 / 19.2.  Summed in one piece 18.9, 25.7, 39.6, 52.7, 16.7: see few_tiles.)
  else if (!aligned && g.k >= 1024 && tiles(g, batch, 64, 64) < cus) HDET_LDS(1, 4, 8);
  // 128 x 128 tiles once there are several rounds of them (256 x 4095, K = 4095, 8 items: 337 | 64 x 64 441; 700 x 1500, K = 576:
  // 14.8 | 10.1; 1788 x 3193, K = 222: 18.4 | 14.7), unless they would be half empty
  else if (tiles(g, batch, 128, 128) >= 4 * cus && g.m > 64 && g.n > 64) {
    if constexpr (AK) {
      if (one_step(g, false, 2, tiles(g, batch, 128, 128))) HDET_LDS(2, 1);
      else HDET_LDS(2, 4);
    } else {
      HDET_LDS(2, 4);
    }
  } else {
    if (one_step(g, !AK, 1, tiles(g, batch, 64, 64))) HDET_LDS(1, 1);
    else HDET_LDS(1, 4);
  }
#undef HDET_LDS
  return hipGetLastError();
}

}  // namespace

hipError_t hdet_launch_bgemm(const hdet_bgemm_args& g_in, bool a_kmajor, bool b_kmajor, int epi, int batch,
                             hipStream_t s) {
  hdet_bgemm_args g = g_in;
  if (g.n1 < 1) g.n1 = 1;
  if (g.n2 < 1) g.n2 = 1;
  // The LDS-direct kernel where the operands allow it, except for products of few tiles in the epilogues that the general kernels
  // have.  Weight gradients stay: the update that the LDS-direct kernel can apply to them (HDET_EPI_ADAMW) has to see the same sums.
  const bool plain = epi <= HDET_EPI_BIAS_BF16 && !g.colsum && a_kmajor;
  // Forward products of up to two 64 x 64 tiles a CU, of one row or column of tiles up to one: their time is the chain of one block, and four times
  // the blocks of 128 x 128 count for more than loads that pass the registers by.  us, this file's kernel / LDS-direct, operands cold:
  // 200 x 1000, K = 3000, 2 items 23.5 / 42.7;  96 x 704, K = 1504, 6 items 16.8 / 25.4;  96 x 1504, K = 784 16.0 / 19.0;  128 x 1024, K = 1024,
  // 8 items 16.4 / 19.5;  256 x 640, K = 640, 5 items 11.5 / 14.0;  200 x 512, K = 512, 6 items 9.9 / 12.4;  32 x 2048, K = 512, 4 items
  // 10.2 / 9.8;  256 x 2048, K = 256, 3 items 9.8 / 9.8;  beyond 256 tiles 128 x 2048, K = 4096, 6 items 65 / 73;  512 x 512, K = 4096, 6 items
  // 48 / 64;  256 x 768, K = 1536, 8 items 25 / 29;  256 x 1024, K = 8192, 6 items 91 / 122.  One row or column of tiles reads its long
  // operand once in either kernel, and beyond a tile a CU the 128 x 128 tiles keep more of it in flight: 64 x 2048, K = 2048, 8 items (256 tiles)
  // 33 / 40;  64 x 4096, K = 4096, 5 items (320) 83 / 66;  K = 1024, 8 items (512) 30.5 / 26.8;  64 x 2048, K = 1024, 9 items (288) 25.9 / 19.3;
  // 8192 x 64, K = 1600, 4 items (512) 41.4 / 28.8;  2600 x 64, K = 2560, 8 items (328) 57.6 / 42.4;  3000 x 40, K = 512, 6 items (282) 11.6 / 12.2.
  // (Gradients of such layers stay: 96 x 1500, K = 700 16.4 / 14.5.)
  const bool small_grid = plain && b_kmajor && tiles(g, batch, 64, 64) <= (g.m > 64 && g.n > 64 ? 2 : 1) * (int64_t)hdet_compute_units();
  const bool aligned = hdet_bgemm_dma_eligible(g, a_kmajor, b_kmajor, epi);
  if (aligned && !small_grid && !(plain && few_tiles(g, batch)))
    return hdet_launch_bgemm_dma(g, a_kmajor, b_kmajor, epi, batch, s);
  if (a_kmajor && b_kmajor) {            // forward
    switch (epi) {
      case HDET_EPI_F32: return launch_general<true, true, HDET_EPI_F32>(g, batch, aligned, s);
      case HDET_EPI_BIAS_F32: return launch_general<true, true, HDET_EPI_BIAS_F32>(g, batch, aligned, s);
      case HDET_EPI_BIAS_RELU_BF16: return launch_general<true, true, HDET_EPI_BIAS_RELU_BF16>(g, batch, aligned, s);
      case HDET_EPI_BIAS_BF16: return launch_general<true, true, HDET_EPI_BIAS_BF16>(g, batch, aligned, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (a_kmajor) {                        // dgrad
    if (epi == HDET_EPI_MASK_BF16) return launch_general<true, false, HDET_EPI_MASK_BF16>(g, batch, aligned, s);
    if (epi == HDET_EPI_BF16) return launch_general<true, false, HDET_EPI_BF16>(g, batch, aligned, s);
    return hipErrorInvalidValue;
  }
  if (!b_kmajor) {                       // wgrad
    if (epi == HDET_EPI_F32) return launch_general<false, false, HDET_EPI_F32>(g, batch, aligned, s);
    if (epi == HDET_EPI_BF16) return launch_general<false, false, HDET_EPI_BF16>(g, batch, aligned, s);
  }
  return hipErrorInvalidValue;
}
