// Causal self-attention of the transformer replicas in mixed precision, forward and backward,
// with the scores kept on chip ("Forward + backward" of Algorithm 1 for the attention part of a
// block).  For head size 64 and sequence lengths that are multiples of 64 this replaces five
// batched GEMMs, two softmax kernels and the [S][S] score and probability tensors in HBM by
// three kernels that stream 64-row tiles of k, v (or q and the output gradient) through LDS.
//
// Arithmetic: products and sums as the unfused path forms them, with bf16 operands and fp32 accumulation:
//   forward   s = (q k^T) * scale (fp32), causal mask, p = exp(s - max s) / sum exp(s - max s), a = bf16(p) v
//   backward  dot = sum_c da_c a_c (fp32, a before it was rounded), dp = da v^T - dot,
//             ds = bf16(bf16(p) dp), dq = (ds k) scale, dk = (ds^T q) scale, dv = bf16(p)^T da
// with scale = 1 / (sqrt(d_head) tau_r), tau_r the replica's attention temperature when that is
// an explored channel (Remark 1).  Because p is rounded after the normalisation, as the unfused path does it, the forward
// walks its tiles twice: for the row sums, then for the product (rounding exp(s - max) instead, in one walk, moves the loss
// of a small model by 5e-4).  It leaves each row's maximum and the reciprocal of its sum ([rows] fp32 each), from which all three kernels
// form p by the same operations, hence bit for bit alike, and what rounding took off a (a_rest), so that dot
// comes from the fp32 a and the backward kernels walk their tiles once.  The dp accumulators start at minus dot.
//
// What bounds them: neither pipe is full (matrix cores busy 21 to 24 % of the cycles at S = 512, 10 to 14 % at S = 256); a wavefront's chain from
// its LDS reads over the products and the exponentials to the next products, with the 2 to 4 wavefronts a SIMD holds, and below S = 512 what a block
// does before and after its few tiles.  us in a step, forward / dq / dk and dv:
//   8 replicas x 16 sequences x 16 heads, S = 512   198 / 338 / 305 -> 204 / 241 / 293
//   4 x 2 x 8, S = 2048                             107 / 179 / 134 -> 80 / 81 / 91
//   8 x 16 x 8, S = 256                             43 / 66 / 54 -> 48 / 57 / 58
// The backward kernels' include the column sums of sum_columns (1 to 2 % of dq, 3 to 6 % of dk and dv), which were a pass of their own of 77 us at
// S = 512 and 23 at S = 256.  The forward has become slower up to S = 512: it writes what rounding took off a beside a, for one walk less in dq.
// (before: dq walked its tiles twice, tiles went through registers into LDS, results of the paths of a tile were copied together, and every grid
// had the first order of remap_block.)  Measured and not kept: both 32 x 32 blocks of a
// tile in one basic block, 211 to 256 registers, 20 to 30 % slower in the backward kernels; dk and dv with 3 wavefronts
// a SIMD, 313 us (registers spill); launches of 1 to 4 replicas at a time, so that dk and dv find in the memory-side cache what dq read, 5 to 50 %
// slower; ds from the unrounded p, which moves the gradients of a small model by 5e-3.
//
// Layout: qkv [N][B][S][3d] bf16 (q | k | v, head h in columns h*64..), a and da [N][B][S][d],
// dqkv like qkv.  A block is 4 wavefronts; a wavefront owns 32 rows (queries in the forward and
// in the dq kernel, keys in the dk/dv kernel) whose operand fragments it loads once from global
// memory into registers, and walks the 64-row tiles of the other side, which go from global memory straight into
// LDS one or two tiles ahead (three in the forward's first walk), with one barrier per tile.  The tiles at the diagonal have a loop of their own,
// a 32 x 32 block at a time; the others need no tests.  Products are v_mfma_f32_32x32x16_bf16 blocks.  The first
// product is formed with the wavefront's own rows as the accumulator's COLUMNS, so that a lane
// holds one of its rows and 16 entries of the other side per block: row reductions stay inside
// a lane (plus one exchange between the half-wavefronts at the very end), and the accumulator
// registers, rounded to bf16, are directly the second product's B operand (contraction index =
// accumulator row) -- probabilities and ds never pass through LDS.  The accumulator keeps the
// rows of a 16-row step in the order (0..3, 8..11 | 4..7, 12..15) over the two half-wavefronts;
// the A operand of the second product is read from its LDS tile in that same order with the
// transposing LDS load, so nothing is transposed or permuted in memory.
// Every sum has a fixed order: results do not depend on scheduling.

#include "hdet_internal.h"
#include "hdet_elem.h"
#include "hdet_lds.h"

// the exponent is one explicit fma in all three kernels, nothing else is contracted
#pragma clang fp contract(off)

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));
typedef unsigned short us4 __attribute__((ext_vector_type(4)));

constexpr int DH = 64;            // head size
constexpr int TB = 64;            // rows of a streamed LDS tile
constexpr int PT = DH + 8;        // pitch of a strip of results
constexpr int WR = 32;            // rows a wavefront owns
constexpr int NWV = 4;            // wavefronts per block
constexpr int RB = WR * NWV;      // rows a block owns
constexpr int THREADS = 64 * NWV;
constexpr int TILE = TB * DH;     // elements of one LDS tile
constexpr int SMAX = 16384;       // longest sequence accepted
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ unsigned short f2bf(float x) { return __builtin_bit_cast(unsigned short, (__bf16)x); }
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
// What rounding to bf16 took off an fp32 number, in 16 bits: the difference of the two as integers, in units of fp32's last place.  Only a
// number halfway between two bf16 may have been 2^15 such units above its bf16 and is kept as 2^15 - 1.
__device__ __forceinline__ unsigned short rest_of(float x) {
  const int d = (int)(__float_as_uint(x) - ((unsigned)f2bf(x) << 16));
  return (unsigned short)(d > 32767 ? 32767 : d < -32768 ? -32768 : d);
}
// the fp32 number from its bf16 and rest
__device__ __forceinline__ float with_rest(unsigned short hi, unsigned short rest) { return __uint_as_float(((unsigned)hi << 16) + (unsigned)(int)(short)rest); }

// Tiles lie in LDS as [64][64], the eight 16-byte chunks of row r permuted by XOR with swz(r): the 32 rows of a k-contiguous fragment
// and the 4 rows x 64 bytes that half a wavefront of the transposing read touches both fall on disjoint banks.
__device__ __forceinline__ int swz(int r) { return ((r & 2) << 1) | ((r >> 2) & 3); }
// Where a lane's fragments begin inside a tile (elements)
struct frag_address {
  int k[4], t[2][2];
  __device__ __forceinline__ explicit frag_address(int lane) {
    const int row = lane & 31, p = lane & 15;
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) k[k4] = row * DH + (((2 * k4 + (lane >> 5)) ^ swz(row)) << 3);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int kr = ((lane >> 5) << 2) + (p >> 2) + 8 * u;
        t[dt][u] = kr * DH + (((4 * dt + ((lane >> 4) & 1) * 2 + ((p & 3) >> 1)) ^ swz(kr)) << 3) + ((p & 1) << 2);
      }
  }
  // MFMA 32x32x16 operand fragment of lane l: (row = l % 32, k = 16 k4 + 8 * (l / 32) + 0..7) of a tile's 32 rows from `tile` on
  __device__ __forceinline__ bf16x8 rows(const uint16_t* tile, int k4) const { return *reinterpret_cast<const bf16x8*>(tile + k[k4]); }
  // Fragment of an operand that is contracted along its tile's ROW index (its rows are the tile's columns 32 dt ..),
  // with the 16 k of the step in accumulator order: half-wavefront h holds k = ks + 4h + 0..3 and
  // ks + 8 + 4h + 0..3.  Within a 16-lane group, lane p points at the 4 elements
  // (k = kb + p / 4, columns cb + 4 * (p % 4) .. + 3) and lane i receives (k = kb .. kb + 3, column cb + i)
  // from the transposing read.
  __device__ __forceinline__ bf16x8 cols(const uint16_t* tile, int dt, int ks) const {
    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(tile + ks * DH + t[dt][0]));
    const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(tile + ks * DH + t[dt][1]));
    const s8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, both);
  }
};
// Fragment (row = l % 32, k = ks + 8 * (l / 32) + 0..7) from global memory (row pitch ld elements)
__device__ __forceinline__ bf16x8 frag_g(const uint16_t* src, int64_t ld, int ks, int lane) {
  return *reinterpret_cast<const bf16x8*>(src + (int64_t)(lane & 31) * ld + ks + ((lane >> 5) << 3));
}
__device__ __forceinline__ f16v mfma(bf16x8 a, bf16x8 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f16v all16(float x) {
  f16v z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = x;
  return z;
}
__device__ __forceinline__ f16v zero16() { return all16(0.f); }
// accumulator element e of lane l sits at (row = (e / 4) * 8 + (l / 32) * 4 + e % 4, col = l % 32) of its 32x32 block
__device__ __forceinline__ int acc_row(int e, int lane) { return ((e >> 2) << 3) + ((lane >> 5) << 2) + (e & 3); }
// elements 8 j .. 8 j + 7 of an accumulator block as the B fragment of contraction step j
__device__ __forceinline__ bf16x8 acc_frag(const f16v& x, int j) {
  bf16x8 f;
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = (__bf16)x[8 * j + t];
  return f;
}
__device__ __forceinline__ float other_half(float x) { return __shfl_xor(x, 32); }
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
// The probability, before it is rounded to bf16, from the raw score s, the row's maximum of s c and 1 / (row sum).  The maximum's rounding
// cancels in the normalisation; that of one statistic for both, maximum plus log2 sum, does not: half an ulp of a number as large as the scores.
__device__ __forceinline__ float prob(float s, float c, float mx, float inv) { return exp2_fast(__builtin_fmaf(s, c, -mx)) * inv; }

// entries of an accumulator block whose row index (row0 + row in block) exceeds `limit` become `fill`
__device__ __forceinline__ void fill_above(f16v& x, int row0, int limit, int lane, float fill) {
  const int last = limit - row0 - acc_row(0, lane);
#pragma unroll
  for (int e = 0; e < 16; ++e) x[e] = acc_row(e, 0) > last ? fill : x[e];
}
// ... whose row index is below `limit`
__device__ __forceinline__ void fill_below(f16v& x, int row0, int limit, int lane, float fill) {
  const int first = limit - row0 - acc_row(0, lane);
#pragma unroll
  for (int e = 0; e < 16; ++e) x[e] = acc_row(e, 0) < first ? fill : x[e];
}

// The 64 x 64 bf16 tiles of a matrix (row pitch ld), from global memory straight to LDS: two instructions a wavefront and tile
struct tile_stream {
  const uint16_t* src;
  int64_t ld;
  uint32_t off;            // byte offset of this lane's first chunk inside a tile
  int wave;
  __device__ __forceinline__ tile_stream(const uint16_t* src_, int64_t ld_, int tid, int wave_) : src(src_), ld(ld_), wave(wave_) {
    off = (uint32_t)(((tid >> 3) * ld + (((tid & 7) ^ swz(tid >> 3)) << 3)) * 2);
  }
  // tile t to the LDS bytes [at, at + 8192); zeros if it does not exist
  __device__ __forceinline__ void load(int t, bool exists, uint32_t at) const {
    const hdet_rsrc rs = make_rsrc(src + (int64_t)t * TB * ld, exists ? (uint32_t)(((TB - 1) * ld + DH) * 2) : 0u);
    lds_load16(rs, at + wave * 1024, off);
    lds_load16(rs, at + 4096 + wave * 1024, off + (uint32_t)(64 * ld));
  }
};

struct attn_args {
  const uint16_t* qkv;      // [N][B][S][3d]
  uint16_t* a;              // forward: [N][B][S][d] output
  uint16_t* a_rest;         // ... and what rounding took off it (rest_of)
  const uint16_t* da;       // backward: gradient at a
  uint16_t* dqkv;           // backward: [N][B][S][3d]
  float* row_max;           // [N][B][heads][S] the row's maximum of s c, c = scale log2 e
  float* row_inv;           // 1 / the row's sum of exp2(s c - maximum)
  float* row_ndot;          // minus the row's dot
  float* colsum;            // backward: sums of dqkv over the rows of a block, [N][B][S / 128][3d], or null
  const hdet_ctrl* ctrl;
  int temp_channel;
  float scale;              // 1 / sqrt(d_head)
  int B, S, heads, d;
  bool heavy_first;         // order of the blocks (remap_block)
};

__device__ __forceinline__ float replica_scale(const attn_args& g, int r) {
  return g.temp_channel >= 0 ? g.scale / (float)hdet_channel_value(g.ctrl, g.temp_channel, r, 0.0) : g.scale;
}

// Blocks reach the chip's 8 XCDs round-robin in launch order, and with causal masking the work of
// a block grows with its position in the sequence: left alone, an XCD would always receive the
// same position.  Launch index -> (row block counted from the longest, sequence and head, replica) such that every XCD
// works through a contiguous range of (replica, sequence, head), in one of two orders:
//  * all row blocks of each together, which keeps the tiles they share in one L2;
//  * heavy_first: the longest row blocks of all of them, then the next ones.  In the first order the blocks of the last
//    round are of any length (S = 2048, 1024 blocks: the CUs are busy 60 to 65 % of the kernel's time).
// heavy_first_order says when.
struct block_id { int x, bh, r; };
__device__ __forceinline__ block_id remap_block(bool heavy_first) {
  const unsigned nx = gridDim.x, ny = gridDim.y, heads = ny * gridDim.z, total = nx * heads;
  unsigned lin = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
  block_id b;
  unsigned grp;
  if (heavy_first) {
    if ((heads & 7u) == 0u) {
      const unsigned own = heads >> 3, j = lin >> 3;
      b.x = j / own;
      grp = (lin & 7u) * own + j % own;
    } else {
      b.x = lin / heads;
      grp = lin % heads;
    }
  } else {
    if ((total & 7u) == 0u) lin = (lin & 7u) * (total >> 3) + (lin >> 3);
    grp = lin / nx;
    // within an XCD the blocks go round-robin over shader engines and their CUs as well: rotate the
    // row block from one (sequence, head) to the next so that no unit keeps seeing the same one
    b.x = (lin % nx + grp + (grp >> 3) + (grp >> 6)) % nx;
  }
  b.bh = grp % ny;
  b.r = grp / ny;
  return b;
}

// The wavefront's [32 rows][64] result, held transposed in two accumulator blocks (block dt:
// columns 32 dt .., lane = row), goes to `dst` (row pitch ld) as to16(value) through the wavefront's LDS strip
// so that every global store writes 16 bytes of a row.
template <typename F>
__device__ __forceinline__ void store_rows(const f16v (&o)[2], F&& to16, uint16_t* stg, uint16_t* dst, int64_t ld, bool on, int lane) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const us4 x = {to16(o[dt][4 * e4]), to16(o[dt][4 * e4 + 1]), to16(o[dt][4 * e4 + 2]), to16(o[dt][4 * e4 + 3])};
      *reinterpret_cast<us4*>(stg + (lane & 31) * PT + dt * 32 + acc_row(4 * e4, lane)) = x;
    }
  __syncthreads();
  if (on) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = lane + 64 * i, row = c >> 3, col = (c & 7) << 3;
      *reinterpret_cast<us8*>(dst + (int64_t)row * ld + col) = *reinterpret_cast<const us8*>(stg + row * PT + col);
    }
  }
}

// The block's 64 column sums over its 128 rows, as stored, from the wavefronts' strips (stage 1 of the qkv bias gradient, which was a pass
// over dqkv of 77 us at S = 512, where the two kernels grow by 13; 23 against 4 at S = 256): one product of each strip against ones, then the
// four wavefronts in the order of their rows.
// Every thread calls it; all 128 rows exist.
__device__ __forceinline__ void sum_columns(const uint16_t* strips, float* sums, float* dst, int tid) {
  const int lane = tid & 63, w = tid >> 6, p = lane & 15;
  const us8 o = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const uint16_t* from = strips + w * WR * PT + (((lane >> 5) << 2) + (p >> 2)) * PT + ((lane >> 4) & 1) * 16 + ((p & 3) << 2);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    f16v x = zero16();
#pragma unroll
    for (int ks = 0; ks < WR; ks += 16) {
      const uint16_t* q = from + ks * PT + 32 * dt;
      const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(q));
      const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(q + 8 * PT));
      const s8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      x = mfma(__builtin_bit_cast(bf16x8, o), __builtin_bit_cast(bf16x8, both), x);
    }
    if (lane < 32) sums[w * DH + 32 * dt + lane] = x[0];
  }
  __syncthreads();
  if (tid < DH) dst[tid] = (sums[tid] + sums[DH + tid]) + (sums[2 * DH + tid] + sums[3 * DH + tid]);
}

// ---------------------------------------------------------------------------------------------
// forward: block = 128 queries of one (replica, sequence, head)
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(THREADS, 4) void attn_fwd_kernel(const attn_args g) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[4 * TILE];      // a ring of tiles: the keys, then keys and values in turn
  const block_id blk = remap_block(g.heavy_first);
  const int qblk = gridDim.x - 1 - blk.x, bh = blk.bh, r = blk.r;         // longest blocks first
  const int b = bh / g.heads, h = bh - b * g.heads;
  const int tid = threadIdx.x, lane = tid & 63, qi = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ld = 3 * (int64_t)g.d;
  const int64_t tok0 = ((int64_t)r * g.B + b) * g.S;
  const uint16_t* base = g.qkv + tok0 * ld + h * DH;
  const int q0 = qblk * RB, wq0 = q0 + w * WR;
  const bool on = wq0 < g.S;                                               // S is a multiple of 64, not of 128
  const int nfull = q0 / TB;                                               // key tiles below the diagonal for all wavefronts
  const int nkb = (q0 + RB < g.S ? q0 + RB : g.S) / TB;                    // ... that the block walks

  const tile_stream keys(base + g.d, ld, tid, w), vals(base + 2 * g.d, ld, tid, w);
  const uint32_t s_addr = lds_addr_of(smem);
  // entry j of the ring: key tiles 0 .. nkb - 1, then key and value tiles 0, 0, 1, 1, ..; past the end zeros
  auto request = [&](int j) {
    const uint32_t at = s_addr + (j & 3) * (TILE * 2);
    const int u = j - nkb;
    if (u < 0) keys.load(j, true, at);
    else if (u & 1) vals.load(u >> 1, u < 2 * nkb, at);
    else keys.load(u >> 1, u < 2 * nkb, at);
  };
  request(0); request(1); request(2);
  const float c = replica_scale(g, r) * kLog2e;
  bf16x8 fq[4];
#pragma unroll
  for (int k4 = 0; k4 < 4; ++k4) fq[k4] = frag_g(base + (int64_t)(on ? wq0 : 0) * ld, ld, k4 * 16, lane);
  const frag_address fa(lane);

  // raw scores of a 32-key block, [key][query]
  auto scores = [&](const uint16_t* kt) {
    f16v s = zero16();
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) s = mfma(fa.rows(kt, k4), fq[k4], s);
    return s;
  };
  // the wavefront's 32-key blocks of a tile at the diagonal: f(block, first key, across the diagonal)
  auto at_diagonal = [&](int kb, auto&& f) {
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {
      const int key0 = kb * TB + 32 * i;
      if (on && key0 <= wq0) f(i, key0, key0 == wq0);
    }
  };

  // pass 1: row maximum (of the raw scores) and sum, each half-wavefront over its own keys
  float m = -1e30f, l = 0.f;
  auto sum_block = [&](f16v& x) {
    float top = m, sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) top = fmaxf(top, x[e]);
    const float tc = top * c;
#pragma unroll
    for (int e = 0; e < 16; ++e) sum += exp2_fast(__builtin_fmaf(x[e], c, -tc));
    l = l * exp2_fast((m - top) * c) + sum;
    m = top;
  };
  for (int kb = 0; kb < nfull; ++kb) {
    wait_and_barrier<4>();
    request(kb + 3);
    const uint16_t* kt = smem + (kb & 3) * TILE;
    f16v x0 = scores(kt), x1 = scores(kt + 32 * DH);
    sum_block(x0);
    sum_block(x1);
  }
  for (int kb = nfull; kb < nkb; ++kb) {
    wait_and_barrier<4>();
    request(kb + 3);
    at_diagonal(kb, [&](int i, int key0, bool across) {
      f16v x = scores(smem + (kb & 3) * TILE + 32 * i * DH);
      if (across) fill_above(x, key0, wq0 + qi, lane, -INFINITY);
      sum_block(x);
    });
  }
  const float mo = other_half(m), lo = other_half(l), top = fmaxf(m, mo);
  const float mx = top * c;
  const float inv = 1.f / (l * exp2_fast((m - top) * c) + lo * exp2_fast((mo - top) * c));

  // pass 2: a^T = v^T p^T, [column][query]
  f16v o[2] = {zero16(), zero16()};
  auto add_block = [&](f16v& x, const uint16_t* vt) {
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = prob(x[e], c, mx, inv);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 pf = acc_frag(x, j);
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) o[dt] = mfma(fa.cols(vt, dt, 16 * j), pf, o[dt]);
    }
  };
  const uint16_t *kt, *vt;
  auto next = [&](int kb) {
    const int j = nkb + 2 * kb;
    if (kb == 0) {
      wait_and_barrier<2>();
    } else {
      wait_and_barrier<0>();
      request(j + 2);
    }
    request(j + 3);
    kt = smem + (j & 3) * TILE;
    vt = smem + ((j + 1) & 3) * TILE;
  };
  for (int kb = 0; kb < nfull; ++kb) {
    next(kb);
    f16v x0 = scores(kt);
    add_block(x0, vt);
    f16v x1 = scores(kt + 32 * DH);
    add_block(x1, vt + 32 * DH);
  }
  for (int kb = nfull; kb < nkb; ++kb) {
    next(kb);
    at_diagonal(kb, [&](int i, int key0, bool across) {
      f16v x = scores(kt + 32 * i * DH);
      if (across) fill_above(x, key0, wq0 + qi, lane, -INFINITY);
      add_block(x, vt + 32 * i * DH);
    });
  }
  wait_and_barrier<0>();
  if (on && lane < 32) {
    const int64_t gr = (((int64_t)r * g.B + b) * g.heads + h) * g.S + wq0 + qi;
    g.row_max[gr] = mx;
    g.row_inv[gr] = inv;
  }
  const int64_t out = (tok0 + (on ? wq0 : 0)) * g.d + h * DH;
  store_rows(o, f2bf, smem + w * WR * PT, g.a + out, g.d, on, lane);
  store_rows(o, rest_of, smem + w * WR * PT, g.a_rest + out, g.d, on, lane);
}

// ---------------------------------------------------------------------------------------------
// backward, step 1: the row dots and dq; block = 128 queries
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(THREADS, 3) void attn_bwd_dq_kernel(const attn_args g) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[3 * 2 * TILE];  // keys and values, three stages
  const block_id blk = remap_block(g.heavy_first);
  const int qblk = gridDim.x - 1 - blk.x, bh = blk.bh, r = blk.r;
  const int b = bh / g.heads, h = bh - b * g.heads;
  const int tid = threadIdx.x, lane = tid & 63, qi = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ld = 3 * (int64_t)g.d;
  const int64_t tok0 = ((int64_t)r * g.B + b) * g.S;
  const uint16_t* base = g.qkv + tok0 * ld + h * DH;
  const int q0 = qblk * RB, wq0 = q0 + w * WR;
  const bool on = wq0 < g.S;
  const int nfull = q0 / TB;
  const int nkb = (q0 + RB < g.S ? q0 + RB : g.S) / TB;
  const int64_t gr = (((int64_t)r * g.B + b) * g.heads + h) * g.S + (on ? wq0 : 0) + qi;

  const tile_stream keys(base + g.d, ld, tid, w), vals(base + 2 * g.d, ld, tid, w);
  const uint32_t s_addr = lds_addr_of(smem);
  auto request = [&](int t, int stage) {
    keys.load(t, t < nkb, s_addr + stage * (4 * TILE));
    vals.load(t, t < nkb, s_addr + stage * (4 * TILE) + 2 * TILE);
  };
  bf16x8 fq[4], fda[4];
  float ndot = 0.f;                        // minus the row's dot = sum over the columns of da a, in fp32: 32 columns a half-wavefront
  {
    const int64_t row = (tok0 + (on ? wq0 : 0)) * g.d + h * DH;
    us8 hi[4], rest[4];
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) {
      fda[k4] = frag_g(g.da + row, g.d, k4 * 16, lane);
      hi[k4] = __builtin_bit_cast(us8, frag_g(g.a + row, g.d, k4 * 16, lane));
      rest[k4] = __builtin_bit_cast(us8, frag_g(g.a_rest + row, g.d, k4 * 16, lane));
    }
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
      for (int t = 0; t < 8; ++t) ndot = __builtin_fmaf(-(float)fda[k4][t], with_rest(hi[k4][t], rest[k4][t]), ndot);
  }
  request(0, 0);
  request(1, 1);
#pragma unroll
  for (int k4 = 0; k4 < 4; ++k4) fq[k4] = frag_g(base + (int64_t)(on ? wq0 : 0) * ld, ld, k4 * 16, lane);
  const float mx = g.row_max[gr], inv = g.row_inv[gr];
  const float scale = replica_scale(g, r);
  const float c = scale * kLog2e;
  ndot += other_half(ndot);
  const frag_address fa(lane);

  f16v o[2] = {zero16(), zero16()};        // dq^T = k^T ds^T, [column][query]
  auto block = [&](const uint16_t* kt, int key0, bool across) {
    const uint16_t* vt = kt + TILE;
    f16v s = zero16(), dp = all16(ndot);   // [key][query]; dp = v da^T - dot
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) s = mfma(fa.rows(kt, k4), fq[k4], s);
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) dp = mfma(fa.rows(vt, k4), fda[k4], dp);
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = prob(s[e], c, mx, inv);
    if (across) fill_above(s, key0, wq0 + qi, lane, 0.f);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 pf = acc_frag(s, j);
#pragma unroll
      for (int t = 0; t < 8; ++t) dp[8 * j + t] *= (float)pf[t];
      const bf16x8 dsf = acc_frag(dp, j);
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) o[dt] = mfma(fa.cols(kt, dt, 16 * j), dsf, o[dt]);
    }
  };
  int stage = 0, ahead = 2;
  auto next = [&](int kb) {                // waits for tile kb, requests kb + 2
    wait_and_barrier<4>();
    request(kb + 2, ahead);
    const uint16_t* kt = smem + stage * (2 * TILE);
    ahead = stage;
    stage = stage == 2 ? 0 : stage + 1;
    return kt;
  };
  for (int kb = 0; kb < nfull; ++kb) {
    const uint16_t* kt = next(kb);
#pragma unroll 1
    for (int i = 0; i < 2; ++i) block(kt + 32 * i * DH, 0, false);
  }
  for (int kb = nfull; kb < nkb; ++kb) {
    const uint16_t* kt = next(kb);
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {
      const int key0 = kb * TB + 32 * i;
      if (on && key0 <= wq0) block(kt + 32 * i * DH, key0, key0 == wq0);
    }
  }
  wait_and_barrier<0>();
  if (on && lane < 32) g.row_ndot[gr] = ndot;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] *= scale;
  store_rows(o, f2bf, smem + w * WR * PT, g.dqkv + (tok0 + (on ? wq0 : 0)) * ld + h * DH, ld, on, lane);
  if (g.colsum) sum_columns(smem, reinterpret_cast<float*>(smem + RB * PT), g.colsum + (tok0 + q0) / RB * ld + h * DH, tid);
}

// ---------------------------------------------------------------------------------------------
// backward, step 2: dk and dv; block = 128 keys, walks the query tiles at or below the diagonal
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(THREADS, 2) void attn_bwd_dkv_kernel(const attn_args g) {
  // queries, output gradients and the queries' three row statistics (a wavefront each, the last one twice): three stages
  constexpr int STAGE = 2 * TILE + NWV * TB * 2;
  __shared__ __attribute__((aligned(1024))) uint16_t smem[3 * STAGE];
  const block_id blk = remap_block(g.heavy_first);
  const int kblk = blk.x, bh = blk.bh, r = blk.r;                          // the first blocks walk the most tiles
  const int b = bh / g.heads, h = bh - b * g.heads;
  const int tid = threadIdx.x, lane = tid & 63, ki = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ld = 3 * (int64_t)g.d;
  const int64_t tok0 = ((int64_t)r * g.B + b) * g.S;
  const uint16_t* base = g.qkv + tok0 * ld + h * DH;
  const int64_t gr0 = (((int64_t)r * g.B + b) * g.heads + h) * g.S;
  const int k0 = kblk * RB, wk0 = k0 + w * WR;
  const bool on = wk0 < g.S;
  const int qb0 = k0 / TB, nqb = g.S / TB;

  const tile_stream qs(base, ld, tid, w), das(g.da + tok0 * g.d + h * DH, g.d, tid, w);
  const float* const stats = (w == 0 ? g.row_max : w == 1 ? g.row_inv : g.row_ndot) + gr0;
  const uint32_t s_addr = lds_addr_of(smem);
  auto request = [&](int t, int stage) {
    const uint32_t at = s_addr + stage * (2 * STAGE);
    qs.load(t, t < nqb, at);
    das.load(t, t < nqb, at + 2 * TILE);
    lds_load4(make_rsrc(stats + (int64_t)t * TB, t < nqb ? TB * 4 : 0), at + 4 * TILE + w * (TB * 4), lane * 4);
  };
  bf16x8 fk[4], fv[4];
#pragma unroll
  for (int k4 = 0; k4 < 4; ++k4) {
    fk[k4] = frag_g(base + g.d + (int64_t)(on ? wk0 : 0) * ld, ld, k4 * 16, lane);
    fv[k4] = frag_g(base + 2 * g.d + (int64_t)(on ? wk0 : 0) * ld, ld, k4 * 16, lane);
  }
  request(qb0, 0);
  request(qb0 + 1, 1);
  const float scale = replica_scale(g, r);
  const float c = scale * kLog2e;
  const frag_address fa(lane);

  f16v dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};        // [column][key]
  // a 32-query block: its tile rows, its statistics
  auto block = [&](const uint16_t* qt, const float* st, int qr0, bool across) {
    const uint16_t* dat = qt + TILE;
    f16v s = zero16(), dp;                                                 // [query][key]; dp = da v^T - dot
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {                                       // 4 consecutive queries at a time
      const f4 nd = *reinterpret_cast<const f4*>(st + 2 * TB + acc_row(4 * e4, lane));
#pragma unroll
      for (int u = 0; u < 4; ++u) dp[4 * e4 + u] = nd[u];
    }
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) s = mfma(fa.rows(qt, k4), fk[k4], s);
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) dp = mfma(fa.rows(dat, k4), fv[k4], dp);
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const f4 mx = *reinterpret_cast<const f4*>(st + acc_row(4 * e4, lane));
      const f4 inv = *reinterpret_cast<const f4*>(st + TB + acc_row(4 * e4, lane));
#pragma unroll
      for (int u = 0; u < 4; ++u) s[4 * e4 + u] = prob(s[4 * e4 + u], c, mx[u], inv[u]);
    }
    if (across) fill_below(s, qr0, wk0 + ki, lane, 0.f);                   // causal: query >= key
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 pf = acc_frag(s, j);
#pragma unroll
      for (int t = 0; t < 8; ++t) dp[8 * j + t] *= (float)pf[t];
      const bf16x8 dsf = acc_frag(dp, j);
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        dv[dt] = mfma(fa.cols(dat, dt, 16 * j), pf, dv[dt]);
        dk[dt] = mfma(fa.cols(qt, dt, 16 * j), dsf, dk[dt]);
      }
    }
  };
  int stage = 0, ahead = 2;
  auto next = [&](int qb) {                // waits for tile qb, requests qb + 2
    wait_and_barrier<5>();
    request(qb + 2, ahead);
    const uint16_t* qt = smem + stage * STAGE;
    ahead = stage;
    stage = stage == 2 ? 0 : stage + 1;
    return qt;
  };
  int qb = qb0;
  for (; qb < qb0 + RB / TB && qb < nqb; ++qb) {
    const uint16_t* qt = next(qb);
    const float* st = reinterpret_cast<const float*>(qt + 2 * TILE);
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {
      const int qr0 = qb * TB + 32 * i;
      if (on && qr0 >= wk0) block(qt + 32 * i * DH, st + 32 * i, qr0, qr0 == wk0);
    }
  }
  for (; qb < nqb; ++qb) {
    const uint16_t* qt = next(qb);
    const float* st = reinterpret_cast<const float*>(qt + 2 * TILE);
#pragma unroll 1
    for (int i = 0; i < 2; ++i) block(qt + 32 * i * DH, st + 32 * i, 0, false);
  }
  wait_and_barrier<0>();
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) dk[dt][e] *= scale;
  uint16_t* dst = g.dqkv + (tok0 + (on ? wk0 : 0)) * ld + h * DH;
  store_rows(dk, f2bf, smem + w * WR * PT, dst + g.d, ld, on, lane);
  store_rows(dv, f2bf, smem + (NWV + w) * WR * PT, dst + 2 * g.d, ld, on, lane);
  if (g.colsum) {
    float* const sums = reinterpret_cast<float*>(smem + 2 * RB * PT);
    float* const at = g.colsum + (tok0 + k0) / RB * ld + h * DH;
    sum_columns(smem, sums, at + g.d, tid);
    sum_columns(smem + RB * PT, sums + NWV * DH, at + 2 * g.d, tid);
  }
}

dim3 attn_grid(const hdet_attn_desc& a) { return dim3((a.seq_len + RB - 1) / RB, a.batch * a.heads, a.n_replicas); }

// Longest row blocks first: while the grid has few rounds, so that the length of the last one counts for more than the tiles that
// the blocks of a head find in the L2.  Forward / dq / dk and dv, time in this order over time in the other:
//   S = 2048, 1024 blocks 0.84 / 0.83 / 0.81, 4096 blocks 0.93 / 0.97 / 0.96, 8192 blocks 1.00 / 1.03 / 1.03;
//   S = 1024, 1024 blocks 0.90 / 1.00 / 0.85, 4096 blocks 0.97 / 1.00 / 0.99, 8192 blocks 1.05 / 1.10 / 1.04;
//   S = 512,  1024 blocks 0.92 / 1.00 / 0.92, 2048 blocks 0.94 / 1.02 / 0.98, 4096 blocks 1.02 / 1.06 / 0.98;
//   S = 256,  512 blocks 0.90 / 0.91 / 0.84, 2048 blocks 1.00 / 1.00 / 0.98;  S = 4096, 1152 blocks 0.76 / 0.89 / 0.84
bool heavy_first_order(const hdet_attn_desc& a) {
  const dim3 g = attn_grid(a);
  const int64_t blocks = (int64_t)g.x * g.y * g.z;
  return blocks <= (int64_t)(g.x >= 8 ? 16 : 8) * hdet_compute_units();
}

attn_args make_args(const hdet_attn_desc& a) {
  attn_args g;
  g.qkv = a.qkv; g.a = a.a; g.a_rest = a.a_rest; g.da = a.da; g.dqkv = a.dqkv;
  g.row_max = a.row_max; g.row_inv = a.row_inv; g.row_ndot = a.row_ndot; g.colsum = a.colsum;
  g.ctrl = a.ctrl; g.temp_channel = a.temp_channel; g.scale = a.scale;
  g.B = a.batch; g.S = a.seq_len; g.heads = a.heads; g.d = a.d_model;
  g.heavy_first = heavy_first_order(a);
  return g;
}

}  // namespace

bool hdet_attn_fusable(int seq_len, int d_model, int heads, int batch) {
  return heads > 0 && batch > 0 && d_model == heads * DH && seq_len % TB == 0 && seq_len >= TB && seq_len <= SMAX &&
         (int64_t)batch * heads <= 65535;
}

hipError_t hdet_launch_attn_fwd(const hdet_attn_desc& a, hipStream_t s) {
  if (!hdet_attn_fusable(a.seq_len, a.d_model, a.heads, a.batch)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attn_fwd_kernel, attn_grid(a), dim3(THREADS), 0, s, make_args(a));
  return hipGetLastError();
}

hipError_t hdet_launch_attn_bwd(const hdet_attn_desc& a, hipStream_t s) {
  if (!hdet_attn_fusable(a.seq_len, a.d_model, a.heads, a.batch) || (a.colsum && a.seq_len % RB)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attn_bwd_dq_kernel, attn_grid(a), dim3(THREADS), 0, s, make_args(a));
  hipLaunchKernelGGL(attn_bwd_dkv_kernel, attn_grid(a), dim3(THREADS), 0, s, make_args(a));
  return hipGetLastError();
}
