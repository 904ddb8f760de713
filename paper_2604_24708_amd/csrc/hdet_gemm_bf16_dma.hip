// Replica-batched bf16 GEMM on the gfx950 matrix cores, fast path: operand tiles go from
// global memory straight into LDS (buffer_load ... lds), several K steps ahead, and never pass
// through registers.  Same contract as the register-staged kernel in hdet_gemm_bf16.hip
// ("Forward + backward" of Algorithm 1 in mixed precision, N independent weight sets):
//
//   C(m,n) = sum_k A(m,k) * B(k,n)          A, B bfloat16; fp32 accumulation; C fp32 or bfloat16
//
// with the three operand orders of a Linear layer (forward NT, dgrad NN, wgrad TN).  The host
// routes a product here when every 8-element chunk of A and B is 16-byte aligned and either whole
// or absent and C can be written 4 columns at a time; everything else takes the other kernel.
//
// Design
//  * Block tile TM x TN, WGM x WGN wavefronts, each owning (TM/WGM) x 64.  K step TK = 32 or 64, NST LDS stages of one K step each.
//    Kernels with K steps of 64 work on 16x16 blocks of v_mfma_f32_16x16x32_bf16: on random
//    data the chip holds 2.03 PFLOP/s of these from registers, 1.82 of the 32x32x16 form, at whose larger blocks every accumulator
//    is read and written twice as often per operation.  With K steps of 32 a 16x16x32 block is the whole step, and its fragments are not read
//    while others multiply: those kernels keep 32x32x16, two sub-steps (weight gradients 3072 x 1024, K = 4096, 8 items 185 us, 205 with
//    16x16x32; K = 2048 94 and 101; gradients through GELU 4096 x 8192, K = 1024, 8 items 691 and 698).  The sums are the same to the bit.
//  * LDS-direct loads: one instruction moves 64 lanes x 16 bytes into 1 KiB of consecutive LDS.
//    Which global chunk a lane fetches is chosen so that the tile lands already swizzled:
//      - operand contiguous along k: tile [row][TK], the 16-byte chunks of a row XOR-permuted by
//        a function of the row, so that the 128-bit fragment reads hit disjoint banks;
//      - operand contiguous along the output axis: tile [k][ROWS], chunks XOR-permuted by
//        a function of k, so that the eight k-rows that half a wavefront of the transposing LDS read
//        (ds_read_b64_tr_b16) touches fall on disjoint banks.  No padding anywhere.
//    The loads go through a buffer descriptor whose extent is the operand of this batch item:
//    chunks outside it (ragged m, n, k edges) are given an out-of-range offset and arrive as
//    zeros, so the loop has no edge cases.
//  * Pipeline: the stage NST K steps ahead is requested as soon as its buffer is free.  One
//    barrier per K step, placed before the last MFMA sub-step: by then every wavefront has read
//    the whole current stage into registers, so the stage is refilled at once, and the next
//    stage has landed (s_waitcnt vmcnt leaves the younger stages in flight).  Fragments are
//    double-buffered in registers across sub-steps, LDS reads and load issue are dealt out
//    between the MFMAs, and the order is pinned with sched_barrier.  The 256 x 256 tile has a kernel of its own (hdet_bgemm_alt_kernel).
//  * Epilogue through LDS: accumulators (lane = row, 4 consecutive columns) go through a
//    per-wavefront staging strip so that every global store writes whole rows, 4 columns per
//    lane; bias / ReLU / ReLU-gate / bf16 rounding (hardware round-to-nearest-even) fused.
//  * Launch order is remapped so that each XCD (own L2) works on a contiguous range of tiles, walked in groups
//    of tile rows so that concurrent blocks share operand tiles of both kinds.

#include "hdet_internal.h"
#include "hdet_elem.h"
#include "hdet_lds.h"
#include "hdet_update_math.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef hdet_rsrc i4;
typedef unsigned short us4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kAbsent = 0x80000000u;   // offset beyond every extent the host lets through

__device__ __forceinline__ unsigned short f2bf(float x) {      // round to nearest even
  return __builtin_bit_cast(unsigned short, (__bf16)x);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// The MFMA of a tile kernel, BLK x BLK with SK of the contraction.  Rows of C are the second operand's, so that a lane's accumulators come in
// fours of consecutive columns of one row.
template <int BLK> struct block;
template <> struct block<16> {
  static constexpr int SK = 32;
  typedef f4 acc;
  static __device__ __forceinline__ acc multiply(bf16x8 a, bf16x8 b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, c, 0, 0, 0); }
};
template <> struct block<32> {
  static constexpr int SK = 16;
  typedef f16v acc;
  static __device__ __forceinline__ acc multiply(bf16x8 a, bf16x8 b, acc c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0); }
};
// ... by K step (see the top of the file)
template <int TK> constexpr int kBlock = TK == 32 ? 32 : 16;

// One operand tile: ROWS rows of the output dimension x TK of the contraction.
// KMAJOR: element (row, k) at src[row * ld + k], LDS tile [row][TK];
// otherwise at src[k * ld + row], LDS tile [k][ROWS].
template <bool KMAJOR, int ROWS, int THREADS, int TK>
struct lds_tile {
  static constexpr int NI = ROWS * TK * 2 / (THREADS * 16);   // load instructions per thread and stage
  static constexpr int RCH = ROWS / 8;                        // chunks per k-row of a [k][ROWS] tile
  static constexpr int CPR = TK / 8;                          // chunks per row of a [row][TK] tile
  static_assert(KMAJOR || ROWS >= 128, "the chunk permutation of a [k][ROWS] tile needs at least 16 chunks per k-row");
  static_assert(TK == 32 || TK == 64, "K step");
  // chunk permutation inside a [row][TK] row: 64-byte rows by row / 4, 128-byte rows by row / 2
  static __device__ __forceinline__ int swz(int r) { return TK == 32 ? (r >> 2) & 3 : (r >> 1) & 7; }
  // ... of a [k][ROWS] row: a 32-lane half of the transposing read takes 64 bytes of each of 4 k-rows, or (16 x 16 blocks) 32 bytes of
  // each of 8 (k mod 4 and k / 8 differ)
  static __device__ __forceinline__ int swz_k(int k) { return ((k & 3) << 2) | (kBlock<TK> == 16 ? ((k >> 3) & 1) << 1 : 0); }
  uint32_t off[NI];     // byte offset of this lane's chunk at K step 0, or kAbsent
  int kofs[NI];         // k index of the chunk inside a K step
  uint32_t kstep;       // bytes per K step
  __device__ __forceinline__ void init(int row0, int rows, int64_t ld, int tid) {
    kstep = KMAJOR ? TK * 2 : (uint32_t)(ld * TK * 2);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = tid + i * THREADS;          // chunk slot in LDS order: LDS byte 16 c
      if (KMAJOR) {
        const int r = c / CPR, cg = (c % CPR) ^ swz(r);
        const int row = row0 + r;
        kofs[i] = cg * 8;
        off[i] = row < rows ? (uint32_t)((row * ld + cg * 8) * 2) : kAbsent;
      } else {
        const int kk = c / RCH, cg = (c % RCH) ^ swz_k(kk);
        const int row = row0 + cg * 8;
        kofs[i] = kk;
        off[i] = row < rows ? (uint32_t)((kk * ld + row) * 2) : kAbsent;
      }
    }
  }
  __device__ __forceinline__ void issue_one(int i, i4 rsrc, uint32_t tile_addr, int kt, int kdim, int wave) const {
    const uint32_t v = (kt * TK + kofs[i] < kdim) ? off[i] + (uint32_t)kt * kstep : kAbsent;
    lds_load16(rsrc, tile_addr + (i * THREADS + wave * 64) * 16, v);
  }
  // MFMA operand fragment: lane l gets (row = r0 + l % BLK, k = ks + 8 * (l / BLK) + 0..7).
  static __device__ __forceinline__ bf16x8 fragment(const uint16_t* tile, int r0, int ks, int lane) {
    constexpr int BLK = kBlock<TK>;
    if (KMAJOR) {
      const int row = r0 + lane % BLK;
      const int chunk = ((ks >> 3) + lane / BLK) ^ swz(row);
      return *reinterpret_cast<const bf16x8*>(tile + row * TK + (chunk << 3));
    }
    // Transposing read: within a 16-lane group, lane p points at the 4 elements
    // (k = kb + p / 4, rows r0 + 4 * (p % 4) .. + 3) and lane i receives (k = kb .. kb + 3, row r0 + i).
    const int p = lane & 15;
    const int row = r0 + (lane & (BLK - 16)) + ((p & 3) << 2);
    const int k = ks + ((lane / BLK) << 3) + (p >> 2);
    const uint16_t* q = tile + k * ROWS + (((row >> 3) ^ swz_k(k)) << 3) + (row & 7);
    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(q));
    const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4 __attribute__((address_space(3)))*)(q + 4 * ROWS));
    const s8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, both);
  }
};

// What lanes 32 .. 63 of a hold for what lanes 0 .. 31 of b hold; odd rows of 16 lanes of a for even rows of b
__device__ __forceinline__ void swap32(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void swap16(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0]; b = r[1];
}

// a reduction over the four groups of 16 lanes, the same value in each
template <typename F>
__device__ __forceinline__ float over_groups(float x, F op) {
  unsigned a = __float_as_uint(x), b = a;
  swap32(a, b);
  x = op(__uint_as_float(a), __uint_as_float(b));
  a = b = __float_as_uint(x);
  swap16(a, b);
  return op(__uint_as_float(a), __uint_as_float(b));
}

// Launch order -> tile: each XCD (own L2; blocks are dealt to the XCDs round-robin) works through a contiguous
// range of tiles, and inside a batch item consecutive tiles walk groups of tile_group tile rows column by column,
// so that the blocks an XCD runs at one time share operand tiles of both kinds in its L2.
struct tile_id { int bx, by, bz; };
__device__ __forceinline__ tile_id tile_of_index(unsigned t, unsigned gx, unsigned gy, unsigned total, int tile_group) {
  {   // XCD x = launch index mod 8 takes the x-th of eight contiguous ranges (the first total mod 8 ranges one tile longer)
    const unsigned x = t & 7u, rem = total & 7u;
    t = x * (total >> 3) + (x < rem ? x : rem) + (t >> 3);
  }
  tile_id id;
  const unsigned per = gx * gy;
  id.bz = t / per;
  const unsigned r = t - id.bz * per;
  const unsigned gm = tile_group > 1 ? (unsigned)tile_group : 1u;
  const unsigned gsz = gm * gx;
  const unsigned grp = r / gsz, first = grp * gm;
  const unsigned rows = gy - first < gm ? gy - first : gm;
  const unsigned q = r - grp * gsz;
  id.by = first + q % rows;
  id.bx = q / rows;
  return id;
}
__device__ __forceinline__ tile_id tile_of_block(int tile_group) {
  return tile_of_index(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x, gridDim.y, gridDim.x * gridDim.y * gridDim.z, tile_group);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr double kLn2 = 0.6931471805599453;

// The block's TM x TN tile to memory.  Accumulators go through LDS as fp32, the wavefront's own 32 rows x 64 columns at a time, and are read
// back with 4 consecutive columns a lane, so that every global access is made of whole rows of the strip.  (Strips of 16 rows x 256 columns
// shared by four wavefronts, whose accesses are whole 1 KiB rows, measured the same or, with the update, 6 % slower.)
// LDS serves one wavefront's accesses in order, so a strip needs no barrier.
// STREAM: results are written past the L2 (stream_result).  `S`: the stage buffers, which no wavefront reads or loads into any more.
template <int EPI, int TM, int TN, int WGM, int WGN, int BLK, bool STREAM, int LDS_BYTES>
__device__ __forceinline__ void store_tile(const hdet_bgemm_args& g, const typename block<BLK>::acc (&acc)[TM / WGM / BLK][TN / WGN / BLK], uint16_t* S,
                                           int bx, int by, int z, int64_t c_base, int tid) {
  constexpr int THREADS = 64 * WGM * WGN;
  constexpr int SR = 32, CW = 64, EP = CW + 4, LPR = CW / 4, RPI = 64 / LPR;      // pitch EP: both sides free of bank conflicts
  constexpr int NIT = SR / RPI, NSTRIP = TM / WGM / SR;
  static_assert(TN / WGN == CW, "a wavefront owns 64 columns");
  static_assert(WGM * WGN * SR * EP * 4 <= LDS_BYTES, "staging area exceeds the stage buffers");
  const int m0 = by * TM, n0 = bx * TN, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / WGN) * (TM / WGM), wn = (wave % WGN) * 64;
  float* const stg = reinterpret_cast<float*>(S) + wave * (SR * EP);
  const int lr = lane / LPR, lc = (lane % LPR) * 4;
  const int col = n0 + wn + lc;
  const bool col_ok = col < g.n;                             // n is a multiple of 4: the 4 columns exist together
  auto put = [&](auto* p, auto v) {
    if (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
  };
  constexpr bool kBias = EPI == HDET_EPI_BIAS_RELU_BF16 || EPI == HDET_EPI_BIAS_F32 || EPI == HDET_EPI_BIAS_BF16 ||
                         EPI == HDET_EPI_BIAS_GELU_BF16 || EPI == HDET_EPI_BIAS_RESID_BF16 || EPI == HDET_EPI_BIAS_DROP_RESID_BF16;
  // the second operand of the gating epilogues (the activations a ReLU or GELU gradient looks at) is
  // fetched one strip ahead, so that its latency hides behind the previous strip's pass through LDS
  constexpr bool kGate = EPI == HDET_EPI_MASK_BF16 || EPI == HDET_EPI_GELUGRAD_BF16 || EPI == HDET_EPI_BIAS_RESID_BF16 ||
                         EPI == HDET_EPI_BIAS_DROP_RESID_BF16;
  us4 gate[2][NIT];
  auto fetch_gate = [&](int strip, us4 (&dst)[NIT]) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int row = m0 + wm + strip * SR + it * RPI + lr;
      dst[it] = us4{0, 0, 0, 0};
      if (row < g.m && col_ok)
        dst[it] = *reinterpret_cast<const us4*>(g.mask + (int64_t)z * g.mask_bs + (int64_t)row * g.mask_ld + col);
    }
  };
  uint32_t drop_thresh = 0u;
  float drop_scale = 1.f;
  if (EPI == HDET_EPI_BIAS_DROP_RESID_BF16) {
    const float p = (float)hdet_channel_value(g.drop_ctrl, g.drop_channel, z, 0.0);
    drop_thresh = (uint32_t)floor((double)p * 4294967296.0);
    drop_scale = 1.f / (1.f - p);
  }
  // HDET_EPI_ADAMW: the tile is the replica's gradient of a weight matrix and is applied at once (Eq. 2 with the
  // replica's rate); the matrix's parameters and moments of a strip are requested before the strip goes through LDS
  constexpr bool kUpd = EPI == HDET_EPI_ADAMW;
  hdet_um::rep_scalars us = {0.f, 0.f, 0.f, 0.f};
  if (kUpd) {
    us = hdet_um::replica_scalars(g.upd, z);
    if (bx == 0 && by == 0 && tid == 0 && g.upd.lr_channel == 0) g.upd.ctrl_out->lr_used[z] = us.lr;
  }
  f4 uth[kUpd ? NIT : 1], um[kUpd ? NIT : 1], uv[kUpd ? NIT : 1];
  auto fetch_upd = [&](int strip) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int row = m0 + wm + strip * SR + it * RPI + lr;
      if (row < g.m && col_ok) {
        const int64_t off = c_base + (int64_t)row * g.ldc + col;
        uth[it] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(g.upd.theta + off));
        um[it] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(g.upd.m + off));
        uv[it] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(g.upd.v + off));
      }
    }
  };
  // column sums of the stored result over the rows this lane stores, for its 4 columns
  constexpr bool kColsum = EPI == HDET_EPI_GELUGRAD_BF16 || EPI == HDET_EPI_MASK_BF16;
  f4 csum = {0.f, 0.f, 0.f, 0.f};
  if (kGate) fetch_gate(0, gate[0]);
  f4 bias = {0.f, 0.f, 0.f, 0.f};
  if (kBias && col_ok) bias = *reinterpret_cast<const f4*>(g.bias + (int64_t)z * g.bias_bs + col);
#pragma unroll
  for (int strip = 0; strip < NSTRIP; ++strip) {
    if (kGate && strip + 1 < NSTRIP) fetch_gate(strip + 1, gate[(strip + 1) & 1]);
    if (kUpd) fetch_upd(strip);
    // accumulator element e of lane l is C(row, col) with row = l % BLK, col = (e / 4) * 8 + (l / BLK) * 4 + e % 4 inside its block
#pragma unroll
    for (int ib = 0; ib < SR / BLK; ++ib)
#pragma unroll
      for (int j = 0; j < CW / BLK; ++j) {
        const typename block<BLK>::acc& x = acc[strip * (SR / BLK) + ib][j];
#pragma unroll
        for (int e = 0; e < BLK * BLK / 64; e += 4)
          *reinterpret_cast<f4*>(stg + (ib * BLK + lane % BLK) * EP + j * BLK + e * 2 + (lane / BLK) * 4) = f4{x[e], x[e + 1], x[e + 2], x[e + 3]};
      }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      f4 v = *reinterpret_cast<const f4*>(stg + (it * RPI + lr) * EP + lc);
      const int row = m0 + wm + strip * SR + it * RPI + lr;
      if (row < g.m && col_ok) {
        const int64_t off = c_base + (int64_t)row * g.ldc + col;
        if (kBias) v += bias;
        if (EPI == HDET_EPI_BIAS_RELU_BF16) {
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = v[q] > 0.f ? v[q] : 0.f;
        }
        if (EPI == HDET_EPI_MASK_BF16) {    // gradient through the ReLU of the layer below
          const us4 a = gate[strip & 1][it];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = bf2f(a[q]) > 0.f ? v[q] : 0.f;
        }
        if (EPI == HDET_EPI_BIAS_RESID_BF16) {  // the layer's output is rounded as the unfused path stores it, then added
          const us4 a = gate[strip & 1][it];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = bf2f(a[q]) + bf2f(f2bf(v[q]));
        }
        if (EPI == HDET_EPI_BIAS_DROP_RESID_BF16) {   // ... dropped out (one Philox block per 4 elements), then added
          const us4 a = gate[strip & 1][it];
          hdet_philox4 w = {{0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu}};
          if (drop_thresh != 0u)
            w = hdet_philox4x32_10((uint32_t)(((int64_t)row * g.ldc + col) >> 2), g.drop_step, (uint32_t)z * 65536u + g.drop_site,
                                   g.drop_stream, g.drop_seed_lo, g.drop_seed_hi);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float y = bf2f(f2bf(v[q]));
            if (drop_thresh != 0u) y = w.x[q] >= drop_thresh ? y * drop_scale : 0.f;
            v[q] = bf2f(a[q]) + y;
          }
        }
        if (EPI == HDET_EPI_GELUGRAD_BF16) {  // the incoming gradient is rounded as the unfused path stores it
          const us4 a = gate[strip & 1][it];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = bf2f(f2bf(v[q])) * hdet_gelu_tanh_grad_fast(bf2f(a[q]));
        }
        if (EPI == HDET_EPI_ADAMW) {
          f4 th = uth[it], mm = um[it], vv = uv[it];
          hdet_um::update_one<HDET_ADAMW, f4>(th, v, mm, vv, g.upd, us);
          __builtin_nontemporal_store(mm, reinterpret_cast<f4*>(g.upd.m + off));
          __builtin_nontemporal_store(vv, reinterpret_cast<f4*>(g.upd.v + off));
          __builtin_nontemporal_store(th, reinterpret_cast<f4*>(g.upd.theta + off));
          if (g.upd.shadow) {
            const us4 o = {hdet_um::to_bf16(th[0]), hdet_um::to_bf16(th[1]), hdet_um::to_bf16(th[2]), hdet_um::to_bf16(th[3])};
            __builtin_nontemporal_store(o, reinterpret_cast<us4*>(g.upd.shadow + off));
          }
        } else if (EPI == HDET_EPI_F32 || EPI == HDET_EPI_BIAS_F32) {
          put(reinterpret_cast<f4*>(reinterpret_cast<float*>(g.c) + off), v);
        } else if (EPI == HDET_EPI_BIAS_GELU_BF16) {
          const us4 pre = {f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
          put(reinterpret_cast<us4*>(reinterpret_cast<uint16_t*>(g.c) + off), pre);
          const us4 o = {f2bf(hdet_gelu_tanh_fast(bf2f(pre[0]))), f2bf(hdet_gelu_tanh_fast(bf2f(pre[1]))),
                         f2bf(hdet_gelu_tanh_fast(bf2f(pre[2]))), f2bf(hdet_gelu_tanh_fast(bf2f(pre[3])))};
          put(reinterpret_cast<us4*>(reinterpret_cast<uint16_t*>(g.c2) + off), o);
        } else {
          const us4 o = {f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
          put(reinterpret_cast<us4*>(reinterpret_cast<uint16_t*>(g.c) + off), o);
          if (kColsum) {
#pragma unroll
            for (int q = 0; q < 4; ++q) csum[q] += bf2f(o[q]);
          }
        }
      }
    }
  }
  // Stage 1 of the column sums: a lane has added its rows in ascending order; the RPI lanes that hold the same
  // columns are added by exchanges (a fixed tree), then the wavefronts that share a 128-row block in the order of
  // their rows.  Every (128-row block, column) of C is written by exactly one block of the grid.
  if (kColsum && g.colsum) {
    static_assert(TM % 128 == 0 && TM / WGM <= 128 && 128 % (TM / WGM) == 0, "wavefronts must tile 128-row blocks");
    float* cbuf = reinterpret_cast<float*>(S);         // [WGM * WGN wavefronts][CW columns]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float x = csum[q];
#pragma unroll
      for (int o = LPR; o < 64; o <<= 1) x += __shfl_xor(x, o);
      csum[q] = x;
    }
    __syncthreads();                                   // the strips are no longer in use
    if (lane < LPR) *reinterpret_cast<f4*>(cbuf + wave * CW + lc) = csum;
    __syncthreads();
    constexpr int WPC = 128 / (TM / WGM),              // wavefronts (along m) per 128-row block
                  CHUNKS = TM / 128;
    const int nchunks = (g.m + 127) / 128;
    for (int t = tid; t < CHUNKS * TN; t += THREADS) {
      const int ch = t / TN, cn = t % TN;              // 128-row block of the tile, column of the tile
      float a = 0.f;
#pragma unroll
      for (int u = 0; u < WPC; ++u) a += cbuf[((ch * WPC + u) * WGN + cn / CW) * CW + cn % CW];
      const int chunk = m0 / 128 + ch, c = n0 + cn;
      if (chunk < nchunks && c < g.n) g.colsum[((int64_t)z * nchunks + chunk) * g.n + c] = a;
    }
  }
}

}  // namespace

// Two blocks share a CU when their stages fit twice into the 160 KiB of LDS; the register budget
// follows (second launch-bound argument: wavefronts per SIMD).
template <bool A_KMAJOR, bool B_KMAJOR, int EPI, int TM, int TN, int WGM, int WGN, int NST, int TK, bool STREAM>
__global__ __launch_bounds__(64 * WGM * WGN, 160 * 1024 / (NST * (TM + TN) * TK * 2) * (WGM * WGN / 4))
void hdet_bgemm_dma_kernel(const hdet_bgemm_args g) {
  constexpr int THREADS = 64 * WGM * WGN;
  constexpr int WMT = TM / WGM / 32, WNT = TN / WGN / 32;
  constexpr int STAGE = (TM + TN) * TK;           // elements per stage: A tile then B tile
  __shared__ __attribute__((aligned(1024))) uint16_t S[NST * STAGE];
  typedef lds_tile<A_KMAJOR, TM, THREADS, TK> ta;
  typedef lds_tile<B_KMAJOR, TN, THREADS, TK> tb;
  constexpr int LPT = ta::NI + tb::NI;            // load instructions per thread and stage

  const tile_id id = tile_of_block(g.tile_group);
  const int bx = id.bx, by = id.by, bz = id.bz;
  const hdet_batch_index bi = hdet_split_batch(bz, g.n1, g.n2);
  const int z = bi.z0;            // replica: bias and mask are per replica
  const uint16_t* A = g.a + hdet_batch_offset(bi, g.a_s);
  const uint16_t* B = g.b + hdet_batch_offset(bi, g.b_s);
  const int64_t c_base = hdet_batch_offset(bi, g.c_s);
  const int m0 = by * TM, n0 = bx * TN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / WGN) * (32 * WMT), wn = (wave % WGN) * (32 * WNT);

  // byte extent of each operand for this batch item: the bound that turns absent chunks into zeros
  const uint32_t a_bytes = (uint32_t)(((int64_t)((A_KMAJOR ? g.m : g.k) - 1) * g.lda + (A_KMAJOR ? g.k : g.m)) * 2);
  const uint32_t b_bytes = (uint32_t)(((int64_t)((B_KMAJOR ? g.n : g.k) - 1) * g.ldb + (B_KMAJOR ? g.k : g.n)) * 2);
  const i4 ra = make_rsrc(A, a_bytes), rb = make_rsrc(B, b_bytes);
  const uint32_t s_addr = lds_addr_of(S);

  ta la; tb lb;
  la.init(m0, g.m, g.lda, tid);
  lb.init(n0, g.n, g.ldb, tid);

  constexpr int BLK = kBlock<TK>, SK = block<BLK>::SK, MB = TM / WGM / BLK, NB = TN / WGN / BLK;
  typename block<BLK>::acc acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < BLK * BLK / 64; ++e) acc[i][j][e] = 0.f;

  const int nk = (g.k + TK - 1) / TK;
#define STAGE_PTR(s) (S + (s) * STAGE)
#define STAGE_ADDR(s) (s_addr + (s) * STAGE * 2)
  // K steps 0 .. NST-1 are requested up front; steps past the end load nothing (all chunks absent)
#pragma unroll
  for (int s = 0; s < NST; ++s) {
#pragma unroll
    for (int i = 0; i < ta::NI; ++i) la.issue_one(i, ra, STAGE_ADDR(s), s, g.k, wave);
#pragma unroll
    for (int i = 0; i < tb::NI; ++i) lb.issue_one(i, rb, STAGE_ADDR(s) + TM * TK * 2, s, g.k, wave);
  }
  wait_and_barrier<(NST - 1) * LPT>();

  // Fragments are double-buffered in registers over the NSS = TK / SK MFMA sub-steps of a K step:
  // while the MFMAs of sub-step ss run on fa/fb[ss & 1], the fragments of the next sub-step (of
  // the next stage after the last one) are read into the other set.
  constexpr int NSS = TK / SK, NM = MB * NB, NR = MB + NB;
  constexpr int IPA = (NR + NM - 1) / NM, IPB = (NR + LPT + NM - 1) / NM;
  bf16x8 fa[2][MB], fb[2][NB];
  auto read_frag = [&](bf16x8* a, bf16x8* b, const uint16_t* st, int ks, int idx) {
    // order: a[0], b[0..], a[1..] -- what the first MFMAs of the next sub-step need first
    if (idx == 0) a[0] = ta::fragment(st, wm, ks, lane);
    else if (idx <= NB) b[idx - 1] = tb::fragment(st + TM * TK, wn + (idx - 1) * BLK, ks, lane);
    else if (idx < NR) a[idx - NB] = ta::fragment(st, wm + (idx - NB) * BLK, ks, lane);
  };
  auto multiply = [&](int set, int q) { acc[q / NB][q % NB] = block<BLK>::multiply(fa[set][q / NB], fb[set][q % NB], acc[q / NB][q % NB]); };
#pragma unroll
  for (int idx = 0; idx < NR; ++idx) read_frag(fa[0], fb[0], S, 0, idx);

  for (int kt0 = 0; kt0 < nk; kt0 += NST) {
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      const int kt = kt0 + s;
      if (kt >= nk) break;
      const uint16_t* cur = STAGE_PTR(s);
      const uint16_t* nxt = STAGE_PTR((s + 1) % NST);
#pragma unroll
      for (int ss = 0; ss < NSS - 1; ++ss) {
#pragma unroll
        for (int q = 0; q < NM; ++q) {
          multiply(ss & 1, q);
#pragma unroll
          for (int u = 0; u < IPA; ++u) read_frag(fa[(ss + 1) & 1], fb[(ss + 1) & 1], cur, (ss + 1) * SK, q * IPA + u);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // every wavefront has read all of stage `cur`; stage `nxt` (K step kt + 1) has landed
      wait_and_barrier<(NST - 2) * LPT>();
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        multiply((NSS - 1) & 1, q);
#pragma unroll
        for (int u = 0; u < IPB; ++u) {
          const int it = q * IPB + u;
          if (it < ta::NI) la.issue_one(it, ra, STAGE_ADDR(s), kt + NST, g.k, wave);
          else if (it < LPT) lb.issue_one(it - ta::NI, rb, STAGE_ADDR(s) + TM * TK * 2, kt + NST, g.k, wave);
          else read_frag(fa[0], fb[0], nxt, 0, it - LPT);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
#undef STAGE_PTR
#undef STAGE_ADDR
  // every wavefront is done with the stage buffers (and the loads past the end have drained):
  // they become the staging area of the epilogue
  wait_and_barrier<0>();

  store_tile<EPI, TM, TN, WGM, WGN, BLK, STREAM, NST * STAGE * 2>(g, acc, S, bx, by, z, c_base, tid);
}

namespace {

// A tile of the kernel below: ROWS rows of the output dimension x 64 of the contraction, loaded by 512 threads.
// KMAJOR: LDS [row][64], otherwise [k][ROWS], chunks permuted as in lds_tile.  SPLIT: LDS rows 64 .. 127 are the operand's rows 128 .. 191.
// Rows (KMAJOR) or k (otherwise) past the operand's end lie past its extent as they are; the other edge is masked.  One offset a
// lane: what the loads of a tile differ by is uniform (an offset and a k index for each load, as in lds_tile, spill).
template <bool KMAJOR, int ROWS, bool SPLIT>
struct half_tile {
  static constexpr int NI = ROWS / 64, RCH = ROWS / 8;
  typedef lds_tile<KMAJOR, ROWS, 512, 64> tile;
  uint32_t off;          // byte offset of this lane's first chunk at K step 0, or kAbsent
  __device__ __forceinline__ void init(int row0, int rows, int64_t ld, int tid) {
    if (KMAJOR) off = (uint32_t)(((row0 + (tid >> 3)) * ld + chunk_k(tid)) * 2);
    else {
      const int kk = tid / RCH, r = ((tid % RCH) ^ tile::swz_k(kk)) * 8, row = row0 + (SPLIT ? r + (r & 64) : r);
      off = row < rows ? (uint32_t)((kk * ld + row) * 2) : kAbsent;
    }
  }
  // k index of a thread's chunk inside a K step (KMAJOR)
  static __device__ __forceinline__ int chunk_k(int tid) { return ((tid & 7) ^ tile::swz(tid >> 3)) * 8; }
  // load instruction i: 64 further rows (KMAJOR), 4096 / ROWS further k (otherwise)
  __device__ __forceinline__ void load(int i, i4 rsrc, uint32_t addr, int kt, int64_t ld, bool k_ok, int wave) const {
    const uint32_t step = KMAJOR ? (uint32_t)(kt * 128 + (int64_t)(SPLIT ? 128 * i : 64 * i) * ld * 2) : (uint32_t)((kt * 64 + i * (4096 / ROWS)) * ld * 2);
    lds_load16(rsrc, addr + (i * 512 + wave * 64) * 16, !KMAJOR || k_ok ? off + step : kAbsent);
  }
};

}  // namespace

// The 256 x 256 tile.  What bounds the long products is the power that the chip may draw, then the cycles in which no MFMA runs.
//  * Eight wavefronts of 128 x 64 in two groups of four, one of each group on every SIMD: while one group multiplies (32 MFMAs, 512 cycles), the
//    other reads its next fragments from LDS and requests a later stage; the block's barriers hand the matrix cores from one to the other, and
//    s_setprio keeps the reading wavefront from delaying the multiplying one.  A K step of 64 is two such turns: rows 0-63 of the wavefront
//    with all of its columns, then rows 64-127 with the column fragments still in registers.
//  * Two stages of 64 KiB.  The half of A that the first turn reads, and B, are free for K step kt + 2 from the second turn of kt on, the other half
//    from the first turn of kt + 1 on, so every load has five or six turns (2500-3000 cycles) to land and each turn waits for all
//    but the newest eight of the wavefront's loads.  A turn's LDS reads are complete before its first barrier, which is what lets the other
//    group (one turn behind) and this one request into what they read.
// Per replica 8192 x 1024, K = 4096, 8 replicas: input gradients 454 -> 391 us (1.41 PFLOP/s), with bias and residual 472 -> 412; weight gradients
// 4096 x 1024, K = 8192: 439 -> 390 (all eight wavefronts in step before, as in the kernel above: matrix cores busy 59 % of the cycles at
// 1.94 GHz, now 70 % at 1.9; the weight gradients 69 % at 1.76 and 73 % at 1.87).  Measured and not kept: loads requested between the MFMAs with the
// barrier's wait on LDS left out, 1-6 % slower; handing over 2 or 4 MFMAs before the end of a turn, 8-12 % slower; 256 x 128 tiles
// in three stages, 5 % faster than kLong on long products and no faster where the weights are streamed.
template <bool A_KMAJOR, bool B_KMAJOR, int EPI, bool STREAM>
__global__ __launch_bounds__(512, 2) void hdet_bgemm_alt_kernel(const hdet_bgemm_args g) {
  constexpr int TM = 256, TN = 256, TK = 64, HALF = 128 * TK, WGM = 2, WGN = 4, MB = TM / WGM / 16;
  __shared__ __attribute__((aligned(1024))) uint16_t S[8 * HALF];
  typedef half_tile<A_KMAJOR, 128, true> ta;
  typedef half_tile<B_KMAJOR, TN, false> tb;
  const tile_id id = tile_of_block(g.tile_group);
  const hdet_batch_index bi = hdet_split_batch(id.bz, g.n1, g.n2);
  const uint16_t* A = g.a + hdet_batch_offset(bi, g.a_s);
  const uint16_t* B = g.b + hdet_batch_offset(bi, g.b_s);
  const int64_t c_base = hdet_batch_offset(bi, g.c_s);
  const int m0 = id.by * TM, n0 = id.bx * TN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = (wave % WGN) * 64, hr = (wave / WGN) * 64;
  const uint32_t a_bytes = (uint32_t)(((int64_t)((A_KMAJOR ? g.m : g.k) - 1) * g.lda + (A_KMAJOR ? g.k : g.m)) * 2);
  const uint32_t b_bytes = (uint32_t)(((int64_t)((B_KMAJOR ? g.n : g.k) - 1) * g.ldb + (B_KMAJOR ? g.k : g.n)) * 2);
  const i4 ra = make_rsrc(A, a_bytes), rb = make_rsrc(B, b_bytes);
  const uint32_t s_addr = lds_addr_of(S);

  ta la[2]; tb lb;
  la[0].init(m0, g.m, g.lda, tid);
  la[1].init(m0 + 64, g.m, g.lda, tid);
  lb.init(n0, g.n, g.ldb, tid);
  const int ck = ta::chunk_k(tid);

  f4 acc[MB][4];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  // LDS, in units of 128 rows x 64: half h of A of stage s at 2 h + s, B at 4 + 2 s
  const int nk = (g.k + TK - 1) / TK;
  auto load_a = [&](int h, int s, int kt) {
    const uint32_t at = s_addr + (2 * h + s) * HALF * 2;
#pragma unroll
    for (int i = 0; i < ta::NI; ++i) la[h].load(i, ra, at, kt, g.lda, ck + kt * TK < g.k, wave);
  };
  auto load_b = [&](int s, int kt) {
    const uint32_t at = s_addr + (4 + 2 * s) * HALF * 2;
#pragma unroll
    for (int i = 0; i < tb::NI; ++i) lb.load(i, rb, at, kt, g.ldb, ck + kt * TK < g.k, wave);
  };
  bf16x8 fa[2][4], fb[2][4];
  auto read_a = [&](int h, int s) {
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[ss][i] = ta::tile::fragment(S + (2 * h + s) * HALF, hr + i * 16, ss * 32, lane);
  };
  auto read_b = [&](int s) {
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[ss][j] = tb::tile::fragment(S + (4 + 2 * s) * HALF, wn + j * 16, ss * 32, lane);
  };
  auto multiply = [&](int h) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[4 * h + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ss][j], fa[ss][i], acc[4 * h + i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto meet = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  load_a(0, 0, 0); load_b(0, 0); load_a(1, 0, 0);
  load_a(0, 1, 1); load_b(1, 1);
  wait_and_barrier<8>();
  if (wave >= 4) meet();
  for (int kt0 = 0; kt0 < nk; kt0 += 2) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int kt = kt0 + s;
      if (kt >= nk) break;
      read_a(0, s);
      read_b(s);
      load_a(1, s ^ 1, kt + 1);
      wait_and_barrier<8>();
      multiply(0);
      meet();
      read_a(1, s);
      load_a(0, s, kt + 2);
      load_b(s, kt + 2);
      wait_and_barrier<8>();
      multiply(1);
      meet();
    }
  }
  if (wave < 4) meet();
  wait_and_barrier<0>();
  store_tile<EPI, TM, TN, WGM, WGN, 16, STREAM, 8 * HALF * 2>(g, acc, S, id.bx, id.by, bi.z0, c_base, tid);
}

// Forward products whose blocks walk over tiles of 256 x 256: the main loop of the kernel above, with the next tile's first two K steps requested in
// the last two of the tile before, so that the pipeline never drains, and a tile's end in registers alone, under the loads in flight.
//  * The bias (in LDS, requested a tile ahead) is added to the finished sums, as the other kernels do: the same bits.  As what the first MFMAs add to
//    it cost no addition, but every partial sum was rounded at its size.
//  * Results change places between the four groups of 16 lanes (v_permlane32_swap, v_permlane16_swap) until a lane has 16 consecutive columns
//    of its row: two 16-byte stores, no LDS.
//  * Stores count in vmcnt with the loads: they are always issued (rows and columns that do not exist lie outside the descriptor), and the first
//    K step of the next tile waits for the loads before them, not for them (kStores).
//  * The group that is a turn behind ends its tile as soon as its products are done, beside the other group, not after it.
//  * Exponentials of logits are exp2(z log2(e) - r), one fused operation and the hardware's exp2, with r the whole number next to max log2(e): what tiles
//    and rows refer to differs by exact powers of two, and nothing that is rounded once for the maximum fails to cancel between the sums and the
//    gradient.  Simulated against 64 bits, logits of size 0.5 to 30, 1000 to 16000 classes: probabilities off by 3e-8 to 1.1e-7 (rms, relative), those of the
//    loss kernels (hdet_mlp.hip) by 4e-8 to 3.6e-7; row losses by 0.6 to 1.0 times as much as theirs.  With r = max log2(e) rounded, a tile's own for its
//    sum and the row's for the gradient, 1.0e-7 to 7e-7, and 2e-5 where the maxima of several tiles lie next to each other at 300.
// Built for the output layer with its loss (hdet_launch_head_loss; products with a bias take it too, launch_shape), whose two passes cost less than writing and reading fp32 logits:  K = 512,
// 4096 x 32000, 8 replicas, 1502 to 1575 us of product and 1152 of loss kernel -> 948 (statistics) + 19 (merge) + 1205 (gradient) in a training step
// (cards differ by up to 10 % in these).  Of a tile's 15 and 19 us the main loop takes 11 (1.6 PFLOP/s, 70 % of the matrix cores' cycles), exponentials
// 3.4, stores 3.5.  Not kept, gradient pass, beside 1190 on one card: results through LDS 1216 (rows of bf16), past the L2 1358 (pieces of 16 bytes), both
// groups' ends in turn 1240; the kernel above with these epilogues 1019 and 1400.
template <int EPI>
__global__ __launch_bounds__(512, 2) void hdet_bgemm_walk_kernel(const hdet_bgemm_args g, unsigned gx, unsigned gy, unsigned total) {
  constexpr int TM = 256, TN = 256, TK = 64, HALF = 128 * TK;
  constexpr bool kStat = EPI == HDET_EPI_XENT_STAT, kGrad = EPI == HDET_EPI_XENT_GRAD;
  constexpr int kStores = kStat ? 0 : 16;
  constexpr int kBiasAt = 8 * HALF * 2, kRowsAt = kBiasAt + 2 * TN * 4;           // bytes: bias [2][TN], then what the epilogue needs
  constexpr int kExtra = 2 * TN * 4 + (kStat ? 4 * TM * 8 : kGrad ? 3 * TM * 4 : 0);
  __shared__ __attribute__((aligned(1024))) uint16_t S[8 * HALF + kExtra / 2];
  typedef lds_tile<true, 128, 512, TK> ta;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = (wave % 4) * 64, hr = (wave / 4) * 64, wm = (wave / 4) * 128;
  // what a lane derives from its number outside the K loop is computed where it is used, the number itself too: kept over the tiles it would spill
  auto lane_now = [] {
    int x;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
    return x;
  };
  const uint32_t s_addr = lds_addr_of(S);
  float* const s_bias = reinterpret_cast<float*>(S) + kBiasAt / 4;
  float* const s_rows = reinterpret_cast<float*>(S) + kRowsAt / 4;
  const int nk = ((g.k + TK - 1) / TK + 1) & ~1;                 // K steps of a tile, an even number (steps beyond K are zeros)

  struct tile { int m0, n0, bx, z; i4 ra, rb, rbias; };
  auto tile_at = [&](unsigned t) {
    tile r;
    const tile_id id = tile_of_index(t < total ? t : total - 1, gx, gy, total, g.tile_group);
    r.m0 = id.by * TM; r.n0 = id.bx * TN; r.bx = id.bx; r.z = id.bz;
    const bool ok = t < total;
    r.ra = make_rsrc(g.a + id.bz * g.a_s[0] + (int64_t)r.m0 * g.lda, ok ? (uint32_t)(((int64_t)(g.m - r.m0 - 1) * g.lda + g.k) * 2) : 0u);
    r.rb = make_rsrc(g.b + id.bz * g.b_s[0] + (int64_t)r.n0 * g.ldb, ok ? (uint32_t)(((int64_t)(g.n - r.n0 - 1) * g.ldb + g.k) * 2) : 0u);
    r.rbias = make_rsrc(g.bias + id.bz * g.bias_bs + r.n0, ok ? (uint32_t)(g.n - r.n0) * 4u : 0u);
    return r;
  };
  const int ck = ((tid & 7) ^ ta::swz(tid >> 3)) * 8;            // k of this thread's chunks inside a K step
  uint32_t off_a = (uint32_t)(((tid >> 3) * g.lda + ck) * 2), off_b = (uint32_t)(((tid >> 3) * g.ldb + ck) * 2);
  // LDS, in units of 128 rows x 64: half h of A of stage s at 2 h + s (its rows 64 .. 127 are the tile's 128 .. 191 of that half), B at 4 + 2 s
  auto load_a = [&](const i4& r, int h, int s, int kt) {
    const uint32_t at = s_addr + (2 * h + s) * HALF * 2;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      lds_load16(r, at + (i * 512 + wave * 64) * 16, ck + kt * TK < g.k ? off_a + (uint32_t)(kt * 128 + (64 * h + 128 * i) * g.lda * 2) : kAbsent);
  };
  auto load_b = [&](const i4& r, int s, int kt) {
    const uint32_t at = s_addr + (4 + 2 * s) * HALF * 2;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      lds_load16(r, at + (i * 512 + wave * 64) * 16, ck + kt * TK < g.k ? off_b + (uint32_t)(kt * 128 + 64 * i * g.ldb * 2) : kAbsent);
  };
  auto load_bias = [&](const tile& t, int slot) {
    if (wave < 4) lds_load4(t.rbias, s_addr + kBiasAt + slot * TN * 4 + wave * 256, (uint32_t)(wave * 64 + lane_now()) * 4u);
  };
  auto load_rows = [&](const tile& t) {                          // reference, factor and label of the tile's rows
    const int ln = lane_now();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int q = wave + 8 * u, row = t.m0 + (q & 3) * 64 + ln;
      if (q < 12) {
        const void* src = q < 4 ? (const void*)g.xent.row_ref : q < 8 ? (const void*)g.xent.row_a : (const void*)g.xent.labels;
        lds_load4(make_rsrc((const float*)src + (int64_t)t.z * g.m, (uint32_t)g.m * 4u), s_addr + kRowsAt + q * 256, row < g.m ? (uint32_t)row * 4u : kAbsent);
      }
    }
  };
  f4 acc[8][4];
  bf16x8 fa[2][4], fb[2][4];
  // fragment i of sub-step ss is 16 i rows behind fragment 0, whose chunk permutation it shares: two addresses an operand
  const uint16_t *pa[2], *pb[2];
#pragma unroll
  for (int ss = 0; ss < 2; ++ss) {
    const int at = (lane & 15) * TK + (((ss * 4 + (lane >> 4)) ^ ta::swz(lane & 15)) << 3);
    pa[ss] = S + hr * TK + at;
    pb[ss] = S + 4 * HALF + wn * TK + at;
  }
  auto read_a = [&](int h, int s) {
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[ss][i] = *reinterpret_cast<const bf16x8*>(pa[ss] + (2 * h + s) * HALF + i * 16 * TK);
  };
  auto read_b = [&](int s) {
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[ss][j] = *reinterpret_cast<const bf16x8*>(pb[ss] + 2 * s * HALF + j * 16 * TK);
  };
  auto multiply = [&](int h, bool first) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[4 * h + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ss][j], fa[ss][i], first && ss == 0 ? f4{0.f, 0.f, 0.f, 0.f} : acc[4 * h + i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto meet = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // a group's four wavefronts have left reference and sum of their 64 columns for the group's 128 rows; 32 rows each
  auto put_stats = [&](const auto& t) {
    const int ln = lane_now(), tr = wm + (wave % 4) * 32 + (ln & 31);
    const float2* buf = reinterpret_cast<const float2*>(s_rows) + tr;
    float2 p[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) p[w] = buf[w * TM];
    const float mx = fmaxf(fmaxf(p[0].x, p[1].x), fmaxf(p[2].x, p[3].x));
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += p[w].x == -INFINITY ? p[w].y : p[w].y * __builtin_amdgcn_exp2f(p[w].x - mx);
    if (ln < 32 && t.m0 + tr < g.m) g.xent.part[((int64_t)t.z * gx + t.bx) * g.m + t.m0 + tr] = float2{mx, s};
  };
  auto finish = [&](const tile& t, int slot) {
    __builtin_amdgcn_sched_barrier(0);
    const int ln = lane_now(), cg = ln >> 4, lr = ln & 15;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f4 bias = *reinterpret_cast<const f4*>(s_bias + slot * TN + wn + j * 16 + cg * 4);
      if (kStat && t.n0 + wn + j * 16 + cg * 4 >= g.n) bias = f4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i][j] += bias;
    }
    if constexpr (kStat) {
      float mx[8], sum[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        mx[i] = acc[i][0][0];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) mx[i] = fmaxf(mx[i], acc[i][j][e]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) mx[i] = over_groups(mx[i], [](float x, float y) { return fmaxf(x, y); });
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        mx[i] = rintf(mx[i] * kLog2e);
        const float ml = mx[i] == -INFINITY ? 0.f : mx[i];
        sum[i] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[i] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][e], kLog2e, -ml));
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) sum[i] = over_groups(sum[i], [](float x, float y) { return x + y; });
      if (ln < 16) {
#pragma unroll
        for (int i = 0; i < 8; ++i) reinterpret_cast<float2*>(s_rows)[(wave % 4) * TM + wm + i * 16 + ln] = float2{mx[i], sum[i]};
      }
    } else {
      const auto rc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint16_t*>(g.c) + t.z * g.c_s[0] + (int64_t)t.m0 * g.ldc + t.n0, 0, 0x7fffffff, 0x00020000);
      const int col = wn + cg * 16;
      const bool ok0 = t.n0 + col < g.n, ok1 = t.n0 + col + 8 < g.n;
      f4 csum[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) csum[j] = f4{0.f, 0.f, 0.f, 0.f};
      float rref[8], ra[8];
      int rlab[8];
      if (kGrad) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int tr = wm + i * 16 + lr;
          rref[i] = s_rows[tr]; ra[i] = s_rows[TM + tr]; rlab[i] = __float_as_int(s_rows[2 * TM + tr]);
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int tr = wm + i * 16 + lr;
        const bool row_ok = t.m0 + tr < g.m;
        f4 v[4];
        if constexpr (kGrad) {
          const float ref = row_ok ? rref[i] : INFINITY, a = ra[i];
          const int yc = row_ok ? rlab[i] - (t.n0 + wn + cg * 4) : -1;
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[j][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][e], kLog2e, -ref)) * a;
          if (__builtin_expect((unsigned)yc < 64u && (yc & 12) == 0, 0)) {      // the row's label is among this lane's columns
            float zy = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (yc == j * 16 + e) { zy = acc[i][j][e]; v[j][e] -= g.xent.invb; }
            const int64_t at = (int64_t)t.z * g.m + t.m0 + tr;
            g.xent.row_loss[at] = (float)((g.xent.row_lse[at] - (double)zy * (double)kLog2e) * kLn2);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) csum[j] += v[j];
        }
        if constexpr (!kGrad) {
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = acc[i][j];
        }
        unsigned d[4][2];
#pragma unroll
        for (int j = 0; j < 4; ++j) { d[j][0] = hdet_bf16_pack(v[j][0], v[j][1]); d[j][1] = hdet_bf16_pack(v[j][2], v[j][3]); }
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          swap32(d[0][w], d[2][w]); swap32(d[1][w], d[3][w]);
          swap16(d[0][w], d[1][w]); swap16(d[2][w], d[3][w]);
        }
        const uint32_t at = (uint32_t)((tr * (int)g.ldc + col) * 2);
        __builtin_amdgcn_raw_buffer_store_b128(hdet_u4v{d[0][0], d[0][1], d[1][0], d[1][1]}, rc, row_ok && ok0 ? at : kAbsent, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(hdet_u4v{d[2][0], d[2][1], d[3][0], d[3][1]}, rc, row_ok && ok1 ? at + 16 : kAbsent, 0, 0);
      }
      if (kGrad && g.colsum) {                                   // a wavefront's 128 rows are one chunk of the column sums
        f4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float x = csum[j][e];
            x += hdet_dpp<0xB1>(x);
            x += hdet_dpp<0x4E>(x);
            x += hdet_dpp<0x141>(x);
            x += hdet_dpp<0x140>(x);
            if (lr == j) out[e] = x;
          }
        const int nchunks = (g.m + 127) / 128, chunk = (t.m0 + wm) / 128, c = t.n0 + wn + lr * 16 + cg * 4;
        if (lr < 4 && chunk < nchunks && c < g.n) *reinterpret_cast<f4*>(g.colsum + ((int64_t)t.z * nchunks + chunk) * g.n + c) = out;
      }
    }
  };

  unsigned t = blockIdx.x;
  tile cur = tile_at(t);
  struct { int m0, bx, z; } prev = {0, 0, 0};
  int slot = 0;
  load_bias(cur, 0);
  load_a(cur.ra, 0, 0, 0); load_b(cur.rb, 0, 0); load_a(cur.ra, 1, 0, 0);
  load_a(cur.ra, 0, 1, 1); load_b(cur.rb, 1, 1);
  wait_and_barrier<8>();
  if (wave >= 4) meet();
  for (bool begun = false;; begun = true) {
    tile nxt;
    asm volatile("" : "+v"(off_a), "+v"(off_b));
    auto pair = [&](int kt0, bool first) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int kt = kt0 + s;
        const bool fs = first && s == 0;
        auto wait = [&] {
          if (kStores && fs && begun) wait_and_barrier<8 + kStores>();
          else wait_and_barrier<8>();
        };
        read_a(0, s);
        read_b(s);
        if (first || kt + 1 < nk) load_a(cur.ra, 1, s ^ 1, kt + 1); else load_a(nxt.ra, 1, s ^ 1, 0);
        wait();
        multiply(0, fs);
        meet();
        read_a(1, s);
        if (first || kt + 2 < nk) { load_a(cur.ra, 0, s, kt + 2); load_b(cur.rb, s, kt + 2); }
        else { load_a(nxt.ra, 0, s, kt + 2 - nk); load_b(nxt.rb, s, kt + 2 - nk); }
        if (first && s == 0) {                                   // under the other group's products
          t += gridDim.x;
          nxt = tile_at(t);
          if (kStat && begun) put_stats(prev);
        }
        if (first && s == 1) {
          load_bias(nxt, slot ^ 1);
          if (kGrad) load_rows(cur);
        }
        wait();
        multiply(1, fs);
        if (s == 0) meet();
      }
    };
    pair(0, true);
    for (int kt0 = 2; kt0 < nk; kt0 += 2) { meet(); pair(kt0, false); }
    // the first group ends its tile under the second's last products, the second at once, not when the first is done
    if (wave < 4) meet();
    finish(cur, slot);
    if (wave >= 4) meet();
    if (t >= total) break;
    prev = {cur.m0, cur.bx, cur.z};
    cur = nxt;
    slot ^= 1;
  }
  if (wave < 4) meet();
  wait_and_barrier<0>();
  if (kStat) put_stats(cur);
}

// The rows' reference and sum from the column tiles' (hdet_launch_head_loss).  Block = 64 rows x 4 phases; phase q takes tiles q, q + 4, ..., the
// phases are added in their order.  References are whole numbers, so that a tile's sum comes to the row's by an exact power of two, and the sum over a
// hundred tiles is in 64 bits.  A label that names no class has no column that would write the row's loss: it counts as a logit of 0.
__global__ __launch_bounds__(256) void hdet_head_rows_kernel(const hdet_xent_epi x, int m, int classes) {
  __shared__ float ref[4][64];
  __shared__ double part[4][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6, z = blockIdx.y, row = blockIdx.x * 64 + lane, tiles = (classes + 255) / 256;
  float mx = -INFINITY;
  double s = 0.0;
  if (row < m) {
    const float2* p = x.part + (int64_t)z * tiles * m + row;
#pragma unroll 8
    for (int t = q; t < tiles; t += 4) {
      const float2 v = p[(int64_t)t * m];
      const float mn = fmaxf(mx, v.x);
      if (v.x != -INFINITY) s = s * (double)__builtin_amdgcn_exp2f(mx - mn) + (double)(v.y * __builtin_amdgcn_exp2f(v.x - mn));
      else s += v.y;
      mx = mn;
    }
  }
  ref[q][lane] = mx;
  part[q][lane] = s;
  __syncthreads();
  if (q == 0 && row < m) {
    float r[4];
    double p[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) { r[w] = ref[w][lane]; p[w] = part[w][lane]; }
    const float top = fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]));
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) sum += r[w] == -INFINITY && p[w] == 0.0 && top != -INFINITY ? 0.0 : p[w] * (double)__builtin_amdgcn_exp2f(r[w] - top);
    const int64_t at = (int64_t)z * m + row;
    x.row_ref[at] = top;
    x.row_a[at] = (float)((double)x.invb / sum);
    const double lse = (double)top + log2(sum);
    x.row_lse[at] = lse;
    if ((unsigned)x.labels[at] >= (unsigned)classes) x.row_loss[at] = (float)(lse * kLn2);
  }
}

namespace {

bool chunk_regular(const void* base, int64_t ld, const int64_t* bs, int chunk_extent) {
  return (ld & 7) == 0 && ((bs[0] | bs[1] | bs[2]) & 7) == 0 && (chunk_extent & 7) == 0 &&
         (reinterpret_cast<uintptr_t>(base) & 15) == 0;
}

// compute units of the current device (queried once per device; 256 on MI355X)
int compute_units() { return hdet_compute_units(); }

}  // namespace

int hdet_compute_units() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    cached[dev] = (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) ? n : 256;
  }
  return cached[dev];
}

namespace {

// Whether a launch writes its results past the L2, where they would push out the operand tiles that the blocks of an XCD share.
// That wins while the rows are whole 128-byte lines, also where the next kernel reads the result at once.  Rows that begin inside
// a line leave partial lines on either side of every tile, which the L2 puts together and the memory does not: such results go
// through the L2 unless the product is long enough, by epilogue, to hide that.  us, past / through (M = 4096, 8 items; pitch mod 128):
//   whole lines: logits 4096 wide K = 128 100 / 127, K = 512 178 / 211, 30016 wide K = 64 714 / 817;  both GELU outputs K = 512,
//                4 items 98 / 109;  ReLU 4096 wide K = 256 109 / 132;  2048 x 2048 weight gradients K = 512 43 / 45, K = 64 27 / 25
//   half lines (64): logits 30000 wide K = 256 956 / 1207, 10000 wide K = 64 292 / 260;  weight gradients K = 64 31 / 26, K = 1024 93 / 91
//   others: logits 5000 wide (32) K = 64 207 / 143, K = 256 213 / 201, K = 1024 362 / 375, 29996 wide K = 128 1477 / 1113;
//           both GELU outputs 2056 wide (16) K = 64 154 / 71, K = 512 150 / 127, 6168 wide K = 2048 843 / 918;
//           input gradient 2056 wide K = 256 70 / 62, K = 1024 155 / 148;  weight gradients 2056 wide K = 256 49 / 37;
//           bias 6168 wide (48) K = 128 188 / 151, K = 512 259 / 264, 2056 wide K = 512 104 / 96;  ReLU 4104 wide K = 128 104 / 112;
//           ReLU gate 2056 wide K = 128 79 / 79, K = 512 106 / 131;  residual 2056 wide K = 512 117 / 133, 1000 wide K = 256 46 / 39;
//           GELU gradient 2056 wide K = 64 83 / 87, K = 512 122 / 146
// (the update epilogue writes no result)
template <int EPI> constexpr bool kAlwaysStream = EPI == HDET_EPI_ADAMW || EPI == HDET_EPI_GELUGRAD_BF16;
bool stream_result(const hdet_bgemm_args& g, int epi, int batch) {
  const int64_t size = epi == HDET_EPI_F32 || epi == HDET_EPI_BIAS_F32 ? 4 : 2;
  const uint64_t part = (reinterpret_cast<uintptr_t>(g.c) | (uint64_t)((g.ldc | g.c_s[0] | g.c_s[1] | g.c_s[2]) * size)) & 127;
  if (part == 0) return true;
  if (part == 64 && epi != HDET_EPI_F32) return epi != HDET_EPI_BIAS_F32 || g.k >= 128;
  const bool large = (int64_t)batch * g.m * g.n * size > (int64_t)256 << 20;       // more than the memory-side cache holds
  switch (epi) {
    case HDET_EPI_MASK_BF16: return g.k >= 256;
    case HDET_EPI_BIAS_RESID_BF16: case HDET_EPI_BIAS_DROP_RESID_BF16: return g.k >= 512;
    case HDET_EPI_BIAS_F32: return large && g.k >= 512;
    case HDET_EPI_BIAS_RELU_BF16: return large && g.k >= 128;
    case HDET_EPI_BIAS_BF16: return large && g.k >= 256;
    case HDET_EPI_BIAS_GELU_BF16: case HDET_EPI_BF16: return large && g.k >= 2048;
  }
  return false;
}

// Which tile a product takes: the one whose time by
//   base + rounds (epi share + slope K / 1000)  us,     rounds = ceil(tiles / CUs) / (blocks per CU), at least `least`
// is the lowest.  `epi` is what the epilogue of a 256 x 256 tile takes where nothing hides it; a smaller tile takes `share` of it, less where a
// second block of the CU multiplies meanwhile.  The constants come from sweeps of every tile over 18 grids of 72 to 1536 tiles of
// 256 x 256, K = 64 .. 4096, with ten epilogues, the operands cold (another gigabyte of them each launch: with warm ones the smaller tiles, which
// read their operands more often, look 10 to 30 % better than they are in a training step).  Against the fastest tile of each product in that
// range this choice loses 0.2 to 1 % on average by epilogue, 21 % at most (384 tiles at K = 1024 with both GELU outputs); lines by K and tile
// count lost up to 34 %.  The alternating kernel is left out below K = 512 (1024 for weight gradients, 2048 for the GELU gradient, whose
// epilogue takes as long as 1024 of K: 719 against 690 us for 8192 x 4096 x 8 in a step), where the model flatters it; but see long_logits.
struct tile_shape { int tm, tn, per_cu; float base, share, slope, least; };
constexpr tile_shape kAlternating = {256, 256, 1, 1.6f, 1.f, 19.f, 1.f};       // hdet_bgemm_alt_kernel
constexpr tile_shape kPair = {256, 128, 2, 3.6f, 0.53f, 32.f, 0.52f};          // K step 32, three stages, two blocks a CU
constexpr tile_shape kPairWgrad = {256, 128, 2, 3.6f, 0.53f, 27.3f, 0.52f};
constexpr tile_shape kLong = {256, 128, 1, 2.35f, 0.51f, 13.6f, 1.f};          // K step 64, three stages
constexpr tile_shape kSmall = {128, 128, 2, 3.1f, 0.44f, 18.1f, 0.8f};         // K step 64, two stages, two blocks a CU
// Up to one 128 x 128 tile a CU (below the sweeps' range) nothing but the length of a block's own chain counts: such tiles, from K = 512 on with
// four stages of K = 64 in flight instead of two, whose longer start costs 1 us.  us, four stages / two / what the cost would choose, operands cold:
//   32 x 1024, K = 2048, 4 items, ReLU gate at K = 1024 14.7 / 17.0 / 17.7;  64 x 512, K = 4096, 3 items 38.6 / 54.1 / 48.4;
//   96 x 704, K = 1504, 6 items 25.0 / 30.3 / 26.8;  200 x 1000, K = 3000, 2 items 42.8 / 51.6 / 61.2;  96 x 1504, K = 784 19.0 / 19.5 / 19.8;
//   32 x 2048, K = 512, 4 items 10.1 / 11.6 / 12.2;  128 x 1024, K = 256, 8 items 10.1 / 9.3 / 9.9;  gradients of K = 32 to 256 7 to 15 % slower
constexpr tile_shape kDeep = {128, 128, 1, 0.f, 0.f, 0.f, 0.f};                // K step 64, four stages
template <int EPI> constexpr float kEpiTime =
    EPI == HDET_EPI_ADAMW ? 80.f : EPI == HDET_EPI_GELUGRAD_BF16 || EPI == HDET_EPI_BIAS_DROP_RESID_BF16 ? 20.f
    : EPI == HDET_EPI_MASK_BF16 || EPI == HDET_EPI_BIAS_RESID_BF16 || EPI == HDET_EPI_BIAS_GELU_BF16 ? 15.f
    : EPI == HDET_EPI_F32 || EPI == HDET_EPI_BIAS_F32 ? 12.f : EPI == HDET_EPI_BIAS_RELU_BF16 ? 9.f : 8.f;

// What hdet_bgemm_walk_kernel asks for beyond the LDS-direct kernels: whole groups of 8 columns, results and their rows 16-byte aligned, four K steps
bool walkable(const hdet_bgemm_args& g) {
  return g.n1 * g.n2 == 1 && g.k >= 192 && (g.n & 7) == 0 && ((g.ldc | g.c_s[0]) & 7) == 0 &&
         (reinterpret_cast<uintptr_t>(g.c) & 15) == 0 && g.ldc < 1 << 22 && g.m < 1 << 28 &&
         ((int64_t)g.m + 256) * g.lda * 2 < (int64_t)1 << 31 && ((int64_t)g.n + 256) * g.ldb * 2 < (int64_t)1 << 31;
}
int tile_group_of(unsigned columns) { return columns >= 64 ? 4 : columns >= 12 ? 2 : 1; }
template <int EPI>
void launch_walk(hdet_bgemm_args g, int batch, hipStream_t s) {
  const unsigned gx = (g.n + 255) / 256, gy = (g.m + 255) / 256, total = gx * gy * (unsigned)batch, cus = (unsigned)compute_units();
  g.tile_group = tile_group_of(gx);
  hipLaunchKernelGGL(hdet_bgemm_walk_kernel<EPI>, dim3(total < cus ? total : cus), dim3(512), 0, s, g, gx, gy, total);
}

template <bool AK, bool BK, int EPI>
hipError_t launch_shape(const hdet_bgemm_args& g, int batch, hipStream_t s) {
  constexpr bool wgrad = !AK && !BK, update = EPI == HDET_EPI_ADAMW;
  const int cus = compute_units();
  const float epi = kEpiTime<EPI>;
  auto time_of = [&](const tile_shape& t, float more_k = 0.f) {
    const int64_t tiles = (int64_t)((g.m + t.tm - 1) / t.tm) * ((g.n + t.tn - 1) / t.tn) * batch;
    const float rounds = (float)((tiles + cus - 1) / cus) / t.per_cu;
    return t.base + (rounds > t.least ? rounds : t.least) * (epi * t.share + t.slope * 1e-3f * (g.k + more_k));
  };
  // the alternating kernel leaves the far edge of its tiles to the bounds of the buffer: no offset of a tile may wrap
  const int64_t a_ext = ((int64_t)(AK ? g.m : g.k) + 256) * g.lda * 2, b_ext = ((int64_t)(BK ? g.n : g.k) + 256) * g.ldb * 2;
  const bool fits = a_ext < (int64_t)1 << 31 && b_ext < (int64_t)1 << 31;
  const bool alternating = g.k >= (update ? 1 : EPI == HDET_EPI_GELUGRAD_BF16 ? 2048 : wgrad ? 1024 : 512) && fits;
  // Weight gradients in it take longer beyond K = 4096 than the sweeps up to there say: between one round of 256 x 256 tiles and one and a half,
  // the pair tiles stay the faster ones.  us in a step, alternating / pair:  3072 x 1024, K = 8192, 6, 7, 8 items (288, 336, 384 tiles) 350 / 319,
  // 364 / 337, 413 / 375;  8 items, K = 6144 297 / 279, K = 12288 536 / 518;  2304 x 2048, K = 8192, 4 items (288) 336 / 307;  6144 x 2048,
  // K = 6144, 2 items (384) 277 / 257.  With every K beyond 4096 counted 1.2 times the line lies there.
  const float t_alt = alternating ? time_of(kAlternating, wgrad && !update && g.k > 4096 ? 0.2f * (g.k - 4096) : 0.f) : 3e38f;
  // Forward products with fp32 results of three rounds of 256 x 256 tiles and more, from K = 384 on: there the pair tiles fall 20 to 30 % behind their
  // cost, and the last round counts for less than a whole one.  us, alternating / pair: 8192 x 2048, 4 items, K = 256 68 / 62, K = 384 81 / 99,
  // K = 448 84 / 111;  12410 x 1296, 7 items (8.04 rounds), K = 256 128 / 115, K = 384 152 / 192, K = 640 212 / 259, K = 768 221 / 289;
  // 9064 x 3776, 7 items, K = 384 252 / 247, K = 448 276 / 287.  (With ReLU, K = 384: 8192 x 1600, 4 items 65 / 57.)
  const bool long_logits = AK && BK && (EPI == HDET_EPI_F32 || EPI == HDET_EPI_BIAS_F32) && g.k >= 384 && fits &&
                           (int64_t)((g.m + 255) / 256) * ((g.n + 255) / 256) * batch >= 3 * (int64_t)cus;
  const bool stream = kAlwaysStream<EPI> || stream_result(g, EPI, batch);
  auto launch = [&](auto kernel, const tile_shape& t, int threads) {
    const dim3 grid((g.n + t.tn - 1) / t.tn, (g.m + t.tm - 1) / t.tm, batch);
    hdet_bgemm_args ga = g;
    // Tile order inside a batch item: with many tile columns, the 32 blocks an XCD runs at a time would share one
    // operand tile of A and none of B; walking groups of 4 (2) tile rows column by column cuts the operand bytes its L2
    // has to fetch by up to two thirds (head product of the transformer, 125 tile columns: 1505 us row by row, 1346 in groups of 4).
    // Updates go row by row: what they stream is theta and the moments (4096 x 4096 x 8, K = 256: 638 us, 668 in groups of 2).
    ga.tile_group = update ? 1 : tile_group_of(grid.x);
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, ga);
  };
#define HDET_TILE(SHAPE, THREADS, KERNEL, ...)                                                        \
  do {                                                                                                \
    if (stream) launch(&KERNEL<AK, BK, EPI, __VA_ARGS__ true>, SHAPE, THREADS);                       \
    else if constexpr (!kAlwaysStream<EPI>) launch(&KERNEL<AK, BK, EPI, __VA_ARGS__ false>, SHAPE, THREADS); \
  } while (0)
  if constexpr (update) {
    if (t_alt <= time_of(kSmall)) HDET_TILE(kAlternating, 512, hdet_bgemm_alt_kernel, );
    else HDET_TILE(kSmall, 256, hdet_bgemm_dma_kernel, 128, 128, 2, 2, 2, 64,);
  } else {
    const float t_pair = time_of(wgrad ? kPairWgrad : kPair), t_small = time_of(kSmall), t_long = time_of(kLong);
    if ((int64_t)((g.m + 127) / 128) * ((g.n + 127) / 128) * batch <= cus) {
      if (g.k >= 512) HDET_TILE(kDeep, 256, hdet_bgemm_dma_kernel, 128, 128, 2, 2, 4, 64,);
      else HDET_TILE(kSmall, 256, hdet_bgemm_dma_kernel, 128, 128, 2, 2, 2, 64,);
    }
    else if (long_logits || (t_alt <= t_pair && t_alt <= t_small && t_alt <= t_long)) {
      // From two rounds of tiles on a product with bias goes to blocks that walk over them: 4096 x 1536, K = 512, 8 items (3 rounds) 63 -> 57 us, 8192 x 3072,
      // K = 1024 (12) 376 -> 346.  With both GELU outputs, twice the stores in pieces of 16 bytes, K = 512 104 -> 106, K = 1024 629 -> 616: left as it was.
      bool walk = false;
      if constexpr (EPI == HDET_EPI_BIAS_BF16) {
        walk = walkable(g) && (int64_t)((g.m + 255) / 256) * ((g.n + 255) / 256) * batch >= 2 * (int64_t)cus;
        if (walk) launch_walk<EPI>(g, batch, s);
      }
      if (!walk) HDET_TILE(kAlternating, 512, hdet_bgemm_alt_kernel, );
    }
    else if (t_pair <= t_small && t_pair <= t_long)
      HDET_TILE(kPair, 512, hdet_bgemm_dma_kernel, 256, 128, 4, 2, 3, 32,);
    else if (t_small <= t_long) HDET_TILE(kSmall, 256, hdet_bgemm_dma_kernel, 128, 128, 2, 2, 2, 64,);
    else HDET_TILE(kLong, 512, hdet_bgemm_dma_kernel, 256, 128, 4, 2, 3, 64,);
  }
#undef HDET_TILE
  return hipGetLastError();
}

}  // namespace

bool hdet_bgemm_dma_eligible(const hdet_bgemm_args& g, bool a_kmajor, bool b_kmajor, int epi) {
  const bool f32_out = epi == HDET_EPI_F32 || epi == HDET_EPI_BIAS_F32;
  const bool has_bias = epi == HDET_EPI_BIAS_F32 || epi == HDET_EPI_BIAS_BF16 || epi == HDET_EPI_BIAS_RELU_BF16 ||
                        epi == HDET_EPI_BIAS_GELU_BF16 || epi == HDET_EPI_BIAS_RESID_BF16 || epi == HDET_EPI_BIAS_DROP_RESID_BF16;
  if (g.m < 1 || g.n < 1 || g.k < 1) return false;
  // a chunk is 8 elements along the operand's contiguous axis: k if k-major, else the row axis
  if (!chunk_regular(g.a, g.lda, g.a_s, a_kmajor ? g.k : g.m)) return false;
  if (!chunk_regular(g.b, g.ldb, g.b_s, b_kmajor ? g.k : g.n)) return false;
  // operand extents of one batch item as 32-bit byte offsets below the "absent" mark
  const int64_t a_bytes = ((int64_t)((a_kmajor ? g.m : g.k) - 1) * g.lda + (a_kmajor ? g.k : g.m)) * 2;
  const int64_t b_bytes = ((int64_t)((b_kmajor ? g.n : g.k) - 1) * g.ldb + (b_kmajor ? g.k : g.n)) * 2;
  // the K loop may form offsets up to one stage row past the extent before they are replaced
  const int64_t slack = 64 * 2 * (a_kmajor ? 1 : g.lda) + 64 * 2 * (b_kmajor ? 1 : g.ldb);
  if (a_bytes + slack >= (int64_t)1 << 31 || b_bytes + slack >= (int64_t)1 << 31) return false;
  // C (and bias, mask) four columns at a time
  if ((g.ldc & 3) || ((g.c_s[0] | g.c_s[1] | g.c_s[2]) & 3) || (g.n & 3)) return false;
  if (reinterpret_cast<uintptr_t>(g.c) & (f32_out ? 15 : 7)) return false;
  if (has_bias && ((g.bias_bs & 3) || (reinterpret_cast<uintptr_t>(g.bias) & 15))) return false;
  if (epi == HDET_EPI_BIAS_DROP_RESID_BF16 && (!g.drop_ctrl || g.drop_channel < 0 || g.n1 * g.n2 != 1 || g.c_s[0] >= ((int64_t)1 << 34)))
    return false;        // the replica is the batch index; the element counter has 32 bits
  if ((epi == HDET_EPI_MASK_BF16 || epi == HDET_EPI_GELUGRAD_BF16 || epi == HDET_EPI_BIAS_RESID_BF16 || epi == HDET_EPI_BIAS_DROP_RESID_BF16) &&
      (!g.mask || (g.mask_ld & 3) || (g.mask_bs & 3) || (reinterpret_cast<uintptr_t>(g.mask) & 7)))
    return false;
  if (epi == HDET_EPI_BIAS_GELU_BF16 && (!g.c2 || (reinterpret_cast<uintptr_t>(g.c2) & 7))) return false;
  if (epi == HDET_EPI_ADAMW &&
      (g.n1 * g.n2 != 1 || !g.upd.theta || !g.upd.m || !g.upd.v || !g.upd.ctrl || !g.upd.ctrl_out ||
       ((reinterpret_cast<uintptr_t>(g.upd.theta) | reinterpret_cast<uintptr_t>(g.upd.m) | reinterpret_cast<uintptr_t>(g.upd.v)) & 15) ||
       (reinterpret_cast<uintptr_t>(g.upd.shadow) & 7)))
    return false;
  // instantiated combinations: what the MLP and the transformer use
  if (a_kmajor && b_kmajor)
    return epi == HDET_EPI_BIAS_RELU_BF16 || epi == HDET_EPI_BIAS_F32 || epi == HDET_EPI_BIAS_BF16 || epi == HDET_EPI_F32 ||
           epi == HDET_EPI_BIAS_GELU_BF16 || epi == HDET_EPI_BIAS_RESID_BF16 || epi == HDET_EPI_BIAS_DROP_RESID_BF16;
  if (a_kmajor && !b_kmajor) return epi == HDET_EPI_MASK_BF16 || epi == HDET_EPI_BF16 || epi == HDET_EPI_GELUGRAD_BF16;
  if (!a_kmajor && !b_kmajor) return epi == HDET_EPI_F32 || epi == HDET_EPI_BF16 || epi == HDET_EPI_ADAMW;
  return false;
}

hipError_t hdet_launch_bgemm_dma(const hdet_bgemm_args& g_in, bool a_kmajor, bool b_kmajor, int epi, int batch,
                                 hipStream_t s) {
  hdet_bgemm_args g = g_in;
  if (g.n1 < 1) g.n1 = 1;
  if (g.n2 < 1) g.n2 = 1;
  if (!hdet_bgemm_dma_eligible(g, a_kmajor, b_kmajor, epi)) return hipErrorInvalidValue;
  if (a_kmajor && b_kmajor) {            // forward
    switch (epi) {
      case HDET_EPI_BIAS_RELU_BF16: return launch_shape<true, true, HDET_EPI_BIAS_RELU_BF16>(g, batch, s);
      case HDET_EPI_BIAS_F32: return launch_shape<true, true, HDET_EPI_BIAS_F32>(g, batch, s);
      case HDET_EPI_BIAS_BF16: return launch_shape<true, true, HDET_EPI_BIAS_BF16>(g, batch, s);
      case HDET_EPI_BIAS_GELU_BF16: return launch_shape<true, true, HDET_EPI_BIAS_GELU_BF16>(g, batch, s);
      case HDET_EPI_BIAS_RESID_BF16: return launch_shape<true, true, HDET_EPI_BIAS_RESID_BF16>(g, batch, s);
      case HDET_EPI_BIAS_DROP_RESID_BF16: return launch_shape<true, true, HDET_EPI_BIAS_DROP_RESID_BF16>(g, batch, s);
      default: return launch_shape<true, true, HDET_EPI_F32>(g, batch, s);
    }
  }
  if (a_kmajor) {                        // dgrad
    if (epi == HDET_EPI_MASK_BF16) return launch_shape<true, false, HDET_EPI_MASK_BF16>(g, batch, s);
    if (epi == HDET_EPI_GELUGRAD_BF16) return launch_shape<true, false, HDET_EPI_GELUGRAD_BF16>(g, batch, s);
    return launch_shape<true, false, HDET_EPI_BF16>(g, batch, s);
  }
  if (epi == HDET_EPI_F32) return launch_shape<false, false, HDET_EPI_F32>(g, batch, s);   // wgrad
  if (epi == HDET_EPI_ADAMW) return launch_shape<false, false, HDET_EPI_ADAMW>(g, batch, s);
  return launch_shape<false, false, HDET_EPI_BF16>(g, batch, s);
}

bool hdet_head_loss_eligible(const hdet_bgemm_args& g, int batch) {
  return walkable(g) && hdet_bgemm_dma_eligible(g, true, true, HDET_EPI_BIAS_BF16);
}

size_t hdet_head_loss_scratch(int m, int n, int batch) {
  return (size_t)batch * m * (8 * (size_t)((n + 255) / 256) + 16) + 1024;
}

hipError_t hdet_launch_head_loss(const hdet_bgemm_args& g_in, int batch, void* scratch, hipStream_t s) {
  hdet_bgemm_args g = g_in;
  if (!hdet_head_loss_eligible(g, batch) || !scratch || !g.xent.labels || !g.xent.row_loss) return hipErrorInvalidValue;
  const unsigned gx = (g.n + 255) / 256;
  const size_t rows = (size_t)batch * g.m;
  char* at = (char*)scratch;
  g.xent.part = (float2*)at; at += rows * gx * sizeof(float2);
  g.xent.row_lse = (double*)at; at += rows * sizeof(double);
  g.xent.row_ref = (float*)at; at += rows * sizeof(float);
  g.xent.row_a = (float*)at;
  g.xent.invb = 1.f / (float)g.m;
  launch_walk<HDET_EPI_XENT_STAT>(g, batch, s);
  hipLaunchKernelGGL(hdet_head_rows_kernel, dim3((g.m + 63) / 64, batch), dim3(256), 0, s, g.xent, g.m, g.n);
  launch_walk<HDET_EPI_XENT_GRAD>(g, batch, s);
  return hipGetLastError();
}
