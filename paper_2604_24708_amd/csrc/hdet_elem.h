// Element access for activation tensors that are fp32 in full precision and bfloat16 (stored
// as uint16_t, round to nearest even) in mixed precision.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

__device__ __forceinline__ float hdet_ld(const float* p) { return *p; }
__device__ __forceinline__ float hdet_ld(const uint16_t* p) { return __uint_as_float((unsigned)(*p) << 16); }
__device__ __forceinline__ void hdet_st(float* p, float x) { *p = x; }
__device__ __forceinline__ void hdet_st(uint16_t* p, float x) { *p = __builtin_bit_cast(unsigned short, (__bf16)x); }

// Eight consecutive elements (16-byte aligned for bf16, 32-byte for fp32) in one or two
// 128-bit accesses.
struct hdet_f8 { float v[8]; };
typedef float hdet_f4v __attribute__((ext_vector_type(4)));
typedef unsigned int hdet_u4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ hdet_f8 hdet_ld8(const float* p) {
  const hdet_f4v a = *reinterpret_cast<const hdet_f4v*>(p), b = *reinterpret_cast<const hdet_f4v*>(p + 4);
  hdet_f8 r = {{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}};
  return r;
}
__device__ __forceinline__ hdet_f8 hdet_ld8(const uint16_t* p) {
  const hdet_u4v u = *reinterpret_cast<const hdet_u4v*>(p);
  hdet_f8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.v[2 * i] = __uint_as_float(u[i] << 16);
    r.v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
  }
  return r;
}
__device__ __forceinline__ unsigned hdet_bf16_bits(float x) {      // round to nearest even (the hardware conversion)
  return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)x);
}
// two values rounded and packed, lo in the low half: one conversion instruction
typedef float hdet_f2v __attribute__((ext_vector_type(2)));
typedef __bf16 hdet_bf2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned hdet_bf16_pack(float lo, float hi) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((hdet_f2v){lo, hi}, hdet_bf2v));
}
__device__ __forceinline__ void hdet_st8(float* p, const hdet_f8& x) {
  *reinterpret_cast<hdet_f4v*>(p) = (hdet_f4v){x.v[0], x.v[1], x.v[2], x.v[3]};
  *reinterpret_cast<hdet_f4v*>(p + 4) = (hdet_f4v){x.v[4], x.v[5], x.v[6], x.v[7]};
}
__device__ __forceinline__ void hdet_st8(uint16_t* p, const hdet_f8& x) {
  hdet_u4v u;
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = hdet_bf16_pack(x.v[2 * i], x.v[2 * i + 1]);
  *reinterpret_cast<hdet_u4v*>(p) = u;
}

// Four consecutive elements in one access (16 B fp32, 8 B bf16).
struct hdet_f4 { float v[4]; };
typedef unsigned int hdet_u2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ hdet_f4 hdet_ld4(const float* p) {
  const hdet_f4v a = *reinterpret_cast<const hdet_f4v*>(p);
  hdet_f4 r = {{a[0], a[1], a[2], a[3]}};
  return r;
}
__device__ __forceinline__ hdet_f4 hdet_ld4(const uint16_t* p) {
  const hdet_u2v u = *reinterpret_cast<const hdet_u2v*>(p);
  hdet_f4 r = {{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u),
                __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xffff0000u)}};
  return r;
}
__device__ __forceinline__ void hdet_st4(float* p, const hdet_f4& x) {
  *reinterpret_cast<hdet_f4v*>(p) = (hdet_f4v){x.v[0], x.v[1], x.v[2], x.v[3]};
}
__device__ __forceinline__ void hdet_st4(uint16_t* p, const hdet_f4& x) {
  hdet_u2v u = {hdet_bf16_pack(x.v[0], x.v[1]), hdet_bf16_pack(x.v[2], x.v[3])};
  *reinterpret_cast<hdet_u2v*>(p) = u;
}

// the same accesses marked non-temporal: data that is touched once and is larger than the caches
__device__ __forceinline__ hdet_f4 hdet_ld4_stream(const float* p) {
  const hdet_f4v a = __builtin_nontemporal_load(reinterpret_cast<const hdet_f4v*>(p));
  hdet_f4 r = {{a[0], a[1], a[2], a[3]}};
  return r;
}
__device__ __forceinline__ void hdet_st4_stream(float* p, const hdet_f4& x) {
  __builtin_nontemporal_store((hdet_f4v){x.v[0], x.v[1], x.v[2], x.v[3]}, reinterpret_cast<hdet_f4v*>(p));
}
__device__ __forceinline__ void hdet_st4_stream(uint16_t* p, const hdet_f4& x) {
  const hdet_u2v u = {hdet_bf16_pack(x.v[0], x.v[1]), hdet_bf16_pack(x.v[2], x.v[3])};
  __builtin_nontemporal_store(u, reinterpret_cast<hdet_u2v*>(p));
}

// x of another lane of the same row of 16 lanes, by a data-parallel primitive: CTRL 0xB1 / 0x4E = quad
// permutations [1,0,3,2] / [2,3,0,1], 0x141 / 0x140 = mirror within 8 / 16 lanes
template <int CTRL>
__device__ __forceinline__ float hdet_dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
// Reductions over the wavefront, the same value in every lane: four steps inside each row of 16 lanes
// (pairs, quads, 8, 16), then two exchanges between rows.  The order is fixed.
__device__ __forceinline__ float hdet_wave_sum(float x) {
  x += hdet_dpp<0xB1>(x);
  x += hdet_dpp<0x4E>(x);
  x += hdet_dpp<0x141>(x);
  x += hdet_dpp<0x140>(x);
  x += __shfl_xor(x, 16);
  x += __shfl_xor(x, 32);
  return x;
}
__device__ __forceinline__ float hdet_wave_max(float x) {
  x = fmaxf(x, hdet_dpp<0xB1>(x));
  x = fmaxf(x, hdet_dpp<0x4E>(x));
  x = fmaxf(x, hdet_dpp<0x141>(x));
  x = fmaxf(x, hdet_dpp<0x140>(x));
  x = fmaxf(x, __shfl_xor(x, 16));
  x = fmaxf(x, __shfl_xor(x, 32));
  return x;
}

// GELU in its tanh form and its derivative (the transformer's MLP activation).  With u = c (z + 0.044715 z^3) and e = exp(-2u):
// 0.5 (1 + tanh u) = 1 / (1 + e) = s, and gelu' = s (1 + z (1 - s) 2 u'), 1 - s = e s, so that nothing cancels where tanh is close to -1 or 1.
__device__ __forceinline__ float hdet_gelu_exp(float z, float z2) {
  const float k1 = -1.5957691216057308f, k2 = -0.07135481282592269f;      // -2 c, -2 c 0.044715
  return expf(z * __builtin_fmaf(k2, z2, k1));
}
// With h = e(|z|) / (1 + e(|z|)), at most 1/2: z h below 0, z - z h above, so that only the last rounding is of the result's size.  Normal arguments of
// size 1 and 2, rms from 64 bits: 1.9e-8 and 3.5e-8 (a last rounding alone 1.7e-8 and 3.4e-8; 0.5 z (1 + tanh u) 2.6e-8 and 4.8e-8; z / (1 + e(z)) 2.8e-8
// and 5.7e-8).  Above 10 h is 0, also where z h would be infinity times that.
__device__ __forceinline__ float hdet_gelu_tanh(float z) {
  const float e = hdet_gelu_exp(fabsf(z), z * z), h = e / (1.f + e);
  return z < 0.f ? z * h : __builtin_fmaf(z > 10.f ? -10.f : -z, h, z);
}
// Below -10 the derivative is less than 1e-35 in size and s runs out of exponents while the rest still grows with z^3: 0 from there on.  Above 10 it
// is 1 and formed at 10, where nothing overflows.  (NaN takes neither branch.)
__device__ __forceinline__ float hdet_gelu_tanh_grad(float z) {
  const float k3 = 1.5957691216057308f, k4 = 0.21406444881780076f;        // 2 u' = k3 + k4 z^2
  const float x = z > 10.f ? 10.f : z, x2 = x * x, e = hdet_gelu_exp(x, x2), s = 1.f / (1.f + e);
  return z < -10.f ? 0.f : s * __builtin_fmaf(x * (e * s), __builtin_fmaf(k4, x2, k3), 1.f);
}

// The same two functions for results that are rounded to bfloat16 anyway, on the hardware exp2 and reciprocal
// (absolute error of a few 1e-7).  With u = c (z + 0.044715 z^3):  0.5 (1 + tanh u) = sigma(2u) = 1 / (1 + exp(-2u)), so
//   gelu(z)  = z sigma(2u),        exp(-2u) = exp2(z (k1 + k2 z^2)),  k1 = -2 c log2(e),  k2 = 0.044715 k1
//   gelu'(z) = sigma + z sigma (1 - sigma) 2 u'(z) = sigma (1 + z (1 - sigma) (k3 + k4 z^2)),  k3 = 2 c,  k4 = 6 c 0.044715
// z -> -inf gives exp2 = inf, sigma = 0 and the limits 0 and 0; z -> +inf gives sigma = 1 and the limits z and 1.  The derivative is formed within +-20,
// where it has its limits and z (1 - sigma) z^2 is finite (from -1e13 on it was not).  A NaN z has made the loss NaN, and with it what this is multiplied by.
__device__ __forceinline__ float hdet_gelu_sigma_fast(float z, float z2) {
  const float k1 = -2.302208198144325f, k2 = -0.1029432395800235f;
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(z * __builtin_fmaf(k2, z2, k1)));
}
__device__ __forceinline__ float hdet_gelu_tanh_fast(float z) {
  return z * hdet_gelu_sigma_fast(z, z * z);
}
__device__ __forceinline__ float hdet_gelu_tanh_grad_fast(float z) {
  const float k3 = 1.5957691216057308f, k4 = 0.21406444881780076f;
  const float x = __builtin_amdgcn_fmed3f(z, -20.f, 20.f), x2 = x * x;
  const float sg = hdet_gelu_sigma_fast(x, x2);
  return __builtin_fmaf(sg, (x * (1.f - sg)) * __builtin_fmaf(k4, x2, k3), sg);
}

// Philox-4x32 with 10 rounds (Salmon et al., SC'11); used for dropout masks and the warm initialisation.  From the fourth
// round on all four words differ from lane to lane and the two exclusive ors of a word are one v_bitop3 (which the compiler
// does not form from the written-out ones); before that most operands are uniform or do not change between replicas and are
// left to the scalar unit and to hoisting.
struct hdet_philox4 { uint32_t x[4]; };
__device__ __forceinline__ hdet_philox4 hdet_philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                           uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int rnd = 0; rnd < 10; ++rnd) {
    if (rnd > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t h0 = (uint32_t)(p0 >> 32), h1 = (uint32_t)(p1 >> 32);
    const uint32_t n0 = rnd < 3 ? h1 ^ c1 ^ k0 : __builtin_amdgcn_bitop3_b32(h1, c1, k0, 0x96);
    const uint32_t n1 = (uint32_t)p1;
    const uint32_t n2 = rnd < 3 ? h0 ^ c3 ^ k1 : __builtin_amdgcn_bitop3_b32(h0, c3, k1, 0x96);
    const uint32_t n3 = (uint32_t)p0;
    c0 = n0; c1 = n1; c2 = n2; c3 = n3;
  }
  hdet_philox4 o = {{c0, c1, c2, c3}};
  return o;
}

// Mean of one replica's row losses in a fixed tree order, the step loss l(theta_r, B_r) of Algorithm 1, and its accumulation
// into L_acc (Sec. 3.4).  One block of 256 threads; part: four doubles of LDS.
template <typename CTRL>
__device__ __forceinline__ void hdet_reduce_loss(const float* row_loss, int rows, CTRL* ctrl, int r, double* part) {
  double s = 0.0;
  for (int b = threadIdx.x; b < rows; b += 256) s += (double)row_loss[(int64_t)r * rows + b];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double mean = (part[0] + part[1] + part[2] + part[3]) / (double)rows;
    ctrl->l_step[r] = (float)mean;
    ctrl->l_acc[r] += mean;
  }
}
