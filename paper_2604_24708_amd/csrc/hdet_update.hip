// Fan-out update (Sec. 3.2, Eq. 2 generalised to SGD-momentum / AdamW), the gradient
// exchange of Algorithm 1 and the converge of Sec. 3.3 (Eq. 3) as single-pass HBM streams.
//
// Layout: every tensor is [N][stride] fp32, plane r = replica r.  The unit of work is one
// 16-byte column (4 consecutive parameters) of one replica:
//   * each of theta, g, m, v is read once and theta, m, v written once per step
//     (28 B per replica-element for AdamW, 20 B for SGD-momentum, +2 B with a bf16 copy);
//   * the replica mean of the gradients (shared mode) and the replica mean of the updated
//     parameters (fused converge) are formed on chip and cost no extra traffic.
// Loads and stores are 128-bit, coalesced along the parameter axis and non-temporal (every
// byte is touched exactly once per step, far beyond any cache).
//
// Four kernels:
//   plane  -- one thread per (replica, column), replica on blockIdx.y; steps that need no
//             exchange along the replica axis.  One column per thread and a grid that covers
//             the plane exactly streamed fastest on MI355X (about 6.4 TB/s, against 5.9 for
//             persistent blocks with a grid-stride loop).
//   wave   -- the wavefronts of a block are the replicas of one 64-column group (beyond 16 replicas
//             up to four replicas a wavefront); gradients (shared mode) and updated parameters (fused converge) cross the
//             replica axis through LDS, each wavefront then writes its own plane.  Keeps
//             the register footprint of the plane kernel instead of N columns per thread.
//   state  -- the wave kernel's form for one set of moments and whole columns.
//   loop   -- one thread walks the replica axis of a column; on request (hdet_set_launch_shape), for
//             planes of more columns than a grid holds, and beyond 16 replicas at the sizes that
//             loop_walks_better names.
// The P mod 4 trailing parameters are one more column in the plane and wave kernels, read and
// written element by element (ld_col / st_col): a launch of their own cost 3 to 6 us, as much as
// the whole update of a small model.
// With AdamW on the mean gradient the moments are the same for every replica; they can be kept
// once (one plane each), which takes a step from 28 N to 12 N + 16 bytes per element.

#include "hdet_internal.h"
#include "hdet_update_math.h"

#pragma clang fp contract(off)

namespace {

using namespace hdet_um;
typedef double d4 __attribute__((ext_vector_type(4)));

// fp64 companions of the column types, for the replica mean of the gradients
__device__ __forceinline__ d4 widen(f4 x) { return __builtin_convertvector(x, d4); }
__device__ __forceinline__ double widen(float x) { return (double)x; }
__device__ __forceinline__ f4 narrow(d4 x) { return __builtin_convertvector(x, f4); }
__device__ __forceinline__ float narrow(double x) { return (float)x; }

constexpr int kThreads = 256;

template <typename T> __device__ __forceinline__ T ld(const float* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const T*>(p));
}
template <typename T> __device__ __forceinline__ void st(float* p, T x) {
  __builtin_nontemporal_store(x, reinterpret_cast<T*>(p));
}

__device__ __forceinline__ void st_bf16(uint16_t* p, f4 x) {
  us4 o = {to_bf16(x[0]), to_bf16(x[1]), to_bf16(x[2]), to_bf16(x[3])};
  __builtin_nontemporal_store(o, reinterpret_cast<us4*>(p));
}
__device__ __forceinline__ void st_bf16(uint16_t* p, float x) { *p = to_bf16(x); }

// Column i of a plane of which `cnt` elements exist: 4, or P mod 4 in the last column (the others read as 0).
__device__ __forceinline__ f4 ld_col(const float* p, int cnt) {
  if (cnt >= 4) return ld<f4>(p);
  f4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c < cnt) x[c] = ld<float>(p + c);
  return x;
}
__device__ __forceinline__ void st_col(float* p, f4 x, int cnt) {
  if (cnt >= 4) { st<f4>(p, x); return; }
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c < cnt) st<float>(p + c, x[c]);
}
__device__ __forceinline__ void st_bf16_col(uint16_t* p, f4 x, int cnt) {
  if (cnt >= 4) { st_bf16(p, x); return; }
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c < cnt) st_bf16(p + c, x[c]);
}
__device__ __forceinline__ int col_elements(int64_t n_params, int64_t i) {      // <= 0: no such column
  const int64_t left = n_params - (i << 2);
  return left < 4 ? (int)left : 4;
}

// ---------------------------------------------------------------------------------------
// plane kernel: thread = (replica blockIdx.y, column blockIdx.x * 256 + threadIdx.x)
// ---------------------------------------------------------------------------------------
template <int OPT>
__global__ __launch_bounds__(kThreads) void hdet_update_plane_kernel(const hdet_update_args a) {
  const int r = blockIdx.y;
  const rep_scalars s = replica_scalars(a, r);
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.lr_channel == 0) a.ctrl_out->lr_used[r] = s.lr;
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= ((a.n_params + 3) >> 2)) return;
  const int cnt = col_elements(a.n_params, i);
  const int64_t off = (int64_t)r * a.stride + (i << 2);
  f4 th = ld_col(a.theta + off, cnt);
  f4 g = ld_col(a.grad + (int64_t)r * a.grad_stride + (i << 2), cnt);
  if (a.grad_stride == 0) g = g * a.grad_scale;
  f4 m = ld_col(a.m + off, cnt);
  f4 v = splat<f4>(0.f);
  if (OPT == HDET_ADAMW) v = ld_col(a.v + off, cnt);
  update_one<OPT, f4>(th, g, m, v, a, s);
  st_col(a.m + off, m, cnt);
  if (OPT == HDET_ADAMW) st_col(a.v + off, v, cnt);
  st_col(a.theta + off, th, cnt);
  if (a.shadow) st_bf16_col(a.shadow + off, th, cnt);
}

// ---------------------------------------------------------------------------------------
// wave kernel: block = `groups` column groups x W wavefronts, W = ceil(N / R); wavefront (grp, w)
// owns the 64 columns of group grp in the replicas w, w + W, ... (R of them at most; R = 1 up to
// 16 replicas).  ex carries a column across the replica axis.
// R > 1 against one thread per column that walks the replicas (the loop kernel), N = 32 and one set of moments: the
// loads of all replicas are in flight together, and 16 wavefronts share a column's exchange.
// ---------------------------------------------------------------------------------------
constexpr int kMaxWaves = 16;

// LDS staging for a mean along the replica axis, structure-of-arrays so that every access
// is free of bank conflicts.  val[grp * N + r][c][lane]: component c of replica r's column.
template <int R> struct exchange_buf {
  float val[kMaxWaves * R][4][64];
  float mean[R == 1 ? kMaxWaves : 1][4][64];      // indexed by group (R > 1: one group)
};

// Every wavefront of group `grp` hands in its columns x; all get back the group's replica
// mean.  The 256 scalars of a group are shared out over its threads, each summed once in
// fp64 in the order r = 0..N-1 and rounded to fp32 once (same bits as the loop kernel).
// Ends with every thread past both barriers, so the buffer can be reused at once.
template <int R>
__device__ __forceinline__ f4 exchange_mean(exchange_buf<R>& e, const f4 (&x)[R], int grp, int w, int waves, int n, int lane) {
#pragma unroll
  for (int k = 0; k < R; ++k)
    if (R == 1 || w + k * waves < n) {
#pragma unroll
      for (int c = 0; c < 4; ++c) e.val[grp * n + w + k * waves][c][lane] = x[k][c];
    }
  __syncthreads();
  const double inv_n = 1.0 / (double)n;
  for (int sidx = w * 64 + lane; sidx < 256; sidx += waves * 64) {
    const int c = sidx >> 6, l = sidx & 63;
    double sum = 0.0;
    for (int q = 0; q < n; ++q) sum += (double)e.val[grp * n + q][c][l];
    e.mean[grp][c][l] = (float)(sum * inv_n);
  }
  __syncthreads();
  return (f4){e.mean[grp][0][lane], e.mean[grp][1][lane], e.mean[grp][2][lane], e.mean[grp][3][lane]};
}

// SSTATE (AdamW on the mean gradient): m and v are single planes; the wavefront of replica 0
// reads, advances and writes them, and hands m / (sqrt(v)/sqrt(1-b2^t) + eps) to the other
// wavefronts of its group through LDS.
template <int OPT, bool SHARED, bool CONV, bool SSTATE, int R>
__global__ __launch_bounds__(kMaxWaves * 64) void hdet_update_wave_kernel(const hdet_update_args a,
                                                                          const int groups, const int waves) {
  static_assert(!SSTATE || (SHARED && OPT == HDET_ADAMW), "one set of moments needs AdamW on the mean gradient");
  __shared__ exchange_buf<R> ex;
  const int n = a.n_replicas;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = R == 1 ? wid / waves : 0, w = wid - grp * waves;
  rep_scalars s[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = w + k * waves;
    s[k] = replica_scalars(a, r < n ? r : 0);
    if (blockIdx.x == 0 && grp == 0 && lane == 0 && a.lr_channel == 0 && r < n) a.ctrl_out->lr_used[r] = s[k].lr;
  }
  const int64_t i = ((int64_t)blockIdx.x * groups + grp) * 64 + lane;
  const int cnt = col_elements(a.n_params, i);
  const bool ok = cnt > 0;
  constexpr int RM = SSTATE ? 1 : R;                   // sets of moments a thread may hold
  f4 th[R], g[R], m[RM], v[RM];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = w + k * waves;
    const bool on = ok && (R == 1 || r < n);
    const int64_t off = (int64_t)r * a.stride + (i << 2);
    th[k] = g[k] = splat<f4>(0.f);
    if (on) {
      th[k] = ld_col(a.theta + off, cnt);
      g[k] = ld_col(a.grad + (int64_t)r * a.grad_stride + (i << 2), cnt);
      if (a.grad_stride == 0) g[k] = g[k] * a.grad_scale;
    }
    if (k < RM) {
      m[k] = v[k] = splat<f4>(0.f);
      if (on && (!SSTATE || w == 0)) {
        m[k] = ld_col(a.m + (SSTATE ? (i << 2) : off), cnt);
        if (OPT == HDET_ADAMW) v[k] = ld_col(a.v + (SSTATE ? (i << 2) : off), cnt);
      }
    }
  }
  // the paper's gradient AllReduce: every replica applies the replica mean
  if (SHARED) {
    const f4 gbar = exchange_mean<R>(ex, g, grp, w, waves, n, lane);
#pragma unroll
    for (int k = 0; k < R; ++k) g[k] = gbar;
  }
  if (SSTATE) {
    if (w == 0) {
      const f4 ratio = adamw_moments<f4>(g[0], m[0], v[0], a);
#pragma unroll
      for (int c = 0; c < 4; ++c) ex.mean[grp][c][lane] = ratio[c];
    }
    __syncthreads();
    const f4 ratio = {ex.mean[grp][0][lane], ex.mean[grp][1][lane], ex.mean[grp][2][lane], ex.mean[grp][3][lane]};
#pragma unroll
    for (int k = 0; k < R; ++k) adamw_apply<f4>(th[k], ratio, s[k]);
    if (CONV) __syncthreads();                        // ex.mean is written again below
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) update_one<OPT, f4>(th[k], g[k], m[k], v[k], a, s[k]);
  }
#pragma unroll
  for (int k = 0; k < RM; ++k) {
    const int r = w + k * waves;
    const int64_t moff = SSTATE ? (i << 2) : (int64_t)r * a.stride + (i << 2);
    if (ok && (R == 1 || r < n) && (!SSTATE || w == 0)) {
      st_col(a.m + moff, m[k], cnt);
      if (OPT == HDET_ADAMW) st_col(a.v + moff, v[k], cnt);
    }
  }
  // Eq. 3 on the freshly updated parameters
  if (CONV) {
    const f4 mean = exchange_mean<R>(ex, th, grp, w, waves, n, lane);
#pragma unroll
    for (int k = 0; k < R; ++k) th[k] = mean;
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = w + k * waves;
    const int64_t off = (int64_t)r * a.stride + (i << 2);
    if (ok && (R == 1 || r < n)) {
      st_col(a.theta + off, th[k], cnt);
      if (a.shadow) st_bf16_col(a.shadow + off, th[k], cnt);
    }
  }
}

// The wave kernel for one set of moments and 2 to 16 replicas: whole columns only, 16-byte accesses without a mask of their own.
// The order in which the streams reach the memory decides here: the general form, whose accesses are masked one by one, is up
// to 5 % slower (and up to 10 % faster in the other forms of update), but has the trailing parameters in the same launch.  With
// some, a launch of their own (3 to 4 us) pays from 9 replicas and 4 million parameters on.  One kernel that holds both forms
// needs more than 64 registers a lane: up to 50 % slower.  us, this / general:
//   none trailing:   N = 5, P = 8e6 108 / 113;  N = 8, P = 20e6 370 / 368;  N = 12, P = 20e6 595 / 607;  N = 16, P = 4e6 146 / 154
//   some, with their launch:  N = 2, P = 4e6 31 / 28;  N = 8, P = 4e6 79 / 75, P = 12e6 224 / 225, P = 90e6 1694 / 1698;
//                             N = 9, P = 8e6 180 / 194;  N = 12, P = 3e6 99 / 93, P = 12e6 356 / 364;  N = 16, P = 30e6 1129 / 1166
template <bool CONV>
__global__ __launch_bounds__(kMaxWaves * 64) void hdet_update_state_kernel(const hdet_update_args a, const int groups) {
  __shared__ exchange_buf<1> ex;
  const int n = a.n_replicas;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = wid / n, r = wid - grp * n;
  const rep_scalars s = replica_scalars(a, r);
  if (blockIdx.x == 0 && grp == 0 && lane == 0 && a.lr_channel == 0) a.ctrl_out->lr_used[r] = s.lr;
  const int64_t i = ((int64_t)blockIdx.x * groups + grp) * 64 + lane;
  const bool ok = i < (a.n_params >> 2);
  const int64_t off = (int64_t)r * a.stride + (i << 2);
  const int64_t moff = i << 2;
  const bool mine = ok && r == 0;                     // this thread holds the moments
  f4 th = splat<f4>(0.f), m = th, v = th;
  f4 g[1] = {th};
  if (ok) {
    th = ld<f4>(a.theta + off);
    g[0] = ld<f4>(a.grad + (int64_t)r * a.grad_stride + (i << 2));
    if (a.grad_stride == 0) g[0] = g[0] * a.grad_scale;
  }
  if (mine) {
    m = ld<f4>(a.m + moff);
    v = ld<f4>(a.v + moff);
  }
  const f4 gbar = exchange_mean<1>(ex, g, grp, r, n, n, lane);
  if (r == 0) {
    const f4 ratio = adamw_moments<f4>(gbar, m, v, a);
#pragma unroll
    for (int c = 0; c < 4; ++c) ex.mean[grp][c][lane] = ratio[c];
  }
  __syncthreads();
  const f4 ratio = {ex.mean[grp][0][lane], ex.mean[grp][1][lane], ex.mean[grp][2][lane], ex.mean[grp][3][lane]};
  adamw_apply<f4>(th, ratio, s);
  if (CONV) __syncthreads();                          // ex.mean is written again below
  if (mine) {
    st<f4>(a.m + moff, m);
    st<f4>(a.v + moff, v);
  }
  if (CONV) {
    const f4 x[1] = {th};
    th = exchange_mean<1>(ex, x, grp, r, n, n, lane);
  }
  if (ok) {
    st<f4>(a.theta + off, th);
    if (a.shadow) st_bf16(a.shadow + off, th);
  }
}

// Standalone converge (Eq. 3) in the same shape: 4 B read + 4 B written per replica-element.
template <int R>
__global__ __launch_bounds__(kMaxWaves * 64) void hdet_converge_wave_kernel(const hdet_converge_args a,
                                                                            const int groups, const int waves) {
  __shared__ exchange_buf<R> ex;
  const int n = a.n_replicas;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = R == 1 ? wid / waves : 0, w = wid - grp * waves;
  const int64_t i = ((int64_t)blockIdx.x * groups + grp) * 64 + lane;
  const int cnt = col_elements(a.n_params, i);
  const bool ok = cnt > 0;
  f4 th[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = w + k * waves;
    th[k] = splat<f4>(0.f);
    if (ok && (R == 1 || r < n)) th[k] = ld_col(a.theta + (int64_t)r * a.stride + (i << 2), cnt);
  }
  const f4 mean = exchange_mean<R>(ex, th, grp, w, waves, n, lane);
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = w + k * waves;
    const int64_t off = (int64_t)r * a.stride + (i << 2);
    if (ok && (R == 1 || r < n)) {
      st_col(a.theta + off, mean, cnt);
      if (a.shadow) st_bf16_col(a.shadow + off, mean, cnt);
    }
  }
}

// ---------------------------------------------------------------------------------------
// loop kernel: one thread walks the replica axis of a column of width T (f4 or float).  Bound by the loads in flight: a
// column's replicas are a chain of memory latencies, which only many columns at a time hide.
// ---------------------------------------------------------------------------------------

template <int OPT, bool SHARED, bool CONV, bool SSTATE, typename T>
__device__ __forceinline__ void update_column(const hdet_update_args& a, const rep_scalars* s,
                                              int64_t col) {
  const int n = a.n_replicas;
  T gbar = splat<T>(0.f);
  if (SHARED) {
    // The paper's gradient AllReduce: mean over the replica axis, r ascending.  Summed in
    // fp64 and rounded to fp32 once: Adam's first steps move by lr * g/(|g| + eps), which
    // magnifies a last-place difference in a near-zero mean gradient ten-thousandfold.
    auto sum = widen(splat<T>(0.f));
    if (a.grad_stride == 0) {
      gbar = ld<T>(a.grad + col) * a.grad_scale;
    } else {
      for (int q = 0; q < n; ++q) sum = sum + widen(ld<T>(a.grad + (int64_t)q * a.grad_stride + col));
      gbar = narrow(sum * (1.0 / (double)n));
    }
  }
  T ratio = splat<T>(0.f);
  if (SSTATE) {                        // one set of moments for all replicas
    T m = ld<T>(a.m + col), v = ld<T>(a.v + col);
    ratio = adamw_moments<T>(gbar, m, v, a);
    st<T>(a.m + col, m);
    st<T>(a.v + col, v);
  }
  // Eq. 3 accumulator, fp64: the sum of N fp32 values is then exact up to 2^-53, the mean is
  // rounded to fp32 once, and averaging identical replicas returns them bit for bit.
  auto acc = widen(splat<T>(0.f));
  for (int r = 0; r < n; ++r) {
    const int64_t off = (int64_t)r * a.stride + col;
    T th = ld<T>(a.theta + off);
    if (SSTATE) {
      adamw_apply<T>(th, ratio, s[r]);
    } else {
      T g = SHARED ? gbar : ld<T>(a.grad + (int64_t)r * a.grad_stride + col);
      if (!SHARED && a.grad_stride == 0) g = g * a.grad_scale;
      T m = ld<T>(a.m + off);
      T v = splat<T>(0.f);
      if (OPT == HDET_ADAMW) v = ld<T>(a.v + off);
      update_one<OPT, T>(th, g, m, v, a, s[r]);
      st<T>(a.m + off, m);
      if (OPT == HDET_ADAMW) st<T>(a.v + off, v);
    }
    if (CONV) {
      acc = acc + widen(th);          // Eq. 3: sum in the order r = 0..N-1
    } else {
      st<T>(a.theta + off, th);
      if (a.shadow) st_bf16(a.shadow + off, th);
    }
  }
  if (CONV) {
    const T mean = narrow(acc * (1.0 / (double)n));
    for (int r = 0; r < n; ++r) {
      const int64_t off = (int64_t)r * a.stride + col;
      st<T>(a.theta + off, mean);
      if (a.shadow) st_bf16(a.shadow + off, mean);
    }
  }
}

template <int OPT, bool SHARED, bool CONV, bool SSTATE>
__global__ __launch_bounds__(kThreads) void hdet_update_loop_kernel(const hdet_update_args a) {
  __shared__ rep_scalars s[HDET_MAX_REPLICAS];
  if ((int)threadIdx.x < a.n_replicas) {
    s[threadIdx.x] = replica_scalars(a, threadIdx.x);
    if (blockIdx.x == 0 && a.lr_channel == 0) a.ctrl_out->lr_used[threadIdx.x] = s[threadIdx.x].lr;
  }
  __syncthreads();
  const int64_t nvec = a.n_params >> 2;
  const int tail = (a.n_params & 3) != 0;                   // loop_grid
  if (blockIdx.x < (unsigned)tail) {
    if ((int)threadIdx.x < (int)(a.n_params & 3)) update_column<OPT, SHARED, CONV, SSTATE, float>(a, s, (nvec << 2) + threadIdx.x);
    return;
  }
  const int64_t gstride = (int64_t)(gridDim.x - tail) * kThreads;
  for (int64_t i = (int64_t)(blockIdx.x - tail) * kThreads + threadIdx.x; i < nvec; i += gstride)
    update_column<OPT, SHARED, CONV, SSTATE, f4>(a, s, i << 2);
}

// Standalone converge (Eq. 3): 4 B read + 4 B written per replica-element.
template <typename T>
__device__ __forceinline__ void converge_column(const hdet_converge_args& a, int64_t col) {
  const int n = a.n_replicas;
  auto acc = widen(splat<T>(0.f));     // fp64 sum, one rounding to fp32 (see update_column)
#pragma unroll 4
  for (int q = 0; q < n; ++q) acc = acc + widen(ld<T>(a.theta + (int64_t)q * a.stride + col));
  const T mean = narrow(acc * (1.0 / (double)n));
  for (int q = 0; q < n; ++q) {
    const int64_t off = (int64_t)q * a.stride + col;
    st<T>(a.theta + off, mean);
    if (a.shadow) st_bf16(a.shadow + off, mean);
  }
}

__global__ __launch_bounds__(kThreads) void hdet_converge_kernel(const hdet_converge_args a) {
  const int64_t nvec = a.n_params >> 2;
  const int tail = (a.n_params & 3) != 0;
  if (blockIdx.x < (unsigned)tail) {
    if ((int)threadIdx.x < (int)(a.n_params & 3)) converge_column<float>(a, (nvec << 2) + threadIdx.x);
    return;
  }
  const int64_t gstride = (int64_t)(gridDim.x - tail) * kThreads;
  for (int64_t i = (int64_t)(blockIdx.x - tail) * kThreads + threadIdx.x; i < nvec; i += gstride)
    converge_column<f4>(a, i << 2);
}

// bf16 copy of the parameters (creation / resume).
__global__ __launch_bounds__(kThreads) void hdet_shadow_kernel(const float* theta, uint16_t* shadow,
                                                               int64_t n_params, int64_t stride) {
  const int64_t base = (int64_t)blockIdx.y * stride;
  const int64_t nvec = n_params >> 2;
  const int64_t gstride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += gstride)
    st_bf16(shadow + base + (i << 2), *reinterpret_cast<const f4*>(theta + base + (i << 2)));
  if (blockIdx.x == gridDim.x - 1) {
    const int64_t col = (nvec << 2) + threadIdx.x;
    if (col < n_params) st_bf16(shadow + base + col, theta[base + col]);
  }
}

int clamp_blocks(int64_t n_params, int blocks) {
  int64_t need = ((n_params >> 2) + kThreads - 1) / kThreads;
  if (need < 1) need = 1;
  return (int)(need < blocks ? need : blocks);
}

// The loop kernels' grid: blocks of whole columns behind one for the P mod 4 trailing parameters, if there are any.  That one
// walks the replicas like any other thread, and starts first: at the end of the last block the walk stood alone (N = 64,
// P = 1673131, SGD on the mean gradient 457 us, with it in front 412).
int loop_grid(int64_t n_params, int blocks) { return clamp_blocks(n_params, blocks) + ((n_params & 3) != 0); }

constexpr int kStateReplicas = 9;              // see hdet_update_state_kernel
constexpr int64_t kStateParams = 4000000;

// Shape of a wave-kernel launch: R replicas per wavefront, 512-thread blocks of several column groups while R = 1.
struct wave_shape {
  int r, groups, waves;
  int64_t bx;
};
wave_shape wave_launch(int64_t n_params, int n) {
  wave_shape w;
  w.r = (n + kMaxWaves - 1) / kMaxWaves;
  w.waves = (n + w.r - 1) / w.r;
  w.groups = w.r == 1 && n < 8 ? 8 / n : 1;
  const int64_t ncol = (n_params + 3) >> 2;        // the last one may hold fewer than four parameters
  w.bx = (ncol + 64 * (int64_t)w.groups - 1) / (64 * (int64_t)w.groups);
  return w;
}

// Beyond 16 replicas: whether the loop kernel takes a launch.  Up to a block or two of 256 columns per CU it is bound by the
// latency of a thread's walk along the replicas, two to five times slower than the wave kernel; from there on it walks the
// planes one after the other, which the memory side likes better than the wave kernel's N planes side by side, until its grid
// no longer runs in one piece.  With one set of moments and 33 replicas or more it stays ahead for good: the wave kernel then
// has a block of up to 16 wavefronts per CU and its exchanges stand alone.  The lines are in blocks per CU (a quarter each), by
// what crosses the replica axis.  Single sizes scatter by 10 % with the planes' distance, so the figures are wave / loop, the
// geometric mean over one to three sizes in each range of P (256 CUs):
//                            0.12-0.2e6 0.3-0.4e6 0.4-0.5e6 0.5-0.62e6 0.8-1e6 1.2-1.5e6 1.5-1.9e6 1.9-2.5e6 3.5-5.5e6
//   one set,       N = 32      0.40      0.65      0.82      0.85      1.12     1.11      1.11      0.94      0.97
//   one set,       N = 48      0.42      0.74      0.92      1.05      1.23     1.19      1.35      1.09      1.10
//   one set, conv, N = 48      0.72      0.97      1.15      1.13      1.28     1.26      1.30      1.25      1.21
//   AdamW, mean,   N = 32      0.36      0.77      0.97      0.91      1.10     1.00      1.03      0.99      1.00
//   SGD, mean,     N = 48      0.47      0.88      1.00      0.95      1.03     1.01      1.12      0.99      0.97
//   AdamW, conv,   N = 48      0.78      1.06      1.20      1.01      1.01     0.94      1.01      0.97      0.96
//   converge alone (with a plane update), N = 32  0.96  1.08  1.06  1.00  1.04  0.99      0.99      0.98      0.99
struct crossing { bool mean, one_set, conv; };      // gradients; ... with one set of moments; parameters
bool loop_walks_better(int64_t n_params, int n, const crossing& x) {
  if (n <= kMaxWaves) return false;
  const int64_t quarters = (n_params >> 2) * 4 / (kThreads * (int64_t)hdet_compute_units());
  if (x.one_set && n > 2 * kMaxWaves) return quarters >= (x.conv ? 8 : 10);
  if (x.mean) return quarters >= 10 && quarters < 28;
  return quarters >= 6 && quarters < 16;
}
bool converge_loop_walks_better(int64_t n_params, int n) {
  const int64_t quarters = (n_params >> 2) * 4 / (kThreads * (int64_t)hdet_compute_units());
  return n > kMaxWaves && quarters >= 3 && quarters < 16;
}

template <int OPT, bool SHARED, bool CONV, bool SSTATE = false>
void launch_variant(const hdet_update_args& a, int variant, int blocks, hipStream_t stream) {
  const int n = a.n_replicas;
  const bool exchange = SHARED || CONV;
  // with one gradient plane for all replicas the wave kernel is taken as well: the replicas of a column share a
  // block, so the plane comes from memory once
  if (variant == 0 && !exchange && !(a.grad_stride == 0 && n > 1 && n <= kMaxWaves)) {
    const int64_t bx = (((a.n_params + 3) >> 2) + kThreads - 1) / kThreads;
    if (bx <= 0x7fffffff) {
      hipLaunchKernelGGL((hdet_update_plane_kernel<OPT>), dim3((unsigned)bx, n), dim3(kThreads), 0, stream, a);
      return;
    }
  } else if (variant == 0 && !loop_walks_better(a.n_params, n, {SHARED, SSTATE, CONV})) {
    const wave_shape w = wave_launch(a.n_params, n);
    if (w.bx <= 0x7fffffff) {
      const dim3 grid((unsigned)w.bx), block(64 * w.groups * w.waves);
      if constexpr (SSTATE) {
        if (w.r == 1 && n > 1 && ((a.n_params & 3) == 0 || (n >= kStateReplicas && a.n_params >= kStateParams))) {
          hipLaunchKernelGGL((hdet_update_state_kernel<CONV>), grid, block, 0, stream, a, w.groups);
          const int64_t whole = a.n_params & ~(int64_t)3;
          if (whole == a.n_params) return;
          hdet_update_args t = a;                     // the trailing parameters, in the general form
          t.theta += whole; t.grad += whole; t.m += whole; t.v += whole;
          if (t.shadow) t.shadow += whole;
          t.n_params -= whole;
          hipLaunchKernelGGL((hdet_update_wave_kernel<OPT, SHARED, CONV, SSTATE, 1>), dim3(1), block, 0, stream, t, w.groups, w.waves);
          return;
        }
      }
      if (w.r == 1) hipLaunchKernelGGL((hdet_update_wave_kernel<OPT, SHARED, CONV, SSTATE, 1>), grid, block, 0, stream, a, w.groups, w.waves);
      else if (w.r == 2) hipLaunchKernelGGL((hdet_update_wave_kernel<OPT, SHARED, CONV, SSTATE, 2>), grid, block, 0, stream, a, w.groups, w.waves);
      else if (w.r == 3) hipLaunchKernelGGL((hdet_update_wave_kernel<OPT, SHARED, CONV, SSTATE, 3>), grid, block, 0, stream, a, w.groups, w.waves);
      else hipLaunchKernelGGL((hdet_update_wave_kernel<OPT, SHARED, CONV, SSTATE, 4>), grid, block, 0, stream, a, w.groups, w.waves);
      return;
    }
  }
  hipLaunchKernelGGL((hdet_update_loop_kernel<OPT, SHARED, CONV, SSTATE>), dim3(loop_grid(a.n_params, blocks)),
                     dim3(kThreads), 0, stream, a);
}

template <int OPT>
void launch_update_opt(const hdet_update_args& a, bool shared, bool conv, int variant, int blocks,
                       hipStream_t stream) {
  if (shared && conv) launch_variant<OPT, true, true>(a, variant, blocks, stream);
  else if (shared) launch_variant<OPT, true, false>(a, variant, blocks, stream);
  else if (conv) launch_variant<OPT, false, true>(a, variant, blocks, stream);
  else launch_variant<OPT, false, false>(a, variant, blocks, stream);
}

}  // namespace

hipError_t hdet_launch_update(const hdet_update_args& a, int optimizer, bool shared, bool fuse_converge,
                              int variant, int blocks, hipStream_t stream) {
  if (a.shared_state) {
    if (optimizer != HDET_ADAMW || !shared) return hipErrorInvalidValue;
    if (fuse_converge) launch_variant<HDET_ADAMW, true, true, true>(a, variant, blocks, stream);
    else launch_variant<HDET_ADAMW, true, false, true>(a, variant, blocks, stream);
    return hipGetLastError();
  }
  if (optimizer == HDET_ADAMW) launch_update_opt<HDET_ADAMW>(a, shared, fuse_converge, variant, blocks, stream);
  else launch_update_opt<HDET_SGDM>(a, shared, fuse_converge, variant, blocks, stream);
  return hipGetLastError();
}

hipError_t hdet_launch_converge(const hdet_converge_args& a, int variant, int blocks, hipStream_t stream) {
  const wave_shape w = wave_launch(a.n_params, a.n_replicas);
  if (variant == 0 && w.bx <= 0x7fffffff && !converge_loop_walks_better(a.n_params, a.n_replicas)) {
    const dim3 grid((unsigned)w.bx), block(64 * w.groups * w.waves);
    if (w.r == 1) hipLaunchKernelGGL(hdet_converge_wave_kernel<1>, grid, block, 0, stream, a, w.groups, w.waves);
    else if (w.r == 2) hipLaunchKernelGGL(hdet_converge_wave_kernel<2>, grid, block, 0, stream, a, w.groups, w.waves);
    else if (w.r == 3) hipLaunchKernelGGL(hdet_converge_wave_kernel<3>, grid, block, 0, stream, a, w.groups, w.waves);
    else hipLaunchKernelGGL(hdet_converge_wave_kernel<4>, grid, block, 0, stream, a, w.groups, w.waves);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(hdet_converge_kernel, dim3(loop_grid(a.n_params, blocks)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t hdet_launch_shadow(const float* theta, uint16_t* shadow, int64_t n_params, int64_t stride,
                              int n_replicas, int blocks, hipStream_t stream) {
  dim3 grid(clamp_blocks(n_params, blocks), n_replicas);
  hipLaunchKernelGGL(hdet_shadow_kernel, grid, dim3(kThreads), 0, stream, theta, shadow, n_params, stride);
  return hipGetLastError();
}
