// Shared parts of the per-atom kernels (gnn.hip, repformer.hip, node_fit.hip; the descriptors through
// dp_desc.h; fitting.hip): MFMA products in the transposed form -- weights as A operand, features
// along the accumulator rows, 16 angles, edges, tokens or atoms along the columns -- in which
// lane (q = lane / 16, c = lane % 16) holds features 16 t + 4 q + i of column c, the layout of
// float4 rows in memory, of an accumulator and of the next product's B operand alike.
#pragma once
#include "dp_internal.h"

namespace dp {
namespace {

__device__ __forceinline__ bool failed(const unsigned *flags) { return (flags[0] & FLAG_ERRORS) != 0u; }
__device__ __forceinline__ f4 ldf4(const float *p) { return *reinterpret_cast<const f4 *>(p); }
__device__ __forceinline__ void stf4(float *p, f4 v) { *reinterpret_cast<f4 *>(p) = v; }
// Sum over the four lane groups (the lanes of one column): a swap of a value's odd rows of 16 lanes with
// its own even rows leaves one of a pair of rows in both lanes of the pair, and the other in the second
// result; likewise the halves of the wave.  In registers; __shfl_xor goes through LDS.
__device__ __forceinline__ float sumq(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float maxq(float v) {  // likewise the largest
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ f4 sum16(f4 v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = dp::sum16(v[i]);
  return v;
}
// Ordering of LDS traffic between the lanes of one wave.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// The lane index through an empty asm statement: inside a loop over atoms the compiler then
// forms lane-derived addresses where they are used instead of keeping (and spilling) them all.
__device__ __forceinline__ int lane() {
  int l = lane_id();
  asm volatile("" : "+v"(l));
  return l;
}
// Keeps the loads of one tile from being scheduled across another's products.
__device__ __forceinline__ void tile_barrier() { __builtin_amdgcn_sched_barrier(0); }

// B operand over 16 NK features (tiles x[t], features 16 t + 4 q + i), and an A operand tile
// of 16 outputs over the same contraction from fragment order: float32, tile t at
// ((t NK + kb) 64 + lane) 4; bf16, two tiles of features per step, at ((t NK/2 + kp) 64 +
// lane) 8, the first four values from tile 2 kp, the others from tile 2 kp + 1.
template <typename T, int NK> struct X;
template <typename T, int NK> struct W;
template <int NK> struct X<float, NK> {
  f4 v[NK];
  __device__ __forceinline__ explicit X(const f4 (&x)[NK]) {
#pragma unroll
    for (int k = 0; k < NK; ++k) v[k] = x[k];
  }
};
template <int NK> struct W<float, NK> {
  f4 v[NK];
  __device__ __forceinline__ void load(const float *__restrict__ p, int t) {
#pragma unroll
    for (int k = 0; k < NK; ++k) v[k] = ldf4(p + ((t * NK + k) * 64 + lane_id()) * 4);
  }
  __device__ __forceinline__ f4 operator()(const X<float, NK> &x, f4 acc) const {
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v[k][s], x.v[k][s], acc, 0, 0, 0);
    return acc;
  }
};
template <int NK> struct X<bf16_t, NK> {
  bf8 v[NK / 2];
  __device__ __forceinline__ explicit X(const f4 (&x)[NK]) {
#pragma unroll
    for (int k = 0; k < NK / 2; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[k][e] = (__bf16)x[2 * k + e / 4][e % 4];
  }
};
template <int NK> struct W<bf16_t, NK> {
  bf8 v[NK / 2];
  __device__ __forceinline__ void load(const bf16_t *__restrict__ p, int t) {
#pragma unroll
    for (int k = 0; k < NK / 2; ++k) v[k] = *reinterpret_cast<const bf8 *>(p + ((t * (NK / 2) + k) * 64 + lane_id()) * 8);
  }
  __device__ __forceinline__ f4 operator()(const X<bf16_t, NK> &x, f4 acc) const {
#pragma unroll
    for (int k = 0; k < NK / 2; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[k], x.v[k], acc, 0, 0, 0);
    return acc;
  }
};
// The four 16-output tiles of a product over the NK feature tiles x, one after the other:
// use(k, acc) with acc = W_k x + init(k).  The contraction goes in pieces of 64 features, and
// the next piece's weights are loaded while the current one is used.
template <typename T, int NK, class Init, class Use>
__device__ __forceinline__ void tiles(const T *__restrict__ p, const f4 (&x)[NK], const Init &init, const Use &use) {
  constexpr int H = NK / 4;  // pieces; fragment order makes piece h of tile k the tile k H + h of 64
  W<T, 4> cur;
  cur.load(p, 0);
  f4 acc;
#pragma unroll
  for (int s = 0; s < 4 * H; ++s) {
    W<T, 4> nxt = cur;
    if (s + 1 < 4 * H) nxt.load(p, s + 1);
    tile_barrier();
    const f4 xs[4] = {x[4 * (s % H)], x[4 * (s % H) + 1], x[4 * (s % H) + 2], x[4 * (s % H) + 3]};
    if (s % H == 0) acc = init(s / H);
    acc = cur(X<T, 4>(xs), acc);
    if (s % H == H - 1) use(s / H, acc);
    tile_barrier();
    cur = nxt;
  }
}

// 16 x 16 tile in LDS, element (token, key) swizzled so that neither access has a bank conflict:
// put writes a lane's four keys of its token, get reads token 4 q + s of key c.
__device__ __forceinline__ void put_tile(float *tile, f4 y) {
  const int q = lane() >> 4, c = lane() & 15, h = c >> 2;
  stf4(tile + 16 * (4 * h + ((c & 3) ^ h)) + 4 * (q ^ h), y);
}
__device__ __forceinline__ f4 get_tile(const float *tile) {
  const int q = lane() >> 4, c = lane() & 15;
  f4 o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o[s] = tile[16 * (4 * q + (s ^ q)) + (c ^ (4 * q))];
  return o;
}

// Copy of N 16-byte pieces from global memory to LDS by a workgroup of NT threads: loaded first, stored
// when their place is free.
template <int N, int NT> struct Copy16 {
  static constexpr int R = (N + NT - 1) / NT;
  f4 v[R];
  static __device__ __forceinline__ int thread() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));  // as lane()
    return t;
  }
  __device__ __forceinline__ Copy16() {}
  __device__ __forceinline__ explicit Copy16(const void *__restrict__ w) { load(w); }
  __device__ __forceinline__ void load(const void *__restrict__ w) {
    const int t = thread();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int k = t + r * NT;
      v[r] = ldf4(static_cast<const float *>(w) + 4 * (k < N ? k : 0));
    }
  }
  // pieces A .. B - 1 only, to d
  template <int A = 0, int B = N> __device__ __forceinline__ void store(void *d) const {
    const int t = thread();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int k = t + r * NT;
      if (k >= A && k < B) stf4(static_cast<float *>(d) + 4 * (k - A), v[r]);
    }
  }
};

// tanh of the layers' hot loops, from the hardware exponential and reciprocal:
// tanh |x| = (1 - t) / (1 + t), t = exp(-2 |x|).  The difference is exact or rounded with the product, so
// near zero only t's own rounding is left: absolute error 0.9e-8 in the mean and 2.4e-8 at most below 0.05,
// 3.8e-8 and 1.3e-7 over |x| < 5.  (1 - 2 / (1 + exp(2 x)) is an instruction less but cancels: 4.6e-8 and
// 1.2e-7 below 0.05.)
__device__ __forceinline__ float act(float x) {
  const float t = __builtin_amdgcn_exp2f(-2.885390081777927f * fabsf(x));
  const float r = __builtin_amdgcn_rcpf(1.f + t);
  return copysignf(fmaf(-t, r, r), x);
}
__device__ __forceinline__ f4 act(f4 v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = act(v[i]);
  return v;
}
// tanh without branches: up to 0.6 x + x^3 p(x^2), where p interpolates (tanh x / x - 1) / x^2 at the six
// Chebyshev nodes of [0, 0.36] (relative error 4e-10; Taylor's series of the same length is off by 2e-8 at
// 0.45, the same way for every argument), beyond it 1 - 2 t / (1 + t) with t = exp(-2 |x|) from the hardware
// exponential and reciprocal, the rounding of the exponent, of 1 + t and of the quotient put back.  Within
// 3 units in the last place in a simulation with the hardware functions off by one, 0.3 in the mean;
// tanhf's branches took a third of the descriptor's embedding.
__device__ __forceinline__ float tanh_fast(float x) {
  constexpr float C = 2.885390043258667f, CL = 3.851926e-8f;  // 2 / ln 2
  const float ax = fminf(fabsf(x), 32.f), y = -C * ax, yl = fmaf(-C, ax, -y) - CL * ax;  // finite: 1 from 9.1 on
  float t = __builtin_amdgcn_exp2f(y);
  t = fmaf(t, yl * 0.6931471805599453f, t);
  const float d = 1.f + t, dl = t - (d - 1.f), r = __builtin_amdgcn_rcpf(d), q = 2.f * t * r;
  const float big = 1.f - fmaf(fmaf(-dl, q, fmaf(-d, q, 2.f * t)), r, q);
  const float z = x * x;
  float p = fmaf(fmaf(2.3707656e-3f, z, -8.4100708e-3f), z, 2.1788322e-2f);
  p = fmaf(fmaf(fmaf(p, z, -5.3961552e-2f), z, 1.3333313e-1f), z, -3.3333333e-1f);
  return !(fabsf(x) >= 0.6f) ? fmaf(p * z, x, x) : copysignf(big, x);  // NaN by the series
}

// Initial features tanh(x w + b) of a lane's four features, with tanhf or tanh_fast.  The repformer takes
// tanhf: an error that all atoms share shows enlarged in its virial, and tanh_fast saves nothing there.
template <float (*Tanh)(float)>
__device__ __forceinline__ f4 init4(float x, const float *__restrict__ w, const float *__restrict__ b) {
  const f4 wv = ldf4(w), bv = ldf4(b);
  f4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = Tanh(x * wv[i] + bv[i]);
  return v;
}

// out[c] = sum_k x[k] Wm[k][c] for threads c < C of a group of NT threads (tid within it; x in
// LDS, Wm row-major): the rows split over the group, the parts (in `part`, one float per
// thread) added in order.  Starts with a workgroup barrier, which every thread passes.
template <int NT, int K, int C>
__device__ __forceinline__ float matvec(const float *__restrict__ Wm, const float *x, float *part, int tid) {
  constexpr int SEG = NT / C, PER = (K + SEG - 1) / SEG;
  static_assert(SEG >= 1, "at least one thread per output");
  const int c = tid % C, sg = tid / C;
  __syncthreads();
  float v = 0.f;
  if (sg < SEG)
#pragma unroll 16
    for (int k = sg * PER; k < min(K, (sg + 1) * PER); ++k) v += x[k] * Wm[k * C + c];
  part[tid] = v;
  __syncthreads();
  float r = 0.f;
  if (tid < C)
#pragma unroll
    for (int s = 0; s < SEG; ++s) r += part[s * C + c];
  return r;
}

}  // namespace
}  // namespace dp
