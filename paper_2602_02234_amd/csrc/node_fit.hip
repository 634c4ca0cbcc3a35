// The message-passing models' fitting net (node_fit.h): 16 atoms per workgroup, one output tile of
// 16 hidden units per wave, all products transposed (dp_tiles.h) on 16x16x4 float32 MFMA;
// activations meet in LDS once per product, a lane's own stay in its registers.
// Bound: latency of the weights (L2) at few atoms.  Inside the last layer's kernel, atom by atom, the net read
// its 192 KB of weights for every atom: 185 us of a 9,999-atom repformer step, 75 us of a GNN one.
#include "node_fit.h"

#include "dp_tiles.h"

namespace dp {
namespace {

constexpr int IN = NodeFit::IN, WID = NodeFit::WID;
constexpr int LDR = WID + 4;  // row stride in LDS

// W x with x = 16 NK features of the lane's atom in LDS: the contraction in parts of two tiles, summed by
// themselves and then pairwise (the energy weighs these sums with factors that make one long
// sum's rounding visible).
template <int NK> __device__ __forceinline__ f4 product(const W<float, NK> &w, const float *row) {
  f4 acc[NK / 2];
#pragma unroll
  for (int p = 0; p < NK / 2; ++p) {
    acc[p] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f4 x = ldf4(row + 32 * p + 16 * h + 4 * (lane_id() >> 4));
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.v[2 * p + h][s], x[s], acc[p], 0, 0, 0);
    }
  }
#pragma unroll
  for (int n = NK / 2; n > 1; n /= 2)
#pragma unroll
    for (int p = 0; p < n / 2; ++p) acc[p] = acc[2 * p] + acc[2 * p + 1];
  return acc[0];
}

__global__ void __launch_bounds__(512) k_node_fit(NodeFit w, float *__restrict__ rows, int n, double *__restrict__ Ei,
                                                  const unsigned *__restrict__ flags) {
  __shared__ float X[2][16][LDR] __attribute__((aligned(16)));
  __shared__ double ep[16][WID / 16];
  if (failed(flags)) return;
  const int l = lane_id(), q = l >> 4, c = l & 15, t = wave_id();
  const int a0 = blockIdx.x * 16, col = 16 * t + 4 * q;
  W<float, IN / 16> w1;
  W<float, WID / 16> w2;
  w1.load(w.G1, t);
  if (threadIdx.x < 256) {
    const int a = threadIdx.x >> 4, k = threadIdx.x & 15;
    stf4(&X[0][a][4 * k], ldf4(rows + (size_t)min(a0 + a, n - 1) * IN + 4 * k));
  }
  const f4 b1 = ldf4(w.d1 + col), b2 = ldf4(w.d2 + col), g3 = ldf4(w.G3 + col);
  w2.load(w.G2, t);
  __syncthreads();
  f4 y1, t2, d;
  const f4 z1 = product(w1, X[0][c]) + b1;
#pragma unroll
  for (int i = 0; i < 4; ++i) y1[i] = tanhf(z1[i]);
  stf4(&X[1][c][col], y1);
  __syncthreads();
  const f4 z2 = product(w2, X[1][c]) + b2;
  w2.load(w.G2T, t);
  double e = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    t2[i] = tanhf(z2[i]);
    e += (double)(t2[i] + y1[i]) * w.G3d[col + i];
  }
  d = g3 * (1.f - t2 * t2);
  e += __shfl_xor(e, 16);
  e += __shfl_xor(e, 32);
  if (q == 0) ep[c][t] = e;
  stf4(&X[0][c][col], d);
  __syncthreads();
  if (threadIdx.x < 16 && a0 + (int)threadIdx.x < n) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < WID / 16; ++k) s += ep[threadIdx.x][k];
    Ei[a0 + threadIdx.x] = w.d3 + s;
  }
  d = (product(w2, X[0][c]) + g3) * (1.f - y1 * y1);
  if (t < IN / 16) w2.load(w.G1T, t);
  stf4(&X[1][c][col], d);
  __syncthreads();
  if (t < IN / 16) {
    const f4 dn = product(w2, X[1][c]);
    if (a0 + c < n) stf4(rows + (size_t)(a0 + c) * IN + col, dn);
  }
}

}  // namespace

void launch_node_fit(const NodeFit &w, float *rows, int n, double *Ei, const unsigned *flags, hipStream_t st) {
  hipLaunchKernelGGL(k_node_fit, dim3((n + 15) / 16), dim3(512), 0, st, w, rows, n, Ei, flags);
}

}  // namespace dp
