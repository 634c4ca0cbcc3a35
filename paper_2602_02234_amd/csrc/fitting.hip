// Fitting net on gfx950: per-atom energy from the descriptor and, for the backward pass,
// dE_i/dT (paper, Section II: a fitting net maps each atom's representation to its energy;
// E is the sum of the atomic energies).
//   D = T T_<16^T;  y1 = tanh(D F1 + c1);  y2 = tanh(y1 F2 + c2) + y1;  y3 = tanh(y2 F3 + c3) + y2
//   E_i = y3 . F4 + c4 + ebias[t_i]    (per fitting head: E_i = sum_h hw_h E_i^h)
//
// Three kernels, 16 (or 32) atoms per workgroup.  The products with F1 (384,000 of the
// 499,200 multiplications each way) are split over column groups and, along the
// contraction, over the waves, so that even ten atom tiles fill the chip; one kernel for
// the whole net ran 150 atoms on ten CUs in 0.59 ms (float32).  The descriptor D (1600
// values per atom) is never stored: its entries come from T (400 values) where they are
// needed, and dE/dD is contracted to dE/dT in the registers it is formed in.
//   k_fit_in   y1, workgroup = atom tile x 3 column tiles x head;
//   k_fit_mid  the two hidden layers, E_i and dE/dpre1, workgroup = atom tile, one column
//              tile per wave; activations meet in LDS once per product, a lane's own
//              values stay in its registers;
//   k_fit_out  dE/dD = sum_h dE/dpre1^h F1^hT and from it dE/dT, workgroup = atom tile x
//              34 of the 100 rows m.
// All products are transposed (weights as A operand: hidden units or descriptor entries
// along the accumulator rows, atoms along the columns), weights in MFMA fragment order.
// Bound: the matrix cores at many atoms, latency of the weight loads (L2) at few.  Measured
// against one kernel for the whole net (forward and backward): float32 150 atoms 594 -> 56 us,
// 9,999 atoms 1.81 -> 0.30 ms; bfloat16 192 atoms 80 -> 45 us, 24,999 atoms 0.48 -> 0.49 ms,
// where the descriptor kernels gain 0.16 ms by neither writing D nor contracting dE/dD.
//
// Both precisions share the kernels.  F32: 16x16x4 float32 products.  B16: the energy is
// read off this net directly, so its products carry the bfloat16 path's largest rounding
// sensitivity; each runs on bf16 MFMA with both operands split into two bf16 terms,
// x = x_hi + x_lo, and three products x_hi w_hi + x_hi w_lo + x_lo w_hi accumulated in
// fp32 (the dropped lo*lo term is 2^-16 relative).
#include "dp_internal.h"

namespace dp {
namespace {

constexpr int KH = 256;      // hidden width padded along k
constexpr int LDA = KH + 4;  // LDS row stride (floats) of hidden activations
constexpr int LDT = 4 * M + 4;  // ... of staged T rows
constexpr int NHT = FH / 16;    // 15 hidden column tiles
constexpr int NWI = 10, CTI = 3;  // k_fit_in: waves, column tiles per workgroup
constexpr int NWO = 12, NGO = 3, MGO = 34;  // k_fit_out: waves, groups of rows m, rows per group
static_assert(NHT % CTI == 0 && NGO * MGO >= M && NWO * 3 >= MGO, "the tiles cover the net");

// Per-atom row of ws.fit (ND floats): y1, then dE/dpre1, of each head; dE/dT (its sum over
// a) and the NGO partial sums over m' of its first 16 rows.
constexpr int ROW_Y = 0, ROW_DT = MAXH * FH, ROW_PART = ROW_DT + 4 * M;
static_assert(ROW_PART + NGO * 4 * M2 <= ND, "the fitting net's row fits");
static_assert(ROW_DT == FIT_DT && ROW_PART == FIT_PART && NGO == FIT_NPART, "as the descriptor backward reads it");

__device__ __forceinline__ f4 ldf4(const float *p) { return *reinterpret_cast<const f4 *>(p); }
__device__ __forceinline__ bf8 ldb8(const bf16_t *p) { return *reinterpret_cast<const bf8 *>(p); }

// A precision: k steps of KS, a lane holding PER consecutive k of a step (k = KS s + PER q
// + e), A fragments of the weights and B operands made from float32 values.
struct F32 {
  static constexpr int KS = 16, PER = 4, KHS = FH / KS;  // KHS: steps over the hidden width
  struct Mat { const float *p; };
  struct Fin { Mat F1T, F2T, F3T, F1, F2, F3; };
  struct A { f4 v; };
  struct B { f4 v; };
  static __device__ __forceinline__ A load(const Mat &m, size_t frag) { return {ldf4(m.p + frag * 256 + 4 * lane_id())}; }
  static __device__ __forceinline__ B make(const f4 (&x)[1]) { return {x[0]}; }
  static __device__ __forceinline__ f4 mma(const A &a, const B &b, f4 acc) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[s], b.v[s], acc, 0, 0, 0);
    return acc;
  }
};
struct B16 {
  static constexpr int KS = 32, PER = 8, KHS = KH / KS;
  struct Mat { const bf16_t *hi, *lo; };
  struct Fin { Mat F1T, F2T, F3T, F1, F2, F3; };
  struct A { bf8 h, l; };
  struct B { bf8 h, l; };
  static __device__ __forceinline__ A load(const Mat &m, size_t frag) {
    return {ldb8(m.hi + frag * 512 + 8 * lane_id()), ldb8(m.lo + frag * 512 + 8 * lane_id())};
  }
  static __device__ __forceinline__ B make(const f4 (&x)[2]) {
    B b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = x[e / 4][e % 4];
      const __bf16 h = (__bf16)v;
      b.h[e] = h;
      b.l[e] = (__bf16)(v - (float)h);
    }
    return b;
  }
  static __device__ __forceinline__ f4 mma(const A &a, const B &b, f4 acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, acc, 0, 0, 0);
  }
};

template <class P> struct Heads { typename P::Fin f[MAXH]; };

// The B operand of step s from a row of float32 values.
template <class P> __device__ __forceinline__ typename P::B from_row(const float *row, int s) {
  f4 x[P::PER / 4];
#pragma unroll
  for (int e = 0; e < P::PER / 4; ++e) x[e] = ldf4(row + P::KS * s + P::PER * (lane_id() >> 4) + 4 * e);
  return P::make(x);
}

// ------------------------------------------------------------ y1 = tanh(D F1 + c1)
template <class P, int AT>
__global__ void __launch_bounds__(NWI * 64) k_fit_in(Tables w, Heads<P> hd, const float *__restrict__ Tsave, int c0,
                                                     int c1, float *__restrict__ fit) {
  constexpr int S = ND / P::KS;  // k steps, dealt to the waves in turn
  static_assert(S % NWI == 0, "whole turns");
  __shared__ union {
    float T[16 * AT][LDT];
    float red[NWI][AT * CTI][256];
  } sm __attribute__((aligned(16)));
  const int a0 = c0 + blockIdx.x * 16 * AT, h = blockIdx.z, t0 = blockIdx.y * CTI;
  const int l = lane_id(), q = l >> 4, c = l & 15, wv = wave_id();
  const typename P::Mat F = hd.f[h].F1T;
  for (int x = threadIdx.x; x < 16 * AT * M; x += NWI * 64) {
    const int a = x / M, m = x % M;
    *reinterpret_cast<f4 *>(&sm.T[a][4 * m]) = ldf4(Tsave + ((size_t)min(a0 + a, c1 - 1) * M + m) * 4);
  }
  typename P::A wn[CTI];
#pragma unroll
  for (int u = 0; u < CTI; ++u) wn[u] = P::load(F, (size_t)(t0 + u) * S + wv);
  __syncthreads();
  // step s covers descriptor entries 16 m + a: rows m = (KS / 16) s + ..., the lane's a fixed
  const int mo = (P::PER * q) / M2, ab = (P::PER * q) % M2;
  f4 Ta[AT][P::PER];
#pragma unroll
  for (int at = 0; at < AT; ++at)
#pragma unroll
    for (int e = 0; e < P::PER; ++e) Ta[at][e] = ldf4(&sm.T[16 * at + c][4 * (ab + e)]);
  f4 acc[AT][CTI] = {};
#pragma unroll
  for (int turn = 0; turn < S / NWI; ++turn) {
    const int s = wv + NWI * turn;
    __builtin_amdgcn_sched_barrier(0);
    typename P::A wc[CTI];
#pragma unroll
    for (int u = 0; u < CTI; ++u) {
      wc[u] = wn[u];
      wn[u] = P::load(F, (size_t)(t0 + u) * S + min(s + NWI, S - 1));
    }
#pragma unroll
    for (int at = 0; at < AT; ++at) {
      const f4 tm = ldf4(&sm.T[16 * at + c][4 * ((P::KS / M2) * s + mo)]);
      f4 x[P::PER / 4];
#pragma unroll
      for (int e = 0; e < P::PER; ++e) {
        const f4 ta = Ta[at][e];
        x[e / 4][e % 4] = tm[0] * ta[0] + tm[1] * ta[1] + tm[2] * ta[2] + tm[3] * ta[3];
      }
      const typename P::B b = P::make(x);
#pragma unroll
      for (int u = 0; u < CTI; ++u) acc[at][u] = P::mma(wc[u], b, acc[at][u]);
    }
  }
  __syncthreads();  // T is no longer needed
#pragma unroll
  for (int at = 0; at < AT; ++at)
#pragma unroll
    for (int u = 0; u < CTI; ++u) *reinterpret_cast<f4 *>(&sm.red[wv][at * CTI + u][4 * l]) = acc[at][u];
  __syncthreads();
  for (int x = threadIdx.x; x < AT * CTI * 64; x += NWI * 64) {
    const int tile = x / 64, ll = x % 64, at = tile / CTI, u = tile % CTI;
    f4 v = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < NWI; ++k) v += ldf4(&sm.red[k][tile][4 * ll]);
    const int col = 16 * (t0 + u) + 4 * (ll >> 4), a = a0 + 16 * at + (ll & 15);
    const f4 bias = ldf4(w.c1[h] + col);
    f4 y;
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = tanhf(v[i] + bias[i]);
    if (a < c1) *reinterpret_cast<f4 *>(fit + (size_t)a * ND + ROW_Y + h * FH + col) = y;
  }
}

// ------------------------------------------------------------ hidden layers, E_i, dE/dpre1
template <class P>
__global__ void __launch_bounds__(NHT * 64) k_fit_mid(Tables w, Heads<P> hd, const int *__restrict__ types, int c0, int c1,
                                                      float *__restrict__ fit, double *__restrict__ Ei,
                                                      double *__restrict__ Eh, int backward) {
  __shared__ float X[2][16][LDA] __attribute__((aligned(16)));  // columns 240 .. 255 stay zero
  __shared__ double ep[16][16];
  constexpr int S = P::KHS;
  const int a0 = c0 + blockIdx.x * 16;
  const int l = lane_id(), q = l >> 4, c = l & 15, t = wave_id();
  const int col = 16 * t + 4 * q, a = a0 + c;  // the lane's hidden units col .. col + 3 and its atom
  for (int x = threadIdx.x; x < 2 * 16 * (KH - FH); x += NHT * 64) X[x / (16 * (KH - FH))][x / (KH - FH) % 16][FH + x % (KH - FH)] = 0.f;
  double esum = 0.0;
  const auto product = [&](const typename P::A (&wf)[S], int b) {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < S; ++s) acc = P::mma(wf[s], from_row<P>(X[b][c], s), acc);
    return acc;
  };
  const auto weights = [&](const typename P::Mat &m, typename P::A (&wf)[S]) {  // issued ahead of a barrier
#pragma unroll
    for (int s = 0; s < S; ++s) wf[s] = P::load(m, (size_t)t * S + s);
  };
  for (int h = 0; h < w.nheads; ++h) {
    const float hw = (float)w.hw[h];
    float *row = fit + (size_t)min(a, c1 - 1) * ND + ROW_Y + h * FH + col;
    typename P::A wf[S];
    weights(hd.f[h].F2T, wf);
    const f4 y1 = ldf4(row);
    *reinterpret_cast<f4 *>(&X[0][c][col]) = y1;
    __syncthreads();
    f4 acc = product(wf, 0);
    weights(hd.f[h].F3T, wf);
    f4 t2, y2, t3;
    const f4 b2 = ldf4(w.c2[h] + col), b3 = ldf4(w.c3[h] + col), F4 = ldf4(w.F4[h] + col);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t2[i] = tanhf(acc[i] + b2[i]);
      y2[i] = t2[i] + y1[i];
    }
    *reinterpret_cast<f4 *>(&X[1][c][col]) = y2;
    __syncthreads();
    acc = product(wf, 1);
    const bool bwd = backward && w.hw[h] != 0.0;
    if (bwd) weights(hd.f[h].F3, wf);
    // E_i = y3 . F4 + c4 + ebias in float64
    double p = 0.0;
    f4 d;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t3[i] = tanhf(acc[i] + b3[i]);
      p += (double)(t3[i] + y2[i]) * w.F4d[h][col + i];
      d[i] = hw * F4[i] * (1.f - t3[i] * t3[i]);  // dE/dpre3
    }
    p += __shfl_xor(p, 16);
    p += __shfl_xor(p, 32);
    if (q == 0) ep[c][t] = p;
    *reinterpret_cast<f4 *>(&X[0][c][col]) = d;
    __syncthreads();
    if ((int)threadIdx.x < 16 && a0 + (int)threadIdx.x < c1) {
      const int r = threadIdx.x;
      int ty = types[a0 + r];
      ty = ty < 0 ? 0 : (ty >= NTYPES ? NTYPES - 1 : ty);
      double e = 0.0;
      for (int k = 0; k < NHT; ++k) e += ep[r][k];
      e += w.c4[h] + w.ebias[h][ty];
      esum += w.hw[h] * e;
      if (w.nheads > 1) Eh[(size_t)(a0 + r) * MAXH + h] = e;
    }
    if (bwd) {
      // dy2 = dpre3 F3^T + hw F4;  dpre2 = dy2 (1 - t2^2)
      const f4 dy2 = product(wf, 0) + hw * F4;
      weights(hd.f[h].F2, wf);
      *reinterpret_cast<f4 *>(&X[1][c][col]) = dy2 * (1.f - t2 * t2);
      __syncthreads();
      // dy1 = dpre2 F2^T + dy2;  dpre1 = dy1 (1 - y1^2)
      const f4 dy1 = product(wf, 1) + dy2;
      if (a < c1) *reinterpret_cast<f4 *>(row) = dy1 * (1.f - y1 * y1);
    }
    __syncthreads();  // the next head overwrites X and ep
  }
  if ((int)threadIdx.x < 16 && a0 + (int)threadIdx.x < c1) Ei[a0 + threadIdx.x] = esum;
}

// ------------------------------------------------------------ dE/dT
// dT_m = sum_a dD_ma T_a + [m < 16] sum_m' dD_m'm T_m'; the second sum is left as one part
// per workgroup, added up by the descriptor backward.
template <class P, int AT>
__global__ void __launch_bounds__(NWO * 64) k_fit_out(Tables w, Heads<P> hd, const float *__restrict__ Tsave, int c0, int c1,
                                                      float *__restrict__ fit) {
  __shared__ union {
    float X[16 * AT][LDA];
    float red[NWO][64][16 + 1];
  } sm __attribute__((aligned(16)));
  constexpr int S = P::KHS;
  const int a0 = c0 + blockIdx.x * 16 * AT;
  const int m0 = blockIdx.y * MGO, m1 = min(M, m0 + MGO);
  const int l = lane_id(), q = l >> 4, c = l & 15, wv = wave_id();
  f4 acc[AT][3] = {};
  for (int h = 0; h < w.nheads; ++h) {
    if (w.hw[h] == 0.0) continue;
    const typename P::Mat F = hd.f[h].F1;
    __syncthreads();
    for (int x = threadIdx.x; x < 16 * AT * (KH / 4); x += NWO * 64) {
      const int a = x / (KH / 4), k = 4 * (x % (KH / 4));
      const f4 zero = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f4 *>(&sm.X[a][k]) = k < FH ? ldf4(fit + (size_t)min(a0 + a, c1 - 1) * ND + ROW_Y + h * FH + k) : zero;
    }
    typename P::A wn[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) wn[u] = P::load(F, (size_t)min(m0 + wv + NWO * u, M - 1) * S);
    __syncthreads();
#pragma unroll 2
    for (int s = 0; s < S; ++s) {
      typename P::A wc[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        wc[u] = wn[u];
        wn[u] = P::load(F, (size_t)min(m0 + wv + NWO * u, M - 1) * S + min(s + 1, S - 1));
      }
#pragma unroll
      for (int at = 0; at < AT; ++at) {
        const typename P::B b = from_row<P>(sm.X[16 * at + c], s);
#pragma unroll
        for (int u = 0; u < 3; ++u) acc[at][u] = P::mma(wc[u], b, acc[at][u]);
      }
    }
  }
#pragma unroll
  for (int at = 0; at < AT; ++at) {
    const int a = min(a0 + 16 * at + c, c1 - 1);
    const float *T = Tsave + (size_t)a * M * 4;
    float *row = fit + (size_t)a * ND;
    f4 Ta[4], part[4] = {};  // the lane's axis rows a = 4 q + i
#pragma unroll
    for (int i = 0; i < 4; ++i) Ta[i] = ldf4(T + 4 * (4 * q + i));
    const bool ok = a0 + 16 * at + c < c1;
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int m = m0 + wv + NWO * u;
      if (m < m1) {
        const f4 Tm = ldf4(T + 4 * m);
        f4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v += acc[at][u][i] * Ta[i];
          part[i] += acc[at][u][i] * Tm;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          v[k] += __shfl_xor(v[k], 16);
          v[k] += __shfl_xor(v[k], 32);
        }
        if (q == 0 && ok) *reinterpret_cast<f4 *>(row + ROW_DT + 4 * m) = v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) sm.red[wv][l][4 * i + k] = part[i][k];
    __syncthreads();
    for (int x = threadIdx.x; x < 64 * 16; x += NWO * 64) {
      const int ll = x / 16, k = x % 16;
      float v = 0.f;
      for (int u = 0; u < NWO; ++u) v += sm.red[u][ll][k];
      const int aa = a0 + 16 * at + (ll & 15);  // entry 4 a + component, a = 4 q + i
      if (aa < c1) fit[(size_t)aa * ND + ROW_PART + blockIdx.y * 4 * M2 + 16 * (ll >> 4) + k] = v;
    }
  }
}

// From AT2_FROM atoms on, the products with F1 take 32 atoms per workgroup, which halves
// the weight traffic from L2; below it the smaller tiles keep more CUs busy.
constexpr int AT2_FROM = 4096;

template <class P>
void launch(const Tables &w, const Heads<P> &hd, const Workspace &ws, const int *types, int c0, int c1, bool backward,
            hipStream_t st) {
  const int n = c1 - c0, at = n >= AT2_FROM ? 2 : 1, tiles = (n + 16 * at - 1) / (16 * at);
  const dim3 gin(tiles, NHT / CTI, w.nheads), gout(tiles, NGO);
  if (at == 2) hipLaunchKernelGGL((k_fit_in<P, 2>), gin, dim3(NWI * 64), 0, st, w, hd, ws.Tsave, c0, c1, ws.fit);
  else hipLaunchKernelGGL((k_fit_in<P, 1>), gin, dim3(NWI * 64), 0, st, w, hd, ws.Tsave, c0, c1, ws.fit);
  hipLaunchKernelGGL((k_fit_mid<P>), dim3((n + 15) / 16), dim3(NHT * 64), 0, st, w, hd, types, c0, c1, ws.fit, ws.Ei,
                     ws.Eh, backward ? 1 : 0);
  if (!backward) return;
  if (at == 2) hipLaunchKernelGGL((k_fit_out<P, 2>), gout, dim3(NWO * 64), 0, st, w, hd, ws.Tsave, c0, c1, ws.fit);
  else hipLaunchKernelGGL((k_fit_out<P, 1>), gout, dim3(NWO * 64), 0, st, w, hd, ws.Tsave, c0, c1, ws.fit);
}

}  // namespace

void launch_fitting(const Weights<float> &w, const Workspace &ws, const int *types, int c0, int c1, bool backward,
                    hipStream_t st) {
  Heads<F32> hd{};
  for (int h = 0; h < w.nheads; ++h)
    hd.f[h] = {{w.F1T[h]}, {w.F2T[h]}, {w.F3T[h]}, {w.F1[h]}, {w.F2[h]}, {w.F3[h]}};
  launch<F32>(w, hd, ws, types, c0, c1, backward, st);
}

void launch_fitting_b16(const Tables &w, const WeightsB16 &wp, const Workspace &ws, const int *types, int c0, int c1,
                        bool backward, hipStream_t st) {
  Heads<B16> hd{};
  const auto m = [](const bf16_t *const (&p)[2]) { return B16::Mat{p[0], p[1]}; };
  for (int h = 0; h < w.nheads; ++h)
    hd.f[h] = {m(wp.F1T[h]), m(wp.F2T[h]), m(wp.F3T[h]), m(wp.F1[h]), m(wp.F2[h]), m(wp.F3[h])};
  launch<B16>(w, hd, ws, types, c0, c1, backward, st);
}

}  // namespace dp
