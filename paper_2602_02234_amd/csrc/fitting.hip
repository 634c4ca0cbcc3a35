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
// Bound: at few atoms the latency of the weight loads (L2) and of the chain of four hidden products,
// at many the instructions around the products (the entries of D, splitting them in two bf16 terms)
// and the reading of the weights, with the matrix cores a third busy.  Measured against one kernel for
// the whole net (forward and backward): float32 150 atoms 594 -> 53 us, 9,999 atoms 1.81 -> 0.28 ms;
// bfloat16 192 atoms 80 -> 34 us, 24,999 atoms 0.48 -> 0.38 ms, where the descriptor kernels gain
// another 0.16 ms by neither writing D nor contracting dE/dD.  Of that: hidden activations split where
// they are written instead of by each wave that reads them, k_fit_mid 23 -> 14 us (192 atoms) and, with
// 32 atoms per workgroup, 163 -> 93 us (24,999); loads of a workgroup's rows issued together.
//
// Both precisions share the kernels.  F32: 16x16x4 float32 products.  B16: the energy is
// read off this net directly, so its products carry the bfloat16 path's largest rounding
// sensitivity; each runs on bf16 MFMA with both operands split into two bf16 terms,
// x = x_hi + x_lo, and three products x_hi w_hi + x_hi w_lo + x_lo w_hi accumulated in
// fp32 (the dropped lo*lo term is 2^-16 relative).
#include "dp_tiles.h"

namespace dp {
namespace {

constexpr int KH = 256;      // hidden width padded along k
constexpr int LDA = KH + 4;  // LDS row stride (floats) of hidden activations
constexpr int LDB = KH + 8;  // ... (bf16) of their hi and lo parts
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

__device__ __forceinline__ bf8 ldb8(const bf16_t *p) { return *reinterpret_cast<const bf8 *>(p); }

// A precision: k steps of KS, a lane holding PER consecutive k of a step (k = KS s + PER q
// + e), A fragments of the weights, B operands made from float32 values, and rows of hidden
// activations in LDS, kept as B operands (split once, where they are written: every wave reads them).
struct F32 {
  static constexpr int KS = 16, PER = 4, KHS = FH / KS;  // KHS: steps over the hidden width
  static constexpr int MID = 1;  // atom tiles of k_fit_mid in large systems
  struct Mat { const float *p; };
  struct Fin { Mat F1T, F2T, F3T, F1, F2, F3; };
  struct A { f4 v; };
  struct B { f4 v; };
  static __device__ __forceinline__ A load(const Mat &m, size_t frag) { return {ldf4(m.p + frag * 256 + 4u * (unsigned)lane())}; }
  static __device__ __forceinline__ B make(const f4 (&x)[1]) { return {x[0]}; }
  template <int R> struct Rows {
    float v[R][LDA] __attribute__((aligned(16)));
    __device__ __forceinline__ void put(int row, int k, f4 x) { stf4(&v[row][k], x); }
    __device__ __forceinline__ B get(int row, int s) const { return {ldf4(&v[row][KS * s + PER * (lane_id() >> 4)])}; }
  };
  static __device__ __forceinline__ f4 mma(const A &a, const B &b, f4 acc) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[s], b.v[s], acc, 0, 0, 0);
    return acc;
  }
};
struct B16 {
  static constexpr int KS = 32, PER = 8, KHS = KH / KS;
  static constexpr int MID = 2;
  struct Mat { const bf16_t *hi, *lo; };
  struct Fin { Mat F1T, F2T, F3T, F1, F2, F3; };
  struct A { bf8 h, l; };
  struct B { bf8 h, l; };
  static __device__ __forceinline__ A load(const Mat &m, size_t frag) {
    const unsigned o = 8u * (unsigned)lane();
    return {ldb8(m.hi + frag * 512 + o), ldb8(m.lo + frag * 512 + o)};
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
  template <int R> struct Rows {
    typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
    bf16_t h[R][LDB] __attribute__((aligned(16))), l[R][LDB] __attribute__((aligned(16)));
    __device__ __forceinline__ void put(int row, int k, f4 x) {
      bf4 a, b;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = (__bf16)x[e];
        b[e] = (__bf16)(x[e] - (float)a[e]);
      }
      *reinterpret_cast<bf4 *>(&h[row][k]) = a;
      *reinterpret_cast<bf4 *>(&l[row][k]) = b;
    }
    __device__ __forceinline__ B get(int row, int s) const {
      const int k = KS * s + PER * (lane_id() >> 4);
      return {ldb8(&h[row][k]), ldb8(&l[row][k])};
    }
  };
  static __device__ __forceinline__ f4 mma(const A &a, const B &b, f4 acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, acc, 0, 0, 0);
  }
};

template <class P> struct Heads { typename P::Fin f[MAXH]; };

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
  const int l = lane_id(), q = l >> 4, c = l & 15, wv = __builtin_amdgcn_readfirstlane(wave_id());
  const typename P::Mat F = hd.f[h].F1T;
  constexpr int NC = 16 * AT * M, RC = (NC + NWI * 64 - 1) / (NWI * 64);
  f4 tv[RC];  // all rows on their way before the first is stored
#pragma unroll
  for (int r = 0; r < RC; ++r) {
    const int x = min((int)threadIdx.x + r * NWI * 64, NC - 1);
    tv[r] = ldf4(Tsave + ((size_t)min(a0 + x / M, c1 - 1) * M + x % M) * 4);
  }
  typename P::A wn[CTI];
#pragma unroll
  for (int u = 0; u < CTI; ++u) wn[u] = P::load(F, (size_t)(t0 + u) * S + wv);
#pragma unroll
  for (int r = 0; r < RC; ++r) {
    const int x = threadIdx.x + r * NWI * 64;
    if (x < NC) stf4(&sm.T[x / M][4 * (x % M)], tv[r]);
  }
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
template <class P, int AT>
__global__ void __launch_bounds__(NHT * 64) k_fit_mid(Tables w, Heads<P> hd, const int *__restrict__ types, int c0, int c1,
                                                      float *__restrict__ fit, double *__restrict__ Ei,
                                                      double *__restrict__ Eh, int backward) {
  __shared__ typename P::template Rows<16 * AT> X[2];  // columns 240 .. 255 stay zero
  __shared__ double ep[16 * AT][16];
  constexpr int S = P::KHS, H = (S + 1) / 2;
  const int a0 = c0 + blockIdx.x * 16 * AT;
  const int l = lane_id(), q = l >> 4, c = l & 15, t = __builtin_amdgcn_readfirstlane(wave_id());
  const int col = 16 * t + 4 * q;  // the lane's hidden units col .. col + 3, of the atoms a0 + 16 at + c
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  for (int x = threadIdx.x; x < 2 * 16 * AT * 4; x += NHT * 64) X[x / (64 * AT)].put(x / 4 % (16 * AT), FH + 4 * (x % 4), zero);
  double esum = 0.0;
  // The first half of a matrix is loaded ahead of a barrier, the second while the first is used: both ahead
  // take half of the registers (the bfloat16 instance with 32 atoms spills 16 as it is).
  const auto weights = [&](const typename P::Mat &m, typename P::A (&wf)[H]) {
#pragma unroll
    for (int s = 0; s < H; ++s) wf[s] = P::load(m, (size_t)t * S + s);
  };
  const auto product = [&](const typename P::Mat &m, const typename P::A (&wf)[H], int b, f4 (&acc)[AT]) {
    typename P::A wl[S - H];
#pragma unroll
    for (int s = H; s < S; ++s) wl[s - H] = P::load(m, (size_t)t * S + s);
    tile_barrier();
#pragma unroll
    for (int at = 0; at < AT; ++at) acc[at] = zero;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (s % 4 == 0) tile_barrier();
#pragma unroll
      for (int at = 0; at < AT; ++at) acc[at] = P::mma(s < H ? wf[s % H] : wl[s < H ? 0 : s - H], X[b].get(16 * at + c, s), acc[at]);
    }
    tile_barrier();
  };
  for (int h = 0; h < w.nheads; ++h) {
    const float hw = (float)w.hw[h];
    const auto row = [&](int at) { return fit + (size_t)min(a0 + 16 * at + c, c1 - 1) * ND + ROW_Y + h * FH + col; };
    typename P::A wf[H];
    weights(hd.f[h].F2T, wf);
    f4 y1[AT], y2[AT], t2[AT], acc[AT];
#pragma unroll
    for (int at = 0; at < AT; ++at) {
      y1[at] = ldf4(row(at));
      X[0].put(16 * at + c, col, y1[at]);
    }
    __syncthreads();
    product(hd.f[h].F2T, wf, 0, acc);
    weights(hd.f[h].F3T, wf);
    const f4 b2 = ldf4(w.c2[h] + col), b3 = ldf4(w.c3[h] + col), F4 = ldf4(w.F4[h] + col);
#pragma unroll
    for (int at = 0; at < AT; ++at) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        t2[at][i] = tanhf(acc[at][i] + b2[i]);
        y2[at][i] = t2[at][i] + y1[at][i];
      }
      X[1].put(16 * at + c, col, y2[at]);
    }
    __syncthreads();
    product(hd.f[h].F3T, wf, 1, acc);
    const bool bwd = backward && w.hw[h] != 0.0;
    if (bwd) weights(hd.f[h].F3, wf);
    // E_i = y3 . F4 + c4 + ebias in float64
#pragma unroll
    for (int at = 0; at < AT; ++at) {
      double p = 0.0;
      f4 d;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float t3 = tanhf(acc[at][i] + b3[i]);
        p += (double)(t3 + y2[at][i]) * w.F4d[h][col + i];
        d[i] = hw * F4[i] * (1.f - t3 * t3);  // dE/dpre3
      }
      p += __shfl_xor(p, 16);
      p += __shfl_xor(p, 32);
      if (q == 0) ep[16 * at + c][t] = p;
      X[0].put(16 * at + c, col, d);
    }
    __syncthreads();
    if ((int)threadIdx.x < 16 * AT && a0 + (int)threadIdx.x < c1) {
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
      f4 dy2[AT];
      product(hd.f[h].F3, wf, 0, dy2);
      weights(hd.f[h].F2, wf);
#pragma unroll
      for (int at = 0; at < AT; ++at) {
        dy2[at] += hw * F4;
        X[1].put(16 * at + c, col, dy2[at] * (1.f - t2[at] * t2[at]));
      }
      __syncthreads();
      // dy1 = dpre2 F2^T + dy2;  dpre1 = dy1 (1 - y1^2)
      product(hd.f[h].F2, wf, 1, acc);
#pragma unroll
      for (int at = 0; at < AT; ++at)
        if (a0 + 16 * at + c < c1) stf4(row(at), (acc[at] + dy2[at]) * (1.f - y1[at] * y1[at]));
    }
    __syncthreads();  // the next head overwrites X and ep
  }
  if ((int)threadIdx.x < 16 * AT && a0 + (int)threadIdx.x < c1) Ei[a0 + threadIdx.x] = esum;
}

// ------------------------------------------------------------ dE/dT
// dT_m = sum_a dD_ma T_a + [m < 16] sum_m' dD_m'm T_m'; the second sum is left as one part
// per workgroup, added up by the descriptor backward.
template <class P, int AT>
__global__ void __launch_bounds__(NWO * 64) k_fit_out(Tables w, Heads<P> hd, const float *__restrict__ Tsave, int c0, int c1,
                                                      float *__restrict__ fit) {
  __shared__ union {
    typename P::template Rows<16 * AT> X;
    float red[AT][NWO][64][16 + 1];
  } sm __attribute__((aligned(16)));
  constexpr int S = P::KHS;
  const int a0 = c0 + blockIdx.x * 16 * AT;
  const int m0 = blockIdx.y * MGO, m1 = min(M, m0 + MGO);
  const int l = lane_id(), q = l >> 4, c = l & 15, wv = __builtin_amdgcn_readfirstlane(wave_id());
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  f4 acc[AT][3] = {};
  for (int h = 0; h < w.nheads; ++h) {
    if (w.hw[h] == 0.0) continue;
    const typename P::Mat F = hd.f[h].F1;
    constexpr int NX = 16 * AT * (KH / 4), RX = (NX + NWO * 64 - 1) / (NWO * 64);
    f4 xv[RX];
#pragma unroll
    for (int r = 0; r < RX; ++r) {
      const int x = min((int)threadIdx.x + r * NWO * 64, NX - 1), k = 4 * (x % (KH / 4));
      xv[r] = ldf4(fit + (size_t)min(a0 + x / (KH / 4), c1 - 1) * ND + ROW_Y + h * FH + min(k, FH - 4));
    }
    typename P::A wn[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) wn[u] = P::load(F, (size_t)min(m0 + wv + NWO * u, M - 1) * S);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RX; ++r) {
      const int x = threadIdx.x + r * NWO * 64, k = 4 * (x % (KH / 4));
      if (x < NX) sm.X.put(x / (KH / 4), k, k < FH ? xv[r] : zero);
    }
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
        const typename P::B b = sm.X.get(16 * at + c, s);
#pragma unroll
        for (int u = 0; u < 3; ++u) acc[at][u] = P::mma(wc[u], b, acc[at][u]);
      }
    }
  }
  // the rows of T of both tiles, on their way together
  f4 Ta[AT][4], Tm[AT][3];  // the lane's axis rows a = 4 q + i, and the wave's rows m
#pragma unroll
  for (int at = 0; at < AT; ++at) {
    const float *T = Tsave + (size_t)min(a0 + 16 * at + c, c1 - 1) * M * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) Ta[at][i] = ldf4(T + 4 * (4 * q + i));
#pragma unroll
    for (int u = 0; u < 3; ++u) Tm[at][u] = ldf4(T + 4 * min(m0 + wv + NWO * u, M - 1));
  }
  __syncthreads();
#pragma unroll
  for (int at = 0; at < AT; ++at) {
    const int a = a0 + 16 * at + c;
    f4 part[4] = {};
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int m = m0 + wv + NWO * u;
      if (m < m1) {
        f4 v = zero;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v += acc[at][u][i] * Ta[at][i];
          part[i] += acc[at][u][i] * Tm[at][u];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = sumq(v[k]);
        if (q == 0 && a < c1) stf4(fit + (size_t)a * ND + ROW_DT + 4 * m, v);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) sm.red[at][wv][l][4 * i + k] = part[i][k];
  }
  __syncthreads();
  for (int x = threadIdx.x; x < AT * 64 * 16; x += NWO * 64) {
    const int at = x / 1024, ll = x / 16 % 64, k = x % 16;
    float v = 0.f;
    for (int u = 0; u < NWO; ++u) v += sm.red[at][u][ll][k];
    const int aa = a0 + 16 * at + (ll & 15);  // entry 4 a + component, a = 4 q + i
    if (aa < c1) fit[(size_t)aa * ND + ROW_PART + blockIdx.y * 4 * M2 + 16 * (ll >> 4) + k] = v;
  }
}

// From AT2_FROM atoms on, 32 atoms per workgroup: that halves the weight traffic from L2, and k_fit_mid,
// one workgroup per CU, would otherwise go over the chip a second time; below it the smaller tiles keep
// more CUs busy.  k_fit_mid in float32 stays at 16 (9,999 atoms: 74 us, with 32 atoms 90 us: matrix
// instructions bound it, and its registers spill).
constexpr int AT2_FROM = 4096;

template <class P>
void launch(const Tables &w, const Heads<P> &hd, const Workspace &ws, const int *types, int c0, int c1, bool backward,
            hipStream_t st) {
  const int n = c1 - c0, at = n >= AT2_FROM ? 2 : 1, tiles = (n + 16 * at - 1) / (16 * at);
  const dim3 gin(tiles, NHT / CTI, w.nheads), gout(tiles, NGO);
  const auto go = [&](auto A, auto AM) {
    hipLaunchKernelGGL((k_fit_in<P, A()>), gin, dim3(NWI * 64), 0, st, w, hd, ws.Tsave, c0, c1, ws.fit);
    hipLaunchKernelGGL((k_fit_mid<P, AM()>), dim3((n + 16 * AM() - 1) / (16 * AM())), dim3(NHT * 64), 0, st, w, hd, types, c0,
                       c1, ws.fit, ws.Ei, ws.Eh, backward ? 1 : 0);
    if (backward)
      hipLaunchKernelGGL((k_fit_out<P, A()>), gout, dim3(NWO * 64), 0, st, w, hd, ws.Tsave, c0, c1, ws.fit);
  };
  if (at == 2) go(std::integral_constant<int, 2>{}, std::integral_constant<int, P::MID>{});
  else go(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
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
