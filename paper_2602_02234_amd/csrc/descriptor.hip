// Per-atom descriptor kernels of the float32 path on gfx950: environment matrix,
// type-embedded embedding net, two gated self-attention layers over the atom's
// neighbours and the descriptor contraction (forward), and the hand-written backward
// that turns dE/dT into g_ij = dE_i/dDelta_ij.
//
// Model (paper, Section II: embedding net over an atom and its neighbours,
// self-attention layers updating that representation residually; sizes of the
// attention model studied here):
//   r = |Delta|, sw = quintic switch (1 below rcs, 0 from rc), s = sw / r,
//   rhat = Delta / r, Rt = (s, s rhat);
//   h1 = tanh(s w1s + B[t_i][t_j]) (type part of the first layer folded into B),
//   h2 = tanh(h1 W2 + b2) + [h1, h1], G = tanh(h2 W3 + b3) + [h2, h2];
//   per layer: S = G (WQ WK^T / sqrt d) G^T, P = sw-weighted row softmax of S,
//   A = P * (rhat_j . rhat_k), Y = A G (WV WO), G <- gamma LN(G + Y) + beta;
//   T = G^T Rt / sel, D = T T_<16^T.
// With one head and no projection biases, Q K^T = G (WQ WK^T) G^T and
// (A V) WO = (A G)(WV WO), so each layer needs the two 100x100 products only;
// they are formed once at model load.
//
// Bound: the float32 MFMA rate (157 TFLOP/s), then the weights' way through L1 in the forward, spills and
// the stages between barriers in the backward.  Per 16-neighbour block and layer the
// forward issues 668 and the backward 1,389 MFMAs 16x16x4 of 32 cycles at 96 neighbours.  Measured
// at 9,999 atoms: forward 1.86 ms (MFMAs alone 1.07), backward 4.42 ms; the step, which took 26.7 ms with
// kernels that passed every operand through LDS, 6.85 ms; 150 atoms, one to a CU: 66 and 144 us.
//
// Layout: one workgroup per atom, one wave per block of 16 neighbours (tokens).  A wave
// keeps everything that belongs to its tokens in registers, transposed (features or keys
// along the accumulator rows, its 16 tokens along the columns): lane (q = lane / 16,
// c = lane % 16) holds features 16 t + 4 q + i of token c.  In that form the accumulator
// of one product is, register by register, the B operand of the next (k step i of tile t
// takes k = 16 t + 4 q + i), so U, S, softmax, H, Y, LayerNorm and their gradients follow
// one another without a trip through LDS; softmax and LayerNorm reduce over registers and
// two lane exchanges.  Only the keys' rows G are shared: [token][100] float32 in LDS, a
// stride for which both the 16-byte row reads and the reads along tokens spread over all
// banks.  Weights come from L2 in fragment order, one output tile ahead.
//
// Instances (dp_desc.h): two atoms of up to 6 blocks (96 neighbours, nine in ten in water) to a
// workgroup of 12 waves with at most 168 registers, so that every SIMD has three; an atom of
// more to one of 8 waves, on a second stream.
#include "dp_desc.h"

namespace dp {
namespace {

constexpr int LDX = 68;   // row stride of a wave's transposition scratch [16 tokens][64]
constexpr int LDW = 20;   // ... of a 16 x 16 tile in it
static_assert(M == 100 && E1 == 25 && E2 == 50, "the fragment layouts below are written for these widths");

// out = W x (ADD: out += W x, summed by itself first) for a 100 x 100 matrix W[out][k] in fragment order: tile t (outputs
// 16 t + row for t < 6; 96 + row / 4 for t = 6) at 1600 t, its k = 16 kb + 4 q + s at
// + 256 kb + 4 lane + s, its k = 96 + q at + 1536 + lane.  The next tile's operands are
// loaded while the current one's 25 products run.
template <bool ADD = false>
__device__ __forceinline__ void wmul(F100 &out, const float *__restrict__ w, const F100 &x) {
  const int l = lane();
  f4 a[6];
  float at;
  const float *p = w + 4 * l;
#pragma unroll
  for (int kb = 0; kb < 6; ++kb) a[kb] = ldf4(p + 256 * kb);
  at = w[1536 + l];
#pragma unroll
  for (int t = 0; t < 7; ++t) {
    f4 b[6];
    float bt = 0.f;
    if (t < 6) {
#pragma unroll
      for (int kb = 0; kb < 6; ++kb) b[kb] = ldf4(p + 1600 * (t + 1) + 256 * kb);
      bt = w[1600 * (t + 1) + 1536 + l];
    }
    tile_barrier();
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 6; ++kb)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = mfma(a[kb][s], x[kb][s], acc);
    acc = mfma(at, x[6][0], acc);
    if (ADD) out[t] += acc;
    else out[t] = acc;
    if (t < 6) {
#pragma unroll
      for (int kb = 0; kb < 6; ++kb) a[kb] = b[kb];
      at = bt;
    }
  }
}

// s[kt] = G x over the keys of tile kt < nb: rows key 16 kt + 4 q + i, columns tokens.
template <int NB>
__device__ __forceinline__ void keys_dot(f4 (&s)[NB], const float *G, const F100 &x, int nb) {
  const int l = lane(), q = l >> 4, c = l & 15;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt) {
    s[kt] = f4{0.f, 0.f, 0.f, 0.f};
    if (kt < nb) {
      tile_barrier();
      const float *g = G + (16 * kt + c) * LDG;
      f4 a[6];
#pragma unroll
      for (int kb = 0; kb < 6; ++kb) a[kb] = ldf4(g + 16 * kb + 4 * q);
      const float at = g[96 + q];
#pragma unroll
      for (int kb = 0; kb < 6; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[kt] = mfma(a[kb][e], x[kb][e], s[kt]);
      s[kt] = mfma(at, x[6][0], s[kt]);
    }
  }
}

// acc = G^T y, y(kt)[i] the value of key 16 kt + 4 q + i, kt < nb.
template <int NB, class Y>
__device__ __forceinline__ void keys_sum(F100 &acc, const float *G, const Y &y, int nb) {
  const int l = lane(), q = l >> 4, c = l & 15;
#pragma unroll
  for (int t = 0; t < 7; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < NB; ++kt)
    if (kt < nb) {
      tile_barrier();
      const f4 v = y(kt);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        tile_barrier();
        const float *g = G + (16 * kt + 4 * q + s) * LDG;
        float a[7];
#pragma unroll
        for (int t = 0; t < 6; ++t) a[t] = g[16 * t + c];
        a[6] = g[96 + (c >> 2)];
#pragma unroll
        for (int t = 0; t < 7; ++t) acc[t] = mfma(a[t], v[s], acc[t]);
      }
    }
}

// out[og] = W in over NI input groups: tile it = 2 og + u at it NI 512, piece p at + 256 p.  With AHEAD
// the tiles' weights are loaded two tiles ahead, the first two by the constructor, which a caller
// runs early (32 NI registers).
template <int NI, int NO, bool AHEAD> struct Emul {
  f4 a[2][2 * NI];
  const float *w;
  __device__ __forceinline__ void fetch(f4 (&x)[2 * NI], int it) const {
#pragma unroll
    for (int p = 0; p < 2 * NI; ++p) x[p] = ldf4(w + (it * 2 * NI + p) * 256);
  }
  __device__ __forceinline__ explicit Emul(const float *__restrict__ wm) : w(wm + 4 * lane()) {
    if (AHEAD) {
      fetch(a[0], 0);
      fetch(a[1], 1);
    }
  }
  __device__ __forceinline__ void operator()(S7 (&out)[NO], const S7 (&in)[NI]) {
#pragma unroll
    for (int it = 0; it < 2 * NO; ++it) {
      f4 n[2 * NI];
      if (!AHEAD) fetch(a[it & 1], it);
      else if (it + 2 < 2 * NO) fetch(n, it + 2);
      tile_barrier();
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ig = 0; ig < NI; ++ig)
#pragma unroll
        for (int r = 0; r < 7; ++r) acc = mfma(a[it & 1][2 * ig + r / 4][r % 4], in[ig][r], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * (it & 1) + i < 7) out[it / 2][4 * (it & 1) + i] = acc[i];
      if (AHEAD && it + 2 < 2 * NO)
#pragma unroll
        for (int p = 0; p < 2 * NI; ++p) a[it & 1][p] = n[p];
    }
  }
};

// h1, t2 = h2 - [h1, h1] and t3 = G - [h2, h2] of the lane's token.
template <bool AHEAD>
__device__ __forceinline__ void embed(const Weights<float> &w, float s, int ti, int tj, S7 (&h1)[1], S7 (&t2)[2], S7 (&t3)[4]) {
  const int q = lane() >> 4;
  Emul<1, 2, AHEAD> e2(w.W2T);
  Emul<2, 4, AHEAD> e3(w.W3T);
  const float *bt = w.Bt + (ti * NTYPES + tj) * E1;
#pragma unroll
  for (int r = 0; r < 7; ++r) {
    const int f = slot_ok(r) ? 4 * r + q : 0;
    const float v = tanh_fast(s * w.w1s[f] + bt[f]);
    h1[0][r] = slot_ok(r) ? v : 0.f;
  }
  e2(t2, h1);
  S7 h2[2];
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      const int f = slot_ok(r) ? 25 * g + 4 * r + q : 0;
      const float v = tanh_fast(t2[g][r] + w.b2[f]);
      t2[g][r] = slot_ok(r) ? v : 0.f;
      h2[g][r] = t2[g][r] + h1[0][r];
    }
  e3(t3, h2);
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      const int f = slot_ok(r) ? 25 * g + 4 * r + q : 0;
      const float v = tanh_fast(t3[g][r] + w.b3[f]);
      t3[g][r] = slot_ok(r) ? v : 0.f;
    }
}

// ======================================================================== forward
template <int NB> struct SmemFwd {
  float G[16 * NB * LDG] __attribute__((aligned(16)));
  float part[NB][M * 4] __attribute__((aligned(16)));
  EnvF<NB> e;
};

template <int NB, int NA>
__device__ __forceinline__ void desc_fwd(int blk, int count, SmemFwd<NB> *smem, Weights<float> w, const double *__restrict__ X, const int *__restrict__ types, int natoms, const int *__restrict__ idx, int c0,
           const int *__restrict__ nlist, const int *__restrict__ nnei, const Grid *__restrict__ grids,
           const int *__restrict__ sys_of, float rc, float rcs, float ln_eps, float *__restrict__ Gsave,
           float *__restrict__ Tsave) {
  const Part<NB, NA> pt(blk, idx, c0, count, nnei);
  SmemFwd<NB> &sm = smem[pt.half];
  const int i = pt.i, n = pt.n, nb = pt.nb, jb = pt.jb, tid = pt.tid;
  const Grid g = grids[sys_of[i]];
  const int ti = clamp_type(types[i]);
  const int l = lane(), q = l >> 4, c = l & 15;
  const bool act = jb < nb;
  build_envf(sm.e, tid, X, types, nlist, i, n, natoms, g, rc, rcs);
  __syncthreads();
  const int j = 16 * jb + c;  // the lane's token
  float *row = sm.G + j * LDG;
  if (act) {
    S7 h1[1], t2[2], t3[4];
    embed<true>(w, sm.e.s[j], ti, sm.e.tj[j], h1, t2, t3);
    put_embedding(row, h1, t2, t3);
  }
  __syncthreads();
  const float hj[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
#pragma unroll 1
  for (int layer = 0; layer < NATTN; ++layer) {
    F100 y = {};
    if (act) {
      F100 x, u;
      get_row(x, row);
      wmul(u, w.WqkT[layer], x);  // U
      f4 s[NB];
      keys_dot<NB>(s, sm.G, u, nb);  // S = U G^T
      softmax_keys<NB>(s, sm.e, n, [](float v) { return expf(v); });
      // H = A G with A = sw E gate
      keys_sum<NB>(x, sm.G, [&](int kt) { return s[kt] * gate4(sm.e, kt, hj) * ldf4(sm.e.sw + 16 * kt + 4 * q); }, nb);
      wmul(y, w.WvoT[layer], x);     // Y, summed by itself and then added: starting from G would round at G's size
      get_row(x, row);
#pragma unroll
      for (int t = 0; t < 7; ++t) y[t] += x[t];
      // LayerNorm; the centred rows are what the backward reads
      const float mu = sum100([&](int t, int k) { return y[t][k]; }) / (float)M;
#pragma unroll
      for (int t = 0; t < 7; ++t) y[t] -= mu;
      save_block(Gsave + ((size_t)i * NATTN + layer) * GSAVE_LAYER + 1600 * jb, y);
      normalise(y, ln_eps);
      F100 ga, be;
      get_table(ga, w.gamma[layer]);
      get_table(be, w.beta[layer]);
#pragma unroll
      for (int t = 0; t < 7; ++t) y[t] = ga[t] * y[t] + be[t];
    }
    __syncthreads();  // every wave is done with the layer's input
    if (act) put_row(row, y);
    __syncthreads();
  }
  // T = G^T Rt / sel: each wave's 16 tokens on MFMA (T^T = Rt^T G, rows c < 4 of the 16
  // used, step s taking token 4 s + q), then the waves' parts in order
  if (act) {
    f4 acc[7];
#pragma unroll
    for (int t = 0; t < 7; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 16 * jb + 4 * s + q;
      const float sk = sm.e.s[k];
      const float rt = c == 0 ? sk : (c < 4 ? sk * sm.e.rh[c - 1][k] : 0.f);
      const float *gk = sm.G + k * LDG;
#pragma unroll
      for (int t = 0; t < 7; ++t) acc[t] = mfma(rt, gk[t < 6 ? 16 * t + c : 96 + (c & 3)], acc[t]);
    }
    if (q == 0)
#pragma unroll
      for (int t = 0; t < 7; ++t)
        if (t < 6 || c < 4) *reinterpret_cast<f4 *>(sm.part[jb] + 4 * (16 * t + c)) = acc[t];
  }
  __syncthreads();
  for (int k = tid; k < (nb ? M * 4 : 0); k += 64 * NB) {
    float acc = 0.f;
    for (int v = 0; v < nb; ++v) acc += sm.part[v][k];
    Tsave[(size_t)i * M * 4 + k] = acc / (float)SEL;
  }
}

// One workgroup per NA atoms of its instance's list; the 8-wave instance loops over its list
// with at most one workgroup per CU.
template <int NB, int NA>
__global__ void __launch_bounds__(64 * NB * NA) __attribute__((amdgpu_waves_per_eu(NB == NB_SMALL ? 3 : 2)))
k_desc_fwd(Weights<float> w, const double *__restrict__ X, const int *__restrict__ types, int natoms,
           const int *__restrict__ idx, const int *__restrict__ cnt, int c0, int ncen, const int *__restrict__ nlist,
           const int *__restrict__ nnei, const Grid *__restrict__ grids, const int *__restrict__ sys_of, float rc, float rcs,
           float ln_eps, float *__restrict__ Gsave, float *__restrict__ Tsave) {
  __shared__ SmemFwd<NB> smem[NA];
  const int count = idx ? *cnt : ncen;
  if constexpr (NB == NB_SMALL) {  // without the loop, which would keep its invariants in registers
    const int b = blockIdx.x;
    if (b * NA < count)
      desc_fwd<NB, NA>(b, count, smem, w, X, types, natoms, idx, c0, nlist, nnei, grids, sys_of, rc, rcs, ln_eps, Gsave, Tsave);
  } else {
    for (int b = blockIdx.x; b * NA < count; b += gridDim.x) {
      desc_fwd<NB, NA>(b, count, smem, w, X, types, natoms, idx, c0, nlist, nnei, grids, sys_of, rc, rcs, ln_eps, Gsave, Tsave);
      __syncthreads();
    }
  }
}

// ======================================================================== backward
template <int NB> struct SmemBwd {
  float G[16 * NB * LDG] __attribute__((aligned(16)));      // a layer's input, then dE/dG
  float scr[NB][16 * LDX] __attribute__((aligned(16)));     // per-wave transposition scratch
  float drhw[NB][16 * NB * 3];                              // each wave's column sums of dC rhat
  float drh[16 * NB * 3], dswa[16 * NB];
  float dRt[16 * NB * 4] __attribute__((aligned(16)));
  float dT[M * 4] __attribute__((aligned(16)));
  EnvF<NB> e;
};

// A wave's 16 x 100 block x as the A operand of products that contract over its tokens:
// o[t][s] = feature 16 t + c (t < 6) or 96 + c / 4 of token 4 q + s.
__device__ __forceinline__ void transpose_block(f4 (&o)[7], const F100 &x, float *scr) {
  const int l = lane(), q = l >> 4, c = l & 15;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    wave_sync();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (4 * h + t < 6) *reinterpret_cast<f4 *>(scr + c * LDX + 16 * t + 4 * q) = x[4 * h + t];
      if (4 * h + t == 6) scr[c * LDX + 16 * t + q] = x[6][0];
    }
    wave_sync();
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (4 * h + t < 6) o[4 * h + t][s] = scr[(4 * q + s) * LDX + 16 * t + c];
        if (4 * h + t == 6) o[6][s] = scr[(4 * q + s) * LDX + 16 * t + (c >> 2)];
      }
  }
  wave_sync();
}

// A key tile y (rows keys, columns tokens) as the B operand contracting over tokens:
// o[s] = y of token 4 q + s, key c.  scr: 16 x LDW floats.
__device__ __forceinline__ f4 transpose_tile(const f4 &y, float *scr) {
  const int l = lane(), q = l >> 4, c = l & 15;
  *reinterpret_cast<f4 *>(scr + c * LDW + 4 * q) = y;
  wave_sync();
  f4 o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o[s] = scr[(4 * q + s) * LDW + c];
  return o;
}

// Tile t of a per-feature table, in a token's arrangement.
__device__ __forceinline__ f4 tab4(const float *__restrict__ p, int t) {
  const int q = lane() >> 4;
  return t < 6 ? ldf4(p + 16 * t + 4 * q) : f4{p[96 + q], 0.f, 0.f, 0.f};
}

// Backward of one layer, its input rows in sm.G.  go: the gradient of the layer's output
// for the wave's tokens; saved: the layer's centred rows.  On return sm.G holds the
// gradient of the layer's input and every thread has passed a barrier.
//   Row part (per token j): dX through the LayerNorm, dH = Wvo dX; U, S, E recomputed;
//   dA = G dH, then per key P = sw E, dP = dA gate, rho = sum P dP, W = E (dP - rho),
//   dS = sw W, dU = G^T dS, and dG_j = dX + Wqk dU.
//   Column part (per key k): dG_k += sw_k sum_j (E gate)_jk dH_j + W_jk U_j and
//   dsw_k += sum_j W_jk.  In step p the wave of block j adds its tokens' share to key block
//   (j + p) mod nb; a barrier ends each step, so each sum has a fixed order.
template <int NB>
__device__ __forceinline__ void layer_bwd(const Weights<float> &w, int layer, SmemBwd<NB> &sm, F100 &go,
                                          const float *__restrict__ saved, int jb, int n, int nb, int steps,
                                          float ln_eps) {
  const int l = lane(), q = l >> 4, c = l & 15;
  const int j = 16 * jb + c;
  float *row = sm.G + j * LDG;
  float *scr = sm.scr[jb];
  F100 u, dh, dx;
  f4 E[NB], W[NB];
  const float hj[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
  {
    {  // LayerNorm backward: dX = (dxh - mean(dxh) - xh mean(dxh xh)) / sigma, dxh = gamma dG_out
      F100 xh;
      load_block(xh, saved + 1600 * jb);
      const float is = normalise(xh, ln_eps);
#pragma unroll
      for (int t = 0; t < 7; ++t) dx[t] = tab4(w.gamma[layer], t) * go[t];
      const float s0 = sum100([&](int t, int k) { return dx[t][k]; }) / (float)M;
      const float s1 = sum100([&](int t, int k) { return dx[t][k] * xh[t][k]; }) / (float)M;
#pragma unroll
      for (int t = 0; t < 7; ++t) dx[t] = (dx[t] - s0 - xh[t] * s1) * is;
    }
    wmul(dh, w.Wvo[layer], dx);
    {
      F100 x;
      get_row(x, row);
      wmul(u, w.WqkT[layer], x);
    }
    keys_dot<NB>(E, sm.G, u, nb);
    softmax_keys<NB>(E, sm.e, n, [](float v) { return expf(v); });
    keys_dot<NB>(W, sm.G, dh, nb);  // dA
    float rho = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
    // columns of dC rhat: sum_j rhat_j (dA E)_jk, A operand rhat of token 4 q + s in rows a < 3
    float rj[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) rj[s] = c < 3 ? sm.e.rh[c][16 * jb + 4 * q + s] : 0.f;
#pragma unroll
    for (int kt = 0; kt < NB; ++kt)
      if (kt < nb) {
        tile_barrier();
        const int k = 16 * kt + 4 * q;
        const f4 sw = ldf4(sm.e.sw + k), rx = ldf4(sm.e.rh[0] + k), ry = ldf4(sm.e.rh[1] + k), rz = ldf4(sm.e.rh[2] + k);
        const f4 gt = rx * hj[0] + ry * hj[1] + rz * hj[2];
        const f4 cc = W[kt] * E[kt];
        const f4 dC = sw * cc, dP = W[kt] * gt, pr = sw * E[kt] * dP;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          rho += pr[i];
          hx += dC[i] * rx[i];
          hy += dC[i] * ry[i];
          hz += dC[i] * rz[i];
        }
        W[kt] = dP;
        wave_sync();
        const f4 ct = transpose_tile(cc, scr);
        f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = mfma(rj[s], ct[s], acc);
        if (q == 0) {
          const float swk = sm.e.sw[16 * kt + c];
          float *o = sm.drhw[jb] + 3 * (16 * kt + c);
          o[0] = swk * acc[0]; o[1] = swk * acc[1]; o[2] = swk * acc[2];
        }
      }
    rho = sumq(rho);
    hx = sumq(hx); hy = sumq(hy); hz = sumq(hz);
    if (q == 0) {
      sm.drh[3 * j] += hx; sm.drh[3 * j + 1] += hy; sm.drh[3 * j + 2] += hz;
    }
    F100 du;
    keys_sum<NB>(du, sm.G, [&](int kt) {
      W[kt] = E[kt] * (W[kt] - rho);
      return ldf4(sm.e.sw + 16 * kt + 4 * q) * W[kt];  // dS
    }, nb);
    wmul<true>(dx, w.Wqk[layer], du);
  }
  __syncthreads();  // the layer's input is no longer needed
  f4 ut[7], ht[7];
  {
    put_row(row, dx);
    transpose_block(ut, u, scr);
    transpose_block(ht, dh, scr);
    // rows 4 q' + 1 of tile 6 collect sum_j W_jk
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if ((c & 3) == 1) {
        ut[6][s] = 1.f;
        ht[6][s] = 0.f;
      }
    }
  }
#pragma unroll 1
  for (int p = 0; p < steps; ++p) {
    __syncthreads();
    if (p < nb) {
      int kb = jb + p;
      if (kb >= nb) kb -= nb;
      wave_sync();
#pragma unroll
      for (int kt = 0; kt < NB; ++kt)
        if (kt == kb) {
          *reinterpret_cast<f4 *>(scr + c * LDW + 4 * q) = E[kt] * gate4(sm.e, kt, hj);
          *reinterpret_cast<f4 *>(scr + 16 * LDW + c * LDW + 4 * q) = W[kt];
        }
      wave_sync();
      f4 ya, yw;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        ya[s] = scr[(4 * q + s) * LDW + c];
        yw[s] = scr[16 * LDW + (4 * q + s) * LDW + c];
      }
      F100 acc = {};
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 7; ++t) acc[t] = mfma(ht[t][s], ya[s], acc[t]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 7; ++t) acc[t] = mfma(ut[t][s], yw[s], acc[t]);
      const int k = 16 * kb + c;
      const float swk = sm.e.sw[k];
      float *gk = sm.G + k * LDG;
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        f4 *o = reinterpret_cast<f4 *>(gk + 16 * t + 4 * q);
        *o = *o + swk * acc[t];
      }
      gk[96 + q] += swk * acc[6][0];
      if (q == 0) sm.dswa[k] += acc[6][1];
    }
  }
  __syncthreads();
  if (q < 3) {  // the wave's keys: component q of their gate gradients
    float v = sm.drh[3 * j + q];
    for (int u2 = 0; u2 < nb; ++u2) v += sm.drhw[u2][3 * j + q];
    sm.drh[3 * j + q] = v;
  }
}

template <int NB, int NA>
__device__ __forceinline__ void desc_bwd(int blk, int count, SmemBwd<NB> *smem, Weights<float> w, const double *__restrict__ X, const int *__restrict__ types, int natoms, const int *__restrict__ idx, int c0,
           const int *__restrict__ nlist, const int *__restrict__ nnei, const Grid *__restrict__ grids,
           const int *__restrict__ sys_of, float rc, float rcs, float ln_eps, const float *__restrict__ Gsave,
           const float *__restrict__ fit, float4 *__restrict__ gout) {
  const Part<NB, NA> pt(blk, idx, c0, count, nnei);
  SmemBwd<NB> &sm = smem[pt.half];
  const int i = pt.i, n = pt.n, nb = pt.nb, jb = pt.jb, tid = pt.tid;
  const Grid g = grids[sys_of[i]];
  const int ti = clamp_type(types[i]);
  const int l = lane(), q = l >> 4, c = l & 15;
  const float *gs = Gsave + (size_t)i * NATTN * GSAVE_LAYER;
  build_envf(sm.e, tid, X, types, nlist, i, n, natoms, g, rc, rcs);
  for (int k = tid; k < 16 * NB; k += 64 * NB) {
    sm.dswa[k] = 0.f;
    for (int a = 0; a < 3; ++a) sm.drh[3 * k + a] = 0.f;
  }
  const float *dTi = fit + (size_t)i * ND;
  for (int k = tid; k < M * 4; k += 64 * NB) {
    float v = dTi[FIT_DT + k];
    if (k < 4 * M2)
      for (int p = 0; p < FIT_NPART; ++p) v += dTi[FIT_PART + 4 * M2 * p + k];
    sm.dT[k] = v;
  }
  for (int k = nb ? 16 * nb + tid : SEL; k < SEL; k += 64 * NB) gout[(size_t)i * SEL + k] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  // A wave without tokens only passes the others' barriers, on a path of its own, so that no register
  // of their work is carried past a branch around it.
  if (jb >= nb) {
    for (int k = 0; k < 2 * (pt.steps + 2) + 4; ++k) __syncthreads();
    return;
  }
  const int j = 16 * jb + c;
  float *row = sm.G + j * LDG;
  F100 go;
  {
    F100 x;
    // the top layer's input: layer 0's output
    load_block(x, gs + 1600 * jb);
    normalise(x, ln_eps);
#pragma unroll
    for (int t = 0; t < 7; ++t) x[t] = tab4(w.gamma[0], t) * x[t] + tab4(w.beta[0], t);
    put_row(row, x);
    // dG = Rt dT^T / sel for its output, and dRt = G dT / sel
    load_block(x, gs + GSAVE_LAYER + 1600 * jb);
    normalise(x, ln_eps);
    const float sj = sm.e.s[j];
    const float rt1 = sj * sm.e.rh[0][j], rt2 = sj * sm.e.rh[1][j], rt3 = sj * sm.e.rh[2][j];
    f4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 7; ++t) {
      tile_barrier();
      const f4 gv = tab4(w.gamma[1], t) * x[t] + tab4(w.beta[1], t);
#pragma unroll
      for (int k = 0; k < (t < 6 ? 4 : 1); ++k) {
        const f4 d = ldf4(sm.dT + 4 * (t < 6 ? 16 * t + 4 * q + k : 96 + q));
        go[t][k] = (sj * d[0] + rt1 * d[1] + rt2 * d[2] + rt3 * d[3]) / (float)SEL;
        p += gv[k] * d;
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) p[a] = sumq(p[a]) / (float)SEL;
    if (q == 0) *reinterpret_cast<f4 *>(sm.dRt + 4 * j) = p;
  }
  __syncthreads();
  layer_bwd<NB>(w, 1, sm, go, gs + GSAVE_LAYER, jb, n, nb, pt.steps, ln_eps);
  get_row(go, row);
  __syncthreads();
  {
    S7 h1[1], t2[2], t3[4];
    embed<(NB > NB_SMALL)>(w, sm.e.s[j], ti, sm.e.tj[j], h1, t2, t3);
    put_embedding(row, h1, t2, t3);
  }
  __syncthreads();
  layer_bwd<NB>(w, 0, sm, go, gs, jb, n, nb, pt.steps, ln_eps);
  __syncthreads();
  // embedding backward and the pair gradients of the wave's tokens
  {
    S7 h1[1], t2[2], t3[4];
    embed<(NB > NB_SMALL)>(w, sm.e.s[j], ti, sm.e.tj[j], h1, t2, t3);
    tile_barrier();
    Emul<4, 2, (NB > NB_SMALL)> e3(w.W3);
    S7 dh2[2], d[4];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
      for (int r = 0; r < 7; ++r) {
        const float v = slot_ok(r) ? row[25 * g4 + 4 * r + q] : 0.f;
        d[g4][r] = v;
        t3[g4][r] = v * (1.f - t3[g4][r] * t3[g4][r]);  // dpre3
      }
    e3(dh2, t3);
    tile_barrier();
    Emul<2, 1, true> e2(w.W2);
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2)
#pragma unroll
      for (int r = 0; r < 7; ++r) {
        dh2[g2][r] += d[g2][r] + d[g2 + 2][r];
        t2[g2][r] = dh2[g2][r] * (1.f - t2[g2][r] * t2[g2][r]);  // dpre2
      }
    S7 dh1[1];
    e2(dh1, t2);
    float ds = 0.f;
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      const float v = dh1[0][r] + dh2[0][r] + dh2[1][r];
      if (slot_ok(r)) ds += v * (1.f - h1[0][r] * h1[0][r]) * w.w1s[4 * r + q];
    }
    ds = sumq(ds);
    if (q == 0 && j < SEL) {
      float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
      if (j < n) {
        const float h[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
        out = pair_gradient(sm.e.s[j], sm.e.sw[j], sm.e.r[j], h, ds, sm.dRt + 4 * j, sm.drh + 3 * j, sm.dswa[j], rc, rcs);
      }
      gout[(size_t)i * SEL + j] = out;
    }
  }
}

// One workgroup per NA atoms of its instance's list; the 8-wave instance loops over its list
// with at most one workgroup per CU.
template <int NB, int NA>
__global__ void __launch_bounds__(64 * NB * NA) __attribute__((amdgpu_waves_per_eu(NB == NB_SMALL ? 3 : 2)))
k_desc_bwd(Weights<float> w, const double *__restrict__ X, const int *__restrict__ types, int natoms,
           const int *__restrict__ idx, const int *__restrict__ cnt, int c0, int ncen, const int *__restrict__ nlist,
           const int *__restrict__ nnei, const Grid *__restrict__ grids, const int *__restrict__ sys_of, float rc, float rcs,
           float ln_eps, const float *__restrict__ Gsave, const float *__restrict__ fit, float4 *__restrict__ gout) {
  __shared__ SmemBwd<NB> smem[NA];
  const int count = idx ? *cnt : ncen;
  if constexpr (NB == NB_SMALL) {  // without the loop, which would keep its invariants in registers
    const int b = blockIdx.x;
    if (b * NA < count)
      desc_bwd<NB, NA>(b, count, smem, w, X, types, natoms, idx, c0, nlist, nnei, grids, sys_of, rc, rcs, ln_eps, Gsave, fit, gout);
  } else {
    for (int b = blockIdx.x; b * NA < count; b += gridDim.x) {
      desc_bwd<NB, NA>(b, count, smem, w, X, types, natoms, idx, c0, nlist, nnei, grids, sys_of, rc, rcs, ln_eps, Gsave, fit, gout);
      __syncthreads();
    }
  }
}

// Lists the centres c0 .. c1-1 for the two instances, one addition per wave and instance
// (one per atom, in the neighbour search, cost 30 us at 3,000 atoms).  The order only
// changes scheduling.
__global__ void __launch_bounds__(256) k_class_lists(const int *__restrict__ nnei, int c0, int c1, int *__restrict__ idx,
                                                     int *__restrict__ cnt, int cap) {
  const int i = c0 + blockIdx.x * 256 + threadIdx.x;
  const int l = lane_id();
  const bool small = i < c1 && nnei[i] <= 16 * NB_SMALL;
  for (int cls = 0; cls < 2; ++cls) {
    const unsigned long long mask = __ballot(i < c1 && small == (cls == 0));
    if (!mask) continue;
    const int first = __ffsll(mask) - 1;
    int base = 0;
    if (l == first) base = atomicAdd(cnt + cls, __popcll(mask));
    base = __shfl(base, first);
    const int pos = base + __popcll(mask & ((1ull << l) - 1ull));
    if ((mask >> l & 1ull) && pos < cap) idx[(size_t)cls * cap + pos] = i;
  }
}

}  // namespace

void launch_descriptor_lists(const Workspace &ws, int n, int c0, int c1, hipStream_t st) {
  if (n >= PAIR_FROM)
    hipLaunchKernelGGL(k_class_lists, dim3((c1 - c0 + 255) / 256), dim3(256), 0, st, ws.nnei, c0, c1, ws.bidx, ws.bcnt,
                       (int)ws.cap);
}

void launch_descriptor_fwd(const Weights<float> &w, const Workspace &ws, const double *coords, const int *types, int n,
                           int c0, int c1, float rc, float rcs, float ln_eps, hipStream_t st) {
  launch_descriptor_lists(ws, n, c0, c1, st);
  launch_instances(ws, n, c1 - c0, k_desc_fwd<NB_SMALL, 2>, k_desc_fwd<8, 1>, st,
                   [&](auto kernel, int groups, int threads, const int *idx, const int *cnt, hipStream_t s) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(threads), 0, s, w, coords, types, n, idx, cnt, c0, c1 - c0, ws.nlist,
                       ws.nnei, ws.grids, ws.sys_of, rc, rcs, ln_eps, ws.Gsave, ws.Tsave);
  });
}

void launch_descriptor_bwd(const Weights<float> &w, const Workspace &ws, const double *coords, const int *types, int n,
                           int c0, int c1, float rc, float rcs, float ln_eps, hipStream_t st) {
  launch_instances(ws, n, c1 - c0, k_desc_bwd<NB_SMALL, 2>, k_desc_bwd<8, 1>, st,
                   [&](auto kernel, int groups, int threads, const int *idx, const int *cnt, hipStream_t s) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(threads), 0, s, w, coords, types, n, idx, cnt, c0, c1 - c0, ws.nlist,
                       ws.nnei, ws.grids, ws.sys_of, rc, rcs, ln_eps, ws.Gsave, ws.fit, ws.g);
  });
}

}  // namespace dp
