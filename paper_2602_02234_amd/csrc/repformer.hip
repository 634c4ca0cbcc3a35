// Repformer-style model kernels for gfx950: one launch per layer, forward and backward (a
// layer's pair update and convolution read the neighbours' g1 of the layer before, so
// layers meet at launch boundaries).
//
// A wave owns a block of 16 of the centre's neighbours (tokens) and keeps all that belongs to
// them in registers, transposed (dp_tiles.h): the pair update, its query, the scores of its
// tokens as queries against every key, softmax, the attention output, and their gradients.
// Only what other waves read goes through LDS: the keys' rows K and V, and, in the backward,
// the gradients that meet at a key.  The products run on MFMA (16x16x4 f32).
//   forward   g2a = g2 + tanh([g2, g1_j] Wa + ba); Q, K, V; E = exp(S - max) / Z over the keys;
//             g2 <- g2a + sum_k sw_k E gate V_k; T = sum_j g2_j R_j^T and the convolution sums;
//             the node update (the last layer's into dnl, where the fitting net takes it).
//   backward  the same recomputed but for the layer's output, which is stored; per token j
//             dA = V dY, per key P = sw E, dP = dA gate, rho = sum P dP, W = E (dP - rho),
//             dQ = K^T (sw W) / sqrt 32; per key k dV_k = sw_k sum_j E gate dY_j, dK_k = sw_k sum_j
//             W Q_j / sqrt 32, dsw_k = sum_j W: the wave reads its column of the tiles of E gate
//             and W, which the waves of all blocks leave in LDS.
// Every sum has a fixed order: results are deterministic.
//
// Up to ONE_UP_TO atoms each has a workgroup of 8 waves; above, atoms of up to 6 blocks go two
// to a workgroup of 12 waves, so that every SIMD has three (a second group of 6 waves is never
// placed beside the first: each brings two waves to the same two SIMDs, and 168 registers
// leave room for three), and atoms of 7 or 8 blocks take 8 of the 12.
// Bound: matrix cores, then the latency of the stages between barriers.  At 96 neighbours
// a forward layer has 1,250 MFMAs of 32 cycles per atom (0.16 ms at 9,999 atoms on 256 CUs), a
// backward layer 2,900 (0.38 ms).  Measured at 9,999 atoms of chain density, per layer: 0.93 ->
// 0.39 .. 0.42 ms forward, 1.97 -> 0.76 .. 0.87 ms backward, against kernels that staged every product's
// operands in LDS and had one atom per CU; at 768 atoms 76 -> 42 .. 45 and 157 -> 82 .. 88 us.
#include <algorithm>

#include "dp_env.h"
#include "dp_tiles.h"
#include "repformer.h"

namespace dp {
namespace rep {
namespace {

constexpr int LK = G2D + 4;   // row stride of the keys' rows in LDS: row reads and reads along keys without conflicts
constexpr int PMAT = 3072;     // floats of one of the pair matrices Pa, Pqkv, Pqkvt, Pat (which lie in this order)
constexpr int NB_SMALL = 6;   // blocks up to which two atoms share a workgroup of 12 waves
constexpr int NB_MAX = 8;     // blocks of the longest list
constexpr int ONE_UP_TO = 256;  // atoms up to which each has a workgroup (and a CU) of its own
constexpr int NLONG = 256;    // workgroups of 12 waves that take the longer lists: one per CU

__device__ __forceinline__ f4 mfma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// The part of a workgroup's work a wave takes: NA atoms (entries blk NA .. of the list, or
// atom blk without one), NB waves each.  Past the end of the list nb = 0; steps is the largest nb, so that
// the waves of both atoms pass the same barriers.
template <int NB, int NA> struct Part {
  int half, jb, tid, i, n, nb, steps;
  __device__ __forceinline__ Part(int blk, const int *__restrict__ idx, int count, const int *__restrict__ nnei) {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));  // as lane()
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    half = NA == 1 ? 0 : wv / NB;
    jb = wv - half * NB;
    tid = t - half * 64 * NB;
    steps = 0;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const int k = idx ? idx[min(blk * NA + a, count - 1)] : blk;
      const int nk = min(max(nnei[k], 0), SEL);
      const int b = blk * NA + a < count ? min(nk > 0 ? (nk + 15) / 16 : 1, NB) : 0;
      steps = max(steps, b);
      if (a == half) {
        i = k;
        n = nk;
        nb = b;
      }
    }
  }
};

// Environment of one atom, padded to whole blocks (s = sw = dsw = 0, r = 1, rhat = 0 past the list).
template <int NB> struct EnvN {
  float sw[16 * NB] __attribute__((aligned(16)));
  float rh[3][16 * NB] __attribute__((aligned(16)));
  float r[16 * NB], dsw[16 * NB], s[16 * NB];
  int jn[16 * NB], tj[16 * NB];
};

template <int NB>
__device__ void build_envn(EnvN<NB> &e, int tid, const double *__restrict__ X, const int *__restrict__ types,
                           const int *__restrict__ nlist, int i, int nn, int n, const Grid &g, const Geo &geo) {
  for (int j = tid; j < 16 * NB; j += 64 * NB) {
    float r = 1.f, sw = 0.f, dsw = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
    int nj = i, tj = 0;
    if (j < nn) {
      nj = nlist[(size_t)i * SEL + j];
      if (nj < 0 || nj >= n) nj = i;
      tj = clamp_type(types[nj]);
      double d[3];
      for (int a = 0; a < 3; ++a) {
        double v = X[3 * nj + a] - X[3 * i + a];
        if (g.periodic) v -= g.L[a] * rint(v * g.invL[a]);
        d[a] = v;
      }
      const float dx = (float)d[0], dy = (float)d[1], dz = (float)d[2];
      r = sqrtf(dx * dx + dy * dy + dz * dz);
      const float u = (r - geo.rcs) / (geo.rc - geo.rcs);
      if (r < geo.rcs) {
        sw = 1.f;
      } else if (r < geo.rc) {
        sw = u * u * u * (-6.f * u * u + 15.f * u - 10.f) + 1.f;
        dsw = -30.f * u * u * (1.f - u) * (1.f - u) / (geo.rc - geo.rcs);
      }
      hx = dx / r; hy = dy / r; hz = dz / r;
    }
    e.sw[j] = sw; e.dsw[j] = dsw; e.r[j] = r; e.s[j] = sw / r;
    e.rh[0][j] = hx; e.rh[1][j] = hy; e.rh[2][j] = hz;
    e.jn[j] = nj; e.tj[j] = tj;
  }
}

__device__ __forceinline__ size_t erow2(const Buffers &b, int l, int i, int j) {
  return (((size_t)l * b.cap + i) * SEL + j) * G2D;
}

// The layer's input of token j: x = [g2 (2 tiles), g1 of the neighbour (4 tiles)], zero past the list.
template <int NB>
__device__ __forceinline__ void token_in(const Weights &w, const Buffers &b, const EnvN<NB> &e, int l, int i, int j,
                                         int nn, f4 (&x)[6]) {
  const int q = lane() >> 4;
  if (j < nn) {
    const float *g1 = l == 0 ? w.TN + e.tj[j] * G1D : b.g1f + ((size_t)(l - 1) * b.cap + e.jn[j]) * G1D;
#pragma unroll
    for (int t = 0; t < 4; ++t) x[2 + t] = ldf4(g1 + 16 * t + 4 * q);
#pragma unroll
    for (int t = 0; t < 2; ++t)
      x[t] = l == 0 ? init4<tanhf>(e.s[j], w.Wp0 + 16 * t + 4 * q, w.bp0 + 16 * t + 4 * q) : ldf4(b.g2f + erow2(b, l - 1, i, j) + 16 * t + 4 * q);
  } else {
#pragma unroll
    for (int t = 0; t < 6; ++t) x[t] = f4{0.f, 0.f, 0.f, 0.f};
  }
}

// out[t] = W_t x + bias (16 t + 4 q ..) for a product with NT output tiles.
template <int NK, int NT>
__device__ __forceinline__ void product(f4 (&out)[NT], const float *__restrict__ wf, const f4 (&x)[NK]) {
  const X<float, NK> xo(x);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    W<float, NK> wt;
    wt.load(wf, t);
    out[t] = wt(xo, out[t]);
  }
}

// W x with x = [g2, g1_j], the 32 features of g2 and the halves of g1_j each summed by themselves: shorter
// sums round less, and g1_j's rounding, alike in all neighbours of one type (in the first layer
// its parts take five values), does not average out.  The virial cancels to a twelfth of its terms and shows it: in one
// sum, started from the bias, its error over 8 boxes of 192 atoms was 4.9e-7 of it in the mean, in parts 0.8e-7 .. 2.6e-7 (with
// either form of tanh).
__device__ __forceinline__ f4 sum_of_parts(const W<float, 6> &wt, const f4 (&x)[6]) {
  f4 p[3] = {};
#pragma unroll
  for (int k = 0; k < 6; ++k)
#pragma unroll
    for (int s = 0; s < 4; ++s) p[k / 2] = mfma(wt.v[k][s], x[k][s], p[k / 2]);
  return p[0] + (p[1] + p[2]);
}

// Pair update and projections of the lane's token: ta = tanh([g2, g1_j] Wa + ba), g2a = g2 + ta,
// q its query; its key and value rows go to LDS.  wl: Pa and Pqkv in LDS.
__device__ __forceinline__ void pair_and_qkv(const Weights &w, const float *wl, int l, const f4 (&x)[6], f4 (&ta)[2],
                                             f4 (&g2a)[2], f4 (&qr)[2], float *Krow, float *Vrow) {
  const int q = lane() >> 4;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    W<float, 6> wt;
    wt.load(wl, t);
    const f4 z = sum_of_parts(wt, x) + ldf4(w.ba[l] + 16 * t + 4 * q);
    ta[t] = act(z);
    g2a[t] = x[t] + ta[t];
  }
  f4 qkv[6] = {};
  product<2, 6>(qkv, wl + PMAT, g2a);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    qr[t] = qkv[t];
    stf4(Krow + 16 * t + 4 * q, qkv[2 + t]);
    stf4(Vrow + 16 * t + 4 * q, qkv[4 + t]);
  }
}

// s[kt] = (rows of R) x for key tile kt < nb: rows key 16 kt + 4 q + i, columns tokens.
template <int NB>
__device__ __forceinline__ void keys_dot(f4 (&s)[NB], const float *R, const f4 (&x)[2], int nb) {
  const int q = lane() >> 4, c = lane() & 15;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt) {
    s[kt] = f4{0.f, 0.f, 0.f, 0.f};
    if (kt < nb)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const f4 a = ldf4(R + (16 * kt + c) * LK + 16 * t + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[kt] = mfma(a[e], x[t][e], s[kt]);
      }
  }
}
// acc = R^T y, y(kt)[i] the value of key 16 kt + 4 q + i, kt < nb.
template <int NB, class Y>
__device__ __forceinline__ void keys_sum(f4 (&acc)[2], const float *R, const Y &y, int nb) {
  const int q = lane() >> 4, c = lane() & 15;
  acc[0] = acc[1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < NB; ++kt)
    if (kt < nb) {
      const f4 v = y(kt);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = mfma(R[(16 * kt + 4 * q + s) * LK + 16 * t + c], v[s], acc[t]);
    }
}

// E = exp((S - max) / sqrt 32) / Z over the keys in place of the scores (0 past the list), with
// Z = sum_k sw_k exp(...).
template <int NB>
__device__ __forceinline__ void softmax_keys(f4 (&s)[NB], const EnvN<NB> &e, int n) {
  const int q = lane() >> 4;
  const float isq = 0.17677669529663687f;  // 1 / sqrt(32)
  float m = -INFINITY;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[kt][i] = 16 * kt + 4 * q + i < n ? s[kt][i] * isq : -INFINITY;
      m = fmaxf(m, s[kt][i]);
    }
  m = maxq(m);
  if (m == -INFINITY) m = 0.f;
  float z = 0.f;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt) {
    const f4 sw = ldf4(e.sw + 16 * kt + 4 * q);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[kt][i] = __expf(s[kt][i] - m);
      z += sw[i] * s[kt][i];
    }
  }
  z = sumq(z);
  const float iz = z > 0.f ? 1.f / z : 0.f;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt) s[kt] *= iz;
}

// A block's rows x (16 tokens x 32 features) with the token along the lane group: o[t][s] =
// feature 16 t + c of token 4 q + s.  scr: [16][LK].
__device__ __forceinline__ void transpose_block(f4 (&o)[2], const f4 (&x)[2], float *scr) {
  const int q = lane() >> 4, c = lane() & 15;
  wave_sync();
#pragma unroll
  for (int t = 0; t < 2; ++t) stf4(scr + c * LK + 16 * t + 4 * q, x[t]);
  wave_sync();
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int s = 0; s < 4; ++s) o[t][s] = scr[(4 * q + s) * LK + 16 * t + c];
  wave_sync();
}
// The node update's W1 (224 x 64) in the registers of a workgroup of NW waves, a quarter-wave to a
// row: row 4 (wave + NW r) + q, columns 4 c ..  One load serves every atom of the workgroup,
// and W1 x and W1^T dz alike.
template <int NW> struct NodeW {
  static constexpr int R = (XD / 4 + NW - 1) / NW;
  f4 w[R];
  int wave;
  __device__ __forceinline__ int row(int r) const { return 4 * (wave + NW * r) + (lane() >> 4); }
  __device__ __forceinline__ NodeW(const float *__restrict__ W1, int wv) : wave(wv) {
#pragma unroll
    for (int r = 0; r < R; ++r) w[r] = row(r) < XD ? ldf4(W1 + row(r) * G1D + 4 * (lane() & 15)) : f4{0.f, 0.f, 0.f, 0.f};
  }
  // The wave's part of sum_k x[k] W1[k][:], to part[64].
  __device__ __forceinline__ void forward(const float *x, float *part) const {
    f4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < R; ++r) v += x[min(row(r), XD - 1)] * w[r];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = sumq(v[i]);
    if (lane() < 16) stf4(part + 4 * lane(), v);
  }
  // dx[k] = sum_o W1[k][o] dz[o] for the wave's rows.
  __device__ __forceinline__ void backward(const float *dz, float *dx) const {
    const f4 z = ldf4(dz + 4 * (lane() & 15));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float v = dp::sum16(fmaf(w[r][0], z[0], w[r][1] * z[1]) + fmaf(w[r][2], z[2], w[r][3] * z[3]));
      if ((lane() & 15) == 0 && row(r) < XD) dx[row(r)] = v;
    }
  }
};

// The wave's share of T^T = sum_j R_j g2_j^T (4 x 32) and of the convolution sums c = sum_j
// sw_j g2_j * g1_j[:32]: 5 rows of 32 in part.  The A operand has R in rows a < 4 and ones in row 4.
template <int NB>
__device__ __forceinline__ void node_parts(const EnvN<NB> &e, int jb, const f4 (&g2)[2], const f4 (&g1)[2], float *scr,
                                           float (*part)[G2D]) {
  const int q = lane() >> 4, c = lane() & 15;
  f4 gt[2], pt[2], p[2], acc[2] = {};
  const float swj = e.sw[16 * jb + c];
#pragma unroll
  for (int t = 0; t < 2; ++t) p[t] = swj * g2[t] * g1[t];
  transpose_block(gt, g2, scr);
  transpose_block(pt, p, scr);
  const float one = c == 4 ? 1.f : 0.f;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int j = 16 * jb + 4 * q + s;
    const float r = c == 0 ? e.s[j] : (c < 4 ? e.s[j] * e.rh[c < 4 ? max(c - 1, 0) : 0][j] : 0.f);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      acc[t] = mfma(r, gt[t][s], acc[t]);
      acc[t] = mfma(one, pt[t][s], acc[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (q == 0)
#pragma unroll
      for (int a = 0; a < 4; ++a) part[a][16 * t + c] = acc[t][a];
    if (q == 1) part[4][16 * t + c] = acc[t][0];
  }
}

// T[m][a] and the node-update input xs = [g1_i, D, c] with D = T T[:4]^T, from the waves' shares
// (added in order).  Passes three barriers, the first before the shares are read.
template <int NB>
__device__ __forceinline__ void node_inputs(int tid, int nb, const float (*part)[5][G2D], const float *g1i, float inv_sel,
                                            float *T, float *xs) {
  __syncthreads();
  if (tid < 5 * G2D) {
    const int a = tid / G2D, m = tid % G2D;
    float v = 0.f;
    for (int u = 0; u < nb; ++u) v += part[u][a][m];
    if (a < 4) T[4 * m + a] = v * inv_sel;
    else xs[G1D + G2D * NAX + m] = v * inv_sel;
  } else if (tid >= 5 * G2D && tid < 5 * G2D + G1D) {
    xs[tid - 5 * G2D] = g1i[tid - 5 * G2D];
  }
  __syncthreads();
  if (tid < G2D * NAX) {
    const int c = tid >> 2, bb = tid & 3;  // D[c][b], flattened c * 4 + b
    float v = 0.f;
    for (int a = 0; a < 4; ++a) v += T[c * 4 + a] * T[bb * 4 + a];
    xs[G1D + tid] = v;
  }
  __syncthreads();
}

// ------------------------------------------------------------------ forward
template <int NB> struct SmemF {
  EnvN<NB> e;
  float K[16 * NB * LK] __attribute__((aligned(16)));
  float V[16 * NB * LK] __attribute__((aligned(16)));
  float scr[NB][16 * LK] __attribute__((aligned(16)));
  float part[NB][5][G2D];
  float T[G2D * 4];
  float zp[2 * NB_SMALL][G1D] __attribute__((aligned(16)));  // the waves' parts of the node update
  float g1i[G1D], xs[XD];
};

template <int NB, int NA>
__device__ __forceinline__ void layer_fwd(int blk, int count, SmemF<NB> *smem, float *wl, const Weights &w, const Buffers &b,
                                          const double *__restrict__ Xc, const int *__restrict__ types,
                                          const int *__restrict__ nlist, const int *__restrict__ nnei,
                                          const Grid *__restrict__ grids, int natoms, int l, const Geo &geo,
                                          const int *__restrict__ idx) {
  const Part<NB, NA> pt(blk, idx, count, nnei);
  SmemF<NB> &sm = smem[pt.half];
  const int i = pt.i, nn = pt.n, nb = pt.nb, jb = pt.jb, tid = pt.tid;
  const int ln = lane(), q = ln >> 4, c = ln & 15;
  const bool act_ = jb < nb, live = nb > 0;
  const Copy16<PMAT / 2, 64 * NB * NA> cw(w.Pa[l]);
  build_envn<NB>(sm.e, tid, Xc, types, nlist, i, nn, natoms, grids[0], geo);
  if (tid < G1D)
    sm.g1i[tid] = l == 0 ? w.TN[clamp_type(types[i]) * G1D + tid] : b.g1f[((size_t)(l - 1) * b.cap + i) * G1D + tid];
  cw.store(wl);
  __syncthreads();
  const int j = 16 * jb + c;
  f4 x[6], ta[2], g2a[2], qr[2];
  if (act_) {
    token_in<NB>(w, b, sm.e, l, i, j, nn, x);
    pair_and_qkv(w, wl, l, x, ta, g2a, qr, sm.K + j * LK, sm.V + j * LK);
  }
  const NodeW<NA * NB> w1(w.W1[l], pt.half * NB + jb);
  tile_barrier();
  __syncthreads();
  if (act_) {
    f4 s[NB], y[2];
    keys_dot<NB>(s, sm.K, qr, nb);
    softmax_keys<NB>(s, sm.e, nn);
    const float hx = sm.e.rh[0][j], hy = sm.e.rh[1][j], hz = sm.e.rh[2][j];
    keys_sum<NB>(y, sm.V, [&](int kt) {
      const int k = 16 * kt + 4 * q;
      return s[kt] * ldf4(sm.e.sw + k) * (hx * ldf4(sm.e.rh[0] + k) + hy * ldf4(sm.e.rh[1] + k) + hz * ldf4(sm.e.rh[2] + k));
    }, nb);
    f4 g1[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      y[t] += g2a[t];
      g1[t] = x[2 + t];
      if (j < nn) stf4(b.g2f + erow2(b, l, i, j) + 16 * t + 4 * q, y[t]);
    }
    node_parts<NB>(sm.e, jb, y, g1, sm.scr[jb], sm.part[jb]);
  }
  node_inputs<NB>(tid, nb, sm.part, sm.g1i, geo.inv_sel, sm.T, sm.xs);
#pragma unroll
  for (int a = 0; a < NA; ++a) w1.forward(smem[a].xs, smem[a].zp[w1.wave]);
  __syncthreads();
  const size_t li = (size_t)l * b.cap + i;
  if (tid < G1D) {
    float z = w.b1[l][tid];
#pragma unroll
    for (int u = 0; u < NA * NB; ++u) z += sm.zp[u][tid];
    const float t = tanhf(z);
    if (live) b.tn[li * G1D + tid] = t;
    if (live) (l < NLAYER - 1 ? b.g1f + li * G1D : b.dnl + (size_t)i * G1D)[tid] = sm.g1i[tid] + t;
  }
  if (live && tid < 4 * G2D) b.Tn[li * (4 * G2D) + tid] = sm.T[tid];
}

// ------------------------------------------------------------------ backward
template <int NB> struct SmemB {
  EnvN<NB> e;
  float K[16 * NB * LK] __attribute__((aligned(16)));  // the keys' rows, then the queries'
  float V[16 * NB * LK] __attribute__((aligned(16)));  // the values' rows, then those of dY
  float tile[NB][NB][256] __attribute__((aligned(16)));  // E gate, then W: tokens' block, keys' block
  float drhw[NB][16 * NB * 3];  // each wave's column sums of dC rhat
  float T[G2D * 4];
  float dT[G2D * 4] __attribute__((aligned(16)));
  float dxn[XD] __attribute__((aligned(16)));
  float dg1[G1D], zz[G1D] __attribute__((aligned(16)));
  float rows[NB][G1D] __attribute__((aligned(16)));
  int slot[16 * NB];
};

template <int NB, int NA>
__device__ __forceinline__ void layer_bwd(int blk, int count, SmemB<NB> *smem, const Weights &w, const Buffers &b,
                                          const double *__restrict__ Xc, const int *__restrict__ types,
                                          const int *__restrict__ nlist, const int *__restrict__ nnei,
                                          const Grid *__restrict__ grids, int natoms, int l, const Geo &geo,
                                          const int *__restrict__ idx, float4 *__restrict__ gout) {
  const Part<NB, NA> pt(blk, idx, count, nnei);
  SmemB<NB> &sm = smem[pt.half];
  constexpr int NT = 64 * NB;
  const int i = pt.i, nn = pt.n, nb = pt.nb, jb = pt.jb, tid = pt.tid;
  const int ln = lane(), q = ln >> 4, c = ln & 15;
  const bool act_ = jb < nb, live = nb > 0, top = l == NLAYER - 1;
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  const float isq = 0.17677669529663687f;
  float *wl = &smem[0].tile[0][0][0];  // the tiles' place, until the scores
  const Copy16<PMAT / 2, 64 * NB * NA> cw(w.Pa[l]);
  build_envn<NB>(sm.e, tid, Xc, types, nlist, i, nn, natoms, grids[0], geo);
  for (int k = tid; k < 16 * NB; k += NT) sm.slot[k] = !top && k < nn ? b.slot[(size_t)i * SEL + k] : -1;
  const size_t li = (size_t)l * b.cap + i;
  float tn = 0.f, dni = 0.f;
  if (tid < G1D) {
    tn = b.tn[li * G1D + tid];
    dni = b.dnl[(size_t)i * G1D + tid];
  }
  if (tid < 4 * G2D) sm.T[tid] = b.Tn[li * (4 * G2D) + tid];
  cw.store(wl);
  __syncthreads();
  const int j = 16 * jb + c;
  const bool ok = act_ && j < nn;
  // dE/dg1_i after this layer: the neighbours' edge parts, sixteen lanes a row, the row groups in
  // turn through the list and added in order
  constexpr int G = 4 * NB, R = 4;
  f4 v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = (tid >> 4) + G * r, sk = sm.slot[k];
    v[r] = sk >= 0 ? ldf4(b.dnj + (size_t)((l + 1) & 1) * b.cap * SEL * G1D + ((size_t)sm.e.jn[k] * SEL + sk) * G1D + 4 * c) : zero;
  }
  // the layer's forward again: pair update, projections; its output is stored
  f4 ta[2], qr[2], g1[2], g2b[2], dy[2];
  if (act_) {
    f4 x[6], g2a[2];
    token_in<NB>(w, b, sm.e, l, i, j, nn, x);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      g2b[t] = ok ? ldf4(b.g2f + erow2(b, l, i, j) + 16 * t + 4 * q) : zero;
      dy[t] = ok && !top ? ldf4(b.dg2 + ((size_t)i * SEL + j) * G2D + 16 * t + 4 * q) : zero;
      g1[t] = x[2 + t];
    }
    pair_and_qkv(w, wl, l, x, ta, g2a, qr, sm.K + j * LK, sm.V + j * LK);
  }
  {
    f4 dn = v[0] + v[1] + v[2] + v[3];
#pragma unroll
    for (int k = 0; k < 4; ++k) dn[k] = sumq(dn[k]);
    if (q == 0) stf4(sm.rows[jb] + 4 * c, dn);
  }
  const NodeW<NA * NB> w1(w.W1[l], pt.half * NB + jb);
  tile_barrier();
  __syncthreads();
  // node backward: dz = dg1 (1 - t^2), dxn = W1 dz, and meanwhile the tokens' softmax
  if (tid < G1D) {
#pragma unroll
    for (int u = 0; u < NB; ++u) dni += sm.rows[u][tid];
    sm.dg1[tid] = dni;
    sm.zz[tid] = dni * (1.f - tn * tn);
  }
  f4 E[NB], Wg[NB], dq[2];
  if (act_) {
    keys_dot<NB>(E, sm.K, qr, nb);
    softmax_keys<NB>(E, sm.e, nn);
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < NA; ++a) w1.backward(smem[a].zz, smem[a].dxn);
  __syncthreads();
  // dT from dD = dxn[64:192] (D[c][b] = sum_a T[c][a] T[b][a], b < 4), then / sel; the sums over c
  // of the b < 4 rows by the whole first wave
  if (tid < G2D * 4) {
    const int m = tid >> 2, a = tid & 3;
    float d = 0.f;
    for (int bb = 0; bb < 4; ++bb) d += sm.dxn[G1D + m * 4 + bb] * sm.T[bb * 4 + a];
    if (jb == 0) {
      float u = 0.f;
#pragma unroll
      for (int k = 0; k < G2D / 4; ++k) u += sm.dxn[G1D + (4 * k + q) * 4 + (c >> 2)] * sm.T[(4 * k + q) * 4 + a];
      u = sumq(u);
      if (tid < 16) d += u;
    }
    sm.dT[tid] = d * geo.inv_sel;
  }
  __syncthreads();
  const float *dc = sm.dxn + G1D + G2D * NAX;  // dE/dc (times sel: divided where used)
  // the token's gradients: dE/dg2 of the output, and of s, sw and rhat (eg)
  float eg[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
  const float hj[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
  if (act_) {
    const float sj = sm.e.s[j], swj = sm.e.sw[j];
    f4 dR = zero;
    float dswc = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f4 dcv = ldf4(dc + 16 * t + 4 * q) * geo.inv_sel;
      dy[t] += swj * dcv * g1[t];
      const f4 pc = dcv * g2b[t] * g1[t];
      dswc += (pc[0] + pc[1]) + (pc[2] + pc[3]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f4 d = ldf4(sm.dT + 4 * (16 * t + 4 * q + k));
        dy[t][k] += sj * (d[0] + d[1] * hj[0] + d[2] * hj[1] + d[3] * hj[2]);
        dR += g2b[t][k] * d;
      }
    }
    dswc = sumq(dswc);
#pragma unroll
    for (int a = 0; a < 4; ++a) dR[a] = sumq(dR[a]);
    eg[0] = dR[0] + dR[1] * hj[0] + dR[2] * hj[1] + dR[3] * hj[2];
    eg[1] = dswc;
#pragma unroll
    for (int a = 0; a < 3; ++a) eg[2 + a] = sj * dR[1 + a];
    // the tokens as queries
    keys_dot<NB>(Wg, sm.V, dy, nb);  // dA
    float rho = 0.f, h0 = 0.f, h1 = 0.f, h2 = 0.f, rj[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) rj[s] = c < 3 ? sm.e.rh[c][16 * jb + 4 * q + s] : 0.f;
#pragma unroll
    for (int kt = 0; kt < NB; ++kt)
      if (kt < nb) {
        tile_barrier();
        const int k = 16 * kt + 4 * q;
        const f4 sw = ldf4(sm.e.sw + k), rx = ldf4(sm.e.rh[0] + k), ry = ldf4(sm.e.rh[1] + k), rz = ldf4(sm.e.rh[2] + k);
        const f4 cc = Wg[kt] * E[kt], dC = sw * cc, gate = rx * hj[0] + ry * hj[1] + rz * hj[2];
        const f4 dP = Wg[kt] * gate, pr = sw * E[kt] * dP;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          rho += pr[s];
          h0 += dC[s] * rx[s];
          h1 += dC[s] * ry[s];
          h2 += dC[s] * rz[s];
        }
        Wg[kt] = dP;
        // columns of dC rhat: sum_j rhat_j (dA E)_jk
        float *tile = sm.tile[jb][kt];
        put_tile(tile, cc);
        wave_sync();
        const f4 ct = get_tile(tile);
        wave_sync();
        put_tile(tile, E[kt] * gate);
        f4 acc = zero;
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = mfma(rj[s], ct[s], acc);
        if (q == 0) {
          const float swk = sm.e.sw[16 * kt + c];
          float *o = sm.drhw[jb] + 3 * (16 * kt + c);
          o[0] = swk * acc[0]; o[1] = swk * acc[1]; o[2] = swk * acc[2];
        }
      }
    rho = sumq(rho);
    eg[2] += sumq(h0);
    eg[3] += sumq(h1);
    eg[4] += sumq(h2);
    keys_sum<NB>(dq, sm.K, [&](int kt) {
      Wg[kt] = E[kt] * (Wg[kt] - rho);
      return ldf4(sm.e.sw + 16 * kt + 4 * q) * Wg[kt] * isq;  // dS
    }, nb);
  }
  // the tokens as keys: the wave reads its column of tiles and the rows of every block
  const auto column = [&](const float *rows, auto use, f4 (&acc)[2]) {
    acc[0] = acc[1] = zero;
#pragma unroll
    for (int jt = 0; jt < NB; ++jt) {
      if (jt >= nb) continue;
      const f4 y = get_tile(sm.tile[jt][jb]);
      use(y);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = mfma(rows[(16 * jt + 4 * q + s) * LK + 16 * t + c], y[s], acc[t]);
    }
  };
  f4 dk[2], dv[2];
  float wsum = 0.f;
  __syncthreads();
  if (act_)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      stf4(sm.K + j * LK + 16 * t + 4 * q, qr[t]);
      stf4(sm.V + j * LK + 16 * t + 4 * q, dy[t]);
    }
  __syncthreads();
  const Copy16<PMAT / 2, 64 * NB * NA> ct(w.Pqkvt[l]);
  if (act_) column(sm.V, [](f4) {}, dv);
  __syncthreads();
  ct.template store<0, PMAT / 4>(smem[0].V);  // the rows of dY are no longer needed
  if (NA == 2) ct.template store<PMAT / 4, PMAT / 2>(smem[NA - 1].V);
  if (act_)
#pragma unroll
    for (int kt = 0; kt < NB; ++kt)
      if (kt < nb) put_tile(sm.tile[jb][kt], Wg[kt]);
  __syncthreads();
  if (!act_) {
    if (l > 0 && live && tid < G1D) b.dnl[(size_t)i * G1D + tid] = sm.dg1[tid] + sm.dxn[tid];
    return;
  }
  column(sm.K, [&](f4 y) { wsum += (y[0] + y[1]) + (y[2] + y[3]); }, dk);
  // the token's key terms, then the projections and the pair update backward
  eg[1] += sumq(wsum);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float v = 0.f;
    for (int u = 0; u < nb; ++u) v += sm.drhw[u][3 * j + a];
    eg[2 + a] += v;
  }
  f4 dqkv[6], dg[2], dz[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    dqkv[t] = dq[t];
    dqkv[2 + t] = sm.e.sw[j] * isq * dk[t];
    dqkv[4 + t] = sm.e.sw[j] * dv[t];
    dg[t] = zero;
  }
  product<6, 2>(dg, smem[0].V, dqkv);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    dg[t] += dy[t];  // dE/dg2a
    dz[t] = dg[t] * (1.f - ta[t] * ta[t]);
  }
  f4 dx[6] = {};
  if (NA == 2) product<2, 6>(dx, smem[NA - 1].V, dz);
  else product<2, 6>(dx, w.Pat[l], dz);
#pragma unroll
  for (int t = 0; t < 2; ++t) dg[t] += dx[t];  // dE/dg2 of the layer's input
  if (l > 0) {
    if (ok) {
      float *dst = b.dnj + (size_t)(l & 1) * b.cap * SEL * G1D + ((size_t)i * SEL + j) * G1D + 4 * q;
      const float sc = sm.e.sw[j] * geo.inv_sel;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        stf4(b.dg2 + ((size_t)i * SEL + j) * G2D + 16 * t + 4 * q, dg[t]);
        stf4(dst + 16 * t, dx[2 + t] + sc * ldf4(dc + 16 * t + 4 * q) * g2b[t]);
        stf4(dst + 32 + 16 * t, dx[4 + t]);
      }
      if (q == 0) {
        float *g = b.gs + ((size_t)i * SEL + j) * GSN;
#pragma unroll
        for (int a = 0; a < 5; ++a) g[a] = top ? eg[a] : g[a] + eg[a];
      }
    }
    if (tid < G1D) b.dnl[(size_t)i * G1D + tid] = sm.dg1[tid] + sm.dxn[tid];
    return;
  }
  // layer 0: g2 = tanh(s Wp0 + bp0) adds to dE/ds; then g_ij = dE/dDelta_ij
  float ds = 0.f;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const f4 g0 = init4<tanhf>(sm.e.s[j], w.Wp0 + 16 * t + 4 * q, w.bp0 + 16 * t + 4 * q);
    const f4 g = dg[t] * (1.f - g0 * g0) * ldf4(w.Wp0 + 16 * t + 4 * q);
    ds += (g[0] + g[1]) + (g[2] + g[3]);
  }
  ds = sumq(ds);
  if (ok && q == 0) {
    const float *g = b.gs + ((size_t)i * SEL + j) * GSN;
#pragma unroll
    for (int a = 0; a < 5; ++a) eg[a] += g[a];
    ds += eg[0];
    const float rr = sm.e.r[j], sw = sm.e.sw[j];
    const float dr = ds * (sm.e.dsw[j] / rr - sw / (rr * rr)) + eg[1] * sm.e.dsw[j];
    const float proj = eg[2] * hj[0] + eg[3] * hj[1] + eg[4] * hj[2];
    gout[(size_t)i * SEL + j] = make_float4((eg[2] - proj * hj[0]) / rr + dr * hj[0], (eg[3] - proj * hj[1]) / rr + dr * hj[1],
                                            (eg[4] - proj * hj[2]) / rr + dr * hj[2], 0.f);
  }
}

// One atom per workgroup, any list length.
__global__ void __launch_bounds__(64 * NB_MAX) __attribute__((amdgpu_waves_per_eu(2)))
k_rep_fwd_one(Weights w, Buffers b, const double *__restrict__ Xc, const int *__restrict__ types,
              const int *__restrict__ nlist, const int *__restrict__ nnei, const Grid *__restrict__ grids, int n, int l,
              Geo geo, const unsigned *__restrict__ flags) {
  __shared__ SmemF<NB_MAX> sm;
  __shared__ float wl[2 * PMAT] __attribute__((aligned(16)));
  if (failed(flags)) return;
  layer_fwd<NB_MAX, 1>(blockIdx.x, n, &sm, wl, w, b, Xc, types, nlist, nnei, grids, n, l, geo, nullptr);
}
__global__ void __launch_bounds__(64 * NB_MAX) __attribute__((amdgpu_waves_per_eu(2)))
k_rep_bwd_one(Weights w, Buffers b, const double *__restrict__ Xc, const int *__restrict__ types,
              const int *__restrict__ nlist, const int *__restrict__ nnei, const Grid *__restrict__ grids, int n, int l,
              Geo geo, float4 *__restrict__ gout, const unsigned *__restrict__ flags) {
  __shared__ SmemB<NB_MAX> sm;
  if (failed(flags)) return;
  layer_bwd<NB_MAX, 1>(blockIdx.x, n, &sm, w, b, Xc, types, nlist, nnei, grids, n, l, geo, nullptr, gout);
}
// 12 waves: the first NLONG workgroups go through the long lists' atoms, eight waves each (the
// others end at once), the rest take two atoms each.
__global__ void __launch_bounds__(128 * NB_SMALL) __attribute__((amdgpu_waves_per_eu(3)))
k_rep_fwd(Weights w, Buffers b, const double *__restrict__ Xc, const int *__restrict__ types, const int *__restrict__ nlist,
          const int *__restrict__ nnei, const Grid *__restrict__ grids, int n, int l, Geo geo, const int *__restrict__ cnt,
          const unsigned *__restrict__ flags) {
  __shared__ union { SmemF<NB_SMALL> two[2]; SmemF<NB_MAX> one; } sm;
  __shared__ float wl[2 * PMAT] __attribute__((aligned(16)));
  if (failed(flags)) return;
  const int blk = blockIdx.x - NLONG;
  if (blk >= 0) {
    if (2 * blk < cnt[0]) layer_fwd<NB_SMALL, 2>(blk, cnt[0], sm.two, wl, w, b, Xc, types, nlist, nnei, grids, n, l, geo, b.idx);
    return;
  }
  if (threadIdx.x >= 64 * NB_MAX) return;
  for (int k = blockIdx.x; k < cnt[1]; k += NLONG) {
    layer_fwd<NB_MAX, 1>(k, cnt[1], &sm.one, wl, w, b, Xc, types, nlist, nnei, grids, n, l, geo, b.idx + b.cap);
    __syncthreads();
  }
}
__global__ void __launch_bounds__(128 * NB_SMALL) __attribute__((amdgpu_waves_per_eu(3)))
k_rep_bwd(Weights w, Buffers b, const double *__restrict__ Xc, const int *__restrict__ types, const int *__restrict__ nlist,
          const int *__restrict__ nnei, const Grid *__restrict__ grids, int n, int l, Geo geo, const int *__restrict__ cnt,
          float4 *__restrict__ gout, const unsigned *__restrict__ flags) {
  __shared__ union { SmemB<NB_SMALL> two[2]; SmemB<NB_MAX> one; } sm;
  if (failed(flags)) return;
  const int blk = blockIdx.x - NLONG;
  if (blk >= 0) {
    if (2 * blk < cnt[0]) layer_bwd<NB_SMALL, 2>(blk, cnt[0], sm.two, w, b, Xc, types, nlist, nnei, grids, n, l, geo, b.idx, gout);
    return;
  }
  if (threadIdx.x >= 64 * NB_MAX) return;
  for (int k = blockIdx.x; k < cnt[1]; k += NLONG) {
    layer_bwd<NB_MAX, 1>(k, cnt[1], &sm.one, w, b, Xc, types, nlist, nnei, grids, n, l, geo, b.idx + b.cap, gout);
    __syncthreads();
  }
}

// The edge count, and the atoms of the two instances (up to 96 neighbours, or more; the order
// only changes scheduling).  A truncated list is an error: the model needs complete ones.
__global__ void __launch_bounds__(1024) k_edge_count(const int *__restrict__ nnei, int n, int64_t *__restrict__ host_etot,
                                                     int *__restrict__ idx, int *__restrict__ cnt, int cap,
                                                     unsigned *__restrict__ flags) {
  __shared__ int64_t part[1024];
  const int l = lane();
  int64_t s = 0;
  for (int k0 = 0; k0 < n; k0 += 1024) {
    const int k = k0 + threadIdx.x;
    const int nk = k < n ? min(max(nnei[k], 0), SEL) : 0;
    s += nk;
    for (int cls = 0; cls < 2; ++cls) {
      const unsigned long long mask = __ballot(k < n && (nk > 16 * NB_SMALL) == (cls == 1));
      if (!mask) continue;
      const int first = __ffsll(mask) - 1;
      int base = 0;
      if (l == first) base = atomicAdd(cnt + cls, __popcll(mask));
      base = __shfl(base, first);
      if (mask >> l & 1ull) idx[(size_t)cls * cap + base + __popcll(mask & ((1ull << l) - 1ull))] = k;
    }
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *host_etot = part[0];
    if (flags[1] != 0u) atomicOr(flags, (unsigned)FLAG_INCOMPLETE);
  }
}

}  // namespace

void launch_edge_count(const Buffers &b, const Workspace &ws, int n, int64_t *host_etot, hipStream_t st) {
  hipLaunchKernelGGL(k_edge_count, dim3(1), dim3(1024), 0, st, ws.nnei, n, host_etot, b.idx, ws.bcnt, (int)b.cap, ws.flags);
}

void launch_layer_fwd(const Weights &w, const Buffers &b, const Workspace &ws, const double *coords,
                      const int *types, int n, int layer, const Geo &geo, hipStream_t st) {
  if (n <= ONE_UP_TO)
    hipLaunchKernelGGL(k_rep_fwd_one, dim3(n), dim3(64 * NB_MAX), 0, st, w, b, coords, types, ws.nlist, ws.nnei, ws.grids, n,
                       layer, geo, ws.flags);
  else
    hipLaunchKernelGGL(k_rep_fwd, dim3(NLONG + (n + 1) / 2), dim3(128 * NB_SMALL), 0, st, w, b, coords, types, ws.nlist,
                       ws.nnei, ws.grids, n, layer, geo, ws.bcnt, ws.flags);
}

void launch_layer_bwd(const Weights &w, const Buffers &b, const Workspace &ws, const double *coords,
                      const int *types, int n, int layer, const Geo &geo, hipStream_t st) {
  if (n <= ONE_UP_TO)
    hipLaunchKernelGGL(k_rep_bwd_one, dim3(n), dim3(64 * NB_MAX), 0, st, w, b, coords, types, ws.nlist, ws.nnei, ws.grids, n,
                       layer, geo, ws.g, ws.flags);
  else
    hipLaunchKernelGGL(k_rep_bwd, dim3(NLONG + (n + 1) / 2), dim3(128 * NB_SMALL), 0, st, w, b, coords, types, ws.nlist,
                       ws.nnei, ws.grids, n, layer, geo, ws.bcnt, ws.g, ws.flags);
}

}  // namespace rep
}  // namespace dp
