// What the descriptor kernels of both precisions share: the transposed layout of a token's
// features and of its environment, the embedding's feature groups, softmax and LayerNorm over
// registers, and the split of the atoms over workgroups.
#pragma once
#include <algorithm>

#include "dp_env.h"
#include "dp_tiles.h"

namespace dp {
namespace {

constexpr int LDG = M;       // row stride (floats) of float32 [token][feature] arrays in LDS: 100
constexpr int NB_SMALL = 6;  // blocks up to which two atoms share a workgroup

// A vector over the 100 features of a lane's token: x[t][i] = feature 16 t + 4 q + i for
// t < 6, x[6][0] = feature 96 + q (x[6][1..3] are never read as features).
typedef f4 F100[7];

__device__ __forceinline__ f4 mfma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// A token's features from / to a row of G.
__device__ __forceinline__ void get_row(F100 &x, const float *row) {
  const int q = lane() >> 4;
#pragma unroll
  for (int t = 0; t < 6; ++t) x[t] = ldf4(row + 16 * t + 4 * q);
  x[6] = f4{row[96 + q], 0.f, 0.f, 0.f};
}
__device__ __forceinline__ void put_row(float *row, const F100 &x) {
  const int q = lane() >> 4;
#pragma unroll
  for (int t = 0; t < 6; ++t) *reinterpret_cast<f4 *>(row + 16 * t + 4 * q) = x[t];
  row[96 + q] = x[6][0];
}
// A per-feature table (bias, gain) in the same arrangement.
__device__ __forceinline__ void get_table(F100 &x, const float *__restrict__ p) { get_row(x, p); }

// A block's features in global memory: 1600 floats, every access one contiguous piece.
__device__ __forceinline__ void save_block(float *__restrict__ p, const F100 &x) {
  const int l = lane();
#pragma unroll
  for (int t = 0; t < 6; ++t) *reinterpret_cast<f4 *>(p + 256 * t + 4 * l) = x[t];
  p[1536 + l] = x[6][0];
}
__device__ __forceinline__ void load_block(F100 &x, const float *__restrict__ p) {
  const int l = lane();
#pragma unroll
  for (int t = 0; t < 6; ++t) x[t] = ldf4(p + 256 * t + 4 * l);
  x[6] = f4{p[1536 + l], 0.f, 0.f, 0.f};
}

// Sum over a token's 100 features of f(t, i) (t = 6: i = 0 only).
template <class Fn> __device__ __forceinline__ float sum100(const Fn &f) {
  float v = f(6, 0);
#pragma unroll
  for (int t = 0; t < 6; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) v += f(t, i);
  return sumq(v);
}

// 1 / sigma of a centred row d, and xh = d / sigma in place.  (Means are quotients: float32's 1 / 100 is off by
// 2.2e-8 and its 1 / 120 by 5.2e-8, the same way for every row, which shows in all forces alike.)
__device__ __forceinline__ float normalise(F100 &d, float eps) {
  const float var = sum100([&](int t, int i) { return d[t][i] * d[t][i]; }) / (float)M;
  const float is = 1.f / sqrtf(var + eps);
#pragma unroll
  for (int t = 0; t < 7; ++t) d[t] *= is;
  return is;
}

// The environment of one atom, padded to whole blocks; padded tokens (j >= n) have
// s = sw = dsw = 0, r = 1, rhat = 0.
template <int NB> struct EnvF {
  float s[16 * NB], sw[16 * NB] __attribute__((aligned(16)));
  float r[16 * NB];
  float rh[3][16 * NB] __attribute__((aligned(16)));
  int tj[16 * NB];
};

// The neighbour of token j as listed (its load can be issued ahead of others), and the entry made from it.
__device__ __forceinline__ int env_neighbour(const int *__restrict__ nlist, int i, int j, int n) {
  return j < n ? nlist[(size_t)i * SEL + j] : i;
}
template <int NB>
__device__ __forceinline__ void env_entry(EnvF<NB> &e, int j, int nj, const double *__restrict__ X,
                                          const int *__restrict__ types, int i, int n, int natoms, const Grid &g, float rc,
                                          float rcs) {
  if (j >= 16 * NB) return;
  float s = 0.f, sw = 0.f, r = 1.f, hx = 0.f, hy = 0.f, hz = 0.f;
  int tj = 0;
  if (j < n) {
    if (nj < 0 || nj >= natoms) nj = i;  // never read outside the coordinate array
    tj = clamp_type(types[nj]);
    double d[3];
    for (int a = 0; a < 3; ++a) {
      double v = X[3 * nj + a] - X[3 * i + a];
      if (g.periodic) v -= g.L[a] * rint(v * g.invL[a]);
      d[a] = v;
    }
    const float dx = (float)d[0], dy = (float)d[1], dz = (float)d[2];
    r = sqrtf(dx * dx + dy * dy + dz * dz);
    const float u = (r - rcs) / (rc - rcs);
    if (r < rcs) sw = 1.f;
    else if (r < rc) sw = u * u * u * (-6.f * u * u + 15.f * u - 10.f) + 1.f;
    s = sw / r;
    hx = dx / r; hy = dy / r; hz = dz / r;
  }
  e.s[j] = s; e.sw[j] = sw; e.r[j] = r; e.tj[j] = tj;
  e.rh[0][j] = hx; e.rh[1][j] = hy; e.rh[2][j] = hz;
}

template <int NB>
__device__ __forceinline__ void build_envf(EnvF<NB> &e, int tid, const double *__restrict__ X, const int *__restrict__ types,
                                           const int *__restrict__ nlist, int i, int n, int natoms, const Grid &g, float rc,
                                           float rcs) {
  env_entry(e, tid, env_neighbour(nlist, i, tid, n), X, types, i, n, natoms, g, rc, rcs);
}

// ------------------------------------------------------------ embedding net
// Its widths 25, 50 = 2 x 25, 100 = 4 x 25 are kept as groups of 25 features, slot r of
// lane group q holding feature 4 r + q of the group (r < 7; r = 6 only for q = 0, zero
// elsewhere), so that the residuals [h, h] add registers of the same lane.  h1[r];
// h2[g][r] with feature 25 g + 4 r + q; G[g][r] likewise for g < 4.  Weights in fragment
// order: an output group's slots 0-3 and 4-7 are two tiles (row 4 q + i of tile u is slot
// 4 u + i); a contraction group's 8 slots are two pieces of 4 k steps.
typedef float S7[7];
__device__ __forceinline__ bool slot_ok(int r) { return r < 6 || lane() < 16; }

// The embedding's G into the token's row.
__device__ __forceinline__ void put_embedding(float *row, const S7 (&h1)[1], const S7 (&t2)[2], const S7 (&t3)[4]) {
  const int q = lane() >> 4;
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int r = 0; r < 7; ++r)
      if (slot_ok(r)) row[25 * g + 4 * r + q] = t3[g][r] + (t2[g & 1][r] + h1[0][r]);
}

// E = exp(S - max) / Z over the keys in place of the scores (0 past the list), with
// Z = sum_k sw_k exp(S_k - max).
template <int NB, class Exp>
__device__ __forceinline__ void softmax_keys(f4 (&s)[NB], const EnvF<NB> &e, int n, const Exp &ex) {
  const int q = lane() >> 4;
  float m = -INFINITY;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (16 * kt + 4 * q + i >= n) s[kt][i] = -INFINITY;
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
      s[kt][i] = ex(s[kt][i] - m);
      z += sw[i] * s[kt][i];
    }
  }
  z = sumq(z);
  const float iz = z > 0.f ? 1.f / z : 0.f;
#pragma unroll
  for (int kt = 0; kt < NB; ++kt) s[kt] *= iz;
}

// rhat_k . h for the four keys of tile kt the lane holds.
template <int NB>
__device__ __forceinline__ f4 gate4(const EnvF<NB> &e, int kt, const float (&h)[3]) {
  const int k = 16 * kt + 4 * (lane() >> 4);
  return ldf4(e.rh[0] + k) * h[0] + ldf4(e.rh[1] + k) * h[1] + ldf4(e.rh[2] + k) * h[2];
}

// The part of a workgroup's work a wave takes: NA atoms (entries blk NA .. of the
// instance's list, or from atom c0 on without one), NB waves each.  Past the end of the list nb = 0; steps is the largest
// nb, so that the waves of both atoms pass the same barriers.
template <int NB, int NA> struct Part {
  int half, jb, tid, i, n, nb, steps;
  __device__ __forceinline__ Part(int blk, const int *__restrict__ idx, int c0, int count, const int *__restrict__ nnei) {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));  // as lane()
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    half = NA == 1 ? 0 : wv / NB;
    jb = wv - half * NB;
    tid = t - half * 64 * NB;
    steps = 0;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const int p = min(blk * NA + a, count - 1), k = idx ? idx[p] : c0 + p;
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

// Two atoms share a workgroup where there is more than one atom per CU (256): the waves of
// a workgroup go to the SIMDs in turn, so that 12 waves put three on each, while a second
// workgroup of 6 waves does not fit beside a first (two SIMDs would hold four waves of 168
// registers; 9,999 atoms that way, float32: forward 2.73 ms, backward 6.9 ms, against 2.10 and
// 4.85 ms in pairs, when both were measured).  Up to 256 atoms run one to a workgroup of eight waves, whatever their
// lists, without the lists of atoms and the second stream.
constexpr int PAIR_FROM = 257;
constexpr int NCU = 256;

// launch(kernel, workgroups, threads, atoms, their number on the device, stream) over the centres
// c0 .. c1-1 of n atoms: the pair kernel for lists of up to 16 NB_SMALL, the large one for the others
// beside it on the second stream, or for all (no list) in small systems.
template <class Pair, class Large, class Launch>
void launch_instances(const Workspace &ws, int n, int ncen, Pair pair, Large large, hipStream_t st, const Launch &launch) {
  if (n < PAIR_FROM) {
    launch(large, ncen, 64 * 8, (const int *)nullptr, (const int *)nullptr, st);
    return;
  }
  (void)hipEventRecord(ws.fork_ev, st);
  (void)hipStreamWaitEvent(ws.side, ws.fork_ev, 0);
  launch(large, std::min(ncen, NCU), 64 * 8, ws.bidx + ws.cap, ws.bcnt + 1, ws.side);
  launch(pair, (ncen + 1) / 2, 64 * 2 * NB_SMALL, ws.bidx, ws.bcnt, st);
  (void)hipEventRecord(ws.join_ev, ws.side);
  (void)hipStreamWaitEvent(st, ws.join_ev, 0);
}

}  // namespace
}  // namespace dp
