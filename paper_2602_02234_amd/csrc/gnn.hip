// GNN-variant descriptor kernels for gfx950: one workgroup per centre atom and one launch
// per message-passing layer, forward and backward (a layer's edge update reads the
// neighbours' node features of the layer before, so layers meet at launch boundaries).
//
// Every product of a feature tile with a weight matrix runs on MFMA (f32 or bf16 operands,
// f32 accumulation) transposed: weights as A operand, features along the accumulator rows,
// 16 angles or 16 edges along the columns.  Lane (q = lane / 16, c = lane % 16) then holds
// features 16 t + 4 q + i of angle or edge c, which is at once the layout of the float4
// rows in memory and the B operand of the next product (k step i of tile t is feature
// 16 t + 4 q + i), so a tile goes from memory through all its products and back without
// passing through LDS.  Weights come in that fragment order; the angle weights of a layer
// stay in each wave's registers.  Features are stored in float32.
//
// Forward, layer l, centre i:
//   per angle-list edge x, once: PQ[x] = the terms that its edge features add to the angle
//           products (with the biases);
//   angles  a wave owns rows p (p = wave, wave + NW, ...) and walks q in tiles of 16:
//           a' = a + tanh([a, e_ip, e_iq] Waa + b), and m_ip += sw_a(r_ip) sw_a(r_iq) / asel
//           tanh([a', e_iq] Wea + b);
//   edges   tiles of 16: e' = e + tanh([n_i, n_j, e] Wee + b) + m;
//   node    n' = n + tanh([n, sum_j sw_e e' / sel] Wnn + b); after the last layer the
//           fitting net, E_i in float64, and dE/dn_i.
// Backward, layer l (activations recomputed from the stored layer inputs): dE/dn_i is
// gathered from the edges (j, i) of the neighbours in list order.  A wave owns columns q
// and walks p: the gradients that meet at edge q, which enter through two weight products,
// are summed in registers and multiplied by the weights once per edge instead of once per
// angle; those of edge p go to a per-wave LDS array, and the waves' arrays are added in
// wave order, so every sum has a fixed order.  Layer 0 turns the accumulated gradients of
// s, sw_e, sw_a and rhat into g_ij = dE/dDelta_ij for the shared force gather.
//
// Bound: the products' and the activations' issue, one after the other in a tile, with two or three
// waves per SIMD to overlap them, then the angle rows' traffic.  At the 9,999-atom box a forward layer moves
// up to 1.7 GB of angle rows (0.33 ms at the copy rate) and has 0.46 ms of float32 MFMA work, a
// backward layer up to 2.6 GB (0.5 ms) and 0.95 ms.  Measured per layer there, float32: forward 3.06 ->
// 1.0 .. 1.2 ms, backward 6.89 -> 2.0 .. 2.4 ms, against kernels that staged every tile in LDS, one wave
// to a SIMD; 2,931 atoms in bfloat16, a step 7.4 -> 2.2 ms.
#include "dp_env.h"
#include "dp_tiles.h"
#include "gnn.h"

namespace dp {
namespace gnn {
namespace {

constexpr int LPQ = 132;  // row stride of the per-edge terms [angle-list edge][128]
constexpr int LMS = 68;   // ... of [angle-list edge][64]
constexpr int LSZ = 100;  // backward: per-edge terms of edge q [96], later the sums over its angles [96 + 4]
constexpr int LPP = 36;   // backward: sums of edge p [32 features, sw_a, rhat], and its terms [32]

template <typename T> __device__ __forceinline__ const T *frag(const Frag &f);
template <> __device__ __forceinline__ const float *frag<float>(const Frag &f) { return f.f32; }
template <> __device__ __forceinline__ const bf16_t *frag<bf16_t>(const Frag &f) { return f.b16; }

struct GEnv {
  float r[SEL], swe[SEL], dswe[SEL], swa[SEL], dswa[SEL], s[SEL];
  float rh[SEL * 3];
  int jn[SEL], tj[SEL], cpos[SEL];  // neighbour, its type, its angle-list position (-1: none)
  int cl[ASEL];                      // edge slot of each angle-list position
  int nn, nc;
};

__device__ __forceinline__ float quintic(float r, float rc, float rcs, float &dsw) {
  const float u = (r - rcs) / (rc - rcs);
  dsw = 0.f;
  if (r < rcs) return 1.f;
  if (r >= rc) return 0.f;
  dsw = -30.f * u * u * (1.f - u) * (1.f - u) / (rc - rcs);
  return u * u * u * (-6.f * u * u + 15.f * u - 10.f) + 1.f;
}

// Geometry of centre i's edges and its angle list (the first asel neighbours, in list
// order, closer than rca; the test is made in float64 on the minimum-image vector).
template <int NT> __device__ void build_genv(GEnv &e, const double *__restrict__ X, const int *__restrict__ types,
                           const int *__restrict__ nlist, const int *__restrict__ nnei, int i, int n,
                           const Grid &g, const Geo &geo) {
  const int nn = min(max(nnei[i], 0), SEL);
  for (int j = threadIdx.x; j < SEL; j += NT) {
    float r = 1.f, sw = 0.f, dsw = 0.f, sa = 0.f, dsa = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
    int nj = i, tj = 0, close = 0;
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
      close = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) < (double)geo.rca;
      const float dx = (float)d[0], dy = (float)d[1], dz = (float)d[2];
      r = sqrtf(dx * dx + dy * dy + dz * dz);
      sw = quintic(r, geo.rc, geo.rcs, dsw);
      sa = quintic(r, geo.rca, geo.rcs, dsa);
      hx = dx / r; hy = dy / r; hz = dz / r;
    }
    e.r[j] = r; e.swe[j] = sw; e.dswe[j] = dsw; e.swa[j] = sa; e.dswa[j] = dsa; e.s[j] = sw / r;
    e.rh[3 * j] = hx; e.rh[3 * j + 1] = hy; e.rh[3 * j + 2] = hz;
    e.jn[j] = nj; e.tj[j] = tj; e.cpos[j] = close;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int base = 0;
    for (int j0 = 0; j0 < nn; j0 += 64) {
      const int j = j0 + lane;
      const bool flag = j < nn && e.cpos[j] != 0;
      const unsigned long long mask = __ballot(flag);
      const int rank = base + __popcll(mask & ((1ull << lane) - 1ull));
      const bool in = flag && rank < geo.asel;
      if (j < nn) e.cpos[j] = in ? rank : -1;
      if (in) e.cl[rank] = j;
      base += __popcll(mask);
    }
    if (lane == 0) {
      e.nn = nn;
      e.nc = min(base, geo.asel);
    }
  }
  __syncthreads();
}

__device__ __forceinline__ float cosang(const GEnv &e, int jp, int jq) {
  return e.rh[3 * jp] * e.rh[3 * jq] + e.rh[3 * jp + 1] * e.rh[3 * jq + 1] + e.rh[3 * jp + 2] * e.rh[3 * jq + 2];
}

__device__ __forceinline__ size_t erow(const Buffers &b, int l, int i, int j) {
  return (((size_t)l * b.cap + i) * SEL + j) * EDIM;
}

// ------------------------------------------------------------------ angle offsets
// One wave per atom.
__global__ void __launch_bounds__(256) k_angle_count(const double *__restrict__ Xc, const int *__restrict__ nlist,
                                                     const int *__restrict__ nnei, const Grid *__restrict__ grids,
                                                     int n, Geo geo, int64_t *__restrict__ aoff) {
  const int i = blockIdx.x * 4 + wave_id(), l = lane_id();
  if (i >= n) return;
  const Grid g = grids[0];
  const int nn = min(max(nnei[i], 0), SEL);
  int nc = 0;
  for (int j0 = 0; j0 < nn; j0 += 64) {
    const int j = j0 + l;
    bool close = false;
    if (j < nn) {
      const int nj = nlist[(size_t)i * SEL + j];
      if (nj >= 0 && nj < n) {
        double d[3];
        for (int a = 0; a < 3; ++a) {
          double v = Xc[3 * nj + a] - Xc[3 * i + a];
          if (g.periodic) v -= g.L[a] * rint(v * g.invL[a]);
          d[a] = v;
        }
        close = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) < (double)geo.rca;
      }
    }
    nc += __popcll(__ballot(close));
  }
  nc = min(nc, geo.asel);
  if (l == 0) aoff[i + 1] = (int64_t)nc * (nc - 1);
  if (i == 0 && l == 0) aoff[0] = 0;
}

// Inclusive prefix of aoff[1 .. n] in one workgroup: each thread sums a contiguous run,
// the 1024 run totals are scanned, then each run is rewritten.
// The same workgroup also writes to host_tot the angles, the edges (sum of nnei) and the
// angle-list edges of the atoms that have angles (sum of nc, from nc (nc - 1)), and sets the
// step's error bits: a truncated list, or more than acap angles.
__global__ void __launch_bounds__(1024) k_angle_scan(int64_t *__restrict__ aoff, const int *__restrict__ nnei, int n,
                                                     int64_t acap, int64_t *__restrict__ host_tot,
                                                     unsigned *__restrict__ flags) {
  __shared__ int64_t part[1024];
  __shared__ int64_t epart[1024], cpart[1024];
  const int t = threadIdx.x;
  const int per = (n + 1023) / 1024;
  const int b0 = 1 + t * per, b1 = min(n + 1, b0 + per);
  int64_t s = 0, se = 0, sc = 0;
  for (int k = b0; k < b1; ++k) {
    const int64_t cnt = aoff[k];
    s += cnt;
    se += min(max(nnei[k - 1], 0), SEL);
    // cnt = nc (nc - 1) with nc <= 48 (0 for no angles)
    sc += cnt > 0 ? (int)(0.5f + sqrtf((float)cnt + 0.25f)) : 0;
  }
  part[t] = s;
  epart[t] = se;
  cpart[t] = sc;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (t < off) {
      epart[t] += epart[t + off];
      cpart[t] += cpart[t + off];
    }
    __syncthreads();
  }
  if (t == 0) {
    host_tot[1] = epart[0];
    host_tot[2] = cpart[0];
  }
  for (int off = 1; off < 1024; off <<= 1) {
    const int64_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  if (t == 1023) {
    host_tot[0] = part[t];
    unsigned f = flags[1] != 0u ? FLAG_INCOMPLETE : 0u;  // a truncated list: the model needs complete ones
    if (part[t] > acap) f |= FLAG_ANGLES;
    if (f) atomicOr(flags, f);
  }
  int64_t run = t > 0 ? part[t - 1] : 0;
  for (int k = b0; k < b1; ++k) {
    run += aoff[k];
    aoff[k] = run;
  }
}

// The layer's input features e_ij of edge slot j, features 16 t + 4 q .. + 3.
__device__ __forceinline__ f4 edge_in(const Weights &w, const Buffers &b, const GEnv &e, int l, int i, int j, int f) {
  return l == 0 ? init4<tanh_fast>(e.s[j], w.We0 + f, w.be0 + f) : ldf4(b.ef + erow(b, l - 1, i, j) + f);
}
// ... and n of the neighbour of slot j.
__device__ __forceinline__ f4 node_in(const Weights &w, const Buffers &b, const GEnv &e, int l, int j, int f) {
  return l == 0 ? ldf4(w.TN + e.tj[j] * NDIM + f) : ldf4(b.nf + ((size_t)(l - 1) * b.cap + e.jn[j]) * NDIM + f);
}

// The terms an angle's products take from its two edges depend on the edge alone; for every
// angle-list edge x, in float32: [e_x[:32] Waa[32:64] (edge p's), e_x[:32] Waa[64:96] + baa,
// e_x[:32] Wea[32:64] + bea], 128 columns, given to put(x, column, four values).
template <int NW, class Put>
__device__ __forceinline__ void edge_terms(const Weights &w, const Buffers &b, const GEnv &e, int l, int i, const Put &put) {
  const int q = lane_id() >> 4, c = lane_id() & 15;
  for (int x0 = 0; x0 < e.nc; x0 += 16) {
    const int x = x0 + c;
    const bool ok = x < e.nc;
    f4 ev[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) ev[t] = ok ? edge_in(w, b, e, l, i, e.cl[x], 16 * t + 4 * q) : f4{0.f, 0.f, 0.f, 0.f};
    const X<float, 2> xo(ev);
    for (int ot = wave_id(); ot < 8; ot += NW) {
      W<float, 2> wt;
      wt.load(w.PQ[l], ot);
      const int col = 16 * ot + 4 * q;
      const f4 bias = ot < 2 ? f4{0.f, 0.f, 0.f, 0.f} : (ot < 4 ? ldf4(w.baa[l] + col - 32) : ldf4(w.bea[l] + col - 64));
      const f4 v = wt(xo, bias);
      if (ok) put(x, col, v);
    }
  }
}

// ------------------------------------------------------------------ forward
template <int NW> struct SmemF {
  GEnv env;
  float PQ[ASEL * LPQ] __attribute__((aligned(16)));   // per-edge terms of the angle products
  float Msg[ASEL * LMS] __attribute__((aligned(16)));  // m_ip
  float nbias[EDIM] __attribute__((aligned(16))), aggw[NW][EDIM] __attribute__((aligned(16)));
  float ni[NDIM], xs[2 * NDIM], part[NW * 64];
  float y1[FWID], t2[FWID], dp[FWID];
};

template <typename T, int NW>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW == 4 ? 3 : 2)))
k_layer_fwd(Weights w, Buffers b, const double *__restrict__ Xc, const int *__restrict__ types,
            const int *__restrict__ nlist, const int *__restrict__ nnei, const Grid *__restrict__ grids, int n, int layer,
            Geo geo, double *__restrict__ Ei, const unsigned *__restrict__ flags) {
  __shared__ SmemF<NW> sm;
  const int i = blockIdx.x;
  if (i >= n || failed(flags)) return;
  const int tid = threadIdx.x, wv = wave_id(), ln = lane_id(), q = ln >> 4, c = ln & 15;
  const int l = layer;
  build_genv<NW * 64>(sm.env, Xc, types, nlist, nnei, i, n, grids[0], geo);
  const GEnv &e = sm.env;
  const int nn = e.nn, nc = e.nc;
  if (tid < NDIM)
    sm.ni[tid] = l == 0 ? w.TN[clamp_type(types[i]) * NDIM + tid] : b.nf[((size_t)(l - 1) * b.cap + i) * NDIM + tid];
  edge_terms<NW>(w, b, e, l, i, [&](int x, int col, f4 v) { stf4(sm.PQ + x * LPQ + col, v); });
  {  // the centre's part of every edge update: bee + n_i Wee[0:64]
    const float v = matvec<NW * 64, NDIM, EDIM>(w.Wee[l], sm.ni, sm.part, threadIdx.x);
    if (tid < EDIM) sm.nbias[tid] = v + w.bee[l][tid];
  }
  __syncthreads();

  // ---------------- angles and messages
  const int na = nc - 1;  // angles per row p
  const int64_t abase = b.aoff[i];
  {
    W<T, 2> wa[2], wm[4];
#pragma unroll
    for (int t = 0; t < 2; ++t) wa[t].load(frag<T>(w.A[l]), t);
#pragma unroll
    for (int t = 0; t < 4; ++t) wm[t].load(frag<T>(w.Mg[l]), t);
    const auto rows_in = [&](int p, int t0, f4 (&v)[2]) {  // a of angle t0 + c of row p (layers > 0)
      const int t = t0 + c;
      const float *ap = b.af + ((size_t)(l - 1) * b.acap + abase + (int64_t)p * na + t) * ADIM + 4 * q;
#pragma unroll
      for (int k = 0; k < 2; ++k) v[k] = t < na ? ldf4(ap + 16 * k) : f4{0.f, 0.f, 0.f, 0.f};
    };
    f4 nxt[2];
    if (l > 0 && wv < nc && na > 0) rows_in(wv, 0, nxt);
    for (int p = wv; p < nc; p += NW) {
      const int jp = e.cl[p];
      const float swp = e.swa[jp] * geo.inv_asel;
      f4 bp[2], m[4] = {};
#pragma unroll
      for (int k = 0; k < 2; ++k) bp[k] = ldf4(sm.PQ + p * LPQ + 16 * k + 4 * q);
      for (int t0 = 0; t0 < na; t0 += 16) {
        const int t = t0 + c;
        const bool ok = t < na;
        const int qr = ok ? t + (t >= p) : p;  // columns past the end read a valid row, unused
        f4 a[2];
        if (l > 0) {
          a[0] = nxt[0];
          a[1] = nxt[1];
          const bool more = t0 + 16 < na;  // the next tile's rows are read while this one is processed
          const int pn = more ? p : p + NW;
          if (pn < nc) rows_in(pn, more ? t0 + 16 : 0, nxt);
        } else {
          const float cs = cosang(e, jp, e.cl[qr]);
#pragma unroll
          for (int k = 0; k < 2; ++k) a[k] = init4<tanh_fast>(cs, w.Wa0 + 16 * k + 4 * q, w.ba0 + 16 * k + 4 * q);
        }
        const float *pq = sm.PQ + qr * LPQ + 4 * q;
        {
          const X<T, 2> x(a);
#pragma unroll
          for (int k = 0; k < 2; ++k) a[k] += act(wa[k](x, bp[k] + ldf4(pq + 32 + 16 * k)));
        }
        if (ok && l < NLAYER - 1) {
          float *ao = b.af + ((size_t)l * b.acap + abase + (int64_t)p * na + t) * ADIM + 4 * q;
          stf4(ao, a[0]);
          stf4(ao + 16, a[1]);
        }
        const X<T, 2> x(a);
        const float wr = ok ? swp * e.swa[e.cl[qr]] : 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) m[k] += wr * act(wm[k](x, ldf4(pq + 64 + 16 * k)));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f4 v = sum16(m[k]);
        if (c == 0) stf4(sm.Msg + p * LMS + 16 * k + 4 * q, v);
      }
    }
  }
  __syncthreads();

  // ---------------- edges
  f4 aw[4] = {};
  for (int j0 = wv * 16; j0 < nn; j0 += NW * 16) {
    const bool ok = j0 + c < nn;
    const int j = ok ? j0 + c : 0;
    f4 x[8];  // [n_j, e_ij]; n_i enters through nbias
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = node_in(w, b, e, l, j, 16 * k + 4 * q);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[4 + k] = edge_in(w, b, e, l, i, j, 16 * k + 4 * q);
    const X<T, 8> xo(x);
    const int cp = ok ? e.cpos[j] : -1;
    const float swj = ok ? e.swe[j] : 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      tile_barrier();
      W<T, 8> wt;  // not loaded ahead: more registers would spill at three waves per SIMD (float32 1.23 -> 1.34 ms)
      wt.load(frag<T>(w.E[l]), k);
      f4 v = x[4 + k] + act(wt(xo, ldf4(sm.nbias + 16 * k + 4 * q)));
      if (cp >= 0) v += ldf4(sm.Msg + cp * LMS + 16 * k + 4 * q);
      if (ok) stf4(b.ef + erow(b, l, i, j) + 16 * k + 4 * q, v);
      aw[k] += swj * v;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f4 v = sum16(aw[k]);
    if (c == 0) stf4(sm.aggw[wv] + 16 * k + 4 * q, v);
  }
  __syncthreads();

  // ---------------- node
  if (tid < NDIM) {
    float v = 0.f;
    for (int u = 0; u < NW; ++u) v += sm.aggw[u][tid];
    sm.xs[tid] = sm.ni[tid];
    sm.xs[NDIM + tid] = v * geo.inv_sel;
  }
  const float z = matvec<NW * 64, 2 * NDIM, NDIM>(w.Wnn[l], sm.xs, sm.part, threadIdx.x);
  float n1 = 0.f;
  if (tid < NDIM) {
    n1 = sm.ni[tid] + tanhf(z + w.bnn[l][tid]);
    if (l < NLAYER - 1) b.nf[((size_t)l * b.cap + i) * NDIM + tid] = n1;
    else if (NW == 4) b.dnl[(size_t)i * NDIM + tid] = n1;  // for launch_node_fit
  }
  if (NW == 4) return;
  if (l < NLAYER - 1) return;

  // ---------------- fitting net, E_i and dE/dn_i (up to WIDE_UP_TO atoms: 4 us at 192 atoms, where a
  // kernel over tiles of 16 atoms takes 9 and a launch; from 2,931 atoms on that kernel takes 9 .. 17 us, this 30 and more)
  if (tid < NDIM) sm.xs[tid] = n1;
  const float z1 = matvec<NW * 64, NDIM, FWID>(w.G1, sm.xs, sm.part, threadIdx.x);
  if (tid < FWID) sm.y1[tid] = tanhf(z1 + w.d1[tid]);
  const float z2 = matvec<NW * 64, FWID, FWID>(w.G2, sm.y1, sm.part, threadIdx.x);
  if (tid < FWID) {
    const float t2 = tanhf(z2 + w.d2[tid]);
    sm.t2[tid] = t2;
    sm.dp[tid] = w.G3[tid] * (1.f - t2 * t2);
  }
  const float z3 = matvec<NW * 64, FWID, FWID>(w.G2T, sm.dp, sm.part, threadIdx.x);  // its first barrier: t2 is complete
  if (wv == 0) {
    double E = (double)(sm.t2[ln] + sm.y1[ln]) * w.G3d[ln] + (double)(sm.t2[ln + 64] + sm.y1[ln + 64]) * w.G3d[ln + 64];
    for (int off = 32; off > 0; off >>= 1) E += __shfl_xor(E, off);
    if (ln == 0) Ei[i] = w.d3 + E;
  }
  float dp1 = 0.f;
  if (tid < FWID) dp1 = (z3 + w.G3[tid]) * (1.f - sm.y1[tid] * sm.y1[tid]);
  __syncthreads();
  if (tid < FWID) sm.dp[tid] = dp1;
  const float dn = matvec<NW * 64, FWID, NDIM>(w.G1T, sm.dp, sm.part, threadIdx.x);
  if (tid < NDIM) b.dnl[(size_t)i * NDIM + tid] = dn;
}

// ------------------------------------------------------------------ backward
template <int NW> struct SmemB {
  GEnv env;
  float P[NW][ASEL * LPP] __attribute__((aligned(16)));  // per-wave sums of the terms of edge p
  float SZ[ASEL * LSZ] __attribute__((aligned(16)));     // terms of edge q; once its wave is done with q, sums over its angles
  float PP[ASEL * LPP] __attribute__((aligned(16)));     // terms of edge p
  float DM[ASEL * LMS] __attribute__((aligned(16)));     // dE/dm_ip
  float nbias[EDIM] __attribute__((aligned(16))), dagg[NDIM] __attribute__((aligned(16)));
  float dnsum[NW][NDIM] __attribute__((aligned(16))), aggw[NW][NDIM] __attribute__((aligned(16)));
  union {  // the reverse slots are read before the edges, ds written by them
    int slot[SEL];
    float ds[SEL];
  };
  float dn[NDIM], ni[NDIM], xs[2 * NDIM], zz[NDIM], part[NW * 64];
};

template <typename T, int NW>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
k_layer_bwd(Weights w, Buffers b, const double *__restrict__ Xc, const int *__restrict__ types,
            const int *__restrict__ nlist, const int *__restrict__ nnei, const Grid *__restrict__ grids, int n, int layer,
            Geo geo, float4 *__restrict__ gout, const unsigned *__restrict__ flags) {
  __shared__ SmemB<NW> sm;
  const int i = blockIdx.x;
  if (i >= n || failed(flags)) return;
  const int tid = threadIdx.x, wv = wave_id(), ln = lane_id(), q = ln >> 4, c = ln & 15;
  build_genv<NW * 64>(sm.env, Xc, types, nlist, nnei, i, n, grids[0], geo);
  const GEnv &e = sm.env;
  const int nn = e.nn, nc = e.nc, l = layer;
  const bool top = l == NLAYER - 1;
  const f4 zero = {0.f, 0.f, 0.f, 0.f};

  if (tid < NDIM)
    sm.ni[tid] = l == 0 ? w.TN[clamp_type(types[i]) * NDIM + tid] : b.nf[((size_t)(l - 1) * b.cap + i) * NDIM + tid];
  edge_terms<NW>(w, b, e, l, i, [&](int x, int col, f4 v) {
    if (col < ADIM) stf4(sm.PP + x * LPP + col, v);
    else stf4(sm.SZ + x * LSZ + col - ADIM, v);
  });
  for (int k = tid; k < NW * nc * LPP; k += NW * 64) sm.P[k / (nc * LPP)][k % (nc * LPP)] = 0.f;
  // ---------------- dE/dn_i after this layer: own part + the neighbours' edge parts, and agg
  // from the stored output edges.  Sixteen lanes read a row; the 4 NW row groups walk the
  // list in turn, four rows in flight each, and are added in order.
  for (int j = tid; j < nn; j += NW * 64) sm.slot[j] = top ? -1 : b.slot[(size_t)i * SEL + j];
  __syncthreads();
  {
    constexpr int G = 4 * NW, R = (SEL + G - 1) / G;
    const float *src = b.dnj + (size_t)((l + 1) & 1) * b.cap * SEL * EDIM;
    const int g0 = tid >> 4;
    f4 dn = zero, agg = zero;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += 4) {
      f4 vd[4], ve[4];
      float sw[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = g0 + G * (r0 + r);
        const bool ok = j < nn;
        const int sj = ok ? sm.slot[j] : -1;
        sw[r] = ok ? e.swe[j] : 0.f;
        vd[r] = sj >= 0 ? ldf4(src + ((size_t)e.jn[j] * SEL + sj) * EDIM + 4 * c) : zero;
        ve[r] = ok ? ldf4(b.ef + erow(b, l, i, j) + 4 * c) : zero;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dn += vd[r];
        agg += sw[r] * ve[r];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      dn[k] = sumq(dn[k]);
      agg[k] = sumq(agg[k]);
    }
    if (q == 0) {
      stf4(sm.dnsum[wv] + 4 * c, dn);
      stf4(sm.aggw[wv] + 4 * c, agg);
    }
  }
  __syncthreads();
  if (tid < NDIM) {
    float dn = b.dnl[(size_t)i * NDIM + tid], agg = 0.f;
    for (int u = 0; u < NW; ++u) {
      dn += sm.dnsum[u][tid];
      agg += sm.aggw[u][tid];
    }
    sm.dn[tid] = dn;
    sm.xs[tid] = sm.ni[tid];
    sm.xs[NDIM + tid] = agg * geo.inv_sel;
  }
  // ---------------- node backward (and the centre's part of every edge update)
  {
    const float v = matvec<NW * 64, NDIM, EDIM>(w.Wee[l], sm.ni, sm.part, threadIdx.x);
    if (tid < EDIM) sm.nbias[tid] = v + w.bee[l][tid];
    const float z = matvec<NW * 64, 2 * NDIM, NDIM>(w.Wnn[l], sm.xs, sm.part, threadIdx.x);
    if (tid < NDIM) {
      const float t = tanhf(z + w.bnn[l][tid]);
      sm.zz[tid] = sm.dn[tid] * (1.f - t * t);
    }
    const float d = matvec<NW * 64, NDIM, 2 * NDIM>(w.WnnT[l], sm.zz, sm.part, threadIdx.x);
    if (tid < NDIM) sm.dn[tid] += d;  // now dE/dn_i of this layer's input, without the edge terms
    else if (tid < 2 * NDIM) sm.dagg[tid - NDIM] = d * geo.inv_sel;
  }
  __syncthreads();

  // ---------------- edges
  f4 dns[4] = {};
  for (int j0 = wv * 16; j0 < nn; j0 += NW * 16) {
    const bool ok = j0 + c < nn;
    const int j = ok ? j0 + c : 0;
    f4 ein[4], de1[4], dz[4];
    float rs = 0.f;
    {
      f4 x[8];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = node_in(w, b, e, l, j, 16 * k + 4 * q);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[4 + k] = edge_in(w, b, e, l, i, j, 16 * k + 4 * q);
      f4 eo[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        ein[k] = x[4 + k];
        eo[k] = ldf4(b.ef + erow(b, l, i, j) + 16 * k + 4 * q);
        de1[k] = top ? zero : ldf4(b.de + ((size_t)i * SEL + j) * EDIM + 16 * k + 4 * q);
      }
      const float swj = e.swe[j];
      tiles<T, 8>(frag<T>(w.E[l]), x, [&](int k) { return ldf4(sm.nbias + 16 * k + 4 * q); }, [&](int k, f4 z) {
        const f4 te = act(z);
        const f4 dg = ldf4(sm.dagg + 16 * k + 4 * q);
        const f4 pr = eo[k] * dg;
        rs += (pr[0] + pr[1]) + (pr[2] + pr[3]);
        de1[k] = ok ? de1[k] + swj * dg : zero;
        dz[k] = de1[k] * (1.f - te * te);
        dns[k] += dz[k];
      });
    }
    rs = sumq(rs);
    if (ok && q == 0) {
      float *g = b.gs + ((size_t)i * SEL + j) * 2;
      g[0] = top ? rs : g[0] + rs;
    }
    if (l > 0) {  // edge (i, j)'s part of dE/dn_j
      float *dst = b.dnj + (size_t)(l & 1) * b.cap * SEL * EDIM + ((size_t)i * SEL + j) * EDIM + 4 * q;
      tiles<T, 4>(frag<T>(w.N[l]), dz, [&](int) { return zero; }, [&](int k, f4 v) {
        if (ok) stf4(dst + 16 * k, v);
      });
    }
    const int cp = ok ? e.cpos[j] : -1;
    float ds = 0.f;
    tiles<T, 4>(frag<T>(w.D[l]), dz, [&](int) { return zero; }, [&](int k, f4 d) {
      const f4 v = de1[k] + d;  // dE/de of the layer's input; the angle terms are added below
      const int f = 16 * k + 4 * q;
      if (cp >= 0) stf4(sm.DM + cp * LMS + f, de1[k]);
      if (l > 0) {
        if (ok) stf4(b.de + ((size_t)i * SEL + j) * EDIM + f, v);
      } else {
        const f4 g = v * (1.f - ein[k] * ein[k]) * ldf4(w.We0 + f);
        ds += (g[0] + g[1]) + (g[2] + g[3]);
      }
    });
    if (l == 0) {
      ds = sumq(ds);
      if (ok && q == 0) sm.ds[j] = ds;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f4 v = sum16(dns[k]);
    if (c == 0) stf4(sm.dnsum[wv] + 16 * k + 4 * q, v);
  }
  __syncthreads();

  // ---------------- angles
  const int na = nc - 1;
  const int64_t abase = b.aoff[i];
  {
    W<T, 2> wm[4], wa[2], wy[2];  // recomputation, and the transposed products
    W<T, 4> wx[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) wm[k].load(frag<T>(w.Mg[l]), k);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      wa[k].load(frag<T>(w.A[l]), k);
      wx[k].load(frag<T>(w.Xt[l]), k);
      wy[k].load(frag<T>(w.Yt[l]), k);
    }
    float *P = sm.P[wv];
    // the rows of angle (p, qq) at column t0 + c of edge qq's walk; past the end the atom's first
    const auto angle = [&](int qq, int t0) -> int64_t {
      const int t = t0 + c, p = t + (t >= qq);
      return t < na ? abase + (int64_t)p * na + qq - (qq > p) : abase;
    };
    const auto rows = [&](const float *src, int64_t idx, f4 (&v)[2]) {
#pragma unroll
      for (int k = 0; k < 2; ++k) v[k] = ldf4(src + (size_t)idx * ADIM + 16 * k + 4 * q);
    };
    const float *a0s = b.af + (size_t)max(l - 1, 0) * b.acap * ADIM;
    f4 a0[2];
    if (wv < nc && na > 0 && l > 0) rows(a0s, angle(wv, 0), a0);
    for (int qq = wv; qq < nc; qq += NW) {
      const int jq = e.cl[qq];
      const float swq = e.swa[jq] * geo.inv_asel;
      const float rq[3] = {e.rh[3 * jq], e.rh[3 * jq + 1], e.rh[3 * jq + 2]};
      float *row = sm.SZ + qq * LSZ;
      f4 za[2] = {}, zm[4] = {};
      float sq = 0.f, hq[3] = {0.f, 0.f, 0.f};  // dE/dsw_a(r_iq), dE/drhat_iq
      for (int t0 = 0; t0 < na; t0 += 16) {
        const int t = t0 + c;
        const bool ok = t < na;
        const int p = ok ? t + (t >= qq) : 0;  // columns past the end read a valid row, unused
        const int jp = e.cl[p];
        const int64_t idx = angle(qq, t0);
        // the next tile's rows of a are read as soon as this one has used its own
        const bool same = t0 + 16 < na, more = same || qq + NW < nc;
        const int64_t nidx = more ? angle(same ? qq : qq + NW, same ? t0 + 16 : 0) : abase;
        f4 da[2] = {zero, zero};
        if (!top) rows(b.da, idx, da);  // needed after most of the tile's products only
        if (l == 0) {
          const float cs = cosang(e, jp, jq);
#pragma unroll
          for (int k = 0; k < 2; ++k) a0[k] = init4<tanh_fast>(cs, w.Wa0 + 16 * k + 4 * q, w.ba0 + 16 * k + 4 * q);
        }
        // the angle update again: a' = a + tanh(...) (recomputed rather than stored: a quarter of the
        // angles' traffic)
        f4 ta[2], a1[2];
        {
          const X<T, 2> x(a0);
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            ta[k] = act(wa[k](x, ldf4(row + 16 * k + 4 * q) + ldf4(sm.PP + p * LPP + 16 * k + 4 * q)));
            a1[k] = a0[k] + ta[k];
          }
        }
        if (l > 0) rows(a0s, nidx, a0);
        tile_barrier();
        // the message: dE/dw and dz_m = w dE/dm (1 - tanh^2)
        const float wr = ok ? e.swa[jp] * swq : 0.f;
        float d = 0.f;
        f4 dz[4];
        {
          const X<T, 2> x(a1);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const f4 tm = act(wm[k](x, ldf4(row + ADIM + 16 * k + 4 * q)));
            const f4 dm = ldf4(sm.DM + p * LMS + 16 * k + 4 * q);
            const f4 g = dm * tm;
            d += (g[0] + g[1]) + (g[2] + g[3]);
            dz[k] = wr * dm * (1.f - tm * tm);
            zm[k] += dz[k];
          }
        }
        tile_barrier();
        d = sumq(d);
        d = ok ? d : 0.f;
        // dE/da' and dz_a
        f4 za1[2];
        {
          const X<T, 4> x(dz);
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const f4 v = wx[k](x, da[k]);  // outside the selection: matrix instructions ignore the lane mask
            da[k] = ok ? v : zero;
            za1[k] = da[k] * (1.f - ta[k] * ta[k]);
            za[k] += za1[k];
          }
        }
        {
          const X<T, 2> x(za1);
#pragma unroll
          for (int k = 0; k < 2; ++k) da[k] = wy[k](x, da[k]);
        }
        float dc = 0.f;
        if (l == 0) {
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const f4 g = da[k] * (1.f - a0[k] * a0[k]) * ldf4(w.Wa0 + 16 * k + 4 * q);
            dc += (g[0] + g[1]) + (g[2] + g[3]);
          }
          dc = sumq(dc);
        }
        if (ok) {
          float *pp = P + p * LPP;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            if (l > 0) stf4(b.da + (size_t)idx * ADIM + 16 * k + 4 * q, da[k]);
            stf4(pp + 16 * k + 4 * q, ldf4(pp + 16 * k + 4 * q) + za1[k]);
          }
          const float sp = e.swa[jp] * geo.inv_asel;
          sq += d * sp;
          if (l == 0)
            for (int a = 0; a < 3; ++a) hq[a] += dc * e.rh[3 * jp + a];
          if (q == 0) {
            f4 s = ldf4(pp + ADIM);
            s[0] += d * swq;
            if (l == 0)
              for (int a = 0; a < 3; ++a) s[1 + a] += dc * rq[a];
            stf4(pp + ADIM, s);
          }
        }
      }
      // the sums over the angles of edge q, in place of its terms
#pragma unroll
      for (int k = 0; k < 2; ++k) za[k] = sum16(za[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k) zm[k] = sum16(zm[k]);
      const f4 sh = sum16(f4{sq, hq[0], hq[1], hq[2]});
      wave_sync();
      if (c == 0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) stf4(row + 16 * k + 4 * q, za[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) stf4(row + ADIM + 16 * k + 4 * q, zm[k]);
        if (q == 0) stf4(row + ADIM + EDIM, sh);
      }
    }
  }
  __syncthreads();

  // ---------------- the angle terms of each angle-list edge: the waves' sums of edge p in wave
  // order (sw_a and rhat complete with edge q's), then the weights once per edge
  for (int k = tid; k < nc * LPP; k += NW * 64) {
    const int x = k / LPP, f = k % LPP;
    float v = sm.P[0][k];
    for (int u = 1; u < NW; ++u) v += sm.P[u][k];
    if (f >= ADIM) v += sm.SZ[x * LSZ + ADIM + EDIM + f - ADIM];
    sm.P[0][k] = v;
  }
  if (tid < NDIM) {
    float s = 0.f;
    for (int u = 0; u < NW; ++u) s += sm.dnsum[u][tid];
    sm.zz[tid] = s;
  }
  __syncthreads();
  for (int x0 = 0; x0 < nc; x0 += 16) {
    const bool ok = x0 + c < nc;
    const int x = ok ? x0 + c : 0;
    const int j = e.cl[x];
    if (x0 / 16 % NW != wv) continue;
    f4 v[8];  // [sum of dz_a over row p, over column q, sum of dz_m over column q]
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      v[k] = ldf4(sm.P[0] + x * LPP + 16 * k + 4 * q);
      v[2 + k] = ldf4(sm.SZ + x * LSZ + 16 * k + 4 * q);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) v[4 + k] = ldf4(sm.SZ + x * LSZ + ADIM + 16 * k + 4 * q);
    const X<float, 8> xo(v);
    float ds = 0.f;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      W<float, 8> wt;
      wt.load(w.PS[l], k);
      const f4 d = wt(xo, zero);
      const int f = 16 * k + 4 * q;
      if (l > 0) {
        float *o = b.de + ((size_t)i * SEL + j) * EDIM + f;
        if (ok) stf4(o, ldf4(o) + d);
      } else {
        const f4 e0 = edge_in(w, b, e, 0, i, j, f);
        const f4 g = d * (1.f - e0 * e0) * ldf4(w.We0 + f);
        ds += (g[0] + g[1]) + (g[2] + g[3]);
      }
    }
    if (l == 0) {
      ds = sumq(ds);
      if (ok && q == 0) sm.ds[j] += ds;
    }
  }
  for (int j = tid; j < nn; j += NW * 64) {
    const int cp = e.cpos[j];
    float *g = b.gs + ((size_t)i * SEL + j) * 2;
    const float dsa = cp >= 0 ? sm.P[0][cp * LPP + ADIM] : 0.f;
    g[1] = top ? dsa : g[1] + dsa;
  }
  if (l > 0) {
    const float v = matvec<NW * 64, NDIM, NDIM>(w.WeeT[l], sm.zz, sm.part, threadIdx.x);
    if (tid < NDIM) b.dnl[(size_t)i * NDIM + tid] = sm.dn[tid] + v;
    return;
  }
  __syncthreads();
  // ---------------- layer 0: g_ij = dE/dDelta_ij
  for (int j = tid; j < nn; j += NW * 64) {
    const float ds = sm.ds[j];
    const float *g2 = b.gs + ((size_t)i * SEL + j) * 2;
    const int cp = e.cpos[j];
    const float rr = e.r[j], sw = e.swe[j];
    const float dr = ds * (e.dswe[j] / rr - sw / (rr * rr)) + g2[0] * e.dswe[j] + g2[1] * e.dswa[j];
    const float hx = e.rh[3 * j], hy = e.rh[3 * j + 1], hz = e.rh[3 * j + 2];
    float gx = 0.f, gy = 0.f, gz = 0.f;
    if (cp >= 0) {
      gx = sm.P[0][cp * LPP + ADIM + 1];
      gy = sm.P[0][cp * LPP + ADIM + 2];
      gz = sm.P[0][cp * LPP + ADIM + 3];
    }
    const float proj = gx * hx + gy * hy + gz * hz;
    gout[(size_t)i * SEL + j] = make_float4((gx - proj * hx) / rr + dr * hx, (gy - proj * hy) / rr + dr * hy,
                                            (gz - proj * hz) / rr + dr * hz, 0.f);
  }
}

}  // namespace

void launch_angle_offsets(const Buffers &b, const Workspace &ws, const double *coords, int n, const Geo &geo,
                          int64_t *host_tot, hipStream_t st) {
  hipLaunchKernelGGL(k_angle_count, dim3((n + 3) / 4), dim3(256), 0, st, coords, ws.nlist, ws.nnei, ws.grids, n, geo,
                     b.aoff);
  hipLaunchKernelGGL(k_angle_scan, dim3(1), dim3(1024), 0, st, b.aoff, ws.nnei, n, b.acap, host_tot, ws.flags);
}

template <typename T>
void launch_layer_fwd(const Weights &w, const Buffers &b, const Workspace &ws, const double *coords,
                      const int *types, int n, int layer, const Geo &geo, double *Ei, hipStream_t st) {
  const auto go = [&](auto kernel, int nw) {
    hipLaunchKernelGGL(kernel, dim3(n), dim3(nw * 64), 0, st, w, b, coords, types, ws.nlist, ws.nnei, ws.grids, n, layer,
                       geo, Ei, ws.flags);
  };
  if (n <= WIDE_UP_TO) go(k_layer_fwd<T, 8>, 8);
  else go(k_layer_fwd<T, 4>, 4);
}

template <typename T>
void launch_layer_bwd(const Weights &w, const Buffers &b, const Workspace &ws, const double *coords,
                      const int *types, int n, int layer, const Geo &geo, hipStream_t st) {
  const auto go = [&](auto kernel, int nw) {
    hipLaunchKernelGGL(kernel, dim3(n), dim3(nw * 64), 0, st, w, b, coords, types, ws.nlist, ws.nnei, ws.grids, n, layer,
                       geo, ws.g, ws.flags);
  };
  if (n <= WIDE_UP_TO) go(k_layer_bwd<T, 8>, 8);
  else go(k_layer_bwd<T, 4>, 4);
}

template void launch_layer_fwd<float>(const Weights &, const Buffers &, const Workspace &, const double *,
                                      const int *, int, int, const Geo &, double *, hipStream_t);
template void launch_layer_fwd<bf16_t>(const Weights &, const Buffers &, const Workspace &, const double *,
                                       const int *, int, int, const Geo &, double *, hipStream_t);
template void launch_layer_bwd<float>(const Weights &, const Buffers &, const Workspace &, const double *,
                                      const int *, int, int, const Geo &, hipStream_t);
template void launch_layer_bwd<bf16_t>(const Weights &, const Buffers &, const Workspace &, const double *,
                                       const int *, int, int, const Geo &, hipStream_t);

}  // namespace gnn
}  // namespace dp
