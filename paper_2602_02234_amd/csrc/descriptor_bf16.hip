// Per-atom descriptor kernels of the bfloat16 path on gfx950, forward and backward: the model
// and the split over waves of the float32 kernels (descriptor.hip, dp_desc.h), with the
// products on 16x16x32 bfloat16 MFMA.  Rounded to bfloat16 are the operands of the products
// only: G, U, the attention weights, H, dY, dH, dS, dU and the embedding's h1, h2 and
// pre-activation gradients; accumulators, residuals, softmax, LayerNorm, the sums of the
// softmax and gate gradients and T = G^T Rt / sel are float32.
//
// A wave carries the 16 tokens of its block in registers, transposed: lane (q = lane / 16,
// c = lane % 16) holds features (or keys) 16 t + 4 q + i of token c.  Two tiles t = 2 p, 2 p + 1
// of that form are the eight k of the lane in step p of the next product (k = 32 p + 8 q + e
// stands for feature 32 p + 4 q + e, or 32 p + 16 + 4 q + e - 4 from e = 4), so an accumulator is
// rounded and used without a trip through LDS; features 96 + q take the first k of step 3.
// Rows that other waves read are kept in LDS in that order, 128 values in sixteen 16-byte
// pieces (piece 4 p + q; 12 + q: feature 96 + q and zeros), the pieces of row r exchanged by
// r's low bits so that 16 rows' reads of one piece and 4 rows' transposed reads of four
// (ds_read_tr: four rows of 16 columns, a column to a lane) both spread over all banks.  One
// copy serves contractions over features and over tokens.
//
// In the backward a key's sums over the queries, A^T dH + dS^T U, are formed by the key's wave
// from the waves' rows of E gate and dH, then W and U, left in LDS between barriers; the factor
// sw_k multiplies the float32 sum.
//
// Bound: vector instructions (softmax, LayerNorm, tanh, conversions), then the latency of the
// stages between barriers; the matrix cores' share is about a fifth (101 MFMAs of 16 cycles per
// block and layer forward, 232 backward, at 96 neighbours).  In the backward vector instructions and
// LDS are each busy for two fifths of the time.  Measured at 24,999 atoms: forward 2.72 -> 1.18 ms,
// backward 5.95 -> 2.87 ms, against one atom per CU with G in LDS twice and rows of 16 keys gathered
// through it; at 192 atoms, one to a CU, 22 and 49 us.  The 12-wave backward spills 39 registers a
// wave; with 84 (a matrix loaded two products early, dE/dRt kept to the end) it took 2.94 ms.
#include "dp_desc.h"

namespace dp {
namespace {

constexpr int RW = 128;   // values in a bfloat16 row in LDS
constexpr int LDH = 52;   // stride (floats) of the rows a block's features are rearranged in (16 fit its rows)
constexpr int WMAT = 11264;                        // values of an attention matrix in fragment order
constexpr int W2T_N = 4 * 512, W3T_N = 14 * 512;   // ... of the embedding's
typedef short s4 __attribute__((ext_vector_type(4)));
static_assert(M == 100 && E1 == 25 && E2 == 50, "the fragment layouts below are written for these widths");

__device__ __forceinline__ f4 mma(bf8 a, bf8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ bf8 ld8(const bf16_t *p) { return *reinterpret_cast<const bf8 *>(p); }

__device__ __forceinline__ bf8 pack(f4 a, f4 b) {
  bf8 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = (__bf16)a[e];
    v[4 + e] = (__bf16)b[e];
  }
  return v;
}
// A token's features as a B operand.
struct XB {
  bf8 v[4];
  __device__ __forceinline__ XB() {}
  __device__ __forceinline__ explicit XB(const F100 &x) {
#pragma unroll
    for (int p = 0; p < 3; ++p) v[p] = pack(x[2 * p], x[2 * p + 1]);
    v[3] = pack(f4{x[6][0], 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f});
  }
};
// Offset in a block (16 rows) of piece 4 p + q of row c: the lane's eight values of step p.  The row's
// low bits are exchanged in, so step p differs from step 0 in the bits of 32 p alone.
__device__ __forceinline__ int piece0() {
  const int l = lane(), q = l >> 4, c = l & 15;
  return c * RW + 8 * (4 * (c & 3) + (q ^ (c >> 2)));
}
__device__ __forceinline__ int piece(int p0, int p) { return p0 ^ (32 * p); }
__device__ __forceinline__ void put_block(bf16_t *block, const XB &x) {
  const int p0 = piece0();
#pragma unroll
  for (int p = 0; p < 4; ++p) *reinterpret_cast<bf8 *>(block + piece(p0, p)) = x.v[p];
}
// Where the lane reads the values of column 16 t + c in rows 4 q .. 4 q + 3 of a block (t = 6: feature
// 96 + c / 4 for c a multiple of 4): for t = 0 and, by the bits of t / 2, for the others.
__device__ __forceinline__ int column0() {
  const int l = lane(), q = l >> 4, c = l & 15, r = c >> 2;
  return (4 * q + r) * RW + 8 * (4 * r + ((c & 3) ^ q));
}
__device__ __forceinline__ s4 read_tr(const bf16_t *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4 *)p);
}
// ... of two consecutive blocks, cu = (column0 ^ 32 (t / 2)) + 4 (t & 1): the eight k of a
// contraction over 32 rows.
__device__ __forceinline__ bf8 column8(const bf16_t *block, int cu) {
  typedef short s8 __attribute__((ext_vector_type(8)));
  const s4 a = read_tr(block + cu), b = read_tr(block + 16 * RW + cu);
  return __builtin_bit_cast(bf8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// acc += W x for a 100 x 100 matrix in fragment order, in LDS: step p < 3 of tile t at (7 p + t) 512 + 8 lane,
// the seven tiles' k = 96 + q at 10752 + 8 lane + t.  A step's seven tiles are independent
// products, and the next step's operands are loaded while they run.
__device__ __forceinline__ void wmul(F100 &acc, const bf16_t *w, const XB &x) {
  const bf16_t *p = w + 8 * lane();
  bf8 a[7];
#pragma unroll
  for (int t = 0; t < 7; ++t) a[t] = ld8(p + 512 * t);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    bf8 b[7];
    if (k < 2) {
#pragma unroll
      for (int t = 0; t < 7; ++t) b[t] = ld8(p + 512 * (7 * (k + 1) + t));
    } else if (k == 2) {
      const bf8 tail = ld8(p + 10752);
#pragma unroll
      for (int t = 0; t < 7; ++t) {
        b[t] = bf8{};
        b[t][0] = tail[t];
      }
    }
    tile_barrier();
#pragma unroll
    for (int t = 0; t < 7; ++t) acc[t] = mma(a[t], x.v[k], acc[t]);
    tile_barrier();
    if (k < 3)
#pragma unroll
      for (int t = 0; t < 7; ++t) a[t] = b[t];
  }
}

// s[kt] = G x over the keys of tile kt < nb: rows key 16 kt + 4 q + i, columns tokens.
template <int NB>
__device__ __forceinline__ void keys_dot(f4 (&s)[NB], const bf16_t *G, const XB &x, int nb) {
#pragma unroll
  for (int kt = 0; kt < NB; ++kt) s[kt] = f4{0.f, 0.f, 0.f, 0.f};
  const int p0 = piece0();
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    tile_barrier();
    const bf16_t *g = G + piece(p0, p);
#pragma unroll
    for (int kt = 0; kt < NB; ++kt)
      if (kt < NB_SMALL - 2 || kt < nb) s[kt] = mma(ld8(g + 16 * kt * RW), x.v[p], s[kt]);
  }
}

// acc += R^T y over rows 32 p .. 32 p + 31 of R, y(p) the lane's eight values of them, for
// 2 p < nb.  Rows of a block past nb are zero.
template <int NB, class Y>
__device__ __forceinline__ void rows_sum(F100 &acc, const bf16_t *R, const Y &y, int nb) {
  const int cu = column0();
#pragma unroll
  for (int p = 0; p < NB / 2; ++p)
    if (2 * p < nb) {
      const bf8 v = y(p);
      bf8 a[7];
#pragma unroll
      for (int t = 0; t < 7; ++t) a[t] = column8(R + 32 * p * RW, (cu ^ (32 * (t >> 1))) + 4 * (t & 1));
#pragma unroll
      for (int t = 0; t < 7; ++t) acc[t] = mma(a[t], v, acc[t]);
      tile_barrier();
    }
}

// ------------------------------------------------------------ embedding net
// Feature groups as in the float32 kernels; a group's seven slots are the lane's k of one step.
// Weights in fragment order: tile u of output group og, input group ig at ((og 2 + u) NI + ig) 512.
template <int NI, int NO>
__device__ __forceinline__ void emul(S7 (&out)[NO], const bf16_t *w, const S7 (&in)[NI]) {
  bf8 x[NI];
  const bf16_t *wl = w + 8 * lane();
#pragma unroll
  for (int ig = 0; ig < NI; ++ig)
    x[ig] = pack(f4{in[ig][0], in[ig][1], in[ig][2], in[ig][3]}, f4{in[ig][4], in[ig][5], in[ig][6], 0.f});
#pragma unroll
  for (int og = 0; og < NO; ++og)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ig = 0; ig < NI; ++ig) acc = mma(ld8(wl + ((og * 2 + u) * NI + ig) * 512), x[ig], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * u + i < 7) out[og][4 * u + i] = acc[i];
    }
}

// The small tables of one atom in LDS, where a read is a short wait and needs no address of its own.
struct Tab {
  float gamma[NATTN][M] __attribute__((aligned(16)));
  float beta[NATTN][M] __attribute__((aligned(16)));
  float b3[M], b2[E2], w1s[E1], Bt[NTYPES * E1];  // Bt: the centre's type
};
// Tile t of a per-feature table, in a token's arrangement.
__device__ __forceinline__ f4 tab4(const float *p, int t) {
  const int q = lane() >> 4;
  return t < 6 ? ldf4(p + 16 * t + 4 * q) : f4{p[96 + q], 0.f, 0.f, 0.f};
}
// By 128 threads (k from 0); every load is issued before the first is waited for.
__device__ __forceinline__ void load_tab(Tab &t, const Tables &w, int ti, int k) {
  static_assert(NTYPES * E1 <= 128 && NATTN == 2, "one entry of each table per thread");
  const int km = min(k, M - 1), k2 = min(k, E2 - 1), k1 = min(k, E1 - 1);
  const float bt = w.Bt[ti * NTYPES * E1 + min(k, NTYPES * E1 - 1)];
  const float g0 = w.gamma[0][km], g1 = w.gamma[1][km], b0 = w.beta[0][km], b1 = w.beta[1][km];
  const float b3 = w.b3[km], b2 = w.b2[k2], w1 = w.w1s[k1];
  if (k < NTYPES * E1) t.Bt[k] = bt;
  if (k < M) {
    t.gamma[0][k] = g0;
    t.gamma[1][k] = g1;
    t.beta[0][k] = b0;
    t.beta[1][k] = b1;
    t.b3[k] = b3;
  }
  if (k < E2) t.b2[k] = b2;
  if (k < E1) t.w1s[k] = w1;
}

// h1 and t2 = h2 - [h1, h1] by groups and t3 = G - [h2, h2] of the lane's token; w2T, w3T: the
// weights, in LDS.  h2 is left in scr (float32, [16][LDH]), from where residual() adds it.
__device__ __forceinline__ void embed(const Tab &w, const bf16_t *w2T, const bf16_t *w3T, float s, int tj, float *scr,
                                      S7 (&h1)[1], S7 (&t2)[2], F100 &t3) {
  const int l = lane(), q = l >> 4, c = l & 15;
  const float *bt = w.Bt + tj * E1;
#pragma unroll
  for (int r = 0; r < 7; ++r) {
    const int f = slot_ok(r) ? 4 * r + q : 0;
    const float v = act(s * w.w1s[f] + bt[f]);
    h1[0][r] = slot_ok(r) ? v : 0.f;
  }
  emul<1, 2>(t2, w2T, h1);
  bf8 x[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    float h[8] = {};
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      const int f = slot_ok(r) ? 25 * g + 4 * r + q : 0;
      const float v = act(t2[g][r] + w.b2[f]);
      t2[g][r] = slot_ok(r) ? v : 0.f;
      h[r] = t2[g][r] + h1[0][r];
      if (slot_ok(r)) scr[c * LDH + 25 * g + 4 * r + q] = h[r];
    }
    x[g] = pack(f4{h[0], h[1], h[2], h[3]}, f4{h[4], h[5], h[6], h[7]});
  }
#pragma unroll
  for (int t = 0; t < 7; ++t) {
    f4 acc = tab4(w.b3, t);
#pragma unroll
    for (int g = 0; g < 2; ++g) acc = mma(ld8(w3T + (2 * t + g) * 512 + 8 * l), x[g], acc);
#pragma unroll
    for (int k = 0; k < (t < 6 ? 4 : 1); ++k) t3[t][k] = act(acc[k]);
  }
}
// [h2, h2] in a token's arrangement: feature f is h2[f % 50].
__device__ __forceinline__ f4 residual(const float *scr, int t) {
  const int l = lane(), q = l >> 4;
  const float *h = scr + (l & 15) * LDH + 4 * q;
  typedef float f2 __attribute__((ext_vector_type(2)));
  if (t < 3) return ldf4(h + 16 * t);
  if (t == 6) return f4{scr[(l & 15) * LDH + 46 + q], 0.f, 0.f, 0.f};
  // 16 t + 4 q + i - 50, even; at t = 3, q = 0 the first two are still 48, 49
  const f2 a = *reinterpret_cast<const f2 *>(t == 3 && q == 0 ? h + 48 : h + 16 * t - 50);
  const f2 b = *reinterpret_cast<const f2 *>(h + 16 * t - 48);
  return f4{a[0], a[1], b[0], b[1]};
}

template <int N, int NT> using Fetch = Copy16<N / 8, NT>;
template <int NT> struct FetchEmb {  // W2^T, then W3^T
  Fetch<W2T_N, NT> a;
  Fetch<W3T_N, NT> b;
  __device__ __forceinline__ explicit FetchEmb(const WeightsB16 &wp) : a(wp.W2T), b(wp.W3T) {}
  __device__ __forceinline__ void store(bf16_t *d) const {
    a.store(d);
    b.store(d + W2T_N);
  }
};

// ======================================================================== forward
template <int NB> struct AtomFwd {
  bf16_t G[16 * NB * RW] __attribute__((aligned(16)));  // the layer's input, every token
  EnvF<NB> e;
  Tab tab;
};
template <int NB, int NA> struct SmemFwd {
  AtomFwd<NB> a[NA];
  bf16_t E[W2T_N + W3T_N] __attribute__((aligned(16)));
  union {
    bf16_t W[2][WMAT] __attribute__((aligned(16)));       // the layer's Wqk^T, Wvo^T
    float part[NA][NB][M * 4];                            // the waves' parts of T
  };
};

__device__ __forceinline__ void zero_block(bf16_t *block) {
#pragma unroll
  for (int p = 0; p < 4; ++p) *reinterpret_cast<bf8 *>(block + piece(piece0(), p)) = bf8{};
}

// The weights go through LDS: twelve waves reading 22 KB each for a product from the vector cache, at
// 64 bytes a cycle, took 4,100 cycles where the copy takes 350 and the LDS reads half.  A wave
// without tokens takes a path of its own, with the same copies and barriers, so that no register
// of the others' work is carried past a branch around it.
template <int NB, int NA>
__device__ __forceinline__ void desc_fwd(int blk, int count, SmemFwd<NB, NA> &sh, const Tables &w, const WeightsB16 &wp,
                                         const double *__restrict__ X, const int *__restrict__ types, int natoms,
                                         const int *__restrict__ idx, int c0, const int *__restrict__ nlist,
                                         const int *__restrict__ nnei, const Grid *__restrict__ grids,
                                         const int *__restrict__ sys_of, float rc, float rcs, float ln_eps,
                                         float *__restrict__ Gsave, float *__restrict__ Tsave) {
  constexpr int NT = 64 * NB * NA;
  const Part<NB, NA> pt(blk, idx, c0, count, nnei);
  AtomFwd<NB> &sm = sh.a[pt.half];
  const int i = pt.i, n = pt.n, nb = pt.nb, jb = pt.jb, tid = pt.tid;
  const Grid g = grids[sys_of[i]];
  const int l = lane(), q = l >> 4, c = l & 15;
  {
    const FetchEmb<NT> fe(wp);
    const Fetch<WMAT, NT> fu(wp.WqkT[0]), fy(wp.WvoT[0]);
    if (tid < 128) build_envf(sm.e, tid, X, types, nlist, i, n, natoms, g, rc, rcs);
    else if (tid < 256) load_tab(sm.tab, w, clamp_type(types[i]), tid - 128);
    fe.store(sh.E);
    fu.store(sh.W[0]);
    fy.store(sh.W[1]);
  }
  __syncthreads();
  const int j = 16 * jb + c;  // the lane's token
  bf16_t *block = sm.G + 16 * jb * RW;
  if (jb >= nb) {
    zero_block(block);
    __syncthreads();
    for (int layer = 1; layer < NATTN; ++layer) {
      const Fetch<WMAT, NT> fu(wp.WqkT[layer]), fy(wp.WvoT[layer]);
      __syncthreads();
      fu.store(sh.W[0]);
      fy.store(sh.W[1]);
      __syncthreads();
    }
    __syncthreads();
  } else {
    F100 x;  // the token's G
    XB xb;
    float *scr = reinterpret_cast<float *>(block);
    {
      S7 h1[1], t2[2];
      embed(sm.tab, sh.E, sh.E + W2T_N, sm.e.s[j], sm.e.tj[j], scr, h1, t2, x);
      wave_sync();
#pragma unroll
      for (int t = 0; t < 7; ++t) x[t] += residual(scr, t);
      wave_sync();
      xb = XB(x);
      put_block(block, xb);
    }
    __syncthreads();
    const float hj[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
#pragma unroll 1
    for (int layer = 0; layer < NATTN; ++layer) {
      f4 s[NB];
      {
        F100 u = {};
        wmul(u, sh.W[0], xb);  // U
        keys_dot<NB>(s, sm.G, XB(u), nb);  // S = U G^T
      }
      softmax_keys<NB>(s, sm.e, n, [](float v) { return __expf(v); });
      // the next layer's weights, on their way during the rest of this one
      const int next = layer + 1 < NATTN ? layer + 1 : layer;
      const Fetch<WMAT, NT> fu(wp.WqkT[next]), fy(wp.WvoT[next]);
      {
        F100 h = {};
        // H = A G with A = sw E gate
        rows_sum<NB>(h, sm.G, [&](int p) {
          const int k = 32 * p + 4 * q;
          return pack(s[2 * p] * gate4(sm.e, 2 * p, hj) * ldf4(sm.e.sw + k),
                      s[2 * p + 1] * gate4(sm.e, 2 * p + 1, hj) * ldf4(sm.e.sw + k + 16));
        }, nb);
        wmul(x, sh.W[1], XB(h));  // G + Y
      }
      // LayerNorm; the centred rows are what the backward reads
      const float mu = sum100([&](int t, int k) { return x[t][k]; }) * (1.f / M);
#pragma unroll
      for (int t = 0; t < 7; ++t) x[t] -= mu;
      save_block(Gsave + ((size_t)i * NATTN + layer) * GSAVE_LAYER + 1600 * jb, x);
      normalise(x, ln_eps);
#pragma unroll
      for (int t = 0; t < 7; ++t) x[t] = tab4(sm.tab.gamma[layer], t) * x[t] + tab4(sm.tab.beta[layer], t);
      __syncthreads();  // every wave is done with the layer's input and weights
      if (layer == NATTN - 1) break;
      xb = XB(x);
      put_block(block, xb);
      fu.store(sh.W[0]);
      fy.store(sh.W[1]);
      __syncthreads();
    }
    // T = G^T Rt / sel: each wave's 16 tokens on float32 MFMA (T^T = Rt^T G, rows c < 4 of the 16
    // used, step s taking token 4 s + q), three tiles of G at a time through the block's rows;
    // then the waves' parts in order
    float rt[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 16 * jb + 4 * s + q;
      const float sk = sm.e.s[k];
      rt[s] = c == 0 ? sk : (c < 4 ? sk * sm.e.rh[c - 1][k] : 0.f);
    }
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      wave_sync();
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        if (3 * h + t < 6) stf4(scr + c * LDH + 16 * t + 4 * q, x[3 * h + t]);
        if (3 * h + t == 6) scr[c * LDH + q] = x[6][0];
      }
      wave_sync();
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        if (3 * h + t > 6) continue;
        f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = mfma(rt[s], scr[(4 * s + q) * LDH + 16 * t + (h < 2 ? c : c & 3)], acc);
        if (q == 0 && (h < 2 || c < 4)) stf4(sh.part[pt.half][jb] + 4 * (48 * h + 16 * t + c), acc);
      }
    }
  }
  __syncthreads();
  for (int k = tid; k < (nb ? M * 4 : 0); k += 64 * NB) {
    float acc = 0.f;
    for (int v = 0; v < nb; ++v) acc += sh.part[pt.half][v][k];
    Tsave[(size_t)i * M * 4 + k] = acc * (1.f / (float)SEL);
  }
}

// One workgroup per NA atoms of its list; the 8-wave instance loops over its atoms with at most
// one workgroup per CU (or as many as there are atoms, without a list).
template <int NB, int NA>
__global__ void __launch_bounds__(64 * NB * NA) __attribute__((amdgpu_waves_per_eu(NB == NB_SMALL ? 3 : 2)))
k_desc_fwd_b16(Tables w, WeightsB16 wp, const double *__restrict__ X, const int *__restrict__ types, int natoms,
               const int *__restrict__ idx, const int *__restrict__ cnt, int c0, int ncen, const int *__restrict__ nlist,
               const int *__restrict__ nnei, const Grid *__restrict__ grids, const int *__restrict__ sys_of, float rc, float rcs,
               float ln_eps, float *__restrict__ Gsave, float *__restrict__ Tsave) {
  __shared__ SmemFwd<NB, NA> smem;
  const int count = idx ? *cnt : ncen;
  for (int b = blockIdx.x; b * NA < count; b += gridDim.x) {
    desc_fwd<NB, NA>(b, count, smem, w, wp, X, types, natoms, idx, c0, nlist, nnei, grids, sys_of, rc, rcs, ln_eps, Gsave, Tsave);
    if (NB == NB_SMALL) break;  // as many workgroups as atoms
    __syncthreads();
  }
}

// ======================================================================== backward
template <int NB> struct AtomBwd {
  bf16_t G[16 * NB * RW] __attribute__((aligned(16)));     // a layer's input, then dH, then U
  bf16_t K[16 * NB * RW] __attribute__((aligned(16)));     // the queries' rows of E gate, then of W
  float drhw[NB][16 * NB * 3];                             // each wave's column sums of dC rhat
  float wsum[NB][16 * NB] __attribute__((aligned(16)));    // ... of W
  float dT[M * 4] __attribute__((aligned(16)));
  EnvF<NB> e;
  Tab tab;
  float dRt[16 * NB][4] __attribute__((aligned(16)));      // dE/dRt of the tokens
  float dge[16 * NB][4] __attribute__((aligned(16)));      // the top layer's part of dE/drhat and dE/dsw
};
// Wvo and Wqk^T of a layer are read before the first rows go to K, so they are kept there (in the
// two atoms' K, or, with one atom, the second beside it); Wqk, and between the layers the
// embedding's weights, have space of their own.
template <int NB, int NA> struct SmemBwd {
  AtomBwd<NB> a[NA];
  bf16_t W[NA == 2 ? 1 : 2][WMAT] __attribute__((aligned(16)));
  float tile[NA == 2 ? 1 : NB][NA == 2 ? 4 : 256] __attribute__((aligned(16)));
  __device__ __forceinline__ bf16_t *wvo() { return a[0].K; }
  __device__ __forceinline__ bf16_t *wqkT() { return NA == 2 ? a[NA - 1].K : W[NA == 2 ? 0 : 1]; }
};
static_assert(sizeof(AtomBwd<NB_SMALL>::K) >= sizeof(bf16_t) * WMAT && WMAT >= W2T_N + W3T_N, "the weights fit");
static_assert(sizeof(AtomBwd<8>::G) * 2 >= sizeof(float) * 16 * 8 * LDG, "float32 rows of every token fit over G and K");

// Row r of a wave's 16 x 16 float32 tile: in the quarter of the block's rows of K that 96 keys leave
// free, or in `tile`.  put: the lane's four keys of token c; get: o[s] = token 4 q + (s ^ q), key c
// (s permuted so that the four lane groups are in different banks).
template <int NB> __device__ __forceinline__ float *tile_row(bf16_t *kblock, float *tile, int r) {
  return NB == NB_SMALL ? reinterpret_cast<float *>(kblock + r * RW + 32 * (3 ^ (r & 3))) : tile + 16 * r;
}
template <int NB> __device__ __forceinline__ void tile_put(bf16_t *kblock, float *tile, f4 y) {
  const int l = lane(), q = l >> 4, c = l & 15;
  stf4(tile_row<NB>(kblock, tile, c) + 4 * (q ^ (c >> 2)), y);
}
template <int NB> __device__ __forceinline__ f4 tile_get(bf16_t *kblock, float *tile) {
  const int l = lane(), q = l >> 4, c = l & 15;
  f4 o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o[s] = tile_row<NB>(kblock, tile, 4 * q + (s ^ q))[c ^ (4 * q)];
  return o;
}

// LayerNorm backward in place: dX = (dxh - mean(dxh) - xh mean(dxh xh)) / sigma, dxh = gamma dG_out.
__device__ __forceinline__ void norm_bwd(F100 &go, const F100 &xh, float is, const float *gamma) {
#pragma unroll
  for (int t = 0; t < 7; ++t) go[t] = tab4(gamma, t) * go[t];
  const float s0 = sum100([&](int t, int k) { return go[t][k]; }) * (1.f / M);
  const float s1 = sum100([&](int t, int k) { return go[t][k] * xh[t][k]; }) * (1.f / M);
#pragma unroll
  for (int t = 0; t < 7; ++t) go[t] = (go[t] - s0 - xh[t] * s1) * is;
}

// Backward of one layer, its input rows in sm.G.  go: in, the gradient of the LayerNorm's input
// (dX) for the wave's tokens, out, of the layer's input.  drh and dsw, the gradients of the
// token's rhat and sw, are added to.  Ends after a barrier; sm.G and sm.K are then free.
//   Row part (per token j): dH = Wvo dX; U, S, E recomputed; dA = G dH, then per key P = sw E,
//   dP = dA gate, rho = sum P dP, W = E (dP - rho), dS = sw W, dU = G^T dS, and dG_j = dX + Wqk dU.
//   (dH comes first: beside E the products' operands would not fit the registers.)
//   Column part (per key k): dG_k += sw_k sum_j (E gate)_jk dH_j + W_jk U_j, dsw_k += sum_j W_jk.
// What the column part needs of the row part: U, and W of the token's keys.
template <int NB> struct Column {
  XB ub;
  bf8 w[NB / 2];
};

template <int NB, int NA>
__device__ __forceinline__ void layer_bwd_rows(const WeightsB16 &wp, int layer, SmemBwd<NB, NA> &sh, AtomBwd<NB> &sm,
                                               F100 &go, Column<NB> &col, int jb, int n, int nb, float (&drh)[3]) {
  constexpr int NT = 64 * NB * NA;
  const int l = lane(), q = l >> 4, c = l & 15;
  const int j = 16 * jb + c;
  bf16_t *block = sm.G + 16 * jb * RW, *kblock = sm.K + 16 * jb * RW;
  float *tile = sh.tile[NA == 2 ? 0 : jb];
  XB &ub = col.ub, hb;
  const int p0 = piece0();
  const float hj[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
  {
    F100 dh = {};
    wmul(dh, sh.wvo(), XB(go));
    hb = XB(dh);
  }
  {
    F100 u = {};
#pragma unroll
    for (int p = 0; p < 4; ++p) ub.v[p] = ld8(block + piece(p0, p));
    wmul(u, sh.wqkT(), ub);
    ub = XB(u);
  }
  const Fetch<WMAT, NT> f(wp.Wqk[layer]);  // earlier it would wait in scratch memory
  f4 E[NB], W[NB];
  keys_dot<NB>(E, sm.G, ub, nb);
  f.store(sh.W[0]);
  softmax_keys<NB>(E, sm.e, n, [](float v) { return __expf(v); });
  keys_dot<NB>(W, sm.G, hb, nb);  // dA
  __syncthreads();  // K is free, Wqk is there
  float rho = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
  // columns of dC rhat: sum_j rhat_j (dA E)_jk, A operand rhat of the tile's tokens in rows a < 3
  float rj[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) rj[s] = c < 3 ? sm.e.rh[c][16 * jb + 4 * q + (s ^ q)] : 0.f;
  // a tile is read back while the next one's terms are formed
  const auto column_sums = [&](int kt) {
    const f4 ct = tile_get<NB>(kblock, tile);
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = mfma(rj[s], ct[s], acc);
    if (q == 0) {
      const float swk = sm.e.sw[16 * kt + c];
      float *o = sm.drhw[jb] + 3 * (16 * kt + c);
      o[0] = swk * acc[0]; o[1] = swk * acc[1]; o[2] = swk * acc[2];
    }
  };
#pragma unroll
  for (int p = 0; p < NB / 2; ++p)
    if (2 * p < nb) {
      f4 ea[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        tile_barrier();
        const int kt = 2 * p + h, k = 16 * kt + 4 * q;
        const f4 sw = ldf4(sm.e.sw + k), rx = ldf4(sm.e.rh[0] + k), ry = ldf4(sm.e.rh[1] + k), rz = ldf4(sm.e.rh[2] + k);
        const f4 gt = rx * hj[0] + ry * hj[1] + rz * hj[2];
        const f4 cc = W[kt] * E[kt];
        const f4 dC = sw * cc, dP = W[kt] * gt;  // P dP = dC gate
        if (kt > 0) column_sums(kt - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          rho = fmaf(dC[i], gt[i], rho);
          hx += dC[i] * rx[i];
          hy += dC[i] * ry[i];
          hz += dC[i] * rz[i];
        }
        W[kt] = dP;
        ea[h] = E[kt] * gt;
        wave_sync();
        tile_put<NB>(kblock, tile, cc);
        wave_sync();
      }
      *reinterpret_cast<bf8 *>(kblock + piece(p0, p)) = pack(ea[0], ea[1]);
    }
  column_sums(2 * ((nb + 1) / 2) - 1);
  rho = sumq(rho);
  drh[0] += sumq(hx);
  drh[1] += sumq(hy);
  drh[2] += sumq(hz);
  bf8 ds[NB / 2];  // dS
#pragma unroll
  for (int p = 0; p < NB / 2; ++p) {
    f4 d[2], v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kt = 2 * p + h;
      v[h] = E[kt] * (W[kt] - rho);
      d[h] = ldf4(sm.e.sw + 16 * kt + 4 * q) * v[h];
      const f4 s = sum16(v[h]);
      if (c == 0) stf4(sm.wsum[jb] + 16 * kt + 4 * q, s);
    }
    col.w[p] = pack(v[0], v[1]);
    ds[p] = pack(d[0], d[1]);
  }
  F100 du = {};
  rows_sum<NB>(du, sm.G, [&](int p) { return ds[p]; }, nb);
  wmul(go, sh.W[0], XB(du));
  const FetchEmb<NT> fe(wp);
  __syncthreads();  // the layer's input and weights are no longer needed
  fe.store(sh.W[0]);
  put_block(block, hb);
  __syncthreads();
}

// The rest, in two steps around the sums over dH: `between` may issue loads there.
template <int NB, int NA, class Fn>
__device__ __forceinline__ void layer_bwd_columns(AtomBwd<NB> &sm, F100 &go, const Column<NB> &col, int jb, int nb,
                                                  float (&drh)[3], float &dsw, const Fn &between) {
  const int l = lane(), c = l & 15;
  const int j = 16 * jb + c;
  bf16_t *block = sm.G + 16 * jb * RW, *kblock = sm.K + 16 * jb * RW;
  const int p0 = piece0();
  F100 acc = {};
  const int cj = (column0() ^ (32 * (jb >> 1))) + 4 * (jb & 1);
  const auto column = [&](int p) { return column8(sm.K + 32 * p * RW, cj); };
  rows_sum<NB>(acc, sm.G, column, nb);
  __syncthreads();
  between();
  put_block(block, col.ub);
#pragma unroll
  for (int p = 0; p < NB / 2; ++p)
    if (2 * p < nb) *reinterpret_cast<bf8 *>(kblock + piece(p0, p)) = col.w[p];
  __syncthreads();
  rows_sum<NB>(acc, sm.G, column, nb);
  const float swj = sm.e.sw[j];
#pragma unroll
  for (int t = 0; t < 7; ++t) go[t] += swj * acc[t];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const float ws = sm.wsum[u][j], d0 = sm.drhw[u][3 * j], d1 = sm.drhw[u][3 * j + 1], d2 = sm.drhw[u][3 * j + 2];
    if (u < nb) {
      dsw += ws;
      drh[0] += d0;
      drh[1] += d1;
      drh[2] += d2;
    }
  }
  __syncthreads();
}

// The same copies and barriers for a wave without tokens.
template <int NB, int NA>
__device__ __forceinline__ void layer_bwd_idle(const WeightsB16 &wp, int layer, SmemBwd<NB, NA> &sh, bf16_t *kblock) {
  constexpr int NT = 64 * NB * NA;
  {
    const Fetch<WMAT, NT> f(wp.Wqk[layer]);
    f.store(sh.W[0]);
  }
  __syncthreads();
  const FetchEmb<NT> fe(wp);
  zero_block(kblock);
  __syncthreads();
  fe.store(sh.W[0]);
  for (int k = 0; k < 4; ++k) __syncthreads();
}

template <int NB, int NA>
__device__ __forceinline__ void desc_bwd(int blk, int count, SmemBwd<NB, NA> &sh, const Tables &w, const WeightsB16 &wp,
                                         const double *__restrict__ X, const int *__restrict__ types, int natoms,
                                         const int *__restrict__ idx, int c0, const int *__restrict__ nlist,
                                         const int *__restrict__ nnei, const Grid *__restrict__ grids,
                                         const int *__restrict__ sys_of, float rc, float rcs, float ln_eps,
                                         const float *__restrict__ Gsave, const float *__restrict__ fit,
                                         float4 *__restrict__ gout) {
  constexpr int NT = 64 * NB * NA;
  const Part<NB, NA> pt(blk, idx, c0, count, nnei);
  AtomBwd<NB> &sm = sh.a[pt.half];
  const int i = pt.i, n = pt.n, nb = pt.nb, jb = pt.jb, tid = pt.tid;
  const Grid g = grids[sys_of[i]];
  const int l = lane(), q = l >> 4, c = l & 15;
  const float *gs = Gsave + (size_t)i * NATTN * GSAVE_LAYER + 1600 * jb;
  bf16_t *block = sm.G + 16 * jb * RW, *kblock = sm.K + 16 * jb * RW;
  F100 x, xh;  // the centred rows of layers 0 and 1
  {
    const int nj = tid < 128 ? env_neighbour(nlist, i, tid, n) : 0;
    load_block(x, gs);
    load_block(xh, gs + GSAVE_LAYER);
    const Fetch<WMAT, NT> fv(wp.Wvo[NATTN - 1]), fq(wp.WqkT[NATTN - 1]);
    if (tid < 128) {
      env_entry(sm.e, tid, nj, X, types, i, n, natoms, g, rc, rcs);
    } else if (tid < 256) {
      load_tab(sm.tab, w, clamp_type(types[i]), tid - 128);
    } else {
      const float *dTi = fit + (size_t)i * ND;
#pragma unroll
      for (int u = 0; u < (M * 4 + 64 * NB - 257) / (64 * NB - 256); ++u) {
        const int k = tid - 256 + u * (64 * NB - 256);
        if (k < M * 4) {
          float v = dTi[FIT_DT + k];
          if (k < 4 * M2)
#pragma unroll
            for (int p = 0; p < FIT_NPART; ++p) v += dTi[FIT_PART + 4 * M2 * p + k];
          sm.dT[k] = v;
        }
      }
    }
    fv.store(sh.wvo());
    fq.store(sh.wqkT());
    for (int k = nb ? 16 * nb + tid : SEL; k < SEL; k += 64 * NB) gout[(size_t)i * SEL + k] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (jb >= nb) {
    zero_block(block);
    __syncthreads();
    __syncthreads();
    layer_bwd_idle<NB, NA>(wp, 1, sh, kblock);
    {
      const Fetch<WMAT, NT> fv(wp.Wvo[0]), fq(wp.WqkT[0]);
      fv.store(sh.wvo());
      fq.store(sh.wqkT());
    }
    __syncthreads();
    layer_bwd_idle<NB, NA>(wp, 0, sh, kblock);
    return;
  }
  __syncthreads();
  const int j = 16 * jb + c;
  F100 go;
  float drh[3] = {0.f, 0.f, 0.f}, dsw = 0.f;
  {
    // the top layer's input: layer 0's output
    normalise(x, ln_eps);
#pragma unroll
    for (int t = 0; t < 7; ++t) x[t] = tab4(sm.tab.gamma[0], t) * x[t] + tab4(sm.tab.beta[0], t);
    put_block(block, XB(x));
    tile_barrier();
    // dG = Rt dT^T / sel for its output, and dRt = G dT / sel
    const float is = normalise(xh, ln_eps);
    const float inv_sel = 1.f / (float)SEL;
    const float sj = sm.e.s[j] * inv_sel;
    const float rt1 = sj * sm.e.rh[0][j], rt2 = sj * sm.e.rh[1][j], rt3 = sj * sm.e.rh[2][j];
    f4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 7; ++t) {
      tile_barrier();
      const f4 gv = tab4(sm.tab.gamma[1], t) * xh[t] + tab4(sm.tab.beta[1], t);
#pragma unroll
      for (int k = 0; k < (t < 6 ? 4 : 1); ++k) {
        const f4 d = ldf4(sm.dT + 4 * (t < 6 ? 16 * t + 4 * q + k : 96 + q));
        go[t][k] = sj * d[0] + rt1 * d[1] + rt2 * d[2] + rt3 * d[3];
        p += gv[k] * d;
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) p[a] = sumq(p[a]) * inv_sel;
    if (q == 0) stf4(sm.dRt[j], p);
    tile_barrier();
    norm_bwd(go, xh, is, sm.tab.gamma[1]);
    tile_barrier();
  }
  __syncthreads();
  Column<NB> col;
  layer_bwd_rows<NB, NA>(wp, 1, sh, sm, go, col, jb, n, nb, drh);
  {
    F100 x0, t3;
    Fetch<WMAT, NT> fv, fq;
    layer_bwd_columns<NB, NA>(sm, go, col, jb, nb, drh, dsw, [&] {  // layer 0's weights and rows, on their way from here
      fv.load(wp.Wvo[0]);
      fq.load(wp.WqkT[0]);
      load_block(x0, gs);
    });
    S7 h1[1], t2[2];
    float *scr = reinterpret_cast<float *>(block);
    embed(sm.tab, sh.W[0], sh.W[0] + W2T_N, sm.e.s[j], sm.e.tj[j], scr, h1, t2, t3);
    wave_sync();
#pragma unroll
    for (int t = 0; t < 7; ++t) t3[t] += residual(scr, t);
    wave_sync();
    put_block(block, XB(t3));
    fv.store(sh.wvo());
    fq.store(sh.wqkT());
    const float is = normalise(x0, ln_eps);
    norm_bwd(go, x0, is, sm.tab.gamma[0]);
    if (q == 0) stf4(sm.dge[j], f4{drh[0], drh[1], drh[2], dsw});  // registers spill
    drh[0] = drh[1] = drh[2] = dsw = 0.f;
  }
  __syncthreads();
  layer_bwd_rows<NB, NA>(wp, 0, sh, sm, go, col, jb, n, nb, drh);
  layer_bwd_columns<NB, NA>(sm, go, col, jb, nb, drh, dsw, [] {});
  // embedding backward and the pair gradients of the wave's tokens
  float *row = reinterpret_cast<float *>(sm.G) + j * LDG;  // over G and K
  S7 h1[1], t2[2], dh2[2];
  {
    F100 t3;
    float *scr = reinterpret_cast<float *>(sm.G) + 16 * jb * LDG;  // the block's rows, before dG is put there
    embed(sm.tab, sh.W[0], sh.W[0] + W2T_N, sm.e.s[j], sm.e.tj[j], scr, h1, t2, t3);
    wave_sync();
    put_row(row, go);
#pragma unroll
    for (int t = 0; t < 7; ++t) t3[t] = go[t] * (1.f - t3[t] * t3[t]);  // dpre3
    const XB d(t3);
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < 4; ++p) acc = mma(ld8(wp.W3 + ((2 * g2 + u) * 4 + p) * 512 + 8 * l), d.v[p], acc);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (4 * u + k < 7) dh2[g2][4 * u + k] = acc[k];
      }
  }
  wave_sync();
#pragma unroll
  for (int g2 = 0; g2 < 2; ++g2)
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      const float v = slot_ok(r) ? row[25 * g2 + 4 * r + q] + row[E2 + 25 * g2 + 4 * r + q] : 0.f;
      dh2[g2][r] += v;
      t2[g2][r] = dh2[g2][r] * (1.f - t2[g2][r] * t2[g2][r]);  // dpre2
    }
  S7 dh1[1];
  emul<2, 1>(dh1, wp.W2, t2);
  float ds = 0.f;
#pragma unroll
  for (int r = 0; r < 7; ++r) {
    const float v = dh1[0][r] + dh2[0][r] + dh2[1][r];
    if (slot_ok(r)) ds += v * (1.f - h1[0][r] * h1[0][r]) * sm.tab.w1s[4 * r + q];
  }
  ds = sumq(ds);
  if (q == 0 && j < SEL) {
    float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < n) {
      const float h[3] = {sm.e.rh[0][j], sm.e.rh[1][j], sm.e.rh[2][j]};
      const float dRt[4] = {sm.dRt[j][0], sm.dRt[j][1], sm.dRt[j][2], sm.dRt[j][3]};
      const f4 ge = ldf4(sm.dge[j]);
      for (int a = 0; a < 3; ++a) drh[a] += ge[a];
      out = pair_gradient(sm.e.s[j], sm.e.sw[j], sm.e.r[j], h, ds, dRt, drh, dsw + ge[3], rc, rcs);
    }
    gout[(size_t)i * SEL + j] = out;
  }
}

template <int NB, int NA>
__global__ void __launch_bounds__(64 * NB * NA) __attribute__((amdgpu_waves_per_eu(NB == NB_SMALL ? 3 : 2)))
k_desc_bwd_b16(Tables w, WeightsB16 wp, const double *__restrict__ X, const int *__restrict__ types, int natoms,
               const int *__restrict__ idx, const int *__restrict__ cnt, int c0, int ncen, const int *__restrict__ nlist,
               const int *__restrict__ nnei, const Grid *__restrict__ grids, const int *__restrict__ sys_of, float rc, float rcs,
               float ln_eps, const float *__restrict__ Gsave, const float *__restrict__ fit, float4 *__restrict__ gout) {
  __shared__ SmemBwd<NB, NA> smem;
  const int count = idx ? *cnt : ncen;
  for (int b = blockIdx.x; b * NA < count; b += gridDim.x) {
    desc_bwd<NB, NA>(b, count, smem, w, wp, X, types, natoms, idx, c0, nlist, nnei, grids, sys_of, rc, rcs, ln_eps, Gsave, fit, gout);
    if (NB == NB_SMALL) break;
    __syncthreads();
  }
}

}  // namespace

void launch_descriptor_fwd_b16(const Tables &w, const WeightsB16 &wp, const Workspace &ws, const double *coords,
                               const int *types, int n, int c0, int c1, float rc, float rcs, float ln_eps, hipStream_t st) {
  launch_descriptor_lists(ws, n, c0, c1, st);
  launch_instances(ws, n, c1 - c0, k_desc_fwd_b16<NB_SMALL, 2>, k_desc_fwd_b16<8, 1>, st,
                   [&](auto kernel, int groups, int threads, const int *idx, const int *cnt, hipStream_t s) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(threads), 0, s, w, wp, coords, types, n, idx, cnt, c0, c1 - c0, ws.nlist,
                       ws.nnei, ws.grids, ws.sys_of, rc, rcs, ln_eps, ws.Gsave, ws.Tsave);
  });
}

void launch_descriptor_bwd_b16(const Tables &w, const WeightsB16 &wp, const Workspace &ws, const double *coords,
                               const int *types, int n, int c0, int c1, float rc, float rcs, float ln_eps, hipStream_t st) {
  launch_instances(ws, n, c1 - c0, k_desc_bwd_b16<NB_SMALL, 2>, k_desc_bwd_b16<8, 1>, st,
                   [&](auto kernel, int groups, int threads, const int *idx, const int *cnt, hipStream_t s) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(threads), 0, s, w, wp, coords, types, n, idx, cnt, c0, c1 - c0, ws.nlist,
                       ws.nnei, ws.grids, ws.sys_of, rc, rcs, ln_eps, ws.Gsave, ws.fit, ws.g);
  });
}

}  // namespace dp
