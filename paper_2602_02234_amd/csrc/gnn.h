// The GNN-variant descriptor (the paper's second model family, Section II: message
// passing over bonds and angles in place of attention): sizes, device weights and
// buffers, launchers.
//
// Model (the functional form the library implements; the paper gives none):
//   edges (i, j), j in N(i) (r_ij < rc); angles at i: ordered pairs (p, q), p != q, of
//   the first asel neighbours of i (list order) with r < rca;
//   n_i = TN[t_i];  e_ij = tanh(s_ij We0 + be0), s = sw_e(r) / r;
//   a_ipq = tanh(c_ipq Wa0 + ba0), c = rhat_ip . rhat_iq;
//   three layers, each: a <- a + tanh([a, e_ip[:32], e_iq[:32]] Waa + baa);
//     m_ip = sum_q sw_a(r_ip) sw_a(r_iq) / asel tanh([a, e_iq[:32]] Wea + bea);
//     e_ij <- e_ij + tanh([n_i, n_j, e_ij] Wee + bee) + m_ij;
//     n_i <- n_i + tanh([n_i, sum_j sw_e(r_ij) e_ij / sel] Wnn + bnn);
//   E_i = y2 G3 + d3, y2 = tanh(y1 G2 + d2) + y1, y1 = tanh(n_i G1 + d1).
#pragma once
#include "dp_internal.h"

namespace dp {
namespace gnn {

constexpr int NDIM = 64;   // node width
constexpr int EDIM = 64;   // edge width
constexpr int ADIM = 32;   // angle width (and the edge columns angles read)
constexpr int NLAYER = 3;
constexpr int FWID = 128;  // fitting width
constexpr int ASEL = 48;   // largest angle-neighbour count a model may set

// A weight matrix in the MFMA fragment order of the layer kernels (see gnn.hip), in the
// precision of the model's products.
struct Frag {
  const float *f32 = nullptr;
  const bf16_t *b16 = nullptr;
};

// Device weights: float32, row-major [in][out] as in the model file (the T-named copies
// transposed), and the fragment-ordered operands.
struct Weights {
  const float *TN;                // [NTYPES][64]
  const float *We0, *be0;         // [64]
  const float *Wa0, *ba0;         // [32]
  const float *baa[NLAYER], *bea[NLAYER];  // [32], [64]  (Waa and Wea are read in fragment order only)
  const float *Wee[NLAYER], *bee[NLAYER];  // [192][64], [64]
  const float *Wnn[NLAYER], *bnn[NLAYER];  // [128][64], [64]
  const float *G1, *d1, *G2, *d2, *G3;     // [64][128], [128], [128][128], [128], [128]
  const float *G1T, *G2T;         // [128][64], [128][128]
  const float *WnnT[NLAYER];      // [64][128]
  const float *WeeT[NLAYER];      // [64][64]  of Wee[0:64]
  Frag A[NLAYER], Mg[NLAYER];     // a -> Waa[0:32] (32 outputs), a' -> Wea[0:32] (64)
  Frag Xt[NLAYER], Yt[NLAYER];    // dz_m -> Wea[0:32]^T (32 outputs of 64), dz_a -> Waa[0:32]^T
  Frag E[NLAYER];                 // [n_j, e] -> Wee[64:192] (64 outputs of 128)
  Frag N[NLAYER], D[NLAYER];      // dz_e -> Wee[64:128]^T and Wee[128:192]^T
  const float *PQ[NLAYER];        // e[:32] -> [Waa[32:64], Waa[64:96], Wea[32:64]] (128 outputs of 32), float32
  const float *PS[NLAYER];        // edge sums -> dE/de[:32] (32 outputs of 128), float32
  const double *G3d;              // [128]  last layer in float64 (energy sum)
  double d3;
};

// Per-step device buffers.  Edge rows use the neighbour-list stride SEL; angles of atom
// i start at aoff[i] (p-major: angle (p, q) at aoff[i] + p (nc_i - 1) + q - (q > p)).
struct Buffers {
  int64_t cap = 0, acap = 0;  // atoms, angles
  int64_t *aoff = nullptr;    // [cap + 1]: angle offsets
  float *nf = nullptr;        // [2][cap][64]       n after layers 1, 2
  float *ef = nullptr;        // [3][cap][SEL][64]  e after layers 1, 2, 3
  float *af = nullptr;        // [2][acap][32]      a after layers 1, 2 (the backward recomputes layer 3's)
  float *da = nullptr;        // [acap][32]         dE/da, updated in place layer by layer
  float *de = nullptr;        // [cap][SEL][64]     dE/de, likewise
  float *dnj = nullptr;       // [2][cap][SEL][64]  edge (i, j)'s part of dE/dn_j, by layer parity
  float *dnl = nullptr;       // [cap][64]          atom i's own part of dE/dn_i
  float *gs = nullptr;        // [cap][SEL][2]      dE/dsw_e, dE/dsw_a per edge over the layers
  int *slot = nullptr;        // [cap][SEL]         position of i in the list of its j-th neighbour, or -1
};

struct Geo {
  float rc, rcs, rca, inv_sel, inv_asel;
  int asel;
};

// aoff[1 .. n]: angle counts of every atom, then their inclusive prefix (aoff[0] = 0).
// host_tot (pinned host memory): the step's angles, edges (sum of the list lengths) and
// angle-list edges.  Sets FLAG_INCOMPLETE if a list was truncated, and FLAG_ANGLES if the
// angle buffers are too small: the step's later kernels then write nothing.
void launch_angle_offsets(const Buffers &b, const Workspace &ws, const double *coords, int n, const Geo &geo,
                          int64_t *host_tot, hipStream_t st);
// Up to this many atoms every CU holds at most one workgroup of four waves on each SIMD
// pair; eight waves per atom then shorten the step, and take the fitting net along.
constexpr int WIDE_UP_TO = 512;
inline bool separate_fit(int n) { return n > WIDE_UP_TO; }
// Layer `layer` (0 .. 2) forward over all n atoms.  After the last one the fitting net gives E_i (Ei)
// and dE/dn (dnl): within the layer's kernel, or (separate_fit) by launch_node_fit from the rows n
// that the layer leaves in dnl.
template <typename T>
void launch_layer_fwd(const Weights &w, const Buffers &b, const Workspace &ws, const double *coords,
                      const int *types, int n, int layer, const Geo &geo, double *Ei, hipStream_t st);
// Layer `layer` backward (called for 2, 1, 0); layer 0 writes g_ij = dE/dDelta_ij into ws.g.
template <typename T>
void launch_layer_bwd(const Weights &w, const Buffers &b, const Workspace &ws, const double *coords,
                      const int *types, int n, int layer, const Geo &geo, hipStream_t st);

}  // namespace gnn
}  // namespace dp
