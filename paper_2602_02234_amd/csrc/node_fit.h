// Fitting net of the message-passing models over node rows: E_i = y2 . G3 + d3,
// y2 = tanh(y1 G2 + d2) + y1, y1 = tanh(n_i G1 + d1), widths 64 -> 128 -> 128, and dE_i/dn_i.
#pragma once
#include <vector>

#include "dp_internal.h"

namespace dp {

struct NodeFit {
  static constexpr int IN = 64, WID = 128;
  const float *G1, *G2, *G2T, *G1T;  // MFMA fragment order, outputs by inputs: 128 x 64, 128 x 128 (twice), 64 x 128
  const float *d1, *d2, *G3;
  const double *G3d;
  double d3;
};
// rows: [n][64], node features in, dE_i/dn_i out; Ei [n].  Writes nothing after an error.
void launch_node_fit(const NodeFit &w, float *rows, int n, double *Ei, const unsigned *flags, hipStream_t st);

// W[out][k], outs and K multiples of 16, in the fragment order of dp_tiles.h (float32).
template <class F> std::vector<float> node_fragments(int outs, int K, const F &W) {
  std::vector<float> v((size_t)outs * K);
  for (int t = 0; t < outs / 16; ++t)
    for (int k = 0; k < K / 16; ++k)
      for (int l = 0; l < 64; ++l)
        for (int s = 0; s < 4; ++s)
          v[((size_t)(t * (K / 16) + k) * 64 + l) * 4 + s] = (float)W(16 * t + l % 16, 16 * k + 4 * (l / 16) + s);
  return v;
}

}  // namespace dp
