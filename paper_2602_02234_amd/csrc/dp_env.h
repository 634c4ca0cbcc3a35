// Per-atom environment (shared by the descriptor kernels of both precisions).
//   Delta = x_j - x_i (minimum image), r = |Delta|, u = (r - rcs) / (rc - rcs),
//   sw = 1 below rcs, u^3 (-6u^2 + 15u - 10) + 1 up to rc, 0 beyond (quintic, C2);
//   s = sw / r, rhat = Delta / r, Rt = (s, s rhat).  Padded tokens (j >= n) are zero.
#pragma once
#include "dp_internal.h"

namespace dp {

__device__ __forceinline__ int clamp_type(int t) { return t < 0 ? 0 : (t >= NTYPES ? NTYPES - 1 : t); }

// The last step of the backward pass for one token: combine the gradients that reached
// s (ds_emb through the embedding input, dRt through Rt), rhat (drh, through the gate;
// and through Rt) and sw (dswa, through the softmax weights) into g = dE_i / dDelta_ij;
// the switch derivative is formed here from r.
__device__ __forceinline__ float4 pair_gradient(float s, float sw, float rr, const float *h, float ds_emb,
                                                const float *dRt, const float *drh, float dswa, float rc, float rcs) {
  const float hx = h[0], hy = h[1], hz = h[2];
  const float u = (rr - rcs) / (rc - rcs);
  const float dsw = (rr >= rcs && rr < rc) ? -30.f * u * u * (1.f - u) * (1.f - u) / (rc - rcs) : 0.f;
  const float ds = ds_emb + dRt[0] + dRt[1] * hx + dRt[2] * hy + dRt[3] * hz;
  const float gx = drh[0] + s * dRt[1];
  const float gy = drh[1] + s * dRt[2];
  const float gz = drh[2] + s * dRt[3];
  const float dswt = dswa + ds / rr;
  const float dr = -ds * sw / (rr * rr) + dswt * dsw;
  const float proj = gx * hx + gy * hy + gz * hz;
  return make_float4((gx - proj * hx) / rr + dr * hx, (gy - proj * hy) / rr + dr * hy, (gz - proj * hz) / rr + dr * hz,
                     0.f);
}

}  // namespace dp
