// Device-side building blocks shared by the gfx950 kernels: sizes, vector types, cross-lane
// row reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dp {

// ---------------------------------------------------------------- model sizes
constexpr int NTYPES = 5;
constexpr int TEBD = 8;
constexpr int E1 = 25;       // embedding widths 17 -> 25 -> 50 -> 100
constexpr int E2 = 50;
constexpr int M = 100;       // neighbour representation width
constexpr int NATTN = 2;     // attention layers
constexpr int DATTN = 128;   // attention width (enters through the fused 100x100 products)
constexpr int M2 = 16;       // axis neurons
constexpr int ND = M * M2;   // descriptor length 1600
constexpr int FH = 240;      // fitting width
// An atom's row of Workspace::fit as the descriptor backward reads it: dE/dT [M][4] at
// FIT_DT, to which FIT_NPART partial sums [16][4] from FIT_PART on are added.
constexpr int FIT_DT = 960, FIT_PART = 1360, FIT_NPART = 3;
constexpr int SEL = 120;     // neighbour capacity
constexpr int NPMAX = 128;   // tokens per atom after padding to a multiple of 16
constexpr int GSAVE_LAYER = NPMAX * M;  // floats per atom and layer of the saved layer inputs

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16_t;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

// Cross-lane moves within a row of 16 lanes by DPP (no LDS round trip): the value of
// the partner lane.  Quad permutations 0xB1 (lane ^ 1) and 0x4E (lane ^ 2), half-row
// mirror 0x141 (lane ^ 7 within 8), row mirror 0x140 (lane ^ 15 within 16) and row
// rotation by 8, 0x128 (lane ^ 8 within 16).  Every lane of the wave must be active.
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// Sum over the 16 lanes sharing lane/16 (one tile row group); the same value in all of
// them (each step adds a partner's value, and a + b == b + a exactly).
__device__ __forceinline__ float sum16(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  return v;
}

}  // namespace dp
