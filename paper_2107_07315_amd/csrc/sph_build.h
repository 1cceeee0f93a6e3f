// Parts of the candidate-list builds: the operands of the matrix-core pair test (and, in sph_listout.h, a
// target's list in the making).
#pragma once
#include "sph_internal.h"
#include "sph_listout.h"

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t dpp_or(uint32_t v) {   // OR over the wave, in lane 63
#define SPH_DPP_OR(ctrl, rows) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, true)
  SPH_DPP_OR(0x111, 0xf);   // row_shr 1, 2, 4, 8
  SPH_DPP_OR(0x112, 0xf);
  SPH_DPP_OR(0x114, 0xf);
  SPH_DPP_OR(0x118, 0xf);
  SPH_DPP_OR(0x142, 0xa);   // row_bcast 15, 31
  SPH_DPP_OR(0x143, 0xc);
#undef SPH_DPP_OR
  return v;
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)dpp_or(v), 63); }

// exchanges the upper 32 lanes of a with the lower 32 lanes of b
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
// The operands of both 32-wide blocks from one particle per lane: 16 FP16 components k, of which
// lane l < 32 of a block's operand holds 0..7 of the block's particle l and lane l >= 32 holds 8..15
// of particle l - 32.  TARGET: the target's side (B), else the candidate's (A).
template <bool TARGET>
__device__ __forceinline__ void lift_operands(float x, float y, float z, float h, float w, f16x8 op[2]) {
  const float s = TARGET ? 1.f : -2.f;
  const float v[5] = {s * x, s * y, s * z, s * h, w};
  _Float16 hi[5], lo[5];
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    hi[d] = (_Float16)v[d];
    lo[d] = (_Float16)(v[d] - (float)hi[d]);
  }
  const _Float16 one = (_Float16)1.f;
  _Float16 k[16];
#pragma unroll
  for (int d = 0; d < 4; ++d) {   // candidate (hi, hi, lo) by target (hi, lo, hi)
    k[3 * d] = hi[d];
    k[3 * d + 1] = TARGET ? lo[d] : hi[d];
    k[3 * d + 2] = TARGET ? hi[d] : lo[d];
  }
  k[12] = TARGET ? one : hi[4];
  k[13] = TARGET ? one : lo[4];
  k[14] = TARGET ? hi[4] : one;
  k[15] = TARGET ? lo[4] : one;
  uint32_t a[4], b[4];
  __builtin_memcpy(a, k, sizeof(a));
  __builtin_memcpy(b, k + 8, sizeof(b));
#pragma unroll
  for (int i = 0; i < 4; ++i) swap32(a[i], b[i]);
  __builtin_memcpy(&op[0], a, sizeof(a));
  __builtin_memcpy(&op[1], b, sizeof(b));
}

}  // namespace
