// Projection added to the residual stream in its epilogue.
#include "gemm_ring.h"

namespace trj {

// ---- epilogue: x[t][n_out] += acc (fp32); 4 consecutive features per access
struct EpiResidual {
  static constexpr bool kScaled = false;
  float* x;
  int ld, T;
  __device__ void operator()(const f32x16& acc, int tile, int ttile, int lane, int) const {
    const int t = ttile * 32 + (lane & 31);
    if (t >= T) return;
    float* row = x + (size_t)t * ld + tile * 32 + 4 * (lane >> 5);
    f32x4 v[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) v[g] = *reinterpret_cast<const f32x4*>(row + 8 * g);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[g][e] += acc[4 * g + e];
      *reinterpret_cast<f32x4*>(row + 8 * g) = v[g];
    }
  }
};

int launch_gemm_residual(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, float* x,
                         hipStream_t st) {
  return launch_gemm(xp, w, tp, n_in, n_out, 1, EpiResidual{x, n_out, T}, st);
}

}  // namespace trj
