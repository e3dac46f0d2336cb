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

// ---- epilogue: the same, and the next norm's input bf16(x * g) in the tiled activation layout (zeros in
// rows T .. tp-1); returns the sum of x^2 over the tile's 32 features, which gemm_pair_kernel adds up per
// workgroup and writes to ssq[row group][row].  As a launch of its own behind the projection
// (reduce_norm_kernel) this read and wrote the whole stream again, 10.5 us at 1024 x 4096.  Steps of two
// layers with 1024 rows 1325 -> 1292 us, 768 rows 1061 -> 1056, a prompt of 1000 886 -> 871; the readers pay
// 1 to 2 us for 32 sums per row instead of four.
struct EpiResidualNorm {
  static constexpr bool kScaled = false;
  float* x;
  int ld, T;
  const float* g;
  uint16_t* hp;
  int tp;
  float* ssq;
  __device__ float operator()(const f32x16& acc, int tile, int ttile, int lane, int) const {
    const int t = ttile * 32 + (lane & 31), f = tile * 32 + 4 * (lane >> 5);
    float ss = 0.f;
    if (t < T) {
      float* row = x + (size_t)t * ld + f;
      f32x4 v[4], gv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = *reinterpret_cast<const f32x4*>(row + 8 * i);
        gv[i] = *reinterpret_cast<const f32x4*>(g + f + 8 * i);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[i][e] += acc[4 * i + e];
          ss += v[i][e] * v[i][e];
        }
        *reinterpret_cast<f32x4*>(row + 8 * i) = v[i];
        const u32x2 pk = {pack2bf(v[i][0] * gv[i][0], v[i][1] * gv[i][1]), pack2bf(v[i][2] * gv[i][2], v[i][3] * gv[i][3])};
        *reinterpret_cast<u32x2*>(hp + a_off(t, f + 8 * i, tp)) = pk;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x2*>(hp + a_off(t, f + 8 * i, tp)) = u32x2{0, 0};
    }
    return ss + __shfl_xor(ss, 32);
  }
};
// Where one workgroup per compute unit takes turns (gemm_pair.h): the other shapes own too few features of a
// row for a sum worth writing, or run split along k; whole row groups.
bool gemm_residual_norm_runs(int tp, int n_in, int n_out, const void* xp, const void* w) {
  return (((uintptr_t)xp | (uintptr_t)w) & 15) == 0 && n_out % 128 == 0 && plan_gemm(tp, n_in, n_out, 1).pair;
}
int launch_gemm_residual_norm(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, float* x,
                              const float* g, uint16_t* hp, float* ssq, hipStream_t st) {
  launch_pair(xp, w, tp, n_in, n_out, EpiResidualNorm{x, n_out, T, g, hp, tp, ssq}, st);
  return check_launch();
}

int launch_gemm_residual(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, float* x,
                         hipStream_t st) {
  return launch_gemm(xp, w, tp, n_in, n_out, 1, EpiResidual{x, n_out, T}, st);
}

}  // namespace trj
