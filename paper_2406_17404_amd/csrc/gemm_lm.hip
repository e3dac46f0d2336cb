// LM head: logits and the greedy argmax, both in the projection's epilogue.
#include "gemm_ring.h"

namespace trj {

// acc layout of v_mfma_f32_32x32x16: lane l, register v -> tile row 8*(v/4) + 4*(l/32) +
// v%4, tile column l%32.  Rows are output features, columns are token rows.

// ---- epilogue: greedy argmax (Eq. 1's arg max taken where the logits are born) and, if the
// caller wants them, the fp32 logits.  Every wavefront reduces the 32 vocabulary rows of its
// tile for each of its 32 token columns and writes one candidate (value, index) per (token,
// row tile); a second, small kernel picks the winner among a token's candidates.  Lowest
// index wins ties, NaN never wins (a candidate that saw nothing keeps index INT32_MAX).
// Reading the logits back for the argmax took 6.4 us at 5 rows x 32000 and 17 us at 69 x
// 128256, the candidates' kernel 4.6.
struct EpiLm {
  static constexpr bool kScaled = true;
  RowScale rs;
  ArgmaxCand* cand;  // [T][n_tiles], null: none
  float* logits;     // [T][32 n_tiles], null: none
  int T, n_tiles;
  __device__ void operator()(const f32x16& acc, int tile, int ttile, int lane, int) const {
    float bv = -INFINITY;
    int bi = INT32_MAX;
#pragma unroll
    for (int v = 0; v < 16; ++v) {  // ascending row index within the lane
      const int row = tile * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      if (acc[v] > bv || (acc[v] == bv && row < bi)) { bv = acc[v]; bi = row; }
    }
    const float ov = __shfl_xor(bv, 32);
    const int oi = __shfl_xor(bi, 32);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    const int t = ttile * 32 + (lane & 31);
    if (t >= T) return;
    if (cand && lane < 32) cand[(size_t)t * n_tiles + tile] = ArgmaxCand{bv, bi};
    if (!logits) return;
    float* row = logits + ((size_t)t * n_tiles + tile) * 32 + 4 * (lane >> 5);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
      *reinterpret_cast<f32x4*>(row + 8 * g) = v;
    }
  }
};

// argmax_out[t] = lowest index of the row maximum of x W^T; cand: T * n_out / 32 candidates
__global__ __launch_bounds__(256) void argmax_cand_kernel(const ArgmaxCand* __restrict__ cand,
                                                          int n_tiles, int32_t* __restrict__ out) {
  const ArgmaxCand* row = cand + (size_t)blockIdx.x * n_tiles;
  float bv = -INFINITY;
  int bi = INT32_MAX;
  for (int j0 = threadIdx.x; j0 < n_tiles; j0 += 256 * 8) {  // 8 loads in flight (clamped index)
    ArgmaxCand c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = row[min(j0 + u * 256, n_tiles - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (c[u].v > bv || (c[u].v == bv && c[u].i < bi)) { bv = c[u].v; bi = c[u].i; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(bv, o);
    const int oi = __shfl_xor(bi, o);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  __shared__ float sv[4];
  __shared__ int si[4];
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = bv; si[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (sv[w] > bv || (sv[w] == bv && si[w] < bi)) { bv = sv[w]; bi = si[w]; }
    out[blockIdx.x] = bi == INT32_MAX ? 0 : bi;
  }
}
int launch_gemm_lm(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, const RowScale& rs,
                   float* logits, void* cand, int32_t* argmax_out, hipStream_t st) {
  EpiLm e{rs, static_cast<ArgmaxCand*>(cand), logits, T, n_out / 32};
  int rc = launch_gemm(xp, w, tp, n_in, n_out, 1, e, st);
  if (rc != TRJ_OK || !cand || !argmax_out) return rc;
  argmax_cand_kernel<<<T, 256, 0, st>>>(static_cast<const ArgmaxCand*>(cand), n_out / 32, argmax_out);
  return check_launch();
}

}  // namespace trj
