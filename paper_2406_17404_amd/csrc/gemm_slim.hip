// Projection of up to eight rows into the residual stream, with the sum, the residual add and the next
// norm's input in one launch.
//
// What bounds it: with so few rows the weights stream at the rate HBM gives (7.1 TB/s), and every launch
// costs some 4 us on top, whatever it does.  A projection split along k over workgroups needs a second
// launch for the sum of its parts (reduce_norm_kernel).  Here a workgroup owns 16 output features and the
// whole k range, so that 4096 features are a workgroup for each compute unit and nothing is left to add.
// The price is activations: with half a weight tile per workgroup, eight rows of them are half as many
// bytes as the weights, read from L2.  Whole steps of two layers of the 7B shape on 777 slots, us, split
// with a sum behind it -> this: 1 row 236.0 -> 226.8, 5 rows 239.5 -> 229.3, 8 rows 240.2 -> 230.4; grouped-query
// 8B shape, 5 rows 364.1 -> 355.8.  From nine rows on the activations are as many bytes as the weights
// and more: 16 rows 242.8 -> 244.2 (with the down projection split as before 241.1, but of the 8B shape 369.1
// -> 370.1), 32 rows 247.0 -> 267.3.
#include "gemm_ring.h"

namespace trj {

constexpr int SLIM_WAVES = 8, SLIM_ROWS = 8;

// Eight wavefronts; wavefront kw multiplies every eighth pair of k-steps (v_mfma_f32_16x16x32_bf16: lane l
// holds feature or token l % 16 and the 8 columns 8 * (l / 16) .. of 32, which in the 32 x 16 tiles of both
// operands is 16 bytes).  Nobody shares an operand, so all of them go straight to registers, U pairs at a
// time, the next U asked for before the current ones are used.  Token columns 8 .. 15 repeat 0 .. 7.
template <int U>
__global__ __launch_bounds__(SLIM_WAVES * 64, 2) void gemm_slim_kernel(const uint16_t* __restrict__ xp,
                                                                       const uint16_t* __restrict__ w, int pairs, int T,
                                                                       int d, float* __restrict__ x,
                                                                       const float* __restrict__ g,
                                                                       uint16_t* __restrict__ hp,
                                                                       float* __restrict__ ssq) {
  __shared__ float part[SLIM_WAVES][16 * SLIM_ROWS];
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int f0 = blockIdx.x * 16;
  // workgroups start at different places of the k range and go round, as in gemm_ring_kernel
  const int first = (int)((blockIdx.x * 40503u & 0xffffu) * (uint32_t)pairs >> 16);
  const int op = (lane >> 5) * 1024 + ((lane >> 4) & 1) * 512;  // k-step and half of this lane's 16 bytes
  const uint8_t* wl = reinterpret_cast<const uint8_t*>(w) + (size_t)(f0 >> 5) * pairs * 2048 + op + ((f0 & 16) + (lane & 15)) * 16;
  const uint8_t* xl = reinterpret_cast<const uint8_t*>(xp) + op + (lane & (SLIM_ROWS - 1)) * 16;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  u32x4 wa[2][U], xa[2][U];
  auto load = [&](int j0, int s) {  // pairs past the end are read from the last one and cleared below
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int p = min((j0 + u) * SLIM_WAVES + kw, pairs - 1) + first;
      if (p >= pairs) p -= pairs;
      wa[s][u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wl + (size_t)p * 2048));
      xa[s][u] = *reinterpret_cast<const u32x4*>(xl + (size_t)p * 2048);
    }
  };
  auto multiply = [&](int j0, int s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((j0 + u) * SLIM_WAVES + kw >= pairs) wa[s][u] = xa[s][u] = u32x4{0, 0, 0, 0};  // uniform
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[s][u]),
                                                    __builtin_bit_cast(bf16x8, xa[s][u]), acc, 0, 0, 0);
    }
  };
  const int n = (pairs + SLIM_WAVES - 1) / SLIM_WAVES;
  load(0, 0);
  // thread e ends with feature e % 16 of row e / 16
  const int e = threadIdx.x, row = e >> 4, f = f0 + (e & 15);
  const float gv = g[f], xv = x[(size_t)min(row, T - 1) * d + f];
  int j = 0;
  for (; j + 2 * U < n; j += 2 * U) {
    load(j + U, 1);
    multiply(j, 0);
    load(j + 2 * U, 0);
    multiply(j + U, 1);
  }
  if (j + U < n) {
    load(j + U, 1);
    multiply(j, 0);
    multiply(j + U, 1);
  } else {
    multiply(j, 0);
  }
  // lane l, register v: feature 4 * (l / 16) + v of token l % 16
  if ((lane & 15) < SLIM_ROWS)
    *reinterpret_cast<f32x4*>(&part[kw][(lane & 15) * 16 + (lane >> 4) * 4]) = acc;
  __syncthreads();
  if (e >= 16 * SLIM_ROWS) return;  // whole wavefronts
  float s = xv;
#pragma unroll
  for (int k = 0; k < SLIM_WAVES; ++k) s += part[k][e];  // fixed order
  const bool live = row < T;
  if (live) x[(size_t)row * d + f] = s;
  hp[a_off(row, f, 32)] = live ? (uint16_t)(pack2bf(s * gv, 0.f) & 0xffffu) : 0;
  float ss = s * s;
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if (live && (e & 15) == 0) ssq[(size_t)row * (d >> 4) + blockIdx.x] = ss;
}

// At least half of the compute units with a workgroup, and no more parts per row than the wavefronts
// of the consuming projection read with one load (4 x 64).  A k range of at most so many rounds of 2048
// columns (SLIM_STEPS pairs of k-steps for each wavefront, as long for a part of one): a workgroup's time grows with
// the rounds alone, that of a projection split over all compute units with the product, so the narrower the
// output the sooner the split one is ahead in spite of its sum.  us of one projection, this less split with
// its sum, 1 to 8 rows alike:
//   outputs  2048  4 rounds -0.5 (8192 columns) +0.6 (6176)    5 rounds +2.2 (10240) +2.9 (8224)
//            2560  5        -0.7 (10240)        -0.1 (8224)    6        -0.5 (12288) +0.9 (10272)
//            3072  6        -1.4 (12288)        -0.1 (10272)   7         0.0 (14336) +1.3 (12800)
//            3328  8        -1.9 (16384)        -1.2 (14368)   9        +1.1 (17408)
//            4096  8        -0.7 (16384)        +0.2 (14368)   9        +1.4 (18432) +3.2 (16416)
constexpr int SLIM_STEPS = 8;
static int slim_rounds(int n_out) { return n_out < 2560 ? 4 : n_out < 2816 ? 5 : n_out < 3328 ? 6 : 8; }
bool gemm_slim_runs(int T, int n_in, int n_out, const void* xp, const void* w) {
  return T <= SLIM_ROWS && n_in % 32 == 0 && n_out % 64 == 0 && n_out >= 2048 && n_out <= 4096 &&
         n_in <= slim_rounds(n_out) * SLIM_STEPS * SLIM_WAVES * 32 && (((uintptr_t)xp | (uintptr_t)w) & 15) == 0;
}
int launch_gemm_slim(const uint16_t* xp, const uint16_t* w, int T, int n_in, int n_out, float* x, const float* g,
                     uint16_t* hp, float* ssq, hipStream_t st) {
  gemm_slim_kernel<SLIM_STEPS><<<n_out / 16, SLIM_WAVES * 64, 0, st>>>(xp, w, n_in / 32, T, n_out, x, g, hp, ssq);
  return check_launch();
}

}  // namespace trj
