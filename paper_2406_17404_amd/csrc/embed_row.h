// Token rows' embedding, as a piece of a launch that does other things too: in bf16 mode
// with the first projection's input, exactly what reduce_norm_kernel writes for a row that
// comes from the embedding table (same column parts, same order of every sum).
#pragma once
#include "common.h"
#include "kernels.h"

namespace trj {

// rows of a workgroup of PREP_THREADS: in bf16 as many as fit side by side (d = 4096: two)
__host__ __device__ inline int embed_rows(const EmbedRow& e) {
  return e.hp ? PREP_THREADS / (e.parts * e.part_threads) : 1;
}
inline int embed_blocks(const EmbedRow& e) {
  return e.x ? ((e.hp ? e.tp : e.T) + embed_rows(e) - 1) / embed_rows(e) : 0;
}

// workgroup `block` of PREP_THREADS; a thread owns 8 columns (bf16: at most 8192 of them)
__device__ inline void embed_row(const EmbedRow& e, int block) {
  if (!e.hp) {  // fp32: one row alone
    const int tid = threadIdx.x, t = block;
    int id = e.tok[t];
    id = id < 0 ? 0 : (id >= e.vocab ? e.vocab - 1 : id);
    const float* row = static_cast<const float*>(e.embed) + (size_t)id * e.d;
    for (int c = tid; c < e.d; c += PREP_THREADS) e.x[(size_t)t * e.d + c] = row[c];
    return;
  }
  __shared__ float wsum[PREP_THREADS / WAVE];
  const int row_threads = e.parts * e.part_threads, sub = threadIdx.x / row_threads;
  const int tid = threadIdx.x - sub * row_threads;  // within the row; parts are whole wavefronts
  const int t = block * embed_rows(e) + sub;
  const bool mine = sub < embed_rows(e) && t < e.tp, live = mine && tid < (e.d >> 3);
  float ss = 0.f;
  if (t >= e.T) {
    const u32x4 z = {0, 0, 0, 0};
    if (live) *reinterpret_cast<u32x4*>(e.hp + a_off(t, tid * 8, e.tp)) = z;
  } else if (live) {
    int id = e.tok[t];
    id = id < 0 ? 0 : (id >= e.vocab ? e.vocab - 1 : id);
    const u32x4 v = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(e.embed) + (size_t)id * e.d + tid * 8);
    const f32x4 g0 = *reinterpret_cast<const f32x4*>(e.g + tid * 8);
    const f32x4 g1 = *reinterpret_cast<const f32x4*>(e.g + tid * 8 + 4);
    const f32x4 a = {__builtin_bit_cast(float, v[0] << 16), __builtin_bit_cast(float, v[0] & 0xffff0000u),
                     __builtin_bit_cast(float, v[1] << 16), __builtin_bit_cast(float, v[1] & 0xffff0000u)};
    const f32x4 b = {__builtin_bit_cast(float, v[2] << 16), __builtin_bit_cast(float, v[2] & 0xffff0000u),
                     __builtin_bit_cast(float, v[3] << 16), __builtin_bit_cast(float, v[3] & 0xffff0000u)};
    float* xr = e.x + (size_t)t * e.d + tid * 8;
    *reinterpret_cast<f32x4*>(xr) = a;
    *reinterpret_cast<f32x4*>(xr + 4) = b;
    const u32x4 pk = {pack2bf(a[0] * g0[0], a[1] * g0[1]), pack2bf(a[2] * g0[2], a[3] * g0[3]),
                      pack2bf(b[0] * g1[0], b[1] * g1[1]), pack2bf(b[2] * g1[2], b[3] * g1[3])};
    *reinterpret_cast<u32x4*>(e.hp + a_off(t, tid * 8, e.tp)) = pk;
#pragma unroll
    for (int i = 0; i < 4; ++i) ss += a[i] * a[i] + b[i] * b[i];
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (mine && tid < e.parts) {
    const int w0 = (sub * row_threads + tid * e.part_threads) / WAVE;
    float tot = 0.f;
    for (int w = 0; w < e.part_threads / WAVE; ++w) tot += wsum[w0 + w];
    e.ssq[(size_t)tid * e.tp + t] = tot;
  }
}

}  // namespace trj
