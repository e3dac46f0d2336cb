// The bf16 projection of many rows with two groups of wavefronts that take turns: while one
// multiplies a phase out of its registers, the other reads its next phase from LDS and requests
// later ones.  Same operands, tiles and epilogues as gemm_ring_kernel (gemm_ring.h).
//
// What bounds it: a 128 x 128 tile per compute unit takes as long as its operands take to arrive
// (8 KiB per k-step at 60-65 GB/s, of which the products are a third).  With all wavefronts in
// step the requests come in bursts behind the meetings and nothing covers the time of reading
// operands from LDS.  Taking turns, a SIMD always has a wavefront with everything in registers, and
// with one workgroup on the compute unit the ring may take all of its LDS.  1024 rows, us,
// gemm_ring_kernel -> this: 4096 x 11008 99 -> 91 (in the packed step, which had split it in two
// with 20 us for the sum behind it: 92 + 20 -> 97 + 11), 4096 x 4096 45 -> 42.5 in the step.  The
// 256 x 256 tile, which the products' power limit binds, did not gain in the step (12288 x 4096
// 111.9, 110.6), nor did 128 x 256 (22016 x 4096 175, 176).
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace trj {

// Workgroup = 2 x 2 wavefronts x 2 k-parts, wavefront tile = 2 x 2 tiles of 32 x 32, phases of PH
// k-steps in a ring of NB buffers; n_in / 16 is a multiple of PH.  Wavefronts 0..3 are the first
// group and take the even phases, 4..7 (one behind the other on each SIMD) the odd ones.  Time goes
// in steps with a meeting of all behind each: phase b is read in step b and multiplied in step b+1.
//   Requests: whoever reads in step t requests phase t+NB-1 (its buffer was last read in step t-1),
//   which with NB odd is one of its own; at the end of the step in which a group multiplies, t, its
//   pieces of phase t+1 are there and those of t+3 may not be.
// Phases behind the last are requested from the last one again, into buffers nobody reads any more.
template <int PH, int NB, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_pair_kernel(const uint16_t* xp, const uint16_t* w, int n_in, int n_out, int tp,
    int phases_per_split, Epi epi) {
  const GemmArgs a{xp, w, n_in, n_out, tp, phases_per_split};
  constexpr int RT = 2, CT = 2, WT = 2, MT = 2, WR = RT * WT, XC = CT * MT;
  constexpr int XP = PH * XC, P = XP + PH * WR, PL = P / 4, BUF = P * 1024;  // PL: of one wavefront
  static_assert(NB == 5 && XP % 4 == 0 && P % 4 == 0 && NB * BUF <= 160 * 1024 && 16 * 4096 <= NB * BUF, "shape");
  extern __shared__ __align__(16) uint8_t smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wv >> 2;
  const int rt = wv & 1, ct = (wv >> 1) & 1;
  const int ksteps = a.n_in >> 4, n = a.phases_per_split;  // no k-splits; >= 1
  const int ttiles = a.tp >> 5, ntiles = a.n_out >> 5, tblocks = (ttiles + XC - 1) / XC;
  int tb = 0, rg = blockIdx.x;  // as in gemm_ring_kernel: the same weight rows on one die
  if (tblocks > 1) {
    const int slot = blockIdx.x >> 3;
    tb = slot % tblocks;
    rg = (slot / tblocks) * 8 + (blockIdx.x & 7);
  }
  if (rg * WR >= ntiles) return;  // uniform
  const int tile0 = rg * WR, tt0 = tb * XC;
  float rsf[Epi::kScaled ? MT : 1], ssq[Epi::kScaled ? MT : 1][RS_MAX_PARTS];
  if constexpr (Epi::kScaled) row_scale_load<MT>(epi.rs, tt0 + ct * MT, ttiles, lane, ssq);

  const uint8_t* xs = reinterpret_cast<const uint8_t*>(a.xp) + (size_t)tt0 * 1024;
  const uint8_t* ws = reinterpret_cast<const uint8_t*>(a.w) + (size_t)tile0 * ksteps * 1024;
  const int rw = wv & 3;  // this wavefront's pieces of its group's phases: rw, rw + 4, ..
  uint32_t voff[PL];
#pragma unroll
  for (int j = 0; j < PL; ++j) {  // tiles past the matrix' end are read from the last one instead
    const int p = j * 4 + rw, pw = p - XP;
    voff[j] = p < XP ? (uint32_t)(p / XC * ttiles + min(p % XC, ttiles - 1 - tt0)) * 1024 + lane * 16
                     : (uint32_t)(min(pw / PH, ntiles - 1 - tile0) * ksteps + pw % PH) * 1024 + lane * 16;
  }
  auto request = [&](int ph) {
    const int q = min(ph, n - 1);
    const uint8_t* x = xs + (size_t)q * PH * ttiles * 1024;
    const uint8_t* w = ws + (size_t)q * PH * 1024;
    const uint32_t b = lds0 + (uint32_t)(ph % NB) * BUF + rw * 1024;
#pragma unroll
    for (int j = 0; j < PL; ++j)
      load_to_lds<false>(j * 4 < XP ? x : w, voff[j], __builtin_amdgcn_readfirstlane(b + j * 4096));
  };

  f32x16 acc[WT][MT];
#pragma unroll
  for (int r = 0; r < WT; ++r)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[r][m][v] = 0.f;
  u32x4 wa[PH][WT], xb[PH][MT];
  auto read = [&](int buffer) {
    const u32x4* lx = reinterpret_cast<const u32x4*>(smem + buffer * BUF) + lane;
#pragma unroll
    for (int q = 0; q < PH; ++q) {
#pragma unroll
      for (int r = 0; r < WT; ++r) wa[q][r] = lx[(XP + (rt * WT + r) * PH + q) * 64];
#pragma unroll
      for (int m = 0; m < MT; ++m) xb[q][m] = lx[(q * XC + ct * MT + m) * 64];
    }
  };
  auto multiply = [&]() {  // ahead of the other wavefront of its SIMD, whose turn it is to read
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < PH; ++q)
#pragma unroll
      for (int r = 0; r < WT; ++r)
#pragma unroll
        for (int m = 0; m < MT; ++m)
          acc[r][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wa[q][r]),
                                                              __builtin_bit_cast(bf16x8, xb[q][m]), acc[r][m], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
  };
  // every wavefront comes to the same number of meetings: the second group starts with one while
  // the first reads, and ends without one behind its last products
  constexpr int ALL = 63;  // more than are ever on the way: waits for none of the loads
  const int turns = (n + 1) / 2;
  for (int p = grp; p < NB - 1; p += 2) request(p);
  wait_and_meet<0>();
  if (grp == 1) wait_and_meet<ALL>();
  int buffer = grp;
  for (int i = 0; i < turns; ++i) {
    const int p = 2 * i + grp;
    read(buffer);
    request(p + NB - 1);
    buffer = buffer + 2 >= NB ? buffer + 2 - NB : buffer + 2;
    __builtin_amdgcn_sched_barrier(0);
    wait_and_meet<ALL>();
    __builtin_amdgcn_sched_barrier(0);
    if (p >= n) {  // the second group's turn behind an odd number of phases adds nothing
#pragma unroll
      for (int q = 0; q < PH; ++q) {
#pragma unroll
        for (int r = 0; r < WT; ++r) wa[q][r] = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < MT; ++m) xb[q][m] = u32x4{0, 0, 0, 0};
      }
    }
    multiply();
    if (grp == 0 || i + 1 < turns) wait_and_meet<PL>();
  }
  wait_and_meet<0>();  // nothing may land in what is used for the sums, or behind the end
  if constexpr (Epi::kScaled) {
#pragma unroll
    for (int m = 0; m < MT; ++m) rsf[m] = row_scale_factor(epi.rs, ssq[m]);
    if (epi.rs.ssq && epi.rs.parts > RS_MAX_PARTS) {  // uniform
      float* factor = reinterpret_cast<float*>(smem) + 16 * 1024;  // behind what the sums below use
      row_factors<XC * 32>(epi.rs, tt0 * 32, factor);
#pragma unroll
      for (int m = 0; m < MT; ++m) rsf[m] = factor[(ct * MT + m) * 32 + (lane & 31)];
    }
  }
  // an epilogue that returns a sum per token row (gemm_residual.hip)
  constexpr bool SUMS = !std::is_void_v<decltype(epi(acc[0][0], 0, 0, 0, 0))>;
  float* sums = reinterpret_cast<float*>(smem) + 16 * 1024;  // behind what the next sums use
  // tile i of both k-parts is added by group i % 2
  float* red = reinterpret_cast<float*>(smem) + (size_t)(wv & 3) * WT * MT * 1024 + lane;
#pragma unroll
  for (int i = 0; i < WT * MT; ++i)
    if (grp != i % 2)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[i * 1024 + v * 64] = acc[i / MT][i % MT][v];
  wait_and_meet<0>();
#pragma unroll
  for (int i = 0; i < WT * MT; ++i)
    if (grp == i % 2)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i / MT][i % MT][v] += red[i * 1024 + v * 64];
#pragma unroll
  for (int r = 0; r < WT; ++r) {
    const int tile = tile0 + rt * WT + r;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int tt = tt0 + ct * MT + m;
      if (tile >= ntiles || tt >= ttiles || grp != (r * MT + m) % 2) continue;  // uniform
      if constexpr (Epi::kScaled) epi(scaled(acc[r][m], rsf[m]), tile, tt, lane, 0);
      else if constexpr (SUMS) {
        const float ss = epi(acc[r][m], tile, tt, lane, 0);
        if (lane < 32) sums[(rt * WT + r) * XC * 32 + (ct * MT + m) * 32 + lane] = ss;
      } else epi(acc[r][m], tile, tt, lane, 0);
    }
  }
  if constexpr (SUMS) {  // of the workgroup's features, in order
    __syncthreads();
    const int t = tt0 * 32 + tid;
    if (tid < XC * 32 && t < a.tp) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < WR; ++r) s += sums[r * XC * 32 + tid];
      epi.ssq[(size_t)rg * a.tp + t] = s;
    }
  }
}

constexpr int PAIR_PHASE = 4, PAIR_BUFFERS = 5;
template <class Epi>
static void launch_pair(const uint16_t* xp, const uint16_t* w, int tp, int n_in, int n_out, const Epi& epi,
                        hipStream_t st) {
  const int rgs = (n_out / 32 + 3) / 4, tblocks = (tp / 32 + 3) / 4;
  auto kern = gemm_pair_kernel<PAIR_PHASE, PAIR_BUFFERS, Epi>;
  constexpr size_t lds = (size_t)PAIR_BUFFERS * PAIR_PHASE * 8 * 1024;
  static DeviceOnce once;  // per instantiation
  allow_lds(once, kern, lds);
  kern<<<tblocks == 1 ? rgs : (rgs + 7) / 8 * 8 * tblocks, 512, lds, st>>>(xp, w, n_in, n_out, tp,
                                                                             (n_in >> 4) / PAIR_PHASE, epi);
}

}  // namespace trj
