// The bf16 projection kernel, shared by the files that instantiate it with their epilogue:
//   Y^T[n_out, T] = W[n_out, n_in] * X^T[n_in, T],  fp32 accumulation on the MFMA units.
// W is stored in 32x16 tiles and X in 32-row tiles per k-step that are, 1 KiB each, exactly
// one v_mfma_f32_32x32x16_bf16 operand (16 bytes per lane).
//
// Both operands go from memory to LDS without passing through registers (global_load_lds,
// 1 KiB per wavefront instruction) into a ring of NB phase buffers of PH k-steps each, and
// from there into MFMA operand registers.  What bounds the kernel and why it looks so:
//  - Up to 128 token rows it is the stream of W from HBM plus the activations that every
//    workgroup reads again from L2.  A compute unit returns loads in order, so the L2 hits
//    queue behind the HBM misses and both together arrive at 50-65 GB/s per compute unit
//    (a probe with separate wavefronts for the two streams; L2 hits alone reach 120).  What
//    helps is to keep that queue full at every moment: register staging, with the loads of a
//    phase waited for one phase later, drained it at every phase end and took about 3 us a
//    phase at 65..128 rows whatever the phase held.  The ring keeps NB - 1 phases in flight
//    and costs no registers.  W carries the streaming hint (5.9 -> 7.2 TB/s in a bare read).
//    us per launch inside the step, register staging -> ring: 128 rows, 12288 x 4096: 51.3 ->
//    34.1, 22016 x 4096: 53.6 -> 48.6; 96 rows, 6144 x 4096: 53.9 -> 24.1, 28672 x 4096: 46.8
//    -> 44.7, 128256 x 4096: 218 -> 178; 64 rows, 12288 x 4096: 27.5 -> 26.0, 22016 x 4096:
//    34.8 -> 32.1; 32 rows: 30.3 -> 29.6 (6.1 TB/s of weights).
//  - Packed batches (from 256 padded rows) are bound by the MFMA units and the LDS together:
//    a 256 x 256 tile of 8 wavefronts reads 48 KiB and writes 16 KiB of LDS per k-step, as
//    many cycles (128 B each) as its MFMAs take.  Operands of a k-step are requested before
//    the MFMAs of the previous one, across phase boundaries too, and interleaved with them.
//    1024 rows, weights straight to registers -> both through the ring: 12288 x 4096 137 -> 117
//    us, 22016 x 4096 218 -> 176, 32000 x 4096 277 -> 250 (1.07 PFLOP/s).
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace trj {

struct GemmArgs {
  const uint16_t* xp;  // activations, tiled (a_off), tp rows
  const uint16_t* w;   // weights, tiled (w_off)
  int n_in, n_out, tp;
  int phases_per_split;
};

// this lane's token row of each of MT token tiles: the partial sums of squares (all parts
// asked for at once, clamped index; parts beyond the last are ignored when they are summed)
template <int MT>
__device__ inline void row_scale_load(const RowScale& rs, int ttile0, int ttiles, int lane,
                                      float (&ssq)[MT][RS_MAX_PARTS]) {
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int p = 0; p < RS_MAX_PARTS; ++p) ssq[m][p] = 0.f;
  if (!rs.ssq || rs.fine || rs.parts > RS_MAX_PARTS) return;  // uniform
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int t = min(ttile0 + m, ttiles - 1) * 32 + (lane & 31);
#pragma unroll
    for (int p = 0; p < RS_MAX_PARTS; ++p)  // no arithmetic on the loaded value here: it would wait for it
      ssq[m][p] = rs.ssq[(size_t)min(p, rs.parts - 1) * rs.tp + t];
  }
}
__device__ inline float row_scale_factor(const RowScale& rs, const float (&ssq)[RS_MAX_PARTS]) {
  if (!rs.ssq || rs.fine || rs.parts > RS_MAX_PARTS) return 1.0f;
  float s = 0.f;
#pragma unroll
  for (int p = 0; p < RS_MAX_PARTS; ++p) s += p < rs.parts ? ssq[p] : 0.f;  // fixed order
  return 1.0f / sqrtf(s * rs.inv_d + rs.eps);
}
// Many rows with sums in more parts (gemm_residual.hip): a thread per token row of the workgroup adds its
// parts in order and hands the factor on through `factor` (LDS that nothing uses any more, once all
// wavefronts are here).  Behind the main loop; 32 parts of 256 rows are 32 KiB per workgroup.
template <int ROWS>
__device__ inline void row_factors(const RowScale& rs, int row0, float* factor) {
  __syncthreads();
  if ((int)threadIdx.x < ROWS) {
    const float* p = rs.ssq + min(row0 + (int)threadIdx.x, rs.tp - 1);
    float s = 0.f;
    for (int k0 = 0; k0 < rs.parts; k0 += 16) {
      float v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = p[(size_t)min(k0 + k, rs.parts - 1) * rs.tp];
#pragma unroll
      for (int k = 0; k < 16; ++k) s += k0 + k < rs.parts ? v[k] : 0.f;
    }
    factor[threadIdx.x] = 1.0f / sqrtf(s * rs.inv_d + rs.eps);
  }
  __syncthreads();
}
// a scaled copy for the epilogue (the accumulators themselves stay where they are)
__device__ inline f32x16 scaled(const f32x16& acc, float f) {
  f32x16 r;
#pragma unroll
  for (int v = 0; v < 16; ++v) r[v] = acc[v] * f;
  return r;
}

// all but the newest N loads of this wavefront have landed and its LDS reads are done; then
// the workgroup meets.  (Loads the compiler issues by itself only make the wait stricter.)
template <int N>
__device__ __forceinline__ void wait_and_meet() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Workgroup = RT row groups x CT token groups x KW k-parts of wavefronts, wavefront tile =
// WT x MT tiles of 32 x 32.  A phase is PH k-steps: XP + WP pieces of 1 KiB, dealt to the
// wavefronts round robin.  Wavefront (.., kw) multiplies k-steps kw*WS .. of every phase.
//
// Ring: phases ph .. ph+NB-1 are in their buffers or on the way.  At the end of phase ph every
// wavefront waits until its own pieces of phase ph+1 have landed (NB-2 younger phases stay in
// flight) and its own operand reads of phase ph are done; behind the barrier the buffer of
// phase ph is therefore free for phase ph+NB and phase ph+1 is complete for everybody.
//
// If n_in/16 is not a multiple of PH the last phase has k-steps beyond it: they are loaded
// from the last real one and both operands cleared (0 * 0, so that no infinity or NaN of the
// repeated step gets in), in the last phase and in front of the MFMA only: a mask right
// behind the LDS read makes the wavefront wait for the read there (22016 x 4096 at 128 rows
// 56.0 against 48.6 us).
//
// ALIGNED: xp and w start at multiples of 16 bytes, as loads to LDS need.  Else the pieces of a
// phase wait in registers from its request to the end of the next phase, when they are written
// to their buffer in front of the barrier: one phase in flight besides the two in LDS, so
// phases are long where they are small (8 k-steps up to 32 rows: 22016 x 4096 41 against 48 us;
// beyond, 4 leave room for a second workgroup on the compute unit: 128 rows 64 against 88).
// 22016 x 4096 with weights one element off: 64 rows 45 us (33 aligned), 1024 rows 264 (181);
// copied to LDS at once and waited for, in one shape for all rows: 64 and 750.
//
// What the first loads need are plain arguments in front: those come in scalar registers when a
// wavefront starts (build.py's kernarg preload; members of a struct do not) and save it a read of
// memory that nothing has in a cache yet.  Steps of two layers, 20 launches, us: 777 x 5 242.2 -> 239.4,
// 1024 x 64 283.8 -> 281.1, 4096 x 128 390.8 -> 387.5.
template <int RT, int CT, int KW, int WT, int MT, int PH, int NB, bool NT, bool ALIGNED, class Epi>
__global__ __launch_bounds__(RT* CT* KW * 64, 2) void gemm_ring_kernel(const uint16_t* xp, const uint16_t* w, int n_in,
                                                                       int n_out, int tp, int phases_per_split,
                                                                       Epi epi) {
  const GemmArgs a{xp, w, n_in, n_out, tp, phases_per_split};
  constexpr int NW = RT * CT * KW, WR = RT * WT, XC = CT * MT, WS = PH / KW;
  constexpr int XP = PH * XC, P = XP + PH * WR, PL = (P + NW - 1) / NW, REM = P % NW;
  constexpr int BUF = P * 1024;
  // wavefront tiles of at most 8 keep the accumulators in 256 registers (two per SIMD)
  static_assert(PH % KW == 0 && NB >= 2 && NB <= 4 && NB * BUF <= 160 * 1024 && WT * MT <= 8, "shape");
  extern __shared__ __align__(16) uint8_t smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform, and the compiler knows
  const int rt = wv % RT, ct = (wv / RT) % CT, kw = wv / (RT * CT);
  const int ksteps = a.n_in >> 4, nph = (ksteps + PH - 1) / PH;
  const int ph0 = blockIdx.y * a.phases_per_split;
  const int n = min(nph, ph0 + a.phases_per_split) - ph0;  // phases of this workgroup, >= 1 if ALIGNED
  const int ttiles = a.tp >> 5, ntiles = a.n_out >> 5, tblocks = (ttiles + XC - 1) / XC;
  // Workgroup ids go round-robin over the 8 dies (XCDs), each with its own L2.  With several
  // token blocks the workgroups that stream the SAME weight rows get ids that land on one die,
  // next to each other in its dispatch order, so that the rows come from HBM once.
  int tb = 0, rg = blockIdx.x;
  if (tblocks > 1) {
    const int slot = blockIdx.x >> 3;
    tb = slot % tblocks;
    rg = (slot / tblocks) * 8 + (blockIdx.x & 7);
  }
  if (rg * WR >= ntiles) return;  // padding of the row groups to a multiple of 8 (uniform)
  const int tile0 = rg * WR, tt0 = tb * XC;

  // the token rows' sums of squares: oldest loads of the wavefront, used behind the main loop
  float rsf[Epi::kScaled ? MT : 1], ssq[Epi::kScaled ? MT : 1][RS_MAX_PARTS];
  if constexpr (Epi::kScaled) row_scale_load<MT>(epi.rs, tt0 + ct * MT, ttiles, lane, ssq);

  const uint8_t* xs = reinterpret_cast<const uint8_t*>(a.xp) + ((size_t)ph0 * PH * ttiles + tt0) * 1024;
  const uint8_t* ws = reinterpret_cast<const uint8_t*>(a.w) + ((size_t)tile0 * ksteps + (size_t)ph0 * PH) * 1024;
  const size_t xstep = (size_t)PH * ttiles * 1024;
  // Few rows: every workgroup starts at another phase of its k range (spread by the golden ratio)
  // and goes round.  In step, all of them would ask the same memory channels for W (row tiles lie
  // whole multiples of 4 KiB apart), and activations that the launch before has just written would
  // miss in a die's L2 for all its workgroups at once; spread out, each fetches its share for the
  // others.  Up to 1 MiB of activations (128 x 4096), which stay in the L2 together; not with a
  // single row tile, where activations are most of what is read; and where all phases are whole.
  // In the step, us: 22016 x 4096 at 128 rows 49.0 -> 44.6, 12288 x 4096 at 128 35.3 -> 34.3, at 64
  // 25.7 -> 25.2, 128256 x 4096 at 96 180 -> 166, 32000 x 4096 at 64 47.5 -> 45.1, 4096 x 4096 at
  // 32 9.1 -> 7.8.  Left out: 4096 x 11008 at 128 rows 26.9 -> 27.3, 6144 x 4096 at 96 23.4 -> 23.9.
  // Launches that do not rotate are not back where they were without the rotation in the kernel (the
  // down projection in the step at 64 rows 19.3 -> 19.7, at 128 26.1 -> 27.0; why is not known, the wrap in
  // the loop is not the reason).
  const bool tail = ksteps % PH != 0;
  const bool spread = NT && WR > 1 && !tail && a.tp * a.n_in <= 1 << 19;
  const int rot = spread ? (int)(((blockIdx.x >> 3) * 40503u + (blockIdx.x & 7) * 8192u & 0xffffu) * n >> 16) : 0;
  xs += rot * xstep;
  ws += (size_t)rot * PH * 1024;
  // piece p of a phase: X (k-step p / XC, token tile p % XC), then W (row tile, k-step);
  // tiles past the matrix' end and k-steps past kmax are read from the last one instead
  auto piece = [&](int p, int kmax) -> uint32_t {
    if (p < XP) return (uint32_t)(min(p / XC, kmax) * ttiles + min(p % XC, ttiles - 1 - tt0)) * 1024 + lane * 16;
    const int pw = p - XP;
    return (uint32_t)(min(pw / PH, ntiles - 1 - tile0) * ksteps + min(pw % PH, kmax)) * 1024 + lane * 16;
  };
  uint32_t voff[PL];
#pragma unroll
  for (int j = 0; j < PL; ++j) voff[j] = piece(min(j * NW + wv, P - 1), PH - 1);
  int iph = ph0;                         // requests made, from ph0 on
  uint32_t ibuf = lds0 + wv * 1024;      // this wavefront's first piece in its buffer
  u32x4 held[ALIGNED ? 1 : PL];          // pieces of the youngest phase, and where they belong
  uint32_t hbuf = 0;
  bool holds = false;
  auto store_held = [&]() {
    if constexpr (!ALIGNED) {
      if (!holds) return;  // uniform
#pragma unroll
      for (int j = 0; j < PL; ++j)
        if (REM == 0 || j < PL - 1 || j * NW + wv < P)
          *reinterpret_cast<u32x4*>(smem + (hbuf - lds0) + j * NW * 1024 + lane * 16) = held[j];
      holds = false;
    }
  };
  auto request = [&]() {
    if (iph == nph - 1 && tail) {
#pragma unroll
      for (int j = 0; j < PL; ++j) voff[j] = piece(min(j * NW + wv, P - 1), ksteps - 1 - iph * PH);
    }
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      const int p = j * NW + wv;
      if (REM != 0 && j == PL - 1 && p >= P) break;
      if constexpr (!ALIGNED) {
        held[j] = *reinterpret_cast<const u32x4*>((p < XP ? xs : ws) + voff[j]);
        continue;
      }
      if ((j + 1) * NW <= XP || (j * NW < XP && p < XP)) load_to_lds<false>(xs, voff[j], ibuf + j * NW * 1024);
      else load_to_lds<NT>(ws, voff[j], ibuf + j * NW * 1024);
    }
    hbuf = ibuf;
    holds = true;
    xs += xstep;
    ws += PH * 1024;
    ++iph;
    if (NT && iph == ph0 + n - rot) {  // round
      xs -= n * xstep;
      ws -= (size_t)n * PH * 1024;
    }
    ibuf = ibuf + BUF >= lds0 + NB * BUF ? ibuf + BUF - NB * BUF : ibuf + BUF;
  };
  auto wait_younger = [&](auto k_c) {  // everything but the youngest K phases has landed
    constexpr int K = decltype(k_c)::value;
    store_held();
    if (REM == 0 || wv < REM) wait_and_meet<K * PL>();
    else wait_and_meet<K * (PL - 1)>();
  };

  f32x16 acc[WT][MT];
#pragma unroll
  for (int r = 0; r < WT; ++r)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[r][m][v] = 0.f;
  u32x4 wa[2][WT], xb[2][MT];  // operands of the current and the next k-step
  uint32_t rbuf = 0;
  auto read = [&](int q, int s) {
    const u32x4* lx = reinterpret_cast<const u32x4*>(smem + rbuf) + lane;
    const int ksl = kw * WS + q;
#pragma unroll
    for (int r = 0; r < WT; ++r) wa[s][r] = lx[(XP + (rt * WT + r) * PH + ksl) * 64];
#pragma unroll
    for (int m = 0; m < MT; ++m) xb[s][m] = lx[(ksl * XC + ct * MT + m) * 64];
  };
  auto multiply = [&](int s) {
#pragma unroll
    for (int r = 0; r < WT; ++r)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        acc[r][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wa[s][r]),
                                                            __builtin_bit_cast(bf16x8, xb[s][m]), acc[r][m], 0, 0, 0);
    // alternate the MFMAs with the LDS reads of the next k-step (without this the compiler
    // bunches the reads in front of their use: 12288 x 4096 at 1024 rows 96.6 against 92 us)
#pragma unroll
    for (int i = 0; i < WT + MT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if (WT * MT > WT + MT) __builtin_amdgcn_sched_group_barrier(0x008, WT * MT - WT - MT, 0);
  };
  auto clear_beyond = [&](int q) {  // last phase: operands of k-step q are zero if it is beyond n_in
    const uint32_t keep = (ph0 + n - 1) * PH + kw * WS + q < ksteps ? 0xffffffffu : 0u;
#pragma unroll
    for (int r = 0; r < WT; ++r) wa[q & 1][r] &= keep;
#pragma unroll
    for (int m = 0; m < MT; ++m) xb[q & 1][m] &= keep;
  };
  auto phase = [&](auto k_c, auto request_c, auto last_c) {
    constexpr bool REQUEST = decltype(request_c)::value, LAST = decltype(last_c)::value;
#pragma unroll
    for (int q = 0; q < WS - 1; ++q) {
      read(q + 1, (q + 1) & 1);
      if constexpr (LAST) clear_beyond(q);
      multiply(q & 1);
    }
    if constexpr (!LAST) {
      wait_younger(k_c);
      if constexpr (REQUEST) request();
      rbuf = rbuf + BUF == NB * BUF ? 0 : rbuf + BUF;
      read(0, WS & 1);
    } else {
      clear_beyond(WS - 1);
    }
    multiply((WS - 1) & 1);
    if constexpr ((WS & 1) && !LAST) {  // the next phase starts from operand set 0
#pragma unroll
      for (int r = 0; r < WT; ++r) wa[0][r] = wa[1][r];
#pragma unroll
      for (int m = 0; m < MT; ++m) xb[0][m] = xb[1][m];
    }
  };
  constexpr std::integral_constant<int, 0> k0{};
  constexpr std::integral_constant<int, 1> k1{};
  constexpr std::integral_constant<int, 2> k2{};
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if (ALIGNED || n > 0)
    for (int p = 0; p < NB && p < n; ++p) {
      request();
      store_held();
    }
  // sums in many parts: each wavefront takes some of the (up to eight) rows and hands their factors on
  // through LDS
  constexpr bool FINE = Epi::kScaled && NT && MT == 1;
  constexpr int FR = (8 + NW - 1) / NW;
  f32x4 fine[FINE ? FR : 1];
  if constexpr (FINE) {
    if (epi.rs.fine) {  // uniform
#pragma unroll
      for (int j = 0; j < FR; ++j)
        if (j * NW + wv < epi.rs.fine)
          fine[j] = *reinterpret_cast<const f32x4*>(epi.rs.ssq + (size_t)(j * NW + wv) * epi.rs.parts + min(lane * 4, epi.rs.parts - 4));
    }
  }
  if (ALIGNED || n > 0) {
    if (n >= NB) wait_younger(std::integral_constant<int, NB - 1>{});
    else if (NB > 3 && n == 3) wait_younger(k2);
    else if (NB > 2 && n == 2) wait_younger(k1);
    else wait_younger(k0);
    read(0, 0);
    int ph = 0;
    for (; ph + NB < n; ++ph) phase(std::integral_constant<int, NB - 2>{}, yes, no);
    // the last phases have nothing left to request and ever fewer phases behind them
    if constexpr (NB > 3) {
      if (n - 1 - ph > 2) { phase(k2, no, no); ++ph; }
    }
    if constexpr (NB > 2) {
      if (n - 1 - ph > 1) { phase(k1, no, no); ++ph; }
    }
    if (n - 1 - ph > 0) phase(k0, no, no);
    phase(k0, no, yes);
  }
  // only now: the compiler, which does not count the ring's loads, waits for all of them here
  if constexpr (Epi::kScaled) {
#pragma unroll
    for (int m = 0; m < MT; ++m) rsf[m] = row_scale_factor(epi.rs, ssq[m]);
  }
  if constexpr (FINE) {
    if (epi.rs.fine) {  // uniform
      float* factor = reinterpret_cast<float*>(smem);  // the ring is done with once all are here
      wait_and_meet<0>();
#pragma unroll
      for (int j = 0; j < FR; ++j) {
        if (j * NW + wv >= epi.rs.fine) break;
        float s = lane * 4 < epi.rs.parts ? (fine[j][0] + fine[j][1]) + (fine[j][2] + fine[j][3]) : 0.f;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) factor[j * NW + wv] = 1.0f / sqrtf(s * epi.rs.inv_d + epi.rs.eps);
      }
      __syncthreads();
      rsf[0] = factor[min(lane & 31, epi.rs.fine - 1)];
    }
  }

  if constexpr (Epi::kScaled && !NT) {
    if (epi.rs.ssq && epi.rs.parts > RS_MAX_PARTS) {  // uniform
      float* factor = reinterpret_cast<float*>(smem);
      row_factors<XC * 32>(epi.rs, tt0 * 32, factor);
#pragma unroll
      for (int m = 0; m < MT; ++m) rsf[m] = factor[(ct * MT + m) * 32 + (lane & 31)];
    }
  }

  // The k-parts of a tile are added through LDS, tile i by k-part i % KW (own part first, then
  // the others in ascending order: deterministic), so that sums and epilogue are spread over
  // all wavefronts.
  if constexpr (KW > 1) {
    float* red = reinterpret_cast<float*>(smem) + (size_t)(ct * RT + rt) * WT * MT * (KW - 1) * 1024 + lane;
    wait_and_meet<0>();
#pragma unroll
    for (int i = 0; i < WT * MT; ++i)
      if (kw != i % KW) {
        float* dst = red + (i * (KW - 1) + (kw < i % KW ? kw : kw - 1)) * 1024;
#pragma unroll
        for (int v = 0; v < 16; ++v) dst[v * 64] = acc[i / MT][i % MT][v];
      }
    wait_and_meet<0>();
#pragma unroll
    for (int i = 0; i < WT * MT; ++i)
      if (kw == i % KW) {
#pragma unroll
        for (int q = 0; q < KW - 1; ++q)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i / MT][i % MT][v] += red[(i * (KW - 1) + q) * 1024 + v * 64];
      }
  }
#pragma unroll
  for (int r = 0; r < WT; ++r) {
    const int tile = tile0 + rt * WT + r;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int tt = tt0 + ct * MT + m;
      if (tile >= ntiles || tt >= ttiles || kw != (r * MT + m) % KW) continue;  // uniform
      if constexpr (Epi::kScaled) epi(scaled(acc[r][m], rsf[m]), tile, tt, lane, blockIdx.y);
      else epi(acc[r][m], tile, tt, lane, blockIdx.y);
    }
  }
}

}  // namespace trj
#include "gemm_pair.h"
namespace trj {

// ---- launch plan (gemm_bf16.hip)
enum GemmShape {  // {row groups, token groups, k-parts} of wavefronts x {row, token} tiles per wavefront
  GS_4x1, GS_2x4, GS_2x2, GS_4x2, GS_1x4, GS_3x2,  // RT row tiles x KW k-parts, all token tiles of the pass
  GS_16,                                            // 8 row groups x 2 row tiles
  GS_MANY_2, GS_MANY_4x4, GS_MANY_4x8, GS_MANY_8x8  // several token blocks: row x token tiles per workgroup
};
struct GemmPlan {
  GemmShape shape;
  int mt;               // token tiles of a pass (small shapes), of a workgroup (many rows)
  int rows, kw, wt;     // row tiles per workgroup, k-parts per workgroup, row tiles per wavefront
  int split_k;
  bool many;
  bool pair;            // gemm_pair_kernel
};
GemmPlan plan_gemm(int tp, int n_in, int n_out, int split_k);
// k-steps per phase; with it the number of phases and the k-splits a request really gets
constexpr int gemm_phase(GemmShape s) {
  return s == GS_2x4 || s == GS_1x4 || s == GS_3x2 || s == GS_MANY_2 ? 8 : (s == GS_16 || s >= GS_MANY_4x4 ? 2 : 4);
}

template <int RT, int CT, int KW, int WT, int MT, int PH, int NB, bool NT, bool ALIGNED = true, class Epi>
static void launch_ring_t(const uint16_t* xp, const uint16_t* w, int tp, int n_in, int n_out, int split_k,
                          const Epi& epi, hipStream_t st) {
  constexpr int WR = RT * WT, XC = CT * MT;
  const int nph = ((n_in >> 4) + PH - 1) / PH, pps = (nph + split_k - 1) / split_k;
  const int rgs = (n_out / 32 + WR - 1) / WR, tblocks = (tp / 32 + XC - 1) / XC;
  // (the unaligned form stands in for a shape with more phases: its last splits may be empty)
  dim3 grid(tblocks == 1 ? rgs : (rgs + 7) / 8 * 8 * tblocks, ALIGNED ? (nph + pps - 1) / pps : split_k);
  constexpr size_t lds_x = (size_t)NB * PH * (XC + WR) * 1024, lds_r = (size_t)(KW - 1) * CT * WR * MT * 4096;
  constexpr size_t lds = lds_x > lds_r ? lds_x : lds_r;
  static_assert(lds <= 160 * 1024, "LDS");
  auto kern = gemm_ring_kernel<RT, CT, KW, WT, MT, PH, NB, NT, ALIGNED, Epi>;
  static DeviceOnce once;  // per instantiation
  allow_lds(once, kern, 160 * 1024);
  kern<<<grid, RT * CT * KW * 64, lds, st>>>(xp, w, n_in, n_out, tp, pps, epi);
}
template <int M, class Epi>
static void launch_ring_few(const GemmPlan& g, const uint16_t* xp, const uint16_t* w, int tp, int n_in, int n_out,
                            const Epi& epi, hipStream_t st) {
#define TRJ_RING(S, RT, KW, WT, NB) \
  launch_ring_t<RT, 1, KW, WT, M, gemm_phase(S), NB, true>(xp, w, tp, n_in, n_out, g.split_k, epi, st)
  switch (g.shape) {  // ring depths: what fits 160 KiB, at most 4 phases
    case GS_4x1: TRJ_RING(GS_4x1, 4, 1, 1, 4); break;
    case GS_2x4: TRJ_RING(GS_2x4, 2, 4, 1, (M == 4 ? 3 : 4)); break;
    case GS_2x2: TRJ_RING(GS_2x2, 2, 2, 1, 4); break;
    case GS_4x2: TRJ_RING(GS_4x2, 4, 2, 1, 4); break;
    case GS_1x4: TRJ_RING(GS_1x4, 1, 4, 1, 4); break;
    case GS_3x2: TRJ_RING(GS_3x2, 3, 2, 1, (M == 4 ? 2 : 3)); break;
    default: TRJ_RING(GS_16, 8, 1, 2, 4); break;
  }
#undef TRJ_RING
}

template <class Epi>
static int launch_gemm(const uint16_t* xp, const uint16_t* w, int tp, int n_in, int n_out, int split_k,
                       const Epi& epi, hipStream_t st) {
  if (tp < 32 || (tp & 31) || (n_in & 15) || (n_out & 31)) return TRJ_ERR_BAD_SHAPE;
  const GemmPlan g = plan_gemm(tp, n_in, n_out, split_k);
  if ((((uintptr_t)xp | (uintptr_t)w) & 15) != 0) {  // callers' odd pointers
#define TRJ_HELD(RT, CT, KW, WT, MT, PH) \
  launch_ring_t<RT, CT, KW, WT, MT, PH, 2, false, false>(xp, w, tp, n_in, n_out, g.split_k, epi, st)
    if (g.shape == GS_MANY_8x8) TRJ_HELD(2, 4, 1, 4, 2, 4);
    else if (g.shape == GS_MANY_4x8) TRJ_HELD(2, 2, 1, 2, 4, 3);
    else if (g.shape == GS_MANY_4x4) TRJ_HELD(2, 2, 1, 2, 2, 4);
    else if (g.many) TRJ_HELD(2, 1, 4, 1, 4, 8);
    else if (g.mt == 1) TRJ_HELD(2, 1, 2, 1, 1, 8);
    else if (g.mt == 2) TRJ_HELD(2, 1, 2, 1, 2, 4);
    else if (g.mt == 3) TRJ_HELD(2, 1, 2, 1, 3, 4);
    else TRJ_HELD(2, 1, 2, 1, 4, 4);
#undef TRJ_HELD
    return check_launch();
  }
  switch (g.shape) {
    case GS_MANY_2:
      launch_ring_t<2, 1, 4, 1, 4, gemm_phase(GS_MANY_2), 3, false>(xp, w, tp, n_in, n_out, g.split_k, epi, st);
      break;
    case GS_MANY_4x4:
      if (g.pair) launch_pair(xp, w, tp, n_in, n_out, epi, st);
      else launch_ring_t<2, 2, 1, 2, 2, gemm_phase(GS_MANY_4x4), 4, false>(xp, w, tp, n_in, n_out, g.split_k, epi, st);
      break;
    case GS_MANY_4x8:
      launch_ring_t<2, 2, 1, 2, 4, gemm_phase(GS_MANY_4x8), 3, false>(xp, w, tp, n_in, n_out, g.split_k, epi, st);
      break;
    case GS_MANY_8x8:
      launch_ring_t<2, 4, 1, 4, 2, gemm_phase(GS_MANY_8x8), 4, false>(xp, w, tp, n_in, n_out, g.split_k, epi, st);
      break;
    default:
      if (g.mt == 1) launch_ring_few<1>(g, xp, w, tp, n_in, n_out, epi, st);
      else if (g.mt == 2) launch_ring_few<2>(g, xp, w, tp, n_in, n_out, epi, st);
      else if (g.mt == 3) launch_ring_few<3>(g, xp, w, tp, n_in, n_out, epi, st);
      else launch_ring_few<4>(g, xp, w, tp, n_in, n_out, epi, st);
  }
  return check_launch();
}

}  // namespace trj
