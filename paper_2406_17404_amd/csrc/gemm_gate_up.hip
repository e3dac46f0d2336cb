// Gate/up projection with SiLU(gate) * up in its epilogue.
#include "gemm_ring.h"

namespace trj {

// acc layout of v_mfma_f32_32x32x16: lane l, register v -> tile row 8*(v/4) + 4*(l/32) +
// v%4, tile column l%32.  Rows are output features, columns are token rows.

// ---- epilogue: act = silu(gate) * up, written bf16 in the tiled activation layout.
// A TRJ_PACK_GATE_UP tile holds gate rows 16*tile.. in tile rows 0..15 and the matching
// up rows in tile rows 16..31, i.e. register v pairs with register v + 8.
struct EpiGateUp {
  static constexpr bool kScaled = true;
  RowScale rs;
  uint16_t* act;  // tiled, tp rows, d_ffn columns
  int tp;
  __device__ void operator()(const f32x16& acc, int tile, int ttile, int lane, int) const {
    int t = ttile * 32 + (lane & 31);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      float r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float gate = acc[4 * g + i], up = acc[8 + 4 * g + i];
        r[i] = gate / (1.0f + __expf(-gate)) * up;
      }
      int f = 16 * tile + 8 * g + 4 * (lane >> 5);
      u32x2 pk = {pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
      *reinterpret_cast<u32x2*>(act + a_off(t, f, tp)) = pk;
    }
  }
};

int launch_gemm_gate_up(const uint16_t* xp, const uint16_t* w, int tp, int n_in, int d_ffn,
                        const RowScale& rs, uint16_t* act, hipStream_t st) {
  EpiGateUp e{rs, act, tp};
  return launch_gemm(xp, w, tp, n_in, 2 * d_ffn, 1, e, st);
}

}  // namespace trj
