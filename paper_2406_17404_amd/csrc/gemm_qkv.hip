// QKV projection with the rotary rotation and the K/V cache write in its epilogue.
#include "gemm_ring.h"

namespace trj {

// acc layout of v_mfma_f32_32x32x16: lane l, register v -> tile row 8*(v/4) + 4*(l/32) +
// v%4, tile column l%32.  Rows are output features, columns are token rows.

// ---- epilogue: rotary on q and k, q stored plain [T][H][dh], k and v into the pool.
struct EpiQKV {
  static constexpr bool kScaled = true;
  RowScale rs;
  const float2* cs;         // [.][dh/2] cos, sin: row t of the table, or row cs_row[t] if given
  const int32_t* cs_row;    // optional: the table is indexed by position, this is each row's
  const int32_t* row_slot;  // pool slot of each row, -1 = skip
  uint16_t* q;
  uint16_t* k_layer;
  uint16_t* v_layer;
  int T, n_heads, n_kv_heads, dh, s_pool;
  int tile0;  // row tile of W that the launch starts at (all of them: 0; K and V only: behind q)
  __device__ void operator()(const f32x16& acc, int launch_tile, int ttile, int lane, int) const {
    const int tile = tile0 + launch_tile;
    int t = ttile * 32 + (lane & 31);
    if (t >= T) return;
    int slot = row_slot[t];
    if (slot < 0) return;
    // row tiles: n_heads*tph of q, then n_kv_heads*tph of k, then as many of v
    const int tph = dh >> 5, q_tiles = n_heads * tph, kv_tiles = n_kv_heads * tph, half = dh >> 1;
    const int sec = tile < q_tiles ? 0 : (tile < q_tiles + kv_tiles ? 1 : 2);
    const int rel = tile - (sec == 0 ? 0 : (sec == 1 ? q_tiles : q_tiles + kv_tiles));
    const int head = rel / tph, jt = rel % tph;
    const int hh = lane >> 5;
    if (sec < 2) {
      const float2* csr = cs + (size_t)(cs_row ? cs_row[t] : t) * half;
      uint16_t* plane = k_layer + (size_t)head * s_pool * dh;
      uint16_t* qrow = q + ((size_t)t * n_heads + head) * dh;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        int c = 16 * jt + 8 * g + 4 * hh;
        float ra[4], rb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float2 sc = csr[c + i];
          float a = acc[4 * g + i], b = acc[8 + 4 * g + i];
          ra[i] = a * sc.x - b * sc.y;
          rb[i] = b * sc.x + a * sc.y;
        }
        u32x2 pa = {pack2bf(ra[0], ra[1]), pack2bf(ra[2], ra[3])};
        u32x2 pb = {pack2bf(rb[0], rb[1]), pack2bf(rb[2], rb[3])};
        if (sec == 0) {
          *reinterpret_cast<u32x2*>(qrow + c) = pa;
          *reinterpret_cast<u32x2*>(qrow + c + half) = pb;
        } else {
          *reinterpret_cast<u32x2*>(plane + k_off(slot, c, dh)) = pa;
          *reinterpret_cast<u32x2*>(plane + k_off(slot, c + half, dh)) = pb;
        }
      }
    } else {
      uint16_t* plane = v_layer + (size_t)head * s_pool * dh;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        int c = 32 * jt + 8 * (v >> 2) + 4 * hh + (v & 3);
        plane[v_off(slot, c, dh)] = f2bf(acc[v]);
      }
    }
  }
};

int launch_gemm_qkv(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_heads,
                    int n_kv_heads, int dh, int s_pool, const RowScale& rs, const float2* cs,
                    const int32_t* cs_row, const int32_t* row_slot, uint16_t* q, uint16_t* k_layer,
                    uint16_t* v_layer, hipStream_t st) {
  // without q only the K and V rows of W are read: its row tiles are stored one after the other
  const int skip = q ? 0 : n_heads * dh;
  EpiQKV e{rs, cs, cs_row, row_slot, q, k_layer, v_layer, T, n_heads, n_kv_heads, dh, s_pool, skip / 32};
  return launch_gemm(xp, w + (size_t)skip * n_in, tp, n_in, (n_heads + 2 * n_kv_heads) * dh - skip, 1, e, st);
}

}  // namespace trj
