// fp32 mode of the verify step (fp32 storage, fp32 arithmetic): used for the tiny fp32
// workload and as a tight-tolerance check of the data layouts.  Launches of a tiny model are
// latency: a step of two layers was 25 launches and 218 us, of which the serial loops of one
// thread per output (a k range of 1024, a row's scores and values) were half.  Now every
// output is summed by 32 threads whose loads are in flight together, and norm, rotary rotation
// with the K/V write, and SiLU(g) * u are part of the projection next to them: 14 launches, 65 us, and the result is closer to the
// 64-bit one (3.4e-7 against 8.1e-7).
// They read the same tiled weight / KV layouts as the bf16 kernels.  The rotary table at the
// top serves both modes.
#include <type_traits>

#include "common.h"
#include "f32_rule.h"
#include "kernels.h"
#include "tree_vis.h"

namespace trj {

// ------------------------------------------------------------------ rotary table
// cs[t][j] = (cos, sin) of row_pos[t] * theta^(-2j/dh), evaluated in double; without
// row_pos the table is over positions themselves (row t = position t).
__global__ void rope_table_kernel(const int32_t* __restrict__ row_pos, int T, int dh, float theta,
                                  float2* __restrict__ cs) {
  int half = dh >> 1;
  int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= T * half) return;
  int t = idx / half, j = idx % half;
  double ang = (double)(row_pos ? row_pos[t] : t) * pow((double)theta, -2.0 * j / dh);
  cs[idx] = make_float2((float)cos(ang), (float)sin(ang));
}
int launch_rope_table(const int32_t* row_pos, int T, int dh, float theta, float2* cs,
                      hipStream_t st) {
  int n = T * (dh >> 1);
  rope_table_kernel<<<(n + 255) / 256, 256, 0, st>>>(row_pos, T, dh, theta, cs);
  return check_launch();
}

// ------------------------------------------------------------------ embedding
// x[t][:] = E[tok[t]][:] where the prologue does not do it (more than PREP_MAX_SEQS sequences).
// Token ids outside [0, vocab) are clamped.
__global__ void embed_kernel(const float* __restrict__ embed, const int32_t* __restrict__ tok, int d, int vocab,
                             float* __restrict__ x) {
  int t = blockIdx.x;
  int id = tok[t];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
  for (int c = threadIdx.x; c < d; c += blockDim.x) x[(size_t)t * d + c] = embed[(size_t)id * d + c];
}
int launch_embed(const float* embed, const int32_t* tok, int T, int d, int vocab, float* x, hipStream_t st) {
  embed_kernel<<<T, 256, 0, st>>>(embed, tok, d, vocab, x);
  return check_launch();
}

// ------------------------------------------------------------------ GEMM (fp32)
// y[t][r] = sum_k x[t][k] * W(r, k) for packed rows r.  Workgroup: one tile of 32 packed rows x
// TT tokens; thread (part, row) sums every 32nd granule of 8 k values for all TT tokens, the
// 32 parts are added in order through LDS.  With a gain `g` the input is RMSNorm(x): the
// products use x * g and the sum is divided by the token's norm, whose sum of squares comes
// from the same reads.
constexpr int F32_THREADS = 32 * F32_PARTS;
struct GemmF32Args {
  const float *x, *w, *g;
  int T, n_in;
  float eps;
};
template <bool VEC>
__device__ inline void load8(const float* p, float (&v)[8]) {
  if constexpr (VEC) {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[e];
  }
}
// UN granules of a thread are asked for together (past the last: the last one again, not added);
// they are added in the same order whatever UN is.
template <int TT, int UN, bool NORM, bool VEC>
__device__ inline void gemm_f32_sums(const GemmF32Args& a, int rt, int t0, int part, int rl, float (&acc)[TT],
                                     float (&ss)[TT]) {
  const int ng = a.n_in >> 3;
  const float* wt = a.w + (size_t)rt * (a.n_in >> 4) * 512 + rl * 8;
  for (int g0 = part; g0 < ng; g0 += F32_PARTS * UN) {
    float wv[UN][8], gv[UN][8], xv[UN][TT][8];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int gi = min(g0 + u * F32_PARTS, ng - 1);
      load8<true>(wt + (size_t)gi * 256, wv[u]);  // granule = (k-step, half): 32 rows of 8 values
      if (NORM) load8<VEC>(a.g + gi * 8, gv[u]);
#pragma unroll
      for (int i = 0; i < TT; ++i) load8<VEC>(a.x + (size_t)min(t0 + i, a.T - 1) * a.n_in + gi * 8, xv[u][i]);
    }
    if (UN > 1) __builtin_amdgcn_sched_barrier(0);  // all loads first
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (UN > 1 && g0 + u * F32_PARTS >= ng) break;
#pragma unroll
      for (int i = 0; i < TT; ++i) {
        if (NORM) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            ss[i] = fmaf(xv[u][i][e], xv[u][i][e], ss[i]);
            xv[u][i][e] *= gv[u][e];
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i] = fmaf(wv[u][e], xv[u][i][e], acc[i]);
      }
    }
  }
}
template <int TT, int UN, bool NORM, class Epi>
__global__ __launch_bounds__(F32_THREADS) void gemm_f32_kernel(const float* x, const float* w, const float* g, int T, int n_in,
                                                            float eps, Epi epi) {
  const GemmF32Args a{x, w, g, T, n_in, eps};  // plain arguments: in scalar registers from the start (build.py)
  __shared__ float red[F32_PARTS][TT][32], sq[F32_PARTS][TT];
  const int rl = threadIdx.x & 31, part = threadIdx.x >> 5;
  const int rt = blockIdx.x, t0 = blockIdx.y * TT;
  float acc[TT], ss[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) acc[i] = ss[i] = 0.f;
  // 16-byte loads of the input where the caller's pointers allow them (uniform)
  const bool vec = ((reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.g)) & 15) == 0;
  if (vec) gemm_f32_sums<TT, UN, NORM, true>(a, rt, t0, part, rl, acc, ss);
  else gemm_f32_sums<TT, UN, NORM, false>(a, rt, t0, part, rl, acc, ss);
#pragma unroll
  for (int i = 0; i < TT; ++i) {
    red[part][i][rl] = acc[i];
    if (rl == 0) sq[part][i] = ss[i];
  }
  __syncthreads();
  const int i = threadIdx.x >> 5, t = t0 + i;
  if (i >= TT || t >= a.T) return;  // whole half-wavefronts: the epilogues exchange within one
  float v = 0.f, s = 0.f;
#pragma unroll
  for (int p = 0; p < F32_PARTS; ++p) {
    v += red[p][i][rl];
    s += sq[p][i];
  }
  if (NORM) v *= 1.0f / sqrtf(s / a.n_in + a.eps);
  epi(v, rt, rl, t);
}

struct EpiF32Store {
  float* y;
  int n_out, add_to;
  __device__ void operator()(float v, int rt, int rl, int t) const {
    float* o = y + (size_t)t * n_out + rt * 32 + rl;
    *o = add_to ? *o + v : v;
  }
};
// logits, and of every row the largest of this tile with its index (ArgmaxCand)
struct EpiF32Lm {
  float* y;
  ArgmaxCand* cand;
  int n_out;
  __device__ void operator()(float v, int rt, int rl, int t) const {
    y[(size_t)t * n_out + rt * 32 + rl] = v;
    float bv = -INFINITY;
    int bi = INT32_MAX;
    if (v == v) { bv = v; bi = rt * 32 + rl; }  // NaN never wins
    for (int o = 16; o > 0; o >>= 1) {          // within the row's 32 lanes
      const float ov = __shfl_xor(bv, o);
      const int oi = __shfl_xor(bi, o);
      if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (rl == 0) cand[(size_t)t * (n_out >> 5) + rt] = ArgmaxCand{bv, bi};
  }
};
// tile rows 0..15 are gate rows 16 rt .., rows 16..31 the matching up rows
struct EpiF32GateUp {
  float* act;
  int F;
  __device__ void operator()(float v, int rt, int rl, int t) const {
    const float u = __shfl_xor(v, 16);
    if (rl < 16) act[(size_t)t * F + 16 * rt + rl] = v / (1.0f + expf(-v)) * u;
  }
};
// q (rotated) plain, K (rotated) and V into the pool at the row's slot; a q or k tile holds
// the rotary partners j and j + dh/2 16 rows apart
struct EpiF32QKV {
  const float2* cs;       // [.][dh/2]: row t of the table, or row cs_row[t] if given
  const int32_t* cs_row;
  const int32_t* row_slot;
  float *q, *k_layer, *v_layer;
  int n_heads, n_kv_heads, dh, s_pool;
  __device__ void operator()(float v, int rt, int rl, int t) const {
    const float other = __shfl_xor(v, 16);
    const int slot = row_slot[t];
    if (slot < 0) return;  // row of a malformed sequence
    const int tph = dh >> 5, q_tiles = n_heads * tph, kv_tiles = n_kv_heads * tph, half = dh >> 1;
    const int sec = rt < q_tiles ? 0 : (rt < q_tiles + kv_tiles ? 1 : 2);
    const int rel = rt - (sec == 0 ? 0 : (sec == 1 ? q_tiles : q_tiles + kv_tiles));
    const int head = rel / tph, jt = rel % tph;
    if (sec == 2) {
      v_layer[(size_t)head * s_pool * dh + v_off(slot, 32 * jt + rl, dh)] = v;
      return;
    }
    const int j = 16 * jt + (rl & 15), c = rl < 16 ? j : j + half;
    const float2 sc = cs[(size_t)(cs_row ? cs_row[t] : t) * half + j];
    const float r = rl < 16 ? v * sc.x - other * sc.y : v * sc.x + other * sc.y;
    if (sec == 0) q[((size_t)t * n_heads + head) * dh + c] = r;
    else k_layer[(size_t)head * s_pool * dh + k_off(slot, c, dh)] = r;
  }
};
// tokens per workgroup: gemm_f32_tokens; behind a norm four or eight
template <class Epi>
static int gemm_f32(const GemmF32Args& a, int n_out, const Epi& e, hipStream_t st) {
  if (a.T < 1 || a.n_in < 16 || n_out < 32 || (a.n_in & 15) || (n_out & 31)) return TRJ_ERR_BAD_SHAPE;
  const dim3 by4(n_out / 32, (a.T + 3) / 4), by8(n_out / 32, (a.T + 7) / 8);
  if (a.g) {
    if (a.T <= 16) gemm_f32_kernel<4, 1, true><<<by4, F32_THREADS, 0, st>>>(a.x, a.w, a.g, a.T, a.n_in, a.eps, e);
    else gemm_f32_kernel<8, 1, true><<<by8, F32_THREADS, 0, st>>>(a.x, a.w, a.g, a.T, a.n_in, a.eps, e);
  } else if constexpr (std::is_same_v<Epi, EpiF32Store>) {  // the others follow a norm
    const int tokens = gemm_f32_tokens(a.T, a.n_in, n_out);
    if (tokens == 2)
      gemm_f32_kernel<2, 4, false><<<dim3(n_out / 32, (a.T + 1) / 2), F32_THREADS, 0, st>>>(a.x, a.w, a.g, a.T, a.n_in, a.eps, e);
    else if (tokens == 4) gemm_f32_kernel<4, 1, false><<<by4, F32_THREADS, 0, st>>>(a.x, a.w, a.g, a.T, a.n_in, a.eps, e);
    else gemm_f32_kernel<8, 1, false><<<by8, F32_THREADS, 0, st>>>(a.x, a.w, a.g, a.T, a.n_in, a.eps, e);
  } else {
    return TRJ_ERR_NULLPTR;
  }
  return check_launch();
}
int launch_gemm_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int n_out, int add_to,
                    float* y, hipStream_t st) {
  return gemm_f32({x, w, g, T, n_in, eps}, n_out, EpiF32Store{y, n_out, add_to}, st);
}
int launch_gemm_lm_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int n_out, float* y,
                       ArgmaxCand* cand, hipStream_t st) {
  return gemm_f32({x, w, g, T, n_in, eps}, n_out, EpiF32Lm{y, cand, n_out}, st);
}
int launch_gemm_gate_up_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int F,
                            float* act, hipStream_t st) {
  return gemm_f32({x, w, g, T, n_in, eps}, 2 * F, EpiF32GateUp{act, F}, st);
}
int launch_gemm_qkv_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int n_heads,
                        int n_kv_heads, int dh, int s_pool, const float2* cs, const int32_t* cs_row,
                        const int32_t* row_slot, float* q, float* k_layer, float* v_layer, hipStream_t st) {
  return gemm_f32({x, w, g, T, n_in, eps}, (n_heads + 2 * n_kv_heads) * dh,
                  EpiF32QKV{cs, cs_row, row_slot, q, k_layer, v_layer, n_heads, n_kv_heads, dh, s_pool}, st);
}

// ------------------------------------------------------------------ tree attention (fp32)
// One workgroup per (row, head).  Scores of all visible slots are kept in LDS (max_slots
// floats), so the sequence length is limited by the LDS size.  A thread owns a key for the
// scores (its row in pieces of 8 values) and, for the values, a column and every FA_PARTS-th
// group of 4 keys, which are contiguous in a V plane; the parts are added in order through LDS.
constexpr int FA_THREADS = 512;
// Groups of a thread's values in flight together, the first of them from the start: 160 keys with
// heads of 64.  One after the other behind the softmax the kernel took 11.4 us at 143 keys, now 6.2.
constexpr int FA_EARLY = 5;
__global__ __launch_bounds__(FA_THREADS) void tree_attn_f32_kernel(
    const int32_t* __restrict__ row_seq, const int32_t* __restrict__ node_off,
    const int32_t* __restrict__ kv_off, const int32_t* __restrict__ prefix_len,
    const int32_t* __restrict__ status_dev, const float* __restrict__ q, const float* __restrict__ k_layer,
    const float* __restrict__ v_layer, const uint64_t* __restrict__ anc, int n_heads, int group, int dh, int s_pool,
    int max_slots, float scale, float* __restrict__ out) {
  extern __shared__ float lds[];
  float* qs = lds;            // dh
  float* sc = lds + dh;       // max_slots, then (values' parts) at least FA_THREADS
  __shared__ float wred[FA_THREADS / WAVE];
  const int t = blockIdx.x, head = blockIdx.y, tid = threadIdx.x;
  float* o = out + ((size_t)t * n_heads + head) * dh;
  const int s = row_seq[t];
  const int L = s < 0 ? 0 : prefix_len[s], i = s < 0 ? 0 : t - node_off[s];
  const int base = s < 0 ? 0 : kv_off[s];
  const int nk = L + i + 1;  // ancestors have smaller indices than i
  if (s < 0 || status_dev[s] != 0 || nk > max_slots) {  // uniform
    for (int c = tid; c < dh; c += FA_THREADS) o[c] = 0.f;
    return;
  }
  const float* kp = k_layer + (size_t)(head / group) * s_pool * dh;  // the group's K/V head
  const float* vp = v_layer + (size_t)(head / group) * s_pool * dh;
  const float* qr = q + ((size_t)t * n_heads + head) * dh;
  for (int c = tid; c < dh; c += FA_THREADS) qs[c] = qr[c];
  // values: columns [c0, c0 + cols) by `parts` threads each.  A thread's first groups are asked for
  // here, with the keys, instead of behind the softmax one after the other
  const int cols = dh < FA_THREADS ? dh : FA_THREADS, parts = FA_THREADS / cols;
  const int col = tid % cols, part = tid / cols, last4 = (nk - 1) & ~3;
  float early[FA_EARLY][4];
  auto load_group = [&](int k4, int c, float (&v)[4]) {  // kv_off is a multiple of 32: groups of 4 stay together
    const float* vg = vp + v_off(base + min(k4, last4), c, dh);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = vg[e];
  };
#pragma unroll
  for (int j = 0; j < FA_EARLY; ++j) load_group(4 * (part + j * parts), col, early[j]);
  __syncthreads();
  const uint64_t a0 = anc[2 * (size_t)t], a1 = anc[2 * (size_t)t + 1];
  float mx = -INFINITY;
  for (int kk = tid; kk < nk; kk += FA_THREADS) {
    float sv = -INFINITY;
    if (tree_key_visible(kk, L, a0, a1)) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      for (int c = 0; c < dh; c += 32) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float* kg = kp + k_off(base + kk, c + 8 * g, dh);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[g] = fmaf(qs[c + 8 * g + e], kg[e], acc[g]);
        }
      }
      sv = ((acc[0] + acc[1]) + (acc[2] + acc[3])) * scale;
    }
    sc[kk] = sv;
    mx = fmaxf(mx, sv);
  }
  auto block_reduce = [&](float v, auto op) {  // the same value in every thread, fixed order
    for (int o2 = 32; o2 > 0; o2 >>= 1) v = op(v, __shfl_xor(v, o2));
    if ((tid & 63) == 0) wred[tid >> 6] = v;
    __syncthreads();
    v = wred[0];
    for (int w = 1; w < FA_THREADS / WAVE; ++w) v = op(v, wred[w]);
    __syncthreads();
    return v;
  };
  mx = block_reduce(mx, [](float a, float b) { return fmaxf(a, b); });
  float sum = 0.f;
  for (int kk = tid; kk < nk; kk += FA_THREADS) {
    const float p = sc[kk] == -INFINITY ? 0.f : expf(sc[kk] - mx);
    sc[kk] = p;
    sum += p;
  }
  sum = block_reduce(sum, [](float a, float b) { return a + b; });
  const float inv = 1.0f / sum;
  float* red = sc + ((nk + 3) & ~3);  // parts x cols
  for (int c0 = 0; c0 < dh; c0 += cols) {
    const int c = c0 + col;
    float acc = 0.f;
    auto add_group = [&](int k4, const float (&v)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p = k4 + e < nk ? sc[min(k4 + e, nk - 1)] : 0.f;
        acc = p != 0.f ? fmaf(p, v[e], acc) : acc;  // slots nobody sees may hold anything
      }
    };
    if (part < parts && c < dh) {
      int k4 = 4 * part;
      if (c0 == 0) {
#pragma unroll
        for (int j = 0; j < FA_EARLY; ++j) add_group(4 * (part + j * parts), early[j]);
        k4 += 4 * FA_EARLY * parts;
      }
      for (; k4 < nk; k4 += 4 * FA_EARLY * parts) {
        float v[FA_EARLY][4];
#pragma unroll
        for (int j = 0; j < FA_EARLY; ++j) load_group(k4 + 4 * j * parts, c, v[j]);
#pragma unroll
        for (int j = 0; j < FA_EARLY; ++j) add_group(k4 + 4 * j * parts, v[j]);
      }
    }
    if (part < parts) red[part * cols + col] = acc;
    __syncthreads();
    if (part == 0 && c < dh) {
      for (int p = 1; p < parts; ++p) acc += red[p * cols + col];
      o[c] = acc * inv;
    }
    __syncthreads();
  }
}
// LDS of the attention: query, scores (with the padding to groups of 4), the values' parts
static size_t attn_f32_lds(int dh, int max_slots) {
  return (size_t)(dh + max_slots + 4 + FA_THREADS) * sizeof(float);
}
int launch_tree_attn_f32(const float* q, const float* k_layer, const float* v_layer,
                         const uint64_t* anc, const int32_t* row_seq, const int32_t* node_off,
                         const int32_t* kv_off, const int32_t* prefix_len,
                         const int32_t* status_dev, int T, int n_heads, int n_kv_heads, int dh,
                         int s_pool, int max_slots, float scale, float* out, hipStream_t st) {
  if ((size_t)(dh + max_slots) * sizeof(float) > 64 * 1024) return TRJ_ERR_BAD_SHAPE;
  const size_t lds = attn_f32_lds(dh, max_slots);
  static DeviceOnce once;
  allow_lds(once, tree_attn_f32_kernel, 96 * 1024);  // a little more than 64 KiB at the limit
  dim3 grid(T, n_heads);
  tree_attn_f32_kernel<<<grid, FA_THREADS, lds, st>>>(row_seq, node_off, kv_off, prefix_len, status_dev, q,
                                              k_layer, v_layer, anc, n_heads,
                                              n_heads / n_kv_heads, dh, s_pool, max_slots, scale,
                                              out);
  return check_launch();
}

}  // namespace trj
