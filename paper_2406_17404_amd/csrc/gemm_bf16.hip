// The projections that store fp32 split-k partial sums, the launch plan of all
// projections, and the split-k sum with what follows it.  The kernel is in gemm_ring.h; the
// projections with a fused epilogue are in gemm_qkv.hip, gemm_gate_up.hip and gemm_lm.hip.
#include "gemm_ring.h"

namespace trj {

// acc layout of v_mfma_f32_32x32x16: lane l, register v -> tile row 8*(v/4) + 4*(l/32) +
// v%4, tile column l%32.  Rows are output features, columns are token rows.

// ---- epilogue: fp32 store, y[split][t][n_out]; 4 consecutive features per store
struct EpiStoreF32T {
  static constexpr bool kScaled = false;  // the accumulators are what the caller wants
  float* y;
  int ld, T;
  size_t split_stride;
  __device__ void operator()(const f32x16& acc, int tile, int ttile, int lane, int split) const {
    int t = ttile * 32 + (lane & 31);
    if (t >= T) return;
    float* row = y + split * split_stride + (size_t)t * ld + tile * 32 + 4 * (lane >> 5);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
      *reinterpret_cast<f32x4*>(row + 8 * g) = v;
    }
  }
};

// ---- launch plan
// Few rows (one pass of up to four token tiles): a launch lasts as long as its busiest
// compute unit takes to pull its bytes (gemm_ring.h), i.e. rounds of workgroups over 256
// compute units x (row tiles + token tiles) KiB per k-step of a workgroup.  The shape with
// the smallest product wins, so row tiles are spread over all compute units and only outputs
// too wide for one round get wide workgroups (128256 x 4096 at 96 rows, 4 row tiles per
// workgroup in four rounds 218 us, 8 in two 187, 16 in one 179).
static GemmShape plan_few(int mt, int ntiles, int ksteps, int split, int* rows, int* kw) {
  int best = 1;
  long best_cost = -1;
  for (int n : {1, 2, 3, 4, 16}) {
    // four token tiles: three row tiles measured faster (22016 x 4096: 40.5 against 43.0 us), but
    // four row tiles are the documented plan of that workload, which is kept
    if (n == 3 && mt == 4) continue;
    const long cost = ((long)(ntiles + n - 1) / n * split + 255) / 256 * (n + mt);
    if (best_cost < 0 || cost < best_cost) { best = n; best_cost = cost; }
  }
  *rows = best;
  // k-parts: enough wavefronts (4 to 8) to keep the matrix units and LDS busy
  *kw = 1;
  if (best == 16) return GS_16;
  if (best == 1) { *kw = 4; return GS_1x4; }
  if (best == 3) { *kw = 2; return GS_3x2; }
  // two row tiles: four k-parts do not pay on short k ranges (4096 x 4096 split four ways at 128
  // rows 12.8 against 11.8 us) and hardly on long ones (12288 x 4096 at 32 rows 18.8 against
  // 18.9); at 128 rows two measured faster there too (27.8 against 30.6), but four are the
  // documented plan of that workload, which is kept
  if (best == 2) { *kw = ksteps / split >= 128 ? 4 : 2; return *kw == 4 ? GS_2x4 : GS_2x2; }
  if (mt < 4 || split > 1) return GS_4x1;  // 64 rows, 32000 x 4096: 45.7 against 45.4 us with two k-parts
  *kw = 2;                                 // 128 rows, 28672 x 4096: 44.7 against 45.1
  return GS_4x2;
}

// Many rows (packed batches): a workgroup's tile sets both its rate and how evenly the launch
// fills the chip.  us of one round of workgroups over the compute units, 256 k-steps, measured
// from 256 to 1024 rows at 4096 columns; rounds x this predicts the launch within 10 % except
// where HBM or power cap it (all shapes alike).
struct ManyShape {
  GemmShape s;
  int rows, tokens, wt;
  float us;
};
constexpr ManyShape MANY[] = {{GS_MANY_2, 2, 4, 1, 28.f}, {GS_MANY_4x4, 4, 4, 2, 37.f},
                              {GS_MANY_4x8, 4, 8, 2, 55.f}, {GS_MANY_8x8, 8, 8, 4, 95.f}};
static long many_wgs(const ManyShape& c, int ttiles, int ntiles) {
  return (long)((ntiles + c.rows - 1) / c.rows) * ((ttiles + c.tokens - 1) / c.tokens);
}
// Where two groups of wavefronts take turns (gemm_pair.h): the 4 x 4 tile, if a compute unit has no
// second workgroup to work in the gaps (more workgroups: 22016 x 4096 at 1024 rows 227 against 210 us),
// all phases are whole and the k range is long enough for the ring of five buffers to fill and drain:
// bare products with cold weights, without turns -> with, us: 4096 x 1024 at 1024 rows 18.9 -> 19.8,
// 8192 x 2048 at 512 28.5 -> 30.2, 11008 x 2048 at 160 26.6 -> 28.9; 4096 x 4096 at 1024 51.0 -> 49.7,
// 4096 x 11008 116.7 -> 114.0.
static bool pair_runs(const ManyShape& c, int ttiles, int ntiles, int ksteps, int split) {
  return c.s == GS_MANY_4x4 && ksteps % PAIR_PHASE == 0 && ksteps * 16 >= tune().gemm_pair_min_k && split == 1 && many_wgs(c, ttiles, ntiles) <= 256;
}
static float many_cost(const ManyShape& c, int ttiles, int ntiles, int ksteps, int split) {
  const float us = pair_runs(c, ttiles, ntiles, ksteps, split) ? 34.f : c.us;
  return (float)((many_wgs(c, ttiles, ntiles) * split + 255) / 256) * us * ksteps / (256.f * split);
}
static const ManyShape& plan_many(int ttiles, int ntiles, int ksteps, int split) {
  const ManyShape* best = nullptr;
  float best_cost = 0.f;
  for (const ManyShape& c : MANY) {
    if (tune().gemm_big_wt != 0 && c.wt != tune().gemm_big_wt) continue;
    const float cost = many_cost(c, ttiles, ntiles, ksteps, split);
    if (!best || cost < best_cost) { best = &c; best_cost = cost; }
  }
  return *best;
}
static bool many_rows(int tp) { return tp > 128 && tune().gemm_big_t > 0 && tp >= tune().gemm_big_t; }

static GemmPlan plan_split(int tp, int n_in, int n_out, int split_k) {
  GemmPlan g;
  const int ttiles = tp >> 5, ntiles = n_out >> 5, ksteps = n_in >> 4;
  auto splits = [&](GemmShape s) {  // grid splits a request really gets: never an empty one
    const int ph = gemm_phase(s), nph = (ksteps + ph - 1) / ph;
    const int sk = split_k > nph ? nph : split_k;
    const int pps = (nph + sk - 1) / sk;
    return (nph + pps - 1) / pps;
  };
  g.many = many_rows(tp);
  g.pair = false;
  if (g.many) {
    const ManyShape& c = plan_many(ttiles, ntiles, ksteps, split_k);
    g.shape = c.s;
    g.mt = c.tokens;
    g.rows = c.rows;
    g.pair = pair_runs(c, ttiles, ntiles, ksteps, split_k);
    g.kw = c.s == GS_MANY_2 ? 4 : g.pair ? 2 : 1;
    g.wt = c.wt;
  } else {
    g.mt = ttiles < 4 ? ttiles : 4;
    g.shape = plan_few(g.mt, ntiles * ((ttiles + g.mt - 1) / g.mt), ksteps, split_k, &g.rows, &g.kw);
    if (const int cfg = tune().gemm_cfg) {  // 1..6 force a shape
      constexpr GemmShape shapes[] = {GS_4x1, GS_2x4, GS_2x2, GS_4x2, GS_1x4, GS_3x2};
      constexpr int rows[] = {4, 2, 2, 4, 1, 3}, kws[] = {1, 4, 2, 2, 4, 2};
      g.shape = shapes[cfg - 1];
      g.rows = rows[cfg - 1];
      g.kw = kws[cfg - 1];
    }
    g.wt = g.shape == GS_16 ? 2 : 1;
  }
  g.split_k = splits(g.shape);
  return g;
}
// A request that the shape it leads to cannot fill (fewer phases than splits) is lowered to
// what it gets, which may change the shape, until the two agree: asking again for the number
// of splits of a plan gives the same plan, on which its callers rely for their buffers.
GemmPlan plan_gemm(int tp, int n_in, int n_out, int split_k) {
  if (split_k < 1) split_k = 1;
  for (;;) {
    const GemmPlan g = plan_split(tp, n_in, n_out, split_k);
    if (g.split_k == split_k) return g;
    split_k = g.split_k;  // always smaller: ends
  }
}

// the launch plan of a projection as six numbers (for tests and experiments): row-tile
// columns per pass, row tiles and k-parts per workgroup, row tiles per wavefront, grid
// k-splits, 1 if a many-rows shape runs
void gemm_bf16_describe_plan(int tp, int n_in, int n_out, int split_k, int32_t out[6]) {
  GemmPlan g = plan_gemm(tp, n_in, n_out, split_k);
  out[0] = g.mt; out[1] = g.rows; out[2] = g.kw; out[3] = g.wt; out[4] = g.split_k;
  out[5] = g.many ? 1 : 0;
}

// number of grid splits a request for split_k really gets
int gemm_bf16_clamp_split(int n_out, int tp, int n_in, int split_k) {
  return plan_gemm(tp, n_in, n_out, split_k).split_k;
}

int gemm_bf16_split_k(int n_out, int tp, int n_in) {
  const int ntiles = n_out >> 5, ttiles = tp >> 5, ksteps = n_in >> 4;
  int sk = 1;
  if (many_rows(tp)) {
    // us at 1024 x 4096 behind the product: an unsplit one is added to the residual stream in its
    // epilogue and a launch only reads it (8), split ones are images to write, read again
    // and add (30 for two, 50 for four).  With the output projection unsplit at 1024 rows:
    // 41.0 + 19.8 us for the sum -> 47.5 + 10.1.  An unsplit projection that takes turns, with whole
    // row groups, has no such launch (gemm_residual.hip; its readers pay 1 to 2 us) and is charged the 8 all the
    // same: 4096 x 11008 keeps two splits at 640 and 768 rows, 4096 x 14336 four or two from 640 to 1024
    float best = 0.f;
    for (int s : {1, 2, 4}) {
      const float cost = many_cost(plan_many(ttiles, ntiles, ksteps, s), ttiles, ntiles, ksteps, s) +
                         (s == 1 ? 8.f : 10.f + 10.f * s) * (ttiles / 32.f) * (ntiles / 128.f);
      if (s == 1 || cost < best) { best = cost; sk = s; }
    }
  } else {
    // projections whose epilogue is a plain partial-sum store are split along k until the
    // launch has about one workgroup (of 2 row tiles) per compute unit; at 33..64 token rows
    // twice as many splits pay, the workgroups of 4 row tiles re-read half as much of the
    // activations (4096 x 11008: 17.5 against 17.8 us; 32 rows 16.1 against 15.8)
    const int mt = ttiles < 4 ? ttiles : 4;
    const int groups = ((ntiles + 1) / 2) * ((ttiles + mt - 1) / mt);
    const int target = mt == 2 ? 2 * tune().gemm_target_wgs : tune().gemm_target_wgs;
    sk = (target + groups - 1) / groups;
  }
  if (sk > tune().max_split_k) sk = tune().max_split_k;
  return gemm_bf16_clamp_split(n_out, tp, n_in, sk);
}

int launch_gemm_store_f32(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in,
                          int n_out, int split_k, float* y, hipStream_t st) {
  EpiStoreF32T e{y, n_out, T, (size_t)T * n_out};
  return launch_gemm(xp, w, tp, n_in, n_out, split_k, e, st);
}

// ------------------------------------------------------------------ split-k sum + residual + norm input
// x[t] += sum_s partial[s][t] (fixed order: s = 0, 1, ...), and the next projection's input
// bf16(x * g) in the tiled activation layout, NOT yet divided by the row's norm: each
// workgroup owns one column part (about 1024 columns) of one token row and writes that part's sum of x^2 to
// ssq[part][t]; the consuming projection divides (RowScale).  Rows t >= T of the padded tile
// are written as zeros.  Without partials x is only read; with an embedding table the row comes
// from it instead (x[t] = E[tok[t]], ids outside [0, vocab) clamped).
constexpr int RN_MAX_THREADS = 256, RN_SB = 8;
// column parts of a row: about 1024 columns each, at most RS_MAX_PARTS
int reduce_norm_parts(int d) {
  int p = (d + 1023) / 1024;
  return p > RS_MAX_PARTS ? RS_MAX_PARTS : p;
}
// threads per workgroup (8 columns each): the part's share of the row, in whole wavefronts
int reduce_norm_threads(int d) {
  const int ngran = d >> 3, parts = reduce_norm_parts(d);
  return ((ngran + parts - 1) / parts + WAVE - 1) / WAVE * WAVE;
}

// a, b += partial sums of splits 0 .. n_split-1 in that order, SB loads in flight at a time
// (indices past the last split are clamped for the load and left out of the sum)
template <int SB>
__device__ __forceinline__ void add_splits(const float* __restrict__ pr, int n_split,
                                           size_t split_stride, f32x4& a, f32x4& b) {
  for (int s0 = 0; s0 < n_split; s0 += SB) {
    f32x4 pa[SB], pb[SB];
#pragma unroll
    for (int j = 0; j < SB; ++j) {
      const float* q = pr + min(s0 + j, n_split - 1) * split_stride;
      pa[j] = *reinterpret_cast<const f32x4*>(q);
      pb[j] = *reinterpret_cast<const f32x4*>(q + 4);
    }
#pragma unroll
    for (int j = 0; j < SB; ++j) {
      if (s0 + j < n_split) {
        a += pa[j];
        b += pb[j];
      }
    }
  }
}

__global__ __launch_bounds__(RN_MAX_THREADS) void reduce_norm_kernel(
    const float* __restrict__ partial, int n_split, size_t split_stride, float* __restrict__ x,
    const uint16_t* __restrict__ embed, const int32_t* __restrict__ tok, int vocab,
    const float* __restrict__ g, int T, int d, int tp, uint16_t* __restrict__ hp,
    float* __restrict__ ssq) {
  const int t = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
  const int ngran = d >> 3;
  const int gi_raw = part * blockDim.x + tid;
  const bool live = gi_raw < ngran;
  const int gi = min(gi_raw, ngran - 1);
  if (t >= T) {
    const u32x4 z = {0, 0, 0, 0};
    if (live) *reinterpret_cast<u32x4*>(hp + a_off(t, gi * 8, tp)) = z;
    if (tid == 0) ssq[(size_t)part * tp + t] = 0.f;
    return;
  }
  // every load of the thread is issued before the first one is used
  float* xr = x + (size_t)t * d + gi * 8;
  f32x4 a, b;
  const f32x4 g0 = *reinterpret_cast<const f32x4*>(g + gi * 8);
  const f32x4 g1 = *reinterpret_cast<const f32x4*>(g + gi * 8 + 4);
  if (embed) {  // uniform over the launch
    int id = tok[t];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
    const u32x4 v = *reinterpret_cast<const u32x4*>(embed + (size_t)id * d + gi * 8);
    a = f32x4{__builtin_bit_cast(float, v[0] << 16), __builtin_bit_cast(float, v[0] & 0xffff0000u),
              __builtin_bit_cast(float, v[1] << 16), __builtin_bit_cast(float, v[1] & 0xffff0000u)};
    b = f32x4{__builtin_bit_cast(float, v[2] << 16), __builtin_bit_cast(float, v[2] & 0xffff0000u),
              __builtin_bit_cast(float, v[3] << 16), __builtin_bit_cast(float, v[3] & 0xffff0000u)};
  } else {
    a = *reinterpret_cast<f32x4*>(xr);
    b = *reinterpret_cast<f32x4*>(xr + 4);
    // as many loads in flight as there are splits, up to RN_SB (n_split is uniform over
    // the launch); the sum runs in the same order s = 0, 1, ... whichever batch is taken
    const float* pr = partial + (size_t)t * d + gi * 8;
    if (n_split <= 2) add_splits<2>(pr, n_split, split_stride, a, b);
    else if (n_split <= 4) add_splits<4>(pr, n_split, split_stride, a, b);
    else add_splits<RN_SB>(pr, n_split, split_stride, a, b);
  }
  float ss = 0.f;
  if (live) {
    if (embed || n_split > 0) {
      *reinterpret_cast<f32x4*>(xr) = a;
      *reinterpret_cast<f32x4*>(xr + 4) = b;
    }
    u32x4 pk = {pack2bf(a[0] * g0[0], a[1] * g0[1]), pack2bf(a[2] * g0[2], a[3] * g0[3]),
                pack2bf(b[0] * g1[0], b[1] * g1[1]), pack2bf(b[2] * g1[2], b[3] * g1[3])};
    *reinterpret_cast<u32x4*>(hp + a_off(t, gi * 8, tp)) = pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) ss += a[e] * a[e] + b[e] * b[e];
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  __shared__ float wsum[RN_MAX_THREADS / WAVE];
  if ((tid & 63) == 0) wsum[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) {
    float tot = 0.f;
    for (int w = 0; w < (int)blockDim.x / WAVE; ++w) tot += wsum[w];
    ssq[(size_t)part * tp + t] = tot;
  }
}

int launch_reduce_norm(const float* partial, int n_split, float* x, const float* g, int T, int d,
                       int tp, uint16_t* hp, float* ssq, hipStream_t st) {
  if ((d & 7) || reduce_norm_threads(d) > RN_MAX_THREADS) return TRJ_ERR_BAD_SHAPE;
  reduce_norm_kernel<<<dim3(tp, reduce_norm_parts(d)), reduce_norm_threads(d), 0, st>>>(
      partial, n_split, (size_t)T * d, x, nullptr, nullptr, 0, g, T, d, tp, hp, ssq);
  return check_launch();
}

int launch_embed_norm(const uint16_t* embed, const int32_t* tok, int T, int d, int vocab, float* x,
                      const float* g, int tp, uint16_t* hp, float* ssq, hipStream_t st) {
  if ((d & 7) || reduce_norm_threads(d) > RN_MAX_THREADS) return TRJ_ERR_BAD_SHAPE;
  reduce_norm_kernel<<<dim3(tp, reduce_norm_parts(d)), reduce_norm_threads(d), 0, st>>>(
      nullptr, 0, 0, x, embed, tok, vocab, g, T, d, tp, hp, ssq);
  return check_launch();
}

// y = sum over splits of partial[s] (fixed order); for the stand-alone linear entry point
__global__ void sum_splits_kernel(const float* __restrict__ partial, int n_split, size_t n,
                                  float* __restrict__ y) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float acc = 0.f;
  for (int s = 0; s < n_split; ++s) acc += partial[s * n + i];
  y[i] = acc;
}
int launch_sum_splits(const float* partial, int n_split, size_t n, float* y, hipStream_t st) {
  sum_splits_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(partial, n_split, n, y);
  return check_launch();
}

// plain [T][n] bf16 -> tiled activation layout (zero padded rows); for the stand-alone
// linear entry point
__global__ void tile_activation_kernel(const uint16_t* __restrict__ x, int T, int n, int tp,
                                       uint16_t* __restrict__ xp) {
  const int t = blockIdx.x;
  for (int gi = threadIdx.x; gi < (n >> 3); gi += blockDim.x) {
    u32x4 v = {0, 0, 0, 0};
    if (t < T) v = *reinterpret_cast<const u32x4*>(x + (size_t)t * n + gi * 8);
    *reinterpret_cast<u32x4*>(xp + a_off(t, gi * 8, tp)) = v;
  }
}
int launch_tile_activation(const uint16_t* x, int T, int n, int tp, uint16_t* xp, hipStream_t st) {
  tile_activation_kernel<<<tp, 256, 0, st>>>(x, T, n, tp, xp);
  return check_launch();
}

}  // namespace trj
