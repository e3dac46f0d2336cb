// Tree-masked attention, bf16 storage, fp32 softmax and accumulation.
//
// The work is streaming the sequence's K/V once.  A workgroup owns a contiguous range of
// 32-slot blocks of one (sequence, head) and one group of query rows (tree nodes), in tiles of
// 32; wavefront (key stream, tile) walks every KS-th block of the range for one tile.  K and V
// blocks are tiled in memory so that each lane's 16 bytes are directly an MFMA A operand:
//   S^T[keys, queries] = K[keys, dh] * Q^T          (v_mfma_f32_32x32x16_bf16)
//   O^T[dh, queries]  += V^T[dh, keys] * P^T[keys, queries]
// With keys as the MFMA row dimension each lane holds one query column, so the online
// softmax state (running max, sum, rescale factor) is per lane, and the S^T registers
// are, after conversion to bf16, exactly the B operand of the second product (the V
// tiling stores keys in the order in which S^T leaves them in the registers).
// The ancestor bit rows mask only the blocks that overlap the tree's own slots.
//
// What bounds it: on long sequences the rate at which K/V arrive, i.e. how much is in flight
// and that no byte is asked for twice; on short ones (up to about 1000 slots) some 8 us of
// launch, first loads, merge and stores, one after the other (100 slots x 5 rows, from the first
// workgroup's start: sequence known 1.0 us, parents there 2.7, K there 3.3, the tree's block done
// 6.2, streams merged 6.9, stored 7.9).  Three forms of the walk, chosen by the launch plan
// (figures at attn_bf16_plan):
//  - registers: every wavefront loads its blocks by itself, the next K while this block's
//    softmax and P*V run and the next V behind them.  No wavefront waits for another before the
//    merge; the tiles of a stream find each other's blocks in the caches.
//  - rings: a key stream's wavefronts share a ring of D blocks in LDS that the loads fill without
//    passing through registers; each fetches its part of every half block, K of block i+D as
//    soon as K of block i has been read by all of them.  More is in flight and each byte is
//    asked for once, which pays for the two meetings per block and the second way through LDS
//    where K/V stream from HBM.
//  - at once: up to two blocks per stream, all requested together into LDS, with one meeting for
//    K and one for V.
// Loads of blocks that no other workgroup (rings) or wavefront (registers) reads carry the
// streaming hint.
// The wavefronts of a workgroup merge their (m, l, O) through LDS in a fixed order.  If
// the workgroup covers the whole sequence it writes the normalised rows; otherwise it
// writes an un-normalised partial and a second, small kernel merges the partials of a
// row in split order.  (Merging inside the same launch by "last workgroup to arrive"
// needs device-scope fences; on this multi-die part each of them writes back and
// invalidates a whole L2, which measured 3-4x the cost of the separate launch.)
#include <type_traits>

#include "attn_parts.h"
#include "common.h"
#include "kernels.h"
#include "tree_vis.h"

namespace trj {

constexpr float NEG_BIG = -1e30f;
constexpr float SOFTMAX_LAG = 8.f;  // see softmax_tile_prefix; smaller weights are below a bf16 step of the largest

struct AttnArgs {
  const uint16_t* q;
  const uint16_t* k_layer;
  const uint16_t* v_layer;
  const uint64_t* anc;
  const int32_t* node_off;
  const int32_t* kv_off;
  const int32_t* prefix_len;
  const int32_t* status_dev;
  int n_heads, s_pool, bpwg, nsplit_max, qg_max;
  // Query heads that share a K/V head are worked on together, 1 << pack of them: query p of a
  // sequence is (node p >> pack, head p & ..), `columns` packed heads in all, `group` per K/V head
  int pack, columns, group;
  int n_kv_groups;  // items x K/V heads: sets of workgroups that share K/V blocks
  // work items (sequence, key split, query group) that exist, longest sequence first, and their number
  // (written by the prep kernels): workgroups past the list's end leave at once, and they
  // are the LAST ids of the launch, so the live ones spread evenly over the compute units
  // One record of 8 words per item: sequence, query group, first row, rows, prefix
  // length, first K/V block of the sequence, key split; a workgroup needs nothing else
  // from memory to find its work, and reads record and count together.
  const int32_t* items;
  const int32_t* n_items;  // and, behind it, whether packed heads are walked without splits (attn_parts.h)
  float scale_log2e;
  float lag;  // of the softmax reference behind the running maximum, log2
  // un-normalised partials, one per (query tile, column, split), stored as the
  // image of the wavefront's accumulator registers: element (mt*16 + v)*64 + lane, so that
  // every store and every load of the merge kernel is a contiguous 256-byte row
  float* po;        // [part_tiles][columns][nsplit_max][DH/32 * 16 * 64]
  float* pm;        // [part_tiles][columns][nsplit_max][32] running max (log2 domain)
  float* pl;        // [part_tiles][columns][nsplit_max][32] sum of weights
  int tiles_per_seq;
  uint16_t* out;
  int tiled, tp;
  // one sequence, nothing prepared (SELF)
  const int32_t* parent;
  int32_t* status;  // written: 1 if the sequence is malformed
  int T, max_seq_slots;
};


// Online-softmax update of one query tile with one block of 32 keys: S^T accumulators in,
// packed bf16 probabilities out (the B operand of the second product), running maximum `top`,
// reference m and sum l of this lane's query updated, `alpha` = factor for the O accumulators.
// Weights are 2^(score - m).  The key whose score is m has weight 1, which bf16 holds exactly,
// and the largest weights are what rounding to bf16 costs precision on: the more keys set the
// reference, the closer the result.  With lag 0 the reference is the running maximum, set by a
// few keys per stream.  With lag > 0 every block's largest key sets it, down to 2^-lag of the
// running maximum (below, rounding no longer matters), at the price of rescaling O at every
// block: for walks that have fewer streams or splits than a sequence of that size could have.
// Error against 64 bits of 16 rows on 512 slots: eight streams 2.02e-3, four 2.06e-3 without
// lag, 2.02e-3 with; twelve sequences of 80 rows on up to 2048 slots with two unsplit streams
// 2.175e-3 without, 2.02e-3 with, with four streams 2.135e-3.
// Blocks that lie wholly in the prefix (all but the last few of a sequence) take this
// lean form: no visibility tests; the max works on the raw scores and the scale
// (log2 e / sqrt(dh), > 0) goes into one fused multiply-add per key; v_exp_f32 directly
// (results below the normal range flush to zero, as they should).
__device__ inline void softmax_tile_prefix(const f32x16& sacc, float scale, float lag, float& top, float& m, float& l,
                                           float& alpha, u32x4 (&pk)[2]) {
  float mx = sacc[0];
#pragma unroll
  for (int v = 1; v < 16; ++v) mx = fmaxf(mx, sacc[v]);
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  top = fmaxf(top, mx * scale);
  const float m_new = fmaxf(mx * scale, top - lag);
  alpha = __builtin_amdgcn_exp2f(m - m_new);
  float lsum = 0.f;
  float p[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    p[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[v], scale, -m_new));
    lsum += p[v];
  }
  l = l * alpha + lsum;
  m = m_new;
#pragma unroll
  for (int kg = 0; kg < 2; ++kg)
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[kg][e] = pack2bf(p[8 * kg + 2 * e], p[8 * kg + 2 * e + 1]);
}

// Blocks that overlap the tree's own slots (at most 5 per sequence): ancestor bits decide
// which keys a query sees; a key that is not visible contributes exactly 0, also while
// nothing is visible yet (m == NEG_BIG).
__device__ inline void softmax_tile_tree(const f32x16& sacc, int key0, int hh, int L, uint64_t anc0,
                                         uint64_t anc1, float scale, float lag, float& top, float& m, float& l,
                                         float& alpha, u32x4 (&pk)[2]) {
  float sv[16];
  float mx = NEG_BIG;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int kk = key0 + 8 * (v >> 2) + 4 * hh + (v & 3);
    const bool vis = tree_key_visible(kk, L, anc0, anc1);
    sv[v] = vis ? sacc[v] * scale : NEG_BIG;
    mx = fmaxf(mx, sv[v]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  top = fmaxf(top, mx);
  const float m_new = fmaxf(mx, top - lag);
  alpha = exp2f(m - m_new);
  float lsum = 0.f;
  float p[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    p[v] = sv[v] > -1e29f ? exp2f(sv[v] - m_new) : 0.f;
    lsum += p[v];
  }
  l = l * alpha + lsum;
  m = m_new;
#pragma unroll
  for (int kg = 0; kg < 2; ++kg)
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[kg][e] = pack2bf(p[8 * kg + 2 * e], p[8 * kg + 2 * e + 1]);
}

// O accumulators times alpha; skipped when no query of the wavefront moved its maximum
// (alpha == 1 in every lane), which is the common case once a few blocks have been seen
template <int MTV>
__device__ inline void rescale_o(f32x16 (&o)[MTV], float alpha) {
  if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) == 0) return;
#pragma unroll
  for (int mt = 0; mt < MTV; ++mt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[mt][v] *= alpha;
}

template <int DH>
__device__ inline void attn_store_row(const AttnArgs& a, int t, int head, int c, u32x2 v) {
  uint16_t* dst = a.tiled ? a.out + a_off(t, head * DH + c, a.tp)
                          : a.out + ((size_t)t * a.n_heads + head) * DH + c;
  *reinterpret_cast<u32x2*>(dst) = v;
}

// All but the newest N of this wavefront's loads have landed and its LDS reads are in
// registers; with two wavefronts per key stream the workgroup then meets, so that both halves
// of what the stream shares have landed and what both have read may be overwritten.
template <int N, bool MEET>
__device__ __forceinline__ void attn_wait() {
  if constexpr (MEET) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
  else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// NTW query tiles x KS key streams of wavefronts.  AF_RING: a stream's blocks come through a ring of
// D blocks in LDS; AF_ONCE: at most D of them, all at once; all operands start at multiples of 16
// bytes.  AF_REGISTERS: every wavefront loads
// its blocks into registers by itself, the next K while this block's softmax and P*V run and the
// next V behind them, and never meets the others before the merge; operands may start anywhere.
// SELF: one sequence and no prologue launch: every workgroup checks the sequence and works the
// ancestor bits out for itself (pointer doubling on the lanes of each wavefront), which saves a
// launch of 5 to 6 us.  The parents are asked for first and the bits worked out only by streams
// that come to the tree (see own_bits).
// The arguments in front of the struct come in scalar registers when a wavefront starts (build.py's kernarg
// preload): what the chain of first loads begins with.  SELF: node_off, kv_off, prefix_len, parent; else
// items, n_items.  us of a call, 512 x 16 10.9 -> 10.5, 3001 x 69 on 8 K/V heads 20.0 -> 19.3, 8192 x 64 35.4
// -> 35.0.
template <int DH, int NTW, int KS, int D, AttnForm FORM, bool SELF>
__global__ __launch_bounds__(KS* NTW * 64, 2) void tree_attn_bf16_kernel(
    const int32_t* first0, const int32_t* first1, const int32_t* first2, const int32_t* first3, int group,
    int n_kv_groups, int columns, int qg_max, AttnArgs rest) {
  AttnArgs a = rest;
  if constexpr (SELF) {
    a.node_off = first0;
    a.kv_off = first1;
    a.prefix_len = first2;
    a.parent = first3;
  } else {
    a.items = first0;
    a.n_items = first1;
  }
  a.group = group;
  a.n_kv_groups = n_kv_groups;
  a.columns = columns;
  a.qg_max = qg_max;
  constexpr int KSTEPS = DH / 16, MTV = DH / 32, SLOTS = 2 * D;
  constexpr int OW = MTV * 16 * 64;     // floats of one wavefront's O tile
  constexpr int HALF = KSTEPS;          // 1-KiB pieces of a block's K, and of its V
  constexpr int HP = HALF / NTW;        // of these, requested by one wavefront
  constexpr int SLOT = HALF * 1024;     // bytes of a ring slot
  constexpr bool MEET = NTW > 1;
  static_assert(D == 2 || D == 3, "the tail below");
  extern __shared__ __align__(16) uint8_t smem[];  // rings: KS x SLOTS slots; then the parts handed over
  __shared__ float sm_m[KS * NTW][32], sm_l[KS * NTW][32];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = wv % NTW, ks = wv / NTW;
  // Workgroup ids go round-robin over the 8 dies (XCDs), each with its own L2.  The
  // workgroups that walk the SAME K/V blocks (with grouped-query attention the query heads
  // of a K/V head) get ids that fall on one die, next to each other in its dispatch order,
  // so that the blocks come from HBM once; the query groups of one (sequence, split) are
  // neighbours in the item list, which puts them n_kv ids apart on the same die whenever
  // the number of K/V heads is a multiple of 8.
  const int slot = blockIdx.x >> 3, kvg = (slot / a.group) * 8 + (blockIdx.x & 7);
  if (kvg >= a.n_kv_groups) return;  // padding to a multiple of 8 (uniform)
  const int n_kv = a.columns / a.group;
  const int column = (kvg % n_kv) * a.group + slot % a.group;
  const int item = kvg / n_kv;
  int s, qg, r0, n, L, blk_base, sp;
  bool whole = false;  // no splits, whatever the plan
  bool several;  // another query group or sequence reads the same blocks
  const int head0 = column << a.pack;  // the column's first head
  auto zero_rows = [&](int t0, int t1) {  // rows without a valid sequence read as zeros (this column's part)
    const u32x2 z = {0, 0};
    const int quads = (DH / 4) << a.pack;  // of a row; columns of neighbouring heads follow each other
    for (int i = tid; i < (t1 - t0) * quads; i += KS * NTW * 64)
      attn_store_row<DH>(a, t0 + i / quads, head0, i % quads * 4, z);
  };
  if constexpr (SELF) {
    s = 0;
    qg = item % a.qg_max;
    sp = item / a.qg_max;
    r0 = a.node_off[0];
    const int r1 = a.node_off[1], ko = a.kv_off[0];
    L = a.prefix_len[0];
    n = r1 - r0;
    const bool range_ok = r0 >= 0 && r1 <= a.T && n > 0 && n <= TRJ_N_MAX;
    const bool ok = range_ok && !(ko < 0 || (ko & (TRJ_KV_BLOCK - 1)) || L < 0 || (long)ko + L + n > (long)a.s_pool ||
                                  (long)L + n > (long)a.max_seq_slots);
    if (qg == 0 && sp == 0) {  // rows that the sequence does not own, for all its workgroups of this head
      zero_rows(0, ok ? r0 : a.T);
      if (ok) zero_rows(r1, a.T);
      if (!ok && column == 0 && tid == 0) a.status[0] = 1;
    }
    if (!ok) return;  // uniform over the launch
    blk_base = ko >> 5;
    several = n << a.pack > 32 * NTW;
  } else {
    const int32_t* rec = a.items + (size_t)item * 8;  // inside the list's memory for every id
    s = rec[0], qg = rec[1], r0 = rec[2], n = rec[3], L = rec[4], blk_base = rec[5], sp = rec[6];
    several = rec[7] != 0;
    if constexpr (FORM != AF_ONCE) whole = a.pack > 0 && a.n_items[1] != 0;  // (at once: never)
    if (item >= a.n_items[0]) return;  // uniform over the workgroup, before any barrier
  }
  const int total = L + n;
  const int nb = (total + 31) >> 5;
  const int bpwg = whole ? nb : a.bpwg;
  const int nsplit = (nb + bpwg - 1) / bpwg;
  const int nq = n << a.pack;  // queries of the column
  if (sp >= nsplit || qg * 32 * NTW >= nq) return;  // uniform as well
  const int b0 = sp * bpwg, b1 = min(nb, b0 + bpwg);
  const int n32 = lane & 31, hh = lane >> 5;
  // no other workgroup reads these blocks (one query group, no sequence with the same slots, one
  // query head per K/V head): the loads carry the streaming hint; with a second reader through
  // L2 it costs a second trip to HBM
  const bool stream = a.group == 1 && !several;

  const size_t plane = (size_t)(column / a.group) * a.s_pool * DH;  // the K/V head
  // this stream's blocks: b0 + ks, b0 + ks + KS, ..
  const int nblk = b0 + ks < b1 ? (b1 - b0 - ks + KS - 1) / KS : 0;
  // queries past the last read the last one instead (never stored, always finite) and see no
  // tree node; a wavefront without any query computes nothing
  const int qi = (qg * NTW + nt) * 32 + n32, qc = min(qi, nq - 1);
  const int node = qc >> a.pack, head = head0 + (qc & ((1 << a.pack) - 1));
  const bool live = (qg * NTW + nt) * 32 < nq;

  f32x16 o[MTV];
#pragma unroll
  for (int mt = 0; mt < MTV; ++mt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[mt][v] = 0.f;
  float top = NEG_BIG, m = NEG_BIG, l = 0.f;
  bf16x8 qreg[KSTEPS];
  u32x4 kreg[KSTEPS], vreg[2 * MTV];  // 1-KiB pieces of a block; V piece mt * 2 + kg
  uint64_t anc0, anc1;
  auto scores = [&]() {
    f32x16 sacc;
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[v] = 0.f;
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k)
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kreg[k]), qreg[k], sacc, 0, 0, 0);
    return sacc;
  };
  auto softmax = [&](const f32x16& sacc, int key0, float& alpha, u32x4 (&pk)[2]) {
    if (key0 + 32 > L)  // uniform
      softmax_tile_tree(sacc, key0, hh, L, anc0, anc1, a.scale_log2e, a.lag, top, m, l, alpha, pk);
    else
      softmax_tile_prefix(sacc, a.scale_log2e, a.lag, top, m, l, alpha, pk);
  };
  auto add_values = [&](int key0, float alpha, const u32x4 (&pk)[2]) {
    if (key0 + 32 > total) {
      // slots past the sequence's last row may hold anything (NaN bit patterns too):
      // clear them in the V operand, their probabilities are exactly zero
#pragma unroll
      for (int kg = 0; kg < 2; ++kg)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          int key = key0 + 16 * kg + 4 * hh + 8 * (e >> 2) + (e & 3);
          if (key >= total) {
            uint32_t keep = (e & 1) ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
            for (int mt = 0; mt < MTV; ++mt) vreg[mt * 2 + kg][e >> 1] &= keep;
          }
        }
    }
    rescale_o<MTV>(o, alpha);
#pragma unroll
    for (int kg = 0; kg < 2; ++kg)
#pragma unroll
      for (int mt = 0; mt < MTV; ++mt)
        o[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vreg[mt * 2 + kg]),
                                                        __builtin_bit_cast(bf16x8, pk[kg]), o[mt], 0, 0, 0);
  };
  // SELF: the ancestor bits from the parents, par[h] = parent of node lane + 64 h (anything
  // from node n on); false if the tree is malformed (the same in every wavefront).  Only streams
  // that come to the tree's own slots need the bits, and trees of up to 64 nodes only half of the
  // work.  Parents behind the queries and all bits in every wavefront took, us of a call: 16 rows on
  // 512 slots 13.3 (now 12.1), 32 on 900 15.6 (14.5), 64 on 8192 36.7 (35.2).
  const bool meets_tree = nblk > 0 && (b0 + ks + (nblk - 1) * KS) * 32 + 32 > L;  // uniform
  auto bits_of = [&](const int (&par)[2], auto halves_c) {
    constexpr int HV = decltype(halves_c)::value, W = 2 * HV;  // nodes per lane, words of a row
    int jump[2], b[W][2];  // nearest ancestor whose bit is not in the row yet (255: none); the row's words
    auto value = [&](const int (&v)[2], int node) { return HV == 1 ? __shfl(v[0], node & 63) : from_node(v, node); };
#pragma unroll
    for (int h = 0; h < HV; ++h) {
      const int i = lane + 64 * h, p = i < n ? par[h] : -1;
      jump[h] = p < 0 ? 255 : p & 127;
#pragma unroll
      for (int w = 0; w < W; ++w) b[w][h] = i >> 5 == w ? (int)(1u << (i & 31)) : 0;
    }
    while (__ballot(jump[0] != 255 || (HV > 1 && jump[HV - 1] != 255))) {
      int u[W + 1][2];
#pragma unroll
      for (int h = 0; h < HV; ++h) {
        u[W][h] = value(jump, jump[h] & 127);
#pragma unroll
        for (int w = 0; w < W; ++w) u[w][h] = value(b[w], jump[h] & 127);
      }
#pragma unroll
      for (int h = 0; h < HV; ++h) {
        if (jump[h] == 255) continue;
#pragma unroll
        for (int w = 0; w < W; ++w) b[w][h] |= u[w][h];
        jump[h] = u[W][h];
      }
    }
    uint32_t r[4] = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int word = value(b[w], node);
      r[w] = qi < nq ? (uint32_t)word : 0u;
    }
    anc0 = (uint64_t)r[1] << 32 | r[0];
    anc1 = (uint64_t)r[3] << 32 | r[2];
  };
  auto own_bits = [&](const int (&par)[2]) -> bool {
    bool bad = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = lane + 64 * h;
      bad = bad || (i < n && (i == 0 ? par[h] != -1 : (par[h] < 0 || par[h] >= i)));
    }
    if (__ballot(bad)) return false;
    anc0 = anc1 = 0;
    if (!meets_tree) return true;
    if (n <= 64) bits_of(par, std::integral_constant<int, 1>{});
    else bits_of(par, std::integral_constant<int, 2>{});
    return true;
  };
  auto self_status = [&](bool ok) {  // the verdict on the tree, and zeros for its rows if it is malformed
    if (sp != 0) return;
    const int rows = 32 * NTW >> a.pack;
    if (!ok) zero_rows(r0 + qg * rows, min(r0 + n, r0 + (qg + 1) * rows));
    if (qg == 0 && column == 0 && tid == 0) a.status[0] = !ok;
  };

  if constexpr (FORM != AF_REGISTERS) {
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem;
    const uint32_t ring = __builtin_amdgcn_readfirstlane(lds0 + ks * SLOTS * SLOT);
    const u32x4* ring_r = reinterpret_cast<const u32x4*>(smem + (size_t)ks * SLOTS * SLOT + lane * 16);
    const int rounds = (b1 - b0 + KS - 1) / KS;
    const size_t first = (size_t)(blk_base + b0 + ks) * SLOT + nt * HP * 1024;
    const uint8_t* kp = reinterpret_cast<const uint8_t*>(a.k_layer + plane) + first;
    const uint8_t* vp = reinterpret_cast<const uint8_t*>(a.v_layer + plane) + first;
    auto request = [&](const uint8_t*& p, int sl) {  // this wavefront's pieces of the next K (or V) into slot sl
      const uint32_t dst = ring + sl * SLOT + nt * HP * 1024;
#pragma unroll
      for (int k = 0; k < HP; ++k) {
        if (stream) load_to_lds<true>(p + k * 1024, lane * 16, dst + k * 1024);
        else load_to_lds<false>(p + k * 1024, lane * 16, dst + k * 1024);
      }
      p += (size_t)KS * SLOT;
    };

    // The queries (as operands of the first product) and their ancestor bits come through LDS
    // too: registers that the compiler had loaded itself it would wait for together with the
    // whole ring.  The streams share them, each fetching its part of every tile.
    constexpr int QAT = KS * SLOTS * SLOT, ANC_AT = QAT + NTW * SLOT, QP = KSTEPS / KS;
    {
      auto fetch = [&](const void* base, uint32_t voff, int at) {
        load_to_lds<false>(base, voff, __builtin_amdgcn_readfirstlane(lds0 + at));
      };
      const uint16_t* qh = a.q + ((size_t)r0 * a.n_heads + head0) * DH;
#pragma unroll
      for (int j = 0; j < QP; ++j) {
        const int k = ks * QP + j;
        fetch(qh, (uint32_t)((node * a.n_heads + head - head0) * DH + hh * 8 + 16 * k) * 2, QAT + nt * SLOT + k * 1024);
      }
      if constexpr (SELF) {
        if (wv == 0) {
          load_words_to_lds(a.parent + r0, min(lane, n - 1) * 4, __builtin_amdgcn_readfirstlane(lds0 + ANC_AT));
          load_words_to_lds(a.parent + r0, min(lane + 64, n - 1) * 4, __builtin_amdgcn_readfirstlane(lds0 + ANC_AT + 256));
        }
      } else if (ks == 0) {
        fetch(a.anc + 2 * (size_t)r0, (uint32_t)node * 16, ANC_AT + nt * 1024);
      }
    }
    if constexpr (FORM == AF_RING) {
#pragma unroll
      for (int i = 0; i < D; ++i)
        if (i < nblk) {
          request(kp, 2 * i);
          request(vp, 2 * i + 1);
        }
    } else {  // all of the range (the plan keeps it to D blocks per stream), K first
#pragma unroll
      for (int i = 0; i < D; ++i)
        if (i < nblk) request(kp, 2 * i);
#pragma unroll
      for (int i = 0; i < D; ++i)
        if (i < nblk) request(vp, 2 * i + 1);
    }

    auto read = [&](u32x4 (&r)[KSTEPS], int sl) {
#pragma unroll
      for (int k = 0; k < KSTEPS; ++k) r[k] = ring_r[(sl * HALF + k) * 64];
    };
    // queries, bits and K of the first block: behind it its V and the blocks already requested (at
    // once: every K has landed, the V are on the way)
    if constexpr (FORM == AF_ONCE) {
      if (nblk >= 2) attn_wait<2 * HP, true>();
      else if (nblk == 1) attn_wait<HP, true>();
      else attn_wait<0, true>();
    } else if (nblk >= D) attn_wait<(2 * D - 1) * HP, true>();
    else if (D > 2 && nblk == 2) attn_wait<3 * HP, true>();
    else if (nblk == 1) attn_wait<HP, true>();
    else attn_wait<0, true>();
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k)
      qreg[k] = __builtin_bit_cast(bf16x8, reinterpret_cast<const u32x4*>(smem + QAT + nt * SLOT)[k * 64 + lane]);
    if constexpr (SELF) {
      const int32_t* words = reinterpret_cast<const int32_t*>(smem + ANC_AT);
      const int par[2] = {words[lane], words[lane + 64]};
      const bool ok = own_bits(par);
      if (!ok) attn_wait<0, true>();  // nothing may arrive after the end
      self_status(ok);
      if (!ok) return;
    } else {
      const u32x4 bits = reinterpret_cast<const u32x4*>(smem + ANC_AT + nt * 1024)[lane];
      anc0 = qi < nq ? (uint64_t)bits[1] << 32 | bits[0] : 0;
      anc1 = qi < nq ? (uint64_t)bits[3] << 32 | bits[2] : 0;
    }
    if constexpr (FORM == AF_ONCE) {
      // only one more meeting, for V, behind the first block's scores and softmax
      static_assert(D == 2, "waits above");
      const int key0 = (b0 + ks) * 32;
      float alpha;
      u32x4 pk[2];
      const bool some = live && nblk > 0;
      if (some) {
        read(kreg, 0);
        softmax(scores(), key0, alpha, pk);
      }
      attn_wait<0, true>();
      if (some) {
        read(vreg, 1);
        add_values(key0, alpha, pk);
      }
      if (live && nblk > 1) {
        read(kreg, 2);
        read(vreg, 3);
        softmax(scores(), key0 + KS * 32, alpha, pk);
        add_values(key0 + KS * 32, alpha, pk);
      }
    }
    // Block i of this stream: its K is in kreg; its V and the next blocks are on the way (slots
    // 2(i%D)+1, ..).  AHEAD: blocks behind it, D when there are at least as many; then block i+D
    // is requested into the slots that get free.  V is read under S^T and softmax, the next K
    // under P*V; at every wait 2(D-1) half blocks of the stream stay in flight.  A wavefront
    // without a row only requests and meets.
    int cur = 0;  // slot of this block's K
    auto block = [&](int i, auto ahead_c) {
      constexpr int AHEAD = decltype(ahead_c)::value;
      const int key0 = (b0 + ks + i * KS) * 32, next = cur + 2 == SLOTS ? 0 : cur + 2;
      f32x16 sacc;
      if (live) sacc = scores();
      attn_wait<(AHEAD < D ? 2 * AHEAD : 2 * (D - 1)) * HP, MEET>();
      if constexpr (AHEAD == D) request(kp, cur);
      float alpha;
      u32x4 pk[2];
      if (live) {
        read(vreg, cur + 1);
        softmax(sacc, key0, alpha, pk);
      }
      attn_wait<(AHEAD == 0 ? 0 : (AHEAD < D ? 2 * AHEAD - 1 : 2 * (D - 1))) * HP, MEET>();
      if constexpr (AHEAD == D) request(vp, cur + 1);
      cur = next;
      if (!live) return;
      if constexpr (AHEAD > 0) read(kreg, next);
      add_values(key0, alpha, pk);
    };
    if (FORM == AF_RING && nblk > 0) {
      read(kreg, 0);
      int i = 0;
      for (; i + D < nblk; ++i) block(i, std::integral_constant<int, D>{});
      if constexpr (D > 2) {
        if (nblk - 1 - i >= 2) block(i++, std::integral_constant<int, 2>{});
      }
      if (nblk - 1 - i >= 1) block(i++, std::integral_constant<int, 1>{});
      block(i, std::integral_constant<int, 0>{});
    }
    if (FORM == AF_RING && MEET && nblk < rounds) {  // a stream with a block less than the others meets them as often
      attn_wait<0, MEET>();
      attn_wait<0, MEET>();
    }
  } else {
    const u32x4* kb = reinterpret_cast<const u32x4*>(a.k_layer + plane) + (size_t)(blk_base + b0 + ks) * KSTEPS * 64 + lane;
    const u32x4* vb = reinterpret_cast<const u32x4*>(a.v_layer + plane) + (size_t)(blk_base + b0 + ks) * KSTEPS * 64 + lane;
    auto load = [&](u32x4 (&r)[KSTEPS], const u32x4*& p) {
#pragma unroll
      for (int k = 0; k < KSTEPS; ++k) {
        // the wavefronts of a stream load the same blocks: with the hint each from HBM again
        if (NTW == 1 && stream) r[k] = __builtin_nontemporal_load(p + k * 64);
        else r[k] = p[k * 64];
      }
      p += (size_t)KS * KSTEPS * 64;
    };
    const uint16_t* qp = a.q + ((size_t)(r0 + node) * a.n_heads + head) * DH + hh * 8;
    int par[2];
    if constexpr (SELF) {  // first: they are needed first
#pragma unroll
      for (int h = 0; h < 2; ++h) par[h] = a.parent[r0 + min(lane + 64 * h, n - 1)];
    }
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) qreg[k] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qp + 16 * k));
    if constexpr (!SELF) {
      anc0 = a.anc[2 * (size_t)(r0 + node)];
      anc1 = a.anc[2 * (size_t)(r0 + node) + 1];
    }
    const int mine = live ? nblk : 0;
    if (mine > 0) {
      load(kreg, kb);
      load(vreg, vb);
    }
    if constexpr (SELF) {
      const bool ok = own_bits(par);
      self_status(ok);
      if (!ok) return;
    } else if (qi >= nq) {
      anc0 = anc1 = 0;
    }
    // the last block has a copy of the code to itself: behind a condition the compiler would wait
    // for all loads wherever it waits for some
    auto block = [&](int i, auto more_c) {
      constexpr bool MORE = decltype(more_c)::value;
      const int key0 = (b0 + ks + i * KS) * 32;
      const f32x16 sacc = scores();
      if constexpr (MORE) load(kreg, kb);  // in flight during the softmax and P*V
      float alpha;
      u32x4 pk[2];
      softmax(sacc, key0, alpha, pk);
      add_values(key0, alpha, pk);
      if constexpr (MORE) load(vreg, vb);  // in flight during the next S^T and softmax
    };
    if (mine > 1) {
      // Once, for all loads.  The wait for the parents leaves the first V on the way; coming from
      // there the loop would wait for V wherever it waits for K, in every turn (heads of 64, 32 on 8
      // K/V heads, 16 rows on 32000 slots 39.6 against 30.2 us; of 128, 31 rows 49.6, 47.2).
      if constexpr (SELF) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      for (int i = 0; i + 1 < mine; ++i) block(i, std::true_type{});
    }
    if (mine > 0) block(mine - 1, std::false_type{});
  }

  // ---- merge the KS key streams of every query tile (fixed order, deterministic)
  const float lt = l + __shfl_xor(l, 32);
  if (hh == 0) {
    sm_m[wv][n32] = m;
    sm_l[wv][n32] = lt;
  }
  __syncthreads();  // the rings are free too
  float* red_all = reinterpret_cast<float*>(smem);
  float mg = NEG_BIG;
#pragma unroll
  for (int k = 0; k < KS; ++k) mg = fmaxf(mg, sm_m[nt + NTW * k][n32]);
  float lg = 0.f;
#pragma unroll
  for (int k = 0; k < KS; ++k) lg += sm_l[nt + NTW * k][n32] * exp2f(sm_m[nt + NTW * k][n32] - mg);
  {
    const float sc = exp2f(m - mg);
#pragma unroll
    for (int mt = 0; mt < MTV; ++mt)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[mt][v] *= sc;
  }
  // Every key stream keeps the 32-column parts of the output tile it owns (part mt belongs
  // to stream mt % KS) and hands the others over through LDS: one barrier, and the final
  // sums and stores are spread over all wavefronts.  The order of the sum is fixed
  // (own part first, then the other streams in ascending order): deterministic.
  constexpr int PART = 16 * 64;  // floats of one 32-column part of a wavefront's tile
#pragma unroll
  for (int mt = 0; mt < MTV; ++mt) {
    const int owner = mt % KS;
    if (ks != owner) {
      float* dst = red_all + (((nt * MTV + mt) * (KS - 1)) + (ks < owner ? ks : ks - 1)) * PART + lane;
#pragma unroll
      for (int v = 0; v < 16; ++v) dst[v * 64] = o[mt][v];
    }
  }
  __syncthreads();
  if (!live) return;  // no query, no partial; the barriers are behind
  const size_t pidx = ((size_t)(part_first(a.pack, a.tiles_per_seq, s, r0) + qg * NTW + nt) * a.columns + column) * a.nsplit_max + sp;
  if (nsplit != 1 && ks == 0 && hh == 0) {
    a.pm[pidx * 32 + n32] = mg;
    a.pl[pidx * 32 + n32] = lg;
  }
  const float inv = 1.0f / lg;
#pragma unroll
  for (int mt = 0; mt < MTV; ++mt) {
    if (ks != mt % KS) continue;
    const float* src = red_all + ((nt * MTV + mt) * (KS - 1)) * PART + lane;
#pragma unroll
    for (int k = 0; k < KS - 1; ++k)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[mt][v] += src[(k * 16 + v) * 64];
    if (nsplit == 1) {
      // the workgroup saw every key: write the normalised rows
      if (qi < nq) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          u32x2 v = {pack2bf(o[mt][4 * g] * inv, o[mt][4 * g + 1] * inv),
                     pack2bf(o[mt][4 * g + 2] * inv, o[mt][4 * g + 3] * inv)};
          attn_store_row<DH>(a, r0 + node, head, 32 * mt + 8 * g + 4 * hh, v);
        }
      }
    } else {
      // un-normalised partial (merged by attn_combine_kernel): the whole register tile,
      // rows that do not exist included (finite, never read back)
      float* img = a.po + pidx * OW + mt * PART + lane;
#pragma unroll
      for (int v = 0; v < 16; ++v) img[v * 64] = o[mt][v];
    }
  }
}


// Merge the partials of one (sequence, query tile, head) in split order.  512 threads: the
// thread (lane, mt, half) owns the 8 accumulator registers v = 8*half .. 8*half+7 of tile mt
// that lane `lane` of the attention wavefront held, i.e. query lane%32, 8 columns.  The loads
// of a batch of splits are all issued together (clamped, never predicated).
template <int DH, int CB>
__global__ __launch_bounds__(512) void attn_combine_kernel(const int32_t* status_dev, const int32_t* node_off,
                                                           const int32_t* prefix_len, int tiles_per_seq, int pack,
                                                           int columns, int nsplit_max, float* po, AttnArgs rest) {
  AttnArgs a = rest;
  a.status_dev = status_dev;
  a.node_off = node_off;
  a.prefix_len = prefix_len;
  a.tiles_per_seq = tiles_per_seq;
  a.pack = pack;
  a.columns = columns;
  a.nsplit_max = nsplit_max;
  a.po = po;
  constexpr int MTV = DH / 32, OW = MTV * 16 * 64;
  const int tile = blockIdx.x % a.tiles_per_seq, s = blockIdx.x / a.tiles_per_seq;
  const int column = blockIdx.y;
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int mt = grp >> 1, v0 = (grp & 1) * 8;
  if (mt >= MTV) return;
  const int n32 = lane & 31, hh = lane >> 5;
  // The first splits' partials are asked for together with what says how many there are: waiting
  // for one after the other was a third of this launch (4.2 -> 3.1 us for three splits of 16 rows).
  // Splits that do not exist are left out of maximum and sum, whatever their memory holds.
  const int status = a.status_dev[s], r0 = a.node_off[s], r1 = a.node_off[s + 1], L = a.prefix_len[s];
  const bool whole = a.pack > 0 && !a.parent && a.n_items[1] != 0;  // (a.parent: there is no list)
  // packed: the tile may have no place, and r0 of an invalid sequence be anything
  if (a.pack > 0 && s > 0 && (status != 0 || tile * 32 >= (r1 - r0) << a.pack)) return;
  const int there = a.pack > 0 && s == 0 ? min(tile, (a.T << a.pack) >> 5) : tile;
  const int place = part_first(a.pack, a.tiles_per_seq, s, r0) + there;
  const size_t base = ((size_t)place * a.columns + column) * a.nsplit_max;
  float ms[CB], ls[CB], x[CB][8];
  auto load = [&](int k0, int last) {
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const int k = min(k0 + j, last);
      ms[j] = a.pm[(base + k) * 32 + n32];
      ls[j] = a.pl[(base + k) * 32 + n32];
      const float* img = a.po + (base + k) * OW + (mt * 16 + v0) * 64 + lane;
#pragma unroll
      for (int e = 0; e < 8; ++e) x[j][e] = img[e * 64];
    }
  };
  load(0, a.nsplit_max - 1);
  const int n = r1 - r0, nq = n << a.pack;
  if (status != 0 || tile * 32 >= nq || whole) return;  // rows of malformed sequences stay zero
  const int nb = (L + n + 31) >> 5;
  const int nsplit = (nb + a.bpwg - 1) / a.bpwg;
  if (nsplit == 1) return;  // written by the attention kernel itself
  float mrun = NEG_BIG, lrun = 0.f;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int k0 = 0; k0 < nsplit; k0 += CB) {
    if (k0 > 0) load(k0, nsplit - 1);
#pragma unroll
    for (int j = 0; j < CB; ++j)
      if (k0 + j >= nsplit) {
        ms[j] = NEG_BIG;
        ls[j] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[j][e] = 0.f;
      }
    float mb = mrun;
#pragma unroll
    for (int j = 0; j < CB; ++j) mb = fmaxf(mb, ms[j]);
    const float resc = exp2f(mrun - mb);
    lrun *= resc;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= resc;
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const float wgt = exp2f(ms[j] - mb);
      lrun += wgt * ls[j];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += wgt * x[j][e];
    }
    mrun = mb;
  }
  const int qi = tile * 32 + n32;
  if (qi >= nq) return;
  const int node = qi >> a.pack, head = (column << a.pack) + (qi & ((1 << a.pack) - 1));
  const float inv = 1.0f / lrun;
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    u32x2 v = {pack2bf(acc[4 * g] * inv, acc[4 * g + 1] * inv),
               pack2bf(acc[4 * g + 2] * inv, acc[4 * g + 3] * inv)};
    attn_store_row<DH>(a, r0 + node, head, 32 * mt + 8 * ((v0 >> 2) + g) + 4 * hh, v);
  }
}

// Launch shape: form of the walk, query tiles per workgroup, query groups, blocks per workgroup,
// splits.  Figures: us of the attention kernel with its merge in a step of 12 layers, where K/V
// come from HBM, 32 heads of 128; R register form, 2r / 4r ring with two / four tiles.
AttnPlan attn_bf16_plan(int B, int rows_T, int all_heads, int dh, bool shared_kv, int max_seq_slots, int pack) {
  AttnPlan p;
  // queries and columns take the place of rows and heads
  const int T = rows_T << pack, n_heads = all_heads >> pack;
  const int nmax = (rows_T < TRJ_N_MAX ? rows_T : TRJ_N_MAX) << pack;
  int nb = (max_seq_slots + 31) / 32;
  if (nb < 1) nb = 1;
  // The ring pays where so many blocks stream from HBM that it matters how much is in flight
  // and that none is asked for twice: from 48 blocks of 32 heads (of 16 KiB each) for one query
  // tile, 96 for two and 128 for more, as blocks with more queries are worked on for longer
  // and four tiles then share them.  Query heads that share K/V find it
  // in L2, as do the chunks of a prompt (1000 tokens: ring 29.8, R 27.2), and halves of it
  // (heads of 64) arrive in time anyway.
  //   rows x slots        5x1024 5x2048 5x4096 33x2048 33x4096 97x1024 97x2048 97x4096
  //   blocks / limit        0.7   1.4    2.7     0.7     1.4     0.3     0.5     1.0
  //   ring                 12.7   15.5   20.3    18.0    22.6    20.2    24.6  4r 31.1
  //   R                    12.3   15.3   20.6    17.5    23.3    18.2    22.3    30.1
  // (69 rows on 4096: 4r 26.4, R 27.8; 128 with K/V of three inputs in turn: 4r 25.5, R 26.4.)
  // 16 packed sequences of 64 rows, up to 2048 slots: ring 69.6, R 85.7; four query heads per
  // K/V head, 97 rows on 4096 slots: ring 30.8, R 28.2, 16 sequences of 16 rows 72.1, 63.1.
  // Heads of 64 with one tile are the exception: two short blocks in flight from the start save
  // 1 us of a call at every length (16 heads, 512 slots: 11.4, 12.6).
  const int tiles = T > 64 * B ? 4 : T > 32 * B ? 2 : 1;  // on average: the sizes are device data
  const long pairs = (long)nb * B * n_heads, xchg = tune().attn_xchg_min_blocks;
  const long least = xchg > 1 ? 32 * xchg * (tiles == 4 ? 8 : 3 * tiles) / 3 : 0;
  p.ring = !shared_kv && (dh == 128 ? pairs >= least : nmax <= 32);
  // Query tiles per workgroup: one or two with four key streams; and four with two streams, so
  // that a tree of more than 64 rows needs no second pass over the sequence, where this fills
  // the chip evenly: one sequence's splits do, several sequences' ragged ones only down to two
  // (and with every tile full the two streams take longer than two workgroups), unsplit ones
  // from one and a half rounds on.  4r against 2r: 69 rows on 4096 slots 26.8, 28.7; four
  // sequences of 69 rows 40.7, 46.5, of 128 66.1, 61.8; two of 97 35.1, 33.4; three (three
  // quarters of the chip) of 128 44.3, 37.5; eight of 128 62.2, 57.3; twelve of 128 115, 135.
  p.ntw = nmax <= 32 ? 1 : 2;
  const long target = tune().attn_target_wgs;
  if (p.ring && tiles == 4) {
    const long cols = (long)B * n_heads, split = cols < target ? target / cols : 1;
    const bool even = split == 1 ? 2 * cols >= 3 * target
                                 : 8 * cols * split >= 7 * target && (B == 1 || (split == 2 && T <= 112 * B));
    if (even) p.ntw = 4;
  }
  // A sequence with more rows than a workgroup takes has several groups.
  p.qg_max = (nmax + 32 * p.ntw - 1) / (32 * p.ntw);
  // the host does not know the trees' sizes (they are device data): the number of work
  // items lies between max(B, T / rows per item) and B * qg_max; the lower figure sizes
  // the split (too few workgroups cost more than too many), the upper one the launch
  const int rows = 32 * p.ntw;
  const int items_est = B > (T + rows - 1) / rows ? B : (T + rows - 1) / rows;
  const long cols = (long)items_est * n_heads;
  int b;
  if (p.ntw == 4 || pack > 0) {  // whole rounds of workgroups at most
    const long split = cols < target ? target / cols : 1;
    b = (int)((nb + split - 1) / split);
  } else {
    b = (int)((nb * cols + target - 1) / target);
  }
  // shortest walk worth a workgroup, in blocks: one per key stream for 33..64 rows, two else
  // (64 rows on 1024 slots: 13.7 against 14.1 us; 128 rows on 1024 18.9 against 21.4)
  const int min_b = tune().attn_min_bpw > 0 ? tune().attn_min_bpw * (p.ntw == 4 ? 2 : 4)
                                            : (p.ntw == 4 || (p.ntw == 2 && nmax <= 64) ? 4 : 8);
  if (b < min_b) b = min_b;
  // one and four tiles have half the key streams that workgroups of eight wavefronts could have, and
  // packed heads fewer splits than single ones (20 rows on 8192 slots 2.11e-3 without
  // lag, 2.03e-3 with; single heads 2.03e-3)
  p.lag = p.ntw == 2 && pack == 0 ? 0.f : SOFTMAX_LAG;
  // up to 16 blocks (four per stream) the walk is shorter than the merge launch that a split
  // needs: 16 rows on 300 slots 11.9 against 13.6 us a call, 64 rows on 128 12.9 against 15.1,
  // on 512 (18 blocks) 17.2 against 15.9; with one query tile up to 24 (16 rows on 512 slots 11.9 split,
  // 11.0 whole, 600 12.1, 11.2, 8 on 700 12.7, 11.5, two sequences of 16 on 660 17.2, 15.4, 16 rows of 16
  // heads on 512 11.2, 10.5; heads of 64 that share K/V, 12 rows on 724 12.1, 9.4, four sequences of 7 on 655
  // 15.6, 12.8, 60 sizes 0.76 to 1.01 of the time; from 25 blocks on it turns, 5 on 777 11.2, 11.7).  Eight key streams instead
  // of four take longer in one workgroup (16 rows on 480 slots 10.4 -> 11.7)
  if (tune().attn_min_bpw == 0 && nb <= (p.ntw == 1 && pack == 0 && !p.ring ? 24 : 16) && b < nb) {
    b = nb;
    p.lag = SOFTMAX_LAG;
  }
  if (b > nb) b = nb;
  p.bpwg = b;
  p.nsplit_max = (nb + b - 1) / b;
  // Two tiles whose workgroup has at most two blocks per stream: all of it at once into LDS, where
  // both tiles read it and nobody waits for a block behind another, if the streams have equally many:
  // one each, or two.  Where some have two and some one, the meetings make them wait for each other,
  // in the last split too.  us of a call of 32 heads, registers -> at once, by blocks of a workgroup:
  // 3 (33 rows on 60 slots) 9.1 -> 9.0, 4 (64 on 60) 10.5 -> 9.4, 5 (33 on 100) 9.3 -> 11.2, 6 (64 on
  // 100, behind a prologue) 15.3 -> 16.1, 8 (128 on 100, the same) 18.2 -> 17.4.  Of splits: 4 (56 on
  // 850) 23.0 -> 22.5, 6 (33 on 1250) 17.9 -> 21.1, 8 (33 on 2000) 19.1 -> 21.0; with more rows registers
  // cost more, as every tile's wavefronts load the blocks for themselves: 8, 8, 8 and 1 (96 on 700)
  // 22.8 -> 21.9, but 8, 8, 8 and 6 (on 850) 22.0 -> 23.1.  5 (64 rows) where the last has 2 to 4 and
  // units stay free for those that wait (224 workgroups, 1024 slots 18.3 -> 18.0; 256, 1072 to 1184 18.0
  // to 18.5 -> 18.3 to 20.6) or heads share K/V (1024: 17.7 -> 16.6).  One tile has nothing to share (16
  // rows on 512: 12.1 -> 12.8).
  const int last = nb - (p.nsplit_max - 1) * b;  // several sequences' are device data
  const bool fours = b <= 4 || (b == 8 && (p.nsplit_max == 1 || T > 64 * B) && (B > 1 || last <= 4 || last == 8));
  const bool fives = b == 5 && p.nsplit_max > 1 && last >= 2 && last <= 4 && (shared_kv || 8 * cols * p.nsplit_max <= 7 * target);
  p.once = dh == 128 && p.ntw == 2 && !p.ring && (fours || fives);
  // not for packed heads of several sequences, which may have to be walked whole (attn_parts.h); there
  // the form gained 1.3 % with more than 64 queries and lost 2.5 % with up to 32
  p.once = p.once && (pack == 0 || B == 1);
  return p;
}

// Beyond 16 blocks, where a group of 2, 4 or 8 heads fills tiles of 32 queries that a tree by itself
// leaves partly empty (69 rows, four heads: 9 tiles instead of 12): the packing with the fewest tiles for
// trees of the average size, of those that pay.  Up to 16 blocks a call is the latency of one workgroup
// (30 rows on 300 slots: 10.5 against 13.1 us packed).  What pays, us of a call of 32 heads of 128 on
// 8 K/V heads, single -> packed, K/V from HBM, from 2004 sizes with all packings each:
//  - trees of up to 32 rows whose packed queries are one tile too, while workgroups stay as they
//    are (5 rows on 12000 slots 25.7 -> 19.6; sixteen sequences of 16 up to 520 28.2 -> 20.1).  Not
//    where only the packed ones need splits and their merge launch (eight of 16 up to 520: 17.6 ->
//    27.4) or an idle second tile (two of 9 up to 700: 14.3 -> 16.4), unless the launch needs fewer
//    rounds of workgroups (32 of 1 up to 520: 36.0 -> 26.3) or the walk is long (eight of 5 up to 3000:
//    36.4 -> 27.5).  Up to 24 blocks, where single heads of
//    one tile are not split, only for fewer rounds (5 rows on 520: 9.8 packed, 9.5 single; four sequences
//    of 5 up to 600 18.2 packed in splits, 14.6);
//  - one tile packed into two is twice the work per block (20 rows on 1000: 13.2 -> 15.3): only for
//    half of the rounds (sixteen of 20 up to 520: 29.0 -> 22.0; not sixteen up to 3000, two rounds of far
//    walks: 52.4 -> 57.1; 26 of 17 on four K/V heads 80.0 -> 56.3) or splits of 24 blocks and more (20
//    on 12000: 25.8 -> 23.3);
//  - more rows: one sequence (69 on 4000: 24.5 -> 21.5), but not 33 to 64 rows of eight heads per K/V
//    head, which L2 feeds, on less than 128 blocks (33 on 1000: 15.5 -> 16.2); several where the
//    rounds get fewer (four of 69 up to 1000: 38.7 -> 23.7; eight of 33 up to 520, as many: 19.1 -> 19.8).
// Heads of 64 have half the bytes per block, so there is less to save: one-tile packings only on long
// walks (two sequences of 1 up to 520 11.2 -> 12.2; 5 rows on 12000 17.3 -> 14.1) and nothing below 32 heads in all (16 on 4
// K/V heads, 5 rows on 12000: 14.4 -> 16.7) but for fewer rounds (32 of 5 up to 1000 42.6 -> 23.9).
int attn_bf16_pack(int B, int T, int n_heads, int n_kv_heads, int dh, int max_seq_slots, bool common_kv) {
  const int share = n_heads / n_kv_heads;
  if (const int forced = tune().attn_pack) return forced <= 4 && share % (1 << (forced - 1)) == 0 ? forced - 1 : 0;
  if (max_seq_slots <= 16 * 32) return 0;
  const int n = (T + B - 1) / B, nb = (max_seq_slots + 31) / 32;
  const bool walks_far = nb >= 64;
  constexpr int CUS = 256;
  struct Launch {
    AttnPlan p;
    int tiles;  // of a group of heads
    long wgs;   // with trees of equal size and length
  };
  auto launch = [&](int pack) {
    Launch l;
    l.p = attn_bf16_plan(B, T, n_heads, dh, common_kv || n_heads >> pack != n_kv_heads, max_seq_slots, pack);
    const int nq = n << pack, rows = 32 * l.p.ntw;
    l.tiles = (share >> pack) * ((nq + 31) / 32);
    l.wgs = (long)B * ((nq + rows - 1) / rows) * (n_heads >> pack) * l.p.nsplit_max;
    return l;
  };
  const Launch single = launch(0);
  const bool half = dh == 64, few = half && n_heads * B < 32;
  const long round = half && single.p.ntw == 1 ? 2 * CUS : CUS;  // two small workgroups share a compute unit
  int best = 0, fewest = single.tiles;
  for (int pack = 1; pack <= 3 && share % (1 << pack) == 0; ++pack) {
    const Launch l = launch(pack);
    if (l.tiles >= fewest) continue;
    const bool unsplit = l.p.nsplit_max == 1;
    const bool fewer_rounds = unsplit && single.wgs > round && 5 * l.wgs <= 4 * single.wgs;
    bool pays;
    if (n <= 32 && n << pack <= 32 && nb <= 24 && single.p.ntw == 1)
      pays = fewer_rounds;
    else if (n <= 32 && n << pack <= 32)
      pays = fewer_rounds || (walks_far && l.p.bpwg >= 24 && !few) ||
             (l.p.ntw == single.p.ntw && (unsplit || single.p.nsplit_max > 1) && (!half || (walks_far && !few)));
    else if (n <= 32)
      pays = (single.p.nsplit_max > 1 && l.p.bpwg >= 24 && !few) ||
             (fewer_rounds && 2 * l.wgs <= single.wgs && (!walks_far || single.wgs > 3 * CUS));
    else if (B == 1)
      pays = half ? share <= 4 && !few : share <= 4 || n > 64 || nb >= 128;
    else
      pays = unsplit ? fewer_rounds || (walks_far && l.wgs <= single.wgs)
                     : l.wgs <= CUS && single.wgs > CUS && !(half && walks_far);
    if (pays) { best = pack; fewest = l.tiles; }
  }
  return best;
}

// Loads without registers need operands on multiples of 16 bytes.  Several query groups of a sequence
// that the kernel checks itself find each other's blocks in the caches while the ancestor bits are
// worked out, which at once has to wait for (100 rows on 600 slots 17.0 against 19.8 us, 128 on 760
// 18.4, 18.2; behind a prologue, 96 rows on 500 in the step, at once is 1 us a layer ahead).
AttnForm attn_bf16_form(const AttnPlan& p, bool self, bool aligned) {
  if (!aligned) return AF_REGISTERS;
  if (p.ring) return AF_RING;
  return p.once && (p.qg_max == 1 || !self) ? AF_ONCE : AF_REGISTERS;
}

// scratch for either answer to "do query heads share K/V": the workspace queries do not know
size_t attn_bf16_ws_floats(int B, int T, int n_heads, int dh, int max_seq_slots, int pack) {
  size_t most = 64;  // no partials needed when every sequence fits one workgroup
  for (bool shared : {false, true}) {
    const AttnPlan p = attn_bf16_plan(B, T, n_heads, dh, shared, max_seq_slots, pack);
    const size_t n = p.nsplit_max > 1 ? part_tiles(B, T, pack, p.qg_max * p.ntw) * (n_heads >> pack) * p.nsplit_max * (dh / 32 * 1024 + 64) : 0;
    most = n > most ? n : most;
  }
  return most;
}
size_t attn_bf16_item_words(int B, int T, int n_heads, int dh, int max_seq_slots, int pack) {
  size_t most = 0;
  for (bool shared : {false, true}) {
    const AttnPlan p = attn_bf16_plan(B, T, n_heads, dh, shared, max_seq_slots, pack);
    const size_t n = (size_t)B * p.qg_max * p.nsplit_max * 8 + 8;
    most = n > most ? n : most;
  }
  return most;
}

int launch_tree_attn_bf16(const uint16_t* q, const uint16_t* k_layer, const uint16_t* v_layer,
                          const uint64_t* anc, const int32_t* node_off,
                          const int32_t* kv_off, const int32_t* prefix_len,
                          const int32_t* status_dev, const int32_t* items, int B, int T,
                          int n_heads, int n_kv_heads, bool shared_kv, int pack, int dh, int s_pool, int max_seq_slots,
                          float scale, float* ws, int tiled, int tp, uint16_t* out, const int32_t* parent,
                          int32_t* status, hipStream_t st) {
  if (dh != 64 && dh != 128) return TRJ_ERR_BAD_SHAPE;
  const AttnPlan p = attn_bf16_plan(B, T, n_heads, dh, shared_kv, max_seq_slots, pack);
  const int columns = n_heads >> pack, group = columns / n_kv_heads;
  const int ntw = p.ntw, qg_max = p.qg_max, bpwg = p.bpwg, nsplit_max = p.nsplit_max;
  const int tiles_per_seq = qg_max * ntw;
  size_t parts = nsplit_max > 1 ? part_tiles(B, T, pack, tiles_per_seq) * columns * nsplit_max : 0;
  float* po = ws;
  float* pm = ws + parts * (dh / 32 * 1024);
  float* pl = pm + parts * 32;
  AttnArgs a{q, k_layer, v_layer, anc, node_off, kv_off, prefix_len, status_dev, n_heads, s_pool, bpwg, nsplit_max, qg_max,
             pack, columns, group, B * qg_max * nsplit_max * n_kv_heads, items,
             items + (size_t)B * qg_max * nsplit_max * 8, scale * 1.4426950408889634f, p.lag, po, pm, pl, tiles_per_seq, out, tiled, tp,
             parent, status, T, max_seq_slots};
  if (parent && (B != 1 || tiled)) return TRJ_ERR_BAD_SHAPE;
  dim3 grid((B * qg_max * n_kv_heads * nsplit_max + 7) / 8 * 8 * group);
  {
    ProfScope ps_(KC_ATTN, st);
    const bool aligned = (((uintptr_t)q | (uintptr_t)k_layer | (uintptr_t)v_layer | (uintptr_t)anc) & 15) == 0;
    const AttnForm form = attn_bf16_form(p, parent != nullptr, aligned);
    const bool ring = form == AF_RING, once = form == AF_ONCE;
#define TRJ_ATTN_A(DH, Q, KS, D, FORM, SELF)                                                      \
  do {                                                                                          \
    constexpr size_t rings = (size_t)(KS * 2 * D + Q) * DH * 64 + Q * 1024;                     \
    constexpr size_t handed = (size_t)Q * DH * (KS - 1) * 128;                                  \
    constexpr size_t lds = FORM != AF_REGISTERS && rings > handed ? rings : handed;                                     \
    auto kern = tree_attn_bf16_kernel<DH, Q, KS, D, FORM, SELF>;                                  \
    static DeviceOnce once; /* per instantiation */                                             \
    allow_lds(once, kern, lds);                                                                 \
    if (SELF) kern<<<grid, KS * Q * 64, lds, st>>>(node_off, kv_off, prefix_len, parent, a.group, a.n_kv_groups, columns, qg_max, a); \
    else kern<<<grid, KS * Q * 64, lds, st>>>(a.items, a.n_items, nullptr, nullptr, a.group, a.n_kv_groups, columns, qg_max, a); \
  } while (0)
#define TRJ_ATTN(DH, Q, KS, D, FORM)                                                            \
  do {                                                                                          \
    if (parent) TRJ_ATTN_A(DH, Q, KS, D, FORM, true);                                           \
    else TRJ_ATTN_A(DH, Q, KS, D, FORM, false);                                                 \
  } while (0)
    if (dh == 128) {
      if (once) TRJ_ATTN(128, 2, 4, 2, AF_ONCE);
      else if (ring && ntw == 1) TRJ_ATTN(128, 1, 4, 2, AF_RING);
      else if (ring && ntw == 2) TRJ_ATTN(128, 2, 4, 2, AF_RING);
      else if (ring) TRJ_ATTN(128, 4, 2, 3, AF_RING);
      else if (ntw == 1) TRJ_ATTN(128, 1, 4, 2, AF_REGISTERS);
      else if (ntw == 2) TRJ_ATTN(128, 2, 4, 2, AF_REGISTERS);
      else TRJ_ATTN(128, 4, 2, 3, AF_REGISTERS);  // planned for the ring, operands off the grid
    } else {
      if (ring) TRJ_ATTN(64, 1, 4, 2, AF_RING);
      else if (ntw == 1) TRJ_ATTN(64, 1, 4, 2, AF_REGISTERS);
      else TRJ_ATTN(64, 2, 4, 2, AF_REGISTERS);
    }
#undef TRJ_ATTN
#undef TRJ_ATTN_A
  }
  int rc = check_launch();
  if (rc || nsplit_max == 1) return rc;
  ProfScope ps_(KC_ATTN_COMBINE, st);
  dim3 cgrid(B * tiles_per_seq, columns);
  if (dh == 128 && nsplit_max <= 4) attn_combine_kernel<128, 4><<<cgrid, 512, 0, st>>>(status_dev, node_off, prefix_len, tiles_per_seq, pack, columns, nsplit_max, po, a);
  else if (dh == 128) attn_combine_kernel<128, 8><<<cgrid, 512, 0, st>>>(status_dev, node_off, prefix_len, tiles_per_seq, pack, columns, nsplit_max, po, a);
  else if (nsplit_max <= 4) attn_combine_kernel<64, 4><<<cgrid, 512, 0, st>>>(status_dev, node_off, prefix_len, tiles_per_seq, pack, columns, nsplit_max, po, a);
  else attn_combine_kernel<64, 8><<<cgrid, 512, 0, st>>>(status_dev, node_off, prefix_len, tiles_per_seq, pack, columns, nsplit_max, po, a);
  return check_launch();
}

}  // namespace trj
