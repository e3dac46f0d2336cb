// Integer / byte kernels of the verify step: tree bookkeeping (depth, ancestor bit
// rows), greedy argmax, longest accepted path, KV compaction, and the layout
// converters.  All results here are exact (no floating point decides anything except
// the comparisons inside argmax).
#include "attn_parts.h"
#include "common.h"
#include "embed_row.h"
#include "kernels.h"

namespace trj {

// ------------------------------------------------------------------ tree bookkeeping
// One workgroup of TRJ_N_MAX threads per sequence.  A tree is well formed when
// parent[0] == -1 and 0 <= parent[i] < i; then walking parents strictly decreases the
// index, so every walk ends at the root.  When the KV arrays are given, the sequence's
// slot range must also lie inside the pool, start on a block boundary and hold at most
// max_seq_slots slots (the bound the host sized its launches and scratch with).  Rows of a
// malformed sequence get depth 0, empty bit rows and row_slot -1, which makes every
// later kernel skip them.
__global__ void fill_i32_kernel(int32_t* p, int32_t v, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ __launch_bounds__(TRJ_N_MAX) void tree_prep_kernel(
    const int32_t* __restrict__ parent, const int32_t* __restrict__ node_off,
    const int32_t* __restrict__ kv_off, const int32_t* __restrict__ prefix_len, int T, int s_pool,
    int max_seq_slots, int32_t* __restrict__ depth, uint64_t* __restrict__ anc, int32_t* __restrict__ status_dev,
    int32_t* __restrict__ row_slot, int32_t* __restrict__ row_pos, int32_t* __restrict__ row_seq) {
  __shared__ int32_t par[TRJ_N_MAX];
  __shared__ int32_t bad;
  const int s = blockIdx.x, i = threadIdx.x;
  int r0 = node_off[s], r1 = node_off[s + 1];
  // row range must lie inside [0, T] and hold 1..TRJ_N_MAX rows
  bool range_ok = r0 >= 0 && r1 <= T && r1 > r0 && (r1 - r0) <= TRJ_N_MAX;
  int n = range_ok ? r1 - r0 : 0;
  if (i == 0) {
    int b = range_ok ? 0 : 1;
    if (kv_off && range_ok) {
      int ko = kv_off[s], L = prefix_len[s];
      if (ko < 0 || (ko & (TRJ_KV_BLOCK - 1)) || L < 0 || (long)ko + L + n > (long)s_pool ||
          (long)L + n > (long)max_seq_slots)
        b = 1;
    }
    bad = b;
  }
  __syncthreads();
  if (i < n) {
    int p = parent[r0 + i];
    par[i] = p;
    if (i == 0 ? p != -1 : (p < 0 || p >= i)) atomicOr(&bad, 1);
  }
  __syncthreads();
  const int is_bad = bad;
  if (i == 0) status_dev[s] = is_bad;
  if (i >= n) return;  // nothing is written outside a valid row range
  uint64_t lo = 0, hi = 0;
  int d = 0;
  if (!is_bad) {
    d = -1;
    for (int j = i; j >= 0; j = par[j]) {
      if (j < 64) lo |= 1ull << j; else hi |= 1ull << (j - 64);
      ++d;
    }
  }
  depth[r0 + i] = d;
  anc[2 * (size_t)(r0 + i)] = lo;
  anc[2 * (size_t)(r0 + i) + 1] = hi;
  if (row_slot) {
    int L = prefix_len[s];
    row_slot[r0 + i] = is_bad ? -1 : kv_off[s] + L + i;
    row_pos[r0 + i] = is_bad ? 0 : L + d;
    row_seq[r0 + i] = is_bad ? -1 : s;
  }
}

// rows that no valid sequence covers must read as "skip": one launch clears all five arrays,
// and a further buffer of the caller's (the attention output, whose padding rows and rows of
// malformed sequences must read as zeros)
__global__ void prep_clear_kernel(int32_t* depth, int32_t* anc_words, int32_t* row_slot,
                                  int32_t* row_pos, int32_t* row_seq, int T, uint32_t* zero,
                                  size_t zero_words) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < zero_words) zero[i] = 0;
  if (i < (size_t)4 * T) anc_words[i] = 0;
  if (i < T) {
    depth[i] = 0;
    if (row_slot) {
      row_slot[i] = -1;
      row_pos[i] = 0;
      row_seq[i] = -1;
    }
  }
}

// One workgroup of 1024 threads builds the attention launch's item list.  Chunks of 1024
// sequences: thread i owns sequence base + i, counts its items (query groups x key splits
// of blocks_per_item 32-slot blocks; 0 when its status is not 0), and an inclusive scan
// over the chunk gives every sequence its place.  With one
// chunk (B <= 1024) the sequences are first ranked by length, longest first (ties by
// index), so that the long ones start early and the launch ends evenly.
// The last word of an item: another query group of the sequence, or another sequence (a prompt
// pass packs chunks of one prompt that share its slots; up to 1024 sequences are compared),
// reads the same blocks.
//
// Every sequence's place in the order longest first (ties by index) and whether another one's
// slots meet its own, from all lengths (-1: no valid sequence) and first slots in LDS, into two
// arrays in LDS.  Called by 1024 threads, which share the others that a sequence is compared
// with: by one thread per sequence 100 sequences took 9 to 15 us longer.
__device__ inline void compare_sequences(const int32_t* len, const int32_t* first, int B, int32_t* place, int32_t* common) {
  int per = 64;
  while (per < B) per <<= 1;
  const int parts = 1024 / per, s = threadIdx.x / parts, part = threadIdx.x % parts;
  int before = 0, meets = 0;
  if (s < B) {
    const int l = len[s], f = first[s];
    for (int j = part; j < B; j += parts) {
      const int ol = len[j], of = first[j];
      before += (ol > l) | ((ol == l) & (j < s));
      meets |= (j != s) & (ol > 0) & (l > 0) & (f < of + ol) & (of < f + l);
    }
  }
  for (int o = parts >> 1; o > 0; o >>= 1) {  // parts are neighbours in a wavefront, at most 16
    before += __shfl_xor(before, o);
    meets |= __shfl_xor(meets, o);
  }
  if (part == 0 && s < B) {
    place[s] = before;
    common[s] = meets;
  }
  __syncthreads();
}
__device__ inline void attn_items_body(
    const int32_t* __restrict__ node_off, const int32_t* __restrict__ prefix_len,
    const int32_t* __restrict__ kv_off, const int32_t* __restrict__ status, int B,
    int rows_per_item, int qg_max, int blocks_per_item, int nsplit_max,
    int32_t* __restrict__ items, int32_t* key, int32_t* cnt, int32_t* scan) {
  const int tid = threadIdx.x;
  __shared__ int32_t first[1024];
  int carry = 0;
  bool descends = false;
  for (int base = 0; base < B; base += 1024) {
    const int s = base + tid;
    descends |= s < B && range_descends(node_off, s);
    int n = 0, len = -1;
    if (s < B && status[s] == 0) {
      n = node_off[s + 1] - node_off[s];
      len = prefix_len[s] + n;
    }
    int ng = (n + rows_per_item - 1) / rows_per_item;
    if (ng > qg_max) ng = qg_max;
    int nsp = (((len + 31) >> 5) + blocks_per_item - 1) / blocks_per_item;
    if (nsp > nsplit_max) nsp = nsplit_max;
    const int nq = len < 0 ? 0 : ng * nsp;
    int place = tid;  // position of this sequence within the chunk
    bool common = false;
    if (B <= 1024) {
      const int slot0 = nq > 0 ? kv_off[s] : 0;
      key[tid] = len;
      first[tid] = slot0;
      __syncthreads();
      compare_sequences(key, first, B, cnt, scan);
      if (s < B) {
        place = cnt[tid];
        common = scan[tid] != 0;
      }
    }
    __syncthreads();
    if (s < B) cnt[place] = nq;
    else if (tid >= B - base) cnt[tid] = 0;
    __syncthreads();
    scan[tid] = cnt[tid];
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
      int v = tid >= d ? scan[tid - d] : 0;
      __syncthreads();
      scan[tid] += v;
      __syncthreads();
    }
    if (s < B) {
      const int at = carry + scan[place] - nq;
      for (int j = 0; j < nq; ++j) {  // the query groups of a split next to each other
        int32_t* rec = items + (size_t)(at + j) * 8;
        rec[0] = s;
        rec[1] = j % ng;
        rec[2] = node_off[s];
        rec[3] = n;
        rec[4] = len - n;
        rec[5] = kv_off[s] >> 5;
        rec[6] = j / ng;
        rec[7] = ng > 1 || common;
      }
    }
    carry += scan[1023];
    __syncthreads();
  }
  const int any = __syncthreads_or(descends);
  if (tid == 0) {
    items[(size_t)B * qg_max * nsplit_max * 8] = carry;
    items[(size_t)B * qg_max * nsplit_max * 8 + 1] = any;
  }
}

__global__ __launch_bounds__(1024) void attn_items_kernel(
    const int32_t* __restrict__ node_off, const int32_t* __restrict__ prefix_len,
    const int32_t* __restrict__ kv_off, const int32_t* __restrict__ status, int B,
    int rows_per_item, int qg_max, int blocks_per_item, int nsplit_max,
    int32_t* __restrict__ items) {
  __shared__ int32_t key[1024], cnt[1024], scan[1024];
  attn_items_body(node_off, prefix_len, kv_off, status, B, rows_per_item, qg_max, blocks_per_item,
                  nsplit_max, items, key, cnt, scan);
}

int launch_attn_items(const int32_t* node_off, const int32_t* prefix_len, const int32_t* kv_off,
                      const int32_t* status_dev, int B, int rows_per_item, int qg_max,
                      int blocks_per_item, int nsplit_max, int32_t* items, hipStream_t st) {
  if (qg_max < 1 || rows_per_item < 1 || blocks_per_item < 1 || nsplit_max < 1) return TRJ_ERR_BAD_SHAPE;
  attn_items_kernel<<<1, 1024, 0, st>>>(node_off, prefix_len, kv_off, status_dev, B, rows_per_item,
                                        qg_max, blocks_per_item, nsplit_max, items);
  return check_launch();
}

int launch_tree_prep(const int32_t* parent, const int32_t* node_off, const int32_t* kv_off,
                     const int32_t* prefix_len, int B, int T, int s_pool, int max_seq_slots,
                     int32_t* depth, uint64_t* anc, int32_t* status_dev, int32_t* row_slot, int32_t* row_pos,
                     int32_t* row_seq, void* zero, size_t zero_bytes, hipStream_t st) {
  const size_t zw = zero ? zero_bytes / 4 : 0, n = zw > (size_t)4 * T ? zw : (size_t)4 * T;
  prep_clear_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(
      depth, reinterpret_cast<int32_t*>(anc), row_slot, row_pos, row_seq, T,
      static_cast<uint32_t*>(zero), zw);
  tree_prep_kernel<<<B, TRJ_N_MAX, 0, st>>>(parent, node_off, kv_off, prefix_len, T, s_pool,
                                            max_seq_slots, depth, anc, status_dev, row_slot, row_pos, row_seq);
  return check_launch();
}

// ------------------------------------------------------------------ step prologue
// Everything a call needs before its first projection or attention launch, in ONE launch for
// up to PREP_MAX_SEQS sequences: the pieces depend on each other only through a sequence's
// tree, which is small enough (at most 128 parents) to be worked out again by every workgroup
// that needs it.  A launch of its own for each piece costs 2-5 us of dispatch and drain for
// next to no work: clear, tree checks, rotary table, work list and embedding together 19 us of
// a step, in one launch 7 us (5 rows).  Roles by workgroup id:
//   B * chunks   sequence s, rows 16c..: tree checks, depth and ancestor bits by pointer
//                doubling (7 rounds at most, where walking the parents of a 128-node chain
//                took 14 us); chunk 0 writes the tree's rows, every chunk the rotary table of
//                its rows (double precision sine and cosine, the longest part, hence chunks)
//   1            validity of all sequences, the attention work list, rows that no valid
//                sequence covers
//   tp - T       padding rows of the attention output
//   tp / rows    embedding and first norm input of embed_rows rows (bf16), or T: the embedding
//                of one row (fp32)
// Above PREP_MAX_SEQS the launches stay separate: the one workgroup that sees all sequences
// would take longer than they do.
__device__ inline void zero_row(const StepPrep& a, int t, int first, int stride) {
  if (!a.zero) return;
  if (a.zero_tp > 0) {
    const u32x4 z = {0, 0, 0, 0};
    for (int g = first; g < (a.zero_cols >> 3); g += stride)
      *reinterpret_cast<u32x4*>(a.zero + a_off(t, g * 8, a.zero_tp)) = z;
  } else {
    uint32_t* p = reinterpret_cast<uint32_t*>(a.zero + (size_t)t * a.zero_cols);
    for (int g = first; g < (a.zero_cols >> 1); g += stride) p[g] = 0;
  }
}
__device__ inline bool slots_ok(int ko, int L, int n, int s_pool, int max_seq_slots) {
  return !(ko < 0 || (ko & (TRJ_KV_BLOCK - 1)) || L < 0 || (long)ko + L + n > (long)s_pool ||
           (long)L + n > (long)max_seq_slots);
}

__device__ inline void prep_sequence(const StepPrep& a, int s, int chunk) {
  __shared__ int32_t jump[TRJ_N_MAX], dep[TRJ_N_MAX];
  __shared__ uint64_t lo[TRJ_N_MAX], hi[TRJ_N_MAX];
  __shared__ int32_t bad;
  const int i = threadIdx.x, r0 = a.node_off[s], r1 = a.node_off[s + 1];
  const bool range_ok = r0 >= 0 && r1 <= a.T && r1 > r0 && (r1 - r0) <= TRJ_N_MAX;
  if (!range_ok) {  // its rows are not its own to write: the workgroup that sees all rows does
    if (chunk == 0 && i == 0) a.status[s] = 1;
    return;
  }
  const int n = r1 - r0, row0 = chunk * PREP_CHUNK;
  if (row0 >= n) return;
  const int L = a.prefix_len[s], ko = a.kv_off[s];
  if (i == 0) bad = !slots_ok(ko, L, n, a.s_pool, a.max_seq_slots);
  __syncthreads();
  if (i < n) {
    const int p = a.parent[r0 + i];
    if (i == 0 ? p != -1 : (p < 0 || p >= i)) atomicOr(&bad, 1);
    jump[i] = p;  // nearest ancestor whose bit is not in the row yet, -1: none
    dep[i] = i > 0;
    lo[i] = i < 64 ? 1ull << i : 0;
    hi[i] = i < 64 ? 0 : 1ull << (i - 64);
  }
  __syncthreads();
  const int is_bad = bad;
  while (!is_bad) {  // parents precede their children, so every jump ends at the root
    int j = i < n ? jump[i] : -1, jj = -1, dj = 0;
    uint64_t l = 0, h = 0;
    if (j >= 0) { jj = jump[j]; dj = dep[j]; l = lo[j]; h = hi[j]; }
    if (!__syncthreads_or(j >= 0)) break;
    if (j >= 0) { jump[i] = jj; dep[i] += dj; lo[i] |= l; hi[i] |= h; }
    __syncthreads();
  }
  if (chunk == 0) {
    if (i == 0) a.status[s] = is_bad;
    if (i < n) {
      const int t = r0 + i;
      a.depth[t] = is_bad ? 0 : dep[i];
      a.anc[2 * (size_t)t] = is_bad ? 0 : lo[i];
      a.anc[2 * (size_t)t + 1] = is_bad ? 0 : hi[i];
      a.row_slot[t] = is_bad ? -1 : ko + L + i;
      a.row_pos[t] = is_bad ? 0 : L + dep[i];
      a.row_seq[t] = is_bad ? -1 : s;
    }
    if (is_bad)
      for (int t = r0; t < r1; ++t) zero_row(a, t, i, PREP_THREADS);
  }
  if (!a.cs) return;
  const int half = a.dh >> 1, rows = min(PREP_CHUNK, n - row0);
  for (int idx = i; idx < rows * half; idx += PREP_THREADS) {
    const int r = row0 + idx / half, j = idx % half;
    const double ang = (double)(is_bad ? 0 : L + dep[r]) * pow((double)a.theta, -2.0 * j / a.dh);
    a.cs[(size_t)(r0 + r) * half + j] = make_float2((float)cos(ang), (float)sin(ang));
  }
}

// The attention work list for up to PREP_MAX_SEQS sequences: the records of attn_items_body,
// one thread per record instead of one per sequence.  bad[s] (LDS or global): no record.
__device__ inline void few_items_body(const int32_t* node_off, const int32_t* prefix_len, const int32_t* kv_off,
                                      const int32_t* bad, int B, int rows_per_item, int qg_max,
                                      int blocks_per_item, int nsplit_max, int32_t* items) {
  __shared__ int32_t len[PREP_MAX_SEQS], first[PREP_MAX_SEQS], at[PREP_MAX_SEQS], shared[PREP_MAX_SEQS];
  __shared__ int32_t order[PREP_MAX_SEQS], groups[PREP_MAX_SEQS], end[PREP_MAX_SEQS];
  const int tid = threadIdx.x;
  int n = 0, l = -1, slot0 = 0;
  static_assert(PREP_MAX_SEQS == WAVE, "the vote");
  uint64_t descends = 0;  // sequences whose range does (asked for here: at the end it took 0.6 us of a call)
  if (tid < PREP_MAX_SEQS) {
    const int s = min(tid, B - 1), r0 = node_off[s], r1 = node_off[s + 1];
    if (tid < B && bad[tid] == 0) {
      n = r1 - r0;
      l = prefix_len[tid] + n;
      slot0 = kv_off[tid];
    }
    descends = __ballot(r1 < r0);
    len[tid] = l;
    first[tid] = slot0;
    order[tid] = tid;  // places past the last sequence: nothing
    groups[tid] = end[tid] = 0;
  }
  __syncthreads();
  compare_sequences(len, first, B, at, shared);
  if (tid < B) {
    const int place = at[tid];
    const int ng = min((n + rows_per_item - 1) / rows_per_item, qg_max);
    const int nsp = min((((l + 31) >> 5) + blocks_per_item - 1) / blocks_per_item, nsplit_max);
    order[place] = tid;
    groups[place] = ng;
    end[place] = l < 0 ? 0 : ng * nsp;
    if (ng > 1) shared[tid] = 1;
  }
  __syncthreads();
  if (tid < WAVE) {  // inclusive sum over the places by one wavefront
    int v = tid < PREP_MAX_SEQS ? end[tid] : 0;
    for (int d = 1; d < PREP_MAX_SEQS; d <<= 1) {
      const int u = __shfl_up(v, d);
      if (tid >= d) v += u;
    }
    if (tid < PREP_MAX_SEQS) end[tid] = v;
  }
  __syncthreads();
  const int total = end[PREP_MAX_SEQS - 1];
  for (int r = tid; r < total; r += blockDim.x) {
    int p = 0;
    while (end[p] <= r) ++p;
    const int s = order[p], ng = groups[p], j = r - (p ? end[p - 1] : 0);
    const int rows = node_off[s + 1] - node_off[s];
    int32_t* rec = items + (size_t)r * 8;
    rec[0] = s;
    rec[1] = j % ng;  // the query groups of a split next to each other
    rec[2] = node_off[s];
    rec[3] = rows;
    rec[4] = len[s] - rows;
    rec[5] = first[s] >> 5;
    rec[6] = j / ng;
    rec[7] = shared[s];
  }
  if (tid == 0) {
    items[(size_t)B * qg_max * nsplit_max * 8] = total;
    items[(size_t)B * qg_max * nsplit_max * 8 + 1] = descends != 0;
  }
}

__device__ inline void prep_all_sequences(const StepPrep& a) {
  __shared__ int32_t first[PREP_MAX_SEQS], last[PREP_MAX_SEQS], bad[PREP_MAX_SEQS];
  const int tid = threadIdx.x;
  if (tid < a.B) {
    const int r0 = a.node_off[tid], r1 = a.node_off[tid + 1];
    const bool ok = r0 >= 0 && r1 <= a.T && r1 > r0 && (r1 - r0) <= TRJ_N_MAX;
    first[tid] = r0;
    last[tid] = ok ? r1 : r0;  // an impossible range covers nothing
    bad[tid] = !ok || !slots_ok(a.kv_off[tid], a.prefix_len[tid], r1 - r0, a.s_pool, a.max_seq_slots);
  }
  __syncthreads();
  for (int t = tid; t < a.T; t += PREP_THREADS) {
    const int p = a.parent[t];
    bool covered = false;
    for (int s = 0; s < a.B; ++s) {
      const int i = t - first[s];
      if (i < 0 || t >= last[s]) continue;
      covered = true;
      if (i == 0 ? p != -1 : (p < 0 || p >= i)) atomicOr(&bad[s], 1);
    }
    if (covered) continue;
    a.depth[t] = 0;
    a.anc[2 * (size_t)t] = a.anc[2 * (size_t)t + 1] = 0;
    a.row_slot[t] = -1;
    a.row_pos[t] = 0;
    a.row_seq[t] = -1;
    zero_row(a, t, 0, 1);
  }
  __syncthreads();
  if (a.items)
    few_items_body(a.node_off, a.prefix_len, a.kv_off, bad, a.B, a.rows_per_item, a.qg_max, a.blocks_per_item,
                   a.nsplit_max, a.items);
}

__global__ __launch_bounds__(PREP_THREADS) void step_prep_kernel(StepPrep a, EmbedRow e, int chunks, int pad_rows) {
  int b = blockIdx.x;
  if (b < a.B * chunks) { prep_sequence(a, b / chunks, b % chunks); return; }
  b -= a.B * chunks;
  if (b == 0) { prep_all_sequences(a); return; }
  b -= 1;
  if (b < pad_rows) { zero_row(a, a.T + b, threadIdx.x, PREP_THREADS); return; }
  embed_row(e, b - pad_rows);
}

int launch_step_prep(const StepPrep& a, const EmbedRow& e, hipStream_t st) {
  const int chunks = a.cs ? ((a.T < TRJ_N_MAX ? a.T : TRJ_N_MAX) + PREP_CHUNK - 1) / PREP_CHUNK : 1;
  const int pad_rows = a.zero && a.zero_tp > 0 ? a.zero_tp - a.T : 0;
  step_prep_kernel<<<a.B * chunks + 1 + pad_rows + embed_blocks(e), PREP_THREADS, 0, st>>>(a, e, chunks, pad_rows);
  return check_launch();
}

// ------------------------------------------------------------------ static tree template
// The paper verifies with ONE fixed sparse tree in every step (appendix "Templates for
// Token Tree"), so everything that depends on the tree alone is computed once into a
// caller-owned buffer: validity, depth and ancestor bits of every row, the row -> sequence
// map, and the rotary table over positions 0..max_pos-1.  A step then needs one small
// kernel for what depends on the prefix lengths: slot range checks, slot and position of
// every row, the attention launch's work list, and the zero fill of the step's padding.
constexpr int32_t TMPL_MAGIC = 0x54724a54;

__global__ void tmpl_finish_kernel(const int32_t* __restrict__ node_off, int B, int T, int dh,
                                   int max_pos, const int32_t* __restrict__ tstatus,
                                   int32_t* __restrict__ hdr, int32_t* __restrict__ tnoff,
                                   int32_t* __restrict__ tseq) {
  // one workgroup per sequence; tseq was cleared to -1 before
  const int s = blockIdx.x, i = threadIdx.x;
  if (s == 0 && i == 0) {
    hdr[0] = TMPL_MAGIC; hdr[1] = B; hdr[2] = T; hdr[3] = dh; hdr[4] = max_pos;
    hdr[5] = hdr[6] = hdr[7] = 0;
    tnoff[B] = node_off[B];
  }
  if (i == 0) tnoff[s] = node_off[s];
  if (tstatus[s] != 0) return;  // a malformed sequence owns no rows
  const int r0 = node_off[s], n = node_off[s + 1] - r0;
  if (i < n) tseq[r0 + i] = s;
}

int launch_template_prepare(const int32_t* parent, const int32_t* node_off, int B, int T, int dh,
                            int max_pos, float theta, const TemplateView& v, hipStream_t st) {
  int rc = launch_tree_prep(parent, node_off, nullptr, nullptr, B, T, 0, 0, v.depth, v.anc, v.tstatus,
                            nullptr, nullptr, nullptr, nullptr, 0, st);
  if (rc != TRJ_OK) return rc;
  fill_i32_kernel<<<(T + 255) / 256, 256, 0, st>>>(v.tseq, -1, T);
  tmpl_finish_kernel<<<B, TRJ_N_MAX, 0, st>>>(node_off, B, T, dh, max_pos, v.tstatus, v.hdr, v.tnoff,
                                              v.tseq);
  rc = check_launch();
  if (rc != TRJ_OK) return rc;
  return launch_rope_table(nullptr, max_pos, dh, theta, v.cs, st);
}

__global__ __launch_bounds__(1024) void tmpl_step_prep_kernel(
    TemplateView v, const int32_t* __restrict__ node_off, const int32_t* __restrict__ kv_off,
    const int32_t* __restrict__ prefix_len, int B, int T, int dh, int max_pos, int s_pool,
    int max_seq_slots, int32_t* __restrict__ status_dev, int32_t* __restrict__ row_slot,
    int32_t* __restrict__ row_pos, int32_t* __restrict__ row_seq, int rows_per_item, int qg_max,
    int blocks_per_item, int nsplit_max, int32_t* __restrict__ items, uint32_t* __restrict__ zero,
    size_t zero_words, int zero_wgs, EmbedRow e) {
  const int tid = threadIdx.x;
  if (blockIdx.x > zero_wgs) {  // embedding and first norm input, embed_rows rows each
    embed_row(e, blockIdx.x - 1 - zero_wgs);
    return;
  }
  if (blockIdx.x > 0) {  // these clear the step's padding
    for (size_t i = (size_t)(blockIdx.x - 1) * 1024 + tid; i < zero_words; i += (size_t)zero_wgs * 1024)
      zero[i] = 0;
    return;
  }
  __shared__ int32_t key[1024], cnt[1024], scan[1024];
  __shared__ int32_t hdr_bad;
  if (tid == 0)
    hdr_bad = !(v.hdr[0] == TMPL_MAGIC && v.hdr[1] == B && v.hdr[2] == T && v.hdr[3] == dh &&
                v.hdr[4] == max_pos);
  __syncthreads();
  for (int s = tid; s < B; s += 1024) {
    // the step's row ranges must be the template's (which were validated when it was made)
    bool ok = !hdr_bad && v.tstatus[s] == 0 && node_off[s] == v.tnoff[s] &&
              node_off[s + 1] == v.tnoff[s + 1];
    if (ok) {
      const int n = v.tnoff[s + 1] - v.tnoff[s];
      const int ko = kv_off[s], L = prefix_len[s];
      if (ko < 0 || (ko & (TRJ_KV_BLOCK - 1)) || L < 0 || (long)ko + L + n > (long)s_pool ||
          (long)L + n > (long)max_seq_slots || (long)L + n > (long)max_pos)
        ok = false;
    }
    status_dev[s] = ok ? 0 : 1;
  }
  __threadfence_block();
  __syncthreads();
  for (int t = tid; t < T; t += 1024) {
    const int s = hdr_bad ? -1 : v.tseq[t];
    const bool bad = s < 0 || s >= B || status_dev[s] != 0;
    const int L = bad ? 0 : prefix_len[s];
    row_slot[t] = bad ? -1 : kv_off[s] + L + (t - v.tnoff[s]);
    row_pos[t] = bad ? 0 : L + v.depth[t];
    row_seq[t] = bad ? -1 : s;
  }
  if (items) {
    __syncthreads();
    if (B <= PREP_MAX_SEQS)
      few_items_body(node_off, prefix_len, kv_off, status_dev, B, rows_per_item, qg_max, blocks_per_item,
                     nsplit_max, items);
    else
      attn_items_body(node_off, prefix_len, kv_off, status_dev, B, rows_per_item, qg_max,
                      blocks_per_item, nsplit_max, items, key, cnt, scan);
  }
}

int launch_template_step_prep(const TemplateView& v, const int32_t* node_off, const int32_t* kv_off,
                              const int32_t* prefix_len, int B, int T, int dh, int max_pos, int s_pool,
                              int max_seq_slots, int32_t* status_dev, int32_t* row_slot,
                              int32_t* row_pos, int32_t* row_seq, int rows_per_item, int qg_max,
                              int blocks_per_item, int nsplit_max, int32_t* items, void* zero,
                              size_t zero_bytes, const EmbedRow& e, hipStream_t st) {
  const size_t zw = zero ? zero_bytes / 4 : 0;
  size_t zwgs = (zw + 16 * 1024 - 1) / (16 * 1024);  // 16 words per thread and pass
  if (zwgs > 512) zwgs = 512;
  tmpl_step_prep_kernel<<<(unsigned)(1 + zwgs + embed_blocks(e)), 1024, 0, st>>>(
      v, node_off, kv_off, prefix_len, B, T, dh, max_pos, s_pool, max_seq_slots, status_dev, row_slot,
      row_pos, row_seq, rows_per_item, qg_max, blocks_per_item, nsplit_max, items,
      static_cast<uint32_t*>(zero), zw, (int)zwgs, e);
  return check_launch();
}

// ------------------------------------------------------------------ greedy argmax
// One workgroup per row; lowest index wins ties; NaN never compares greater.
// One workgroup per row; every thread keeps ARGMAX_UNROLL 16-byte loads in flight (the row
// is read once, so the kernel is a latency chain unless the loads are batched: a row of 32000
// is one batch of eight, 64 such rows 7.0 -> 6.5 us in the kernel; accept_path with kv_compact,
// three launches, does not show it).
constexpr int ARGMAX_THREADS = 1024, ARGMAX_UNROLL = 8;
__device__ inline void amax_merge(float& bv, int& bi, float v, int i) {
  if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
}
__global__ __launch_bounds__(ARGMAX_THREADS) void argmax_kernel(const float* __restrict__ logits,
                                                                int V, int32_t* __restrict__ out) {
  const float* row = logits + (size_t)blockIdx.x * V;
  float bv = -INFINITY;
  int bi = INT32_MAX;
  const int tid = threadIdx.x;
  if ((V & 3) == 0 && (((uintptr_t)row) & 15) == 0) {
    const float4* r4 = reinterpret_cast<const float4*>(row);
    const int n4 = V >> 2;
    for (int i0 = tid; i0 < n4; i0 += ARGMAX_THREADS * ARGMAX_UNROLL) {
      float4 x[ARGMAX_UNROLL];
#pragma unroll
      for (int u = 0; u < ARGMAX_UNROLL; ++u) x[u] = r4[min(i0 + u * ARGMAX_THREADS, n4 - 1)];
#pragma unroll
      for (int u = 0; u < ARGMAX_UNROLL; ++u) {
        const int i = i0 + u * ARGMAX_THREADS;
        if (i < n4) {
          amax_merge(bv, bi, x[u].x, 4 * i);
          amax_merge(bv, bi, x[u].y, 4 * i + 1);
          amax_merge(bv, bi, x[u].z, 4 * i + 2);
          amax_merge(bv, bi, x[u].w, 4 * i + 3);
        }
      }
    }
  } else {
    for (int i = tid; i < V; i += ARGMAX_THREADS) amax_merge(bv, bi, row[i], i);
  }
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(bv, o);
    int oi = __shfl_xor(bi, o);
    amax_merge(bv, bi, ov, oi);
  }
  __shared__ float sv[ARGMAX_THREADS / WAVE];
  __shared__ int si[ARGMAX_THREADS / WAVE];
  if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; }
  __syncthreads();
  if (tid < ARGMAX_THREADS / WAVE) {
    bv = sv[tid];
    bi = si[tid];
    for (int o = ARGMAX_THREADS / WAVE / 2; o > 0; o >>= 1) amax_merge(bv, bi, __shfl_xor(bv, o), __shfl_xor(bi, o));
    if (tid == 0) out[blockIdx.x] = bi == INT32_MAX ? 0 : bi;
  }
}

int launch_argmax(const float* logits, int T, int V, int32_t* out, hipStream_t st) {
  argmax_kernel<<<T, ARGMAX_THREADS, 0, st>>>(logits, V, out);
  return check_launch();
}

// ------------------------------------------------------------------ accept
// ONE wavefront finds a sequence's longest accepted path, two nodes per lane (node = lane and
// lane + 64): node i is accepted when its token is the prediction at its parent and the parent
// is accepted (the root always is); best = max over accepted nodes of (depth, -index).  Depth
// and acceptance come by pointer doubling on registers passed between lanes, at most 7 rounds
// and no barrier (64 rows, the kernel alone: walking the parents in LDS 2.9 us, doubling in LDS
// with barriers 4.3, this 2.7; a 128-node chain takes 127 steps to walk).
struct Accepted {
  int depth, best, bonus;  // depth of the best node, -1 for a malformed sequence; uniform
  int path[2];             // nodes lane and lane + 64 of the path, root first; -1 behind its end
};
// what a sequence's nodes bring with them, nodes lane and lane + 64: asked for ahead of the predictions
// where these have still to be worked out
struct AcceptNodes {
  int r0, n, par[2], tk[2];
  bool bad;  // this lane's verdict
};
__device__ inline AcceptNodes accept_nodes(const int32_t* __restrict__ tok, const int32_t* __restrict__ parent,
                                           const int32_t* __restrict__ node_off, int T, int s) {
  const int lane = threadIdx.x & 63;
  const int r0 = node_off[s], r1 = node_off[s + 1];
  const bool range_ok = r0 >= 0 && r1 <= T && r1 > r0 && (r1 - r0) <= TRJ_N_MAX;
  AcceptNodes a{r0, range_ok ? r1 - r0 : 0, {-1, -1}, {0, 0}, !range_ok};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h;
    if (i >= a.n) continue;
    a.par[h] = parent[r0 + i];
    a.tk[h] = tok[r0 + i];
  }
  return a;
}
__device__ inline Accepted accept_sequence(const AcceptNodes& a, const int32_t* argmax, bool known_bad) {
  const int lane = threadIdx.x & 63, n = a.n;
  const int (&par)[2] = a.par, (&tk)[2] = a.tk;
  Accepted r{-1, -1, -1, {-1, -1}};
  int am[2];
  bool bad = a.bad || known_bad;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h;
    am[h] = i < n ? argmax[a.r0 + i] : 0;
    if (i < n) bad = bad || (i == 0 ? par[h] != -1 : (par[h] < 0 || par[h] >= i));
  }
  if (__ballot(bad)) return r;
  // one word per node: nearest ancestor not yet accounted for (255: none), distance to it,
  // and whether the nodes up to it (itself included, that one not) carry the right tokens
  int w[2];
  {
    int g[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) g[h] = from_node(am, max(par[h], 0));
#pragma unroll
    for (int h = 0; h < 2; ++h) w[h] = par[h] < 0 ? 255 | 1 << 16 : par[h] | 1 << 8 | (tk[h] == g[h]) << 16;
  }
  while (__ballot((w[0] & 255) != 255 || (w[1] & 255) != 255)) {
    int u[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) u[h] = from_node(w, w[h] & 127);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if ((w[h] & 255) != 255)
        w[h] = (u[h] & 255) | ((w[h] & 0xff00) + (u[h] & 0xff00)) | (w[h] & u[h] & 0x10000);
  }
  int key = -1;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h;
    if (i < n && (w[h] & 0x10000)) key = max(key, (w[h] & 0xff00) | (255 - i));
  }
  for (int o = 32; o > 0; o >>= 1) key = max(key, __shfl_xor(key, o));
  r.depth = key >> 8;  // the root is always accepted
  r.best = 255 - (key & 255);
  r.bonus = from_node(am, r.best);
  for (int j = r.best, k = r.depth; j >= 0; j = from_node(par, j), --k) {
    if (lane == k) r.path[0] = j;
    if (lane + 64 == k) r.path[1] = j;
  }
  return r;
}
__device__ inline void accept_store(const Accepted& r, int s, int32_t* accept_len, int32_t* best_node, int32_t* path,
                                    int32_t* bonus_tok) {
  const int lane = threadIdx.x & 63;
  path[(size_t)s * TRJ_N_MAX + lane] = r.path[0];
  path[(size_t)s * TRJ_N_MAX + 64 + lane] = r.path[1];
  if (lane == 0) {
    accept_len[s] = r.depth;
    best_node[s] = r.best;
    bonus_tok[s] = r.bonus;
  }
}

__global__ __launch_bounds__(WAVE) void accept_kernel(
    const int32_t* __restrict__ argmax, const int32_t* __restrict__ tok,
    const int32_t* __restrict__ parent, const int32_t* __restrict__ node_off, int T,
    int32_t* __restrict__ accept_len, int32_t* __restrict__ best_node, int32_t* __restrict__ path,
    int32_t* __restrict__ bonus_tok, int32_t* __restrict__ status_dev) {
  const int s = blockIdx.x;
  const Accepted r = accept_sequence(accept_nodes(tok, parent, node_off, T, s), argmax, false);
  accept_store(r, s, accept_len, best_node, path, bonus_tok);
  if (threadIdx.x == 0) status_dev[s] = r.depth < 0;
}

int launch_accept(const int32_t* argmax, const int32_t* tok, const int32_t* parent, const int32_t* node_off, int B,
                  int T, int32_t* accept_len, int32_t* best_node, int32_t* path, int32_t* bonus_tok,
                  int32_t* status_dev, hipStream_t st) {
  accept_kernel<<<B, WAVE, 0, st>>>(argmax, tok, parent, node_off, T, accept_len, best_node, path, bonus_tok,
                                    status_dev);
  return check_launch();
}

// ------------------------------------------------------------------ KV compaction
// One workgroup per (sequence, layer*head) plane; a thread owns head_dim columns.  Row j of
// the accepted path moves from slot base+path[j] to base+j.  path is increasing with
// path[j] >= j, so copying in increasing j never overwrites a row that is still to be read,
// and a thread reads and writes its own columns only: no barrier.  (Bound by the scattered
// reach over 2 x 1024 planes, not by the rows: eight rows requested together, or K rows as
// 16-byte pieces, took 7.3-7.8 us for a path of 6 in 32 x 32 planes, row by row 6.2.)
template <typename E>
__device__ __forceinline__ void compact_plane(E* __restrict__ kp, E* __restrict__ vp, const int32_t* pth, int a,
                                              int base, int dh, int s_pool) {
  for (int j = 0; j <= a && j < TRJ_N_MAX; ++j) {
    const int src = pth[j];
    if (src <= j || src >= TRJ_N_MAX || base + src >= s_pool) continue;  // uniform over the workgroup
    for (int c = threadIdx.x; c < dh; c += blockDim.x) {
      const E kk = kp[k_off(base + src, c, dh)];
      const E vv = vp[v_off(base + src, c, dh)];
      kp[k_off(base + j, c, dh)] = kk;
      vp[v_off(base + j, c, dh)] = vv;
    }
  }
}
template <typename E>
__global__ void kv_compact_kernel(E* __restrict__ k_pool, E* __restrict__ v_pool,
                                  size_t layer_stride, const int32_t* __restrict__ path,
                                  const int32_t* __restrict__ accept_len,
                                  const int32_t* __restrict__ kv_off,
                                  const int32_t* __restrict__ prefix_len, int n_heads, int dh,
                                  int s_pool, int32_t* __restrict__ new_len) {
  const int s = blockIdx.x, plane = blockIdx.y;
  const int a = accept_len[s];
  const int L = prefix_len[s], ko = kv_off[s];
  if (plane == 0 && threadIdx.x == 0) new_len[s] = a < 0 ? L : L + a + 1;
  if (a < 0 || L < 0 || ko < 0) return;
  const size_t off = (plane / n_heads) * layer_stride + (size_t)(plane % n_heads) * s_pool * dh;
  compact_plane(k_pool + off, v_pool + off, path + (size_t)s * TRJ_N_MAX, a, ko + L, dh, s_pool);
}

int launch_kv_compact(void* k_pool, void* v_pool, size_t layer_stride, const int32_t* path,
                      const int32_t* accept_len, const int32_t* kv_off, const int32_t* prefix_len,
                      int B, int n_layers, int n_heads, int dh, int s_pool, int dtype,
                      int32_t* new_len, hipStream_t st) {
  dim3 grid(B, n_layers * n_heads);
  int threads = dh < 64 ? 64 : (dh > 256 ? 256 : dh);
  if (dtype == TRJ_BF16)
    kv_compact_kernel<uint16_t><<<grid, threads, 0, st>>>((uint16_t*)k_pool, (uint16_t*)v_pool,
                                                          layer_stride, path, accept_len, kv_off,
                                                          prefix_len, n_heads, dh, s_pool, new_len);
  else
    kv_compact_kernel<uint32_t><<<grid, threads, 0, st>>>((uint32_t*)k_pool, (uint32_t*)v_pool,
                                                          layer_stride, path, accept_len, kv_off,
                                                          prefix_len, n_heads, dh, s_pool, new_len);
  return check_launch();
}

// picked[t] = the winner among row t's candidates, for T rows, by TRJ_N_MAX threads: equally many per row, up
// to a wavefront, each with PICK_LOADS candidates on the way at a time.  Lowest index wins ties, NaN never wins.
__device__ inline void pick_argmax(const ArgmaxCand* __restrict__ cand, int n_cand, int T, int32_t* picked) {
  const int per = pick_threads(T);
  const int t = threadIdx.x / per, j0 = threadIdx.x % per;
  float bv = -INFINITY;
  int bi = INT32_MAX;
  if (t < T) {
    const ArgmaxCand* row = cand + (size_t)t * n_cand;
    for (int j = j0; j < n_cand; j += PICK_LOADS * per) {
      ArgmaxCand c[PICK_LOADS];
#pragma unroll
      for (int u = 0; u < PICK_LOADS; ++u) c[u] = row[min(j + u * per, n_cand - 1)];  // the last again: changes nothing
#pragma unroll
      for (int u = 0; u < PICK_LOADS; ++u) amax_merge(bv, bi, c[u].v, c[u].i);
    }
  }
  for (int o = per >> 1; o > 0; o >>= 1) amax_merge(bv, bi, __shfl_xor(bv, o), __shfl_xor(bi, o));
  if (t < T && j0 == 0) picked[t] = bi == INT32_MAX ? 0 : bi;
}

// Acceptance and compaction of a step in one launch: every plane's workgroup works the path
// out for itself (three 512-byte reads and a few rounds on registers) instead of waiting for a launch
// that does only this; plane 0 writes it out.  Tail of a step 9.4 -> 5.0 us.
template <typename E>
__global__ __launch_bounds__(TRJ_N_MAX) void accept_compact_kernel(
    E* __restrict__ k_pool, E* __restrict__ v_pool, size_t layer_stride, const ArgmaxCand* __restrict__ cand, int n_cand,
    int32_t* argmax, const int32_t* __restrict__ tok, const int32_t* __restrict__ parent,
    const int32_t* __restrict__ node_off, const int32_t* __restrict__ kv_off, const int32_t* __restrict__ prefix_len,
    int32_t* status_dev, int T, int n_heads, int dh, int s_pool, int32_t* __restrict__ accept_len, int32_t* __restrict__ best_node,
    int32_t* __restrict__ path, int32_t* __restrict__ bonus_tok, int32_t* __restrict__ new_len) {
  __shared__ int32_t pth[TRJ_N_MAX];
  __shared__ int32_t depth;
  __shared__ int32_t picked[TRJ_N_MAX];
  const int s = blockIdx.x, plane = blockIdx.y;
  const int L = prefix_len[s], ko = kv_off[s];
  AcceptNodes nodes{};
  bool known_bad = false;
  if (threadIdx.x < WAVE) {
    // the prologue's verdict on tree and slots stands; what only parent[] shows (a prepared template
    // is not compared with it) is added.  Every plane reads the word while plane 0 may write it and
    // comes to the same end with either value.
    nodes = accept_nodes(tok, parent, node_off, T, s);
    known_bad = status_dev[s] != 0;
  }
  if (cand) {  // uniform; one sequence
    pick_argmax(cand, n_cand, T, picked);
    __syncthreads();
    if (plane == 0 && (int)threadIdx.x < T) argmax[threadIdx.x] = picked[threadIdx.x];
  }
  if (threadIdx.x < WAVE) {
    const Accepted r = cand ? accept_sequence(nodes, picked, known_bad) : accept_sequence(nodes, argmax, known_bad);
    if (plane == 0) {
      accept_store(r, s, accept_len, best_node, path, bonus_tok);
      if (threadIdx.x == 0) {
        new_len[s] = r.depth < 0 ? L : L + r.depth + 1;
        if (r.depth < 0) status_dev[s] = 1;
      }
    }
    pth[threadIdx.x] = r.path[0];
    pth[threadIdx.x + WAVE] = r.path[1];
    if (threadIdx.x == 0) depth = r.depth;
  }
  __syncthreads();
  const int d = depth;
  if (d < 0) return;  // the prologue checked kv_off and prefix_len of every sequence left
  const size_t off = (plane / n_heads) * layer_stride + (size_t)(plane % n_heads) * s_pool * dh;
  compact_plane(k_pool + off, v_pool + off, pth, d, ko + L, dh, s_pool);
}

int launch_accept_compact(void* k_pool, void* v_pool, size_t layer_stride, const ArgmaxCand* cand, int n_cand,
                          int32_t* argmax, const int32_t* tok,
                          const int32_t* parent, const int32_t* node_off, const int32_t* kv_off,
                          const int32_t* prefix_len, int32_t* status_dev, int B, int T, int n_layers,
                          int n_heads, int dh, int s_pool, int dtype, int32_t* accept_len, int32_t* best_node,
                          int32_t* path, int32_t* bonus_tok, int32_t* new_len, hipStream_t st) {
  dim3 grid(B, n_layers * n_heads);
  if (dtype == TRJ_BF16)
    accept_compact_kernel<uint16_t><<<grid, TRJ_N_MAX, 0, st>>>(
        (uint16_t*)k_pool, (uint16_t*)v_pool, layer_stride, cand, n_cand, argmax, tok, parent, node_off, kv_off, prefix_len,
        status_dev, T, n_heads, dh, s_pool, accept_len, best_node, path, bonus_tok, new_len);
  else
    accept_compact_kernel<uint32_t><<<grid, TRJ_N_MAX, 0, st>>>(
        (uint32_t*)k_pool, (uint32_t*)v_pool, layer_stride, cand, n_cand, argmax, tok, parent, node_off, kv_off, prefix_len,
        status_dev, T, n_heads, dh, s_pool, accept_len, best_node, path, bonus_tok, new_len);
  return check_launch();
}

// ------------------------------------------------------------------ layout converters
template <typename E, bool PACK>
__global__ void kv_convert_kernel(E* __restrict__ k_pool, E* __restrict__ v_pool,
                                  E* __restrict__ k_plain, E* __restrict__ v_plain, int dh,
                                  int s_pool, int slot0, int n_slots) {
  const int head = blockIdx.y;
  size_t total = (size_t)n_slots * dh;
  E* kp = k_pool + (size_t)head * s_pool * dh;
  E* vp = v_pool + (size_t)head * s_pool * dh;
  E* kl = k_plain + (size_t)head * n_slots * dh;
  E* vl = v_plain + (size_t)head * n_slots * dh;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    int sl = (int)(i / dh), c = (int)(i % dh);
    if (PACK) {
      kp[k_off(slot0 + sl, c, dh)] = kl[i];
      vp[v_off(slot0 + sl, c, dh)] = vl[i];
    } else {
      kl[i] = kp[k_off(slot0 + sl, c, dh)];
      vl[i] = vp[v_off(slot0 + sl, c, dh)];
    }
  }
}

int launch_kv_convert(void* k_pool, void* v_pool, void* k_plain, void* v_plain, int n_heads,
                      int dh, int s_pool, int slot0, int n_slots, int dtype, bool pack,
                      hipStream_t st) {
  if (n_slots == 0) return TRJ_OK;
  size_t total = (size_t)n_slots * dh;
  int bx = (int)((total + 255) / 256);
  if (bx > 1024) bx = 1024;
  dim3 grid(bx, n_heads);
#define TRJ_KVC(E, P)                                                                         \
  kv_convert_kernel<E, P><<<grid, 256, 0, st>>>((E*)k_pool, (E*)v_pool, (E*)k_plain,          \
                                                (E*)v_plain, dh, s_pool, slot0, n_slots)
  if (dtype == TRJ_BF16) {
    if (pack) TRJ_KVC(uint16_t, true); else TRJ_KVC(uint16_t, false);
  } else {
    if (pack) TRJ_KVC(uint32_t, true); else TRJ_KVC(uint32_t, false);
  }
#undef TRJ_KVC
  return check_launch();
}

// one thread per 8-element granule of the packed matrix
template <typename E>
__global__ void pack_weight_kernel(E* __restrict__ dst, const E* __restrict__ src, int n_out,
                                   int n_in, int kind, int n_heads, int dh) {
  size_t granules = (size_t)n_out * (n_in >> 3);
  for (size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x; g < granules;
       g += (size_t)gridDim.x * blockDim.x) {
    // granule g of the packed buffer: decode (tile row, k-step, half, row in tile)
    size_t tile = g >> 6;
    int lane = (int)(g & 63);
    int ksteps = n_in >> 4;
    int rt = (int)(tile / ksteps), ks = (int)(tile % ksteps);
    int r = rt * 32 + (lane & 31), k = ks * 16 + (lane >> 5) * 8;
    const E* s = src + (size_t)logical_row(r, kind, n_out, n_heads, dh) * n_in + k;
    E* d = dst + g * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = s[e];
  }
}

int launch_pack_weight(void* dst, const void* src, int n_out, int n_in, int dtype, int kind,
                       int n_heads, int dh, hipStream_t st) {
  size_t granules = (size_t)n_out * (n_in >> 3);
  int bx = (int)((granules + 255) / 256);
  if (bx > 65536) bx = 65536;
  if (dtype == TRJ_BF16)
    pack_weight_kernel<uint16_t><<<bx, 256, 0, st>>>((uint16_t*)dst, (const uint16_t*)src, n_out,
                                                     n_in, kind, n_heads, dh);
  else
    pack_weight_kernel<uint32_t><<<bx, 256, 0, st>>>((uint32_t*)dst, (const uint32_t*)src, n_out,
                                                     n_in, kind, n_heads, dh);
  return check_launch();
}

}  // namespace trj
