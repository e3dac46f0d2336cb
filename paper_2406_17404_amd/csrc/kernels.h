// Internal launcher declarations shared by the .hip files.  Every launcher only
// enqueues on the given stream and returns a trj_status.
#pragma once
#include "common.h"

namespace trj {

struct Tunables {
  int gemm_target_wgs = 256;   // split-k is raised until a GEMM has this many workgroups
  int max_split_k = 8;
  int gemm_cfg = 0;            // 0: choose the workgroup shape per GEMM; 1..6 force one
  int gemm_big_t = 256;        // padded token rows from which wavefronts own two row tiles (0: never)
  int gemm_pair_min_k = 4096;  // k range from which two groups of wavefronts may take turns (gemm_pair.h)
  int attn_target_wgs = 256;   // attention workgroups per launch aimed at (one per CU)
  int gemm_big_wt = 0;         // row tiles per wavefront of the many-rows kernel (2, 4; 0 = choose)
  int attn_xchg_min_blocks = 48;  // blocks of 32 heads from which K/V go through rings, one query tile (1: always)
  int attn_pack = 0;           // 0: choose; 1, 2, 3, 4: work on 1, 2, 4, 8 query heads of a K/V head together
  int attn_min_bpw = 0;        // 32-slot blocks per key stream, at least (0: chosen from the tree size)
};
// trj_set_tunable writes the process-wide set; every entry point copies it once on entry
// (TuneScope) and every launch plan of that call, on that thread, reads the copy, so the
// workspace a call carves and the launches it makes always come from the same values.
const Tunables& tune();
struct TuneScope {
  Tunables snap;
  const Tunables* prev;
  TuneScope();
  ~TuneScope();
};

// per-kernel timing hooks (api.hip): when kernel class `cls` is being profiled, a HIP
// event is recorded on the stream before and after the launch
enum KernelClass {
  KC_NONE = 0, KC_GEMM_QKV = 1, KC_ATTN = 2, KC_ATTN_COMBINE = 3, KC_GEMM_O = 4,
  KC_REDUCE_NORM = 5, KC_GEMM_GATE_UP = 6, KC_GEMM_DOWN = 7, KC_GEMM_LM = 8, KC_ARGMAX = 9,
  KC_ACCEPT = 10, KC_KV_COMPACT = 11, KC_SETUP = 12
};
void prof_begin(int cls, hipStream_t st);
void prof_end(int cls, hipStream_t st);
struct ProfScope {
  int cls;
  hipStream_t st;
  ProfScope(int c, hipStream_t s) : cls(c), st(s) { prof_begin(cls, st); }
  ~ProfScope() { prof_end(cls, st); }
};

// tree_kernels.hip
int launch_tree_prep(const int32_t* parent, const int32_t* node_off, const int32_t* kv_off,
                     const int32_t* prefix_len, int B, int T, int s_pool, int max_seq_slots,
                     int32_t* depth, uint64_t* anc, int32_t* status_dev, int32_t* row_slot, int32_t* row_pos,
                     int32_t* row_seq, void* zero, size_t zero_bytes, hipStream_t st);
// One launch for all of a call's bookkeeping (see step_prep_kernel), for up to PREP_MAX_SEQS
// sequences; kv_off and prefix_len are not null.  Optional parts: cs (rotary table [T][dh/2]),
// items (attention work list), zero (bf16 attention output whose rows without a valid sequence
// read as zeros: plain rows of zero_cols, or tiled with zero_tp rows, padding rows included),
// the embedding (EmbedRow::x).
constexpr int PREP_MAX_SEQS = 64, PREP_THREADS = 1024, PREP_CHUNK = 16;
struct StepPrep {
  const int32_t *parent, *node_off, *kv_off, *prefix_len;
  int B, T, s_pool, max_seq_slots;
  int32_t* depth;
  uint64_t* anc;
  int32_t *status, *row_slot, *row_pos, *row_seq;
  float2* cs;
  int dh;
  float theta;
  int32_t* items;
  int rows_per_item, qg_max, blocks_per_item, nsplit_max;
  uint16_t* zero;
  int zero_cols, zero_tp;
};
// x[t] = E[tok[t]] for T rows; with hp (bf16 mode) the first projection's input for tp rows
// too, see launch_reduce_norm.  x null: nothing.
struct EmbedRow {
  const void* embed;
  const int32_t* tok;
  int T, d, vocab;
  float* x;
  const float* g;
  int tp;
  uint16_t* hp;
  float* ssq;
  int parts, part_threads;
};
int launch_step_prep(const StepPrep& a, const EmbedRow& e, hipStream_t st);
// List of the (sequence, key split, query group) triples that exist, for the bf16 attention
// launch: n records of 8 words {sequence, group, first row, rows, prefix length,
// kv_off / 32, split, 1 if another group or sequence reads the same slots}, sequences ordered by length (prefix + tree), longest first, when
// B <= 1024 (else in index order); word 8 * B * qg_max * nsplit_max holds n.  Sequences
// whose status is not 0 are left out.  Must follow launch_tree_prep on the stream.
int launch_attn_items(const int32_t* node_off, const int32_t* prefix_len, const int32_t* kv_off,
                      const int32_t* status_dev, int B, int rows_per_item, int qg_max,
                      int blocks_per_item, int nsplit_max, int32_t* items, hipStream_t st);
// A prepared tree template (device pointers into the caller's buffer): what depends on the
// tree alone.  hdr: 8 words {magic, B, T, head_dim, max_pos}; tstatus[B]: 1 = malformed tree;
// tnoff[B+1]: the row ranges it was made for; tseq[T]: row -> sequence (-1: none);
// cs[max_pos][head_dim/2]: cos, sin of position * theta^(-2j/head_dim).
struct TemplateView {
  int32_t* hdr;
  int32_t* depth;
  uint64_t* anc;
  int32_t* tstatus;
  int32_t* tnoff;
  int32_t* tseq;
  float2* cs;
};
int launch_template_prepare(const int32_t* parent, const int32_t* node_off, int B, int T, int dh,
                            int max_pos, float theta, const TemplateView& v, hipStream_t st);
// Everything a step needs besides the template: slot checks (status_dev), slot / position /
// sequence of every row, the bf16 attention work list (items may be null), zero fill.
int launch_template_step_prep(const TemplateView& v, const int32_t* node_off, const int32_t* kv_off,
                              const int32_t* prefix_len, int B, int T, int dh, int max_pos, int s_pool,
                              int max_seq_slots, int32_t* status_dev, int32_t* row_slot,
                              int32_t* row_pos, int32_t* row_seq, int rows_per_item, int qg_max,
                              int blocks_per_item, int nsplit_max, int32_t* items, void* zero,
                              size_t zero_bytes, const EmbedRow& e, hipStream_t st);
// The largest of a tile of 32 logits and its index (INT32_MAX: no value that is a number), [row][n_out / 32].
struct ArgmaxCand {
  float v;
  int32_t i;
};
int launch_argmax(const float* logits, int T, int V, int32_t* out, hipStream_t st);
int launch_accept(const int32_t* argmax, const int32_t* tok, const int32_t* parent, const int32_t* node_off, int B,
                  int T, int32_t* accept_len, int32_t* best_node, int32_t* path, int32_t* bonus_tok,
                  int32_t* status_dev, hipStream_t st);
// One sequence with so few candidates (16 KiB) that the acceptance launch picks among them by itself, in every
// workgroup: a launch less for one or two rounds of loads, PICK_LOADS of each thread, one behind the other.
// From the LM head's launch to the end of acceptance, bf16, less than with a launch for the pick, us, in models
// of 8, 256 and 1024 layers x K/V heads (a workgroup each): one round (1 row of 512 candidates, 8 of 128) 1.0 to 1.6,
// two (1 of 1000, 4 of 512, 16 of 128, 31 of 64) 0.3 to 1.2 (128 rows of 16 1.7, 1.4, -0.4), three (1 of 1536, 3 of
// 682) -0.3 to 0.2, four (1 of 2048, 5 of 406, 17 of 120) -0.2 to -0.9 (65 of 31 0.7, 0.3, -0.3).  Steps of the
// tiny fp32 model (15 rows, 64 candidates each, one round) 62.0 -> 60.7.  fp32 has no other candidates, and an
// argmax that reads logits takes longer the longer a row is: up to four rows, whose candidates in three and
// four rounds are more than 512 each, the pick stays 1 to 3 us ahead (1 of 2048 3.0, 3 of 682 1.0; 5 of 406 -0.2,
// 17 of 120 -0.2).
constexpr int PICK_LOADS = 8;
// threads that pick among one row's candidates, a power of two, of one wavefront
__host__ __device__ inline int pick_threads(int T) {
  int per = WAVE;
  while (per * T > TRJ_N_MAX) per >>= 1;
  return per;
}
inline bool accept_picks(int B, int T, int vocab, bool fp32) {
  if (B != 1 || T > TRJ_N_MAX || (long)T * (vocab >> 5) > 2048) return false;
  return (vocab >> 5) <= 2 * PICK_LOADS * pick_threads(T) || (fp32 && T <= 4);
}
// both of a step; status_dev: as the prologue wrote it, 1 is added for a malformed parent[]; cand (may be
// null): argmax is not there yet and is written from these (accept_picks)
int launch_accept_compact(void* k_pool, void* v_pool, size_t layer_stride, const ArgmaxCand* cand, int n_cand,
                          int32_t* argmax, const int32_t* tok,
                          const int32_t* parent, const int32_t* node_off, const int32_t* kv_off,
                          const int32_t* prefix_len, int32_t* status_dev, int B, int T, int n_layers,
                          int n_heads, int dh, int s_pool, int dtype, int32_t* accept_len, int32_t* best_node,
                          int32_t* path, int32_t* bonus_tok, int32_t* new_len, hipStream_t st);
int launch_kv_compact(void* k_pool, void* v_pool, size_t layer_stride, const int32_t* path,
                      const int32_t* accept_len, const int32_t* kv_off, const int32_t* prefix_len,
                      int B, int n_layers, int n_heads, int dh, int s_pool, int dtype,
                      int32_t* new_len, hipStream_t st);
int launch_kv_convert(void* k_pool, void* v_pool, void* k_plain, void* v_plain, int n_heads,
                      int dh, int s_pool, int slot0, int n_slots, int dtype, bool pack,
                      hipStream_t st);
int launch_pack_weight(void* dst, const void* src, int n_out, int n_in, int dtype, int kind,
                       int n_heads, int dh, hipStream_t st);

// f32_kernels.hip
int launch_rope_table(const int32_t* row_pos, int T, int dh, float theta, float2* cs,
                      hipStream_t st);
int launch_embed(const float* embed, const int32_t* tok, int T, int d, int vocab, float* x, hipStream_t st);
// g: RMSNorm's gain, applied to x with its division (null: x as it is); add_to: y += instead of y =
int launch_gemm_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int n_out, int add_to,
                    float* y, hipStream_t st);
// logits y and candidates of their argmax, behind a norm
int launch_gemm_lm_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int n_out, float* y,
                       ArgmaxCand* cand, hipStream_t st);
int launch_gemm_gate_up_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int F,
                            float* act, hipStream_t st);
int launch_gemm_qkv_f32(const float* x, const float* g, float eps, const float* w, int T, int n_in, int n_heads,
                        int n_kv_heads, int dh, int s_pool, const float2* cs, const int32_t* cs_row,
                        const int32_t* row_slot, float* q, float* k_layer, float* v_layer, hipStream_t st);
int launch_tree_attn_f32(const float* q, const float* k_layer, const float* v_layer,
                         const uint64_t* anc, const int32_t* row_seq, const int32_t* node_off,
                         const int32_t* kv_off, const int32_t* prefix_len,
                         const int32_t* status_dev, int T, int n_heads, int n_kv_heads, int dh,
                         int s_pool, int max_slots, float scale, float* out, hipStream_t st);

// gemm_bf16.hip
// RMSNorm with the division deferred to the consumer: the producer of the activations
// writes bf16(x * g) (not yet divided by the row's norm) and, per row, partial sums of x^2
// over `parts` column parts; a projection of those activations multiplies its accumulators
// by 1 / sqrt(mean(x^2) + eps) of the token row before its epilogue.  (x*g*inv and (x*g)*inv
// round to bf16 with the same relative error, and the product with W is linear in inv.)
// The producer then needs no row-wide reduction and spreads over the whole chip.
constexpr int RS_MAX_PARTS = 4;
struct RowScale {
  const float* ssq;  // [parts][tp], more than RS_MAX_PARTS only for many rows; nullptr: activations are used as they are
  int parts, tp;
  float inv_d, eps;
  int fine;          // this many rows, sums as [row][parts], up to 256 parts (gemm_slim.hip); 0: as above
};
// A projection into the residual stream and the next norm's input in one launch, for few rows:
// x += xp w^T, hp = bf16(x * g) tiled (rows T .. 7 of 32 as zeros, the others are left alone), n_out / 16
// sums of squares per row, [row][part] (at 16-byte boundaries: RowScale::fine).
bool gemm_slim_runs(int T, int n_in, int n_out, const void* xp, const void* w);
int launch_gemm_slim(const uint16_t* xp, const uint16_t* w, int T, int n_in, int n_out, float* x, const float* g,
                     uint16_t* hp, float* ssq, hipStream_t st);
int reduce_norm_parts(int d);    // column parts of a row
int reduce_norm_threads(int d);  // threads per part, 8 columns each, in whole wavefronts
int gemm_bf16_split_k(int n_out, int tp, int n_in);
int gemm_bf16_clamp_split(int n_out, int tp, int n_in, int split_k);
void gemm_bf16_describe_plan(int tp, int n_in, int n_out, int split_k, int32_t out[6]);
int launch_gemm_store_f32(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in,
                          int n_out, int split_k, float* y, hipStream_t st);
// x += the whole product (no k-split)
int launch_gemm_residual(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, float* x,
                         hipStream_t st);
// the same for many rows with the next norm's input (RowScale: [n_out / 128][tp] sums of squares)
bool gemm_residual_norm_runs(int tp, int n_in, int n_out, const void* xp, const void* w);
int launch_gemm_residual_norm(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, float* x,
                              const float* g, uint16_t* hp, float* ssq, hipStream_t st);
// fp32 logits (null: none) and the greedy argmax of every row, from candidates of the epilogue
// (cand null: the logits alone; argmax_out null: the candidates stay)
int launch_gemm_lm(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_out, const RowScale& rs,
                   float* logits, void* cand, int32_t* argmax_out, hipStream_t st);
int launch_gemm_gate_up(const uint16_t* xp, const uint16_t* w, int tp, int n_in, int d_ffn,
                        const RowScale& rs, uint16_t* act, hipStream_t st);
// q may be null: then only K and V are computed and written (the last layer of a prompt pass)
int launch_gemm_qkv(const uint16_t* xp, const uint16_t* w, int T, int tp, int n_in, int n_heads,
                    int n_kv_heads, int dh, int s_pool, const RowScale& rs, const float2* cs,
                    const int32_t* cs_row, const int32_t* row_slot, uint16_t* q, uint16_t* k_layer,
                    uint16_t* v_layer, hipStream_t st);
// x[t] = E[tok[t]] (more than PREP_MAX_SEQS sequences), or x[t] += the split-k partial sums
// (n_split == 0: x is complete already and only read); hp = bf16(x * g) tiled and the rows'
// partial sums of squares for the consumer's RowScale, one launch
int launch_embed_norm(const uint16_t* embed, const int32_t* tok, int T, int d, int vocab, float* x,
                      const float* g, int tp, uint16_t* hp, float* ssq, hipStream_t st);
int launch_reduce_norm(const float* partial, int n_split, float* x, const float* g, int T, int d,
                       int tp, uint16_t* hp, float* ssq, hipStream_t st);
int launch_sum_splits(const float* partial, int n_split, size_t n, float* y, hipStream_t st);
int launch_tile_activation(const uint16_t* x, int T, int n, int tp, uint16_t* xp, hipStream_t st);

// attn_bf16.hip
enum AttnForm { AF_REGISTERS, AF_RING, AF_ONCE };  // how K/V come to a wavefront
struct AttnPlan {
  int ntw, qg_max;       // query tiles of 32 per workgroup, groups of them per sequence at most
  int bpwg, nsplit_max;  // 32-slot blocks per workgroup, key splits per sequence at most
  bool ring;             // K/V through rings in LDS, else registers
  bool once;             // no ring: all of a workgroup's K/V to LDS at once
  float lag;             // how far the softmax reference may fall behind the running maximum (log2)
};
// log2 of the query heads of a K/V head that are worked on together as one column.  common_kv: the
// sequences read the same K/V
int attn_bf16_pack(int B, int T, int n_heads, int n_kv_heads, int dh, int max_seq_slots, bool common_kv);
// the form in which a plan runs.  self: one sequence that the kernel checks itself; aligned: all
// operands start at multiples of 16 bytes
AttnForm attn_bf16_form(const AttnPlan& p, bool self, bool aligned);
// shared_kv: several workgroups besides a sequence's query groups read the same K/V
AttnPlan attn_bf16_plan(int B, int T, int n_heads, int dh, bool shared_kv, int max_seq_slots, int pack);
size_t attn_bf16_ws_floats(int B, int T, int n_heads, int dh, int max_seq_slots, int pack);
size_t attn_bf16_item_words(int B, int T, int n_heads, int dh, int max_seq_slots, int pack);
// parent (one sequence, plain `out`): no prologue launch came before, the kernel checks the
// sequence itself, writes its status and the rows it does not own; anc and items are not read
int launch_tree_attn_bf16(const uint16_t* q, const uint16_t* k_layer, const uint16_t* v_layer,
                          const uint64_t* anc, const int32_t* node_off,
                          const int32_t* kv_off, const int32_t* prefix_len,
                          const int32_t* status_dev, const int32_t* items, int B, int T,
                          int n_heads, int n_kv_heads, bool shared_kv, int pack, int dh, int s_pool, int max_seq_slots,
                          float scale, float* ws, int tiled, int tp, uint16_t* out, const int32_t* parent,
                          int32_t* status, hipStream_t st);

// api.hip: the forward pass behind tr_verify_step (with_head == false: decoder layers
// only, for prompt passes), its workspace need, and the model-descriptor check
int step_impl(const trj_model_desc* desc, const trj_weights* weights, void* k_pool, void* v_pool,
              size_t kv_layer_stride, int32_t s_pool, const int32_t* tok, const int32_t* parent,
              const int32_t* node_off, const int32_t* kv_off, const int32_t* prefix_len,
              int32_t B, int32_t T, int32_t max_seq_slots, void* workspace, size_t ws_bytes,
              float* logits, int32_t* argmax_out, int32_t* accept_len, int32_t* best_node,
              int32_t* path, int32_t* bonus_tok, int32_t* new_len, int32_t* status_dev,
              bool with_head, hipStream_t st, const TemplateView* tmpl = nullptr, int max_pos = 0);
size_t template_carve(void* base, int B, int T, int dh, int max_pos, TemplateView* v);
size_t step_workspace_bytes(const trj_model_desc& m, int B, int T, int max_seq_slots);
int check_model(const trj_model_desc* m);

// token rows are padded to whole 32-row MFMA tiles: 1, 2, 3 or 4 tiles per workgroup pass,
// beyond that blocks of 4
inline int padded_rows(int T) { return T <= 96 ? (T <= 32 ? 32 : (T + 31) / 32 * 32) : (T + 127) / 128 * 128; }

}  // namespace trj
