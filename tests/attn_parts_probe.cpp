// Host build of the places of the attention's partial sums for tests/test_attention_parts_cpu.py:
// marks every place that the valid sequences of a batch write, as the kernels count them.
#include "../paper_2406_17404_amd/csrc/attn_parts.h"

// returns the number of places that two sequences share or that lie outside the memory
extern "C" int trj_test_parts(const int32_t* node_off, int B, int T, int pack, int ntw, int n_max, int32_t* owner) {
  const int qg_max = ((T < n_max ? T : n_max) * (1 << pack) + 32 * ntw - 1) / (32 * ntw), per = qg_max * ntw;
  const long tiles = (long)trj::part_tiles(B, T, pack, per);
  int wrong = 0;
  for (int s = 0; s < B; ++s)  // no splits, no partial sums
    if (pack > 0 && trj::range_descends(node_off, s)) return 0;
  for (long i = 0; i < tiles; ++i) owner[i] = -1;
  for (int s = 0; s < B; ++s) {
    const int r0 = node_off[s], n = node_off[s + 1] - r0;
    if (r0 < 0 || node_off[s + 1] > T || n < 1 || n > n_max) continue;  // malformed: writes nothing
    for (int t = 0; t * 32 < n << pack; ++t) {
      const long at = trj::part_first(pack, per, s, r0) + t;
      if (at < 0 || at >= tiles || owner[at] != -1) ++wrong;
      else owner[at] = s;
    }
  }
  return wrong;
}
