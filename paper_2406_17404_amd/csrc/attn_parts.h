// Where the attention's partial sums lie (attn_bf16.hip): one place per query tile of every
// sequence whose keys are split.  Compiled for the host by a test that checks that no two
// sequences meet, whatever row ranges a batch states.
#pragma once
#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define TRJ_PARTS_HD __host__ __device__
#else
#define TRJ_PARTS_HD
#endif

namespace trj {

// Place of a sequence's first query tile among the partials' (of part_tiles).  Single heads: every
// sequence has room for the most tiles one could have.  Packed, that would be many times the tiles
// there are (sequences of 20 rows: 16 for 3): behind the rows in front of it, and one more per
// sequence for their last tiles that are not full.  The first sequence's place does not depend on
// its rows, so that the merge of a single one need not wait for them.
TRJ_PARTS_HD inline int part_first(int pack, int tiles_per_seq, int s, int r0) {
  return pack == 0 ? s * tiles_per_seq : s == 0 ? 0 : ((r0 << pack) >> 5) + s;
}
inline size_t part_tiles(int B, int T, int pack, int tiles_per_seq) {
  return pack == 0 ? (size_t)B * tiles_per_seq : ((size_t)T << pack >> 5) + B;
}
// Packed places keep sequences apart only where the row ranges ascend.  A malformed range may lie
// between valid ones that do not ({100, 128, 0, 50}: the middle one is refused, its neighbours are
// not): if any range of a batch descends, its packed sequences are walked without splits.
TRJ_PARTS_HD inline bool range_descends(const int32_t* node_off, int s) { return node_off[s + 1] < node_off[s]; }

}  // namespace trj
