// Launch shape of the fp32 projections (f32_kernels.hip), on the host; a test compiles it alone.
#pragma once

namespace trj {

constexpr int F32_PARTS = 32;  // threads that share an output's sum

// Tokens per workgroup of a projection without a norm: four while that keeps the launch within the
// chip, eight beyond (every group of tokens reads the weights again).  Two, whose threads ask for
// several granules at a time, where a thread has enough granules whose latencies would otherwise
// follow one another, and where a second round of workgroups does not cost more (one round is 256;
// against eight tokens, of which half as many workgroups run at once, two).  us, without -> with:
// 256 x 1024 at 15 rows 6.7 -> 4.7, at 32 10.7 -> 4.9, 1024 x 4096 at 32 35.8 -> 25.5; beyond the
// limit 4096 x 1024 at 16 11.9 -> 16.1, 4096 x 4096 at 32 78.7 -> 110.6, 32000 x 4096 at 32 755 -> 1424.
constexpr int gemm_f32_tokens(int T, int n_in, int n_out) {
  const int few = T <= 16;
  const long wgs = (long)(n_out / 32) * ((T + 1) / 2);
  const bool granules = n_in > 8 * F32_PARTS * (few ? 2 : 1);
  if (T <= 32 && granules && (T <= 2 || wgs <= (few ? 256 : 512))) return 2;
  return few ? 4 : 8;
}

}  // namespace trj
