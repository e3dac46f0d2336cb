// Host build of the fp32 projections' launch rule for tests/test_f32_rule_cpu.py.
#include "../paper_2406_17404_amd/csrc/f32_rule.h"

extern "C" int trj_test_f32_tokens(int T, int n_in, int n_out) { return trj::gemm_f32_tokens(T, n_in, n_out); }
