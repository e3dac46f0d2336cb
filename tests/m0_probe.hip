// Compiled, never run, by tests/test_lds_load_registers_cpu.py: a compiler-made load to LDS on
// either side of the hand-written one, to the same LDS address, so that the compiler would
// leave out setting m0 again if it did not know that the hand-written one changes it.
#include "../paper_2406_17404_amd/csrc/common.h"

typedef const __attribute__((address_space(1))) void gptr;
typedef __attribute__((address_space(3))) void lptr;

template <int FORM>
__global__ void probe_kernel(const char* a, const char* b, float* out) {
  __shared__ __align__(16) float lds[1024];
  const uint32_t other = (uint32_t)(size_t)(lptr*)lds + 2048;
  const int lane = threadIdx.x;
  __builtin_amdgcn_global_load_lds((gptr*)(a + lane * 4), (lptr*)lds, 4, 0, 0);
  if (FORM == 0) trj::load_to_lds<false>(b, lane * 16, __builtin_amdgcn_readfirstlane(other));
  if (FORM == 1) trj::load_to_lds<true>(b, lane * 16, __builtin_amdgcn_readfirstlane(other));
  if (FORM == 2) trj::load_words_to_lds(b, lane * 4, __builtin_amdgcn_readfirstlane(other));
  __builtin_amdgcn_global_load_lds((gptr*)(a + 256 + lane * 4), (lptr*)lds, 4, 0, 0);
  __syncthreads();
  out[lane] = lds[lane] + lds[512 + lane];
}
template __global__ void probe_kernel<0>(const char*, const char*, float*);
template __global__ void probe_kernel<1>(const char*, const char*, float*);
template __global__ void probe_kernel<2>(const char*, const char*, float*);
