// The arithmetic with carries in inline assembly, in kernels small enough to
// compile for the device in a moment and read the instructions of.  One chain
// each: nothing else to put between a carry's writer and its reader.
#include "../../paper_2605_17222_amd/csrc/modarith.hpp"

using namespace ckks;

__global__ void sums(uint64_t* out, const uint64_t* a, const uint64_t* b, uint64_t q, uint64_t mu, int s, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  U128 x = {0, 0};
#pragma clang loop unroll(disable)
  for (int m = 0; m < n; ++m) mac128(x, a[m * 64 + t], b[m * 64 + t]);
  out[t] = barrett_sum(x, q, mu, s);
}

__global__ void butterfly(uint64_t* v, const uint64_t* w, uint64_t q) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  v[t] = shoup_add(v[t], v[t + 64], w[t], w[t + 64], q);
}
