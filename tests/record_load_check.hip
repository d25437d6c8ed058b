// Compiled to assembly by tests/test_host_record_load.py: the accumulate pass's rows of records, two of them a lane,
// requested through a buffer whose bound is the item's end.
#include <stdint.h>

#include "bwd_record.hpp"

template <typename IT, int F>
__global__ void rows_of_records(const uint32_t* records, uint32_t first, uint32_t n, uint32_t row_bytes, uint32_t* out) {
  using Rec = hg::Record<IT, F>;
  const auto item = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(records) + (uint64_t)first * Rec::kWords, 0,
                                                      n * Rec::kWords * 4u, hg::kBufferWord3);
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t j = 0; j < 3; ++j) {
    const auto r = Rec::load_from(item, threadIdx.x * Rec::kWords * 4u + (j == 2 ? row_bytes : j * 1024u * Rec::kWords * 4u));
    for (uint32_t q = 0; q < Rec::kWords; ++q) sum ^= r.w[q];
  }
  out[threadIdx.x] = sum;
}
template __global__ void rows_of_records<_Float16, 1>(const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*);
template __global__ void rows_of_records<_Float16, 2>(const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*);
template __global__ void rows_of_records<_Float16, 4>(const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*);
template __global__ void rows_of_records<_Float16, 8>(const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*);
template __global__ void rows_of_records<float, 2>(const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*);
template __global__ void rows_of_records<float, 8>(const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*);
