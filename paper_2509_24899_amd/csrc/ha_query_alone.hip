// The query kernel with one wave per SIMD, one workgroup of four waves per CU, for problems whose 128-query tiles do not outnumber the
// CUs (launch_query's rule).  gfx950 only.
//
// Bound: latency of one wave's chain.  Nothing else hides it, so the epilogue is the pipeline of the state pass (mlp128_pipelined, whose
// 270 live registers need a wave's full 512), fragments are requested ahead of their use, and the file is compiled with the matrix
// instructions in vector-register form (otherwise the accumulators sit in the accumulator file and every rescale, exponential and
// output passes through copies: 1388 of them, 400 in the loop).  H = 12, N = 1560, R = 4 (156 workgroups, 13 key blocks), whole
// call: 43.1 us with 84 workgroups of eight waves, 39.2 with four waves and the operands in LDS, 37.4 with the pipelined epilogue, 36.2 with
// accumulators in vector registers.
#include "ha_query_kernel.h"

namespace ha {

hipError_t launch_query_alone(const Plan &pl, const QueryArgs &a, dim3 grid, hipStream_t st) {
  if (a.lin) {
    if (pl.f32) query_kernel_ring<128, 128, 128, 4, 8, 2, true, true><<<grid, 256, 0, st>>>(a);
    else query_kernel_ring<128, 128, 128, 4, 8, 2, false, true><<<grid, 256, 0, st>>>(a);
  } else if (pl.D == 64) {
    if (pl.f32) query_kernel_ring<64, 64, 64, 4, 8, 2, true><<<grid, 256, 0, st>>>(a);
    else query_kernel_ring<64, 64, 64, 4, 8, 2, false><<<grid, 256, 0, st>>>(a);
  } else {
    if (pl.f32) query_kernel_ring<128, 128, 128, 4, 8, 2, true><<<grid, 256, 0, st>>>(a);
    else query_kernel_ring<128, 128, 128, 4, 8, 2, false><<<grid, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

}  // namespace ha
