// The query kernel with one wave per SIMD, one workgroup of four waves per CU, for problems whose 128-query tiles do not outnumber the
// CUs (launch_query's rule).  gfx950 only.
//
// Bound: latency of one wave's chain.  Nothing else hides it, so the epilogue is the pipeline of the state pass (mlp128_pipelined, whose
// 270 live registers need a wave's full 512), fragments are requested ahead of their use, and the file is compiled with the matrix
// instructions in vector-register form (otherwise the accumulators sit in the accumulator file and every rescale, exponential and
// output passes through copies: 1388 of them, 400 in the loop).  H = 12, N = 1560, R = 4 (156 workgroups, 13 key blocks), whole
// call: 43.1 us with 84 workgroups of eight waves, 39.2 with four waves and the operands in LDS, 37.4 with the pipelined epilogue, 36.2 with
// accumulators in vector registers.
//   With the map in the call and a loop of up to 256 key blocks the workgroup has a second set of four waves, which evaluate phi_q and its
// product with the state (MapRole, ha_query_kernel.h) while the first walk the keys: the epilogue is an exchange through LDS.  The same case:
// kernel 19.7 -> 16.5 us, whole call 35.6 -> 32.7.  Stamps (cycles): first request at 2700, first blocks there at 6000, 13 steps of 1530, the
// exchange and the store 3300; the map's pieces, of about a step each, fill all of the loop.  (Before its pieces were cut to that size
// the activation alone held the loop up for 3000 cycles; two copies of the step cost a cold instruction fetch of 2500 in a short loop.)
// Others, one role / two: d = 64, H = 2, N = 1024, R = 4, fp32 20.6 / 19.2; H = 12, N = 2600, R = 2 51.1 / 49.4; H = 6, N = 5000, R = 2 (79 blocks)
// 66.5 / 66.1; d = 64, H = 1, R = 2: N = 20000 (313 blocks) 119.4 / 118.0, N = 32000, fp32 (500) 180.6 / 184.1: a barrier per step instead of two.
#include "ha_query_kernel.h"

namespace ha {

hipError_t launch_query_alone(const Plan &pl, const QueryArgs &a, dim3 grid, hipStream_t st) {
  if (a.lin) {
    if (pl.f32) query_kernel_ring<128, 128, 128, 4, 8, 2, true, true><<<grid, 256, 0, st>>>(a);
    else query_kernel_ring<128, 128, 128, 4, 8, 2, false, true><<<grid, 256, 0, st>>>(a);
  } else if (a.has_linear && a.NS <= 256 * 32) {
    if (pl.D == 64) {
      if (pl.f32) query_kernel_ring<64, 64, 64, 4, 8, 1, true, false, 0, true><<<grid, 512, 0, st>>>(a);
      else query_kernel_ring<64, 64, 64, 4, 8, 1, false, false, 0, true><<<grid, 512, 0, st>>>(a);
    } else {
      if (pl.f32) query_kernel_ring<128, 128, 128, 4, 4, 1, true, false, 0, true><<<grid, 512, 0, st>>>(a);
      else query_kernel_ring<128, 128, 128, 4, 4, 1, false, false, 0, true><<<grid, 512, 0, st>>>(a);
    }
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
