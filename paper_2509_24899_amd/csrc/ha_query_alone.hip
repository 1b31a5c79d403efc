// The query kernel where 128-query tiles do not outnumber the CUs (launch_query's rule): one workgroup per CU, its first four waves
// with a SIMD each for the key loop.  gfx950 only.
//
// Bound: latency of one wave's chain.  Nothing else hides it, so fragments are requested ahead of their use and the file is compiled with the matrix
// instructions in vector-register form (otherwise the accumulators sit in the accumulator file and every rescale, exponential and
// output passes through copies: 1388 of them, 400 in the loop).  H = 12, N = 1560, R = 4 (156 workgroups, 13 key blocks), whole
// call: 43.1 us with 84 workgroups of eight waves; with four waves of a SIMD each, the map behind the loop and its operands in LDS, 36.2.
//   Where the call has a map, a second set of four waves evaluates phi_q and its product with the state (MapRole, ha_query_kernel.h) while the first
// walk the keys: the epilogue is an exchange through LDS.  The same case: kernel 19.7 -> 16.5 us, whole call 36.2 -> 33.5.  Stamps (cycles): first
// request at 2700, first blocks there at 6000, 13 steps of 1530, the exchange and the store 3300; the map's pieces, of about a step each, fill all of
// the loop.  (Before its pieces were cut to that size the activation alone held the loop up for 3000 cycles; two copies of the step cost
// a cold instruction fetch of 2500 in a short loop.)
#include "ha_query_kernel.h"

namespace ha {

// Beside the loop the map saves 1.5 - 2 us at any length, but the loop has a barrier per key block there instead of one every two: in the bf16 instances
// a block takes as long either way, in the fp32 instance of d = 64 10 ns more, so that it is behind from about 160 blocks on.  Whole calls,
// behind / beside, us: bf16: d = 128, H = 6, R = 2: N = 1000 33.6 / 31.3, 5300 (83 blocks) 69.4 / 68.3; d = 64: H = 2, N = 1024, R = 4 18.2 / 16.5, H = 1, R = 2:
// N = 8000 (125) 56.4 / 54.7, 20000 (313) 120.1 / 118.3, 32760 (512) 184.1 / 182.6.  fp32: d = 128: 37.0 / 35.4, 77.1 / 76.9; d = 64: 19.9 / 18.5, N = 8000
// 58.5 / 58.1, 12000 (188) 80.1 / 80.6, H = 2, N = 16000 (250) 101.9 / 102.8, H = 1, N = 32760 185.3 / 189.2.  (d = 128 has the map in the call from six heads
// on, hence at most 171 blocks.)
constexpr int kMaxKeysBesideMapF32 = 160 * 32;

hipError_t launch_query_alone(const Plan &pl, const QueryArgs &a, dim3 grid, hipStream_t st) {
  const bool map = a.has_linear && !a.lin;                // the call evaluates phi_q
  // (The instances' code stands in the order in which they are named here: with the last two first the 128-wide ones with a map fall elsewhere and
  // take longer, H = 12, N = 1560, R = 4 32.1 us instead of 31.8.)
  if (pl.D == 128 && !map) {
    if (pl.f32) query_kernel_ring<128, 128, 128, 4, 8, 2, true, true><<<grid, 256, 0, st>>>(a);
    else query_kernel_ring<128, 128, 128, 4, 8, 2, false, true><<<grid, 256, 0, st>>>(a);
  } else if (pl.D == 64 && map && (!pl.f32 || a.NS <= kMaxKeysBesideMapF32)) {
    if (pl.f32) query_kernel_ring<64, 64, 64, 4, 8, 1, true, false, 0, true><<<grid, 512, 0, st>>>(a);
    else query_kernel_ring<64, 64, 64, 4, 8, 1, false, false, 0, true><<<grid, 512, 0, st>>>(a);
  } else if (pl.D == 128) {
    if (pl.f32) query_kernel_ring<128, 128, 128, 4, 4, 1, true, false, 0, true><<<grid, 512, 0, st>>>(a);
    else query_kernel_ring<128, 128, 128, 4, 4, 1, false, false, 0, true><<<grid, 512, 0, st>>>(a);
  } else if (map) {
    query_kernel_ring<64, 64, 64, 4, 8, 2, true><<<grid, 256, 0, st>>>(a);
  } else {
    if (pl.f32) query_kernel_ring<64, 64, 64, 4, 8, 2, true, true><<<grid, 256, 0, st>>>(a);
    else query_kernel_ring<64, 64, 64, 4, 8, 2, false, true><<<grid, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

}  // namespace ha
