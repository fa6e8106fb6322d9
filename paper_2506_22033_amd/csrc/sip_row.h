// Streaming and finishing in one workgroup: it streams a whole row (sip_stream.h), and what it then
// has in hand -- the list in registers, the masses, the row's parameters -- it finishes
// (sip_finish.h).  For batches of several rows per compute unit: while one workgroup of a compute unit
// is in the finishing part's chain of barriers, which leaves the memory and most issue slots idle, the
// other one streams, and the set-up (sample, threshold, history) is paid once a row instead of once a
// chunk.  Two workgroups per compute unit: the finishing tables take 70 KB of LDS, and 128 registers a
// lane pay for four 16-byte loads in flight per tile instead of two.  (One row per compute unit and less:
// row_rescue_kernel, sip_fused.h.)
// Measured against the two kernels, us a call: 256 rows of V = 128256 bf16 32.5 -> 28.7, of V = 200000 fp32 53.6 ->
// 49.3; 800 rows of V = 152064 bf16 88.2 -> 85.0 (sip.hip has the line between them, and both sides of it).
// What bounds it: bf16, 1024 rows of V = 129280 (109 us with lists of one length for every nucleus, now 89), vector
// issue, 65 % of the slots, one row's set-up and finishing beside the other's streaming; fp32, 2048 rows of V =
// 256000 (490 us), HBM while it streams (4.3 TB/s over the whole kernel).
#pragma once
#include "sip_finish.h"
#include "sip_stream.h"

namespace sip {

template <int DT, bool SH, bool IDS>
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void row_kernel(Args a_by_value) {
  (void)a_by_value;
  const Args& a = *(const Args*)__builtin_amdgcn_kernarg_segment_ptr();
  warm_kernel_arguments();
  static_assert(kStreamThreads == kFinThreads, "one workgroup shape for both parts");
  __shared__ union __align__(16) Both { RowStreamShared<DT> stream; FinShared fin; __device__ Both() {} } u;
  static_assert(sizeof(u) <= 80 * 1024, "two workgroups per compute unit");
  // Workgroups go to the 8 XCDs round-robin by their id.  Every eight rows are dealt out turned by one
  // against the eight before, so that a batch whose rows alternate (every other one greedy, say) loads
  // all XCDs alike (V = 256000, 2048 rows,
  // half of them greedy: four XCDs were done after 444 us, four after 527; now all after 495).
  int b = blockIdx.x;
  if (b < (a.B & ~7)) b = (b & ~7) | ((b + (b >> 3)) & 7);
  RowHand hand;
  int code = 2;
  if (stream_part<DT, SH, true, IDS>(a, b, u.stream.front, u.stream.tables, &hand)) {                      // uniform
    __syncthreads();                       // the list is written, and the tables are free
    if (IDS && hand.greedy) code = finish_greedy(a, b, hand.best);             // uniform
    else code = finish_row<true>(a, b, u.fin, nullptr, &hand);
  }
  if (threadIdx.x == 0) {
    a.row_path[b] = code;
    a.row_why[b] = code == kFinWholeRow ? 1 : code;                            // anything but 1: the rescue kernel's
  }
}

}  // namespace sip
