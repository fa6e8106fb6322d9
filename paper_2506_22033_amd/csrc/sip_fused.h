// finish_kernel and rescue_kernel in one, for batches of at most one row per compute unit: a
// workgroup finishes its row from the list (finish_row) and, if the list does not settle it,
// goes on with the heavier logic (rescue_row) itself, at once.  No queue, no second launch
// behind it -- whose four microseconds, the latency of starting any kernel, are a fifteenth of
// such a call.  The price is the LDS of the heavier logic for every workgroup (one workgroup per
// compute unit), which a batch this small does not feel.
#pragma once
#include "sip_final.h"
#include "sip_finish.h"
#include "sip_row.h"

namespace sip {

constexpr size_t kAloneLds = 144 * 1024;    // sample, queues and tables of a chunk that has a compute unit to itself
constexpr size_t kFusedRawBytes = 122880;   // final_lds_fixed() of the largest vocabulary of the single-pass kernels
static_assert(sizeof(FinShared) <= kFusedRawBytes, "the finishing tables lie inside the same LDS");

// rescue_row() for the kernels that hardly ever need it, as a function of its own: inlined, its registers made the part
// that every row goes through keep 540 to 620 scalar registers in lanes of vector registers, now 2 to 28, and 18 to 37
// vector registers in scratch, now none.  us a call: one row of V = 128256 bf16 18.2 / 17.9, 64 rows 25.8 / 25.5, 256 rows of
// V = 152064 fp32 with everything on 50.0 / 49.7.  LDS goes along as offsets, the arguments as an address, so that both
// are reached by the instructions meant for them.
// Not marked as a tail call, which a call at a kernel's end otherwise is: a function that may be one has to save 108 of
// the 256 registers it uses, 432 bytes a lane, for nobody.  That frame costs more than its traffic: it sets the distance between
// the waves' scratch for every kernel of the queue, and at 32 KB (500 bytes a lane) the small frames of others collide in
// the caches (1024 rows of V = 128256 fp32, ids only, 113 / 117).  us a call, inlined / with the registers saved / so: rows of
// V = 40000 whose nuclei outgrow their lists 128 fp32 70.2 / 71.9 / 66.1, 256 bf16 69.0 / 78.9 / 67.4; in pieces, inlined / so: 200
// rows of V = 152064 in four, nucleus, bf16 33.4 / 32.7, no filter 99.0 / 96.8, fp32 137.8 / 120.0.
template <typename T>
__device__ __forceinline__ uint32_t lds_offset(T& x) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) T*)&x;
}
template <typename T>
__device__ __forceinline__ T& at_lds_offset(uint32_t o) {
  return *(T*)(__attribute__((address_space(3))) T*)(uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)o);
}
template <int DT, bool SH>
__device__ __attribute__((noinline, not_tail_called)) void rescue_apart(unsigned long long args, int b, uint32_t raw, uint32_t ex, uint32_t fs, int why,
                                                       float m, float zmax, float T) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)args);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(args >> 32));
  const Args& a = *(const Args*)(const __attribute__((address_space(4))) Args*)(((unsigned long long)hi << 32) | lo);
  RescueSeen seen;
  seen.why = __builtin_amdgcn_readfirstlane(why);
  seen.m = m; seen.zmax = zmax; seen.T = T;
  rescue_row<DT, SH>(a, __builtin_amdgcn_readfirstlane(b), &at_lds_offset<unsigned char>(raw), at_lds_offset<ExactShared>(ex),
                     at_lds_offset<FastShared>(fs), seen);
}

template <int DT, bool SH>
__global__ __launch_bounds__(kFinalThreads) void finish_rescue_kernel(Args a_by_value) {
  (void)a_by_value;
  const Args& a = *(const Args*)__builtin_amdgcn_kernarg_segment_ptr();
  warm_kernel_arguments();
  __shared__ union __align__(16) { FinShared fs; unsigned char raw[kFusedRawBytes]; } u;
  __shared__ ExactShared ex;
  __shared__ FastShared fsr;
  static_assert(kFinThreads == kFinalThreads, "one workgroup shape for both parts");
  const int b = blockIdx.x;
  FinHint hint;
  const int code = finish_row<false>(a, b, u.fs, &hint);
  if (threadIdx.x == 0) {
    a.row_path[b] = code;
    a.row_why[b] = code == kFinWholeRow ? 1 : code;
  }
  if (code == 1 || code == kFinWholeRow) return;                     // uniform
  __syncthreads();
  RescueSeen seen;
  if (hint.valid) { seen.why = code; seen.m = hint.m; seen.zmax = hint.zmax; seen.T = hint.T; }
  rescue_apart<DT, SH>((unsigned long long)&a, b, lds_offset(u.raw[0]), lds_offset(ex), lds_offset(fsr), seen.why, seen.m, seen.zmax, seen.T);
}

// The same for a workgroup that has streamed its row itself (sip_row.h).
template <int DT, bool SH, bool IDS>
__global__ __launch_bounds__(kFinalThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void row_rescue_kernel(Args a_by_value) {
  (void)a_by_value;
  const Args& a = *(const Args*)__builtin_amdgcn_kernarg_segment_ptr();
  warm_kernel_arguments();
  __shared__ union __align__(16) Tables {
    RowStreamShared<DT> stream; FinShared fin; unsigned char raw[kFusedRawBytes];
    __device__ Tables() {}
  } u;
  static_assert(sizeof(u) == kFusedRawBytes, "");
  __shared__ ExactShared ex;
  __shared__ FastShared fsr;
  const int b = blockIdx.x;
  RowHand hand;
  FinHint hint;
  int code = 2;
  if (stream_part<DT, SH, true, IDS>(a, b, u.stream.front, u.stream.tables, &hand)) {                      // uniform
    __syncthreads();                       // the list is written, and the tables are free
    if (IDS && hand.greedy) code = finish_greedy(a, b, hand.best);             // uniform
    else code = finish_row<true>(a, b, u.fin, &hint, &hand);
  }
  if (threadIdx.x == 0) {
    a.row_path[b] = code;
    a.row_why[b] = code == kFinWholeRow ? 1 : code;
  }
  if (code == 1 || code == kFinWholeRow) return;                     // uniform
  __syncthreads();
  RescueSeen seen;
  if (hint.valid) { seen.why = code; seen.m = hint.m; seen.zmax = hint.zmax; seen.T = hint.T; }
  rescue_apart<DT, SH>((unsigned long long)&a, b, lds_offset(u.raw[0]), lds_offset(ex), lds_offset(fsr), seen.why, seen.m, seen.zmax, seen.T);
}

// The same where the batch is so small that a row's chunks have a compute unit each: the last of a row's workgroups
// to be done with its chunk finishes the row.  What a second kernel costs -- 2.4 us until it starts, cold arguments and
// records -- goes; what the workgroups pay to agree is 1 us: their stores' way to memory (put(): written back from
// the XCD's L2 by each of them instead, 64 rows of V = 128256 bf16 took 29.6 us for 26.3), the addition to the row's word, its
// answer.  Times and the rule for it are at make_plan().  What bounds it: latency, the set-up's chain of 5 us, 4 us from the
// last chunk to the finishing and 11 us of that.
template <int DT, bool SH, bool IDS>
__global__ __launch_bounds__(kFinalThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void chunk_rescue_kernel(Args a_by_value) {
  (void)a_by_value;
  const Args& a = *(const Args*)__builtin_amdgcn_kernarg_segment_ptr();
  warm_kernel_arguments();
  __shared__ union Tables {
    uint4 stream[kAloneLds / 16]; FinShared fin; unsigned char raw[kFusedRawBytes];
    __device__ Tables() {}
  } u;
  __shared__ ExactShared ex;
  __shared__ FastShared fsr;
  __shared__ bool last;
  static_assert(sizeof(u) + sizeof(ex) + sizeof(fsr) + 64 <= 160 * 1024, "a compute unit's LDS");
  // (a row's chunks on one XCD, as in stream_kernel)
  int wg = blockIdx.x;
  if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int b = wg / a.S;
  unsigned char* const front = reinterpret_cast<unsigned char*>(u.stream);
  RowHand hand;
  RowWord word{reinterpret_cast<unsigned long long*>(a.rowinfo + b), 0ull};
  stream_part<DT, SH, false, IDS, true>(a, wg, front,
      *reinterpret_cast<StreamTables<DT, false, true>*>(front + stream_front_bytes<DT, false>(a.cap_c / kStreamWaves)), &hand, &word);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                             // every wave's part of the list is written
  __syncthreads();
  if (threadIdx.x == kFinalThreads - kWave) last = word.arrive((uint32_t)a.S);
  __syncthreads();
  if (!last) return;                                                 // uniform
  FinHint hint;
  int code;
  if (IDS && hand.greedy) {                                          // uniform
    unsigned long long best = 0;
    for (int i = 0; i < a.S; ++i) {
      const unsigned long long x = *reinterpret_cast<const unsigned long long*>(a.chunks + (size_t)b * (size_t)a.S + i);
      best = x > best ? x : best;
    }
    __syncthreads();                       // (finish_greedy() may write there)
    code = finish_greedy(a, b, best);
  } else {
    code = finish_row<false, true>(a, b, u.fin, &hint, &hand);
  }
  if (threadIdx.x == 0) {
    a.row_path[b] = code;
    a.row_why[b] = code == kFinWholeRow ? 1 : code;
  }
  if (code == 1 || code == kFinWholeRow) return;                     // uniform
  __syncthreads();
  RescueSeen seen;
  if (hint.valid) { seen.why = code; seen.m = hint.m; seen.zmax = hint.zmax; seen.T = hint.T; }
  rescue_apart<DT, SH>((unsigned long long)&a, b, lds_offset(u.raw[0]), lds_offset(ex), lds_offset(fsr), seen.why, seen.m, seen.zmax, seen.T);
}

}  // namespace sip
