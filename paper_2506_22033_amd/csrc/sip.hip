// Host side of the C boundary declared in include/sip.h: argument checks, workspace
// carving and kernel launches.  No allocation, no synchronisation.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <atomic>
#include <chrono>
#include <mutex>

#include "../../include/sip.h"
#include "../../include/sip_diag.h"
#include "sip_device.h"
#include "sip_exact.h"
#include "sip_final.h"
#include "sip_finish.h"
#include "sip_fused.h"
#include "sip_handoff.h"
#include "sip_resident.h"
#include "sip_row.h"
#include "sip_state.h"
#include "sip_stream.h"

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Launch shape of the single-pass path; a function of (B, V, dtype) only.
struct Cut {
  int S, cap_c, nc_cap;                                  // see Args
};
struct Plan {
  bool fast;       // false: vocabulary outside what the single-pass kernels are built for
  Cut cut;         // of a row, for the streaming kernel
  Cut beside;      // the same for chunks that have a compute unit each, with room on the chip beside them; S = 0: not so
  Cut alone;       // and on all of the chip
  int room;        // segments of kChunkCap entries a row has in the workspace
  size_t final_lds;
};

// Rows up to here fit the registers of one workgroup (16 waves x 128; sip_resident.h).
constexpr int kResidentMaxV = SIP_MAX_RESIDENT_V;
static_assert(kResidentMaxV == 1024 * 32, "the largest variant launched below");
// Kernels that use more than the default 64 KB of dynamic LDS have to be told so once per device.
constexpr int kMaxDynLds = 144 * 1024;
constexpr int kFastMinV = 16384;
constexpr int kFastMaxV = 262144;
constexpr int kFastMinPiece = 8192;      // smallest vocabulary shard: its sample blocks (at most 32 of 256 elements) must fit

// `t` > 0: the logits come in t vocabulary shards of V / t elements (0: one piece).  `small_chunks`: see
// plan_for().
Plan make_plan(int32_t B, int32_t V, int dtype, int t, bool small_chunks = true) {
  Plan p{};
  const int pieces = t > 0 ? t : 1;
  const int Vp = V / pieces;                           // elements per piece
  p.fast = V >= kFastMinV && V <= kFastMaxV && Vp >= kFastMinPiece && pieces <= sip::kMaxChunks;
  if (!p.fast) return p;
  const int tile = dtype == SIP_F32 ? sip::StreamShape<SIP_F32, false>::kTile : sip::StreamShape<SIP_BF16, false>::kTile;
  const int n_tiles = (Vp + tile - 1) / tile * pieces;
  // `n` chunks a row, as the kernels can have them.
  auto fit = [&](int n, int most = sip::kChunkBitsMax) {
    // A chunk holds at least two tiles; where the batch is small, one: a short bf16 row would else be one or
    // two chunks, whose queues overflow under a long history.  (V = 24275 bf16, 61 rows of 3034 tokens on a
    // state, one chunk: half of the rows took the exact path, 254 us; three: 78.)  The workspace grows with
    // the chunks, so for at most 256 of them.
    n = std::max(1, std::min({n, sip::kMaxChunks, std::max({1, n_tiles / 2, small_chunks ? std::min(n_tiles, 256 / B) : 0})}));
    if (n >= pieces) {
      n = n / pieces * pieces;                           // a chunk is part of one piece: a multiple of their number
    } else {
      // a chunk is several whole pieces: the divisor of their number nearest to `n` (by ratio)
      int best = pieces;
      for (int dv = 1; dv <= pieces; ++dv)
        if (pieces % dv == 0) {
          const double r0 = std::fabs(std::log((double)best / n)), r1 = std::fabs(std::log((double)dv / n));
          if (r1 < r0 || (r1 == r0 && dv > best)) best = dv;
        }
      n = best;
    }
    // the streaming kernel marks a chunk's history tokens in an LDS bitmap of `most` bits:
    // cut finer (first at the piece boundaries, then inside the pieces) until a chunk fits
    const int unit = sip::kChunkUnit;
    const int n_units = (Vp + unit - 1) / unit;
    auto max_chunk = [&](int S) {
      return S >= pieces ? (n_units + S / pieces - 1) / (S / pieces) * unit : pieces / S * Vp;
    };
    while (max_chunk(n) > most) {
      n = n >= pieces ? n + pieces : pieces;
      if (n > sip::kMaxChunks) return 0;
    }
    return n;                                            // <= n_tiles
  };
  // Room in the workspace.  Up to 256 rows: for as many chunks as fit on the chip at once, 4 per compute
  // unit.  Larger batches run in rounds of that many workgroups, and every workgroup pays a fixed set-up
  // (sample, threshold, history bitmap: about what streaming 38 elements per lane costs) before it
  // streams its V / (S * 512) elements per lane: the S with the cheapest rounds x (set-up + stream).
  // (256 units, whatever device the call will run on: how large a workspace is and how a row is cut are the same for
  // every device, and known without one.  A partition of the chip with fewer units gets as many chunks; only its speed
  // is not what is said below.)
  constexpr int kUnits = 256, kResident = kUnits * 4;
  int want;
  if (B * 4 <= kResident) {
    want = kResident / B;
  } else {
    // (from 2 on: one chunk's queues alone are short for a long list plus a long history)
    double best_cost = 0.0;
    want = 2;
    for (int S = 2; S <= sip::kMaxChunks; ++S) {
      const double rounds = std::ceil((double)B * S / kResident);
      const double cost = rounds * (38.0 + (double)V / (S * (double)sip::kStreamThreads));
      if (S == 2 || cost < best_cost) { best_cost = cost; want = S; }
    }
  }
  p.room = p.cut.S = fit(want);
  if (p.room == 0) { p.fast = false; return p; }
  // Chunks per row.  Up to 256 rows the room's worth of chunks is often too many: each pays the set-up, and what
  // counts is how many a compute unit gets.  With w of them its time grows as w * (set-up + stream), the set-up
  // being worth 32 KB of the row, and a compute unit that has only one streams at 4/5 of the speed.  us a call, at 1024
  // workgroups / at 256 / as chosen: V = 128256 fp32, 64 rows 27.5 / 23.2 / 23.2, 128 rows 29.6 / 27.7 / 27.0; bf16, 64
  // rows 23.1 / 22.1 / 22.1, 128 rows 29.6 / 26.3 / 26.8; V = 200000 fp32, 128 rows 32.8 / - / 31.5; bf16 31.8 / - /
  // 29.5.
  int load = 4;                                          // chunks of a compute unit
  if (B <= kUnits) {
    const double set_up = dtype == SIP_F32 ? 8192.0 : 16384.0;                 // in elements
    double best_cost = 0.0;
    const int room = p.room;
    for (int w = 1; w <= 4; ++w) {
      const int S = w * kUnits >= B ? fit(w * kUnits / B) : 0;
      if (S == 0 || S > room) continue;
      const int per_unit = (B * S + kUnits - 1) / kUnits;
      const double cost = per_unit * (set_up + (per_unit == 1 ? 1.25 : 1.0) * V / S);
      if (best_cost == 0.0 || cost < best_cost) { best_cost = cost; p.cut.S = S; load = per_unit; }
    }
  }
  // Fewer chunks share the row's room in the workspace and their compute unit's LDS: longer queues and segments.
  constexpr int kTables = sip::stream_lds_bytes<SIP_F32>(sip::kQueueCap) - sip::kChunkCap * (int)sizeof(uint2);
  constexpr int kAloneTables = (int)sizeof(sip::StreamTables<SIP_F32, false, true>);
  static_assert(kAloneTables + 16384 <= (int)sip::kAloneLds && sizeof(sip::StreamTables<SIP_BF16, false, true>) <= kAloneTables + 8192 &&
                kMaxDynLds <= (int)sip::kAloneLds, "bf16 tables are larger by less than its queues are shorter");
  auto share = [&](Cut& c, int load, int tables) {
    const int lds = std::min(kMaxDynLds, 160 * 1024 / load);
    const int queue = std::min(sip::kQueueCap * p.room / c.S, (lds - tables) / (sip::kStreamWaves * (int)sizeof(uint2))) / 32 * 32;
    c.cap_c = sip::kStreamWaves * std::max(queue, sip::kQueueCap);
    // the longest list a row may have: what the heavier per-row logic holds in registers, and what
    // the row's chunks can hand over
    c.nc_cap = std::min(sip::kFinalThreads * sip::kCandLong, c.S * c.cap_c);
  };
  share(p.cut, load, kTables);
  // A compute unit for each chunk, and the last of a row's workgroups finishes it (chunk_rescue_kernel).  That saves a launch and
  // what the second kernel waits for at its start.  But such a workgroup leaves its compute unit no room for another one (the
  // heavier logic's 256 registers a lane), where the streaming kernel's chunks of two batches in flight lie side by side.
  // With 176 workgroups the finishing ones of another batch, and some of its chunks, find room.  us a call, two kernels / as many
  // chunks as compute units / 176 (nucleus 0.95, Student-t, 600 tokens), one batch at a time; two batches in flight, each
  // on a stream:
  //   V = 60000 bf16 16 rows 18.4 / 17.7 / 17.7; 10.0 / 9.1 / 9.1, 32 rows 18.6 / 17.7 / 18.3; 10.7 / 12.3 / 9.9
  //   V = 128256 bf16 16 rows 18.6 / 17.7 / 18.1; 10.8 / 12.2 / 9.6, 32 rows 19.3 / 18.5 / 19.4; 11.4 / 13.2 / 10.7, 40 rows 20.1 /
  //   19.0 / 20.2; 12.1 / 13.6 / 12.2, 64 rows (192 workgroups) 20.9 / 20.0 / 21.0; 13.2 / 17.7 / 14.2
  //   V = 128256 fp32 16 rows 18.6 / 18.1 / 18.4; 11.1 / 12.6 / 9.5, 32 rows 19.7 / 18.9 / 19.9; 12.1 / 13.7 / 11.1, 40 rows 20.3 /
  //   19.7 / 20.7; 14.2 / 14.3 / 13.3
  //   V = 200000 bf16 24 rows 19.6 / 18.6 / 19.6; 11.7 / 12.9 / 10.6, 32 rows 20.4 / 19.3 / 20.6; fp32 24 rows 20.2 / 19.3 / 20.1;
  //   12.4 / 13.8 / 11.2, 32 rows 20.7 / 20.0 / 21.6
  //   V = 128256 bf16 35 rows without a filter 23.1 / 23.0 / 23.8; 13.5 / 17.2 / 15.1, V = 40000 21.8 / 21.8 / 21.8; 11.5 / 13.5 / 13.4
  // So with 176, up to 32 rows and chunks of 36 K elements.
  auto alone = [&](Cut& c, int units, int rows, int most) {
    c.S = B <= rows ? fit(units / B, most) : 0;
    if (c.S < 2 || c.S > p.room || B * c.S > units) c.S = 0;
    else share(c, 1, kAloneTables);
  };
  alone(p.beside, 176, 32, 36 * 1024);
  // Greedy rows of which only the ids are wanted have next to nothing to finish, and where that does not serve them gain from
  // every compute unit, also with two batches in flight.  us a call, two kernels / one, one batch; two: V = 128256 64 rows bf16 8.0 /
  // 7.0; 5.6 / 5.6, fp32 9.4 / 7.4; 9.4 / 7.5, 128 rows bf16 10.9 / 8.4; 7.7 / 7.1, fp32 15.8 / 14.7; 12.1 / 10.8; V = 262144 fp32 100 rows 21.5
  // / 19.5; 17.5 / 13.9.  (16 rows of V = 128256 bf16 two kernels / 256 workgroups / 176: 7.5 / 8.2 / 7.5; 4.3 / 5.7 / 4.2, fp32 7.6 / 8.0 / 7.7; 4.4 / 5.9 /
  // 4.4; 32 rows bf16 7.5 / 6.9 / 7.0; 4.4 / 5.3 / 4.1.)
  alone(p.alone, kUnits, kUnits / 2, sip::kAloneBitsMax);
  p.final_lds = sip::final_lds_fixed(V);
  return p;
}

struct Layout {
  size_t row_path, tick, side_z, side_c, rowinfo, chunks, cand, gather, total;
};

thread_local hipEvent_t g_prof[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};   // one-shot, see sip_profile_kernel_events()

constexpr int kMaxDevices = 64;
constexpr int kRescueGrid = 256;         // workgroups of the rescue kernel (one per compute unit)

// Built-in scratch of sip_sample_noalloc(): one copy per device, at that device's own address.
// In host code the name below is only a handle for hipGetSymbolAddress; the address the kernels
// get is the one looked up in device_setup().
constexpr size_t kNoallocBytes = (size_t)40 << 20;     // holds a call of 256 rows at V = 152064 (33.6 MB)
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

struct DeviceSetup {
  std::atomic<int> state{0};                // 0: not done, 1: done
  void* scratch_ptr = nullptr;
  int compute_units = 0;
};
DeviceSetup g_dev[kMaxDevices];
std::mutex g_dev_mutex;

// Per-device set-up (see sip_init in the header).  Returns the device's entry, or nullptr.
DeviceSetup* device_setup() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return nullptr; }
  DeviceSetup& d = g_dev[dev];
  if (d.state.load(std::memory_order_acquire) == 1) return &d;
  std::lock_guard<std::mutex> lock(g_dev_mutex);
  if (d.state.load(std::memory_order_acquire) == 1) return &d;
  const void* big[] = {
      reinterpret_cast<const void*>(sip::exact_kernel<SIP_F32, false>), reinterpret_cast<const void*>(sip::exact_kernel<SIP_BF16, false>),
      reinterpret_cast<const void*>(sip::exact_kernel<SIP_F32, true>),  reinterpret_cast<const void*>(sip::exact_kernel<SIP_BF16, true>),
      reinterpret_cast<const void*>(sip::rescue_kernel<SIP_F32, false>), reinterpret_cast<const void*>(sip::rescue_kernel<SIP_BF16, false>),
      reinterpret_cast<const void*>(sip::rescue_kernel<SIP_F32, true>),  reinterpret_cast<const void*>(sip::rescue_kernel<SIP_BF16, true>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_F32, false, false>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_BF16, false, false>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_F32, true, false>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_BF16, true, false>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_F32, false, true>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_BF16, false, true>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_F32, true, true>),
      reinterpret_cast<const void*>(sip::stream_kernel<SIP_BF16, true, true>)};
  for (const void* k : big)
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynLds) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return nullptr; }
  d.scratch_ptr = p;
  if (hipDeviceGetAttribute(&d.compute_units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    d.compute_units = 0;
  }
  d.state.store(1, std::memory_order_release);
  return &d;
}

bool shape_ok(int32_t B, int32_t V, int dtype, int64_t nnz, int32_t k_lp) {
  return B > 0 && V > 0 && (dtype == SIP_F32 || dtype == SIP_BF16) && nnz >= 0 && k_lp >= -1;
}

// `gather_row_bytes` > 0 (sharded logits): room for B whole rows.
Layout make_layout(int32_t B, const Plan& p, int64_t nnz, size_t gather_row_bytes = 0) {
  Layout l;
  size_t off = 0;
  l.row_path = off; off += align_up((size_t)2 * B * sizeof(int));            // first, so that callers can find it: path
                                                                             // codes, then the finishing kernel's own
                                                                             // codes
  l.tick = off; off += align_up(sizeof(unsigned long long));                 // the state's call counter as taken by this call
  l.side_z = off; off += align_up((size_t)nnz * sizeof(float));
  l.side_c = off; off += align_up((size_t)nnz * sizeof(unsigned int));
  l.rowinfo = off;
  if (p.fast) off += align_up((size_t)B * sizeof(sip::RowInfo));
  l.chunks = off;
  if (p.fast) off += align_up((size_t)B * p.room * sizeof(sip::ChunkOut));
  l.cand = off;
  if (p.fast) off += align_up((size_t)B * p.room * (size_t)sip::kChunkCap * sizeof(uint2));
  l.gather = off; off += align_up((size_t)B * gather_row_bytes);
  l.total = off ? off : kAlign;
  return l;
}

// A call's plan.  Chunks of one tile take up to 7.9 MB of workspace more than chunks of two (256 segments
// of 30 KB): where that alone would put a call with a history of millions of tokens beyond the built-in
// scratch, its chunks hold two tiles -- through every entry point, so that all of them give the same bits.
Plan plan_for(int32_t B, int32_t V, int dtype, int t, int64_t nnz, size_t gather_row_bytes = 0, bool* coarse = nullptr) {
  const Plan p = make_plan(B, V, dtype, t);
  if (make_layout(B, p, nnz, gather_row_bytes).total <= kNoallocBytes) return p;
  const Plan two = make_plan(B, V, dtype, t, false);
  const bool give_way = make_layout(B, two, nnz, gather_row_bytes).total <= kNoallocBytes;
  if (coarse) *coarse = give_way && two.room != p.room;
  return give_way ? two : p;
}

// What the size functions report.  A call's own need falls where its chunks of one tile become chunks of
// two, with a longer history as above or with more rows (256 / B in make_plan()).  A caller that sized its
// workspace for its longest histories and largest batch is served on every smaller call all the same: the
// largest need of the batches up to this one that are cut into chunks of one tile counts, and for a
// history beyond which they give way the built-in scratch's size, which bounds the need up to there.
size_t workspace_need(int32_t B, int32_t V, int dtype, int t, int64_t nnz, size_t gather_row_bytes = 0) {
  // (Batches with the same 256 / b have chunks of the same length, and the need grows with b among them: the
  // largest of each counts, and below 256 / kMaxChunks they are all alike.  One batch after the other, this
  // took 16 us where a caller leaves the workspace to the binding, V = 24275 bf16 and 255 rows; now 4.)
  size_t need = 0;
  for (int32_t b = std::min(B, 256 / sip::kMaxChunks); ; b = std::min(B, b < 256 ? 256 / (256 / (b + 1)) : B)) {
    if (b < B && make_plan(b, V, dtype, t).room == make_plan(b, V, dtype, t, false).room) b = B;   // (from here on they all agree)
    bool coarse = false;
    const size_t own = make_layout(b, plan_for(b, V, dtype, t, nnz, gather_row_bytes, &coarse), nnz, gather_row_bytes).total;
    need = std::max(need, coarse ? kNoallocBytes : own);
    if (b >= B) return need;
  }
}

// Where a call's token histories come from: a CSR handed in by the caller, or the slots of a
// device-resident state.
struct HistSource {
  const int64_t* indptr = nullptr;
  const int32_t* tokens = nullptr;
  int64_t nnz = 0;                                   // entries the side tables of the workspace are sized for
  const int64_t* p_indptr = nullptr;                 // separate prompt tokens (CSR), or none
  const int32_t* p_tokens = nullptr;
  int64_t p_nnz = 0;
  const int32_t* slot = nullptr;
  sip::StateView state{};                            // valid when slot != nullptr
  int L_max = 0, slots = 0;
};

// Vocabulary shards of a call (sip_sample_sharded); t == 0: the logits are one matrix.
struct ShardSource {
  const void* const* base = nullptr;                 // host array of t device pointers
  int t = 0, V_shard = 0;
  int64_t stride = 0;
};

// A number for a call (Args::call_mark): never 0 in the upper 56 bits.
uint64_t new_call_mark() {
  static const uint64_t seed = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^
                               (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull ^
                               (uint64_t)reinterpret_cast<uintptr_t>(&g_dev) << 20;
  static std::atomic<uint64_t> calls{0};
  for (;;) {
    uint64_t x = seed + 0x9E3779B97F4A7C15ull * calls.fetch_add(1, std::memory_order_relaxed);
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x = (x ^ (x >> 31)) & ~255ull;
    if (x) return x;
  }
}

void set_cut(sip::Args& a, const Cut& c) {
  a.S = c.S; a.cap_c = c.cap_c; a.nc_cap = c.nc_cap;
  a.fin_tps = c.S > 0 ? sip::kFinThreads / c.S : sip::kFinThreads;
  a.fin_inv = (65536 + a.fin_tps - 1) / a.fin_tps;
}

template <bool SH>
sip_status launch(const sip::Args& a, int32_t B, int dtype, const Plan& plan, bool state, sip::StateHeader* head,
                  unsigned long long* tick_room, hipStream_t stream);

// Where both ways serve a row (16384 to 32768 entries): whether it is held in registers.  That takes
// a compute unit for a row and 9 to 34 us, whatever the row's filters keep; a batch of more rows than
// compute units takes as many rounds of it.  The streaming and finishing kernels overlap their rows,
// but pay for a row that its list does not settle: a nucleus that outgrows it, or queues that overflow
// (bf16 rows of one chunk under a wide min-p).  Which rows are like that, or greedy, is not known here;
// which parameters the call has is.  us, by streaming / in registers (fp32 unless said, 256 compute units,
// the present kernels on both sides; normal logits of standard deviation 2.5 unless said; "Student-t" has a spike a row):
//   up to one row per compute unit, V = 32768, 64 rows: greedy 15 / 10; no filter 22 / 12.5; min-p 20 / 13;
//   top-k and top-p 18.5 / 21; top-p, peaked rows 22 / 22, Student-t 18 / 16; all parameters, 512 tokens of history,
//   best 20: 25 / 32, V = 24000 bf16, 256 rows 25 / 28.  16 rows, whose chunks one kernel streams and finishes: greedy 13.5 / 10,
//   no filter 20 / 12, min-p 17.5 / 13, top-k and top-p 17 / 21, top-p, peaked 20 / 22, Student-t 17 / 16, all parameters
//   23.5 / 32.
//   V = 32000, rows of all four modes (greedy, top-k, top-p 0.9, min-p), 256 tokens of history, best 5: normal logits, whose
//   nuclei outgrow their lists, 4 to 64 rows 65 to 73 / 27; Student-t 17 to 19 / 30.
//   So: in registers, up to a third slower on rows that a list settles (up to three quarters with best-n
//   beside a spike) and several times faster where one of them is not; but rows without any filter that ask for best-n,
//   which are always settled from a list, by streaming: V = 32768, 64 rows, best 5, greedy 16 / 15 normal, 16 / 24 Student-t;
//   sampled 22 / 17.5, 22 / 27.
//   V = 24000, 2048 rows: greedy 74 / 75; no filter 106 / 93; min-p 93.5 / 99, V = 32000 and 512 tokens
//   of history 111 / 143, 600 rows of it 49 / 54; top-k and top-p 87 / 150; top-p, peaked 107 / 144.
//   So: in registers without a filter, min-p alone up to three rounds.
bool resident_is_chosen(const sip_params& params, int32_t k_lp, int32_t B, bool state, int compute_units) {
  // A state's call would have to take its number in a launch of its own before this kernel (the
  // streaming kernel does it in passing): bf16 V = 28532, 4 rows, hand-off: 56.8 us an iteration
  // against 53.4; V = 28092, 13 rows: 59.3 against 53.7.
  if (state) return false;
  const bool top = params.top_k || params.top_p, best = k_lp > 0;
  if (B <= compute_units) return top || params.min_p || !best;
  return !top && !best && (!params.min_p || B <= 3 * compute_units);
}

// Whether a row's workgroup streams and finishes it (sip_row.h) or the row is streamed in chunks for the
// finishing kernel.  A row to a workgroup pays the set-up once and overlaps one row's finishing with
// another's streaming, or at least needs no second kernel; but up to one row per compute unit it leaves
// chip idle that chunks would use, and beyond that the rows come in rounds of two per compute unit.
// us a call in chunks for two kernels / a row to a workgroup (256 compute units; nucleus 0.95, Student-t, 600 tokens):
//   V = 40000 bf16 (80 KB): 64 rows 19.7 / 20.1, 96 21.0 / 20.2, 256 25.0 / 20.9; fp32 (160 KB): 96 21.6 / 21.5, 128
//   22.0 / 21.8
//   V = 128256 bf16 (256 KB): 128 26.3 / 28.0, 144 28.1 / 28.1, 176 30.0 / 28.3, 256 32.5 / 28.7
//   V = 128256 fp32 (513 KB): 160 29.3 / 32.4, 192 31.8 / 32.5, 200 33.4 / 33.0, 256 36.8 / 35.6
//   V = 200000 bf16 (400 KB): 144 31.2 / 33.3, 192 33.4 / 33.7, 224 36.6 / 33.7; fp32 (800 KB): 160 35.9 / 40.1, 192
//   41.0 / 40.8, 224 49.5 / 45.0 (without a filter 192 rows 38.1 / 39.8 bf16, 44.6 / 50.6 fp32; 224 always a row to a
//   workgroup)
//   V = 110000 bf16 380 rows 41.2 / 41.2, fp32 53.7 / 52.4; V = 152064 bf16 300 44.5 / 46.6, 380 49.8 / 46.9, fp32
//   380 72.4 / 65.1; V = 230000 fp32 380 95.4 / 92.6
//   V = 100000 and 200000, both types: 520 rows 8 % more to 4 % less, 600 2 % more
//   to 8 % less, 700 and 1030 2 to 17 % less.
// So up to one row per compute unit from a number of rows on that grows with the row's bytes, to 3/4 of
// the compute units (where three chunks to a compute unit no longer fit the batch); above, not in the first
// part of a round -- unless the row is short -- but in the third and later rounds always.  A state's call
// would have to take its number in a launch of its own ahead of it: with 600 tokens a slot, V = 152064, 128
// rows 34.6 / 38.9 bf16, 35.2 / 44.2 fp32; 256 41.6 / 40.5, 46.3 / 46.4; 520 76.2 / 77.8, 99.7 / 102.7; 1030 130.9
// / 120.4, 181.9 / 167.5.  (The line is on the safe side: 700 rows 88.7 / 79.9, 121.4 / 110.3; V = 40000 bf16, 512 rows
// 43.1 / 40.1.)
bool row_is_chosen(int32_t B, int32_t V, int dtype, bool state, int compute_units) {
  const int64_t row_bytes = (int64_t)V * (dtype == SIP_F32 ? 4 : 2), cu = compute_units;
  if (state) return B >= 4 * cu;
  if (B <= cu) return B > std::min(cu * 3 / 4, cu * 3 / 16 + row_bytes / 2200);
  if (row_bytes <= 200 * 1024) return true;
  return B <= 2 * cu ? B >= cu * 23 / 16 : B >= cu * 75 / 32;
}

// Whether a call's rows are greedy ones of which only the ids are wanted, as far as can be told here: no filter is handed in, and
// no log-probabilities are asked for.  (Rows sampled without any filter look the same, and beyond 32 of them pay with two batches in
// flight for what greedy ones gain: us a call, two kernels / one, one batch; two: 64 rows of V = 128256 bf16 24.5 / 23.7; 15.1 / 20.5, fp32
// 26.7 / 26.1; 18.0 / 21.8.)
bool greedy_ids(const sip_params& params, int32_t k_lp) { return k_lp < 0 && !params.top_k && !params.top_p && !params.min_p; }

// The kernels of a call, and how its rows are cut where they are cut at all.
struct Way {
  sip_route route;
  const Cut* cut = nullptr;
};
// A batch of no more rows than the device has compute units, in chunks or a row to a workgroup: the workgroup that finishes
// a row also takes it through the heavier logic if the list does not settle it (sip_fused.h).  Larger batches: the lean kernel,
// two workgroups per compute unit, and a small fixed grid behind it for the rows (normally none) that need more.
Way choose_way(const Plan& plan, const sip_params& params, int32_t k_lp, int32_t B, int32_t V, int dtype, bool state, int compute_units) {
  if (V <= kResidentMaxV && (!plan.fast || resident_is_chosen(params, k_lp, B, state, compute_units))) return {SIP_ROUTE_RESIDENT};
  if (!plan.fast) return {SIP_ROUTE_EXACT};
  const bool fused = B <= compute_units && (size_t)plan.final_lds <= sip::kFusedRawBytes &&
                     2 * (((size_t)V + 31) / 32) * sizeof(uint32_t) <= sip::kFusedRawBytes;
  // (Where a row would have a workgroup of its own if it were not for chunks on a compute unit each -- 80 to 128 short rows of
  // which the ids are asked for --, it has: greedy ones, chunks / a row to a workgroup, recorded calls, one batch; two in flight, V = 33000
  // bf16 86 rows 7.0 / 5.1; 4.5 / 2.8, V = 40000 128 rows bf16 6.8 / 5.3; 5.2 / 3.1, fp32 6.9 / 5.4; 6.1 / 4.0, V = 60000 bf16 7.1 / 5.9; 5.5 / 3.4;
  // sampled ones V = 40000 fp32 23.8 / 24.8; 20.2 / 13.8.)
  if (row_is_chosen(B, V, dtype, state, compute_units)) return {fused ? SIP_ROUTE_ROW_FUSED : SIP_ROUTE_ROW};
  const Cut& each = greedy_ids(params, k_lp) && !plan.beside.S ? plan.alone : plan.beside;
  if (each.S && fused && !state) return {SIP_ROUTE_CHUNKS_ALONE, &each};
  return {fused ? SIP_ROUTE_CHUNKS_FUSED : SIP_ROUTE_CHUNKS, &plan.cut};
}

// Argument checks common to the entry points, workspace carving and the kernel launches.
sip_status sample_impl(const void* logits, int32_t B, int32_t V, int64_t row_stride, sip_dtype dtype,
                       const sip_params* params, const HistSource& h, uint64_t seed, uint64_t step,
                       int32_t* out_ids, int32_t* out_lp_ids, float* out_lp, int32_t k_logprobs, void* workspace,
                       size_t workspace_bytes, hipStream_t stream, const ShardSource& sh = ShardSource{}) {
  if (!shape_ok(B, V, (int)dtype, h.nnz, k_logprobs) || h.p_nnz < 0) return SIP_ERR_INVALID_ARG;
  if (!out_ids) return SIP_ERR_INVALID_ARG;
  if ((k_logprobs >= 0) != (out_lp_ids != nullptr) || (k_logprobs >= 0) != (out_lp != nullptr))
    return SIP_ERR_INVALID_ARG;
  const size_t esz = dtype == SIP_F32 ? 4 : 2;
  if (sh.t == 0) {
    if (!logits || row_stride < V) return SIP_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(logits) & 15u) != 0 || ((size_t)row_stride * esz) % 16 != 0)
      return SIP_ERR_INVALID_ARG;
  } else {
    if (!sh.base || sh.stride < sh.V_shard) return SIP_ERR_INVALID_ARG;
    if (((size_t)sh.V_shard * esz) % 16 != 0 || ((size_t)sh.stride * esz) % 16 != 0) return SIP_ERR_INVALID_ARG;
    for (int i = 0; i < sh.t; ++i)
      if (!sh.base[i] || (reinterpret_cast<uintptr_t>(sh.base[i]) & 15u) != 0) return SIP_ERR_INVALID_ARG;
  }
  if (B > SIP_MAX_B || V > SIP_MAX_V || k_logprobs > SIP_MAX_K_LOGPROBS) return SIP_ERR_UNSUPPORTED;
  const Plan plan = plan_for(B, V, (int)dtype, sh.t, h.nnz + h.p_nnz, sh.t ? (size_t)V * esz : 0);
  const Layout lay = make_layout(B, plan, h.nnz + h.p_nnz, sh.t ? (size_t)V * esz : 0);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0 || workspace_bytes < lay.total)
    return SIP_ERR_WORKSPACE;

  sip::Args a;
  a.logits = logits;
  a.B = B; a.V = V; a.row_stride = row_stride;
  for (int i = 0; i < 8; ++i) a.shard[i] = nullptr;
  a.t_shards = 1; a.V_shard = V; a.shard_stride = row_stride;
  if (sh.t) {
    // whole-row code paths read the row from the workspace, where its workgroup puts it together first
    a.logits = static_cast<char*>(workspace) + lay.gather;
    a.row_stride = V;
    for (int i = 0; i < sh.t; ++i) a.shard[i] = sh.base[i];
    a.t_shards = sh.t; a.V_shard = sh.V_shard; a.shard_stride = sh.stride;
  }
  a.inv_V_shard = 1.0f / (float)a.V_shard;
  {
    const int epl = dtype == SIP_F32 ? 4 : 8, unit = sip::kWave * epl;
    const int nsb = sip::kSampleSize / (sip::kStreamThreads * epl) * sip::kStreamWaves;   // sample blocks per row
    a.smp_bps = (nsb + a.t_shards - 1) / a.t_shards;
    a.smp_inv = (65536 + a.smp_bps - 1) / a.smp_bps;
    a.smp_step = a.V_shard / a.smp_bps / unit * unit;
  }
  if (params) a.p = *params; else a.p = sip_params{};
  a.indptr = reinterpret_cast<const long long*>(h.indptr);
  a.tokens = h.tokens;
  a.nnz = h.slot ? (long long)h.slots * h.L_max : ((h.indptr && h.tokens) ? h.nnz : 0);
  a.p_indptr = reinterpret_cast<const long long*>(h.p_indptr);
  a.p_tokens = h.p_tokens;
  a.p_nnz = (h.p_indptr && h.p_tokens) ? h.p_nnz : 0;
  a.slot = h.slot; a.L_max = h.L_max; a.slots = h.slots;
  a.st_len = h.state.len; a.st_ndist = h.state.ndist; a.st_tokens = h.state.tokens; a.st_table = h.state.table;
  a.st_tick = h.slot ? &h.state.head->tick : nullptr;
  a.st_overflow = h.slot ? &h.state.head->overflow : nullptr;
  a.call_tick = nullptr;
  a.seed = seed; a.step = step;
  a.out_ids = out_ids; a.out_lp_ids = out_lp_ids; a.out_lp = out_lp; a.k_lp = k_logprobs;
  char* ws = static_cast<char*>(workspace);
  a.row_path = reinterpret_cast<int*>(ws + lay.row_path);
  a.side_z = reinterpret_cast<float*>(ws + lay.side_z);
  a.side_c = reinterpret_cast<unsigned int*>(ws + lay.side_c);
  a.rowinfo = reinterpret_cast<sip::RowInfo*>(ws + lay.rowinfo);
  a.chunks = reinterpret_cast<sip::ChunkOut*>(ws + lay.chunks);
  a.cand = reinterpret_cast<uint2*>(ws + lay.cand);
  a.bf16 = dtype == SIP_BF16;
  set_cut(a, plan.cut);
  a.row_why = a.row_path + B;
  a.one_seg = 0;
  a.call_mark = 0;

  sip::StateHeader* head = h.slot ? h.state.head : nullptr;
  unsigned long long* const tick_room = reinterpret_cast<unsigned long long*>(ws + lay.tick);     // room for a.call_tick
  return sh.t ? launch<true>(a, B, (int)dtype, plan, h.slot != nullptr, head, tick_room, stream)
              : launch<false>(a, B, (int)dtype, plan, h.slot != nullptr, head, tick_room, stream);
}

template <bool SH>
sip_status launch(const sip::Args& a_in, int32_t B, int dtype, const Plan& plan, bool state, sip::StateHeader* head,
                  unsigned long long* tick_room, hipStream_t stream) {
  const DeviceSetup* dev = device_setup();
  if (!dev) return SIP_ERR_HIP;
  sip::Args a = a_in;
  hipEvent_t ev[6];
  for (int i = 0; i < 6; ++i) { ev[i] = g_prof[i]; g_prof[i] = nullptr; }
  const bool timed = ev[0] || ev[1] || ev[2] || ev[3] || ev[4] || ev[5];
  const Way way = choose_way(plan, a.p, a.k_lp, B, a.V, dtype, state, dev->compute_units);
  if (way.route == SIP_ROUTE_RESIDENT) {
    // a workgroup holds its whole row in registers: one kernel
    if (state) {
      a.call_tick = tick_room;
      hipLaunchKernelGGL(sip::state_take_tick_kernel, dim3(1), dim3(64), 0, stream, head, a.call_tick);
    }
    const bool f32 = dtype == SIP_F32;
    auto kern = a.V <= 4096    ? (f32 ? sip::resident_kernel<SIP_F32, 512, 8> : sip::resident_kernel<SIP_BF16, 512, 8>)
                : a.V <= 8192  ? (f32 ? sip::resident_kernel<SIP_F32, 1024, 8> : sip::resident_kernel<SIP_BF16, 1024, 8>)
                : a.V <= 16384 ? (f32 ? sip::resident_kernel<SIP_F32, 1024, 16> : sip::resident_kernel<SIP_BF16, 1024, 16>)
                               : (f32 ? sip::resident_kernel<SIP_F32, 1024, 32> : sip::resident_kernel<SIP_BF16, 1024, 32>);
    const dim3 threads(a.V <= 4096 ? 512 : 1024);
    if (timed) {
      hipExtLaunchKernelGGL(kern, dim3(B), threads, 0, stream, ev[0], ev[1], 0, a);
      for (int i = 2; i < 6; ++i)
        if (ev[i]) (void)hipEventRecord(ev[i], stream);     // no second and third kernel: empty intervals
    } else {
      hipLaunchKernelGGL(kern, dim3(B), threads, 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
  }
  const size_t words = ((size_t)a.V + 31) / 32;
  if (way.route == SIP_ROUTE_EXACT) {
    // every row takes the exact multi-pass path
    const size_t dyn = 2 * words * sizeof(uint32_t);
    auto kern = dtype == SIP_F32 ? sip::exact_kernel<SIP_F32, SH> : sip::exact_kernel<SIP_BF16, SH>;
    hipLaunchKernelGGL(kern, dim3(B), dim3(sip::kExactThreads), dyn, stream, a);
    if (hipGetLastError() != hipSuccess) return SIP_ERR_HIP;
    if (state) {
      hipLaunchKernelGGL(sip::state_tick_kernel, dim3(1), dim3(64), 0, stream, head);
      if (hipGetLastError() != hipSuccess) return SIP_ERR_HIP;
    }
    return SIP_OK;
  }
  a.call_tick = state ? tick_room : nullptr;   // the streaming kernel takes the state's counter and leaves it here
  const bool ids = a.k_lp < 0;                   // token ids only
  auto k_stream = dtype == SIP_F32 ? (ids ? sip::stream_kernel<SIP_F32, SH, true> : sip::stream_kernel<SIP_F32, SH, false>)
                                   : (ids ? sip::stream_kernel<SIP_BF16, SH, true> : sip::stream_kernel<SIP_BF16, SH, false>);
  auto k_rescue = dtype == SIP_F32 ? sip::rescue_kernel<SIP_F32, SH> : sip::rescue_kernel<SIP_BF16, SH>;
  const size_t dyn = std::max(plan.final_lds, 2 * words * sizeof(uint32_t));
  // A row streamed and finished by one workgroup, or the pass over the logits in chunks, then one
  // workgroup per row on what it left.
  if (way.route == SIP_ROUTE_CHUNKS_ALONE) {
    // a compute unit for every chunk: streaming, finishing and the heavier logic in one kernel
    a.call_mark = new_call_mark();
    set_cut(a, *way.cut);
    auto k_alone = dtype == SIP_F32 ? (ids ? sip::chunk_rescue_kernel<SIP_F32, SH, true> : sip::chunk_rescue_kernel<SIP_F32, SH, false>)
                                    : (ids ? sip::chunk_rescue_kernel<SIP_BF16, SH, true> : sip::chunk_rescue_kernel<SIP_BF16, SH, false>);
    if (timed) {
      hipExtLaunchKernelGGL(k_alone, dim3(B * a.S), dim3(sip::kStreamThreads), 0, stream, ev[0], ev[1], 0, a);
      for (int i = 2; i < 6; ++i)
        if (ev[i]) (void)hipEventRecord(ev[i], stream);       // one kernel: empty intervals
    } else {
      hipLaunchKernelGGL(k_alone, dim3(B * a.S), dim3(sip::kStreamThreads), 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
  }
  a.one_seg = way.route == SIP_ROUTE_ROW_FUSED || way.route == SIP_ROUTE_ROW;
  if (a.one_seg) {
    // the row's workgroup streams and finishes it, and the rescue kernel is behind it
    a.S = plan.room; a.cap_c = sip::kChunkCap;       // (one segment of them all)
    a.nc_cap = std::min(sip::kFinalThreads * sip::kCandLong, a.S * a.cap_c);
    if (state) hipLaunchKernelGGL(sip::state_take_tick_kernel, dim3(1), dim3(64), 0, stream, head, a.call_tick);
    if (way.route == SIP_ROUTE_ROW_FUSED) {
      auto k_both = dtype == SIP_F32 ? (ids ? sip::row_rescue_kernel<SIP_F32, SH, true> : sip::row_rescue_kernel<SIP_F32, SH, false>)
                                     : (ids ? sip::row_rescue_kernel<SIP_BF16, SH, true> : sip::row_rescue_kernel<SIP_BF16, SH, false>);
      if (timed) {
        hipExtLaunchKernelGGL(k_both, dim3(B), dim3(sip::kStreamThreads), 0, stream, ev[0], ev[1], 0, a);
        for (int i = 2; i < 6; ++i)
          if (ev[i]) (void)hipEventRecord(ev[i], stream);     // one kernel: empty intervals
      } else {
        hipLaunchKernelGGL(k_both, dim3(B), dim3(sip::kStreamThreads), 0, stream, a);
      }
      return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
    }
    auto k_row = dtype == SIP_F32 ? (ids ? sip::row_kernel<SIP_F32, SH, true> : sip::row_kernel<SIP_F32, SH, false>)
                                  : (ids ? sip::row_kernel<SIP_BF16, SH, true> : sip::row_kernel<SIP_BF16, SH, false>);
    const int n_rescue_wg = std::min<int>(B, kRescueGrid);
    if (timed) {
      hipExtLaunchKernelGGL(k_row, dim3(B), dim3(sip::kStreamThreads), 0, stream, ev[0], ev[1], 0, a);
      for (int i = 2; i < 4; ++i)
        if (ev[i]) (void)hipEventRecord(ev[i], stream);       // no finishing kernel: an empty interval
      hipExtLaunchKernelGGL(k_rescue, dim3(n_rescue_wg), dim3(sip::kFinalThreads), dyn, stream, ev[4], ev[5], 0, a);
    } else {
      hipLaunchKernelGGL(k_row, dim3(B), dim3(sip::kStreamThreads), 0, stream, a);
      hipLaunchKernelGGL(k_rescue, dim3(n_rescue_wg), dim3(sip::kFinalThreads), dyn, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
  }
  const uint32_t stream_lds = (uint32_t)(dtype == SIP_F32 ? sip::stream_lds_bytes<SIP_F32>(a.cap_c / sip::kStreamWaves)
                                                        : sip::stream_lds_bytes<SIP_BF16>(a.cap_c / sip::kStreamWaves));
  if (timed) hipExtLaunchKernelGGL(k_stream, dim3(B * a.S), dim3(sip::kStreamThreads), stream_lds, stream, ev[0], ev[1], 0, a);
  else hipLaunchKernelGGL(k_stream, dim3(B * a.S), dim3(sip::kStreamThreads), stream_lds, stream, a);
  if (way.route == SIP_ROUTE_CHUNKS_FUSED) {
    auto k_fused = dtype == SIP_F32 ? sip::finish_rescue_kernel<SIP_F32, SH> : sip::finish_rescue_kernel<SIP_BF16, SH>;
    if (timed) {             // the events take the dispatches' own begin / end time stamps
      hipExtLaunchKernelGGL(k_fused, dim3(B), dim3(sip::kFinalThreads), 0, stream, ev[2], ev[3], 0, a);
      if (ev[4]) (void)hipEventRecord(ev[4], stream);       // no third kernel: an empty interval
      if (ev[5]) (void)hipEventRecord(ev[5], stream);
    } else {
      hipLaunchKernelGGL(k_fused, dim3(B), dim3(sip::kFinalThreads), 0, stream, a);
    }
  } else {
    const int n_rescue_wg = std::min<int>(B, kRescueGrid);
    if (timed) {
      hipExtLaunchKernelGGL(sip::finish_kernel, dim3(B), dim3(sip::kFinThreads), 0, stream, ev[2], ev[3], 0, a);
      hipExtLaunchKernelGGL(k_rescue, dim3(n_rescue_wg), dim3(sip::kFinalThreads), dyn, stream, ev[4], ev[5], 0, a);
    } else {
      hipLaunchKernelGGL(sip::finish_kernel, dim3(B), dim3(sip::kFinThreads), 0, stream, a);
      hipLaunchKernelGGL(k_rescue, dim3(n_rescue_wg), dim3(sip::kFinalThreads), dyn, stream, a);
    }
  }
  if (hipGetLastError() != hipSuccess) return SIP_ERR_HIP;
  return SIP_OK;
}

bool state_shape_ok(int32_t slots, int32_t L_max) {
  return slots > 0 && L_max > 0 && slots <= SIP_MAX_SLOTS && L_max <= SIP_MAX_L;
}
bool state_ok(const void* state, size_t state_bytes, int32_t slots, int32_t L_max) {
  return state && (reinterpret_cast<uintptr_t>(state) & (kAlign - 1)) == 0 &&
         state_bytes >= sip::state_total(slots, L_max);
}

}  // namespace

extern "C" {

size_t sip_workspace_bytes(int32_t B, int32_t V, sip_dtype dtype, int64_t hist_nnz, int32_t k_logprobs) {
  if (!shape_ok(B, V, (int)dtype, hist_nnz, k_logprobs)) return 0;
  if (B > SIP_MAX_B || V > SIP_MAX_V || k_logprobs > SIP_MAX_K_LOGPROBS) return 0;
  return workspace_need(B, V, (int)dtype, 0, hist_nnz);
}

sip_status sip_sample(const void* logits, int32_t B, int32_t V, int64_t row_stride, sip_dtype dtype,
                      const sip_params* params, const int64_t* hist_indptr, const int32_t* hist_tokens,
                      int64_t hist_nnz, uint64_t seed, uint64_t step, int32_t* out_ids, int32_t* out_lp_ids,
                      float* out_lp, int32_t k_logprobs, void* workspace, size_t workspace_bytes,
                      void* hip_stream) {
  if (hist_nnz > 0 && (!hist_indptr || !hist_tokens)) return SIP_ERR_INVALID_ARG;
  HistSource h;
  h.indptr = hist_indptr; h.tokens = hist_tokens; h.nnz = hist_nnz;
  return sample_impl(logits, B, V, row_stride, dtype, params, h, seed, step, out_ids, out_lp_ids, out_lp,
                     k_logprobs, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

sip_status sip_init(void) { return device_setup() ? SIP_OK : SIP_ERR_HIP; }

size_t sip_noalloc_scratch_bytes(void) { return kNoallocBytes; }

sip_status sip_sample_noalloc(const void* logits, int32_t B, int32_t V, int64_t row_stride, sip_dtype dtype,
                              const sip_params* params, const int64_t* hist_indptr, const int32_t* hist_tokens,
                              int64_t hist_nnz, uint64_t seed, uint64_t step, int32_t* out_ids,
                              int32_t* out_lp_ids, float* out_lp, int32_t k_logprobs, void* hip_stream) {
  if (!logits || !out_ids) return SIP_ERR_INVALID_ARG;     // (the rest is checked by sample_impl, before anything is enqueued)
  if (hist_nnz > 0 && (!hist_indptr || !hist_tokens)) return SIP_ERR_INVALID_ARG;
  if (!shape_ok(B, V, (int)dtype, hist_nnz, k_logprobs)) return SIP_ERR_INVALID_ARG;
  if (B > SIP_MAX_B || V > SIP_MAX_V || k_logprobs > SIP_MAX_K_LOGPROBS) return SIP_ERR_UNSUPPORTED;
  const size_t need = make_layout(B, plan_for(B, V, (int)dtype, 0, hist_nnz), hist_nnz).total;
  if (need > kNoallocBytes) return SIP_ERR_SCRATCH;
  DeviceSetup* d = device_setup();                 // the current device's copy of the array
  if (!d) return SIP_ERR_HIP;
  // Nothing in the workspace has to start at zero: every kernel writes what it later reads.
  HistSource h;
  h.indptr = hist_indptr; h.tokens = hist_tokens; h.nnz = hist_nnz;
  return sample_impl(logits, B, V, row_stride, dtype, params, h, seed, step, out_ids, out_lp_ids, out_lp,
                     k_logprobs, d->scratch_ptr, kNoallocBytes, static_cast<hipStream_t>(hip_stream));
}

size_t sip_workspace_bytes_sharded(int32_t B, int32_t V_shard, int32_t t, sip_dtype dtype, int64_t hist_nnz,
                                   int32_t k_logprobs) {
  if (t < 1 || t > SIP_MAX_SHARDS || V_shard <= 0 || (int64_t)V_shard * t > SIP_MAX_V || B > SIP_MAX_B) return 0;
  const int32_t V = V_shard * t;
  if (!shape_ok(B, V, (int)dtype, hist_nnz, k_logprobs) || k_logprobs > SIP_MAX_K_LOGPROBS) return 0;
  const size_t row_bytes = (size_t)V * (dtype == SIP_F32 ? 4 : 2);
  return workspace_need(B, V, (int)dtype, t, hist_nnz, row_bytes);
}

sip_status sip_sample_sharded(const void* const* shard_logits, int32_t t, int32_t B, int32_t V_shard,
                              int64_t shard_stride, sip_dtype dtype, const sip_params* params,
                              const int64_t* hist_indptr, const int32_t* hist_tokens, int64_t hist_nnz,
                              uint64_t seed, uint64_t step, int32_t* out_ids, int32_t* out_lp_ids, float* out_lp,
                              int32_t k_logprobs, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (t < 1 || t > SIP_MAX_SHARDS || V_shard <= 0 || !shard_logits) return SIP_ERR_INVALID_ARG;
  if ((int64_t)V_shard * t > SIP_MAX_V || B > SIP_MAX_B) return SIP_ERR_UNSUPPORTED;
  if (hist_nnz > 0 && (!hist_indptr || !hist_tokens)) return SIP_ERR_INVALID_ARG;
  HistSource h;
  h.indptr = hist_indptr; h.tokens = hist_tokens; h.nnz = hist_nnz;
  ShardSource sh;
  sh.base = shard_logits; sh.t = t; sh.V_shard = V_shard; sh.stride = shard_stride;
  return sample_impl(nullptr, B, V_shard * t, 0, dtype, params, h, seed, step, out_ids, out_lp_ids, out_lp,
                     k_logprobs, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream), sh);
}

size_t sip_state_bytes(int32_t slots, int32_t L_max) {
  if (!state_shape_ok(slots, L_max)) return 0;
  return sip::state_total(slots, L_max);
}

sip_status sip_state_init(void* state, size_t state_bytes, int32_t slots, int32_t L_max, void* hip_stream) {
  if (!state_shape_ok(slots, L_max)) return SIP_ERR_INVALID_ARG;
  if (!state_ok(state, state_bytes, slots, L_max)) return SIP_ERR_WORKSPACE;
  const sip::StateView v = sip::state_view(state, slots, L_max);
  hipLaunchKernelGGL(sip::state_init_kernel, dim3(slots), dim3(sip::kStateThreads), 0,
                     static_cast<hipStream_t>(hip_stream), v.head, v.len, v.ndist, v.table, slots);
  return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
}

sip_status sip_state_assign(void* state, size_t state_bytes, int32_t slots, int32_t L_max, int32_t n,
                            const int32_t* slot_ids, const int64_t* indptr, const int32_t* tokens, int64_t nnz,
                            void* hip_stream) {
  if (!state_shape_ok(slots, L_max) || n < 0 || nnz < 0) return SIP_ERR_INVALID_ARG;
  if (n > 0 && !slot_ids) return SIP_ERR_INVALID_ARG;
  if (nnz > 0 && (!indptr || !tokens)) return SIP_ERR_INVALID_ARG;
  if (!state_ok(state, state_bytes, slots, L_max)) return SIP_ERR_WORKSPACE;
  if (n == 0) return SIP_OK;
  const sip::StateView v = sip::state_view(state, slots, L_max);
  hipLaunchKernelGGL(sip::state_assign_kernel, dim3(n), dim3(sip::kStateThreads), 0,
                     static_cast<hipStream_t>(hip_stream), v.head, v.len, v.ndist, v.tokens, v.table, slots, L_max, slot_ids,
                     reinterpret_cast<const long long*>(indptr), tokens, (long long)nnz);
  return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
}

sip_status sip_sample_state(const void* logits, int32_t B, int32_t V, int64_t row_stride, sip_dtype dtype,
                            const sip_params* params, void* state, size_t state_bytes, int32_t slots,
                            int32_t L_max, const int32_t* slot_of_row, uint64_t seed, uint64_t step,
                            int32_t* out_ids, int32_t* out_lp_ids, float* out_lp, int32_t k_logprobs,
                            void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!state_shape_ok(slots, L_max) || !slot_of_row || B <= 0) return SIP_ERR_INVALID_ARG;
  if (!state_ok(state, state_bytes, slots, L_max)) return SIP_ERR_WORKSPACE;
  HistSource h;
  h.state = sip::state_view(state, slots, L_max);
  h.tokens = h.state.tokens; h.nnz = (int64_t)B * L_max;
  h.slot = slot_of_row; h.L_max = L_max; h.slots = slots;
  // the kernels append the ids to the slots and count the call themselves
  return sample_impl(logits, B, V, row_stride, dtype, params, h, seed, step, out_ids, out_lp_ids, out_lp,
                     k_logprobs, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

namespace {
// Checks of a sip_call that sample_impl does not make, and its two sources.
sip_status call_sources(const sip_call* c, HistSource& h, ShardSource& sh, int32_t& V) {
  if (!c || c->B <= 0) return SIP_ERR_INVALID_ARG;
  if (c->t_shards < 0 || c->t_shards > SIP_MAX_SHARDS) return SIP_ERR_INVALID_ARG;
  if (c->t_shards > 0) {
    if (c->V_shard <= 0 || !c->shard_logits) return SIP_ERR_INVALID_ARG;
    if ((int64_t)c->V_shard * c->t_shards > SIP_MAX_V || c->B > SIP_MAX_B) return SIP_ERR_UNSUPPORTED;
    sh.base = c->shard_logits; sh.t = c->t_shards; sh.V_shard = c->V_shard; sh.stride = c->shard_stride;
    V = c->V_shard * c->t_shards;
  } else {
    V = c->V;
  }
  if (c->state) {
    if (c->hist_indptr || c->hist_tokens || c->hist_nnz != 0) return SIP_ERR_INVALID_ARG;   // one source of history
    if (!state_shape_ok(c->slots, c->L_max) || !c->slot_of_row) return SIP_ERR_INVALID_ARG;
    if (!state_ok(c->state, c->state_bytes, c->slots, c->L_max)) return SIP_ERR_WORKSPACE;
    h.state = sip::state_view(c->state, c->slots, c->L_max);
    h.tokens = h.state.tokens; h.nnz = (int64_t)c->B * c->L_max;
    h.slot = c->slot_of_row; h.L_max = c->L_max; h.slots = c->slots;
  } else {
    if (c->hist_nnz < 0 || (c->hist_nnz > 0 && (!c->hist_indptr || !c->hist_tokens))) return SIP_ERR_INVALID_ARG;
    h.indptr = c->hist_indptr; h.tokens = c->hist_tokens; h.nnz = c->hist_nnz;
  }
  if (c->prompt_nnz < 0 || (c->prompt_nnz > 0 && (!c->prompt_indptr || !c->prompt_tokens))) return SIP_ERR_INVALID_ARG;
  if (c->prompt_nnz > 0 && c->state) return SIP_ERR_INVALID_ARG;      // a state's slots hold prompt and output as one history
  h.p_indptr = c->prompt_indptr; h.p_tokens = c->prompt_tokens; h.p_nnz = c->prompt_nnz;
  if ((c->host_ids != nullptr) != (c->host_flag != nullptr)) return SIP_ERR_INVALID_ARG;
  if (c->host_flag && ((reinterpret_cast<uintptr_t>(c->host_flag) & 7u) != 0 ||
                       (reinterpret_cast<uintptr_t>(c->host_ids) & 3u) != 0))
    return SIP_ERR_INVALID_ARG;
  return SIP_OK;
}
}  // namespace

size_t sip_call_workspace_bytes(const sip_call* c) {
  HistSource h; ShardSource sh; int32_t V = 0;
  if (call_sources(c, h, sh, V) != SIP_OK) return 0;
  if (!shape_ok(c->B, V, (int)c->dtype, h.nnz, c->k_logprobs)) return 0;
  if (c->B > SIP_MAX_B || V > SIP_MAX_V || c->k_logprobs > SIP_MAX_K_LOGPROBS) return 0;
  const size_t esz = c->dtype == SIP_F32 ? 4 : 2;
  const size_t row_bytes = sh.t ? (size_t)V * esz : 0;
  return workspace_need(c->B, V, (int)c->dtype, sh.t, h.nnz + h.p_nnz, row_bytes);
}

sip_status sip_sample_call(const sip_call* c) {
  HistSource h; ShardSource sh; int32_t V = 0;
  const sip_status ok = call_sources(c, h, sh, V);
  if (ok != SIP_OK) return ok;
  hipStream_t stream = static_cast<hipStream_t>(c->hip_stream);
  const sip_status st = sample_impl(c->logits, c->B, V, c->row_stride, c->dtype, c->params, h, c->seed, c->step,
                                    c->out_ids, c->out_lp_ids, c->out_lp, c->k_logprobs, c->workspace,
                                    c->workspace_bytes, stream, sh);
  if (st != SIP_OK || !c->host_flag) return st;
  return sip_publish_ids(c->out_ids, c->B, c->host_ids, c->host_flag, c->ticket, c->hip_stream);
}

sip_status sip_publish_ids(const int32_t* ids, int32_t B, int32_t* host_ids, uint64_t* host_flag, uint64_t ticket,
                           void* hip_stream) {
  if (!ids || !host_ids || !host_flag || B <= 0) return SIP_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(host_flag) & 7u) != 0 || (reinterpret_cast<uintptr_t>(host_ids) & 3u) != 0)
    return SIP_ERR_INVALID_ARG;
  hipLaunchKernelGGL(sip::publish_kernel, dim3(1), dim3(sip::kPublishThreads), 0,
                     static_cast<hipStream_t>(hip_stream), ids, B, host_ids,
                     reinterpret_cast<unsigned long long*>(host_flag), (unsigned long long)ticket);
  return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
}

sip_status sip_wait_ids(const uint64_t* host_flag, uint64_t ticket, uint64_t timeout_ns) {
  if (!host_flag || (reinterpret_cast<uintptr_t>(host_flag) & 7u) != 0) return SIP_ERR_INVALID_ARG;
  const auto t0 = std::chrono::steady_clock::now();
  unsigned spins = 0;
  for (;;) {
    if (__atomic_load_n(host_flag, __ATOMIC_ACQUIRE) >= ticket) return SIP_OK;
    __builtin_ia32_pause();
    if ((++spins & 1023u) == 0 && timeout_ns != UINT64_MAX) {
      const auto dt = std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - t0);
      if ((uint64_t)dt.count() >= timeout_ns) return SIP_ERR_TIMEOUT;
    }
  }
}

sip_status sip_probe_read(const void* src, size_t bytes, int32_t workgroups, void* workspace,
                          size_t workspace_bytes, void* start_event, void* stop_event, void* hip_stream) {
  if (!src || bytes < 16 || workgroups <= 0 || workgroups > 65536) return SIP_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(src) & 15u) != 0) return SIP_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < (size_t)workgroups * sizeof(float)) return SIP_ERR_WORKSPACE;
  hipExtLaunchKernelGGL(sip::probe_read_kernel, dim3(workgroups), dim3(sip::kProbeThreads), 0,
                        static_cast<hipStream_t>(hip_stream), static_cast<hipEvent_t>(start_event),
                        static_cast<hipEvent_t>(stop_event), 0, static_cast<const uint4*>(src), bytes / 16,
                        (int)workgroups, static_cast<float*>(workspace));
  return hipGetLastError() == hipSuccess ? SIP_OK : SIP_ERR_HIP;
}

int32_t sip_plan_chunks(int32_t B, int32_t V, sip_dtype dtype, int32_t t_shards) {
  if (B <= 0 || B > SIP_MAX_B || V <= 0 || (dtype != SIP_F32 && dtype != SIP_BF16) || t_shards < 0 || t_shards > SIP_MAX_SHARDS) return -1;
  if (t_shards > 0 && V % t_shards != 0) return -1;
  const Plan p = make_plan(B, V, (int)dtype, t_shards);
  return p.fast ? p.cut.S : 0;
}

int32_t sip_call_route(int32_t B, int32_t V, sip_dtype dtype, int32_t t_shards, int32_t on_state, const sip_params* params,
                       int64_t hist_nnz, int32_t k_logprobs, int32_t compute_units, int32_t* chunks) {
  if (!shape_ok(B, V, (int)dtype, hist_nnz, k_logprobs) || B > SIP_MAX_B || V > SIP_MAX_V || k_logprobs > SIP_MAX_K_LOGPROBS) return -1;
  if (t_shards < 0 || t_shards > SIP_MAX_SHARDS || (t_shards > 0 && V % t_shards != 0) || compute_units < 0) return -1;
  const size_t gather = t_shards ? (size_t)V * (dtype == SIP_F32 ? 4 : 2) : 0;
  const Plan p = plan_for(B, V, (int)dtype, t_shards, hist_nnz, gather);
  const Way way = choose_way(p, params ? *params : sip_params{}, k_logprobs, B, V, (int)dtype, on_state != 0, compute_units ? compute_units : 256);
  if (chunks) *chunks = way.cut ? way.cut->S : 1;
  return way.route;
}

const char* sip_status_string(sip_status status) {
  switch (status) {
    case SIP_OK: return "ok";
    case SIP_ERR_INVALID_ARG: return "invalid argument";
    case SIP_ERR_UNSUPPORTED: return "unsupported shape";
    case SIP_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case SIP_ERR_HIP: return "HIP runtime error";
    case SIP_ERR_TIMEOUT: return "timed out";
    case SIP_ERR_SCRATCH: return "call needs more scratch than the library's built-in array holds";
  }
  return "unknown status";
}

void sip_profile_kernel_events(void* stream_start, void* stream_stop, void* finish_start, void* finish_stop,
                               void* rescue_start, void* rescue_stop) {
  g_prof[0] = static_cast<hipEvent_t>(stream_start);
  g_prof[1] = static_cast<hipEvent_t>(stream_stop);
  g_prof[2] = static_cast<hipEvent_t>(finish_start);
  g_prof[3] = static_cast<hipEvent_t>(finish_stop);
  g_prof[4] = static_cast<hipEvent_t>(rescue_start);
  g_prof[5] = static_cast<hipEvent_t>(rescue_stop);
}

int sip_version(void) { return 100; }

}  // extern "C"
