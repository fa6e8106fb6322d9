// Small vocabularies: one workgroup holds its whole row in registers and answers everything from
// there -- one kernel, one read of the logits, no list, no threshold estimate and no second look
// at memory whatever the row's filters keep.
//
// A thread owns NPT elements, loaded 16 bytes at a time, so that element order is (load, thread,
// element of the load).  Steps (Sec. 2.1 step 3; Sec. 5.1 ApplyPenalty / temperature / softmax /
// filters / draw), every sum an integer sum in units of 2^-40 of the maximum's mass:
//   (1) multiplicity of every token in the history: one 16-bit counter per vocabulary entry in
//       LDS (bit 15: the token is in the separate prompt); a thread reads the counters of its own
//       elements, penalises them in registers, no table to search;
//   (2) s = z'/tau, maximum, lowest finite value;
//   (3) mass of every element; count and mass per value bin (2048 linear bins between the maximum
//       and the lowest value, or 28 below the maximum, where masses are zero);
//   (4) one descending scan over the bins locates the bins of the k-th largest, of the n-th best
//       and of the nucleus cut; their members, gathered from the registers, are compared all
//       pairs;
//   (5) draw: mass kept per block of 64 lanes x one load (these are in vocabulary order), prefix
//       over the blocks, and the wave that holds the crossing finds it in its registers.
//
// What bounds it: vector issue of the one compute unit that has the row (16 waves, 4 to a SIMD, so
// an instruction per element costs V / 1024 x 16 cycles; 58 % of the slots at V = 32000) and the chain of
// its barriers.  Hence what is done once per row is done
// by one wave, parameters that are off take part with their neutral value instead of a branch,
// temperature and repetition penalty are products with a double reciprocal (RowDivisor), masses
// become integers through a double's low bits, and bins cost three instructions; with the
// straightforward forms of these V = 32000 took 34.5 us, then 25.3 (fp32, 4 rows, one of each kind
// of filter); with the block masses of a wave's loads added up together (row_sums_u64(): eight sums over 64 lanes
// one by one were a fifth of what a thread issues for the draw), min-p taken out of the masses once, and the
// gathering of a cut's members passing over loads whose largest value is below, 24.5.  Without a filter, V = 16000,
// 64 rows 13.7 -> 12.7, 1500 rows 81.4 -> 75.5; top-p 97.9 -> 95.3.  (Counting only bins that the k-th or n-th best
// can be in, by the least of 128 groups' maxima, made everything 1 to 5 % slower: the LDS additions are hidden, the
// test is not.)  Against exact_kernel, which vocabularies below 16384 used to go through: V = 4096, 64 rows, top-k
// and top-p: 53 -> 11 us; V = 12556, 468 rows, no filter: 99 -> 19 us.  Which of the larger ones come here:
// resident_is_chosen().
//
// What this cannot settle -- more than kResList members in a bin of a cut (all-equal rows), top_p <= 0,
// no finite maximum -- goes through exact_row() in the same workgroup.
#pragma once
#include "sip_device.h"
#include "sip_exact.h"
#include "sip_finish.h"
#include "sip_stream.h"

namespace sip {

constexpr int kResBins = 2048;
constexpr int kResList = 1024;             // members of a cut's bin / entries at or above the bin of the n-th best
constexpr int kResMaxCount = 32767;        // longest history that 15-bit counters hold whatever it repeats
constexpr uint32_t kResFold = 16384;       // longer ones: taken out of a count beyond it, and noted
constexpr float kResSpan = 28.6f;          // exp(-28.6) * 2^40 < 1/2: nothing further below the maximum has mass

template <int NT, int NPT>
struct __align__(16) ResShared {
  union {
    uint32_t cnt[NT * NPT / 2];            // two 16-bit counters per word, token 2i in the low half
    uint32_t dyn[NT * NPT / 16];           // exact_row(): bitmap and ranks
  } u;
  uint32_t hcnt[kResBins];                 // entries per bin
  uint32_t hoff[kResBins];                 // entries in all higher bins
  unsigned long long hmass[kResBins];      // mass per bin; after the scan: mass of all higher bins
  uint32_t a_key[kResList], a_idx[kResList];           // entries at or above the bin of the n-th best
  uint32_t m_key[kResList];                            // members of a cut's bin
  unsigned long long m_E[kResList];
  unsigned long long blk[NT * NPT / (kWave * 4)];      // kept mass per (load, wave)
  unsigned long long r64[16], r64b[16];
  uint32_t r32[16], rkey[16], rlow[16];
  uint32_t n_a, n_m, m_lo, m_hi, n_best, key_k, key_p;
  unsigned long long s1_part;
  int bin_k, bin_n, bin_p;
  uint32_t arg_max;
  float t_minp;
  double ln_z;
  unsigned long long j24;
  double recip[2];                          // of the temperature and of the repetition penalty
  ExactShared ex;
};

// Sums of N values over the 16 lanes of a DPP row: lane l has that of t[l % N].  Half of the values go to
// the other lane of a pair at each of the first steps, so that eight take 10 additions, not 32.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_mov_u64(unsigned long long v) {
  return ((unsigned long long)dpp_mov<CTRL, 0xf>(0u, (uint32_t)(v >> 32)) << 32) | dpp_mov<CTRL, 0xf>(0u, (uint32_t)v);
}
template <int CTRL, int HALF, int N>
__device__ __forceinline__ void halve_u64(unsigned long long (&t)[N], bool upper) {
#pragma unroll
  for (int j = 0; j < HALF; ++j) {
    const unsigned long long keep = upper ? t[j + HALF] : t[j], give = upper ? t[j] : t[j + HALF];
    t[j] = keep + dpp_mov_u64<CTRL>(give);
  }
}
template <int N>
__device__ __forceinline__ unsigned long long row_sums_u64(unsigned long long (&t)[N], int lane) {
  static_assert(N == 2 || N == 4 || N == 8, "");
  if constexpr (N >= 8) halve_u64<0x141, 4>(t, lane & 4);                      // from the other end of eight lanes
  if constexpr (N >= 4) halve_u64<0x4E, 2>(t, lane & 2);                       // lane ^ 2
  halve_u64<0xB1, 1>(t, lane & 1);                                             // lane ^ 1
  unsigned long long v = t[0] + dpp_mov_u64<0x128>(t[0]);                      // rotations by 8, 4, 2
  if constexpr (N <= 4) v += dpp_mov_u64<0x124>(v);
  if constexpr (N <= 2) v += dpp_mov_u64<0x122>(v);
  return v;
}

// `NT` threads, `NPT` elements each: V <= NT * NPT.
template <int DT, int NT, int NPT>
__global__ __launch_bounds__(NT) void resident_kernel(Args a_by_value) {
  (void)a_by_value;
  const Args& a = *(const Args*)__builtin_amdgcn_kernarg_segment_ptr();
  warm_kernel_arguments();
  constexpr int EPL = (DT == SIP_F32) ? 4 : 8;
  constexpr int ESZ = (DT == SIP_F32) ? 4 : 2;
  constexpr int NL = NPT / EPL;
  constexpr int NW = NT / kWave;
  constexpr int BPT = kResBins / NT;
  constexpr int NBLK = NL * NW;
  static_assert(NPT % EPL == 0 && NW <= 16 && NBLK <= 2 * kWave, "");
  __shared__ ResShared<NT, NPT> fs;
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
  const int b = blockIdx.x;
  const int V = a.V;
  const bool sharded = a.shard[0] != nullptr;          // uniform

  // ---- (0) the whole row is requested at once; the row's parameters and history extent meanwhile
  uint4 q[NL];
  {
    const int e_last = ((V - 1) / EPL) * EPL;
    if (!sharded) {
      const char* row = reinterpret_cast<const char*>(a.logits) + (size_t)b * (size_t)a.row_stride * ESZ;
#pragma unroll
      for (int j = 0; j < NL; ++j)
        q[j] = *reinterpret_cast<const uint4*>(row + (size_t)min((j * NT + tid) * EPL, e_last) * ESZ);
    } else {
      // a 16-byte load never straddles two pieces: V_shard * ESZ is a multiple of 16
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const int e0 = min((j * NT + tid) * EPL, e_last);
        int sh = (int)((float)e0 * a.inv_V_shard);
        sh += (sh + 1) * a.V_shard <= e0;
        sh -= sh * a.V_shard > e0;
        q[j] = *reinterpret_cast<const uint4*>(shard_base(a, sh) +
                                               ((size_t)b * (size_t)a.shard_stride + (size_t)(e0 - sh * a.V_shard)) * ESZ);
      }
    }
  }
  const RowParams rp = load_row_params(a, b);
  const PenaltyPlan pen = penalty_plan(a, b, rp.theta, rp.phi, rp.psi);
  const bool minp_on = !rp.greedy && rp.min_p > 0.0f;
  const bool k_act = !rp.greedy && rp.top_k >= 2 && rp.top_k < V;
  const bool p_act = !rp.greedy && rp.top_p < 1.0f;
  const uint32_t n_top = (uint32_t)max(0, min(a.k_lp, V));
  const bool bins_on = k_act || p_act || n_top > 0;
  {
    uint4* z4 = reinterpret_cast<uint4*>(fs.hcnt);
    if (bins_on)
      for (int i = tid; i < kResBins * 4 / 16; i += NT) z4[i] = make_uint4(0, 0, 0, 0);
    z4 = reinterpret_cast<uint4*>(fs.hmass);
    if (p_act)
      for (int i = tid; i < kResBins * 8 / 16; i += NT) z4[i] = make_uint4(0, 0, 0, 0);
    z4 = reinterpret_cast<uint4*>(fs.u.cnt);
    if (pen.any)
      for (int i = tid; i < NT * NPT * 2 / 16; i += NT) z4[i] = make_uint4(0, 0, 0, 0);
    if (NL > 1 && tid < NBLK) fs.blk[tid] = 0;
    if (tid == 0) {
      fs.n_a = 0; fs.n_m = 0; fs.m_lo = kFinNone; fs.m_hi = 0; fs.key_k = 0; fs.key_p = kFinNone; fs.s1_part = 0;
      fs.bin_k = -1; fs.bin_n = -1; fs.bin_p = 1 << 30; fs.arg_max = kFinNone;
    }
  }
  // (what is worked out once for the row is one wave's work: sixteen waves doing the same cost the
  // compute unit sixteen times its instructions)
  if (wave == NW - 1 && !rp.greedy) {
    const float t = minp_on ? (float)log((double)rp.min_p) : -INFINITY;
    const unsigned long long u = (unsigned long long)(philox_word0(a.seed, rp.row_id, step_of(a)) >> 8);
    if (lane == 0) { fs.t_minp = t; fs.j24 = u; }
  }
  if (wave == NW - 2) {
    const double r = 1.0 / (double)(lane == 0 ? (rp.greedy ? 1.0f : rp.tau) : rp.theta);
    if (lane < 2) fs.recip[lane] = r;
  }
  const bool counts = rp.phi != 0.0f;                  // otherwise "occurs" is all that matters
  const bool long_hist = counts && pen.h.hi - pen.h.lo > kResMaxCount;               // uniform
  int code = (pen.any && counts && pen.h.hi - pen.h.lo > (long long)kResFold * kResList) ? 4 : 0;   // uniform, like every `code` below
  uint32_t n_fold = 0;                                 // uniform: notes (m_key: token) of kResFold each
  __syncthreads();

  // ---- (1) multiplicities
  if (pen.any && code == 0) {
    const long long lo = pen.h.lo, hi = pen.h.hi;
    for (long long i0 = lo; i0 < hi; i0 += 4 * NT) {
      int t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const long long i = i0 + tid + (long long)j * NT;
        t[j] = i < hi ? a.tokens[i] : -1;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (t[j] >= 0 && t[j] < V) {
          const uint32_t one = (t[j] & 1) ? 0x10000u : 1u;
          if (long_hist) {
            const uint32_t old = atomicAdd(&fs.u.cnt[t[j] >> 1], one);
            if (((t[j] & 1) ? old >> 16 : old & 0xFFFFu) == kResFold) {
              const uint32_t q = atomicAdd(&fs.n_m, 1u);                       // (at most one for every kResFold tokens)
              if (q < (uint32_t)kResList) fs.m_key[q] = (uint32_t)t[j];
            }
          } else if (counts) {
            atomicAdd(&fs.u.cnt[t[j] >> 1], one);
          } else {
            atomicOr(&fs.u.cnt[t[j] >> 1], one);
          }
        }
      if (long_hist) {
        // what has grown beyond kResFold gives it up again before the next batch could take it beyond 15 bits
        static_assert(kResFold + 4 * 1024 < 32768, "a batch on top of what folding leaves");
        __syncthreads();
        const uint32_t n = min(fs.n_m, (uint32_t)kResList);
        for (uint32_t q = n_fold + tid; q < n; q += NT)
          atomicSub(&fs.u.cnt[fs.m_key[q] >> 1], (fs.m_key[q] & 1) ? kResFold << 16 : kResFold);
        n_fold = n;
        __syncthreads();
      }
    }
    for (long long i0 = pen.p_lo; i0 < pen.p_hi; i0 += 4 * NT) {
      int t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const long long i = i0 + tid + (long long)j * NT;
        t[j] = i < pen.p_hi ? a.p_tokens[i] : -1;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (t[j] >= 0 && t[j] < V) atomicOr(&fs.u.cnt[t[j] >> 1], (t[j] & 1) ? 0x80000000u : 0x8000u);
    }
    __syncthreads();
  }

  // ---- (2) penalised values, s = z' / tau, maximum and lowest value
  // (parameters that are off take part with the value that changes nothing: no branch per element)
  float s[NPT];
  {
    const RowDivisor by_tau(uniform_f64(fs.recip[0])), by_theta(uniform_f64(fs.recip[1]));
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int e0 = (j * NT + tid) * EPL;
      if (j * NT * EPL >= V) {                         // workgroup-uniform: nothing in this load
#pragma unroll
        for (int i = 0; i < EPL; ++i) s[j * EPL + i] = -INFINITY;
        continue;
      }
      const uint32_t w[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
      float z[EPL];
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        z[i] = DT == SIP_F32 ? __uint_as_float(w[i]) : __uint_as_float((i & 1) ? (w[i / 2] & 0xFFFF0000u) : (w[i / 2] << 16));
      if (pen.any) {                                   // (past the end of the row: counters that stay zero)
        uint32_t c[EPL / 2];
        bool some = false;
#pragma unroll
        for (int i = 0; i < EPL / 2; ++i) { c[i] = fs.u.cnt[e0 / 2 + i]; some |= c[i] != 0u; }
        if (__any(some)) {
          uint32_t ci[EPL], n[EPL];
#pragma unroll
          for (int i = 0; i < EPL; ++i) {
            ci[i] = (i & 1) ? c[i / 2] >> 16 : c[i / 2] & 0xFFFFu;
            n[i] = ci[i] & 0x7FFFu;
          }
#pragma nounroll
          for (uint32_t o = 0; o < n_fold; ++o) {                              // hardly ever any
            const uint32_t at = fs.m_key[o] - (uint32_t)e0;
#pragma unroll
            for (int i = 0; i < EPL; ++i) n[i] += at == (uint32_t)i ? kResFold : 0u;
          }
#pragma unroll
          for (int i = 0; i < EPL; ++i)
            z[i] = ci[i] ? penalise_shared(z[i], n[i], by_theta, rp.theta, rp.phi, rp.psi) : z[i];
        }
      }
#pragma unroll
      for (int i = 0; i < EPL; ++i) z[i] = by_tau.of(z[i]);
      if ((j + 1) * NT * EPL <= V) {                   // workgroup-uniform: whole loads
#pragma unroll
        for (int i = 0; i < EPL; ++i) { mx = fmaxf(mx, z[i]); mn = fminf(mn, z[i]); }
      } else {
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const bool in = e0 + i < V;
          mn = in ? fminf(mn, z[i]) : mn;
          z[i] = in ? z[i] : -INFINITY;
          mx = fmaxf(mx, z[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < EPL; ++i) s[j * EPL + i] = z[i];
    }
    const uint32_t wk = wave_max_u32(key_of(mx)), wl = wave_min_u32(key_of(mn));
    if (lane == 0) { fs.rkey[wave] = wk; fs.rlow[wave] = wl; }
  }
  __syncthreads();
  const float m = value_of(wave_max_u32(fs.rkey[lane & (NW - 1)]));
  const float low = value_of(wave_min_u32(fs.rlow[lane & (NW - 1)]));
  if (long_hist && tid == 0) fs.n_m = 0;               // (from here on the members')
  if (!(m > -3.0e38f && m < 3.0e38f)) code = 6;
  const float lo_s = fmaxf(low, __fsub_rn(m, kResSpan));
  const float span = __fsub_rn(m, lo_s);
  const float scale = span > 0.0f ? (float)(kResBins - 1) / span : 0.0f;
  // monotone in s (one rounding of v * scale + shift); -inf and what lies below lo_s share bin 0
  const float shift = __fmaf_rn(-m, scale, (float)(kResBins - 1));
  auto bin_of = [&](float v) -> int {
    return (int)__builtin_amdgcn_fmed3f(__fmaf_rn(v, scale, shift), 0.0f, (float)(kResBins - 1));
  };
  const float t_minp = rp.greedy ? -INFINITY : fs.t_minp;                      // (no min-p: -inf)
  auto emit = [&](uint32_t token, float sv, double lnZ) {                      // one thread
    a.out_ids[b] = (int)token;
    if (a.k_lp >= 0) {
      const int cols = 1 + a.k_lp;
      a.out_lp_ids[(size_t)b * cols] = (int)token;
      a.out_lp[(size_t)b * cols] = (float)((double)sv - (double)m - lnZ);
    }
    a.row_path[b] = a.S > 0 ? 1 : 14; a.row_why[b] = 1;  // 14: no shape of the single-pass kernels
    if (a.slot) state_append_row(a, b);
  };
  if (rp.greedy && code == 0) {
    uint32_t at = kFinNone;
#pragma unroll
    for (int j = NL - 1; j >= 0; --j)
#pragma unroll
      for (int i = EPL - 1; i >= 0; --i)
        if (s[j * EPL + i] == m) at = (uint32_t)((j * NT + tid) * EPL + i);
    at = wave_min_u32(at);
    if (lane == 0 && at != kFinNone) atomicMin(&fs.arg_max, at);
    if (a.k_lp < 0) {
      __syncthreads();
      if (tid == 0) emit(fs.arg_max, m, 0.0);
      return;
    }
  }

  // ---- (3) masses and bins
  float e[NPT];
  if (code == 0) {
    unsigned long long mine = 0;
    int n_mine = 0;                                    // summands, each with kMagicBits in it
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      if (j * NT * EPL >= V) {                         // workgroup-uniform
#pragma unroll
        for (int i = 0; i < EPL; ++i) e[j * EPL + i] = 0.0f;
        continue;
      }
      n_mine += EPL;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        const float v = s[j * EPL + i];
        const float x = exp_nonpos(__fsub_rn(v, m));
        e[j * EPL + i] = x;
        const unsigned long long E = mass_bits(x);
        mine += E;
        if (bins_on) {
          // (bin 0, which a row with far outliers has most of its elements in, is what is left over)
          const int bin = bin_of(v);
          if (bin > 0) {
            atomicAdd(&fs.hcnt[bin], 1u);
            if (p_act) atomicAdd(&fs.hmass[bin], E - kMagicBits);
          }
        }
      }
    }
    mine = wave_add_u64(mine - (unsigned long long)n_mine * kMagicBits);
    if (lane == 0) fs.r64[wave] = mine;
  }
  __syncthreads();
  const unsigned long long S0 = wave_add_u64(lane < NW ? fs.r64[lane] : 0ull);
  auto ln_total = [&]() -> double { return log((double)S0) - (double)kFixShift * 0.6931471805599453094; };
  // One wave works it out while the others are at the elements, instead of whoever needs it at the end of the chain
  // (V = 16000 without a filter 12.7 -> 12.3, everything on 21.2 -> 20.9 us; not with eight waves: 1500 rows of 4096,
  // top-p, 60.8 / 62.0).
  constexpr bool kAhead = NW == 16;
  auto note_ln_total = [&]() {
    if (kAhead && wave == NW / 2) {
      const double z = ln_total();
      if (lane == 0) fs.ln_z = z;
    }
  };
  auto noted_ln_total = [&]() -> double { return kAhead ? fs.ln_z : ln_total(); };

  // ---- (4) descending scan: thread t owns bins kResBins-1-BPT*t .. kResBins-BPT*(t+1)
  auto limit_of = [&](unsigned long long mass1) -> unsigned long long {
    const double lim = ceil((double)rp.top_p * (double)mass1);
    return lim > 0.0 ? (unsigned long long)lim : 0ull;
  };
  const int b0 = kResBins - 1 - BPT * tid;
  uint32_t c[BPT];
  unsigned long long mex[BPT];
  unsigned long long limit = (p_act && !k_act) ? limit_of(S0) : 0ull;
  // the lowest non-empty bin, from `lowest` up, whose elements may still be in the nucleus
  auto find_nucleus_bin = [&](int lowest) {
    int at = 1 << 30;
#pragma unroll
    for (int j = 0; j < BPT; ++j)
      if (b0 - j >= lowest && c[j] && mex[j] < limit) at = b0 - j;             // descending: the last hit is the lowest
    const uint32_t wmin = wave_min_u32((uint32_t)at);
    if (lane == 0 && wmin < (1u << 30)) atomicMin(&fs.bin_p, (int)wmin);
  };
  if (bins_on && code == 0) {
    uint32_t csum = 0;
    unsigned long long msum = 0, w[BPT];
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      c[j] = fs.hcnt[b0 - j]; csum += c[j];
      w[j] = p_act ? fs.hmass[b0 - j] : 0ull; msum += w[j];
    }
    const uint32_t cinc = dpp_scan_add_u32(csum);
    unsigned long long minc = 0;
    if (p_act) minc = dpp_scan_add_u64(msum);
    if (lane == kWave - 1) { fs.r32[wave] = cinc; fs.r64b[wave] = minc; }
    __syncthreads();
    const uint32_t before = wave_add_u32(lane < wave ? fs.r32[lane & 15] : 0u);
    uint32_t cex = before + cinc - csum;
    unsigned long long mx_ = minc - msum;
    if (p_act) mx_ += wave_add_u64(lane < wave ? fs.r64b[lane & 15] : 0ull);
    const uint32_t k = (uint32_t)rp.top_k;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int bin = b0 - j;
      if (bin == 0) { c[j] = (uint32_t)V - cex; fs.hcnt[0] = c[j]; }           // (its mass is never asked for)
      fs.hoff[bin] = cex;
      if (p_act) fs.hmass[bin] = mx_;
      mex[j] = mx_;
      if (k_act && cex < k && k <= cex + c[j]) fs.bin_k = bin;
      if (n_top > 0 && cex < n_top && n_top <= cex + c[j]) fs.bin_n = bin;
      cex += c[j]; mx_ += w[j];
    }
    if (p_act && !k_act) find_nucleus_bin(0);
    __syncthreads();
    const int bin_k = fs.bin_k, bin_n = fs.bin_n;
    // (a k-th largest that far below the maximum cuts off nothing that has mass)
    const bool k_cut = k_act && !(bin_k == 0 && low < lo_s);
    int bin_m = k_cut ? bin_k : (p_act && !k_act ? fs.bin_p : -1);             // the bin whose members decide the first cut
    if ((k_act && bin_k < 0) || (n_top > 0 && bin_n < 0) || (p_act && !k_act && bin_m >= kResBins)) code = 8;
    // The n-th best may lie where masses are zero (a dominant token, a temperature near 0): bin 0
    // is then cut once more, by count, between the lowest value and lo_s.
    const bool deep = n_top > 0 && bin_n == 0 && low < lo_s;
    float low2 = low, scale2 = 0.0f;
    auto bin2_of = [&](float v) -> int { return (int)__builtin_amdgcn_fmed3f(__fsub_rn(v, low2) * scale2, 0.0f, (float)(kResBins - 1)); };
    int bin_n2 = 0;
    uint32_t n_best = 0;                               // entries at or above the bin of the n-th best
    if (n_top > 0 && code == 0) n_best = fs.hoff[bin_n] + fs.hcnt[bin_n];
    if (deep && code == 0) {
      uint32_t* h2 = fs.a_key;                         // a_key and a_idx, one behind the other: not in use yet
      static_assert(2 * kResList == kResBins, "");
      for (int i = tid; i < kResBins; i += NT) h2[i] = 0;
      float mn = lo_s;                                 // lowest finite value
#pragma unroll
      for (int r = 0; r < NPT; ++r) mn = s[r] > -INFINITY ? fminf(mn, s[r]) : mn;
      const uint32_t wl = wave_min_u32(key_of(mn));
      if (lane == 0) fs.rlow[wave] = wl;
      __syncthreads();
      low2 = value_of(wave_min_u32(fs.rlow[lane & (NW - 1)]));
      scale2 = (float)(kResBins - 1) / fmaxf(__fsub_rn(lo_s, low2), 1.0e-30f);
#pragma unroll
      for (int j = 0; j < NL; ++j)
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const float v = s[j * EPL + i];
          if ((j * NT + tid) * EPL + i < V && bin_of(v) == 0) atomicAdd(&h2[bin2_of(v)], 1u);
        }
      __syncthreads();
      uint32_t c2[BPT], sum = 0;
#pragma unroll
      for (int j = 0; j < BPT; ++j) { c2[j] = h2[b0 - j]; sum += c2[j]; }
      const uint32_t inc = dpp_scan_add_u32(sum);
      if (lane == kWave - 1) fs.r32[wave] = inc;
      __syncthreads();
      uint32_t ex = fs.hoff[0] + wave_add_u32(lane < wave ? fs.r32[lane & 15] : 0u) + inc - sum;
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        if (ex < n_top && n_top <= ex + c2[j]) { fs.bin_n = b0 - j; fs.n_best = ex + c2[j]; }
        ex += c2[j];
      }
      __syncthreads();
      bin_n2 = fs.bin_n; n_best = fs.n_best;
    }
    if (code == 0 && n_best > (uint32_t)kResList) code = 9;
    // ---- members of the cut's bin, their least and largest key, and the entries the best-n are chosen from
    auto gather = [&](int bin_a, int bin_b) {
      uint32_t lo = kFinNone, hi = 0;
      const int first = min(bin_a >= 0 ? bin_a : 1 << 30, bin_b >= 0 ? bin_b : 1 << 30);
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        if (j * NT * EPL >= V) continue;               // workgroup-uniform
        if (NPT >= 16 && first > 0) {                  // (a shorter row's loads have one nearly always)
          float hi = s[j * EPL];
#pragma unroll
          for (int i = 1; i < EPL; ++i) hi = fmaxf(hi, s[j * EPL + i]);
          if (!(__fmaf_rn(hi, scale, shift) >= (float)first)) continue;        // every bin_of() below `first`
        }
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const int v = (j * NT + tid) * EPL + i;
          const float x = s[j * EPL + i];
          const int bin = bin_of(x);
          if (bin >= first && v < V) {
            if (bin_a >= 0 && bin >= bin_a && (!deep || bin > 0 || bin2_of(x) >= bin_n2)) {
              const uint32_t at = atomicAdd(&fs.n_a, 1u);
              if (at < (uint32_t)kResList) { fs.a_key[at] = key_of(x); fs.a_idx[at] = (uint32_t)v; }
            }
            if (bin == bin_b) {
              const uint32_t at = atomicAdd(&fs.n_m, 1u), key = key_of(x);
              if (at < (uint32_t)kResList) { fs.m_key[at] = key; fs.m_E[at] = mass_units(e[j * EPL + i]); }
              lo = min(lo, key); hi = max(hi, key);
            }
          }
        }
      }
      if (__any(hi != 0u)) {
        lo = wave_min_u32(lo); hi = wave_max_u32(hi);
        if (lane == 0) { atomicMin(&fs.m_lo, lo); atomicMax(&fs.m_hi, hi); }
      }
    };
    // Logits that take few different values (quantised ones, rows of equal values) put thousands of
    // equal entries into the bin of a cut: then there is nothing to compare, however many they are.
    auto members_equal = [&]() { return fs.m_lo == fs.m_hi; };
    // the smallest member (of K1) whose strictly larger mass stays below the limit
    auto nucleus_in_bin = [&](unsigned long long above, uint32_t nm, uint32_t key_k) {
      for (uint32_t t = tid; t < nm; t += NT) {
        const uint32_t kt = fs.m_key[t];
        unsigned long long G = above;
#pragma unroll 8
        for (uint32_t o = 0; o < nm; ++o) G += fs.m_key[o] > kt ? fs.m_E[o] : 0ull;
        if (kt >= key_k && G < limit) atomicMin(&fs.key_p, kt);
      }
    };
    if (code == 0) {
      if (n_top > 0) note_ln_total();
      gather(n_top > 0 ? bin_n : -1, bin_m);
      __syncthreads();
      if (bin_m >= 0) {
        const uint32_t nm = fs.n_m;
        if (members_equal()) {
          if (tid == 0 && k_cut) { fs.key_k = fs.m_lo; fs.s1_part = nm * fs.m_E[0]; }
          if (tid == 0 && !k_cut) fs.key_p = fs.m_lo;
        } else if (nm > (uint32_t)kResList) {
          code = 9;
        } else if (k_cut) {
          const uint32_t k_rem = k - fs.hoff[bin_k];                           // 1 <= k_rem <= members
          for (uint32_t t = tid; t < nm; t += NT) {
            const uint32_t kt = fs.m_key[t];
            uint32_t gt = 0, ge = 0;
            unsigned long long sum_ge = 0;
#pragma unroll 8
            for (uint32_t o = 0; o < nm; ++o) {
              const uint32_t ko = fs.m_key[o];
              gt += ko > kt; ge += ko >= kt;
              sum_ge += ko >= kt ? fs.m_E[o] : 0ull;
            }
            if (gt < k_rem && k_rem <= ge) { fs.key_k = kt; fs.s1_part = sum_ge; }        // equal members agree
          }
        } else {
          nucleus_in_bin(fs.hmass[bin_m], nm, 0u);
        }
      }
      if (n_top > 0) {
        // (from the other end of the workgroup, so that it is other waves' work)
        const uint32_t na = min(fs.n_a, (uint32_t)kResList);
        const int cols = 1 + a.k_lp;
        for (uint32_t t = NT - 1 - tid; t < na; t += NT) {
          const uint32_t kt = fs.a_key[t], v = fs.a_idx[t];
          uint32_t rank = 0;
#pragma unroll 8
          for (uint32_t o = 0; o < na; ++o) {
            const uint32_t ko = fs.a_key[o];
            rank += (ko > kt || (ko == kt && fs.a_idx[o] < v)) ? 1u : 0u;
          }
          if (rank < n_top) {
            a.out_lp_ids[(size_t)b * cols + 1 + rank] = (int)v;
            a.out_lp[(size_t)b * cols + 1 + rank] = (float)((double)value_of(kt) - (double)m - noted_ln_total());
          }
        }
        for (int o = (int)n_top + tid; o < a.k_lp; o += NT) {                  // vocabulary smaller than k_logprobs
          a.out_lp_ids[(size_t)b * cols + 1 + o] = -1;
          a.out_lp[(size_t)b * cols + 1 + o] = -INFINITY;
        }
      }
      if (bin_m >= 0) __syncthreads();
      if (k_act && p_act && code == 0) {
        // ---- top-p on the mass that survived top-k
        const uint32_t key_k = fs.key_k;
        limit = limit_of(fs.hmass[bin_k] + fs.s1_part);
        find_nucleus_bin(bin_k);
        if (tid == 0) { fs.n_m = 0; fs.m_lo = kFinNone; fs.m_hi = 0; }
        __syncthreads();
        bin_m = fs.bin_p;
        if (bin_m >= kResBins) {
          code = 10;
        } else {
          gather(-1, bin_m);
          __syncthreads();
          const uint32_t nm = fs.n_m;
          if (members_equal()) {
            if (tid == 0) fs.key_p = fs.m_lo;
          } else if (nm > (uint32_t)kResList) {
            code = 9;
          } else {
            nucleus_in_bin(fs.hmass[bin_m], nm, key_k);
          }
          __syncthreads();
        }
      }
      if (code == 0 && p_act && fs.key_p == kFinNone) code = 10;
    }
  }

  // ---- (5) draw
  if (code == 0 && rp.greedy) {
    if (tid == 0) emit(fs.arg_max, m, n_top > 0 ? noted_ln_total() : ln_total());
    return;
  }
  if (code == 0) {
    float s_cut = -INFINITY;
    if (fs.key_k) s_cut = value_of(fs.key_k);
    if (p_act) s_cut = fmaxf(s_cut, value_of(fs.key_p));
    if (minp_on) {                                     // (a mass less costs the other rows nothing)
#pragma unroll
      for (int r = 0; r < NPT; ++r) e[r] = __fsub_rn(s[r], m) >= t_minp ? e[r] : 0.0f;
    }
    auto kept = [&](int r) { return s[r] >= s_cut; };
    auto lane_mass = [&](int j) -> unsigned long long {
      unsigned long long t = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i) t += mass_bits(kept(j * EPL + i) ? e[j * EPL + i] : 0.0f);
      return t - (unsigned long long)EPL * kMagicBits;
    };
    if (n_top == 0 && a.k_lp >= 0) note_ln_total();
    unsigned long long t_of[NL];
    // (wave-uniform.  Most waves of a row that keeps few tokens have none: V = 19513 fp32, 3 rows, 13.6 us a call with a
    // sum for each load that has one, 14.2 with the sums of all loads together in every wave, 13.6 with both)
    bool has = false;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      t_of[j] = 0;
      if (j * NT * EPL < V) {                          // workgroup-uniform
        bool some = false;
#pragma unroll
        for (int i = 0; i < EPL; ++i) some |= kept(j * EPL + i);
        if (__any(some)) { t_of[j] = lane_mass(j); has = true; }
      }
    }
    if constexpr (NL == 1) {
      const unsigned long long t = wave_add_u64(t_of[0]);
      if (lane == 0) fs.blk[wave] = t;
    } else if (has) {
      const unsigned long long t = row_sums_u64(t_of, lane);
      if ((lane & 15) < NL) atomicAdd(&fs.blk[(lane & 15) * NW + wave], t);
    }
    __syncthreads();
    const unsigned long long w0 = 2 * lane < NBLK ? fs.blk[2 * lane] : 0ull;
    const unsigned long long w1 = 2 * lane + 1 < NBLK ? fs.blk[2 * lane + 1] : 0ull;
    const unsigned long long incl = dpp_scan_add_u64(w0 + w1);
    const unsigned long long S3 = last_lane_u64(incl);
    const unsigned long long j24 = fs.j24;
    const unsigned long long target = (__umul64hi(j24, S3) << 40) | ((j24 * S3) >> 24);    // floor(j * S3 / 2^24)
    unsigned long long ex = incl - w0 - w1;
    int hit = -1;
    if (ex <= target && target < ex + w0) hit = 2 * lane;
    else if (ex + w0 <= target && target < incl) { hit = 2 * lane + 1; ex += w0; }
    const unsigned long long ball = __ballot(hit >= 0);
    if (!ball) {
      code = 14;                                                               // no kept mass
    } else {
      const int src = __ffsll((long long)ball) - 1;
      const int blk = __builtin_amdgcn_readlane(hit, src);
      const unsigned long long before = readlane_u64(ex, src);
      if (wave == (blk & (NW - 1))) {                                          // the wave that holds the crossing
        uint32_t token = kFinNone;
        float sv = 0.0f;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          if (j == blk / NW) {
            const unsigned long long t = lane_mass(j);
            unsigned long long C = before + dpp_scan_add_u64(t) - t;
            const bool mine = C <= target && target < C + t;
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
              const int r = j * EPL + i;
              C += kept(r) ? mass_units(e[r]) : 0ull;
              if (mine && token == kFinNone && C > target) { token = (uint32_t)((j * NT + tid) * EPL + i); sv = s[r]; }
            }
          }
        }
        if (token != kFinNone) emit(token, sv, a.k_lp >= 0 ? noted_ln_total() : 0.0);                    // one lane
      }
      return;
    }
  }

  // ---- the general multi-pass path for what the above could not settle
  __syncthreads();
  if (sharded) { if (DT == SIP_F32) gather_row<SIP_F32>(a, b); else gather_row<SIP_BF16>(a, b); }
  exact_row<DT>(a, b, in_lds(&fs.u.dyn[0]), in_lds(&fs.ex));
  if (tid == 0) { a.row_path[b] = a.S > 0 ? code : 14; a.row_why[b] = code; }
  if (a.slot) {
    __syncthreads();
    if (tid == 0) state_append_row(a, b);
  }
}

}  // namespace sip
