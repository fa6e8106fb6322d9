// The heavier per-row logic of the single-pass path, for the rows that the finishing kernel
// (sip_finish.h) cannot settle from the list the streaming kernel left behind: rescue_row(),
// run by rescue_kernel on the rows passed on to it or, in small batches, by the workgroup that
// just tried (sip_fused.h).  It tries, in this order,
//   - the row's list again in register variants that hold up to 24 entries per thread
//     (fast_row: lists of up to 12288 entries, as top_k in the thousands makes them), with the
//     history tokens' multiplicities from a bitmap over the vocabulary, popcount ranks and side
//     tables in LDS;
//   - a second, longer list, made by reading the row once more with a lower threshold
//     (restream_row), and the same logic on that one (rows under min-p, and lists that lack the k-th or n-th);
//   - the continuations over the whole row (whole_row_finish): a nucleus that reaches below the
//     list is cut and drawn from in one read of the row, or two, and a row without any filter is drawn
//     over all its elements;
//   - the exact multi-pass path (sip_exact.h).
//
// fast_row keeps the list in registers: every thread holds its share of the entries (key,
// index, mass, value bin) from the moment they are read until the end.  Every sum is an
// integer sum (masses in units of 2^-40 of the maximum's mass), so no result depends on the
// order in which threads add.  Selection works on 2048 linear value bins between the
// completeness threshold and the maximum: one histogram locates the bin that holds the k-th
// largest value, the nucleus cut or the n-th best, and the handful of entries in that bin are
// then resolved by all-pairs comparison.  The draw does the same over 2048 bins of the
// vocabulary index.
//
// Whenever a list cannot prove the answer (a cut falls below the completeness threshold,
// a bin or a segment overflows, too many distinct history tokens, ...) fast_row returns a
// reason code > 1 and rescue_row goes on to the next of the above; 1 means the row is finished.
#pragma once
#include <type_traits>

#include "sip_device.h"
#include "sip_exact.h"
#include "sip_stream.h"

namespace sip {

constexpr int kFinalThreads = 512;
constexpr int kFinalWaves = kFinalThreads / kWave;
constexpr int kBins = 2048;
constexpr int kBinsPerThread = kBins / kFinalThreads;
constexpr int kMembers = 256;        // entries of one bin that can be resolved by all-pairs comparison
constexpr int kSideMax = 4096;       // distinct history tokens per row the fast path handles
constexpr int kMaxChunks = 16;       // chunks (= list segments) per row
constexpr int kTopList = kFinalThreads / 2 < 256 ? kFinalThreads / 2 : 256;        // entries at or above the bin of the n-th best (half a workgroup ranks them)
constexpr int kTokRegs = 8;          // history tokens a thread keeps in registers between phases
constexpr int kWordRegs = 16;        // bitmap words a thread owns (2^18 / 32 / kFinalThreads)
constexpr uint32_t kNoIdx = 0xFFFFFFFFu;
constexpr int kNeedLong = 30;        // internal: more history tokens than this variant holds per thread
constexpr int kNeedLongList = 31;    // internal: more candidates than this variant holds per thread
constexpr int kWholeRowCut = 32;     // internal: the nucleus cut lies below the list -- settle it, and draw, over the whole row
constexpr int kWholeRow = 33;        // internal: no filter at all -- draw over the whole row
constexpr int kCandLong = 24;        // candidate entries per thread of the largest variant

struct FastShared {
  float Tc[kMaxChunks];
  double unit;
  unsigned long long bulk[kMaxChunks];
  uint32_t segoff[kMaxChunks + 1];
  unsigned long long r64[kFinalWaves];
  uint32_t r32[kFinalWaves];
  uint32_t rkey[kFinalWaves];
  uint32_t ridx[kFinalWaves];
  uint32_t fail_seg, anyc, dropped;
  float m_out, zmax_out, trow_out;      // for a second attempt: max of s, max of z', threshold used
  unsigned long long limit_out;         // for the whole-row continuation: top-p limit, ln Z, whether penalties apply
  double lnz_out;
  int has_pen_out;
  int second_list_out;                  // min-p bounds the kept set: a second list can be cut there
  uint32_t rq_n;                         // candidates found by the second pass
  const char* shard_row[8];             // sharded logits: this row's piece in every shard
  int ndist_out;                        // distinct history tokens of the row, -1 while not counted (thread 0 only)
  int bin_k, bin_n, bin_p, bin_low, bin_d;
  uint32_t above_k, above_n;
  uint32_t key_k, key_p, token_key;
  int token;
  unsigned long long s1_part, before_d;
  uint32_t n_memb, n_memb2, n_memb3;
  uint32_t m_key[kMembers];
  uint32_t m_idx[kMembers];
  unsigned long long m_E[kMembers];
  uint32_t n_top;
  uint32_t t_key[kTopList];
  uint32_t t_idx[kTopList];
  int w_lo[2], w_hi[2];                 // whole_row_window: first and last bin of two windows, elements of the sample
  uint32_t w_n0[2], w_n1[2];            // below the first and up to the last
  float w_sq;                           // sum of the squared masses below the place where the cut is expected
};

// Bytes of dynamic LDS the finishing kernel needs for vocabulary V, before the candidates.
__host__ __device__ inline size_t final_lds_fixed(int V) {
  const size_t W = ((size_t)V + 31) / 32;
  return ((W * 4 + W * 2 + 15) / 16) * 16 + (size_t)kBins * 20 + (size_t)kSideMax * 8;
}

template <int DT>
__device__ __forceinline__ float load_elem(const char* row, int v) {
  if (DT == SIP_F32) return reinterpret_cast<const float*>(row)[v];
  return __uint_as_float((uint32_t)reinterpret_cast<const unsigned short*>(row)[v] << 16);
}


// One attempt at finishing row b from its candidate list.  CR / SR = candidate entries /
// distinct history tokens a thread can hold in registers: the list, once read, never goes to
// memory again -- each thread keeps its share with key, index, mass and value bin in
// registers, and the phases below talk to each other only through the LDS histograms and a few
// small gathered lists.  Every register round is unrolled code that costs time even when it
// holds nothing (0.5-0.7 us each), hence several instantiations and a caller that picks the
// smallest one that fits.  Returns 1 (finished), kNeedLong / kNeedLongList (the row does not fit
// SR / CR entries per thread) or a reason code > 1; outputs written before a failure are overwritten
// by the path that takes the row over.
template <int DT, int CR, int SR, bool SH>
__device__ __forceinline__ int fast_row(const Args& a, const int b, const RowParams& rp, unsigned char* dyn,
                                        FastShared& fs, const int S, const int cap_c) {
  constexpr int NT = kFinalThreads;
  constexpr int NE = CR + SR;                               // register entries per thread
  constexpr bool STORE = CR <= 8;
  typedef typename std::conditional<(NE <= 32), uint32_t, unsigned long long>::type mask_t;                           // keep mass and bin in registers too
  constexpr int NS = STORE ? NE : 1;
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int V = a.V;
  const int W = (V + 31) >> 5;
  // ---- LDS carving
  uint32_t* bm = reinterpret_cast<uint32_t*>(dyn);
  unsigned short* pre = reinterpret_cast<unsigned short*>(dyn + (size_t)W * 4);
  unsigned char* p2 = dyn + (((size_t)W * 6 + 15) / 16) * 16;
  unsigned long long* hm = reinterpret_cast<unsigned long long*>(p2);      // value bins: mass
  unsigned long long* hd = hm + kBins;                                      // index bins: kept mass
  uint32_t* hc = reinterpret_cast<uint32_t*>(hd + kBins);                   // value bins: count
  uint32_t* cnt = hc + kBins;                                               // multiplicity per history slot
  uint32_t* stok = cnt + kSideMax;                                          // token per history slot
  const char* row = reinterpret_cast<const char*>(a.logits) + (size_t)b * (size_t)a.row_stride * (DT == SIP_F32 ? 4 : 2);
  auto scaled_s = [&](float z) { return rp.greedy ? z : __fdiv_rn(z, rp.tau); };

  // ---- (0) chunk summaries, history extent; clear the LDS tables meanwhile
  const PenaltyPlan pen = penalty_plan(a, b, rp.theta, rp.phi, rp.psi);
  const long long lo = pen.h.lo, hi = pen.h.hi;
  const bool has_pen = pen.any;
  const int nseg = S;                                       // one list segment per chunk
  if (tid == 0) {
    fs.fail_seg = 0; fs.anyc = 0; fs.dropped = 0;
    fs.bin_k = -1; fs.bin_n = -1; fs.bin_p = 1 << 30; fs.bin_low = 1 << 30; fs.bin_d = -1;
    fs.key_p = 0xFFFFFFFFu; fs.n_memb = 0; fs.n_memb2 = 0; fs.n_memb3 = 0; fs.n_top = 0;
    fs.token = 0x7FFFFFFF; fs.key_k = 0; fs.s1_part = 0;
  }
  if (SH && tid == 0) {                   // constant indices: the piece pointers come through scalar loads
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < a.t_shards)
        fs.shard_row[i] = reinterpret_cast<const char*>(a.shard[i]) + (size_t)b * (size_t)a.shard_stride * (DT == SIP_F32 ? 4 : 2);
  }
  if (tid < S) {
    const ChunkOut co = a.chunks[(size_t)b * a.S + tid];
    fs.Tc[tid] = co.Tc; if (tid == 0) fs.unit = co.unit; fs.bulk[tid] = co.bulk;
    fs.segoff[tid] = co.cnt;
  }
  // history tokens of this thread (the first kTokRegs rounds stay in registers)
  int tok[kTokRegs];
#pragma unroll
  for (int j = 0; j < kTokRegs; ++j) {
    const long long i = lo + tid + (long long)j * NT;
    tok[j] = (has_pen && i < hi) ? a.tokens[i] : -1;
  }
  {
    uint4* z4 = reinterpret_cast<uint4*>(p2);               // hm, hd, hc: kBins * 20 bytes
    for (int i = tid; i < kBins * 20 / 16; i += NT) z4[i] = make_uint4(0, 0, 0, 0);
  }
  if (has_pen) {
    for (int w = tid; w < W; w += NT) bm[w] = 0;
    for (int i = tid; i < kSideMax; i += NT) cnt[i] = 0;
  }
  // row constants that take long arithmetic, worked out while the loads above travel
  const bool minp_on = !rp.greedy && rp.min_p > 0.0f;
  const float t_minp = minp_on ? (float)log((double)rp.min_p) : 0.0f;
  const unsigned long long j24 = rp.greedy ? 0ull : (unsigned long long)(philox_word0(a.seed, rp.row_id, step_of(a)) >> 8);
  __syncthreads();

  // ---- (1) prefix of the segment sizes (wave 0); presence bitmap of the history (everyone)
  if (wave == 0) {
    const uint32_t c0 = 2 * lane < nseg ? fs.segoff[2 * lane] : 0u;
    const uint32_t c1 = 2 * lane + 1 < nseg ? fs.segoff[2 * lane + 1] : 0u;
    const uint32_t incl = dpp_scan_add_u32(c0 + c1);
    const uint32_t total = last_lane_u32(incl);
    if (c0 > (uint32_t)cap_c || c1 > (uint32_t)cap_c) fs.fail_seg = 1;       // a queue overflowed
    if (c0 + c1 < c0 || incl < c0 + c1) fs.fail_seg = 1;                       // (the overflow mark wraps the sums)
    if (2 * lane < nseg) fs.segoff[2 * lane] = incl - c0 - c1;
    if (2 * lane + 1 < nseg) fs.segoff[2 * lane + 1] = incl - c1;
    if (lane == 0) fs.segoff[nseg] = total;
  }
  if (has_pen) {
#pragma unroll
    for (int j = 0; j < kTokRegs; ++j) {
      const int t = tok[j];
      if (t >= 0 && t < V) atomicOr(&bm[t >> 5], 1u << (t & 31));
    }
    for (long long i = lo + tid + (long long)kTokRegs * NT; i < hi; i += NT) {
      const int t = a.tokens[i];
      if (t >= 0 && t < V) atomicOr(&bm[t >> 5], 1u << (t & 31));
    }
    for (long long i = pen.p_lo + tid; i < pen.p_hi; i += NT) {             // a separate prompt: presence only
      const int t = a.p_tokens[i];
      if (t >= 0 && t < V) atomicOr(&bm[t >> 5], 1u << (t & 31));
    }
  }
  __syncthreads();
  // (the chunks of a row share threshold and unit)
  const float T_row = value_of(key_of(fs.Tc[0]));
  if (fs.fail_seg || !(T_row == T_row)) return 3;                             // uniform
  const uint32_t total_seg = fs.segoff[nseg];
  if (total_seg > (uint32_t)a.nc_cap) return 5;                               // uniform
  if (total_seg > (uint32_t)(NT * CR)) return kNeedLongList;                  // uniform

  // ---- (2) The two dependent global reads of this kernel -- the candidate segments and the raw
  // logits of the history tokens -- are issued as early as their addresses are known and
  // consumed as late as possible, with the LDS work in between.
  // (2a) thread t takes list positions per*t .. per*t + per-1: one segment search, then it walks along
  const uint2* segs = a.cand + (size_t)b * (size_t)a.S * (size_t)a.cap_c;
  const int per = (int)((total_seg + NT - 1) / NT);                           // uniform, <= CR
  uint2 creg[CR];
  {
    const uint32_t i0 = (uint32_t)(tid * per);
    int sg = 0;
    if (i0 < total_seg) {
      int s1 = nseg;
      while (s1 - sg > 1) {
        const int mid = (sg + s1) >> 1;
        if (fs.segoff[mid] <= i0) sg = mid; else s1 = mid;
      }
    }
    uint32_t lo_off = fs.segoff[sg], hi_off = fs.segoff[sg + 1];
#pragma unroll
    for (int r = 0; r < CR; ++r) {
      creg[r] = make_uint2(0u, kNoIdx);
      if (r < per) {
        const uint32_t i = i0 + (uint32_t)r;
        if (i < total_seg) {
          while (i >= hi_off) { ++sg; lo_off = hi_off; hi_off = fs.segoff[sg + 1]; }   // skips empty segments too
          creg[r] = segs[(size_t)sg * cap_c + (i - lo_off)];
        }
      }
    }
  }
  // (2b) slots of the distinct history tokens, in token order: each thread owns a contiguous
  // run of bitmap words
  uint32_t ndist = 0;
  if (has_pen) {
    const int perw = (W + NT - 1) / NT;                   // <= kWordRegs because V <= 262144
    const int w0 = tid * perw;
    uint32_t wd[kWordRegs];                                // all reads go out together
#pragma unroll
    for (int j = 0; j < kWordRegs; ++j) wd[j] = bm[min(w0 + j, W - 1)];
    uint32_t local = 0;
#pragma unroll
    for (int j = 0; j < kWordRegs; ++j) {
      if (!(j < perw && w0 + j < W)) wd[j] = 0;
      local += (uint32_t)__popc(wd[j]);
    }
    const uint32_t incl = dpp_scan_add_u32(local);
    if (lane == kWave - 1) fs.r32[wave] = incl;
    __syncthreads();
    uint32_t slot = incl - local;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) {
      const uint32_t t = fs.r32[ww];
      if (ww < wave) slot += t;
      ndist += t;
    }
    if (tid == 0) fs.ndist_out = (int)ndist;
    if (ndist > (uint32_t)kSideMax) return 4;                                 // uniform
    if (ndist > (uint32_t)(NT * SR)) return kNeedLong;                        // uniform
#pragma unroll
    for (int j = 0; j < kWordRegs; ++j) {
      uint32_t bits = wd[j];
      if (bits) pre[w0 + j] = (unsigned short)slot;
      while (bits) {                                                          // token of each slot
        stok[slot] = (uint32_t)(((w0 + j) << 5) + __ffs((int)bits) - 1);
        bits &= bits - 1;
        ++slot;
      }
    }
    __syncthreads();
  }
  // Register entries: 0..CR-1 candidates, CR..NE-1 history tokens.  idx == kNoIdx: no entry.
  uint32_t idx[NE], key[NE];                 // key[] holds the bits of z' until (5) turns them into keys
  // (2c) request the raw logits of this thread's history tokens
  float raw[SR];
#pragma unroll
  for (int r = 0; r < SR; ++r) {
    idx[CR + r] = kNoIdx; raw[r] = 0.0f;
    if ((uint32_t)(r * NT) < ndist) {                                        // uniform
      const uint32_t i = (uint32_t)(r * NT + tid);
      const uint32_t t = stok[min(i, (uint32_t)kSideMax - 1)];
      if (i < ndist) idx[CR + r] = t;
    }
  }
#pragma unroll
  for (int r = 0; r < SR; ++r)
    if (idx[CR + r] != kNoIdx) {
      if (!SH) {
        raw[r] = load_elem<DT>(row, (int)idx[CR + r]);
      } else {                                  // the token's shard, then its place inside it
        const int v = (int)idx[CR + r];
        int sh = min((int)((float)v * a.inv_V_shard), a.t_shards - 1);
        sh += (v >= (sh + 1) * a.V_shard) - (v < sh * a.V_shard);
        raw[r] = load_elem<DT>(fs.shard_row[sh], v - sh * a.V_shard);
      }
    }
  // ---- (3) multiplicities of the history tokens
  if (has_pen && pen.counts) {
    auto count = [&](int t) {
      if (t >= 0 && t < V) {
        const uint32_t word = bm[t >> 5];
        atomicAdd(&cnt[pre[t >> 5] + __popc(word & ((1u << (t & 31)) - 1u))], 1u);
      }
    };
    const int rounds = (int)min((long long)kTokRegs, (hi - lo + NT - 1) / NT);   // uniform
    uint32_t cw[kTokRegs], cp[kTokRegs];
#pragma unroll
    for (int j = 0; j < kTokRegs; ++j) {
      if (j < rounds) {
        const int t = min(max(tok[j], 0), V - 1);
        cw[j] = bm[t >> 5]; cp[j] = pre[t >> 5];
      }
    }
#pragma unroll
    for (int j = 0; j < kTokRegs; ++j) {
      const int t = tok[j];
      if (j < rounds && t >= 0 && t < V) atomicAdd(&cnt[cp[j] + __popc(cw[j] & ((1u << (t & 31)) - 1u))], 1u);
    }
    for (long long i = lo + tid + (long long)kTokRegs * NT; i < hi; i += NT) count(a.tokens[i]);
  }
  // (2d) candidates that carry a penalty are dropped: they come back with their penalised value
  // as history entries
  bool anyc = false;
  uint32_t fw[CR];
#pragma unroll
  for (int r = 0; r < CR; ++r) {
    fw[r] = 0;
    if (r < per && creg[r].y != kNoIdx) creg[r].y &= ~kTagBit;                  // the tag repeats what the bitmap says
    if (r < per && has_pen) fw[r] = bm[min(creg[r].y, (uint32_t)V - 1) >> 5];   // uniform condition
  }
#pragma unroll
  for (int r = 0; r < CR; ++r) {
    const uint2 e = creg[r];
    const bool keep = (r < per) & (e.y < (uint32_t)V) & (((fw[r] >> (e.y & 31)) & 1u) == 0);
    idx[r] = keep ? e.y : kNoIdx;
    key[r] = e.x;
    anyc |= keep & (__uint_as_float(e.x) >= T_row);
  }
  __syncthreads();

  // ---- (4) penalised values of the history entries; maximum of the list (lowest index on ties)
  // (the streaming pass, and restream_row, keep history tokens out of the bulk mass, so nothing
  // has to be taken back out of it)
  uint32_t bkey = 0, bidx = kNoIdx;
  {
    // everything these rounds read from LDS is requested first, then used
    uint32_t mult[SR];
#pragma unroll
    for (int r = 0; r < SR; ++r)
      if ((uint32_t)(r * NT) < ndist) mult[r] = pen.counts ? cnt[r * NT + tid] : pen.dflt;   // uniform
#pragma unroll
    for (int r = 0; r < SR; ++r) {
      if ((uint32_t)(r * NT) < ndist && idx[CR + r] != kNoIdx)
        key[CR + r] = __float_as_uint(penalise(raw[r], mult[r], rp.theta, rp.phi, rp.psi));
    }
  }
#pragma unroll
  for (int r = 0; r < NE; ++r) {
    if (idx[r] != kNoIdx) {
      const uint32_t kz = key_of(__uint_as_float(key[r]));
      if (kz > bkey || (kz == bkey && idx[r] < bidx)) { bkey = kz; bidx = idx[r]; }
    }
  }
  {
    const uint32_t wk = last_lane_u32(dpp_scan_max_u32(bkey));
    const uint32_t wi = last_lane_u32(dpp_scan_min_u32(bkey == wk ? bidx : kNoIdx));
    if (lane == kWave - 1) { fs.rkey[wave] = wk; fs.ridx[wave] = wi; }
    if (__any(anyc) && lane == 0) fs.anyc = 1;
  }
  __syncthreads();
  bkey = 0; bidx = kNoIdx;
#pragma unroll
  for (int w = 0; w < kFinalWaves; ++w) {
    const uint32_t ok = fs.rkey[w], oi = fs.ridx[w];
    if (ok > bkey || (ok == bkey && oi < bidx)) { bkey = ok; bidx = oi; }
  }
  // an unpenalised candidate at or above T_row proves that nothing outside the list is larger
  if (!fs.anyc || bidx == kNoIdx) return 6;                                   // uniform
  const int best_i = (int)bidx;
  const float m = scaled_s(value_of(bkey));
  const float s_c = scaled_s(T_row);            // entries with s > s_c: every such element of the row is in the list
  const uint32_t key_c = key_of(s_c);
  if (tid == 0) { fs.m_out = m; fs.zmax_out = value_of(bkey); fs.trow_out = T_row; }
  const float span = __fsub_rn(m, s_c);
  if (!(span >= 0.0f) || !(span < 3.0e38f)) return 7;                         // uniform
  const float binscale = span > 0.0f ? (float)(kBins - 2) / span : 0.0f;
  const bool big_k = !rp.greedy && rp.top_k >= 512 && rp.top_k < V;
  auto bin_of = [&](float s, uint32_t k) -> int {
    if (k <= key_c) return 0;
    // A large k lies just above the threshold, where a heavy-tailed row has thousands of entries in
    // the few lowest of 2046 equal bins, more than can be compared.  So for these the bin is the least
    // of three lines: half of the bins over the first 2 % of the span, a quarter up to 8 %, the rest
    // beyond; each is monotone in s, and so is their minimum.  (bf16 V = 49402, Student-t logits,
    // top_k 4000: such a row used to end in exact_row; the call took 296 us, now 57.  Bins like these
    // in finish_row, for every row or chosen per row, cost the ordinary rows 1 us of 19.)
    float x = __fsub_rn(s, s_c) * binscale;
    if (big_k) x = fminf(fminf(24.0f * x, 4.0f * x + 853.0f), 0.272f * x + 1489.0f);
    return 1 + min(kBins - 2, max((int)x, 0));
  };
  auto mass = [&](float s) { return fix_of(expf(__fsub_rn(s, m))); };
  // which register rounds hold anything at all (workgroup-uniform)
  auto live = [&](int r) { return r < CR ? r < per : (uint32_t)((r - CR) * NT) < ndist; };

  // ---- (5) keys, masses, value histogram (count and mass per bin)
  unsigned long long Ereg[NS];
  short breg[NS];
#pragma unroll
  for (int r = 0; r < NE; ++r) {
    if (live(r)) {
      unsigned long long E = 0;
      int bin = -1;
      uint32_t k = 0;
      if (idx[r] != kNoIdx) {
        const float s = scaled_s(__uint_as_float(key[r]));
        k = key_of(s);
        bin = bin_of(s, k);
        E = mass(s);
        atomicAdd(&hc[bin], 1u);
        if (E) atomicAdd(&hm[bin], E);
      }
      key[r] = k;
      if (r >= CR) cnt[(r - CR) * NT + tid] = k;      // slot -> key, for the whole-row draw (this thread's own slot)
      if constexpr (STORE) { Ereg[r] = E; breg[r] = (short)bin; }
    } else {
      key[r] = 0;
      if constexpr (STORE) { Ereg[r] = 0; breg[r] = -1; }
    }
  }
  auto E_of = [&](int r) -> unsigned long long {
    if constexpr (STORE) return Ereg[r]; else return mass(value_of(key[r]));
  };
  auto b_of = [&](int r) -> int {
    if constexpr (STORE) return (int)breg[r]; else return bin_of(value_of(key[r]), key[r]);
  };
  __syncthreads();
  const bool k_act = !rp.greedy && rp.top_k >= 2 && rp.top_k < V;
  const uint32_t n_top = (uint32_t)max(0, min(a.k_lp, V));
  unsigned long long S_cand;
  {
    // thread t owns bins kBins-1-4t .. kBins-4-4t; scan in descending bin order
    const int b0 = kBins - 1 - kBinsPerThread * tid;
    uint32_t c[kBinsPerThread];
    unsigned long long w[kBinsPerThread];
    uint32_t csum = 0;
    unsigned long long msum = 0;
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) { c[j] = hc[b0 - j]; w[j] = hm[b0 - j]; csum += c[j]; msum += w[j]; }
    const uint32_t cinc = dpp_scan_add_u32(csum);
    const unsigned long long minc = dpp_scan_add_u64(msum);
    if (lane == kWave - 1) { fs.r32[wave] = cinc; fs.r64[wave] = minc; }
    __syncthreads();
    uint32_t cex = cinc - csum;
    unsigned long long mex = minc - msum, mtot = 0;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) {
      if (ww < wave) { cex += fs.r32[ww]; mex += fs.r64[ww]; }
      mtot += fs.r64[ww];
    }
    S_cand = mtot;
    const uint32_t k = (uint32_t)rp.top_k;
    int mylow = 1 << 30;
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) {
      const int bin = b0 - j;
      hm[bin] = mex;                                                         // exclusive suffix mass
      if (bin >= 1) {                                                        // bin 0 is the incomplete region
        if (k_act && cex < k && k <= cex + c[j]) { fs.bin_k = bin; fs.above_k = cex; }
        if (n_top > 0 && cex < n_top && n_top <= cex + c[j]) { fs.bin_n = bin; fs.above_n = cex; }
        if (c[j]) mylow = bin;                                               // bins descend: the last one wins
      }
      cex += c[j]; mex += w[j];
    }
    const uint32_t wlow = last_lane_u32(dpp_scan_min_u32((uint32_t)mylow));
    if (lane == kWave - 1 && wlow < (1u << 30)) atomicMin(&fs.bin_low, (int)wlow);
  }
  __syncthreads();
  if ((k_act && fs.bin_k < 0) || (n_top > 0 && fs.bin_n < 0)) return 8;      // uniform: k-th / n-th not provably in the list
  const int bin_k = k_act ? fs.bin_k : 0, bin_n = fs.bin_n;

  // bulk mass -> units of 2^-40 relative to the maximum
  unsigned long long bulk;
  {
    const unsigned long long bc = fs.bulk[min(lane, S - 1)];
    bulk = last_lane_u64(dpp_scan_add_u64(lane < S ? bc : 0ull));
  }
  // 2^x with x split into integer and fraction: the fraction goes through the hardware exp2 (1 ulp,
  // far inside the accuracy of the fp32 bulk sums), the integer part is an exponent shift
  const double ln2 = 0.6931471805599453094;
  const double x = fmin(fmax(bulk_exponent(fs.unit, m) + 10.0, -2000.0), 2000.0);
  const double xi = floor(x);
  const double bulk_rel = ldexp((double)bulk * (double)__builtin_amdgcn_exp2f((float)(x - xi)), (int)xi);
  const unsigned long long S0 = S_cand + (bulk_rel < 9.0e18 ? (unsigned long long)bulk_rel : 0ull);
  // ln S0 from exponent and mantissa: S0 = f * 2^e, f in [0.5, 1)
  int e2;
  const float f2 = (float)frexp((double)S0, &e2);
  const double lnZ = ((double)__builtin_amdgcn_logf(f2) + (double)(e2 - kFixShift)) * ln2;

  // ---- (6) gather the bin of the k-th largest and everything at or above the bin of the n-th best
  if (k_act || n_top > 0) {
    mask_t mk = 0, mt = 0;            // bit r: register entry r lies in the bin of the k-th / belongs to the top list
#pragma unroll
    for (int r = 0; r < NE; ++r) {
      if (live(r) && idx[r] != kNoIdx) {
        const int bin = b_of(r);
        mk |= (mask_t)(k_act & (bin == bin_k)) << r;
        mt |= (mask_t)((n_top > 0) & (bin >= bin_n)) << r;
      }
    }
    uint32_t qk = 0, qt = 0;            // one reservation per thread and list
    if (mk) qk = atomicAdd(&fs.n_memb, (uint32_t)__popcll((unsigned long long)mk));
    if (mt) qt = atomicAdd(&fs.n_top, (uint32_t)__popcll((unsigned long long)mt));
    if (mk | mt) {
#pragma unroll
      for (int r = 0; r < NE; ++r) {
        if ((mk >> r) & 1u) {
          if (qk < (uint32_t)kMembers) { fs.m_key[qk] = key[r]; fs.m_E[qk] = E_of(r); }
          ++qk;
        }
        if ((mt >> r) & 1u) {
          if (qt < (uint32_t)kTopList) { fs.t_key[qt] = key[r]; fs.t_idx[qt] = idx[r]; }
          ++qt;
        }
      }
    }
    __syncthreads();
    if (fs.n_memb > (uint32_t)kMembers || fs.n_top > (uint32_t)kTopList) return 9;   // uniform
  }
  // best-n (upper half of the workgroup) and the k-th largest (lower half) side by side
  // The gathered list holds every element at or above the bin of the n-th best, so an entry's
  // rank in this list is its rank in the row.  Up to 64 entries are ranked by one wave out of
  // its own registers; longer lists by half the workgroup out of LDS.
  const uint32_t nt_all = (a.k_lp >= 0 && n_top > 0) ? (uint32_t)__builtin_amdgcn_readfirstlane((int)fs.n_top) : 0u;
  if (nt_all > 0 && nt_all <= (uint32_t)kWave) {
    if (wave == 1) {
      const int cols = 1 + a.k_lp;
      const uint32_t kt = fs.t_key[lane], v = fs.t_idx[lane];
      uint32_t rank = 0;
      for (uint32_t q = 0; q < nt_all; ++q) {
        const uint32_t kq = (uint32_t)__builtin_amdgcn_readlane((int)kt, (int)q);
        const uint32_t iq = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)q);
        rank += (uint32_t)((kq > kt) | ((kq == kt) & (iq < v)));
      }
      if ((uint32_t)lane < nt_all && rank < n_top) {
        a.out_lp_ids[(size_t)b * cols + 1 + rank] = (int)v;
        a.out_lp[(size_t)b * cols + 1 + rank] = (float)((double)value_of(kt) - (double)m - lnZ);
      }
    }
  } else if (nt_all > 0 && tid >= NT / 2) {
    const int cols = 1 + a.k_lp;
    const uint32_t nt = nt_all;
    const uint32_t t = (uint32_t)(tid - NT / 2);
    if (t < nt) {
      const uint32_t kt = fs.t_key[t], v = fs.t_idx[t];
      uint32_t rank = 0;
#pragma unroll 8
      for (uint32_t q = 0; q < nt; ++q) {
        const uint32_t kq = fs.t_key[q];
        rank += (kq > kt || (kq == kt && fs.t_idx[q] < v)) ? 1u : 0u;
      }
      if (rank < n_top) {
        a.out_lp_ids[(size_t)b * cols + 1 + rank] = (int)v;
        a.out_lp[(size_t)b * cols + 1 + rank] = (float)((double)value_of(kt) - (double)m - lnZ);
      }
    }
  }
  uint32_t key_k = 0;
  unsigned long long S1 = S0;
  if (k_act) {
    const uint32_t nm = (uint32_t)__builtin_amdgcn_readfirstlane((int)fs.n_memb), k_rem = (uint32_t)rp.top_k - fs.above_k;
    if (nm <= (uint32_t)kWave) {
      if (wave == 0) {                    // members in the lanes of one wave, compared through readlane
        const uint32_t kt = fs.m_key[lane];
        const unsigned long long Et = fs.m_E[lane];
        uint32_t gt = 0, ge = 0;
        unsigned long long sum_ge = 0;
        for (uint32_t q = 0; q < nm; ++q) {
          const uint32_t kq = (uint32_t)__builtin_amdgcn_readlane((int)kt, (int)q);
          const unsigned long long Eq = readlane_u64(Et, (int)q);
          gt += kq > kt; ge += kq >= kt;
          sum_ge += kq >= kt ? Eq : 0ull;
        }
        if ((uint32_t)lane < nm && gt < k_rem && k_rem <= ge) { fs.key_k = kt; fs.s1_part = sum_ge; }
      }
    } else if ((uint32_t)tid < nm) {
      const uint32_t kt = fs.m_key[tid];
      uint32_t gt = 0, ge = 0;
      unsigned long long sum_ge = 0;
#pragma unroll 8
      for (uint32_t q = 0; q < nm; ++q) {
        const uint32_t kq = fs.m_key[q];
        gt += kq > kt; ge += kq >= kt;
        sum_ge += kq >= kt ? fs.m_E[q] : 0ull;
      }
      // the k-th largest of the row: ties write the same two values
      if (gt < k_rem && k_rem <= ge) { fs.key_k = kt; fs.s1_part = sum_ge; }
    }
    __syncthreads();
    key_k = fs.key_k;
    S1 = hm[bin_k] + fs.s1_part;
  }

  int token = best_i;
  uint32_t token_key = key_of(m);
  if (!rp.greedy) {
    // ---- (7) top-p
    // every element missing from the list fails min-p  <=>  the completeness threshold itself fails it
    const bool minp_bounds = minp_on && !(__fsub_rn(s_c, m) >= t_minp);
    uint32_t key_cut = key_k;
    bool whole_row = false;
    if (rp.top_p < 1.0f) {
      const double lim = ceil((double)rp.top_p * (double)S1);
      const unsigned long long limit = lim > 0.0 ? (unsigned long long)lim : 0ull;
      const int lowbin = k_act ? bin_k : 1;
      {
        const int b0 = kBins - 1 - kBinsPerThread * tid;
        int mine = 1 << 30;
#pragma unroll
        for (int j = 0; j < kBinsPerThread; ++j) {
          const int bin = b0 - j;
          if (bin >= lowbin && hc[bin] && hm[bin] < limit) mine = bin;       // bins descend: the last one wins
        }
        const uint32_t wmin = last_lane_u32(dpp_scan_min_u32((uint32_t)mine));
        if (lane == kWave - 1 && wmin < (1u << 30)) atomicMin(&fs.bin_p, (int)wmin);
      }
      __syncthreads();
      const int bin_p = fs.bin_p;
      if (bin_p >= kBins) return 10;                                          // uniform (p <= 0)
      {
        mask_t mp = 0;
#pragma unroll
        for (int r = 0; r < NE; ++r)
          if (live(r) && idx[r] != kNoIdx) mp |= (mask_t)((key[r] >= key_k) & (b_of(r) == bin_p)) << r;
        if (mp) {
          uint32_t q = atomicAdd(&fs.n_memb2, (uint32_t)__popcll((unsigned long long)mp));
#pragma unroll
          for (int r = 0; r < NE; ++r) {
            if ((mp >> r) & 1u) {
              if (q < (uint32_t)kMembers) { fs.m_key[q] = key[r]; fs.m_E[q] = E_of(r); }
              ++q;
            }
          }
        }
      }
      __syncthreads();
      const uint32_t nm = (uint32_t)__builtin_amdgcn_readfirstlane((int)fs.n_memb2);
      if (nm > (uint32_t)kMembers) {                                          // uniform
        if (k_act) return 9;
        // (without top-k what settles a cut below the list settles this one too)
        if (tid == 0) { fs.limit_out = limit; fs.lnz_out = lnZ; fs.has_pen_out = has_pen; fs.second_list_out = 0; }
        return kWholeRowCut;
      }
      if (nm <= (uint32_t)kWave) {
        if (wave == 0) {
          const uint32_t kt = fs.m_key[lane];
          const unsigned long long Et = fs.m_E[lane];
          unsigned long long G = hm[bin_p];
          for (uint32_t q = 0; q < nm; ++q) {
            const uint32_t kq = (uint32_t)__builtin_amdgcn_readlane((int)kt, (int)q);
            const unsigned long long Eq = readlane_u64(Et, (int)q);
            G += kq > kt ? Eq : 0ull;
          }
          const bool member = (uint32_t)lane < nm;
          const uint32_t kp = last_lane_u32(dpp_scan_min_u32((member && G < limit) ? kt : 0xFFFFFFFFu));
          const bool drop = __any(member && !(G < limit));
          if (lane == 0) { fs.key_p = kp; if (drop) fs.dropped = 1; }
        }
      } else if ((uint32_t)tid < nm) {
        const uint32_t kt = fs.m_key[tid];
        unsigned long long G = hm[bin_p];
#pragma unroll 8
        for (uint32_t q = 0; q < nm; ++q)
          if (fs.m_key[q] > kt) G += fs.m_E[q];
        if (G < limit) atomicMin(&fs.key_p, kt); else fs.dropped = 1;
      }
      __syncthreads();
      const bool inside = k_act || bin_p > fs.bin_low || fs.dropped != 0;
      if (!inside && !minp_bounds) {
        // uniform: the cut may lie below the list; it is settled, and the token drawn, over the
        // whole row by the caller (out of this function: code that is rarely needed slows it down)
        if (tid == 0) {
          fs.limit_out = limit; fs.lnz_out = lnZ; fs.has_pen_out = has_pen;
          fs.second_list_out = minp_on;
        }
        return kWholeRowCut;
      }
      key_cut = max(key_k, fs.key_p);
    } else if (!k_act && !minp_bounds) {
      if (minp_on) return 12;                                                 // uniform: min-p reaches below the list
      whole_row = true;                                                       // no filter at all: every token is kept
    }

    if (whole_row) {
      if (tid == 0) { fs.limit_out = 0; fs.lnz_out = lnZ; fs.has_pen_out = has_pen; }
      return kWholeRow;                                                       // uniform: finished by the caller
    } else {
      // ---- (8) draw: kept mass per index bin, prefix, then resolve inside the crossing bin
      auto kept = [&](uint32_t k) {
        return k >= key_cut && k > key_c && (!minp_on || __fsub_rn(value_of(k), m) >= t_minp);
      };
      int ishift = 0;
      while (((V - 1) >> ishift) >= kBins) ++ishift;
      mask_t keptmask = 0;                                // bit r: register entry r is in the kept set
#pragma unroll
      for (int r = 0; r < NE; ++r) {
        if (live(r) && idx[r] != kNoIdx && kept(key[r])) {
          const unsigned long long E = E_of(r);
          if (E) { atomicAdd(&hd[idx[r] >> ishift], E); keptmask |= (mask_t)1 << r; }
        }
      }
      __syncthreads();
      unsigned long long target;
      {
        const int b0 = kBinsPerThread * tid;                 // ascending index order
        unsigned long long w[kBinsPerThread], msum = 0;
#pragma unroll
        for (int j = 0; j < kBinsPerThread; ++j) { w[j] = hd[b0 + j]; msum += w[j]; }
        const unsigned long long minc = dpp_scan_add_u64(msum);
        if (lane == kWave - 1) fs.r64[wave] = minc;
        __syncthreads();
        unsigned long long ex = minc - msum, S3 = 0;
#pragma unroll
        for (int ww = 0; ww < kFinalWaves; ++ww) {
          if (ww < wave) ex += fs.r64[ww];
          S3 += fs.r64[ww];
        }
        target = (__umul64hi(j24, S3) << 40) | ((j24 * S3) >> 24);             // floor(j * S3 / 2^24)
#pragma unroll
        for (int j = 0; j < kBinsPerThread; ++j) {
          if (ex <= target && target < ex + w[j]) { fs.bin_d = b0 + j; fs.before_d = ex; }
          ex += w[j];
        }
      }
      __syncthreads();
      const int bin_d = fs.bin_d;
      if (bin_d < 0) return 13;                                               // uniform (no kept mass)
      {
        mask_t md = 0;
#pragma unroll
        for (int r = 0; r < NE; ++r) md |= (mask_t)(((keptmask >> r) & 1u) & (mask_t)((int)(idx[r] >> ishift) == bin_d)) << r;
        if (md) {
          uint32_t q = atomicAdd(&fs.n_memb3, (uint32_t)__popcll((unsigned long long)md));
#pragma unroll
          for (int r = 0; r < NE; ++r) {
            if ((md >> r) & 1u) {
              if (q < (uint32_t)kMembers) { fs.m_key[q] = key[r]; fs.m_idx[q] = idx[r]; fs.m_E[q] = E_of(r); }
              ++q;
            }
          }
        }
      }
      __syncthreads();
      const uint32_t nm = (uint32_t)__builtin_amdgcn_readfirstlane((int)fs.n_memb3);
      if (nm > (uint32_t)kMembers) return 9;                                  // uniform
      if (nm <= (uint32_t)kWave) {
        if (wave == 0) {
          const uint32_t v = fs.m_idx[lane], kt = fs.m_key[lane];
          const unsigned long long Et = fs.m_E[lane];
          unsigned long long C = fs.before_d;
          for (uint32_t q = 0; q < nm; ++q) {
            const uint32_t iq = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)q);
            const unsigned long long Eq = readlane_u64(Et, (int)q);
            C += iq <= v ? Eq : 0ull;
          }
          // members have mass > 0 and distinct indices: exactly one of them is the first crossing
          if ((uint32_t)lane < nm && C > target && C - Et <= target) { fs.token = (int)v; fs.token_key = kt; }
        }
      } else if ((uint32_t)tid < nm) {
        const uint32_t v = fs.m_idx[tid];
        unsigned long long C = fs.before_d;
#pragma unroll 8
        for (uint32_t q = 0; q < nm; ++q)
          if (fs.m_idx[q] <= v) C += fs.m_E[q];
        // members have mass > 0 and distinct indices: exactly one of them is the first crossing
        if (C > target && C - fs.m_E[tid] <= target) { fs.token = (int)v; fs.token_key = fs.m_key[tid]; }
      }
      __syncthreads();
      token = fs.token;
      if (token == 0x7FFFFFFF) return 13;                                     // uniform
      token_key = fs.token_key;
    }
  }

  // ---- (9) the token and its logprob.  Past this point nothing can fail.
  if (tid == 0) {
    a.out_ids[b] = token;
    if (a.k_lp >= 0) {
      const int cols = 1 + a.k_lp;
      a.out_lp_ids[(size_t)b * cols] = token;
      a.out_lp[(size_t)b * cols] = (float)((double)value_of(token_key) - (double)m - lnZ);
    }
  }
  return 1;
}

// Second attempt for a row whose candidate list turned out too short: this workgroup reads
// the row again (it is still in the last-level cache) with a lower threshold `Tc` and leaves
// the result where the first attempt's data was: one segment of S * cap_c entries and one
// chunk summary.  Same arithmetic as stream_kernel; `bm` (if not null) is the row's history
// bitmap that the first attempt left in LDS: tokens in it stay out of the bulk mass.
template <int DT>
__device__ __attribute__((noinline)) void restream_row(const Args& a, const int b, const RowParams rp, const float Tc,
                                                       lds_ptr<FastShared> fs_lds, lds_ptr<const uint32_t> bm_lds) {
  FastShared& fs = *(FastShared*)fs_lds;
  const uint32_t* const bm = (const uint32_t*)bm_lds;
  constexpr int NT = kFinalThreads;
  constexpr int EPL = (DT == SIP_F32) ? 4 : 8;
  constexpr int ESZ = (DT == SIP_F32) ? 4 : 2;
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int V = a.V;
  const char* row = reinterpret_cast<const char*>(a.logits) + (size_t)b * (size_t)a.row_stride * ESZ;
  uint2* region = a.cand + (size_t)b * (size_t)a.S * (size_t)a.cap_c;
  const uint32_t cap = (uint32_t)(a.S * a.cap_c);
  const BulkRef ref = make_bulk_ref(Tc, log2_scale(rp));
  __syncthreads();
  if (tid == 0) fs.rq_n = 0;
  __syncthreads();
  float acc = 0.0f;
  constexpr int UNR = 4;                                    // loads in flight per thread
  for (int t0 = 0; t0 < V; t0 += UNR * NT * EPL) {
    uint4 q[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int e0 = t0 + (u * NT + tid) * EPL;
      q[u] = e0 < V ? *reinterpret_cast<const uint4*>(row + (size_t)e0 * ESZ) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int e0 = t0 + (u * NT + tid) * EPL;
      float z[EPL];
      if (DT == SIP_F32) {
        z[0] = __uint_as_float(q[u].x); z[1] = __uint_as_float(q[u].y);
        z[2] = __uint_as_float(q[u].z); z[3] = __uint_as_float(q[u].w);
      } else {
        const uint32_t w[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          z[2 * i] = __uint_as_float(w[i] << 16);
          z[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
      }
      float g = 0.0f;
      // the elements of one load share a bitmap word (e0 is a multiple of EPL <= 8)
      const uint32_t hw = bm ? bm[min(e0, V - 1) >> 5] >> (e0 & 31) : 0u;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        if (e0 + i >= V) z[i] = -INFINITY;
        const bool hit = z[i] >= ref.Tc;
        if (hit) {
          const uint32_t pos = atomicAdd(&fs.rq_n, 1u);
          if (pos < cap) region[pos] = make_uint2(__float_as_uint(z[i]), (uint32_t)(e0 + i));
        }
        float e = bulk_term(bulk_arg(z[i], ref));
        e = (hit || ref.none || ((hw >> i) & 1u)) ? 0.0f : e;
        g += e;
      }
      acc += g;
    }
  }
  const unsigned long long wsum = dpp_scan_add_u64(bulk_units(acc));
  if (lane == kWave - 1) fs.r64[wave] = wsum;
  __syncthreads();
  if (tid == 0) {
    ChunkOut o;
    o.bulk = 0;
    for (int w = 0; w < kFinalWaves; ++w) o.bulk += fs.r64[w];
    o.Tc = ref.Tc; o.off = published_off(ref);
    o.cnt = fs.rq_n;
    o.n_blk = 0; o.unit = ref.unit;
    a.chunks[(size_t)b * a.S] = o;
  }
  // what this workgroup wrote to global memory is read back by other waves of it
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// Rarely needed continuations, defined after the kernel (see there).
template <int DT>
__device__ int whole_row_finish(const Args& a, const int b, const RowParams rp, lds_ptr<unsigned char> dyn_lds,
                                lds_ptr<FastShared> fs_lds, const bool cut);

// Runs the smallest instantiation of fast_row that can hold the row: the history length bounds
// the number of distinct tokens; a variant that turns out too small says so early and the next
// one starts over.  Three variants, one after the other: every further instantiation in this
// kernel was measured to slow all of them down (0.6-1 us each).
template <int DT, bool SH>
__device__ __forceinline__ int fast_any(const Args& a, const int b, const RowParams& rp, unsigned char* dyn,
                                        FastShared& fs, const int S, const int cap_c, const long long ndist_ub) {
  constexpr int NT = kFinalThreads;
  int r = kNeedLong;
  if (ndist_ub <= 2 * NT) r = fast_row<DT, 8, 2, SH>(a, b, rp, dyn, fs, S, cap_c);
  if (r == kNeedLong) r = fast_row<DT, 8, 8, SH>(a, b, rp, dyn, fs, S, cap_c);
  if (r == kNeedLong || r == kNeedLongList) r = fast_row<DT, kCandLong, 8, SH>(a, b, rp, dyn, fs, S, cap_c);
  return (r == kNeedLong || r == kNeedLongList) ? 5 : r;
}

// One row that the finishing logic could not settle from its list is taken through the heavier
// logic below -- the same list in larger register variants, a second and longer list, the
// continuations over the whole row, the exact multi-pass path -- by the calling workgroup.
// `dynraw`: final_lds_fixed(V) (and at least 2 * ceil(V / 32) words) of LDS.
// Bitmap over the vocabulary of the row's history (and prompt) tokens, as restream_row() wants it.
__device__ __forceinline__ void history_bitmap(const Args& a, const int b, const PenaltyPlan& pen, uint32_t* bm) {
  const int W = (a.V + 31) / 32, V = a.V;
  for (int w = threadIdx.x; w < W; w += kFinalThreads) bm[w] = 0;
  __syncthreads();
  for (long long i = pen.h.lo + threadIdx.x; i < pen.h.hi; i += kFinalThreads) {
    const int t = a.tokens[i];
    if (t >= 0 && t < V) atomicOr(&bm[t >> 5], 1u << (t & 31));
  }
  for (long long i = pen.p_lo + threadIdx.x; i < pen.p_hi; i += kFinalThreads) {
    const int t = a.p_tokens[i];
    if (t >= 0 && t < V) atomicOr(&bm[t >> 5], 1u << (t & 31));
  }
  __syncthreads();
}

// `seen`: what a finishing attempt on the row's first list has already found out (finish_row()
// in the same workgroup), or nothing.
struct RescueSeen {
  int why = 0;               // finish_row()'s code; 0 = nothing is known
  float m = 0.0f, zmax = 0.0f, T = 0.0f;
};
template <int DT, bool SH>
__device__ __forceinline__ void rescue_row(const Args& a, const int b, unsigned char* dynraw, ExactShared& ex,
                                           FastShared& fs, const RescueSeen seen = RescueSeen()) {
  const RowParams rp = load_row_params(a, b);
  int how = 2;                                   // 2: not eligible for the single-pass path
  int code = 0;
  bool gathered = false;                         // sharded logits: the row has been put together in the workspace
  const int target = candidate_target(rp, a);
  if (target != 0) {
    // Upper bound on the row's distinct history tokens, which decides the instantiation that is
    // tried first: the history's length, or what a device-resident state remembers from the
    // slot's previous call.
    const PenaltyPlan pen0 = penalty_plan(a, b, rp.theta, rp.phi, rp.psi);
    const HistRange hr = pen0.h;
    long long ndist_ub = (hr.hi - hr.lo) + (pen0.p_hi - pen0.p_lo);
    if (a.slot && hr.hi > hr.lo) {
      const int hint = a.st_ndist[a.slot[b]];
      if (hint >= 0 && hint < ndist_ub) ndist_ub = hint;
    }
    if (threadIdx.x == 0) fs.ndist_out = -1;
    // At most two attempts, and a look at the first list again, written as a loop so that the kernel holds one copy
    // of the code.
    int S = a.one_seg ? 1 : a.S, cap_c = a.one_seg ? a.S * a.cap_c : a.cap_c;
#pragma nounroll
    for (int attempt = 0; attempt < 3; ++attempt) {
      int r;
      bool cut_below = false;
      const bool skipped = attempt == 0 && (seen.why == 12 || (seen.why == 11 && rp.min_p > 0.0f));
      if (skipped) {
        // The first list has been looked at already and is known to be too short for a cut whose
        // place a second list can reach: go straight on to that one.
        r = seen.why;
        cut_below = seen.why == 11;
        if (threadIdx.x == 0) { fs.m_out = seen.m; fs.zmax_out = seen.zmax; fs.trow_out = seen.T; }
      } else {
        r = fast_any<DT, SH>(a, b, rp, dynraw, fs, S, cap_c, ndist_ub);
      }
      if (attempt == 0 && r == kWholeRowCut) {
        // with min-p on, the kept set ends at the min-p threshold at the latest, which is known exactly by now:
        // a second list cut there settles the row if it fits.  (Without it the row's one read in
        // whole_row_window() is no dearer than a second list, which besides may turn out too short: V = 128256
        // bf16, 256 rows, 244 with nuclei beyond their lists, 247 us a call with second lists, 130 without.)
        __syncthreads();
        if (fs.second_list_out) { r = 11; cut_below = true; }
      }
      if (attempt == 2) { how = r; break; }
      if (attempt == 1) {
        const bool fine = r == 1 || r == kWholeRowCut || r == kWholeRow;
        how = fine ? r : 16 + r;                 // 17..29: failed again after the retry
        if (fine) code = 15;                     // 15: finished by the retry (still one HBM pass)
        break;
      }
      how = r;
      if (r != 8 && r != 11 && r != 12) break;
      // The list was complete but too short.  Where min-p is on, the threshold that bounds the
      // kept set is known exactly now that the maximum is; otherwise lower the threshold by
      // three tenths of its distance to the maximum.  One retry, then the exact path.
      __syncthreads();
      const float m = fs.m_out, zmax = fs.zmax_out, t_old = fs.trow_out;
      float t_new = t_old - 0.3f * (zmax - t_old);
      if (rp.min_p > 0.0f && !rp.greedy) {
        const float zt = (m + (float)log((double)rp.min_p)) * rp.tau;
        t_new = fminf(t_new, zt - 1.0e-5f * fabsf(zt) - 1.0e-30f);
        if (r != 8) t_new = zt - 1.0e-5f * fabsf(zt) - 1.0e-30f;
      }
      if (!(t_new < t_old)) break;
      if (SH && !gathered) { gather_row<DT>(a, b); gathered = true; }
      const PenaltyPlan pen1 = penalty_plan(a, b, rp.theta, rp.phi, rp.psi);
      const uint32_t* bm1 = pen1.any ? reinterpret_cast<const uint32_t*>(dynraw) : nullptr;
      if (skipped && pen1.any) history_bitmap(a, b, pen1, reinterpret_cast<uint32_t*>(dynraw));   // (else the first attempt left it there)
      restream_row<DT>(a, b, rp, t_new, in_lds(&fs), in_lds(bm1));
      S = 1; cap_c = a.S * a.cap_c;
      if (cut_below && fs.rq_n > (uint32_t)min(kFinalThreads * kCandLong, a.S * a.cap_c)) {
        // The second list does not fit either: the cut is settled over the whole row, from the
        // tables of an attempt on the first list -- which are there, untouched, unless that
        // attempt was skipped: then the first list is made again (the second one lies where it
        // was) and looked at now.
        how = kWholeRowCut;
        if (!skipped) break;
        restream_row<DT>(a, b, rp, t_old, in_lds(&fs), in_lds(bm1));
        attempt = 1;
      }
    }
  }
  if (how == kWholeRowCut || how == kWholeRow) {
    // rows that are finished over the whole row: nucleus cut below the list, or no filter at all
    if (SH && !gathered) { gather_row<DT>(a, b); gathered = true; }
    how = whole_row_finish<DT>(a, b, rp, in_lds(dynraw), in_lds(&fs), how == kWholeRowCut);
    code = how == 1 ? 16 : 0;                    // 16: finished over the whole row by this workgroup
  }
  if (how != 1) {
    __syncthreads();
    if (SH && !gathered) { gather_row<DT>(a, b); gathered = true; }
    exact_row<DT>(a, b, in_lds(reinterpret_cast<uint32_t*>(dynraw)), in_lds(&ex));
  }
  if (threadIdx.x == 0) a.row_path[b] = code ? code : how;
  if (a.slot) {                                  // device-resident history: the row's id joins it
    __syncthreads();
    if (threadIdx.x == 0) state_append_row(a, b);
  }
}

// The rows that the kernel before it could not settle (row_why is not 1), one workgroup per row at a
// time.  Launched with a fixed, small grid; every wave looks at all the codes for itself, so that nothing
// has to be counted (and nothing set to zero) ahead of it, and no wave waits for another to find that
// there is nothing to do.  Nothing to rescue, 1024 rows: 4.2 us (6.3 with the codes counted through LDS and a
// frame of 504 bytes a lane, which also cost the kernel before it 2 us of 111).
template <int DT, bool SH>
__global__ __launch_bounds__(kFinalThreads) void rescue_kernel(Args a_by_value) {
  // The arguments are read where they are used, straight from the kernel-argument segment
  // (the struct is the only parameter, so it starts at offset 0), instead of being held in
  // scalar registers from the first instruction on: there are more of them than registers.
  (void)a_by_value;
  const Args& a = *(const Args*)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __align__(16) unsigned char dynraw[];
  __shared__ ExactShared ex;
  __shared__ FastShared fs;
  // Every wave looks at the codes for itself, kSpan rows at a time: nothing to share, and nothing to wait for.
  constexpr int kLook = 16, kSpan = kLook * kWave;
  const int lane = lane_id();
  int base = 0;
  uint32_t seen = 0;                                   // unsettled rows ahead of `base`
  auto row_of = [&](uint32_t rank) -> int {            // the row with that rank among the unsettled, -1 = none
#pragma nounroll
    for (; base < a.B; base += kSpan) {
      int code[kLook];
#pragma unroll
      for (int j = 0; j < kLook; ++j) code[j] = a.row_why[min(base + j * kWave + lane, a.B - 1)];
      uint32_t before = seen;
      int row = -1;
#pragma unroll
      for (int j = 0; j < kLook; ++j) {
        const unsigned long long bad = __ballot(code[j] != 1 && base + j * kWave + lane < a.B);
        const uint32_t n = (uint32_t)__popcll(bad), k = rank - before;
        if (row < 0 && k < n) {
          const uint32_t mine = __builtin_amdgcn_mbcnt_hi((uint32_t)(bad >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bad, 0u));
          const unsigned long long at = __ballot(((bad >> lane) & 1ull) && mine == k);
          row = base + j * kWave + __ffsll((long long)at) - 1;
        }
        before += n;
      }
      if (row >= 0) return row;
      seen = before;
    }
    return -1;
  };
#pragma nounroll
  for (uint32_t round = 0;; ++round) {
    // (every round is dealt out turned by one against the round before, so that a batch whose rows alternate
    // between cheap and dear does not give one workgroup the dear ones of several rounds.  V = 42037 bf16, 351
    // rows on the exact path, every other one greedy: 801 us a call, 562 so.)
    const int b = row_of(round * gridDim.x + (blockIdx.x + round) % gridDim.x);
    if (b < 0) return;                                 // uniform: all waves have seen the same codes
    rescue_row<DT, SH>(a, b, dynraw, ex, fs);
    __syncthreads();                                   // done with the tables in LDS
  }
}

// Where fast_row() leaves its tables in LDS, for what continues over the whole row.
struct WholeRowTables {
  const uint32_t* bm;                       // the row's history, one bit per token
  const unsigned short* pre;                // history tokens ahead of a word of it
  unsigned long long *hm, *hd;              // kBins each
  uint32_t* hc;                             // kBins
  const uint32_t* cnt;                      // keys of the history tokens' values, in the order of their ids
  __device__ __forceinline__ WholeRowTables(unsigned char* dyn, const int V) {
    const int W = (V + 31) >> 5;
    bm = reinterpret_cast<const uint32_t*>(dyn);
    pre = reinterpret_cast<const unsigned short*>(dyn + (size_t)W * 4);
    hm = reinterpret_cast<unsigned long long*>(dyn + (((size_t)W * 6 + 15) / 16) * 16);
    hd = hm + kBins;
    hc = reinterpret_cast<uint32_t*>(hd + kBins);
    cnt = hc + kBins;
  }
};

// Draw over the whole row, for a row without any filter (plain temperature sampling).  Maximum,
// total mass and best-n came from the list; the draw itself needs every element's mass in
// vocabulary order, so the row is read once more here (it is still in the last-level cache),
// plus the one block in which the running mass crosses the target.  Out of line: rarely needed,
// and the finishing kernel gets slower with every piece of code inlined into it.  Leaves the
// token and its key in fs; returns 1, or 13 if there is no mass to draw from.
template <int DT>
__device__ __attribute__((noinline)) int whole_row_draw(const char* row, const int V, const bool has_pen,
                                                        lds_ptr<unsigned char> dyn_lds, lds_ptr<FastShared> fs_lds,
                                                        const float tau, const bool greedy, const float m,
                                                        const float zmax, const float c_row,
                                                        const unsigned long long j24) {
  const WholeRowTables tables((unsigned char*)dyn_lds, V);
  const uint32_t* const bm = tables.bm; const unsigned short* const pre = tables.pre; const uint32_t* const cnt = tables.cnt;
  unsigned long long* const hd = tables.hd;
  FastShared& fs = *(FastShared*)fs_lds;
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  auto scaled_s = [&](float z) { return greedy ? z : __fdiv_rn(z, tau); };
  constexpr int EPL = (DT == SIP_F32) ? 4 : 8;
  constexpr int ESZ = (DT == SIP_F32) ? 4 : 2;
  const int e_last = ((V - 1) / EPL) * EPL;
  auto ldrow = [&](int e0) {                            // clamped: always a valid address
    return load_global(row + (size_t)min(e0, e_last) * ESZ);
  };
  // Masses as fp32, relative to the maximum; a lane adds those of one 16-byte load in a fixed
  // order and only the sum becomes an integer (units of 2^-40), so that both reads of the row
  // agree bit for bit on every partial sum while converting once per load, not per element.
  auto masses = [&](const uint4& q, int e0, float (&E)[EPL], uint32_t (&keys)[EPL]) {
    float z[EPL];
    if (DT == SIP_F32) {
      z[0] = __uint_as_float(q.x); z[1] = __uint_as_float(q.y);
      z[2] = __uint_as_float(q.z); z[3] = __uint_as_float(q.w);
    } else {
      const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[2 * i] = __uint_as_float(w4[i] << 16);
        z[2 * i + 1] = __uint_as_float(w4[i] & 0xFFFF0000u);
      }
    }
    // the elements of one load share a bitmap word (e0 is a multiple of EPL <= 8)
    const uint32_t word = has_pen ? bm[min(e0, V - 1) >> 5] : 0u;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int v = e0 + i;
      E[i] = 0.0f; keys[i] = 0;
      if (v < V) {
        if ((word >> (v & 31)) & 1u) {                                     // carries a penalty: value from the list
          const float sv = value_of(cnt[pre[v >> 5] + __popc(word & ((1u << (v & 31)) - 1u))]);
          keys[i] = key_of(sv);
          E[i] = expf(__fsub_rn(sv, m));
        } else {
          // exp(z/tau - max) as 2^((z - zmax) * c): no division, hardware exp2; the two passes
          // below use the same expression, which is all the draw needs
          keys[i] = __float_as_uint(z[i]);                                 // raw bits, turned into a key on a hit
          E[i] = __builtin_amdgcn_exp2f(__fmul_rn(__fsub_rn(z[i], zmax), c_row));
        }
      }
    }
  };
  // first read: mass of every block of BLK consecutive elements (one block = UNR loads per
  // lane of one wave) into hd[] (still all zero); waves take contiguous runs of blocks
  constexpr int UNR = 4;
  constexpr int BLK = UNR * kWave * EPL;
  const int nblk = (V + BLK - 1) / BLK;                 // <= kBins because V <= 262144
  const int per_wave = (nblk + kFinalWaves - 1) / kFinalWaves;
  for (int blk = wave * per_wave; blk < min(nblk, (wave + 1) * per_wave); ++blk) {
    const int base = blk * BLK;
    uint4 q[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) q[u] = ldrow(base + (u * kWave + lane) * EPL);
    unsigned long long mine = 0;
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      float E[EPL];
      uint32_t keys[EPL];
      masses(q[u], base + (u * kWave + lane) * EPL, E, keys);        // zero past the end of the row
      float part = 0.0f;
#pragma unroll
      for (int i = 0; i < EPL; ++i) part += E[i];
      mine += fix_of(part);
    }
    mine = dpp_scan_add_u64(mine);
    if (lane == kWave - 1) hd[blk] = mine;
  }
  __syncthreads();
  // prefix over the blocks, find the block that holds the crossing
  unsigned long long target;
  {
    const int b0 = kBinsPerThread * tid;
    unsigned long long w[kBinsPerThread], msum = 0;
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) { w[j] = hd[b0 + j]; msum += w[j]; }
    const unsigned long long minc = dpp_scan_add_u64(msum);
    if (lane == kWave - 1) fs.r64[wave] = minc;
    __syncthreads();
    unsigned long long ex = minc - msum, S3 = 0;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) {
      if (ww < wave) ex += fs.r64[ww];
      S3 += fs.r64[ww];
    }
    target = (__umul64hi(j24, S3) << 40) | ((j24 * S3) >> 24);           // floor(j * S3 / 2^24)
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) {
      if (ex <= target && target < ex + w[j]) { fs.bin_d = b0 + j; fs.before_d = ex; }
      ex += w[j];
    }
  }
  __syncthreads();
  const int blk_d = fs.bin_d;
  if (blk_d < 0) return 13;                                               // uniform (no mass at all)
  // second read, one block, one wave: lane prefixes in vocabulary order
  if (wave == 0) {
    const int base = blk_d * BLK;
    unsigned long long running = fs.before_d;
    int found = -1;
    uint32_t found_key = 0;
    uint4 q[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) q[u] = ldrow(base + (u * kWave + lane) * EPL);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int e0 = base + (u * kWave + lane) * EPL;
      float E[EPL];
      uint32_t keys[EPL];
      masses(q[u], e0, E, keys);
      float part = 0.0f;
#pragma unroll
      for (int i = 0; i < EPL; ++i) part += E[i];
      const unsigned long long lane_tot = fix_of(part);
      const unsigned long long incl = dpp_scan_add_u64(lane_tot);
      const unsigned long long c = running + incl - lane_tot;
      int hit = -1;
      uint32_t hit_key = 0;
      float upto = 0.0f;                             // same additions in the same order as `part`
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        upto += E[i];
        if (hit < 0 && E[i] > 0.0f && c + fix_of(upto) > target) { hit = e0 + i; hit_key = keys[i]; }   // key, or raw bits if unpenalised
      }
      const unsigned long long ball = __ballot(hit >= 0);
      if (ball && found < 0) {
        const int src = __ffsll((long long)ball) - 1;
        found = __builtin_amdgcn_readlane(hit, src);
        found_key = (uint32_t)__builtin_amdgcn_readlane((int)hit_key, src);
      }
      running += last_lane_u64(incl);
    }
    if (lane == 0) {
      if (found >= 0 && !(has_pen && ((bm[found >> 5] >> (found & 31)) & 1u)))
        found_key = key_of(scaled_s(__uint_as_float(found_key)));
      fs.token = found; fs.token_key = found_key;
    }
  }
  __syncthreads();
  const int token = fs.token;
  return (token == 0x7FFFFFFF || token < 0) ? 13 : 1;
}

// Nucleus and draw of a row whose cut lies below the candidate list (top-p alone on a flat
// distribution keeps tens of thousands of tokens), in two reads of the row (it is in the last-level
// cache).  The first puts the mass of every element into one of 2048 bins over the exact fp32 s,
// monotone in s so that equal values never part; the bin in which the mass of everything larger first
// stays short of the limit holds the cut.  The second sums, per block of consecutive elements, what lies
// above that bin and what lies in it, and lists the latter; once the cut among them is known (all equal:
// they are all kept) the kept ones join their blocks' sums, and one block is read again for the token.
// More members than the list takes, and not all equal: the bin becomes the interval of another pair of
// reads, at most kLevels of them.  All sums are integers.  Returns 1 (fs.token, fs.token_key), or a code:
// the caller then takes the row to the exact path.
// What bounds it: vector issue of one compute unit (about 25 instructions an element and read) and the
// first read's 64-bit LDS additions.  One row of V = 213087 bf16 whose cut falls among equal values: 1060 ->
// 261 us for the call (count and mass bins on each of up to three levels, a read to gather at most 256
// members, a read for the block masses; more equal members than that went to the exact path); eleven rows
// of V = 44143 fp32, three wide nuclei among them, 144 -> 127.  A flat row of V = 213087 bf16: 264, and 232 since
// the reads take two loads of eight elements at a time instead of four and nothing is spilled.
template <int DT>
__device__ __attribute__((noinline)) int whole_row_nucleus(const char* row, const int V, const bool has_pen,
                                                           lds_ptr<unsigned char> dyn_lds, lds_ptr<FastShared> fs_lds,
                                                           const double inv_tau, const float m, const unsigned long long limit,
                                                           const unsigned long long j24, const bool minp_on, const float t_minp) {
  const WholeRowTables tables((unsigned char*)dyn_lds, V);
  const uint32_t* const bm = tables.bm; const unsigned short* const pre = tables.pre; const uint32_t* const cnt = tables.cnt;
  unsigned long long* const hm = tables.hm; unsigned long long* const hd = tables.hd;
  FastShared& fs = *(FastShared*)fs_lds;
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  constexpr int NT = kFinalThreads;
  constexpr int EPL = (DT == SIP_F32) ? 4 : 8;
  constexpr int ESZ = (DT == SIP_F32) ? 4 : 2;
  constexpr int UNR = 16 / EPL;                           // loads in flight per thread (32 elements at once: 230 bytes of scratch a lane)
  constexpr int kLevels = 3;
  constexpr float kSpan = 28.0f;                          // exp(-28) * 2^40 < 1: nothing below has mass
  constexpr int BLK = UNR * kWave * EPL;                  // elements of a block: one wave's loads
  constexpr uint32_t kList = kBins;                       // members listed (key, block) where the bins were
  static_assert(262144 / BLK <= kBins / 2, "two sums per block in hd[]");
  const RowDivisor by_tau(inv_tau);
  const int e_last = ((V - 1) / EPL) * EPL;
  auto ldrow = [&](int e0) { return *reinterpret_cast<const uint4*>(row + (size_t)min(e0, e_last) * ESZ); };
  // s of every element of one 16-byte load (penalised elements take theirs from the slot table); NaN past the end
  auto svals = [&](const uint4& q, int e0, float (&sv)[EPL]) {
    float z[EPL];
    if (DT == SIP_F32) {
      z[0] = __uint_as_float(q.x); z[1] = __uint_as_float(q.y);
      z[2] = __uint_as_float(q.z); z[3] = __uint_as_float(q.w);
    } else {
      const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[2 * i] = __uint_as_float(w4[i] << 16);
        z[2 * i + 1] = __uint_as_float(w4[i] & 0xFFFF0000u);
      }
    }
    // the elements of one load share a bitmap word (e0 is a multiple of EPL <= 8)
    const uint32_t word = has_pen ? bm[min(e0, V - 1) >> 5] : 0u;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int v = e0 + i;
      sv[i] = v < V ? by_tau.of(z[i]) : __uint_as_float(0x7FC00000u);
      if (v < V && ((word >> (v & 31)) & 1u)) sv[i] = value_of(cnt[pre[v >> 5] + __popc(word & ((1u << (v & 31)) - 1u))]);
    }
  };
  auto mass = [&](float sv) { return mass_units(exp_nonpos(__fsub_rn(sv, m))); };   // as a list's, which the limit is from
  auto kept_minp = [&](float sv) { return !minp_on || __fsub_rn(sv, m) >= t_minp; };
  float lo[kLevels] = {m - kSpan, 0.0f, 0.0f}, sc[kLevels] = {};       // (indexed with constants only)
  int pick[kLevels] = {};
  auto bin_at = [&](int l, float sv) { return min(kBins - 1, max(0, (int)(__fsub_rn(sv, lo[l]) * sc[l]))); };
  // where s lies against the interval of level n (the picked bins of the levels above it): -1 below, 0 in it, 1 above
  auto side = [&](int n, float sv) {
    int r = 0;
#pragma unroll
    for (int l = 0; l < kLevels; ++l)
      if (l < n && r == 0) { const int d = bin_at(l, sv) - pick[l]; r = d > 0 ? 1 : (d < 0 ? -1 : 0); }
    return r;
  };
  float cur_lo = m - kSpan, cur_w = kSpan;
  unsigned long long above = 0;                           // mass of everything larger than the current interval
  const int nblk = (V + BLK - 1) / BLK;
  uint32_t key_cut = 0;
  // One interval: 1 = the cut is found, 0 = it lies among more than kList members, 11 = nothing qualifies.  (One
  // copy for the first, which settles most rows, and one for all others, with the level in a register: for the
  // first, that costs a tenth of the time.)
  auto interval = [&](auto is_first, const int level) -> int {
    constexpr bool FIRST = decltype(is_first)::value;
    const float cur_sc = (float)kBins / cur_w;
    if constexpr (FIRST) {
      lo[0] = cur_lo; sc[0] = cur_sc;
    } else {
#pragma unroll
      for (int l = 1; l < kLevels; ++l)
        if (l == level) { lo[l] = cur_lo; sc[l] = cur_sc; }
    }
    // ---- first read: mass per bin of the current interval
    __syncthreads();
    for (int i = tid; i < kBins; i += NT) { hm[i] = 0; hd[i] = 0; }
    if (tid == 0) { fs.bin_p = 1 << 30; fs.n_memb2 = 0; fs.key_p = 0xFFFFFFFFu; fs.key_k = 0; fs.bin_d = -1; fs.token = 0x7FFFFFFF; }
    __syncthreads();
    for (int t0 = tid * EPL; t0 < V; t0 += UNR * NT * EPL) {
      uint4 q[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) q[u] = ldrow(t0 + u * NT * EPL);
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float sv[EPL];
        svals(q[u], t0 + u * NT * EPL, sv);
#pragma unroll
        for (int i = 0; i < EPL; ++i)
          // (who is in the interval, bin_at() alone says: the interval's rounded lower end can lie an ulp above
          // a value of the bin that it was)
          if (sv[i] >= lo[0] && (FIRST || side(level, sv[i]) == 0)) {
            const unsigned long long E = mass(sv[i]);
            if (E) atomicAdd(&hm[min(kBins - 1, max(0, (int)(__fsub_rn(sv[i], cur_lo) * cur_sc)))], E);
          }
      }
    }
    __syncthreads();
    {
      // thread t owns bins kBins-1-4t .. kBins-4-4t; exclusive suffix mass in descending bin order
      const int b0 = kBins - 1 - kBinsPerThread * tid;
      unsigned long long w[kBinsPerThread], msum = 0;
#pragma unroll
      for (int j = 0; j < kBinsPerThread; ++j) { w[j] = hm[b0 - j]; msum += w[j]; }
      const unsigned long long minc = dpp_scan_add_u64(msum);
      if (lane == kWave - 1) fs.r64[wave] = minc;
      __syncthreads();
      unsigned long long mex = above + minc - msum;
#pragma unroll
      for (int ww = 0; ww < kFinalWaves; ++ww)
        if (ww < wave) mex += fs.r64[ww];
      int mine = 1 << 30;
      unsigned long long mex_j[kBinsPerThread];
#pragma unroll
      for (int j = 0; j < kBinsPerThread; ++j) {
        mex_j[j] = mex;
        if (w[j] && mex < limit) mine = b0 - j;           // bins descend: the last one wins
        mex += w[j];
      }
      const uint32_t wmin = last_lane_u32(dpp_scan_min_u32((uint32_t)mine));
      if (lane == kWave - 1 && wmin < (1u << 30)) atomicMin(&fs.bin_p, (int)wmin);
      __syncthreads();
      const int bp = fs.bin_p;
#pragma unroll
      for (int j = 0; j < kBinsPerThread; ++j)
        if (b0 - j == bp) fs.before_d = mex_j[j];
    }
    __syncthreads();
    const int bp = fs.bin_p;
    if (bp >= kBins) return 11;                           // uniform (limit of 0)
    if constexpr (FIRST) {
      pick[0] = bp;
    } else {
#pragma unroll
      for (int l = 1; l < kLevels; ++l)
        if (l == level) pick[l] = bp;
    }
    above = fs.before_d;
    // ---- second read: sums per block, members of the bin
    uint2* const list = reinterpret_cast<uint2*>(hm);     // (the bins are done with)
    const int per_wave = (nblk + kFinalWaves - 1) / kFinalWaves;
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0;
    for (int blk = wave * per_wave; blk < min(nblk, (wave + 1) * per_wave); ++blk) {
      const int base = blk * BLK;
      uint4 q[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) q[u] = ldrow(base + (u * kWave + lane) * EPL);
      unsigned long long A = 0, M = 0;
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float sv[EPL];
        svals(q[u], base + (u * kWave + lane) * EPL, sv);
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const int r = sv[i] >= lo[0] && kept_minp(sv[i]) ? side(FIRST ? 1 : level + 1, sv[i]) : -1;
          const unsigned long long E = r >= 0 ? mass(sv[i]) : 0ull;
          A += r > 0 ? E : 0ull;
          const bool member = r == 0 && E != 0;
          const unsigned long long ball = __ballot(member);
          if (ball) {
            M += member ? E : 0ull;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&fs.n_memb2, (uint32_t)__popcll(ball));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(ball >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball, 0u));
            if (member) {
              const uint32_t k = key_of(sv[i]);
              kmin = min(kmin, k); kmax = max(kmax, k);
              if (at < kList) list[at] = make_uint2(k, (uint32_t)blk);
            }
          }
        }
      }
      A = dpp_scan_add_u64(A); M = dpp_scan_add_u64(M);
      if (lane == kWave - 1) { hd[blk] = A; hd[kBins / 2 + blk] = M; }
    }
    if (kmax) { atomicMin(&fs.key_p, kmin); atomicMax(&fs.key_k, kmax); }
    __syncthreads();
    const uint32_t n = fs.n_memb2;
    kmin = fs.key_p; kmax = fs.key_k;
    if (kmin == kmax) {                                   // uniform: all equal, and the first of them is kept
      key_cut = kmin;
      for (int i = tid; i < nblk; i += NT) hd[i] += hd[kBins / 2 + i];
      __syncthreads();
      return 1;
    }
    if (n <= kList) {
      // the smallest key above which the mass stays short of the limit: bisection, kmax being one
      uint32_t k_lo = kmin, k_hi = kmax;                  // the answer lies in [k_lo, k_hi]
      while (k_lo < k_hi) {                               // uniform
        const uint32_t mid = k_lo + ((k_hi - k_lo) >> 1);
        unsigned long long g = 0;
        for (uint32_t q = tid; q < n; q += NT) {
          const uint32_t k = list[q].x;
          if (k > mid) g += mass(value_of(k));
        }
        g = dpp_scan_add_u64(g);
        __syncthreads();
        if (lane == kWave - 1) fs.r64[wave] = g;
        __syncthreads();
        unsigned long long G = above;
#pragma unroll
        for (int ww = 0; ww < kFinalWaves; ++ww) G += fs.r64[ww];
        if (G < limit) k_hi = mid; else k_lo = mid + 1;
      }
      key_cut = k_hi;
      for (uint32_t q = tid; q < n; q += NT)
        if (list[q].x >= key_cut) atomicAdd(&hd[list[q].y], mass(value_of(list[q].x)));
      __syncthreads();
      return 1;
    }
    cur_w = cur_w * (1.0f / (float)kBins);
    cur_lo = cur_lo + (float)bp * cur_w;
    return 0;
  };
  int found_cut = interval(std::true_type{}, 0);
#pragma nounroll
  for (int level = 1; level < kLevels && found_cut == 0; ++level) found_cut = interval(std::false_type{}, level);       // uniform
  if (found_cut != 1) return 11;                          // uniform
  // ---- prefix over the blocks, and the block that holds the crossing
  unsigned long long target;
  {
    static_assert(kBins / 2 <= 2 * NT, "two blocks per thread");
    const unsigned long long w0 = 2 * tid < nblk ? hd[2 * tid] : 0ull, w1 = 2 * tid + 1 < nblk ? hd[2 * tid + 1] : 0ull;
    const unsigned long long minc = dpp_scan_add_u64(w0 + w1);
    __syncthreads();
    if (lane == kWave - 1) fs.r64[wave] = minc;
    __syncthreads();
    unsigned long long ex = minc - w0 - w1, S3 = 0;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) {
      if (ww < wave) ex += fs.r64[ww];
      S3 += fs.r64[ww];
    }
    target = (__umul64hi(j24, S3) << 40) | ((j24 * S3) >> 24);               // floor(j * S3 / 2^24)
    if (ex <= target && target < ex + w0) { fs.bin_d = 2 * tid; fs.before_d = ex; }
    ex += w0;
    if (ex <= target && target < ex + w1) { fs.bin_d = 2 * tid + 1; fs.before_d = ex; }
  }
  __syncthreads();
  const int blk_d = fs.bin_d;
  if (blk_d < 0) return 13;                                                   // uniform (no mass at all)
  if (wave == 0) {                                                            // lane prefixes in vocabulary order
    const int base = blk_d * BLK;
    unsigned long long running = fs.before_d;
    bool found = false;
#pragma nounroll
    for (int u = 0; u < UNR && !found; ++u) {
      const int e0 = base + (u * kWave + lane) * EPL;
      float sv[EPL];
      svals(ldrow(e0), e0, sv);
      unsigned long long E[EPL], tot = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        E[i] = sv[i] >= lo[0] && kept_minp(sv[i]) && key_of(sv[i]) >= key_cut ? mass(sv[i]) : 0ull;
        tot += E[i];
      }
      const unsigned long long incl = dpp_scan_add_u64(tot);
      unsigned long long c = running + incl - tot;
      int hit = -1;
      uint32_t hit_key = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        c += E[i];
        if (hit < 0 && E[i] && c > target) { hit = e0 + i; hit_key = key_of(sv[i]); }
      }
      const unsigned long long ball = __ballot(hit >= 0);
      found = ball != 0;
      if (found && lane == __ffsll((long long)ball) - 1) { fs.token = hit; fs.token_key = hit_key; }
      running += last_lane_u64(incl);
    }
  }
  __syncthreads();
  return fs.token == 0x7FFFFFFF ? 13 : 1;
}

// The same in one read of the row, for rows that no min-p bounds.  A sample of 8192 elements says about where
// the cut lies: the mass below it is known (total less limit), so the cut lies where the sample's elements
// from below add up to their share of that, give or take three standard deviations of such a sum (2 to 3 % of
// it each on flat rows, 8 on rows whose tail is a few hundred elements).  The read then sums, per block of 1024
// elements, what lies above that window, and lists what lies in it (some thousand elements, to where the row's
// candidates were); bins over the window, and the members of one of them, settle the cut; and one block is read again
// for the token. Every decision is taken on the exact fp32 s; masses are exp_nonpos() like a list's, every element's an
// integer.  (Added up in fp32 over a load first, what weighs less than 2^-24 of its neighbour could not be drawn, and
// v_exp_f32 of a rounded product is off by 1e-6 some twenty below the maximum: that was 115 us in place of 133 in the
// first of the calls below, 96 in place of 103 in the fourth.)  Returns 1 (fs.token, fs.token_key), 13 (no mass), or
// 0: the window is too long for the room, or the cut not in it (whole_row_nucleus() then does without one).
// What bounds it: vector issue of one compute unit (some 40 instructions an element).  us a call, against a second
// list and two reads: 1 row of V = 256000 fp32, flat 269 -> 138, V = 213087 bf16 234 -> 126; V = 200000 fp32, 64
// rows, 16 of them flat 267 -> 140; V = 128256 bf16, 256 rows, 244 of them spiked at top-p 0.9 291 -> 103; V = 166557
// fp32, 1883 rows, 471 flat 752 -> 497.
template <int DT>
__device__ __attribute__((noinline)) int whole_row_window(const char* row_any, const int V_any, const bool has_pen_any,
                                                          lds_ptr<unsigned char> dyn_lds, lds_ptr<FastShared> fs_lds,
                                                          uint2* region_any, const uint32_t cap_any, const double inv_tau,
                                                          const float m, const unsigned long long limit, const float top_p,
                                                          const unsigned long long j24) {
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
  constexpr int NT = kFinalThreads;
  constexpr int EPL = (DT == SIP_F32) ? 4 : 8;
  constexpr int ESZ = (DT == SIP_F32) ? 4 : 2;
  constexpr int BLK = 1024;
  constexpr int UNR = BLK / (kWave * EPL);                // loads of a block per lane
  constexpr int SL = kSampleSize / (NT * EPL);            // sample loads per thread
  constexpr float kSpan = 28.0f;                          // exp(-28) * 2^40 < 1: nothing below has mass
  constexpr float kWide[2] = {3.0f, 1.5f};                // standard deviations on either side
  // (what a function is handed lies in vector registers, and pointers may be to anything: said to be uniform, and
  // global, they leave the loop without exec-masked branches and flat accesses: 130 -> 98 us in the fourth of these,
  // together with barriers alone, no device-wide fences, around the list)
  typedef __attribute__((address_space(1))) char global_char;
  typedef __attribute__((address_space(1))) unsigned long long global_u64;
  auto uniform_at = [](const void* p) {
    const unsigned long long at = (unsigned long long)(uintptr_t)p;
    return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
  };
  const int V = __builtin_amdgcn_readfirstlane(V_any);
  const WholeRowTables tables((unsigned char*)dyn_lds, V);
  const uint32_t* const bm = tables.bm; const unsigned short* const pre = tables.pre; const uint32_t* const cnt = tables.cnt;
  unsigned long long* const hm = tables.hm; unsigned long long* const hd = tables.hd;
  uint32_t* const hc = tables.hc;
  FastShared& fs = *(FastShared*)fs_lds;
  const bool has_pen = __builtin_amdgcn_readfirstlane(has_pen_any ? 1 : 0) != 0;
  const uint32_t cap = (uint32_t)__builtin_amdgcn_readfirstlane((int)cap_any);
  global_char* const row = (global_char*)uniform_at(row_any);
  global_u64* const region = (global_u64*)uniform_at(region_any);             // key of s | element << 32
  const RowDivisor by_tau(inv_tau);
  const int e_last = ((V - 1) / EPL) * EPL;
  typedef __attribute__((address_space(1))) const u32x4 global_x4;
  auto ldrow = [&](int e0) {
    const u32x4 q = *(global_x4*)(row + (uint32_t)min(e0, e_last) * (uint32_t)ESZ);
    return make_uint4(q.x, q.y, q.z, q.w);
  };
  auto raw = [&](const uint4& q, float (&z)[EPL]) {
    if (DT == SIP_F32) {
      z[0] = __uint_as_float(q.x); z[1] = __uint_as_float(q.y);
      z[2] = __uint_as_float(q.z); z[3] = __uint_as_float(q.w);
    } else {
      const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[2 * i] = __uint_as_float(w4[i] << 16);
        z[2 * i + 1] = __uint_as_float(w4[i] & 0xFFFF0000u);
      }
    }
  };
  // s of a load's elements; of what carries a penalty, and past the end, -inf
  auto svals = [&](const uint4& q, int e0, bool end, float (&sv)[EPL]) {
    float z[EPL];
    raw(q, z);
#pragma unroll
    for (int i = 0; i < EPL; ++i) sv[i] = by_tau.of(z[i]);
    if (has_pen) {                                        // uniform (the elements of a load share a bitmap word)
      const uint32_t bits = bm[min(e0, V - 1) >> 5] >> (e0 & 31);
#pragma unroll
      for (int i = 0; i < EPL; ++i) sv[i] = (bits >> i) & 1u ? -INFINITY : sv[i];
    }
    if (end) {
#pragma unroll
      for (int i = 0; i < EPL; ++i) sv[i] = e0 + i < V ? sv[i] : -INFINITY;
    }
  };
  auto rel = [&](float sv) { return exp_nonpos(__fsub_rn(sv, m)); };
  auto mass = [&](float sv) { return mass_units(rel(sv)); };
  // every penalised token: f(s, token) per lane that has one, all lanes of the wave together
  auto each_penalised = [&](auto&& f) {
    if (!has_pen) return;
    const int W = (V + 31) >> 5;
    for (int w0 = wave * kWave; w0 < W; w0 += NT) {
      const int w = w0 + lane;
      const uint32_t word = w < W ? bm[w] : 0u;
      uint32_t left = word;
      while (__any(left != 0u)) {
        const uint32_t bit = left & (0u - left);
        f(left != 0u, left ? value_of(cnt[pre[w] + __popc(word & (bit - 1u))]) : 0.0f, (uint32_t)(w << 5) + (uint32_t)__popc(bit - 1u));
        left &= left - 1u;
      }
    }
  };
  // ---- the window, from the sample: bins from the lowest value (or m - 28) to m, mass and number of elements
  // (Four lanes to a piece of 64 bytes.  In pieces of a wave's load, 16 of a bf16 row, a part of the ids that holds
  // most of the mass had a piece too many or too few, and the cut lay beside the window: V = 152816 bf16, 50 rows
  // with all that is likely in a sixth of the ids, 313 us a call, 174 so.  And bins from m - 28 for every row are few
  // for one whose values are all about the same, and its window too long: V = 180525 bf16, 109 rows of standard
  // deviation 0.02, 515 us, 174 so.)
  constexpr uint32_t NP = (uint32_t)(SL * NT / 4), P0 = (uint32_t)(4 * EPL);
  static_assert(16384 / NP >= P0, "the shortest row is that long: every piece lies inside");
  float smp[SL][EPL], low = INFINITY;
#pragma unroll
  for (int j = 0; j < SL; ++j) {
    const int e0 = (int)((uint32_t)(j * NT + tid) / 4u * (uint32_t)V / NP / P0 * P0) + (tid & 3) * EPL;
    svals(ldrow(e0), e0, true, smp[j]);
#pragma unroll
    for (int i = 0; i < EPL; ++i) low = smp[j][i] > -INFINITY ? fminf(low, smp[j][i]) : low;
  }
  each_penalised([&](bool have, float sv, uint32_t) { low = have && sv > -INFINITY ? fminf(low, sv) : low; });
  const uint32_t low_key = last_lane_u32(dpp_scan_min_u32(key_of(low)));
  __syncthreads();
  if (lane == 0) fs.rkey[wave] = low_key;
  for (int i = tid; i < kBins; i += NT) { hm[i] = 0; hc[i] = 0; }
  if (tid < 2) { fs.w_lo[tid] = -1; fs.w_hi[tid] = -1; }
  if (tid == 0) {
    fs.bin_p = 1 << 30; fs.bin_d = -1; fs.n_memb2 = 0; fs.key_p = 0xFFFFFFFFu; fs.key_k = 0; fs.token = 0x7FFFFFFF;
    fs.w_sq = -1.0f; fs.rq_n = 0;
  }
  __syncthreads();
  uint32_t lowest = fs.rkey[0];
#pragma unroll
  for (int ww = 1; ww < kFinalWaves; ++ww) lowest = min(lowest, fs.rkey[ww]);
  const float massless = m - kSpan, lo0 = fmaxf(massless, value_of(lowest)), span0 = m - lo0;
  if (!(span0 > 1e-30f)) return 0;                        // uniform: a sample of one value, or of none
  const float sc0 = (float)kBins / span0;
  auto bin0 = [&](float sv) { return min(kBins - 1, max(0, (int)(__fsub_rn(sv, lo0) * sc0))); };
  __syncthreads();                                        // (rkey is used again)
#pragma unroll
  for (int j = 0; j < SL; ++j)
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (smp[j][i] >= massless) {
        const int bin = bin0(smp[j][i]);
        atomicAdd(&hm[bin], mass(smp[j][i]));
        atomicAdd(&hc[bin], 1u);
      }
  // The sample's elements carry no penalty.  Those that do are all at hand, so each of them counts for its share
  // of a sample: left out, thousands put the estimate beside the cut, and the row was read twice more (V = 65536
  // fp32, 22 flat rows of 3500 tokens 205 us a call, 130 so; V = 40001, 300 rows 335, 235).
  const double share = (double)kSampleSize / (double)V;
  each_penalised([&](bool have, float sv, uint32_t) {
    if (have && sv >= massless) atomicAdd(&hm[bin0(sv)], (unsigned long long)((double)mass(sv) * share));
  });
  __syncthreads();
  {
    // thread t has bins 4t .. 4t + 3, ascending
    unsigned long long w[kBinsPerThread], msum = 0;
    uint32_t c[kBinsPerThread], csum = 0;
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) {
      w[j] = hm[kBinsPerThread * tid + j]; msum += w[j];
      c[j] = hc[kBinsPerThread * tid + j]; csum += c[j];
    }
    float sq[kBinsPerThread], ssum = 0.0f;                // squares, a bin's elements taken to weigh the same
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) { sq[j] = c[j] ? (float)w[j] / (float)c[j] * (float)w[j] : 0.0f; ssum += sq[j]; }
    const unsigned long long minc = dpp_scan_add_u64(msum);
    const uint32_t cinc = dpp_scan_add_u32(csum);
    const float sinc = dpp_scan_add_f32(ssum);
    if (lane == kWave - 1) { fs.r64[wave] = minc; fs.r32[wave] = cinc; fs.rkey[wave] = __float_as_uint(sinc); }
    __syncthreads();
    unsigned long long ex0 = minc - msum;
    uint32_t n0 = cinc - csum;
    float sq0 = sinc - ssum;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww)
      if (ww < wave) { ex0 += fs.r64[ww]; n0 += fs.r32[ww]; sq0 += __uint_as_float(fs.rkey[ww]); }
    const double below = (double)limit * (1.0 - (double)top_p) / (double)top_p * ((double)kSampleSize / (double)V);
    {
      unsigned long long ex = ex0;
      float q = sq0;
#pragma unroll
      for (int j = 0; j < kBinsPerThread; ++j) {
        if ((double)ex <= below && below < (double)(ex + w[j]))
          fs.w_sq = fmaxf(q, 0.0f) + sq[j] * (float)((below - (double)ex) / (double)w[j]);
        ex += w[j]; q += sq[j];
      }
    }
    __syncthreads();
    const double dev = sqrt((double)fmaxf(fs.w_sq, 0.0f));
    unsigned long long ex = ex0;
    uint32_t n = n0;
    double ends[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double wide = fmax((double)kWide[k >> 1] * dev, 0.02 * below);
      ends[k] = fs.w_sq < 0.0f ? -1.0 : (k & 1) ? below + wide : fmax(below - wide, 0.0);
    }
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if ((double)ex <= ends[k] && ends[k] < (double)(ex + w[j])) {
          if (k & 1) { fs.w_hi[k >> 1] = kBinsPerThread * tid + j; fs.w_n1[k >> 1] = n + c[j]; }
          else { fs.w_lo[k >> 1] = kBinsPerThread * tid + j; fs.w_n0[k >> 1] = n; }
        }
      ex += w[j]; n += c[j];
    }
  }
  __syncthreads();
  int pick = -1;
#pragma unroll
  for (int k = 1; k >= 0; --k)                            // the wider one where it fits (an eighth of the room to spare)
    if (fs.w_lo[k] >= 0 && fs.w_hi[k] >= 0 &&
        (unsigned long long)(fs.w_n1[k] - fs.w_n0[k]) * (unsigned long long)V <
            (unsigned long long)(cap - cap / 8) * (unsigned long long)kSampleSize)
      pick = k;
  if (pick < 0) return 0;                                 // uniform
  const float s_lo = lo0 + (float)fs.w_lo[pick] / sc0, s_hi = lo0 + (float)(fs.w_hi[pick] + 1) / sc0;
  if (!(s_lo < s_hi)) return 0;                           // uniform
  for (int i = tid; i < kBins; i += NT) { hm[i] = 0; hd[i] = 0; }
  __syncthreads();
  // ---- the read: sums per block of what lies above, list of what lies in the window
  const int nblk = (V + BLK - 1) / BLK;
  const int per_wave = (nblk + kFinalWaves - 1) / kFinalWaves;
  // The list is dealt out in pages of a wave's size, as they are asked for: a wave's share of the row may hold most of
  // the window (ids in order of frequency, a piece with a tail of its own).  Fixed eighths ran over there, and the
  // row was read twice more: 400 rows of V = 131072 fp32 with their tail in an eighth of the ids, top-p 0.5, 454 ->
  // 249 us; what did not run over takes 0 to 5 % longer.
  constexpr uint32_t kPage = kWave;
  const uint32_t room = cap / kPage * kPage;
  const uint32_t key_none = key_of(-INFINITY);            // of places left empty
  uint32_t at = 0, end = 0;                               // wave-uniform: the rest of the wave's page
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  lds_u32* const pages = (lds_u32*)&fs.rq_n;              // (as a flat address its answer would wait for the loads under way)
  auto push = [&](const unsigned long long mask, const bool mine, auto&& entry) {                // by all lanes
    const uint32_t to = at + (uint32_t)__popcll(mask);
    uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, at));
    if (__builtin_expect(to > end, 0)) {                  // uniform
      uint32_t page = 0;
      if (lane == 0) page = __hip_atomic_fetch_add(pages, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      page = (uint32_t)__builtin_amdgcn_readfirstlane((int)page) * kPage;
      if (pos >= end) pos = page + (pos - end);
      at = page + (to - end);
      end = page + kPage;
    } else {
      at = to;
    }
    if (mine && pos < room) region[pos] = entry();
  };
  // mass above the window; bit EPL-1-i of `in`: element i lies in it
  auto part_of = [&](const float (&sv)[EPL], uint32_t& in) -> unsigned long long {
    uint32_t not_lo = ~0u, not_hi = ~0u;
    unsigned long long part = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const float a_lo = __fsub_rn(sv[i], s_lo), a_hi = __fsub_rn(sv[i], s_hi);               // (a difference has the comparison's sign)
      not_lo = __builtin_amdgcn_alignbit(not_lo, __float_as_uint(a_lo), 31);
      not_hi = __builtin_amdgcn_alignbit(not_hi, __float_as_uint(a_hi), 31);
      part += mass_bits(a_hi >= 0.0f ? rel(sv[i]) : 0.0f);
    }
    in = ~not_lo & not_hi & ((1u << EPL) - 1u);
    return part - (unsigned long long)EPL * kMagicBits;
  };
  uint4 q[UNR], next[UNR];                                // (a block's loads and the next one's)
#pragma unroll
  for (int u = 0; u < UNR; ++u) q[u] = ldrow(wave * per_wave * BLK + (u * kWave + lane) * EPL);
  for (int blk = wave * per_wave; blk < min(nblk, (wave + 1) * per_wave); ++blk) {
    const int base = blk * BLK;
#pragma unroll
    for (int u = 0; u < UNR; ++u) next[u] = ldrow(base + BLK + (u * kWave + lane) * EPL);
    unsigned long long A = 0;
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int e0 = base + (u * kWave + lane) * EPL;
      float sv[EPL];
      svals(q[u], e0, base + BLK > V, sv);                // (uniform)
      uint32_t in;
      A += part_of(sv, in);
      unsigned long long mask = __ballot(in != 0u);
      while (mask) {
        push(mask, in != 0u, [&]() {
          const int i = EPL - __ffs((int)in);
          float z[EPL], x = 0.0f;
          raw(q[u], z);
#pragma unroll
          for (int k = 0; k < EPL; ++k) x = k == i ? z[k] : x;
          return ((unsigned long long)(uint32_t)(e0 + i) << 32) | key_of(by_tau.of(x));
        });
        in &= in - 1u;
        mask = __ballot(in != 0u);
      }
    }
    A = dpp_scan_add_u64(A);
    if (lane == kWave - 1) hd[blk] = A;
#pragma unroll
    for (int u = 0; u < UNR; ++u) q[u] = next[u];
  }
  __syncthreads();
  each_penalised([&](bool have, float sv, uint32_t v) {
    const bool above = have && sv >= s_hi, in = have && sv >= s_lo && !above;
    if (above) atomicAdd(&hd[v / BLK], mass(sv));
    const unsigned long long mask = __ballot(in);
    if (mask) push(mask, in, [&]() { return ((unsigned long long)v << 32) | key_of(sv); });
  });
  for (uint32_t i = at + (uint32_t)lane; i < min(end, room); i += kWave) region[i] = key_none;
  __syncthreads();                                        // (a workgroup's own stores are visible to it behind a barrier)
  const uint32_t n_list = fs.rq_n * kPage;
  if (n_list > room) return 0;                            // uniform
  // ---- the cut: bins over the window, then the members of one
  const float sc = (float)kBins / __fsub_rn(s_hi, s_lo);
  auto bin_at = [&](float sv) { return min(kBins - 1, max(0, (int)(__fsub_rn(sv, s_lo) * sc))); };
  // every entry, four of a lane under way at a time
  auto each_entry = [&](auto&& f) {
    for (uint32_t i0 = (uint32_t)tid; i0 < n_list; i0 += 4 * NT) {             // (wave-uniform: whole pages)
      uint2 en[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned long long w = region[min(i0 + (uint32_t)(k * NT), n_list - 1u)];
        en[k] = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + (uint32_t)(k * NT) < n_list && en[k].x != key_none) f(en[k]);
    }
  };
  each_entry([&](const uint2& en) {
    const float sv = value_of(en.x);
    const unsigned long long E = mass(sv);
    if (E) atomicAdd(&hm[bin_at(sv)], E);
  });
  unsigned long long above = 0;                           // mass above the window, later above the bin
  {
    const unsigned long long a2 = dpp_scan_add_u64((tid < nblk ? hd[tid] : 0ull) + (tid + NT < nblk ? hd[tid + NT] : 0ull));
    if (lane == kWave - 1) fs.r64[wave] = a2;
    __syncthreads();
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) above += fs.r64[ww];
    __syncthreads();
    // thread t has bins kBins-1-4t .. kBins-4-4t, descending
    const int b0 = kBins - 1 - kBinsPerThread * tid;
    unsigned long long w[kBinsPerThread], msum = 0;
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) { w[j] = hm[b0 - j]; msum += w[j]; }
    const unsigned long long minc = dpp_scan_add_u64(msum);
    if (lane == kWave - 1) fs.r64[wave] = minc;
    __syncthreads();
    unsigned long long ex = above + minc - msum;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww)
      if (ww < wave) ex += fs.r64[ww];
#pragma unroll
    for (int j = 0; j < kBinsPerThread; ++j) {
      if (ex < limit && limit <= ex + w[j]) { fs.bin_p = b0 - j; fs.before_d = ex; }         // one bin at most
      ex += w[j];
    }
  }
  __syncthreads();
  const int bp = fs.bin_p;
  if (bp >= kBins) return 0;                              // uniform: the cut lies above or below the window
  above = fs.before_d;
  __syncthreads();
  constexpr uint32_t kList = kBins;
  uint32_t* const list = reinterpret_cast<uint32_t*>(hm); // (the bins are done with)
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0;
  each_entry([&](const uint2& en) {
    const float sv = value_of(en.x);
    const int bin = bin_at(sv);
    const unsigned long long E = mass(sv);
    if (E && bin > bp) atomicAdd(&hd[en.y / BLK], E);
    if (E && bin == bp) {
      const uint32_t at = atomicAdd(&fs.n_memb2, 1u);
      if (at < kList) list[at] = en.x;
      kmin = min(kmin, en.x); kmax = max(kmax, en.x);
    }
  });
  if (kmax) { atomicMin(&fs.key_p, kmin); atomicMax(&fs.key_k, kmax); }
  __syncthreads();
  const uint32_t n = fs.n_memb2;
  // the smallest key above which the mass stays short of the limit lies in [k_lo, k_hi]
  uint32_t k_lo = fs.key_p, k_hi = fs.key_k;
  if (k_lo != k_hi && n > kList) return 0;                // uniform
  while (k_lo < k_hi) {                                   // uniform
    const uint32_t mid = k_lo + ((k_hi - k_lo) >> 1);
    unsigned long long g = 0;
    for (uint32_t i = tid; i < n; i += NT)
      if (list[i] > mid) g += mass(value_of(list[i]));
    g = dpp_scan_add_u64(g);
    __syncthreads();
    if (lane == kWave - 1) fs.r64[wave] = g;
    __syncthreads();
    unsigned long long G = above;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) G += fs.r64[ww];
    if (G < limit) k_hi = mid; else k_lo = mid + 1;
  }
  const uint32_t key_cut = k_hi;
  each_entry([&](const uint2& en) {
    const float sv = value_of(en.x);
    if (en.x >= key_cut && bin_at(sv) == bp) atomicAdd(&hd[en.y / BLK], mass(sv));
  });
  __syncthreads();
  // ---- prefix over the blocks, and the block that holds the crossing
  unsigned long long target;
  {
    static_assert(262144 / BLK <= NT, "a block per thread");
    const unsigned long long w = tid < nblk ? hd[tid] : 0ull;
    const unsigned long long minc = dpp_scan_add_u64(w);
    if (lane == kWave - 1) fs.r64[wave] = minc;
    __syncthreads();
    unsigned long long ex = minc - w, S3 = 0;
#pragma unroll
    for (int ww = 0; ww < kFinalWaves; ++ww) {
      if (ww < wave) ex += fs.r64[ww];
      S3 += fs.r64[ww];
    }
    target = (__umul64hi(j24, S3) << 40) | ((j24 * S3) >> 24);                // floor(j * S3 / 2^24)
    if (ex <= target && target < ex + w) { fs.bin_d = tid; fs.before_d = ex; }
  }
  __syncthreads();
  const int blk_d = fs.bin_d;
  if (blk_d < 0) return 13;                                                   // uniform (no mass at all)
  if (wave == 0) {                                                            // lane prefixes in vocabulary order
    const int base = blk_d * BLK;
    unsigned long long running = fs.before_d;
    bool found = false;
#pragma nounroll
    for (int u = 0; u < UNR && !found; ++u) {
      const int e0 = base + (u * kWave + lane) * EPL;
      const uint4 q = ldrow(e0);
      float sv[EPL];
      svals(q, e0, true, sv);
      const uint32_t word = has_pen ? bm[min(e0, V - 1) >> 5] : 0u;
      unsigned long long E[EPL], tot = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        if (e0 + i < V && ((word >> ((e0 + i) & 31)) & 1u))
          sv[i] = value_of(cnt[pre[(e0 + i) >> 5] + __popc(word & ((1u << ((e0 + i) & 31)) - 1u))]);
        E[i] = sv[i] > -INFINITY && key_of(sv[i]) >= key_cut ? mass(sv[i]) : 0ull;
        tot += E[i];
      }
      const unsigned long long incl = dpp_scan_add_u64(tot);
      unsigned long long c = running + incl - tot;
      int hit = -1;
      uint32_t hit_key = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        c += E[i];
        if (hit < 0 && E[i] && c > target) { hit = e0 + i; hit_key = key_of(sv[i]); }
      }
      const unsigned long long ball = __ballot(hit >= 0);
      found = ball != 0;
      if (found && lane == __ffsll((long long)ball) - 1) { fs.token = hit; fs.token_key = hit_key; }
      running += last_lane_u64(incl);
    }
  }
  __syncthreads();
  return fs.token == 0x7FFFFFFF ? 13 : 1;
}

// Continuation of fast_row for the two kinds of row that are finished over the whole row
// (codes kWholeRowCut and kWholeRow): nucleus cut if asked for, draw, token and its logprob.
// The best-n list is already written.  Returns 1, or a code that sends the row to the exact path.
template <int DT>
__device__ __attribute__((noinline)) int whole_row_finish(const Args& a, const int b, const RowParams rp,
                                                          lds_ptr<unsigned char> dyn_lds, lds_ptr<FastShared> fs_lds, const bool cut) {
  FastShared& fs = *(FastShared*)fs_lds;
  const int V = a.V;
  const char* row = reinterpret_cast<const char*>(a.logits) + (size_t)b * (size_t)a.row_stride * (DT == SIP_F32 ? 4 : 2);
  __syncthreads();
  const float m = fs.m_out, zmax = fs.zmax_out;
  const unsigned long long limit = fs.limit_out;
  const double lnZ = fs.lnz_out;
  const bool has_pen = fs.has_pen_out != 0;
  const bool minp_on = cut && rp.min_p > 0.0f;
  const float t_minp = minp_on ? (float)log((double)rp.min_p) : 0.0f;
  const unsigned long long j24 = (unsigned long long)(philox_word0(a.seed, rp.row_id, step_of(a)) >> 8);
  if (cut) {
    int r = 0;
    if (!minp_on)
      r = whole_row_window<DT>(row, V, has_pen, dyn_lds, fs_lds, a.cand + (size_t)b * (size_t)a.S * (size_t)a.cap_c,
                               (uint32_t)(a.S * a.cap_c), 1.0 / (double)rp.tau, m, limit, rp.top_p, j24);
    if (r == 0) r = whole_row_nucleus<DT>(row, V, has_pen, dyn_lds, fs_lds, 1.0 / (double)rp.tau, m, limit, j24,
                                        minp_on, t_minp);
    if (r != 1) return r == 11 ? 10 : r;                                      // uniform
  } else if (whole_row_draw<DT>(row, V, has_pen, dyn_lds, fs_lds, rp.tau, rp.greedy, m, zmax, (float)log2_scale(rp), j24) != 1) {
    return 13;                                                                // uniform
  }
  if (threadIdx.x == 0) {
    const int token = fs.token;
    a.out_ids[b] = token;
    if (a.k_lp >= 0) {
      const int cols = 1 + a.k_lp;
      a.out_lp_ids[(size_t)b * cols] = token;
      a.out_lp[(size_t)b * cols] = (float)((double)value_of(fs.token_key) - (double)m - lnZ);
    }
  }
  return 1;
}

}  // namespace sip
