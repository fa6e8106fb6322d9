// Single pass over the logits: the only kernel that touches all B*V elements.
//
// A row is cut into S chunks, one 512-thread workgroup each.  The workgroup never learns the
// row's maximum; instead it picks, from a 8192-element sample spread over the row, a value
// threshold Tc such that only the top ~1-3 % of the row lies at or above it, and then streams
// its chunk once:
//   * elements >= Tc ("candidates") are collected, value and index, in per-wave LDS queues
//     (a wave that finds more than its queue holds reports an overflow and the row falls back
//     to the exact path) and written out at the end as the chunk's one segment of the workspace
//     (a workgroup that finishes its row itself keeps them in registers, sip_row.h) --
//     every question that needs exact
//     values (top-k, top-p, min-p, draw, best-n, maximum) is answered later from these few
//     thousand entries per row;
//   * all other elements only contribute their softmax mass, 2^(z*c + off) with c = log2(e)/tau and
//     off = -Tc*c.  Because z < Tc, every term is < 1: no running maximum, no rescaling
//     (Sec. 5.1 row-wise softmax, here fused with temperature scaling).  Each thread adds its
//     terms in fp32 in a fixed order; the per-thread sums are combined as integers in units
//     of 2^-30.
// What bounds it: fp32 rows HBM (V = 152064, 256 rows 33.1 -> 29.6 us, 5.3 TB/s), bf16 rows vector issue (V =
// 129280, 1024 rows 86.4 -> 74.7 us, and a minimum per element more since), both against a loop that compared,
// selected and pushed element by element and waited for loads it had just issued.
// History penalties (Sec. 5.1 ApplyPenalty) touch at most |history| elements of a row.  The
// workgroup marks the row's history tokens that fall into its chunk in an LDS bitmap (one bit
// per element of the chunk); an element whose bit is set goes into the list whatever its
// value, tagged, and stays out of the bulk mass, so that the finishing kernel finds the raw
// logit of every token it has to penalise in the list and never reads the logits itself.
#pragma once
#include <type_traits>

#include "sip_device.h"

namespace sip {

constexpr int kStreamThreads = 512;
constexpr int kStreamWaves = kStreamThreads / kWave;
static_assert(kStreamWaves == 8, "a chunk's segment is made of eight wave queues");
constexpr int kSampleBins = 8192;           // see sample_bin()
constexpr int kSampleSize = 8192;           // elements of a row the threshold is estimated from
constexpr int kQueueCap = 480;              // entries of one wave's LDS candidate queue where four workgroups share a compute unit
constexpr int kChunkCap = kStreamWaves * kQueueCap;   // entries of such a chunk's segment in the workspace
constexpr int kChunkBitsMax = 73728;        // most elements a chunk may have (history bitmap: 9 KB of LDS)
constexpr int kAloneBitsMax = 131072;       // one that has a compute unit to itself (16 KB; only where ids alone are asked for that long)
constexpr int kRowBitsMax = 262144;         // and a row that one workgroup streams (32 KB)
// What differs between a workgroup that streams one chunk of a row for the finishing kernel (ROW =
// false: four workgroups per compute unit, 40 KB of LDS and 64 registers each) and one that streams the
// whole row and finishes it itself (sip_row.h: two, with 80 KB and 128 registers).  ALONE: a chunk whose workgroup
// has a compute unit to itself (sip_fused.h).
template <int DT, bool ROW, bool ALONE = false>
struct StreamShape {
  static constexpr int EPL = DT == SIP_F32 ? 4 : 8;                    // elements per 16-byte load
  static constexpr int kLoads = ROW || ALONE ? 4 : 2;                           // 16-byte loads per thread per tile, of which two are held
  static constexpr int kTile = kStreamThreads * kLoads * EPL;
  typedef typename std::conditional<DT == SIP_F32, uint2, uint32_t>::type entry_t;      // of a queue, see `process`
  static constexpr int kQueue = DT == SIP_F32 ? 704 : 1280;             // ROW: entries of one wave's queue (chunks: an eighth of Args::cap_c)
  static constexpr int kTags = 1 << EPL;                               // history bits of one load
  static constexpr int kBits = ROW ? kRowBitsMax : ALONE ? kAloneBitsMax : kChunkBitsMax;      // most elements a workgroup streams
  static constexpr int kBlocks = kBits / kBlkElems;
  static constexpr int kHistRegs = ROW || ALONE ? 8 : 4;                         // history tokens a thread requests with the sample
  // Load numbers of p whole pieces, each rounded up to tiles: they have kLoadBits in a bf16 queue entry.
  static constexpr int kLoadBits = ROW ? 7 : ALONE ? 6 : 5;
  static constexpr int load_numbers(int p) { return p * kLoads * ((kBits / p + kTile - 1) / kTile); }
  static constexpr int most_load_numbers(int p) {
    return p == 0 ? 0 : load_numbers(p) > most_load_numbers(p - 1) ? load_numbers(p) : most_load_numbers(p - 1);
  }
};
static_assert(StreamShape<SIP_BF16, false>::most_load_numbers(SIP_MAX_SHARDS) <= 1 << StreamShape<SIP_BF16, false>::kLoadBits, "see `process`");
static_assert(StreamShape<SIP_BF16, false, true>::most_load_numbers(SIP_MAX_SHARDS) <= 1 << StreamShape<SIP_BF16, false, true>::kLoadBits, "see `process`");
static_assert(StreamShape<SIP_BF16, true>::most_load_numbers(SIP_MAX_SHARDS) <= 1 << StreamShape<SIP_BF16, true>::kLoadBits, "see `process`");
constexpr float kBulkScale = 1073741824.0f; // 2^30

// Per-row decisions shared by the streaming and the finishing kernel.
struct RowParams {
  float tau, top_p, min_p, theta, phi, psi;
  int top_k;
  unsigned long long row_id;
  bool greedy;
};

__device__ __forceinline__ RowParams load_row_params(const Args& a, int b) {
  RowParams r;
  r.tau = a.p.temperature ? a.p.temperature[b] : 1.0f;
  r.top_k = a.p.top_k ? a.p.top_k[b] : 0;
  r.top_p = a.p.top_p ? a.p.top_p[b] : 1.0f;
  r.min_p = a.p.min_p ? a.p.min_p[b] : 0.0f;
  r.theta = a.p.repetition_penalty ? a.p.repetition_penalty[b] : 1.0f;
  r.phi = a.p.frequency_penalty ? a.p.frequency_penalty[b] : 0.0f;
  r.psi = a.p.presence_penalty ? a.p.presence_penalty[b] : 0.0f;
  r.row_id = a.p.row_id ? (unsigned long long)a.p.row_id[b] : (unsigned long long)b;
  r.greedy = (r.tau == 0.0f) || (r.top_k == 1);
  return r;
}

// The threshold of a row whose list is to hold `target` entries is the j-th largest value of a
// sample, j = target * (sample size) / V, so the list comes out at target * (1 +- 1/sqrt(j)).
// Lists of kWholeFrom entries and more are the ones that may outgrow the 4096 entries of the
// finishing kernel's faster variants (twice the time for that row), so they are estimated from
// the whole sample of kSampleSize elements as long as that keeps j small (<= kTailRank); every other
// list from every other sample block.  Of the whole sample, and of the half where j is small (<= kTailRank
// / 2), a thread only tracks its three largest values.  (Up to three times that rank it would find 99 in 100 of
// the j largest were they spread over the row; with all of them in a sixth of the ids it finds half, and the
// list takes in what lies far below: V = 65936 bf16 in two pieces, 5 rows under min-p, 124 us, 330 so.)
constexpr int kTailRank = 256;
constexpr int kWholeFrom = 2048;
__device__ __forceinline__ bool whole_sample(int target, int V) {
  // ceil(target * kSampleSize / V) <= kTailRank, without the division (target <= 2^14, V <= 2^19)
  return target >= kWholeFrom && (uint32_t)target * (uint32_t)kSampleSize <= (uint32_t)kTailRank * (uint32_t)V;
}

// No filter at all: every element of the row may be drawn (rp.greedy excluded by the caller).
__device__ __forceinline__ bool unfiltered(const RowParams& r, int V) {
  return !(r.top_k >= 2 && r.top_k < V) && !(r.top_p < 1.0f) && !(r.min_p > 0.0f);
}

// Whether anything is asked for that takes the mass of the whole row: a log-probability, or a share of it that is
// drawn from or that top-p leaves out.  (Not so the largest element, a draw from the k largest, top-p among
// these, or a draw from what min-p keeps.)
__device__ __forceinline__ bool total_is_used(const RowParams& r, const Args& a) {
  if (a.k_lp >= 0) return true;
  return !r.greedy && !(r.top_k >= 2 && r.top_k < a.V) && (r.top_p < 1.0f || !(r.min_p > 0.0f));
}

// How many of the row's largest elements the candidate list should hold; 0 = this row
// cannot be finished from a candidate list (k is too large) and takes the exact multi-pass
// path instead.
__device__ __forceinline__ int candidate_target(const RowParams& r, const Args& a) {
  if (!(r.tau >= 0.0f)) return 0;
  if (r.greedy) return 512;
  const int k = (r.top_k >= 2 && r.top_k < a.V) ? r.top_k : 0;
  const bool p_on = r.top_p < 1.0f, minp_on = r.min_p > 0.0f;
  if (k == 0 && !p_on && !minp_on) return 512;        // plain temperature sampling: the list serves the maximum
                                                      // and best-n, as with greedy rows
  int t;
  if (k > 0) {
    // top-k needs its k largest in the list.  The threshold is the j-th largest of kSampleSize
    // sampled values, j = t * kSampleSize / V, so the list comes out t * (1 +- 1/sqrt(j)): ask
    // for 3.5 such deviations more than k (whatever top-p and min-p do afterwards happens
    // inside those k)
    t = k + 256 + (int)(3.5f * sqrtf((float)k * (float)a.V * (1.0f / (float)kSampleSize)));
    if (!whole_sample(t, a.V)) t = k + 256 + (int)(3.5f * sqrtf((float)k * (float)a.V * (2.0f / (float)kSampleSize)));
  } else {
    // a nucleus with nothing else to bound it tends to be longer than one cut by min-p, so it
    // starts from a longer list -- as long as still fits the 8 entries per thread of the
    // finishing kernel's faster variants
    t = minp_on ? 1920 : 2816;
    // min-p keeps what lies within tau * ln(1/min_p) of the maximum: the list must reach that
    // far down, and how many elements that is grows quickly with the temperature
    if (minp_on && r.min_p < 1.0f) t = max(t, 1280 + (int)(400.0f * r.tau * -__logf(r.min_p)));
  }
  // the threshold comes from a sample: allow for a list a quarter longer than asked for
  if (t + (t >> 2) > a.nc_cap) return 0;
  return t;
}

// log2(e)/tau (greedy rows: tau = 1)
__device__ __forceinline__ double log2_scale(const RowParams& r) { return 1.4426950408889634074 / (r.greedy ? 1.0 : (double)r.tau); }

// One fused multiply-add answers both questions the stream asks of an element: x = z * c + off with
// c = log2(e)/tau and off = -Tc*c (rounded) is negative exactly if z < Tc -- rounding keeps a sign, and
// Tc is put, by an ulp at most, where z * c + off changes it -- and 2^x is then the element's softmax
// mass in units of 2^-off, a number that whoever reads the sums works out from Tc and off
// (bulk_exponent()).  Negligible terms apart x is small, so its one rounding leaves the term as
// accurate as the fp32 result; what c's own rounding does to Tc*c is in the unit, exactly.  z = -inf
// gives 0.
struct BulkRef {
  float Tc, c, off;
  bool none;               // no element below the threshold has any mass
  double unit;             // log2 of the terms' unit (masses being 2^(z * log2(e)/tau))
};
// `Tc`: where the threshold should lie; the result's is where it lies (every reader takes that one).
// At temperatures so small that whatever lies below the threshold has less than 2^-64 of its mass the
// multiply-add only tells which side an element is on.
// `c`: log2_scale() of the row.
__device__ __forceinline__ BulkRef make_bulk_ref(float Tc, const double c) {
  BulkRef r;
  r.c = (float)c; r.Tc = Tc;
  double tc = (double)Tc * (double)r.c;
  r.none = !(fabs(tc) < 1073741824.0) || !(r.c < INFINITY);
  r.unit = 0.0;
  if (r.none) { r.c = 1.0f; r.off = 0.0f - Tc; return r; }
  if (fabs(tc) < 0x1p-100) { r.Tc = 0.0f; tc = 0.0; }                          // (so that off has its 24 bits)
  r.off = 0.0f - (float)tc;
  // the smallest z with z * c + off >= 0: off is within half an ulp of -Tc*c, z within one of Tc
  // (products of two fp32 numbers are exact in double)
  const uint32_t k = key_of(r.Tc);
  const double at = -(double)r.off;
  const float lower = value_of(k - 1u), upper = value_of(k + 1u);
  if ((double)lower * (double)r.c >= at) r.Tc = lower;
  else if (!((double)r.Tc * (double)r.c >= at)) r.Tc = upper;
  r.unit = at + (double)r.Tc * (c - (double)r.c);
  return r;
}
// `off` as the chunk summaries carry it
__device__ __forceinline__ float published_off(const BulkRef& r) { return r.none ? INFINITY : r.off; }
// The same from a chunk summary (but for the unit).
__device__ __forceinline__ BulkRef published_ref(float Tc, float off, const RowParams& rp) {
  BulkRef r;
  r.Tc = Tc; r.c = (float)log2_scale(rp); r.off = off; r.none = !(off < INFINITY); r.unit = 0.0;
  return r;
}
// log2 of (unit of the bulk terms / mass of the maximum m).  m >= Tc / tau as rounded, so what comes
// out above 0 is the rounding of m, and no term is left of that size.
__device__ __forceinline__ double bulk_exponent(double unit, float m) { return unit - (double)m * 1.4426950408889634074; }
__device__ __forceinline__ float bulk_arg(float z, const BulkRef& r) { return __fmaf_rn(z, r.c, r.off); }
// What an element adds to the running sum: its mass if x < 0, nothing if it belongs to the list, that is
// for x >= 0 and for a NaN.  Read as integers the bits of a negative number lie below those of -inf, and
// those of everything else at or above them: one minimum instead of a comparison and a selection.
__device__ __forceinline__ float bulk_term(float x) {
  return __builtin_amdgcn_exp2f(__int_as_float(min(__float_as_int(x), (int)0xFF800000u)));
}
// Bulk terms of one 16-byte load, added in the order of its elements, as an integer in units of
// 2^-41 of a term of 1, that is at most 2^-40 of the maximum's mass: added to 2^11 a double's last bit
// is 2^-41, so the low bits of the sum are the integer (a load's terms add up to at most 8).
constexpr unsigned long long kBlkMagic = 0x40A0000000000000ull;       // 2^11
constexpr int kBlkUnitShift = 41;
__device__ __forceinline__ unsigned long long blk_bits(float g) {      // + kBlkMagic
  return (unsigned long long)__double_as_longlong((double)g + 2048.0);
}
__device__ __forceinline__ unsigned long long blk_units(float g) { return blk_bits(g) - kBlkMagic; }
// per-thread fp32 partial sum -> integer units of 2^-30
__device__ __forceinline__ unsigned long long bulk_units(float acc) {
  return acc > 0.0f ? (unsigned long long)(acc * kBulkScale) : 0ull;
}

// The sample's histogram has a bin per sign, exponent and 9 mantissa bits for 1 <= |z| < 128, in ascending order
// of z; below 1 the bins are 2^-9 wide, and what lies beyond 128 joins the outermost bin of its sign.  (With 8 mantissa
// bits a row of thousands of elements on each of two neighbouring values had both in its list.)  A row whose
// threshold lies in an outermost bin -- nearly always one that is masked with -inf -- or among more values around 0
// than these bins tell apart has its sample read again: 2 us of a call for the masked, 3 to 4 for logits beyond
// 128 or all below 0.01.
// (One level.  13-bit keys first and then the found bin split by 5 bits more, by wave 0 from all threads' largest
// keys, took 2000 to 3000 cycles longer, 1 us of every call: one row of V = 128256 bf16 20.5 -> 19.6 us.)
// (The range: with bins of z's own exponent from 1/4 to 64, V = 128256, one row, logits around 100 cost 25.7 us a
// call bf16, 25.1 fp32, of 1/30 the size 21.7 and 22.1, masked rows 28.4 and 28.9; now 20.0, 19.4, 18.8, 19.5, 20.8 and
// 21.6.  Bins put around what the row's middle holds cost every call the wait for that, 0.3 us.)
constexpr float kLow = 0.5f;
constexpr int kGroup = 32;                             // bins of a sixteenth of their values
__device__ __forceinline__ uint32_t sample_bin(float z) {
  // (positive floats, the former the larger one from 1 on, compared as integers)
  const uint32_t y = max(__float_as_uint(fabsf(z)), __float_as_uint(__fmaf_rn(fabsf(z), 0.5f, kLow)));
  const uint32_t t = min((y >> 14) - (__float_as_uint(kLow) >> 14), 4095u);
  return (t | 4096u) ^ ((uint32_t)(__float_as_int(z) >> 31) & 8191u);
}
__device__ __forceinline__ bool outermost_bin(uint32_t i) { return ((i + 1u) & 8191u) <= 1u; }
__device__ __forceinline__ bool bin_around_0(uint32_t i) { return i - 4064u < 64u; }      // |z| < 1/16
// Smallest value of bin i (of one that is not an outermost one).  Bin 4096 begins at 0.
__device__ __forceinline__ float sample_floor(uint32_t i) {
  const uint32_t b = __float_as_uint(kLow) >> 14;
  const float y = __uint_as_float(i >= 4096u ? (i - 4096u + b) << 14 : ((4096u - i + b) << 14) - 1u);
  const float z = fminf(y, 2.0f * (y - kLow));
  return i >= 4096u ? z : -z;
}

// A row that top-p or min-p bounds asks for a list that reaches far down (candidate_target()), which a
// peaked row does not need.  Its sample says how far down is enough: this looks, from the
// threshold asked for upwards, for the highest group of bins such that in the sample
//   - at least `least` values lie in it or above (the maximum and the best-n come from the list), and
//   - min-p keeps nothing below, or the mass below is at most a half (with a penalty on, a quarter) of the
//     share that top-p leaves out,
// values below counting as their group's upper end and those above as its lower end.  A few of the row's
// largest may be history tokens that a penalty takes away, or be in the sample by chance: the fourth (with
// a penalty on, eighth) largest sample value stands for the maximum, and those above it count as much as
// it does.  (What a thread's sample holds beyond its three largest counts as at the lowest group, so the mass
// below is rather too small: a matter of speed, as a row whose list ends too high is settled over the whole row.  Of
// 72576 rows -- normal, Student-t, spiked and peaked, top-p 0.5, 0.9 and 0.99, V = 50000 to 200000, 16 to 512 of
// them, both types -- 31561 left their lists; with lists of one length 31590, no fewer at any of the 30 shapes.)
// Returns that group (its lower end is the threshold), or G.
// What it gives, us a call: Student-t logits, lists of 540 instead of 2830 entries, V = 129280 bf16, 1024 rows
// 110.0 -> 93.3; V = 152064 bf16 in pieces, 200 rows 38.8 -> 34.2; V = 128256 bf16, 32 rows of 8600 tokens under
// min-p 32.6 -> 27.3.  A row that keeps the long list pays 0.3 for the question.
// For one wave.  G: group of bins the threshold lies in; above: sample values above
// that group; c: log2_scale() of the row.
__device__ __forceinline__ uint32_t raised_group(const uint32_t G, const uint32_t above, const uint32_t* hist, const RowParams& rp,
                                                 const float c, const bool has_pen, const uint32_t least,
                                                 const uint32_t n_smp) {
  constexpr int kUp = 44;                              // lane l has group G + kUp - l
  const int lane = lane_id(), g = (int)G + kUp - lane;
  const bool in = g >= 0 && g < kSampleBins / kGroup;
  const uint4* const h4 = reinterpret_cast<const uint4*>(hist) + kGroup / 8 * min(max(g, 0), kSampleBins / kGroup - 1);
  uint32_t both = 0;                                   // (both counters of a word at once: 8192 values at most)
#pragma unroll
  for (int i = 0; i < kGroup / 8; ++i) { const uint4 q = h4[i]; both += q.x + q.y + q.z + q.w; }
  const uint32_t n = in ? (both & 0xFFFFu) + (both >> 16) : 0u;
  auto floor_of = [](int gr) { return sample_floor((uint32_t)(kGroup * max(gr, 0))); };
  const float z0 = floor_of((int)G);
  const float x_lo = fminf((floor_of(g) - z0) * c, 100.0f), x_hi = (floor_of(g + 1) - z0) * c;
  const uint32_t scan = dpp_scan_add_u32(n);
  const uint32_t beyond = above - min(above, (uint32_t)__builtin_amdgcn_readlane((int)scan, kUp - 1));     // above the lanes' groups
  const uint32_t n_from = beyond + scan;               // in this group or above
  const unsigned long long flat = __ballot(in && n_from >= (has_pen ? 8u : 4u));
  const int at = flat ? __ffsll((long long)flat) - 1 : kWave - 1;
  const float x_top = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x_lo), at));
  const float head = (float)beyond * __builtin_amdgcn_exp2f(x_top) +
                     dpp_scan_add_f32(n ? (float)n * __builtin_amdgcn_exp2f(fminf(x_lo, x_top)) : 0.0f);
  const float up = dpp_scan_add_f32(lane >= at && n ? (float)n * __builtin_amdgcn_exp2f(x_hi) : 0.0f);
  const float rest = (float)(n_smp - min(n_smp, last_lane_u32(n_from))) *
                     __builtin_amdgcn_exp2f(__uint_as_float(last_lane_u32(__float_as_uint(x_lo))));
  const float tail = rest + (__uint_as_float(last_lane_u32(__float_as_uint(up))) - up);
  const bool by_p = rp.top_p < 1.0f && tail <= (has_pen ? 0.25f : 0.5f) * (1.0f - rp.top_p) * (tail + head);
  const bool by_minp = rp.min_p > 0.0f && x_lo <= x_top + __log2f(rp.min_p);
  const unsigned long long ok = __ballot(in && lane >= at && lane < kUp && n_from >= least && (by_p || by_minp));
  return ok ? G + (uint32_t)(kUp + 1 - __ffsll((long long)ok)) : G;
}

// LDS: first the sample histogram (two 16-bit counters per word, 16 KB), then, in its
// place, the per-wave candidate queues (a chunk's: fp32 30 KB, bf16 15 KB, up to four times
// that where fewer than four share a compute unit; a row's: 44 or 40 KB); then the history
// bitmap (9, 16 or 32 KB) and the tag words (fp32 256 bytes, bf16 4 KB).
template <int DT, bool ROW, bool ALONE = false>
struct __align__(16) StreamTables {
  typedef StreamShape<DT, ROW, ALONE> Sh;
  uint32_t bmw[Sh::kBits / 32];            // (first: a queue that overflows may write up to 4 KB past the last wave's end)
  uint4 tag_words[Sh::kTags];              // history bits of a load -> what is or-ed into its four words
  unsigned long long blk_mass[Sh::kBlocks];
  union {
    uint32_t sub_hist[32];                 // a bin of 13-bit keys, split by the next 5 key bits (dead once the threshold is found)
    struct {
      unsigned long long red64[kStreamWaves];
      uint32_t red32[kStreamWaves];
    };
  };
  BulkRef ref;
  uint32_t seg_cnt;                        // entries of the segment so far
  uint32_t key_thr;                        // how the threshold came about, see there
};
// Bytes ahead of them: the histogram, later queues of `cap` entries.
template <int DT, bool ROW>
__host__ __device__ constexpr int stream_front_bytes(int cap) {
  const int q = kStreamWaves * cap * (int)sizeof(typename StreamShape<DT, ROW>::entry_t);
  return q > kSampleBins * 2 ? q : kSampleBins * 2;
}
template <int DT>
constexpr int stream_lds_bytes(int cap) { return stream_front_bytes<DT, false>(cap) + (int)sizeof(StreamTables<DT, false>); }
static_assert(stream_lds_bytes<SIP_F32>(kQueueCap) <= 40 * 1024 && stream_lds_bytes<SIP_BF16>(kQueueCap) <= 40 * 1024,
              "four workgroups per compute unit");
static_assert(stream_lds_bytes<SIP_F32>(2 * kQueueCap) <= 80 * 1024, "two with queues of twice the length");
template <int DT>
struct __align__(16) RowStreamShared {
  unsigned char front[stream_front_bytes<DT, true>(StreamShape<DT, true>::kQueue)];
  StreamTables<DT, true> tables;
};

// What a workgroup that finishes its row itself takes from here to there (ROW; all of it uniform).
constexpr int kRowRegs = 10;               // list entries a thread holds in registers
struct RowHand {
  RowInfo ri;
  ChunkOut co;
  uint32_t longest;                        // entries of the longest queue
  bool greedy = false;                     // the arg max is all that is asked for, and `best` is it (the chunk's)
  unsigned long long best;                 // key of the value, complement of the vocabulary id: the larger the better
  bool direct;                             // the queues went to registers, lane l's entry r being entry 64 * r + l of its wave's
  uint2 list[kRowRegs];                    // (per thread)
};

// Streams chunk wg % S of row wg / S (ROW: row wg).  False: the row cannot be finished from a list.  `front` and
// `sm`: LDS, one behind the other.  IDS: a call that asks for token ids only (a kernel of its own, see `masses`).
// ALONE: `hand` gets the row's record, whose place has the row's word (opened here by the last wave's first thread).
template <int DT, bool SH, bool ROW, bool IDS = false, bool ALONE = false>
__device__ __forceinline__ bool stream_part(const Args& a, const int wg, unsigned char* const front, StreamTables<DT, ROW, ALONE>& sm,
                                            RowHand* hand, RowWord* word = nullptr) {
  typedef StreamShape<DT, ROW, ALONE> Sh;
  typedef typename Sh::entry_t entry_t;
  constexpr int EPL = Sh::EPL;
  constexpr int ESZ = (DT == SIP_F32) ? 4 : 2;
  constexpr int NL = Sh::kLoads;
  constexpr int SUB = kStreamThreads * EPL;         // elements per workgroup-wide load
  constexpr int TILE = Sh::kTile;
  constexpr int SLOADS = kSampleSize / SUB;         // sample loads per thread (4 fp32, 2 bf16)
  constexpr int NSB = SLOADS * kStreamWaves;        // 1 KB sample blocks spread over the row
  uint32_t* const bmw = sm.bmw;
  uint32_t* const hist = reinterpret_cast<uint32_t*>(front);
  const int queue_cap = ROW ? Sh::kQueue : a.cap_c / kStreamWaves;

  // Where several bf16 chunks share a compute unit, the set-up's chain and the queues' way out go ahead of other chunks'
  // streaming: us a call, without / so, V = 152064, 150 rows 27.9 / 27.2, 300 rows 44.6 / 43.6.  Not for fp32, whose streaming
  // the memory bounds and which must not stop asking (520 rows of V = 128256 90.0 / 94.9), nor for a row to a workgroup (1024 bf16
  // rows of V = 129280 88.2 / 89.9, streaming first 88.7; 2048 fp32 rows of V = 256000 502 / 506, 509).
  constexpr bool CHAIN_FIRST = DT == SIP_BF16 && !ROW && !ALONE;
  if (CHAIN_FIRST) __builtin_amdgcn_s_setprio(2);
  // (the wave's number, and further down r0, in a scalar register: as vector registers they were
  // spilled, and a store to scratch ahead of the loads makes every wait for one of them a wait for
  // all -- 3 us of the 33 at fp32 V = 152064, 256 rows)
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
  const int S = ROW ? 1 : a.S;
  const int b = ROW ? wg : wg / S, ch = ROW ? 0 : wg - b * S;
  const int V = a.V;
  // SH (vocabulary-sharded logits): the row's chunks are dealt out to the shards, S / t_shards
  // each, and a chunk lies inside its shard; c0, c1 and every element index below are then
  // relative to the shard, `ibase` being the shard's first vocabulary id.
  // With more chunks than shards a chunk is a part of one shard (np = 1 piece); with fewer, it is
  // np whole shards in a row, streamed one after the other.
  const bool split = !SH || S >= a.t_shards;         // uniform
  const int S_sh = !SH ? S : (split ? S / a.t_shards : 1);
  const int np = (SH && !split) ? a.t_shards / S : 1;
  const int sh = !SH ? 0 : (split ? ch / S_sh : ch * np);
  const int lc = !SH ? ch : (split ? ch - sh * S_sh : 0);
  const int Vl = SH ? a.V_shard : V;
  const uint32_t ibase = SH ? (uint32_t)(sh * Vl) : 0u;
  const int c0 = chunk_begin(lc, Vl, S_sh, kChunkUnit);
  const int c1 = chunk_begin(lc + 1, Vl, S_sh, kChunkUnit);
  if (c0 >= c1) return false;                        // host guarantees every chunk is non-empty
  const char* row = SH ? shard_base(a, sh) + (size_t)b * (size_t)a.shard_stride * ESZ      // (moves on with the pieces)
                       : reinterpret_cast<const char*>(a.logits) + (size_t)b * (size_t)a.row_stride * ESZ;

  // Loads are unconditional (a select on the loaded value would make the wave wait for it at
  // once): lanes past the end of the chunk re-read its last 16 bytes and `process` discards
  // what they hold by index.
  const int e_last = ((c1 - 1) / EPL) * EPL;
  auto load_tile = [&](int t0, uint4 (&buf)[NL]) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const uint32_t e0 = (uint32_t)min(t0 + j * SUB + tid * EPL, e_last);     // (a scalar base and 32 bits beside it)
      buf[j] = *reinterpret_cast<const uint4*>(row + e0 * (uint32_t)ESZ);
    }
  };
  auto unpack = [&](const uint4& q, float (&z)[EPL]) {
    if (DT == SIP_F32) {
      z[0] = __uint_as_float(q.x); z[1] = __uint_as_float(q.y);
      z[2] = __uint_as_float(q.z); z[3] = __uint_as_float(q.w);
    } else {
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[2 * i] = __uint_as_float(w[i] << 16);
        z[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
      }
    }
  };

  // ---- The row's small records -- parameters, history and prompt extents -- are read first, all
  // at once and without a branch in between (where branches meet, the compiler waits for every
  // load in flight).  Their addresses are the same for the whole workgroup and nothing has been
  // stored by this kernel so far, so the compiler reads them through the scalar cache into scalar
  // registers: one round trip, and no vector registers held while they travel.  What a call does
  // not have (a NULL parameter array, no history) is read from memory that is there anyway and
  // replaced by its default afterwards.
  const char* const dummy = reinterpret_cast<const char*>(a.chunks);
  auto rec = [&](const void* arr, size_t off) { return arr ? reinterpret_cast<const char*>(arr) + off : dummy; };
  const bool csr_on = !a.slot && a.indptr && a.tokens && a.nnz > 0;
  const bool prompt_csr = a.p_indptr && a.p_tokens && a.p_nnz > 0;
  const float r_tau = *reinterpret_cast<const float*>(rec(a.p.temperature, 4 * (size_t)b));
  const int r_k = *reinterpret_cast<const int*>(rec(a.p.top_k, 4 * (size_t)b));
  const float r_p = *reinterpret_cast<const float*>(rec(a.p.top_p, 4 * (size_t)b));
  const float r_minp = *reinterpret_cast<const float*>(rec(a.p.min_p, 4 * (size_t)b));
  const float r_theta = *reinterpret_cast<const float*>(rec(a.p.repetition_penalty, 4 * (size_t)b));
  const float r_phi = *reinterpret_cast<const float*>(rec(a.p.frequency_penalty, 4 * (size_t)b));
  const float r_psi = *reinterpret_cast<const float*>(rec(a.p.presence_penalty, 4 * (size_t)b));
  const long long r_id = *reinterpret_cast<const long long*>(rec(a.p.row_id, 8 * (size_t)b));
  const long long r_h0 = *reinterpret_cast<const long long*>(rec(csr_on ? a.indptr : nullptr, 8 * (size_t)b));
  const long long r_h1 = *reinterpret_cast<const long long*>(rec(csr_on ? a.indptr : nullptr, 8 * (size_t)b + 8));
  const long long r_p0 = *reinterpret_cast<const long long*>(rec(prompt_csr ? a.p_indptr : nullptr, 8 * (size_t)b));
  const long long r_p1 = *reinterpret_cast<const long long*>(rec(prompt_csr ? a.p_indptr : nullptr, 8 * (size_t)b + 8));
  const int r_slot = *reinterpret_cast<const int*>(rec(a.slot, 4 * (size_t)b));
  // (all of them are named here, once: otherwise the compiler moves each read to the branch that
  // first looks at its value, and the round trips follow one another)
  asm volatile("" ::"s"(r_tau), "s"(r_k), "s"(r_p), "s"(r_minp), "s"(r_theta), "s"(r_phi), "s"(r_psi), "s"(r_id),
               "s"(r_h0), "s"(r_h1), "s"(r_p0), "s"(r_p1), "s"(r_slot));
  // ---- the records: defaults for what the call does not have
  RowParams rp;
  rp.tau = a.p.temperature ? r_tau : 1.0f;
  rp.top_k = a.p.top_k ? r_k : 0;
  rp.top_p = a.p.top_p ? r_p : 1.0f;
  rp.min_p = a.p.min_p ? r_minp : 0.0f;
  rp.theta = a.p.repetition_penalty ? r_theta : 1.0f;
  rp.phi = a.p.frequency_penalty ? r_phi : 0.0f;
  rp.psi = a.p.presence_penalty ? r_psi : 0.0f;
  rp.row_id = a.p.row_id ? (unsigned long long)r_id : (unsigned long long)b;
  rp.greedy = (rp.tau == 0.0f) || (rp.top_k == 1);
  const int target = candidate_target(rp, a);
  // ---- What one thread of the grid does for the whole call.  Device-resident history: the call
  // takes its number from the state's call counter (one atomic add, so that calls in flight at once
  // on one state each get their own) and leaves it in the workspace, where the kernels behind this
  // one read it (step_of()).  (A workgroup that goes on to finish its row finds it there.)
  // (Here, on the one path that every workgroup takes, and not before the records above have been
  // read: with no store ahead of them in the kernel the compiler reads them through the scalar
  // cache.)
  if (!ROW && a.call_tick && blockIdx.x == 0 && tid == 0) *a.call_tick = atomicAdd(a.st_tick, 1ull);
  if (ALONE && tid == kStreamThreads - kWave) word->look();
  if (target == 0) {
    if (ALONE) {
      hand->ri.target = 0;
      if (tid == kStreamThreads - kWave) word->open(a.call_mark);
    }
    if (!ROW && !ALONE && ch == 0 && tid == 0) a.rowinfo[b].target = 0;                // the finishing kernel looks at nothing else
    return false;
  }
  // ---- A greedy row without penalties of which only the id is asked for: no threshold, no list.  Every thread keeps
  // the largest of its values, the load that has the first of them and that load's place.  What bounds it: the memory.
  // us a call, by way of a list / so: one row of V = 128256 bf16 11.9 / 7.9, 64 rows fp32 15.5 / 9.7, 128 rows of V = 152064 bf16
  // 17.7 / 11.0, 256 rows 22.9 / 14.4, 1024 rows of V = 129280 62.5 / 49.4; in chunks that a second kernel compares 128 rows of V = 152064
  // 18.1 / 12.6, 150 rows 19.1 / 13.6, 300 rows of V = 60000 fp32 30.8 / 21.2, on a state 64 rows of V = 60000 bf16 37.5 / 30.9.
  if constexpr (IDS) {
    const bool arg_max = rp.greedy &&
                         ((rp.theta == 1.0f && rp.phi == 0.0f && rp.psi == 0.0f) || !(a.slot || csr_on || prompt_csr));
    if (ROW || ALONE) hand->greedy = arg_max;
    if (arg_max) {                                   // uniform
      if (CHAIN_FIRST) __builtin_amdgcn_s_setprio(0);
      if (ALONE && tid == kStreamThreads - kWave) word->open(a.call_mark);
      float top = -INFINITY;
      uint4 top_q = make_uint4(0, 0, 0, 0);
      uint32_t top_v = 0;                            // vocabulary id of the load's first element
      auto look = [&](const uint4& q, uint32_t v, int left) {                  // `left`: elements inside the piece
        float z[EPL];
        unpack(q, z);
        if (left < EPL) {
#pragma unroll
          for (int i = 0; i < EPL; ++i) z[i] = i < left ? z[i] : -INFINITY;
        }
        float x = z[0];
#pragma unroll
        for (int i = 1; i < EPL; ++i) x = z[i] > x ? z[i] : x;
        if (x > top) { top = x; top_q = q; top_v = v; }
      };
      for (int pc = 0; pc < np; ++pc) {
        if (SH) row = shard_base(a, sh + pc) + (size_t)b * (size_t)a.shard_stride * ESZ;
        const uint32_t v0 = ibase + (uint32_t)(SH ? pc * Vl : 0);
        uint4 now[2][NL];
        load_tile(c0, now[0]);
        load_tile(c0 + TILE, now[1]);
        auto turn = [&](const uint4 (&q)[NL], int t0) {
          if (t0 + TILE <= c1) {                     // uniform
#pragma unroll
            for (int j = 0; j < NL; ++j) look(q[j], v0 + (uint32_t)(t0 + j * SUB + tid * EPL), EPL);
          } else {
#pragma unroll
            for (int j = 0; j < NL; ++j) {
              const int e0 = t0 + j * SUB + tid * EPL;
              if (e0 < c1) look(q[j], v0 + (uint32_t)e0, c1 - e0);
            }
          }
        };
        for (int t0 = c0;;) {
          turn(now[0], t0);
          load_tile(t0 + 2 * TILE, now[0]);
          if ((t0 += TILE) >= c1) break;
          turn(now[1], t0);
          load_tile(t0 + 2 * TILE, now[1]);
          if ((t0 += TILE) >= c1) break;
        }
      }
      uint32_t at = 0;
      {
        float z[EPL];
        unpack(top_q, z);
#pragma unroll
        for (int i = EPL - 1; i >= 0; --i) at = z[i] == top ? (uint32_t)i : at;
      }
      // (nothing above -inf: 0)
      unsigned long long mine = top > -INFINITY ? (unsigned long long)key_of(top) << 32 | (uint32_t)~(top_v + at) : 0ull;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long other = __shfl_xor(mine, o, kWave);
        mine = other > mine ? other : mine;
      }
      if (lane == 0) sm.red64[wave] = mine;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kStreamWaves; ++w) mine = sm.red64[w] > mine ? sm.red64[w] : mine;
      if (ROW || ALONE) hand->best = mine;
      if (!ROW && tid == 0) put<ALONE>(&a.chunks[wg].bulk, mine);
      if (!ROW && !ALONE && ch == 0 && tid == 0) a.rowinfo[b].target = kArgMaxOnly;
      return true;
    }
  }
  // ---- threshold: the same 8192-element sample (1 KB blocks spread evenly over the row) is
  // read by every chunk of the row, so all chunks agree on Tc = the lower end of the bin of the j-th
  // largest sample value, j / 8192 = target / V
  // (for long lists: half of the blocks, j / 4096 = target / V; see whole_sample())
  // All blocks are requested, whether or not the row's rank calls for the whole sample: a branch
  // around a load makes the compiler wait for that load where the branches meet, one exposed
  // memory latency per block.
  auto load_sample = [&](int j) -> uint4 {
    const int sb = wave * SLOADS + j;                  // even j: every other block of the row
    if (!SH) {
      const uint32_t base = (uint32_t)sb * (uint32_t)V / (uint32_t)NSB / (uint32_t)(kWave * EPL) * (uint32_t)(kWave * EPL);
      return reinterpret_cast<const uint4*>(row + (size_t)base * ESZ)[lane];     // base + 64 * EPL <= V since V >= 16384
    }
    // the same NSB blocks for every chunk of the row, smp_bps to a shard (the last shard may get
    // fewer), evenly spread inside it; V_shard >= 8192, so a block fits
    // (wave-uniform, and said so: with a per-lane index the table of piece pointers would be read
    // through a vector load from the kernel-argument segment, and a wait for that one)
    const int ssh = __builtin_amdgcn_readfirstlane((sb * a.smp_inv) >> 16);   // sb / smp_bps
    const int e0 = (sb - ssh * a.smp_bps) * a.smp_step + lane * EPL;
    const char* srow = shard_base(a, ssh) + (size_t)b * (size_t)a.shard_stride * ESZ;
    return *reinterpret_cast<const uint4*>(srow + (size_t)e0 * ESZ);
  };
  uint4 smp[SLOADS];
#pragma unroll
  for (int j = 0; j < SLOADS; ++j) smp[j] = load_sample(j);
  // ---- history bitmap of the chunk: bit (v - g0) for every history token v in [g0, g1), the
  // vocabulary ids this workgroup streams.  Requested here, entered while wave 0 looks for the
  // threshold, by the seven others.  (A device-resident state's extent takes a read of its own.)
  HistRange hr{0, 0, 0};
  int slot = -1, ndist = -1;
  if (a.slot) {                                      // uniform
    hr.side = (long long)b * a.L_max;
    if (r_slot >= 0 && r_slot < a.slots) {
      const int n = a.st_len[r_slot];
      slot = r_slot; ndist = a.st_ndist[r_slot];
      hr.lo = (long long)r_slot * a.L_max;
      hr.hi = hr.lo + (n < 0 ? 0 : (n > a.L_max ? a.L_max : n));
    }
  } else {
    hr = hist_range_csr(a, r_h0, r_h1);
  }
  const PenaltyPlan pen = penalty_plan_of(a, hr, r_p0, r_p1, rp.theta, rp.phi, rp.psi);
  const bool has_pen = pen.any;                                                                       // uniform
  const int g0 = (int)ibase + c0;
  const int g1 = (!SH || split) ? (int)ibase + c1 : (int)ibase + np * Vl;
  constexpr int MT = kStreamThreads - kWave;         // threads that enter tokens
  // (Without a branch, like the sample: what is not there is read from memory that is.)
  const long long n_hist = has_pen ? hr.hi - hr.lo : 0;
  const int* const first_tok = n_hist > 0 ? a.tokens + hr.lo : reinterpret_cast<const int*>(dummy);
  const uint32_t last_tok = (uint32_t)min(max(n_hist, 1ll), 1ll << 20) - 1u;
  int htok[Sh::kHistRegs];
#pragma unroll
  for (int j = 0; j < Sh::kHistRegs; ++j) htok[j] = first_tok[min((uint32_t)(tid - kWave + j * MT), last_tok)];
  // ---- the first tiles of the chunk, which travel while the threshold is worked out.  (Behind sample
  // and tokens: loads come back in the order of their requests.)
  uint4 buf[2][NL];
  int tnext = c0;                                    // first element of the next tile to request
  int n_pj = 0;                                      // SH: the piece it is in
  auto roll = [&]() {                                // SH: on to the next piece (a piece can be a single tile)
    if (tnext >= c1 && n_pj < np) {                  // (behind the last piece: on with its last 16 bytes)
      if (++n_pj < np) tnext = c0;
      if (n_pj < np) row = shard_base(a, sh + n_pj) + (size_t)b * (size_t)a.shard_stride * ESZ;
    }
  };
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    load_tile(tnext, buf[k]);                        // (past the chunk's end: its last 16 bytes again, never looked at)
    tnext += TILE;
    if (SH) roll();
  }

  if (ROW || ALONE || (ch == 0 && tid == 0)) {      // the row's record for the finishing kernel
    RowInfo ri;
    ri.tau = rp.tau; ri.top_p = rp.top_p; ri.min_p = rp.min_p; ri.theta = rp.theta; ri.phi = rp.phi; ri.psi = rp.psi;
    ri.top_k = rp.top_k; ri.target = target | (pen.prompt_on ? kPromptFlag : 0);
    ri.row_id = rp.row_id; ri.lo = hr.lo; ri.hi = hr.hi;
    ri.slot = slot; ri.ndist = ndist;
    if (ROW || ALONE) hand->ri = ri; else a.rowinfo[b] = ri;
  }
  {
    uint4* z4 = reinterpret_cast<uint4*>(hist);
    for (int i = tid; i < kSampleBins * 2 / 16; i += kStreamThreads) z4[i] = make_uint4(0, 0, 0, 0);
    z4 = reinterpret_cast<uint4*>(bmw);
    const int n_bits = ROW ? min((V + 127) / 128, Sh::kBits / 128) : Sh::kBits / 128;
    for (int i = tid; i < n_bits; i += kStreamThreads) z4[i] = make_uint4(0, 0, 0, 0);
  }
  if (tid < Sh::kTags) {                   // (bit p is element EPL - 1 - p, see `process`)
    auto word = [&](int i) -> uint32_t {
      if constexpr (DT == SIP_F32) return (tid >> (3 - i)) & 1 ? ~0u : 0u;
      else return ((tid >> (7 - 2 * i)) & 1 ? 0xFFFFu : 0u) | ((tid >> (6 - 2 * i)) & 1 ? 0xFFFF0000u : 0u);
    };
    sm.tag_words[tid] = make_uint4(word(0), word(1), word(2), word(3));
  }
  const double scale = log2_scale(rp);     // (worked out while the sample travels)
  if (tid < Sh::kBlocks) sm.blk_mass[tid] = 0ull;
  if (tid == 0) sm.seg_cnt = 0;
  __syncthreads();
  // Only the upper tail of the sample matters.  When j is small, a thread enters just the
  // three largest of its values: far fewer LDS atomics, and hardly any on the same word.
  // (Should one thread hold more than three of the j largest, the threshold comes out a
  // little low, which only lengthens the candidate list.)
  const bool bounded = !rp.greedy && !(rp.top_k >= 2 && rp.top_k < V) && (rp.top_p < 1.0f || rp.min_p > 0.0f);   // by top-p or min-p alone
  const bool whole = whole_sample(target, V);        // workgroup-uniform, like everything about the threshold
  const int n_smp = whole ? kSampleSize : kSampleSize / 2;
  uint32_t want = ((uint32_t)target * (uint32_t)n_smp + (uint32_t)V - 1u) / (uint32_t)V;     // < 2^32: target <= 2^14
  if (want < 2u) want = 2u;
  if (want > (uint32_t)n_smp) want = (uint32_t)n_smp;
  const uint32_t j = want;
  const bool tail_only = whole || j <= (uint32_t)(kTailRank / 2);
  auto count_in = [&](uint32_t bin) { atomicAdd(&hist[bin >> 1], (bin & 1u) ? 0x10000u : 1u); };
  // the three largest as floats, one maximum and two medians per value
  float f0 = -INFINITY, f1 = -INFINITY, f2 = -INFINITY;
  auto best = [&](const uint4& q) {
    float z[EPL];
    unpack(q, z);
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const float x = z[i];
      f2 = __builtin_amdgcn_fmed3f(f1, f2, x);
      f1 = __builtin_amdgcn_fmed3f(f0, f1, x);
      f0 = fmaxf(f0, x);
    }
  };
  if (tail_only) {
#pragma unroll
    for (int l = 0; l < SLOADS; ++l) {
      if (!whole && (l & 1)) continue;
      best(smp[l]);
    }
    count_in(sample_bin(f0)); count_in(sample_bin(f1)); count_in(sample_bin(f2));
  } else {
#pragma unroll
    for (int l = 0; l < SLOADS; l += 2) {
      float z[EPL];
      unpack(smp[l], z);
#pragma unroll
      for (int i = 0; i < EPL; ++i) count_in(sample_bin(z[i]));
    }
  }
  __syncthreads();
  // ---- wave 0 alone finds the bin of the j-th largest (between barriers of all eight the same took
  // twice as long), `need` being what is still wanted from inside it and `above` the values above its
  // group of bins.
  auto find_bin = [&](uint32_t& need, uint32_t& above) -> uint32_t {
    constexpr int WPL = kSampleBins / 2 / kWave;     // words per lane (64), lane 0 owning the highest bins
    const uint4* mine = reinterpret_cast<const uint4*>(hist + kSampleBins / 2 - (lane + 1) * WPL);
    uint32_t s = 0;                                  // (both counters of a word at once: 8192 values at most)
#pragma unroll 4
    for (int i = 0; i < WPL / 4; ++i) { const uint4 w = mine[(i + lane) % (WPL / 4)]; s += w.x + w.y + w.z + w.w; }
    const uint32_t local = (s & 0xFFFFu) + (s >> 16), incl = dpp_scan_add_u32(local);
    const unsigned long long at = __ballot(incl >= j);
    const int src = at ? __ffsll((long long)at) - 1 : kWave - 1;
    uint32_t run = (uint32_t)__builtin_amdgcn_readlane((int)(incl - local), src);          // sample values above its words
    const int word = kSampleBins / 2 - 1 - src * WPL - lane;
    const uint32_t w = hist[word], incl2 = run + dpp_scan_add_u32((w & 0xFFFFu) + (w >> 16));
    const unsigned long long at2 = __ballot(incl2 >= j);
    const int src2 = at2 ? __ffsll((long long)at2) - 1 : kWave - 1;
    const uint32_t cw = (uint32_t)__builtin_amdgcn_readlane((int)w, src2);
    static_assert(WPL % (kGroup / 2) == 0, "a lane's words are whole groups");
    const int ahead = src2 & ~(kGroup / 2 - 1);
    above = ahead ? (uint32_t)__builtin_amdgcn_readlane((int)incl2, ahead - 1) : run;
    run = (uint32_t)__builtin_amdgcn_readlane((int)incl2, src2) - (cw & 0xFFFFu) - (cw >> 16);
    const bool upper = run + (cw >> 16) >= j;
    need = j - run - (upper ? 0u : cw >> 16);
    return 2u * (uint32_t)(kSampleBins / 2 - 1 - src * WPL - src2) + (upper ? 1u : 0u);
  };
  if (wave == 0) {
    uint32_t need, above;
    const uint32_t K = find_bin(need, above);
    bool out = outermost_bin(K);
    if (__builtin_expect(bin_around_0(K), 0)) out = ((hist[K >> 1] >> (K & 1u) * 16u) & 0xFFFFu) - need > j / 4u + 8u;
    float at = sample_floor(K);
    if (!out && bounded) {
      const uint32_t G = raised_group(K / kGroup, above, hist, rp, (float)scale, has_pen,
                                      max(2u, (512u * (uint32_t)n_smp + (uint32_t)V - 1u) / (uint32_t)V), (uint32_t)n_smp);
      // (Put below the group's lower end by as little as still tells the two apart when divided by the temperature:
      // what equals the threshold counts as outside the list, and logits on coarse values, whole numbers say, lie on
      // that end by the hundred, having been counted as kept.  64 rows of V = 152064 fp32, whole numbers, top-p 0.99
      // at 0.3: 20 of them left their lists.)
      if (G != K / kGroup) { at = sample_floor(G * kGroup); at -= fmaxf(fabsf(at), kLow) * 0x1p-18f; }
    }
    const BulkRef r = make_bulk_ref(out ? 0.0f : at, scale);
    if (lane == 0) { sm.key_thr = out ? 1u : 0u; sm.ref = r; }
  }
  if (ALONE && tid == kStreamThreads - kWave) word->open(a.call_mark);
  if (has_pen && wave > 0) {
    auto mark = [&](int t) {
      const uint32_t r = (uint32_t)(t - g0) ^ (uint32_t)(EPL - 1);             // (last element of a load first, see `process`)
      if (t >= g0 && t < g1) atomicOr(&bmw[r >> 5], 1u << (r & 31));
    };
#pragma unroll
    for (int j = 0; j < Sh::kHistRegs; ++j)
      if (tid - kWave + j * MT < n_hist) mark(htok[j]);
    // (A round's last requests may lie beyond the list's end: its last token again, for all lanes.  Entered,
    // these would go to one word of LDS one after the other, so rows of MT tokens beyond the end are skipped.
    // V = 40000 fp32, 128 rows of 2000 tokens: streaming kernel 19.3 us with them, 14.6 without.)
    auto mark_all = [&](const int* tok, long long lo, long long hi) {
      constexpr int N = 8;                           // requests at once
      for (long long i0 = lo; i0 < hi; i0 += (long long)N * MT) {
        const int* const from = tok + i0;            // (uniform)
        const uint32_t last = (uint32_t)min(hi - i0, (long long)N * MT) - 1u;
        int t[N];
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] = from[min((uint32_t)(tid - kWave + j * MT), last)];
#pragma unroll
        for (int j = 0; j < N; ++j)
          if ((uint32_t)(j * MT) <= last) mark(t[j]); // (uniform)
      }
    };
    mark_all(a.tokens, hr.lo + (long long)Sh::kHistRegs * MT, hr.hi);
    mark_all(a.p_tokens, pen.p_lo, pen.p_hi);                                  // separate prompt
  }
  __syncthreads();                                   // also: the histogram is dead from here on
  if (__builtin_expect(sm.key_thr != 0u, 0)) {                                    // workgroup-uniform
    // The bins do not tell where the j-th largest lies.  The sample once more (read again, a load at a time: held
    // until here, it costs registers): its lowest finite value, how many there are in the blocks that count, the
    // threads' three largest.
    f0 = f1 = f2 = -INFINITY;
    float lo = INFINITY;
    uint32_t n_fin = 0;
#pragma nounroll
    for (int l = 0; l < SLOADS; ++l) {
      const bool counts = whole || !(l & 1);
      const uint4 q = load_sample(l);
      float z[EPL];
      unpack(q, z);
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (z[i] > -INFINITY) { lo = fminf(lo, z[i]); n_fin += counts ? 1u : 0u; }
      if (counts) best(q);
    }
    uint32_t klo = last_lane_u32(dpp_scan_min_u32(lo == INFINITY ? 0xFFFFFFFFu : key_of(lo)));
    n_fin = last_lane_u32(dpp_scan_add_u32(n_fin));
    if (lane == 0) { sm.red32[wave] = klo; sm.red64[wave] = n_fin; }
    uint4* const z4 = reinterpret_cast<uint4*>(hist);
    for (int i = tid; i < kSampleBins * 2 / 16; i += kStreamThreads) z4[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    klo = sm.red32[0]; n_fin = (uint32_t)sm.red64[0];
#pragma unroll
    for (int w = 1; w < kStreamWaves; ++w) { klo = min(klo, sm.red32[w]); n_fin += (uint32_t)sm.red64[w]; }
    if (n_fin < j) {                                                              // workgroup-uniform
      // A row that is masked almost everywhere (-inf for all but a few hundred tokens, as a grammar
      // constraint leaves it) has fewer finite values in its sample than the list asks for.  Then the
      // lowest of them is the threshold: the list takes every finite element from there up, and what
      // lies below it is bulk as usual.  (No finite sample value at all: the lowest finite float,
      // which makes the finishing kernel pass the row on.)
      const uint32_t k18 = klo == 0xFFFFFFFFu ? 512u : max(klo >> 14, 512u);
      if (tid == 0) sm.ref = make_bulk_ref(value_of(k18 << 14), scale);
    } else {
      // Else over 13-bit keys (sign, exponent, 4 mantissa bits), the bin that holds the j-th largest then split by the
      // next 5.
      auto each_key = [&](auto&& f) {
        if (tail_only) {
          f(key_of(f0)); f(key_of(f1)); f(key_of(f2));
        } else {
#pragma nounroll
          for (int l = 0; l < SLOADS; l += 2) {
            float z[EPL];
            unpack(load_sample(l), z);
#pragma unroll
            for (int i = 0; i < EPL; ++i) f(key_of(z[i]));
          }
        }
      };
      each_key([&](uint32_t k) { count_in(k >> 19); });
      __syncthreads();
      if (tid < 32) sm.sub_hist[tid] = 0;              // (where the waves' sums were)
      uint32_t need = 1, above;
      if (wave == 0) {
        const uint32_t K = find_bin(need, above);
        if (lane == 0) sm.key_thr = K;
      }
      __syncthreads();
      const uint32_t K = sm.key_thr;
      each_key([&](uint32_t k) { if ((k >> 19) == K) atomicAdd(&sm.sub_hist[(k >> 14) & 31u], 1u); });
      __syncthreads();
      if (wave == 0) {
        // lane l: sub-bin 31 - l, descending
        const uint32_t c = lane < 32 ? sm.sub_hist[31 - min(lane, 31)] : 0u;
        const uint32_t incl = dpp_scan_add_u32(c);
        const unsigned long long reach = __ballot(lane < 32 && incl >= need);
        const uint32_t first = reach ? (uint32_t)__ffsll((long long)reach) - 1u : 31u;
        const uint32_t k18 = max((K << 5) | (31u - first), 512u);              // 18-bit key, of a finite value
        const BulkRef r = make_bulk_ref(value_of(k18 << 14), scale);
        if (lane == 0) sm.ref = r;
      }
    }
    __syncthreads();
  }
  BulkRef ref = sm.ref;
  auto uniform = [](float x) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x))); };
  ref.Tc = uniform(ref.Tc); ref.c = uniform(ref.c); ref.off = uniform(ref.off);

  // ---- stream
  if (CHAIN_FIRST) __builtin_amdgcn_s_setprio(0);
  entry_t* const queue = reinterpret_cast<entry_t*>(front) + wave * queue_cap;       // this wave's LDS queue
  const unsigned char* bm8 = reinterpret_cast<const unsigned char*>(bmw);
  uint32_t qn = 0;                          // wave-uniform: list entries in the queue
  float acc = 0.0f;                         // this thread's bulk mass, fixed order of additions

  uint32_t ib = ibase;                      // SH: first vocabulary id of the piece being processed
  // Block masses of a row without any filter.  One scalar branch per load for every other row; a
  // copy of the loop for these rows alone cost all of them registers (bf16 V = 129280, 1024 rows:
  // streaming kernel 90 -> 115 us).  bf16 V = 151643, 256 rows, no filter: finishing kernel 72.6 ->
  // 16 us, streaming kernel 28 us as before, call 99.4 -> 43 us; with the sums in fp32 26.5 + 14.8 us,
  // but fewer bits than the draw by re-reading the row has.
  const bool plain = !SH && !rp.greedy && unfiltered(rp, V);                   // workgroup-uniform
  // Where nothing takes the row's mass it is not summed, which is a third of what a load costs.  (One more branch a
  // load for everybody else took 1 to 2 % of bf16 calls, hence a kernel of its own.)
  const bool masses = !IDS || total_is_used(rp, a);                            // workgroup-uniform
  // Per element a multiply-add, its sign shifted into a mask, a minimum, an exponential and an addition; the
  // elements at or above the threshold and the history tokens (`hb`) are then pushed lane by lane, one
  // of each lane at a time, which takes one or two rounds of a load at the usual list lengths.
  // Bit p of mask and `hb` is element EPL - 1 - p.  A history token's bits are all set for the sum, a NaN,
  // which bulk_term() leaves out: what belongs to the list must not pass through the fp32 sums, not even to be
  // taken out again (6000 tokens around the threshold, penalised away: 3e-5 of the total was left behind).  `it`: the
  // wave's load number in its chunk.  A queue entry is the element's value and its place: fp32 (bits, vocabulary
  // id); bf16 one word, the value's 16 bits above load number, lane and element (5, 6 or 7 + 6 + 3 bits).
  // Whether it is a history token is looked up again when the queue goes out.
  auto process = [&](const uint4& q, int e0, int it, bool guard, uint32_t hb, const uint4& tg) {
    float z[EPL];
    unpack(make_uint4(q.x | tg.x, q.y | tg.y, q.z | tg.z, q.w | tg.w), z);
    if (guard) {
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (e0 + i >= c1) z[i] = -INFINITY;
    }
    uint32_t below = ~0u;
    float x[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      x[i] = bulk_arg(z[i], ref);
      below = __builtin_amdgcn_alignbit(below, __float_as_uint(x[i]), 31);
    }
    uint32_t hits = ~below | hb;
    if (guard) hits = e0 < c1 ? hits & (~0u << max(e0 + EPL - c1, 0)) : 0u;
    const uint32_t place = DT == SIP_F32 ? (uint32_t)(e0 + EPL - 1) + (SH ? ib : 0u) : ((uint32_t)it << 9) | ((uint32_t)lane << 3) | 7u;
    // (a queue that is full is looked at once per load: what it gets beyond its room lies in the next
    // waves' or in the bitmap, and the chunk is given up)
    if (__builtin_amdgcn_readfirstlane((int)qn) <= queue_cap) {
      for (;;) {
        const unsigned long long mask = __ballot(hits != 0);
        if (!mask) break;
        const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, qn));
        if (hits) {
          const uint32_t p = (uint32_t)__ffs((int)hits) - 1u, y = place - p;
          if constexpr (DT == SIP_F32) {
            const uint32_t hi = (p & 1u) ? q.x : q.y, lo = (p & 1u) ? q.z : q.w;
            queue[pos] = make_uint2(p < 2u ? lo : hi, y);
          } else {
            const unsigned long long w = p < 4u ? ((unsigned long long)q.w << 32) | q.z : ((unsigned long long)q.y << 32) | q.x;
            queue[pos] = ((uint32_t)(w >> ((y << 4) & 63u)) << 16) | y;
          }
        }
        hits &= hits - 1u;
        qn += (uint32_t)__popcll(mask);
      }
    }
    if (IDS && !masses) return;
    float g = bulk_term(x[0]);
#pragma unroll
    for (int i = 1; i < EPL; ++i) g += bulk_term(x[i]);
    acc += g;
    if (!SH && plain) {
      // (in two halves of 24 and 20 bits: 32-bit sums over 16 lanes, and four atomics of the wave for the rest)
      const unsigned long long t = blk_bits(g);
      const uint32_t t0 = row16_sum_u32((uint32_t)t & 0xFFFFFFu), t1 = row16_sum_u32((uint32_t)(t >> 24) & 0xFFFFFFu);
      static_assert(((kBlkMagic >> 24) & 0xFFFFFFu) == 0, "neither half holds any of the magic bits");
      if ((lane & 15) == 15) atomicAdd(&sm.blk_mass[(uint32_t)(e0 - c0) / (uint32_t)kBlkElems], ((unsigned long long)t1 << 24) + t0);
    }
  };
  // Element e0 of the piece being processed is bit (ib - ibase) + e0 - c0 of the bitmap, a
  // multiple of EPL: the bits of one 16-byte load are half a byte (fp32) or one byte (bf16).
  // Lanes past the end of the chunk read the last byte; `process` discards what they get.  (e0 =
  // t0 + tid * EPL + a multiple of 64, so that one address serves the loads of a tile.)
  auto hist_bits = [&](int t0, int j, bool guard) -> uint32_t {
    uint32_t bit0 = (uint32_t)(t0 - c0 + tid * EPL) + (SH ? ib - ibase : 0u);
    uint32_t at = (bit0 >> 3) + (uint32_t)(j * (SUB / 8));
    if (guard) at = min(at, (uint32_t)(Sh::kBits / 8 - 1));
    const uint32_t byte = bm8[at];
    return DT == SIP_F32 ? (byte >> (bit0 & 4u)) & 0xFu : byte;
  };
  int it0 = 0;                              // number of the tile's first load
  auto process_tile = [&](const uint4 (&buf)[NL], int t0) {
    uint32_t hb[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) hb[j] = hist_bits(t0, j, false);
    uint4 tg[NL];                           // (looked up for rows without a penalty too: behind a branch a load they took 1 us more of 36)
#pragma unroll
    for (int j = 0; j < NL; ++j) tg[j] = sm.tag_words[hb[j]];
#pragma unroll
    for (int j = 0; j < NL; ++j) process(buf[j], t0 + j * SUB + tid * EPL, it0 + j, false, hb[j], tg[j]);
    it0 += NL;
  };
  auto process_end = [&](const uint4 (&buf)[NL], int t0) {                     // a tile that the chunk ends in
#pragma unroll
    for (int j = 0; j < NL; ++j)
      if (t0 + j * SUB < c1) {               // workgroup-uniform condition
        const uint32_t hb = hist_bits(t0, j, true);
        process(buf[j], t0 + j * SUB + tid * EPL, it0 + j, true, hb, sm.tag_words[hb]);
      }
    it0 += NL;
  };
  // A queue goes out to the segment, behind what other queues have put there so far (in the order in
  // which the waves get here).
  const uint32_t seg_cap = (uint32_t)(ROW ? a.S * a.cap_c : a.cap_c);
  uint2* const seg = a.cand + (size_t)wg * (size_t)seg_cap;
  const int lpp = NL * ((c1 - c0 + TILE - 1) / TILE);                          // load numbers of one piece
  bool lost = false;                        // wave-uniform: the queue overflowed
  // entry i of the queue, as the list has it
  auto taken_out = [&](uint32_t i) -> uint2 {
    uint2 en;
    if constexpr (DT == SIP_F32) {
      en = queue[i];
    } else {
      const uint32_t w = queue[i];
      uint32_t it = (w >> 9) & ((1u << Sh::kLoadBits) - 1), base = ibase + (uint32_t)c0;
      if (SH) { const uint32_t pc = it / (uint32_t)lpp; it -= pc * (uint32_t)lpp; base += pc * (uint32_t)Vl; }
      en = make_uint2(w & 0xFFFF0000u, base + it * (uint32_t)SUB + (uint32_t)wave * (uint32_t)(kWave * EPL) + (w & 511u));
    }
    const uint32_t bit = (en.y - (uint32_t)g0) ^ (uint32_t)(EPL - 1);
    if ((bmw[min(bit >> 5, (uint32_t)(Sh::kBits / 32 - 1))] >> (bit & 31u)) & 1u) en.y |= kTagBit;
    return en;
  };
  uint32_t n_flushed = 0;                   // entries that went out ahead of the end
  auto queue_place = [&](uint32_t& n_out) -> uint32_t {
    n_out = min((uint32_t)__builtin_amdgcn_readfirstlane((int)qn), (uint32_t)queue_cap);
    lost |= qn > (uint32_t)queue_cap;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&sm.seg_cnt, n_out);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
  };
  auto flush = [&]() {
    uint32_t n_out;
    const uint32_t at = queue_place(n_out);
    for (uint32_t i = lane; i < n_out; i += kWave) {
      const uint2 en = taken_out(i);
      if (!ROW || at + i < seg_cap) put<ALONE>(&seg[at + i], en);
    }
    n_flushed += n_out;
    qn = 0;
  };
  // ROW: a queue that is half full goes out, and one that a further pair of tiles like the last would fill.
  // (Half full alone let rows overflow whose pairs of tiles fill a little less than half: V = 50001 fp32, 224
  // rows of 9000 tokens, 174 of them: 645 us, now 54.  After every tile instead of every pair: 2 to 3 % more
  // for every call.)
  uint32_t q_seen = 0;                      // wave-uniform: its entries when last looked at
  auto make_room = [&]() {
    if constexpr (ROW) {
      const int q = __builtin_amdgcn_readfirstlane((int)qn), more = q - (int)q_seen;
      if (q > Sh::kQueue / 2 || q + more + more / 4 + 32 > Sh::kQueue) flush();
      q_seen = (uint32_t)__builtin_amdgcn_readfirstlane((int)qn);
    }
  };

  // Two register buffers in turn: while one tile is processed the other's loads are in flight.  Every
  // tile processed is followed by a request, also where nothing is left to request (it repeats the last
  // 16 bytes), and the loop is left from its middle: with a request that may not have been made the
  // compiler counts the outstanding loads as if it had not, and waits for the loads just issued.
  // (ROW: a whole row may fill a queue several times, so between two of its pairs of tiles a queue may go
  // out.  Stores in the loop cost the waits that come next, so no earlier than make_room() says.)
  if (!SH) {
    int tcur = c0;
    while (tcur + TILE < c1) {
      process_tile(buf[0], tcur);
      load_tile(tnext, buf[0]);
      tnext += TILE; tcur += TILE;
      if (tcur + TILE >= c1) {
#pragma unroll
        for (int j = 0; j < NL; ++j) buf[0][j] = buf[1][j];
        break;
      }
      process_tile(buf[1], tcur);
      load_tile(tnext, buf[1]);
      tnext += TILE; tcur += TILE;
      make_room();
    }
    process_end(buf[0], tcur);
  } else {
    // the same over np pieces: every piece is [c0, c1) of its shard; the requests run ahead of the
    // processing across the piece boundaries (`row` is what load_tile reads from)
    int c_pj = 0, tcur = c0;                         // tile being processed
    auto on = [&]() {
      tcur += TILE;
      if (tcur >= c1) { ++c_pj; tcur = c0; ib += (uint32_t)Vl; }
      return c_pj < np;
    };
    for (;;) {
      if (tcur + TILE <= c1) process_tile(buf[0], tcur); else process_end(buf[0], tcur);
      load_tile(tnext, buf[0]); tnext += TILE; roll();
      if (!on()) break;
      if (tcur + TILE <= c1) process_tile(buf[1], tcur); else process_end(buf[1], tcur);
      load_tile(tnext, buf[1]); tnext += TILE; roll();
      if (!on()) break;
      make_room();
    }
  }
  // ---- the queues go out (ROW = false: only now, all of them), and the chunk's summary
  if (CHAIN_FIRST) __builtin_amdgcn_s_setprio(2);
  uint32_t n_last = 0;
  if constexpr (ROW) {
    // What is left in the queue also stays in registers, so that finishing need not read it back (it does
    // where a queue has gone out before, or is longer); all rounds are under way at once.
    const uint32_t at = queue_place(n_last);
#pragma unroll
    for (int r = 0; r < kRowRegs; ++r) {
      hand->list[r] = make_uint2(0u, kTagBit);
      if ((uint32_t)(r * kWave) < n_last) hand->list[r] = taken_out(min((uint32_t)(r * kWave + lane), n_last - 1u));       // uniform condition
    }
#pragma unroll
    for (int r = 0; r < kRowRegs; ++r) {
      const uint32_t i = (uint32_t)(r * kWave + lane);
      if (i < n_last) {
        if (at + i < seg_cap) seg[at + i] = hand->list[r];
      } else {
        hand->list[r] = make_uint2(0u, 0xFFFFFFFFu);
      }
    }
    for (uint32_t i = (uint32_t)(kRowRegs * kWave + lane); i < n_last; i += kWave) {
      const uint2 en = taken_out(i);
      if (at + i < seg_cap) seg[at + i] = en;
    }
  } else {
    flush();
  }
  const unsigned long long wsum = dpp_scan_add_u64(bulk_units(acc));
  // (31: the queue overflowed; 30: part of it went out early; below: its entries at the end)
  if (lane == kWave - 1) { sm.red64[wave] = wsum; sm.red32[wave] = n_last | (n_flushed ? 1u << 30 : 0u) | (lost ? 1u << 31 : 0u); }
  __syncthreads();
  uint32_t marks = 0, longest = 0;
#pragma unroll
  for (int w = 0; w < kStreamWaves; ++w) { marks |= sm.red32[w]; longest = max(longest, sm.red32[w] & ~(3u << 30)); }
  bool overflow = (marks >> 31) != 0u;
  const uint32_t tot = sm.seg_cnt;
  overflow |= tot > seg_cap;
  const bool blocks = plain && tot <= seg_cap - (uint32_t)Sh::kBlocks;           // workgroup-uniform
  const int n_blk = blocks ? (c1 - c0 + kBlkElems - 1) / kBlkElems : 0;
  if (tid < n_blk) put<ALONE>(reinterpret_cast<unsigned long long*>(seg + seg_cap) - n_blk + tid, ref.none ? 0ull : sm.blk_mass[tid]);
  if (ROW || tid == 0) {
    ChunkOut o;
    o.bulk = 0;
#pragma unroll
    for (int w = 0; w < kStreamWaves; ++w) o.bulk += sm.red64[w];
    if (ref.none) o.bulk = 0;
    o.Tc = ref.Tc;
    o.off = published_off(ref);
    o.cnt = overflow ? kCntOverflow : tot;
    o.n_blk = (uint32_t)n_blk;
    o.unit = sm.ref.unit;
    if (ROW) {                             // (scalar registers: vector registers are short there)
      hand->co = o;
      hand->co.bulk = readlane_u64(o.bulk, 0);
      hand->co.unit = __longlong_as_double((long long)readlane_u64((unsigned long long)__double_as_longlong(o.unit), 0));
      hand->co.cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)o.cnt);
      hand->co.n_blk = (uint32_t)__builtin_amdgcn_readfirstlane((int)o.n_blk);
      hand->longest = (uint32_t)__builtin_amdgcn_readfirstlane((int)longest);
      hand->direct = __builtin_amdgcn_readfirstlane(!(marks >> 30) && longest <= (uint32_t)(kRowRegs * kWave)) != 0;
    }
    if (tid == 0) put<ALONE>(&a.chunks[ROW ? (size_t)b * (size_t)a.S : (size_t)wg], o);
  }
  return true;
}

// IDS: for calls that ask for token ids only.  us a call: V = 152064 bf16, 128 greedy rows 19.9 -> 17.9; V = 83007
// bf16, 287 rows under min-p 39.8 -> 35.8.
template <int DT, bool SH, bool IDS>
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void stream_kernel(Args a) {
  extern __shared__ __align__(16) unsigned char stream_lds[];                  // stream_lds_bytes()
  // Workgroups are handed to the 8 XCDs round-robin by their id.  The chunks of one row read
  // the same sample, so they are renumbered to land on the same XCD (and its L2): id i works
  // on logical chunk (i % 8) * (n / 8) + i / 8 when n, the grid size, is a multiple of 8.
  int wg = blockIdx.x;
  if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  unsigned char* const tables = stream_lds + stream_front_bytes<DT, false>(a.cap_c / kStreamWaves);
  stream_part<DT, SH, false, IDS>(a, wg, stream_lds, *reinterpret_cast<StreamTables<DT, false>*>(tables), nullptr);
}

}  // namespace sip
