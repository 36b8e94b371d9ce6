// The selection of one row whose scores fit the registers of a workgroup, and what the other forms share with it (see
// tb_select.hip for the scheme).
#pragma once

#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

constexpr int kWaveTile = kWave * 4;  // scores per wave tile: one float4 per lane
constexpr int kHistBins = 4096;       // LDS histogram size (12 bits per level)
constexpr int kTopShift = 20;         // key >> 20 = top 12 bits

struct SelectArgs {
  const float* scores;
  int64_t score_stride;
  int64_t N;
  int32_t kk, lo, hi;  // selection: the kk largest of the candidates [lo, hi)
  int32_t* idx;
  int32_t* count;
  int64_t idx_cap;
  int32_t tiles_per_wave;  // of a workgroup that takes the whole row
  // Selection by pieces.  Stage A cuts the row into `pieces` pieces and keeps, per piece, the
  // candidates whose key is not below a threshold that a sample of the whole row puts safely
  // under the kk-th largest key: pairs (score bits, position in the whole row) go to cand
  // [unit][piece][cap] in position order, and the piece's header {number found, b_lo, b_hi, cut}
  // to piece_hdr[unit][piece] (the cut in a row's first piece only, and only where a kernel before
  // stage A has found the bracket; stage B reads the bracket there).  Stage B selects the kk largest among the kept
  // ones, read as one row through the table of the pieces' counts; if the pieces hold fewer
  // than kk keys together or more than stage B has registers for -- the sample misled -- it
  // selects on the original row instead.
  int32_t pieces;
  int64_t piece_len;
  int64_t cap;
  int64_t units;  // rows of the launch (stage A maps its workgroups to rows and pieces itself)
  uint2* cand;
  uint32_t* piece_hdr;
};

// The W per-wave values in s_w (complete after a barrier): returns the sum of the entries of
// the waves before this one and, in `total`, the sum of all.  Every wave scans the values in
// one DPP row (lane i < W of each row holds entry i) instead of adding up W LDS reads per thread.
template <int W>
__device__ inline uint32_t wave_entries_scan(const uint32_t* s_w, uint32_t& total) {
  static_assert(W <= 16, "one DPP row holds the per-wave entries");
  constexpr int kRowShr = 0x110;
  const int l16 = threadIdx.x & 15;
  const uint32_t v = l16 < W ? s_w[l16] : 0u;
  uint32_t incl = v;
  incl += __builtin_amdgcn_update_dpp(0u, incl, kRowShr + 1, 0xF, 0xF, false);
  incl += __builtin_amdgcn_update_dpp(0u, incl, kRowShr + 2, 0xF, 0xF, false);
  if (W > 4) incl += __builtin_amdgcn_update_dpp(0u, incl, kRowShr + 4, 0xF, 0xF, false);
  if (W > 8) incl += __builtin_amdgcn_update_dpp(0u, incl, kRowShr + 8, 0xF, 0xF, false);
  total = __builtin_amdgcn_readlane(incl, W - 1);
  return __builtin_amdgcn_readlane(incl - v, wave_id());
}

// A wave-uniform bound as a value of its own, so that a second pass over the scores compares again: the masks of the
// first pass would otherwise be kept for it, two scalar registers per score, most of them spilled.
__device__ inline uint32_t compared_anew(uint32_t bound) {
  uint32_t b = __builtin_amdgcn_readfirstlane(bound);
  asm volatile("" : "+s"(b));
  return b;
}

// A count of lane masks, added up at this point (left alone, the compiler keeps the masks of a whole pass and counts at
// its end, again with most of them spilled).
__device__ inline void settle(uint32_t& count) {
  asm volatile("" : "+s"(count));
}

constexpr uint32_t kNoScore = 0x7FC00000u;  // a NaN, in the place of what is no candidate: no compare holds for it

// Result of a histogram walk, published in LDS for the whole workgroup.
struct Found {
  uint32_t bin_a, above_a;  // bin in which the running count (from the top bin down) reaches target a, count above it
  uint32_t bin_b, above_b;  // same for target b
  uint32_t extra_total;     // block-wide sum of `extra`
  uint32_t total;           // sum of all bins
  uint32_t need_a, need_b;  // the targets that were searched
  uint32_t count_a;         // entries in bin_a (the histogram itself may be cleared for reuse once the walk is done)
  uint32_t count_b;         // entries in bin_b
  uint32_t pad[2];
};
static_assert(sizeof(Found) == 48, "three 128-bit LDS reads");
constexpr int kFoundWords = sizeof(Found) / 4;

// Walk the 4096-entry LDS histogram (entries the caller does not use are 0) from the highest
// bin down and find, for each of two targets, the bin in which the running count reaches it
// and the count in strictly higher bins.  A target of 0 or beyond the total finds nothing and
// leaves the preset {0, 0}.  The targets may depend on a second block-wide sum: every wave
// brings its `extra` (the same in every lane), and `targets(extra_total, need_a, need_b)` turns the total into
// the targets.
//
// All W waves take part: wave w owns the 4096/W bins below 4096 - (4096/W) w, lane l a run of
// BL = 64/W adjacent bins (128-bit reads), so that (wave, lane, slot) ascending is bin
// descending.  A DPP scan gives the running count inside the wave, the wave totals go through
// LDS and are scanned by every wave; the one lane whose bins contain a target resolves it and
// publishes the result.  Three barriers: the first completes the histogram that the callers
// fill with LDS atomics.  s_extra (W words) is per call site, s_wsum (W words) may be shared by
// all call sites, s_found is per call site and preset to 0.
template <int W, typename Targets>
__device__ inline Found find_bins(const uint32_t* s_hist, uint32_t extra, uint32_t* s_extra, uint32_t* s_wsum,
                                  Found* s_found, Targets&& targets) {
  constexpr int BW = kHistBins / W;  // bins per wave
  constexpr int BL = BW / kWave;     // bins per lane
  static_assert(BL >= 4 && BL % 4 == 0, "whole 128-bit reads per lane");
  const int lane = lane_id();
  const int wave = wave_id();
  if (lane == 0) s_extra[wave] = extra;
  __syncthreads();  // the histogram and s_extra are complete
  const uint32_t bin0 = static_cast<uint32_t>(kHistBins - BW * (wave + 1) + BL * (kWave - 1 - lane));
  uint32_t c[BL];  // ascending bins bin0 .. bin0 + BL - 1
  uint32_t lsum = 0;
#pragma unroll
  for (int i = 0; i < BL / 4; ++i) {
    const uint4 q = *reinterpret_cast<const uint4*>(s_hist + bin0 + 4 * i);
    c[4 * i] = q.x;
    c[4 * i + 1] = q.y;
    c[4 * i + 2] = q.z;
    c[4 * i + 3] = q.w;
    lsum += (q.x + q.y) + (q.z + q.w);
  }
  const uint32_t incl = wave_incl_scan_u32(lsum);
  if (lane == kWave - 1) s_wsum[wave] = incl;
  __syncthreads();
  uint32_t total, extra_total;
  const uint32_t before = wave_entries_scan<W>(s_wsum, total) + incl - lsum;  // count in bins above this lane's
  wave_entries_scan<W>(s_extra, extra_total);
  uint32_t need[2];
  targets(extra_total, need[0], need[1]);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (before < need[t] && need[t] <= before + lsum) {  // at most one thread of the workgroup
      uint32_t run = before, bin = bin0 + BL - 1, cnt = c[BL - 1];
#pragma unroll
      for (int i = BL - 2; i >= 0; --i) {
        if (need[t] > run + cnt) {  // not in this bin: go one down
          run += cnt;
          cnt = c[i];
          --bin;
        }
      }
      if (t == 0) {
        s_found->bin_a = bin;
        s_found->above_a = run;
        s_found->count_a = cnt;
      } else {
        s_found->bin_b = bin;
        s_found->above_b = run;
        s_found->count_b = cnt;
      }
    }
  }
  if (threadIdx.x == 0) {
    s_found->extra_total = extra_total;
    s_found->total = total;
    s_found->need_a = need[0];
    s_found->need_b = need[1];
  }
  __syncthreads();
  return *s_found;
}

// The bracket of top-12-bit bins that a sample of n_s keys (histogram s_hist) gives for the
// kk-th largest of n_cand candidates: the rank of the threshold inside the sample and its
// spread (binomial), in fp32 -- a heuristic only: exact counts decide afterwards whether the
// bracket holds.
template <int W>
__device__ inline void sample_bracket(const uint32_t* s_hist, uint32_t n_valid, uint32_t* s_extra, uint32_t* s_wsum,
                                      Found* s_found, int kk, int64_t n_cand, uint32_t& b_lo, uint32_t& b_hi,
                                      uint32_t* key_lo = nullptr) {
  const Found fb = find_bins<W>(s_hist, n_valid, s_extra, s_wsum, s_found, [&](uint32_t n_s, uint32_t& na, uint32_t& nb) {
    // (hardware reciprocal and square root: approximate, which is all a heuristic needs)
    const float frac = static_cast<float>(kk) * __builtin_amdgcn_rcpf(static_cast<float>(n_cand));
    const float ks_f = frac * static_cast<float>(n_s);
    const float margin = 6.0f * __builtin_amdgcn_sqrtf(ks_f * (1.0f - frac)) + 4.0f;
    const float hi_f = ks_f - margin, lo_f = ks_f + margin;
    na = hi_f < 1.0f ? 0u : static_cast<uint32_t>(hi_f);  // 0: no bin is safely above T
    nb = lo_f >= static_cast<float>(n_s) ? n_s + 1u : static_cast<uint32_t>(lo_f) + 1u;
  });
  b_hi = fb.need_a ? fb.bin_a : (kHistBins - 1);         // top bin of the bracket
  const bool have_lo = fb.need_b <= fb.extra_total && fb.bin_b >= 1u;
  b_lo = have_lo ? fb.bin_b : 1u;                        // bottom bin of the bracket (bin 0 holds only "not a candidate")
  if (b_hi < b_lo) b_hi = b_lo;
  if (key_lo) {
    // A key inside the bottom bin from which up a filter may keep: the bin is a sixteenth of an
    // octave wide, and a distribution that is dense around the threshold puts several times the
    // budget into it.  The sample's target rank is its j-th largest entry of count_b; with the
    // bin's entries taken as evenly spread, everything from one spacing below that entry up is
    // kept (a heuristic like the bracket itself: what decides is the exact count afterwards).
    uint32_t lo_key = b_lo << kTopShift;
    if (have_lo && fb.count_b > 0u) {
      const uint32_t j = fb.need_b - fb.above_b;  // 1 .. count_b
      const uint32_t width = 1u << kTopShift;
      const uint32_t below = fb.count_b > j + 1u ? fb.count_b - (j + 1u) : 0u;  // spacings between the bin's lower edge and the cut
      lo_key += static_cast<uint32_t>((static_cast<unsigned long long>(width) * below) / fb.count_b);
    }
    *key_lo = lo_key;
  }
}

constexpr int kMaxLevels = 4;    // bracketed level (possibly repeated once over all bins) + up to 2 levels of low bits

// LDS of one selection (shared by the bodies that run one after the other in a kernel).
template <int W>
struct SelLds {
  __attribute__((aligned(16))) uint32_t hist[2][kHistBins];  // of alternating levels
  __attribute__((aligned(16))) Found found[kMaxLevels + 1];
  uint32_t part[2][W];
  uint32_t wsum[W];
  uint32_t wgt[W], weq[W];
  uint32_t ntiny;  // keys gathered from a sparsely populated sub-bin
  uint32_t tiny[kWave];
  uint32_t spare[kWave];  // where lanes without an entry store
};
// Stage B: where the pieces' kept keys lie in the row that stage B selects on.
struct PieceTab {
  uint32_t start[kMaxPieces];  // position of piece c's first kept key in that row (pieces padded to multiples of 4)
  uint32_t n[kMaxPieces];      // kept keys of piece c
  uint32_t len;                // length of the row
  uint32_t b_lo, b_hi;         // the bracket the pieces agreed on
  uint32_t ok;                 // the row of kept keys can be selected on
};

// The always-kept ranges, sink prefix [0, lo) and local window [hi, N), and the list's length.  Written last: a
// global store that is still on its way would hold up whatever waits for memory after it.
template <int W, typename Put>
__device__ __forceinline__ void write_fixed_ranges(const SelectArgs& a, const int u, Put&& put) {
  constexpr int kThreads = W * kWave;
  const int tid = threadIdx.x;
  for (int64_t n = tid; n < a.lo; n += kThreads) put(n, static_cast<int32_t>(n));
  for (int64_t n = a.hi + tid; n < a.N; n += kThreads) put(a.lo + a.kk + (n - a.hi), static_cast<int32_t>(n));
  if (tid == 0) a.count[u] = static_cast<int32_t>(a.lo + a.kk + (a.N - a.hi));
}

// Level state of the radix descent: candidates are the keys with lo_key <= key < lo_key + span, histogrammed by
// (key - lo_key) >> shift; keys above `above_key` (only on the first, bracketed level) are counted instead.
struct Level {
  uint32_t lo_key, span, above_key, need;
  int shift;
};
__device__ inline Level bracketed_level(uint32_t b_lo, uint32_t b_hi, int kk) {
  const uint32_t nb = b_hi - b_lo + 1;                         // 12-bit bins in the bracket
  const int e = 31 - __clz(static_cast<int>(kHistBins / nb));  // extra bits of resolution
  return Level{b_lo << kTopShift, nb << kTopShift, (b_hi == kHistBins - 1) ? 0xFFFFFFFFu : ((b_hi + 1) << kTopShift) - 1u,
               static_cast<uint32_t>(kk), kTopShift - e};
}
// the sample misled us (possible on the bracketed level only): every real bin (bin 0 holds only "not a candidate")
__device__ inline void widen_level(Level& v) {
  v.lo_key = 1u << kTopShift;
  v.span = static_cast<uint32_t>(kHistBins - 1) << kTopShift;
  v.shift = kTopShift;
  v.above_key = 0xFFFFFFFFu;
}
// the low bits of the chosen sub-bin
__device__ inline void next_level(Level& v) {
  v.span = 1u << v.shift;
  v.shift = v.shift > 12 ? v.shift - 12 : 0;
  v.above_key = 0xFFFFFFFFu;
}

// The selection of one row whose keys fit the workgroup's registers (NT tiles of 256 per wave).
// STAGE 0: a row of scores; 2: stage B of a selection by pieces (the row is what the pieces kept, read through
// the piece table); 3: a row of scores in LDS (row), whose list goes to LDS (list) as well.  u: the row (b*Hq + h) this
// workgroup selects for.  region: LDS, CAP words per wave, in which a wave collects its part of the list (STAGE 0
// and 3: the histograms, which are done with by then).
//
// One compute unit per row, so what counts is the instructions per score and what a phase waits for:
//  * the sample is loaded first, and its histogram and walk run while the row itself is on its way;
//  * where the bracket lies above zero (a budget below about half of the candidates) no keys are made: the scores' own
//    bits are ordered there; what is no candidate is a NaN that no compare holds for.  A threshold below that, or a cut
//    through equal scores, turns the scores into keys once, in their registers (made again in every pass: 32 rows of 32768,
//    half of the scores kept 18.9 us, now 16.5; 65536 negative scores, a tenth kept 20.8 and 16.5);
//  * histogram adds of scores outside the bracket go to a spare word of the lane instead of being branched around (the
//    exec-mask bookkeeping of a branch per score cost more than the adds: 10.4 -> 9.6 us on a row of 32768);
//  * the output is one pass: a compare per score, the lane masks (scalar registers) give every kept score its place in
//    the wave's LDS region, and after the one barrier that tells the waves where their parts begin the region is copied out 64
//    entries a store (counting first and storing from the registers, 32 stores of a few lanes each: 10.6 -> 10.0).  A
//    wave that keeps more than its region holds counts first after all, and so do all where the budget says so;
//  * nothing derived from a score is kept in registers for a later pass (lane_pos, compared_anew, settle): 58 registers
//    for 8 tiles, so that two workgroups share a compute unit, and none is spilled.
// Selection alone, 32 rows, a tenth kept, us before and now: 1024 scores 6.4 and 4.2, 4096 5.3 and 4.9, 16384 7.7 and 6.9, 32768
// 11.2 and 9.4, 65536 19.8 and 14.8; 512 rows of 16384 14.6 and 12.4, of 32768 27.4 and 19.3.  (1000 vector instructions a
// wave for 32768 scores, now 650; half of a wave's time is waiting for barriers and LDS.)
template <int W, int NT, int STAGE, int CAP>
__device__ __forceinline__ void select_regs(const SelectArgs& a, const int u, const PieceTab* tab, SelLds<W>& sl, uint32_t* region,
                                            const float* row = nullptr, int32_t* list = nullptr) {
  constexpr int kThreads = W * kWave;
  constexpr int kTileElts = W * kWaveTile;  // scores per workgroup-wide tile
  constexpr bool kStageB = STAGE == 2;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int kk = a.kk;
  // stage B: the row is the concatenation of the pieces' kept keys, every piece padded to a
  // multiple of 4; every key of it is a candidate
  const int N = kStageB ? static_cast<int>(tab->len) : static_cast<int>(a.N);
  const int lo = kStageB ? 0 : a.lo, hi = kStageB ? N : a.hi;
  int32_t* out = a.idx + static_cast<int64_t>(u) * a.idx_cap;
  auto put = [&](int64_t i, int32_t n) {  // entry i of the row's list
    out[i] = n;
    if constexpr (STAGE == 3) list[i] = n;
  };
  if (kk == 0) {
    write_fixed_ranges<W>(a, u, put);
    return;
  }
  // stage B: as many tiles per wave as the row needs (its length is not known at launch)
  const int tpw_b = (N + kTileElts - 1) / kTileElts;
  const int tpw = kStageB ? (tpw_b < 1 ? 1 : (tpw_b < NT ? tpw_b : NT)) : NT;
  const int wspan = wave * tpw * kWaveTile;  // first position of the wave's span (the same in every lane)
  const bool refine = kk < hi - lo;
  auto init_lds = [&]() {
    uint4* z = reinterpret_cast<uint4*>(&sl.hist[0][0]);
    for (int i = tid; i < 2 * kHistBins / 4; i += kThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = tid; i < (kMaxLevels + 1) * kFoundWords; i += kThreads) reinterpret_cast<uint32_t*>(&sl.found[0])[i] = 0;
    if (tid == 0) sl.ntiny = 0;
    __syncthreads();
  };
  float s4[NT][4];                    // the scores
  int32_t cidx[kStageB ? NT : 1][4];  // stage B: positions in the original row, -1 where there is no entry
  float sample = 0.f;
  int sample_pos = 0;
  if constexpr (kStageB) {
    // where position n (a multiple of 4) of the row lies in the [piece][cap] arrays, and how
    // many of the four entries from there on are real (the rest is padding)
    const uint2* cand = a.cand + static_cast<int64_t>(u) * a.pieces * a.cap;
    uint4 r01[NT], r23[NT];  // (score bits, position) of entries 0 and 1, 2 and 3
    int valid[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n0 = wspan + j * kWaveTile + lane * 4;
      valid[j] = 0;
      int64_t phys = 0;
      if (j < tpw && n0 < N) {
        int c = 0;  // the last piece that starts at or before n0 (binary search over the starts)
#pragma unroll
        for (int step = kMaxPieces / 2; step >= 1; step >>= 1)
          if (c + step < a.pieces && static_cast<int>(tab->start[c + step]) <= n0) c += step;
        const int off = n0 - static_cast<int>(tab->start[c]);
        valid[j] = static_cast<int>(tab->n[c]) - off;
        phys = c * a.cap + off;
      }
      const uint4* src = reinterpret_cast<const uint4*>(cand + phys);
      r01[j] = src[0];
      r23[j] = src[1];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const uint32_t kv[4] = {r01[j].x, r01[j].z, r23[j].x, r23[j].z};
      const uint32_t iv[4] = {r01[j].y, r01[j].w, r23[j].y, r23[j].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        s4[j][c] = __uint_as_float(c < valid[j] ? kv[c] : kNoScore);
        cidx[kStageB ? j : 0][c] = c < valid[j] ? static_cast<int32_t>(iv[c]) : -1;
      }
    }
  } else {
    const float* s = STAGE == 3 ? row : a.scores + static_cast<int64_t>(u) * a.score_stride;
    const char* s_bytes = reinterpret_cast<const char*>(s);
    // the sample: four adjacent scores at each of kThreads / 4 places spread evenly over the candidates (the
    // lanes of a place share its cache line), one score per thread
    sample_pos = ((lo + (tid >> 2) * (hi - lo) / (kThreads / 4)) & ~3) + (tid & 3);
    sample = s[sample_pos < N ? sample_pos : N - 1];
    __builtin_amdgcn_sched_barrier(0);
    init_lds();
    __builtin_amdgcn_sched_barrier(0);
    // A row's allocation covers score_stride >= N entries and score_stride is a multiple of 4, so the vector that
    // holds the last score lies inside it; positions past it are clamped to it (and are no candidates)
    const uint32_t last = static_cast<uint32_t>((N - 1) & ~3) * 4u;
    float4 raw[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const uint32_t off = static_cast<uint32_t>(wspan + j * kWaveTile + lane * 4) * 4u;
      raw[j] = *reinterpret_cast<const float4*>(s_bytes + (off < last ? off : last));
    }
    __builtin_amdgcn_sched_barrier(0);  // every load of the thread is issued before the first is used
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      s4[j][0] = raw[j].x;
      s4[j][1] = raw[j].y;
      s4[j][2] = raw[j].z;
      s4[j][3] = raw[j].w;
    }
  }
  // The lane's first position, relative to lo, as a value of its own for every pass over the scores: what is derived from it
  // (a position per score, a test per score) would otherwise be kept in registers from one pass for the next.
  auto lane_pos = [&]() -> int {
    int p = wspan + lane * 4 - lo;
    asm volatile("" : "+v"(p));
    return p;
  };
  auto candidate = [&](int p, int j, int c) -> bool {
    if constexpr (kStageB) return cidx[kStageB ? j : 0][c] >= 0;
    return static_cast<uint32_t>(p + j * kWaveTile + c) < static_cast<uint32_t>(hi - lo);
  };
  const bool inside = wspan >= lo && wspan + NT * kWaveTile <= hi;  // every score of the wave is a candidate (not in stage B)
  if constexpr (kStageB) init_lds();
  auto for_each_tile = [&](auto&& body) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
      if (!kStageB || j < tpw) body(j, s4[j]);
  };

  // The kept scores: all whose key is at least T_key (ties: of those equal to it the first r_eq), from 1 up every candidate.
  uint32_t T_key = 1;
  uint32_t r_eq = 0;
  Level v{};
  bool found = false, whole = false;  // whole: every score from lo_key up is kept, none is cut
  int call = 1;
  bool dense = true;
  auto targets = [&](uint32_t c_above, uint32_t& na, uint32_t& nb) {
    na = (c_above < v.need) ? v.need - c_above : 0u;
    nb = 0u;
  };
  // A handful of scores share the chosen sub-bin (the usual case after the bracketed level: its
  // sub-bins are a few thousand key values wide): instead of another histogram level,
  // they have been gathered, one lane each (x: something that is ordered like them), and are ranked against each
  // other in every wave.  Returns the threshold's x and reduces v.need to how many equal to it are needed.
  auto rank_tiny = [&](uint32_t count, bool& whole) -> uint32_t {
    __syncthreads();
    const int n_tiny = static_cast<int>(count);
    const uint32_t mine = lane < n_tiny ? sl.tiny[lane] : 0u;
    uint32_t greater = 0, equal = 0;
    for (int j = 0; j < n_tiny; ++j) {
      const uint32_t other = __builtin_amdgcn_readlane(mine, j);
      greater += other > mine ? 1u : 0u;
      equal += other == mine ? 1u : 0u;
    }
    // the one whose ranks (greater, greater + equal] contain `need` is the threshold
    const unsigned long long hit = ballot64(lane < n_tiny && greater < v.need && v.need <= greater + equal);
    const int L = __ffsll(hit) - 1;  // (several lanes when the threshold value repeats: they agree)
    v.need -= static_cast<uint32_t>(__builtin_amdgcn_readlane(greater, L));
    whole = v.need == static_cast<uint32_t>(__builtin_amdgcn_readlane(equal, L));
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(mine, L));
  };
  if (refine) {
    uint32_t b_lo, b_hi;
    if constexpr (kStageB) {
      // the pieces have already derived the bracket from their sample of the row
      b_lo = tab->b_lo;
      b_hi = tab->b_hi;
    } else {
      const bool valid = sample_pos >= lo && sample_pos < hi;
      if (valid) atomicAdd(&sl.hist[0][score_key(sample) >> kTopShift], 1u);
      sample_bracket<W>(sl.hist[0], popc64(ballot64(valid)), sl.part[0], sl.wsum, &sl.found[0], kk, hi - lo, b_lo, b_hi);
    }
    __builtin_amdgcn_sched_barrier(0);  // (the row's scores are waited for from here on)
    if constexpr (!kStageB) {
      if (!inside) {  // (scalar)
        const int p = lane_pos();
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int c = 0; c < 4; ++c) s4[j][c] = candidate(p, j, c) ? s4[j][c] : __uint_as_float(kNoScore);
      }
    }
    v = bracketed_level(b_lo, b_hi, kk);
    constexpr uint32_t kSign = 0x80000000u, kPastInf = 0x7F800001u;
    if (v.lo_key > kSign) {
      // The bracket lies above zero (a budget below about half of the candidates): the bits of the scores
      // themselves are ordered there, and those of what is negative, NaN or no candidate lie outside every range that
      // ends at +inf, so no key has to be made (four instructions a score).
      const uint32_t lo_bits = v.lo_key ^ kSign;
      const uint32_t span = min(v.span, kPastInf - lo_bits);
      const float f_above = __uint_as_float(v.above_key ^ kSign);  // (past +inf: a NaN, nothing is above)
      uint32_t n_above = 0;
      for_each_tile([&](int, const float(&f4)[4]) {
        uint32_t* w[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t d = __float_as_uint(f4[c]) - lo_bits;
          n_above += popc64(ballot64(f4[c] > f_above));
          w[c] = d < span ? &sl.hist[1][d >> v.shift] : &sl.spare[lane];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) atomicAdd(w[c], 1u);
        settle(n_above);
      });
      const Found f = find_bins<W>(sl.hist[1], n_above, sl.part[1], sl.wsum, &sl.found[1], targets);
      call = 2;
      if (f.need_a >= 1u && f.need_a <= f.total) {
        v.lo_key += f.bin_a << v.shift;
        v.need = f.need_a - f.above_a;
        if (v.need == f.count_a) {
          found = whole = true;  // every score of this sub-bin is needed: no reason to look at its low bits
        } else if (v.shift == 0) {
          found = true;
        } else if (f.count_a <= static_cast<uint32_t>(kWave)) {
          const uint32_t bin_bits = v.lo_key ^ kSign;
          const uint32_t sub = min(1u << v.shift, kPastInf - bin_bits);
          for_each_tile([&](int, const float(&f4)[4]) {
            const uint32_t d0 = __float_as_uint(f4[0]) - bin_bits, d1 = __float_as_uint(f4[1]) - bin_bits;
            const uint32_t d2 = __float_as_uint(f4[2]) - bin_bits, d3 = __float_as_uint(f4[3]) - bin_bits;
            const uint32_t dmin = min(min(d0, d1), min(d2, d3));
            if (ballot64(dmin < sub) != 0ull) {
              const uint32_t d[4] = {d0, d1, d2, d3};
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (d[c] < sub) sl.tiny[atomicAdd(&sl.ntiny, 1u)] = d[c];
            }
          });
          v.lo_key += rank_tiny(f.count_a, whole);
          found = true;
        } else {
          next_level(v);
          dense = false;
        }
      } else {
        widen_level(v);
      }
    }
  }
  // Unless the threshold is known and a positive score that cuts no ties, what follows is over keys (0: not a candidate; no
  // real score has a key below 0x007FFFFF), which take the scores' registers.
  const bool keyed = __builtin_amdgcn_readfirstlane(!(found && whole)) != 0;
  if (keyed) {
    const int p = lane_pos();
    // (one score after the other, in place: left alone, the compiler keeps scores beside their keys, and spills)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        asm volatile("" : "+v"(s4[j][c]));
        s4[j][c] = __uint_as_float(!kStageB || candidate(p, j, c) ? score_key(s4[j][c]) : 0u);
        asm volatile("" : "+v"(s4[j][c]));
      }
    if (!kStageB && !inside) {  // (scalar)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) s4[j][c] = candidate(p, j, c) ? s4[j][c] : 0.f;
    }
  }
  if (refine) {
    if (!found) {
      auto key4 = [](const float(&f4)[4], uint32_t(&k4)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) k4[c] = __float_as_uint(f4[c]);
      };
#pragma nounroll
      for (; call <= kMaxLevels; ++call) {
        uint32_t* h = sl.hist[call & 1];
        if (call > 1) {  // (it held an earlier level, or the sample)
          uint4* z = reinterpret_cast<uint4*>(h);
          for (int i = tid; i < kHistBins / 4; i += kThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
          __syncthreads();
        }
        uint32_t n_above = 0;
        if (dense) {
          // a sizeable share of the keys falls into the range: test every key on its own.
          // (key > above_key implies key - lo_key >= span, so the two cases are disjoint.)
          for_each_tile([&](int, const float(&f4)[4]) {
            uint32_t k4[4];
            key4(f4, k4);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const uint32_t d = k4[c] - v.lo_key;  // wraps to a large value for keys below lo_key
              n_above += popc64(ballot64(k4[c] > v.above_key));
              if (d < v.span) atomicAdd(&h[d >> v.shift], 1u);
            }
            settle(n_above);
          });
        } else {
          // only the keys of one sub-bin take part: skip wave-uniformly
          for_each_tile([&](int, const float(&f4)[4]) {
            uint32_t k4[4];
            key4(f4, k4);
            const uint32_t d0 = k4[0] - v.lo_key, d1 = k4[1] - v.lo_key, d2 = k4[2] - v.lo_key, d3 = k4[3] - v.lo_key;
            const uint32_t dmin = min(min(d0, d1), min(d2, d3));
            if (ballot64(dmin < v.span) != 0ull) {
              if (d0 < v.span) atomicAdd(&h[d0 >> v.shift], 1u);
              if (d1 < v.span) atomicAdd(&h[d1 >> v.shift], 1u);
              if (d2 < v.span) atomicAdd(&h[d2 >> v.shift], 1u);
              if (d3 < v.span) atomicAdd(&h[d3 >> v.shift], 1u);
            }
          });
        }
        const Found f = find_bins<W>(h, n_above, sl.part[call & 1], sl.wsum, &sl.found[call], targets);
        if (f.need_a >= 1u && f.need_a <= f.total) {  // T lies inside this level's range: descend
          v.lo_key += f.bin_a << v.shift;
          v.need = f.need_a - f.above_a;
          if (v.need == f.count_a) {
            whole = true;
            break;
          }
          if (v.shift == 0) break;
          if (f.count_a <= static_cast<uint32_t>(kWave)) {
            const uint32_t sub = 1u << v.shift;
            for_each_tile([&](int, const float(&f4)[4]) {
              uint32_t k4[4];
              key4(f4, k4);
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                const uint32_t d = k4[c] - v.lo_key;
                if (d < sub) sl.tiny[atomicAdd(&sl.ntiny, 1u)] = d;
              }
            });
            v.lo_key += rank_tiny(f.count_a, whole);
            break;
          }
          next_level(v);
          dense = false;
        } else {
          widen_level(v);
          dense = true;
        }
      }
    }
    T_key = v.lo_key;
    r_eq = whole ? 0u : v.need;
  }

  auto value = [&](int p, int j, int c) -> int32_t {  // what the list holds for score c of tile j (p: lane_pos() + lo)
    return kStageB ? cidx[kStageB ? j : 0][c] : p + j * kWaveTile + c;
  };
  // ---- ordered output, no score equal to T to cut (the usual case).  bound: the bits of T, or T_key; kept(f, bound): the test.
  // Where the budget alone is more than the regions hold, the first pass only counts.
  constexpr bool kFits = NT * kWaveTile <= CAP;  // a wave's region holds all of its scores
  const uint32_t room = kk > W * CAP ? 0u : static_cast<uint32_t>(CAP);
  auto emit = [&](const uint32_t bound, auto&& kept) {
    uint32_t* const part = region + wave * CAP;
    const int p = lane_pos() + lo;
    uint32_t run = 0;  // kept scores of the wave so far (the same in every lane)
    for_each_tile([&](int j, const float(&f4)[4]) {
      const bool t0 = kept(f4[0], bound), t1 = kept(f4[1], bound), t2 = kept(f4[2], bound), t3 = kept(f4[3], bound);
      const unsigned long long m0 = ballot64(t0), m1 = ballot64(t1), m2 = ballot64(t2), m3 = ballot64(t3);
      const uint32_t tot = popc64(m0) + popc64(m1) + popc64(m2) + popc64(m3);
      if (kFits || run + tot <= room) {
        uint32_t* w = part + run + mbcnt64(m3, mbcnt64(m2, mbcnt64(m1, mbcnt64(m0, 0u))));  // after the entries of lower lanes and earlier tiles
        if (t0) *w++ = static_cast<uint32_t>(value(p, j, 0));
        if (t1) *w++ = static_cast<uint32_t>(value(p, j, 1));
        if (t2) *w++ = static_cast<uint32_t>(value(p, j, 2));
        if (t3) *w = static_cast<uint32_t>(value(p, j, 3));
      }
      run += tot;
      settle(run);
    });
    if (lane == 0) sl.wgt[wave] = run;
    __syncthreads();
    uint32_t total;
    uint32_t at = wave_entries_scan<W>(sl.wgt, total);  // kept scores of the waves before
    if (kFits || run <= room) {
      if (at + run <= static_cast<uint32_t>(kk))  // (always, when the counts add up)
        for (uint32_t e = lane; e < run; e += kWave) put(a.lo + at + e, static_cast<int32_t>(part[e]));
    } else {
      // more than the wave's region holds (large scores crowded into its span): from the registers
      const uint32_t again = compared_anew(bound);
      const int p = lane_pos() + lo;
      for_each_tile([&](int j, const float(&f4)[4]) {
        bool t[4];
        unsigned long long m[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          t[c] = kept(f4[c], again);
          m[c] = ballot64(t[c]);
        }
        uint32_t o = mbcnt64(m[3], mbcnt64(m[2], mbcnt64(m[1], mbcnt64(m[0], at))));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (t[c]) {
            if (o < static_cast<uint32_t>(kk)) put(a.lo + o, value(p, j, c));
            ++o;
          }
        }
        at += popc64(m[0]) + popc64(m[1]) + popc64(m[2]) + popc64(m[3]);
      });
    }
  };
  if (r_eq == 0u) {
    if (keyed)  // (scalar)
      emit(T_key, [](float f, uint32_t bound) { return __float_as_uint(f) >= bound; });
    else
      emit(__float_as_uint(score_of_key(T_key)), [](float f, uint32_t bound) { return f >= __uint_as_float(bound); });
  } else {
    // ---- ordered output with ties at the threshold: {key > T} and the first r_eq of {key == T}.
    // Pass A: the wave's totals of both.
    uint32_t run_gt = 0, run_eq = 0;
    for_each_tile([&](int, const float(&f4)[4]) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t k = __float_as_uint(f4[c]);
        run_gt += popc64(ballot64(k > T_key));
        run_eq += popc64(ballot64(k == T_key));
      }
      settle(run_gt);
      settle(run_eq);
    });
    if (lane == 0) {
      sl.wgt[wave] = run_gt;
      sl.weq[wave] = run_eq;
    }
    __syncthreads();
    uint32_t unused;
    uint32_t base_gt = wave_entries_scan<W>(sl.wgt, unused);
    uint32_t base_eq = wave_entries_scan<W>(sl.weq, unused);
    // Pass B: position of a kept score = (#greater before it) + min(#equal before it, r_eq)
    const uint32_t T2 = compared_anew(T_key);
    const int p = lane_pos() + lo;
    for_each_tile([&](int j, const float(&f4)[4]) {
      uint32_t gt = base_gt, eq = base_eq, k4[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        k4[c] = __float_as_uint(f4[c]);
        const unsigned long long mg = ballot64(k4[c] > T2), me = ballot64(k4[c] == T2);
        gt = mbcnt64(mg, gt);
        eq = mbcnt64(me, eq);
        base_gt += popc64(mg);
        base_eq += popc64(me);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bool is_gt = k4[c] > T2, is_eq = k4[c] == T2;
        const uint32_t pos = gt + (eq < r_eq ? eq : r_eq);
        if ((is_gt || (is_eq && eq < r_eq)) && pos < static_cast<uint32_t>(kk)) put(a.lo + pos, value(p, j, c));
        gt += is_gt ? 1u : 0u;
        eq += is_eq ? 1u : 0u;
      }
    });
  }
  write_fixed_ranges<W>(a, u, put);
}

}  // namespace
}  // namespace tb
