// Top-k selection under the policy "candidates = [lo, hi); keep the kk largest scores, lowest
// index wins ties; emit ascending".
//
// The selection of one row (b,h) by one workgroup of W waves: wave w owns the contiguous span
// [w*span, (w+1)*span) of the row's scores and keeps them in registers (up to 64 per thread;
// longer rows are streamed again in every phase).  They are compared through order-preserving
// 32-bit keys: positive scores by their own bits, which are ordered alike, others by keys that take
// their place in the registers.  The exact threshold key T (the kk-th largest) and the number r
// of keys equal to T that are still needed are found by an MSB-first radix descent over LDS
// histograms:
//
//   bracket   a 12-bit histogram of a SAMPLE (one score per thread, four adjacent ones at each
//             of as many places spread evenly over the candidates) gives a range of top-12-bit
//             bins [b_lo, b_hi] that contains T unless the sample is wildly unrepresentative
//             (the rank of T in the sample, +- 6 standard deviations);
//   level 1   exact: every key above the bracket is counted, every key inside it goes into a
//             histogram of up to 4096 sub-bins; if the exact counts show that T is NOT inside
//             the bracket, the level is repeated with the bracket widened to all bins (slow
//             path, same result);
//   level 2+  the remaining low bits, 12 at a time, over the few keys of the chosen sub-bin.
//
// Output: {key > T} U {first r keys == T by index} in ascending order.  Positions come from
// counts (lane masks inside a 256-score wave tile, DPP scans where a row is streamed, running totals along
// the wave's span, the wave totals across the workgroup) -- no atomic slot grabbing, so the result
// is ordered and reproducible.
//
// Launch forms:
//   select_kernel                      one workgroup per row (1024 threads, 512 up to 4096 scores), no global scratch;
//   prefilter_kernel + stage_b_kernel  long rows: the row is cut into pieces, one workgroup per
//                                      piece keeps the keys at or above the lower end of a bracket
//                                      that every piece derives from the same sample of the row
//                                      (or, for a small budget of a very long row, finds ready from
//                                      bracket_kernel), and a second kernel selects among the kept keys;
//   score_bracket_kernel + scoring     long rows of a whole step: the bracket comes from a sample that is scored for it, the
//   kernel + stage_b_kernel            scoring kernel keeps what lies above its lower end.
#include "tb_select_regs.h"

namespace tb {
namespace {

// The four scores at positions n0 .. n0+3 (n0 a multiple of 4) as one 128-bit load without any
// branch, so that a thread's loads can all be in flight together.  A row's allocation covers
// score_stride >= N entries and score_stride is a multiple of 4, so the vector that holds the
// last score lies inside it; a position past that vector (`last4`) is clamped to it, and
// keys_of4 -- which gets the unclamped position -- masks what was read.
__device__ inline float4 load_scores4(const float* s, int64_t last4, int64_t n0) {
  return *reinterpret_cast<const float4*>(s + (n0 < last4 ? n0 : last4));
}

// Keys of the positions n0 .. n0+3.  Positions outside the candidate range [lo, hi) get key 0
// (no real score has a key below 0x007FFFFF).
__device__ inline void keys_of4(const float4& f, int lo, int hi, int64_t n0, uint32_t (&key)[4]) {
  const float v[4] = {f.x, f.y, f.z, f.w};
  if (n0 >= lo && n0 + 3 < hi) {  // the usual case: all four are candidates
#pragma unroll
    for (int c = 0; c < 4; ++c) key[c] = score_key(v[c]);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int64_t n = n0 + c;
      key[c] = (n >= lo && n < hi) ? score_key(v[c]) : 0u;
    }
  }
}

constexpr int kListCap = 16384;  // keys inside the bracket that a streamed row keeps in LDS
constexpr int kStreamBatch = 8;  // tiles in flight per wave while streaming

// Streamed rows: keys inside the bracket (with the wave whose span they come from), every wave's count of keys
// above it, and per-(counting wave, owning wave) tallies of kept / tied keys.
template <int W>
struct ListLds {
  uint32_t ckey[kListCap];
  uint8_t cwave[kListCap];
  uint32_t n;  // keys appended (the list is unusable when beyond its capacity)
  uint32_t wabove[W];
  uint32_t lcnt[W][W][2];
};

// The selection of one row by a workgroup that streams it again in every phase (rows too long for the registers, and
// the fall-back of a selection by pieces); the keys inside the bracket are kept in LDS, so that only two passes read
// the scores.
template <int W>
__device__ __forceinline__ void select_stream(const SelectArgs& a, const int u, SelLds<W>& sl, ListLds<W>& ll) {
  constexpr int kThreads = W * kWave;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int kk = a.kk;
  const int64_t N = a.N;
  const int lo = a.lo, hi = a.hi;
  const float* s = a.scores + static_cast<int64_t>(u) * a.score_stride;
  int32_t* out = a.idx + static_cast<int64_t>(u) * a.idx_cap;
  if (kk == 0) {
    write_fixed_ranges<W>(a, u, [&](int64_t i, int32_t n) { out[i] = n; });
    return;
  }
  const int tpw = a.tiles_per_wave;
  const int64_t wbase = static_cast<int64_t>(wave) * tpw * kWaveTile + lane * 4;
  const bool refine = kk < hi - lo;
  const int64_t last4 = N > 0 ? ((N - 1) & ~int64_t{3}) : 0;  // the vector that holds the last score
  for (int i = tid; i < 2 * kHistBins; i += kThreads) (&sl.hist[0][0])[i] = 0;
  for (int i = tid; i < (kMaxLevels + 1) * kFoundWords; i += kThreads) reinterpret_cast<uint32_t*>(&sl.found[0])[i] = 0;
  if (tid == 0) ll.n = 0;

  // visit every tile of this wave's span: body(j, keys of the tile).  The loads of kStreamBatch tiles are issued
  // before the first tile is used (one load per iteration would leave a wave with 1 KiB in flight and the pass
  // latency-bound)
  auto for_each_tile = [&](auto&& body) {
    for (int j0 = 0; j0 < tpw; j0 += kStreamBatch) {
      float4 raw[kStreamBatch];
#pragma unroll
      for (int t = 0; t < kStreamBatch; ++t)  // tiles past the wave's span read a clamped address and are dropped
        raw[t] = load_scores4(s, last4, wbase + static_cast<int64_t>(j0 + t) * kWaveTile);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < kStreamBatch; ++t) {
        if (j0 + t < tpw) {
          uint32_t k4[4];
          keys_of4(raw[t], lo, hi, wbase + static_cast<int64_t>(j0 + t) * kWaveTile, k4);
          body(j0 + t, k4);
        }
      }
    }
  };

  uint32_t T = 0;        // threshold key: everything above is kept
  uint32_t r_eq = 0;     // how many keys equal to T are kept (lowest indices first)
  bool list_ok = false;  // the LDS list holds every key inside the bracket
  if (refine) {
    __syncthreads();  // LDS initialised
    // bracket from a sample: one key per thread, the first key of a tile that varies with the lane so that the sample
    // is spread over the wave's span.  (More keys would narrow the bracket a little, but they land in a handful of
    // exponent bins and their LDS atomics serialise.)
    uint32_t b_lo, b_hi;
    uint32_t k4[4];
    {
      const int64_t n0 = wbase + static_cast<int64_t>(lane % tpw) * kWaveTile;
      keys_of4(load_scores4(s, last4, n0), lo, hi, n0, k4);
      if (k4[0]) atomicAdd(&sl.hist[0][k4[0] >> kTopShift], 1u);
    }
    sample_bracket<W>(sl.hist[0], popc64(ballot64(k4[0] != 0u)), sl.part[0], sl.wsum, &sl.found[0], kk, hi - lo, b_lo, b_hi);

    Level v = bracketed_level(b_lo, b_hi, kk);
    int cur = 1;  // sl.hist[cur] is clear and becomes this level's histogram
    bool dense = true, take_whole_bin = false;
#pragma nounroll
    for (int call = 1; call <= kMaxLevels; ++call) {
      uint32_t* h = sl.hist[cur];
      uint32_t n_above = 0;
      if (call == 1) {
        // the bracketed level: the keys inside the bracket are also appended to the LDS list (one slot reservation
        // per wave tile)
        for_each_tile([&](int, const uint32_t(&k4)[4]) {
          uint32_t d[4], nin = 0;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            d[c] = k4[c] - v.lo_key;  // wraps to a large value for keys below lo_key
            n_above += (k4[c] > v.above_key) ? 1u : 0u;
            if (d[c] < v.span) {
              atomicAdd(&h[d[c] >> v.shift], 1u);
              ++nin;
            }
          }
          const uint32_t incl = wave_incl_scan_u32(nin);
          const uint32_t tot = __builtin_amdgcn_readlane(incl, kWave - 1);
          if (tot) {
            uint32_t base = 0;
            if (lane == kWave - 1) base = atomicAdd(&ll.n, tot);
            uint32_t pos = __builtin_amdgcn_readlane(base, kWave - 1) + incl - nin;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              if (d[c] < v.span) {
                if (pos < static_cast<uint32_t>(kListCap)) {
                  ll.ckey[pos] = k4[c];
                  ll.cwave[pos] = static_cast<uint8_t>(wave);
                }
                ++pos;
              }
            }
          }
        });
      } else if (dense) {
        for_each_tile([&](int, const uint32_t(&k4)[4]) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const uint32_t d = k4[c] - v.lo_key;
            n_above += (k4[c] > v.above_key) ? 1u : 0u;
            if (d < v.span) atomicAdd(&h[d >> v.shift], 1u);
          }
        });
      } else if (list_ok) {
        // the keys of the chosen sub-bin are all in the LDS list
        const uint32_t nl = ll.n;
        for (uint32_t i = tid; i < nl; i += kThreads) {
          const uint32_t d = ll.ckey[i] - v.lo_key;
          if (d < v.span) atomicAdd(&h[d >> v.shift], 1u);
        }
      } else {
        // only the handful of keys of one sub-bin take part: skip wave-uniformly
        for_each_tile([&](int, const uint32_t(&k4)[4]) {
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
      // clear the other histogram for the next level while this one is being filled
      for (int i = tid; i < kHistBins; i += kThreads) sl.hist[cur ^ 1][i] = 0;
      const uint32_t n_above_wave = __builtin_amdgcn_readlane(wave_incl_scan_u32(n_above), kWave - 1);
      const Found f = find_bins<W>(h, n_above_wave, sl.part[call & 1], sl.wsum, &sl.found[call],
                                   [&](uint32_t c_above, uint32_t& na, uint32_t& nb) {
                                     na = (c_above < v.need) ? v.need - c_above : 0u;
                                     nb = 0u;
                                   });
      if (call == 1) {
        list_ok = ll.n <= static_cast<uint32_t>(kListCap);
        if (tid < W) ll.wabove[tid] = sl.part[1][tid];  // per-wave counts of keys above the bracket
      }
      cur ^= 1;
      if (f.need_a >= 1u && f.need_a <= f.total) {  // T lies inside this level's range: descend
        v.lo_key += f.bin_a << v.shift;
        v.need = f.need_a - f.above_a;
        if (v.need == f.count_a) {
          // every key of this sub-bin is needed: no reason to look at its low bits
          take_whole_bin = true;
          break;
        }
        if (v.shift == 0) break;
        next_level(v);
        dense = false;
      } else {
        widen_level(v);
        list_ok = false;
      }
    }
    T = v.lo_key;
    r_eq = v.need;
    if (take_whole_bin) {  // keep everything from the start of the sub-bin upwards
      T = v.lo_key - 1u;
      r_eq = 0u;
    }
  }
  // kk == hi - lo: T = 0 keeps every candidate (all real keys are > 0)

  // ---- ordered output.  Pass A: the wave's totals of {key > T} and {key == T} (packed: low and high half per tile)
  int32_t* sel_out = out + a.lo;
  auto tile_count = [&](const uint32_t(&k4)[4]) {
    uint32_t cnt = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      cnt += k4[c] > T ? 1u : 0u;
      cnt += (k4[c] == T && r_eq != 0u) ? 0x10000u : 0u;
    }
    return cnt;
  };
  if (list_ok) {
    // the per-wave totals come from the list instead of another pass over the scores (a key above the bracket is kept
    // for sure; a key below it never is)
    for (int i = tid; i < W * W * 2; i += kThreads) (&ll.lcnt[0][0][0])[i] = 0;
    __syncthreads();
    const uint32_t nl = ll.n;
    for (uint32_t i = tid; i < nl; i += kThreads) {
      const uint32_t key = ll.ckey[i];
      const uint32_t w = ll.cwave[i];
      if (key > T) {
        atomicAdd(&ll.lcnt[wave][w][0], 1u);
      } else if (key == T) {
        atomicAdd(&ll.lcnt[wave][w][1], 1u);
      }
    }
    __syncthreads();
    if (tid < W) {
      uint32_t gt = ll.wabove[tid], eq = 0;
      for (int cw = 0; cw < W; ++cw) {
        gt += ll.lcnt[cw][tid][0];
        eq += ll.lcnt[cw][tid][1];
      }
      sl.wgt[tid] = gt;
      sl.weq[tid] = eq;
    }
  } else {
    uint32_t run_gt = 0, run_eq = 0;
    for_each_tile([&](int, const uint32_t(&k4)[4]) {
      const uint32_t tot = __builtin_amdgcn_readlane(wave_incl_scan_u32(tile_count(k4)), kWave - 1);
      run_gt += tot & 0xFFFFu;
      run_eq += tot >> 16;
    });
    if (lane == 0) {
      sl.wgt[wave] = run_gt;
      sl.weq[wave] = run_eq;
    }
  }
  __syncthreads();
  // kept / tied keys in the spans of the waves before this one
  uint32_t unused_total;
  uint32_t base_gt = wave_entries_scan<W>(sl.wgt, unused_total);
  uint32_t base_eq = r_eq != 0u ? wave_entries_scan<W>(sl.weq, unused_total) : 0u;

  // Pass B: position of a kept key = (#greater before it) + min(#equal before it, r_eq)
  for_each_tile([&](int j, const uint32_t(&k4)[4]) {
    const uint32_t cnt = tile_count(k4);
    const uint32_t excl = wave_incl_scan_u32(cnt) - cnt;
    const uint32_t tot = __builtin_amdgcn_readlane(excl + cnt, kWave - 1);
    uint32_t gt_before = base_gt + (excl & 0xFFFFu);
    uint32_t eq_before = base_eq + (excl >> 16);
    const int32_t nn = static_cast<int32_t>(wbase + static_cast<int64_t>(j) * kWaveTile);
    auto emit = [&](uint32_t pos, int c) {
      if (pos < static_cast<uint32_t>(kk)) sel_out[pos] = nn + c;
    };
    if ((tot >> 16) == 0) {
      // no key of this wave tile equals T: the tie count is the same for every slot
      uint32_t pos = gt_before + (eq_before < r_eq ? eq_before : r_eq);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (k4[c] > T) {
          emit(pos, c);
          ++pos;
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bool gt = k4[c] > T;
        const bool eq = k4[c] == T;
        if (gt || (eq && eq_before < r_eq)) emit(gt_before + (eq_before < r_eq ? eq_before : r_eq), c);
        gt_before += gt ? 1u : 0u;
        eq_before += eq ? 1u : 0u;
      }
    }
    base_gt += tot & 0xFFFFu;
    base_eq += tot >> 16;
  });
  write_fixed_ranges<W>(a, u, [&](int64_t i, int32_t n) { out[i] = n; });
}

// ---- moving the scores at or above a bound into a list, with few instructions per score ----------
// A SIMD issues about one instruction in four cycles whatever its kind, so a pass over a row
// costs what it spends per score.  This pass spends one floating-point compare per score (the
// lane masks of a wave tile's four compares stay in scalar registers), eight mask-count
// instructions per tile for the number of entries in lower lanes, and per score one store of
// (score bits, position) -- to the next free slot of the wave's region in LDS, or to a spare
// slot of the lane when the score is below the bound, instead of a branch.  The regions hold
// their entries in position order.
template <int W, int NT, int CAP_PER_TILE>
struct RegionLds {
  static constexpr int kCap = NT * CAP_PER_TILE;  // entries per wave (a tile has 256 scores)
  // The waves' regions one after the other, then one spare slot per lane.  pos mirrors key at a
  // fixed distance, so that one instruction writes both.  A wave with more entries than its
  // region holds runs on into what follows -- the caller then discards the list, but the stores
  // must stay inside the arrays: the last wave's can reach NT * 256 - kCap entries past its
  // region, which `spill` covers.
  uint32_t key[W * kCap + kWave];  // raw score bits
  int32_t pos[W * kCap + kWave];   // position in the row
  uint32_t spill[NT * kWaveTile - kCap];
  uint32_t cnt[W];
};


// Appends the candidates (positions in [lo, hi)) among the wave's NT tiles `raw` -- tile j holds
// the positions pos0 + 256 j + 4 lane .. + 3 -- whose score is at least f_lo (`all`: every
// candidate, NaN included) to the wave's region, and returns their number, the same in every
// lane; beyond RegionLds::kCap the region has overflowed.
template <int W, int NT, int CPT>
__device__ __forceinline__ uint32_t append_at_least(const float4 (&raw)[NT], const int pos0, const int lo, const int hi,
                                                    const float f_lo, const bool all, RegionLds<W, NT, CPT>& rl, const int wave,
                                                    const int lane) {
  using R = RegionLds<W, NT, CPT>;
  constexpr int kCap = R::kCap;
  constexpr int kPosOff = static_cast<int>(sizeof(rl.key) / 4);  // pos[i] is key[i + kPosOff]
  static_assert(offsetof(R, pos) == sizeof(rl.key), "pos follows key");
  static_assert(offsetof(R, spill) == offsetof(R, pos) + sizeof(rl.pos), "the spill area follows pos");
  uint32_t* const lkey = rl.key + wave * kCap;
  uint32_t* const spare = rl.key + W * kCap + lane;
  uint32_t run = 0;
  auto append = [&](int j, bool t0, bool t1, bool t2, bool t3) {
    const float v0 = raw[j].x, v1 = raw[j].y, v2 = raw[j].z, v3 = raw[j].w;
    const int p0 = pos0 + j * kWaveTile + lane * 4;
    const unsigned long long m0 = ballot64(t0), m1 = ballot64(t1), m2 = ballot64(t2), m3 = ballot64(t3);
    uint32_t* w = lkey + run + mbcnt64(m3, mbcnt64(m2, mbcnt64(m1, mbcnt64(m0, 0u))));  // after the entries of lower lanes and earlier tiles
    uint32_t* d;
    d = t0 ? w : spare;
    d[0] = __float_as_uint(v0);
    d[kPosOff] = static_cast<uint32_t>(p0);
    w += t0 ? 1 : 0;
    d = t1 ? w : spare;
    d[0] = __float_as_uint(v1);
    d[kPosOff] = static_cast<uint32_t>(p0 + 1);
    w += t1 ? 1 : 0;
    d = t2 ? w : spare;
    d[0] = __float_as_uint(v2);
    d[kPosOff] = static_cast<uint32_t>(p0 + 2);
    w += t2 ? 1 : 0;
    d = t3 ? w : spare;
    d[0] = __float_as_uint(v3);
    d[kPosOff] = static_cast<uint32_t>(p0 + 3);
    run += popc64(m0) + popc64(m1) + popc64(m2) + popc64(m3);  // (scalar instructions)
  };
  if (pos0 >= lo && pos0 + NT * kWaveTile <= hi) {  // the usual case: every score of the wave's span is a candidate
#pragma unroll
    for (int j = 0; j < NT; ++j) append(j, all || raw[j].x >= f_lo, all || raw[j].y >= f_lo, all || raw[j].z >= f_lo, all || raw[j].w >= f_lo);
  } else {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n_t = pos0 + j * kWaveTile;
      if (n_t >= hi || n_t + kWaveTile <= lo) continue;
      const int p0 = n_t + lane * 4;
      append(j, (all || raw[j].x >= f_lo) && p0 >= lo && p0 < hi, (all || raw[j].y >= f_lo) && p0 + 1 >= lo && p0 + 1 < hi,
             (all || raw[j].z >= f_lo) && p0 + 2 >= lo && p0 + 2 < hi, (all || raw[j].w >= f_lo) && p0 + 3 >= lo && p0 + 3 < hi);
    }
  }
  return run;
}

constexpr int kSelWaves = 16;  // one workgroup per row
constexpr int kSelThreads = kSelWaves * kWave;

template <int NT, int W = kSelWaves>
__global__ __launch_bounds__(W * kWave, (NT >= 1 && NT <= 8) ? 8 : 4)  // up to 8 tiles: two workgroups to a compute unit
void select_kernel(SelectArgs a) {
  __shared__ SelLds<W> sl;
  if constexpr (NT == 0) {
    __shared__ ListLds<kSelWaves> ll;
    select_stream<kSelWaves>(a, blockIdx.x, sl, ll);
  } else {
    select_regs<W, NT, 0, 2 * kHistBins / W>(a, blockIdx.x, nullptr, sl, &sl.hist[0][0]);
  }
}

template <int W>
struct SampleLds {
  uint32_t hist[kHistBins];
  __attribute__((aligned(16))) Found found;
  uint32_t part[W], wsum[W];
};

// The sample of a row: four adjacent scores at each of THREADS * M positions spread evenly over the
// candidates.
template <int THREADS, int M>
__device__ inline int64_t sample_pos(const SelectArgs& a, int i) {
  const int64_t place = static_cast<int64_t>(i) * THREADS + threadIdx.x;
  return (a.lo + place * (a.hi - a.lo) / (THREADS * M)) & ~int64_t{3};
}
template <int THREADS, int M>
__device__ inline void sample_load(const SelectArgs& a, const float* row, float4 (&raw)[M]) {
  const int64_t last4 = (a.N - 1) & ~int64_t{3};
#pragma unroll
  for (int i = 0; i < M; ++i) raw[i] = load_scores4(row, last4, sample_pos<THREADS, M>(a, i));
}
// The bracket of the sample, by the whole workgroup (starts with a barrier, ends with one).
template <int W, int M, typename Lds>
__device__ __forceinline__ void bracket_of_sample(const SelectArgs& a, const float4 (&raw)[M], int64_t span, Lds& sl, uint32_t& b_lo,
                                                  uint32_t& b_hi, uint32_t& t_lo) {
  constexpr int kThreads = W * kWave;
  const int tid = threadIdx.x;
  uint4* z = reinterpret_cast<uint4*>(sl.hist);
  for (int i = tid; i < kHistBins / 4; i += kThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < kFoundWords) reinterpret_cast<uint32_t*>(&sl.found)[tid] = 0;
  __syncthreads();
  uint32_t n_valid = 0;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    uint32_t sk[4];
    keys_of4(raw[i], a.lo, a.hi, sample_pos<kThreads, M>(a, i), sk);  // (the four may straddle an end of the candidate range)
    // all four enter the histogram: a narrower bracket means fewer kept keys to store and to
    // select among
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (sk[e]) atomicAdd(&sl.hist[sk[e] >> kTopShift], 1u);
      n_valid += popc64(ballot64(sk[e] != 0u));
    }
  }
  sample_bracket<W>(sl.hist, n_valid, sl.part, sl.wsum, &sl.found, a.kk, span, b_lo, b_hi, &t_lo);
}

// The bracket of a row from one larger sample, taken once (one workgroup per row): b_lo, b_hi and the
// cut go to the header of the row's first piece.  Bound by its chain of phases (7.6 us for 32 rows).
__global__ __launch_bounds__(kSelThreads) void bracket_kernel(SelectArgs a) {
  constexpr int M = kRowSample / (4 * kSelThreads);
  __shared__ SampleLds<kSelWaves> sl;
  const int u = blockIdx.x, tid = threadIdx.x;
  float4 raw[M];
  sample_load<kSelThreads, M>(a, a.scores + static_cast<int64_t>(u) * a.score_stride, raw);
  __builtin_amdgcn_sched_barrier(0);
  uint32_t b_lo, b_hi, t_lo;
  bracket_of_sample<kSelWaves, M>(a, raw, a.hi - a.lo, sl, b_lo, b_hi, t_lo);
  if (tid < 3) a.piece_hdr[static_cast<int64_t>(u) * a.pieces * 4 + 1 + tid] = tid == 0 ? b_lo : (tid == 1 ? b_hi : t_lo);
}

// The bracket of a row whose scores are not there yet: the workgroup scores a sample of its candidates itself (SAMPLE rows,
// four adjacent ones at each of SAMPLE / 4 places, so that a place is one or two cache lines), and leaves b_lo, b_hi and the cut
// in the header of the row's first piece for the scoring kernel that follows.  A heuristic, as every bracket: the sums
// need not round as that kernel's do.  Bound by its chain: the trips to memory, the histogram, its walk: 6.4 us for 256 rows
// and 2048 scored, 12.8 us for 32 rows and 8192 (with 4096 9.0, but the second stage then takes 20.8 us instead of 13.8).
// The heads of a KV group read the same rows; they are placed on one XCD (workgroups go to the eight round-robin).
struct SampleArgs {
  const void* q_imp;
  const void* Kimp;
  int64_t ki_stride_b, ki_stride_h, ki_stride_n;
  int32_t Hkv, g, n_groups;
  float scale;
};
template <typename T, int DIMP, int SAMPLE>
__global__ __launch_bounds__(kSelThreads) void score_bracket_kernel(SelectArgs a, SampleArgs s) {
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int LPR = DIMP / EPL;             // lanes per projected row
  constexpr int RPP = kSelThreads / LPR;      // rows per pass of the workgroup
  constexpr int PASSES = SAMPLE / RPP;
  constexpr int BATCH = PASSES < 8 ? PASSES : 8;  // loads in flight per lane (two batches are, while one is used)
  constexpr int OWN = SAMPLE / kSelThreads;   // scores that a lane takes over
  static_assert(PASSES % BATCH == 0 && BATCH % LPR == 0 && OWN >= 1, "every lane of a row takes over whole passes");
  __shared__ SampleLds<kSelWaves> sl;
  const int tid = threadIdx.x;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int kvg = xcd + 8 * (slot / s.g);
  if (kvg >= s.n_groups) return;  // (the launch is padded to a multiple of eight groups)
  const int b = kvg / s.Hkv, hkv = kvg % s.Hkv;
  const int u = kvg * s.g + slot % s.g;  // row b*Hq + h
  const int N = static_cast<int>(a.N);
  const int part = tid % LPR, rsub = tid / LPR;
  const T* kbase = static_cast<const T*>(s.Kimp) + b * s.ki_stride_b + hkv * s.ki_stride_h + part * EPL;
  const uint32_t span = static_cast<uint32_t>(a.hi - a.lo);
  static_assert(kSelectMaxN * (SAMPLE / 4) <= (int64_t{1} << 32), "place times span fits 32 bits");
  auto pos_of = [&](int r) -> int {  // row r of the sample
    return ((a.lo + static_cast<int>(static_cast<uint32_t>(r >> 2) * span / (SAMPLE / 4))) & ~3) + (r & 3);
  };
  typename Pack16<T>::Raw kraw[BATCH];
  auto load = [&](int p0) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int n = pos_of((p0 + i) * RPP + rsub);
      kraw[i] = Pack16<T>::load_raw(kbase + (n < N ? n : N - 1) * s.ki_stride_n);
    }
  };
  load(0);
  float qv[EPL];
  Pack16<T>::load(static_cast<const T*>(s.q_imp) + static_cast<int64_t>(u) * DIMP + part * EPL, qv);
  __builtin_amdgcn_sched_barrier(0);
  uint4* z = reinterpret_cast<uint4*>(sl.hist);
  for (int i = tid; i < kHistBins / 4; i += kSelThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < kFoundWords) reinterpret_cast<uint32_t*>(&sl.found)[tid] = 0;
  __syncthreads();
  uint32_t n_valid = 0;
#pragma nounroll
  for (int p0 = 0; p0 < PASSES; p0 += BATCH) {
    float own[BATCH / LPR];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      float kf[EPL], x = 0.f;
      Pack16<T>::unpack(kraw[i], kf);
#pragma unroll
      for (int e = 0; e < EPL; ++e) x = fmaf(qv[e], kf[e], x);
      x = group_allreduce_sum<LPR>(x);
      if (i % LPR == part) own[i / LPR] = x * s.scale;
    }
    if (p0 + BATCH < PASSES) load(p0 + BATCH);
#pragma unroll
    for (int o = 0; o < BATCH / LPR; ++o) {
      const int n = pos_of((p0 + o * LPR + part) * RPP + rsub);
      const bool valid = n >= a.lo && n < a.hi;  // (the four may straddle an end of the candidate range)
      if (valid) atomicAdd(&sl.hist[score_key(own[o]) >> kTopShift], 1u);
      n_valid += popc64(ballot64(valid));
    }
  }
  uint32_t b_lo, b_hi, t_lo;
  sample_bracket<kSelWaves>(sl.hist, n_valid, sl.part, sl.wsum, &sl.found, a.kk, span, b_lo, b_hi, &t_lo);
  if (tid < 3) a.piece_hdr[static_cast<int64_t>(u) * a.pieces * 4 + 1 + tid] = tid == 0 ? b_lo : (tid == 1 ? b_hi : t_lo);
}

template <typename T, int DIMP>
tb_status launch_score_bracket_d(const SelectArgs& a, const SampleArgs& s, int sample, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>((s.n_groups + 7) / 8 * 8 * s.g)), block(kSelThreads);
  if (sample <= kScoredSample)
    hipLaunchKernelGGL((score_bracket_kernel<T, DIMP, kScoredSample>), grid, block, 0, st, a, s);
  else
    hipLaunchKernelGGL((score_bracket_kernel<T, DIMP, kScoredSampleLarge>), grid, block, 0, st, a, s);
  return hip_status(hipGetLastError());
}
template <typename T>
tb_status launch_score_bracket(const ScoreLaunch& S, const SelectArgs& a, const SelectPlan& plan, hipStream_t st) {
  const tb_cache_desc& d = *S.desc;
  const SampleArgs s{S.q_imp, S.Kimp, d.ki_stride_b, d.ki_stride_h, d.ki_stride_n, d.Hkv, d.Hq / d.Hkv, d.B * d.Hkv, S.scale};
  const int sample = plan.row_sample ? kScoredSampleLarge : kScoredSample;
  if (d.Dimp == 16) return launch_score_bracket_d<T, 16>(a, s, sample, st);
  if constexpr (sizeof(T) == 2)
    if (d.Dimp == 32) return launch_score_bracket_d<T, 32>(a, s, sample, st);
  return TB_ERR_UNSUPPORTED;
}

// ---- selection of a row by pieces, stage A.  The piece's scores are in registers (NT tiles per
// wave).  Every piece of a row takes the same sample of the row's candidates (one 128-bit load
// per thread at positions spread evenly over [lo, hi)) and so arrives at the same bracket as its
// siblings (OWN), or reads the bracket that bracket_kernel has left in the header of the row's first
// piece.  The scores whose keys are at or above the bracket's lower end are kept, in position
// order: collected per wave in LDS, then copied out behind the entries of the waves before.
constexpr int kPieceCapPerTile = 56;  // a wave's region holds 22% of its span: several times what a piece keeps
template <int W, int NT, bool OWN>
struct PieceLds {
  SampleLds<OWN ? W : 1> sample[OWN ? 1 : 0];
  RegionLds<W, NT, kPieceCapPerTile> reg;
};

template <int W, int NT, bool OWN>
__device__ __forceinline__ void piece_body(const SelectArgs& a, const int u, const int c, PieceLds<W, NT, OWN>& pl) {
  constexpr int kThreads = W * kWave;
  constexpr int kCap = RegionLds<W, NT, kPieceCapPerTile>::kCap;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int64_t base = c * a.piece_len;
  int64_t n_c = a.N - base;
  n_c = n_c < 0 ? 0 : (n_c > a.piece_len ? a.piece_len : n_c);
  const float* row = a.scores + static_cast<int64_t>(u) * a.score_stride;
  const float* s = row + base;
  const int last4 = n_c > 0 ? static_cast<int>((n_c - 1) & ~int64_t{3}) : 0;
  const int wspan0 = wave * NT * kWaveTile;  // the wave's span, as positions inside the piece
  uint2* out = a.cand + (static_cast<int64_t>(u) * a.pieces + c) * a.cap;
  uint32_t* row_hdr = a.piece_hdr + static_cast<int64_t>(u) * a.pieces * 4;
  uint32_t* hdr = row_hdr + c * 4;
  float4 raw[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n0 = wspan0 + j * kWaveTile + lane * 4;
    raw[j] = *reinterpret_cast<const float4*>(s + (n0 < last4 ? n0 : last4));  // (past the piece's end: excluded by position below)
  }
  uint32_t t_lo;  // keys from here up are kept (inside the bracket's bottom bin)
  if constexpr (OWN) {
    float4 sraw[1];
    const int64_t span = a.hi - a.lo;
    sample_load<kThreads, 1>(a, row, sraw);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t b_lo, b_hi;
    bracket_of_sample<W, 1>(a, sraw, span, pl.sample[0], b_lo, b_hi, t_lo);
    if (tid < 2) hdr[1 + tid] = tid == 0 ? b_lo : b_hi;
  } else {
    t_lo = row_hdr[3];
  }
  // a score is kept when it is at least f_lo; a lower end at or below the key of -inf keeps
  // every candidate (NaN, whose key is that of -inf, included)
  const bool all = t_lo <= kKeyOfMinusInf;
  const float f_lo = all ? 0.f : score_of_key(t_lo);

  // positions are those of the whole row; candidates past the piece's end do not exist (the
  // last piece ends with the row, and hi <= N)
  const int pos0 = static_cast<int>(base) + wspan0;
  const uint32_t run = append_at_least<W, NT>(raw, pos0, a.lo, a.hi, f_lo, all, pl.reg, wave, lane);
  if (lane == 0) pl.reg.cnt[wave] = run;
  __syncthreads();
  uint32_t total;
  const uint32_t wave_base = wave_entries_scan<W>(pl.reg.cnt, total);
  const int l16 = lane & 15;
  const bool overflowed = ballot64(l16 < W && pl.reg.cnt[l16 < W ? l16 : 0] > static_cast<uint32_t>(kCap)) != 0ull;
  if (tid == 0) hdr[0] = total;
  if (!overflowed) {
    const uint32_t* lkey = pl.reg.key + wave * kCap;
    const int32_t* lpos = pl.reg.pos + wave * kCap;
    for (uint32_t e = lane; e < run; e += kWave) {
      const uint32_t at = wave_base + e;
      if (at < static_cast<uint32_t>(a.cap)) out[at] = make_uint2(lkey[e], static_cast<uint32_t>(lpos[e]));
    }
    return;
  }

  // A wave of this piece holds more kept scores than its region (a dense cluster of large
  // scores).  The counts of the pass above are right all the same, so every wave knows where
  // its kept scores go: they are stored from the registers, positions from the compare masks.
  uint32_t at = wave_base;  // kept scores of the waves and tiles before (the same in every lane)
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n_t = pos0 + j * kWaveTile;
    if (n_t >= a.hi || n_t + kWaveTile <= a.lo) continue;
    const int p0 = n_t + lane * 4;
    const float v[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
    bool t[4];
    unsigned long long m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      t[e] = (all || v[e] >= f_lo) && p0 + e >= a.lo && p0 + e < a.hi;  // (the test of the pass above)
      m[e] = ballot64(t[e]);
    }
    uint32_t o = mbcnt64(m[3], mbcnt64(m[2], mbcnt64(m[1], mbcnt64(m[0], at))));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (t[e]) {
        if (o < static_cast<uint32_t>(a.cap)) out[o] = make_uint2(__float_as_uint(v[e]), static_cast<uint32_t>(p0 + e));
        ++o;
      }
    }
    at += popc64(m[0]) + popc64(m[1]) + popc64(m[2]) + popc64(m[3]);
  }
}

// ---- stage B.  One workgroup per row: builds the table of the pieces' kept keys and selects
// among them, or -- when the pieces kept fewer than kk keys, one of them ran out of room, or they
// kept more than this instance holds in registers -- selects on the original row (one streaming
// workgroup: slow, but it only happens when the sample of stage A was wildly unrepresentative).
template <int NT>
__global__ __launch_bounds__(kSelThreads, 4) void stage_b_kernel(SelectArgs a) {
  constexpr int W = kSelWaves;
  __shared__ SelLds<W> sl;
  __shared__ ListLds<W> ll;
  __shared__ PieceTab tab;
  __shared__ uint32_t s_part[3][W];
  const int tid = threadIdx.x;
  const int u = blockIdx.x;
  const uint32_t* hdr = a.piece_hdr + static_cast<int64_t>(u) * a.pieces * 4;
  uint32_t n = 0;
  if (tid < a.pieces) n = hdr[tid * 4];
  const uint32_t padded = (n + 3u) & ~3u;
  const uint32_t incl = wave_incl_scan_u32(padded), incl_n = wave_incl_scan_u32(n);
  if (lane_id() == kWave - 1) {
    s_part[0][wave_id()] = incl;
    s_part[1][wave_id()] = incl_n;
  }
  const bool over = ballot64(n > static_cast<uint32_t>(a.cap)) != 0ull;
  if (lane_id() == 0) s_part[2][wave_id()] = over ? 1u : 0u;
  __syncthreads();
  uint32_t len, kept, overs;
  const uint32_t start = wave_entries_scan<W>(s_part[0], len) + incl - padded;
  wave_entries_scan<W>(s_part[1], kept);
  wave_entries_scan<W>(s_part[2], overs);
  if (tid < kMaxPieces) {
    tab.start[tid] = start;
    tab.n[tid] = n;
  }
  if (tid == 0) {
    tab.len = len;
    tab.b_lo = hdr[1];
    tab.b_hi = hdr[2];
    tab.ok = (overs == 0u && len <= static_cast<uint32_t>(NT * W * kWaveTile) && kept >= static_cast<uint32_t>(a.kk)) ? 1u : 0u;
  }
  __syncthreads();
  if (tab.ok) {
    select_regs<W, NT, 2, kListCap / W>(a, u, &tab, sl, ll.ckey);
  } else {
    select_stream<W>(a, u, sl, ll);
  }
}

// Stage A.  All pieces of a row run on one XCD (workgroups go to the eight XCDs round-robin by
// their linear index), close together in time: the sample of the row that every piece takes is
// then served by that XCD's L2, out of the lines that the row's pieces fetch anyway.
template <int W, int NT, bool OWN>
__global__ __launch_bounds__(W * kWave) void prefilter_kernel(SelectArgs a) {
  __shared__ PieceLds<W, NT, OWN> sl;
  const int64_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int64_t u = (slot / a.pieces) * 8 + xcd;
  if (u >= a.units) return;  // (the launch is padded to a multiple of eight rows)
  // the pieces of a row from its end backwards: with scores that favour recent positions the
  // last pieces keep the most and take the longest, so they should not be the last to start
  piece_body<W, NT, OWN>(a, static_cast<int>(u), a.pieces - 1 - static_cast<int>(slot % a.pieces), sl);
}

template <int W, bool OWN>
tb_status launch_prefilter_w(const SelectArgs& a, int tiles, dim3 grid, hipStream_t st) {
  const dim3 block(W * kWave);
  if (tiles <= 2)
    hipLaunchKernelGGL((prefilter_kernel<W, 2, OWN>), grid, block, 0, st, a);
  else if (tiles <= 4)
    hipLaunchKernelGGL((prefilter_kernel<W, 4, OWN>), grid, block, 0, st, a);
  else if (tiles <= 8)
    hipLaunchKernelGGL((prefilter_kernel<W, 8, OWN>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((prefilter_kernel<W, 16, OWN>), grid, block, 0, st, a);
  return hip_status(hipGetLastError());
}

tb_status launch_whole(const SelectArgs& a, int64_t units, hipStream_t st) {
  SelectArgs b = a;
  const int32_t tiles = static_cast<int32_t>((a.N + kSelWaves * kWaveTile - 1) / (kSelWaves * kWaveTile));  // per wave
  b.tiles_per_wave = tiles;
  dim3 grid(static_cast<unsigned>(units));
  dim3 block(kSelThreads);
  // A workgroup costs what its tiles per wave cost, so there is an instance for (almost) every number (20011 scores, five
  // tiles: 10.3 us as eight, 8.1 now).  Up to 4096 scores eight waves do: their barriers are cheaper than what the
  // other eight would take off them (1024 scores: 4.9 us with sixteen, 4.2; 4096: 5.0 and 4.8; 8192: 5.5 and 6.1).
  constexpr int kFewWaves = 8;
  const dim3 few(kFewWaves * kWave);
  if (a.N <= kFewWaves * kWaveTile)
    hipLaunchKernelGGL((select_kernel<1, kFewWaves>), grid, few, 0, st, b);
  else if (a.N <= 2 * kFewWaves * kWaveTile)
    hipLaunchKernelGGL((select_kernel<2, kFewWaves>), grid, few, 0, st, b);
  else if (tiles <= 2)
    hipLaunchKernelGGL(select_kernel<2>, grid, block, 0, st, b);
  else if (tiles <= 3)
    hipLaunchKernelGGL(select_kernel<3>, grid, block, 0, st, b);
  else if (tiles <= 4)
    hipLaunchKernelGGL(select_kernel<4>, grid, block, 0, st, b);
  else if (tiles <= 5)
    hipLaunchKernelGGL(select_kernel<5>, grid, block, 0, st, b);
  else if (tiles <= 6)
    hipLaunchKernelGGL(select_kernel<6>, grid, block, 0, st, b);
  else if (tiles <= 8)
    hipLaunchKernelGGL(select_kernel<8>, grid, block, 0, st, b);
  else if (tiles <= 10)
    hipLaunchKernelGGL(select_kernel<10>, grid, block, 0, st, b);
  else if (tiles <= 12)
    hipLaunchKernelGGL(select_kernel<12>, grid, block, 0, st, b);
  else if (tiles <= 16)
    hipLaunchKernelGGL(select_kernel<16>, grid, block, 0, st, b);
  else
    hipLaunchKernelGGL(select_kernel<0>, grid, block, 0, st, b);
  return hip_status(hipGetLastError());
}

// Arguments of a selection; with a plan of several pieces, its scratch is [units][pieces][cap] pairs, then the pieces' headers.
SelectArgs select_args(const SelectLaunch& L, const SelectPlan* plan) {
  SelectArgs a;
  a.scores = L.scores;
  a.score_stride = L.score_stride;
  a.N = L.N;
  a.kk = L.kk;
  a.lo = L.lo;
  a.hi = L.hi;
  a.idx = L.idx;
  a.count = L.count;
  a.idx_cap = L.idx_cap;
  a.tiles_per_wave = static_cast<int32_t>((L.N + kSelWaves * kWaveTile - 1) / (kSelWaves * kWaveTile));  // of a workgroup on the whole row
  a.pieces = plan ? plan->pieces : 1;
  a.piece_len = plan ? plan->piece_len : 0;
  a.cap = plan ? plan->cap : 0;
  a.units = L.units;
  a.cand = plan ? static_cast<uint2*>(L.scratch) : nullptr;
  a.piece_hdr = plan ? reinterpret_cast<uint32_t*>(a.cand + L.units * plan->pieces * plan->cap) : nullptr;
  return a;
}

// Second stage over kept keys that are in place.
tb_status launch_stage_b(const SelectArgs& a, const SelectPlan& plan, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(a.units)), block(kSelThreads);
  if (plan.stage_b_tiles <= 2)
    hipLaunchKernelGGL(stage_b_kernel<2>, grid, block, 0, st, a);
  else if (plan.stage_b_tiles <= 4)
    hipLaunchKernelGGL(stage_b_kernel<4>, grid, block, 0, st, a);
  else if (plan.stage_b_tiles <= 8)
    hipLaunchKernelGGL(stage_b_kernel<8>, grid, block, 0, st, a);
  else  // (more than 65536 kept keys falls back to the whole row inside the kernel)
    hipLaunchKernelGGL(stage_b_kernel<16>, grid, block, 0, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace

tb_status launch_select(const SelectLaunch& L, hipStream_t st) {
  if (L.units == 0) return TB_OK;
  const SelectPlan plan = select_plan(L.units, L.hi - L.lo, L.N, L.kk);
  if (plan.pieces <= 1 || !L.scratch || L.scratch_bytes < select_scratch_bytes(L.units, plan))
    return launch_whole(select_args(L, nullptr), L.units, st);

  const SelectArgs a = select_args(L, &plan);
  const dim3 grid(static_cast<unsigned>((L.units + 7) / 8 * 8 * plan.pieces));
  const bool own = !plan.row_sample;
  if (!own) {
    hipLaunchKernelGGL(bracket_kernel, dim3(static_cast<unsigned>(L.units)), dim3(kSelThreads), 0, st, a);
    if (hipGetLastError() != hipSuccess) return TB_ERR_HIP;
  }
  tb_status rc;
  if (plan.piece_waves == 4)
    rc = own ? launch_prefilter_w<4, true>(a, plan.piece_tiles, grid, st) : launch_prefilter_w<4, false>(a, plan.piece_tiles, grid, st);
  else
    rc = own ? launch_prefilter_w<8, true>(a, plan.piece_tiles, grid, st) : launch_prefilter_w<8, false>(a, plan.piece_tiles, grid, st);
  if (rc != TB_OK) return rc;
  return launch_stage_b(a, plan, st);
}

tb_status launch_score_select(const ScoreLaunch& S, const SelectLaunch& L, const SelectPlan& plan, hipStream_t st) {
  const SelectArgs a = select_args(L, &plan);
  tb_status rc = S.desc->dtype == TB_F32 ? launch_score_bracket<float>(S, a, plan, st) : launch_score_bracket<bf16_t>(S, a, plan, st);
  if (rc != TB_OK) return rc;
  rc = launch_score_filter(S, FilterOut{a.cand, a.piece_hdr, plan.pieces, plan.piece_len, plan.cap, L.lo, L.hi, plan.pieces / (S.desc->B * S.desc->Hkv)}, st);
  if (rc != TB_OK) return rc;
  return launch_stage_b(a, plan, st);
}

}  // namespace tb
