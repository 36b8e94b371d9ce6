// Neighbour fetching on an ascending, duplicate-free index list; one workgroup per (b,h) list.
//
// mode 0 (radius): the output is the union of [i-r, i+r] clipped to [0,N).  Because the input
// ascends, entry j adds exactly the positions of its interval that lie beyond the interval of
// entry j-1, so the output length is a prefix sum and every entry writes its own run.
//
// mode 1 (cluster-aware): every selected token adds the next free position past its cluster.
// With D_j = number of still-owed positions right after entry j (itself counted) and
// gap_j = free positions between entries j and j+1, D_j = max(D_{j-1} - gap_{j-1}, 0) + 1 and
// entry j is followed by min(D_j, gap_j) fetched positions.  The recurrence is a composition
// of maps x -> max(x + a, c), which is associative, so it runs as a block-wide prefix scan.
//
// Bound by the chain of phases of one workgroup per list: the list is staged in LDS where it fits
// (coalesced, read several times from there), the arithmetic is 32-bit (N <= 2^30) and a scan costs one
// barrier.  64 lists of 1408 entries, cluster-aware:
// 7.7 -> 5.0 us (17 -> 10 behind a selection, its list not in the L2); 2 lists of 60000: 301 -> 160; 128 lists of
// 4096, radius 1: 11.0 -> 10.0 (its stores lie a run per thread apart).
#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

constexpr int kExpThreads = 1024;
constexpr int kExpWaves = kExpThreads / kWave;

// Entries of a list that are staged in LDS: what 64 KiB hold beside the kernels' own arrays, so that no
// launch has to ask for a larger limit.
constexpr int kExpOwnLds = 256;
constexpr int kExpStaged = (64 * 1024 - kExpOwnLds) / 4;
constexpr int64_t kExpMaxEntries = int64_t{1} << 30;  // N, and so an ascending list, is no longer

struct ExpandArgs {
  int32_t N, radius;
  const int32_t* idx_in;
  const int32_t* count_in;
  int64_t cap_in;  // also the distance between two lists
  int32_t* idx_out;
  int32_t* count_out;
  int64_t cap_out;
};

extern __shared__ int32_t s_list[];

// The list of this workgroup (in LDS when STAGED), its length, and the entries [j0, j1) of this thread.
template <bool STAGED>
__device__ inline const int32_t* open_list(const ExpandArgs& a, int& c, int& j0, int& j1) {
  const int64_t u = blockIdx.x;
  const int32_t* in = a.idx_in + u * a.cap_in;
  const int64_t cnt = a.count_in[u];
  const int64_t most = a.cap_in < kExpMaxEntries ? a.cap_in : kExpMaxEntries;
  c = static_cast<int>(cnt < 0 ? 0 : (cnt > most ? most : cnt));
  const int per = (c + kExpThreads - 1) / kExpThreads;
  j0 = min(static_cast<int>(threadIdx.x) * per, c);
  j1 = min(j0 + per, c);
  if constexpr (STAGED) {
    for (int i = threadIdx.x; i < c; i += kExpThreads) s_list[i] = in[i];
    __syncthreads();
    return s_list;
  } else {
    return in;
  }
}

// Sum over the threads before this one; `total` over all.
__device__ inline uint32_t threads_before(uint32_t v, uint32_t* s_wave, uint32_t& total) {
  const uint32_t incl = wave_incl_scan_u32(v);
  const int wave = wave_id();
  if (lane_id() == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kExpWaves; ++w) {
    const uint32_t t = s_wave[w];
    before += w < wave ? t : 0u;
    total += t;
  }
  return before + incl - v;
}

__device__ inline void write_count(const ExpandArgs& a, uint32_t total) {
  if (threadIdx.x == 0) a.count_out[blockIdx.x] = static_cast<int32_t>(total < static_cast<uint64_t>(a.cap_out) ? total : a.cap_out);
}

template <bool STAGED>
__global__ __launch_bounds__(kExpThreads) void expand_radius_kernel(ExpandArgs a) {
  __shared__ uint32_t s_wave[kExpWaves];
  int c, j0, j1;
  const int32_t* in = open_list<STAGED>(a, c, j0, j1);
  int32_t* out = a.idx_out + static_cast<int64_t>(blockIdx.x) * a.cap_out;
  const int r = a.radius, last = a.N - 1;
  auto hi_of = [&](int i) { return min(i + r, last); };
  const int covered = (j0 > 0 && j0 < j1) ? hi_of(in[j0 - 1]) : -1;  // last position emitted by earlier entries
  uint32_t mine = 0;
  int cov = covered;
  for (int j = j0; j < j1; ++j) {
    const int i = in[j];
    const int s = max(max(i - r, 0), cov + 1), e = hi_of(i);
    if (e >= s) {
      mine += static_cast<uint32_t>(e - s + 1);
      cov = e;
    }
  }
  uint32_t total;
  uint32_t pos = threads_before(mine, s_wave, total);
  cov = covered;
  for (int j = j0; j < j1; ++j) {
    const int i = in[j];
    const int s = max(max(i - r, 0), cov + 1), e = hi_of(i);
    for (int p = s; p <= e; ++p) {
      if (pos < static_cast<uint64_t>(a.cap_out)) out[pos] = p;
      ++pos;
    }
    if (e >= s) cov = e;
  }
  write_count(a, total);
}

// x -> max(x + add, floor): the debt carried across a run of entries.  A debt never exceeds the
// number of entries (< 2^30), so an add of -2^30 or less leaves the floor in any case: adds are kept at
// -2^30 at least, and no sum leaves 32 bits.
struct DebtMap {
  int add, floor;
};
constexpr int kNegBig = -(1 << 30);
__device__ inline DebtMap compose(const DebtMap& first, const DebtMap& then) {
  // then(first(x)) = max(max(x + a1, c1) + a2, c2) = max(x + a1 + a2, max(c1 + a2, c2))
  return DebtMap{max(first.add + then.add, kNegBig), max(first.floor + then.add, then.floor)};
}

template <bool STAGED>
__global__ __launch_bounds__(kExpThreads) void expand_cluster_kernel(ExpandArgs a) {
  __shared__ uint32_t s_wave[kExpWaves];
  __shared__ DebtMap s_map[kExpWaves];
  static_assert(sizeof(s_wave) + sizeof(s_map) <= kExpOwnLds, "the staged list and these fit 64 KiB");
  const int lane = lane_id(), wave = wave_id();
  int c, j0, j1;
  const int32_t* in = open_list<STAGED>(a, c, j0, j1);
  int32_t* out = a.idx_out + static_cast<int64_t>(blockIdx.x) * a.cap_out;

  // map of entry j applied to the debt after entry j-1: D_j = max(D_{j-1} - gap_{j-1}, 0) + 1
  DebtMap mine{0, kNegBig};  // identity
  {
    int prev = j0 > 0 && j0 < j1 ? in[j0 - 1] : 0;
    for (int j = j0; j < j1; ++j) {
      const int i = in[j];
      mine = compose(mine, DebtMap{j > 0 ? 1 - (i - prev - 1) : kNegBig, 1});
      prev = i;
    }
  }
  // inclusive scan of the maps across the wave, then across waves (thread order = list order)
  DebtMap incl = mine;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const DebtMap o{__shfl_up(incl.add, off, kWave), __shfl_up(incl.floor, off, kWave)};
    if (lane >= off) incl = compose(o, incl);
  }
  if (lane == kWave - 1) s_map[wave] = incl;
  __syncthreads();
  DebtMap before{0, kNegBig};
  for (int w = 0; w < wave; ++w) before = compose(before, s_map[w]);
  {
    const DebtMap prev{__shfl_up(incl.add, 1, kWave), __shfl_up(incl.floor, 1, kWave)};
    if (lane > 0) before = compose(before, prev);
  }
  // debt after the last entry handled by earlier threads (0 before the first entry)
  const int debt0 = j0 == 0 ? 0 : max(before.add, before.floor);  // map applied to x = 0

  // visits the thread's entries: body(entry, free positions taken behind it)
  auto walk = [&](auto&& body) {
    int debt = debt0;
    int prev = j0 > 0 && j0 < j1 ? in[j0 - 1] : 0, i = j0 < j1 ? in[j0] : 0;
    for (int j = j0; j < j1; ++j) {
      const int next = j + 1 < c ? in[j + 1] : a.N;
      debt = max(j > 0 ? debt - (i - prev - 1) : 0, 0) + 1;
      body(i, max(min(debt, next - i - 1), 0));
      prev = i;
      i = next;
    }
  };
  uint32_t mine_out = 0;
  walk([&](int, int fill) { mine_out += 1u + static_cast<uint32_t>(fill); });
  uint32_t total;
  uint32_t pos = threads_before(mine_out, s_wave, total);
  walk([&](int i, int fill) {
    for (int f = 0; f <= fill; ++f) {
      if (pos < static_cast<uint64_t>(a.cap_out)) out[pos] = i + f;
      ++pos;
    }
  });
  write_count(a, total);
}

}  // namespace

tb_status launch_expand(int64_t units, int64_t N, int32_t radius, int32_t mode, const int32_t* idx_in,
                        const int32_t* count_in, int64_t cap_in, int32_t* idx_out, int32_t* count_out,
                        int64_t cap_out, hipStream_t st) {
  if (units == 0) return TB_OK;
  ExpandArgs a{static_cast<int32_t>(N), radius, idx_in, count_in, cap_in, idx_out, count_out, cap_out};
  const dim3 grid(static_cast<unsigned>(units)), block(kExpThreads);
  const bool staged = cap_in <= kExpStaged;
  const size_t lds = staged ? static_cast<size_t>(cap_in) * 4 : 0;
  if (mode == 0 && staged)
    hipLaunchKernelGGL(expand_radius_kernel<true>, grid, block, lds, st, a);
  else if (mode == 0)
    hipLaunchKernelGGL(expand_radius_kernel<false>, grid, block, lds, st, a);
  else if (staged)
    hipLaunchKernelGGL(expand_cluster_kernel<true>, grid, block, lds, st, a);
  else
    hipLaunchKernelGGL(expand_cluster_kernel<false>, grid, block, lds, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace tb
