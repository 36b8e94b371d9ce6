// Decode attention over a per-head list of selected rows (gather fused into the kernel: no
// intermediate "important buffer" copy is made).
//
// Work split: nsplit workgroups per (b, h) (placed per XCD when heads share KV rows, see the
// kernel).  The head's list is cut into tiles of 4*GPW rows that go round all its waves (tile t to
// wave t % 4 of workgroup t / 4 % nsplit), where GPW = 64/LPR row groups and LPR = D*sizeof(T)/16
// lanes cover one row with a 128-bit load each (bf16, D=128: 16 lanes per 256 B row, 4 rows per
// wave instruction, 16-row tiles).  All K and V loads of a tile are issued before the first one is consumed, so a wave keeps 8 KiB of gathers in
// flight (measured best: 32-row tiles were 3-5% slower on the batched configurations).  Every lane group runs its own online softmax (running max, running sum, fp32
// accumulator slice of D/LPR elements) in the base-2 domain; groups are merged by wave
// shuffles, waves through LDS, and workgroups through fp32 partials in the workspace: the
// last workgroup of a head to arrive (device-scope counter) combines the partials in split
// order, so the result does not depend on arrival order.  The counter is reset by that
// workgroup, which leaves the workspace ready for the next call.
//
// Why the tiles go round: a head's waves then walk its ascending list together, and so do the heads
// that share a KV head, so the rows of the cache that are being read at any time lie close
// together and a row that several heads list is still in their XCD's L2 when the next one asks for
// it.  With a contiguous slice per wave the heads' positions drift apart by sqrt(slot) / density
// rows, in as many places as there are waves.  And a list shorter than max_count (a widened one)
// still occupies every wave.  Interval of 8 steps, 4 x 32 heads, 65536 rows, widened lists: 908 -> 850 us;
// 2 x 64 heads (eight to a group), 30001 rows: 477 -> 370; 16 x 32 heads, 2048 of 16384 rows, one
// workgroup a head: unchanged.  More workgroups than two a compute unit still lose (768: 893 and 366,
// 1024: 865 and 419 us on these two).
//
// Few KV groups (one, two or four: no placement per XCD, below): the splits of a head lie on the XCDs
// split % 8, and with the tiles going round all of them every XCD fetches the rows of all heads.  There
// (where the splits divide by eight) the list is cut into eight shares, one per XCD, and its tiles go round the
// waves of that XCD.  The first list entry then waits for the count: 0.07 us.  4 groups of eight heads, fp32,
// 2839 of 11356 rows: 15.5 us without shares, 13.2 with them, 6000 of 18000 rows: 24.3 and 18.7; 4 groups of four,
// bf16, 6000 of 18000 rows: 11.7 and 10.9.
//
// Non-temporal gathers: a load that allocates in the last-level cache (256 MB) pays for what it displaces there.  Where a
// launch reads more than that cache keeps for the next one, and heads seldom pick each other's rows (whose lines such a load
// lets go of early), rows are read without.  streams_rows has the rule; 16 x 32 heads on 8, 2048 of 16384 rows 81.5 -> 76.5 us, 16 x 8 heads
// on 8, 8000 rows 97.7 -> 84.5 (537 and 524 MB listed; rows read and folded, nothing else, 76 and 92 us, non-temporally 70 and 78).
//
// A row that arrives in the three-buffer layout's ring comes with the attention of its step: as a launch of its own the copy took
// 4.2 us, all of them launch and one trip to memory.  Interval of 16 steps and a wrap, 2 x 32 heads, 2816 rows a head: 480 -> 418 us.
//
// Head-less lists (one list per batch element for all heads) go through the same kernel with
// the list shared, or, when there are enough KV groups to fill the chip, through
// attn_group_kernel: one workgroup per (b, kv head, split) that serves all query heads of the
// KV head, so that every listed row is loaded once.
#include "tb_attn_rows.h"

namespace tb {
namespace {

constexpr int kGroupWaves = kAttnGroupWaves;  // of a workgroup that serves a KV group on the matrix cores
// occupancy the register allocation is held to: 4 waves per SIMD = 4 workgroups per CU, so that a
// launch of up to 1024 workgroups is resident at once (no second round of workgroups)
constexpr int kAttnWavesPerSimd = 4;

struct AttnArgs {
  const void* q;
  const void* K;
  const void* V;
  const int32_t* idx;
  const int32_t* count;
  int64_t idx_cap, max_count, tail_begin, tail_end, N;
  int64_t k_stride_b, k_stride_h, k_stride_n;
  int64_t v_stride_b, v_stride_h, v_stride_n;
  float sm_scale_log2;
  float* out;
  float* lse;
  float* partials;  // of the splits: accumulators [units][nsplit][D], then (max, sum) pairs [units][nsplit]
  int64_t pairs_off;  // floats before the pairs
  uint32_t* counters;
  int32_t Hq, Hkv, g, nsplit, n_kv_groups, xcd_map;
  int32_t shared_list;  // one list and count per batch element, read by all of its heads
  // buffered form: the listed rows have been copied to per-query-head buffers
  // [B][Hq][buf_cap][D] in list order (slot i of the list is buffer row i); idx is unused
  const void* Kbuf;
  const void* Vbuf;
  int64_t buf_cap;
  // buffered form: row new_row of the cache is on its way there (-1: none).  The workgroup of a KV head's first split copies
  // it from new_from, and everybody reads it from there, so nobody depends on the copy.
  const char* new_from[2];  // K and V: the row of the first KV head
  char* new_to[2];
  int64_t new_from_b[2], new_from_h[2], new_to_b[2], new_to_h[2];  // strides in bytes
  int32_t new_row;
  // buffered form, lists migrated on the way: the rows that `idx` names between its first skip_front and last skip_back entries are
  // taken from the cache src and left in the buffers
  const char* src[2];  // K and V
  int64_t src_b[2], src_h[2], src_n[2];  // strides in bytes
  int64_t src_N;
  int32_t skip_front, skip_back;
  int32_t* count_out;
};

// Asks for the lines of the kernel's arguments together.  A line is a trip to memory the first time that a compute unit
// reads it, and left alone the compiler reads each where it is first used, one trip behind the other.
__device__ __forceinline__ void fetch_args(const AttnArgs& a) {
  asm volatile("" ::"s"(a.q), "s"(a.tail_end), "s"(a.out), "s"(a.g), "s"(a.xcd_map));
}

constexpr int32_t kTailFlag = 0x40000000;  // buffered form: the row number refers to the cache, not the buffer

// Waits until every vector-memory operation this wave has issued, stores included, has been
// acknowledged (s_waitcnt with all counters at zero).
__device__ inline void publish_fence() { __builtin_amdgcn_s_waitcnt(0); }

// A workgroup's (max, sum) of a split, handed over as one 64-bit word.
__device__ inline void store_pair(float* p, float m, float l) {
  const unsigned long long x = __float_as_uint(m) | static_cast<unsigned long long>(__float_as_uint(l)) << 32;
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kAgentScope = 16;  // cache policy of a buffer load that agent-scope stores are visible to (sc1)
// The splits of GH heads where the workgroups have left them (partials `po`, pairs `pp` of the first of them): 128
// bits of an accumulator and its pair per load.  With a scalar load each for value, max and sum (24 instructions
// a thread for 16 splits instead of 4) the kernel took 15.0 us instead of 14.6 (32 heads, 3277 of 32768 rows, cold);
// of these the ticket costs 0.7 and the combination 1.1.
template <int D, int GH, int NW>
__device__ __forceinline__ void combine_published(const float* po, const float* pp, const int nsplit, float* out, float* lse,
                                                  float (&s_m)[NW][GH], float (&s_l)[NW][GH], float (&s_acc)[NW][GH][D]) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(po), 0, GH * nsplit * D * static_cast<int>(sizeof(float)), 0x00027000);
  combine_splits<D, GH, NW>(
      nsplit, out, lse, s_m, s_l, s_acc,
      [&](int at) { return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(pp) + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
      [&](int at, int d) -> u32x4 {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (at * D + d) * static_cast<int>(sizeof(float)), 0, kAgentScope);
      });
}

// SHARES: the list is cut into one share per XCD (nsplit divides by their number).  NT: rows are read non-temporally.  MIG: the
// buffered form of a step that has new lists: a listed row comes from the cache and is stored in its slot of the buffer by the wave
// that attends to it, so that it is not read again: migration 27 us and attention 15.6 apart for 2 x 32 heads, 2816 rows a head, an
// interval of 16 steps and a wrap with two of them 403 -> 372 us.
template <typename T, int D, bool BUF, bool SHARES, bool NT, bool MIG = false>
__global__ __launch_bounds__(kAttnThreads, kAttnWavesPerSimd) void attn_kernel(AttnArgs a) {
  constexpr int EPL = Pack16<T>::kElts;    // elements per lane
  constexpr int LPR = D / EPL;             // lanes per row
  constexpr int GPW = kWave / LPR;         // row groups per wave
  constexpr int TILE = kLoadsPerTile * GPW;  // rows per wave tile
  static_assert(LPR >= 4 && LPR <= 32, "row must span 4..32 lanes");
  static_assert(BUF || !MIG, "rows migrate to buffers");

  __shared__ float s_m[kAttnWaves][1], s_l[kAttnWaves][1];
  __shared__ __attribute__((aligned(16))) float s_acc[kAttnWaves][1][D];
  __shared__ uint32_t s_last;

  fetch_args(a);
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int grp = lane / LPR;
  const int sub = lane % LPR;
  // Workgroups go to the 8 XCDs round-robin by their linear index, and every XCD has an L2 of
  // its own: with grouped queries, the query heads that share a KV head are given to one XCD, so
  // that rows picked by several of them are fetched into one L2 once.  KV group (b, hkv) number
  // k lives on XCD k % 8; slot s of an XCD is (its k-th group, head of the group, split).  (If
  // the hardware places workgroups differently, the mapping is just another order of the work.)
  int split, h, b, hkv;
  if (a.xcd_map) {  // (XCD, split, its k-th group's heads)
    const int k = blockIdx.z / a.g, kvg = blockIdx.x + kXcds * k;
    if (kvg >= a.n_kv_groups) return;  // the last round of groups does not fill all XCDs
    split = blockIdx.y;
    b = kvg / a.Hkv;
    hkv = kvg - b * a.Hkv;
    h = hkv * a.g + (blockIdx.z - k * a.g);
  } else {
    split = blockIdx.x;
    h = blockIdx.y;
    b = blockIdx.z;
    hkv = h / a.g;
  }
  const int64_t u = static_cast<int64_t>(b) * a.Hq + h;

  // The tiles of the list, or of an XCD's share of it, go round the waves (see the head of this file)
  int64_t w_beg = static_cast<int64_t>(split * kAttnWaves + wave) * TILE;
  int64_t stride = static_cast<int64_t>(a.nsplit) * kAttnWaves * TILE;
  int64_t cnt, total;  // set once the count has arrived (first-tile block below); total: this wave's end

  const char* kbase = reinterpret_cast<const char*>(static_cast<const T*>(a.K) + b * a.k_stride_b +
                                                   hkv * a.k_stride_h) + sub * 16;
  const char* vbase = reinterpret_cast<const char*>(static_cast<const T*>(a.V) + b * a.v_stride_b +
                                                   hkv * a.v_stride_h) + sub * 16;
  const uint32_t k_row_bytes = static_cast<uint32_t>(a.k_stride_n * sizeof(T));
  const uint32_t v_row_bytes = static_cast<uint32_t>(a.v_stride_n * sizeof(T));
  const int64_t lu = (!BUF && a.shared_list) ? b : u;  // which list this head reads
  const char* kbuf = nullptr;
  const char* vbuf = nullptr;
  if (BUF) {
    kbuf = reinterpret_cast<const char*>(static_cast<const T*>(a.Kbuf) + u * a.buf_cap * D) + sub * 16;
    vbuf = reinterpret_cast<const char*>(static_cast<const T*>(a.Vbuf) + u * a.buf_cap * D) + sub * 16;
  }
  const char* ksrc = nullptr;
  const char* vsrc = nullptr;
  if (MIG) {
    ksrc = a.src[0] + b * a.src_b[0] + hkv * a.src_h[0] + sub * 16;
    vsrc = a.src[1] + b * a.src_b[1] + hkv * a.src_h[1] + sub * 16;
  }
  const char* knew = nullptr;
  const char* vnew = nullptr;
  int32_t n_new = INT32_MIN;  // the new row as row_at names it (this value: nobody's name)
  if (BUF && a.new_row >= 0) {
    n_new = a.new_row | kTailFlag;
    knew = a.new_from[0] + b * a.new_from_b[0] + hkv * a.new_from_h[0] + sub * 16;
    vnew = a.new_from[1] + b * a.new_from_b[1] + hkv * a.new_from_h[1] + sub * 16;
    if (split == 0 && h % a.g == 0 && tid < LPR) {  // (sub == tid)
      const uint4 kr = *reinterpret_cast<const uint4*>(knew), vr = *reinterpret_cast<const uint4*>(vnew);
      *reinterpret_cast<uint4*>(a.new_to[0] + b * a.new_to_b[0] + hkv * a.new_to_h[0] + sub * 16) = kr;
      *reinterpret_cast<uint4*>(a.new_to[1] + b * a.new_to_b[1] + hkv * a.new_to_h[1] + sub * 16) = vr;
    }
  }

  RowSoftmax<T, D> rows;
  rows.init(static_cast<const T*>(a.q) + u * D + sub * EPL, a.sm_scale_log2);

  // Row numbers of a tile: lane i (modulo the tile) has slot i, an entry of the selected list, then of the dense tail; -1
  // marks a slot past the end.  An entry is read without waiting for the count or asking whether there is one (clamped into the
  // max_count entries that the call names: the list may end with them), ahead of the gathers of the tile before, and looked at when
  // its own tile begins: read under a condition it was waited for on the spot, and with it every gather of the tile before.  With the arguments and the first entries fetched
  // together: steps of 32 heads on 8, 3277 of 32768 rows 27.9 -> 27.2 us, 16 x 32, 2048 of 16384 118.1 -> 116.1, 3 x 32, 2433 of 20011
  // 35.9 -> 34.6; an interval of 8 steps of 4 x 32 heads, 65536 rows 823 -> 814.
  const int64_t last_slot = a.max_count > 0 ? a.max_count - 1 : 0;
  const int32_t* entries = BUF && !MIG ? nullptr : (a.max_count > 0 ? a.idx + lu * a.idx_cap : a.count);
  auto fetch_entry = [&](int64_t t0) -> int32_t {
    if (BUF && !MIG) return 0;  // slot i of the list is row i of the buffer
    const int64_t i = t0 + (lane & (TILE - 1)) + (MIG ? a.skip_front : 0);
    return entries[i < last_slot ? i : last_slot];
  };
  auto row_at = [&](int64_t t0, int32_t entry) -> int32_t {
    const int64_t i = t0 + (lane & (TILE - 1));
    int64_t n = i < cnt ? static_cast<int64_t>(entry) : a.tail_begin + (i - cnt);
    n = n < 0 ? 0 : (n >= a.N ? a.N - 1 : n);  // keep the gather inside the cache whatever the list holds
    int32_t row = static_cast<int32_t>(n);
    if (BUF) row = i < cnt ? static_cast<int32_t>(i) : row | kTailFlag;  // (the tail is read from the cache)
    if (MIG && i < cnt) row = static_cast<int32_t>(entry < 0 ? 0 : (entry >= a.src_N ? a.src_N - 1 : entry));
    return i < total ? row : -1;
  };
  int32_t entry = 0;
  const int32_t cnt_read = a.count[lu];
  if (!SHARES) entry = fetch_entry(w_beg);
  __builtin_amdgcn_sched_barrier(0);  // query, count and entries come in one trip to memory
  cnt = cnt_read < 0 ? 0 : (cnt_read > a.max_count ? a.max_count : cnt_read);
  if (MIG) {
    cnt = max(cnt - a.skip_front - a.skip_back, int64_t{0});
    if (split == 0 && tid == 0) a.count_out[u] = static_cast<int32_t>(cnt);
  }
  total = cnt + (a.tail_end - a.tail_begin);
  if (SHARES) {  // whole tiles per XCD
    const int64_t share = (total + kXcds * TILE - 1) / (kXcds * TILE) * TILE, beg = (split % kXcds) * share;
    w_beg = beg + static_cast<int64_t>(split / kXcds * kAttnWaves + wave) * TILE;
    stride = static_cast<int64_t>(a.nsplit / kXcds) * kAttnWaves * TILE;
    total = min(total, beg + share);
    entry = fetch_entry(w_beg);
  }
  for (int64_t t0 = w_beg; t0 < total; t0 += stride) {
    const int32_t n_mine = row_at(t0, entry);
    entry = fetch_entry(t0 + stride);
    __builtin_amdgcn_sched_barrier(0);
    typename Pack16<T>::Raw kraw[kLoadsPerTile], vraw[kLoadsPerTile];  // kept packed until used
    bool valid[kLoadsPerTile];
#pragma unroll
    for (int t = 0; t < kLoadsPerTile; ++t) {
      const int32_t n = __shfl(n_mine, t * GPW + grp, kWave);
      valid[t] = n >= 0;
      // 32-bit byte offsets from a per-workgroup base (the host checks that a head's slab is
      // below 4 GiB): one address register per gather instead of two
      if (BUF) {
        const bool tail = valid[t] && (n & kTailFlag);
        const uint32_t row = valid[t] ? static_cast<uint32_t>(n & (kTailFlag - 1)) : 0u;
        const char* kp = tail ? kbase + row * k_row_bytes : kbuf + row * static_cast<uint32_t>(D * sizeof(T));
        const char* vp = tail ? vbase + row * v_row_bytes : vbuf + row * static_cast<uint32_t>(D * sizeof(T));
        if (MIG && !tail) {  // (a slot past the end: the cache's first row)
          kp = ksrc + static_cast<int64_t>(row) * a.src_n[0];
          vp = vsrc + static_cast<int64_t>(row) * a.src_n[1];
        }
        if (n == n_new) {
          kp = knew;
          vp = vnew;
        }
        kraw[t] = Pack16<T>::template load_raw<NT>(kp);
        vraw[t] = Pack16<T>::template load_raw<NT>(vp);
      } else {
        const uint32_t row = valid[t] ? static_cast<uint32_t>(n) : 0u;
        kraw[t] = Pack16<T>::template load_raw<NT>(kbase + row * k_row_bytes);
        vraw[t] = Pack16<T>::template load_raw<NT>(vbase + row * v_row_bytes);
      }
    }
    // every gather of the tile is in flight before the first one is consumed
    __builtin_amdgcn_sched_barrier(0);
    rows.consume(kraw, vraw, valid);
    if constexpr (MIG) {
#pragma unroll
      for (int t = 0; t < kLoadsPerTile; ++t) {
        const int64_t slot = t0 + t * GPW + grp;
        if (slot < cnt) {  // (the buffers' own alignment and size are the attention's)
          char* ko = const_cast<char*>(kbuf) + slot * static_cast<int64_t>(D * sizeof(T));
          char* vo = const_cast<char*>(vbuf) + slot * static_cast<int64_t>(D * sizeof(T));
          __builtin_memcpy(__builtin_assume_aligned(ko, 16), &kraw[t], 16);
          __builtin_memcpy(__builtin_assume_aligned(vo, 16), &vraw[t], 16);
        }
      }
    }
  }
  rows.merge_groups();
  if (grp == 0) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) s_acc[wave][0][sub * EPL + e] = rows.acc[e];
    if (sub == 0) {
      s_m[wave][0] = rows.m;
      s_l[wave][0] = rows.l;
    }
  }
  __syncthreads();

  // merge the waves of the workgroup: thread d < D owns output element d
  float M = -INFINITY, L = 0.f, o = 0.f;
  if (tid < D) merge_waves<D, kAttnWaves>(&s_m[0], &s_l[0], &s_acc[0], tid, M, L, o);

  if (a.nsplit == 1) {
    if (tid < D) a.out[u * D + tid] = (L > 0.f) ? o / L : 0.f;
    if (tid == 0 && a.lse) a.lse[u] = (L > 0.f) ? M * kLn2 + logf(L) : -INFINITY;
    return;
  }

  // Several workgroups per head: publish the partial, the last one to arrive combines.
  // Partials are written and read with agent-scope accesses, which go through the L2 of the
  // XCD to the memory side where the L2s of all XCDs meet, so the hand-over needs no cache
  // write-back or invalidate.  Ordering: a store counts against the wave's vector-memory
  // counter until the memory side has acknowledged it, so after publish_fence() (s_waitcnt
  // vmcnt(0)) in every storing wave and the workgroup barrier, the partial of this workgroup is
  // in place; only then does thread 0 issue the ticket, a read-modify-write performed at the
  // memory side.  The drawer of the last ticket issues its agent-scope loads after the ticket
  // has returned (branch on its value behind a barrier), so they find every partial whose
  // ticket preceded its own.
  if (tid < D) __hip_atomic_store(&a.partials[(u * a.nsplit + split) * D + tid], o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) store_pair(a.partials + a.pairs_off + (u * a.nsplit + split) * 2, M, L);
  publish_fence();
  __syncthreads();
  if (tid == 0) {
    const uint32_t ticket = __hip_atomic_fetch_add(&a.counters[u * kCounterStrideWords], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (ticket == static_cast<uint32_t>(a.nsplit - 1)) ? 1u : 0u;
  }
  __syncthreads();
  if (!s_last) return;
  combine_published<D, 1, kAttnWaves>(a.partials + u * a.nsplit * D, a.partials + a.pairs_off + u * a.nsplit * 2, a.nsplit, a.out + u * D,
                                   a.lse ? a.lse + u : nullptr, s_m, s_l, s_acc);
  if (tid == 0) __hip_atomic_store(&a.counters[u * kCounterStrideWords], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the workgroups of a KV group share once their rows are streamed: the waves' (max, sum) pairs
// and accumulators per head.
template <int D, int GH, int NW>
struct GroupLds {
  static constexpr int kThreads = NW * kWave;
  static constexpr int kOutsPerThread = (GH * D + kThreads - 1) / kThreads;
  float m[NW][GH], l[NW][GH];
  __attribute__((aligned(16))) float acc[NW][GH][D];
  uint32_t last;
};

// Merges the waves of the workgroup; with several workgroups per KV group publishes the partial, and
// the last one to arrive combines.
template <int D, int GH, int NW>
__device__ __forceinline__ void group_finish(const AttnArgs& a, const int64_t u0, const int split, GroupLds<D, GH, NW>& gl) {
  constexpr int kThreads = NW * kWave;
  constexpr int OUTS = GH * D;                         // outputs of the workgroup
  constexpr int R = GroupLds<D, GH, NW>::kOutsPerThread;   // outputs per thread in the merges
  const int tid = threadIdx.x;
  __syncthreads();
  // merge the waves: thread owns outputs (head, element) number tid, tid + 256, ...
  float M[R], L[R], o[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = tid + r * kThreads;
    const int hh = (e < OUTS) ? e / D : 0, d = e % D;
    M[r] = -INFINITY;
    L[r] = 0.f;
    o[r] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) M[r] = fmaxf(M[r], gl.m[w][hh]);
    if (M[r] > -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float wgt = exp2_safe(gl.m[w][hh] - M[r]);
        L[r] += gl.l[w][hh] * wgt;
        o[r] += gl.acc[w][hh][d] * wgt;
      }
    }
  }

  if (a.nsplit == 1) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int e = tid + r * kThreads;
      if (e < OUTS) {
        const int hh = e / D, d = e % D;
        a.out[(u0 + hh) * D + d] = (L[r] > 0.f) ? o[r] / L[r] : 0.f;
        if (d == 0 && a.lse) a.lse[u0 + hh] = (L[r] > 0.f) ? M[r] * kLn2 + logf(L[r]) : -INFINITY;
      }
    }
    return;
  }

  // several workgroups per KV group: publish the partials (agent-scope accesses and the same
  // ordering as in attn_kernel), take a ticket, the last to arrive combines in split order
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = tid + r * kThreads;
    if (e < OUTS) {
      const int hh = e / D, d = e % D;
      const int64_t at = (u0 + hh) * a.nsplit + split;
      __hip_atomic_store(&a.partials[at * D + d], o[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (d == 0) store_pair(a.partials + a.pairs_off + at * 2, M[r], L[r]);
    }
  }
  publish_fence();
  __syncthreads();
  if (tid == 0) {
    const uint32_t ticket = __hip_atomic_fetch_add(&a.counters[u0 * kCounterStrideWords], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    gl.last = (ticket == static_cast<uint32_t>(a.nsplit - 1)) ? 1u : 0u;
  }
  __syncthreads();
  if (!gl.last) return;
  combine_published<D, GH, NW>(a.partials + u0 * a.nsplit * D, a.partials + a.pairs_off + u0 * a.nsplit * 2, a.nsplit, a.out + u0 * D,
                            a.lse ? a.lse + u0 : nullptr, gl.m, gl.l, gl.acc);
  if (tid == 0) __hip_atomic_store(&a.counters[u0 * kCounterStrideWords], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Head-less lists with grouped queries (fp32, and groups of two): the GH query heads of a KV head read
// the same rows, so one workgroup serves all of them: every listed row is loaded once and used GH times (the
// loads, not the arithmetic, bound this kernel).  Work split and tiling as in attn_kernel, with
// one workgroup per (b, kv head, split); every lane group keeps GH softmax states and GH
// accumulator slices.  The partial hand-over uses the counter of the group's first head.
template <typename T, int D, int GH>
__global__ __launch_bounds__(kAttnThreads) void attn_group_kernel(AttnArgs a) {
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int LPR = D / EPL;
  constexpr int GPW = kWave / LPR;
  constexpr int TILE = kLoadsPerTile * GPW;
  static_assert(LPR >= 4 && LPR <= 32, "row must span 4..32 lanes");

  __shared__ GroupLds<D, GH, kAttnWaves> gl;

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int grp = lane / LPR;
  const int sub = lane % LPR;
  const int split = blockIdx.x, hkv = blockIdx.y, b = blockIdx.z;
  const int64_t u0 = static_cast<int64_t>(b) * a.Hq + static_cast<int64_t>(hkv) * GH;  // first head of the group

  const int64_t w_beg = static_cast<int64_t>(split * kAttnWaves + wave) * TILE;
  const int64_t stride = static_cast<int64_t>(a.nsplit) * kAttnWaves * TILE;

  const char* kbase = reinterpret_cast<const char*>(static_cast<const T*>(a.K) + b * a.k_stride_b +
                                                   hkv * a.k_stride_h) + sub * 16;
  const char* vbase = reinterpret_cast<const char*>(static_cast<const T*>(a.V) + b * a.v_stride_b +
                                                   hkv * a.v_stride_h) + sub * 16;
  const uint32_t k_row_bytes = static_cast<uint32_t>(a.k_stride_n * sizeof(T));
  const uint32_t v_row_bytes = static_cast<uint32_t>(a.v_stride_n * sizeof(T));
  const int32_t* list = a.idx + b * a.idx_cap;

  float qv[GH][EPL];
#pragma unroll
  for (int j = 0; j < GH; ++j) {
    Pack16<T>::load(static_cast<const T*>(a.q) + (u0 + j) * D + sub * EPL, qv[j]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qv[j][e] *= a.sm_scale_log2;
  }
  float m[GH], l[GH], acc[GH][EPL];
#pragma unroll
  for (int j = 0; j < GH; ++j) {
    m[j] = -INFINITY;
    l[j] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[j][e] = 0.f;
  }

  int64_t cnt = a.count[b];
  cnt = cnt < 0 ? 0 : (cnt > a.max_count ? a.max_count : cnt);
  const int64_t total = cnt + (a.tail_end - a.tail_begin);
  // row numbers of a tile: lanes 0..TILE-1 fetch one entry each (list, then the dense tail)
  auto fetch_rows = [&](int64_t t0) -> int32_t {
    const int64_t i = t0 + lane;
    if (lane < TILE && i < total) {
      int64_t n = (i < cnt) ? static_cast<int64_t>(list[i]) : a.tail_begin + (i - cnt);
      n = n < 0 ? 0 : (n >= a.N ? a.N - 1 : n);  // keep the gather inside the cache whatever the list holds
      return static_cast<int32_t>(n);
    }
    return -1;
  };
  int32_t n_next = fetch_rows(w_beg);
  for (int64_t t0 = w_beg; t0 < total; t0 += stride) {
    const int32_t n_mine = n_next;
    typename Pack16<T>::Raw kraw[kLoadsPerTile], vraw[kLoadsPerTile];
    bool valid[kLoadsPerTile];
#pragma unroll
    for (int t = 0; t < kLoadsPerTile; ++t) {
      const int32_t n = __shfl(n_mine, t * GPW + grp, kWave);
      valid[t] = n >= 0;
      const uint32_t row = valid[t] ? static_cast<uint32_t>(n) : 0u;
      kraw[t] = Pack16<T>::load_raw(kbase + row * k_row_bytes);
      vraw[t] = Pack16<T>::load_raw(vbase + row * v_row_bytes);
    }
    n_next = fetch_rows(t0 + stride);
    __builtin_amdgcn_sched_barrier(0);  // every gather of the tile is in flight before the first is consumed
    clear_past_end(vraw, valid);
    float sc[GH][kLoadsPerTile];
#pragma unroll
    for (int t = 0; t < kLoadsPerTile; ++t) {
      float kf[EPL];
      Pack16<T>::unpack(kraw[t], kf);
#pragma unroll
      for (int j = 0; j < GH; ++j) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) s = fmaf(qv[j][e], kf[e], s);
        s = group_allreduce_sum<LPR>(s);
        sc[j][t] = valid[t] ? s : -INFINITY;
      }
    }
#pragma unroll
    for (int j = 0; j < GH; ++j) {
      float tmax = sc[j][0];
#pragma unroll
      for (int t = 1; t < kLoadsPerTile; ++t) tmax = fmaxf(tmax, sc[j][t]);
      const float m_new = fmaxf(m[j], tmax);
      const float m_ref = (m_new > -INFINITY) ? m_new : 0.f;  // nothing seen yet: all weights 0
      const float alpha = exp2_safe(m[j] - m_ref);
      l[j] *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[j][e] *= alpha;
#pragma unroll
      for (int t = 0; t < kLoadsPerTile; ++t) {
        sc[j][t] = exp2_safe(sc[j][t] - m_ref);  // invalid -> 0
        l[j] += sc[j][t];
      }
      m[j] = m_new;
    }
#pragma unroll
    for (int t = 0; t < kLoadsPerTile; ++t) {
      float vf[EPL];
      Pack16<T>::unpack(vraw[t], vf);
#pragma unroll
      for (int j = 0; j < GH; ++j)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[j][e] = fmaf(sc[j][t], vf[e], acc[j][e]);
    }
  }

  // merge the row groups of the wave, head by head
#pragma unroll
  for (int j = 0; j < GH; ++j) {
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1) {
      const float m_o = __shfl_xor(m[j], off, kWave);
      const float l_o = __shfl_xor(l[j], off, kWave);
      const float m_n = fmaxf(m[j], m_o);
      const float wa = (m_n > -INFINITY) ? exp2_safe(m[j] - m_n) : 0.f;
      const float wb = (m_n > -INFINITY) ? exp2_safe(m_o - m_n) : 0.f;
      l[j] = l[j] * wa + l_o * wb;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float a_o = __shfl_xor(acc[j][e], off, kWave);
        acc[j][e] = acc[j][e] * wa + a_o * wb;
      }
      m[j] = m_n;
    }
    if (grp == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) gl.acc[wave][j][sub * EPL + e] = acc[j][e];
      if (sub == 0) {
        gl.m[wave][j] = m[j];
        gl.l[wave][j] = l[j];
      }
    }
  }
  group_finish<D, GH, kAttnWaves>(a, u0, split, gl);
}

// The same for bf16 on the matrix cores.  GH heads that read the same rows make both halves
// contractions, and on the vector ALUs their arithmetic (about 1760 clocks of a SIMD per 16 rows with
// four heads) is as long as the stream of the rows itself.  A wave takes 32 rows a step:
//
//   scores   (16 rows x D) x (D x heads), v_mfma_f32_16x16x32_bf16: lane (i, kb) = (lane % 16, lane / 16)
//            loads 16 bytes of row i, elements 32 c + 8 kb .. + 7 for slice c; the other operand is the
//            same slice of query i (zero past the group's heads).  Accumulator v of lane (j, kb) is
//            (row 4 kb + v, head j).
//   weights  exp2 in fp32, each the exact sum of three bf16 numbers (its upper halves: all 24 bits),
//            so that the products with V are exact and only the fp32 accumulation rounds.
//   output   (heads x 32 rows) x (32 rows x D): lane (j, kb) already holds the weights of head j for
//            the rows 4 kb + v of both 16-row tiles -- the k slots 8 kb .. + 7 of this operand, in an
//            order of their own that the other operand follows: lane (n, kb) loads elements EV n .. of
//            the same rows of V, and element e of them all is column EV n + e.
//
// Invalid slots repeat the wave's first row with weight 0 (a row that is attended anyway, so that an
// infinite value in an unlisted row cannot reach the result).  Infinite and NaN values in attended rows
// of V give what a sum of products gives (see below): a wave whose result holds a NaN goes over
// its rows a second time, all others pay one test.  Relative error against 64 bits on 3661 rows 2.0e-7
// (vector form: 2.4e-7).
//
// Eight waves a workgroup, one workgroup per compute unit as a rule: as many rows in flight as two
// of four waves, and half the partials for the last workgroup to combine (512 workgroups of eight waves:
// 40.6 us instead of 31.7 below).  Bound by its chain of latencies (list, two steps of gathers,
// hand-over, combination) at 3661 rows, by the gathers beyond.  Score to attention, 32 groups of four
// heads, 3661 rows: 36.8 -> 31.7 us; of eight heads, 8576 rows: 85.9 -> 64.3 us.  Two heads a group
// leave 14 of 16 columns idle and stay on the vector form (8576 rows: 60.4 against 61.7 us).
typedef short attn_bf16x8 __attribute__((ext_vector_type(8)));
typedef float attn_f32x4 __attribute__((ext_vector_type(4)));

template <int D, int GH>
__global__ __launch_bounds__(kGroupWaves * kWave, 2) void attn_group_mfma_kernel(AttnArgs a) {
  constexpr int KC = D / 32;  // slices of a row for the scores
  constexpr int EV = D / 16;  // elements of a V row per lane
  constexpr int VW = EV / 2;  // ... in 32-bit words
  constexpr int STEP = 32;
  typedef uint32_t vword __attribute__((ext_vector_type(VW)));
  static_assert(GH <= 16, "one column per head of the group");
  __shared__ GroupLds<D, GH, kGroupWaves> gl;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  const int i16 = lane & 15, kb = lane >> 4;
  const int split = blockIdx.x, hkv = blockIdx.y, b = blockIdx.z;
  const int64_t u0 = static_cast<int64_t>(b) * a.Hq + static_cast<int64_t>(hkv) * GH;  // first head of the group

  const int64_t w_beg = static_cast<int64_t>(split * kGroupWaves + wave) * STEP;
  const int64_t stride = static_cast<int64_t>(a.nsplit) * kGroupWaves * STEP;
  const char* kbase = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.K) + b * a.k_stride_b + hkv * a.k_stride_h) + kb * 16;
  const char* vbase = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.V) + b * a.v_stride_b + hkv * a.v_stride_h) + i16 * (EV * 2);
  const uint32_t k_row_bytes = static_cast<uint32_t>(a.k_stride_n * sizeof(bf16_t));
  const uint32_t v_row_bytes = static_cast<uint32_t>(a.v_stride_n * sizeof(bf16_t));
  const int32_t* list = a.idx + b * a.idx_cap;

  attn_bf16x8 qop[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const bf16_t* qp = static_cast<const bf16_t*>(a.q) + (u0 + (i16 < GH ? i16 : 0)) * D + c * 32 + kb * 8;
    uint4 t = *reinterpret_cast<const uint4*>(qp);
    if (i16 >= GH) t = make_uint4(0u, 0u, 0u, 0u);
    __builtin_memcpy(&qop[c], &t, 16);
  }
  float m, l;  // of head i16 (l: this lane's rows only)
  // accumulator v: head 4 kb + v, column EV i16 + e; the weights' lower parts are summed apart (one
  // rounding a step at the size of the result instead of three)
  attn_f32x4 acc[EV], acc_low[EV];

  // row of slot i of the list (read as `raw`), or of the dense tail behind it
  int64_t cnt, total;
  auto row_of = [&](int64_t i, int32_t raw) -> int32_t {
    int64_t n = (i < cnt) ? static_cast<int64_t>(raw) : a.tail_begin + (i - cnt);
    n = n < 0 ? 0 : (n >= a.N ? a.N - 1 : n);  // keep the gather inside the cache whatever the list holds
    return static_cast<int32_t>(n);
  };
  // lane r (and r + 32) of a step: the row of its slot r.  The first step's entries are read without
  // waiting for the count (clamped into the entries that the call names, whatever the count is).
  int32_t n_next;
  {
    const int64_t i0 = w_beg + (lane & 31);
    const int64_t last = a.max_count - 1;
    const int32_t raw = a.max_count > 0 ? list[i0 < last ? i0 : last] : 0;
    const int32_t raw_first = a.max_count > 0 ? list[w_beg < last ? w_beg : last] : 0;
    const int64_t c = a.count[b];
    cnt = c < 0 ? 0 : (c > a.max_count ? a.max_count : c);
    total = cnt + (a.tail_end - a.tail_begin);
    n_next = i0 < total ? row_of(i0, raw) : row_of(w_beg, raw_first);
  }
  auto fetch_rows = [&](int64_t t0) -> int32_t {
    int64_t i = t0 + (lane & 31);
    i = i < total ? i : w_beg;
    return row_of(i, i < cnt ? list[i] : 0);
  };
  auto clear = [&]() {
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] = acc_low[e] = attn_f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // kInf: elements of V that are infinite or NaN meet the weights' upper parts only (a lower part may be 0,
  // and 0 times infinity is NaN), and the slots past the list's end count as rows of zeros.
  auto step = [&](const int64_t t0, auto inf_tag) {
    constexpr bool kInf = decltype(inf_tag)::value;
    const int32_t n_mine = n_next;
    attn_bf16x8 kraw[2][KC];
    vword vraw[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint32_t row = static_cast<uint32_t>(__shfl(n_mine, 16 * t + i16, kWave));
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const uint4 x = *reinterpret_cast<const uint4*>(kbase + row * k_row_bytes + c * 64);
        __builtin_memcpy(&kraw[t][c], &x, 16);
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t row = static_cast<uint32_t>(__shfl(n_mine, 16 * t + 4 * kb + v, kWave));
        vraw[t][v] = *reinterpret_cast<const vword*>(vbase + row * v_row_bytes);
      }
    if (t0 + stride < total) n_next = fetch_rows(t0 + stride);
    __builtin_amdgcn_sched_barrier(0);  // every gather of the step is in flight before the first is consumed
    if constexpr (kInf) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (t0 + 16 * t + 4 * kb + v >= total) vraw[t][v] = vword{};
    }
    float p[2][4];
    float tmax = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      // every slice on its own, added pairwise: fewer roundings at the size of the whole sum
      attn_f32x4 sc[KC];
#pragma unroll
      for (int c = 0; c < KC; ++c)
        sc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kraw[t][c], qop[c], attn_f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      const attn_f32x4 s = KC == 2 ? sc[0] + sc[1] : (sc[0] + sc[1]) + (sc[KC - 2] + sc[KC - 1]);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool valid = t0 + 16 * t + 4 * kb + v < total;
        p[t][v] = s[v];
        tmax = fmaxf(tmax, valid ? s[v] * a.sm_scale_log2 : -INFINITY);
      }
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16, kWave));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, kWave));
    const float m_new = fmaxf(m, tmax);
    const float m_ref = (m_new > -INFINITY) ? m_new : 0.f;  // nothing seen yet: all weights 0
    if (__any(m_new > m)) {
      const float alpha = exp2_safe(m - m_ref);
      l *= alpha;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float al = __shfl(alpha, 4 * kb + v, kWave);  // (lane j < 16 holds head j)
#pragma unroll
        for (int e = 0; e < EV; ++e) {
          acc[e][v] *= al;
          acc_low[e][v] *= al;
        }
      }
      m = m_new;
    }
    uint32_t part[3][4];  // the weights of the eight rows as three bf16 numbers each, packed in pairs
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t w[3][2];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          // one rounding for the scaled score and its distance to the maximum
          const bool valid = t0 + 16 * t + 4 * kb + 2 * h + o < total;
          const float x = valid ? exp2_safe(fmaf(p[t][2 * h + o], a.sm_scale_log2, -m_ref)) : 0.f;
          l += x;
          w[0][o] = __float_as_uint(x) & 0xFFFF0000u;
          const float r = x - __uint_as_float(w[0][o]);  // exact
          w[1][o] = __float_as_uint(r) & 0xFFFF0000u;
          w[2][o] = __float_as_uint(r - __uint_as_float(w[1][o]));  // at most 8 bits are left
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) part[k][2 * t + h] = __builtin_amdgcn_perm(w[k][1], w[k][0], 0x07060302u);
      }
    attn_bf16x8 pop[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) __builtin_memcpy(&pop[k], &part[k][0], 16);
#pragma unroll
    for (int e = 0; e < EV; ++e) {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;  // element e of two rows side by side
      uint32_t w[4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          w[2 * t + h] = __builtin_amdgcn_perm(vraw[t][2 * h + 1][e / 2], vraw[t][2 * h][e / 2], sel);
      attn_bf16x8 vop, vop_low;
      __builtin_memcpy(&vop, &w[0], 16);
      if constexpr (kInf) {
#pragma unroll
        for (int x = 0; x < 4; ++x) w[x] = bf16x2_finite_or_zero(w[x]);
      }
      __builtin_memcpy(&vop_low, &w[0], 16);
#pragma unroll
      for (int k = 2; k >= 1; --k) acc_low[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pop[k], vop_low, acc_low[e], 0, 0, 0);
      acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pop[0], vop, acc[e], 0, 0, 0);
    }
  };
  clear();
  for (int64_t t0 = w_beg; t0 < total; t0 += stride) step(t0, std::false_type{});
  // A NaN in the result may come from such an element: the wave goes over its rows again with care.
  // (The sum of the results is NaN where one of them is; infinities of both signs make it one, too.)
  float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < EV; ++e)
#pragma unroll
    for (int v = 0; v < 4; ++v) sum[v] += acc[e][v] + acc_low[e][v];
  bool nan = false;
#pragma unroll
  for (int v = 0; v < 4; ++v) nan |= (4 * kb + v < GH) & (sum[v] != sum[v]);
  if (__builtin_expect(__any(nan), 0)) {
    clear();
    n_next = fetch_rows(w_beg);
    for (int64_t t0 = w_beg; t0 < total; t0 += stride) step(t0, std::true_type{});
  }
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);
  if (lane < GH) {
    gl.m[wave][lane] = m;
    gl.l[wave][lane] = l;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (4 * kb + v < GH) {
#pragma unroll
      for (int e = 0; e < EV; ++e) gl.acc[wave][4 * kb + v][EV * i16 + e] = acc[e][v] + acc_low[e][v];
    }
  group_finish<D, GH, kGroupWaves>(a, u0, split, gl);
}

template <typename T, int D, int GH>
tb_status launch_group(const AttnArgs& a, const AttnLaunch& L, hipStream_t st) {
  const tb_cache_desc& d = *L.desc;
  const dim3 grid(L.plan.nsplit, d.Hkv, d.B);
  if constexpr (std::is_same<T, bf16_t>::value && GH >= 4)
    hipLaunchKernelGGL((attn_group_mfma_kernel<D, GH>), grid, dim3(kGroupWaves * kWave), 0, st, a);
  else
    hipLaunchKernelGGL((attn_group_kernel<T, D, GH>), grid, dim3(kAttnThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

// Non-temporal gathers of lists of up to `rows` rows.  With lists that do not depend on each other the g heads of a group read
// `distinct` rows of N and come back to each of them g * rows / distinct times.  A step that has just selected its lists finds little in the
// last-level cache from 100 MB of different rows on; beyond 1.3 readers a row (1.4 where the rows are far more than that cache)
// the lines are wanted again.  Whole steps in us over copies that no cache holds, plain and non-temporal (D = 128, bf16; B x heads on KV
// heads, listed of N): 4 x 16 on 8, 3277 of 32768 (101 MB) 47.7 and 47.9; 3 x 32 on 8, 2600 of 32768 (111 MB) 51.8 and 47.5; 5 x 16 on
// 8, 3277 of 32768 (126 MB) 58.3 and 55.4; 4 x 32 on 8, 3277 of 32768 (182 MB) 67.7 and 63.8; 4 x 32 on 8, 8192 of 131072 (480 MB) 175
// and 161.  Attention alone: 4 x 32 on 8, 12450 of 65536 (612 MB, 1.33) 104.1 and 102.0, an interval of 8 steps that reuse such lists
// 814 and 800; 4 x 32 on 8, 18350 of 65536 (785 MB, 1.53) 130.8 and 139.3; 16 x 64 on 8, 1638 of 16384 (1.4) 112.6 and 119.
// Sizes do not say whether the heads of a group favour the same rows.  With projected keys of Zipf-scaled magnitude, steps: two heads a
// group (1.28 readers a row instead of 1.06) 5 x 16 on 8, 3277 of 32768 53.1 and 52.4, 4 x 16 on 8, 8192 of 131072 118 and 113; four (1.9
// instead of 1.2) 4 x 32 on 8, 3277 of 32768 57.7 and 58.3, 16 x 32 on 8, 1638 of 16384 96.1 and 98.6, 4 x 32 on 8, 8192 of 131072 152
// and 141: 3% lost at most, where independent lists win 3 to 8%.  Eight lose more (attention alone, with an earlier loop, 4 x 64 on 8,
// 4096 of 131072 56.1 and 63.5), and so do lists in shares: both are read plainly (shares, steps: 7 x 16 on 4, 3277 of 32768 66.8 and
// 62.6, 13 x 8 on 4, 6000 of 40000 108 and 101, but Zipf-scaled 7 x 16 on 4 54.4 and 57.8, 9 x 16 on 4, 4000 of 40000 78.2 and 85.4).
// Lists that are handed in may be those of the step before, whose rows
// that cache still holds unless they are far more than it has room for: intervals of 8 steps that reuse lists of 220 MB 339 and
// 349 us, of 295 MB 405 and 411, of 393 MB 508 and 495, of 430 MB 596 and 565.
bool streams_rows(const AttnLaunch& L) {
  const tb_cache_desc& d = *L.desc;
  const int g = d.Hq / d.Hkv;
  if (L.shared_list || g > 4) return false;
  const ListedRows r = listed_rows(g, static_cast<double>(L.max_count + (L.tail_end - L.tail_begin)), static_cast<double>(d.N));
  const double bytes = static_cast<double>(d.B) * d.Hkv * r.distinct * 2 * d.D * (d.dtype == TB_F32 ? 4 : 2);
  return ((L.fresh_lists && bytes >= 100e6 && r.reuse <= kStreamedReuse) || (bytes >= 375e6 && r.reuse <= 1.4)) && in_device_memory(L.K) &&
         in_device_memory(L.V);
}

template <typename T, int D>
tb_status launch_td(const AttnLaunch& L, hipStream_t st) {
  const tb_cache_desc& d = *L.desc;
  AttnArgs a;
  a.q = L.q;
  a.K = L.K;
  a.V = L.V;
  a.idx = L.idx;
  a.count = L.count;
  a.idx_cap = L.idx_cap;
  a.max_count = L.max_count;
  a.tail_begin = L.tail_begin;
  a.tail_end = L.tail_end;
  a.N = d.N;
  a.k_stride_b = d.k_stride_b;
  a.k_stride_h = d.k_stride_h;
  a.k_stride_n = d.k_stride_n;
  a.v_stride_b = d.v_stride_b;
  a.v_stride_h = d.v_stride_h;
  a.v_stride_n = d.v_stride_n;
  a.sm_scale_log2 = L.sm_scale * kLog2e;
  a.out = L.out;
  a.lse = L.lse;
  a.partials = L.partials;
  a.pairs_off = static_cast<int64_t>(d.B) * d.Hq * L.plan.nsplit * D;
  a.counters = L.counters;
  a.Hq = d.Hq;
  a.Hkv = d.Hkv;
  a.g = d.Hq / d.Hkv;
  a.nsplit = L.plan.nsplit;
  a.Kbuf = L.Kbuf;
  a.Vbuf = L.Vbuf;
  a.buf_cap = L.buf_cap;
  a.new_row = -1;
  if (L.append) {
    const NewRow& r = *L.append;
    const int64_t elt = sizeof(T);
    const int64_t from[2][3] = {{r.src->k_stride_b, r.src->k_stride_h, r.src->k_stride_n}, {r.src->v_stride_b, r.src->v_stride_h, r.src->v_stride_n}};
    const int64_t to[2][3] = {{d.k_stride_b, d.k_stride_h, d.k_stride_n}, {d.v_stride_b, d.v_stride_h, d.v_stride_n}};
    const void* in[2] = {r.K, r.V};
    void* out[2] = {r.Kdst, r.Vdst};
    for (int t = 0; t < 2; ++t) {
      a.new_from[t] = static_cast<const char*>(in[t]) + r.src_row * from[t][2] * elt;
      a.new_to[t] = static_cast<char*>(out[t]) + r.dst_row * to[t][2] * elt;
      a.new_from_b[t] = from[t][0] * elt;
      a.new_from_h[t] = from[t][1] * elt;
      a.new_to_b[t] = to[t][0] * elt;
      a.new_to_h[t] = to[t][1] * elt;
    }
    a.new_row = static_cast<int32_t>(r.dst_row);  // (below 2^30: launch conditions)
  }
  if (L.migrate) {
    const GatherLaunch& m = *L.migrate;
    const int64_t elt = sizeof(T);
    a.idx = m.idx;
    a.idx_cap = m.idx_cap;
    a.max_count = m.max_count;
    a.count = m.count;
    a.src[0] = static_cast<const char*>(m.K);
    a.src[1] = static_cast<const char*>(m.V);
    const int64_t strides[2][3] = {{m.desc->k_stride_b, m.desc->k_stride_h, m.desc->k_stride_n}, {m.desc->v_stride_b, m.desc->v_stride_h, m.desc->v_stride_n}};
    for (int t = 0; t < 2; ++t) {
      a.src_b[t] = strides[t][0] * elt;
      a.src_h[t] = strides[t][1] * elt;
      a.src_n[t] = strides[t][2] * elt;
    }
    a.src_N = m.desc->N;
    a.skip_front = m.skip_front;
    a.skip_back = m.skip_back;
    a.count_out = m.count_out;
  }
  a.shared_list = L.shared_list ? 1 : 0;
  a.n_kv_groups = d.B * d.Hkv;
  // per-XCD placement pays when heads share KV rows and the KV groups spread evenly over the XCDs
  const int64_t heads_per_xcd = (static_cast<int64_t>(a.n_kv_groups) + kXcds - 1) / kXcds * a.g;
  a.xcd_map = attn_on_one_xcd(&d) && heads_per_xcd <= 65535 ? 1 : 0;  // (of a grid's third number)
  if (L.grouped) {  // the plan was made for one workgroup per KV group
    if (a.g == 2) return launch_group<T, D, 2>(a, L, st);
    if (a.g == 4) return launch_group<T, D, 4>(a, L, st);
    if (a.g == 8) return launch_group<T, D, 8>(a, L, st);
    return TB_ERR_UNSUPPORTED;
  }
  dim3 grid(L.plan.nsplit, d.Hq, d.B);
  if (a.xcd_map) grid = dim3(kXcds, a.nsplit, static_cast<unsigned>(heads_per_xcd));
  const bool shares = attn_in_shares(&d) && a.nsplit % kXcds == 0;
  // (per-head buffers share no rows: non-temporal whatever the size; against loads that the caches keep, an interval of 2 x 32 heads,
  // 2816 rows a head, 418 and 407 us, of 4 x 32 heads, 9400 rows 1340 and 1209, of 8 heads, 1000 rows no difference)
  if (L.migrate) {
    // (rows that several heads list are kept in the caches for them, as in the migration on its own)
    const GatherLaunch& m = *L.migrate;
    const double listed = static_cast<double>(m.max_count - m.skip_front - m.skip_back);
    const bool nt = listed_rows(a.g, listed > 1.0 ? listed : 1.0, static_cast<double>(m.desc->N)).reuse <= kStreamedReuse &&
                    in_device_memory(m.K) && in_device_memory(m.V);
    if (shares && nt)
      hipLaunchKernelGGL((attn_kernel<T, D, true, true, true, true>), grid, dim3(kAttnThreads), 0, st, a);
    else if (shares)
      hipLaunchKernelGGL((attn_kernel<T, D, true, true, false, true>), grid, dim3(kAttnThreads), 0, st, a);
    else if (nt)
      hipLaunchKernelGGL((attn_kernel<T, D, true, false, true, true>), grid, dim3(kAttnThreads), 0, st, a);
    else
      hipLaunchKernelGGL((attn_kernel<T, D, true, false, false, true>), grid, dim3(kAttnThreads), 0, st, a);
  } else if (L.Kbuf && shares)
    hipLaunchKernelGGL((attn_kernel<T, D, true, true, true>), grid, dim3(kAttnThreads), 0, st, a);
  else if (L.Kbuf)
    hipLaunchKernelGGL((attn_kernel<T, D, true, false, true>), grid, dim3(kAttnThreads), 0, st, a);
  else if (shares)
    hipLaunchKernelGGL((attn_kernel<T, D, false, true, false>), grid, dim3(kAttnThreads), 0, st, a);
  else if (streams_rows(L))
    hipLaunchKernelGGL((attn_kernel<T, D, false, false, true>), grid, dim3(kAttnThreads), 0, st, a);
  else
    hipLaunchKernelGGL((attn_kernel<T, D, false, false, false>), grid, dim3(kAttnThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace

int attn_tile_rows_per_wg(int dtype, int D) {
  const int elt = dtype == TB_F32 ? 4 : 2;
  const int lpr = D * elt / 16;
  return kAttnWaves * kLoadsPerTile * (kWave / lpr);
}

tb_status launch_attn(const AttnLaunch& L, hipStream_t st) {
  const tb_cache_desc& d = *L.desc;
  if (d.B == 0 || d.Hq == 0) return TB_OK;
  if (d.dtype == TB_F32) {
    if (d.D == 64) return launch_td<float, 64>(L, st);
    if (d.D == 128) return launch_td<float, 128>(L, st);
  } else {
    if (d.D == 64) return launch_td<bf16_t, 64>(L, st);
    if (d.D == 128) return launch_td<bf16_t, 128>(L, st);
  }
  return TB_ERR_UNSUPPORTED;
}

}  // namespace tb
