// A whole decode step -- scores, selection, attention -- of short rows in one launch: one workgroup per (b, h).
//
// Three kernels of 3 to 5 us with a boundary between each are bound by their launches and first trips to memory, and
// a caller that launches them one by one by its host.  Here the scores stay in LDS for the selection (and are stored on the
// way), the list stays in LDS for the attention.  A head has one compute unit throughout, so this is for
// launches of no more heads than compute units, rows that one pass of the selection's registers holds and lists that one
// workgroup attends to in a few rounds; step_in_one has the rule and what both sides of it measure.
// Scores, lists and outputs are those of the separate kernels, bit for bit: a score is the same sum, and the splits of the
// attention that the separate kernel would give to workgroups of four waves are groups of four waves here.
// Bound by its chain (a trip to memory for the projected keys, the selection's phases, another trip for the rows, the merges):
// 8 heads, 1024 rows, d' = 16, D = 64, fp32 8.8 us a step in a graph of steps (8.9 traced), in three launches 10.8.
#include "tb_attn_rows.h"
#include "tb_select_regs.h"

namespace tb {
namespace {

constexpr int kStepWaves = 16;
constexpr int kStepThreads = kStepWaves * kWave;
static_assert(kStepMaxN == 4 * kStepThreads, "a thread stores four scores of the longest row");
static_assert(kStepMaxN <= kStepWaves * kWaveTile, "the selection holds the longest row in one tile a wave");
static_assert(kStepMaxSplits * kAttnWaves <= kStepWaves, "every split of the attention has its waves");

struct StepArgs {
  SelectArgs sel;
  const void* q_imp;
  const void* Kimp;
  const void* q;
  const void* K;
  const void* V;
  float* scores;
  float* out;
  float* lse;
  int64_t ki_stride_b, ki_stride_h, ki_stride_n;
  int64_t k_stride_b, k_stride_h, k_stride_n;
  int64_t v_stride_b, v_stride_h, v_stride_n;
  float score_scale, sm_scale_log2;
  int32_t Hkv, g, n_groups, nsplit;
};

typedef short step_bf16x8 __attribute__((ext_vector_type(8)));
typedef float step_f32x4 __attribute__((ext_vector_type(4)));

template <int D>
struct StepLds {
  SelLds<kStepWaves> sel;
  __attribute__((aligned(16))) float scores[kStepMaxN];
  int32_t list[kStepMaxN];
  float m[kStepWaves][1], l[kStepWaves][1];
  __attribute__((aligned(16))) float acc[kStepWaves][1][D];
  // the splits' sums, as the separate kernel's workgroups leave them
  unsigned long long pair[kStepMaxSplits];
  __attribute__((aligned(16))) float part[kStepMaxSplits][D];
  float cm[kAttnWaves][1], cl[kAttnWaves][1];
  __attribute__((aligned(16))) float cacc[kAttnWaves][1][D];
};

template <typename T, int D, int DIMP>
__global__ __launch_bounds__(kStepThreads, 4) void step_kernel(StepArgs a) {
  __shared__ StepLds<D> s;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  // the heads of a KV group on one XCD (workgroups go to the eight round-robin): they read the same projected keys
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int kvg = xcd + 8 * (slot / a.g);
  if (kvg >= a.n_groups) return;  // (the launch is padded to a multiple of eight groups)
  const int b = kvg / a.Hkv, hkv = kvg % a.Hkv;
  const int u = kvg * a.g + slot % a.g;  // b*Hq + h
  const int N = static_cast<int>(a.sel.N);

  // ---- scores, as score_kernel and score_mfma_kernel make them
  {
    constexpr bool kMfma = std::is_same<T, bf16_t>::value && DIMP == 32;
    constexpr int EPL = Pack16<T>::kElts;
    constexpr int LPR = DIMP / EPL;           // lanes per projected row
    constexpr int RPP = kStepThreads / LPR;   // rows per pass of the workgroup
    constexpr int BATCH = 8;                  // passes whose loads are in flight together
    static_assert(kStepMaxN % RPP == 0 && (!kMfma || RPP == 16 * kStepWaves), "whole passes stay within the scores' LDS");
    const int i16 = lane & 15, kb = lane >> 4;
    const int part = kMfma ? kb : tid % LPR;
    const int rsub = kMfma ? wave * 16 + i16 : tid / LPR;
    const T* kbase = static_cast<const T*>(a.Kimp) + b * a.ki_stride_b + hkv * a.ki_stride_h + part * EPL;
    const T* qp = static_cast<const T*>(a.q_imp) + static_cast<int64_t>(u) * DIMP + part * EPL;
    step_bf16x8 qop = {0, 0, 0, 0, 0, 0, 0, 0};
    float qv[EPL];
    if constexpr (kMfma) {
      if (i16 == 0) {  // one column
        const uint4 t = *reinterpret_cast<const uint4*>(qp);
        __builtin_memcpy(&qop, &t, 16);
      }
    } else {
      Pack16<T>::load(qp, qv);
    }
    for (int r0 = 0; r0 < N; r0 += BATCH * RPP) {
      typename Pack16<T>::Raw raw[BATCH];
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {
        const int row = r0 + i * RPP + rsub;
        raw[i] = Pack16<T>::load_raw(kbase + (row < N ? row : N - 1) * a.ki_stride_n);  // clamp: no result of such a row is used
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {
        if (r0 + i * RPP >= N) break;  // (scalar; whole passes stay within kStepMaxN)
        if constexpr (kMfma) {
          step_bf16x8 kop;
          __builtin_memcpy(&kop, &raw[i], 16);
          const step_f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop, qop, step_f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          if (i16 == 0)
            *reinterpret_cast<float4*>(&s.scores[r0 + i * RPP + wave * 16 + 4 * kb]) =
                make_float4(acc[0] * a.score_scale, acc[1] * a.score_scale, acc[2] * a.score_scale, acc[3] * a.score_scale);
        } else {
          float kf[EPL], x = 0.f;
          Pack16<T>::unpack(raw[i], kf);
#pragma unroll
          for (int e = 0; e < EPL; ++e) x = fmaf(qv[e], kf[e], x);
          x = group_allreduce_sum<LPR>(x) * a.score_scale;
          if (part == 0) s.scores[r0 + i * RPP + rsub] = x;
        }
      }
    }
  }
  __syncthreads();
  {
    float* dst = a.scores + static_cast<int64_t>(u) * a.sel.score_stride;
    const int n = 4 * tid;  // (a thread's four: kStepMaxN scores)
    if (n + 3 < N) {
      *reinterpret_cast<float4*>(dst + n) = *reinterpret_cast<const float4*>(&s.scores[n]);
    } else {
      for (int c = n; c < N; ++c) dst[c] = s.scores[c];
    }
  }

  // ---- selection
  select_regs<kStepWaves, 1, 3, 2 * kHistBins / kStepWaves>(a.sel, u, nullptr, s.sel, &s.sel.hist[0][0], s.scores, s.list);
  __syncthreads();

  // ---- attention: split w / 4 of nsplit is waves w / 4 * 4 .. + 3
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int LPR = D / EPL;
  constexpr int GPW = kWave / LPR;
  constexpr int TILE = kLoadsPerTile * GPW;
  const int grp = lane / LPR, sub = lane % LPR;
  const int total = a.sel.lo + a.sel.kk + (N - a.sel.hi);
  const char* kbase = reinterpret_cast<const char*>(static_cast<const T*>(a.K) + b * a.k_stride_b + hkv * a.k_stride_h) + sub * 16;
  const char* vbase = reinterpret_cast<const char*>(static_cast<const T*>(a.V) + b * a.v_stride_b + hkv * a.v_stride_h) + sub * 16;
  const uint32_t k_row_bytes = static_cast<uint32_t>(a.k_stride_n * sizeof(T));
  const uint32_t v_row_bytes = static_cast<uint32_t>(a.v_stride_n * sizeof(T));
  RowSoftmax<T, D> rows;
  rows.init(static_cast<const T*>(a.q) + static_cast<int64_t>(u) * D + sub * EPL, a.sm_scale_log2);
  const int stride = a.nsplit * kAttnWaves * TILE;
  for (int t0 = wave < a.nsplit * kAttnWaves ? wave * TILE : total; t0 < total; t0 += stride) {
    typename Pack16<T>::Raw kraw[kLoadsPerTile], vraw[kLoadsPerTile];
    bool valid[kLoadsPerTile];
#pragma unroll
    for (int t = 0; t < kLoadsPerTile; ++t) {
      const int i = t0 + t * GPW + grp;
      valid[t] = i < total;
      const uint32_t row = min(static_cast<uint32_t>(s.list[valid[t] ? i : 0]), static_cast<uint32_t>(N - 1));
      kraw[t] = Pack16<T>::load_raw(kbase + row * k_row_bytes);
      vraw[t] = Pack16<T>::load_raw(vbase + row * v_row_bytes);
    }
    __builtin_amdgcn_sched_barrier(0);  // every gather of the tile is in flight before the first is consumed
    rows.consume(kraw, vraw, valid);
  }
  rows.merge_groups();
  if (grp == 0) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) s.acc[wave][0][sub * EPL + e] = rows.acc[e];
    if (sub == 0) {
      s.m[wave][0] = rows.m;
      s.l[wave][0] = rows.l;
    }
  }
  __syncthreads();
  const int split = tid / kAttnThreads, d = tid % kAttnThreads;
  float M = -INFINITY, L = 0.f, o = 0.f;
  if (split < a.nsplit && d < D)
    merge_waves<D, kAttnWaves>(&s.m[split * kAttnWaves], &s.l[split * kAttnWaves], &s.acc[split * kAttnWaves], d, M, L, o);
  if (a.nsplit == 1) {
    if (tid < D) a.out[static_cast<int64_t>(u) * D + tid] = (L > 0.f) ? o / L : 0.f;
    if (tid == 0 && a.lse) a.lse[u] = (L > 0.f) ? M * kLn2 + logf(L) : -INFINITY;
    return;
  }
  if (split < a.nsplit && d < D) {
    s.part[split][d] = o;
    if (d == 0) s.pair[split] = __float_as_uint(M) | static_cast<unsigned long long>(__float_as_uint(L)) << 32;
  }
  __syncthreads();
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  combine_splits<D, 1, kAttnWaves>(
      a.nsplit, a.out + static_cast<int64_t>(u) * D, a.lse ? a.lse + u : nullptr, s.cm, s.cl, s.cacc, [&](int at) { return s.pair[at]; },
      [&](int at, int e) -> u32x4 { return *reinterpret_cast<const u32x4*>(&s.part[at][e]); });
}

template <typename T, int D>
tb_status launch_td(const StepArgs& a, int Dimp, dim3 grid, hipStream_t st) {
  const dim3 block(kStepThreads);
  if (Dimp == 16)
    hipLaunchKernelGGL((step_kernel<T, D, 16>), grid, block, 0, st, a);
  else if (Dimp == 32)
    hipLaunchKernelGGL((step_kernel<T, D, 32>), grid, block, 0, st, a);
  else if (Dimp == 64)
    hipLaunchKernelGGL((step_kernel<T, D, 64>), grid, block, 0, st, a);
  else
    return TB_ERR_UNSUPPORTED;
  return hip_status(hipGetLastError());
}

}  // namespace

tb_status launch_step(const ScoreLaunch& S, const SelectLaunch& L, const AttnLaunch& A, hipStream_t st) {
  const tb_cache_desc& d = *S.desc;
  StepArgs a;
  a.sel = SelectArgs{};
  a.sel.score_stride = L.score_stride;
  a.sel.N = L.N;
  a.sel.kk = L.kk;
  a.sel.lo = L.lo;
  a.sel.hi = L.hi;
  a.sel.idx = L.idx;
  a.sel.count = L.count;
  a.sel.idx_cap = L.idx_cap;
  a.q_imp = S.q_imp;
  a.Kimp = S.Kimp;
  a.q = A.q;
  a.K = A.K;
  a.V = A.V;
  a.scores = S.scores;
  a.out = A.out;
  a.lse = A.lse;
  a.ki_stride_b = d.ki_stride_b;
  a.ki_stride_h = d.ki_stride_h;
  a.ki_stride_n = d.ki_stride_n;
  a.k_stride_b = d.k_stride_b;
  a.k_stride_h = d.k_stride_h;
  a.k_stride_n = d.k_stride_n;
  a.v_stride_b = d.v_stride_b;
  a.v_stride_h = d.v_stride_h;
  a.v_stride_n = d.v_stride_n;
  a.score_scale = S.scale;
  a.sm_scale_log2 = A.sm_scale * kLog2e;
  a.Hkv = d.Hkv;
  a.g = d.Hq / d.Hkv;
  a.n_groups = d.B * d.Hkv;
  a.nsplit = A.plan.nsplit;
  const dim3 grid(static_cast<unsigned>((a.n_groups + 7) / 8 * 8 * a.g));
  if (d.dtype == TB_F32) return d.D == 64 ? launch_td<float, 64>(a, d.Dimp, grid, st) : launch_td<float, 128>(a, d.Dimp, grid, st);
  return d.D == 64 ? launch_td<bf16_t, 64>(a, d.Dimp, grid, st) : launch_td<bf16_t, 128>(a, d.Dimp, grid, st);
}

}  // namespace tb
