// Importance scoring: scores[b,h,n] = scale * <q_imp[b,h,:], K_imp[b,h/g,n,:]>.
//
// Bandwidth-bound stream over the projected-key cache.  A projected row is Dimp*sizeof(T)
// bytes (64 B for the Llama-shaped configs); LPR = row_bytes/16 adjacent lanes each take one
// 128-bit load of a row, so a wave instruction reads 1 KiB of consecutive memory.  Every
// loaded row is used for all g query heads of its KV head (the cache is read once per KV
// head).  Each thread issues all of its loads before consuming any of them; workgroups are
// small (256 threads) so that several of them overlap on a compute unit and the memory
// pipeline never drains between them.
#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

typedef uint32_t nt_u32x4 __attribute__((ext_vector_type(4)));
constexpr int64_t kScoreNtStoreBytes = 16 << 20;  // score arrays from this size on bypass the caches
constexpr int kScoreThreads = 256;
constexpr int kLoadsPerThread = 4;
constexpr int kFilterBlock = kWave * 4;  // rows a step of the scoring kernel that filters: one float4 of scores per lane

struct ScoreArgs {
  const void* q_imp;
  const void* Kimp;
  float* scores;
  int64_t N;
  int64_t ki_stride_b, ki_stride_h, ki_stride_n;
  int64_t score_stride;
  int32_t Hq;
  float scale;
  // Large score arrays are stored non-temporally: the selection then reads them from further
  // away (C3: score + select 47.0 -> 48.8 us), but their write-back no longer competes with the
  // gathers of the attention kernel that follows (C3: 95.5 -> 86.1 us inside the step, the step
  // 142.5 -> 135.0 us).  Small ones stay in the caches for the selection (C2: 34.5 against 35.4 us).
  int32_t nt_store;
};

template <typename T, int DIMP, int G>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(ScoreArgs a) {
  constexpr int EPL = Pack16<T>::kElts;      // elements per lane (one 128-bit load)
  constexpr int LPR = DIMP / EPL;            // lanes per projected row
  constexpr int RPP = kScoreThreads / LPR;   // rows per pass of the workgroup
  constexpr int RW = RPP * kLoadsPerThread;  // rows per workgroup
  static_assert(LPR >= 1 && LPR <= 16 && (LPR & (LPR - 1)) == 0, "row must span 1..16 lanes");

  const int tid = threadIdx.x;
  const int part = tid % LPR;
  const int rsub = tid / LPR;
  const int b = blockIdx.z;
  const int hkv = blockIdx.y;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * RW;

  const T* kbase = static_cast<const T*>(a.Kimp) + b * a.ki_stride_b + hkv * a.ki_stride_h + part * EPL;

  // issue every load of this thread first (kept packed until used)
  typename Pack16<T>::Raw kraw[kLoadsPerThread];
#pragma unroll
  for (int i = 0; i < kLoadsPerThread; ++i) {
    int64_t row = row0 + i * RPP + rsub;
    row = row < a.N ? row : a.N - 1;  // clamp: the result of a clamped row is not stored
    {
      // the projected keys are streamed once per step: a non-temporal load keeps them from
      // displacing the scores (which the selection reads next) in the caches
      const nt_u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4*>(kbase + row * a.ki_stride_n));
      __builtin_memcpy(&kraw[i], &t, 16);
    }
  }

  // this lane's slice of the g importance queries
  float qv[G][EPL];
  const T* qbase = static_cast<const T*>(a.q_imp) + (static_cast<int64_t>(b) * a.Hq + hkv * G) * DIMP + part * EPL;
#pragma unroll
  for (int hh = 0; hh < G; ++hh) Pack16<T>::load(qbase + hh * DIMP, qv[hh]);

  // scores of the workgroup's RW rows for the g heads, staged in LDS so that they leave as
  // full 128-bit stores (1 KiB per wave instruction) instead of 64-byte pieces
  __shared__ float s_out[G][RW];
#pragma unroll
  for (int i = 0; i < kLoadsPerThread; ++i) {
    float kf[EPL];
    Pack16<T>::unpack(kraw[i], kf);
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) s = fmaf(qv[hh][e], kf[e], s);
      s = group_allreduce_sum<LPR>(s) * a.scale;
      if ((hh % LPR) == part) s_out[hh][i * RPP + rsub] = s;
    }
  }
  __syncthreads();
  float* sbase = a.scores + (static_cast<int64_t>(b) * a.Hq + hkv * G) * a.score_stride + row0;
  constexpr int V4 = RW / 4;  // float4 groups per head
  for (int v = tid; v < G * V4; v += kScoreThreads) {
    const int hh = v / V4, r4 = (v % V4) * 4;
    float* dst = sbase + hh * a.score_stride + r4;
    if (row0 + r4 + 3 < a.N) {
      if (a.nt_store) {
        typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(*reinterpret_cast<const nt_f32x4*>(&s_out[hh][r4]), reinterpret_cast<nt_f32x4*>(dst));
      } else {
        *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(&s_out[hh][r4]);
      }
    } else {
      for (int c = 0; c < 4; ++c)
        if (row0 + r4 + c < a.N) dst[c] = s_out[hh][r4 + c];
    }
  }
}

// ---- bf16 with Dimp = 32 on the matrix cores ----------------------------------------------------
// The g dot products of a projected row are a (rows x 32) x (32 x g) contraction.  On the vector
// ALUs they cost about 85 instructions per wave and 16 rows, and since the workgroups of a compute
// unit wait for their loads together and then compute together, that arithmetic is not hidden
// behind the stream (C2: 2.3 us of issue per compute unit in a kernel of 6.2 us).  One
// v_mfma_f32_16x16x32_bf16 does the same: the A operand of lane (i, kb) = (lane % 16, lane / 16)
// is its 128-bit load of row i, elements 8 kb .. 8 kb + 7 -- so a wave instruction still reads 1 KiB
// of consecutive memory -- and the B operand is the same slice of importance query j = lane % 16
// (zero for j >= g).  Both operands assign their eight elements to the same k, so the sum runs over
// matching elements whatever the order inside the instruction.  Accumulator v of lane (j, kb) is
// (row 4 kb + v, head j).
typedef short mfma_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

template <int G>
__global__ __launch_bounds__(kScoreThreads) void score_mfma_kernel(ScoreArgs a) {
  constexpr int DIMP = 32;
  constexpr int RPP = kScoreThreads / 4;     // rows per pass of the workgroup: 16 per wave
  constexpr int RW = RPP * kLoadsPerThread;  // rows per workgroup
  static_assert(G <= 16, "one MFMA column per query head of the group");
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int i16 = lane & 15, kb = lane >> 4;
  const int b = blockIdx.z;
  const int hkv = blockIdx.y;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * RW;
  const bf16_t* kbase = static_cast<const bf16_t*>(a.Kimp) + b * a.ki_stride_b + hkv * a.ki_stride_h + kb * 8;

  mfma_bf16x8 kraw[kLoadsPerThread];
#pragma unroll
  for (int i = 0; i < kLoadsPerThread; ++i) {
    int64_t row = row0 + i * RPP + wave * 16 + i16;
    row = row < a.N ? row : a.N - 1;  // clamp: the result of a clamped row is not stored
    const nt_u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4*>(kbase + row * a.ki_stride_n));
    __builtin_memcpy(&kraw[i], &t, 16);
  }
  mfma_bf16x8 qop = {0, 0, 0, 0, 0, 0, 0, 0};
  if (i16 < G) {
    const bf16_t* qp = static_cast<const bf16_t*>(a.q_imp) + (static_cast<int64_t>(b) * a.Hq + hkv * G + i16) * DIMP + kb * 8;
    const uint4 t = *reinterpret_cast<const uint4*>(qp);
    __builtin_memcpy(&qop, &t, 16);
  }

  __shared__ __attribute__((aligned(16))) float s_out[G][RW];
#pragma unroll
  for (int i = 0; i < kLoadsPerThread; ++i) {
    mfma_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kraw[i], qop, acc, 0, 0, 0);
    if (i16 < G) {
      const float4 o = make_float4(acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
      *reinterpret_cast<float4*>(&s_out[i16 < G ? i16 : 0][i * RPP + wave * 16 + 4 * kb]) = o;
    }
  }
  __syncthreads();
  float* sbase = a.scores + (static_cast<int64_t>(b) * a.Hq + hkv * G) * a.score_stride + row0;
  constexpr int V4 = RW / 4;  // float4 groups per head
  for (int v = tid; v < G * V4; v += kScoreThreads) {
    const int hh = v / V4, r4 = (v % V4) * 4;
    float* dst = sbase + hh * a.score_stride + r4;
    if (row0 + r4 + 3 < a.N) {
      if (a.nt_store) {
        typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(*reinterpret_cast<const nt_f32x4*>(&s_out[hh][r4]), reinterpret_cast<nt_f32x4*>(dst));
      } else {
        *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(&s_out[hh][r4]);
      }
    } else {
      for (int c = 0; c < 4; ++c)
        if (row0 + r4 + c < a.N) dst[c] = s_out[hh][r4 + c];
    }
  }
}

// ---- scores of long rows, with the first stage of the selection ----------------------------------
// One workgroup per piece of a row (all heads of its KV group): blocks of 256 rows one after the other, the next
// block's loads in flight while the current one is multiplied and its scores go through LDS.  A wave owns a head (or
// two of eight), so the scores at or above the head's cut go from the registers that store them straight to the
// piece's list, in position order, behind the wave's running count: a compare, a mask count and (for a few lanes) an
// 8-byte store per score, which the stream of projected keys hides (without the filter the kernel is no faster).  Bound
// by the stream, which many workgroups looping over their own pieces cut into more places than one block each does:
// 4 x 8 KV heads, 131072 rows, 8 heads each 67.2 us and 62.5 for the scores alone, whose pass by the selection's first
// stage took 34.4; 8 KV heads, 1M rows, 4 heads each 120 and 108, the pass and its bracket 36.
template <typename T, int DIMP, int G>
__global__ __launch_bounds__(kScoreThreads) void score_filter_kernel(ScoreArgs a, FilterOut f) {
  constexpr bool kMfma = std::is_same<T, bf16_t>::value && DIMP == 32;
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int LPR = DIMP / EPL;           // lanes per projected row
  constexpr int RPP = kScoreThreads / LPR;  // rows per pass of the workgroup
  constexpr int NL = kFilterBlock / RPP;    // loads per lane and block
  constexpr int kWaves = kScoreThreads / kWave;
  constexpr int HPW = (G + kWaves - 1) / kWaves;  // heads per wave
  constexpr int kPitch = kFilterBlock + 16;       // (the heads of a wave's stores start in different banks)
  static_assert(!kMfma || LPR == 4, "a wave's 16 rows a pass");
  __shared__ __attribute__((aligned(16))) float s_out[2][G][kPitch];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int b = blockIdx.z;
  const int hkv = blockIdx.y;
  // (every KV group begins at another piece: with scores that favour recent positions the last pieces keep the most, and one
  // compute unit would get those of all groups: 8 KV heads, 1M rows of ascending scores 204 us a step, 168 now)
  const int at = static_cast<int>(blockIdx.x) + (b * static_cast<int>(gridDim.y) + hkv) * f.turn;
  const int piece = at < f.pieces ? at : at - f.pieces;
  const int64_t base = static_cast<int64_t>(piece) * f.piece_len;
  const int rows = static_cast<int>(a.N - base < f.piece_len ? a.N - base : f.piece_len);  // (a piece has rows: pieces = ceil(N / piece_len))
  // lane's place in a pass: on the matrix cores lane (i, kb) = (lane % 16, lane / 16) holds elements 8 kb .. 8 kb + 7 of row i
  const int i16 = lane & 15, kb = lane >> 4;
  const int part = kMfma ? kb : tid % LPR;
  const int rsub = kMfma ? wave * 16 + i16 : tid / LPR;
  const T* kbase = static_cast<const T*>(a.Kimp) + b * a.ki_stride_b + hkv * a.ki_stride_h + base * a.ki_stride_n + part * EPL;

  nt_u32x4 raw[NL];
  auto load = [&](int r0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      int row = r0 + i * RPP + rsub;
      row = row < rows ? row : rows - 1;  // clamp: the result of a clamped row is not used
      raw[i] = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4*>(kbase + row * a.ki_stride_n));
    }
  };
  load(0);

  mfma_bf16x8 qop = {0, 0, 0, 0, 0, 0, 0, 0};
  float qv[kMfma ? 1 : G][EPL];
  const T* qbase = static_cast<const T*>(a.q_imp) + (static_cast<int64_t>(b) * a.Hq + hkv * G) * DIMP + part * EPL;
  if constexpr (kMfma) {
    if (i16 < G) {
      const uint4 t = *reinterpret_cast<const uint4*>(qbase + i16 * DIMP);
      __builtin_memcpy(&qop, &t, 16);
    }
  } else {
#pragma unroll
    for (int hh = 0; hh < G; ++hh) Pack16<T>::load(qbase + hh * DIMP, qv[hh]);
  }

  // the wave's heads: cut, list and running count
  const int64_t u0 = static_cast<int64_t>(b) * a.Hq + hkv * G;
  float f_lo[HPW];
  bool all[HPW];  // a cut at or below the key of -inf keeps every candidate (NaN, whose key is that of -inf, included)
  uint32_t run[HPW];
#pragma unroll
  for (int k = 0; k < HPW; ++k) {
    const int hh = wave + k * kWaves;
    const uint32_t cut = hh < G ? f.hdr[(u0 + hh) * f.pieces * 4 + 3] : 0xFFFFFFFFu;
    all[k] = cut <= kKeyOfMinusInf;
    f_lo[k] = all[k] ? 0.f : score_of_key(cut);
    run[k] = 0;
  }

  for (int r0 = 0, buf = 0; r0 < rows; r0 += kFilterBlock, buf ^= 1) {
    float (&out)[G][kPitch] = s_out[buf];
    nt_u32x4 cur[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) cur[i] = raw[i];
    if (r0 + kFilterBlock < rows) load(r0 + kFilterBlock);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      if constexpr (kMfma) {
        mfma_bf16x8 kop;
        __builtin_memcpy(&kop, &cur[i], 16);
        mfma_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop, qop, acc, 0, 0, 0);
        if (i16 < G)
          *reinterpret_cast<float4*>(&out[i16 < G ? i16 : 0][i * RPP + wave * 16 + 4 * kb]) =
              make_float4(acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
      } else {
        typename Pack16<T>::Raw kr;
        __builtin_memcpy(&kr, &cur[i], 16);
        float kf[EPL];
        Pack16<T>::unpack(kr, kf);
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
          float s = 0.f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) s = fmaf(qv[kMfma ? 0 : hh][e], kf[e], s);
          s = group_allreduce_sum<LPR>(s) * a.scale;
          if ((hh % LPR) == part) out[hh][i * RPP + rsub] = s;
        }
      }
    }
    __syncthreads();  // (the other buffer's readers are done: they are past the barrier before)
#pragma unroll
    for (int k = 0; k < HPW; ++k) {
      const int hh = wave + k * kWaves;
      if (hh >= G) break;  // (scalar)
      const float4 v = *reinterpret_cast<const float4*>(&out[hh][lane * 4]);
      const int r = r0 + lane * 4;
      const int p = static_cast<int>(base) + r;
      float* dst = a.scores + (u0 + hh) * a.score_stride + base + r;
      if (r + 3 < rows) {
        if (a.nt_store) {
          typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
          const nt_f32x4 o = {v.x, v.y, v.z, v.w};
          __builtin_nontemporal_store(o, reinterpret_cast<nt_f32x4*>(dst));
        } else {
          *reinterpret_cast<float4*>(dst) = v;
        }
      } else {
        const float o[4] = {v.x, v.y, v.z, v.w};
        for (int c = 0; c < 4; ++c)
          if (r + c < rows) dst[c] = o[c];
      }
      bool t0 = v.x >= f_lo[k], t1 = v.y >= f_lo[k], t2 = v.z >= f_lo[k], t3 = v.w >= f_lo[k];
      const int blk = static_cast<int>(base) + r0;
      if (all[k] || blk < f.lo || blk + kFilterBlock > f.hi) {  // (scalar; a block past the row's end is past hi)
        const uint32_t d = static_cast<uint32_t>(p - f.lo), n = static_cast<uint32_t>(f.hi - f.lo);
        t0 = (t0 || all[k]) && d < n;
        t1 = (t1 || all[k]) && d + 1u < n;
        t2 = (t2 || all[k]) && d + 2u < n;
        t3 = (t3 || all[k]) && d + 3u < n;
      }
      const unsigned long long m0 = ballot64(t0), m1 = ballot64(t1), m2 = ballot64(t2), m3 = ballot64(t3);
      uint2* w = f.cand + ((u0 + hh) * f.pieces + piece) * f.cap + run[k] + mbcnt64(m3, mbcnt64(m2, mbcnt64(m1, mbcnt64(m0, 0u))));
      if (t0) *w++ = make_uint2(__float_as_uint(v.x), static_cast<uint32_t>(p));
      if (t1) *w++ = make_uint2(__float_as_uint(v.y), static_cast<uint32_t>(p + 1));
      if (t2) *w++ = make_uint2(__float_as_uint(v.z), static_cast<uint32_t>(p + 2));
      if (t3) *w = make_uint2(__float_as_uint(v.w), static_cast<uint32_t>(p + 3));
      run[k] += popc64(m0) + popc64(m1) + popc64(m2) + popc64(m3);
    }
  }
#pragma unroll
  for (int k = 0; k < HPW; ++k) {
    const int hh = wave + k * kWaves;
    if (hh < G && lane == 0) f.hdr[((u0 + hh) * f.pieces + piece) * 4] = run[k];
  }
}

ScoreArgs score_args(const ScoreLaunch& L) {
  const tb_cache_desc& d = *L.desc;
  ScoreArgs a;
  a.q_imp = L.q_imp;
  a.Kimp = L.Kimp;
  a.scores = L.scores;
  a.N = d.N;
  a.ki_stride_b = d.ki_stride_b;
  a.ki_stride_h = d.ki_stride_h;
  a.ki_stride_n = d.ki_stride_n;
  a.score_stride = L.score_stride;
  a.Hq = d.Hq;
  a.scale = L.scale;
  a.nt_store = static_cast<int64_t>(d.B) * d.Hq * d.N * 4 >= kScoreNtStoreBytes ? 1 : 0;
  return a;
}

template <typename T, int DIMP, int G>
tb_status launch_tdg(const ScoreLaunch& L, const FilterOut* f, hipStream_t st) {
  const tb_cache_desc& d = *L.desc;
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int RW = kScoreThreads / (DIMP / EPL) * kLoadsPerThread;
  const ScoreArgs a = score_args(L);
  if (d.N == 0) return TB_OK;
  if (f) {
    if constexpr (DIMP * sizeof(T) <= 64 && DIMP * sizeof(T) <= 32 * G) {  // (score_select_plan's rule)
      hipLaunchKernelGGL((score_filter_kernel<T, DIMP, G>), dim3(f->pieces, d.Hkv, d.B), dim3(kScoreThreads), 0, st, a, *f);
      return hip_status(hipGetLastError());
    }
    return TB_ERR_UNSUPPORTED;
  }
  dim3 grid(static_cast<unsigned>((d.N + RW - 1) / RW), d.Hkv, d.B);
  if constexpr (std::is_same<T, bf16_t>::value && DIMP == 32) {
    static_assert(RW == kScoreThreads / 4 * kLoadsPerThread, "both kernels cut the rows alike");
    hipLaunchKernelGGL((score_mfma_kernel<G>), grid, dim3(kScoreThreads), 0, st, a);
  } else {
    hipLaunchKernelGGL((score_kernel<T, DIMP, G>), grid, dim3(kScoreThreads), 0, st, a);
  }
  return hip_status(hipGetLastError());
}

template <typename T, int DIMP>
tb_status launch_td(const ScoreLaunch& L, const FilterOut* f, hipStream_t st) {
  switch (L.desc->Hq / L.desc->Hkv) {
    case 1: return launch_tdg<T, DIMP, 1>(L, f, st);
    case 2: return launch_tdg<T, DIMP, 2>(L, f, st);
    case 4: return launch_tdg<T, DIMP, 4>(L, f, st);
    case 8: return launch_tdg<T, DIMP, 8>(L, f, st);
    default: return TB_ERR_UNSUPPORTED;
  }
}

template <typename T>
tb_status launch_t(const ScoreLaunch& L, const FilterOut* f, hipStream_t st) {
  switch (L.desc->Dimp) {
    case 16: return launch_td<T, 16>(L, f, st);
    case 32: return launch_td<T, 32>(L, f, st);
    case 64: return launch_td<T, 64>(L, f, st);
    default: return TB_ERR_UNSUPPORTED;
  }
}

}  // namespace

tb_status launch_score(const ScoreLaunch& L, hipStream_t st) {
  return L.desc->dtype == TB_F32 ? launch_t<float>(L, nullptr, st) : launch_t<bf16_t>(L, nullptr, st);
}

tb_status launch_score_filter(const ScoreLaunch& L, const FilterOut& f, hipStream_t st) {
  return L.desc->dtype == TB_F32 ? launch_t<float>(L, &f, st) : launch_t<bf16_t>(L, &f, st);
}

}  // namespace tb
