// Key-cache projection K_imp = K W: rows [n_begin, n_end) of every (b, kv-head).
//
// Two forms.  project_rows_kernel takes up to four rows (the append of a decode step) with one
// wave per row; project_kernel takes everything else -- a window of appended rows, or the whole
// cache after prefill -- on the matrix cores.
#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

struct ProjectArgs {
  const void* K;
  const void* W;
  void* Kimp;
  int64_t n_begin, n_end;
  int64_t k_stride_b, k_stride_h, k_stride_n;
  int64_t ki_stride_b, ki_stride_h, ki_stride_n;
  int32_t per_head_w;
  int32_t tiles_per_wave;  // project_kernel
};

// ---- many rows on the matrix cores.  The projection is a (Dimp x D) x (D x rows) contraction with up to
// 25 flop per byte (bf16, Dimp = 32): bound by the stream of the cache, and the arithmetic has to stay
// out of its way.  16 output columns are the M side of a 16 x 16 tile, 16 cache rows the N side:
// lane (n, kb) = (lane % 16, lane / 16) loads 16 bytes of row n (elements kb * EPL .. of slice c), so the
// cache passes through no LDS; the lane's part of W stays in registers for all tiles of the wave
// (staged once per workgroup through LDS).  Accumulator v of lane (n, kb) and M tile t is column
// col(4 kb + v, t) of row n; the columns are dealt so that a lane's outputs lie side by side and leave
// as 128-bit stores.  fp32 accumulators, one RNE rounding.  The next tile's loads are issued before
// the current tile is multiplied.
//
// Two forms.  From 2048 rows on, bf16 with Dimp = 16 or 32 takes one 16x16x32 product per load and M
// tile.  Everything else (fp32, Dimp = 64, fewer rows) takes v_mfma_f32_16x16x4_f32, whose sum is the chain
// of fused multiply-adds over its four inputs: with the elements in the order of the head dimension
// (a 4 x 4 transposition over the lanes of a row) the results are those of a scalar chain, bit for bit,
// which is what these shapes have always returned.  bf16 with Dimp = 64 would stream at 26 us instead
// of 53 below in the other form, with other roundings of one value in 10^4.
//
// D = 128, 8 x 32768 rows: bf16 Dimp = 32 17.5 -> 15.2 us (5.5 TB/s; before: the cache through LDS into
// 32x32x8 products), Dimp = 16 17.5 -> 14.0; before with vector FMAs out of LDS: Dimp = 64 97 -> 53, fp32
// Dimp = 32 55 -> 41, fp32 Dimp = 64 (24 x 20001 rows) 166 -> 103 us, a window of 8 rows of 32 heads 8.1 -> 4.4 us.
// The fp32 products bound the chain form with Dimp = 64, the stream the others.
typedef short mfma_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // a 128-bit load kept as a plain vector
constexpr int kProjThreads = 256;
constexpr int kProjWaves = kProjThreads / kWave;
constexpr int kProjTileRows = 16;
constexpr int kProjBf16Rows = 2048;  // bf16 products from here on

// 4 x 4 transposition of the registers f[0..3] over the four lanes (n, 0..3): afterwards register r of
// lane (n, kb) is what register kb of lane (n, r) was.
__device__ inline void lane_transpose4(uint32_t (&f)[4]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto x = __builtin_amdgcn_permlane32_swap(f[i], f[i + 2], false, false);
    f[i] = x[0];
    f[i + 2] = x[1];
  }
#pragma unroll
  for (int i = 0; i < 4; i += 2) {
    const auto x = __builtin_amdgcn_permlane16_swap(f[i], f[i + 1], false, false);
    f[i] = x[0];
    f[i + 1] = x[1];
  }
}

// CHAIN: fp32 products in the order of the head dimension (v_mfma_f32_16x16x4_f32, the four lanes of
// a row hold elements 4 s .. 4 s + 3 at step s); otherwise bf16 products.
template <typename T, int D, int DIMP, bool CHAIN>
__global__ __launch_bounds__(kProjThreads) void project_kernel(ProjectArgs a) {
  constexpr bool kF32 = std::is_same<T, float>::value;
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int KC = D / (4 * EPL);  // 128-bit loads per lane and tile
  constexpr int MT = DIMP / 16;
  static_assert(CHAIN || !kF32, "fp32 has the chain only");
  __shared__ __attribute__((aligned(16))) T s_w[D * DIMP];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int i16 = lane & 15, kb = lane >> 4;
  const int b = blockIdx.z, h = blockIdx.y;
  const T* w = static_cast<const T*>(a.W) + (a.per_head_w ? static_cast<int64_t>(h) * D * DIMP : 0);
  const T* kl = static_cast<const T*>(a.K) + b * a.k_stride_b + h * a.k_stride_h + kb * EPL;
  T* ob = static_cast<T*>(a.Kimp) + b * a.ki_stride_b + h * a.ki_stride_h;
  // tile t of the wave: the four waves of the workgroup read 64 adjacent rows at a time
  const int64_t row00 = a.n_begin + (static_cast<int64_t>(blockIdx.x) * a.tiles_per_wave * kProjWaves + wave) * kProjTileRows + i16;
  constexpr int kTileStep = kProjWaves * kProjTileRows;

  using Raw = typename Pack16<T>::Raw;
  u32x4 v[KC];
  auto load = [&](int64_t row) {
    row = row < a.n_end ? row : a.n_end - 1;  // (computed and dropped)
    const T* p = kl + row * a.k_stride_n;
#pragma unroll
    for (int c = 0; c < KC; ++c) v[c] = *reinterpret_cast<const u32x4*>(p + c * 4 * EPL);
  };
  load(row00);
  for (int i = tid; i < D * DIMP / EPL; i += kProjThreads)
    reinterpret_cast<u32x4*>(s_w)[i] = reinterpret_cast<const u32x4*>(w)[i];
  __syncthreads();
  // column of row i of M tile t: bf16 lanes own 4 MT adjacent columns (4 kb + v <-> i), fp32 lanes 4 of every tile
  auto col = [](int i, int t) { return kF32 ? 16 * t + i : (i >> 2) * (4 * MT) + 4 * t + (i & 3); };
  u32x4 wop[CHAIN ? 1 : KC][MT];
  float wst[CHAIN ? D / 4 : 1][MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    if constexpr (CHAIN) {
#pragma unroll
      for (int st = 0; st < D / 4; ++st) wst[st][t] = to_float(s_w[(4 * st + kb) * DIMP + col(i16, t)]);
    } else {
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        T e[EPL];
#pragma unroll
        for (int x = 0; x < EPL; ++x) e[x] = s_w[(c * 4 * EPL + kb * EPL + x) * DIMP + col(i16, t)];
        __builtin_memcpy(&wop[c][t], e, 16);
      }
    }
  }

  for (int tile = 0; tile < a.tiles_per_wave; ++tile) {
    const int64_t row = row00 + static_cast<int64_t>(tile) * kTileStep;
    if (row - i16 >= a.n_end) break;  // the same for the whole wave
    u32x4 k[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) k[c] = v[c];
    if (tile + 1 < a.tiles_per_wave) load(row + kTileStep);  // clamped rows: always in bounds
    mfma_f32x4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      if constexpr (CHAIN) {
        Raw raw;
        __builtin_memcpy(&raw, &k[c], 16);
        float f[EPL];
        Pack16<T>::unpack(raw, f);
#pragma unroll
        for (int g = 0; g < EPL / 4; ++g) {  // elements EPL kb + 4 g .. + 3 of every lane
          uint32_t x[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = __float_as_uint(f[4 * g + i]);
          lane_transpose4(x);
#pragma unroll
          for (int i = 0; i < 4; ++i) f[4 * g + i] = __uint_as_float(x[i]);
        }
        // register i of group g now belongs to step (EPL i + 4 g) / 4 of this slice
#pragma unroll
        for (int st = 0; st < EPL; ++st)
#pragma unroll
          for (int t = 0; t < MT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wst[c * EPL + st][t], f[4 * (st % (EPL / 4)) + st / (EPL / 4)], acc[t], 0, 0, 0);
      } else {
        mfma_bf16x8 kop, wo;
        __builtin_memcpy(&kop, &k[c], 16);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          __builtin_memcpy(&wo, &wop[c][t], 16);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wo, kop, acc[t], 0, 0, 0);
        }
      }
    }
    if (row < a.n_end) {
      T* o = ob + row * a.ki_stride_n;
      if constexpr (kF32) {
#pragma unroll
        for (int t = 0; t < MT; ++t) *reinterpret_cast<mfma_f32x4*>(o + 16 * t + 4 * kb) = acc[t];
      } else {
        uint32_t r[2 * MT];
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int x = 0; x < 2; ++x)
            r[2 * t + x] = f32_to_bf16_rne(acc[t][2 * x]) | (static_cast<uint32_t>(f32_to_bf16_rne(acc[t][2 * x + 1])) << 16);
        T* dst = o + kb * (4 * MT);
        if constexpr (MT == 1) {
          *reinterpret_cast<uint2*>(dst) = make_uint2(r[0], r[1]);
        } else {
#pragma unroll
          for (int x = 0; x < 2 * MT; x += 4) *reinterpret_cast<uint4*>(dst + 2 * x) = make_uint4(r[x], r[x + 1], r[x + 2], r[x + 3]);
        }
      }
    }
  }
}

// ---- a few rows (the append of a decode step): one wave per cache row, no LDS, no barrier.
// Lane l accumulates output column l % DIMP over the slice l / DIMP of the head dimension (W rows
// are read coalesced, the K element is the same for all lanes of a slice); the slices are then
// added across lanes.  The whole chain is two dependent loads deep.
template <typename T, int D, int DIMP>
__global__ __launch_bounds__(kWave) void project_rows_kernel(ProjectArgs a) {
  constexpr int SLICES = kWave / DIMP;  // 4, 2 or 1 lanes per output column
  constexpr int DS = D / SLICES;        // head-dimension elements per slice
  const int lane = threadIdx.x;
  const int col = lane % DIMP, slice = lane / DIMP;
  const int b = blockIdx.z, h = blockIdx.y;
  const int64_t row = a.n_begin + blockIdx.x;
  const T* w = static_cast<const T*>(a.W) + (a.per_head_w ? static_cast<int64_t>(h) * D * DIMP : 0) +
               static_cast<int64_t>(slice) * DS * DIMP + col;
  const T* k = static_cast<const T*>(a.K) + b * a.k_stride_b + h * a.k_stride_h + row * a.k_stride_n + slice * DS;
  float acc = 0.f;
#pragma unroll 16
  for (int d = 0; d < DS; ++d) acc = fmaf(to_float(k[d]), to_float(w[static_cast<int64_t>(d) * DIMP]), acc);
#pragma unroll
  for (int off = DIMP; off < kWave; off <<= 1) acc += __shfl_xor(acc, off, kWave);
  if (slice == 0) {
    T* o = static_cast<T*>(a.Kimp) + b * a.ki_stride_b + h * a.ki_stride_h + row * a.ki_stride_n + col;
    store_elt(o, acc);
  }
}

template <typename T, int D, int DIMP>
tb_status launch_tdd(const tb_cache_desc& d, ProjectArgs a, hipStream_t st) {
  const int64_t rows = a.n_end - a.n_begin;
  if (rows <= 4) {
    dim3 grid(static_cast<unsigned>(rows), d.Hkv, d.B);
    hipLaunchKernelGGL((project_rows_kernel<T, D, DIMP>), grid, dim3(kWave), 0, st, a);
    return hip_status(hipGetLastError());
  }
  auto wgs = [&](int tiles) {
    const int64_t per_wg = static_cast<int64_t>(kProjWaves) * kProjTileRows * tiles;
    return (rows + per_wg - 1) / per_wg;
  };
  // Tiles of a wave: the more, the less of its time goes into W, the fewer workgroups share the
  // stream.  bf16, D = 128, Dimp = 32: 8 x 32768 rows 15.2 us with 2 tiles, 15.8 with 4, 17.7 with 1; 16 x 4096
  // rows 7.1 with 2, 7.9 with 1; 128 x 16384 rows 125 with 4, 132 with 8; D = 64, 16 x 50000 rows 31.3 with 2,
  // 32.8 with 4.
  const int64_t heads = static_cast<int64_t>(d.Hkv) * d.B;
  const int tiles = wgs(4) * heads >= 4096 ? 4 : (wgs(2) * heads >= 512 ? 2 : 1);
  a.tiles_per_wave = tiles;
  const dim3 grid(static_cast<unsigned>(wgs(tiles)), d.Hkv, d.B);
  if constexpr (std::is_same<T, bf16_t>::value && DIMP <= 32) {
    if (rows >= kProjBf16Rows) {
      hipLaunchKernelGGL((project_kernel<T, D, DIMP, false>), grid, dim3(kProjThreads), 0, st, a);
      return hip_status(hipGetLastError());
    }
  }
  hipLaunchKernelGGL((project_kernel<T, D, DIMP, true>), grid, dim3(kProjThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

template <typename T, int D>
tb_status launch_td(const tb_cache_desc& d, const ProjectArgs& a, hipStream_t st) {
  switch (d.Dimp) {
    case 16: return launch_tdd<T, D, 16>(d, a, st);
    case 32: return launch_tdd<T, D, 32>(d, a, st);
    case 64: return launch_tdd<T, D, 64>(d, a, st);
    default: return TB_ERR_UNSUPPORTED;
  }
}

template <typename T>
tb_status launch_t(const tb_cache_desc& d, const ProjectArgs& a, hipStream_t st) {
  switch (d.D) {
    case 64: return launch_td<T, 64>(d, a, st);
    case 128: return launch_td<T, 128>(d, a, st);
    default: return TB_ERR_UNSUPPORTED;
  }
}

}  // namespace

tb_status launch_project(const tb_cache_desc* d, const void* K, const void* W, int32_t Hw, void* Kimp,
                         int64_t n_begin, int64_t n_end, hipStream_t st) {
  if (n_end <= n_begin || d->B == 0 || d->Hkv == 0) return TB_OK;
  ProjectArgs a;
  a.K = K;
  a.W = W;
  a.Kimp = Kimp;
  a.n_begin = n_begin;
  a.n_end = n_end;
  a.k_stride_b = d->k_stride_b;
  a.k_stride_h = d->k_stride_h;
  a.k_stride_n = d->k_stride_n;
  a.ki_stride_b = d->ki_stride_b;
  a.ki_stride_h = d->ki_stride_h;
  a.ki_stride_n = d->ki_stride_n;
  a.per_head_w = (Hw != 1) ? 1 : 0;
  a.tiles_per_wave = 1;
  return d->dtype == TB_F32 ? launch_t<float>(*d, a, st) : launch_t<bf16_t>(*d, a, st);
}

}  // namespace tb
