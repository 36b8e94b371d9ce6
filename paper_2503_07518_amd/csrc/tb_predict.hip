// Importance-query prediction of a producer layer: q_imp = f(LN(h)) with f a two-layer MLP
// (Sec. 3.1 "Query prediction"; hidden size 512 in the paper's experiments).  At decode time h is
// one hidden state per sequence.
//
// hidden_kernel:      LN over E (two-pass mean / variance, fp32), W1 x over a slice of the inputs
// hidden_sum_kernel:  z = gelu(sum of the slices + b1)
// output_kernel:      y = W2 z + b2, rounded once to the storage type and scattered to
//                     q_imp[slot][b][head][j]   (row o of W2 is (slot, head, j), slot outermost)
#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

constexpr int kPredThreads = 256;
constexpr int kPredWaves = kPredThreads / kWave;
constexpr int kMaxE = 8192;
constexpr int kMaxHidden = 2048;

struct PredictArgs {
  const void* h;
  const void* gamma;
  const void* beta;
  const void* W1;
  const void* b1;
  const void* W2;
  const void* b2;
  float* z;    // [B][hidden] fp32
  float* xln;  // [B][E] fp32: the first layer's partial sums, then LN(h)
  void* q_imp;
  int32_t B, E, hidden, G, Hq, Dimp;
  float eps;
};

// Sum over the 64 lanes with DPP moves (row shifts, then the row broadcasts); every lane gets it.
__device__ inline float wave_total(float v) {
  constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
  auto dpp = [](float x, auto ctrl, auto row_mask) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                      decltype(row_mask)::value, 0xF, false));
  };
  using std::integral_constant;
  v += dpp(v, integral_constant<int, kRowShr + 1>{}, integral_constant<int, 0xF>{});
  v += dpp(v, integral_constant<int, kRowShr + 2>{}, integral_constant<int, 0xF>{});
  v += dpp(v, integral_constant<int, kRowShr + 4>{}, integral_constant<int, 0xF>{});
  v += dpp(v, integral_constant<int, kRowShr + 8>{}, integral_constant<int, 0xF>{});
  v += dpp(v, integral_constant<int, kRowBcast15>{}, integral_constant<int, 0xA>{});
  v += dpp(v, integral_constant<int, kRowBcast31>{}, integral_constant<int, 0xC>{});
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}

// Workgroup-wide sum (kPredWaves waves); every thread gets it.
__device__ inline float block_sum(float v, float* s_red) {
  const float w = wave_total(v);
  __syncthreads();  // s_red may still be read from the previous reduction
  if (lane_id() == 0) s_red[threadIdx.x / kWave] = w;
  __syncthreads();
  float total = 0.f;
#pragma unroll
  for (int k = 0; k < kPredWaves; ++k) total += s_red[k];
  return total;
}

__device__ inline float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// LayerNorm of hidden state b by one workgroup, written as fp32.  The row stays in registers for
// the two passes.
template <typename T>
__device__ inline void ln_row(const PredictArgs& a, int b) {
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int kMaxChunks = kMaxE / EPL / kPredThreads;
  __shared__ float s_red[kPredWaves];
  const int tid = threadIdx.x;
  const int n_chunks = a.E / EPL;
  const T* row = static_cast<const T*>(a.h) + static_cast<int64_t>(b) * a.E;
  typename Pack16<T>::Raw raw[kMaxChunks], graw[kMaxChunks], braw[kMaxChunks];
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {  // every load first; pieces past the row read piece 0 and are dropped
    const int ch = tid + c * kPredThreads;
    const int off = (ch < n_chunks ? ch : 0) * EPL;
    raw[c] = Pack16<T>::load_raw(row + off);
    graw[c] = Pack16<T>::load_raw(static_cast<const T*>(a.gamma) + off);
    braw[c] = Pack16<T>::load_raw(static_cast<const T*>(a.beta) + off);
  }
  float hv[kMaxChunks][EPL];
  float part = 0.f;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    Pack16<T>::unpack(raw[c], hv[c]);
    if (tid + c * kPredThreads < n_chunks) {
#pragma unroll
      for (int i = 0; i < EPL; ++i) part += hv[c][i];
    }
  }
  const float mean = block_sum(part, s_red) / static_cast<float>(a.E);
  part = 0.f;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    if (tid + c * kPredThreads < n_chunks) {
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        hv[c][i] -= mean;
        part += hv[c][i] * hv[c][i];
      }
    }
  }
  const float rstd = 1.0f / sqrtf(block_sum(part, s_red) / static_cast<float>(a.E) + a.eps);
  float* out = a.xln + static_cast<int64_t>(b) * a.E;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const int ch = tid + c * kPredThreads;
    if (ch < n_chunks) {
      float gm[EPL], bt[EPL];
      Pack16<T>::unpack(graw[c], gm);
      Pack16<T>::unpack(braw[c], bt);
#pragma unroll
      for (int i = 0; i < EPL; i += 4)
        *reinterpret_cast<float4*>(out + ch * EPL + i) =
            make_float4(hv[c][i] * rstd * gm[i] + bt[i], hv[c][i + 1] * rstd * gm[i + 1] + bt[i + 1],
                        hv[c][i + 2] * rstd * gm[i + 2] + bt[i + 2], hv[c][i + 3] * rstd * gm[i + 3] + bt[i + 3]);
    }
  }
}

// ---- both layers on the matrix cores.  They are [B x E] x [E x hidden] and [B x hidden] x
// [hidden x out] products: the batch is the M side of 16 x 16 tiles (rows past B are computed on a
// clamped row and dropped), 16 rows of the weight matrix the N side.  A lane loads 16 bytes of its
// weight row and the same inputs of its sequence's activations; any assignment of inputs to the k
// slots of the instructions is right as long as both operands use the same one.  bf16: the fp32
// activations enter as a sum of three bf16 numbers that together hold all 24 bits (the upper halves
// of x, of the remainder and of what is left then), so every product is exact and only the fp32
// accumulation rounds; fp32: v_mfma_f32_16x16x4_f32 takes weights and activations as they are.
// Relative error of z against 64 bits 1.4e-7 (vector FMA form: 1.8e-7; two bf16 parts: 2.5e-6).
//
// What bounds it is neither bytes (8 MiB of weights at E = 4096, hidden 512, 4096 outputs: 1.2 us at
// the read rate) nor arithmetic but the latency of a few round trips and how many compute units
// take part.  The first layer has only hidden / 16 tiles, so the E inputs are split over workgroups
// as well until about one workgroup per compute unit is there.  Every workgroup takes the
// statistics of its rows itself (one pass over bytes that sit in the L2, against a launch of its
// own); the partial sums wait in the LN(h) buffer, are added in slice order by a small second
// kernel, and the third kernel's first workgroups write LN(h) there beside the output tiles.
// From some hundred sequences on it is the arithmetic that prepares the activations (launch_tiles).
// bf16, E = 4096, hidden 512, 4096 outputs, in a graph of such calls: B = 16 23.8 -> 15.4 us (before: 32
// workgroups that each converted all activations, LN in a launch of its own), B = 6 34.7 -> 12.8 and
// B = 1 11.3 -> 10.5 us (before: vector FMAs); fp32 B = 16 39.4 -> 19.9, B = 1 17.3 -> 13.1 us.
typedef short mfma_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

constexpr int kOutWaves = 4;          // waves of an output-layer workgroup: they split the inputs
constexpr int kFoldElements = 512;    // up to so many hidden activations, or
constexpr int kFoldSums = 4096;       // so many partial sums, the output kernel adds the slices itself
constexpr int kHidTargetWgs = 256;    // one hidden-layer workgroup per compute unit

// acc(n)[0] + ... += x . w[n] over one step, n < NT: 8 inputs of a lane (bf16 weights) or 4 (fp32 weights;
// these are summed in kAccs chains, so that no chain is longer than the bf16 form's).
template <typename T>
struct MfmaStep;

template <>
struct MfmaStep<bf16_t> {
  static constexpr int kInputs = 32;  // inputs that a wave covers: 4 lane groups x 8
  static constexpr int kAccs = 1;
  static constexpr bool kSplit = true;  // activations enter in parts: see sum_of_products()
  template <int NT, typename Acc>
  __device__ static inline void run(const float (&x)[8], const uint4 (&w)[NT], Acc&& acc) {
    uint32_t p[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t part[3][2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float v = x[2 * i + e];
        const uint32_t hi = __float_as_uint(v) & 0xFFFF0000u;
        float r = v - __uint_as_float(hi);  // exact
        r = (r == r) ? r : 0.f;             // an infinite (or NaN) activation is its upper half alone
        const uint32_t mid = __float_as_uint(r) & 0xFFFF0000u;
        part[0][e] = hi;
        part[1][e] = mid;
        part[2][e] = __float_as_uint(r - __uint_as_float(mid));  // at most 8 bits are left: a bf16 number
      }
#pragma unroll
      for (int t = 0; t < 3; ++t) p[t][i] = __builtin_amdgcn_perm(part[t][1], part[t][0], 0x07060302u);
    }
    mfma_bf16x8 xv[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) __builtin_memcpy(&xv[t], &p[t][0], 16);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      mfma_bf16x8 wv;
      __builtin_memcpy(&wv, &w[n], 16);
      mfma_f32x4& sum = acc(n)[0];
#pragma unroll
      for (int t = 2; t >= 0; --t)  // the small parts first
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[t], wv, sum, 0, 0, 0);
    }
  }
};

template <>
struct MfmaStep<float> {
  static constexpr int kInputs = 16;
  static constexpr int kAccs = 4;
  static constexpr bool kSplit = false;
  template <int NT, typename Acc>
  __device__ static inline void run(const float (&x)[4], const float4 (&w)[NT], Acc&& acc) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      mfma_f32x4(&sum)[kAccs] = acc(n);
      sum[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0], w[n].x, sum[0], 0, 0, 0);
      sum[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1], w[n].y, sum[1], 0, 0, 0);
      sum[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2], w[n].z, sum[2], 0, 0, 0);
      sum[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[3], w[n].w, sum[3], 0, 0, 0);
    }
  }
};

template <int NA>
__device__ inline mfma_f32x4 total_of(const mfma_f32x4 (&acc)[NA]) {
  if constexpr (NA == 1) return acc[0];
  else return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// `sum` as the matrix cores have it, or, where that is NaN, the plain chain of multiply-adds: a lower part of an
// activation may be 0, and 0 times an infinite weight is NaN, where the product itself is infinite.
template <typename T, typename X>
__device__ inline float sum_of_products(float sum, const T* w, int k0, int k1, X&& x) {
  if (MfmaStep<T>::kSplit && __builtin_expect(sum != sum, 0)) {
    sum = 0.f;
#pragma nounroll
    for (int k = k0; k < k1; ++k) sum = fmaf(x(k), to_float(w[k]), sum);
  }
  return sum;
}

// Partial sums over the inputs [slice * steps * NW waves * kInputs, ...) of NT * 16 hidden units and
// MT * 16 sequences.  n_slices == 1: the sums are whole and leave as z = gelu(sum + b1); otherwise they go to
// part[slice][b][unit].
template <typename T, int MT, int NT, int NW>
__global__ __launch_bounds__(NW * kWave) void hidden_kernel(PredictArgs a, int n_slices, int steps) {
  using Step = MfmaStep<T>;
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int kHeld = 8;             // pieces of a row that a lane keeps between the two passes of the statistics
  constexpr int CH = MT == 1 ? 4 : 2;  // steps whose loads are in flight together
  __shared__ float s_red[NW][MT][256];
  __shared__ float s_mean[MT * 16], s_rstd[MT * 16];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
  const int r = lane % 16, q = lane / 16;
  const int n0 = blockIdx.x * (16 * NT), slice = blockIdx.y, b0 = blockIdx.z * (16 * MT);
  const T* wrow[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
    wrow[t] = static_cast<const T*>(a.W1) + static_cast<int64_t>(min(n0 + 16 * t + r, a.hidden - 1)) * a.E;
  const T* hrow[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int b = b0 + m * 16 + r;
    hrow[m] = static_cast<const T*>(a.h) + static_cast<int64_t>(b < a.B ? b : a.B - 1) * a.E;
  }
  // the wave's steps lie next to each other: lane (r, q) takes pieces of row r, 64 bytes a step
  const int k_first = (slice * NW + wave) * steps * Step::kInputs + q * EPL;

  typename Pack16<T>::Raw wr[CH][NT], gr[CH], br[CH], hr[CH][MT];
  auto load = [&](int s0) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int k = k_first + (s0 + c) * Step::kInputs;
      const int ks = (s0 + c < steps && k < a.E) ? k : 0;
#pragma unroll
      for (int t = 0; t < NT; ++t) wr[c][t] = Pack16<T>::load_raw(wrow[t] + ks);
      gr[c] = Pack16<T>::load_raw(static_cast<const T*>(a.gamma) + ks);
      br[c] = Pack16<T>::load_raw(static_cast<const T*>(a.beta) + ks);
#pragma unroll
      for (int m = 0; m < MT; ++m) hr[c][m] = Pack16<T>::load_raw(hrow[m] + ks);
    }
  };
  load(0);

  // mean and 1 / standard deviation of the workgroup's rows, one row per wave at a time (two passes;
  // pieces past the first kHeld per lane are read again for the second)
  const int n_pieces = a.E / EPL;
  const int n_held = min(kHeld, (n_pieces + kWave - 1) / kWave);
  for (int row_no = wave; row_no < MT * 16; row_no += NW) {
    if (b0 + row_no >= a.B) break;  // the same for the whole wave
    const T* row = static_cast<const T*>(a.h) + static_cast<int64_t>(b0 + row_no) * a.E;
    // rows lie a power of two apart as a rule: every wave begins elsewhere in its row, so that the
    // waves of the chip do not ask one L2 channel after the other together
    const int rot = row_no % n_held;
    typename Pack16<T>::Raw held[kHeld];
    bool has[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
      const int j = i + rot < n_held ? i + rot : i + rot - n_held;
      const int p = lane + j * kWave;
      has[i] = i < n_held && p < n_pieces;
      held[i] = Pack16<T>::load_raw(row + (has[i] ? p : 0) * EPL);
    }
    float sum = 0.f;
    auto add = [&](const typename Pack16<T>::Raw& raw) {
      float f[EPL];
      Pack16<T>::unpack(raw, f);
#pragma unroll
      for (int e = 0; e < EPL; ++e) sum += f[e];
    };
#pragma unroll
    for (int i = 0; i < kHeld; ++i)
      if (has[i]) add(held[i]);
    for (int p = lane + kHeld * kWave; p < n_pieces; p += kWave) add(Pack16<T>::load_raw(row + p * EPL));
    const float mean = wave_total(sum) / static_cast<float>(a.E);
    float dev = 0.f;
    auto add_dev = [&](const typename Pack16<T>::Raw& raw) {
      float f[EPL];
      Pack16<T>::unpack(raw, f);
#pragma unroll
      for (int e = 0; e < EPL; ++e) dev += (f[e] - mean) * (f[e] - mean);
    };
#pragma unroll
    for (int i = 0; i < kHeld; ++i)
      if (has[i]) add_dev(held[i]);
    for (int p = lane + kHeld * kWave; p < n_pieces; p += kWave) add_dev(Pack16<T>::load_raw(row + p * EPL));
    const float rstd = 1.0f / sqrtf(wave_total(dev) / static_cast<float>(a.E) + a.eps);
    if (lane == 0) {
      s_mean[row_no] = mean;
      s_rstd[row_no] = rstd;
    }
  }
  __syncthreads();

  float mean[MT], rstd[MT];
  mfma_f32x4 acc[NT][MT][Step::kAccs];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int rr = b0 + m * 16 + r < a.B ? m * 16 + r : a.B - 1 - b0;  // (rows past the batch use the last one's)
    mean[m] = s_mean[rr];
    rstd[m] = s_rstd[rr];
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int c = 0; c < Step::kAccs; ++c) acc[t][m][c] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < steps; s0 += CH) {
    if (s0 > 0) load(s0);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      if (s0 + c < steps) {  // the same for the whole wave
        const bool in = k_first + (s0 + c) * Step::kInputs < a.E;  // pieces past the row add nothing
        float gm[EPL], bt[EPL];
        Pack16<T>::unpack(gr[c], gm);
        Pack16<T>::unpack(br[c], bt);
        typename Pack16<T>::Raw w[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          w[t] = wr[c][t];
          if (!in) w[t] = typename Pack16<T>::Raw{};
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          float x[EPL];
          Pack16<T>::unpack(hr[c][m], x);
#pragma unroll
          for (int e = 0; e < EPL; ++e) x[e] = in ? (x[e] - mean[m]) * rstd[m] * gm[e] + bt[e] : 0.f;
          Step::template run<NT>(x, w, [&](int t) -> mfma_f32x4(&)[Step::kAccs] { return acc[t][m]; });
        }
      }
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (nt > 0) __syncthreads();  // the sums of the tile before have been read
#pragma unroll
    for (int m = 0; m < MT; ++m)
      *reinterpret_cast<mfma_f32x4*>(&s_red[wave][m][lane * 4]) = total_of(acc[nt][m]);
    __syncthreads();
    // accumulator v of lane l is (sequence 4 * (l / 16) + v, unit l % 16); the waves are summed in order
    for (int t = tid; t < MT * 256; t += NW * kWave) {
      const int m = t / 256, row = t % 256 / 16, n = n0 + 16 * nt + t % 16;
      const int e = (16 * (row / 4) + t % 16) * 4 + row % 4;
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += s_red[w][m][e];
      const int b = b0 + m * 16 + row;
      if (b < a.B && n < a.hidden) {
        const T* h = static_cast<const T*>(a.h) + static_cast<int64_t>(b) * a.E;
        const int span = NW * steps * Step::kInputs, k0 = slice * span;
        sum = sum_of_products(sum, static_cast<const T*>(a.W1) + static_cast<int64_t>(n) * a.E, k0, min(k0 + span, a.E), [&](int k) {
          return (to_float(h[k]) - s_mean[m * 16 + row]) * s_rstd[m * 16 + row] * to_float(static_cast<const T*>(a.gamma)[k]) +
                 to_float(static_cast<const T*>(a.beta)[k]);
        });
        if (n_slices == 1)
          a.z[static_cast<int64_t>(b) * a.hidden + n] = gelu_erf(sum + to_float(static_cast<const T*>(a.b1)[n]));
        else
          a.xln[(static_cast<int64_t>(slice) * a.B + b) * a.hidden + n] = sum;
      }
    }
  }
}

// Elements i, i + stride, ... of [B][hidden] of the first layer, J of them: the slices in order, S of
// them (8 / J) in flight for every element.
template <int J>
__device__ inline void sum_slices(const PredictArgs& a, int64_t i, int64_t stride, int n_slices, float (&sum)[J]) {
  constexpr int S = 8 / J;
  const int64_t n = static_cast<int64_t>(a.B) * a.hidden;
#pragma unroll
  for (int j = 0; j < J; ++j) sum[j] = 0.f;
  for (int s0 = 0; s0 < n_slices; s0 += S) {
    float v[J][S];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s) v[j][s] = a.xln[(s0 + s < n_slices ? s0 + s : s0) * n + (i + j * stride < n ? i + j * stride : i)];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int s = 0; s < S; ++s) sum[j] += s0 + s < n_slices ? v[j][s] : 0.f;
  }
}

// z = gelu(sum over the slices + b1), one element per thread.
template <typename T>
__global__ __launch_bounds__(kPredThreads) void hidden_sum_kernel(PredictArgs a, int n_slices) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kPredThreads + threadIdx.x;
  if (i >= static_cast<int64_t>(a.B) * a.hidden) return;
  const float bias = to_float(static_cast<const T*>(a.b1)[i % a.hidden]);
  float sum[1];
  sum_slices<1>(a, i, 0, n_slices, sum);
  a.z[i] = gelu_erf(sum[0] + bias);
}

// y[b][o] = W2[o] . z[b] + b2[o] for NT * 16 output rows o and MT * 16 sequences per workgroup, rounded
// to the storage type and scattered to q_imp[slot][b][head][j].  The four waves split the inputs
// (one tile per workgroup: four times the workgroups of one tile per wave).
// FOLD (one or two sequences, several slices): every workgroup sums the first layer's partial sums
// itself, into LDS, instead of a launch of its own that would do it; otherwise workgroups
// ahead of those of the tiles write LN(h), whose buffer held the partial sums until now.
template <typename T, int MT, int NT, bool FOLD>
__global__ __launch_bounds__(kOutWaves * kWave) void output_kernel(PredictArgs a, int n_slices) {
  static_assert(kOutWaves * kWave == kPredThreads, "ln_row and sum_slices run on kPredThreads threads");
  using Step = MfmaStep<T>;
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int CH = FOLD ? 8 : (MT == 1 ? 4 : 2);
  constexpr int kStride = kOutWaves * Step::kInputs;
  typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));  // (z need not be 16-byte aligned)
  __shared__ float s_red[kOutWaves][MT][256];
  __shared__ float s_z[FOLD ? kFoldSums / 2 : 4];  // (at least two partial sums per activation)
  int tile = blockIdx.x, group = blockIdx.y;
  if constexpr (!FOLD) {  // LN(h): one group of sequences: by the first workgroups of its row, more: by rows of workgroups ahead of theirs
    const int ahead = a.B <= 16 * MT ? 0 : (a.B + static_cast<int>(gridDim.x) - 1) / static_cast<int>(gridDim.x);
    const int b = group * static_cast<int>(gridDim.x) + tile;
    if (ahead == 0 ? tile < a.B : group < ahead) {
      if (b < a.B) ln_row<T>(a, b);
      return;
    }
    if (ahead == 0) tile -= a.B;
    group -= ahead;
  }
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
  const int r = lane % 16, q = lane / 16;
  const int n_out = a.G * a.Hq * a.Dimp;
  const int n0 = tile * (16 * NT), b0 = group * (16 * MT);
  if (n0 >= n_out) return;
  const T* wrow[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
    wrow[t] = static_cast<const T*>(a.W2) + static_cast<int64_t>(min(n0 + 16 * t + r, n_out - 1)) * a.hidden;
  typename Pack16<T>::Raw wr[CH][NT];
  auto load_w = [&](int k0) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int k = k0 + c * kStride + q * EPL;
#pragma unroll
      for (int t = 0; t < NT; ++t) wr[c][t] = Pack16<T>::load_raw(wrow[t] + (k < a.hidden ? k : 0));
    }
  };
  load_w(wave * Step::kInputs);
  float bias[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) bias[t] = to_float(static_cast<const T*>(a.b2)[min(n0 + 16 * t + tid % 16, n_out - 1)]);
  if constexpr (FOLD) {
    auto fold = [&](auto per_thread) {
      constexpr int J = decltype(per_thread)::value;
      const int n = a.B * a.hidden;
      for (int i = tid; i < n; i += J * kPredThreads) {
        float b1[J], sum[J];
#pragma unroll
        for (int j = 0; j < J; ++j) b1[j] = to_float(static_cast<const T*>(a.b1)[(i + j * kPredThreads) % a.hidden]);
        sum_slices<J>(a, i, kPredThreads, n_slices, sum);
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int at = i + j * kPredThreads;
          if (at < n) {
            const float z = gelu_erf(sum[j] + b1[j]);
            s_z[at] = z;
            if (tile == 0) a.z[at] = z;
          }
        }
      }
    };
    if (n_slices <= 2)
      fold(std::integral_constant<int, 4>{});
    else if (n_slices <= 4)
      fold(std::integral_constant<int, 2>{});
    else
      fold(std::integral_constant<int, 1>{});
    __syncthreads();
  }
  const float* xrow[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int b = b0 + m * 16 + r;
    xrow[m] = (FOLD ? s_z : a.z) + static_cast<int64_t>(b < a.B ? b : a.B - 1) * a.hidden;
  }
  mfma_f32x4 acc[NT][MT][Step::kAccs];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int c = 0; c < Step::kAccs; ++c) acc[t][m][c] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = wave * Step::kInputs; k0 < a.hidden; k0 += CH * kStride) {
    float x[CH][MT][EPL];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int k = k0 + c * kStride + q * EPL;
      const int ks = k < a.hidden ? k : 0;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int e = 0; e < EPL; e += 4) {
          const f32x4_u v = *reinterpret_cast<const f32x4_u*>(xrow[m] + ks + e);
#pragma unroll
          for (int i = 0; i < 4; ++i) x[c][m][e + i] = v[i];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int kc = k0 + c * kStride;
      if (kc < a.hidden) {  // the same for the whole wave
        const bool in = kc + q * EPL < a.hidden;  // pieces past the row add nothing
        typename Pack16<T>::Raw w[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          w[t] = wr[c][t];
          if (!in) w[t] = typename Pack16<T>::Raw{};
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
#pragma unroll
          for (int e = 0; e < EPL; ++e) x[c][m][e] = in ? x[c][m][e] : 0.f;
          Step::template run<NT>(x[c][m], w, [&](int t) -> mfma_f32x4(&)[Step::kAccs] { return acc[t][m]; });
        }
      }
    }
    if (k0 + CH * kStride < a.hidden) load_w(k0 + CH * kStride);
  }
  const int per_slot = a.Hq * a.Dimp;
  const int row = tid / 16;
  const int e = (16 * (row / 4) + tid % 16) * 4 + row % 4;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (nt > 0) __syncthreads();  // the sums of the tile before have been read
#pragma unroll
    for (int m = 0; m < MT; ++m)
      *reinterpret_cast<mfma_f32x4*>(&s_red[wave][m][lane * 4]) = total_of(acc[nt][m]);
    __syncthreads();
    const int o_mine = n0 + 16 * nt + tid % 16;
    const int slot = o_mine / per_slot, rest = o_mine % per_slot;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kOutWaves; ++w) sum += s_red[w][m][e];
      const int b = b0 + m * 16 + row;
      if (b < a.B && o_mine < n_out) {
        const float* z = (FOLD ? s_z : a.z) + static_cast<int64_t>(b) * a.hidden;
        sum = sum_of_products(sum, static_cast<const T*>(a.W2) + static_cast<int64_t>(o_mine) * a.hidden, 0, a.hidden, [&](int k) { return z[k]; });
        store_elt(static_cast<T*>(a.q_imp) + (static_cast<int64_t>(slot) * a.B + b) * per_slot + rest, sum + bias[nt]);
      }
    }
  }
}

template <typename T, int MT>
tb_status launch_tiles(const PredictArgs& a, hipStream_t st) {
  constexpr int kInputs = MfmaStep<T>::kInputs;
  const int tiles = (a.hidden + 15) / 16, groups = (a.B + 16 * MT - 1) / (16 * MT);
  const int out_tiles = (a.G * a.Hq * a.Dimp + 15) / 16;
  // Batches that fill the chip several times over: up to four tiles of a layer per workgroup, as long as
  // one workgroup per compute unit is left, share the LayerNorm and the splitting of their activations (fp32
  // activations are not split: nothing gained)
  // (bf16, 2048 sequences: E = 4096, hidden 512, 4096 outputs 340 -> 170 us, hidden 128, 128 outputs 71.7 -> 45.8,
  // E = 8192, hidden 1024, 1024 outputs 813 -> 369; 256 sequences of the first 49.5 -> 39.6)
  // (an output workgroup is half as large: twice as many of them).
  auto tiles_of = [&](int n, int wgs) { return !MfmaStep<T>::kSplit || MT == 1 || n * groups < 2 * wgs ? 1 : (n * groups < 4 * wgs ? 2 : 4); };
  const int hidden_nt = tiles_of(tiles, kHidTargetWgs), out_nt = tiles_of(out_tiles, 2 * kHidTargetWgs);
  // One or two sequences with few activations or partial sums: the output kernel adds the slices itself (it has
  // no workgroups that write LN(h) then).  Against a launch of its own for the sums: B = 1, bf16, E = 2048, hidden 520,
  // 128 outputs 10.2 and 11.2 us, E = 4096, hidden 1024 12.0 and 12.6; fp32, E = 2048, hidden 1024 12.7 and 14.2; B = 2, E = 3072,
  // hidden 256 (512 activations, twelve slices) 12.8 and 15.7; B = 2, E = 2048, hidden 512, four
  // slices: no difference in a graph, 12.5 and 15.0 launched one by one.
  auto folds = [&](int n_slices) {
    const int n = a.B * a.hidden;
    return MT == 1 && a.B <= 2 && n_slices > 1 && (n <= kFoldElements || n_slices * n <= kFoldSums);
  };
  // slices of E: as many as give up to one workgroup per compute unit (one more round for a few of them
  // would cost the most: a compute unit holds one; bf16, E = 5120, hidden 640, 5120 outputs, B = 1: 17.4 us with
  // 280 workgroups, 13.7 with 200), while every wave has a step of its own and the partial sums fit the
  // LN(h) buffer
  int waves = 8, steps = 0, slices = 0;
  for (;; waves = 16) {
    const int all_steps = (a.E + waves * kInputs - 1) / (waves * kInputs);
    int want = kHidTargetWgs / (tiles * groups);
    if (want > all_steps) want = all_steps;
    if (a.B <= 2 && want > 16) want = 16;  // (two round trips for their sum; fp32, E = 4096, hidden 128, B = 1: 11.4 us with 32, 10.5)
    if (want > a.E / a.hidden) want = a.E / a.hidden;
    // two slices save less than the launch that sums them costs where a whole tile is 64 KiB of weights
    // at most (measured at B = 1 with that launch: bf16, E = 2048, hidden 1024 11.4 us without slices, 12.0 with
    // two; fp32, twice the bytes, 16.7 and 15.4); the same for two sequences that fold (12.2 and 13.1)
    if (want < 2 || (want == 2 && !(a.B == 1 && folds(2)) && 16 * a.E * sizeof(T) <= 64 * 1024)) want = 1;
    steps = (all_steps + want - 1) / want;
    slices = (all_steps + steps - 1) / steps;
    // 8 waves while their steps are in flight together, more waves otherwise (B = 16: 15.4 against
    // 16.5 us at E = 4096, hidden 512; B = 24: 41.7 against 37.6 us at E = 8192, hidden 1024)
    if (steps <= 4 || waves == 16 || hidden_nt > 1) break;
  }
  auto launch_hidden = [&](auto nt, auto nw) {
    constexpr int NT = decltype(nt)::value, NW = decltype(nw)::value;
    hipLaunchKernelGGL((hidden_kernel<T, MT, NT, NW>), dim3((tiles + NT - 1) / NT, slices, groups), dim3(NW * kWave), 0, st, a, slices, steps);
  };
  auto launch_output = [&](auto nt, auto fold) {
    constexpr int NT = decltype(nt)::value;
    constexpr bool FOLD = decltype(fold)::value;
    // (at least 16 workgroups a row, so that the rows of LN(h) stay a few thousand)
    const int wgs = (out_tiles + NT - 1) / NT, row = groups > 1 && wgs < 16 ? 16 : wgs;
    const dim3 grid(groups > 1 || FOLD ? row : a.B + row, groups > 1 ? groups + (a.B + row - 1) / row : 1);
    hipLaunchKernelGGL((output_kernel<T, MT, NT, FOLD>), grid, dim3(kPredThreads), 0, st, a, slices);
  };
  using std::integral_constant;
  const integral_constant<int, 1> one;
  const integral_constant<int, 8> w8;
  const integral_constant<int, 16> w16;
  if constexpr (MT == 2 && MfmaStep<T>::kSplit) {
    const integral_constant<int, 2> two;
    const integral_constant<int, 4> four;
    if (hidden_nt == 4)
      launch_hidden(four, w8);
    else if (hidden_nt == 2)
      launch_hidden(two, w8);
  }
  if (hidden_nt == 1) {
    if (waves == 8)
      launch_hidden(one, w8);
    else
      launch_hidden(one, w16);
  }
  if (hipGetLastError() != hipSuccess) return TB_ERR_HIP;
  if constexpr (MT == 1) {
    if (folds(slices)) {
      launch_output(one, std::true_type{});
      return hip_status(hipGetLastError());
    }
  }
  if (slices > 1) {
    const int64_t n = static_cast<int64_t>(a.B) * a.hidden;
    const dim3 sgrid(static_cast<unsigned>((n + kPredThreads - 1) / kPredThreads));
    hipLaunchKernelGGL((hidden_sum_kernel<T>), sgrid, dim3(kPredThreads), 0, st, a, slices);
    if (hipGetLastError() != hipSuccess) return TB_ERR_HIP;
  }
  if constexpr (MT == 2 && MfmaStep<T>::kSplit) {
    const integral_constant<int, 2> two;
    const integral_constant<int, 4> four;
    if (out_nt == 4)
      launch_output(four, std::false_type{});
    else if (out_nt == 2)
      launch_output(two, std::false_type{});
  }
  if (out_nt == 1) launch_output(one, std::false_type{});
  return hip_status(hipGetLastError());
}

template <typename T>
tb_status launch_t(const PredictArgs& a, hipStream_t st) {
  // 32 sequences per workgroup read every weight once for two M tiles
  return a.B > 16 ? launch_tiles<T, 2>(a, st) : launch_tiles<T, 1>(a, st);
}

}  // namespace

tb_status launch_predict(const PredictLaunch& L, hipStream_t st) {
  if (L.B == 0) return TB_OK;
  if (L.E > kMaxE || L.hidden > kMaxHidden) return TB_ERR_UNSUPPORTED;
  PredictArgs a;
  a.h = L.h;
  a.gamma = L.gamma;
  a.beta = L.beta;
  a.W1 = L.W1;
  a.b1 = L.b1;
  a.W2 = L.W2;
  a.b2 = L.b2;
  a.z = L.z;
  a.xln = L.xln;
  a.q_imp = L.q_imp;
  a.B = L.B;
  a.E = L.E;
  a.hidden = L.hidden;
  a.G = L.G;
  a.Hq = L.Hq;
  a.Dimp = L.Dimp;
  a.eps = L.eps;
  return L.dtype == TB_F32 ? launch_t<float>(a, st) : launch_t<bf16_t>(a, st);
}

}  // namespace tb
