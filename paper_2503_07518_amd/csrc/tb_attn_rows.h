// The softmax over a wave's rows, and the merges of waves and splits: what the split attention and the kernel that
// takes a whole small step have in common, so that both round alike.
#pragma once

#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

constexpr int kAttnThreads = 256;
constexpr int kAttnWaves = kAttnThreads / kWave;
constexpr int kLoadsPerTile = kAttnLoadsPerTile;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ inline float exp2_safe(float d) { return __builtin_amdgcn_exp2f(d); }

// A slot past the list's end adds nothing, whatever row it has loaded: its V counts as zeros (a weight of 0 is not enough:
// 0 times an infinite element is NaN).  Only a wave's last tile has such slots; the others pay a branch (selects in
// every tile: 32 heads, 3277 of 32768 rows 27.2 -> 27.6 us a step).
template <typename Raw>
__device__ __forceinline__ void clear_past_end(Raw (&vraw)[kLoadsPerTile], const bool (&valid)[kLoadsPerTile]) {
  unsigned long long past = 0;
#pragma unroll
  for (int t = 0; t < kLoadsPerTile; ++t) past |= ballot64(!valid[t]);
  if (past == 0) return;
#pragma unroll
  for (int t = 0; t < kLoadsPerTile; ++t)
    if (!valid[t]) vraw[t].x = vraw[t].y = vraw[t].z = vraw[t].w = 0;
}

// The online softmax of a wave whose lane groups take one row each (lane: EPL elements of it), in the base-2 domain.
template <typename T, int D>
struct RowSoftmax {
  static constexpr int EPL = Pack16<T>::kElts;  // elements per lane
  static constexpr int LPR = D / EPL;           // lanes per row
  float qv[EPL], acc[EPL];
  float m, l;

  __device__ __forceinline__ void init(const T* q, const float sm_scale_log2) {
    Pack16<T>::load(q, qv);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qv[e] *= sm_scale_log2;
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
  }

  // kLoadsPerTile rows of every lane group
  __device__ __forceinline__ void consume(const typename Pack16<T>::Raw (&kraw)[kLoadsPerTile], typename Pack16<T>::Raw (&vraw)[kLoadsPerTile],
                                          const bool (&valid)[kLoadsPerTile]) {
    float sc[kLoadsPerTile];
    float tmax = -INFINITY;
#pragma unroll
    for (int t = 0; t < kLoadsPerTile; ++t) {
      float kf[EPL];
      Pack16<T>::unpack(kraw[t], kf);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) s = fmaf(qv[e], kf[e], s);
      s = group_allreduce_sum<LPR>(s);
      sc[t] = valid[t] ? s : -INFINITY;
      tmax = fmaxf(tmax, sc[t]);
    }
    clear_past_end(vraw, valid);
    const float m_new = fmaxf(m, tmax);
    if (m_new > -INFINITY) {
      const float alpha = exp2_safe(m - m_new);  // m = -inf -> 0
      l *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
#pragma unroll
      for (int t = 0; t < kLoadsPerTile; ++t) {
        const float p = exp2_safe(sc[t] - m_new);  // invalid -> 0
        l += p;
        float vf[EPL];
        Pack16<T>::unpack(vraw[t], vf);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
      }
      m = m_new;
    }
  }

  // the lane groups of the wave: afterwards every one of them holds the wave's result
  __device__ __forceinline__ void merge_groups() {
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1) {
      const float m_o = __shfl_xor(m, off, kWave);
      const float l_o = __shfl_xor(l, off, kWave);
      const float m_n = fmaxf(m, m_o);
      const float wa = (m_n > -INFINITY) ? exp2_safe(m - m_n) : 0.f;
      const float wb = (m_n > -INFINITY) ? exp2_safe(m_o - m_n) : 0.f;
      l = l * wa + l_o * wb;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float a_o = __shfl_xor(acc[e], off, kWave);
        acc[e] = acc[e] * wa + a_o * wb;
      }
      m = m_n;
    }
  }
};

// Merges NW waves' (max, sum, accumulators): element `d` of the output.
template <int D, int NW>
__device__ __forceinline__ void merge_waves(const float (*s_m)[1], const float (*s_l)[1], const float (*s_acc)[1][D], const int d, float& M,
                                            float& L, float& o) {
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w][0]);
  if (M > -INFINITY) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wgt = exp2_safe(s_m[w][0] - M);
      L += s_l[w][0] * wgt;
      o += s_acc[w][0][d] * wgt;
    }
  }
}

// Adds up the splits of GH heads and writes their outputs: the work of the last workgroup to arrive, whose time is
// added to the whole launch.  A quad of outputs per thread (pair(at): (max, sum) of head and split number
// at, quad(at, d): its accumulators from element d), the splits dealt round the J thread groups that cover the
// outputs.  All loads of a thread are in flight together: a chain of device-scope loads would cost
// a memory round trip per split, and such a load is paid per instruction even when its result is not needed,
// so the chunk is sized to the split count.  The order of combination is fixed.  (Threads past the NW waves repeat
// their work.)
template <int D, int GH, int NW, typename Pair, typename Quad>
__device__ __forceinline__ void combine_splits(const int nsplit, float* out, float* lse, float (&s_m)[NW][GH], float (&s_l)[NW][GH],
                                               float (&s_acc)[NW][GH][D], Pair&& pair, Quad&& quad_of) {
  constexpr int kThreads = NW * kWave;
  constexpr int QUADS = GH * D / 4;       // threads that cover the outputs
  constexpr int J = kThreads / QUADS;     // thread groups, each taking every J-th split
  constexpr int ROWS = QUADS < kWave ? NW : J;  // partial sums left for LDS
  static_assert(QUADS <= kThreads && ROWS <= NW, "every output has a thread, the sums fit the waves' LDS");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x % kThreads;
  const int quad = tid % QUADS, j = tid / QUADS;
  const int hh = quad / (D / 4), d = quad % (D / 4) * 4;
  float M = -INFINITY, L = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
  auto add = [&](const float m_o, const float l_o, const float (&o_o)[4]) {
    const float m_n = fmaxf(M, m_o);
    if (m_n > -INFINITY) {
      const float wa = exp2_safe(M - m_n), wb = exp2_safe(m_o - m_n);
      L = L * wa + l_o * wb;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = o[e] * wa + o_o[e] * wb;
      M = m_n;
    }
  };
  auto walk = [&](auto ch_tag) {
    constexpr int CH = decltype(ch_tag)::value;
    for (int s0 = j; s0 < nsplit; s0 += J * CH) {
      u32x4 ov[CH];
      unsigned long long pv[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int sp = s0 + c * J < nsplit ? s0 + c * J : nsplit - 1;
        pv[c] = pair(hh * nsplit + sp);
        ov[c] = quad_of(hh * nsplit + sp, d);
      }
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        // (a repeated last split counts as an empty one: a weight of 0 alone would turn an infinite sum into NaN)
        if (s0 + c * J >= nsplit) {
          pv[c] = __float_as_uint(-INFINITY);
          ov[c] = u32x4{0u, 0u, 0u, 0u};
        }
        const float oc[4] = {__uint_as_float(ov[c].x), __uint_as_float(ov[c].y), __uint_as_float(ov[c].z), __uint_as_float(ov[c].w)};
        add(__uint_as_float(static_cast<uint32_t>(pv[c])), __uint_as_float(static_cast<uint32_t>(pv[c] >> 32)), oc);
      }
    }
  };
  if (nsplit <= J)
    walk(std::integral_constant<int, 1>{});
  else if (nsplit <= 2 * J)
    walk(std::integral_constant<int, 2>{});
  else if (nsplit <= 4 * J)
    walk(std::integral_constant<int, 4>{});
  else
    walk(std::integral_constant<int, 8>{});
#pragma unroll
  for (int off = QUADS; off < kWave; off <<= 1) {
    const float m_o = __shfl_xor(M, off, kWave), l_o = __shfl_xor(L, off, kWave);
    float o_o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o_o[e] = __shfl_xor(o[e], off, kWave);
    add(m_o, l_o, o_o);
  }
  // (the LDS arrays were last read before the partial was published)
  const int row = QUADS < kWave ? tid / kWave : j;
  if (QUADS >= kWave || tid % kWave < QUADS) {
    *reinterpret_cast<float4*>(&s_acc[row][hh][d]) = make_float4(o[0], o[1], o[2], o[3]);
    if (d == 0) {
      s_m[row][hh] = M;
      s_l[row][hh] = L;
    }
  }
  __syncthreads();
#pragma unroll
  for (int e0 = 0; e0 < GH * D; e0 += kThreads) {
    const int e = e0 + tid, eh = e / D, ed = e % D;
    if (e < GH * D) {
      float Mt = -INFINITY, Lt = 0.f, ot = 0.f;
#pragma unroll
      for (int r = 0; r < ROWS; ++r) Mt = fmaxf(Mt, s_m[r][eh]);
      if (Mt > -INFINITY) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          const float wgt = exp2_safe(s_m[r][eh] - Mt);
          Lt += s_l[r][eh] * wgt;
          ot += s_acc[r][eh][ed] * wgt;
        }
      }
      out[e] = (Lt > 0.f) ? ot / Lt : 0.f;
      if (ed == 0 && lse) lse[eh] = (Lt > 0.f) ? Mt * kLn2 + logf(Lt) : -INFINITY;
    }
  }
}

}  // namespace
}  // namespace tb
