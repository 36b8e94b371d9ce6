// Migration of the selected K/V rows into per-query-head "important" buffers (the paper's
// physical layout, Sec. 3.3): Kbuf/Vbuf[b,h,i,:] = K/V[b,h/g,idx[b,h,skip_front + i],:] for
// i < count[b,h] - skip_front - skip_back (the entries at the two ends of a list are the sink
// prefix and the local window, which live in buffers of their own).
// A pure copy: LPR = D*sizeof(T)/16 adjacent lanes move one row with a 128-bit load and store
// each; a thread issues the loads of all its rows (K and V) before the first store.
#include "tb_device.h"
#include "tb_internal.h"

namespace tb {
namespace {

constexpr int kGatherThreads = 256;
constexpr int kGatherRowsPerThread = 4;

struct GatherArgs {
  const void* K;
  const void* V;
  const int32_t* idx;
  const int32_t* count;
  int64_t idx_cap, max_count, N;
  int64_t k_stride_b, k_stride_h, k_stride_n;
  int64_t v_stride_b, v_stride_h, v_stride_n;
  void* Kbuf;
  void* Vbuf;
  int64_t buf_cap;
  int32_t Hq, g;
  int32_t skip_front, skip_back;  // list entries left out at the two ends
  int32_t* count_out;             // nullable: receives the number of rows migrated per (b,h)
};

// NT: rows that seldom go to more than one head's buffer are read non-temporally (loads that allocate in the caches pay for
// what they displace there, the buffers that are being written among it).  Intervals with two migrations: 2 x 32 heads, 2816
// of 16384 rows 407 -> 404 us, 2 x 8 heads, fp32, 4300 rows 263 -> 256; 4 x 32 heads on 16, 8000 of 32768 rows (1.5 readers a row) 735 and 754.
template <typename T, int D, bool NT>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(GatherArgs a) {
  constexpr int EPL = Pack16<T>::kElts;
  constexpr int LPR = D / EPL;                  // lanes per row
  constexpr int RPP = kGatherThreads / LPR;     // rows per pass of the workgroup
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x;
  const int sub = tid % LPR, rsub = tid / LPR;
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t u = static_cast<int64_t>(b) * a.Hq + h;
  const int hkv = h / a.g;
  int64_t cnt = a.count[u];
  cnt = cnt < 0 ? 0 : (cnt > a.max_count ? a.max_count : cnt);
  cnt -= a.skip_front + a.skip_back;
  cnt = cnt < 0 ? 0 : cnt;
  if (a.count_out && blockIdx.x == 0 && tid == 0) a.count_out[u] = static_cast<int32_t>(cnt);
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * RPP * kGatherRowsPerThread + rsub;
  if (i0 - rsub >= cnt) return;
  const int32_t* list = a.idx + u * a.idx_cap + a.skip_front;
  const T* kb = static_cast<const T*>(a.K) + b * a.k_stride_b + hkv * a.k_stride_h + sub * EPL;
  const T* vb = static_cast<const T*>(a.V) + b * a.v_stride_b + hkv * a.v_stride_h + sub * EPL;
  T* ko = static_cast<T*>(a.Kbuf) + u * a.buf_cap * D + sub * EPL;
  T* vo = static_cast<T*>(a.Vbuf) + u * a.buf_cap * D + sub * EPL;
  u32x4 kr[kGatherRowsPerThread], vr[kGatherRowsPerThread];
#pragma unroll
  for (int r = 0; r < kGatherRowsPerThread; ++r) {
    const int64_t i = i0 + r * RPP;
    int64_t n = (i < cnt) ? static_cast<int64_t>(list[i]) : 0;
    n = n < 0 ? 0 : (n >= a.N ? a.N - 1 : n);  // stay inside the cache whatever the list holds
    kr[r] = load_128<NT, u32x4>(kb + n * a.k_stride_n);
    vr[r] = load_128<NT, u32x4>(vb + n * a.v_stride_n);
  }
#pragma unroll
  for (int r = 0; r < kGatherRowsPerThread; ++r) {
    const int64_t i = i0 + r * RPP;
    if (i < cnt) {
      *reinterpret_cast<u32x4*>(ko + i * D) = kr[r];
      *reinterpret_cast<u32x4*>(vo + i * D) = vr[r];
    }
  }
}

template <typename T, int D>
tb_status launch_td(const GatherLaunch& L, hipStream_t st) {
  const tb_cache_desc& d = *L.desc;
  GatherArgs a;
  a.K = L.K;
  a.V = L.V;
  a.idx = L.idx;
  a.count = L.count;
  a.idx_cap = L.idx_cap;
  a.max_count = L.max_count;
  a.N = d.N;
  a.k_stride_b = d.k_stride_b;
  a.k_stride_h = d.k_stride_h;
  a.k_stride_n = d.k_stride_n;
  a.v_stride_b = d.v_stride_b;
  a.v_stride_h = d.v_stride_h;
  a.v_stride_n = d.v_stride_n;
  a.Kbuf = L.Kbuf;
  a.Vbuf = L.Vbuf;
  a.buf_cap = L.buf_cap;
  a.Hq = d.Hq;
  a.g = d.Hq / d.Hkv;
  a.skip_front = L.skip_front;
  a.skip_back = L.skip_back;
  a.count_out = L.count_out;
  constexpr int rows_per_wg = kGatherThreads / (D / Pack16<T>::kElts) * kGatherRowsPerThread;
  // (at least one workgroup per list, so that count_out is written for an empty one too)
  const int64_t rows = L.max_count > L.skip_front + L.skip_back ? L.max_count - L.skip_front - L.skip_back : 1;
  dim3 grid(static_cast<unsigned>((rows + rows_per_wg - 1) / rows_per_wg), d.Hq, d.B);
  if (listed_rows(a.g, static_cast<double>(rows), static_cast<double>(d.N)).reuse <= kStreamedReuse && in_device_memory(L.K) &&
      in_device_memory(L.V))
    hipLaunchKernelGGL((gather_kernel<T, D, true>), grid, dim3(kGatherThreads), 0, st, a);
  else
    hipLaunchKernelGGL((gather_kernel<T, D, false>), grid, dim3(kGatherThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

// Arrival of new rows: one 16-byte piece of K and one of V per thread, all KV heads of the batch in one
// launch.  Bound by its launch and one trip to memory (two elementwise copies of one row of 16 heads each: 2 x 3.0 us and the
// gap between them; this: 4.2 us, the row cold; 4.4 with the row found by 64-bit divisions).
struct AppendArgs {
  const char* src[2];
  char* dst[2];
  int64_t src_b[2], src_h[2], src_n[2], dst_b[2], dst_h[2], dst_n[2];  // strides in bytes
  int32_t total, shift;  // 16-byte pieces of all rows; log2 of the pieces per row
};

__global__ __launch_bounds__(kGatherThreads) void append_kernel(AppendArgs a) {
  const int i = blockIdx.x * kGatherThreads + threadIdx.x;
  if (i >= a.total) return;
  const int64_t row = i >> a.shift;
  const int at = (i & ((1 << a.shift) - 1)) * 16;
  const int h = blockIdx.y, b = blockIdx.z;
  uint4 v[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) v[t] = *reinterpret_cast<const uint4*>(a.src[t] + b * a.src_b[t] + h * a.src_h[t] + row * a.src_n[t] + at);
#pragma unroll
  for (int t = 0; t < 2; ++t) *reinterpret_cast<uint4*>(a.dst[t] + b * a.dst_b[t] + h * a.dst_h[t] + row * a.dst_n[t] + at) = v[t];
}

}  // namespace

tb_status launch_gather(const GatherLaunch& L, hipStream_t st) {
  const tb_cache_desc& d = *L.desc;
  if (d.B == 0 || d.Hq == 0 || (L.max_count == 0 && !L.count_out)) return TB_OK;
  if (d.dtype == TB_F32) {
    if (d.D == 64) return launch_td<float, 64>(L, st);
    if (d.D == 128) return launch_td<float, 128>(L, st);
  } else {
    if (d.D == 64) return launch_td<bf16_t, 64>(L, st);
    if (d.D == 128) return launch_td<bf16_t, 128>(L, st);
  }
  return TB_ERR_UNSUPPORTED;
}

tb_status launch_append(const tb_cache_desc& src, const void* K, const void* V, int64_t src_row, const tb_cache_desc& dst, void* Kdst,
                        void* Vdst, int64_t dst_row, int64_t rows, hipStream_t st) {
  if (src.B == 0 || src.Hkv == 0 || rows == 0) return TB_OK;
  const int64_t elt = src.dtype == TB_F32 ? 4 : 2;
  AppendArgs a;
  const int64_t from[2][3] = {{src.k_stride_b, src.k_stride_h, src.k_stride_n}, {src.v_stride_b, src.v_stride_h, src.v_stride_n}};
  const int64_t to[2][3] = {{dst.k_stride_b, dst.k_stride_h, dst.k_stride_n}, {dst.v_stride_b, dst.v_stride_h, dst.v_stride_n}};
  const void* in[2] = {K, V};
  void* out[2] = {Kdst, Vdst};
  for (int t = 0; t < 2; ++t) {
    a.src_b[t] = from[t][0] * elt;
    a.src_h[t] = from[t][1] * elt;
    a.src_n[t] = from[t][2] * elt;
    a.dst_b[t] = to[t][0] * elt;
    a.dst_h[t] = to[t][1] * elt;
    a.dst_n[t] = to[t][2] * elt;
    a.src[t] = static_cast<const char*>(in[t]) + src_row * a.src_n[t];
    a.dst[t] = static_cast<char*>(out[t]) + dst_row * a.dst_n[t];
  }
  const int pieces = static_cast<int>(src.D * elt / 16);  // per row: 8, 16 or 32
  a.shift = 31 - __builtin_clz(pieces);
  a.total = static_cast<int32_t>(rows * pieces);  // (at most 2^20 rows)
  const dim3 grid(static_cast<unsigned>((a.total + kGatherThreads - 1) / kGatherThreads), src.Hkv, src.B);
  const int threads = a.total <= kWave ? kWave : kGatherThreads;
  hipLaunchKernelGGL(append_kernel, grid, dim3(threads), 0, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace tb
