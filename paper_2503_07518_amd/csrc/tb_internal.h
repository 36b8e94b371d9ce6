// Host-side declarations shared by the translation units of libtokenbutler: one launcher per
// kernel family, the workspace layout and the launch plan of the split attention.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "tokenbutler.h"

namespace tb {

constexpr int64_t kSelectMaxN = 1 << 20;
// Arrival counters sit 256 bytes apart so that the device-scope atomics of different heads do
// not queue up on one cache line / memory channel.
constexpr int kCounterStrideWords = 64;

// Workspace layout (byte offsets), fixed by B*Hq so that all operations agree on it:
//   [0, part_off)              uint32 arrival counters, one per (b,h), 256 B apart -- zero between calls
//   [part_off, ...)            fp32 split-attention partials, accumulators [B*Hq][nsplit][D] and
//                              (max, sum) pairs [B*Hq][nsplit][2]; the two-stage
//                              selection of long rows keeps its candidates in the same region
//                              (it has finished before the attention of the same stream starts)
struct WsLayout {
  size_t part_off, total;
};

struct AttnPlan {
  int nsplit;     // workgroups per (b,h): the tiles of its list go round them
  int max_split;  // upper bound of nsplit for any list no longer than the one planned for
  int least;      // splits that a workspace has to have room for
  int multiple;   // of which a smaller workspace leaves a multiple (shares of the list, heads that meet on an XCD)
};

constexpr int kXcds = 8;  // accelerator complex dies of the chip, each with its own L2
// With grouped queries the heads of a KV group are placed on one XCD where the groups spread evenly over the XCDs; elsewhere their
// lists are cut into one share per XCD, if there are enough splits.
inline bool attn_on_one_xcd(const tb_cache_desc* d) {
  const int64_t groups = static_cast<int64_t>(d->B) * d->Hkv;
  return d->Hq > d->Hkv && (groups % kXcds == 0 || groups >= 8 * kXcds);
}
inline bool attn_in_shares(const tb_cache_desc* d) { return d->Hq > d->Hkv && !attn_on_one_xcd(d); }

// `shares`: splits in multiples of the number of XCDs are one share of the list each; one_list: all heads read the same list
AttnPlan attn_plan(int64_t units, int64_t max_rows, int tile_rows_per_wg, bool shares, bool one_list);
// A shared list's KV groups of four heads and more, bf16, are served on the matrix cores.
inline bool attn_group_mfma(const tb_cache_desc* d) { return d->dtype == TB_BF16 && d->Hq >= 4 * d->Hkv; }
AttnPlan attn_group_plan(const tb_cache_desc* d, int64_t max_rows);
bool attn_shared_list_grouped(const tb_cache_desc* d, int64_t max_rows);
WsLayout ws_layout(int64_t units, int D, int nsplit);

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Lists of `rows` of N rows, one for each of the g heads of a KV group, that do not depend on each other: how many different
// rows the group reads, and how often each of them.
struct ListedRows {
  double distinct, reuse;
};
inline ListedRows listed_rows(int g, double rows, double N) {
  const double p = rows < N ? rows / N : 1.0;
  double none = 1.0;  // share of the rows that no head lists
  for (int j = 0; j < g; ++j) none *= 1.0 - p;
  const double distinct = N * (1.0 - none);
  return ListedRows{distinct, distinct > 0.0 ? g * p * N / distinct : 1.0};
}
// Readers a row up to which its line is not kept for the next one (non-temporal loads)
constexpr double kStreamedReuse = 1.3;
// Whether the rows of a cache are in the memory of a GPU: rows of an offloaded one come over the host link, which any second
// reader a row is worth keeping lines for (steps of 4 x 32 heads on 8 over pinned host memory, plain and non-temporal loads: 3277 of
// 32768 rows 3.34 and 3.73 ms, 12288 of 65536 11.1 and 13.7).  Asked at every launch that would read non-temporally, 0.1 us.
bool in_device_memory(const void* p);

struct ScoreLaunch {
  const tb_cache_desc* desc;
  const void* q_imp;
  const void* Kimp;
  float scale;
  float* scores;
  int64_t score_stride;
};
tb_status launch_score(const ScoreLaunch& a, hipStream_t st);

// Long rows are selected in two stages so that several compute units work on a head: the row
// is cut into `pieces` pieces, every piece keeps the candidates that a sample of the row puts
// at or above the k-th largest (stage A, one workgroup per piece), and the final kk are
// selected among the kept ones (stage B, a second kernel).  pieces == 1: one workgroup per row,
// no scratch.
struct SelectPlan {
  int pieces;
  int64_t piece_len;  // scores per piece
  int64_t cap;        // kept keys a piece has room for (a multiple of 4)
  int stage_b_tiles;  // 4096-key tiles of kept keys that stage B holds in registers: 2, 4, 8 or 16
  int piece_waves;    // waves of a stage-A workgroup: 4 or 8
  int piece_tiles;    // 256-key tiles that each of them keeps in registers: 2, 4, 8 or 16
  bool row_sample;    // a kernel before stage A samples the row, once; otherwise every piece does
};
constexpr int kMaxPieces = 256;   // pieces of a row: entries of the second stage's table
constexpr int kRowSample = 8192;  // scores of a row that the kernel before stage A looks at
SelectPlan select_plan(int64_t units, int64_t candidates, int64_t N, int64_t kk);
// The plan of a selection whose first stage is part of the scoring kernel: pieces of whole 256-row blocks with
// room for all of their rows.  pieces == 1: scores and selection are separate.
constexpr int kScoredSample = 2048, kScoredSampleLarge = 8192;  // rows that the kernel before it scores for the bracket
SelectPlan score_select_plan(const tb_cache_desc* d, int64_t candidates, int64_t kk);
// kept (score, position) pairs [units][pieces][cap], then 4 words of header per piece
inline size_t select_scratch_bytes(int64_t units, const SelectPlan& p) {
  return p.pieces > 1 ? static_cast<size_t>(units) * p.pieces * (p.cap * 8 + 16) : 0;
}

struct SelectLaunch {
  int64_t units;
  int64_t N;
  const float* scores;
  int64_t score_stride;
  int32_t kk, lo, hi;
  int32_t* idx;
  int32_t* count;
  int64_t idx_cap;
  void* scratch;         // 16-byte aligned, or NULL
  size_t scratch_bytes;  // below select_scratch_bytes(): one workgroup per row is used instead
};
tb_status launch_select(const SelectLaunch& a, hipStream_t st);
// Scores and selects: a bracket from a sample, then one kernel that stores the scores and keeps what the bracket does not
// rule out, then the selection among the kept (score_select_plan; the scratch has to hold it).
tb_status launch_score_select(const ScoreLaunch& S, const SelectLaunch& L, const SelectPlan& plan, hipStream_t st);
// What the scoring kernel keeps and where: candidates [lo, hi) at or above the cut in the header of a row's first piece.
struct FilterOut {
  uint2* cand;    // [units][pieces][cap] (score bits, position)
  uint32_t* hdr;  // [units][pieces][4]; word 0 receives the number kept, word 3 of piece 0 holds the cut
  int32_t pieces;
  int64_t piece_len, cap;
  int32_t lo, hi;
  int32_t turn;  // pieces by which a KV group begins later than the one before (over all groups at most `pieces`)
};
tb_status launch_score_filter(const ScoreLaunch& S, const FilterOut& f, hipStream_t st);

// A row that reaches the cache with the attention over it: row src_row of src is copied to row dst_row.
struct NewRow {
  const tb_cache_desc* src;
  const void* K;
  const void* V;
  int64_t src_row, dst_row;
  void* Kdst;
  void* Vdst;
};

struct GatherLaunch {
  const tb_cache_desc* desc;
  const void* K;
  const void* V;
  const int32_t* idx;
  const int32_t* count;
  int64_t idx_cap, max_count;
  void* Kbuf;
  void* Vbuf;
  int64_t buf_cap;
  int32_t skip_front = 0, skip_back = 0;  // list entries left out at the two ends
  int32_t* count_out = nullptr;           // receives count - skip_front - skip_back (>= 0) per list
};

struct AttnLaunch {
  const tb_cache_desc* desc;
  const void* q;
  const void* K;
  const void* V;
  const int32_t* idx;
  const int32_t* count;
  int64_t idx_cap, max_count, tail_begin, tail_end;
  float sm_scale;
  float* out;
  float* lse;
  float* partials;
  uint32_t* counters;
  AttnPlan plan;
  // buffered form (Kbuf != NULL): list slot i is row i of the per-query-head buffers
  const void* Kbuf = nullptr;
  const void* Vbuf = nullptr;
  int64_t buf_cap = 0;
  const NewRow* append = nullptr;  // (buffered form)
  const GatherLaunch* migrate = nullptr;  // (buffered form) the rows of these lists come from their cache and are left in the buffers
  // head-less form: idx is [B][idx_cap] and count [B], one list for all heads of a batch element
  bool shared_list = false;
  bool grouped = false;  // shared list served by one workgroup per KV group (plan made for that)
  bool fresh_lists = false;  // the lists have been selected by this call
};

// Scores, selection and attention in one launch (a workgroup per head), for what step_in_one allows.
constexpr int kStepMaxN = 4096;
constexpr int kStepMaxSplits = 4;
bool step_in_one(const tb_cache_desc* d, int64_t rows, int nsplit);
tb_status launch_step(const ScoreLaunch& S, const SelectLaunch& L, const AttnLaunch& A, hipStream_t st);

// Copies the listed rows of K and V into per-query-head buffers [B][Hq][buf_cap][D].
tb_status launch_gather(const GatherLaunch& a, hipStream_t st);
tb_status launch_append(const tb_cache_desc& src, const void* K, const void* V, int64_t src_row, const tb_cache_desc& dst, void* Kdst,
                        void* Vdst, int64_t dst_row, int64_t rows, hipStream_t st);
int attn_tile_rows_per_wg(int dtype, int D);
constexpr int kAttnGroupWaves = 8;    // waves of a workgroup that serves a KV group on the matrix cores
constexpr int kAttnLoadsPerTile = 4;  // K (and V) gathers of a lane per tile
tb_status launch_attn(const AttnLaunch& a, hipStream_t st);

// Query predictor of a producer layer (LN + two-layer MLP), see tb_predict.hip.
struct PredictLaunch {
  int dtype;
  int32_t B, E, hidden, G, Hq, Dimp;
  float eps;
  const void *h, *gamma, *beta, *W1, *b1, *W2, *b2;
  float* z;
  float* xln;
  void* q_imp;
};
tb_status launch_predict(const PredictLaunch& a, hipStream_t st);

tb_status launch_project(const tb_cache_desc* d, const void* K, const void* W, int32_t Hw, void* Kimp,
                         int64_t n_begin, int64_t n_end, hipStream_t st);

tb_status launch_expand(int64_t units, int64_t N, int32_t radius, int32_t mode, const int32_t* idx_in,
                        const int32_t* count_in, int64_t cap_in, int32_t* idx_out, int32_t* count_out,
                        int64_t cap_out, hipStream_t st);

tb_status launch_fill_zero(void* p, size_t bytes, hipStream_t st);
tb_status launch_read_stream(const void* src, size_t bytes, uint32_t* sink, hipStream_t st);

inline tb_status hip_status(hipError_t e) { return e == hipSuccess ? TB_OK : TB_ERR_HIP; }

}  // namespace tb
