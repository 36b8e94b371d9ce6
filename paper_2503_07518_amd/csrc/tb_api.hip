// C ABI of libtokenbutler: argument validation on the host, workspace layout, launch plans.
// Every entry point only enqueues kernels on the caller's stream.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "tb_internal.h"

namespace tb {

constexpr int64_t kAttnCus = 256;         // compute units
constexpr int64_t kAttnMostWgs = 2560;    // workgroups of a launch whose heads are split
constexpr int64_t kAttnGroupTargetWgs = 256;
// Workgroups that the scoring kernel that filters aims at: several rounds of short ones follow the plain kernel's order
// through the cache (4 x 8 KV heads, 131072 rows: 2048 workgroups 72.5 us, 4096 69.7, 8192 67.2, one block each 71.9), but
// every piece costs the second stage some padding.
constexpr int64_t kScoreFilterWgs = 8192;
constexpr int64_t kAttnMinTiles = 2;      // a workgroup is worth its hand-over from two tiles per wave on

// `want` splits or a few less: as many as equal shares of whole granules make
static AttnPlan split_plan(int64_t max_rows, int64_t want, int granule) {
  AttnPlan p{1, static_cast<int>(want), 1, 1};
  int64_t rows = (max_rows + want - 1) / want;
  rows = (rows + granule - 1) / granule * granule;
  p.nsplit = static_cast<int>((max_rows + rows - 1) / rows);
  return p;
}

// Splits per head.  A launch lasts as long as the compute unit with the most workgroups, each costing its rows and a start that
// is worth kStart tiles, so that many splits pay where they even out the last round; every split costs the head's last
// workgroup kHandOver tiles; one workgroup a compute unit does not keep enough gathers in flight (kAlone), and splits in shares, one
// per XCD, read a fifth less from beyond their L2 (kShares; in a launch of one round, which waits for trips more than for bytes,
// kSharesAlone: 8 heads on 2, 1590 rows 9.0 us with 8 splits in shares and 7.8 with 12 without; 16 on 2, 4500 rows 11.2 with 16
// and 10.5 with 24).  bf16, D = 128, us with 512 / units splits rounded up, and now: 3 x 32 heads on 8, 2433 rows 23.6 and 21.1 (6
// splits put a third workgroup on a quarter of the compute units); 5 x 32, 3000 rows 46.1 and 41.2; 14 x 32, 700 rows 27.9 and 24.0;
// 10 x 64, 3000 rows 119 and 108 (two instead of one); 22 x 8 on 1 50.6 and 37.7 (8 instead of 3: shares); fp32 3 x 32, 2400 rows
// 44.5 and 38.4.  The constants were chosen on 179 shapes of 8 to 960 heads, 200 to 12000 rows, both types and sizes of head (the choice
// 0.7% off the best of the numbers tried on average and 11% at most, 512 / units 6.4% on average; 18 of the numbers chosen had not
// been tried, the nearest one stands for them), kSharesAlone on 216 of 4 to 40 heads on 1, 2 or 4 KV heads (0.8% and 7%).  On other
// shapes, drawn at random: 86 of all kinds 1.0% off the best on average, 13% at most (before kSharesAlone), and against 512 / units 3%
// faster on average, 4% slower at most without shares; 60 of few KV groups against 512 / units 9% faster on average, none slower.
// One list for all heads (one_list, for heads that are not on one XCD): split s of head h is on XCD (s + nsplit h) % 8, so that the
// rows of a split go to one XCD's L2 with a multiple of eight splits, to two with another multiple of four, and to all
// eight with an odd number.  Only launches of few workgroups (kFewWgs) take numbers that are no multiple of four.  fp32, 9 x 8 heads
// on 2, D = 64, 5000 rows: 7 splits 35.0 us, 8 19.5; 9 x 16 on 2, 660 rows: 3 19.8, 4 and 8 11.8; bf16, 3 x 32 on 4, 1000 rows: 5 13.7, 4 9.9.
// 162 such shapes 0.9% off the best number tried on average, 15% at most, kFewWgs chosen on them, 108 others 0.9% and 10%
// (512 / units 16% on average and 134% at most, without this rule 3% and 89%).  70 shared lists drawn at random: 12% faster than
// with 512 / units on average, none slower.  Lists of their own keep any number: with this rule 70 shapes took 0.4% longer on average,
// 10% at most, and 31 whose heads favour the same rows (Zipf-scaled projected keys) 1.1% less, 11% at most.
AttnPlan attn_plan(int64_t units, int64_t max_rows, int tile_rows_per_wg, bool shares, bool one_list) {
  constexpr int64_t kFewWgs = 144;
  constexpr double kStart = 1.6, kHandOver = 0.1, kAlone = 1.6, kShares = 0.8, kSharesAlone = 0.91;
  if (max_rows <= 0 || units <= 0) return AttnPlan{1, 1, 1, 1};
  const int64_t most = std::max<int64_t>(1, std::min(max_rows / (kAttnMinTiles * tile_rows_per_wg), kAttnMostWgs / units));
  int64_t want = 1;
  double least = INFINITY;
  auto consider = [&](int64_t n) {
    const int64_t rounds = (units * n + kAttnCus - 1) / kAttnCus;
    double cost = static_cast<double>(rounds) * (static_cast<double>(max_rows) / static_cast<double>(n) + kStart * tile_rows_per_wg);
    if (rounds == 1) cost *= kAlone;
    if (shares && n % kXcds == 0) cost *= rounds == 1 ? kSharesAlone : kShares;
    cost += kHandOver * static_cast<double>(n * tile_rows_per_wg);
    if (cost < least) {
      least = cost;
      want = n;
    }
  };
  const int64_t step = !one_list || most < 2 ? 1 : (most < 4 ? 2 : 4);
  consider(step);
  for (int64_t rounds = 1; rounds * kAttnCus <= kAttnMostWgs; ++rounds) {  // as many splits as these rounds hold
    const int64_t n = std::min(rounds * kAttnCus / units, most);
    if (n > 1 && (step == 1 || units * n <= kFewWgs)) consider(n);
    if (step > 1 && n > step) consider(n / step * step);
    if (shares && n > kXcds) consider(n / kXcds * kXcds);
  }
  const int granule = tile_rows_per_wg / kAttnLoadsPerTile;
  AttnPlan p = split_plan(max_rows, want, granule);
  // (rounded down, it would not be a number that cuts the list into shares: 8 heads on 1, fp32, 8196 rows 15.2 us with 61 splits,
  // 13.6 with 64; 32 on 4, bf16, 3100 rows 13.5 with 15, 12.4 with 16; 8 on 1, 2050 rows 8.1 and 7.9)
  const int64_t multiple = shares && want % kXcds == 0 ? kXcds : (want % step == 0 ? step : 1);
  if (multiple > 1) {
    p.nsplit = static_cast<int>(want);
    p.multiple = static_cast<int>(multiple);
  }
  p.max_split = static_cast<int>(most);
  p.least = std::min(p.nsplit, split_plan(max_rows, std::min(most, (2 * kAttnCus + units - 1) / units), granule).nsplit);
  return p;
}
// A workspace with room for fewer splits than the plan's serves with those, down to `least`: two workgroups a compute unit, or two
// tiles a wave where that is fewer, which is what a workspace made for a list as long as this one always has.
static bool fit_splits(const tb_cache_desc* d, AttnPlan& p, size_t ws_bytes) {
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  const int planned = p.nsplit;
  while (p.nsplit > p.least && ws_bytes < ws_layout(units, d->D, p.nsplit).total) --p.nsplit;
  if (p.nsplit < planned && p.nsplit > p.multiple) p.nsplit -= p.nsplit % p.multiple;
  return ws_bytes >= ws_layout(units, d->D, p.least).total;
}
// (the buffered form is planned alike, so that it adds up in the same order)
static AttnPlan attn_plan(const tb_cache_desc* d, int64_t max_rows, bool shared_list = false) {
  const bool shares = attn_in_shares(d);
  return attn_plan(static_cast<int64_t>(d->B) * d->Hq, max_rows, attn_tile_rows_per_wg(d->dtype, d->D), shares, shares && shared_list);
}

AttnPlan attn_group_plan(const tb_cache_desc* d, int64_t max_rows) {
  const int64_t groups = static_cast<int64_t>(d->B) * d->Hkv;
  if (max_rows <= 0 || groups <= 0 || !attn_group_mfma(d)) return attn_plan(groups, max_rows, attn_tile_rows_per_wg(d->dtype, d->D), false, false);
  // On the matrix cores: 8 waves of 32 rows a step, up to one such workgroup per compute unit (the same
  // rows in flight as two of 4 waves, half the partials to combine).  A compute unit holds one of them at D = 128,
  // so a few more than compute units would take a second round (g = 4, D = 128, 3300 rows, attention alone:
  // 24 groups 18.4 us with 11 splits, 15.9 with 10; 72 groups 37.4 with 4, 27.0 with 3).  More groups than
  // compute units take several rounds anyway: as many splits as make the rounds shortest in all, a round
  // costing its rows and about two steps (304 groups, 3000 rows: 112.5 us with one split, 102.7 with three; 1500
  // rows 53.5 and 52.6).
  const int64_t step = 32 * kAttnGroupWaves, most = max_rows > step ? max_rows / step : 1;
  int64_t want = kAttnGroupTargetWgs / groups, cap = want;
  if (groups > kAttnGroupTargetWgs) {
    auto cost = [&](int64_t n) { return (groups * n + kAttnGroupTargetWgs - 1) / kAttnGroupTargetWgs * (max_rows / n + 2 * step); };
    want = 1;
    cap = 4;
    for (int64_t n = 2; n <= cap && n <= most; ++n)
      if (cost(n) < cost(want)) want = n;
  }
  AttnPlan p = split_plan(max_rows, want < most ? want : most, 4 * kAttnGroupWaves);
  p.max_split = static_cast<int>(cap < most ? cap : most);
  return p;
}

// A shared list with grouped queries: one workgroup per (KV group, split) loads every row once
// for all heads of the group.  That pays when there are enough KV groups to fill the chip with
// few splits each (the last workgroup of a group combines heads x splits partials with
// device-scope loads, about 0.1 us per split); with fewer groups the per-head kernel, whose
// heads share rows through the L2 of their XCD, is faster.  On the matrix cores: 16 groups from 3072 rows on
// (attention alone, per head and grouped, us: 16 groups of four, D = 128: 2500 rows 11.3 and 12.6, 3400 rows 13.6 and
// 13.5, 4200 rows 16.1 and 14.3; 24 groups: 3300 rows 17.5 and 15.9; groups of eight gain from 2000 rows on), the
// narrowest shape from 4096 on (16 groups of four, D = 64: 3300 rows 9.4 and 10.3, 4200 10.7 and 10.9, 6000 12.2 and
// 11.4; from 20 groups on 17.1 and 10.8 at 3300); 8 groups nowhere (score to attention, 3661 rows: 25.0 and 26.8).
bool attn_shared_list_grouped(const tb_cache_desc* d, int64_t max_rows) {
  const int64_t groups = static_cast<int64_t>(d->B) * d->Hkv;
  if (d->Hq <= d->Hkv) return false;
  const int64_t enough = groups < 20 && d->Hq / d->Hkv * d->D <= 256 ? 4096 : 3072;
  return groups >= 32 || (attn_group_mfma(d) && groups >= 16 && max_rows >= enough);
}

// 4096-key tiles of the second stage for the keys that the pieces keep together, give or take: the share of the row above
// the cut (the rank of the threshold in a sample of n_s plus twice the bracket's slack: the cut lies one slack below the
// expected rank, and the other one allows for the sample's own spread), every piece padded to a multiple of 4.
// (32: more than the second stage can hold, it reads them again in every phase.)
static int stage_b_tiles(const SelectPlan& p, int64_t candidates, int64_t kk, double n_s) {
  const double frac = static_cast<double>(kk) / static_cast<double>(candidates);
  const double ks = frac * n_s, slack = 6.0 * sqrt(ks * (1.0 - frac)) + 4.0;
  double kept = (ks + 2.0 * slack) / n_s * static_cast<double>(candidates) + 3.0 * static_cast<double>(p.pieces);
  if (kept > static_cast<double>(p.pieces * p.cap)) kept = static_cast<double>(p.pieces * p.cap);
  const int64_t t4k = (static_cast<int64_t>(kept) + 4095) / 4096;
  return t4k <= 2 ? 2 : (t4k <= 4 ? 4 : (t4k <= 8 ? 8 : (t4k <= 16 ? 16 : 32)));
}
// The larger sample where it saves tiles of a second stage with more than eight.
static void choose_sample(SelectPlan& p, int64_t candidates, int64_t kk, double n_s, double n_large) {
  int tiles = stage_b_tiles(p, candidates, kk, n_s);
  p.row_sample = false;
  if (tiles > 8 && stage_b_tiles(p, candidates, kk, n_large) < tiles) {
    p.row_sample = true;
    tiles = stage_b_tiles(p, candidates, kk, n_large);
  }
  p.stage_b_tiles = tiles < 16 ? tiles : 16;
}

SelectPlan select_plan(int64_t units, int64_t candidates, int64_t N, int64_t kk) {
  SelectPlan p{1, 0, 0, 2, 8, 16, false};
  // worth it when the budget is a small share of the candidates (the kept keys are then a small
  // share of the row as well) and the row is longer than the 65536 scores one workgroup holds in
  // registers (beyond that it would stream the row again in every phase: 44 against 27 us just
  // past 65536); up to 65536 scores two launches cost more than the one-workgroup selection
  if (units <= 0 || kk <= 0 || N <= 65536 || kk * 8 > candidates) return p;
  int waves = 8, tiles = 8;
  auto len_of = [&]() { return static_cast<int64_t>(waves) * 256 * tiles; };
  // few rows (a head-less selection has one per batch element): shorter pieces, so that more
  // compute units take part
  while (units * ((N + len_of() - 1) / len_of()) < 256 && (tiles > 2 || waves > 4)) {
    if (tiles > 2) tiles /= 2; else waves /= 2;
  }
  while ((N + len_of() - 1) / len_of() > kMaxPieces && tiles < 16) tiles *= 2;
  const int64_t len = len_of();
  const int64_t pieces = (N + len - 1) / len;
  if (pieces < 2 || pieces > kMaxPieces) return p;
  p.pieces = static_cast<int>(pieces);
  p.piece_len = len;
  p.piece_waves = waves;
  p.piece_tiles = tiles;
  const int64_t cap = 2 * kk + 4096;                      // the budget, the bracket's slack, a coarse top bin
  p.cap = ((cap < len ? cap : len) + 3) / 4 * 4;
  // A small budget of a very long row is a small rank in a piece's own sample, and the pieces keep
  // several budgets' worth of keys.  Where these would need more than 8 tiles of stage B, one larger
  // sample of the row, taken once, is worth its launch if fewer tiles do then (32 rows of 1M scores, 8192 kept:
  // the selection 73 -> 50 us, stage B 38.8 -> 15.2 of them; 32 rows of 500000, 15625 kept: 53 -> 36); elsewhere it is
  // not (256 rows of 131072: 48 us either way, 32 rows: 2 us slower; 64 rows of 262144, 30840 kept, sixteen tiles
  // either way: 70 -> 72).
  choose_sample(p, candidates, kk, 4.0 * 64 * waves, kRowSample);
  return p;
}

// The first stage inside the scoring kernel pays where a row of the projected cache is short next to the g scores made
// from it: the looped kernel streams that cache at 4.0 TB/s where the plain one reaches 4.3, and a sample of rows is read at
// random by one compute unit, against a pass over the scores that falls away.  Steps in us, separate and together: 32 heads
// on 8, d' = 32 bf16, 131072 rows 51.4 and 46.4, 1M rows 186 and 173; 4 x 64 on 8, 131072 rows 169 and 151; 8 x 16 on 8, 66001 rows
// 86.7 and 82.6; one head a group: d' = 16, 4 x 8, 131072 rows 55.4 and 50.3, d' = 32, 16 x 8, 66001 rows 127 and 132; rows of 128
// bytes: 8 x 8 on 1, 70000 rows 76.4 and 79.5, of 256 bytes: 8 heads, 131072 rows 69.0 and 78.5.
SelectPlan score_select_plan(const tb_cache_desc* d, int64_t candidates, int64_t kk) {
  const int64_t groups = static_cast<int64_t>(d->B) * d->Hkv, N = d->N;
  SelectPlan p = select_plan(static_cast<int64_t>(d->B) * d->Hq, candidates, N, kk);
  if (p.pieces < 2) return p;
  const int row_bytes = d->Dimp * (d->dtype == TB_F32 ? 4 : 2);
  if (row_bytes > 64 || row_bytes > 32 * (d->Hq / d->Hkv)) {
    p.pieces = 1;
    return p;
  }
  int64_t blocks = (groups * N + 256 * kScoreFilterWgs - 1) / (256 * kScoreFilterWgs);  // per piece
  const int64_t fewest = (N + 256 * kMaxPieces - 1) / (256 * kMaxPieces);  // (the table of the second stage)
  if (blocks < fewest) blocks = fewest;
  p.piece_len = blocks * 256;
  p.pieces = static_cast<int>((N + p.piece_len - 1) / p.piece_len);
  p.cap = p.piece_len;
  choose_sample(p, candidates, kk, kScoredSample, kScoredSampleLarge);
  return p;
}

// Scratch for every row of up to N scores and every budget of up to max_count, so that a workspace made for a cache's capacity
// serves it while it fills: fewer rows can be cut into more pieces, or round up to more.  A plan holds between two
// multiples of 2048 rows, of which every piece length is one; with the first stage inside the scoring kernel the pieces together
// are less than a piece longer than the row, and a piece is no longer for fewer rows.
static size_t select_scratch_upto(int64_t units, int64_t N, int64_t max_count) {
  size_t most = 0;
  for (int64_t n = std::min(N, kSelectMaxN); n > 65536; n = (n - 1) / 2048 * 2048)
    most = std::max(most, select_scratch_bytes(units, select_plan(units, n, n, std::min(max_count, n / 8))));
  return most;
}
static size_t score_select_scratch_upto(const tb_cache_desc* d, int64_t max_count) {
  tb_cache_desc longest = *d;
  longest.N = std::min(d->N, kSelectMaxN);
  const SelectPlan p = score_select_plan(&longest, longest.N, std::min(max_count, longest.N / 8));
  return p.pieces > 1 ? static_cast<size_t>(d->B) * d->Hq * ((longest.N + p.piece_len) * 8 + kMaxPieces * 16) : 0;
}

// One launch for a whole step, a workgroup per head, against three: no more heads than compute units, a row that a workgroup
// scores and a list that it attends to in little more than the two launches saved (a compute unit takes about 60 bytes a
// nanosecond).  Separate and in one, us a step in a graph of steps: 8 heads, 1024 rows of d' = 16, 128 kept, D = 64, fp32 10.8 and
// 8.8; D = 128, bf16, d' = 32: 32 heads, 2048 rows, 200 kept (230 KB) 14.4 and 11.7, 4096 rows, 400 kept (460 KB) 15.9 and 15.5, 800
// kept (660 KB) 17.1 and 17.2; 256 heads, 1024 rows, 100 kept 14.7 and 11.6, 4000 rows, 400 kept 23.9 and 20.4; 64 heads, 3000
// rows, 684 kept (540 KB) 18.4 and 18.4; d' = 64, 4096 rows, 600 kept (810 KB) 18.1 and 20.4.  112 heads on 28, 2300 rows of d' = 16, 760
// kept (as many splits as there are waves for since attn_plan evens out the rounds) 23.2 and 16.1.
bool step_in_one(const tb_cache_desc* d, int64_t rows, int nsplit) {
  const int64_t elt = d->dtype == TB_F32 ? 4 : 2;
  return d->N > 0 && d->N <= kStepMaxN && static_cast<int64_t>(d->B) * d->Hq <= 256 && nsplit <= kStepMaxSplits &&
         (d->N * d->Dimp + rows * 2 * d->D) * elt <= 480 * 1024;
}

WsLayout ws_layout(int64_t units, int D, int nsplit) {
  WsLayout w;
  w.part_off = align_up(static_cast<size_t>(units) * kCounterStrideWords * sizeof(uint32_t), 256);
  w.total = w.part_off + align_up(static_cast<size_t>(units) * nsplit * (D + 2) * sizeof(float), 256);
  return w;
}

namespace {

// Scratch of tb_sparse_decode_attn_static: device memory that the library owns, one copy per
// GPU, held from the first use on that GPU until the process ends.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the symbol): the device
// address is looked up once per device and kept.
constexpr size_t kStaticScratchBytes = size_t{4} << 20;
static_assert(kAttnMostWgs * (kCounterStrideWords + 128 + 2) * sizeof(float) + 512 <= kStaticScratchBytes, "heads that are split fit the scratch");
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call per device).
tb_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TB_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TB_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return TB_OK;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

tb_status check_desc(const tb_cache_desc* d) {
  if (!d) return TB_ERR_INVALID_ARG;
  if (d->B < 0 || d->Hq < 0 || d->Hkv < 0 || d->N < 0) return TB_ERR_INVALID_ARG;
  if (d->dtype != TB_F32 && d->dtype != TB_BF16) return TB_ERR_INVALID_ARG;
  if (d->Hkv == 0 ? d->Hq != 0 : (d->Hq % d->Hkv) != 0) return TB_ERR_INVALID_ARG;
  if (d->D != 64 && d->D != 128) return TB_ERR_UNSUPPORTED;
  if (d->Dimp != 16 && d->Dimp != 32 && d->Dimp != 64) return TB_ERR_UNSUPPORTED;
  if (d->Hkv > 0) {
    const int g = d->Hq / d->Hkv;
    if (g != 1 && g != 2 && g != 4 && g != 8) return TB_ERR_UNSUPPORTED;
  }
  if (d->B > 65535 || d->Hq > 65535) return TB_ERR_UNSUPPORTED;
  return TB_OK;
}

tb_status check_strides(const tb_cache_desc* d, int64_t sb, int64_t sh, int64_t sn, int inner) {
  if (sb < 0 || sh < 0 || sn < inner) return TB_ERR_INVALID_ARG;
  if ((sb | sh | sn) % 8) return TB_ERR_UNSUPPORTED;
  (void)d;
  return TB_OK;
}

#define TB_TRY(expr)                 \
  do {                               \
    const tb_status _s = (expr);     \
    if (_s != TB_OK) return _s;      \
  } while (0)

struct Policy {
  int64_t lo, hi, kk, count;
};
Policy policy(int64_t N, int32_t k, int32_t sink, int32_t window) {
  Policy p;
  p.lo = sink < N ? sink : N;
  p.hi = (N - window > p.lo) ? (N - window) : p.lo;
  const int64_t nc = p.hi - p.lo;
  p.kk = k < nc ? k : nc;
  p.count = p.lo + p.kk + (N - p.hi);
  return p;
}

tb_status check_score_args(const tb_cache_desc* d, const void* q_imp, const void* Kimp, const float* scores,
                           int64_t score_stride) {
  TB_TRY(check_desc(d));
  if (!q_imp || !Kimp || !scores) return TB_ERR_INVALID_ARG;
  if (score_stride < d->N) return TB_ERR_INVALID_ARG;
  if (score_stride % 4) return TB_ERR_UNSUPPORTED;
  TB_TRY(check_strides(d, d->ki_stride_b, d->ki_stride_h, d->ki_stride_n, d->Dimp));
  if (!aligned16(q_imp) || !aligned16(Kimp) || !aligned16(scores)) return TB_ERR_UNSUPPORTED;
  return TB_OK;
}

tb_status check_select_args(const tb_cache_desc* d, const float* scores, int64_t score_stride, int32_t k,
                            int32_t sink, int32_t window, const int32_t* idx, const int32_t* count,
                            int64_t idx_cap) {
  TB_TRY(check_desc(d));
  if (!scores || !idx || !count) return TB_ERR_INVALID_ARG;
  if (k < 0 || sink < 0 || window < 0) return TB_ERR_INVALID_ARG;
  if (score_stride < d->N) return TB_ERR_INVALID_ARG;
  if (score_stride % 4 || !aligned16(scores)) return TB_ERR_UNSUPPORTED;
  if (d->N > kSelectMaxN) return TB_ERR_UNSUPPORTED;
  const Policy p = policy(d->N, k, sink, window);
  if (idx_cap < p.count) return TB_ERR_INVALID_ARG;
  return TB_OK;
}

tb_status check_attn_args(const tb_cache_desc* d, const void* q, const void* K, const void* V, const int32_t* idx,
                          const int32_t* count, int64_t idx_cap, int64_t max_count, int64_t tail_begin,
                          int64_t tail_end, const float* out) {
  TB_TRY(check_desc(d));
  if (!q || !K || !V || !idx || !count || !out) return TB_ERR_INVALID_ARG;
  if (idx_cap < 0 || max_count < 0 || max_count > idx_cap) return TB_ERR_INVALID_ARG;
  if (tail_begin < 0 || tail_begin > tail_end || tail_end > d->N) return TB_ERR_INVALID_ARG;
  if (d->N == 0 && max_count > 0) return TB_ERR_INVALID_ARG;
  TB_TRY(check_strides(d, d->k_stride_b, d->k_stride_h, d->k_stride_n, d->D));
  TB_TRY(check_strides(d, d->v_stride_b, d->v_stride_h, d->v_stride_n, d->D));
  if (!aligned16(q) || !aligned16(K) || !aligned16(V)) return TB_ERR_UNSUPPORTED;
  if (max_count + (tail_end - tail_begin) > (int64_t{1} << 30)) return TB_ERR_UNSUPPORTED;
  // the gather addresses rows with 32-bit byte offsets inside one (b, kv-head) slab
  const int64_t elt = d->dtype == TB_F32 ? 4 : 2;
  if (d->N * d->k_stride_n * elt >= (int64_t{1} << 32) || d->N * d->v_stride_n * elt >= (int64_t{1} << 32))
    return TB_ERR_UNSUPPORTED;
  return TB_OK;
}

}  // namespace
}  // namespace tb

using namespace tb;

extern "C" {

tb_status tb_project_keys(const tb_cache_desc* d, const void* K, const void* W, int32_t Hw, void* Kimp,
                          int64_t n_begin, int64_t n_end, void* stream) {
  TB_TRY(check_desc(d));
  if (!K || !W || !Kimp) return TB_ERR_INVALID_ARG;
  if (Hw != 1 && Hw != d->Hkv) return TB_ERR_INVALID_ARG;
  if (n_begin < 0 || n_begin > n_end || n_end > d->N) return TB_ERR_INVALID_ARG;
  TB_TRY(check_strides(d, d->k_stride_b, d->k_stride_h, d->k_stride_n, d->D));
  TB_TRY(check_strides(d, d->ki_stride_b, d->ki_stride_h, d->ki_stride_n, d->Dimp));
  if (!aligned16(K) || !aligned16(W) || !aligned16(Kimp)) return TB_ERR_UNSUPPORTED;
  return launch_project(d, K, W, Hw, Kimp, n_begin, n_end, static_cast<hipStream_t>(stream));
}

tb_status tb_score(const tb_cache_desc* d, const void* q_imp, const void* Kimp, float scale, float* scores,
                   int64_t score_stride, void* stream) {
  TB_TRY(check_score_args(d, q_imp, Kimp, scores, score_stride));
  if (d->B == 0 || d->Hq == 0) return TB_OK;
  ScoreLaunch L{d, q_imp, Kimp, scale, scores, score_stride};
  return launch_score(L, static_cast<hipStream_t>(stream));
}

tb_status tb_select_topk(const tb_cache_desc* d, const float* scores, int64_t score_stride, int32_t k, int32_t sink,
                         int32_t window, int32_t* idx, int32_t* count, int64_t idx_cap, void* ws, size_t ws_bytes,
                         void* stream) {
  TB_TRY(check_select_args(d, scores, score_stride, k, sink, window, idx, count, idx_cap));
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  if (units == 0) return TB_OK;
  const Policy p = policy(d->N, k, sink, window);
  SelectLaunch L;
  L.units = units;
  L.N = d->N;
  L.scores = scores;
  L.score_stride = score_stride;
  L.kk = static_cast<int32_t>(p.kk);
  L.lo = static_cast<int32_t>(p.lo);
  L.hi = static_cast<int32_t>(p.hi);
  L.idx = idx;
  L.count = count;
  L.idx_cap = idx_cap;
  // scratch of the two-stage selection: behind the arrival counters, which stay untouched
  const size_t off = ws_layout(units, d->D, 1).part_off;
  const bool usable = ws && aligned16(ws) && ws_bytes > off;
  L.scratch = usable ? static_cast<char*>(ws) + off : nullptr;
  L.scratch_bytes = usable ? ws_bytes - off : 0;
  return launch_select(L, static_cast<hipStream_t>(stream));
}

tb_status tb_expand_neighbors(int32_t B, int32_t Hq, int64_t N, int32_t radius, int32_t mode, const int32_t* idx_in,
                              const int32_t* count_in, int64_t cap_in, int32_t* idx_out, int32_t* count_out,
                              int64_t cap_out, void* stream) {
  if (B < 0 || Hq < 0 || N < 0 || radius < 0 || cap_in < 0 || cap_out < 0) return TB_ERR_INVALID_ARG;
  if (mode != 0 && mode != 1) return TB_ERR_INVALID_ARG;
  if (!idx_in || !count_in || !idx_out || !count_out) return TB_ERR_INVALID_ARG;
  if (idx_in == idx_out) return TB_ERR_INVALID_ARG;
  if (B > 65535 || Hq > 65535 || N > (int64_t{1} << 30) || radius > (1 << 20)) return TB_ERR_UNSUPPORTED;
  const int64_t mult = (mode == 0) ? (2 * static_cast<int64_t>(radius) + 1) : 2;
  int64_t need = mult * cap_in;
  if (need > N) need = N;
  if (cap_out < need) return TB_ERR_INVALID_ARG;
  return launch_expand(static_cast<int64_t>(B) * Hq, N, radius, mode, idx_in, count_in, cap_in, idx_out, count_out,
                       cap_out, static_cast<hipStream_t>(stream));
}

static tb_status sparse_attn(const tb_cache_desc* d, const void* q, const void* K, const void* V, const int32_t* idx,
                             const int32_t* count, int64_t idx_cap, int64_t max_count, int64_t tail_begin,
                             int64_t tail_end, float sm_scale, float* out, float* lse, void* ws, size_t ws_bytes,
                             void* stream, bool shared_list) {
  TB_TRY(check_attn_args(d, q, K, V, idx, count, idx_cap, max_count, tail_begin, tail_end, out));
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  if (units == 0) return TB_OK;
  const int64_t rows = max_count + (tail_end - tail_begin);
  const bool grouped = shared_list && attn_shared_list_grouped(d, rows);
  const AttnPlan by_head = attn_plan(d, rows, shared_list);
  AttnPlan plan = grouped ? attn_group_plan(d, rows) : by_head;
  if (!ws || !aligned16(ws)) return TB_ERR_WORKSPACE;
  if (grouped && attn_group_mfma(d)) {
    // where a workgroup per KV group splits finer than the forms that such a shape asked room for before it
    // (per head, or one split a group), a workspace of that size still serves, with fewer splits
    const int64_t groups = static_cast<int64_t>(d->B) * d->Hkv;
    const int least = groups > kAttnGroupTargetWgs ? 1 : (groups < 32 ? by_head.least : plan.nsplit);
    plan.least = std::min(plan.nsplit, least);
  }
  if (!fit_splits(d, plan, ws_bytes)) return TB_ERR_WORKSPACE;
  const WsLayout w = ws_layout(units, d->D, plan.nsplit);
  AttnLaunch L{d,   q,   K,   V,
               idx, count, idx_cap, max_count, tail_begin, tail_end,
               sm_scale, out, lse,
               reinterpret_cast<float*>(static_cast<char*>(ws) + w.part_off),
               reinterpret_cast<uint32_t*>(ws), plan};
  L.shared_list = shared_list;
  L.grouped = grouped;
  return launch_attn(L, static_cast<hipStream_t>(stream));
}

tb_status tb_sparse_decode_attn(const tb_cache_desc* d, const void* q, const void* K, const void* V,
                                const int32_t* idx, const int32_t* count, int64_t idx_cap, int64_t max_count,
                                int64_t tail_begin, int64_t tail_end, float sm_scale, float* out, float* lse,
                                void* ws, size_t ws_bytes, void* stream) {
  return sparse_attn(d, q, K, V, idx, count, idx_cap, max_count, tail_begin, tail_end, sm_scale, out, lse, ws,
                     ws_bytes, stream, false);
}

tb_status tb_sparse_decode_attn_shared(const tb_cache_desc* d, const void* q, const void* K, const void* V,
                                       const int32_t* idx, const int32_t* count, int64_t idx_cap,
                                       int64_t max_count, int64_t tail_begin, int64_t tail_end, float sm_scale,
                                       float* out, float* lse, void* ws, size_t ws_bytes, void* stream) {
  return sparse_attn(d, q, K, V, idx, count, idx_cap, max_count, tail_begin, tail_end, sm_scale, out, lse, ws,
                     ws_bytes, stream, true);
}

tb_status tb_sparse_decode_attn_static(const tb_cache_desc* d, const void* q, const void* K, const void* V,
                                       const int32_t* idx, const int32_t* count, int64_t idx_cap,
                                       int64_t max_count, int64_t tail_begin, int64_t tail_end, float sm_scale,
                                       float* out, float* lse, void* stream) {
  TB_TRY(check_attn_args(d, q, K, V, idx, count, idx_cap, max_count, tail_begin, tail_end, out));
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  if (units == 0) return TB_OK;
  const AttnPlan plan = attn_plan(d, max_count + (tail_end - tail_begin));
  const WsLayout w = ws_layout(units, d->D, plan.nsplit);
  if (w.total > kStaticScratchBytes) return TB_ERR_WORKSPACE;  // beyond the library's own scratch
  void* ws = nullptr;
  TB_TRY(static_scratch(&ws));
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the arrival counters must be zero when the kernel starts; the array keeps whatever the
  // last call on this GPU left, so they are cleared here (a fill kernel, not a memset node:
  // callers may be capturing a graph)
  TB_TRY(launch_fill_zero(ws, w.part_off, st));
  AttnLaunch L{d,   q,   K,   V,
               idx, count, idx_cap, max_count, tail_begin, tail_end,
               sm_scale, out, lse,
               reinterpret_cast<float*>(static_cast<char*>(ws) + w.part_off),
               reinterpret_cast<uint32_t*>(ws), plan};
  return launch_attn(L, st);
}

tb_status tb_gather_kv(const tb_cache_desc* d, const void* K, const void* V, const int32_t* idx, const int32_t* count,
                       int64_t idx_cap, int64_t max_count, void* Kbuf, void* Vbuf, int64_t buf_cap, void* stream) {
  TB_TRY(check_desc(d));
  if (!K || !V || !idx || !count || !Kbuf || !Vbuf) return TB_ERR_INVALID_ARG;
  if (idx_cap < 0 || max_count < 0 || max_count > idx_cap || max_count > buf_cap) return TB_ERR_INVALID_ARG;
  if (d->N == 0 && max_count > 0) return TB_ERR_INVALID_ARG;
  TB_TRY(check_strides(d, d->k_stride_b, d->k_stride_h, d->k_stride_n, d->D));
  TB_TRY(check_strides(d, d->v_stride_b, d->v_stride_h, d->v_stride_n, d->D));
  if (!aligned16(K) || !aligned16(V) || !aligned16(Kbuf) || !aligned16(Vbuf)) return TB_ERR_UNSUPPORTED;
  if (max_count > (int64_t{1} << 30)) return TB_ERR_UNSUPPORTED;
  GatherLaunch L{d, K, V, idx, count, idx_cap, max_count, Kbuf, Vbuf, buf_cap};
  return launch_gather(L, static_cast<hipStream_t>(stream));
}

static tb_status check_gather(const tb_cache_desc* d, const void* K, const void* V, const int32_t* idx, const int32_t* count, int64_t idx_cap,
                              int64_t max_count, int32_t skip_front, int32_t skip_back, void* Kbuf, void* Vbuf, int64_t buf_cap, int32_t* count_out,
                              GatherLaunch& L) {
  TB_TRY(check_desc(d));
  if (!K || !V || !idx || !count || !Kbuf || !Vbuf || !count_out) return TB_ERR_INVALID_ARG;
  if (idx_cap < 0 || max_count < 0 || max_count > idx_cap || skip_front < 0 || skip_back < 0) return TB_ERR_INVALID_ARG;
  const int64_t rows = max_count > static_cast<int64_t>(skip_front) + skip_back ? max_count - skip_front - skip_back : 0;
  if (rows > buf_cap) return TB_ERR_INVALID_ARG;
  if (d->N == 0 && max_count > 0) return TB_ERR_INVALID_ARG;
  TB_TRY(check_strides(d, d->k_stride_b, d->k_stride_h, d->k_stride_n, d->D));
  TB_TRY(check_strides(d, d->v_stride_b, d->v_stride_h, d->v_stride_n, d->D));
  if (!aligned16(K) || !aligned16(V) || !aligned16(Kbuf) || !aligned16(Vbuf)) return TB_ERR_UNSUPPORTED;
  if (max_count > (int64_t{1} << 30)) return TB_ERR_UNSUPPORTED;
  L = GatherLaunch{d, K, V, idx, count, idx_cap, max_count, Kbuf, Vbuf, buf_cap, skip_front, skip_back, count_out};
  return TB_OK;
}

tb_status tb_gather_important(const tb_cache_desc* d, const void* K, const void* V, const int32_t* idx,
                              const int32_t* count, int64_t idx_cap, int64_t max_count, int32_t skip_front,
                              int32_t skip_back, void* Kbuf, void* Vbuf, int64_t buf_cap, int32_t* count_out,
                              void* stream) {
  GatherLaunch L;
  TB_TRY(check_gather(d, K, V, idx, count, idx_cap, max_count, skip_front, skip_back, Kbuf, Vbuf, buf_cap, count_out, L));
  return launch_gather(L, static_cast<hipStream_t>(stream));
}

static tb_status check_append(const tb_cache_desc* src, const void* K, const void* V, int64_t src_row, const tb_cache_desc* dst, const void* Kdst,
                              const void* Vdst, int64_t dst_row, int64_t rows) {
  TB_TRY(check_desc(src));
  TB_TRY(check_desc(dst));
  if (!K || !V || !Kdst || !Vdst || rows < 0 || src_row < 0 || dst_row < 0) return TB_ERR_INVALID_ARG;
  if (src->B != dst->B || src->Hkv != dst->Hkv || src->D != dst->D || src->dtype != dst->dtype) return TB_ERR_INVALID_ARG;
  if (rows > src->N - src_row || rows > dst->N - dst_row) return TB_ERR_INVALID_ARG;
  for (const tb_cache_desc* d : {src, dst}) {
    TB_TRY(check_strides(d, d->k_stride_b, d->k_stride_h, d->k_stride_n, d->D));
    TB_TRY(check_strides(d, d->v_stride_b, d->v_stride_h, d->v_stride_n, d->D));
  }
  if (!aligned16(K) || !aligned16(V) || !aligned16(Kdst) || !aligned16(Vdst)) return TB_ERR_UNSUPPORTED;
  if (rows > (int64_t{1} << 20)) return TB_ERR_UNSUPPORTED;
  return TB_OK;
}

static tb_status buffered_attn(const tb_cache_desc* d, const void* q, const void* Kbuf, const void* Vbuf, int64_t buf_cap, const int32_t* count,
                               int64_t max_count, const void* K, const void* V, int64_t tail_begin, int64_t tail_end, float sm_scale, float* out,
                               float* lse, void* ws, size_t ws_bytes, void* stream, const NewRow* append, const GatherLaunch* migrate = nullptr) {
  if (!Kbuf || !Vbuf || buf_cap < 0 || max_count > buf_cap) return TB_ERR_INVALID_ARG;
  // the list itself is not read: its place in the argument check is taken by the count array
  TB_TRY(check_attn_args(d, q, K, V, count, count, buf_cap, max_count, tail_begin, tail_end, out));
  if (!aligned16(Kbuf) || !aligned16(Vbuf)) return TB_ERR_UNSUPPORTED;
  const int64_t elt = d->dtype == TB_F32 ? 4 : 2;
  if (buf_cap * d->D * elt >= (int64_t{1} << 32)) return TB_ERR_UNSUPPORTED;  // 32-bit offsets inside a head's buffer
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  if (units == 0) {
    if (!append) return TB_OK;
    return launch_append(*append->src, append->K, append->V, append->src_row, *d, append->Kdst, append->Vdst, append->dst_row, 1,
                         static_cast<hipStream_t>(stream));
  }
  const int64_t rows = max_count + (tail_end - tail_begin);
  AttnPlan plan = attn_plan(d, rows);
  if (!ws || !aligned16(ws) || !fit_splits(d, plan, ws_bytes)) return TB_ERR_WORKSPACE;
  const WsLayout w = ws_layout(units, d->D, plan.nsplit);
  AttnLaunch L{d,   q,   K,   V,
               nullptr, count, buf_cap, max_count, tail_begin, tail_end,
               sm_scale, out, lse,
               reinterpret_cast<float*>(static_cast<char*>(ws) + w.part_off),
               reinterpret_cast<uint32_t*>(ws), plan};
  L.Kbuf = Kbuf;
  L.Vbuf = Vbuf;
  L.buf_cap = buf_cap;
  L.append = append;
  L.migrate = migrate;
  return launch_attn(L, static_cast<hipStream_t>(stream));
}

tb_status tb_append_kv(const tb_cache_desc* src, const void* K, const void* V, int64_t src_row, const tb_cache_desc* dst,
                       void* Kdst, void* Vdst, int64_t dst_row, int64_t rows, void* stream) {
  TB_TRY(check_append(src, K, V, src_row, dst, Kdst, Vdst, dst_row, rows));
  return launch_append(*src, K, V, src_row, *dst, Kdst, Vdst, dst_row, rows, static_cast<hipStream_t>(stream));
}

tb_status tb_buffered_decode_attn(const tb_cache_desc* d, const void* q, const void* Kbuf, const void* Vbuf,
                                  int64_t buf_cap, const int32_t* count, int64_t max_count, const void* K,
                                  const void* V, int64_t tail_begin, int64_t tail_end, float sm_scale, float* out,
                                  float* lse, void* ws, size_t ws_bytes, void* stream) {
  return buffered_attn(d, q, Kbuf, Vbuf, buf_cap, count, max_count, K, V, tail_begin, tail_end, sm_scale, out, lse, ws, ws_bytes, stream,
                       nullptr);
}

tb_status tb_append_buffered_decode_attn(const tb_cache_desc* src, const void* K_src, const void* V_src, int64_t src_row,
                                         const tb_cache_desc* d, const void* q, const void* Kbuf, const void* Vbuf, int64_t buf_cap,
                                         const int32_t* count, int64_t max_count, void* K, void* V, int64_t dst_row, int64_t tail_begin,
                                         int64_t tail_end, float sm_scale, float* out, float* lse, void* ws, size_t ws_bytes, void* stream) {
  TB_TRY(check_append(src, K_src, V_src, src_row, d, K, V, dst_row, 1));
  const NewRow row{src, K_src, V_src, src_row, dst_row, K, V};
  return buffered_attn(d, q, Kbuf, Vbuf, buf_cap, count, max_count, K, V, tail_begin, tail_end, sm_scale, out, lse, ws, ws_bytes, stream, &row);
}

tb_status tb_migrate_buffered_decode_attn(const tb_cache_desc* src, const void* K_src, const void* V_src, const int32_t* idx,
                                          const int32_t* count, int64_t idx_cap, int64_t max_count, int32_t skip_front, int32_t skip_back,
                                          int32_t* count_out, int64_t src_row, const tb_cache_desc* d, const void* q, void* Kbuf, void* Vbuf,
                                          int64_t buf_cap, void* K, void* V, int64_t dst_row, int64_t tail_begin, int64_t tail_end,
                                          float sm_scale, float* out, float* lse, void* ws, size_t ws_bytes, void* stream) {
  GatherLaunch lists;
  TB_TRY(check_gather(src, K_src, V_src, idx, count, idx_cap, max_count, skip_front, skip_back, Kbuf, Vbuf, buf_cap, count_out, lists));
  TB_TRY(check_desc(d));
  if (src->B != d->B || src->Hq != d->Hq || src->Hkv != d->Hkv || src->D != d->D || src->dtype != d->dtype) return TB_ERR_INVALID_ARG;
  if (src->N > (int64_t{1} << 30)) return TB_ERR_UNSUPPORTED;  // the next bit of a row number names the cache of the dense range
  if (src_row >= 0) TB_TRY(check_append(src, K_src, V_src, src_row, d, K, V, dst_row, 1));
  const NewRow row{src, K_src, V_src, src_row, dst_row, K, V};
  return buffered_attn(d, q, Kbuf, Vbuf, buf_cap, count_out, std::min(max_count, buf_cap), K, V, tail_begin, tail_end, sm_scale, out, lse, ws,
                       ws_bytes, stream, src_row >= 0 ? &row : nullptr, &lists);
}

tb_status tb_predict_queries(const tb_predictor_desc* p, int32_t B, const void* h, const void* gamma,
                             const void* beta, const void* W1, const void* b1, const void* W2, const void* b2,
                             float* hidden_act, float* ln_act, void* q_imp, void* stream) {
  if (!p || B < 0) return TB_ERR_INVALID_ARG;
  if (p->E <= 0 || p->hidden <= 0 || p->G <= 0 || p->Hq <= 0 || p->Dimp <= 0) return TB_ERR_INVALID_ARG;
  if (p->dtype != TB_F32 && p->dtype != TB_BF16) return TB_ERR_INVALID_ARG;
  if (!(p->ln_eps >= 0.f)) return TB_ERR_INVALID_ARG;
  if (!h || !gamma || !beta || !W1 || !b1 || !W2 || !b2 || !hidden_act || !ln_act || !q_imp)
    return TB_ERR_INVALID_ARG;
  if (p->E % 8 || p->hidden % 8 || p->E > 8192 || p->hidden > 2048 || B > 65535) return TB_ERR_UNSUPPORTED;
  if (static_cast<int64_t>(p->G) * p->Hq * p->Dimp > (int64_t{1} << 24)) return TB_ERR_UNSUPPORTED;
  if (!aligned16(W1) || !aligned16(W2) || !aligned16(h) || !aligned16(gamma) || !aligned16(beta) ||
      !aligned16(ln_act))
    return TB_ERR_UNSUPPORTED;
  PredictLaunch L{p->dtype, B, p->E, p->hidden, p->G, p->Hq, p->Dimp, p->ln_eps, h, gamma, beta, W1, b1, W2, b2,
                  hidden_act, ln_act, q_imp};
  return launch_predict(L, static_cast<hipStream_t>(stream));
}

tb_status tb_decode_step(const tb_cache_desc* d, const void* q_imp, const void* Kimp, float score_scale,
                         const void* q, const void* K, const void* V, int32_t k, int32_t sink, int32_t window,
                         float sm_scale, float* scores, int64_t score_stride, int32_t* idx, int32_t* count,
                         int64_t idx_cap, float* out, float* lse, void* ws, size_t ws_bytes, void* stream) {
  TB_TRY(check_score_args(d, q_imp, Kimp, scores, score_stride));
  TB_TRY(check_select_args(d, scores, score_stride, k, sink, window, idx, count, idx_cap));
  const Policy p = policy(d->N, k, sink, window);
  TB_TRY(check_attn_args(d, q, K, V, idx, count, idx_cap, p.count, 0, 0, out));
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  if (units == 0) return TB_OK;
  AttnPlan plan = attn_plan(d, p.count);
  if (!ws || !aligned16(ws) || !fit_splits(d, plan, ws_bytes)) return TB_ERR_WORKSPACE;
  const WsLayout w = ws_layout(units, d->D, plan.nsplit);
  hipStream_t st = static_cast<hipStream_t>(stream);
  ScoreLaunch S{d, q_imp, Kimp, score_scale, scores, score_stride};

  SelectLaunch L;
  L.units = units;
  L.N = d->N;
  L.scores = scores;
  L.score_stride = score_stride;
  L.kk = static_cast<int32_t>(p.kk);
  L.lo = static_cast<int32_t>(p.lo);
  L.hi = static_cast<int32_t>(p.hi);
  L.idx = idx;
  L.count = count;
  L.idx_cap = idx_cap;
  L.scratch = static_cast<char*>(ws) + w.part_off;
  L.scratch_bytes = ws_bytes - w.part_off;
  AttnLaunch A{d,   q,   K,   V,
               idx, count, idx_cap, p.count, 0, 0,
               sm_scale, out, lse,
               reinterpret_cast<float*>(static_cast<char*>(ws) + w.part_off),
               reinterpret_cast<uint32_t*>(ws), plan};
  A.fresh_lists = true;
  if (step_in_one(d, p.count, plan.nsplit)) return launch_step(S, L, A, st);
  const SelectPlan both = score_select_plan(d, p.hi - p.lo, p.kk);
  if (both.pieces > 1 && L.scratch_bytes >= select_scratch_bytes(units, both)) {
    TB_TRY(launch_score_select(S, L, both, st));
  } else {
    TB_TRY(launch_score(S, st));
    TB_TRY(launch_select(L, st));
  }
  return launch_attn(A, st);
}

size_t tb_workspace_bytes(int32_t op, const tb_cache_desc* d, int64_t max_count) {
  if (check_desc(d) != TB_OK || max_count < 0) return 0;
  const int64_t units = static_cast<int64_t>(d->B) * d->Hq;
  // two-stage selection of long rows (none for most shapes): max_count bounds the budget
  const size_t sel = select_scratch_upto(units, d->N, max_count);
  const size_t sel_total = sel ? ws_layout(units, d->D, 1).part_off + align_up(sel, 256) : 0;
  if (op == TB_OP_SELECT) return sel_total;
  if (op == TB_OP_ATTN || op == TB_OP_DECODE_STEP) {
    const AttnPlan plan = attn_plan(d, max_count);
    // sized for the largest split count a shorter list could get, so that one workspace serves
    // every call whose list is no longer than max_count
    size_t att = ws_layout(units, d->D, plan.max_split).total;
    if (attn_shared_list_grouped(d, max_count)) {  // the head-less form splits per KV group, possibly finer
      const AttnPlan gp = attn_group_plan(d, max_count);
      const size_t g_att = ws_layout(units, d->D, gp.max_split).total;
      if (g_att > att) att = g_att;
    }
    if (op == TB_OP_ATTN) return att;
    const size_t both = score_select_scratch_upto(d, max_count);
    const size_t step = both ? ws_layout(units, d->D, 1).part_off + align_up(both, 256) : 0;
    return std::max(std::max(step, sel_total), att);
  }
  return 0;
}

tb_status tb_workspace_init(void* ws, size_t ws_bytes, void* stream) {
  if (!ws && ws_bytes) return TB_ERR_INVALID_ARG;
  if (ws_bytes % 4 || (reinterpret_cast<uintptr_t>(ws) & 3u)) return TB_ERR_INVALID_ARG;
  return launch_fill_zero(ws, ws_bytes, static_cast<hipStream_t>(stream));
}

tb_status tb_read_stream_probe(const void* src, size_t bytes, uint32_t* sink, void* stream) {
  if (!src || !sink) return TB_ERR_INVALID_ARG;
  if (!aligned16(src)) return TB_ERR_UNSUPPORTED;
  return launch_read_stream(src, bytes, sink, static_cast<hipStream_t>(stream));
}

const char* tb_status_string(tb_status s) {
  switch (s) {
    case TB_OK: return "ok";
    case TB_ERR_INVALID_ARG: return "invalid argument";
    case TB_ERR_UNSUPPORTED: return "unsupported shape, dtype or alignment";
    case TB_ERR_WORKSPACE: return "workspace missing or too small";
    case TB_ERR_HIP: return "HIP launch failed";
    default: return "unknown status";
  }
}

int32_t tb_version(void) { return 100; }

}  // extern "C"
