// C-ABI entry points of libbaklava (device part): context, split-K schedule, launches.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <numeric>
#include <vector>

#include "baklava.h"
#include "common.h"
#include "plan.h"

using namespace baklava;

namespace {

thread_local int g_last_hip_error = 0;

inline bool hip_ok(hipError_t e) {
  if (e == hipSuccess) return true;
  g_last_hip_error = (int)e;
  return false;
}

constexpr int kMinChunk = 256;
constexpr int kSizingChunk = 256;  // the workspace is sized for chunks of at least this many rows
constexpr int kDefaultChunk = 512;        // launches over part of the model: shortest run (the item target lengthens it)
constexpr int kDefaultChunkWhole = 256;   // launches over the whole model: shortest run; longer ones come from the item target
constexpr int kWholeItemsPerCu = 5;       // launches over many caches aim at this many work items per compute unit
constexpr int kShortestRun = 64;          // where those would leave compute units idle (see build_schedule)
constexpr int kMostFillItems = 256;       // most work items such short runs are cut for: one per compute unit (sizes the workspace)
constexpr int kMaxChunk = 1 << 22; // row offsets inside a work item stay below 2^32 bytes
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int64_t count_items(const int32_t* cap, int64_t n_caches, int chunk) {
  int64_t n = 0;
  for (int64_t c = 0; c < n_caches; ++c) n += std::max<int64_t>(1, ((int64_t)cap[c] + chunk - 1) / chunk);
  return n;
}

struct WorkspacePlan {
  // index 0: schedule for launches over a layer sub-range, 1: for launches over the whole model, 2: for launches over
  // several layers where that of a single one would cut needlessly short runs (see schedule_for)
  size_t items[3], multi[3];
  size_t part_o, part_ml, final_ml, logits, lag_q, lag_ml, lag_n, lag_cnt, flush_ticket, status, kept, info, order_all, order_layer;
  size_t move_ticket, move_flags, tiles, spread, tile_hist, sel_state, total;
  int64_t n_tiles, n_long;
  int64_t max_items;
};

bool shape_ok(const baklava_desc* d) {
  if (!d) return false;
  if (d->L <= 0 || d->Hq <= 0 || d->Hkv <= 0 || d->batch <= 0) return false;
  if (d->D != 64 && d->D != 128) return false;
  if (d->dtype != BAKLAVA_BF16 && d->dtype != BAKLAVA_F32) return false;
  if (d->Hq % d->Hkv) return false;
  const int G = d->Hq / d->Hkv;
  if (G > 16 || (d->dtype == BAKLAVA_F32 && G > 8)) return false;
  if (d->dtype == BAKLAVA_BF16 && G > 8 && d->D != 128) return false;
  if (d->sink < 0 || d->recent < 0) return false;
  if (d->policy != BAKLAVA_POLICY_SCORE && d->policy != BAKLAVA_POLICY_STREAMING) return false;
  if ((int64_t)d->L * d->batch * d->Hkv > INT32_MAX) return false;
  return true;
}

// Scores are deferred over bf16 rows of 128 elements only (see decode_impl).
bool keeps_records(const baklava_desc* d) { return d->dtype == BAKLAVA_BF16 && d->D == 128; }

WorkspacePlan plan_workspace(const baklava_desc* d, const int32_t* cap) {
  WorkspacePlan w{};
  const int64_t n_caches = (int64_t)d->L * d->batch * d->Hkv;
  const int G = d->Hq / d->Hkv;
  const size_t row_bytes = (size_t)d->D * (d->dtype == BAKLAVA_BF16 ? 2 : 4);
  int64_t total_tokens = 0;
  for (int64_t c = 0; c < n_caches; ++c) total_tokens += cap[c];
  // runs of at least kSizingChunk rows, or the shorter ones of the layers that those would not fill the chip with
  const int64_t cpl = (int64_t)d->batch * d->Hkv;
  w.max_items = 0;
  for (int32_t l = 0; l < d->L; ++l)
    w.max_items += std::max(count_items(cap + l * cpl, cpl, kSizingChunk),
                            std::min<int64_t>(count_items(cap + l * cpl, cpl, kShortestRun), kMostFillItems));
  size_t o = 0;
  for (int k = 0; k < 3; ++k) {  // (the third only where a launch can hold several layers, but not all)
    w.multi[k] = o;   o = align256(o + (k < 2 || d->L > 2 ? (size_t)n_caches * sizeof(MultiCache) : 0));
    w.items[k] = o;   o = align256(o + (k < 2 || d->L > 2 ? (size_t)w.max_items * sizeof(Item) : 0));
  }
  w.part_o = o;       o = align256(o + (size_t)w.max_items * G * d->D * 4);
  w.part_ml = o;      o = align256(o + (size_t)w.max_items * G * 2 * 4);
  w.final_ml = o;     o = align256(o + (size_t)n_caches * G * 2 * 4);
  // score tracking: the record of the pending calls of every cache (32 packed query rows, their (max, 1/sum), the
  // rows each call saw, the count of pending calls per head), or the logits of a call where there are no records
  const bool track = d->track_scores != 0, records = track && keeps_records(d);
  w.logits = o;       o = align256(o + (track && !records ? (size_t)total_tokens * G * 4 : 0));
  w.lag_q = o;        o = align256(o + (records ? (size_t)n_caches * kLagRows * row_bytes : 0));
  w.lag_ml = o;       o = align256(o + (records ? (size_t)n_caches * kLagRows * 2 * 4 : 0));
  w.lag_n = o;        o = align256(o + (size_t)n_caches * kLagCalls * 4);
  w.lag_cnt = o;      o = o + (size_t)n_caches * G * 4;
  w.flush_ticket = o; o = align256(o + (size_t)n_caches * kTicketStride * 4);
  w.status = o;       o = align256(o + 256);
  w.kept = o;         o = align256(o + (size_t)total_tokens * 4);
  w.info = o;         o = align256(o + (size_t)n_caches * sizeof(CompactInfo));
  w.order_all = o;    o = align256(o + (size_t)n_caches * 4);
  w.order_layer = o;  o = align256(o + (size_t)n_caches * 4);
  w.move_ticket = o;  o = align256(o + (size_t)n_caches * 4);
  w.move_flags = o;   o = align256(o + (size_t)(total_tokens / kMoveRowsMin + n_caches) * 4);
  // selection of the caches too long for one workgroup: tile table and per-tile digit counters
  w.n_tiles = 0;
  w.n_long = 0;
  for (int64_t c = 0; c < n_caches; ++c)
    if (cap[c] > kMinLongRows) {  // room for every threshold BAKLAVA_OPT_TILED_SELECT_ROWS may set
      w.n_tiles += ((int64_t)cap[c] + kTileRows - 1) / kTileRows;
      w.n_long += 1;
    }
  w.tiles = o;        o = align256(o + (size_t)w.n_tiles * sizeof(SelTile));
  w.spread = o;       o = align256(o + (size_t)(w.n_tiles + n_caches) * sizeof(SelTile));
  w.tile_hist = o;    o = align256(o + (size_t)w.n_tiles * 4 * 256 * 4);
  w.sel_state = o;    o = align256(o + (size_t)w.n_long * 4 * sizeof(SelState));
  w.total = o;
  return w;
}

}  // namespace

struct baklava_ctx {
  baklava_desc d;
  int64_t n_caches, total_tokens;
  int32_t cpl;  // caches per layer
  int32_t G;
  int32_t row_bytes;
  std::vector<int64_t> off;
  std::vector<int32_t> cap, len, budget;
  std::vector<int32_t> order_all, order_layer;  // caches, longest first (whole model / inside each layer)
  std::vector<MoveCount> move_before;           // cache -> work of the eviction move for the caches before it
  std::vector<int32_t> tile_begin;              // cache -> first tile of the tiled selection (long caches only have any)
  std::vector<int32_t> spread_begin;            // cache -> first tile of the selection by several workgroups per cache
  std::vector<int32_t> n_wide;                  // layer -> caches with more than kNarrowRows rows of capacity
  int32_t kernel_pref;
  bool layer_one_wave;   // default schedule of layer-range launches: one workgroup per compute unit
  int32_t target_items;  // > 0: layer-range launches lengthen their runs until a layer has at most this many items
  int32_t target_items_whole;  // > 0: the same for launches over the whole model
  int32_t n_cus;               // compute units of the device
  int32_t select_long_rows;    // caches with more capacity than this are ranked tile by tile at eviction
  int32_t lag_gp_log2;         // score tracking: log2 of G rounded up to 4, 8 or 16 (rows a call takes in a record)
  struct Schedule {
    int32_t chunk = 0;
    bool fill = false;                 // runs of fewer rows where those would leave compute units idle (the default)
    std::vector<int32_t> max_count;    // layer -> longest work item of the layer, rows
    std::vector<int32_t> max_split;    // layer -> most work items of a cache
    std::vector<int32_t> cib;          // cache -> first item
    std::vector<int32_t> multi_begin;  // layer -> first entry of the list of multi-item caches
  } sched[3];                          // 0: layer sub-range launches, 1: whole-model launches, 2: see schedule_for
  WorkspacePlan plan;
  char* ws;
  int32_t time_kernel;         // 0 off, 1 events recorded around the attention kernel, 2 events carried by its dispatch
  bool track_on;               // score tracking in force (BAKLAVA_OPT_TRACK_SCORES pauses it)
  std::vector<hipEvent_t> ev;  // pairs (before, after); the first 2 * ev_used are recorded
  size_t ev_used;
};

namespace {

// Work items per compute unit that a launch over the whole model aims at: runs long enough to amortise the per-item
// costs (a merge of the wavefronts, and of the split partials), yet enough of them to even out the load.  Two run side by
// side on a compute unit, so two are best while every cache can still be cut into about four (as for one wave of a layer),
// three up to the next line and five beyond; where two would make runs of more than 8192 rows, four, whose scores fit
// the LDS they wait in.  us per call with five / by the rule, attention alone and tracked: bf16, D = 128, four heads, 32
// caches of 4096 rows 17.1 / 16.4 and 24.8 / 22.9, 64 27.9 / 24.9 and 36.6 / 33.0, 128 47.2 / 45.0 and 59.4 / 55.9, 192
// (three) 66.7 / 65.3 and 82.1 / 80.3; D = 64, 64 18.1 / 15.3 and 29.6 / 24.1; fp32, D = 128, 64 53.3 / 47.0 and 68.9 / 55.8;
// 128 caches of 65536 rows (four) 632 / 627 and 733 / 724, with two 628 and 736; 256 of 8192 rows with four instead of five
// 160 / 163 (one head) and 165 / 165, with two 197.
int whole_items_per_cu(int64_t n_caches, int64_t rows, int64_t cus) {
  if (4 * n_caches <= 2 * cus) return rows <= 2 * cus * 8192 ? 2 : 4;
  if (4 * n_caches <= 3 * cus) return 3;
  return kWholeItemsPerCu;
}

// Builds one of the split-K schedules with the host planner and uploads it.  Schedules 0 and 2
// serve launches over a layer sub-range (launch order inside each layer, so a layer range is a
// contiguous slice), schedule 1 launches over the whole model.  The table depends on capacities
// only, so it is uploaded once; the kernels clamp each run to the live length.
//
// fill: the default schedules, until an option asks for a run length or an item count.  A launch whose caches the
// shortest run already cuts, so that it merges partials anyway, but into fewer work items than there are compute units,
// takes runs of 64 rows and more, as long as they make one wave: a compute unit reads some 30 to 45 GB/s whatever it
// is given.  us per call of a layer of 8 caches (shortest run 512) / now, bf16, D = 128, four query heads, tracked:
// 8192 rows in all 13.7 / 12.0, 32768 14.9 / 12.7, 65536 16.1 / 15.0; attention alone, one head, 8192 10.1 / 7.6; fp32,
// D = 128, four heads, 8192 20.1 / 10.1, 32768 22.1 / 13.9.  Runs of at least 128 rows are equal but in the vector kernel
// (8192 rows 12.7).  A launch of unsplit caches stays: cut, it would need a merge (8 bf16 caches of 384 rows 6.2 us, cut
// 7.3; of 128 rows 4.4, cut 7.2), except on the vector kernel from four heads on, whose shortest run is 256 rows (8 caches,
// four heads, D = 128, 320 rows 12.2, cut 9.2, 500 rows 17.1, cut 9.3; D = 64, 264 rows 7.8, cut 8.3, tracked 13.1, cut
// 11.1, 384 rows 8.8, cut 8.2; eight heads 264 rows 12.8, cut 11.1).
int build_schedule(baklava_ctx* ctx, int which, int chunk, bool fill) {
  int64_t n_items = 0;
  // The list of multi-item caches and the work items lie next to each other in the workspace, so they are formed that
  // way here and travel in one copy (each takes about 20 us).
  const size_t front = ctx->plan.items[which] - ctx->plan.multi[which];
  std::unique_ptr<char[]> both(new (std::nothrow) char[front + (size_t)ctx->plan.max_items * sizeof(Item)]);
  if (!both) return BAKLAVA_ENOMEM;
  MultiCache* const multi = reinterpret_cast<MultiCache*>(both.get());
  baklava_work_item* const items = reinterpret_cast<baklava_work_item*>(both.get() + front);
  const int st = plan_schedule(ctx->off.data(), ctx->cap.data(), ctx->d.L, ctx->cpl, chunk,
                               which == 1 ? ctx->target_items_whole : ctx->target_items, kShortestRun,
                               fill ? std::min(ctx->n_cus, kMostFillItems) : 0, which == 1, ctx->plan.max_items,
                               items, &n_items);
  if (st != BAKLAVA_OK) return st;
  if (which == 2 && n_items == ctx->sched[0].cib.back()) return BAKLAVA_OK;  // the same work items: schedule 0 serves
  static_assert(sizeof(baklava_work_item) == sizeof(Item), "work item layouts must match");
  // cache -> first partial slot, and the caches that need the combine kernel (in launch order)
  std::vector<int32_t> cib(ctx->n_caches + 1, 0), multi_begin(ctx->d.L + 1, 0);
  size_t n_multi = 0;
  std::vector<int32_t> max_count(ctx->d.L, 0), max_split(ctx->d.L, 0);
  int32_t slot0 = 0;  // the items of a cache follow each other
  for (int64_t i = 0; i < n_items; ++i) {
    if (items[i].start == 0) slot0 = items[i].slot;
    items[i].reserved = slot0;
    const baklava_work_item& it = items[i];
    max_count[it.cache / ctx->cpl] = std::max(max_count[it.cache / ctx->cpl], it.count);
    max_split[it.cache / ctx->cpl] = std::max(max_split[it.cache / ctx->cpl], it.nsplit);
    if (it.start == 0) {
      cib[it.cache] = it.slot;
      if (it.nsplit > 1) {
        multi[n_multi++] = MultiCache{it.cache, it.slot, it.slot + it.nsplit, 0};
        multi_begin[it.cache / ctx->cpl + 1] += 1;
      }
    }
  }
  cib[ctx->n_caches] = (int32_t)n_items;
  for (int32_t l = 0; l < ctx->d.L; ++l) multi_begin[l + 1] += multi_begin[l];
  if (!hip_ok(hipDeviceSynchronize())) return BAKLAVA_EHIP;  // no launch may still read the old table
  const size_t skip = n_multi ? 0 : front;
  std::memset(multi + n_multi, 0, n_multi ? front - n_multi * sizeof(MultiCache) : 0);
  if (!hip_ok(hipMemcpy(ctx->ws + ctx->plan.multi[which] + skip, both.get() + skip, front - skip + (size_t)n_items * sizeof(Item),
                        hipMemcpyHostToDevice)))
    return BAKLAVA_EHIP;
  ctx->sched[which].cib.swap(cib);
  ctx->sched[which].multi_begin.swap(multi_begin);
  ctx->sched[which].chunk = chunk;
  ctx->sched[which].fill = fill;
  ctx->sched[which].max_count.swap(max_count);
  ctx->sched[which].max_split.swap(max_split);
  return BAKLAVA_OK;
}

// fp32 rows for four query heads and more: the vector kernel is bound by its arithmetic there, so short runs pay earlier.
// The matrix kernel, which takes over from five on, is bound by HBM and indifferent: a layer of 8 caches of 1000 to 32768
// rows within 4% with either rule.
bool slow_rows(const baklava_ctx* ctx) { return ctx->d.dtype == BAKLAVA_F32 && ctx->G >= 4; }

// fp32 rows from five query heads on: the vector kernel, which takes eight then, is bound by its arithmetic, the matrix
// kernel (which always takes sixteen, of which at most eight are there) by HBM.  us per call, vector / matrix kernel,
// without scores and tracked, 32 caches of 4096 rows a layer and 64 in one launch: D = 128, one head 25.0 / 27.5 and 43.9 / 48.8; four 29.7 / 30.0, 32.1 / 31.2 and 49.7 /
// 52.5, 53.7 / 54.9; five 44.0 / 30.5, 47.4 / 33.2 and 69.0 / 51.9, 82.3 / 56.4; eight 44.0 / 31.2, 50.6 / 35.2 and 76.4 /
// 52.2, 85.3 / 60.6; D = 64, four 18.0 / 18.0 and 27.3 / 28.1, eight 26.0 / 19.9 and 38.6 / 30.7.  8 caches of 300 rows,
// D = 128, eight heads 13.3 / 11.9, of 32768 rows 67.7 / 52.2; 40 of 30 rows 7.8 / 7.8, tracked 11.7 / 11.9.
bool f32_on_matrix_cores(const baklava_ctx* ctx) { return ctx->d.dtype == BAKLAVA_F32 && ctx->G >= 5; }

// Which schedule a launch over the layers takes.  The short runs of schedule 0 give a single layer a work item for every
// compute unit; over several layers that is more work items than the launch needs, each with its share of the merge.
// Beyond two for each compute unit (four where rows are slow) a launch takes the runs that the layers would have
// without the fill.  us per call over 2, 3, 4, 5, 7 layers of 8 caches, short runs / without, four query heads:
//   bf16, D = 128    8192 rows a layer   8.7 / 10.9    9.2 / 11.4   10.7 / 11.5   11.9 / 11.7   13.8 / 12.1
//                   32768               12.8 / 12.8   14.5 / 13.5   18.3 / 17.7   19.5 / 19.9   25.4 / 22.2
//                   65536               17.0 / 19.0   21.9 / 21.5   27.3 / 27.8   29.8 / 31.8   41.8 / 41.4
//   D = 64, tracked 16384               12.5 / 12.1   15.1 / 13.5   17.5 / 13.6   20.6 / 16.4   25.8 / 16.9
//   fp32, D = 128    8192               12.2 / 21.3   12.9 / 21.6   14.6 / 21.7   15.2 / 21.9   18.6 / 22.3
//                   32768               19.7 / 22.0   24.1 / 23.1   31.7 / 30.8   33.8 / 35.5   46.1 / 41.8
int schedule_for(const baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count) {
  if (layer_begin == 0 && layer_count == ctx->d.L) return 1;
  const baklava_ctx::Schedule& sc = ctx->sched[0];
  if (layer_count == 1 || !sc.fill || ctx->sched[2].cib.empty()) return 0;
  const int32_t c0 = layer_begin * ctx->cpl, c1 = c0 + layer_count * ctx->cpl;
  return sc.cib[c1] - sc.cib[c0] > (slow_rows(ctx) ? 4 : 2) * ctx->n_cus ? 2 : 0;
}

// Tile tables of the eviction's selection (they depend on capacities and the threshold only), in cache order, so that
// the tiles of a layer range are a contiguous slice: one of the long caches, one of all others (spread; a single entry
// for those of up to kNarrowRows rows).  The two share the tile counters.  Without a cache of several tiles the second
// table is never read, and not uploaded.
int build_tiles(baklava_ctx* ctx) {
  std::vector<SelTile> tiles, spread;
  const int64_t n_caches = ctx->n_caches;
  std::vector<int32_t> tile_begin(n_caches + 1, 0), spread_begin(n_caches + 1, 0);
  int32_t n_long = 0, counters = 0;
  bool any_spread = false;
  for (int64_t c = 0; c < n_caches; ++c) {
    tile_begin[c] = (int32_t)tiles.size();
    spread_begin[c] = (int32_t)spread.size();
    const bool is_long = ctx->cap[c] > ctx->select_long_rows;
    const int32_t nt = is_long || ctx->cap[c] > kNarrowRows ? (int32_t)(((int64_t)ctx->cap[c] + kTileRows - 1) / kTileRows) : 1;
    for (int32_t t = 0; t < nt; ++t)
      (is_long ? tiles : spread).push_back(SelTile{(int32_t)c, t, counters, nt, is_long ? n_long : 0, 0});
    if (is_long || nt > 1) counters += nt;
    any_spread = any_spread || (!is_long && nt > 1);
    n_long += is_long ? 1 : 0;
  }
  tile_begin[n_caches] = (int32_t)tiles.size();
  spread_begin[n_caches] = (int32_t)spread.size();
  if (counters > ctx->plan.n_tiles || (int64_t)spread.size() > ctx->plan.n_tiles + n_caches || n_long > ctx->plan.n_long)
    return BAKLAVA_ECAPACITY;
  if (!hip_ok(hipDeviceSynchronize())) return BAKLAVA_EHIP;  // no launch may still read the old tables
  if ((!tiles.empty() &&
       !hip_ok(hipMemcpy(ctx->ws + ctx->plan.tiles, tiles.data(), tiles.size() * sizeof(SelTile), hipMemcpyHostToDevice))) ||
      (any_spread &&
       !hip_ok(hipMemcpy(ctx->ws + ctx->plan.spread, spread.data(), spread.size() * sizeof(SelTile), hipMemcpyHostToDevice))))
    return BAKLAVA_EHIP;
  ctx->tile_begin.swap(tile_begin);
  ctx->spread_begin.swap(spread_begin);
  return BAKLAVA_OK;
}

// Whether several workgroups rank each of the range's caches of more than kNarrowRows rows.  Every one of them reads the
// scores of its cache, so this pays while they find compute units that would idle: far up to one for each, little from
// there to three for two, beyond which it loses to caches of just over two tiles or without shorter ones beside them
// (which one workgroup ranks, and which otherwise wait for a launch of their own).  us of ranking, one workgroup per
// cache / spread (workgroups of the caches of more than kNarrowRows rows):
//   alone                   16500 rows  29.6 / 30.8 (258)  29.6 / 32.8 (384)  29.7 / 32.6 (510)
//                           32768       33.8 / 22.6 (256)  34.0 / 34.6 (384)  35.1 / 37.6 (512)
//                           65536       43.3 / 28.4 (256)  43.6 / 43.8 (384)  44.2 / 46.3 (512)
//   beside 64 shorter ones  16500       43.1 / 37.8 (258)  43.9 / 39.9 (384)  43.8 / 42.1 (510)
//                           32768       48.0 / 31.1 (256)  48.5 / 42.1 (384)  49.2 / 47.5 (512)
//   beside 500              16500       49.6 / 45.8 (258)  50.2 / 52.4 (384)  50.5 / 54.7 (510)
//                           32768       54.2 / 40.2 (256)  55.0 / 52.1 (384)  54.3 / 65.6 (560)
//                           65536       64.2 / 44.8 (256)  64.2 / 61.1 (384)  64.9 / 64.8 (512)
// Whole evictions: 88 caches of 32768 rows (352) 347 / 346, 44 of 65536 (352) 355 / 353, 96 of 16500 (288) 234 / 234.
bool spread_selection(const baklava_ctx* ctx, int64_t c0, int64_t c1) {
  int64_t tiles = 0;
  for (int64_t c = c0; c < c1; ++c) {
    const int32_t nt = ctx->spread_begin[c + 1] - ctx->spread_begin[c];
    tiles += nt > 1 ? nt : 0;
  }
  return tiles > 0 && 2 * tiles <= 3 * (int64_t)ctx->n_cus;
}

bool range_ok(const baklava_ctx* ctx, int32_t lb, int32_t lc) {
  return lb >= 0 && lc > 0 && (int64_t)lb + lc <= ctx->d.L;
}

// The weights of the calls on record go to the score plane now (see DecodeParams): a pass over the
// K rows of the layer range, after which the records are empty.  Only the MFMA attention kernel over rows of
// 128 elements leaves calls on record.
int flush_records(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count, hipStream_t s) {
  if (!ctx->d.track_scores || !keeps_records(&ctx->d)) return BAKLAVA_OK;
  const int64_t c0 = (int64_t)layer_begin * ctx->cpl;
  const int64_t c1 = c0 + (int64_t)layer_count * ctx->cpl;
  const int which = schedule_for(ctx, layer_begin, layer_count);
  const baklava_ctx::Schedule& sc = ctx->sched[which];
  const int32_t i0 = sc.cib[c0], i1 = sc.cib[c1];
  DecodeParams p{};
  p.k = ctx->d.k; p.score = ctx->d.score;
  p.items = reinterpret_cast<const Item*>(ctx->ws + ctx->plan.items[which]) + i0;
  p.lag_q = ctx->ws + ctx->plan.lag_q;
  p.lag_ml = reinterpret_cast<float*>(ctx->ws + ctx->plan.lag_ml);
  p.lag_n = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.lag_n);
  p.lag_cnt = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.lag_cnt);
  // The flush empties the records itself while no cache has more work items than draw a ticket faster than a launch
  // behind the flush takes (see score_flush_mfma).
  const bool self_clear = *std::max_element(sc.max_split.begin() + layer_begin,
                                            sc.max_split.begin() + layer_begin + layer_count) <= kMostTickets;
  p.flush_ticket = self_clear ? reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.flush_ticket) : nullptr;
  p.G = ctx->G; p.lag_gp_log2 = ctx->lag_gp_log2;
  p.scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)ctx->d.D));
  const int32_t longest = *std::max_element(sc.max_count.begin() + layer_begin,
                                            sc.max_count.begin() + layer_begin + layer_count);
  if (!hip_ok(launch_score_flush_mfma(p, i1 - i0, longest, s))) return BAKLAVA_EHIP;
  if (!self_clear && !hip_ok(launch_fill_i32(p.lag_cnt + c0 * ctx->G, 0, (c1 - c0) * ctx->G, s))) return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}

// The score update of a call on the vector kernel over rows whose calls are otherwise recorded, for the one that
// has just been enqueued.
int score_pass(baklava_ctx* ctx, const DecodeParams& d, int n_items, int longest, hipStream_t s) {
  ScoreParams p;
  p.k = d.k; p.q = d.q;
  p.ml = d.final_ml;
  p.len = d.len;
  p.items = d.items;
  p.score = d.score;
  p.G = d.G; p.Hq = d.Hq; p.Hkv = d.Hkv;
  p.cache_begin = d.cache_begin;
  p.scale_log2e = d.scale_log2e;
  if (!hip_ok(launch_score_pass(p, n_items, longest, s))) return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}

// host_lengths: the host mirror of the lengths is checked and advanced (the calls that take the token
// position by value); otherwise the device tables alone decide and evolve.
int decode_impl(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count, const void* k_new,
                const void* v_new, int32_t token_pos, const int32_t* token_pos_dev, bool host_lengths,
                const void* q, float* out, void* stream) {
  const bool fused = k_new != nullptr;
  const int64_t c0 = (int64_t)layer_begin * ctx->cpl;
  const int64_t c1 = c0 + (int64_t)layer_count * ctx->cpl;
  if (host_lengths) {
    for (int64_t c = c0; c < c1; ++c) {
      if (fused && ctx->len[c] >= ctx->cap[c]) return BAKLAVA_ECAPACITY;
      if (!fused && ctx->len[c] <= 0) return BAKLAVA_ESTATE;
    }
  }
  const int which = schedule_for(ctx, layer_begin, layer_count);
  const baklava_ctx::Schedule& sc = ctx->sched[which];
  const int32_t i0 = sc.cib[c0], i1 = sc.cib[c1];
  hipStream_t s = (hipStream_t)stream;
  const bool use_mfma = ctx->kernel_pref == 2 || (ctx->kernel_pref == 0 && ctx->d.dtype == BAKLAVA_BF16);
  const bool track = ctx->track_on;
  // Scores are deferred over rows of 128 elements only: those of 64 have always been current when a call
  // returns, and callers read them, set them or declare new lengths between calls without a flush.
  const bool defer = track && use_mfma && ctx->d.D == 128;
  // Other calls add their weights right away; weights an earlier call left pending come first, so that the
  // scores grow in the order of the calls.
  if (track && !defer) {
    const int st = flush_records(ctx, layer_begin, layer_count, s);
    if (st != BAKLAVA_OK) return st;
  }
  DecodeParams p;
  p.k = ctx->d.k; p.v = ctx->d.v; p.q = q; p.out = out;
  p.off = ctx->d.off; p.len = ctx->d.len;
  // Slots are numbered cache by cache and the launch order only permutes caches inside a layer
  // (schedule 0), so the launch-ordered table of a layer range is the slice [i0, i1).
  p.items = reinterpret_cast<const Item*>(ctx->ws + ctx->plan.items[which]) + i0;
  p.part_o = reinterpret_cast<float*>(ctx->ws + ctx->plan.part_o);
  p.part_ml = reinterpret_cast<float*>(ctx->ws + ctx->plan.part_ml);
  p.final_ml = reinterpret_cast<float*>(ctx->ws + ctx->plan.final_ml);
  p.lag_q = ctx->ws + ctx->plan.lag_q;
  p.lag_ml = reinterpret_cast<float*>(ctx->ws + ctx->plan.lag_ml);
  p.lag_n = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.lag_n);
  p.lag_cnt = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.lag_cnt);
  p.cap = ctx->d.cap;
  p.score = ctx->d.score;
  p.pos = ctx->d.pos;
  const int32_t m0 = sc.multi_begin[layer_begin], m1 = sc.multi_begin[layer_begin + layer_count];
  p.multi = reinterpret_cast<const MultiCache*>(ctx->ws + ctx->plan.multi[which]) + m0;
  p.k_new = k_new; p.v_new = v_new;
  p.token_pos_dev = token_pos_dev;
  p.status = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.status);
  p.G = ctx->G; p.Hq = ctx->d.Hq; p.Hkv = ctx->d.Hkv; p.batch = ctx->d.batch;
  p.cache_begin = (int32_t)c0;
  p.lag = defer ? 1 : 0;
  p.lag_batch = kLagRows >> ctx->lag_gp_log2;
  p.lag_gp_log2 = ctx->lag_gp_log2;
  p.ring_slots = 0;
  const bool from_logits = track && !keeps_records(&ctx->d);
  p.logits = from_logits ? reinterpret_cast<float*>(ctx->ws + ctx->plan.logits) : nullptr;
  p.logit_stride = ctx->total_tokens;
  const int32_t longest = *std::max_element(sc.max_count.begin() + layer_begin,
                                            sc.max_count.begin() + layer_begin + layer_count);
  p.fused_append = fused ? 1 : 0;
  p.token_pos = token_pos;
  p.row_bytes = ctx->row_bytes;
  p.scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)ctx->d.D));
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  if (ctx->time_kernel) {
    while (ctx->ev.size() < 2 * (ctx->ev_used + 1)) {
      hipEvent_t e;
      if (!hip_ok(hipEventCreate(&e))) return BAKLAVA_EHIP;
      ctx->ev.push_back(e);
    }
    ev0 = ctx->ev[2 * ctx->ev_used];
    ev1 = ctx->ev[2 * ctx->ev_used + 1];
    if (!(ctx->time_kernel == 2 && use_mfma) && !hip_ok(hipEventRecord(ev0, s))) return BAKLAVA_EHIP;
  }
  const bool on_dispatch = ctx->time_kernel == 2 && use_mfma;
  hipError_t e = use_mfma ? launch_decode_mfma(p, ctx->d.D, i1 - i0, longest, i1 - i0 <= ctx->n_cus, s,
                                               on_dispatch ? ev0 : nullptr, on_dispatch ? ev1 : nullptr)
               : ctx->kernel_pref == 0 && f32_on_matrix_cores(ctx)
                          ? launch_decode_mfma_f32(p, ctx->d.D, i1 - i0, longest, i1 - i0 <= ctx->n_cus, s)
                          : launch_decode_valu(p, ctx->d.dtype, ctx->d.D, i1 - i0, longest, i1 - i0 <= ctx->n_cus, s);
  if (!hip_ok(e)) return BAKLAVA_EHIP;
  if (ctx->time_kernel) {
    if (!on_dispatch && !hip_ok(hipEventRecord(ev1, s))) return BAKLAVA_EHIP;
    ctx->ev_used += 1;
  }
  const int32_t most_split = *std::max_element(sc.max_split.begin() + layer_begin,
                                               sc.max_split.begin() + layer_begin + layer_count);
  if (from_logits) {
    if (!hip_ok(launch_finish(p, ctx->d.D, m1 - m0, most_split, i1 - i0, longest, s))) return BAKLAVA_EHIP;
  } else {
    if (!hip_ok(launch_combine(p, ctx->d.D, m1 - m0, most_split, s))) return BAKLAVA_EHIP;
    if (track && !defer) {
      const int st = score_pass(ctx, p, i1 - i0, longest, s);
      if (st != BAKLAVA_OK) return st;
    }
  }
  if (fused && host_lengths)
    for (int64_t c = c0; c < c1; ++c) ctx->len[c] += 1;
  return BAKLAVA_OK;
}

}  // namespace

void baklava::note_hip_error(hipError_t e) { g_last_hip_error = (int)e; }

extern "C" int baklava_last_hip_error(void) { return g_last_hip_error; }

extern "C" size_t baklava_workspace_bytes(const baklava_desc* desc, const int32_t* cap_host,
                                          const int32_t* budget_host) {
  if (!shape_ok(desc) || !cap_host || !budget_host) return 0;
  const int64_t n_caches = (int64_t)desc->L * desc->batch * desc->Hkv;
  for (int64_t c = 0; c < n_caches; ++c)
    if (cap_host[c] < 0) return 0;
  for (int64_t i = 0; i < (int64_t)desc->L * desc->Hkv; ++i)
    if (budget_host[i] < 0) return 0;
  return plan_workspace(desc, cap_host).total;
}

extern "C" int baklava_create(const baklava_desc* desc, const int64_t* off_host, const int32_t* cap_host,
                              const int32_t* len_host, const int32_t* budget_host, baklava_ctx** out) {
  if (!out) return BAKLAVA_EINVAL;
  *out = nullptr;
  if (!shape_ok(desc) || !off_host || !cap_host || !budget_host) return BAKLAVA_EINVAL;
  if (!desc->k || !desc->v || !desc->score || !desc->pos || !desc->off || !desc->cap || !desc->len ||
      !desc->budget || !desc->workspace)
    return BAKLAVA_EINVAL;
  if (((uintptr_t)desc->k | (uintptr_t)desc->v) & 15) return BAKLAVA_EINVAL;
  if ((uintptr_t)desc->workspace & 255) return BAKLAVA_EINVAL;
  const int64_t n_caches = (int64_t)desc->L * desc->batch * desc->Hkv;
  const int64_t m = (int64_t)desc->L * desc->Hkv;
  for (int64_t i = 0; i < m; ++i) {
    if (budget_host[i] < 0) return BAKLAVA_EINVAL;
    const int need = desc->policy == BAKLAVA_POLICY_SCORE ? desc->sink + desc->recent : desc->sink;
    if (budget_host[i] < need) return BAKLAVA_EINFEASIBLE;
  }
  // The arena must be packed as baklava_layout lays it out (off[c] = capacities before c): the
  // workspace planes that run parallel to the arena (kept lists) are indexed by the same offsets.
  int64_t packed = 0;
  for (int64_t c = 0; c < n_caches; ++c) {
    if (cap_host[c] < 0 || off_host[c] != packed) return BAKLAVA_EINVAL;
    packed += cap_host[c];
    if (len_host && (len_host[c] < 0 || len_host[c] > cap_host[c])) return BAKLAVA_ECAPACITY;
  }
  baklava_ctx* ctx = new (std::nothrow) baklava_ctx();
  if (!ctx) return BAKLAVA_ENOMEM;
  ctx->d = *desc;
  ctx->n_caches = n_caches;
  ctx->total_tokens = packed;
  ctx->cpl = desc->batch * desc->Hkv;
  ctx->G = desc->Hq / desc->Hkv;
  ctx->row_bytes = desc->D * (desc->dtype == BAKLAVA_BF16 ? 2 : 4);
  ctx->lag_gp_log2 = ctx->G <= 4 ? 2 : ctx->G <= 8 ? 3 : 4;
  ctx->off.assign(off_host, off_host + n_caches);
  ctx->cap.assign(cap_host, cap_host + n_caches);
  if (len_host) ctx->len.assign(len_host, len_host + n_caches);
  else ctx->len.assign(n_caches, 0);
  ctx->budget.assign(budget_host, budget_host + m);
  ctx->kernel_pref = 0;
  // A launch over part of the layers is one wave of workgroups: at most one per compute unit.
  {
    int dev = 0, cus = 0;
    if (!hip_ok(hipGetDevice(&dev)) ||
        !hip_ok(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev))) {
      delete ctx;
      return BAKLAVA_EHIP;
    }
    // One wave only pays while every cache can still be cut into about four work items; with more
    // caches per layer the runs differ too much in length and several waves of shorter items
    // balance better (measured on llama32-shaped layers: 64 caches per layer, one wave +6%;
    // 128 caches, five items per compute unit +4%; 256 caches, +48%).
    ctx->layer_one_wave = (int64_t)ctx->cpl * 4 <= cus;
    ctx->target_items = ctx->layer_one_wave ? cus : kWholeItemsPerCu * cus;
    ctx->n_cus = cus;
    ctx->target_items_whole = whole_items_per_cu(n_caches, packed, cus) * cus;
  }
  ctx->time_kernel = 0;
  ctx->track_on = desc->track_scores != 0;
  ctx->ev_used = 0;
  ctx->plan = plan_workspace(desc, cap_host);
  ctx->ws = reinterpret_cast<char*>(desc->workspace);
  if (desc->workspace_bytes < ctx->plan.total) { delete ctx; return BAKLAVA_ECAPACITY; }

  // Launch orders: longest caches first, over the whole model and within each layer.
  auto longer = [&](int32_t a, int32_t b) { return ctx->cap[a] > ctx->cap[b]; };
  ctx->order_all.resize(n_caches);
  std::iota(ctx->order_all.begin(), ctx->order_all.end(), 0);
  ctx->order_layer = ctx->order_all;
  std::stable_sort(ctx->order_all.begin(), ctx->order_all.end(), longer);
  for (int32_t l = 0; l < desc->L; ++l)
    std::stable_sort(ctx->order_layer.begin() + (int64_t)l * ctx->cpl,
                     ctx->order_layer.begin() + (int64_t)(l + 1) * ctx->cpl, longer);
  {  // the two lie next to each other in the workspace: one copy (each takes about 20 us)
    std::vector<int32_t> both((ctx->plan.order_layer - ctx->plan.order_all) / 4 + n_caches, 0);
    std::copy(ctx->order_all.begin(), ctx->order_all.end(), both.begin());
    std::copy(ctx->order_layer.begin(), ctx->order_layer.end(), both.end() - n_caches);
    if (!hip_ok(hipMemcpy(ctx->ws + ctx->plan.order_all, both.data(), both.size() * 4, hipMemcpyHostToDevice))) {
      delete ctx;
      return BAKLAVA_EHIP;
    }
  }
  // No call is pending for the score pass, and the status word is clear.
  if (!hip_ok(hipMemset(ctx->ws + ctx->plan.lag_cnt, 0, (size_t)n_caches * (ctx->G + kTicketStride) * 4)) ||
      !hip_ok(hipMemset(ctx->ws + ctx->plan.status, 0, 256))) {
    delete ctx;
    return BAKLAVA_EHIP;
  }
  // Work of the eviction move, at most (rows move from the first evicted one on; none of a cache whose budget is not
  // below its capacity).
  ctx->move_before.assign(n_caches + 1, MoveCount{0, 0});
  for (int64_t c = 0; c < n_caches; ++c) {
    const int64_t rows = move_rows(ctx->row_bytes / 16), most_short = move_short_rows(ctx->row_bytes / 16);
    const int64_t b = ctx->budget[(c / ctx->cpl) * desc->Hkv + c % desc->Hkv];
    MoveCount& m = ctx->move_before[c + 1];
    m = ctx->move_before[c];
    if (b < ctx->cap[c] && b > most_short) m.tiles += (b + rows - 1) / rows;
    if (b < ctx->cap[c] && b <= most_short) m.short_caches += 1;
  }
  // Eviction: a cache of up to kHeldRows rows is ranked by one workgroup that holds its scores in
  // registers, or by several (see spread_selection), a longer one tile by tile.  Measured, us per eviction,
  // one workgroup against tiles: 8 caches of 15000 rows 57 / 90, of 30000 87 / 103, of 60000 121 / 132; 256
  // caches 449 / 489, 862 / 914, 1716 / 1838.
  ctx->select_long_rows = kHeldRows;
  ctx->n_wide.assign(desc->L, 0);
  for (int64_t c = 0; c < n_caches; ++c) ctx->n_wide[c / ctx->cpl] += ctx->cap[c] > kNarrowRows ? 1 : 0;
  {
    const int st = build_tiles(ctx);
    if (st != BAKLAVA_OK) { delete ctx; return st; }
  }
  if (desc->dtype == BAKLAVA_BF16 && !hip_ok(prepare_decode_mfma())) { delete ctx; return BAKLAVA_EHIP; }
  if (desc->dtype == BAKLAVA_F32 && !hip_ok(prepare_decode_mfma_f32())) { delete ctx; return BAKLAVA_EHIP; }
  const int chunk = ctx->layer_one_wave ? kDefaultChunk : kDefaultChunkWhole;
  const int chunk_layer = slow_rows(ctx) ? kDefaultChunkWhole : chunk;  // (see build_schedule)
  int st = build_schedule(ctx, 0, chunk_layer, true);
  if (st == BAKLAVA_OK) st = build_schedule(ctx, 1, kDefaultChunkWhole, true);
  if (st == BAKLAVA_OK && desc->L > 2) st = build_schedule(ctx, 2, chunk, false);
  if (st != BAKLAVA_OK) { delete ctx; return st; }
  *out = ctx;
  return BAKLAVA_OK;
}

extern "C" int baklava_destroy(baklava_ctx* ctx) {
  if (!ctx) return BAKLAVA_EINVAL;
  for (hipEvent_t e : ctx->ev) (void)hipEventDestroy(e);
  delete ctx;
  return BAKLAVA_OK;
}

extern "C" int baklava_set_option(baklava_ctx* ctx, int32_t option, int64_t value) {
  if (!ctx) return BAKLAVA_EINVAL;
  switch (option) {
    case BAKLAVA_OPT_CHUNK_TOKENS:
    case BAKLAVA_OPT_CHUNK_TOKENS_WHOLE: {
      if (value < kMinChunk || value % 64 || value > kMaxChunk) return BAKLAVA_EINVAL;
      const int which = option == BAKLAVA_OPT_CHUNK_TOKENS ? 0 : 1;
      if ((int32_t)value == ctx->sched[which].chunk && !ctx->sched[which].fill) return BAKLAVA_OK;
      return build_schedule(ctx, which, (int32_t)value, false);
    }
    case BAKLAVA_OPT_TARGET_ITEMS:
    case BAKLAVA_OPT_TARGET_ITEMS_WHOLE: {
      if (value < 0 || value > (1 << 20)) return BAKLAVA_EINVAL;
      const int which = option == BAKLAVA_OPT_TARGET_ITEMS ? 0 : 1;
      int32_t& target = which == 0 ? ctx->target_items : ctx->target_items_whole;
      if ((int32_t)value == target && !ctx->sched[which].fill) return BAKLAVA_OK;
      target = (int32_t)value;
      return build_schedule(ctx, which, ctx->sched[which].chunk, false);
    }
    case BAKLAVA_OPT_KERNEL:
      if (value < 0 || value > 2) return BAKLAVA_EINVAL;
      if (value == 2 && !(ctx->d.dtype == BAKLAVA_BF16 && ctx->d.D == 128)) return BAKLAVA_EINVAL;
      if (value == 1 && ctx->G > 8) return BAKLAVA_EINVAL;
      ctx->kernel_pref = (int32_t)value;
      return BAKLAVA_OK;
    case BAKLAVA_OPT_TILED_SELECT_ROWS: {
      if (value < kMinLongRows || value > INT32_MAX) return BAKLAVA_EINVAL;
      if (std::min<int64_t>(value, kHeldRows) == ctx->select_long_rows) return BAKLAVA_OK;
      const int32_t old = ctx->select_long_rows;
      ctx->select_long_rows = (int32_t)std::min<int64_t>(value, kHeldRows);
      const int st = build_tiles(ctx);
      if (st != BAKLAVA_OK) ctx->select_long_rows = old;
      return st;
    }
    case BAKLAVA_OPT_TRACK_SCORES:
      if (value != 0 && value != 1) return BAKLAVA_EINVAL;
      if (value == 1 && !ctx->d.track_scores) return BAKLAVA_EINVAL;  // the workspace holds no records
      ctx->track_on = value == 1;
      return BAKLAVA_OK;
    case BAKLAVA_OPT_TIME_KERNEL:
      if (value < 0 || value > 2) return BAKLAVA_EINVAL;
      if (ctx->ev_used && value != ctx->time_kernel) return BAKLAVA_ESTATE;  // read the pending record first
      ctx->time_kernel = (int32_t)value;
      return BAKLAVA_OK;
    default:
      return BAKLAVA_EINVAL;
  }
}

extern "C" int baklava_profile_read(baklava_ctx* ctx, double* total_ms_out, int64_t* launches_out) {
  if (!ctx || !total_ms_out || !launches_out) return BAKLAVA_EINVAL;
  double total = 0.0;
  for (size_t i = 0; i < ctx->ev_used; ++i) {
    if (!hip_ok(hipEventSynchronize(ctx->ev[2 * i + 1]))) return BAKLAVA_EHIP;
    float ms = 0.f;
    if (!hip_ok(hipEventElapsedTime(&ms, ctx->ev[2 * i], ctx->ev[2 * i + 1]))) return BAKLAVA_EHIP;
    total += ms;
  }
  *total_ms_out = total;
  *launches_out = (int64_t)ctx->ev_used;
  ctx->ev_used = 0;
  return BAKLAVA_OK;
}

extern "C" int baklava_reset(baklava_ctx* ctx, void* stream) {
  if (!ctx) return BAKLAVA_EINVAL;
  if (!hip_ok(launch_fill_i32(ctx->d.len, 0, ctx->n_caches, (hipStream_t)stream))) return BAKLAVA_EHIP;
  if (!hip_ok(launch_fill_i32(reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.lag_cnt), 0, ctx->n_caches * ctx->G,
                              (hipStream_t)stream)))
    return BAKLAVA_EHIP;
  std::fill(ctx->len.begin(), ctx->len.end(), 0);
  return BAKLAVA_OK;
}

extern "C" int baklava_set_lengths(baklava_ctx* ctx, const int32_t* len_host, void* stream) {
  if (!ctx || !len_host) return BAKLAVA_EINVAL;
  for (int64_t c = 0; c < ctx->n_caches; ++c) {
    if (len_host[c] < 0) return BAKLAVA_EINVAL;
    if (len_host[c] > ctx->cap[c]) return BAKLAVA_ECAPACITY;
  }
  ctx->len.assign(len_host, len_host + ctx->n_caches);
  // Weights of a call over the old contents are not owed to the new ones: the records are emptied.
  int32_t* lag_cnt = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.lag_cnt);
  // Lengths that fit one launch's arguments travel with it (17 us for the call, of which most is the wait
  // below; 21 with a fill and a copy); from 1024 caches on the copy is as fast, from 2048 faster.
  if (ctx->n_caches <= kLengthsPerLaunch) {
    LengthsParams p;
    p.len = ctx->d.len; p.lag_cnt = lag_cnt;
    p.count = (int32_t)ctx->n_caches; p.G = ctx->G;
    std::memcpy(p.value, ctx->len.data(), ctx->n_caches * sizeof(int32_t));
    if (!hip_ok(launch_set_lengths(p, (hipStream_t)stream))) return BAKLAVA_EHIP;
  } else {
    if (!hip_ok(launch_fill_i32(lag_cnt, 0, ctx->n_caches * ctx->G, (hipStream_t)stream))) return BAKLAVA_EHIP;
    // The mirror is the staging buffer: wait for the copy so that later appends may change it.
    if (!hip_ok(hipMemcpyAsync(ctx->d.len, ctx->len.data(), ctx->n_caches * 4, hipMemcpyHostToDevice,
                               (hipStream_t)stream)))
      return BAKLAVA_EHIP;
  }
  // (the call has always synchronised: other streams may use the lengths once it returns)
  if (!hip_ok(hipStreamSynchronize((hipStream_t)stream))) return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}

extern "C" int baklava_append(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count,
                              const void* k_new, const void* v_new, int32_t token_pos, void* stream) {
  if (!ctx || !k_new || !v_new || !range_ok(ctx, layer_begin, layer_count)) return BAKLAVA_EINVAL;
  if (((uintptr_t)k_new | (uintptr_t)v_new) & 15) return BAKLAVA_EINVAL;
  const int64_t c0 = (int64_t)layer_begin * ctx->cpl;
  const int64_t c1 = c0 + (int64_t)layer_count * ctx->cpl;
  for (int64_t c = c0; c < c1; ++c)
    if (ctx->len[c] >= ctx->cap[c]) return BAKLAVA_ECAPACITY;
  AppendParams p;
  p.k = ctx->d.k; p.v = ctx->d.v; p.score = ctx->d.score; p.pos = ctx->d.pos;
  p.off = ctx->d.off; p.cap = ctx->d.cap; p.len = ctx->d.len;
  p.k_new = k_new; p.v_new = v_new;
  p.token_pos_dev = nullptr;
  p.cache_begin = (int32_t)c0; p.token_pos = token_pos; p.row_bytes = ctx->row_bytes;
  if (!hip_ok(launch_append(p, (int)(c1 - c0), (hipStream_t)stream))) return BAKLAVA_EHIP;
  for (int64_t c = c0; c < c1; ++c) ctx->len[c] += 1;
  return BAKLAVA_OK;
}

extern "C" int baklava_decode_attn(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count,
                                   const void* q, float* out, void* stream) {
  if (!ctx || !q || !out || !range_ok(ctx, layer_begin, layer_count)) return BAKLAVA_EINVAL;
  if (((uintptr_t)q & 15) || ((uintptr_t)out & 15)) return BAKLAVA_EINVAL;
  return decode_impl(ctx, layer_begin, layer_count, nullptr, nullptr, 0, nullptr, true, q, out, stream);
}

extern "C" int baklava_append_decode_attn(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count,
                                          const void* k_new, const void* v_new, int32_t token_pos,
                                          const void* q, float* out, void* stream) {
  if (!ctx || !q || !out || !k_new || !v_new || !range_ok(ctx, layer_begin, layer_count)) return BAKLAVA_EINVAL;
  if (((uintptr_t)q | (uintptr_t)out | (uintptr_t)k_new | (uintptr_t)v_new) & 15) return BAKLAVA_EINVAL;
  return decode_impl(ctx, layer_begin, layer_count, k_new, v_new, token_pos, nullptr, true, q, out, stream);
}

extern "C" int baklava_append_decode_attn_replay(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count,
                                                 const void* k_new, const void* v_new,
                                                 const int32_t* token_pos_dev, const void* q, float* out,
                                                 void* stream) {
  if (!ctx || !q || !out || !k_new || !v_new || !token_pos_dev || !range_ok(ctx, layer_begin, layer_count))
    return BAKLAVA_EINVAL;
  if (((uintptr_t)q | (uintptr_t)out | (uintptr_t)k_new | (uintptr_t)v_new) & 15) return BAKLAVA_EINVAL;
  if ((uintptr_t)token_pos_dev & 3) return BAKLAVA_EINVAL;
  return decode_impl(ctx, layer_begin, layer_count, k_new, v_new, 0, token_pos_dev, false, q, out, stream);
}

extern "C" int baklava_sync_lengths(baklava_ctx* ctx, void* stream) {
  if (!ctx) return BAKLAVA_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  int32_t status = 0;
  int32_t* status_dev = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.status);
  if (!hip_ok(hipMemcpyAsync(ctx->len.data(), ctx->d.len, ctx->n_caches * 4, hipMemcpyDeviceToHost, s)) ||
      !hip_ok(hipMemcpyAsync(&status, status_dev, 4, hipMemcpyDeviceToHost, s)) ||
      !hip_ok(hipStreamSynchronize(s)))
    return BAKLAVA_EHIP;
  if (status == 0) return BAKLAVA_OK;
  if (!hip_ok(launch_fill_i32(status_dev, 0, 1, s))) return BAKLAVA_EHIP;
  return BAKLAVA_ECAPACITY;
}

extern "C" int baklava_flush_scores(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count, void* stream) {
  if (!ctx || !range_ok(ctx, layer_begin, layer_count)) return BAKLAVA_EINVAL;
  return flush_records(ctx, layer_begin, layer_count, (hipStream_t)stream);
}

extern "C" int baklava_compact(baklava_ctx* ctx, int32_t layer_begin, int32_t layer_count,
                               int32_t* kept_idx_out, void* stream) {
  if (!ctx || !range_ok(ctx, layer_begin, layer_count)) return BAKLAVA_EINVAL;
  const int64_t c0 = (int64_t)layer_begin * ctx->cpl;
  const int64_t c1 = c0 + (int64_t)layer_count * ctx->cpl;
  CompactParams p;
  p.k = ctx->d.k; p.v = ctx->d.v; p.score = ctx->d.score; p.pos = ctx->d.pos;
  p.off = ctx->d.off; p.len = ctx->d.len; p.budget = ctx->d.budget;
  const bool whole = layer_begin == 0 && layer_count == ctx->d.L;
  p.order = whole ? reinterpret_cast<const int32_t*>(ctx->ws + ctx->plan.order_all)
                  : reinterpret_cast<const int32_t*>(ctx->ws + ctx->plan.order_layer) + c0;
  p.kept = kept_idx_out ? kept_idx_out : reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.kept);
  p.info = reinterpret_cast<CompactInfo*>(ctx->ws + ctx->plan.info);
  p.Hkv = ctx->d.Hkv; p.batch = ctx->d.batch;
  p.sink = ctx->d.sink; p.recent = ctx->d.recent; p.policy = ctx->d.policy;
  p.row_bytes = ctx->row_bytes;
  p.write_identity = kept_idx_out ? 1 : 0;
  p.move_ticket = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.move_ticket);
  p.move_flags = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.move_flags);
  hipStream_t s = (hipStream_t)stream;
  // The selection ranks rows by their scores: weights still owed to them are added first.
  {
    const int st = flush_records(ctx, layer_begin, layer_count, s);
    if (st != BAKLAVA_OK) return st;
  }
  p.cap = ctx->d.cap;
  const int32_t t0 = ctx->tile_begin[c0], t1 = ctx->tile_begin[c1];
  p.tiles = reinterpret_cast<const SelTile*>(ctx->ws + ctx->plan.tiles) + t0;
  p.tile_hist = reinterpret_cast<int32_t*>(ctx->ws + ctx->plan.tile_hist);
  p.sel_state = reinterpret_cast<SelState*>(ctx->ws + ctx->plan.sel_state);
  p.long_rows = ctx->select_long_rows;
  const int n_wide = std::accumulate(ctx->n_wide.begin() + layer_begin, ctx->n_wide.begin() + layer_begin + layer_count, 0);
  const int32_t sp0 = ctx->spread_begin[c0], n_spread = ctx->spread_begin[c1] - sp0;
  const bool spread = spread_selection(ctx, c0, c1);
  if (!hip_ok(launch_compact_select(p, (int)(c1 - c0), n_wide, whole || layer_count == 1, t1 - t0,
                                    reinterpret_cast<const SelTile*>(ctx->ws + ctx->plan.spread) + sp0,
                                    spread ? n_spread : 0, ctx->n_cus, s)))
    return BAKLAVA_EHIP;
  if (!hip_ok(launch_compact_move(p, (int)c0, (int)(c1 - c0), ctx->move_before.data() + c0, ctx->n_cus, s))) return BAKLAVA_EHIP;
  for (int64_t c = c0; c < c1; ++c) {
    const int32_t b = ctx->budget[(c / ctx->cpl) * ctx->d.Hkv + c % ctx->d.Hkv];
    ctx->len[c] = std::min(ctx->len[c], b);
  }
  return BAKLAVA_OK;
}

extern "C" size_t baklava_profile_workspace_bytes(int32_t batch, int32_t Hq, int32_t T) {
  if (batch <= 0 || Hq <= 0 || T <= 0) return 0;
  const int64_t n_tiles = ((int64_t)T + 127) / 128;  // 128 tokens per workgroup
  return align256((size_t)batch * Hq * n_tiles * sizeof(float));
}

extern "C" int baklava_profile_similarity(const void* q, const void* k, const void* v, int32_t batch,
                                          int32_t Hq, int32_t Hkv, int32_t T, int32_t D, int32_t dtype,
                                          float* cos_out, float* sim_out, float* lse_out, void* workspace,
                                          size_t workspace_bytes, void* stream) {
  if (!q || !k || !v || !sim_out || !workspace) return BAKLAVA_EINVAL;
  if (batch <= 0 || Hq <= 0 || Hkv <= 0 || T <= 0 || Hq % Hkv) return BAKLAVA_EINVAL;
  if (D != 128 || dtype != BAKLAVA_BF16) return BAKLAVA_EINVAL;
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)workspace) & 15) return BAKLAVA_EINVAL;
  if (((uintptr_t)sim_out | (uintptr_t)cos_out | (uintptr_t)lse_out) & 3) return BAKLAVA_EINVAL;
  if ((int64_t)batch * Hq * (((int64_t)T + 127) / 128) > INT32_MAX) return BAKLAVA_EINVAL;
  if (workspace_bytes < baklava_profile_workspace_bytes(batch, Hq, T)) return BAKLAVA_ECAPACITY;
  if (!hip_ok(launch_profile_similarity(q, k, v, batch, Hq, Hkv, T, cos_out, sim_out, lse_out,
                                        reinterpret_cast<float*>(workspace), (hipStream_t)stream)))
    return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}

extern "C" size_t baklava_layer_workspace_bytes(int32_t n_seq, int32_t T) {
  if (n_seq <= 0 || T <= 0) return 0;
  return align256((size_t)n_seq * (((size_t)T + 15) / 16) * sizeof(float));  // 16 rows per workgroup
}

extern "C" int baklava_layer_similarity(const void* x_in, const void* x_out, int32_t n_seq, int32_t T,
                                        int32_t hidden, int32_t dtype, float* cos_out, float* sim_out,
                                        void* workspace, size_t workspace_bytes, void* stream) {
  if (!x_in || !x_out || !sim_out || !workspace) return BAKLAVA_EINVAL;
  if (n_seq <= 0 || T <= 0 || hidden <= 0 || hidden % 8 || dtype != BAKLAVA_BF16) return BAKLAVA_EINVAL;
  if (((uintptr_t)x_in | (uintptr_t)x_out | (uintptr_t)workspace) & 15) return BAKLAVA_EINVAL;
  if (((uintptr_t)sim_out | (uintptr_t)cos_out) & 3) return BAKLAVA_EINVAL;
  if ((int64_t)n_seq * (((int64_t)T + 15) / 16) > INT32_MAX) return BAKLAVA_EINVAL;
  if (workspace_bytes < baklava_layer_workspace_bytes(n_seq, T)) return BAKLAVA_ECAPACITY;
  if (!hip_ok(launch_layer_similarity(x_in, x_out, n_seq, T, hidden, cos_out, sim_out,
                                      reinterpret_cast<float*>(workspace), (hipStream_t)stream)))
    return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}

extern "C" int baklava_prefill_scores(const void* q, const void* k, const float* lse, const int64_t* row_off,
                                      int32_t batch, int32_t Hq, int32_t Hkv, int32_t T, int32_t D,
                                      int32_t dtype, float* score_out, void* stream) {
  if (!q || !k || !lse || !score_out) return BAKLAVA_EINVAL;
  if (batch <= 0 || Hq <= 0 || Hkv <= 0 || T <= 0 || Hq % Hkv) return BAKLAVA_EINVAL;
  if (D != 128 || dtype != BAKLAVA_BF16) return BAKLAVA_EINVAL;
  if (((uintptr_t)q | (uintptr_t)k) & 15) return BAKLAVA_EINVAL;
  if (((uintptr_t)lse | (uintptr_t)score_out) & 3 || ((uintptr_t)row_off & 7)) return BAKLAVA_EINVAL;
  if ((int64_t)batch * Hkv * (((int64_t)T + 127) / 128) > INT32_MAX) return BAKLAVA_EINVAL;
  if (!hip_ok(launch_prefill_scores(q, k, lse, row_off, batch, Hq, Hkv, T, score_out, (hipStream_t)stream)))
    return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}

extern "C" int baklava_lengths(baklava_ctx* ctx, int32_t* len_host_out) {
  if (!ctx || !len_host_out) return BAKLAVA_EINVAL;
  std::memcpy(len_host_out, ctx->len.data(), ctx->n_caches * sizeof(int32_t));
  return BAKLAVA_OK;
}

extern "C" int baklava_stream_probe(void* dst, const void* src, int64_t bytes, int32_t mode, void* stream) {
  if (!dst || !src || bytes <= 0 || (bytes & 15) || (mode < 0 || mode > 3)) return BAKLAVA_EINVAL;
  if (((uintptr_t)dst | (uintptr_t)src) & 15) return BAKLAVA_EINVAL;
  if (!hip_ok(launch_stream_probe(dst, src, bytes, mode, (hipStream_t)stream))) return BAKLAVA_EHIP;
  return BAKLAVA_OK;
}
