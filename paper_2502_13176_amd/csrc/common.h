// Internal declarations shared by the library's own translation units.
#ifndef BAKLAVA_COMMON_H
#define BAKLAVA_COMMON_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace baklava {

// 16-byte load with the non-temporal hint, for data a kernel reads exactly once.
#ifdef __HIPCC__
typedef uint32_t nt_u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_nt16(const void* ptr) {
  const nt_u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4_t*>(ptr));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_nt16(void* ptr, uint4 v) {
  const nt_u32x4_t x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<nt_u32x4_t*>(ptr));
}
#endif

constexpr int kLagRows = 32;   // packed query rows of a cache's record of pending calls (score tracking)
constexpr int kLagCalls = 8;   // most calls such a record holds
constexpr int kTicketStride = 32;  // words from one cache's flush ticket to the next: a cache line each
constexpr int kMostTickets = 128;  // most work items of a cache that draw them
// Eviction move: destination rows per tile by 16-byte pieces per row (128 KiB of K and V), threads per workgroup, caches
// per launch
constexpr int kMoveRowsMin = 128;
constexpr int move_rows(int pieces) { return pieces > 16 ? kMoveRowsMin : pieces > 8 ? 2 * kMoveRowsMin : 4 * kMoveRowsMin; }
// most rows of a cache that one workgroup moves (half a tile, or a whole one of 512-byte rows)
constexpr int move_short_rows(int pieces) { return pieces > 8 ? kMoveRowsMin : 2 * kMoveRowsMin; }
constexpr int kMoveThreads = 512;
constexpr int kMoveCaches = 8192;
constexpr int kTileRows = 8192;     // rows per tile of a cache that is ranked tile by tile (one workgroup per tile and pass)
constexpr int kHeldRows = 65536;     // most rows of a cache that one workgroup ranks, in its registers
constexpr int kNarrowRows = kHeldRows / 4;  // most rows of a cache of which two such workgroups fit a compute unit
constexpr int kMinLongRows = kTileRows;  // smallest capacity from which a cache may be ranked that way

// One split-K work item (same layout as baklava_work_item of the public header): rows
// [start, start + count) of cache c; its partial result goes to partial slot `slot`.  Rows at or
// beyond the cache's live length are skipped by the kernel.
struct Item {
  int32_t c, start, count, slot;
  int32_t nsplit;  // work items of this cache
  int32_t slot0;   // partial slot of the cache's first item (filled in when the table is uploaded)
  int64_t row0;    // arena row of `start`: off[c] + start
};

// Result of the selection pass for one cache.
struct CompactInfo {
  int32_t new_len;      // rows that survive
  int32_t first_moved;  // smallest evicted row index (== old length when nothing is evicted)
  int32_t old_len;
  int32_t pad;
};

// One tile of a cache that several workgroups rank (or, in the second table, the only one of a short cache).
struct SelTile {
  int32_t c, tile;
  int32_t first_tile;  // index of the counters of the cache's tile 0
  int32_t n_tiles;     // tiles of the cache
  int32_t long_idx;    // index of the cache among the caches that are ranked this way
  int32_t pad;
};

// State of the radix select of a long cache after a pass.
struct SelState {
  uint32_t prefix;   // digits found so far, in place
  int32_t need;      // rank of the wanted key among the keys that match the prefix
  int32_t digit[4];
};

// A cache that the combine kernel serves, with its partial slots [slot_begin, slot_end): one
// 16-byte record, so that the kernel needs a single load before it can fetch the partials.
struct MultiCache {
  int32_t c, slot_begin, slot_end, pad;
};

struct DecodeParams {
  void* k;
  void* v;
  const void* q;
  float* out;
  const int64_t* off;
  int32_t* len;
  const Item* items;               // work items of the launched range, in launch order
  float* part_o;                   // [n_items, G, D] un-normalised partial outputs
  float* part_ml;                  // [n_items, G, 2]  (running max in log2 units, sum)
  float* final_ml;                 // [n_caches, G, 2] (global max, 1 / global sum) of the latest call
  // Score tracking, MFMA kernel: the weights of a call are added to the score plane by a later
  // call over the same caches (or by the score pass that baklava_flush_scores launches), because
  // only then are the softmax normalisers known to every work item.  Each cache keeps a record of
  // up to lag_batch pending calls; their query rows are packed into two 16-row operands (call s,
  // head g -> packed row s * Gp + g, Gp = G rounded up to 4, 8 or 16), so that two extra matrix
  // products per slab serve all of them.  A call that finds lag_batch calls pending adds their
  // weights and starts the record again with itself.
  void* lag_q;                     // [n_caches, kLagRows, D] packed query rows of the pending calls
  float* lag_ml;                   // [n_caches, kLagRows, 2] their (max, 1 / sum), same row numbering
  int32_t* lag_n;                  // [n_caches, kLagCalls] rows that were live at pending call s
  int32_t* lag_cnt;                // [n_caches, G] pending calls (one counter per head, all equal:
                                   // each block of the combine kernel reads and writes its own)
  int32_t* flush_ticket;           // [n_caches * kTicketStride] work items of a flush that are done (0 at rest), or
                                   // null: a launch behind the flush empties the records
  const int32_t* cap;
  float* score;
  int32_t* pos;
  const MultiCache* multi;         // caches of the launched range that have more than one work item
  const void* k_new;               // fused append: [caches of the range, D] rows to add first
  const void* v_new;
  const int32_t* token_pos_dev;    // fused append: the new row's position, read on the device (or null)
  int32_t* status;                 // device status word: bit 0 = a fused append found its cache full
  int32_t G, Hq, Hkv, batch;
  int32_t cache_begin;             // first cache id of the launched range
  int32_t lag;                     // 1: record this call, apply the pending ones when due (MFMA kernel)
  int32_t lag_batch;               // calls a record holds: kLagRows / Gp
  int32_t lag_gp_log2;             // log2(Gp)
  int32_t ring_slots;              // slabs (tiles) per wavefront whose new scores (logits) wait in LDS
  // Score tracking without records: the attention kernel leaves the scaled logits of the call (log2 units) here,
  // head g of arena row r at logits[g * logit_stride + r], and the live rows of each cache in lag_n; the kernel
  // behind it merges the split partials and adds the weights to the scores.  Null: not asked for.
  float* logits;
  int64_t logit_stride;
  int32_t fused_append;            // 1: every cache of the range first receives its new row
  int32_t token_pos;
  int32_t row_bytes;
  float scale_log2e;               // log2(e) / sqrt(D)
};

// Score pass over the K rows alone (bf16 rows of 128 elements on the vector kernel), behind the combine kernel:
// score_j += sum_g 2^(q_g . k_j scale - M_g) / L_g over the live rows of every cache of the range.
struct ScoreParams {
  const void* k;
  const void* q;                   // [layer_count, batch, Hq, D], the call's query rows
  const float* ml;                 // final_ml of the call
  const int32_t* len;
  const Item* items;
  float* score;
  int32_t G, Hq, Hkv;
  int32_t cache_begin;
  float scale_log2e;
};

struct AppendParams {
  void* k;
  void* v;
  float* score;
  int32_t* pos;
  const int64_t* off;
  const int32_t* cap;
  int32_t* len;
  const void* k_new;
  const void* v_new;
  const int32_t* token_pos_dev;  // the row's position, read on the device (or null: token_pos)
  int32_t cache_begin;
  int32_t token_pos;
  int32_t row_bytes;
};

constexpr int kLengthsPerLaunch = 512;
struct LengthsParams {
  int32_t* len;
  int32_t* lag_cnt;                  // [n_caches, G]
  int32_t count, G;                  // all caches of the context
  int32_t value[kLengthsPerLaunch];
};

struct CompactParams {
  void* k;
  void* v;
  float* score;
  int32_t* pos;
  const int64_t* off;
  int32_t* len;
  const int32_t* budget;
  const int32_t* order;  // launch order: blockIdx.x -> cache id
  int32_t* kept;         // [total_tokens], packed by off
  CompactInfo* info;     // [n_caches]
  int32_t Hkv, batch;
  int32_t sink, recent, policy;
  int32_t row_bytes;
  int32_t write_identity;  // 1: also write 0..n-1 for caches that evict nothing
  int32_t* move_ticket;    // [n_caches] tiles that workgroups of a launch of the move have taken (its first cache's counter)
  int32_t* move_flags;     // tiles whose rows have been read (see move_flag_base)
  const int32_t* cap;
  const SelTile* tiles;    // tiles of the long caches of the launched range
  int32_t* tile_hist;      // [all tiles][4 passes][256] digit counters, indexed by first_tile + tile
  SelState* sel_state;     // [long caches][4] state after pass 0..3
  int32_t long_rows;       // caches with more capacity than this are ranked tile by tile
};

// Records a failed HIP call for baklava_last_hip_error() (per host thread).
void note_hip_error(hipError_t e);

// Launchers (defined next to their kernels).  All return hipError_t of the launch.
// max_count: longest work item of the launch (rows); one_wave: the launch has at most one workgroup per
// compute unit, so a workgroup may take the whole LDS (score tracking keeps its new scores or logits there)
hipError_t launch_decode_valu(const DecodeParams& p, int dtype, int D, int n_items, int max_count, bool one_wave,
                              hipStream_t s);
hipError_t launch_decode_mfma(const DecodeParams& p, int D, int n_items, int max_count, bool one_wave, hipStream_t s,
                              hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t prepare_decode_mfma();
hipError_t launch_decode_mfma_f32(const DecodeParams& p, int D, int n_items, int max_count, bool one_wave, hipStream_t s);
hipError_t prepare_decode_mfma_f32();
// the weights of the calls on record, from the K rows alone, after which the records are empty where flush_ticket is not
// null (bf16, D = 128; needs only the lag_*, flush_ticket, k, score, items, G and scale fields, and all work items of a
// cache in the launch)
hipError_t launch_score_flush_mfma(const DecodeParams& p, int n_items, int max_count, hipStream_t s);
hipError_t launch_profile_similarity(const void* q, const void* k, const void* v, int batch, int Hq, int Hkv,
                                     int T, float* cos_out, float* sim_out, float* lse_out, float* tile_sum,
                                     hipStream_t s);
hipError_t launch_layer_similarity(const void* x_in, const void* x_out, int n_seq, int T, int hidden,
                                   float* cos_out, float* sim_out, float* tile_sum, hipStream_t s);
hipError_t launch_prefill_scores(const void* q, const void* k, const float* lse, const int64_t* row_off,
                                 int batch, int Hq, int Hkv, int T, float* score, hipStream_t s);
// most_split: work items of the cache that has most of them
hipError_t launch_combine(const DecodeParams& p, int D, int n_multi, int most_split, hipStream_t s);
// the end of a tracked call without records: split partials merged, weights added to the scores from p.logits
hipError_t launch_finish(const DecodeParams& p, int D, int n_multi, int most_split, int n_items, int max_count,
                         hipStream_t s);
// max_count: the largest row count of a work item in the launched range (or a bound on it)
hipError_t launch_score_pass(const ScoreParams& p, int n_items, int max_count, hipStream_t s);
hipError_t launch_append(const AppendParams& p, int n_caches, hipStream_t s);
hipError_t launch_set_lengths(const LengthsParams& p, hipStream_t s);
hipError_t launch_fill_i32(int32_t* dst, int32_t value, int64_t n, hipStream_t s);
// n_wide: caches of the range with more than kNarrowRows rows of capacity; sorted: they come first in p.order
// n_spread > 0: the caches of up to p.long_rows rows are ranked by the workgroups spread[0 .. n_spread)
hipError_t launch_compact_select(const CompactParams& p, int n_caches, int n_wide, bool sorted, int n_tiles,
                                 const SelTile* spread, int n_spread, int n_cus, hipStream_t s);
// Sums over the caches before one, of those that can evict: tiles of the move for caches of more than move_short_rows rows
// of budget, at most, and caches of no more.
struct MoveCount {
  int64_t tiles;
  int32_t short_caches;
};
// the move of caches c0 .. c0 + n_caches, behind the selection; before[i]: the sums for cache c0 + i
hipError_t launch_compact_move(const CompactParams& p, int c0, int n_caches, const MoveCount* before, int n_cus,
                               hipStream_t s);
hipError_t launch_stream_probe(void* dst, const void* src, int64_t bytes, int mode, hipStream_t s);

}  // namespace baklava
#endif
