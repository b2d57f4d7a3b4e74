// Budget-enforcing eviction (f_evict, Eqs. 5-6): selection of the surviving rows (one workgroup
// per cache, long caches first, or several where few long caches would leave compute units idle; caches
// beyond what a workgroup's registers hold are cut into tiles and go through one kernel per radix pass),
// then a stable in-place move (tiles of rows, several workgroups to a cache).
#include "common.h"

#include <algorithm>

namespace baklava {

namespace {

constexpr int kSelThreads = 512;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelRows = 16;   // consecutive rows per thread in the emit pass (four 16-byte loads)
constexpr int kEmitTile = kSelThreads * kSelRows;

// Order-preserving map from fp32 to uint32 (larger float -> larger key); -0 is folded onto +0 so
// that it ties with it, as a floating-point comparison would.
__device__ __forceinline__ uint32_t score_key(float f) {
  const uint32_t u = __float_as_uint(f + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix sum of `v` over the workgroup; `total` receives the sum.  `sm` holds one
// word per wavefront.  Ends with a barrier, so `sm` can be reused right away.
template <int WAVES = kSelWaves>
__device__ __forceinline__ int block_exclusive_scan(int v, int* sm, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) sm[wave] = incl;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const int x = sm[w];
    if (w < wave) base += x;
    tot += x;
  }
  __syncthreads();
  total = tot;
  return base + incl - v;
}

// What the selection of one cache is after: the middle rows [mid_lo, mid_hi) compete for k places.
struct SelGoal {
  int n, b, k, mid_lo, mid_hi;
};

__device__ __forceinline__ SelGoal sel_goal(const CompactParams& p, int c) {
  SelGoal g;
  g.n = p.len[c];
  const int cpl = p.batch * p.Hkv;
  g.b = p.budget[(c / cpl) * p.Hkv + c % p.Hkv];
  const int s = p.sink;
  const int r = (p.policy == 1) ? (g.b - s) : p.recent;
  g.k = g.b - s - r;  // middle rows that survive, >= 0 (checked at context creation)
  g.mid_lo = s;
  g.mid_hi = g.n - r;
  return g;
}

// First flag of a cache's tiles: each of the caches before it has at most one tile more than its rows fill.
__device__ __forceinline__ int64_t move_flag_base(int64_t off, int c) { return off / kMoveRowsMin + c; }

// The move behind the selection starts at the cache's first tile, with no tile read yet.  By one whole workgroup.  A
// cache within its budget has no tile, and its flags would not hold one per 128 rows of the budget, which may lie above
// the capacity; a cache beyond its budget has more rows of capacity than that.
__device__ __forceinline__ void clear_move_state(const CompactParams& p, int c, int64_t off, const SelGoal& g) {
  int32_t* flags = p.move_flags + move_flag_base(off, c);
  const int n_flags = g.n > g.b ? (int)(((int64_t)g.b + kMoveRowsMin - 1) / kMoveRowsMin) : 0;
  for (int t = threadIdx.x; t < n_flags; t += blockDim.x) flags[t] = 0;
  if (threadIdx.x == 0) p.move_ticket[c] = 0;
}

// One counting pass of the radix select over rows [j_begin, j_end) of the middle: keys whose digits
// above `shift` equal `prefix` are counted by their digit at `shift` into the LDS histogram.
// A thread adds up runs of equal digits among its own keys before it touches the histogram: in
// the first pass most scores share their leading bits, and one atomic per key on the same few
// counters would serialise the whole workgroup.
template <int UNROLL>
__device__ __forceinline__ void count_digits(const float* score, int j_begin, int j_end, uint32_t prefix,
                                             uint32_t mask, int shift, int* hist) {
  const int tid = threadIdx.x;
  for (int j0 = j_begin + tid; j0 < j_end; j0 += kSelThreads * UNROLL) {
    uint32_t key[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int j = j0 + u * kSelThreads;
      key[u] = score_key(j < j_end ? score[j] : 0.f);
    }
    int run_digit = -1, run = 0;
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int j = j0 + u * kSelThreads;
      const bool live = j < j_end && (key[u] & mask) == prefix;
      const int digit = (key[u] >> shift) & 255;
      if (live && digit == run_digit) {
        run += 1;
      } else if (live) {
        if (run) atomicAdd(&hist[run_digit], run);
        run_digit = digit;
        run = 1;
      }
    }
    if (run) atomicAdd(&hist[run_digit], run);
  }
}

// The digit of the need-th largest key given the 256 counters of a pass: thread t looks at digit
// 255 - t; `above` = keys with a larger digit.  Exactly one digit has above < need <= above + its own
// count.  Results through the shared words; ends with a barrier.
__device__ __forceinline__ void find_digit(const int* hist, int need, int* sm_scan, int* sh_digit, int* sh_need) {
  const int tid = threadIdx.x;
  const int mine = tid < 256 ? hist[255 - tid] : 0;
  int all;
  const int above = block_exclusive_scan(mine, sm_scan, all);
  if (tid < 256 && above < need && above + mine >= need) {
    *sh_digit = 255 - tid;
    *sh_need = need - above;
  }
  __syncthreads();
}

// LDS an emit needs: the keys of a tile, padded by one word per 16 so that a thread's 16 consecutive
// keys and its neighbours' fall into different banks; once every thread has read its keys (the
// workgroup scan in between has barriers) the same words collect the tile's part of the kept list.
constexpr int kEmitKeyWords = kEmitTile + kEmitTile / 16;

// Stable emit of the rows [j_begin, j_end) of a cache.  A row survives if it is a sink or recent
// row, if its key exceeds the threshold, or if it is among the first need_eq rows (of the whole
// cache) whose key equals it; its place in the list is the number of survivors before it, i.e.
// (rows of the first two kinds before it) + min(rows with an equal key before it, need_eq).  Both
// counts come from one workgroup scan of a packed pair per tile of kEmitTile rows (at most
// kSelRows * kSelThreads = 2^13 each).  sure_base / eq_base: the two counts over the rows before
// j_begin.  Global memory is touched in whole lines only: the tile's scores are loaded row t,
// t + 512, ... per thread (all loads in flight at once) and handed to the thread that owns 16
// consecutive rows through LDS; the tile's survivors, which occupy consecutive places of the list,
// are collected in LDS and written out together.  The smallest evicted row index of the range goes
// to *sh_first (shared, initialised by the caller to the cache's length).
__device__ __forceinline__ void emit_rows(const float* score, int32_t* kept, const SelGoal& g, uint32_t thr,
                                          int need_eq, int j_begin, int j_end, int sure_base, int eq_base,
                                          int* sm_scan, int* sh_first, uint32_t* lds_key) {
  const int tid = threadIdx.x;
  const int n = g.n;
  int32_t* lds_out = reinterpret_cast<int32_t*>(lds_key);
  for (int j0 = j_begin; j0 < j_end; j0 += kEmitTile) {
    const int live = j_end - j0;  // rows of this tile (a short cache fills only the front of it)
    if (g.k > 0) {
      float sc[kSelRows];
#pragma unroll
      for (int u = 0; u < kSelRows; ++u) {
        const int j = j0 + tid + u * kSelThreads;
        sc[u] = 0.f;
        if (u * kSelThreads < live) sc[u] = (j >= g.mid_lo && j < g.mid_hi && j < j_end) ? score[j] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kSelRows; ++u) {
        const int r = tid + u * kSelThreads;
        if (u * kSelThreads < live) lds_key[r + (r >> 4)] = score_key(sc[u]);
      }
      __syncthreads();
    }
    const int jt = j0 + tid * kSelRows;
    bool sure[kSelRows], eq[kSelRows];
    int n_sure = 0, n_eq = 0;
#pragma unroll
    for (int i = 0; i < kSelRows; ++i) {
      const int j = jt + i;
      const bool in = j < j_end;
      const bool middle = in && j >= g.mid_lo && j < g.mid_hi;
      const uint32_t key = (middle && g.k > 0) ? lds_key[tid * (kSelRows + 1) + i] : 0u;
      sure[i] = (in && !middle) || (middle && g.k > 0 && key > thr);
      eq[i] = middle && g.k > 0 && key == thr;
      n_sure += sure[i] ? 1 : 0;
      n_eq += eq[i] ? 1 : 0;
    }
    int total;
    const int excl = block_exclusive_scan(n_sure | (n_eq << 16), sm_scan, total);
    const int place0 = sure_base + min(eq_base, need_eq);  // place of the tile's first survivor
    int sure_before = sure_base + (excl & 0xffff);
    int eq_before = eq_base + ((uint32_t)excl >> 16);
    int first_out = n;
#pragma unroll
    for (int i = 0; i < kSelRows; ++i) {
      const int j = jt + i;
      const bool keep = sure[i] || (eq[i] && eq_before < need_eq);
      if (keep) lds_out[sure_before + min(eq_before, need_eq) - place0] = j;
      else if (j < j_end) first_out = min(first_out, j);
      sure_before += sure[i] ? 1 : 0;
      eq_before += eq[i] ? 1 : 0;
    }
    // rows leave in ascending order of the tiles, so only the first tile that evicts has to report
    if (first_out < n && first_out < *(volatile int*)sh_first) atomicMin(sh_first, first_out);
    sure_base += total & 0xffff;
    eq_base += (uint32_t)total >> 16;
    const int survivors = sure_base + min(eq_base, need_eq) - place0;
    __syncthreads();
    for (int i = tid; i < survivors; i += kSelThreads) kept[place0 + i] = lds_out[i];
    __syncthreads();  // the LDS areas are free again
  }
}

// ---- caches one workgroup ranks alone ----------------------------------------------------------
// The middle of a cache of up to 1024 * KEYS rows is read once, into registers: row i * 1024 + t of the
// middle is key i of thread t, every load in flight before the first use.  Three radix passes (11, 11
// and 10 bits) count digits in LDS, and the stable emit takes its flags from the same registers: each
// wavefront leaves its counts of surviving rows per block of 1024 rows, one workgroup scan turns them
// into places, and a row's place inside its wavefront is a population count of the ballot below it.
// Bound by vector issue (about 40 instructions per key on one compute unit) and the latency of a dozen
// barriers, not by bandwidth.  Sweeping the scores once per pass (four passes of 8 bits and the emit, 512
// threads) took 90 us for 512 caches of 128 to 32768 rows, this takes 53; tile by tile (below) 8 caches of
// 32768 rows took 46 us in five kernels, here 36 in one.  KEYS = 16 (caches of up to 16384 rows) needs at
// most 64 registers, so two workgroups fit a compute unit; KEYS = 64 needs more, so one does.
constexpr int kHeldThreads = 1024;
constexpr int kHeldWaves = kHeldThreads / 64;
constexpr int kHeldBins = 2048;

// Inclusive prefix sum over the wavefront in six data-parallel-primitive adds: shifts inside the rows
// of 16 lanes, then the last lane of a row to the next one, and lane 31 to the upper half.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Word i of an array that the whole workgroup reads or writes: a uniform base and a 32-bit offset (i < 2^30).
template <typename T>
__device__ __forceinline__ T word_at(const T* base, int i) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (uint32_t)i * 4u);
}
// Word `block` + the thread's number of m, the last one in place of those past it.
template <typename T>
__device__ __forceinline__ T block_word(const T* base, int block, int m) {
  const int b = min(block, m - 1);
  return word_at(base + b, min((int)threadIdx.x, m - 1 - b));
}
template <typename T>
__device__ __forceinline__ void set_word(T* base, int i, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (uint32_t)i * 4u) = v;
}

// Exclusive prefix sum of `v` over the workgroup of kHeldThreads; `sm` holds one word per wavefront and
// is not read again after the barrier of the caller's next step.
__device__ __forceinline__ int held_exclusive_scan(int v, int* sm) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int incl = wave_inclusive_scan(v);
  if (lane == 63) sm[wave] = incl;
  __syncthreads();
  const int sums = wave_inclusive_scan(lane < kHeldWaves ? sm[lane] : 0);
  const int before = __builtin_amdgcn_readlane(sums, max(wave, 1) - 1);
  return (wave > 0 ? before : 0) + incl - v;
}

// One key more of digit `digit`.  64 lanes that meet on one counter would be served one after the other, so a
// wavefront whose active lanes all have the same digit (many equal scores) adds them up first.
__device__ __forceinline__ void count_key(int* hist, int digit) {
  const uint64_t here = __ballot(true);
  if (__ballot(digit == __builtin_amdgcn_readfirstlane(digit)) == here) {
    if (__builtin_amdgcn_mbcnt_hi((uint32_t)(here >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)here, 0)) == 0)
      atomicAdd(&hist[digit], __popcll(here));
  } else {
    atomicAdd(&hist[digit], 1);
  }
}

// LDS of a workgroup that ranks.
template <int KEYS>
struct HeldShared {
  int hist[kHeldBins];
  int scan[2 * kHeldWaves];
  int digit, need, first;
  int sure_before[KEYS * kHeldWaves], eq_before[KEYS * kHeldWaves];
};

// The digit of the need-th largest key from the counters of a pass; need becomes its rank among the keys of that
// digit.  Thread t looks at the digits 2047 - 2t (c_hi keys) and 2046 - 2t (c_lo): exactly one digit has above <
// need <= above + its own count.  Ends with a barrier.
__device__ __forceinline__ int held_find_digit(int c_hi, int c_lo, int& need, int* scan, int* sh_digit, int* sh_need) {
  const int d_hi = kHeldBins - 1 - 2 * threadIdx.x;
  const int above = held_exclusive_scan(c_hi + c_lo, scan);
  if (above < need && above + c_hi >= need) {
    *sh_digit = d_hi;
    *sh_need = need - above;
  } else if (above + c_hi < need && above + c_hi + c_lo >= need) {
    *sh_digit = d_hi - 1;
    *sh_need = need - above - c_hi;
  }
  __syncthreads();
  need = *sh_need;
  return *sh_digit;
}
template <int KEYS>
__device__ __forceinline__ int held_find_digit(HeldShared<KEYS>& sm, int& need) {  // leaves the counters cleared
  const int d_hi = kHeldBins - 1 - 2 * threadIdx.x;
  const int c_hi = sm.hist[d_hi], c_lo = sm.hist[d_hi - 1];
  sm.hist[d_hi] = 0;
  sm.hist[d_hi - 1] = 0;
  return held_find_digit(c_hi, c_lo, need, sm.scan, &sm.digit, &sm.need);
}

// Scores of m rows, row i * 1024 + t as key i of thread t.  Places past the m rows hold key 0, the lowest: no score
// but a NaN of all ones maps there.  Behind every row of the cache neither the threshold nor a survivor's place depends
// on them.  (A base for each block keeps 64 keys from spilling; up to 16 take fewer instructions with one for all: 1500
// caches of up to 2064 rows ranked in 36.6 / 34.7 us.)
template <int KEYS>
__device__ __forceinline__ void held_load(const float* score, int m, uint32_t (&key)[KEYS]) {
#pragma unroll
  for (int i = 0; i < KEYS; ++i)
    key[i] = __float_as_uint(KEYS <= 16 ? score[min(i * kHeldThreads + (int)threadIdx.x, m - 1)] : block_word(score, i * kHeldThreads, m));
}
template <int KEYS>
__device__ __forceinline__ void held_map(int m, uint32_t (&key)[KEYS]) {
#pragma unroll
  for (int i = 0; i < KEYS; ++i) {
    const uint32_t x = score_key(__uint_as_float(key[i]));
    key[i] = i * kHeldThreads + (int)threadIdx.x < m ? x : 0u;
  }
}

// Stable emit of the m rows behind the keys, cache rows row0 .. row0 + m.  A row survives if its key exceeds the
// threshold, or if it is among the first need_eq rows of the cache whose key equals it; its place in `out` is (rows of
// the first kind before it) + min(rows with an equal key before it, need_eq), of which sure_base and eq_base lie
// before row0.  Counts per (block of 1024 rows, wavefront) first: lane i collects its wavefront's counts of block i,
// the workgroup scans them in row order, and lane i gets block i's two places back.  Lowers sm.first to the first row
// (from row0) that does not survive.
template <int KEYS>
__device__ __forceinline__ void held_emit(HeldShared<KEYS>& sm, const uint32_t (&key)[KEYS], int m, uint32_t thr,
                                          int need_eq, int sure_base, int eq_base, int row0, int32_t* out) {
  static_assert(KEYS <= 64, "one lane per block");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n_both = 0;
#pragma unroll
  for (int i = 0; i < KEYS; ++i) {
    if (i * kHeldThreads < m) {
      const int both = __popcll(__ballot(key[i] > thr)) | __popcll(__ballot(key[i] == thr)) << 16;
      n_both = lane == i ? both : n_both;
    }
  }
  if (lane < KEYS) {
    sm.sure_before[lane * kHeldWaves + wave] = n_both & 0xffff;
    sm.eq_before[lane * kHeldWaves + wave] = n_both >> 16;
  }
  __syncthreads();
  int a = 0, e = 0;
  if (tid < KEYS * kHeldWaves) { a = sm.sure_before[tid]; e = sm.eq_before[tid]; }
  if (KEYS * kHeldThreads < 65536) {  // both counts in one scan
    const int both = held_exclusive_scan(a | e << 16, sm.scan);
    a = both & 0xffff;
    e = (uint32_t)both >> 16;
  } else {
    a = held_exclusive_scan(a, sm.scan);
    e = held_exclusive_scan(e, sm.scan + kHeldWaves);
  }
  if (tid < KEYS * kHeldWaves) { sm.sure_before[tid] = a; sm.eq_before[tid] = e; }
  __syncthreads();
  int place_sure = 0, place_eq = 0;
  if (lane < KEYS) {
    place_sure = sm.sure_before[lane * kHeldWaves + wave] + sure_base;
    place_eq = sm.eq_before[lane * kHeldWaves + wave] + eq_base;
  }
  int first_out = m;  // first row of this wavefront that does not survive
#pragma unroll
  for (int i = 0; i < KEYS; ++i) {
    if (i * kHeldThreads < m) {
      const int r = i * kHeldThreads + tid;
      const uint64_t ms = __ballot(key[i] > thr), me = __ballot(key[i] == thr);
      const int eq0 = __builtin_amdgcn_readlane(place_eq, i);
      int sb = __builtin_amdgcn_readlane(place_sure, i) + min(eq0, need_eq);
      bool keep = key[i] > thr;
      sb = __builtin_amdgcn_mbcnt_hi((uint32_t)(ms >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ms, sb));
      if (me != 0 && eq0 < need_eq) {  // uniform over the wavefront
        const int eb = __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0));
        sb += min(eb, need_eq - eq0);
        keep = keep || (key[i] == thr && eq0 + eb < need_eq);
      }
      if (keep) set_word(out, sb, row0 + r);
      const uint64_t gone = __ballot(!keep);
      if (gone != 0) first_out = min(first_out, i * kHeldThreads + wave * 64 + __ffsll((unsigned long long)gone) - 1);
    }
  }
  if (lane == 0) atomicMin(&sm.first, first_out);
  __syncthreads();
}

// The whole selection of one cache of up to 1024 * KEYS rows by this workgroup.
template <int KEYS>
__device__ __forceinline__ void select_whole(const CompactParams& p, int c, HeldShared<KEYS>& sm) {
  const int tid = threadIdx.x;
  const SelGoal g = sel_goal(p, c);
  const int n = g.n;
  const int64_t off = p.off[c];
  int32_t* kept = p.kept + off;
  clear_move_state(p, c, off, g);

  if (n <= g.b) {
    if (p.write_identity)
      for (int j = tid; j < n; j += kHeldThreads) kept[j] = j;
    if (tid == 0) p.info[c] = CompactInfo{n, n, n, 0};
    return;
  }

  // sink and recent rows: the first and the last places
  for (int j = tid; j < g.mid_lo; j += kHeldThreads) kept[j] = j;
  for (int j = g.mid_hi + tid; j < n; j += kHeldThreads) kept[j - (n - g.b)] = j;
  if (g.k <= 0) {  // no middle row survives
    if (tid == 0) p.info[c] = CompactInfo{g.b, g.mid_lo, n, 0};
    return;
  }

  const int m = g.mid_hi - g.mid_lo;  // rows that compete, g.k < m of them survive
  uint32_t key[KEYS];
  held_load(p.score + off + g.mid_lo, m, key);
  sm.hist[tid] = 0;
  sm.hist[tid + kHeldThreads] = 0;
  if (tid == 0) sm.first = m;
  held_map(m, key);
  __syncthreads();

  // radix select of the k-th largest key
  uint32_t prefix = 0, mask = 0;
  int need = g.k;
#pragma unroll 1
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
    const uint32_t digits = pass == 2 ? 1023u : 2047u;
#pragma unroll
    for (int i = 0; i < KEYS; ++i)
      if (i * kHeldThreads < m && (key[i] & mask) == prefix) count_key(sm.hist, (key[i] >> shift) & digits);
    __syncthreads();
    prefix |= (uint32_t)held_find_digit(sm, need) << shift;
    mask |= digits << shift;
  }
  // need: rows whose key equals the threshold that still survive (oldest first)
  held_emit(sm, key, m, prefix, need, 0, 0, g.mid_lo, kept + g.mid_lo);
  if (tid == 0) p.info[c] = CompactInfo{g.b, g.mid_lo + sm.first, n, 0};
}

template <int KEYS>
__global__ __launch_bounds__(kHeldThreads) void compact_select_kernel(CompactParams p, int cap_above, int cap_most) {
  __shared__ HeldShared<KEYS> sm;
  const int c = p.order[blockIdx.x];
  const int cap = p.cap[c];
  if (cap <= cap_above || cap > cap_most) return;  // another launch's
  select_whole<KEYS>(p, c, sm);
}

// Wide caches (the first n_wide of the launch order, of more than kNarrowRows rows) and all others in one launch.
__global__ __launch_bounds__(kHeldThreads) void compact_select_both_kernel(CompactParams p, int n_wide) {
  constexpr int kWide = kHeldRows / kHeldThreads, kNarrow = kNarrowRows / kHeldThreads;
  __shared__ union {
    HeldShared<kWide> wide;
    HeldShared<kNarrow> narrow;
  } sm;
  const int c = p.order[blockIdx.x];
  if (p.cap[c] > p.long_rows) return;  // ranked tile by tile
  if ((int)blockIdx.x < n_wide) select_whole<kWide>(p, c, sm.wide);
  else select_whole<kNarrow>(p, c, sm.narrow);
}

// ---- few caches: several workgroups to each ------------------------------------------------------
// One workgroup on each of a few caches leaves most of the chip idle.  Here a cache is cut into tiles of kTileRows rows,
// one workgroup each, in two kernels.  The first counts the keys of every tile by their leading 11 bits and leaves
// the counters in the workspace.  In the second every workgroup adds up the counters of its cache, finds the threshold's
// leading digit, collects in LDS the keys of the whole cache that have it (an eighth of them, say), ranks those by their
// other bits for itself, and emits its own tile.  Reading the cache's scores once more in every workgroup costs less than
// the launches that would share the work (about 5 us each behind one another).  A cache of up to kNarrowRows rows is
// ranked whole by the first kernel.  us per eviction, one workgroup per cache / spread: 8 caches of 20000 rows 47 / 35, of 32768 56 / 41, of
// 64000 82 / 62; the ranking of 8 caches of 32768 rows takes 20 us in all (35), 5 in the first kernel; of the 15 in the
// second 4.7 pass until the other rows with the digit are collected, 2.7 with the emit and the rest with barriers.
constexpr int kTileKeys = kTileRows / kHeldThreads;
constexpr int kMostTiles = kHeldRows / kTileRows;
constexpr int kListKeys = 2048;  // keys with the threshold's leading digit that LDS holds for each wavefront

// Rows of the middle that a tile holds.
__device__ __forceinline__ void tile_range(const SelGoal& g, int tile, int& lo, int& hi) {
  lo = max(g.mid_lo, tile * kTileRows);
  hi = min(g.mid_hi, (tile + 1) * kTileRows);
}

__global__ __launch_bounds__(kHeldThreads) void compact_spread_count_kernel(CompactParams p) {
  __shared__ HeldShared<kNarrowRows / kHeldThreads> sm;
  const SelTile tl = p.tiles[blockIdx.x];
  if (tl.n_tiles == 1) {
    select_whole<kNarrowRows / kHeldThreads>(p, tl.c, sm);
    return;
  }
  const int tid = threadIdx.x;
  const SelGoal g = sel_goal(p, tl.c);
  if (tl.tile == 0) clear_move_state(p, tl.c, p.off[tl.c], g);
  if (tl.tile == 0 && tid == 0)  // the second kernel lowers first_moved with atomicMin
    p.info[tl.c] = g.n <= g.b ? CompactInfo{g.n, g.n, g.n, 0} : CompactInfo{g.b, g.k > 0 ? g.n : g.mid_lo, g.n, 0};
  if (g.n <= g.b || g.k <= 0) return;
  int lo, hi;
  tile_range(g, tl.tile, lo, hi);
  const int m = max(0, hi - lo);
  uint32_t key[kTileKeys];
  if (m > 0) held_load(p.score + p.off[tl.c] + lo, m, key);
  sm.hist[tid] = 0;
  sm.hist[tid + kHeldThreads] = 0;
  __syncthreads();
  if (m > 0) {
    held_map(m, key);
#pragma unroll
    for (int i = 0; i < kTileKeys; ++i)
      if (i * kHeldThreads + tid < m) count_key(sm.hist, key[i] >> 21);
  }
  __syncthreads();
  // two counters of at most kTileRows each to a word
  uint32_t* out = reinterpret_cast<uint32_t*>(p.tile_hist) + (int64_t)(tl.first_tile + tl.tile) * (kHeldBins / 2);
  out[tid] = (uint32_t)sm.hist[2 * tid] | (uint32_t)sm.hist[2 * tid + 1] << 16;
}

__global__ __launch_bounds__(kHeldThreads) void compact_spread_emit_kernel(CompactParams p) {
  __shared__ HeldShared<kTileKeys> sm;
  __shared__ uint32_t cand[kHeldWaves * kListKeys];
  __shared__ int sure_before, eq_before;
  const SelTile tl = p.tiles[blockIdx.x];
  if (tl.n_tiles == 1) return;  // done
  const int tid = threadIdx.x, lane = tid & 63;
  const SelGoal g = sel_goal(p, tl.c);
  const int n = g.n;
  const int64_t off = p.off[tl.c];
  int32_t* kept = p.kept + off;
  const int j_begin = tl.tile * kTileRows, j_end = min(n, j_begin + kTileRows);
  if (n <= g.b) {
    if (p.write_identity)
      for (int j = j_begin + tid; j < j_end; j += kHeldThreads) kept[j] = j;
    return;
  }
  int lo, hi;
  tile_range(g, tl.tile, lo, hi);
  const int m = hi - lo;
  const bool ranks = g.k > 0 && m > 0;  // uniform over the workgroup
  const int m_all = g.mid_hi - g.mid_lo, front = lo - g.mid_lo;
  const float* score = p.score + off + g.mid_lo;  // the middle: m_all rows, `front` of them before the tile
  auto load_round = [&](float (&x)[kTileKeys], int r0) {
#pragma unroll
    for (int i = 0; i < kTileKeys; ++i) x[i] = block_word(score, r0 + i * kHeldThreads, m_all);
  };
  float first_round[kTileKeys];
  uint32_t w[kMostTiles];
  if (ranks) {
    // counters of this thread's two digits in the cache's tiles
    const uint32_t* th = reinterpret_cast<const uint32_t*>(p.tile_hist) + (int64_t)tl.first_tile * (kHeldBins / 2);
#pragma unroll
    for (int j = 0; j < kMostTiles; ++j) w[j] = th[(int64_t)min(j, tl.n_tiles - 1) * (kHeldBins / 2) + kHeldThreads - 1 - tid];
    load_round(first_round, 0);
  }
  // sink and recent rows of the tile
  for (int j = j_begin + tid; j < min(j_end, g.mid_lo); j += kHeldThreads) kept[j] = j;
  for (int j = max(j_begin, g.mid_hi) + tid; j < j_end; j += kHeldThreads) kept[j - (n - g.b)] = j;
  if (!ranks) return;  // nothing to rank, or none of it here

  sm.hist[tid] = 0;
  sm.hist[tid + kHeldThreads] = 0;
  if (tid == 0) {
    sm.first = m;
    sure_before = eq_before = 0;
  }
  int c_hi = 0, c_lo = 0, f_hi = 0, f_lo = 0;
#pragma unroll
  for (int j = 0; j < kMostTiles; ++j) {
    if (j < tl.n_tiles) { c_hi += w[j] >> 16; c_lo += w[j] & 0xffff; }
    if (j < tl.tile) { f_hi += w[j] >> 16; f_lo += w[j] & 0xffff; }
  }
  int need = g.k;
  const int d1 = held_find_digit(c_hi, c_lo, need, sm.scan, &sm.digit, &sm.need);
  const int t_hi = kHeldBins - 1 - 2 * tid;
  int sure = (t_hi > d1 ? f_hi : 0) + (t_hi - 1 > d1 ? f_lo : 0);  // rows before the tile that survive: larger digits

  // Every row of the middle whose key has that digit, a round of 8192 rows at a time and the next one on its way.
  // The digit is compared as it lies in the score (bits inverted where the key inverts them: scores below zero; -0 is
  // folded onto +0).  f(first row, the scores' bits: those whose leading digit is `lead` count)
  const uint32_t lead = d1 < kHeldBins / 2 ? (uint32_t)(kHeldBins - 1 - d1) : (uint32_t)(d1 - kHeldBins / 2);
  const uint32_t inv = d1 < kHeldBins / 2 ? 0xffffffffu : 0u;
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);  // first row of this wavefront in a block of 1024
  auto sweep = [&](auto f) {
    float next[kTileKeys];
#pragma unroll
    for (int i = 0; i < kTileKeys; ++i) next[i] = first_round[i];
#pragma unroll 1
    for (int r0 = 0; r0 < m_all; r0 += kTileRows) {
      uint32_t x[kTileKeys];
#pragma unroll
      for (int i = 0; i < kTileKeys; ++i) x[i] = __float_as_uint(next[i] + 0.0f);
      if (r0 + kTileRows < m_all) {
        load_round(next, r0 + kTileRows);
      } else {  // places past the last row repeat it: they get another digit
#pragma unroll
        for (int i = 0; i < kTileKeys; ++i) x[i] = r0 + i * kHeldThreads + tid < m_all ? x[i] : (lead ^ 1) << 21;
      }
      f(r0, x);
    }
  };
  // (a list for each wavefront, in the order of the rows: no counter to wait for, and those before the tile come first)
  int n_mine = 0, n_front = 0;
  bool fits = true;
  uint32_t* const mine = cand + wave0 / 64 * kListKeys;
  sweep([&](int r0, const uint32_t (&x)[kTileKeys]) {
    fits = fits && n_mine + 64 * kTileKeys <= kListKeys;
#pragma unroll
    for (int i = 0; i < kTileKeys; ++i) {
      const bool hit = x[i] >> 21 == lead;
      const uint64_t b = __ballot(hit);
      if (fits && hit)
        mine[__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, n_mine))] = x[i];
      n_mine += __popcll(b);
    }
    if (r0 + kTileRows <= front) {
      n_front = n_mine;
    } else if (r0 < front) {  // the tile begins in this round
#pragma unroll
      for (int i = 0; i < kTileKeys; ++i)
        n_front += __popcll(__ballot(x[i] >> 21 == lead && r0 + i * kHeldThreads + tid < front));
    }
  });
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // f(key bits, whether the row lies before the tile) for every candidate, from LDS, or, where they are too many for the
  // list, from another sweep over the scores.
  auto each = [&](auto f) {
    if (fits) {
      for (int r = lane; r < n_mine; r += 64) f(mine[r] ^ inv, r < n_front);
    } else {
      sweep([&](int r0, const uint32_t (&x)[kTileKeys]) {
#pragma unroll 1
        for (int i = 0; i < kTileKeys; ++i) {
          uint32_t v = 0;
#pragma unroll
          for (int k = 0; k < kTileKeys; ++k) v = k == i ? x[k] : v;
          if (v >> 21 == lead) f(v ^ inv, r0 + i * kHeldThreads + tid < front);
        }
      });
    }
  };
  each([&](uint32_t x, bool) { count_key(sm.hist, x >> 10 & 2047); });
  __syncthreads();
  const int d2 = held_find_digit(sm, need);
  each([&](uint32_t x, bool) {
    if ((int)(x >> 10 & 2047) == d2) count_key(sm.hist, x & 1023);
  });
  uint32_t key[kTileKeys];
  held_load(score + front, m, key);
  __syncthreads();
  const int d3 = held_find_digit(sm, need);
  const uint32_t low = (uint32_t)d2 << 10 | (uint32_t)d3;
  int eq = 0;  // candidates before the tile that equal the threshold
  each([&](uint32_t x, bool before) {
    sure += before && (x & 0x1fffffu) > low ? 1 : 0;
    eq += before && (x & 0x1fffffu) == low ? 1 : 0;
  });
  sure = wave_inclusive_scan(sure);
  eq = wave_inclusive_scan(eq);
  if (lane == 63 && sure != 0) atomicAdd(&sure_before, sure);
  if (lane == 63 && eq != 0) atomicAdd(&eq_before, eq);
  held_map(m, key);
  uint32_t thr = (uint32_t)d1 << 21 | low;
  if (thr == 0) {  // rows at the lowest key survive: the places past this tile's rows, in front of the next tile's, do not
#pragma unroll
    for (int i = 0; i < kTileKeys; ++i) key[i] = i * kHeldThreads + tid >= m ? 0u : key[i] == 0 ? 1u : 2u;
    thr = 1;
  }
  __syncthreads();
  held_emit(sm, key, m, thr, need, sure_before, eq_before, lo, kept + g.mid_lo);
  if (tid == 0 && sm.first < m) atomicMin(&p.info[tl.c].first_moved, lo + sm.first);
}

// ---- caches too long for one workgroup -------------------------------------------------------
// A long cache is cut into tiles of kTileRows rows (over its capacity), one workgroup per tile and
// pass.  Pass P (one kernel each, P = 0..3) leaves the 256 counters of every tile in the workspace;
// the counters of a cache are the sums over its tiles, which every workgroup of the next kernel forms
// for itself (a few thousand additions) before it searches the digit: no atomics between workgroups,
// no counters to clear, no waiting on another workgroup, and one kernel per pass.  The last kernel
// knows the threshold, derives from the stored counters how many survivors the tiles before its own
// hold, and emits its tile.

// State of a long cache's selection after pass P - 1, formed by every workgroup of the kernel that
// follows that pass: the state after pass P - 2 (stored by that kernel's predecessor) advanced by
// the digit search on the summed tile counters of pass P - 1.  Tile 0's workgroup stores it for the
// next kernel.  Ends with a barrier; `hist` is free again.
template <int P>
__device__ __forceinline__ SelState state_before_pass(const CompactParams& p, const SelTile& tl, int k, int* hist,
                                                      int* sm_scan, int* sh_digit, int* sh_need) {
  SelState st = SelState{0u, k, {0, 0, 0, 0}};
  if (P == 0) return st;
  if (P >= 2) st = p.sel_state[(int64_t)tl.long_idx * 4 + (P - 2)];
  const int tid = threadIdx.x;
  if (tid < 256) {
    int sum = 0;
    for (int j = 0; j < tl.n_tiles; ++j) sum += p.tile_hist[((int64_t)(tl.first_tile + j) * 4 + (P - 1)) * 256 + tid];
    hist[tid] = sum;
  }
  __syncthreads();
  find_digit(hist, st.need, sm_scan, sh_digit, sh_need);
  st.prefix |= (uint32_t)*sh_digit << (24 - 8 * (P - 1));
  st.need = *sh_need;
  st.digit[P - 1] = *sh_digit;
  __syncthreads();
  if (tl.tile == 0 && tid == 0) p.sel_state[(int64_t)tl.long_idx * 4 + (P - 1)] = st;
  return st;
}

template <int PASS>
__global__ __launch_bounds__(kSelThreads) void compact_tile_count_kernel(CompactParams p) {
  const SelTile tl = p.tiles[blockIdx.x];
  const int c = tl.c;
  const int tid = threadIdx.x;
  const SelGoal g = sel_goal(p, c);
  if (PASS == 0 && tl.tile == 0) clear_move_state(p, c, p.off[c], g);
  if (PASS == 0 && tl.tile == 0 && tid == 0) {
    // the selection's result record; the emit kernel lowers first_moved with atomicMin
    p.info[c] = g.n <= g.b ? CompactInfo{g.n, g.n, g.n, 0} : CompactInfo{g.b, g.n, g.n, 0};
  }
  if (g.n <= g.b || g.k <= 0) return;  // nothing to rank (uniform over the cache's workgroups)
  __shared__ int hist[256];
  __shared__ int sm_scan[kSelWaves];
  __shared__ int sh_digit, sh_need;
  const SelState st = state_before_pass<PASS>(p, tl, g.k, hist, sm_scan, &sh_digit, &sh_need);
  for (int i = tid; i < 256; i += kSelThreads) hist[i] = 0;
  __syncthreads();
  const int shift = 24 - 8 * PASS;
  const uint32_t mask = PASS == 0 ? 0u : (0xffffffffu << (shift + 8));
  const int j_begin = max(g.mid_lo, tl.tile * kTileRows), j_end = min(g.mid_hi, (tl.tile + 1) * kTileRows);
  count_digits<kTileRows / kSelThreads>(p.score + p.off[c], j_begin, j_end, st.prefix, mask, shift, hist);
  __syncthreads();
  if (tid < 256) p.tile_hist[((int64_t)(tl.first_tile + tl.tile) * 4 + PASS) * 256 + tid] = hist[tid];
}

__global__ __launch_bounds__(kSelThreads) void compact_tile_emit_kernel(CompactParams p) {
  const SelTile tl = p.tiles[blockIdx.x];
  const int c = tl.c;
  const int tid = threadIdx.x;
  const SelGoal g = sel_goal(p, c);
  const int n = g.n;
  const int64_t off = p.off[c];
  int32_t* kept = p.kept + off;
  const int j_begin = tl.tile * kTileRows, j_end = min(n, (tl.tile + 1) * kTileRows);
  if (n <= g.b) {
    if (p.write_identity)
      for (int j = j_begin + tid; j < j_end; j += kSelThreads) kept[j] = j;
    return;
  }
  __shared__ int hist[256];
  __shared__ int sm_scan[kSelWaves];
  __shared__ int sh_digit, sh_need, sh_first;
  __shared__ uint32_t lds_key[kEmitKeyWords];
  uint32_t thr = 0;
  int need_eq = 0, sure_base = 0, eq_base = 0;
  if (g.k > 0) {
    const SelState st = state_before_pass<4>(p, tl, g.k, hist, sm_scan, &sh_digit, &sh_need);
    thr = st.prefix;
    need_eq = st.need;
    // Survivors in the tiles before this one, from their counters: keys that some pass ranked above the
    // threshold's digit, and keys equal to the threshold (capped by need_eq where they are used).
    // One wavefront per earlier tile in turn, its 64 lanes over the 256 counters of each pass.
    const int lane = tid & 63, wave = tid >> 6;
    int sure = 0, eq = 0;
    for (int j = wave; j < tl.tile; j += kSelWaves) {
      const int32_t* th = p.tile_hist + (int64_t)(tl.first_tile + j) * 4 * 256;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int d = lane + 64 * q;
#pragma unroll
        for (int ps = 0; ps < 4; ++ps) sure += d > st.digit[ps] ? th[ps * 256 + d] : 0;
        eq += d == st.digit[3] ? th[3 * 256 + d] : 0;
      }
    }
    (void)block_exclusive_scan(sure, sm_scan, sure_base);
    (void)block_exclusive_scan(eq, sm_scan, eq_base);
  }
  const int before = min(j_begin, n);  // rows in front of this tile
  sure_base += min(before, g.mid_lo) + max(0, before - g.mid_hi);
  if (tid == 0) sh_first = n;
  __syncthreads();
  if (j_begin < j_end)
    emit_rows(p.score + off, kept, g, thr, need_eq, j_begin, j_end, sure_base, eq_base, sm_scan, &sh_first, lds_key);
  __syncthreads();
  if (tid == 0 && sh_first < n) atomicMin(&p.info[c].first_moved, sh_first);
}

// The move is stable and in place: row p <- row kept[p], with kept[p] >= p and kept[p] - p <= (rows evicted).  The rows
// of a cache from the first that moves on are cut into tiles.  The tiles of all caches, numbered in a row, are handed
// out in ascending order by a counter (a ticket).  A tile's workgroup loads its rows, waits for them, raises the tile's
// flag, and stores them once the flags of all earlier tiles of the cache are up whose sources may lie in its range:
// those rows have been read.  A ticket is waited for only by later ones, and raising a flag waits for nothing, so every
// wait ends whatever order the workgroups are started in.  No data passes between workgroups (each reads rows that no
// one has written), only the permission to overwrite, so neither side needs a cache to be written back or invalidated:
// the flags are relaxed device-scope atomics, raised behind an explicit wait for the loads.
//
// Bound by HBM.  What reads and writes together reach here depends on how far apart the rows in flight lie: a plain
// copy of 1 GiB runs at 6.1 to 6.3 TB/s in 16 KiB pieces in address order, at 5.4 in pieces of 256 KiB.  Hence tiles in
// order over the whole arena, 128 KiB each (half of it K), and one workgroup to a compute unit.  A workgroup per run of
// 1024 to 4096 rows, behind a kernel that saved the rows which cross a run's end, took 1096 us for 5 million rows of 512
// bytes, of which nearly all move, and 19 for the rows across the ends; this takes 877.  Whole evictions, us: two workgroups
// to a compute unit 901 (904), but 266240 rows 71.0 (65.7) and 135168 rows of 256 bytes 34.3 (30.5); half as many bytes per
// tile 985; the next ticket drawn while a tile's rows are on their way 958 (the rows in flight lie further apart); a
// workgroup for every tile 920, and where few rows move 155 (60.8), for 20000 workgroups that find nothing to do; a counter
// for each cache and four tiles per workgroup 985.
//
// Caches of up to move_short_rows rows are one tile, so they need neither tickets nor flags: a workgroup moves each.  As
// tiles among the others they left a compute unit idle for most of the latency of a ticket, a table and a row, and were
// slower than runs had been.  Whole evictions, us, runs / tiles / this, rows of 256 bytes where nothing else is said: 1263
// caches of 19 rows 41.4 / 54.8 / 38.8, 695 of 50 33.0 / 38.6 / 30.4, 8 of 58 16.4 / 16.8 / 14.8, 2892 of 18 rows of 128
// bytes 79.7 / 111 / 73.9.  Beside longer caches workgroups behind those that draw tickets serve them, two to a compute
// unit, where they are a quarter of all or more (one that finds a longer cache is launched for nothing): 2253 caches of
// up to 751 rows, 93% short, 81.2 / 91.6 / 73.2; 835 caches, 56% short, 51.8 / 51.1 / 46.2; 2292 caches, 27% short, 211 /
// 164 / 161; 3296 caches of 128-byte rows, one of them of 20000, 125 / 145 / 117.

// The rows of a tile on their way.  PIECES: 16-byte pieces per row.
template <int PIECES, int ROWS>
struct MoveTile {
  static_assert(ROWS <= kMoveThreads && ROWS >= kMoveRowsMin, "a thread per score, a flag per tile");
  static constexpr int kPerPlane = ROWS * PIECES / kMoveThreads;  // pieces per thread and plane
  uint4 kb[kPerPlane], vb[kPerPlane];
  float sc;
  int ps;

  // Destination rows p0 .. e of the cache at `off`; ends with a barrier behind which the workgroup has read all of them.
  __device__ __forceinline__ void load(const CompactParams& p, int64_t off, int p0, int e) {
    const uint4* K = reinterpret_cast<const uint4*>(p.k) + off * PIECES;
    const uint4* V = reinterpret_cast<const uint4*>(p.v) + off * PIECES;
    const int32_t* kept = p.kept + off;
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < kPerPlane; ++i) {
      const int idx = tid + i * kMoveThreads;
      const int64_t src = kept[min(p0 + idx / PIECES, e - 1)];  // clamped: a row of this tile
      kb[i] = load_nt16(K + src * PIECES + idx % PIECES);
      vb[i] = load_nt16(V + src * PIECES + idx % PIECES);
    }
    sc = 0.f;
    ps = 0;
    if (tid < e - p0) {
      const int src = kept[p0 + tid];
      sc = p.score[off + src];
      ps = p.pos[off + src];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's rows are here
    __syncthreads();                                  // and those of the others
  }

  __device__ __forceinline__ void store(const CompactParams& p, int64_t off, int p0, int e) const {
    uint4* K = reinterpret_cast<uint4*>(p.k) + off * PIECES;
    uint4* V = reinterpret_cast<uint4*>(p.v) + off * PIECES;
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < kPerPlane; ++i) {
      const int idx = tid + i * kMoveThreads;
      const int row = p0 + idx / PIECES;
      if (row < e) {
        store_nt16(K + (int64_t)row * PIECES + idx % PIECES, kb[i]);
        store_nt16(V + (int64_t)row * PIECES + idx % PIECES, vb[i]);
      }
    }
    if (tid < e - p0) {
      p.score[off + p0 + tid] = sc;
      p.pos[off + p0 + tid] = ps;
    }
  }
};

// The move of a cache of up to move_short_rows rows by one workgroup.
template <int PIECES>
__device__ __forceinline__ void move_short(const CompactParams& p, int c) {
  const CompactInfo info = p.info[c];
  const int first = info.first_moved, b = info.new_len;
  if (first >= b || b > move_short_rows(PIECES)) return;  // no row moves, or the cache has tiles
  const int64_t off = p.off[c];
  MoveTile<PIECES, move_short_rows(PIECES)> tile;
  tile.load(p, off, first, b);
  tile.store(p, off, first, b);
}

// Workgroups 0 .. n_tickets draw tiles; those behind them, if any, take the caches of up to short_rows rows, which then
// have no tiles.
template <int PIECES>
__global__ __launch_bounds__(kMoveThreads, 4) void compact_move_kernel(CompactParams p, int c0, int n_caches, int n_tickets,
                                                                       int short_rows) {
  if ((int)blockIdx.x >= n_tickets) {
    move_short<PIECES>(p, c0 + (int)blockIdx.x - n_tickets);
    return;
  }
  constexpr int ROWS = move_rows(PIECES);
  extern __shared__ int sh_end[];  // tiles of the caches up to and with this one
  __shared__ int sh_scan[kMoveThreads / 64];
  __shared__ int sh_tile;
  const int tid = threadIdx.x;
  int* const ticket = p.move_ticket + c0;
  int next = 0;
  if (tid == 0) next = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int total = 0;
  for (int i0 = 0; i0 < n_caches; i0 += kMoveThreads) {
    const int i = i0 + tid;
    int n = 0;
    if (i < n_caches) {
      const CompactInfo info = p.info[c0 + i];
      n = info.new_len <= short_rows ? 0 : max(0, info.new_len - info.first_moved + ROWS - 1) / ROWS;
      if (blockIdx.x == 0 && info.first_moved < info.old_len) p.len[c0 + i] = info.new_len;
    }
    int all;
    n += block_exclusive_scan<kMoveThreads / 64>(n, sh_scan, all);
    if (i < n_caches) sh_end[i] = total + n;
    total += all;
  }
  for (;;) {
    if (tid == 0) sh_tile = next;
    __syncthreads();
    const int g = sh_tile;
    if (g >= total) return;  // (uniform over the workgroup)
    int lo = 0;              // the first cache that ends behind tile g
    for (int hi = n_caches - 1; lo < hi;) {
      const int mid = (lo + hi) >> 1;
      if (sh_end[mid] > g) hi = mid; else lo = mid + 1;
    }
    const int t = __builtin_amdgcn_readfirstlane(lo > 0 ? g - sh_end[lo - 1] : g), c = __builtin_amdgcn_readfirstlane(c0 + lo);
    const CompactInfo info = p.info[c];
    const int b = info.new_len, first = info.first_moved, evicted = info.old_len - b;
    const int64_t off = p.off[c];
    int32_t* flags = p.move_flags + move_flag_base(off, c);
    const int p0 = first + t * ROWS, e = min(p0 + ROWS, b);
    MoveTile<PIECES, ROWS> tile;
    tile.load(p, off, p0, e);
    if (tid == 0) __hip_atomic_store(flags + t, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // from the first of the earlier tiles that may hold a row whose source is at or past p0
    for (int j = max(0, (t * ROWS - evicted) / ROWS - 1) + tid; j < t; j += kMoveThreads)
      while (__hip_atomic_load(flags + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) __builtin_amdgcn_s_sleep(1);
    __syncthreads();
    tile.store(p, off, p0, e);
    if (total <= n_tickets) return;  // a tile for each
    if (tid == 0) next = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The same for launches in which no cache has more rows.
template <int PIECES>
__global__ __launch_bounds__(kMoveThreads, PIECES > 16 ? 4 : 8) void compact_move_short_kernel(CompactParams p, int c0) {
  const int c = c0 + blockIdx.x;
  if (threadIdx.x == 0) {
    const CompactInfo info = p.info[c];
    if (info.first_moved < info.old_len) p.len[c] = info.new_len;
  }
  move_short<PIECES>(p, c);
}

}  // namespace

// The launch order holds the n_wide caches of more than kNarrowRows rows first when `sorted`.
hipError_t launch_compact_select(const CompactParams& p, int n_caches, int n_wide, bool sorted, int n_tiles,
                                 const SelTile* spread, int n_spread, int n_cus, hipStream_t s) {
  if (n_caches <= 0) return hipSuccess;
  const dim3 held(kHeldThreads);
  CompactParams q = p;
  if (n_spread > 0) {
    q.tiles = spread;
    compact_spread_count_kernel<<<dim3(n_spread), held, 0, s>>>(q);
    compact_spread_emit_kernel<<<dim3(n_spread), held, 0, s>>>(q);
  } else if (sorted && n_wide > 0 && n_wide < n_caches && n_caches - n_wide <= 6 * ((n_cus - n_wide % n_cus) % n_cus)) {
    // One workgroup to a compute unit instead of two, but the narrow caches run beside the wide ones instead of behind
    // them, on the compute units that the last round of those leaves, while there are few enough for that.  us per
    // eviction, two launches / one, wide x rows and narrow x rows: 100 x 32768 and 8 x 8000 65.5 / 53.0, 400 x 8000
    // 77.4 / 58.4, 1000 x 4000 94.9 / 87.1, 2000 x 8000 145 / 158; 200 x 32768 and 150 x 8000 70.8 / 65.6, 400 x 16000
    // 91.0 / 93.7, 1000 x 4000 98.9 / 107; 300 x 30000 and 400 x 8000 117 / 97.5, 2000 x 8000 183 / 186.
    compact_select_both_kernel<<<dim3(n_caches), held, 0, s>>>(p, n_wide);
  } else {
    if (n_wide > 0)
      compact_select_kernel<kHeldRows / kHeldThreads>
          <<<dim3(sorted ? n_wide : n_caches), held, 0, s>>>(p, kNarrowRows, p.long_rows);
    if (n_wide < n_caches) {
      if (sorted) q.order += n_wide;
      compact_select_kernel<kNarrowRows / kHeldThreads>
          <<<dim3(sorted ? n_caches - n_wide : n_caches), held, 0, s>>>(q, -1, std::min(kNarrowRows, p.long_rows));
    }
  }
  if (n_tiles > 0) {
    const dim3 grid(n_tiles), block(kSelThreads);
    compact_tile_count_kernel<0><<<grid, block, 0, s>>>(p);
    compact_tile_count_kernel<1><<<grid, block, 0, s>>>(p);
    compact_tile_count_kernel<2><<<grid, block, 0, s>>>(p);
    compact_tile_count_kernel<3><<<grid, block, 0, s>>>(p);
    compact_tile_emit_kernel<<<grid, block, 0, s>>>(p);
  }
  return hipGetLastError();
}

template <int PIECES>
void launch_move(const CompactParams& p, int c0, int n_caches, int64_t n_tiles, int n_short, int n_cus, hipStream_t s) {
  const dim3 block(kMoveThreads);
  if (n_tiles == 0) {
    compact_move_short_kernel<PIECES><<<dim3(n_caches), block, 0, s>>>(p, c0);
    return;
  }
  const bool apart = 4 * (int64_t)n_short >= n_caches;
  const int n_tickets = (int)std::min<int64_t>(apart ? n_tiles : n_tiles + n_short, n_cus);
  compact_move_kernel<PIECES><<<dim3(n_tickets + (apart ? n_caches : 0)), block, (size_t)n_caches * 4, s>>>(
      p, c0, n_caches, n_tickets, apart ? move_short_rows(PIECES) : 0);
}

hipError_t launch_compact_move(const CompactParams& p, int c0, int n_caches, const MoveCount* before, int n_cus,
                               hipStream_t s) {
  for (int at = 0; at < n_caches; at += kMoveCaches) {
    const int n = std::min(kMoveCaches, n_caches - at);
    const int64_t n_tiles = before[at + n].tiles - before[at].tiles;
    const int n_short = before[at + n].short_caches - before[at].short_caches;
    if (n_tiles == 0 && n_short == 0) continue;  // no cache has more rows than its budget
    switch (p.row_bytes / 16) {
      case 8: launch_move<8>(p, c0 + at, n, n_tiles, n_short, n_cus, s); break;
      case 16: launch_move<16>(p, c0 + at, n, n_tiles, n_short, n_cus, s); break;
      case 32: launch_move<32>(p, c0 + at, n, n_tiles, n_short, n_cus, s); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace baklava
