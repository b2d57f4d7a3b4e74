// Decode attention over ragged caches, vector-ALU version, plus the kernels every decode call
// shares: split combine, score update, append, fill.
//
// Each work item (a run of rows of one cache) is one workgroup.  A 256-byte row is spread over 16
// lanes as 16-byte pieces, so one wavefront load instruction fetches four whole rows, fully
// coalesced.  Each lane group keeps its own running (max, sum, output) for every query head of the
// group (online softmax, Eq. 1 re-associated) and the groups are merged once at the end: no barrier
// and no cross-group traffic inside the streaming loop.
#include "common.h"
#include "decode_tail.h"

#include <algorithm>
#include <type_traits>

namespace baklava {

namespace {

struct bf16x8 { uint4 raw; };

template <typename T> struct Row;
template <> struct Row<float> {
  static constexpr int EPL = 4;  // elements per 16-byte piece
  __device__ static void widen(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
};
template <> struct Row<uint16_t> {  // bf16 storage
  static constexpr int EPL = 8;
  __device__ static void widen(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
  }
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

constexpr float kNegInf = -__builtin_huge_valf();

// Merge two online-softmax states that share a query head.
__device__ __forceinline__ void merge_state(float& m, float& l, float* acc, int n_acc, float mo,
                                            float lo, const float* acco) {
  const float mn = fmaxf(m, mo);
  const float ms = (mn == kNegInf) ? 0.f : mn;
  const float a = fast_exp2(m - ms), b = fast_exp2(mo - ms);
  l = l * a + lo * b;
  for (int e = 0; e < n_acc; ++e) acc[e] = acc[e] * a + acco[e] * b;
  m = mn;
}

// Sum over aligned groups of LPR lanes (8, 16 or 32), every lane of a group receiving it: the pairs of
// a butterfly over lane distances 1, 2, 4, 8, 16, taken with data-parallel-primitive operands instead
// of trips through the LDS crossbar (after the first two steps a quad holds equal values, so mirroring
// a row pairs the same sums as exchanging its halves).
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += dpp(v, std::integral_constant<int, 0xb1>{});   // quad_perm:[1,0,3,2]
  v += dpp(v, std::integral_constant<int, 0x4e>{});   // quad_perm:[2,3,0,1]
  v += dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
  if (LPR >= 16) v += dpp(v, std::integral_constant<int, 0x140>{});  // row_mirror
  if (LPR >= 32) v += __shfl_xor(v, 16);
  return v;
}

// v[i] of N values that every lane holds, i the lane's own: a tree of selects by the bits of i (depth first, so that
// few values wait).
template <int N>
__device__ __forceinline__ float select_own(const float* v, int i) {
  if constexpr (N == 1) {
    return v[0];
  } else {
    const float lo = select_own<N / 2>(v, i), hi = select_own<N / 2>(v + N / 2, i);
    return (i & (N / 2)) ? hi : lo;
  }
}

// Wavefronts per workgroup of a launch that has at most one workgroup per compute unit: they alone must
// keep enough loads in flight (8 KB each, and the next 8 KB during the arithmetic).  Four wavefronts
// without the tile ahead, with lane sums through the LDS crossbar and a rescale on every tile, read the
// 67 MB of 32 fp32 caches (D = 64, two query heads each) in 32 us; this takes 14.  16 where the
// accumulators leave 128 registers, 8 otherwise; up to four query heads the loads bound it, at eight the
// vector ALUs do.  With several workgroups per compute unit those fill it, and items are as short as 256
// rows, one tile for each of eight wavefronts, so the merge at the end weighs more: four wavefronts then
// (88 bf16 caches of 2500 rows per launch, D = 64, four query heads, eight steps of three layers and an
// eviction: 639 us, with eight 1024, as it was before 894).
// (16 at four fp32 query heads leave 128 registers where the loop takes 136, so that it spills and loads less far ahead:
// us per call, 16 / 8, a layer of 32 caches of 4096 rows, D = 128, 29.8 / 28.2, tracked 39.5 / 32.3, 8 caches of 4096
// rows 15.5 / 14.0 and 18.8 / 16.4; D = 64 20.0 / 18.3 and 24.4 / 22.2.)
template <int GT, int EPL> constexpr int wide_waves() { return GT < 4 && GT * EPL <= 16 ? 16 : 8; }

// KEEP (score tracking): the scaled logits of the call go to p.logits for the kernel behind this one.  They wait in
// LDS until the work item is done (or a wavefront's part of the area is full): stores between the loads would slow
// the stream far beyond their bytes.
template <typename T, int D, int GT, int NW, bool KEEP>
__global__ __launch_bounds__(64 * NW) void decode_partial_valu(DecodeParams p) {
  constexpr int EPL = Row<T>::EPL;
  constexpr int LPR = D / EPL;   // lanes per row
  constexpr int RPW = 64 / LPR;  // rows per wavefront load
  constexpr int U = 4;           // rows in flight per lane
  constexpr int TILE = RPW * U;

  const Item it = p.items[blockIdx.x];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPR, rg = lane / LPR;
  const int G = p.G;
  const int n_old = p.len[it.c];
  const int64_t off_c = it.row0 - it.start;
  // a fused append only happens while the cache has room (a full cache sets the status word)
  const int add = (p.fused_append && n_old < p.cap[it.c]) ? 1 : 0;
  const int n = n_old + add;
  const int token_pos = p.token_pos_dev ? *p.token_pos_dev : p.token_pos;
  if (p.fused_append) {
    if (add) append_new_row<64 * NW>(p, it, n_old, off_c, token_pos);
    else if (it.start == 0 && threadIdx.x == 0) *p.status = 1;
  }
  if (KEEP && it.start == 0 && threadIdx.x == 0) p.lag_n[(int64_t)it.c * kLagCalls] = n;
  int cnt = min(it.start + it.count, n) - it.start;
  if (cnt < 0) cnt = 0;
  const int64_t row0 = off_c + it.start;
  const T* Kb = reinterpret_cast<const T*>(p.k) + row0 * D + sub * EPL;
  const T* Vb = reinterpret_cast<const T*>(p.v) + row0 * D + sub * EPL;

  // Rows are clamped to the item's last live one; read once per step: non-temporal, so that the
  // stream does not displace other cached data.
  uint4 kraw[U], vraw[U];
  auto load_tile = [&](int t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(t0 + u * RPW + rg, cnt - 1);
      kraw[u] = load_nt16(Kb + (int64_t)r * D);
      vraw[u] = load_nt16(Vb + (int64_t)r * D);
    }
  };
  int t0 = wave * TILE;
  if (t0 < cnt) load_tile(t0);

  const int c_rel = it.c - p.cache_begin;
  const int64_t qrow0 = (int64_t)c_rel * G;
  float qr[GT][EPL];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    if (g < G) {
      const uint4 raw = *reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(p.q) +
                                                        (qrow0 + g) * D + sub * EPL);
      Row<T>::widen(raw, qr[g]);
#pragma unroll
      for (int e = 0; e < EPL; ++e) qr[g][e] *= p.scale_log2e;
    } else {
#pragma unroll
      for (int e = 0; e < EPL; ++e) qr[g][e] = 0.f;
    }
  }

  float m[GT], l[GT], acc[GT][EPL];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    m[g] = kNegInf; l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
  }

  extern __shared__ __attribute__((aligned(16))) float lds_ring[];
  float* const ring = lds_ring + (KEEP ? wave * p.ring_slots * (GT * TILE) : 0);  // [tile][head][row]
  int ring_n = 0;   // tiles in this wavefront's part
  int ring_t0 = 0;  // first row of the oldest one; the others follow at NW * TILE rows each
  auto flush_ring = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int i = lane;
    asm volatile("" : "+v"(i));  // what follows from it is formed here, not kept in registers over the loop
    for (; i < ring_n * (GT * TILE); i += 64) {
      const int g = i / TILE % GT, r = ring_t0 + i / (GT * TILE) * (NW * TILE) + i % TILE;
      if (g < G && r < cnt) p.logits[g * p.logit_stride + row0 + r] = ring[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the area may be written again
    ring_n = 0;
  };

  for (; t0 < cnt; t0 += NW * TILE) {
    uint4 kc[U], vc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { kc[u] = kraw[u]; vc[u] = vraw[u]; }
    if (t0 + NW * TILE < cnt) load_tile(t0 + NW * TILE);  // the next tile is on its way during this one's arithmetic
    float s[U][GT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[EPL];
      Row<T>::widen(kc[u], kf);
      const int r = t0 + u * RPW + rg;
      const bool live = r < cnt;
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) d = fmaf(qr[g][e], kf[e], d);
        d = group_sum<LPR>(d);
        s[u][g] = live ? d : kNegInf;
      }
    }
    if (KEEP) {  // the lanes of a row hold all of its logits: each stores one
      if (ring_n == 0) ring_t0 = t0;
      constexpr int kPer = U * GT < LPR ? U * GT : LPR;
#pragma unroll
      for (int j = 0; j < U * GT; j += kPer) {
        const int i = j + sub;
        const float mine = select_own<kPer>(&s[0][0] + j, sub);
        if (sub < kPer) ring[(ring_n * GT + i % GT) * TILE + i / GT * RPW + rg] = mine;
      }
      if (++ring_n == p.ring_slots) flush_ring();
    }
    float mx[GT];
    bool moves = false;
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      mx[g] = s[0][g];
#pragma unroll
      for (int u = 1; u < U; ++u) mx[g] = fmaxf(mx[g], s[u][g]);
      moves = moves || mx[g] > m[g];
    }
    // The reference is the running maximum, so weights stay in 0 .. 1 and values whose plain sum over the rows
    // fits fp32 do not overflow.  (Left to lag by up to 8 in log2 units it is 2 to 7% faster at four and eight
    // query heads, 35.2 against 37.5 us for two fp32 caches of 32768 rows, D = 128, eight heads, and equal at
    // one and two, but weights reach 2^8.  Set 8 above a new maximum it is as fast, but the difference to it
    // loses bits: error 2.2e-7 against 1.7e-7.)
    if (__any(moves)) {
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        const float mn = fmaxf(m[g], mx[g]);
        const float alpha = fast_exp2(m[g] - ((mn == kNegInf) ? 0.f : mn));
        m[g] = mn;
        l[g] *= alpha;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] *= alpha;
      }
    }
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      const float ms = (m[g] == kNegInf) ? 0.f : m[g];
#pragma unroll
      for (int u = 0; u < U; ++u) s[u][g] = fast_exp2(s[u][g] - ms);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float vf[EPL];
      Row<T>::widen(vc[u], vf);
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        l[g] += s[u][g];
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(s[u][g], vf[e], acc[g][e]);
      }
    }
  }

  if (KEEP && ring_n > 0) flush_ring();

  // Merge the lane groups of a wavefront (lanes with equal `sub`).
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      float acco[EPL];
      const float mo = __shfl_xor(m[g], o), lo = __shfl_xor(l[g], o);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acco[e] = __shfl_xor(acc[g][e], o);
      merge_state(m[g], l[g], acc[g], EPL, mo, lo, acco);
    }
  }

  // Hand the wavefronts' results over through LDS.
  __shared__ float sm[NW * GT * D + 2 * NW * GT];
  float* sm_o = sm;                  // [NW][GT][D]
  float* sm_m = sm + NW * GT * D;    // [NW][GT]
  float* sm_l = sm_m + NW * GT;      // [NW][GT]
  if (rg == 0) {
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      if (sub == 0) { sm_m[wave * GT + g] = m[g]; sm_l[wave * GT + g] = l[g]; }
#pragma unroll
      for (int e = 0; e < EPL; ++e) sm_o[(wave * GT + g) * D + sub * EPL + e] = acc[g][e];
    }
  }
  __syncthreads();
  finish_item<D, GT, NW>(p, it, G, n, sm_o, sm_m, sm_l);
}

// Merge of the split partials of one (cache, query head):
//   out = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M)
// which is the softmax of Eq. 7 with the sum over rows regrouped by split.  One workgroup per (cache with several work
// items, query head); THREADS / D thread groups share the splits.  A kernel this small is a chain of latencies: what
// does not depend on the maximum M is requested before it is formed (the first kAhead outputs of every group, the
// record's inputs), every wavefront forms M and the splits' factors for itself, one split per lane, and a group then
// reads the factor of a split from its lane, so that the sums over splits are plain multiply-adds, kAhead outputs at a
// time.  A layer of 8 caches of up to 8192 rows: 9.9 us per attention call (10.5 with a running rescale per split and
// integer divisions in front of the first loads), of 131072 rows 48.4 (54).
template <int D, int THREADS>
__device__ __forceinline__ void combine_head(const DecodeParams& p, int multi, int g) {
  constexpr int GROUPS = THREADS / D, kAhead = 8, kHeld = 4;
  const int G = p.G;
  const MultiCache mc = p.multi[multi];
  const int c = mc.c;
  const int tid = threadIdx.x, lane = tid & 63;
  const int d = tid % D, grp = __builtin_amdgcn_readfirstlane(tid / D);  // (D is a multiple of 64)
  const int n_split = mc.slot_end - mc.slot_begin;
  const int64_t first = (int64_t)mc.slot_begin * G + g;  // partial s of this head: first + s * G
  const float2* ml = reinterpret_cast<const float2*>(p.part_ml) + first;
  const float* po = p.part_o + first * D + d;
  const int64_t orow = (int64_t)(c - p.cache_begin) * G + g;
  // Element d of the output, from the sums over the splits, and this head's part of the record a later score pass over
  // the cache needs (see DecodeParams).  Each block reads and writes the pending-call counter of its own head only;
  // the threads that write a record are of one wavefront, and have read the counter before.
  const int slot = p.lag ? lag_slot(p, p.lag_cnt[(int64_t)c * G + g]) : 0;
  uint4 q_piece = make_uint4(0, 0, 0, 0);
  if (p.lag && tid * 16 < p.row_bytes)
    q_piece = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.q) + orow * p.row_bytes)[tid];
  const int n_old = p.len[c];
  const int n_now = n_old + (p.fused_append && n_old < p.cap[c] ? 1 : 0);  // live rows after this call
  auto write_out = [&](float o, float l, float m) {
    const float inv = 1.f / l;
    p.out[orow * D + d] = o * inv;
    if (d == 0) {
      p.final_ml[((int64_t)c * G + g) * 2 + 0] = m;
      p.final_ml[((int64_t)c * G + g) * 2 + 1] = inv;
      if (g == 0 && n_now != n_old) p.len[c] = n_now;  // the fused append's row is now counted
    }
    if (p.lag) {
      const int64_t r = (int64_t)c * kLagRows + (slot << p.lag_gp_log2) + g;
      if (tid * 16 < p.row_bytes) reinterpret_cast<uint4*>(reinterpret_cast<char*>(p.lag_q) + r * p.row_bytes)[tid] = q_piece;
      if (d == 0) {
        p.lag_ml[r * 2 + 0] = m;
        p.lag_ml[r * 2 + 1] = inv;
        if (g == 0) p.lag_n[(int64_t)c * kLagCalls + slot] = n_now;
        p.lag_cnt[(int64_t)c * G + g] = slot + 1;
      }
    }
  };
  // A few splits: launches over many caches have these, and are bound by what a workgroup takes in all.  One thread per
  // element forms everything for itself, without the exchanges between lanes (six for each of two reductions).  us per
  // call over 504 caches of 820 rows on average (mostly two to four work items), all layers at once, with the exchanges
  // / without: D = 128, 4 heads 39.0 / 37.9, 16 heads 49.2 / 46.2, D = 64, 8 heads 24.7 / 22.6; 200 caches of 2048 rows
  // (six), D = 128, 16 heads 50.0 / 49.4.
  auto add_few = [&](auto most) {
    constexpr int N = decltype(most)::value;
    float2 x[N];
    float v[N];
#pragma unroll
    for (int s = 0; s < N; ++s) {
      x[s] = make_float2(kNegInf, 0.f);
      v[s] = 0.f;
      if (s < n_split) {
        x[s] = ml[s * G];
        v[s] = po[(int64_t)s * (G * D)];
      }
    }
    float m = x[0].x;
#pragma unroll
    for (int s = 1; s < N; ++s) m = fmaxf(m, x[s].x);
    m = (m == kNegInf) ? 0.f : m;
    float o = 0.f, l = 0.f;
#pragma unroll
    for (int s = 0; s < N; ++s) {
      if (s < n_split) {
        const float a = fast_exp2(x[s].x - m);
        l = fmaf(a, x[s].y, l);
        o = fmaf(a, v[s], o);
      }
    }
    write_out(o, l, m);
  };
  if (n_split <= 8) {
    if (grp != 0) return;
    if (n_split <= 4) add_few(std::integral_constant<int, 4>{});
    else add_few(std::integral_constant<int, 8>{});
    return;
  }
  float2 held[kHeld];  // split 64 h + lane
#pragma unroll
  for (int h = 0; h < kHeld; ++h) {
    held[h] = make_float2(kNegInf, 0.f);
    if (64 * h + lane < n_split) held[h] = ml[(64 * h + lane) * G];
  }
  auto load_outputs = [&](float (&v)[kAhead], int s0) {  // of splits s0, s0 + GROUPS, ...: past the last one it again
#pragma unroll
    for (int k = 0; k < kAhead; ++k) v[k] = po[(int64_t)min(s0 + k * GROUPS, n_split - 1) * (G * D)];
  };
  float v[kAhead];
  load_outputs(v, grp);

  float m = kNegInf;
#pragma unroll
  for (int h = 0; h < kHeld; ++h) m = fmaxf(m, held[h].x);
  for (int s = 64 * kHeld + lane; s < n_split; s += 64) m = fmaxf(m, ml[s * G].x);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  m = (m == kNegInf) ? 0.f : m;
  float o = 0.f, l = 0.f;
  // 64 splits, one per lane; outputs of kAhead splits per group at a time, the first ones on their way already
  auto add_splits = [&](int s0, float2 mine) {
    const float a = fast_exp2(mine.x - m);
    l += a * mine.y;
    const int end = min(n_split, s0 + 64);
    for (int s = s0 + grp; s < end; s += kAhead * GROUPS) {
      if (s != grp) load_outputs(v, s);
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
        if (s + k * GROUPS < end)
          o = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), s + k * GROUPS - s0)), v[k], o);
    }
  };
  static_assert(64 % GROUPS == 0, "a group's splits of every 64 start at its number");
#pragma unroll
  for (int h = 0; h < kHeld; ++h)
    if (64 * h < n_split) add_splits(64 * h, held[h]);
  for (int s0 = 64 * kHeld; s0 < n_split; s0 += 64)
    add_splits(s0, s0 + lane < n_split ? ml[(s0 + lane) * G] : make_float2(kNegInf, 0.f));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
  __shared__ float red_o[GROUPS][D];
  red_o[grp][d] = o;
  __syncthreads();
  if (grp == 0) {
#pragma unroll
    for (int w = 1; w < GROUPS; ++w) o += red_o[w][d];
    write_out(o, l, m);
  }
}

constexpr int kFinishRowsPerThread = 2;

template <int D, int THREADS>
__global__ __launch_bounds__(THREADS) void combine_kernel(DecodeParams p) {
  combine_head<D, THREADS>(p, blockIdx.x, blockIdx.y);
}

// The end of a tracked call without records: in place of the combine kernel (the first n_combine workgroups, one per
// cache with several work items and query head) and of a pass over the K rows,
//   score_j += sum_g 2^(x_gj - M_g) / L_g   (cumulative attention per cached token, summed over the query heads)
// from the logits x that the attention kernel has left.  The other workgroups take two rows per thread of a work item
// and merge their cache's normalisers from the split partials for themselves, behind the loads of the rows.
// (n_items > 0: a grid of two dimensions, the first row of workgroups for the partials, then one per tile of rows.)
// Reads 4 G bytes per row where a pass over the K rows read the row and formed the products again: 8 tracked calls
// over 67 MB of fp32 caches (D = 64, two query heads) take 167 us (203), four steps of two layers of 32 caches of 4096
// rows, D = 128, eight heads, 377 (499), bf16, D = 64, eight heads, 154 (199).
template <int D, int GT, int THREADS>
__global__ __launch_bounds__(THREADS) void finish_kernel(DecodeParams p, int n_combine, int tiles, int n_items) {
  constexpr int R = kFinishRowsPerThread, kRows = R * THREADS;
  if ((int)blockIdx.x < n_combine && blockIdx.y == 0) {
    combine_head<D, THREADS>(p, (uint32_t)blockIdx.x / (uint32_t)p.G, (uint32_t)blockIdx.x % (uint32_t)p.G);
    return;
  }
  uint32_t item = blockIdx.x, tile = blockIdx.y - 1;
  if (n_items == 0) {
    item = (blockIdx.x - n_combine) / (uint32_t)tiles;
    tile = (blockIdx.x - n_combine) % (uint32_t)tiles;
  } else if (blockIdx.y == 0 || (int)item >= n_items) {
    return;
  }
  const Item it = p.items[item];
  const int G = p.G;
  const int n = p.lag_n[(int64_t)it.c * kLagCalls];  // (len may already count this call's new row, or not yet)
  const int cnt = min(it.start + it.count, n) - it.start;
  const int r_begin = tile * kRows;
  if (r_begin >= cnt) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float x[R][GT], old[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t row = it.row0 + min(r_begin + k * THREADS + tid, cnt - 1);
#pragma unroll
    for (int g = 0; g < GT; ++g) x[k][g] = p.logits[min(g, G - 1) * p.logit_stride + row];
    old[k] = p.score[row];
  }
  // (max, 1 / sum) of every query head over the cache's work items
  __shared__ float sm_m[GT], sm_inv[GT];
  if (it.nsplit > 1) {
    for (int g = wave; g < G; g += THREADS / 64) {
      float m = kNegInf, l = 0.f;
      for (int s = lane; s < it.nsplit; s += 64) m = fmaxf(m, p.part_ml[((int64_t)(it.slot0 + s) * G + g) * 2]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
      m = (m == kNegInf) ? 0.f : m;
      for (int s = lane; s < it.nsplit; s += 64) {
        const float* ml = p.part_ml + ((int64_t)(it.slot0 + s) * G + g) * 2;
        l += ml[1] * fast_exp2(ml[0] - m);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
      if (lane == 0) { sm_m[g] = m; sm_inv[g] = 1.f / l; }
    }
  } else if (tid < G) {
    sm_m[tid] = p.final_ml[((int64_t)it.c * G + tid) * 2];
    sm_inv[tid] = p.final_ml[((int64_t)it.c * G + tid) * 2 + 1];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = r_begin + k * THREADS + tid;
    float w = 0.f;
#pragma unroll
    for (int g = 0; g < GT; ++g)
      if (g < G) w += fast_exp2(x[k][g] - sm_m[g]) * sm_inv[g];
    if (r < cnt) p.score[it.row0 + r] = old[k] + w;
  }
}

// The score update of the vector kernel over rows whose calls are otherwise recorded (bf16, D = 128), right after the
// combine kernel: a pass over the K rows.
// Workgroup (x, y) updates rows [y * kScoreTile, +kScoreTile) of work item x, so that long work
// items still spread over many workgroups.  Row layout as in the attention kernel above: a row
// over D / EPL lanes, 64 / (D / EPL) rows per wavefront load; a wavefront keeps eight of them in
// flight, and lane u of a row's lanes adds the weight of the u-th one, so that the scores of a tile
// are read and written by one instruction each.
constexpr int kScoreTile = 256;
template <typename T, int D, int GT>
__global__ __launch_bounds__(256) void score_pass_kernel(ScoreParams p) {
  constexpr int EPL = Row<T>::EPL;
  constexpr int LPR = D / EPL;
  constexpr int RPW = 64 / LPR;
  constexpr int U = 8;
  static_assert(U <= LPR, "one lane of a row per row in flight");
  const Item it = p.items[blockIdx.x];
  const int G = p.G;
  const int cnt = min(it.start + it.count, p.len[it.c]) - it.start;
  const int r_begin = blockIdx.y * kScoreTile;
  if (r_begin >= cnt) return;
  const int r_end = min(cnt, r_begin + kScoreTile);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPR, rg = lane / LPR;
  const T* Kb = reinterpret_cast<const T*>(p.k) + it.row0 * D + sub * EPL;
  uint4 kraw[U];
  auto load_tile = [&](int r0) {
#pragma unroll
    for (int u = 0; u < U; ++u) kraw[u] = load_nt16(Kb + (int64_t)min(r0 + u * RPW + rg, r_end - 1) * D);
  };
  int r0 = r_begin + wave * (U * RPW);
  if (r0 < r_end) load_tile(r0);
  const int c_rel = it.c - p.cache_begin;
  const int64_t qrow0 = (int64_t)c_rel * G;
  const T* qrows = reinterpret_cast<const T*>(p.q) + qrow0 * D;
  float qr[GT][EPL], M[GT], inv[GT];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    M[g] = 0.f;
    inv[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) qr[g][e] = 0.f;
    if (g < G) {
      Row<T>::widen(*reinterpret_cast<const uint4*>(qrows + g * D + sub * EPL), qr[g]);
#pragma unroll
      for (int e = 0; e < EPL; ++e) qr[g][e] *= p.scale_log2e;
      M[g] = p.ml[((int64_t)it.c * G + g) * 2];
      inv[g] = p.ml[((int64_t)it.c * G + g) * 2 + 1];
    }
  }
  float* sc = p.score + it.row0;
  for (; r0 < r_end; r0 += 4 * U * RPW) {
    const int r = r0 + sub * RPW + rg;  // the row whose score this lane updates (sub < U)
    const bool mine = sub < U && r < r_end;
    const float old = mine ? sc[r] : 0.f;
    float w_mine = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[EPL];
      Row<T>::widen(kraw[u], kf);
      float w = 0.f;
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) d = fmaf(qr[g][e], kf[e], d);
        w += fast_exp2(group_sum<LPR>(d) - M[g]) * inv[g];  // heads beyond G: 2^0 * 0
      }
      w_mine = sub == u ? w : w_mine;
    }
    if (r0 + 4 * U * RPW < r_end) load_tile(r0 + 4 * U * RPW);
    if (mine) sc[r] = old + w_mine;
  }
}

// [K'; K_t], [V'; V_t] of Eq. 7: the new row goes to slot len, then len += 1.
__global__ __launch_bounds__(64) void append_kernel(AppendParams p) {
  const int c = p.cache_begin + blockIdx.x;
  const int n = p.len[c];
  if (n >= p.cap[c]) return;  // the host has already refused this case
  const int64_t row = p.off[c] + n;
  const int pieces = p.row_bytes / 16;
  const int lane = threadIdx.x;
  const int plane = lane / 32, piece = lane % 32;
  if (piece < pieces) {
    const char* src = reinterpret_cast<const char*>(plane ? p.v_new : p.k_new) +
                      (int64_t)blockIdx.x * p.row_bytes + piece * 16;
    char* dst = reinterpret_cast<char*>(plane ? p.v : p.k) + row * p.row_bytes + piece * 16;
    *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
  }
  if (lane == 63) {
    p.score[row] = 0.f;
    p.pos[row] = p.token_pos_dev ? *p.token_pos_dev : p.token_pos;
  }
  __syncthreads();
  if (lane == 0) p.len[c] = n + 1;
}

// Live lengths handed over among the kernel's arguments, and the records of pending calls emptied: one
// small dispatch instead of a fill and a staged copy from pageable memory.
__global__ __launch_bounds__(kLengthsPerLaunch) void set_lengths_kernel(LengthsParams p) {
  const int c = threadIdx.x;
  if (c >= p.count) return;
  p.len[c] = p.value[c];
  for (int g = 0; g < p.G; ++g) p.lag_cnt[c * p.G + g] = 0;
}

__global__ void fill_i32_kernel(int32_t* dst, int32_t value, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = value;
}

// LDS for the logits that wait (KEEP), beside the hand-over area: within the 64 KiB that need no attribute in a launch
// of one workgroup per compute unit, less where several share one.
constexpr int kRingAlone = 60 * 1024, kRingShared = 16 * 1024;

template <typename T, int D, int GT, int NW>
void launch_valu_nw(DecodeParams p, int n_items, int max_count, bool one_wave, hipStream_t s) {
  const dim3 grid(n_items), block(64 * NW);
  if constexpr (Row<T>::EPL == 8 && D == 128) p.logits = nullptr;  // (calls over these rows leave none)
  if (!p.logits) {
    decode_partial_valu<T, D, GT, NW, false><<<grid, block, 0, s>>>(p);
    return;
  }
  if constexpr (!(Row<T>::EPL == 8 && D == 128)) {
    constexpr int kTile = 64 / (D / Row<T>::EPL) * 4, kSlot = GT * kTile * 4;  // rows of a tile, bytes of its logits
    constexpr int kHandOver = (NW * GT * D + 2 * NW * GT) * 4;
    const int room = one_wave ? kRingAlone - kHandOver : kRingShared;
    const int need = (max_count + NW * kTile - 1) / (NW * kTile);
    p.ring_slots = std::max(1, std::min(room / (NW * kSlot), need));
    decode_partial_valu<T, D, GT, NW, true><<<grid, block, (size_t)p.ring_slots * NW * kSlot, s>>>(p);
  }
}

template <typename T, int D, int GT>
void launch_valu(const DecodeParams& p, int n_items, int max_count, bool one_wave, hipStream_t s) {
  constexpr int NW = wide_waves<GT, Row<T>::EPL>();
  if (one_wave) launch_valu_nw<T, D, GT, NW>(p, n_items, max_count, one_wave, s);
  else launch_valu_nw<T, D, GT, 4>(p, n_items, max_count, one_wave, s);
}

template <typename T, int D>
hipError_t launch_valu_g(const DecodeParams& p, int n_items, int max_count, bool one_wave, hipStream_t s) {
  if (p.G <= 1) launch_valu<T, D, 1>(p, n_items, max_count, one_wave, s);
  else if (p.G <= 2) launch_valu<T, D, 2>(p, n_items, max_count, one_wave, s);
  else if (p.G <= 4) launch_valu<T, D, 4>(p, n_items, max_count, one_wave, s);
  else if (p.G <= 8) launch_valu<T, D, 8>(p, n_items, max_count, one_wave, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_valu(const DecodeParams& p, int dtype, int D, int n_items, int max_count, bool one_wave,
                              hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  if (dtype == 0 && D == 128) return launch_valu_g<uint16_t, 128>(p, n_items, max_count, one_wave, s);
  if (dtype == 0 && D == 64) return launch_valu_g<uint16_t, 64>(p, n_items, max_count, one_wave, s);
  if (dtype == 1 && D == 128) return launch_valu_g<float, 128>(p, n_items, max_count, one_wave, s);
  if (dtype == 1 && D == 64) return launch_valu_g<float, 64>(p, n_items, max_count, one_wave, s);
  return hipErrorInvalidValue;
}

// Caches of more work items than this are merged by 1024 threads per head instead of 256.  us per call, 256 / 1024: a
// layer of 8 caches of up to 8192 rows (about 80 work items) 10.2 / 9.9, of 131072 rows 54.8 / 48.4; 32 caches (20) 18.5 /
// 18.0; at 16 and fewer equal.  (n_x: workgroups that the grid's first dimension has to hold.)
constexpr int kManySplits = 16;
constexpr int64_t kMostThreads = (int64_t)1 << 32;  // a grid dimension holds fewer; one of more runs in part, without an error
bool merge_by_1024(int most_split, int64_t n_x) { return most_split > kManySplits && n_x < kMostThreads / 1024; }

hipError_t launch_combine(const DecodeParams& p, int D, int n_multi, int most_split, hipStream_t s) {
  if (n_multi <= 0) return hipSuccess;
  const dim3 grid(n_multi, p.G);
  if (merge_by_1024(most_split, n_multi)) {
    if (D == 128) combine_kernel<128, 1024><<<grid, dim3(1024), 0, s>>>(p);
    else if (D == 64) combine_kernel<64, 1024><<<grid, dim3(1024), 0, s>>>(p);
    else return hipErrorInvalidValue;
  } else {
    if (D == 128) combine_kernel<128, 256><<<grid, dim3(256), 0, s>>>(p);
    else if (D == 64) combine_kernel<64, 256><<<grid, dim3(256), 0, s>>>(p);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D, int THREADS>
hipError_t launch_finish_d(const DecodeParams& p, int n_multi, int n_items, int max_count, hipStream_t s) {
  // One grid dimension while it holds all workgroups; work items times the tiles of the longest one may be 2^32 threads
  // and more (65536 caches, one of 131072 rows), and then take two.  (Two always: a layer of 8 caches of 32768 rows in
  // all, bf16, D = 64, four heads, 10.5 / 11.2 us per call, for the workgroups that have nothing to do.)
  constexpr int kRows = kFinishRowsPerThread * THREADS;
  const int tiles = (max_count + kRows - 1) / kRows, n_combine = n_multi * p.G;
  const int64_t all = n_combine + (int64_t)n_items * tiles;
  const bool flat = all < kMostThreads / THREADS;
  const dim3 grid(flat ? (unsigned)all : (unsigned)std::max(n_combine, n_items), flat ? 1 : 1 + tiles), block(THREADS);
  const int n = flat ? 0 : n_items;
  if (p.G <= 1) finish_kernel<D, 1, THREADS><<<grid, block, 0, s>>>(p, n_combine, tiles, n);
  else if (p.G <= 2) finish_kernel<D, 2, THREADS><<<grid, block, 0, s>>>(p, n_combine, tiles, n);
  else if (p.G <= 4) finish_kernel<D, 4, THREADS><<<grid, block, 0, s>>>(p, n_combine, tiles, n);
  else if (p.G <= 8) finish_kernel<D, 8, THREADS><<<grid, block, 0, s>>>(p, n_combine, tiles, n);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_finish(const DecodeParams& p, int D, int n_multi, int most_split, int n_items, int max_count,
                         hipStream_t s) {
  if (n_items <= 0 || max_count <= 0) return hipSuccess;
  const bool wide = merge_by_1024(most_split, std::max<int64_t>((int64_t)n_multi * p.G, n_items));
  if (D == 128) return wide ? launch_finish_d<128, 1024>(p, n_multi, n_items, max_count, s)
                            : launch_finish_d<128, 256>(p, n_multi, n_items, max_count, s);
  if (D == 64) return wide ? launch_finish_d<64, 1024>(p, n_multi, n_items, max_count, s)
                           : launch_finish_d<64, 256>(p, n_multi, n_items, max_count, s);
  return hipErrorInvalidValue;
}

hipError_t launch_score_pass(const ScoreParams& p, int n_items, int max_count, hipStream_t s) {
  if (n_items <= 0 || max_count <= 0) return hipSuccess;
  const dim3 grid(n_items, (max_count + kScoreTile - 1) / kScoreTile), block(256);
  if (p.G <= 2) score_pass_kernel<uint16_t, 128, 2><<<grid, block, 0, s>>>(p);
  else if (p.G <= 4) score_pass_kernel<uint16_t, 128, 4><<<grid, block, 0, s>>>(p);
  else if (p.G <= 8) score_pass_kernel<uint16_t, 128, 8><<<grid, block, 0, s>>>(p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_append(const AppendParams& p, int n_caches, hipStream_t s) {
  if (n_caches <= 0) return hipSuccess;
  append_kernel<<<dim3(n_caches), dim3(64), 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_set_lengths(const LengthsParams& p, hipStream_t s) {
  if (p.count <= 0) return hipSuccess;
  set_lengths_kernel<<<dim3(1), dim3(kLengthsPerLaunch), 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* dst, int32_t value, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(dst, value, n);
  return hipGetLastError();
}

}  // namespace baklava
