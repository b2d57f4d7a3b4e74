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

// Wavefronts per workgroup of a launch that has at most one workgroup per compute unit: they alone must
// keep enough loads in flight (8 KB each, and the next 8 KB during the arithmetic).  Four wavefronts
// without the tile ahead, with lane sums through the LDS crossbar and a rescale on every tile, read the
// 67 MB of 32 fp32 caches (D = 64, two query heads each) in 32 us; this takes 14.  16 where the
// accumulators leave 128 registers, 8 otherwise; up to four query heads the loads bound it, at eight the
// vector ALUs do.  With several workgroups per compute unit those fill it, and items are as short as 256
// rows, one tile for each of eight wavefronts, so the merge at the end weighs more: four wavefronts then
// (88 bf16 caches of 2500 rows per launch, D = 64, four query heads, eight steps of three layers and an
// eviction: 639 us, with eight 1024, as it was before 894).
template <int REGS> constexpr int wide_waves() { return REGS <= 16 ? 16 : 8; }

template <typename T, int D, int GT, int NW>
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
    if (add) append_new_row(p, it, n_old, off_c, token_pos);
    else if (it.start == 0 && threadIdx.x == 0) *p.status = 1;
  }
  if (p.keep_rows && it.start == 0 && threadIdx.x == 0) p.lag_n[(int64_t)it.c * kLagCalls] = n;
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
  const int64_t qrow0 = (int64_t)(c_rel / p.Hkv) * p.Hq + (int64_t)(c_rel % p.Hkv) * G;
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
// which is the softmax of Eq. 7 with the sum over rows regrouped by split.  One workgroup per
// (cache with several work items, query head); 256 / D thread groups share the splits.
template <int D>
__global__ __launch_bounds__(256) void combine_kernel(DecodeParams p) {
  constexpr int GROUPS = 256 / D;
  const int G = p.G;
  const MultiCache mc = p.multi[blockIdx.x / G];
  const int c = mc.c;
  const int g = blockIdx.x % G;
  const int tid = threadIdx.x;
  const int d = tid % D, grp = tid / D;
  const int ib = mc.slot_begin, ie = mc.slot_end;
  // where this call's record goes; read by every thread before the barrier below, written after it
  const int slot = p.lag ? lag_slot(p, p.lag_cnt[(int64_t)c * G + g]) : 0;
  float m = kNegInf, l = 0.f, o = 0.f;
#pragma unroll 8
  for (int s = ib + grp; s < ie; s += GROUPS) {
    const float ms = p.part_ml[((int64_t)s * G + g) * 2];
    const float ls = p.part_ml[((int64_t)s * G + g) * 2 + 1];
    const float os = p.part_o[((int64_t)s * G + g) * D + d];
    const float mn = fmaxf(m, ms);
    const float msafe = (mn == kNegInf) ? 0.f : mn;
    const float a = fast_exp2(m - msafe), b = fast_exp2(ms - msafe);
    l = l * a + ls * b;
    o = o * a + os * b;
    m = mn;
  }
  __shared__ float red_o[GROUPS][D], red_m[GROUPS], red_l[GROUPS];
  red_o[grp][d] = o;
  if (d == 0) { red_m[grp] = m; red_l[grp] = l; }
  __syncthreads();
  if (grp == 0) {
    float mm = red_m[0];
#pragma unroll
    for (int w = 1; w < GROUPS; ++w) mm = fmaxf(mm, red_m[w]);
    const float ms = (mm == kNegInf) ? 0.f : mm;
    float ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < GROUPS; ++w) {
      const float a = fast_exp2(red_m[w] - ms);
      ll += red_l[w] * a;
      oo += red_o[w][d] * a;
    }
    const float inv = 1.f / ll;
    const int c_rel = c - p.cache_begin;
    const int64_t orow = (int64_t)(c_rel / p.Hkv) * p.Hq + (int64_t)(c_rel % p.Hkv) * G + g;
    int n_now = 0;  // live rows after this call (thread 0 of head 0's block)
    p.out[orow * D + d] = oo * inv;
    if (d == 0) {
      p.final_ml[((int64_t)c * G + g) * 2 + 0] = ms;
      p.final_ml[((int64_t)c * G + g) * 2 + 1] = inv;
      if (g == 0) {
        int n = p.len[c];
        if (p.fused_append && n < p.cap[c]) p.len[c] = ++n;  // the fused append's row is now counted
        n_now = n;
      }
    }
    // This head's part of the record a later score pass over the cache needs (see DecodeParams).
    // Each block reads and writes the pending-call counter of its own head only.
    if (p.lag) {
      const int64_t m = (int64_t)c * kLagRows + (slot << p.lag_gp_log2) + g;
      if (tid * 16 < p.row_bytes) {
        const uint4* src = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.q) + orow * p.row_bytes);
        reinterpret_cast<uint4*>(reinterpret_cast<char*>(p.lag_q) + m * p.row_bytes)[tid] = src[tid];
      }
      if (d == 0) {
        p.lag_ml[m * 2 + 0] = ms;
        p.lag_ml[m * 2 + 1] = inv;
        if (g == 0) p.lag_n[(int64_t)c * kLagCalls + slot] = n_now;
        p.lag_cnt[(int64_t)c * G + g] = slot + 1;
      }
    }
  }
}

// score_j += sum_g 2^(q_g . k_j scale - M_g) / L_g  (cumulative attention per cached token, summed
// over the query heads that share the cache), from the K rows alone once the normalisers of the
// call are final: the score update of the vector-ALU path and of bf16 rows of 64 elements, launched right
// after the attention kernel.
// Workgroup (x, y) updates rows [y * kScoreTile, +kScoreTile) of work item x, so that long work
// items still spread over many workgroups.  Row layout as in the attention kernel above: a row
// over D / EPL lanes, 64 / (D / EPL) rows per wavefront load; a wavefront keeps eight of them in
// flight, and lane u of a row's lanes adds the weight of the u-th one, so that the scores of a tile
// are read and written by one instruction each.  One load in flight per wavefront and 1024 rows per
// workgroup took 35 us for 33 MB of K, this takes 8.
// With MERGE a cache's normalisers are merged from its split partials by every workgroup for itself,
// beside its first K loads, and a last slice of workgroups (one per cache) merges the outputs: the pass
// takes the place of the combine kernel.  That saves a launch (eight tracked calls over 67 MB of fp32
// caches, D = 64: 222 -> 203 us), but each workgroup pays for the merge: the caller's rule says where it is
// taken, with both sides measured.
constexpr int kScoreTile = 256;
template <typename T, int D, int GT, bool MERGE>
__global__ __launch_bounds__(256) void score_pass_kernel(ScoreParams p) {
  constexpr int EPL = Row<T>::EPL;
  constexpr int LPR = D / EPL;
  constexpr int RPW = 64 / LPR;
  constexpr int U = 8;
  static_assert(U <= LPR, "one lane of a row per row in flight");
  const Item it = p.items[blockIdx.x];
  const int G = p.G;
  // (the merge advances len itself)
  const int n = MERGE ? p.rows[(int64_t)it.c * kLagCalls] : p.len[it.c];
  const bool merge = MERGE && blockIdx.y == gridDim.y - 1;
  if (merge && (it.start != 0 || it.nsplit == 1)) return;
  const int cnt = merge ? 0 : min(it.start + it.count, n) - it.start;
  const int r_begin = blockIdx.y * kScoreTile;
  if (!merge && r_begin >= cnt) return;
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
  const int64_t qrow0 = (int64_t)(c_rel / p.Hkv) * p.Hq + (int64_t)(c_rel % p.Hkv) * G;
  // (max, 1 / sum) of every query head over the cache's work items
  __shared__ float sm_m[GT], sm_inv[GT];
  if (!MERGE) {
    // final_ml, read below
  } else if (it.nsplit > 1) {
    for (int g = wave; g < G; g += 4) {
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
  } else if ((int)threadIdx.x < G) {
    sm_m[threadIdx.x] = p.ml[((int64_t)it.c * G + threadIdx.x) * 2];
    sm_inv[threadIdx.x] = p.ml[((int64_t)it.c * G + threadIdx.x) * 2 + 1];
  }
  if (MERGE) __syncthreads();
  if (merge) {
    // out = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M), as in the combine kernel
    for (int idx = threadIdx.x; idx < G * D; idx += 256) {
      const int g = idx / D, d = idx % D;
      const float m = sm_m[g];
      float o = 0.f;
#pragma unroll 8
      for (int s = it.slot0; s < it.slot0 + it.nsplit; ++s)
        o += p.part_o[((int64_t)s * G + g) * D + d] * fast_exp2(p.part_ml[((int64_t)s * G + g) * 2] - m);
      p.out[(qrow0 + g) * D + d] = o * sm_inv[g];
    }
    if (threadIdx.x == 0) p.len[it.c] = n;  // a fused append's row is now counted
    return;
  }
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
      M[g] = MERGE ? sm_m[g] : p.ml[((int64_t)it.c * G + g) * 2];
      inv[g] = MERGE ? sm_inv[g] : p.ml[((int64_t)it.c * G + g) * 2 + 1];
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

template <typename T, int D, int GT>
void launch_valu(const DecodeParams& p, int n_items, bool one_wave, hipStream_t s) {
  constexpr int NW = wide_waves<GT * Row<T>::EPL>();
  if (one_wave) decode_partial_valu<T, D, GT, NW><<<dim3(n_items), dim3(64 * NW), 0, s>>>(p);
  else decode_partial_valu<T, D, GT, 4><<<dim3(n_items), dim3(256), 0, s>>>(p);
}

template <typename T, int D>
hipError_t launch_valu_g(const DecodeParams& p, int n_items, bool one_wave, hipStream_t s) {
  if (p.G <= 1) launch_valu<T, D, 1>(p, n_items, one_wave, s);
  else if (p.G <= 2) launch_valu<T, D, 2>(p, n_items, one_wave, s);
  else if (p.G <= 4) launch_valu<T, D, 4>(p, n_items, one_wave, s);
  else if (p.G <= 8) launch_valu<T, D, 8>(p, n_items, one_wave, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_valu(const DecodeParams& p, int dtype, int D, int n_items, bool one_wave, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  if (dtype == 0 && D == 128) return launch_valu_g<uint16_t, 128>(p, n_items, one_wave, s);
  if (dtype == 0 && D == 64) return launch_valu_g<uint16_t, 64>(p, n_items, one_wave, s);
  if (dtype == 1 && D == 128) return launch_valu_g<float, 128>(p, n_items, one_wave, s);
  if (dtype == 1 && D == 64) return launch_valu_g<float, 64>(p, n_items, one_wave, s);
  return hipErrorInvalidValue;
}

hipError_t launch_combine(const DecodeParams& p, int D, int n_multi, hipStream_t s) {
  if (n_multi <= 0) return hipSuccess;
  const dim3 grid(n_multi * p.G), block(256);
  if (D == 128) combine_kernel<128><<<grid, block, 0, s>>>(p);
  else if (D == 64) combine_kernel<64><<<grid, block, 0, s>>>(p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <typename T, int D, bool MERGE>
hipError_t launch_score_g(const ScoreParams& p, const dim3& grid, hipStream_t s) {
  if (p.G <= 2) score_pass_kernel<T, D, 2, MERGE><<<grid, dim3(256), 0, s>>>(p);
  else if (p.G <= 4) score_pass_kernel<T, D, 4, MERGE><<<grid, dim3(256), 0, s>>>(p);
  else if (p.G <= 8) score_pass_kernel<T, D, 8, MERGE><<<grid, dim3(256), 0, s>>>(p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <bool MERGE>
hipError_t launch_score(const ScoreParams& p, int dtype, int D, const dim3& grid, hipStream_t s) {
  if (dtype == 0 && D == 128) return launch_score_g<uint16_t, 128, MERGE>(p, grid, s);
  if (dtype == 0 && D == 64) return launch_score_g<uint16_t, 64, MERGE>(p, grid, s);
  if (dtype == 1 && D == 128) return launch_score_g<float, 128, MERGE>(p, grid, s);
  if (dtype == 1 && D == 64) return launch_score_g<float, 64, MERGE>(p, grid, s);
  return hipErrorInvalidValue;
}

hipError_t launch_score_pass(const ScoreParams& p, int dtype, int D, int n_items, int max_count, bool merge,
                             hipStream_t s) {
  if (n_items <= 0 || max_count <= 0) return hipSuccess;
  const int tiles = (max_count + kScoreTile - 1) / kScoreTile;
  return merge ? launch_score<true>(p, dtype, D, dim3(n_items, tiles + 1), s)
               : launch_score<false>(p, dtype, D, dim3(n_items, tiles), s);
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
