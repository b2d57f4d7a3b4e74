// Decode attention over ragged caches of fp32 rows, matrix version (D = 128 or 64, up to 8 query heads per KV head, the most
// that fp32 caches may have; taken from five on).
//
// Both products of a tile of 16 rows run on v_mfma_f32_16x16x4_f32, whose operands, products and sums are fp32, with
// the G query heads on the N side (padded to 16):
//
//   S^T[row, g]  = K[row, :] . Q[g, :]          A = K (whole rows staged through LDS), B = Q (registers)
//   O^T[d, g]   += V^T[d, rows] . P^T[rows, g]  A = V^T (straight from the loads), B = P^T
//
// The head-dim elements of the first product are numbered so that one 16-byte read of a lane feeds four instructions:
// step (i, e) takes element 16 i + 4 j + e from the lanes of group j = lane / 16.  The accumulator of S^T (lane (g, j),
// register c: row 4 j + c) is the B operand of step c of the second product once that step takes rows c, 4 + c, 8 + c
// and 12 + c; lane (m, j) then loads 16 bytes of row 4 j + c, elements 64 h + 4 m .. + 3, which are row m of four A
// operands.  So neither the weights nor V pass through LDS or another lane.
//
// Each wavefront streams its own slabs of rows; there is no barrier in the loop.  Bound by HBM: a tile of 16 rows (16 KiB
// of K and V at D = 128) takes 64 instructions of 32 cycles, so the matrix cores of a compute unit follow at about 75 GB/s,
// of which it is given 27.  The vector kernel forms 2 G D products per row on 256 lanes and is bound by that from five
// heads on: 32 caches of 4096 rows, D = 128, eight heads 44.0 us, here 31.2 (19.0 for the bytes).
//
// Rounding.  Every instruction starts at zero and adds four products; logits are sums of these in pairs, outputs grow by
// sums over eight rows.  Against 64 bits the outputs of that call are off by 1.86e-7 (vector kernel 2.04e-7), from caches of 300
// rows both by 1.5e-7; with one sum over a wavefront's rows and one over 32 elements of a logit it was 2.4e-7.
#include "common.h"
#include "decode_tail.h"

#include <algorithm>

namespace baklava {

namespace {

typedef float floatx4_t __attribute__((ext_vector_type(4)));

constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kLowest = -3.402823466e38f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// What follows from the head dimension.
template <int D>
struct Shape {
  static constexpr int kTiles = 128 / D;           // tiles of 16 rows per slab: 8 KiB of K and of V
  static constexpr int kRows = 16 * kTiles;        // rows per wavefront iteration
  static constexpr int kPieces = D / 4;            // 16-byte pieces of a row
  static constexpr int kLoadRows = 64 / kPieces;   // rows per load instruction of K
  static constexpr int kLoads = kRows / kLoadRows; // load instructions per slab and plane
  static constexpr int kHalves = D / 64;           // 64-element parts of a row of V
  static constexpr int kKStride = D * 4 + 16;      // bytes between staged K rows: the 16 bytes that 16 lanes read of
                                                   // 16 consecutive rows spread over all banks
};

// KEEP (score tracking): the scaled logits of the call go to p.logits for the kernel behind this one; they wait in LDS
// until the work item is done (or a wavefront's part of the area is full).
template <int D, int NW, bool KEEP>
__global__ __launch_bounds__(64 * NW, 2) void decode_partial_mfma_f32(DecodeParams p) {
  using S = Shape<D>;
  constexpr int kRows = S::kRows, kKStride = S::kKStride, kStage = kRows * kKStride;
  constexpr int kHandOver = (NW * 16 * D + 2 * NW * 16) * 4;
  __shared__ __attribute__((aligned(16))) unsigned char lds[NW * kStage > kHandOver ? NW * kStage : kHandOver];
  extern __shared__ __attribute__((aligned(16))) float lds_ring[];

  const Item it = p.items[blockIdx.x];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n16 = lane & 15, jg = lane >> 4;
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
  const char* Kb = reinterpret_cast<const char*>(p.k) + row0 * (D * 4);
  const char* Vb = reinterpret_cast<const char*>(p.v) + row0 * (D * 4);
  unsigned char* myk = lds + wave * kStage;

  // Rows are clamped to the item's last live one, so nothing outside the live rows is ever read; read once per step:
  // non-temporal, so that the stream does not displace other cached data.  (Offsets from the item's first row fit 32
  // bits: a work item spans at most 2^22 rows.)
  const int last = cnt - 1;
  const int k_row = lane / S::kPieces, k_piece = lane % S::kPieces;
  uint4 kr[S::kLoads];
  uint4 vr[S::kTiles][4][S::kHalves];
  auto load_k = [&](int t0) {
#pragma unroll
    for (int i = 0; i < S::kLoads; ++i)
      kr[i] = load_nt16(Kb + (uint32_t)(min(t0 + k_row + S::kLoadRows * i, last) * (D * 4) + k_piece * 16));
  };
  auto load_v = [&](int t0) {
#pragma unroll
    for (int T = 0; T < S::kTiles; ++T)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int h = 0; h < S::kHalves; ++h)
          vr[T][c][h] = load_nt16(Vb + (uint32_t)(min(t0 + 16 * T + 4 * jg + c, last) * (D * 4) + 256 * h + 16 * n16));
  };

  int t0 = wave * kRows;
  if (t0 < cnt) load_k(t0);
  // B operand of the first product: lane (g, j), step (i, e) holds Q[g][16 i + 4 j + e], with the scale
  const int64_t qrow0 = (int64_t)(it.c - p.cache_begin) * G;
  floatx4_t qb[D / 16];
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    qb[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    if (n16 < G) qb[i] = *reinterpret_cast<const floatx4_t*>(reinterpret_cast<const float*>(p.q) + (qrow0 + n16) * D + 16 * i + 4 * jg);
#pragma unroll
    for (int e = 0; e < 4; ++e) qb[i][e] *= p.scale_log2e;
  }
  if (t0 < cnt) load_v(t0);

  // Lane (g, j), register i: O[g][64 h + 4 (4 j + i) + e].  Sums over eight rows are formed on their own and then added:
  // one sum over all rows of a wavefront would lose more to rounding than the vector kernel's many.
  floatx4_t o[S::kHalves][4];
#pragma unroll
  for (int h = 0; h < S::kHalves; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[h][e] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // Running max of head n16, log2 units, equal in the 4 lanes of a head, from the lowest finite value on: rows with a
  // logit of -inf weigh 2^-inf = 0, also before the first finite one.
  float m_run = kLowest;
  float l_part = 0.f;  // this lane's share of the running sum

  float* ring = lds_ring + (KEEP ? wave * p.ring_slots * G * kRows : 0);  // [slab][head][row]
  int ring_n = 0;   // slabs held there
  int ring_t0 = 0;  // first row of the oldest one; the others follow at NW * kRows rows each
  auto flush_ring = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // As many heads at a time as a wavefront has lanes for a slab's rows: one head after the other left most of them idle
    // over short caches.  us per tracked call, D = 128, eight heads, 40 caches of 30 rows: vector kernel 11.7, one head at a
    // time 12.8, here 11.9; longer ones, one head at a time / here, 6 of 2092 14.4 / 13.9, 40 of 1104 19.0 / 18.5.
    for (int slab = 0; slab < ring_n; ++slab) {
      const int r = ring_t0 + slab * (NW * kRows) + lane % kRows;
      for (int g = lane / kRows; g < G; g += 64 / kRows)
        if (r < cnt) p.logits[g * p.logit_stride + row0 + r] = ring[(slab * G + g) * kRows + lane % kRows];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the area may be written again
    ring_n = 0;
  };

  for (; t0 < cnt; t0 += NW * kRows) {
    // ---- stage K rows in LDS; the next slab's loads reuse the registers (past the end: the last live row again) ----
#pragma unroll
    for (int i = 0; i < S::kLoads; ++i)
      *reinterpret_cast<uint4*>(myk + (k_row + S::kLoadRows * i) * kKStride + k_piece * 16) = kr[i];
    load_k(t0 + NW * kRows);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // ---- S^T = K Q^T, sums of four elements, added up in pairs as the vector kernel's lanes do -----------------------
    floatx4_t x[S::kTiles];
#pragma unroll
    for (int T = 0; T < S::kTiles; ++T) {
      floatx4_t s[D / 16];
#pragma unroll
      for (int i = 0; i < D / 16; ++i) {
        const floatx4_t a = *reinterpret_cast<const floatx4_t*>(myk + (16 * T + n16) * kKStride + i * 64 + jg * 16);
        floatx4_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const floatx4_t zero = {0.f, 0.f, 0.f, 0.f};
          d[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], qb[i][e], zero, 0, 0, 0);
        }
        s[i] = (d[0] + d[1]) + (d[2] + d[3]);
#pragma unroll
        for (int k = 1; (i + 1) % (2 * k) == 0; k *= 2) s[i + 1 - 2 * k] += s[i + 1 - k];
      }
      x[T] = s[0];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the staging area may be written again

    if (t0 + kRows > cnt) {  // rows past the end: no weight, and nothing that a weight of zero would turn into NaN
#pragma unroll
      for (int T = 0; T < S::kTiles; ++T)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (t0 + 16 * T + 4 * jg + c >= cnt) {
            x[T][c] = kNegInf;
#pragma unroll
            for (int h = 0; h < S::kHalves; ++h) vr[T][c][h] = make_uint4(0, 0, 0, 0);
          }
    }
    if (KEEP) {
      if (ring_n == 0) ring_t0 = t0;
      if (n16 < G) {
#pragma unroll
        for (int T = 0; T < S::kTiles; ++T)
          *reinterpret_cast<floatx4_t*>(ring + (ring_n * G + n16) * kRows + 16 * T + 4 * jg) = x[T];
      }
      if (++ring_n == p.ring_slots) flush_ring();
    }
    // ---- online softmax on the accumulator layout --------------------------------------------------------------------
    float mx = x[0][0];
#pragma unroll
    for (int T = 0; T < S::kTiles; ++T)
#pragma unroll
      for (int c = 0; c < 4; ++c) mx = fmaxf(mx, x[T][c]);
    if (__any(mx > m_run)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mn = fmaxf(m_run, mx);
      const float alpha = fast_exp2(m_run - mn);
      m_run = mn;
      l_part *= alpha;
#pragma unroll
      for (int h = 0; h < S::kHalves; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[h][e] *= alpha;
    }
    // ---- O^T += V^T P^T --------------------------------------------------------------------------------------------
#pragma unroll
    for (int T = 0; T < S::kTiles; ++T) {
      float w[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) w[c] = fast_exp2(x[T][c] - m_run);
      l_part += (w[0] + w[1]) + (w[2] + w[3]);
#pragma unroll
      for (int h = 0; h < S::kHalves; ++h) {
        floatx4_t part[2][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const floatx4_t v = __builtin_bit_cast(floatx4_t, vr[T][c][h]), zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            part[c & 1][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], w[c], c < 2 ? zero : part[c & 1][e], 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) o[h][e] += part[0][e] + part[1][e];
      }
    }
    load_v(t0 + NW * kRows);
  }
  if (KEEP && ring_n > 0) flush_ring();

  // Sum of the four lanes of a head.
  float l_tot = l_part;
  l_tot += __shfl_xor(l_tot, 16);
  l_tot += __shfl_xor(l_tot, 32);

  // Hand the wavefronts' results over through LDS (reusing the staging area).
  __syncthreads();
  float* sm_o = reinterpret_cast<float*>(lds);  // [NW][16][D]
  float* sm_m = sm_o + NW * 16 * D;             // [NW][16]
  float* sm_l = sm_m + NW * 16;                 // [NW][16]
  if (n16 < G) {
#pragma unroll
    for (int h = 0; h < S::kHalves; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        floatx4_t out;
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = o[h][e][i];
        *reinterpret_cast<floatx4_t*>(sm_o + (wave * 16 + n16) * D + 64 * h + 4 * (4 * jg + i)) = out;
      }
    if (jg == 0) {
      sm_m[wave * 16 + n16] = m_run;
      sm_l[wave * 16 + n16] = l_tot;
    }
  }
  __syncthreads();
  finish_item<D, 16, NW>(p, it, G, n, sm_o, sm_m, sm_l);
}

// Dynamic LDS for the logits that wait: what a workgroup alone on its compute unit leaves, or its half of what two leave.
template <int D, int NW> constexpr int ring_bytes() {
  constexpr int stat = std::max(NW * Shape<D>::kRows * Shape<D>::kKStride, (NW * 16 * D + 2 * NW * 16) * 4);
  return NW == 8 ? 160 * 1024 - stat - 512 : (160 * 1024 - 2 * stat - 1024) / 2;
}

template <int D, int NW>
void launch(DecodeParams p, int n_items, int max_count, hipStream_t s) {
  const dim3 grid(n_items), block(64 * NW);
  p.ring_slots = 0;
  if (!p.logits) {
    decode_partial_mfma_f32<D, NW, false><<<grid, block, 0, s>>>(p);
    return;
  }
  const int slot = p.G * Shape<D>::kRows * 4 * NW;  // bytes of a slab of every wavefront
  const int need = (max_count + NW * Shape<D>::kRows - 1) / (NW * Shape<D>::kRows);
  p.ring_slots = std::max(1, std::min(ring_bytes<D, NW>() / slot, need));
  decode_partial_mfma_f32<D, NW, true><<<grid, block, (size_t)p.ring_slots * slot, s>>>(p);
}

template <int D, int NW>
hipError_t prepare() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(decode_partial_mfma_f32<D, NW, true>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, ring_bytes<D, NW>());
}

}  // namespace

// Called when a context over fp32 rows is created on the current device, i.e. outside any stream capture.
hipError_t prepare_decode_mfma_f32() {
  hipError_t e = prepare<128, 8>();
  if (e == hipSuccess) e = prepare<128, 4>();
  if (e == hipSuccess) e = prepare<64, 8>();
  if (e == hipSuccess) e = prepare<64, 4>();
  return e;
}

hipError_t launch_decode_mfma_f32(const DecodeParams& p, int D, int n_items, int max_count, bool one_wave, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  if (p.G > 8 || p.lag || (D != 128 && D != 64)) return hipErrorInvalidValue;
  if (D == 128) one_wave ? launch<128, 8>(p, n_items, max_count, s) : launch<128, 4>(p, n_items, max_count, s);
  else one_wave ? launch<64, 8>(p, n_items, max_count, s) : launch<64, 4>(p, n_items, max_count, s);
  return hipGetLastError();
}

}  // namespace baklava
