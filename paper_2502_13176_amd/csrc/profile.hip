// One-time profiling (Algorithm 1, step 1): for every attention head of a prompt, causal attention
// over the prompt fused with the token-wise cosine between the head's input row v_t and its output
// row softmax(q_t K^T / sqrt(D)) V, and the mean of those cosines.
//
// A dense contraction (2 D T (T + 1) flops per head), so it runs on the matrix cores, as
// v_mfma_f32_32x32x16_bf16:
//
//   S^T[key, token]  = K[key, :] . Q[token, :]          A = K rows from LDS, B = Q (registers)
//   O^T[d, token]   += V^T[d, keys] . P^T[keys, token]   A = V^T (LDS, transposed read), B = P^T
//
// The accumulator of S^T (lane (token, h), register i: key 8 (i / 4) + 4 h + i % 4) is already a valid B
// operand of the second product once the 16 keys of an instruction are numbered the way the lane holds
// them, so the softmax weights never leave their lane; V^T is read from LDS with the same numbering.
//
// A workgroup of 4 wavefronts owns 128 consecutive tokens of one head, 32 per wavefront.  Keys and
// values go from memory to LDS without a stop in registers, in tiles of 64 rows, double-buffered.  The
// tiles wholly below the workgroup's tokens form a software pipeline: the first product of tile n + 1
// runs beside the exponentials of tile n, and those of its second half beside the second product of its
// first half.  The tiles that cross the diagonal follow, masked, one step after the other.  The softmax
// normaliser cancels in the cosine, so the output is never divided.
//
// 32 heads of 8192 tokens take 680 to 734 us box to box (727 to 765 with 16x16x32 instructions, rows staged
// through registers and products and exponentials in turn), two prompts of 700 tokens 21 us (29): the matrix
// pipe is 65% busy at the 1.7 GHz that its power leaves (it was 40% at 2.4 GHz), 1.13 to 1.22 PFLOP/s
// executed.
#include "common.h"

namespace baklava {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));

constexpr int kD = 128;
constexpr int kRow = kD * 2;                       // bytes of a row
constexpr int kChunks = kD / 16;                   // head-dim steps of the first product
constexpr int kWaves = 4;
constexpr int kTokPerWave = 32;
constexpr int kTokPerWg = kWaves * kTokPerWave;    // 128
constexpr int kKeyTile = 64;                       // rows per LDS stage, two slabs of 32
constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kMaxSlack = 8.f;                   // a logit may exceed its token's reference maximum by this much
constexpr float kCosEps = 1e-8f;                   // lower clamp of the product of the two norms

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x8_t as_bf16x8(u32x4_t x) { return __builtin_bit_cast(bf16x8_t, x); }

struct ProfileParams {
  const unsigned char* q;  // [batch, Hq, T, D] bf16
  const unsigned char* k;  // [batch, Hkv, T, D]
  const unsigned char* v;
  float* cos_out;          // [batch, Hq, T] or null
  float* lse_out;          // [batch, Hq, T] or null: log2 of the sum over visible keys of 2^(scaled logit)
  float* tile_sum;         // [batch * Hq, n_tiles] sum of the cosines of each 128-token tile
  int32_t T, Hq, Hkv, n_tiles;
  float scale_log2e;
};

__global__ __launch_bounds__(256, 2) void profile_attn_kernel(ProfileParams p) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_k[2][kKeyTile * kRow];
  __shared__ __attribute__((aligned(16))) unsigned char lds_v[2][kKeyTile * kRow];
  __shared__ float wave_sum[kWaves];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, jh = lane >> 5;
  const int T = p.T;
  // heaviest tiles (the last tokens of the prompt) are launched first; the query heads that share a KV
  // head meet on the same XCDs (consecutive workgroups go round them) and so share its rows in the L2
  const int G = p.Hq / p.Hkv;
  const int n_kv = gridDim.x / (p.n_tiles * G);  // batch * Hkv
  const int64_t kv_head = blockIdx.x % n_kv;
  const int rest = blockIdx.x / n_kv;
  const int tile = p.n_tiles - 1 - rest / G;
  const int bh = (int)kv_head * G + rest % G;    // Hq = Hkv * G: query heads of all prompts in a row
  const unsigned char* Qb = p.q + (int64_t)bh * T * kRow;
  const unsigned char* Kb = p.k + kv_head * T * kRow;
  const unsigned char* Vb = p.v + kv_head * T * kRow;

  const int q0 = tile * kTokPerWg;          // first token of the workgroup
  const int qw0 = q0 + wave * kTokPerWave;  // first token of this wavefront
  const int last_tok = min(q0 + kTokPerWg, T) - 1;
  const int n_key_tiles = last_tok / kKeyTile + 1;
  const int n_full = q0 / kKeyTile;         // tiles without a masked pair (an even number); one or two more follow

  // Staging: a wavefront copies 16 rows of each plane per tile, 4 rows (1 KiB of LDS, in lane order) per
  // instruction.  The 16-byte pieces of a row are permuted on the way: piece c of K row r lies in slot
  // c ^ (r % 16), piece c of V row r in slot c ^ 4 (r % 4), so that the operand reads spread over the
  // banks.  Rows past the prompt (last tile) repeat the last one; their keys are masked.
  // (Written out, with one wait before the barrier that publishes a tile: the only result is in LDS.)
  const int st_row = wave * 16 + lane / 16, st_slot = lane % 16;
  const uint32_t k_off = st_row * kRow + (st_slot ^ (lane / 16)) * 16;          // row 4 i further: ^ 64 i
  const uint32_t v_off = st_row * kRow + (st_slot ^ (4 * (lane / 16))) * 16;
  const uint32_t lds_k0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_k + wave * 16 * kRow;
  const uint32_t lds_v0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_v + wave * 16 * kRow;
  auto copy_rows = [&](uint32_t dst, const unsigned char* plane, int kt, uint32_t off, uint32_t step) {
    const unsigned char* src = plane + (int64_t)kt * (kKeyTile * kRow);
    const int most = T - 1 - kt * kKeyTile;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t o = (off ^ (step * i)) + i * 4 * kRow;
      if (most < kKeyTile - 1) o = min(st_row + 4 * i, most) * kRow + o % kRow;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(dst + i * 4 * kRow), "v"(o), "s"(src) : "memory", "m0");
    }
  };
  auto stage_k = [&](int kt) { copy_rows(lds_k0 + (kt & 1) * (kKeyTile * kRow), Kb, kt, k_off, 64); };
  auto stage_v = [&](int kt) { copy_rows(lds_v0 + (kt & 1) * (kKeyTile * kRow), Vb, kt, v_off, 0); };
  auto publish = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };

  stage_k(0);
  stage_v(0);
  if (n_key_tiles > 1) stage_k(1);

  // B operand of the first product: lane (token, h), chunk c holds Q[token][16c + 8h .. +8).
  const int tok = qw0 + n32;
  const int tok_row = min(tok, T - 1);  // tokens past the prompt repeat the last one and are never written
  bf16x8_t qb[kChunks];
#pragma unroll
  for (int c = 0; c < kChunks; ++c)
    qb[c] = as_bf16x8(*reinterpret_cast<const u32x4_t*>(Qb + (int64_t)tok_row * kRow + c * 32 + jh * 16));

  floatx16_t o[4];  // lane (token, h), register i of block b: O[token][32 b + 8 (i / 4) + 4 h + i % 4]
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
  float m_ref = kNegInf;  // reference maximum of the exponent, log2 units
  float l_part = 0.f;     // this lane's share of the running sum
  const float cs = p.scale_log2e;

  // First product for a tile: lane (key, h) of the A operand reads piece 2 c + h of its row.
  auto logits = [&](floatx16_t (&s)[2], int kt) {
    const unsigned char* base = lds_k[kt & 1] + n32 * kRow;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int slot = ((2 * c + jh) ^ (n32 & 15)) * 16;
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) {
        const u32x4_t a = *reinterpret_cast<const u32x4_t*>(base + sl * 32 * kRow + slot);
        const floatx16_t zero = {};
        s[sl] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), qb[c], c == 0 ? zero : s[sl], 0, 0, 0);
      }
    }
  };
  auto max_of = [&](const floatx16_t (&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int sl = 0; sl < 2; ++sl)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[sl][i]);
    return mx * cs;
  };
  // Lazy running maximum: the reference m_ref of a token only moves when a logit exceeds it by more
  // than kMaxSlack (log2 units), so weights stay below 2^kMaxSlack and the rescale of the accumulators
  // is rare after the first tile.  (First tile: m_ref = -inf, always taken; key 0 is visible to every
  // token, so the new reference is finite.)
  auto follow_max = [&](float mx) {
    if (__any(mx > m_ref + kMaxSlack)) {
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mn = fmaxf(m_ref, mx);
      const float alpha = fast_exp2(m_ref - mn);
      m_ref = mn;
      l_part *= alpha;
#pragma unroll
      for (int b = 0; b < 4; ++b) o[b] *= alpha;
    }
  };
  // Weights of a slab of 32 keys as B operands, 16 keys each.  Each weight is split into a truncated bf16
  // high part and a bf16 residual, so the second product keeps ~16 bits of it (one bf16 term alone costs
  // about 1e-3 on a token's cosine).
  auto weights = [&](const floatx16_t& s, u32x4_t (&ph)[2], bf16x8_t (&pl)[2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const float p0 = fast_exp2(fmaf(s[8 * u + e], cs, -m_ref));
        const float p1 = fast_exp2(fmaf(s[8 * u + e + 1], cs, -m_ref));
        l_part += p0 + p1;
        const uint32_t u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
        ph[u][e / 2] = (u0 >> 16) | (u1 & 0xffff0000u);
        pl[u][e] = (__bf16)(p0 - __uint_as_float(u0 & 0xffff0000u));
        pl[u][e + 1] = (__bf16)(p1 - __uint_as_float(u1 & 0xffff0000u));
      }
  };
  // Second product for a slab.  A transposed read hands lane m of a 16-lane group element m of the 16
  // d values the group points at, for 4 consecutive keys: the group (h, d half) reads keys 4 h .. + 3 of
  // each 8, two reads per 16 keys.
  auto outputs = [&](int kt, int sl, const u32x4_t (&ph)[2], const bf16x8_t (&pl)[2]) {
    const int n16 = lane & 15, half = (lane >> 4) & 1, k4 = n16 >> 2;
    const unsigned char* row = lds_v[kt & 1] + (sl * 32 + 4 * jh + k4) * kRow + half * 32 + (n16 & 3) * 8;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        typedef __attribute__((address_space(3))) s16x4_t* lds_ptr_t;
        const unsigned char* at = row + u * 16 * kRow + (b ^ k4) * 64;
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)at);
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(at + 8 * kRow));
        const bf16x8_t a = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, as_bf16x8(ph[u]), o[b], 0, 0, 0);
        o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pl[u], o[b], 0, 0, 0);
      }
  };

  publish();
  floatx16_t s[2];
  logits(s, 0);
  float mx = max_of(s);
  __syncthreads();  // tile 0's K rows are overwritten by tile 2's in the first step
  u32x4_t ph[2][2];
  bf16x8_t pl[2][2];
  // One pipeline step: tile kt from its logits in `s`, the next tile's logits into `sn`.
  auto step = [&](const floatx16_t (&s)[2], floatx16_t (&sn)[2], int kt) {
    if (kt + 2 < n_key_tiles) stage_k(kt + 2);
    stage_v(kt + 1);
    follow_max(mx);
    logits(sn, kt + 1);
    weights(s[0], ph[0], pl[0]);
    outputs(kt, 0, ph[0], pl[0]);
    weights(s[1], ph[1], pl[1]);
    outputs(kt, 1, ph[1], pl[1]);
    mx = max_of(sn);
    publish();
  };
  int kt = 0;
  for (; kt < n_full; kt += 2) {  // an even number of tiles, and at least one follows
    floatx16_t sn[2];
    step(s, sn, kt);
    step(sn, s, kt + 1);
  }
  for (; kt < n_key_tiles; ++kt) {
    const int kt0 = kt * kKeyTile;
    if (kt + 1 < n_key_tiles) stage_v(kt + 1);
    if (kt0 <= qw0 + kTokPerWave - 1) {  // else wholly above this wavefront's tokens
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kt0 + sl * 32 + 8 * (i / 4) + 4 * jh + i % 4 > tok) s[sl][i] = kNegInf;
      follow_max(max_of(s));
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) {
        weights(s[sl], ph[sl], pl[sl]);
        outputs(kt, sl, ph[sl], pl[sl]);
      }
      if (kt + 1 < n_key_tiles) logits(s, kt + 1);
    }
    publish();
  }

  // ---- cosine between v_t and the (un-normalised) output row, per token --------------------------
  float dot = 0.f, no = 0.f, nv = 0.f;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u32x2_t raw = *reinterpret_cast<const u32x2_t*>(Vb + (int64_t)tok_row * kRow + (b * 32 + q * 8 + jh * 4) * 2);
      const float v0 = __uint_as_float(raw.x << 16), v1 = __uint_as_float(raw.x & 0xffff0000u);
      const float v2 = __uint_as_float(raw.y << 16), v3 = __uint_as_float(raw.y & 0xffff0000u);
      const float o0 = o[b][4 * q], o1 = o[b][4 * q + 1], o2 = o[b][4 * q + 2], o3 = o[b][4 * q + 3];
      dot += o0 * v0 + o1 * v1 + o2 * v2 + o3 * v3;
      no += o0 * o0 + o1 * o1 + o2 * o2 + o3 * o3;
      nv += v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3;
    }
  dot += __shfl_xor(dot, 32);
  no += __shfl_xor(no, 32);
  nv += __shfl_xor(nv, 32);
  const float l_tot = l_part + __shfl_xor(l_part, 32);
  const float inv_l = 1.f / l_tot;
  const float cosv = (dot * inv_l) / fmaxf(sqrtf(no) * inv_l * sqrtf(nv), kCosEps);
  float wsum = 0.f;
  if (tok < T && jh == 0) {
    if (p.cos_out) p.cos_out[(int64_t)bh * T + tok] = cosv;
    if (p.lse_out) p.lse_out[(int64_t)bh * T + tok] = m_ref + __builtin_log2f(l_tot);
    wsum = cosv;
  }
  // sum over the wavefront's tokens (lanes with h = 0 hold them), then over the workgroup, in a fixed order
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) wsum += __shfl_xor(wsum, off);
  if (lane == 0) wave_sum[wave] = wsum;
  __syncthreads();
  if (tid == 0)
    p.tile_sum[(int64_t)bh * p.n_tiles + tile] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
}

// Mean over the prompt: one wavefront per head adds the tile sums in a fixed order.
__global__ __launch_bounds__(64) void profile_mean_kernel(const float* tile_sum, float* sim_out, int n_tiles, int T) {
  const int bh = blockIdx.x;
  float acc = 0.f;
  for (int i = threadIdx.x; i < n_tiles; i += 64) acc += tile_sum[(int64_t)bh * n_tiles + i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (threadIdx.x == 0) sim_out[bh] = acc / (float)T;
}

}  // namespace

hipError_t launch_profile_similarity(const void* q, const void* k, const void* v, int batch, int Hq, int Hkv,
                                     int T, float* cos_out, float* sim_out, float* lse_out, float* tile_sum,
                                     hipStream_t s) {
  ProfileParams p;
  p.q = reinterpret_cast<const unsigned char*>(q);
  p.k = reinterpret_cast<const unsigned char*>(k);
  p.v = reinterpret_cast<const unsigned char*>(v);
  p.cos_out = cos_out;
  p.lse_out = lse_out;
  p.tile_sum = tile_sum;
  p.T = T; p.Hq = Hq; p.Hkv = Hkv;
  p.n_tiles = (T + kTokPerWg - 1) / kTokPerWg;
  p.scale_log2e = 1.4426950408889634f / sqrtf((float)kD);
  const int64_t n_wg = (int64_t)batch * Hq * p.n_tiles;
  if (n_wg <= 0 || n_wg > INT32_MAX) return hipErrorInvalidValue;
  profile_attn_kernel<<<dim3((unsigned)n_wg), dim3(256), 0, s>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  profile_mean_kernel<<<dim3(batch * Hq), dim3(64), 0, s>>>(tile_sum, sim_out, p.n_tiles, T);
  return hipGetLastError();
}

}  // namespace baklava
