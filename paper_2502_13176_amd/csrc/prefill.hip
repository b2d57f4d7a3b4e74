// Attention scores of a whole prompt at once: score_j = sum over the G query heads of a KV head and
// over the prompt tokens t >= j of softmax_j(q_t . k_j / sqrt(D)), i.e. the column sums of the
// causal attention matrices, the accumulated-attention statistic the eviction ranks by, as it
// stands after a prefill of T tokens (before the first decode step and its eviction, Eqs. 5-6).
//
// The row normalisers come from the attention pass that produced the prompt's outputs (its
// log-sum-exp per token, here in log2 units), so this pass needs the first product only:
//
//   S^T[key, token] = K[key, :] . Q[token, :]     A = K rows (registers, fixed per wavefront),
//                                                 B = Q rows (streamed through LDS)
//   score[key]     += 2^(S^T[key, token] * log2(e)/sqrt(D) - lse2[token])   for key <= token
//
// A workgroup of 4 wavefronts owns 128 or 256 consecutive keys of one KV head, 32 or 64 per wavefront,
// and walks over the G query heads and, for each, over the tokens from its first key to the end of the
// prompt in stages of 64, double-buffered in LDS.  Column sums stay in registers (one partial per
// lane and key) and are reduced over the 32 token lanes once, at the end: no atomics, results are
// deterministic.  A key block streams the tokens from its first key on, so a workgroup takes blocks i
// and n_blocks - 1 - i: equal work for every workgroup of a sequence.
#include "common.h"

namespace baklava {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kD = 128;
constexpr int kChunks = kD / 16;                   // 16 head-dim elements per matrix instruction
constexpr int kWaves = 4;
constexpr int kTokTile = 64;                       // tokens per LDS stage
constexpr int kQStride = 272;                      // bytes between staged Q rows (conflict-free operand reads)
constexpr float kNegInf = -__builtin_huge_valf();

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x8_t as_bf16x8(u32x4_t x) { return __builtin_bit_cast(bf16x8_t, x); }

struct PrefillParams {
  const unsigned char* q;    // [batch, Hq, T, D] bf16
  const unsigned char* k;    // K plane; sequence (b, h) starts at row k_off[b * Hkv + h], or is dense
  const float* lse;          // [batch, Hq, T] log2-sum-exp of the scaled logits, log2 units
  const int64_t* row_off;    // [batch * Hkv] or null
  float* score;              // same row addressing as k
  int32_t T, Hq, Hkv, n_blocks;
  float scale_log2e;
};

// TILES: 32-key tiles per wavefront; PIPE: products of one tile beside the weights of the one before.  Bound
// by vector issue: per 32 x 32 tile 16 exponentials of 16 cycles, 16 multiply-adds and 16 additions of 4 and 8
// matrix instructions of 32, about 420 cycles if the matrix pipe runs beside the vector ALUs (the device runs this at about 1.9 GHz); what a stage costs
// beside that (rows to LDS and back, barrier) is shared by twice as many products with two tiles.  16 x
// 16 products one after the other with their weights took 5530 us for 32 heads of 32768 tokens and 160
// for 2048 tokens; this takes 4100-4340 (two tiles) and 122 (one).  Without PIPE a wavefront takes 125
// registers, so four workgroups share a compute unit and cover one another's waits: for launches of many
// workgroups with a few stages each, where filling a pipeline costs more than it gives.
template <int TILES, bool PIPE>
__global__ __launch_bounds__(256, PIPE ? 2 : 4) void prefill_score_kernel(PrefillParams p) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_q[2][kTokTile * kQStride];
  __shared__ float lds_lse[2][kTokTile];
  constexpr int kKeysPerWave = 32 * TILES, kKeysPerWg = kWaves * kKeysPerWave;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = p.T;
  const int n_pairs = (p.n_blocks + 1) / 2;
  const int n_seq = gridDim.x / n_pairs;      // batch * Hkv
  const int seq = blockIdx.x % n_seq;         // (b, kv head)
  const int pair = blockIdx.x / n_seq;
  const int G = p.Hq / p.Hkv;
  const int b = seq / p.Hkv, hk = seq % p.Hkv;
  const int64_t row0 = p.row_off ? p.row_off[seq] : (int64_t)seq * T;
  const unsigned char* Kb = p.k + row0 * (kD * 2);
  const int64_t head0 = (int64_t)b * p.Hq + (int64_t)hk * G;
  const float cs = p.scale_log2e;

#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
  int lane = tid & 63, piece = tid, last_t0 = (T - 1) / kTokTile * kTokTile;
  // four wavefronts per SIMD: a half forms anew what it derives from these, kept it would cost spilled registers
  if constexpr (!PIPE) asm volatile("" : "+v"(lane), "+v"(piece), "+s"(last_t0));
  const int n32 = lane & 31, jh = lane >> 5;
  const int block = half == 0 ? pair : p.n_blocks - 1 - pair;
  if (half == 1 && block == pair) break;      // odd number of blocks: the middle one is alone
  const int j0 = block * kKeysPerWg;          // first key of the block
  const int jw0 = j0 + wave * kKeysPerWave;   // first key of this wavefront

  // A operand: lane (key % 32, j), tile tt, chunk c holds K[key][16c + 8j .. +8); loaded once.
  bf16x8_t ka[TILES][kChunks];
#pragma unroll
  for (int tt = 0; tt < TILES; ++tt) {
    const int row = min(jw0 + tt * 32 + n32, T - 1);  // keys past the prompt repeat the last one, never written
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
      ka[tt][c] = as_bf16x8(*reinterpret_cast<const u32x4_t*>(Kb + (int64_t)row * (kD * 2) + c * 32 + jh * 16));
  }

  // Lane (token, j) of a product holds keys 8 (i / 4) + 4 j + i % 4 of the tile in its register i; so do
  // the column-sum partials, over this lane's tokens.
  float acc[TILES][16];
#pragma unroll
  for (int tt = 0; tt < TILES; ++tt)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[tt][i] = 0.f;

  // Stages: the token tiles from the prompt's last one down to the one holding key j0, and for each of
  // them the query heads of the group.  Every workgroup of a sequence starts at the same tile, so those
  // that run side by side find its Q rows in the L2 (5700 -> 5340 us for 32768 tokens with one tile).
  const int first_tile = j0 / kTokTile;
  const int n_tiles = (T + kTokTile - 1) / kTokTile - first_tile;
  const int n_stages = G * n_tiles;

  // Rows past the prompt (in the last tile only, the first to be staged) repeat the last one; such a
  // token has an infinite normaliser, so its weights are zero.  With PIPE addresses are a uniform base plus
  // an offset that only changes after that tile.
  u32x4_t qreg[4];
  float lreg = 0.f;
  uint32_t q_off[4], l_off = min(lane, T - 1 - last_t0) * 4u;
#pragma unroll
  for (int i = 0; i < 4; ++i) q_off[i] = min(piece / 16 + i * 16, T - 1 - last_t0) * (kD * 2u) + (piece % 16) * 16u;
  int ld_g = 0, ld_t0 = last_t0;  // head and first token of the next stage to load
  auto load_stage = [&]() {
    if constexpr (!PIPE) {  // offsets formed for every stage: kept, they would take registers
      const int most = T - 1 - ld_t0;
      const unsigned char* Qt = p.q + ((head0 + ld_g) * T + ld_t0) * (kD * 2);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        qreg[i] = *reinterpret_cast<const u32x4_t*>(Qt + (uint32_t)(min(piece / 16 + i * 16, most) * (kD * 2) + piece % 16 * 16));
      if (wave == 0) {
        lreg = p.lse[(head0 + ld_g) * T + ld_t0 + min(lane, most)];
        if (lane > most) lreg = -kNegInf;
      }
      if (++ld_g == G) { ld_g = 0; ld_t0 -= kTokTile; }
      return;
    }
    const unsigned char* Qt = p.q + ((head0 + ld_g) * T + ld_t0) * (kD * 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) qreg[i] = *reinterpret_cast<const u32x4_t*>(Qt + q_off[i]);
    if (wave == 0)
      lreg = *reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(p.lse + (head0 + ld_g) * T + ld_t0) + l_off);
    if (wave == 0 && ld_t0 == last_t0) lreg = last_t0 + lane < T ? lreg : -kNegInf;
    if (++ld_g == G) {
      if (ld_t0 == last_t0) {
        l_off = lane * 4u;
#pragma unroll
        for (int i = 0; i < 4; ++i) q_off[i] = (piece / 16 + i * 16) * (kD * 2u) + (piece % 16) * 16u;
      }
      ld_g = 0;
      ld_t0 -= kTokTile;
    }
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<u32x4_t*>(&lds_q[buf][(piece / 16 + i * 16) * kQStride + (piece % 16) * 16]) = qreg[i];
    if (wave == 0) lds_lse[buf][lane] = lreg;
  };

  // A stage holds two column tiles of 32 tokens.  The products of one run on the matrix pipe while the
  // vector ALUs turn the other's logits into weights; the second tile's are turned in the next stage.
  floatx16_t s0[TILES], s1[TILES];
  float nl0 = 0.f, nl1 = 0.f;
  // none yet: logits of -inf, weights of zero
#pragma unroll
  for (int tt = 0; tt < TILES; ++tt)
#pragma unroll
    for (int i = 0; i < 16; ++i) s1[tt][i] = kNegInf;
  // B operands of a column tile: lane (token, j), chunk c holds Q[token][16c + 8j .. +8).
  auto read_tile = [&](bf16x8_t (&qt)[kChunks], float& nl, int buf, int nt) {
    const unsigned char* qrow = &lds_q[buf][(nt * 32 + n32) * kQStride + jh * 16];
    nl = -lds_lse[buf][nt * 32 + n32];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) qt[c] = as_bf16x8(*reinterpret_cast<const u32x4_t*>(qrow + c * 32));
  };
  auto products = [&](floatx16_t (&s)[TILES], const bf16x8_t (&qt)[kChunks]) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
#pragma unroll
      for (int tt = 0; tt < TILES; ++tt) {
        const floatx16_t zero = {};
        s[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[tt][c], qt[c], c == 0 ? zero : s[tt], 0, 0, 0);
      }
  };
  auto add_weights = [&](const floatx16_t (&s)[TILES], float nl) {
#pragma unroll
    for (int tt = 0; tt < TILES; ++tt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[tt][i] += fast_exp2(fmaf(s[tt][i], cs, nl));
  };
  auto mask_tile = [&](floatx16_t (&s)[TILES], int tok0) {
#pragma unroll
    for (int tt = 0; tt < TILES; ++tt)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (jw0 + tt * 32 + 8 * (i / 4) + 4 * jh + i % 4 > tok0 + n32) s[tt][i] = kNegInf;
  };
  // Ends a tile's share of a stage: the weights are summed here, not moved behind the barrier, so that they
  // can be issued while the matrix pipe works.
  auto settle = [&]() {
#pragma unroll
    for (int tt = 0; tt < TILES; ++tt)
      asm volatile("" : "+v"(acc[tt][0]), "+v"(acc[tt][1]), "+v"(acc[tt][2]), "+v"(acc[tt][3]), "+v"(acc[tt][4]),
                        "+v"(acc[tt][5]), "+v"(acc[tt][6]), "+v"(acc[tt][7]), "+v"(acc[tt][8]), "+v"(acc[tt][9]),
                        "+v"(acc[tt][10]), "+v"(acc[tt][11]), "+v"(acc[tt][12]), "+v"(acc[tt][13]),
                        "+v"(acc[tt][14]), "+v"(acc[tt][15]));
  };

  load_stage();
  store_stage(0);
  __syncthreads();
  if (n_stages > 1) load_stage();

  // Tiles that start behind the workgroup's keys have no masked pair; the last ones (a tile per 64 keys
  // of the workgroup) cross the diagonal.
  const int n_below = PIPE ? max(0, (T + kTokTile - 1) / kTokTile - (j0 + kKeysPerWg) / kTokTile) * G : 0;
  int st = 0;
  bf16x8_t qa[kChunks];
  float nla;
  if constexpr (TILES == 1 && PIPE) {
    // The barrier of a stage sits between its two tiles: the rows of the next stage are in LDS before the
    // second tile's products start, so every operand is read one tile ahead of its use.
    bf16x8_t qb[kChunks];
    float nlb;
    if (n_below > 0) read_tile(qa, nla, 0, 0);
    for (; st < n_below; ++st) {  // at least one stage follows
      const int buf = st & 1;
      read_tile(qb, nlb, buf, 1);
      products(s0, qa);
      add_weights(s1, nl1);
      nl0 = nla;
      settle();
      store_stage(buf ^ 1);  // its tiles were read before the previous stage's barrier
      __syncthreads();
      if (st + 2 < n_stages) load_stage();
      read_tile(qa, nla, buf ^ 1, 0);
      products(s1, qb);
      add_weights(s0, nl0);
      nl1 = nlb;
      settle();
    }
  } else if constexpr (PIPE) {
    // no registers left for operands one tile ahead: the other wavefront of the SIMD covers the reads
    for (; st < n_below; ++st) {
      const int buf = st & 1;
      read_tile(qa, nl0, buf, 0);
      products(s0, qa);
      add_weights(s1, nl1);
      settle();
      read_tile(qa, nl1, buf, 1);
      products(s1, qa);
      add_weights(s0, nl0);
      settle();
      store_stage(buf ^ 1);
      __syncthreads();
      if (st + 2 < n_stages) load_stage();
    }
  }
  int t0 = last_t0 - n_below / G * kTokTile, g = 0;
  if constexpr (PIPE && TILES == 1) {
    int tok1 = T;  // first token of the tile in s1
    for (; st < n_stages; ++st) {
      const int buf = st & 1;
      if (t0 + kTokTile - 1 >= jw0) {  // else every token precedes every key of this wavefront
        mask_tile(s1, tok1);
        add_weights(s1, nl1);
        read_tile(qa, nl0, buf, 0);
        products(s0, qa);
        read_tile(qa, nl1, buf, 1);
        products(s1, qa);
        mask_tile(s0, t0);
        add_weights(s0, nl0);
        tok1 = t0 + 32;
      }
      if (st + 1 < n_stages) store_stage(buf ^ 1);
      __syncthreads();
      if (st + 2 < n_stages) load_stage();
      if (++g == G) { g = 0; t0 -= kTokTile; }
    }
    mask_tile(s1, tok1);
    add_weights(s1, nl1);
  } else {
    if (PIPE) add_weights(s1, nl1);
    for (; st < n_stages; ++st) {
      const int buf = st & 1;
#pragma unroll 1
      for (int nt = 0; nt < 2; ++nt) {
        const int tok0 = t0 + nt * 32;
        if (tok0 >= T || tok0 + 31 < jw0) continue;  // past the prompt, or before every key of this wavefront
        const unsigned char* qrow = &lds_q[buf][(nt * 32 + n32) * kQStride + jh * 16];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
          const bf16x8_t q1 = as_bf16x8(*reinterpret_cast<const u32x4_t*>(qrow + c * 32));
#pragma unroll
          for (int tt = 0; tt < TILES; ++tt) {
            const floatx16_t zero = {};
            s0[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[tt][c], q1, c == 0 ? zero : s0[tt], 0, 0, 0);
          }
        }
        nl0 = -lds_lse[buf][nt * 32 + n32];
        if (tok0 < jw0 + kKeysPerWave - 1) {
          asm volatile("" ::: "memory");  // keeps this a branch: below the diagonal nothing is masked
          mask_tile(s0, tok0);
        }
        add_weights(s0, nl0);
      }
      if (st + 1 < n_stages) store_stage(buf ^ 1);
      __syncthreads();
      if (st + 2 < n_stages) load_stage();
      if (++g == G) { g = 0; t0 -= kTokTile; }
    }
  }

  // Sum over the 32 token lanes of each half: at every step a lane keeps one half of its keys and adds the
  // partner's share of them, so lane n32 ends with key register n32 / 2, and the even lanes write.
#pragma unroll
  for (int tt = 0; tt < TILES; ++tt) {
#pragma unroll
    for (int off = 16; off > 1; off >>= 1) {
      const bool upper = n32 & off;
#pragma unroll
      for (int i = 0; i < off / 2; ++i) {
        const float lo = acc[tt][i], hi = acc[tt][i + off / 2];
        acc[tt][i] = (upper ? hi : lo) + __shfl_xor(upper ? lo : hi, off);
      }
    }
    const float sum = acc[tt][0] + __shfl_xor(acc[tt][0], 1);
    const int i = n32 >> 1, key = jw0 + tt * 32 + 8 * (i / 4) + 4 * jh + i % 4;
    if (!(n32 & 1) && key < T) p.score[row0 + key] = sum;
  }
  }
}

template <int TILES, bool PIPE>
hipError_t launch_tiles(PrefillParams p, int64_t n_seq, hipStream_t s) {
  p.n_blocks = (p.T + kWaves * 32 * TILES - 1) / (kWaves * 32 * TILES);
  const int64_t n_wg = n_seq * ((p.n_blocks + 1) / 2);
  if (n_wg <= 0 || n_wg > INT32_MAX) return hipErrorInvalidValue;
  prefill_score_kernel<TILES, PIPE><<<dim3((unsigned)n_wg), dim3(256), 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_scores(const void* q, const void* k, const float* lse, const int64_t* row_off,
                                 int batch, int Hq, int Hkv, int T, float* score, hipStream_t s) {
  PrefillParams p;
  p.q = reinterpret_cast<const unsigned char*>(q);
  p.k = reinterpret_cast<const unsigned char*>(k);
  p.lse = lse;
  p.row_off = row_off;
  p.score = score;
  p.T = T; p.Hq = Hq; p.Hkv = Hkv;
  p.n_blocks = 0;
  p.scale_log2e = 1.4426950408889634f / sqrtf((float)kD);
  // One tile per wavefront, pipelined, while that gives at most two workgroups to each of the 256 compute units.
  // Beyond, two tiles once they fill the chip twice over, if the prompt is long against a workgroup's masked
  // stages (twice as many with two tiles) or the launch is large enough for fewer stages to outweigh them;
  // otherwise the form without pipeline.  us with one tile / two tiles / without pipeline (and with 16 x 16
  // products, one form for all), sequences x tokens x query heads of each:
  //   8 x 8192 x 4       468 /  663 /  716 ( 596)    256 x 1999 x 1    187 /  163 /  176 ( 183)
  //   32 x 8192 x 4     1260 / 1071 / 1289 (1275)    512 x 1300 x 1    199 /  170 /  161 ( 174)
  //   64 x 3000 x 4      399 /  376 /  369 ( 367)    256 x 900 x 4     171 /  163 /  156 ( 166)
  //   128 x 1999 x 4     342 /  311 /  336 ( 347)    1024 x 100 x 4    32 /   45 /   25 (  29)
  //   256 x 1100 x 8     555 /  460 /  497 ( 477)    1024 x 64 x 1     9.6 / 13.0 / 7.2 ( 7.2)
  const int64_t n_seq = (int64_t)batch * Hkv;
  const int64_t narrow = n_seq * ((((int64_t)T + 127) / 128 + 1) / 2);  // workgroups with one tile
  const int64_t wide = n_seq * ((((int64_t)T + 255) / 256 + 1) / 2);    // with two
  const int64_t tokens = (int64_t)(Hq / Hkv) * T;                       // rows of Q that a sequence streams
  if (narrow <= 512) return launch_tiles<1, true>(p, n_seq, s);
  if (wide >= 512 && (T >= 1500 || (double)tokens * wide >= 2.8e6)) return launch_tiles<2, true>(p, n_seq, s);
  return launch_tiles<1, false>(p, n_seq, s);
}

}  // namespace baklava
