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

#include <type_traits>

namespace baklava {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kD = 128;
constexpr int kRow = kD * 2;                       // bytes of a row
constexpr int kChunks = kD / 16;                   // 16 head-dim elements per matrix instruction
constexpr int kWaves = 4;
constexpr int kTokTile = 64;                       // tokens per LDS stage
constexpr float kNegInf = -__builtin_huge_valf();

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x8_t as_bf16x8(u32x4_t x) { return __builtin_bit_cast(bf16x8_t, x); }

// Memory to LDS without a stop in registers: 64 lanes x 16 bytes (or 4) from `base` + the lane's offset to `lds`, in
// lane order.  An instruction's own offset counts for both sides.
__device__ __forceinline__ void copy_rows(uint32_t lds, const void* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void copy_rows_4(uint32_t lds, const void* base, uint32_t o0, uint32_t o1, uint32_t o2, uint32_t o3) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %1\n\tglobal_load_lds_dwordx4 %3, %1 offset:1024\n\t"
               "global_load_lds_dwordx4 %4, %1 offset:2048\n\tglobal_load_lds_dwordx4 %5, %1 offset:3072"
               :: "s"(lds), "s"(base), "v"(o0), "v"(o1), "v"(o2), "v"(o3) : "memory", "m0");
}
__device__ __forceinline__ void copy_words(uint32_t lds, const void* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}

struct PrefillParams {
  const unsigned char* q;    // [batch, Hq, T, D] bf16
  const unsigned char* k;    // K plane; sequence (b, h) starts at row k_off[b * Hkv + h], or is dense
  const float* lse;          // [batch, Hq, T] log2-sum-exp of the scaled logits, log2 units
  const int64_t* row_off;    // [batch * Hkv] or null
  float* score;              // same row addressing as k
  int32_t T, Hq, Hkv, n_blocks;
  float scale_log2e;
};

// TILES: 32-key tiles per wavefront; PIPE: products of one tile beside the weights of the one before.  Bound by power
// and vector issue: a probe of one 32 x 32 tile (8 matrix instructions of 32 cycles, 16 exponentials of 8, 16
// multiply-adds and 16 additions of 4.4) takes 109 ns for the products alone, 107 for the rest, 143 for both, and on
// random data the products alone run at 195 (1.37 PFLOP/s, what a large library product reaches; zeros run faster),
// the whole kernel at 235.  What a stage costs beside that (rows to LDS and back, barrier) is shared by twice as many
// products with two tiles.  Rows through registers, one stage ahead and with a wait for the normalisers in every
// stage, took 4210 us for 32 heads of 32768 tokens, 468 for 8192 and 105 for 2048; this takes 3820, 316 and 84.
// Without PIPE a wavefront takes 113 registers, so four workgroups share a compute unit and cover one another's
// waits: for launches of many workgroups with a few stages each, where filling a pipeline costs more than it gives.
template <int TILES, bool PIPE>
__global__ __launch_bounds__(64 * kWaves, PIPE ? 2 : 4) void prefill_score_kernel(PrefillParams p) {
  constexpr int kBufs = PIPE ? 4 : 2;         // stages in LDS (without pipeline four workgroups share a compute unit)
  constexpr int kRowsPerWave = kTokTile / kWaves, kCopies = kRowsPerWave / 4;  // rows and copies of a wavefront per stage
  __shared__ __attribute__((aligned(16))) unsigned char lds_q[kBufs][kTokTile * kRow];
  __shared__ __attribute__((aligned(16))) float lds_lse[kBufs][kTokTile];
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
  const unsigned char* Kb = p.k + row0 * kRow;
  const int64_t head0 = (int64_t)b * p.Hq + (int64_t)hk * G;
  const float cs = p.scale_log2e;
  const int last_t0 = (T - 1) / kTokTile * kTokTile;  // first token of the prompt's last tile

#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
  int lane = tid & 63;
  // four wavefronts per SIMD: a half forms anew what it derives from this, kept it would cost spilled registers
  if constexpr (!PIPE) asm volatile("" : "+v"(lane));
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
      ka[tt][c] = as_bf16x8(*reinterpret_cast<const u32x4_t*>(Kb + (int64_t)row * kRow + c * 32 + jh * 16));
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

  // Staging: rows of Q and their normalisers go from memory to LDS without a stop in registers, 4 rows (1 KiB of
  // LDS, in lane order) per instruction, kBufs stages ahead: one stage ahead and through registers, every
  // workgroup of a launch with one wavefront per SIMD waited for memory in every stage.  The 16-byte pieces of a
  // row are permuted on the way (piece c of row r lies in slot c ^ (r % 16)), so that the operand reads spread
  // over the banks.  Rows past the prompt (in the last tile, the first to be staged) repeat the last one; such a
  // token's normaliser is taken as infinite where it is read.
  // (Written out: the only result is in LDS.  A wavefront waits for its own copies of a stage before the barrier
  // that publishes it; loads of the compiler's own in flight only make such a wait longer.)
  const int st_row = wave * kRowsPerWave + lane / 16;
  const uint32_t st_slot = ((lane % 16) ^ (st_row & 15)) * 16;  // 4 i rows further: ^ 64 i
  const uint32_t lds_q0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)&lds_q[0][wave * kRowsPerWave * kRow];
  const uint32_t lds_l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)&lds_lse[0][0];
  int ld_g = 0, ld_st = 0;                           // head and number of the next stage to copy
  const int left0 = T - last_t0;                     // tokens of the prompt's last tile
  uint32_t q_off = min(st_row, left0 - 1) * kRow + st_slot, l_off = min(lane, left0 - 1) * 4u;
  const unsigned char* ld_q = p.q + (head0 * T + last_t0) * kRow;
  const float* ld_l = p.lse + head0 * T + last_t0;
  auto copy_stage = [&](int buf) {  // buf = ld_st % kBufs
    const uint32_t dst = lds_q0 + buf * (kTokTile * kRow);
    if (ld_st >= G || left0 == kTokTile) {
      copy_rows_4(dst, ld_q, q_off, q_off ^ 64, q_off ^ 128, q_off ^ 192);
    } else {  // rows of the last tile: none beyond the prompt's last one
#pragma unroll
      for (int i = 0; i < kCopies; ++i)
        copy_rows(dst + i * 4 * kRow, ld_q, min(st_row + 4 * i, left0 - 1) * kRow + (st_slot ^ (64 * i)));
    }
    static_assert(kCopies == 4, "copies written out");
    // every wavefront brings all normalisers: the same values to the same places
    copy_words(lds_l0 + buf * (kTokTile * 4), ld_l, l_off);
    ++ld_st;
    int64_t step = T;
    if (++ld_g == G) {
      ld_g = 0;
      step -= (int64_t)G * T + kTokTile;
      q_off = st_row * kRow + st_slot;
      l_off = lane * 4u;
    }
    ld_q += step * kRow;
    ld_l += step;
  };
  // Ends a stage (in buffer buf): the next one is published, and the buffer, whose rows every wavefront has read,
  // takes the one kBufs further.  At most kBufs - 2 younger stages may be on their way meanwhile.
  auto next_stage = [&](int buf) {  // with kBufs or more stages left after this one
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kBufs - 2) * (kCopies + 1)) : "memory");
    __syncthreads();
    copy_stage(buf);
  };
  auto last_stages = [&](int buf) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (ld_st < n_stages) copy_stage(buf);
  };

  // A stage holds two column tiles of 32 tokens.  The products of one run on the matrix pipe while the
  // vector ALUs turn the other's logits into weights; the second tile's are turned in the next stage.
  floatx16_t s0[TILES], s1[TILES];
  float nl0 = 0.f, nl1 = 0.f;  // their tokens' normalisers
  // none yet: logits of -inf, weights of zero
#pragma unroll
  for (int tt = 0; tt < TILES; ++tt)
#pragma unroll
    for (int i = 0; i < 16; ++i) s1[tt][i] = kNegInf;
  // B operands of a column tile: lane (token, j), chunk c holds Q[token][16c + 8j .. +8).
  auto read_chunk = [&](int buf, int nt, int c) {
    return as_bf16x8(*reinterpret_cast<const u32x4_t*>(&lds_q[buf][(nt * 32 + n32) * kRow + (((2 * c + jh) ^ (n32 & 15)) * 16)]));
  };
  // (left: tokens from the stage's first one to the end of the prompt)
  auto read_norm = [&](int buf, int nt, int left) {
    const float l = lds_lse[buf][nt * 32 + n32];
    return nt * 32 + n32 < left ? l : -kNegInf;
  };
  auto read_tile = [&](bf16x8_t (&qt)[kChunks], int buf, int nt) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c) qt[c] = read_chunk(buf, nt, c);
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
      for (int i = 0; i < 16; ++i) acc[tt][i] += fast_exp2(fmaf(s[tt][i], cs, -nl));
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

#pragma unroll 1
  for (int i = 0; i < min(kBufs, n_stages); ++i) copy_stage(i);
  if (ld_st == kBufs) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kBufs - 1) * (kCopies + 1)) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // Tiles that start behind the workgroup's keys have no masked pair; the last ones (a tile per 64 keys
  // of the workgroup) cross the diagonal.
  const int n_below = PIPE ? max(0, (T + kTokTile - 1) / kTokTile - (j0 + kKeysPerWg) / kTokTile) * G : 0;
  int st = 0, t0 = last_t0, g = 0;  // stage, its first token, its head
  auto advance = [&]() {
    ++st;
    if (++g == G) { g = 0; t0 -= kTokTile; }
  };
  bf16x8_t qa[kChunks];
  if constexpr (PIPE) {
    // (kBufs stages per turn, so that LDS addresses are constant offsets; what is left goes with the masked ones)
    bf16x8_t qb[kChunks];
    float nla, nlb;
    auto stage = [&](auto b) {
      constexpr int buf = decltype(b)::value;
      if constexpr (TILES == 1) {
        // The end of a stage sits between its two tiles: the rows of the next stage are in LDS before the
        // second tile's products start, so every operand is read one tile ahead of its use.
        read_tile(qb, buf, 1);
        nlb = read_norm(buf, 1, T - t0);
        products(s0, qa);
        add_weights(s1, nl1);
        nl0 = nla;
        settle();
        next_stage(buf);
        advance();
        read_tile(qa, (buf + 1) % kBufs, 0);
        nla = read_norm((buf + 1) % kBufs, 0, T - t0);
        products(s1, qb);
        add_weights(s0, nl0);
        nl1 = nlb;
        settle();
      } else {
        // no registers left for operands one tile ahead: the other wavefront of the SIMD covers the reads
        read_tile(qa, buf, 0);
        nl0 = read_norm(buf, 0, T - t0);
        products(s0, qa);
        add_weights(s1, nl1);
        settle();
        read_tile(qa, buf, 1);
        nl1 = read_norm(buf, 1, T - t0);
        products(s1, qa);
        add_weights(s0, nl0);
        settle();
        next_stage(buf);
        advance();
      }
    };
    if (TILES == 1 && n_below >= kBufs) { read_tile(qa, 0, 0); nla = read_norm(0, 0, T - t0); }
    while (st + kBufs <= min(n_below, n_stages - kBufs)) {  // the last of them still has a stage to copy
      stage(std::integral_constant<int, 0>{});
      stage(std::integral_constant<int, 1>{});
      stage(std::integral_constant<int, 2>{});
      stage(std::integral_constant<int, 3>{});
    }
    static_assert(kBufs == 4, "stages written out");
  }
  if constexpr (PIPE && TILES == 1) {
    int tok1 = T;  // first token of the tile in s1
    while (st < n_stages) {
      const int buf = st % kBufs;
      if (t0 + kTokTile - 1 >= jw0) {  // else every token precedes every key of this wavefront
        mask_tile(s1, tok1);
        add_weights(s1, nl1);
        read_tile(qa, buf, 0);
        nl0 = read_norm(buf, 0, T - t0);
        products(s0, qa);
        read_tile(qa, buf, 1);
        nl1 = read_norm(buf, 1, T - t0);
        products(s1, qa);
        mask_tile(s0, t0);
        add_weights(s0, nl0);
        tok1 = t0 + 32;
      }
      last_stages(buf);
      advance();
    }
    mask_tile(s1, tok1);
    add_weights(s1, nl1);
  } else {
    if (PIPE) add_weights(s1, nl1);
    while (st < n_stages) {
      const int buf = st % kBufs;
#pragma unroll 1
      for (int nt = 0; nt < 2; ++nt) {
        const int tok0 = t0 + nt * 32;
        if (tok0 >= T || tok0 + 31 < jw0) continue;  // past the prompt, or before every key of this wavefront
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
          const bf16x8_t q1 = read_chunk(buf, nt, c);
#pragma unroll
          for (int tt = 0; tt < TILES; ++tt) {
            const floatx16_t zero = {};
            s0[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[tt][c], q1, c == 0 ? zero : s0[tt], 0, 0, 0);
          }
        }
        nl0 = read_norm(buf, nt, T - t0);
        if (tok0 < jw0 + kKeysPerWave - 1) {
          asm volatile("" ::: "memory");  // keeps this a branch: below the diagonal nothing is masked
          mask_tile(s0, tok0);
        }
        add_weights(s0, nl0);
      }
      last_stages(buf);
      advance();
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

// The same for launches that would leave compute units idle.  There a workgroup is a serial chain of stages, 0.6 us each,
// and 8 sequences of 2048 tokens are 64 workgroups.  Here eight wavefronts take the same 32 keys, each a tile of 32 tokens
// in a turn.  So that a key's weights are added in the same order as there, and the bits are the same, the wavefronts
// hand their weights over through LDS, and each adds up those of four keys (two of the 16 a lane holds), tile after tile.
// A turn of eight tiles takes 1.6 us, with the wavefronts in step at its two barriers; 32 heads of 2048 tokens 56 us (83).
// Tried: sums for each wavefront, added at the end, 42 us, but other bits; the products of a turn beside the additions of
// the one before, 60 (the rows then come half a turn ahead instead of two).
constexpr int kParts = 8;
__global__ __launch_bounds__(64 * kParts, 2) void prefill_score_shared_kernel(PrefillParams p) {
  constexpr int kTile = 32;
  // Rows of Q of a wavefront's tile, then its weights: both are its own but for the reading of the weights.
  __shared__ __attribute__((aligned(16))) unsigned char lds_q[2][kParts][kTile * kRow];
  __shared__ __attribute__((aligned(16))) float lds_lse[2][kParts][64];

  const int lane = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n32 = lane & 31, jh = lane >> 5;
  const int T = p.T;
  const int n_pairs = (p.n_blocks + 1) / 2;
  const int n_seq = gridDim.x / n_pairs;      // batch * Hkv
  const int seq = blockIdx.x % n_seq;         // (b, kv head)
  const int pair = blockIdx.x / n_seq;
  const int G = p.Hq / p.Hkv;
  const int64_t row0 = p.row_off ? p.row_off[seq] : (int64_t)seq * T;
  const unsigned char* Kb = p.k + row0 * kRow;
  const int64_t head0 = (int64_t)(seq / p.Hkv) * p.Hq + (int64_t)(seq % p.Hkv) * G;
  const float cs = p.scale_log2e;
  const int last_t0 = (T - 1) / kTokTile * kTokTile;  // first token of the prompt's last 64, which are a stage above
  const int left0 = T - last_t0;
  const int nt = part & 1;                            // which 32 tokens of a stage

#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    const int block = half == 0 ? pair : p.n_blocks - 1 - pair;
    if (half == 1 && block == pair) break;  // odd number of blocks: the middle one is alone
    const int j0 = block * 32;
    bf16x8_t ka[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
      ka[c] = as_bf16x8(*reinterpret_cast<const u32x4_t*>(Kb + (int64_t)min(j0 + n32, T - 1) * kRow + c * 32 + jh * 16));
    // this wavefront's keys: registers 2 part and 2 part + 1 of a lane
    float acc[2] = {0.f, 0.f};

    // Stages as above (heads inside tokens, from the prompt's end); part k takes tile k % 2 of every fourth one.
    const int n_stages = G * ((T + kTokTile - 1) / kTokTile - j0 / kTokTile);
    const int n_turns = (2 * n_stages + kParts - 1) / kParts, mine = (n_stages - part / 2 + kParts / 2 - 1) / (kParts / 2);
    struct Place {
      int g, back;  // head, stages of 64 tokens before the prompt's last
    };
    auto next = [&](Place& at) {
#pragma unroll
      for (int k = 0; k < kParts / 2; ++k)
        if (++at.g == G) { at.g = 0; ++at.back; }
    };
    Place ld = {__builtin_amdgcn_readfirstlane((part / 2) % G), __builtin_amdgcn_readfirstlane((part / 2) / G)}, st = ld;
    // Rows to LDS as above, two turns ahead: piece c of row r lies in slot c ^ (r % 16).  Rows past the prompt repeat the
    // last one.  Only this wavefront reads them, so waiting for its own copies is enough.
    const int st_row = lane / 16;
    const uint32_t st_slot = ((lane % 16) ^ st_row) * 16;  // 4 i rows further: ^ 64 i
    const uint32_t lds_q0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)&lds_q[0][part][0];
    const uint32_t lds_l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)&lds_lse[0][part][0];
    auto copy_tile = [&](int buf) {
      const int64_t row = (head0 + ld.g) * T + last_t0 - (int64_t)ld.back * kTokTile;
      const unsigned char* q = p.q + row * kRow;
      const uint32_t dst = lds_q0 + buf * (kParts * kTile * kRow);
      uint32_t l_off = (nt * kTile + n32) * 4u;
      if (ld.back > 0 || left0 == kTokTile) {
        const uint32_t o = (nt * kTile + st_row) * kRow + st_slot;
        copy_rows_4(dst, q, o, o ^ 64, o ^ 128, o ^ 192);
        copy_rows_4(dst + 4096, q + 4096, o, o ^ 64, o ^ 128, o ^ 192);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          copy_rows(dst + i * 1024, q, min(nt * kTile + st_row + 4 * i, left0 - 1) * kRow + (st_slot ^ (64 * (i % 4))));
        l_off = min(nt * kTile + n32, left0 - 1) * 4u;
      }
      copy_words(lds_l0 + buf * (kParts * 64 * 4), p.lse + row, l_off);
      next(ld);
    };
    if (mine > 0) copy_tile(0);
    if (mine > 1) copy_tile(1);

#pragma unroll 1
    for (int turn = 0; turn < n_turns; ++turn) {
      const int buf = turn & 1;
      unsigned char* const my_q = lds_q[buf][part];
      if (turn < mine) {
        if (turn + 1 < mine) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");  // all but the next turn's copies
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        floatx16_t s;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
          const bf16x8_t q = as_bf16x8(*reinterpret_cast<const u32x4_t*>(my_q + n32 * kRow + ((2 * c + jh) ^ (n32 & 15)) * 16));
          const floatx16_t zero = {};
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c], q, c == 0 ? zero : s, 0, 0, 0);
        }
        const int tok0 = last_t0 - st.back * kTokTile + nt * kTile;
        const float nl = tok0 + n32 < T ? lds_lse[buf][part][n32] : -kNegInf;
        if (tok0 < j0 + 31) {  // crosses the diagonal
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (j0 + 8 * (i / 4) + 4 * jh + i % 4 > tok0 + n32) s[i] = kNegInf;
        }
        float* const out = reinterpret_cast<float*>(my_q) + lane * 2;  // [8 pairs of keys][64 lanes][2]
        typedef float floatx2_t __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < 16; i += 2)
          *reinterpret_cast<floatx2_t*>(out + i * 64) =
              floatx2_t{fast_exp2(fmaf(s[i], cs, -nl)), fast_exp2(fmaf(s[i + 1], cs, -nl))};
        next(st);
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kParts; ++k)
        if (turn * kParts + k < 2 * n_stages) {
          const float* in = reinterpret_cast<const float*>(lds_q[buf][k]) + (part * 64 + lane) * 2;
          acc[0] += in[0];
          acc[1] += in[1];
        }
      __syncthreads();
      if (turn + 2 < mine) copy_tile(buf);
    }
    // Sum over the 32 token lanes of each half, in the pairs of the kernel above.
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int off = 16; off > 0; off >>= 1) acc[i] += __shfl_xor(acc[i], off);
      const int r = 2 * part + i, key = j0 + 8 * (r / 4) + 4 * jh + r % 4;
      if (n32 == 0 && key < T) p.score[row0 + key] = acc[i];
    }
  }
}

template <int TILES, bool PIPE>
hipError_t launch_tiles(PrefillParams p, int64_t n_seq, hipStream_t s) {
  constexpr int kKeysPerWg = kWaves * 32 * TILES;
  p.n_blocks = (p.T + kKeysPerWg - 1) / kKeysPerWg;
  const int64_t n_wg = n_seq * ((p.n_blocks + 1) / 2);
  if (n_wg <= 0 || n_wg > INT32_MAX) return hipErrorInvalidValue;
  prefill_score_kernel<TILES, PIPE><<<dim3((unsigned)n_wg), dim3(64 * kWaves), 0, s>>>(p);
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
  // One tile per wavefront, pipelined, while that gives at most two workgroups to each of the 256 compute units (or
  // three, for a prompt of some length), but for very short prompts, and but for the launches of at most two that two
  // tiles turn into one for every compute unit, from 8192 tokens on: 8 sequences of 15873 to 16384 tokens, 4 of 32257
  // to 32768, 2 of twice as many.  One tile / two tiles on both sides of these: 8 x 12000 x 4 810 / 834, 15360 1028 /
  // 984, 15900 1077 / 1022, 16384 1131 / 1074, 16385 1282 / 1142, 17000 1629 / 1680; 4 x 32256 x 1 559 / 543, 32768 565 /
  // 528, 36000 865 / 900 (just below and just above them two tiles would be better as well).
  // Beyond, two tiles once they fill the chip twice over, if the prompt is long against a workgroup's masked stages
  // (twice as many with two tiles) or the launch is large enough for fewer stages to outweigh them; otherwise the form
  // without pipeline.  us with one tile / two tiles / without pipeline, sequences x tokens x query heads of each:
  //   8 x 2000 x 4        84 /  156 /  118      128 x 1999 x 4      295 /  295 /  298
  //   8 x 8192 x 4       316 /  498 /  489      256 x 700 x 4        94 /   93 /   89
  //   8 x 16384 x 4     1072 / 1024 / 1220      256 x 1300 x 8      626 /  626 /  603
  //   32 x 6000 x 4      603 /  648 /  650      512 x 513 x 8       264 /  274 /  224
  //   32 x 8192 x 4     1082 /  972 / 1130      512 x 1300 x 8     1372 / 1177 / 1268
  //   64 x 3000 x 4      310 /  355 /  331      1024 x 100 x 4     30.2 / 39.8 / 23.9
  // Over 334 shapes (8 to 1024 sequences of 64 to 16384 tokens, 1 to 8 heads) this rule is within 0.4% of the best of
  // these forms on average and 15% at worst (512 x 200 x 1: 15.8 against 13.8).
  const int64_t n_seq = (int64_t)batch * Hkv;
  // Eight wavefronts for the same 32 keys while that gives at most one workgroup to each of the 256 compute units (two do
  // not fit), unless a workgroup has so few turns that handing the weights over costs more than the others save.  us with
  // one tile / shared, sequences x tokens x query heads of each:
  //   1 x 2556 x 7   174 /  114      8 x 2013 x 2   44.5 / 32.2      8 x 2120 x 1   28.3 / 37.0 (272 workgroups)
  //   2 x 246 x 7   35.4 / 20.0      8 x 2048 x 4   83.3 / 56.4     16 x 1131 x 2   30.1 / 39.6 (288)
  //   2 x 200 x 1    9.7 /  8.6     16 x 250 x 4    22.8 / 14.1      2 x 110 x 2     7.0 /  8.4
  //   2 x 8192 x 1  78.8 / 55.1     64 x 227 x 1    11.0 /  9.0     16 x 147 x 1     8.9 /  9.3
  //   4 x 1993 x 7   142 / 93.6     32 x 413 x 1    12.3 / 10.7     24 x 71 x 4     10.1 /  9.9
  // Over 203 drawn shapes of up to 330 such workgroups (100 to 16384 tokens, 1 to 16 heads) launches take 0.49 to 1.01
  // times what the rule above alone gives, 0.72 in the median.
  const int64_t shared = n_seq * ((((int64_t)T + 31) / 32 + 1) / 2);
  if (shared <= 256 && T > 128 && (int64_t)(Hq / Hkv) * T >= 200) {
    p.n_blocks = (T + 31) / 32;
    prefill_score_shared_kernel<<<dim3((unsigned)shared), dim3(64 * kParts), 0, s>>>(p);
    return hipGetLastError();
  }
  const int64_t narrow = n_seq * ((((int64_t)T + 127) / 128 + 1) / 2);  // workgroups with one tile
  const int64_t wide = n_seq * ((((int64_t)T + 255) / 256 + 1) / 2);    // with two
  const int64_t tokens = (int64_t)(Hq / Hkv) * T;                       // rows of Q that a sequence streams
  if (narrow <= 512 && T >= 8192 && wide >= 256) return launch_tiles<2, true>(p, n_seq, s);
  if (narrow <= 512 && (T > 256 || n_seq <= 256)) return launch_tiles<1, true>(p, n_seq, s);
  if (narrow <= 768 && T >= 2000) return launch_tiles<1, true>(p, n_seq, s);
  if (wide >= 512 && (T >= 1700 || (double)tokens * wide >= 7e6)) return launch_tiles<2, true>(p, n_seq, s);
  return launch_tiles<1, false>(p, n_seq, s);
}

}  // namespace baklava
