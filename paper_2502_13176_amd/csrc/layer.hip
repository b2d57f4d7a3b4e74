// Layer importance heuristic ("Layer Importance Heuristic"): the cosine between the input and the
// output hidden state of a layer, token by token, and its mean over the prompt.
//
// HBM-bound: every hidden-state row is read once (2 * hidden * 2 bytes per token for bf16).  One
// wavefront per token row, or per two or four short ones: 64 lanes x 16 bytes per load instruction, all
// loads of the row pairs in flight before the first use, non-temporal (read once); three dot products
// per row reduced over the wavefront.  A workgroup takes 16 consecutive rows and writes the sum of their cosines; a
// second small kernel adds the workgroup sums in a fixed order (deterministic, no atomics).
#include <mutex>
#include <type_traits>

#include "baklava.h"
#include "common.h"

namespace baklava {

constexpr int kRowsPerWg = 16;

namespace {

constexpr int kWaves = 4;
constexpr float kCosEps = 1e-8f;

struct LayerParams {
  const unsigned char* x_in;   // [n_seq, T, hidden] bf16
  const unsigned char* x_out;
  float* cos_out;              // [n_seq, T] or null
  float* tile_sum;             // [n_seq, n_tiles]
  int32_t T, hidden, n_tiles;
};

__device__ __forceinline__ void accumulate(uint4 a, uint4 b, float& dot, float& na, float& nb) {
  const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a0 = __uint_as_float(aw[i] << 16), a1 = __uint_as_float(aw[i] & 0xffff0000u);
    const float b0 = __uint_as_float(bw[i] << 16), b1 = __uint_as_float(bw[i] & 0xffff0000u);
    dot = fmaf(a0, b0, dot); dot = fmaf(a1, b1, dot);
    na = fmaf(a0, a0, na);   na = fmaf(a1, a1, na);
    nb = fmaf(b0, b0, nb);   nb = fmaf(b1, b1, nb);
  }
}

// Sum over the 16 lanes of a row of lanes, every lane receiving it: the pairs of a butterfly over lane distances 8, 4,
// 2, 1 (lanes that a rotation reaches in place of the partner hold the same sum as it).
__device__ __forceinline__ float row_sum(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += dpp(v, std::integral_constant<int, 0x128>{});  // row_ror:8
  v += dpp(v, std::integral_constant<int, 0x124>{});  // row_ror:4
  v += dpp(v, std::integral_constant<int, 0x122>{});  // row_ror:2
  v += dpp(v, std::integral_constant<int, 0x121>{});  // row_ror:1
  return v;
}

// A wavefront's four rows are taken ROWS at a time, up to 8 KB of each tensor in flight: row by row, short rows spent
// their time on one memory latency each (hidden 512, 768 and 1024 all took 93 to 97 us for 32 x 4096 tokens).  A sum
// over 64 lanes goes to the 64 / ROWS lanes that keep its row in the first steps, so four rows cost 9 exchanges and 12
// rotations instead of 72 exchanges.
template <int ROWS>
__global__ __launch_bounds__(256) void layer_cosine_kernel(LayerParams p) {
  constexpr int kPieces = 8 / ROWS, kPerWave = kRowsPerWg / kWaves;
  __shared__ float wave_sum[kWaves];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int seq = blockIdx.x / p.n_tiles, tile = blockIdx.x % p.n_tiles;
  const int64_t row_bytes = (int64_t)p.hidden * 2;
  float wsum = 0.f;
  for (int k = 0; k < kPerWave; k += ROWS) {
    const int t0 = tile * kRowsPerWg + wave + k * kWaves;  // rows t0, t0 + 4, ...
    if (t0 >= p.T) break;
    int64_t at[ROWS];
    float dot[ROWS], na[ROWS], nb[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      at[r] = ((int64_t)seq * p.T + min(t0 + r * kWaves, p.T - 1)) * row_bytes;  // past the prompt: its last row
      dot[r] = na[r] = nb[r] = 0.f;
    }
    // (a 4096-wide row is one pass)
    for (int64_t h0 = (int64_t)lane * 16; h0 < row_bytes; h0 += kPieces * 1024) {
      uint4 av[ROWS][kPieces], bv[ROWS][kPieces];
#pragma unroll
      for (int u = 0; u < kPieces; ++u) {
        const int64_t o = h0 + u * 1024;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) av[r][u] = bv[r][u] = make_uint4(0, 0, 0, 0);
        if (o < row_bytes) {
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            av[r][u] = load_nt16(p.x_in + at[r] + o);
            bv[r][u] = load_nt16(p.x_out + at[r] + o);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int u = 0; u < kPieces; ++u) accumulate(av[r][u], bv[r][u], dot[r], na[r], nb[r]);
    }
    // lanes 64 / ROWS * r and on keep row r
    int off = 32;
#pragma unroll
    for (int n = ROWS / 2; n > 0; n /= 2, off /= 2) {
      const bool upper = lane & off;
#pragma unroll
      for (int r = 0; r < n; ++r) {
        auto fold = [&](float (&v)[ROWS]) { v[r] = (upper ? v[r + n] : v[r]) + __shfl_xor(upper ? v[r] : v[r + n], off); };
        fold(dot);
        fold(na);
        fold(nb);
      }
    }
#pragma unroll
    for (; off >= 16; off /= 2) {
      dot[0] += __shfl_xor(dot[0], off);
      na[0] += __shfl_xor(na[0], off);
      nb[0] += __shfl_xor(nb[0], off);
    }
    const float d = row_sum(dot[0]), a = row_sum(na[0]), b = row_sum(nb[0]);
    const float c = d / fmaxf(sqrtf(a) * sqrtf(b), kCosEps);
    const int t = t0 + lane / (64 / ROWS) * kWaves;
    if (lane % (64 / ROWS) == 0 && p.cos_out && t < p.T) p.cos_out[(int64_t)seq * p.T + t] = c;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (t0 + r * kWaves < p.T) wsum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), r * (64 / ROWS)));
  }
  if (lane == 0) wave_sum[wave] = wsum;
  __syncthreads();
  if (threadIdx.x == 0)
    p.tile_sum[(int64_t)seq * p.n_tiles + tile] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
}

__global__ __launch_bounds__(64) void layer_mean_kernel(const float* tile_sum, float* sim_out, int n_tiles, int T) {
  const int seq = blockIdx.x;
  float acc = 0.f;
  for (int i = threadIdx.x; i < n_tiles; i += 64) acc += tile_sum[(int64_t)seq * n_tiles + i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (threadIdx.x == 0) sim_out[seq] = acc / (float)T;
}

}  // namespace

hipError_t launch_layer_similarity(const void* x_in, const void* x_out, int n_seq, int T, int hidden,
                                   float* cos_out, float* sim_out, float* tile_sum, hipStream_t s) {
  LayerParams p;
  p.x_in = reinterpret_cast<const unsigned char*>(x_in);
  p.x_out = reinterpret_cast<const unsigned char*>(x_out);
  p.cos_out = cos_out;
  p.tile_sum = tile_sum;
  p.T = T; p.hidden = hidden;
  p.n_tiles = (T + kRowsPerWg - 1) / kRowsPerWg;
  const int64_t n_wg = (int64_t)n_seq * p.n_tiles;
  if (n_wg <= 0 || n_wg > INT32_MAX) return hipErrorInvalidValue;
  // As many rows at a time as 8 KB of a tensor hold, but one from 3.5 KB on, where enough is in flight anyway.  us, row by
  // row / so, 32 prompts of 4096 tokens: hidden 512 89.9 / 43.9, 768 92.5 / 62.9, 1024 95.8 / 84.4, 1152 (28 prompts)
  // 103 / 82.7, 1536 (21) 84.0 / 81.9, 1792 (18) 83.5 / 81.8, two rows at 2048 (16) 87.2 / 88.3; 32 prompts of 1000
  // tokens: 512 27.4 / 16.2, 1024 30.1 / 24.0, 1536 35.6 / 33.9.
  if (hidden <= 1024) layer_cosine_kernel<4><<<dim3((unsigned)n_wg), dim3(256), 0, s>>>(p);
  else if (hidden <= 1792) layer_cosine_kernel<2><<<dim3((unsigned)n_wg), dim3(256), 0, s>>>(p);
  else layer_cosine_kernel<1><<<dim3((unsigned)n_wg), dim3(256), 0, s>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  layer_mean_kernel<<<dim3(n_seq), dim3(64), 0, s>>>(tile_sum, sim_out, p.n_tiles, T);
  return hipGetLastError();
}

}  // namespace baklava

// ---------------------------------------------------------------------------------------------
// The same pass for callers that cannot allocate and have no workspace to hand over: the
// per-workgroup partial sums live in a fixed device array instead.
// ---------------------------------------------------------------------------------------------

static __device__ __align__(256) float scratch[BAKLAVA_LAYER_STATIC_MAX_TILES];

namespace {

// In host code the array's name is only a handle for the runtime; the device address has to be
// asked for, once per device (every device holds its own copy of the array).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};

int scratch_for_current_device(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) { baklava::note_hip_error(e); return BAKLAVA_EHIP; }
  if (dev < 0 || dev >= kMaxDevices) return BAKLAVA_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    float* ptr = nullptr;
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) { baklava::note_hip_error(e); return BAKLAVA_EHIP; }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return BAKLAVA_OK;
}

}  // namespace

extern "C" int baklava_layer_similarity_static(const void* x_in, const void* x_out, int32_t n_seq, int32_t T,
                                               int32_t hidden, int32_t dtype, float* cos_out, float* sim_out,
                                               void* stream) {
  if (!x_in || !x_out || !sim_out) return BAKLAVA_EINVAL;
  if (n_seq <= 0 || T <= 0 || hidden <= 0 || hidden % 8 || dtype != BAKLAVA_BF16) return BAKLAVA_EINVAL;
  if (((uintptr_t)x_in | (uintptr_t)x_out) & 15) return BAKLAVA_EINVAL;
  if (((uintptr_t)sim_out | (uintptr_t)cos_out) & 3) return BAKLAVA_EINVAL;
  const int64_t tiles = (int64_t)n_seq * (((int64_t)T + baklava::kRowsPerWg - 1) / baklava::kRowsPerWg);
  if (tiles > BAKLAVA_LAYER_STATIC_MAX_TILES) return BAKLAVA_ECAPACITY;
  float* tile_sum = nullptr;
  const int st = scratch_for_current_device(&tile_sum);
  if (st != BAKLAVA_OK) return st;
  // Every partial sum the second kernel reads is written by the first one in this call, so nothing
  // has to be cleared; what earlier calls left in the array is never read.
  const hipError_t e = baklava::launch_layer_similarity(x_in, x_out, n_seq, T, hidden, cos_out, sim_out, tile_sum,
                                                        (hipStream_t)stream);
  if (e != hipSuccess) { baklava::note_hip_error(e); return BAKLAVA_EHIP; }
  return BAKLAVA_OK;
}
