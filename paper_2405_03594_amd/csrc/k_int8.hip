// Sparse-quantized linear layer (paper section 3.4: int8 weights and int8
// activations) and its dense comparator, for gfx950.
//
// acc[m][n] = sum over kept k of Xq[m][k] * Wq[n][k] is accumulated exactly in
// int32 by v_mfma_i32_16x16x64_i8; the epilogue is
//   Y[m][n] = fp16_rne( (float(acc) * sx[m]) * sw[n] )
// with each product rounded to binary32 (no fused multiply-add).
//
// This file: where the sparse layer's launches go (k_int8_quad.hip, k_wide.hip,
// k_prefill.hip), the dense comparator and the activations' quantizer.
#include "spl_common.h"

namespace spl {
namespace {

constexpr int kI8Waves = 8;                 // dense kernel
constexpr int kI8Threads = 64 * kI8Waves;
constexpr int kI8Unroll = 4;                // dense kernel: 64-column steps per wave per group
constexpr int64_t kI8MaxBytes = (int64_t)1 << 31;   // activations of one launch
// Batches of more rows than one batch fragment go to the streaming kernel (q|k|v 12.4 us a launch at 17 rows, 13.8 at
// 32, 25.4 at 127; gate|up 20.2, 21.3, 46.2).
constexpr int64_t kI8WideMinM = 17;
// On up to one row block per CU, where the four-tile kernel waits for its activations most, from 9 rows of up to 3072
// columns, 12 of up to 4096 and 16 past them: its launches / the streaming ones at 9, 12, 14 and 16 rows 3072 x 3072
// 5.6 / 5.4, 5.8 / 5.4, 5.9 / 5.4, 6.1 / 5.4 us (at 8 rows, where only decoding waits, 5.3 to 5.6 / 5.2 to 5.5),
// 4096 x 4096 6.0 / 6.2, 6.2 / 6.2, 6.4 / 6.2, 6.6 / 6.2, 4096 x 11008 at 12, 14 and 16 10.1 / 10.6, 10.4 / 10.7,
// 10.9 / 10.8; 2048 x 2048 at 9 and 12 4.5 / 4.4, 4.65 / 4.4; q|k|v, 3 blocks per CU, 10.9 / 11.2 at 12.
bool i8_wide_small(int64_t M, int64_t blocks, int64_t kmax) {
  return M >= (kmax <= 3072 ? 9 : kmax <= 4096 ? 12 : 16) && blocks <= device_cus();
}

__device__ __forceinline__ i32x4 mfma_i8(u32x4 a, u32x4 b, i32x4 c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0,
                                               0);
}

// Combine the waves' int32 partial sums and run the epilogue.
// part: [W][MT][4][64] int32 in LDS; output (f, r, l): n = n0 + 4*(l/16) + r, m = m0 + 16 f + l%16.
template <int MT, int W>
__device__ __forceinline__ void i8_finish(const i32x4 (&acc)[MT], int32_t* part, int wave, int lane, int64_t n0,
                                          int64_t N, int64_t m0, int64_t M, const float* __restrict__ sx,
                                          const float* __restrict__ sw, uint16_t* __restrict__ Y,
                                          int32_t* __restrict__ acc_out) {
#pragma unroll
  for (int f = 0; f < MT; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[((wave * MT + f) * 4 + r) * 64 + lane] = acc[f][r];
  __syncthreads();
  for (int o = threadIdx.x; o < MT * 4 * 64; o += W * kWave) {
    const int f = o / 256, r = (o / 64) & 3, l = o & 63;
    const int64_t n = n0 + 4 * (l >> 4) + r;
    const int64_t m = m0 + 16 * f + (l & 15);
    if (n < N && m < M) {
      int32_t s = 0;
#pragma unroll
      for (int w = 0; w < W; ++w) s += part[w * MT * 256 + o];
      if (acc_out) acc_out[m * N + n] = s;
      const float a = static_cast<float>(s);
      const float t = __fmul_rn(a, sx[m]);
      const float y = __fmul_rn(t, sw[n]);
      Y[m * N + n] = F16::from_f32(y);
    }
  }
}

struct I8DenseTaskArg {
  const int8_t* Xq;
  const float* sx;
  const int8_t* W;
  int64_t N, K;
  const float* sw;
  uint16_t* Y;
  int32_t* acc;
};
struct I8DenseGroupArg {
  I8DenseTaskArg t[SPL_MAX_GROUP];
  int32_t first[SPL_MAX_GROUP + 1];
  int32_t count;
  int32_t M;
};

template <int MT>
__global__ void __launch_bounds__(kI8Threads) k_dense_int8(const I8DenseGroupArg g) {
  const int ti = find_task(g.first, g.count);
  const I8DenseTaskArg tk = g.t[ti];
  const int8_t* __restrict__ Xq = tk.Xq;
  const float* __restrict__ sx = tk.sx;
  const int8_t* __restrict__ Wq = tk.W;
  const int64_t M = g.M, K = tk.K, N = tk.N;
  const float* __restrict__ sw = tk.sw;
  uint16_t* __restrict__ Y = tk.Y;
  int32_t* __restrict__ acc_out = tk.acc;
  __shared__ int32_t part[kI8Waves * MT * 256];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int fr = lane & 15, fg = lane >> 4;
  const int Q = (int)((K + 63) / 64);                     // 64-column steps
  const int G = (Q + kI8Unroll - 1) / kI8Unroll;
  const int64_t n0 = ((int64_t)blockIdx.x - g.first[ti]) * 16;
  const int64_t m0 = (int64_t)blockIdx.y * 16 * MT;
  const int64_t wrow = (n0 + fr < N ? n0 + fr : N - 1) * K;
  int64_t xrow[MT];
#pragma unroll
  for (int f = 0; f < MT; ++f) {
    const int64_t m = m0 + 16 * f + fr;
    xrow[f] = (m < M ? m : M - 1) * K;
  }
  i32x4 acc[MT];
#pragma unroll
  for (int f = 0; f < MT; ++f) acc[f] = i32x4{0, 0, 0, 0};
  for (int g = wave; g < G; g += kI8Waves) {
    u32x4 a[kI8Unroll];
    u32x4 xb[kI8Unroll][MT];
#pragma unroll
    for (int u = 0; u < kI8Unroll; ++u) {
      const int q = g * kI8Unroll + u;
      int64_t k = (int64_t)q * 64 + 16 * fg;
      const bool kok = k < K && q < Q;
      if (!kok) k = 0;
      u32x4 v = *reinterpret_cast<const u32x4*>(Wq + wrow + k);
      if (!kok) v = u32x4{0u, 0u, 0u, 0u};
      a[u] = v;
#pragma unroll
      for (int f = 0; f < MT; ++f) {
        u32x4 x = *reinterpret_cast<const u32x4*>(Xq + xrow[f] + k);
        if (!kok) x = u32x4{0u, 0u, 0u, 0u};
        xb[u][f] = x;
      }
    }
#pragma unroll
    for (int u = 0; u < kI8Unroll; ++u)
#pragma unroll
      for (int f = 0; f < MT; ++f) acc[f] = mfma_i8(a[u], xb[u][f], acc[f]);
  }
  i8_finish<MT, kI8Waves>(acc, part, wave, lane, n0, N, m0, M, sx, sw, Y, acc_out);
}

int i8_fragments(int64_t M) { return M <= 16 ? 1 : (M <= 32 ? 2 : 4); }

// Per-token activation quantisation (paper section 3.4 quantises the
// activations to int8; symmetric, one binary32 scale per row): one workgroup
// per row of X [M][K] (K % 8 == 0, 16-byte pieces of 8 fp16/bf16 values)
// finds amax = max |x| (a wave reduction, then the 4 wave maxima), sets
// scale = amax / 127 (1 when amax is 0), and writes the codes
// clamp(round-half-even(x / scale), -127, 127); each division is correctly
// rounded.  Rows of up to TH PT pieces stay in registers between the two
// steps (one read of X); PT = 0 re-reads longer rows (from L2).
template <class T, int PT, int TH>
__global__ void __launch_bounds__(TH) k_quantize_rows(const uint16_t* __restrict__ X, int64_t K,
                                                       int8_t* __restrict__ Xq, float* __restrict__ sx) {
  constexpr int R = PT > 0 ? PT : 1;
  __shared__ float wmax[TH / kWave];
  const int64_t m = blockIdx.x;
  const uint16_t* x = X + m * K;
  const int64_t P = K / 8;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  auto amax8 = [](const u32x4& v, float a) {
#pragma unroll
    for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(T::to_f32((v[e >> 1] >> (16 * (e & 1))) & 0xffffu)));
    return a;
  };
  float amax = 0.0f;
  u32x4 v[R];
  if constexpr (PT > 0) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int64_t p = t + TH * i;
      v[i] = p < P ? *reinterpret_cast<const u32x4*>(x + 8 * p) : u32x4{0u, 0u, 0u, 0u};
      amax = amax8(v[i], amax);
    }
  } else {
    for (int64_t p = t; p < P; p += TH) amax = amax8(*reinterpret_cast<const u32x4*>(x + 8 * p), amax);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) amax = fmaxf(amax, __shfl_xor(amax, d));
  if (lane == 0) wmax[wave] = amax;
  __syncthreads();
  amax = wmax[0];
#pragma unroll
  for (int w = 1; w < TH / kWave; ++w) amax = fmaxf(amax, wmax[w]);
  const float scale = amax == 0.0f ? 1.0f : __fdiv_rn(amax, 127.0f);
  if (t == 0) sx[m] = scale;
  int8_t* q = Xq + m * K;
  auto put8 = [&](const u32x4& w, int64_t p) {
    uint32_t c[2] = {0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float r = rintf(__fdiv_rn(T::to_f32((w[e >> 1] >> (16 * (e & 1))) & 0xffffu), scale));
      r = fminf(fmaxf(r, -127.0f), 127.0f);
      c[e >> 2] |= ((uint32_t)(int32_t)r & 0xffu) << (8 * (e & 3));
    }
    *reinterpret_cast<u32x2*>(q + 8 * p) = u32x2{c[0], c[1]};
  };
  if constexpr (PT > 0) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int64_t p = t + TH * i;
      if (p < P) put8(v[i], p);
    }
  } else {
    for (int64_t p = t; p < P; p += TH) put8(*reinterpret_cast<const u32x4*>(x + 8 * p), p);
  }
}

template <class T>
void quantize_rows_launch(const uint16_t* x, int64_t M, int64_t K, int8_t* Xq, float* sx, hipStream_t s) {
  const int64_t P = K / 8;
  const dim3 grid((unsigned)M);
  auto launch = [&](auto* kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, x, K, Xq, sx);
  };
  // Up to one row per CU a launch takes as long as one workgroup, whose divisions the row's threads share: 11008
  // columns on 256 / 1024 threads 4.8 / 4.1 us at one row, 5.3 / 4.5 at 16.
  const bool few = M <= device_cus();
  if (P <= 256)
    launch(k_quantize_rows<T, 1, 256>, 256);
  else if (few && P <= 512)
    launch(k_quantize_rows<T, 1, 512>, 512);
  else if (few && P <= 1024)
    launch(k_quantize_rows<T, 1, 1024>, 1024);
  else if (few && P <= 2048)
    launch(k_quantize_rows<T, 2, 1024>, 1024);
  else if (P <= 512)
    launch(k_quantize_rows<T, 2, 256>, 256);
  else if (P <= 1024)
    launch(k_quantize_rows<T, 4, 256>, 256);
  else if (P <= 2048)
    launch(k_quantize_rows<T, 8, 256>, 256);
  else
    launch(k_quantize_rows<T, 0, 256>, 256);
}

}  // namespace

hipError_t launch_sparse_int8(const spl_int8_task* tasks, int count, int64_t M, hipStream_t s) {
  if (M >= kI8PrefillMinM) {                         // MFMA-tiled kernel with activations shared in LDS
    for (int i = 0; i < count; ++i) {
      const hipError_t e = launch_sparse_prefill_i8(tasks[i], M, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  int64_t blocks = 0, kmax = 0;
  for (int i = 0; i < count; ++i) {
    blocks += tile_blocks(tasks[i].Wq->rows);
    kmax = tasks[i].Wq->cols > kmax ? tasks[i].Wq->cols : kmax;
  }
  bool wide = M >= kI8WideMinM || i8_wide_small(M, blocks, kmax);
  for (int i = 0; i < count; ++i) wide = wide && sparse_wide_fits(M, tasks[i].Wq->cols, 1);
  if (wide) return launch_int8_wide(tasks, count, M, s);
  // Up to one batch fragment four tiles per scan, where 32 bits address the activations: launches of the streaming
  // kernel / that one at 8 rows 4096 x 4096 6.0 / 6.0 us, 4096 x 11008 9.8 / 9.8, q|k|v 10.4 / 9.9, gate|up 16.8 /
  // 15.1.
  bool quad = M <= 16;
  for (int i = 0; i < count; ++i) quad = quad && int8_quad_fits(M, tasks[i].Wq->cols);
  if (quad) return launch_int8_quad(tasks, count, M, s);
  // Activations past 32-bit addressing: as many rows at a time as it takes.
  const int64_t rows = kmax < kI8MaxBytes / M ? M : kI8MaxBytes / kmax;
  for (int64_t m0 = 0; m0 < M; m0 += rows) {
    spl_int8_task t[SPL_MAX_GROUP];
    for (int i = 0; i < count; ++i) {
      t[i] = tasks[i];
      const int64_t N = t[i].Wq->rows;
      t[i].Xq += m0 * t[i].Wq->cols, t[i].x_scales += m0;
      t[i].Y = static_cast<uint16_t*>(t[i].Y) + m0 * N;
      if (t[i].acc_out) t[i].acc_out += m0 * N;
    }
    const hipError_t e = launch_int8_wide(t, count, M - m0 < rows ? M - m0 : rows, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_dense_int8(const spl_dense_int8_task* tasks, int count, int64_t M, hipStream_t s) {
  if (M >= kI8PrefillMinM) {
    for (int i = 0; i < count; ++i) {
      const hipError_t e = launch_dense_prefill_i8(tasks[i], M, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  I8DenseGroupArg g{};
  g.count = count;
  g.M = (int32_t)M;
  g.first[0] = 0;
  for (int i = 0; i < count; ++i) {
    g.t[i] = I8DenseTaskArg{tasks[i].Xq, tasks[i].x_scales, tasks[i].Wq, tasks[i].N, tasks[i].K, tasks[i].w_scales,
                            static_cast<uint16_t*>(tasks[i].Y), tasks[i].acc_out};
    g.first[i + 1] = g.first[i] + (int32_t)((tasks[i].N + 15) / 16);
  }
  const int MT = i8_fragments(M);
  const dim3 grid((unsigned)g.first[count], (unsigned)((M + 16 * MT - 1) / (16 * MT))), block(kI8Threads);
  if (MT == 1)
    hipLaunchKernelGGL((k_dense_int8<1>), grid, block, 0, s, g);
  else if (MT == 2)
    hipLaunchKernelGGL((k_dense_int8<2>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((k_dense_int8<4>), grid, block, 0, s, g);
  return hipGetLastError();
}

hipError_t launch_quantize_rows_i8(const void* X, int32_t dtype, int64_t M, int64_t K, int8_t* Xq, float* sx,
                                   hipStream_t s) {
  const uint16_t* x = static_cast<const uint16_t*>(X);
  if (dtype == SPL_BF16)
    quantize_rows_launch<Bf16>(x, M, K, Xq, sx, s);
  else
    quantize_rows_launch<F16>(x, M, K, Xq, sx, s);
  return hipGetLastError();
}

}  // namespace spl
