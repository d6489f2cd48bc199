// Streaming kernel for sparse linear layers at batches of 2 to about a hundred
// rows (fp16, bf16 and int8 payloads), for gfx950.
//
// At these batches the product is a stream of compressed weights: one
// Llama-2-7B layer at 64 rows is 25 GFLOP against 147 MB.  As in the decode
// kernel a wave expands tiles straight into its MFMA A operand (paper section
// 2.4.2), here with up to four batch fragments of 16 rows per expanded tile
// and R row blocks per wave:
//
//   * a workgroup owns R consecutive 16-row blocks (gated: one of the gate and
//     one of the up matrix) and 8 XG batch rows; its W waves split the k-steps
//     into contiguous ranges and run without a barrier until the reduction;
//   * a wave walks its range in chunks of 128 bytes of an activation row: 64
//     columns (two tiles) of 16-bit payloads, 128 columns (four tiles) of
//     int8.  Everything a chunk needs is loaded one chunk ahead into
//     registers and staged in the wave's own LDS: the blocks' values (16-byte
//     pieces; a slot holds the chunk's tiles even when they are full, so the
//     schedule never depends on the pattern), their bitmask words regrouped by
//     row, and the activations;
//   * the activations pass through LDS because of how they are read: the MFMA
//     operand wants 16 rows in 16 consecutive lanes, and a load of that shape
//     touches a different cache line in each lane, one lane per cycle of the
//     address unit (counters of a version that loaded operands directly: 67
//     cache accesses per instruction, 16 bytes per cycle and CU, the unit busy
//     two thirds of a 4096 x 4096 launch at 64 rows, 19.8 us).  Eight lanes read one
//     row's 128 bytes instead, 64 bytes per cycle; LDS (pieces swizzled by
//     row) turns them: 13.9 us there, and gate|up at 16 rows 26 us (30.5 in the
//     paired decode kernel);
//   * the waves' partial sums are added in LDS in wave order and rounded once
//     (int8: exact sums and the int8 path's epilogue).
//
// What bounds it at 64 rows is the activations' way through L2, L1 and LDS:
// each CU reads all of X once per resident workgroup (512 KB for 4096
// columns, at most 64 bytes per cycle), which R = 2 halves where the grid is
// large enough; below 16 rows it is latency, as in the decode kernel.
#include <type_traits>

#include "spl_common.h"

namespace spl {
namespace {

struct WideI8 {};                // int8 weights and activations

template <class T>
constexpr bool wide_q() { return std::is_same<T, WideI8>::value; }

template <class T>
struct WideAcc {
  using t = f32x4;
  using e = float;
};
template <>
struct WideAcc<WideI8> {
  using t = i32x4;
  using e = int32_t;
};

template <class T>
__device__ __forceinline__ typename WideAcc<T>::t wide_mfma(u32x4 a, u32x4 b, typename WideAcc<T>::t c) {
  if constexpr (wide_q<T>())
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0,
                                                 0);
  else if constexpr (std::is_same<T, Bf16>::value)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

struct WideTaskArg {
  const unsigned char* X;        // [M][K] activations
  uint16_t* Y;                   // [M][N]: the payload type, fp16 for int8
  const uint32_t* bm;
  const unsigned char* values;
  const int32_t* toff;
  int64_t N, K;
  const float* sx;               // int8: activation scales [M], weight scales [N], optional int32 sums [M][N]
  const float* sw;
  int32_t* acc;
};
struct WideGroupArg {
  WideTaskArg t[SPL_MAX_GROUP];       // gated: the gate and the up matrix
  int32_t first[SPL_MAX_GROUP + 1];   // first workgroup of each task; first[count] = grid size along x
  int32_t count;
  int32_t M;
  int32_t rows;                       // batch rows per workgroup (grid y)
};

constexpr uint32_t kWideOob = 0x80000000u;   // a byte offset past any accepted X

// Bytes of a block's value slot: the chunk's full tiles, up to 15 bytes before
// the first value and 12 past the last window, rounded up to 16.
constexpr int kWideSlot = 2048 + 32;
// LDS of a wave: staged activations, then the blocks' value slots.
template <int R, int XG>
constexpr int wide_wave_lds() { return XG * 1024 + R * kWideSlot; }
template <int R, int XG, int W>
constexpr size_t wide_lds() {
  constexpr size_t red = (size_t)W * ((XG + 1) / 2) * 1024, st = (size_t)W * wide_wave_lds<R, XG>();
  return st > red ? st : red;
}

// Sum the waves' partial 16 x 16 MT results (lane l, register i of a fragment:
// row 4 (l / 16) + i, batch row l % 16) in wave order; f(i, e, sum) gets
// element e (fragment e / 256, lane e / 4 % 64, register e % 4) as the
// thread's i-th.
template <class T, int MT, int W, class F>
__device__ __forceinline__ void wide_sum(typename WideAcc<T>::e* red, const typename WideAcc<T>::t (&acc)[MT], F f) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < MT; ++t)
    *reinterpret_cast<typename WideAcc<T>::t*>(red + ((wave * MT + t) * 64 + lane) * 4) = acc[t];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < (256 * MT + W * kWave - 1) / (W * kWave); ++i) {
    const int e = threadIdx.x + i * W * kWave;
    if (256 * MT % (W * kWave) != 0 && e >= 256 * MT) break;
    typename WideAcc<T>::e s = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += red[w * MT * 256 + e];
    f(i, e, s);
  }
}

// The launch bound keeps the registers that the staged chunk needs (up to 160)
// and lets LDS decide the workgroups per CU; one row block of up to four
// staged-row groups on 8 waves is held to 80, so that three share a CU (int8
// at 32 rows took 82: q|k|v 23 us instead of 13.8, with the select below).
template <class T, int R, int XG, int W, bool kGated>
__global__ void __launch_bounds__(W * kWave, W == 16 ? 4 : W == 8 ? (R == 1 && XG <= 4 ? 6 : 2) : 3) k_sparse_wide(const WideGroupArg g) {
  static_assert(!kGated || (R == 2 && !wide_q<T>()), "gated: a gate and an up block");
  constexpr bool kQ = wide_q<T>();
  constexpr int TC = kQ ? 4 : 2;                     // tiles per chunk; MFMA step j takes tile j (int8: 2j, 2j + 1)
  constexpr int PC = kQ ? 16 : 8;                    // columns per 16-byte piece of an activation row
  constexpr int MT = (XG + 1) / 2;                   // batch fragments
  constexpr int NQ = (TC * R + 3) / 4;               // bitmask dwords per lane and chunk
  constexpr int WS = TC * R + (kQ ? 1 : 2);          // words row stride: rows in distinct banks
  using Acc = typename WideAcc<T>::t;
  extern __shared__ __align__(16) unsigned char dsm[];
  __shared__ u32x2 lut[16];                          // 16-bit: nibble_selector16; int8: nibble_selector8 in .x
  __shared__ __align__(16) uint32_t words[W][16 * WS];
  const int ti = kGated ? 0 : find_task(g.first, g.count);
  const WideTaskArg tk = g.t[ti];
  const WideTaskArg tu = g.t[kGated ? 1 : ti];
  const int64_t K = tk.K;
  const int64_t B = tile_blocks(tk.N);
  const int64_t blk0 = (int64_t)(kGated ? 1 : R) * ((int64_t)blockIdx.x - g.first[ti]);
  const int m0 = g.rows * (int)blockIdx.y;
  const int M = g.M - m0 < g.rows ? g.M - m0 : g.rows;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int fr = lane & 15, fg = lane >> 4;
  const int S = (int)tile_steps(K);
  int kbeg, kend;                                    // this wave's k-steps: whole chunks, clipped to S
  {
    const int P = (S + TC - 1) / TC, L = (P + W - 1) / W;
    kbeg = TC * (wave * L < P ? wave * L : P);
    kend = kbeg + TC * L < S ? kbeg + TC * L : S;
    if (kbeg > kend) kbeg = kend;
  }
  // block b: its bitmask words, offsets and values; a block past the matrix aliases the first with zero words
  const uint32_t* bmb[R];
  const int32_t* tob[R];
  const unsigned char* vbs[R];
  bool live[R];
#pragma unroll
  for (int b = 0; b < R; ++b) {
    const int64_t rb = blk0 + (kGated ? 0 : b);
    live[b] = rb < B;
    const WideTaskArg& tb = kGated && b == 1 ? tu : tk;
    const int64_t at = (live[b] ? rb : blk0) * S;
    bmb[b] = tb.bm + at * 16;
    tob[b] = tb.toff + at;
    vbs[b] = tb.values;
  }

  // Activations of a chunk: load i covers rows 8 i .. 8 i + 7, lane l row 8 i + l / 8, piece l % 8 of its 128
  // bytes.  Rows past M and columns past K pass an offset past the buffer, which reads zeros without a fetch.
  constexpr int XB = kQ ? 1 : 2;                     // bytes per activation
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(tk.X + XB * (int64_t)m0 * K), (short)0, (int)(XB * (int64_t)M * K), 0x00020000);
  uint32_t xoff[XG];
#pragma unroll
  for (int i = 0; i < XG; ++i) {
    const int m = 8 * i + (lane >> 3);
    xoff[i] = m < M ? XB * ((uint32_t)m * (uint32_t)K + (uint32_t)(PC * (lane & 7))) : kWideOob;
  }

  // Offsets of the wave's tiles: lane i holds that of tile ob + i (clamped to the range end)
  int ob = kbeg;
  int32_t orng[R];
  auto load_offsets = [&]() {
    const int t = ob + lane < kend ? ob + lane : kend;
#pragma unroll
    for (int b = 0; b < R; ++b) orng[b] = tob[b][t];
  };
  // the chunk in flight
  u32x4 xv[XG];
  u32x4 vv[R][2];                                    // value pieces 0 .. 127 of each block (a 129th is read when staged)
  uint32_t wv[NQ];
  uint32_t a0[R];                                    // first value byte loaded (16-byte aligned)
  int np[R];                                         // 16-byte pieces: at most 129
  uint32_t rel[R][TC];                               // byte of each tile's first value, from a0
  auto issue = [&](int c0) {
    const int r = c0 - ob;
#pragma unroll
    for (int b = 0; b < R; ++b) {
      uint32_t o[TC + 1];                            // tiles past the range: its end
#pragma unroll
      for (int j = 0; j <= TC; ++j) o[j] = (uint32_t)__builtin_amdgcn_readlane(orng[b], r + j);
      a0[b] = (XB * o[0]) & ~15u;
#pragma unroll
      for (int j = 0; j < TC; ++j) rel[b][j] = XB * o[j] - a0[b];
      np[b] = (int)((XB * o[TC] - a0[b] + 15u) >> 4);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (i > 0 && np[b] <= kWave * i) continue;   // wave-uniform
        const uint32_t piece = (uint32_t)(lane + kWave * i);   // past the chunk: its first piece again
        const uint32_t off = a0[b] + (piece < (uint32_t)np[b] ? 16u * piece : 0u);
        vv[b][i] = *reinterpret_cast<const u32x4*>(vbs[b] + off);
      }
    }
    // lane (fr, fg) loads row fr's word of tiles fg, fg + 4, ... of the chunk (tile TC b + j)
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int u = fg + 4 * i, t = c0 + u % TC;
      wv[i] = 0u;
#pragma unroll
      for (int b = 0; b < R; ++b)
        if ((R == 1 || u / TC == b) && (R == 1 || live[b]) && t < kend) wv[i] = bmb[b][t * 16 + fr];
    }
    const bool past = 32 * (int64_t)c0 + 8 * PC > K && 32 * (int64_t)c0 + PC * (lane & 7) >= K;
#pragma unroll
    for (int i = 0; i < XG; ++i)
      xv[i] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, past ? kWideOob : xoff[i], 32 * XB * c0, 0));
  };

  if (kbeg < kend) {
    load_offsets();
    issue(kbeg);
  }
  if (threadIdx.x < 16)
    lut[threadIdx.x] = kQ ? u32x2{nibble_selector8(threadIdx.x), 0u}
                          : u32x2{nibble_selector16(threadIdx.x, 0), nibble_selector16(threadIdx.x, 1)};
  __syncthreads();

  uint32_t* wl = words[wave];
  unsigned char* xs = dsm + wave * wide_wave_lds<R, XG>();
  unsigned char* slot0 = xs + XG * 1024;
  const uint32_t slot_addr = lds_off(slot0);
  const uint32_t lut_addr = lds_off(lut);
  // staged row r, 16-byte piece c sits at piece c ^ (r % 8) of the row's 128 bytes
  unsigned char* xw = xs + 128 * (lane >> 3) + 16 * ((lane & 7) ^ (lane >> 3));
  const uint32_t xrd = lds_off(xs) + 128 * fr;
  const uint32_t xc[2] = {16u * (uint32_t)(fg ^ (fr & 7)), 16u * (uint32_t)((4 + fg) ^ (fr & 7))};
  Acc acc[R][MT];
#pragma unroll
  for (int b = 0; b < R; ++b)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[b][t] = Acc{0, 0, 0, 0};

  for (int c0 = kbeg; c0 < kend; c0 += TC) {
    // 1. stage the chunk (a wave's LDS operations complete in order: the previous chunk's reads are done)
#pragma unroll
    for (int i = 0; i < XG; ++i) *reinterpret_cast<u32x4*>(xw + 1024 * i) = xv[i];
#pragma unroll
    for (int b = 0; b < R; ++b) {
      unsigned char* slot = slot0 + b * kWideSlot;
      *reinterpret_cast<u32x4*>(slot + 16 * lane) = vv[b][0];
      if (np[b] > kWave && lane + kWave < np[b]) *reinterpret_cast<u32x4*>(slot + 16 * (lane + kWave)) = vv[b][1];
      if (np[b] > 2 * kWave && lane == 0)            // full tiles off a 16-byte boundary
        *reinterpret_cast<u32x4*>(slot + 32 * kWave) = *reinterpret_cast<const u32x4*>(vbs[b] + a0[b] + 32 * kWave);
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (TC * R % 4 == 0 || fg + 4 * i < TC * R) wl[fr * WS + fg + 4 * i] = wv[i];
    wave_lds_sync();
    uint32_t tile0[R][TC];                           // LDS byte of each tile's first value
#pragma unroll
    for (int b = 0; b < R; ++b)
#pragma unroll
      for (int j = 0; j < TC; ++j) tile0[b][j] = slot_addr + (uint32_t)(b * kWideSlot) + rel[b][j];

    // 2. the next chunk's loads
    const int c1 = c0 + TC;
    if (c1 < kend) {
      if (c1 - ob + TC > kWave - 1) {                // past the loaded offsets
        ob = c1;
        load_offsets();
      }
      issue(c1);
    }

    // 3. expand and multiply.  A tile's values are in lane order (16-bit: the wave's 64 lanes; int8: the 32
    // lanes of its half of the wave), so a lane's first value is the tile's + the exclusive scan of the
    // lanes' kept counts; one scan serves the chunk's two MFMA steps, in 16-bit halves
    uint32_t wj[R][2], ex[R];
#pragma unroll
    for (int b = 0; b < R; ++b) {
      if constexpr (kQ) {                            // my 16 columns of tiles fg / 2 and 2 + fg / 2
        wj[b][0] = __builtin_amdgcn_ubfe(wl[fr * WS + TC * b + (fg >> 1)], 16 * (fg & 1), 16);
        wj[b][1] = __builtin_amdgcn_ubfe(wl[fr * WS + TC * b + 2 + (fg >> 1)], 16 * (fg & 1), 16);
        const uint32_t pc = __popc(wj[b][0]) | (__popc(wj[b][1]) << 16);
        ex[b] = half_inclusive_scan(pc) - pc;
      } else {                                       // my 8 columns of both tiles
        const u32x2 wp = *reinterpret_cast<const u32x2*>(wl + fr * WS + TC * b);
        wj[b][0] = __builtin_amdgcn_ubfe(wp.x, 8 * fg, 8);
        wj[b][1] = __builtin_amdgcn_ubfe(wp.y, 8 * fg, 8);
        const uint32_t pc = __popc(wj[b][0]) | (__popc(wj[b][1]) << 16);
        ex[b] = wave_inclusive_scan(pc) - pc;
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (c0 + TC / 2 * j < kend) {
        u32x4 xb[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          // (an odd XG: the last fragment's rows 8 .. 15 repeat rows 0 .. 7 and are not stored)
          const uint32_t base = 2 * t + 1 < XG ? xrd : xrd - 128 * (fr & 8);
          xb[t] = lds_load16(base + 2048 * t + xc[j]);
        }
#pragma unroll
        for (int b = 0; b < R; ++b) {
          const uint32_t before = j ? ex[b] >> 16 : ex[b] & 0xffffu;
          u32x4 a;
          if constexpr (kQ) {
            // (an arithmetic select: a conditional one is turned into a load from private memory)
            const uint32_t t0 = tile0[b][2 * j], t1 = tile0[b][2 * j + 1];
            uint32_t p = before + t0 + ((t1 - t0) & (0u - (uint32_t)(fg >> 1)));
#pragma unroll
            for (int q = 0; q < 4; ++q) {            // a nibble's values: an aligned dword pair, realigned
              const uint32_t nib = __builtin_amdgcn_ubfe(wj[b][j], 4 * q, 4);
              const uint32_t d = p & ~3u;
              const uint32_t lo = lds_load4(d), hi = lds_load4(d + 4);
              a[q] = __builtin_amdgcn_perm(0u, __builtin_amdgcn_alignbyte(hi, lo, p), lds_load4(lut_addr + 8u * nib));
              p += __popc(nib);
            }
          } else {
            // the two nibbles' 8-byte windows: aligned dwords, realigned by their address's low 2 bits
            const uint32_t nlo = wj[b][j] & 15u, nhi = wj[b][j] >> 4;
            const uint32_t pa = 2u * before + tile0[b][j], pb = pa + 2u * __popc(nlo);
            const uint32_t da = pa & ~3u, db = pb & ~3u;
            const uint32_t a_0 = lds_load4(da), a_1 = lds_load4(da + 4), a_2 = lds_load4(da + 8);
            const uint32_t b_0 = lds_load4(db), b_1 = lds_load4(db + 4), b_2 = lds_load4(db + 8);
            const uint32_t vlo = __builtin_amdgcn_alignbyte(a_1, a_0, pa);
            const uint32_t vhi = __builtin_amdgcn_alignbyte(a_2, a_1, pa);
            const uint32_t ulo = __builtin_amdgcn_alignbyte(b_1, b_0, pb);
            const uint32_t uhi = __builtin_amdgcn_alignbyte(b_2, b_1, pb);
            const u32x2 slo = lds_load8(lut_addr + 8u * nlo), shi = lds_load8(lut_addr + 8u * nhi);
            a.x = __builtin_amdgcn_perm(vhi, vlo, slo.x);
            a.y = __builtin_amdgcn_perm(vhi, vlo, slo.y);
            a.z = __builtin_amdgcn_perm(uhi, ulo, shi.x);
            a.w = __builtin_amdgcn_perm(uhi, ulo, shi.y);
          }
#pragma unroll
          for (int t = 0; t < MT; ++t) acc[b][t] = wide_mfma<T>(a, xb[t], acc[b][t]);
        }
      }
    }
    wave_lds_sync();                                 // the next chunk overwrites the staged data
  }

  // 4. reduce, block by block (gated: the gate's sums, then the up's)
  auto* red = reinterpret_cast<typename WideAcc<T>::e*>(dsm);
  float gate[(256 * MT + W * kWave - 1) / (W * kWave)];
#pragma unroll
  for (int b = 0; b < R; ++b) {
    __syncthreads();                                 // the staged data, then the previous block's sums, are read
    const int64_t n0 = 16 * (blk0 + (kGated ? 0 : b));
    wide_sum<T, MT, W>(red, acc[b], [&](int i, int e, typename WideAcc<T>::e v) {
      if constexpr (kGated) {
        if (b == 0) {
          gate[i] = v;
          return;
        }
      }
      const int64_t n = n0 + 4 * ((e >> 6) & 3) + (e & 3);
      const int m = 16 * (e >> 8) + ((e >> 2) & 15);
      if (!live[b] || m >= M || n >= tk.N) return;
      const int64_t at = (int64_t)(m0 + m) * tk.N + n;
      if constexpr (kQ) {
        if (tk.acc) tk.acc[at] = v;
        tk.Y[at] = F16::from_f32(__fmul_rn(__fmul_rn((float)v, tk.sx[m0 + m]), tk.sw[n]));
      } else if constexpr (kGated) {
        tk.Y[at] = T::from_f32(gate[i] / (1.0f + expf(-gate[i])) * v);
      } else {
        tk.Y[at] = T::from_f32(v);
      }
    });
  }
}

template <class T, int R, int XG, int W, bool kGated>
hipError_t wide_launch(const WideGroupArg& g, hipStream_t s) {
  auto* kernel = k_sparse_wide<T, R, XG, W, kGated>;
  constexpr size_t lds = wide_lds<R, XG, W>();
  static_assert(lds + W * 16 * (4 * R + 2) * 4 + 256 <= 160 * 1024, "LDS of a CU");
  static PerDeviceFlag lds_set;
  const hipError_t attr = allow_lds_once(lds_set, kernel, lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kernel, dim3((unsigned)g.first[g.count], (unsigned)((g.M + g.rows - 1) / g.rows)),
                     dim3(W * kWave), lds, s, g);
  return hipGetLastError();
}

// Batch rows per workgroup: at most 64 (the activations of a chunk then take
// 32 registers per lane and 8 KB of LDS per wave), the batch split evenly, in
// the staged 8-row groups the kernel is built for: kMin to kMax of them.
int wide_splits(int M) { return (M + 63) / 64; }

template <class T, int R, int W, bool kGated, int kMin, int kMax>
hipError_t wide_rows(WideGroupArg& g, hipStream_t s) {
  for (int i = 0; i < g.count; ++i)
    g.first[i + 1] = g.first[i] + (int32_t)(kGated ? tile_blocks(g.t[i].N) : (tile_blocks(g.t[i].N) + R - 1) / R);
  if (kGated) g.first[g.count = 1] = (int32_t)tile_blocks(g.t[0].N);
  const int splits = wide_splits(g.M);
  g.rows = (g.M + splits - 1) / splits;
  if constexpr (kMin <= 1)
    if (g.rows <= 8) return wide_launch<T, R, 1, W, kGated>(g, s);
  if constexpr (kMin <= 2)
    if (g.rows <= 16) return wide_launch<T, R, 2, W, kGated>(g, s);
  if constexpr (kMin <= 4) {
    if (g.rows <= 24) return wide_launch<T, R, 3, W, kGated>(g, s);
    if (kMax <= 4 || g.rows <= 32) return wide_launch<T, R, 4, W, kGated>(g, s);
  }
  if constexpr (kMax >= 8) {
    if (kMin <= 6 && g.rows <= 48) return wide_launch<T, R, 6, W, kGated>(g, s);
    return wide_launch<T, R, 8, W, kGated>(g, s);
  }
  return hipErrorNotSupported;                       // not reached: the pickers keep to kMin .. kMax
}

// Row blocks (R) and waves (W) per workgroup, from the row blocks per CU
// (4096 x 4096 launches have 1, q|k|v 3, gate|up 5.4) and the rows per
// workgroup.  One workgroup of 16 waves fits a CU, so that form is for up to
// one block per CU: 288 blocks (3 x 1536 x 1536) are two rounds of it.
// Measured, us per launch at 70%, bf16 unless said:
//   up to 32 rows, one block per CU: R 1, W 16 (4096 x 4096 at 16 rows 8.3; W
//     8 9.9); below 3.5 per CU: R 1, W 8 (3 x 1536 x 1536 at 16 rows 7.0; W 16
//     8.8); above: R 2, W 8, whose activations serve two blocks (gate|up at 32
//     rows 31.5; R 1 36.6; 3 x 5120 x 5120 at 16 rows 22.1; 26.1), except up to
//     8 rows, whose activations are few: R 1, W 8 (2 x 9216 x 3072 at 8 rows
//     16.8; R 2 20.2; 2 x 13824 x 5120 33.4; 38.0);
//   more rows, R 1 workgroups (blocks times the splits of the batch) up to one
//     per CU: R 1, W 8 (4096 x 4096 at 64 rows 13.9; W 4 18.2); up to one block
//     per CU in two splits: R 1, W 8 up to 48 rows each, else R 2, W 8
//     (4096 x 11008 at 128 rows 38.9; R 1 54.4); below 3.5 per CU: R 1, W 4
//     (q|k|v at 64 rows int8 19.6; W 8 25.9; R 2 21.2); above, and for 57 to 64
//     rows of 16-bit payloads from two per CU on (q|k|v 30.1; R 1 31.8; at 49
//     30.0; 29.3): R 2, W 4, three workgroups per CU (gate|up at 65 rows 62; R 2
//     W 8 85; at 33 rows 34.8; 44.9).
template <class T>
hipError_t wide_pick(WideGroupArg& g, hipStream_t s) {
  int64_t blocks = 0;
  for (int i = 0; i < g.count; ++i) blocks += tile_blocks(g.t[i].N);
  const int64_t cus = device_cus(), splits = wide_splits(g.M);
  const int64_t rows = (g.M + splits - 1) / splits;
  if (rows <= 32) {
    if (blocks <= cus) return wide_rows<T, 1, 16, false, 1, 4>(g, s);
    if (2 * blocks < 7 * cus || (rows <= 8 && blocks < 16 * cus)) return wide_rows<T, 1, 8, false, 1, 8>(g, s);
    return wide_rows<T, 2, 8, false, 1, 8>(g, s);
  }
  if (blocks * splits <= cus || (blocks <= cus && rows <= 48)) return wide_rows<T, 1, 8, false, 1, 8>(g, s);
  if (blocks <= cus) return wide_rows<T, 2, 8, false, 1, 8>(g, s);
  const bool pair = 2 * blocks * splits >= 7 * cus || (!wide_q<T>() && rows > 56 && blocks >= 2 * cus);
  return pair ? wide_rows<T, 2, 4, false, 6, 8>(g, s) : wide_rows<T, 1, 4, false, 6, 8>(g, s);
}

// The gated half, by its pairs of row blocks: up to 32 rows W 16 up to one pair
// per CU, W 8 above (2 x 5632 x 2048, 352 pairs, at 8 rows 10.3; W 16 12.8);
// more rows: W 8 up to one workgroup per CU, W 4 above (gate|up at 33 rows
// 34.6; W 8 44.0; at 65 62.0; 83.8).
template <class T>
hipError_t wide_pick_gated(WideGroupArg& g, hipStream_t s) {
  const int64_t pairs = tile_blocks(g.t[0].N), cus = device_cus(), splits = wide_splits(g.M);
  const int64_t rows = (g.M + splits - 1) / splits;
  if (rows <= 32)
    return pairs <= cus ? wide_rows<T, 2, 16, true, 1, 4>(g, s) : wide_rows<T, 2, 8, true, 1, 8>(g, s);
  return pairs * splits <= cus ? wide_rows<T, 2, 8, true, 1, 8>(g, s) : wide_rows<T, 2, 4, true, 6, 8>(g, s);
}

WideTaskArg wide_task(const void* X, const spl_matrix& W, void* Y) {
  WideTaskArg t{};
  t.X = static_cast<const unsigned char*>(X);
  t.Y = static_cast<uint16_t*>(Y);
  t.bm = W.bitmask;
  t.values = static_cast<const unsigned char*>(W.values);
  t.toff = W.tile_offsets;
  t.N = W.rows, t.K = W.cols;
  return t;
}

}  // namespace

// The activations of a workgroup's batch rows are addressed with 32-bit byte
// offsets.
bool sparse_wide_fits(int64_t M, int64_t K, int bytes) {
  return M >= 1 && M <= kWideMaxM && bytes * (M < 64 ? M : 64) * K <= (int64_t)kWideOob;
}

hipError_t launch_sparse_wide(const spl_sparse_task* tasks, int count, int64_t M, hipStream_t s) {
  WideGroupArg g{};
  g.M = (int32_t)M;
  for (int i = 0; i < count; ++i) {
    const spl_matrix& W = *tasks[i].W;
    if (!sparse_wide_fits(M, W.cols, 2)) return hipErrorNotSupported;
    // Nothing kept: +0 above the decode kernels' 32 rows, as in the prefill kernels; up to there the product is
    // computed, as at one row (activations that are not finite give NaN).
    if (W.nnz == 0 && M > 32) {
      const hipError_t e = launch_zero_fill(tasks[i].Y, M * W.rows, s);
      if (e != hipSuccess) return e;
    } else {
      g.t[g.count++] = wide_task(tasks[i].X, W, tasks[i].Y);
    }
  }
  if (g.count == 0) return hipSuccess;
  return tasks[0].W->dtype == SPL_BF16 ? wide_pick<Bf16>(g, s) : wide_pick<F16>(g, s);
}

hipError_t launch_gated_wide(const void* X, int64_t M, const spl_matrix& Wg, const spl_matrix& Wu, void* Y,
                             hipStream_t s) {
  if (!sparse_wide_fits(M, Wg.cols, 2)) return hipErrorNotSupported;
  if (Wg.nnz == 0 || Wu.nnz == 0) return launch_zero_fill(Y, M * Wg.rows, s);   // silu(0) u = silu(g) 0 = 0
  WideGroupArg g{};
  g.count = 2;
  g.M = (int32_t)M;
  g.t[0] = wide_task(X, Wg, Y);
  g.t[1] = wide_task(X, Wu, Y);
  return Wg.dtype == SPL_BF16 ? wide_pick_gated<Bf16>(g, s) : wide_pick_gated<F16>(g, s);
}

hipError_t launch_int8_wide(const spl_int8_task* tasks, int count, int64_t M, hipStream_t s) {
  WideGroupArg g{};
  g.count = count;
  g.M = (int32_t)M;
  for (int i = 0; i < count; ++i) {
    const spl_int8_task& t = tasks[i];
    if (!sparse_wide_fits(M, t.Wq->cols, 1)) return hipErrorNotSupported;
    g.t[i] = wide_task(t.Xq, *t.Wq, t.Y);
    g.t[i].sx = t.x_scales, g.t[i].sw = t.w_scales, g.t[i].acc = t.acc_out;
  }
  return wide_pick<WideI8>(g, s);
}

}  // namespace spl
