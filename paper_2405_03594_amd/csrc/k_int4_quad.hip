// Sparse-quantized linear layer with 4-bit payloads (decode batches, M <= 16)
// for gfx950: storage, integer sums and epilogue of k_int4.hip, four tiles per
// scan.
//
// One workgroup per 16-row block, its W waves over contiguous ranges of quads
// (4 tiles, 128 columns, two MFMAs).  What bounds a launch is the expansion's
// vector instructions and, from a few batch rows on, the activations, not the
// memory:
//
//   * lane (fr, fg) owns row fr of the quad's tile fg, and MFMA h multiplies
//     column group h (16 columns) of the four tiles: one 4-step scan over the
//     tile's 16 rows, the counts of both groups in one register, gives the
//     first values of all eight operands of the quad's rows;
//   * a lane's (at most 16) codes of a group are one 12-byte load, shifted into
//     place and then by the counts of its 4-column nibbles in registers (staged
//     in LDS as in k_int8_quad.hip, the step took 6% longer);
//   * a code is used in the upper half of its byte, where it is 16 x the code
//     with no sign extension: for four columns whose codes start at bit 0 of t,
//     the bytes of {t << 4, t} hold them in their upper halves, so one
//     v_perm_b32 (selectors from a 16-entry table, zeros where the bitmask is
//     clear) and one mask make the operand.  The sums are 16 x the codes',
//     divided by 16, exactly, at the end;
//   * a load of the MFMA activation operand touches 16 rows in 16 consecutive
//     lanes, one cache access per lane (64 cycles); from kTurnMinM rows on a
//     wave loads 128-byte runs, 8 lanes per row, and turns them in its own LDS,
//     written one quad ahead (us per launch, direct / turned, at 1, 4, 8 and 16
//     rows: 4096 x 4096 5.3 / 5.5, 5.6 / 5.5, 5.8 / 5.6, 6.5 / 5.8; 11008 x 4096
//     8.6 / 8.9, 9.1 / 8.9, 9.6 / 9.0, 11.2 / 9.2);
//   * words, offsets, codes and activations are buffer loads that end at the
//     wave's range, so nothing is clamped; words and offsets are two quads
//     ahead, codes and activations one.  Direct, no load is waited for in the
//     quad that issues it; turned, the next quad's activations are, at its end,
//     where they go to LDS.
//
// Launches at 70% and cold weights, k_int4.hip's kernel / this one, at 1 and 16
// rows: 4096 x 4096 7.0 / 5.3, 7.4 / 5.8 us; 4096 x 11008 12.7 / 8.4, 13.5 / 9.4;
// 11008 x 4096 12.6 / 8.7, 13.4 / 9.2.
#include "spl_common.h"

namespace spl {
namespace {

typedef unsigned u32x3 __attribute__((ext_vector_type(3)));

constexpr int kTurnMinM = 5;

struct I4QuadArg {
  const int8_t* Xq;          // [M][K]
  const float* sx;           // [M]
  const uint32_t* bm;        // [B*S][16]
  const uint8_t* values;     // nibbles
  const int32_t* toff;       // [B*S + 1]
  const float* sw;           // [N]
  uint16_t* Y;               // [M][N] fp16
  int32_t* acc;              // optional [M][N]
  int64_t N, K;
  uint32_t vbytes;           // size of the values' buffer (16 bytes past the last at least)
  int32_t M;
};

// v_perm_b32 selector of a 4-column nibble of the bitmask: value r has its
// code in the upper half of byte 4, 0, 5 or 1 of {t << 4, t}.
__device__ __forceinline__ uint32_t i4_selector(uint32_t nib) {
  uint32_t sel = 0u;
  for (int j = 0; j < 4; ++j) {
    const uint32_t r = nibble_rank(nib, j);
    sel |= (((nib >> j) & 1u) ? (((r & 1u) ? 0u : 4u) + (r >> 1)) : 0x0Cu) << (8 * j);
  }
  return sel;
}

__device__ __forceinline__ i32x4 i4_mfma(u32x4 a, u32x4 b, i32x4 c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0,
                                               0);
}
__device__ __forceinline__ uint32_t shift64(uint32_t hi, uint32_t lo, uint32_t bits) {   // bits < 64
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> bits);
}

template <int W, bool kTurn>
__global__ void __launch_bounds__(W * kWave) k_int4_quad(const I4QuadArg tk) {
  __shared__ i32x4 part[W][64];
  __shared__ uint32_t sel4[16];
  __shared__ __align__(16) unsigned char xlds[kTurn ? W : 1][kTurn ? 2 * 2048 : 16];   // two quads: 16 rows of 128 B
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  const int64_t b = blockIdx.x;
  const int M = tk.M;
  const int S = (int)tile_steps(tk.K);
  const int Q = (S + 3) / 4;                         // quads of tiles (128 columns each)
  const int L = (Q + W - 1) / W;
  const int pb = wave * L < Q ? wave * L : Q;
  const int pe = pb + L < Q ? pb + L : Q;
  struct Meta {
    uint32_t w, base;   // my row's bitmask word of my tile, the tile's first value
  };
  struct Vals {
    uint32_t w, sh[2];  // the word; where my groups' values start in d (v_alignbit takes the low bits)
    u32x3 d[2];
  };
  // the words and tile offsets of this wave's range: what lies past reads zeros
  const auto rsrc = [](const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
  };
  const uint32_t tiles = (uint32_t)(4 * pe < S ? 4 * pe : S);
  const __amdgpu_buffer_rsrc_t bm_rsrc = rsrc(tk.bm + b * S * 16, 64u * tiles);
  const __amdgpu_buffer_rsrc_t to_rsrc = rsrc(tk.toff + b * S, 4u * tiles);
  const __amdgpu_buffer_rsrc_t x_rsrc = rsrc(tk.Xq, (uint32_t)(M * tk.K));
  const __amdgpu_buffer_rsrc_t v_rsrc = rsrc(tk.values, tk.vbytes);
  auto load_meta = [&](int p) {
    const uint32_t q = (uint32_t)p;
    return Meta{__builtin_amdgcn_raw_buffer_load_b32(bm_rsrc, 256u * q + 64u * (uint32_t)fg + 4u * (uint32_t)fr, 0, 0),
                __builtin_amdgcn_raw_buffer_load_b32(to_rsrc, 16u * q + 4u * (uint32_t)fg, 0, 0)};
  };
  // a lane with no kept value reads at its offset (at most nnz) and uses none of it
  auto load_vals = [&](const Meta& m) {
    Vals v;
    v.w = m.w;
    // kept counts of the row's two groups, 16 bits each (at most 256 over the rows); values are ordered by group,
    // then row
    const uint32_t cnt = __popc(m.w & 0xffffu) + ((uint32_t)__popc(m.w >> 16) << 16);
    const uint32_t inc = row16_inclusive_scan(cnt), ex = inc - cnt;
    const uint32_t tot = __builtin_amdgcn_update_dpp(0u, inc, 0x15F, 0xf, 0xf, false);   // row_newbcast:15
    const uint32_t off[2] = {m.base + (ex & 0xffffu), m.base + (tot & 0xffffu) + (ex >> 16)};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v.d[h] = __builtin_bit_cast(u32x3, __builtin_amdgcn_raw_buffer_load_b96(v_rsrc, (off[h] >> 1) & ~3u, 0, 0));
      v.sh[h] = off[h] << 2;
    }
    return v;
  };
  // Activations.  Columns past K meet zero weights: whatever is read there (the next row's, or zeros) adds nothing.
  // Batch rows past M, and quads past the range, read past the buffer: no fetch.
  struct Acts {
    u32x4 x[2];
  };
  constexpr uint32_t kOob = 0x80000000u;             // (the host bounds M K)
  // direct: operand h of lane (fr, fg) is 16 columns of row fr; turned: piece i of the lane is 16 columns of row
  // 8 i + lane / 8
  const int row = kTurn ? lane >> 3 : fr;
  const uint32_t xbase = kTurn ? 16u * (uint32_t)(lane & 7) : 32u * (uint32_t)fg;
  uint32_t xrow[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = kTurn ? row + 8 * i : row;
    xrow[i] = r < M ? (uint32_t)r * (uint32_t)tk.K + xbase + (kTurn ? 0u : 16u * i) : kOob;
  }
  auto load_x = [&](int p) {
    Acts a;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a.x[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             x_rsrc, p < pe ? xrow[i] + 128u * (uint32_t)p : kOob, 0, 0));
    return a;
  };
  // turned: piece c of row r lies at piece c ^ (r % 8), so that 8 rows' equal pieces are in different banks
  unsigned char* xl = xlds[kTurn ? wave : 0];
  const uint32_t xput = 16u * (uint32_t)(8 * row + ((lane & 7) ^ (row & 7)));
  const uint32_t xget = 16u * (uint32_t)(8 * fr + ((2 * fg) ^ (fr & 7)));   // operand 1: the piece's lowest bit flipped
  auto put_x = [&](const Acts& a, int buf) {
    if constexpr (kTurn) {
#pragma unroll
      for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4*>(xl + 2048 * buf + 1024 * i + xput) = a.x[i];
      wave_lds_sync();
    }
  };
  auto get_x = [&](const Acts& a, int buf) {
    if constexpr (!kTurn) return a;
    Acts o;
#pragma unroll
    for (int h = 0; h < 2; ++h) o.x[h] = *reinterpret_cast<const u32x4*>(xl + 2048 * buf + (xget ^ (16u * h)));
    wave_lds_sync();
    return o;
  };
  // the table's selectors of the word's eight nibbles: read ahead of the next quad's scan, which covers them
  struct Sel {
    uint32_t i[8], s[8];
  };
  auto load_sel = [&](uint32_t w) {
    Sel e;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      e.i[q] = (q == 0 ? w << 2 : w >> (4 * q - 2)) & 0x3Cu;
      e.s[q] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(sel4) + e.i[q]);
    }
    __builtin_amdgcn_sched_barrier(0);
    return e;
  };
  i32x4 acc[2] = {i32x4{0, 0, 0, 0}, i32x4{0, 0, 0, 0}};     // 16 x the sums
  auto mul = [&](const Vals& v, const Sel& e, const Acts& x) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t sh = v.sh[h];
      u32x4 a;
      const uint32_t lo = __builtin_amdgcn_alignbit(v.d[h][1], v.d[h][0], sh);   // codes 0 .. 7
      const uint32_t hi = __builtin_amdgcn_alignbit(v.d[h][2], v.d[h][1], sh);   // codes 8 .. 15
      uint32_t rank = 0u;                          // values before this 4-column nibble: at most 4 q
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t t = q == 0   ? lo
                           : q == 1 ? __builtin_amdgcn_alignbit(hi, lo, 4u * rank)
                                    : shift64(hi, lo, 4u * rank);
        a[q] = __builtin_amdgcn_perm(t << 4, t, e.s[4 * h + q]) & 0xF0F0F0F0u;
        rank += __popc(e.i[4 * h + q]);
      }
      acc[h] = i4_mfma(a, x.x[h], acc[h]);
    }
  };
  // two quads per iteration with the roles of the register sets swapped, so
  // that no loaded register is copied (a copy would wait for its load); a quad
  // past the range has zero words and adds nothing
  const Meta m0 = load_meta(pb);
  Meta m1 = load_meta(pb + 1);
  Acts x0 = load_x(pb);
  if (threadIdx.x < 16) sel4[threadIdx.x] = i4_selector(threadIdx.x);
  Vals v0 = load_vals(m0);
  put_x(x0, 0);
  __syncthreads();
  for (int p = pb; p < pe; p += 2) {
    const Sel e0 = load_sel(v0.w);
    const Meta m2 = load_meta(p + 2);
    const Vals v1 = load_vals(m1);
    const Acts x1 = load_x(p + 1);
    mul(v0, e0, get_x(x0, 0));
    put_x(x1, 1);
    const Sel e1 = load_sel(v1.w);
    m1 = load_meta(p + 3);
    v0 = load_vals(m2);
    x0 = load_x(p + 2);
    mul(v1, e1, get_x(x1, 1));
    put_x(x0, 0);
  }
  part[wave][lane] = (acc[0] >> 4) + (acc[1] >> 4);   // multiples of 16
  __syncthreads();
  if (wave != 0) return;
  i32x4 sum = part[0][lane];
#pragma unroll
  for (int w = 1; w < W; ++w) sum += part[w][lane];
  const int m = lane & 15;
  if (m >= M) return;
  const float xs = tk.sx[m];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t n = b * 16 + 4 * (lane >> 4) + r;
    if (n >= tk.N) continue;
    const int32_t v = sum[r];
    if (tk.acc) tk.acc[(int64_t)m * tk.N + n] = v;
    tk.Y[(int64_t)m * tk.N + n] = F16::from_f32(__fmul_rn(__fmul_rn((float)v, xs), tk.sw[n]));
  }
}

template <int W>
hipError_t i4_launch(const I4QuadArg& g, hipStream_t s) {
  const dim3 grid((unsigned)tile_blocks(g.N)), block(W * kWave);
  if (g.M >= kTurnMinM)
    hipLaunchKernelGGL((k_int4_quad<W, true>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((k_int4_quad<W, false>), grid, block, 0, s, g);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_int4_quad(const int8_t* Xq, const float* sx, int64_t M, const spl_matrix& W4, const float* sw,
                            void* Y, int32_t* acc_out, hipStream_t s) {
  const I4QuadArg g{Xq, sx, W4.bitmask, static_cast<const uint8_t*>(W4.values), W4.tile_offsets, sw,
                    static_cast<uint16_t*>(Y), acc_out, W4.rows, W4.cols,
                    (uint32_t)spl_values_bytes(W4.dtype, W4.nnz), (int32_t)M};
  return int4_quad_waves(W4.rows) == 16 ? i4_launch<16>(g, s) : i4_launch<8>(g, s);
}

}  // namespace spl
