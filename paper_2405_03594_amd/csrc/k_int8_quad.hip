// Sparse-quantized linear layers in int8 (groups, decode batches, M <= 16) for
// gfx950: storage, integer sums and epilogue of k_int8.hip, four tiles per scan.
//
// One workgroup per 16-row block, its W waves over contiguous ranges of quads
// (4 tiles, 128 columns, two MFMAs):
//
//   * lane (fr, fg) owns row fr of the quad's tile fg, and MFMA h multiplies
//     column group h (16 columns) of the four tiles: one 4-step scan over the
//     tile's 16 rows, the counts of both groups in one register, gives the
//     first values of all eight operands of the quad's rows (k_wide.hip takes
//     a 5-step scan per two tiles);
//   * a wave loads a quad's values in 16-byte pieces and stages them in its own
//     LDS (loads at the lanes' own starts, 20 bytes per group, take 64 cycles
//     of the cache's address path each: four layers' step of one row 252 us
//     instead of 236); a lane's (at most 16) values of a group are five dwords
//     there, shifted into place and then by the counts of its 4-column nibbles
//     in registers, where a window per nibble reads eight;
//   * one v_perm_b32 per nibble (selectors from a 16-entry table, zeros where
//     the bitmask is clear) makes the operand;
//   * activations are loaded as the MFMA takes them, one quad ahead (turned in
//     LDS from 128-byte runs the step took 274 us instead of 269 at 16 rows,
//     270 instead of 247 at 8: another round trip before each product);
//   * words, offsets, values and activations are buffer loads that end at the
//     wave's range, so nothing is clamped; words and offsets are two quads
//     ahead, values and activations one.
//
// Four layers' step (hidden 4096, ffn 11008, 70%) with the kernel before, two
// tiles per scan, / this one: 236 / 221 us at one row, 288 / 229 at 8.
#include "spl_common.h"

namespace spl {
namespace {

struct I8QuadTaskArg {
  const int8_t* Xq;          // [M][K]
  const float* sx;           // [M]
  const uint32_t* bm;        // [B*S][16]
  const uint8_t* values;
  const int32_t* toff;       // [B*S + 1]
  const float* sw;           // [N]
  uint16_t* Y;               // [M][N] fp16
  int32_t* acc;              // optional [M][N]
  int64_t N, K;
};
struct I8QuadGroupArg {
  I8QuadTaskArg t[SPL_MAX_GROUP];
  int32_t first[SPL_MAX_GROUP + 1];   // first workgroup of each task; first[count] = grid size
  int32_t count;
  int32_t M;
};

// v_perm_b32 selector of a 4-column nibble of the bitmask: value r is byte r.
__device__ __forceinline__ uint32_t i8q_selector(uint32_t nib) {
  uint32_t sel = 0u;
  for (int j = 0; j < 4; ++j) {
    const uint32_t r = nibble_rank(nib, j);
    sel |= (((nib >> j) & 1u) ? r : 0x0Cu) << (8 * j);
  }
  return sel;
}

__device__ __forceinline__ i32x4 i8q_mfma(u32x4 a, u32x4 b, i32x4 c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0,
                                               0);
}
__device__ __forceinline__ uint32_t shift64(uint32_t hi, uint32_t lo, uint32_t bits) {   // bits < 64
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> bits);
}

// One task: its arguments are loaded without a search for it first.  The
// launch bound leaves three 8-wave workgroups per CU (81 registers otherwise,
// two: 11008 x 4096 at one row 12.2 us instead of 8.9).
template <int W, bool kGroup>
__global__ void __launch_bounds__(W * kWave, W == 8 ? 6 : 1) k_int8_quad(const I8QuadGroupArg g) {
  __shared__ i32x4 part[W][64];
  __shared__ uint32_t sel4[16];
  // a quad's values from a 16-byte boundary (full tiles: kPieces pieces and one more; a lane reads at most 16 bytes
  // past them)
  constexpr int kPieces = 128;                       // 2048 values
  constexpr int kLoads = kPieces / kWave;
  __shared__ __align__(16) unsigned char stage[W][16 * (kPieces + 2)];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  const int ti = kGroup ? find_task(g.first, g.count) : 0;
  const I8QuadTaskArg tk = g.t[ti];
  const int64_t b = (int64_t)blockIdx.x - (kGroup ? g.first[ti] : 0);
  const int M = g.M;
  const int S = (int)tile_steps(tk.K);
  const int Q = (S + 3) / 4;                         // quads of tiles (128 columns each)
  const int L = (Q + W - 1) / W;
  const int pb = wave * L < Q ? wave * L : Q;
  const int pe = pb + L < Q ? pb + L : Q;
  struct Meta {
    uint32_t w, base;   // my row's bitmask word of my tile, the tile's first value
  };
  struct Vals {
    uint32_t w;         // the word
    uint32_t at[2];     // my groups' first values, from the stage's start
    u32x4 d[kLoads];    // the quad's values: pieces lane, 64 + lane
    uint32_t a0;        // their first byte; np: how many (wave-uniform)
    int np;
  };
  // the words and tile offsets of this wave's range: what lies past reads zeros
  const auto rsrc = [](const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
  };
  const uint32_t tiles = (uint32_t)(4 * pe < S ? 4 * pe : S);
  const __amdgpu_buffer_rsrc_t bm_rsrc = rsrc(tk.bm + b * S * 16, 64u * tiles);
  const __amdgpu_buffer_rsrc_t to_rsrc = rsrc(tk.toff + b * S, 4u * tiles);
  const __amdgpu_buffer_rsrc_t x_rsrc = rsrc(tk.Xq, (uint32_t)(M * tk.K));
  auto load_meta = [&](int p) {
    const uint32_t q = (uint32_t)p;
    return Meta{__builtin_amdgcn_raw_buffer_load_b32(bm_rsrc, 256u * q + 64u * (uint32_t)fg + 4u * (uint32_t)fr, 0, 0),
                __builtin_amdgcn_raw_buffer_load_b32(to_rsrc, 16u * q + 4u * (uint32_t)fg, 0, 0)};
  };
  auto load_vals = [&](const Meta& m, int p) {
    Vals v;
    v.w = m.w;
    // kept counts of the row's two groups, 16 bits each (at most 256 over the rows); values are ordered by group,
    // then row
    const uint32_t cnt = __popc(m.w & 0xffffu) + ((uint32_t)__popc(m.w >> 16) << 16);
    const uint32_t inc = row16_inclusive_scan(cnt), ex = inc - cnt;
    const uint32_t tot = __builtin_amdgcn_update_dpp(0u, inc, 0x15F, 0xf, 0xf, false);   // row_newbcast:15
    // the quad's values: from its first tile's to the end of its last one below S
    const int left = S - 4 * p;                      // tiles (none past the range: words, offsets are zeros there)
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane(m.base);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readlane(m.base + (tot & 0xffffu) + (tot >> 16),
                                                             left >= 4 ? 63 : (left > 0 ? 16 * left - 1 : 0));
    v.a0 = first & ~15u;
    v.np = (int)((end - v.a0 + 15u) >> 4);
    const __amdgpu_buffer_rsrc_t v_rsrc = rsrc(tk.values + v.a0, 16u * (uint32_t)v.np);
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      if (i == 0 || v.np > kWave * i)                // wave-uniform
        v.d[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, 16 * lane + 1024 * i, 0, 0));
    const int32_t rel = (int32_t)(m.base - v.a0);   // negative: a tile past S, which uses no value
    const uint32_t base = rel < 0 ? 0u : (uint32_t)rel;
    v.at[0] = base + (ex & 0xffffu);
    v.at[1] = base + (tot & 0xffffu) + (ex >> 16);
    return v;
  };
  // Activations.  Columns past K meet zero weights: whatever is read there (the next row's, or zeros) adds nothing.
  // Batch rows past M, and quads past the range, read past the buffer: no fetch.
  struct Acts {
    u32x4 x[2];
  };
  constexpr uint32_t kOob = 0x80000000u;             // (the host bounds M K)
  // operand h of lane (fr, fg) is 16 columns of row fr
  const uint32_t xrow = fr < M ? (uint32_t)fr * (uint32_t)tk.K + 32u * (uint32_t)fg : kOob;
  auto load_x = [&](int p) {
    Acts a;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a.x[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             x_rsrc, (p < pe ? xrow + 128u * (uint32_t)p : kOob) + 16u * i, 0, 0));
    return a;
  };
  unsigned char* vl = stage[wave];
  const uint32_t vl_addr = lds_off(vl);
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
  // one quad at a time: its loads, one quad old, go to LDS, and the loads of the next are issued before it is expanded
  i32x4 acc[2] = {i32x4{0, 0, 0, 0}, i32x4{0, 0, 0, 0}};
  const Meta m0 = load_meta(pb);
  Meta mn = load_meta(pb + 1);
  Acts xn = load_x(pb);
  if (threadIdx.x < 16) sel4[threadIdx.x] = i8q_selector(threadIdx.x);
  Vals v = load_vals(m0, pb);
  __syncthreads();
  for (int p = pb; p < pe; ++p) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      if (i == 0 || v.np > kWave * i) *reinterpret_cast<u32x4*>(vl + 16 * lane + 1024 * i) = v.d[i];
    if (v.np > kPieces && lane == 0)                 // a full quad off a 16-byte boundary
      *reinterpret_cast<u32x4*>(vl + 16 * kPieces) =
          *reinterpret_cast<const u32x4*>(tk.values + (size_t)v.a0 + (size_t)(16 * kPieces));
    wave_lds_sync();
    uint32_t d[2][5], sh[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t at = vl_addr + (v.at[h] & ~3u);
#pragma unroll
      for (int k = 0; k < 5; ++k) d[h][k] = lds_load4(at + 4 * k);
      sh[h] = v.at[h];                               // v_alignbyte takes the low bits
    }
    const Acts x = xn;
    const Sel e = load_sel(v.w);                     // (and no later load of this quad before these)
    v = load_vals(mn, p + 1);
    mn = load_meta(p + 2);
    xn = load_x(p + 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 a;
      uint32_t s[4];                                 // bytes 0 .. 15
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = __builtin_amdgcn_alignbyte(d[h][k + 1], d[h][k], sh[h]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {                  // s[0]: the nibble's values; then past its (at most 4) bytes
        a[q] = __builtin_amdgcn_perm(0u, s[0], e.s[4 * h + q]);
        const uint32_t past = 8u * (uint32_t)__popc(e.i[4 * h + q]);
#pragma unroll
        for (int k = 0; k + q < 3; ++k) s[k] = shift64(s[k + 1], s[k], past);
      }
      acc[h] = i8q_mfma(a, x.x[h], acc[h]);
    }
    wave_lds_sync();                                 // the next quad overwrites the stage
  }
  part[wave][lane] = acc[0] + acc[1];
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
hipError_t i8q_launch(const I8QuadGroupArg& g, hipStream_t s) {
  auto* kernel = g.count > 1 ? k_int8_quad<W, true> : k_int8_quad<W, false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)g.first[g.count]), dim3(W * kWave), 0, s, g);
  return hipGetLastError();
}

void i8q_add(I8QuadGroupArg& g, const int8_t* Xq, const float* sx, const spl_matrix& W, const float* sw, void* Y,
              int32_t* acc) {
  const int i = g.count++;
  g.t[i] = I8QuadTaskArg{Xq, sx, W.bitmask, static_cast<const uint8_t*>(W.values), W.tile_offsets, sw,
                         static_cast<uint16_t*>(Y), acc, W.rows, W.cols};
  g.first[i + 1] = g.first[i] + (int32_t)tile_blocks(W.rows);
}

}  // namespace

hipError_t launch_int8_quad(const spl_int8_task* tasks, int count, int64_t M, hipStream_t s) {
  I8QuadGroupArg g{};
  g.M = (int32_t)M;
  for (int i = 0; i < count; ++i)
    i8q_add(g, tasks[i].Xq, tasks[i].x_scales, *tasks[i].Wq, tasks[i].w_scales, tasks[i].Y, tasks[i].acc_out);
  // Waves per row block, us per launch at 70%, 8 rows.  Up to one block per CU, where each wave has a quad, 16: 4096 x
  // 4096 6.0, with 8 6.8; 4096 x 11008 9.8, 12.4; but 2 x 2048 x 768 (6 quads) 4.5, 4.2.  Above, 16 waves are one
  // workgroup per CU, so two rounds below two blocks per CU: 3 x 1536 x 1536 (288 blocks) 7.4, with 8 5.8.  Past
  // three per CU, which are all that it holds of 8 waves, 4, six of which fit: 2 x 6208 x 4096 (3.03) at 1 and 16 rows
  // 11.6, 13.5, with 8 12.6, 15.4; gate|up (5.4) 15.1, 19.4; 2 x 13824 x 5120 (6.75) at one row 23.4, 24.4; q|k|v
  // (3) 11.5, 9.9.
  int64_t kmax = 0;
  for (int i = 0; i < count; ++i) kmax = tasks[i].Wq->cols > kmax ? tasks[i].Wq->cols : kmax;
  const int64_t blocks = g.first[g.count], cus = device_cus();
  if (blocks <= cus && kmax >= 16 * 128) return i8q_launch<16>(g, s);
  return blocks <= 3 * cus ? i8q_launch<8>(g, s) : i8q_launch<4>(g, s);
}

}  // namespace spl
