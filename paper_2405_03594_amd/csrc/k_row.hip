// Sparse linear layer of one activation row (the decode step of one sequence,
// paper section 2.4.2) for gfx950: fp16 and bf16 payloads, groups of matrices
// in one launch, and the gated half of a Llama MLP.
//
// A workgroup owns one 16-row block (gated: of the gate matrix in its lower
// waves, of the up matrix in its upper ones); its waves split the k-steps into
// contiguous ranges of quads (4 tiles, 128 columns) and run without a barrier
// until the reduction.  As in the decode kernel the values pass through LDS
// and a wave expands them straight into MFMA operands.  What bounds a launch
// once it streams is that expansion, not the memory: counters of the decode
// kernel on gate|up (2 x 11008 x 4096 at 70%, 21.4 us, of which 66 MB take 11)
// had the vector units and the LDS each busy half of the time, 37 vector
// instructions and 38 LDS cycles per tile.  Here a tile takes 31 and 26:
//
//   * lane (fr, fg) owns row fr of the quad's tile fg instead of column group
//     fg of every tile, and MFMA step q multiplies column group q of the four
//     tiles.  A lane's bitmask word is then its own coalesced load (no
//     regrouping in LDS), and one 4-step scan of the word's four byte counts
//     gives the offsets of 16 operands (6 steps per 2 tiles before);
//   * step q needs columns of the activations in one column of the B operand
//     only.  A lane loads its 16 bytes once, lane (q, fg) those of step q, and
//     each step has an accumulator of its own, of which column q counts: no
//     activation passes through LDS, and no barrier waits for them;
//   * LDS serves 16 lanes per cycle up to 8 aligned bytes each, so a window
//     of three dwords costs three.  The third is read for no window but the
//     last of a step pair: it is used only by four values from an odd start,
//     and is then the first dword of the next window, in a register of this
//     lane or of the next row's;
//   * words, activations and values are raw buffer loads whose size ends at
//     the range, the row or the chunk: what lies past reads zeros without a
//     fetch, and no lane computes a clamped address.
//
// Measured in one stream against the decode kernel (M = 1, bf16 at 70%, cold):
// 4096 x 4096 7.9 -> 6.3 us, q|k|v 14.3 -> 12.9, gate|up 21.3 -> 19.2, gated
// 22.2 -> 18.0, 4096 x 11008 13.5 -> 11.4, 5120 x 13824 26.4 -> 19.8; at 50%
// 9.0 -> 8.1, 17.0 -> 16.0, 26.5 -> 24.3, 26.9 -> 23.9, 16.2 -> 13.8.  A 4096 x
// 4096 launch is 1.7 us of dispatch, two dependent trips to memory (offsets,
// then values) of about 1 us and the expansion of what they bring.
#include <type_traits>

#include "spl_common.h"

namespace spl {
namespace {

template <class T>
__device__ __forceinline__ f32x4 row_mfma(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (std::is_same<T, Bf16>::value)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

struct RowTaskArg {
  const uint16_t* X;
  uint16_t* Y;
  const uint32_t* bm;
  const unsigned char* values;
  const int32_t* toff;
  int64_t N, K;
};
struct RowGroupArg {
  RowTaskArg t[SPL_MAX_GROUP];        // gated: the gate and the up matrix
  int32_t first[SPL_MAX_GROUP + 1];   // first workgroup of each task; first[count] = grid size
  int32_t count;
};

// A wave's LDS: the selector table, then the chunk's values: two quads where
// they fit 256 pieces of 16 bytes (up to 50% kept), otherwise one, of at most
// 257 (full tiles off a 16-byte boundary); a window reads up to 12 bytes past.
constexpr int kRowPieces = 256;
constexpr int kRowTable = 128;
constexpr int kRowSlot = 16 * (kRowPieces + 8);
constexpr int kRowWaveLds = kRowTable + kRowSlot;
static_assert(kRowWaveLds % 128 == 0, "a table's address has no bits in common with an index into it");

// Kept counts of the word's four bytes, one byte each.
__device__ __forceinline__ uint32_t byte_counts(uint32_t w) {
  uint32_t c = w - ((w >> 1) & 0x55555555u);
  c = (c & 0x33333333u) + ((c >> 2) & 0x33333333u);
  return (c + (c >> 4)) & 0x0f0f0f0fu;
}

// Registers: 102 on 16 waves (one workgroup per CU), 80 otherwise, which
// leaves six waves per SIMD.
template <class T, int W, bool kGated>
__global__ void __launch_bounds__(W * kWave, W == 16 ? 4 : 6) k_sparse_row(const RowGroupArg g) {
  constexpr int WK = kGated ? W / 2 : W;             // waves that split a matrix's k-steps
  constexpr bool kDeep = W == 16;                    // one workgroup per CU: registers for more in flight
  constexpr int HG = kDeep ? 4 : 2;                  // column groups whose windows are in registers at a time
  extern __shared__ __align__(128) unsigned char dsm[];
  __shared__ float red[W * 16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  const int ti = kGated ? wave / WK : find_task(g.first, g.count);
  const RowTaskArg tk = g.t[ti];                     // (at most 2^31 bytes of activations: the launchers check)
  const int64_t K = tk.K;
  const int64_t blk = kGated ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - g.first[ti];
  const int S = (int)tile_steps(K);
  int kbeg, kend;                                    // this wave's k-steps: whole quads, clipped to S
  {
    const int Q = (S + 3) / 4, L = (Q + WK - 1) / WK, w = kGated ? wave % WK : wave;
    kbeg = 4 * (w * L < Q ? w * L : Q);
    kend = kbeg + 4 * L < S ? kbeg + 4 * L : S;
    if (kbeg > kend) kbeg = kend;
  }
  const int32_t* tob = tk.toff + blk * S;
  const auto rsrc = [](const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t bm_rsrc = rsrc(tk.bm + blk * S * 16, 64u * (uint32_t)kend);   // past the range: zeros
  const __amdgpu_buffer_rsrc_t x_rsrc = rsrc(tk.X, (uint32_t)(2 * K));                       // columns past K too

  u32x2* lut = reinterpret_cast<u32x2*>(dsm + wave * kRowWaveLds);
  unsigned char* slot = dsm + wave * kRowWaveLds + kRowTable;

  // Offsets of the wave's tiles: lane i holds that of tile ob + i (clamped to the range end)
  int ob = kbeg;
  int32_t orng = 0;
  auto load_offsets = [&]() { orng = tob[ob + lane < kend ? ob + lane : kend]; };
  // the chunk in flight: lane (fr, fg) holds the words of row fr, tiles fg and 4 + fg; lane (q, fg) (q < 4) the
  // activations of their column group q
  u32x4 vv[4], xv[2];
  uint32_t wv[2], a0 = 0;                            // a0: first value byte loaded (16-byte aligned)
  int np = 0;                                        // 16-byte pieces
  bool two = false;                                  // two quads
  const uint32_t xlane = fr < 4 ? 64u * (uint32_t)fg + 16u * (uint32_t)fr : 0x80000000u;
  auto load_x = [&](u32x4 (&x)[2], int c0) {
    const uint32_t xo = xlane + 64u * (uint32_t)c0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      x[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, xo + 256u * i, 0, 0));
  };
  auto issue_words = [&](int c0) {
    const uint32_t wo = 64u * (uint32_t)c0 + 4u * (uint32_t)lane;
#pragma unroll
    for (int i = 0; i < 2; ++i) wv[i] = __builtin_amdgcn_raw_buffer_load_b32(bm_rsrc, wo + 256u * i, 0, 0);
    if constexpr (kDeep) load_x(xv, c0);
  };
  auto issue_values = [&](int c0) {
    const int r = c0 - ob;
    const uint32_t o0 = (uint32_t)__builtin_amdgcn_readlane(orng, r);
    const uint32_t o4 = (uint32_t)__builtin_amdgcn_readlane(orng, r + 4);
    const uint32_t o8 = (uint32_t)__builtin_amdgcn_readlane(orng, r + 8);
    a0 = (2u * o0) & ~15u;
    const uint32_t n8 = (2u * o8 - a0 + 15u) >> 4;
    two = c0 + 4 < kend && n8 <= (uint32_t)kRowPieces;   // (a quad past the range has activations, and 0 x inf)
    np = (int)(two ? n8 : (2u * o4 - a0 + 15u) >> 4);
    const __amdgpu_buffer_rsrc_t v_rsrc = rsrc(tk.values + a0, 16u * (uint32_t)np);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i == 0 || np > kWave * i)                  // wave-uniform
        vv[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, 16 * lane + 1024 * i, 0, 0));
  };

  if (kbeg < kend) {
    load_offsets();
    issue_words(kbeg);
    issue_values(kbeg);
  }
  if (lane < 16) lut[lane] = u32x2{nibble_selector16(lane, 0), nibble_selector16(lane, 1)};
  const uint32_t slot_addr = lds_off(slot);
  const uint32_t lut_addr = lds_off(lut);            // a multiple of 128
  // operands kept in registers, so that an index takes one v_and_or_b32 and a count one v_bcnt_u32_b32
  uint32_t m78 = 0x78u, lut_v = lut_addr, nlut = 0u - (uint32_t)__popc(lut_addr);
  asm("" : "+s"(m78));
  asm("" : "+v"(lut_v));
  asm("" : "+v"(nlut));
  f32x4 acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int c0 = kbeg; c0 < kend;) {
    // 1. stage the chunk's values (a wave's LDS operations complete in order: the previous chunk's reads are done)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i == 0 || np > kWave * i) *reinterpret_cast<u32x4*>(slot + 16 * (lane + kWave * i)) = vv[i];
    if (np > kRowPieces && lane == 0)                // a full quad off a 16-byte boundary
      *reinterpret_cast<u32x4*>(slot + 16 * kRowPieces) =
          *reinterpret_cast<const u32x4*>(tk.values + a0 + (size_t)(16 * kRowPieces));
    wave_lds_sync();
    // its words, activations and the LDS byte of each lane's tile; then the next chunk's loads
    const bool both = two;
    uint32_t w[2], vb[2];
    u32x4 xb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      w[i] = wv[i];
      if constexpr (kDeep) xb[i] = xv[i];
      const uint32_t o = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (c0 - ob + 4 * i + fg), orng);
      vb[i] = 2u * o + (slot_addr - a0);
    }
    if constexpr (!kDeep) load_x(xb, c0);
    const int c1 = c0 + (both ? 8 : 4);
    if (c1 < kend) {
      if (c1 - ob + 8 > kWave - 1) {
        ob = c1;
        load_offsets();
      }
      issue_words(c1);
      issue_values(c1);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (i == 1 && !both) break;
      // 2. a tile's values are ordered by column group, then row: one scan over the 16 rows for the four groups,
      // a byte each (at most 128), and the groups' totals
      const uint32_t cnt = byte_counts(w[i]);
      const uint32_t inc = row16_inclusive_scan(cnt);
      const uint32_t ex2 = (inc - cnt) << 1;         // bytes before my row: at most 240 per group
      const uint32_t tot = __builtin_amdgcn_update_dpp(0u, inc, 0x15F, 0xf, 0xf, false);   // row_newbcast:15
      uint32_t base = vb[i];
#pragma unroll
      for (int h = 0; h < 4 / HG; ++h) {
        uint32_t pa[HG], pb[HG], a_0[HG], a_1[HG], b_0[HG], b_1[HG];
        u32x2 sl[HG], sh[HG];
#pragma unroll
        for (int e = 0; e < HG; ++e) {
          const int q = HG * h + e;
          pa[e] = __builtin_amdgcn_ubfe(ex2, 8 * q, 8) + base;
          if (q < 3) base += 2u * __builtin_amdgcn_ubfe(tot, 8 * q, 8);
          const uint32_t slo = ((q == 0 ? w[i] << 3 : w[i] >> (8 * q - 3)) & m78) | lut_v;
          const uint32_t shi = ((w[i] >> (8 * q + 1)) & m78) | lut_v;
          pb[e] = pa[e] + 2u * (__popc(slo) + nlut);
          const uint32_t da = pa[e] & ~3u, db = pb[e] & ~3u;
          a_0[e] = lds_load4(da), a_1[e] = lds_load4(da + 4);
          b_0[e] = lds_load4(db), b_1[e] = lds_load4(db + 4);
          sl[e] = lds_load8(slo), sh[e] = lds_load8(shi);
        }
        // The third dword of a window is used only by four values from an odd start, and then the next window
        // starts there: the upper nibble's, for the upper one itself the next row's (from row 15 the next
        // column group's).
        const uint32_t last = lds_load4((pb[HG - 1] & ~3u) + 8);
#pragma unroll
        for (int e = 0; e < HG; ++e) {
          uint32_t b_2 = last;
          if (e + 1 < HG) {
            const uint32_t nx = __builtin_amdgcn_update_dpp(0u, a_0[e + 1 < HG ? e + 1 : e], 0x150, 0xf, 0xf, false);   // row_newbcast:0
            b_2 = __builtin_amdgcn_update_dpp(nx, a_0[e], 0x101, 0xf, 0xf, false);                 // row_shl:1
          }
          const uint32_t vlo = __builtin_amdgcn_alignbyte(a_1[e], a_0[e], pa[e]);
          const uint32_t vhi = __builtin_amdgcn_alignbyte(b_0[e], a_1[e], pa[e]);
          const uint32_t ulo = __builtin_amdgcn_alignbyte(b_1[e], b_0[e], pb[e]);
          const uint32_t uhi = __builtin_amdgcn_alignbyte(b_2, b_1[e], pb[e]);
          const u32x4 a = u32x4{__builtin_amdgcn_perm(vhi, vlo, sl[e].x), __builtin_amdgcn_perm(vhi, vlo, sl[e].y),
                                __builtin_amdgcn_perm(uhi, ulo, sh[e].x), __builtin_amdgcn_perm(uhi, ulo, sh[e].y)};
          acc[HG * h + e] = row_mfma<T>(a, xb[i], acc[HG * h + e]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);             // one quad's windows in registers at a time
    }
    wave_lds_sync();                                 // the next chunk overwrites the staged data
    c0 = c1;
  }

  // column q of accumulator q holds the wave's sums of rows 4 fg .. 4 fg + 3 over column group q
  f32x4 r = fr == 0 ? acc[0] : fr == 1 ? acc[1] : fr == 2 ? acc[2] : acc[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    r[e] += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(r[e]), 0xB1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
    r[e] += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(r[e]), 0x4E, 0xf, 0xf, false));   // quad_perm 2,3,0,1
  }
  if (fr == 0) *reinterpret_cast<f32x4*>(red + wave * 16 + 4 * fg) = r;
  __syncthreads();
  if (threadIdx.x >= 16) return;
  const int64_t n = blk * 16 + threadIdx.x;
  float s = 0.f, u = 0.f;
#pragma unroll
  for (int v = 0; v < WK; ++v) s += red[16 * v + threadIdx.x];
  if constexpr (kGated) {
#pragma unroll
    for (int v = 0; v < WK; ++v) u += red[16 * (WK + v) + threadIdx.x];
    s = s / (1.0f + expf(-s)) * u;
  }
  if (n < tk.N) tk.Y[n] = T::from_f32(s);
}

template <class T, int W, bool kGated>
hipError_t row_launch(const RowGroupArg& g, hipStream_t s) {
  auto* kernel = k_sparse_row<T, W, kGated>;
  constexpr size_t lds = (size_t)W * kRowWaveLds;
  static PerDeviceFlag lds_set;
  const hipError_t attr = allow_lds_once(lds_set, kernel, lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kernel, dim3((unsigned)g.first[g.count]), dim3(W * kWave), lds, s, g);
  return hipGetLastError();
}

// Waves per workgroup.  A CU holds one workgroup of 16 waves, three of 8 or six
// of 4 (80 registers).  Measured (us at 16 / 8 / 4 waves, bf16 at 70%): up to
// one row block per CU 16 (4096 x 4096 6.3 / 7.2 / 9.1, 4096 x 11008 11.5 /
// 14.9 / 19.2); up to three 8 (5120 x 5120, 1.25 per CU, 13.1 / 10.7 / 11.7;
// q|k|v, three, 15.4 / 12.9 / 13.2); past them, where 8 waves would take a
// second round, 4 (2 x 6208 x 4096, 3.03 per CU, 8 / 4 waves 14.2 / 13.8, at
// 50% 18.2 / 17.4; 3 x 5120 x 5120 18.2 / 17.4, 24.2 / 22.8; gate|up, 5.4, 19.5 /
// 18.8; 2 x 12288 x 4096, six, 20.0 / 19.2, 28.3 / 25.3), but 8 where those are
// three rounds and 4 waves two of six, if the rounds are long (2 x 13824 x
// 5120, 6.75 per CU, 27.2 / 28.2, 37.2 / 39.6; with 4096 columns 22.4 / 23.3,
// 31.2 / 32.8; with 2048 13.9 / 14.1, and at eight per CU 15.8 / 15.4; nine per
// CU with 4096 27.1 / 27.6, 38.3 / 38.1).  The gated pair, whose waves split
// twice the matrices, keeps 8 (21.3 / 18.0 / 20.2).
template <class T, bool kGated>
hipError_t row_pick(const RowGroupArg& g, hipStream_t s) {
  const int64_t blocks = g.first[g.count], cus = device_cus();
  if (blocks <= cus) return row_launch<T, 16, kGated>(g, s);
  int64_t kmax = 0;
  for (int i = 0; i < g.count; ++i) kmax = g.t[i].K > kmax ? g.t[i].K : kmax;
  const bool third = blocks > 6 * cus && blocks < 9 * cus && kmax >= 4096;
  return blocks <= 3 * cus || third || kGated ? row_launch<T, 8, kGated>(g, s) : row_launch<T, 4, kGated>(g, s);
}

// A row's activations, and a row block's words, are addressed with 32-bit byte offsets.
constexpr int64_t kRowMaxK = (int64_t)1 << 30;

RowTaskArg row_task(const void* X, const spl_matrix& W, void* Y) {
  return RowTaskArg{static_cast<const uint16_t*>(X), static_cast<uint16_t*>(Y),   W.bitmask,
                    static_cast<const unsigned char*>(W.values), W.tile_offsets, W.rows, W.cols};
}

}  // namespace

hipError_t launch_sparse_row(const spl_sparse_task* tasks, int count, hipStream_t s) {
  RowGroupArg g{};
  g.count = count;
  for (int i = 0; i < count; ++i) {
    if (tasks[i].W->cols > kRowMaxK) return hipErrorNotSupported;
    g.t[i] = row_task(tasks[i].X, *tasks[i].W, tasks[i].Y);
    g.first[i + 1] = g.first[i] + (int32_t)tile_blocks(tasks[i].W->rows);
  }
  return tasks[0].W->dtype == SPL_BF16 ? row_pick<Bf16, false>(g, s) : row_pick<F16, false>(g, s);
}

hipError_t launch_gated_row(const void* X, const spl_matrix& Wg, const spl_matrix& Wu, void* Y, hipStream_t s) {
  if (Wg.cols > kRowMaxK) return hipErrorNotSupported;
  if (Wg.nnz == 0 || Wu.nnz == 0) return launch_zero_fill(Y, Wg.rows, s);   // silu(0) u = silu(g) 0 = 0
  RowGroupArg g{};
  g.t[0] = row_task(X, Wg, Y);
  g.t[1] = row_task(X, Wu, Y);
  g.count = 1;
  g.first[1] = (int32_t)tile_blocks(Wg.rows);
  return Wg.dtype == SPL_BF16 ? row_pick<Bf16, true>(g, s) : row_pick<F16, true>(g, s);
}

}  // namespace spl
