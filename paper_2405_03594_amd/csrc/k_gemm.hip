// Prefill-sized sparse products through a decoded copy of the weights in
// matrix-core operand order, for gfx950.
//
// The tiled kernels expand every W tile once per workgroup column of the
// batch, on the same waves that issue the MFMAs, and read both operands from
// LDS.  Where the caller lends scratch memory, the tiles are instead decoded
// once (paper section 2.4.2 decompresses the stored submatrices before the
// matrix units consume them) into *fragments*: 1 KB per 16 x 32 tile (int8:
// per 16 x 64 pair of tiles), lane l's 16 operand bytes at 16 l, a row
// block's fragments consecutive.  The product kernel then needs no LDS for W:
// a wave loads its A operand with one coalesced 1 KB request per fragment,
// straight into registers.
//
// k_frag_gemm: NWN x NWM waves of 16 FN x 16 FM outputs.  K advances by stages
// of 128 bytes of an activation row (two MFMA k-steps).  Activations go from
// global memory straight into LDS, a ring of four stage buffers of 128-byte
// rows whose 16-byte piece c sits at c ^ (row % 8); fragments go into two
// register sets.  Each stage has two halves, one per k-step; a half multiplies
// its k-step while the other k-step's activation operands are read from LDS
// and the requests of later stages are issued, one request or LDS read in
// front of every FN MFMAs.  The one barrier per stage sits between the halves,
// so no wave starts a stage by waiting for LDS: at it a wave has waited for
// its own requests of stage st + 1 (counted: the later ones stay in flight),
// and after it the buffer of stage st - 1 is refilled.  Stages past the last,
// which fill the loop's last iteration, read through empty buffer descriptors
// (zeros).  The loop holds nothing but MFMAs, LDS reads, requests and their
// scalar addresses: with per-lane bounds selects in it the compiler also moved
// accumulators between registers every iteration (4096 x 4096 x 2048 tokens:
// 74.5 us; without 59.6).
//
// Measured on one Llama-2-7B layer, bf16, 70%, cold weights, against the tiled
// kernels that expand in place: 2048 tokens q|k|v 275 -> 39 + 183 us (decoding +
// product, 1126 TFLOP/s), o 87 -> 15 + 69, gated gate|up 530 -> 67 + 350 (1055),
// down 231 -> 36 + 172 (1074), so 157 us of a layer are decoding, in int8 90;
// 397 tokens, both together: q|k|v 130 -> 89, o 44 -> 37, gate|up 182 -> 150,
// down 109 -> 87.
#include <type_traits>

#include "spl_common.h"

namespace spl {
namespace {

struct FgI8 {};                  // int8 weights and activations, exact int32 sums

template <class T>
constexpr bool fg_q() { return std::is_same<T, FgI8>::value; }
// (int8 sums are held as the bits of f32x4)
template <class T>
__device__ __forceinline__ f32x4 fg_mfma(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (fg_q<T>())
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a),
                                                                           __builtin_bit_cast(i32x4, b),
                                                                           __builtin_bit_cast(i32x4, c), 0, 0, 0));
  else if constexpr (std::is_same<T, Bf16>::value)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

// Fragments per row block of a matrix of K columns: 16 rows x 64 bytes of a
// row each (32 columns of 16-bit payloads, 64 of int8), an even number.
template <bool kQ>
__host__ __device__ constexpr int64_t fg_steps(int64_t K) { return kQ ? 2 * ((K + 127) / 128) : 2 * ((K + 63) / 64); }

struct FgTask {
  const unsigned char* X;        // [M][K] activations
  const unsigned char* A;        // fragments [B][fg_steps][1024]
  const unsigned char* A2;       // gated: the up matrix (A is the gate)
  uint16_t* Y;                   // [M][N]
  int64_t N, K;
  int32_t tn;                    // n-blocks
  const float* sx;               // int8: activation scales [M], weight scales [N], optional sums [M][N]
  const float* sw;
  int32_t* acc;
};
struct FgGroupArg {
  FgTask t[SPL_MAX_GROUP];
  int32_t first[SPL_MAX_GROUP + 1];
  int32_t count;
  int32_t M;
};

constexpr uint32_t kFgOob = 0x80000000u;

// 16 bytes per lane from a buffer straight into LDS: lane l fills dst + 16 l (zeros for an offset past the buffer)
__device__ __forceinline__ void fg_dma16(__amdgpu_buffer_rsrc_t src, unsigned char* dst, uint32_t voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

template <int N>
__device__ __forceinline__ void fg_wait_vm() {   // at most N of this wave's vector-memory requests remain
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void fg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

enum { kFgPlain = 0, kFgGated = 1 };

// Waves per SIMD that the registers are held to: one for a 128 x 256 tile on four waves (128 accumulators), else
// two, which is what the stage ring leaves LDS for.
constexpr int fg_waves(int FN, int FM) { return FN * FM > 16 ? 1 : 2; }

// kRagged: rows of X are not whole stages; their missing columns read zeros.
template <class T, int FN, int FM, int NWN, int NWM, int kMode, bool kRagged>
__global__ void __launch_bounds__(64 * NWN * NWM, fg_waves(FN, FM)) k_frag_gemm(const FgGroupArg ga) {
  constexpr bool kQ = fg_q<T>();
  constexpr int BM = 16 * FM * NWM;                  // NWN x NWM waves of 16 FN x 16 FM
  constexpr int XS = BM * 128;                       // bytes of a staged activation stage
  constexpr int XG = BM / 8 / (NWN * NWM);                        // 8-row groups (1 KB requests) per wave and stage
  extern __shared__ __align__(16) unsigned char dsm[];
  const int ti = find_task(ga.first, ga.count);
  const FgTask g = ga.t[ti];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int wn = wave % NWN, wm = wave / NWN;
  const int fr = lane & 15, fg = lane >> 4;
  const int64_t N = g.N, K = g.K;
  const int SP = (int)fg_steps<kQ>(K), nst = SP / 2;
  const int B = (int)tile_blocks(N);
  // workgroup order: the XCDs (blockIdx % 8) take contiguous runs of tiles, four m-blocks to a column of n-blocks
  int bn, bm;
  {
    const int M4 = 4;
    const int tm = (ga.M + BM - 1) / BM, tn = g.tn, total = tm * tn;
    const int w = (int)blockIdx.x - ga.first[ti];
    const int q = total / 8, r = total % 8, x = w % 8, i = w / 8;
    const int t = x * q + (x < r ? x : r) + i;
    const int gsz = M4 * tn, grp = t / gsz, h = tm - grp * M4 < M4 ? tm - grp * M4 : M4, in = t - grp * gsz;
    bm = grp * M4 + in % h;
    bn = in / h;
  }
  const int64_t m0 = (int64_t)bm * BM;
  const int M = (int)(ga.M - m0 < BM ? ga.M - m0 : BM);

  const int abytes = (int)((int64_t)B * SP * 1024);
  const unsigned char* ab[2] = {g.A, kMode == kFgGated ? g.A2 : g.A};
  uint32_t aoff[FN];
#pragma unroll
  for (int i = 0; i < FN; ++i) {
    int rb = kMode == kFgGated ? (FN / 2) * (NWN * bn + wn) + i / 2 : FN * (NWN * bn + wn) + i;
    if (rb >= B) rb = B - 1;                         // its results are not stored
    aoff[i] = (uint32_t)rb * (uint32_t)SP * 1024u + 16u * (uint32_t)lane;
  }
  constexpr int XB = kQ ? 1 : 2;
  const int64_t Kb = XB * K;                         // bytes of an activation row
  const uint32_t xp = 16u * (uint32_t)((lane & 7) ^ (lane >> 3));   // my piece of a row's 128 bytes
  uint32_t xoff[XG];
#pragma unroll
  for (int i = 0; i < XG; ++i) {
    const int row = 8 * (XG * wave + i) + (lane >> 3);
    xoff[i] = row < M ? (uint32_t)row * (uint32_t)Kb + xp : kFgOob;
  }
  u32x4 a[2][2][FN], b[2][FM];
  // a stage past the last reads zeros: its descriptors are empty
  auto load_a = [&](u32x4 (&d)[FN], int i, int st, int ks) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(ab[kMode == kFgGated ? i & 1 : 0]), (short)0, st < nst ? abytes : 0, 0x00020000);
    d[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, aoff[i], 2048 * st + 1024 * ks, 0));
  };
  auto load_x = [&](int i, int st, int slot) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(g.X + m0 * Kb), (short)0, st < nst ? (int)(M * Kb) : 0, 0x00020000);
    uint32_t off = xoff[i];
    if (kRagged && 128 * st + 128 > Kb && 128 * st + (int)xp >= Kb) off = kFgOob;   // columns past K: zeros
    fg_dma16(r, dsm + slot * XS + (XG * wave + i) * 1024, off, 128 * st);
  };
  const uint32_t brow = lds_off(dsm) + 128 * (16 * FM * wm + fr);
  const uint32_t bc[2] = {16u * (uint32_t)(fg ^ (fr & 7)), 16u * (uint32_t)((4 + fg) ^ (fr & 7))};
  auto read_b = [&](u32x4& d, int t, int slot, int ks) { d = lds_load16(brow + (uint32_t)(slot * XS) + 2048 * t + bc[ks]); };

  f32x4 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // prologue: the ring's first three stages, and two stages of fragments but the second one's last half, in the order
  // of their use.  Groups are fenced: the waits count what was issued after a group.
#pragma unroll
  for (int u = 0; u < 3; ++u) {
#pragma unroll
    for (int i = 0; i < XG; ++i) load_x(i, u, u);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2 - u; ++ks)
#pragma unroll
      for (int i = 0; i < FN; ++i) load_a(a[u & 1][ks], i, u, ks);
    __builtin_amdgcn_sched_barrier(0);
  }
  fg_wait_vm<XG + FN>();                             // stages 0 and 1 are staged: after them came A1's half and stage 2
  fg_barrier();
#pragma unroll
  for (int t = 0; t < FM; ++t) read_b(b[0][t], t, 0, 0);

  auto stage = [&](int st, int slot, u32x4 (&as)[2][FN], u32x4 (&next)[2][FN]) {
    // half 0: k-step 0 of stage st; read k-step 1; load the second k-step of stage st + 1
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < FM; ++t) {
      read_b(b[1][t], t, slot, 1);
      if (t < FN) load_a(next[1], t, st + 1, 1);
#pragma unroll
      for (int i = 0; i < FN; ++i) acc[i][t] = fg_mfma<T>(as[0][i], b[0][t], acc[i][t]);
    }
#pragma unroll
    for (int t = 0; t < FM; ++t) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (t < FN) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, FN, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // Stage st + 1's activations were requested in the second half of stage st - 2 (or before the loop); since then
    // two first halves of FN requests and one second half of XG + FN were issued.
    fg_wait_vm<XG + 3 * FN>();
    fg_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // half 1: k-step 1; read k-step 0 of stage st + 1; refill the buffer of stage st - 1
#pragma unroll
    for (int t = 0; t < FM; ++t) {
      read_b(b[0][t], t, (slot + 1) & 3, 0);
      if (t < XG) load_x(t, st + 3, (slot + 3) & 3);
      if (t < FN) load_a(as[0], t, st + 2, 0);
#pragma unroll
      for (int i = 0; i < FN; ++i) acc[i][t] = fg_mfma<T>(as[1][i], b[1][t], acc[i][t]);
    }
#pragma unroll
    for (int t = 0; t < FM; ++t) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (t < XG) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      if (t < FN) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, FN, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(XG <= FM && FN <= FM, "one request per MFMA column");
  for (int st = 0; st < nst; st += 4) {              // stages past the last multiply zeros by zeros
    stage(st, 0, a[0], a[1]);
    stage(st + 1, 1, a[1], a[0]);
    stage(st + 2, 2, a[0], a[1]);
    stage(st + 3, 3, a[1], a[0]);
  }
  fg_wait_vm<0>();
  __syncthreads();

  // epilogue: lane (fr, fg) register r of fragment (i, j): n = 16 i + 4 fg + r, m = 16 j + fr; through LDS so that
  // a row's columns leave as 16-byte pieces
  constexpr int WN = kMode == kFgGated ? 8 * FN : 16 * FN;    // output columns of the wave
  constexpr int CH = WN / 8;                                  // 16-byte pieces per row
  const int64_t n0 = (int64_t)bn * NWN * WN + wn * WN;
  const int mw = 16 * FM * wm;
  auto value = [&](int i, int j, int r, int64_t n) -> uint32_t {
    if constexpr (kQ) {
      const int m = mw + 16 * j + fr;
      const float sx = g.sx[m0 + (m < M ? m : M - 1)], sw = g.sw[n < N ? n : N - 1];
      return F16::from_f32(__fmul_rn(__fmul_rn((float)__float_as_int(acc[i][j][r]), sx), sw));
    } else if constexpr (kMode == kFgGated) {
      const float gs = acc[2 * i][j][r], us = acc[2 * i + 1][j][r];
      return T::from_f32(gs / (1.0f + expf(-gs)) * us);
    } else {
      return T::from_f32(acc[i][j][r]);
    }
  };
  unsigned char* out = dsm + wave * (16 * FM * WN * 2);
#pragma unroll
  for (int j = 0; j < FM; ++j)
#pragma unroll
    for (int i = 0; i < WN / 16; ++i) {
      const int64_t n = n0 + 16 * i + 4 * fg;
      u32x2 p;
      p.x = value(i, j, 0, n) | (value(i, j, 1, n + 1) << 16);
      p.y = value(i, j, 2, n + 2) | (value(i, j, 3, n + 3) << 16);
      const int row = 16 * j + fr, c = 2 * i + (fg >> 1);
      *reinterpret_cast<u32x2*>(out + row * (WN * 2) + 16 * (c ^ (row & (CH - 1))) + 8 * (fg & 1)) = p;
    }
  if constexpr (kQ) {
    if (g.acc) {
#pragma unroll
      for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = mw + 16 * j + fr;
            const int64_t n = n0 + 16 * i + 4 * fg + r;
            if (m < M && n < N) g.acc[(m0 + m) * N + n] = __float_as_int(acc[i][j][r]);
          }
    }
  }
  wave_lds_sync();
  const bool whole = n0 + WN <= N && (N & 7) == 0;
#pragma unroll
  for (int q = 0; q < 16 * FM * CH / 64; ++q) {
    const int e = 64 * q + lane, row = e / CH, c = e % CH;
    const u32x4 v = *reinterpret_cast<const u32x4*>(out + row * (WN * 2) + 16 * (c ^ (row & (CH - 1))));
    const int m = mw + row;
    if (m >= M) continue;
    const int64_t n = n0 + 8 * c;
    uint16_t* y = g.Y + (m0 + m) * N + n;
    if (whole) {
      *reinterpret_cast<u32x4*>(y) = v;
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (n + k < N) y[k] = (uint16_t)(v[k >> 1] >> (16 * (k & 1)));
    }
  }
}

// ------------------------------------------------------------------ decoding

// One launch decodes the matrices of a group: task i owns workgroups
// [first[i], first[i + 1]).
struct FgExpandTask {
  const uint32_t* bm;
  const unsigned char* values;
  const int32_t* toff;
  unsigned char* A;
  int64_t frags;                 // fragments to write
  int32_t S, SP;                 // tile steps; fragments per row block
  int32_t B;                     // row blocks (transposed form)
};
struct FgExpandArg {
  FgExpandTask t[SPL_MAX_GROUP];
  int32_t first[SPL_MAX_GROUP + 1];
  int32_t count;
};
constexpr int kFgTiles = 4;      // fragments per wave, their loads in flight together

// The operand of a lane's byte of a bitmask word: two 8-byte windows from the
// first value of each nibble, placed by the selector table.
__device__ __forceinline__ u32x4 fg_place(uint32_t byte, u32x2 v0, u32x2 v1, const u32x2* lut) {
  const u32x2 slo = lut[byte & 0xfu], shi = lut[byte >> 4];
  return u32x4{__builtin_amdgcn_perm(v0.y, v0.x, slo.x), __builtin_amdgcn_perm(v0.y, v0.x, slo.y),
               __builtin_amdgcn_perm(v1.y, v1.x, shi.x), __builtin_amdgcn_perm(v1.y, v1.x, shi.y)};
}

// 16-bit payloads: fragment (row block b, step s) is tile (b, s); steps past S
// are zeros.  Each value is read once, 1 KB written per tile with one coalesced
// store; bound by a wave's two dependent trips (offsets and words, then values)
// with four fragments in flight rather than by HBM (gate|up 67 us for 66 MB
// read and 180 MB written, 3.7 TB/s, where plain reads reach 6.5).  The windows
// read at most 16 bytes past the last payload, which every values buffer has.
__global__ void __launch_bounds__(256) k_frag_expand16(const FgExpandArg g) {
  __shared__ u32x2 lut[16];
  if (threadIdx.x < 16) lut[threadIdx.x] = u32x2{nibble_selector16(threadIdx.x, 0), nibble_selector16(threadIdx.x, 1)};
  __syncthreads();
  const FgExpandTask& k = g.t[find_task(g.first, g.count)];
  const int64_t f0 = ((int64_t)((int)blockIdx.x - g.first[find_task(g.first, g.count)]) * 4 + (threadIdx.x >> 6)) * kFgTiles;
  if (f0 >= k.frags) return;                         // whole waves leave together
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  const uint16_t* values = reinterpret_cast<const uint16_t*>(k.values);
  uint32_t byte[kFgTiles], oa[kFgTiles];
  int64_t b = f0 / k.SP;
  int s = (int)(f0 - b * k.SP);
#pragma unroll
  for (int i = 0; i < kFgTiles; ++i) {
    const bool live = f0 + i < k.frags && s < k.S;
    const int64_t t = b * k.S + s;
    byte[i] = live ? (k.bm[t * 16 + fr] >> (8 * fg)) & 0xffu : 0u;
    oa[i] = live ? (uint32_t)k.toff[t] : 0u;
    if (++s == k.SP) s = 0, ++b;
  }
#pragma unroll
  for (int i = 0; i < kFgTiles; i += 2) {            // values are in lane order: an exclusive scan, two tiles each
    const uint32_t pc = __popc(byte[i]) | (__popc(byte[i + 1]) << 16);
    const uint32_t ex = wave_inclusive_scan(pc) - pc;
    oa[i] += ex & 0xffffu;
    oa[i + 1] += ex >> 16;
  }
  u32x2 v0[kFgTiles], v1[kFgTiles];
#pragma unroll
  for (int i = 0; i < kFgTiles; ++i) {
    __builtin_memcpy(&v0[i], values + oa[i], 8);
    __builtin_memcpy(&v1[i], values + oa[i] + __popc(byte[i] & 0xfu), 8);
  }
#pragma unroll
  for (int i = 0; i < kFgTiles; ++i) {
    if (f0 + i >= k.frags) break;
    *reinterpret_cast<u32x4*>(k.A + (f0 + i) * 1024 + 16 * lane) = fg_place(byte[i], v0[i], v1[i], lut);
  }
}

// int8 payloads: fragment (b, p) is the pair of tiles 2p (lanes 0-31) and
// 2p + 1 (lanes 32-63); a lane holds 16 columns, its values from the exclusive
// scan over its half of the wave.
__global__ void __launch_bounds__(256) k_frag_expand8(const FgExpandArg g) {
  __shared__ uint32_t lut[80];
  if (threadIdx.x < 80) lut[threadIdx.x] = nibble_selector8(threadIdx.x / 5, threadIdx.x % 5);
  __syncthreads();
  const FgExpandTask& k = g.t[find_task(g.first, g.count)];
  const int64_t f0 = ((int64_t)((int)blockIdx.x - g.first[find_task(g.first, g.count)]) * 4 + (threadIdx.x >> 6)) * kFgTiles;
  if (f0 >= k.frags) return;
  const int lane = threadIdx.x & 63, fr = lane & 15, half = (lane >> 4) & 1;
  uint32_t hw[kFgTiles], oa[kFgTiles];
  int64_t b = f0 / k.SP;
  int p = (int)(f0 - b * k.SP);
#pragma unroll
  for (int i = 0; i < kFgTiles; ++i) {
    const int s = 2 * p + (lane >> 5);
    const bool live = f0 + i < k.frags && s < k.S;
    const int64_t t = b * k.S + s;
    hw[i] = live ? (k.bm[t * 16 + fr] >> (16 * half)) & 0xffffu : 0u;
    oa[i] = live ? (uint32_t)k.toff[t] : 0u;
    if (++p == k.SP) p = 0, ++b;
  }
#pragma unroll
  for (int i = 0; i < kFgTiles; i += 2) {
    const uint32_t pc = __popc(hw[i]) | (__popc(hw[i + 1]) << 16);
    const uint32_t ex = half_inclusive_scan(pc) - pc;
    oa[i] += ex & 0xffffu;
    oa[i + 1] += ex >> 16;
  }
  u32x2 v0[kFgTiles], v1[kFgTiles];                  // 8-byte windows: columns 0-7 and 8-15 of the lane's 16
#pragma unroll
  for (int i = 0; i < kFgTiles; ++i) {
    __builtin_memcpy(&v0[i], k.values + oa[i], 8);
    __builtin_memcpy(&v1[i], k.values + oa[i] + __popc(hw[i] & 0xffu), 8);
  }
#pragma unroll
  for (int i = 0; i < kFgTiles; ++i) {
    if (f0 + i >= k.frags) break;
    const uint32_t q0 = hw[i] & 15u, q1 = (hw[i] >> 4) & 15u, q2 = (hw[i] >> 8) & 15u, q3 = hw[i] >> 12;
    u32x4 v;
    v.x = __builtin_amdgcn_perm(v0[i].y, v0[i].x, lut[5 * q0]);
    v.y = __builtin_amdgcn_perm(v0[i].y, v0[i].x, lut[5 * q1 + __popc(q0)]);
    v.z = __builtin_amdgcn_perm(v1[i].y, v1[i].x, lut[5 * q2]);
    v.w = __builtin_amdgcn_perm(v1[i].y, v1[i].x, lut[5 * q3 + __popc(q2)]);
    *reinterpret_cast<u32x4*>(k.A + (f0 + i) * 1024 + 16 * lane) = v;
  }
}

// Fragments of W transposed (16-bit): row block b' holds columns 16 b' .. + 15
// of W, step s' its rows 32 s' .. + 31.  A wave decodes the tiles (2s', s) and
// (2s' + 1, s) into a 32 x 32 block in LDS (rows of 64 bytes) and reads its
// two fragments b' = 2s, 2s + 1 with LDS transpose reads: in each 16-lane
// quarter, lane l points at 8 bytes of row l / 4, columns 4 (l % 4) .. + 3,
// and receives column l of the quarter's four rows.
__device__ __forceinline__ u32x2 fg_load_tr8(uint32_t addr) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(
      u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)addr));
}
__global__ void __launch_bounds__(256) k_frag_expand16t(const FgExpandArg g) {
  __shared__ u32x2 lut[16];
  __shared__ __align__(16) unsigned char blk[4][2048];
  if (threadIdx.x < 16) lut[threadIdx.x] = u32x2{nibble_selector16(threadIdx.x, 0), nibble_selector16(threadIdx.x, 1)};
  __syncthreads();
  const FgExpandTask& k = g.t[0];
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4, wave = threadIdx.x >> 6;
  const int64_t u = (int64_t)blockIdx.x * 4 + wave;  // block (s', s): s' = u % SP, so that a row's stores follow on
  if (u >= k.frags) return;                          // k.frags: blocks, SP x S
  const int64_t s = u / k.SP;
  const int sp = (int)(u - s * k.SP);
  const uint16_t* values = reinterpret_cast<const uint16_t*>(k.values);
  uint32_t byte[2], oa[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int b = 2 * sp + i;
    const int64_t t = (int64_t)b * k.S + s;
    byte[i] = b < k.B ? (k.bm[t * 16 + fr] >> (8 * fg)) & 0xffu : 0u;
    oa[i] = b < k.B ? (uint32_t)k.toff[t] : 0u;
  }
  const uint32_t pc = __popc(byte[0]) | (__popc(byte[1]) << 16);
  const uint32_t ex = wave_inclusive_scan(pc) - pc;
  oa[0] += ex & 0xffffu;
  oa[1] += ex >> 16;
  u32x2 v0[2], v1[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    __builtin_memcpy(&v0[i], values + oa[i], 8);
    __builtin_memcpy(&v1[i], values + oa[i] + __popc(byte[i] & 0xfu), 8);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)                        // row 16 i + fr, columns 8 fg .. + 7
    *reinterpret_cast<u32x4*>(blk[wave] + 64 * (16 * i + fr) + 16 * fg) = fg_place(byte[i], v0[i], v1[i], lut);
  wave_lds_sync();
  const uint32_t base = lds_off(blk[wave]) + 64 * (8 * fg + (fr >> 2)) + 8 * (fr & 3);
#pragma unroll
  for (int h = 0; h < 2; ++h) {                      // column 16 h + fr, rows 8 fg .. + 7
    const u32x2 lo = fg_load_tr8(base + 32 * h), hi = fg_load_tr8(base + 32 * h + 256);
    *reinterpret_cast<u32x4*>(k.A + ((2 * s + h) * k.SP + sp) * 1024 + 16 * lane) = u32x4{lo.x, lo.y, hi.x, hi.y};
  }
}

// ------------------------------------------------------------------ launches

template <bool kQ>
int64_t fg_bytes(int64_t rows, int64_t cols) { return tile_blocks(rows) * fg_steps<kQ>(cols) * 1024; }

// Decode `count` matrices (16-bit, or int8 with kQ) one after the other into
// scratch; at[i] receives matrix i's fragments.
template <bool kQ>
hipError_t fg_expand(const spl_matrix* const* W, int count, unsigned char* scratch, unsigned char** at,
                     hipStream_t s) {
  FgExpandArg g{};
  g.count = count;
  for (int i = 0; i < count; ++i) {
    FgExpandTask& t = g.t[i];
    t.bm = W[i]->bitmask, t.values = static_cast<const unsigned char*>(W[i]->values), t.toff = W[i]->tile_offsets;
    t.S = (int32_t)tile_steps(W[i]->cols), t.SP = (int32_t)fg_steps<kQ>(W[i]->cols);
    t.frags = tile_blocks(W[i]->rows) * t.SP;
    t.A = at[i] = scratch;
    scratch += t.frags * 1024;
    g.first[i + 1] = g.first[i] + (int32_t)((t.frags + 4 * kFgTiles - 1) / (4 * kFgTiles));
  }
  const dim3 grid((unsigned)g.first[count]);
  if (kQ)
    hipLaunchKernelGGL(k_frag_expand8, grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL(k_frag_expand16, grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

template <class T, int FN, int FM, int NWN, int NWM, int kMode, bool kRagged>
hipError_t fg_launch(FgGroupArg& g, hipStream_t s) {
  constexpr int BM = 16 * FM * NWM, RN = (kMode == kFgGated ? 8 : 16) * FN * NWN;
  constexpr size_t ring = (size_t)4 * BM * 128, out = (size_t)NWN * NWM * 16 * FM * 16 * FN * 2;
  constexpr size_t lds = ring > out ? ring : out;
  auto* kernel = k_frag_gemm<T, FN, FM, NWN, NWM, kMode, kRagged>;
  static PerDeviceFlag lds_set;
  const hipError_t attr = allow_lds_once(lds_set, kernel, lds);
  if (attr != hipSuccess) return attr;
  const int tm = (g.M + BM - 1) / BM;
  g.first[0] = 0;
  for (int i = 0; i < g.count; ++i) {
    g.t[i].tn = (int32_t)((g.t[i].N + RN - 1) / RN);
    g.first[i + 1] = g.first[i] + tm * g.t[i].tn;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)g.first[g.count]), dim3(64 * NWN * NWM), lds, s, g);
  return hipGetLastError();
}

// Workgroup tile of a launch and its cost: the one whose rounds over the chip cost least.
// Costs are us per 64 stages measured on 4096-column launches (bf16): one
// workgroup of 128 x 256 per CU 60; of 128 x 128, two per CU, 32 for one and
// 62 for both; of 64 x 128, four per CU, 24, 42, 60 and 78.  So gate|up at
// 2048 tokens (1376 / 2752 / 5504 tiles) takes 128 x 128 (333 us; 340 with
// 128 x 256), q|k|v there 128 x 256 (179; 185), q at 512 tokens 64 x 128
// (24.5; 31 and 50 with the larger ones).  A stage is as many MFMA cycles in
// fp16, and in int8, where it holds 128 columns.  Over 68 launches of 8 sets of
// widths at 256 to 2048 rows in fp16, int8 and the gated form, each forced to
// all three tiles, the choice is within 5% of the best but for seven: gate|up
// fp16 at 2048 rows 403 us, 375 with 128 x 256; gated at 256, which is expanded
// in place; 2 x 5632 x 2048 at 2048 rows int8 70, gated 115, 64 and 105 with 128
// x 128; and int8 at 512 to 2048 rows on three widths by 5 to 7%.
enum { kFgL, kFgM, kFgS };
struct FgCost {
  int tile;
  int64_t us;                    // per 64 stages
};
FgCost fg_cost(const int64_t* N, int count, int64_t M) {   // rows of each task (gated: of both matrices)
  const int64_t cus = device_cus();
  auto tiles = [&](int rn, int bm) {
    int64_t n = 0;
    for (int i = 0; i < count; ++i) n += (N[i] + rn - 1) / rn;
    return n * ((M + bm - 1) / bm);
  };
  const int64_t l = tiles(128, 256), m = tiles(128, 128), q = tiles(64, 128);
  const int64_t cl = (l + cus - 1) / cus * 60;
  const int64_t mr = m % (2 * cus), cm = m / (2 * cus) * 62 + (mr == 0 ? 0 : mr <= cus ? 32 : 62);
  const int64_t qr = (q % (4 * cus) + cus - 1) / cus, cq = q / (4 * cus) * 78 + (qr == 0 ? 0 : 6 + 18 * qr);
  return cl <= cm && cl <= cq ? FgCost{kFgL, cl} : cm <= cq ? FgCost{kFgM, cm} : FgCost{kFgS, cq};
}

// Us of the kernel that expands N x K in place for M rows of 16-bit payloads
// (gated: N rows of both matrices), from its tiles (k_prefill.hip): 128 x 256,
// one per CU, rounds of 1.38 us a stage of 64 columns; 64 x 128, up to one per
// CU 0.66 (K split), else 0.25 and 0.39 for each tile of a CU.
double fg_inplace_us(int64_t N, int64_t K, int64_t M) {
  const int64_t cus = device_cus(), st = (K + 63) / 64;
  const int64_t large = ((N + 127) / 128) * ((M + 255) / 256), small = ((N + 63) / 64) * ((M + 127) / 128);
  if (large >= cus) return (double)((large + cus - 1) / cus) * (4 + 1.38 * st);
  if (small <= cus) return 4 + 0.66 * st;
  return 4 + (0.25 + 0.39 * ((small + cus - 1) / cus)) * st;
}

// Us of decoding matrices into `bytes` of fragments at 3.3 TB/s and of their
// product: 7 us (gated 9) beside fg_cost, with 8 stages more for the product's
// ends, or reading the fragments at 2.8 TB/s.
double fg_decoded_us(const int64_t* N, int count, int64_t K, int64_t M, int64_t bytes, bool gated) {
  const double product = (double)fg_cost(N, count, M).us * ((K + 63) / 64 + 8) / 72, read = bytes / 2.8e6;
  return (gated ? 9 : 7) + bytes / 3.3e6 + (product > read ? product : read);
}

// Whether a call gains by decoding its matrices into scratch first.  int8
// always does (4096 x 4096 at 129 rows 32 us in place, 27 decoded; q|k|v 93,
// 34), but for one small matrix, where issuing the call from eager code costs
// more than the kernel (18 us with scratch, 12 without; 1024 x 1024 at 129 rows
// takes 16 us in place).  16-bit payloads by the estimates above; in place has to
// come to the 16 us that issuing a call with scratch takes.  Over 1022 launches
// on 31 sets of widths (K 512 to 11008, 113 to 2048 rows) they pick the slower
// way by more than 10% twice.  Where it matters (in place / decoded): gate|up
// gated at 129 rows 91 / 125 us, at 300 176 / 148, at 2048 530 / 395; 2 x 8192 x
// 3072 gated at 512 rows 75 / 87, at 768 136 / 110; 2 x 13824 x 5120 at 256 rows
// 164 / 215; 8192 x 1024 at 256 14 / 24; 4096 x 4096 at 129 44 / 39; 1536 x 1536
// at 397 rows 19.4 / 16.7, at 640 18.6 / 19.5.
bool fg_pays(const spl_matrix* const* W, int count, int64_t M, bool gated) {
  int64_t N[SPL_MAX_GROUP], bytes = 0, kmax = 0;
  double inplace = 0;
  if (W[0]->dtype == SPL_I8) {
    const int64_t small = ((W[0]->rows + 63) / 64) * ((M + 127) / 128);
    return count > 1 || W[0]->cols > 1024 || small > device_cus();
  }
  for (int i = 0; i < count; ++i) {
    const int64_t K = W[i]->cols;
    N[i] = W[i]->rows;
    bytes += fg_bytes<false>(W[i]->rows, K);
    kmax = K > kmax ? K : kmax;
    if (!gated) inplace += fg_inplace_us(N[i], K, M);
  }
  if (gated) {
    N[0] *= 2, count = 1;
    inplace = fg_inplace_us(N[0], kmax, M);
  }
  double decoded = fg_decoded_us(N, count, kmax, M, bytes, gated);
  // one launch of tiles with K split: its activations and outputs are read and written meanwhile
  if (count == 1 && !gated && ((N[0] + 63) / 64) * ((M + 127) / 128) <= device_cus())
    decoded += 2.0 * M * (N[0] + kmax) / 3.5e6;
  return inplace >= 16 && decoded < inplace;
}

template <class T, int kMode, bool kRagged>
hipError_t fg_product_r(FgGroupArg& g, hipStream_t s) {
  int64_t N[SPL_MAX_GROUP];
  for (int i = 0; i < g.count; ++i) N[i] = g.t[i].N * (kMode == kFgGated ? 2 : 1);
  switch (fg_cost(N, g.count, g.M).tile) {
    case kFgL:
      // (eight waves for int8, whose MFMAs the compiler keeps off the accumulation registers)
      if constexpr (!kRagged && fg_q<T>()) return fg_launch<T, 4, 4, 2, 4, kMode, kRagged>(g, s);
      else if constexpr (!kRagged) return fg_launch<T, 4, 8, 2, 2, kMode, kRagged>(g, s);
      // (ragged columns have no large tile, which would give 0 to 5%: 3 x 3000 x 3000 at 2048 rows 142 us, 141 with
      // it; 2 x 8008 x 3000 246, 239; 2 x 8008 x 4072 320, 304)
    case kFgM: return fg_launch<T, 4, 4, 2, 2, kMode, kRagged>(g, s);
    default: return fg_launch<T, 2, 4, 2, 2, kMode, kRagged>(g, s);
  }
}

template <class T, int kMode = kFgPlain>
hipError_t fg_product(FgGroupArg& g, hipStream_t s) {
  bool ragged = false;
  for (int i = 0; i < g.count; ++i) ragged = ragged || g.t[i].K % (fg_q<T>() ? 128 : 64) != 0;
  return ragged ? fg_product_r<T, kMode, true>(g, s) : fg_product_r<T, kMode, false>(g, s);
}

// A product of M rows with a decoded rows x cols matrix is addressable: its
// fragments and a workgroup's activations with 32-bit byte offsets.
template <bool kQ>
bool fg_fits(int64_t M, int64_t rows, int64_t cols) {
  return M >= 1 && M < ((int64_t)1 << 31) && cols <= ((int64_t)1 << 21) &&
         fg_bytes<kQ>(rows, cols) < ((int64_t)1 << 31);
}
// Workgroups of a task in the smallest tiles (64 x 128, 256 threads); a launch
// of them all stays below 2^32 threads up to kFgMaxGroups.
constexpr int64_t kFgMaxGroups = ((int64_t)1 << 24) - 1;
int64_t fg_groups(int64_t M, int64_t rows) { return ((rows + 63) / 64) * ((M + 127) / 128); }

}  // namespace

int64_t frag_linear_bytes(const spl_matrix* const* W, int count, int64_t M, bool gated) {
  int64_t bytes = 0, groups = 0;
  for (int i = 0; i < count; ++i) {
    const bool q = W[i]->dtype == SPL_I8;
    groups += fg_groups(M, W[i]->rows);
    if (!(q ? fg_fits<true>(M, W[i]->rows, W[i]->cols) : fg_fits<false>(M, W[i]->rows, W[i]->cols))) return 0;
    if (W[i]->nnz > 0) bytes += q ? fg_bytes<true>(W[i]->rows, W[i]->cols) : fg_bytes<false>(W[i]->rows, W[i]->cols);
  }
  return groups <= kFgMaxGroups && fg_pays(W, count, M, gated) ? bytes : 0;
}

hipError_t launch_frag_linear(const spl_sparse_task* tasks, int count, int64_t M, void* scratch, hipStream_t s) {
  FgGroupArg g{};
  g.M = (int32_t)M;
  const spl_matrix* W[SPL_MAX_GROUP];
  unsigned char* at[SPL_MAX_GROUP];
  for (int i = 0; i < count; ++i) {
    if (tasks[i].W->nnz == 0) {                      // nothing kept: +0
      const hipError_t e = launch_zero_fill(tasks[i].Y, M * tasks[i].W->rows, s);
      if (e != hipSuccess) return e;
      continue;
    }
    FgTask& t = g.t[g.count];
    t.X = static_cast<const unsigned char*>(tasks[i].X), t.Y = static_cast<uint16_t*>(tasks[i].Y);
    t.N = tasks[i].W->rows, t.K = tasks[i].W->cols;
    W[g.count++] = tasks[i].W;
  }
  if (g.count == 0) return hipSuccess;
  const hipError_t e = fg_expand<false>(W, g.count, static_cast<unsigned char*>(scratch), at, s);
  if (e != hipSuccess) return e;
  for (int i = 0; i < g.count; ++i) g.t[i].A = at[i];
  return W[0]->dtype == SPL_BF16 ? fg_product<Bf16>(g, s) : fg_product<F16>(g, s);
}

hipError_t launch_frag_gated(const void* X, int64_t M, const spl_matrix& Wg, const spl_matrix& Wu, void* Y,
                             void* scratch, hipStream_t s) {
  if (Wg.nnz == 0 || Wu.nnz == 0) return launch_zero_fill(Y, M * Wg.rows, s);   // silu(0) u = silu(g) 0 = 0
  const spl_matrix* W[2] = {&Wg, &Wu};
  unsigned char* at[2];
  const hipError_t e = fg_expand<false>(W, 2, static_cast<unsigned char*>(scratch), at, s);
  if (e != hipSuccess) return e;
  FgGroupArg g{};
  g.M = (int32_t)M, g.count = 1;
  FgTask& t = g.t[0];
  t.X = static_cast<const unsigned char*>(X), t.Y = static_cast<uint16_t*>(Y);
  t.N = Wg.rows, t.K = Wg.cols;
  t.A = at[0], t.A2 = at[1];
  return Wg.dtype == SPL_BF16 ? fg_product<Bf16, kFgGated>(g, s) : fg_product<F16, kFgGated>(g, s);
}

hipError_t launch_frag_int8(const spl_int8_task* tasks, int count, int64_t M, void* scratch, hipStream_t s) {
  FgGroupArg g{};
  g.M = (int32_t)M;
  const spl_matrix* W[SPL_MAX_GROUP];
  unsigned char* at[SPL_MAX_GROUP];
  for (int i = 0; i < count; ++i) {
    const spl_int8_task& k = tasks[i];
    if (k.Wq->nnz == 0) {                            // (float(0) * sx) * sw = +0
      hipError_t e = launch_zero_fill(k.Y, M * k.Wq->rows, s);
      if (e == hipSuccess && k.acc_out) e = launch_zero_fill(k.acc_out, 2 * M * k.Wq->rows, s);
      if (e != hipSuccess) return e;
      continue;
    }
    FgTask& t = g.t[g.count];
    t.X = reinterpret_cast<const unsigned char*>(k.Xq), t.Y = static_cast<uint16_t*>(k.Y);
    t.N = k.Wq->rows, t.K = k.Wq->cols;
    t.sx = k.x_scales, t.sw = k.w_scales, t.acc = k.acc_out;
    W[g.count++] = k.Wq;
  }
  if (g.count == 0) return hipSuccess;
  const hipError_t e = fg_expand<true>(W, g.count, static_cast<unsigned char*>(scratch), at, s);
  if (e != hipSuccess) return e;
  for (int i = 0; i < g.count; ++i) g.t[i].A = at[i];
  return fg_product<FgI8>(g, s);
}

// dX [M][K] = dY [M][N] W: the product with W transposed, decoded as such.
int64_t frag_input_grad_bytes(const spl_matrix& W, int64_t M) {
  if (W.rows % 8 != 0 || !fg_fits<false>(M, 32 * tile_steps(W.cols), W.rows) || fg_groups(M, W.cols) > kFgMaxGroups)
    return 0;
  const int64_t bytes = 2 * tile_steps(W.cols) * fg_steps<false>(W.rows) * 1024;
  // Where W's packed tiles can be read directly, decoding them first has to be the faster way (512 x 4096 at 2048 rows
  // 24 us decoded, 20 directly; 4096 x 4096 70, 95); elsewhere the other way decodes and transposes all of W.
  if (sparse_input_grad_applies(M, W) &&
      fg_decoded_us(&W.cols, 1, W.rows, M, bytes, false) >= fg_inplace_us(W.cols, W.rows, M))
    return 0;
  return bytes;
}

hipError_t launch_frag_input_grad(const void* dY, int64_t M, const spl_matrix& W, void* dX, void* scratch,
                                  hipStream_t s) {
  if (W.nnz == 0) return launch_zero_fill(dX, M * W.cols, s);
  FgExpandArg x{};
  x.count = 1;
  FgExpandTask& k = x.t[0];
  k.bm = W.bitmask, k.values = static_cast<const unsigned char*>(W.values), k.toff = W.tile_offsets;
  k.A = static_cast<unsigned char*>(scratch);
  k.S = (int32_t)tile_steps(W.cols), k.SP = (int32_t)fg_steps<false>(W.rows), k.B = (int32_t)tile_blocks(W.rows);
  k.frags = (int64_t)k.S * k.SP;
  hipLaunchKernelGGL(k_frag_expand16t, dim3((unsigned)((k.frags + 3) / 4)), dim3(256), 0, s, x);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  FgGroupArg g{};
  g.M = (int32_t)M, g.count = 1;
  FgTask& t = g.t[0];
  t.X = static_cast<const unsigned char*>(dY), t.Y = static_cast<uint16_t*>(dX);
  t.N = W.cols, t.K = W.rows;
  t.A = k.A;
  return W.dtype == SPL_BF16 ? fg_product<Bf16>(g, s) : fg_product<F16>(g, s);
}

}  // namespace spl
