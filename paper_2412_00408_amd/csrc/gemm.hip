// gemm.hip — quake_linear_gelu: y = GELU(x w^T) for bfloat16 or binary16
// x [m, k] and w [n, k] (both k-contiguous, the layout of a linear layer's
// input and weight), binary32 accumulation on the matrix cores, the GELU of
// Eq. 7 with QuAKE / QuAKE2 / EXACT applied to the binary32 accumulators in
// the epilogue, output in the input format. This is QuAKE inside a fused consumer: the GELU
// costs no HBM traffic of its own.
//
// What bounds it, and what follows from that (MI355X, random operands):
//  * Power. With random operands the matrix cores pull the clock down to
//    1.6-2.0 GHz, and v_mfma_*_16x16x32 does the same products for less energy
//    than 32x32x16: 1973 against 1584 TFLOP/s in a loop of nothing else. So the
//    blocks are 16 x 16.
//  * Operand delivery. A CU takes 64 bytes per clock from L2, and L2 serves
//    whole 128-byte lines (rows of 64 bytes got half that rate with every CU
//    loading: 30 against 59 bytes per clock and CU), so K advances in slabs of
//    64 elements = one line per row, and the tiles are as wide as registers
//    and LDS allow: 256 x 256 and 256 x 192 need 1/2 and 7/12 of that rate at
//    the full matrix-core rate.
//  * Issue. Slabs go from L2 to LDS directly (global_load_lds, no registers, no
//    ds_write). A burst of those loads stalls every wave that issues it, so
//    they and the fragment reads are placed one by one between the products
//    (4096 x 4096 x 4096 with 256 x 256 tiles of 32 x 32 blocks: 125 us with
//    bursts, 109 us with the loads spread out; 100 us with 16 x 16 blocks).
//  * Latency. The x and w tiles have SA and SB stages in LDS (up to 160 KB), so
//    that a slab is loaded one to four slabs ahead; one barrier per slab.
//  * The output. Where tiles end together, the write is not hidden; it leaves
//    through LDS as whole rows, 16 bytes per lane at any address of y (rows of
//    y are 16-byte aligned only where n is a multiple of 8). Of aligned rows a
//    large output is written non-temporally, so that L2 has little left to
//    write back at the end of the kernel (the product of 16384 x 4096 x 1024:
//    126.8 -> 112.1 us).
//  * Few slabs. The first slab and the output then take most of a tile's time,
//    and only other workgroups of the same CU can hide them: small tiles, and
//    128 x 128 with two or three stages instead of five, of which two fit a
//    CU. With k of one slab a tile has one stage and no refills (with two or
//    three, whose loads past the end of k fetch zeros, such products took 8 %
//    longer over 300 shapes, 12436 x 3713 x 64 37 against 33 us).
// Measured against the kernel this replaced (128-wide tiles of 32 x 32 blocks,
// slabs through registers; back to back, with the GELU): bf16 4096 x 3072 x 768
// 26.5 -> 21.9 us, 4096 x 768 x 3072 (no GELU) 37.2 -> 21.0 us, binary16
// 16384 x 4096 x 1024 (EXACT) 187.0 -> 129.0 us (1065 TFLOP/s).
//
// Operand lane layout of the 16x16x32 16-bit MFMA: lane l holds row l mod 16
// and k = 8 (l / 16) .. +7 of A, column l mod 16 and the same k of B;
// accumulator r of lane l is row 4 (l / 16) + r, column l mod 16. The w
// fragment is passed as A, so that a lane's four accumulators are four
// consecutive columns of one row of y.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "quake_device.hpp"
#include "quake_host.hpp"

namespace qk {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// one 16x16x32 matrix-core step on raw 16-bit operands of format DT
template <int DT>
__device__ __forceinline__ f32x4_t mfma16(u32x4 a, u32x4 b, f32x4_t c) {
  if constexpr (DT == BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a),
                                                  __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

constexpr int kBK = 64;          // elements of k per slab: one 128-byte line per row
constexpr int kSlabRow = 128;    // bytes of an LDS row

struct GemmArgs {
  const uint16_t* x;
  const uint16_t* w;
  uint16_t* y;
  int32_t m, n, k;
  int64_t ldx, ldw, ldy;   // elements
  float c0, c1, a;         // GELU constants (Eq. 7 folded into Eq. 5)
  uint32_t tiles_m, tiles_n;
  int32_t op;              // quake_mode of the GELU, or -1 for the product alone
  uint32_t nt;             // y (rows 16-byte aligned) is written non-temporally
};

// where lanes past the end of k load from
__device__ const u32x4 g_zero16 = {0u, 0u, 0u, 0u};

// the workgroup's barrier, no LDS access of this wave outstanding or moved across
__device__ __forceinline__ void lds_barrier() {
  wait_lds();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The GELU of four accumulators (op uniform: its branches are scalar), as two
// packed pairs.
template <int DT>
__device__ __forceinline__ uint2 gelu4(f32x4_t v, const GemmArgs& g, int op) {
  float f[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (op == EXACT) f[i] = gelu_q<EXACT>(f[i], g.c0, g.c1, g.a);
    else if (op == Q1) f[i] = gelu_q<Q1>(f[i], g.c0, g.c1, g.a);
    else if (op == Q2) f[i] = gelu_q<Q2>(f[i], g.c0, g.c1, g.a);
    else if (op == Q2M) f[i] = gelu_q<Q2M>(f[i], g.c0, g.c1, g.a);
  }
  uint2 o;
  o.x = DT == BF16 ? pack_bf16(f[0], f[1]) : pack_f16(f[0], f[1]);
  o.y = DT == BF16 ? pack_bf16(f[2], f[3]) : pack_f16(f[2], f[3]);
  return o;
}

// Stores to y at any address: gfx950 takes vector stores there (the compiler
// emits the same global_store_dwordx4 for this type). Unaligned rows cost 0-9 %
// more than aligned ones that way; element by element they cost 24-43 % more
// (13020 x 1666 x 128: 37.6 -> 24.6 us, 10308 x 3341 x 360: 72.7 -> 53.4, 2045 x 3069
// x 200: 14.7 -> 12.0; put together from dwords of LDS to aligned vectors and 2-byte
// row ends, 13020 x 1666 x 128 took as long as this and 6469 x 4028 x 72 10 % more).
// Not non-temporal: their vectors share lines with the next tile's, which L2 has
// to merge (8210 x 3081 x 16: 27.5 against 38.4 us).
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));
// the first n (1 to 7) elements of v to p
__device__ __forceinline__ void store_head(uint16_t* p, uint32_t n, const u32x4 v) {
  if (n & 4) *reinterpret_cast<u32x2_any*>(p) = u32x2_any{v[0], v[1]};
  if (n & 2) *reinterpret_cast<u32_any*>(p + (n & 4)) = (n & 4) ? v[2] : v[0];
  if (n & 1)
    *reinterpret_cast<u16_any*>(p + (n & 6)) =
        (uint16_t)((n & 4) ? ((n & 2) ? v[3] : v[2]) : ((n & 2) ? v[1] : v[0]));
}

// WM x WN waves over a BM x BN tile, SA / SB stages of its x / w slab
// (|SA - SB| <= 1, both at least 2; or one each, for k of one slab, where
// nothing is refilled); registers for two waves per SIMD.
template <int DT, int BM, int BN, int WM, int WN, int SA, int SB>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_kernel(GemmArgs g) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;         // 16 x 16 blocks per wave
  constexpr int IA = BM / 8 / NW, IB = BN / 8 / NW;           // loads per wave and slab
  constexpr int NV = IA + IB;
  constexpr uint32_t kA = BM * kSlabRow, kB = BN * kSlabRow;  // bytes of a stage
  constexpr uint32_t kB0 = SA * kA;                           // first w stage
  constexpr int P = TN * 32 + 16;                             // row pitch of the epilogue's staging
  constexpr bool kOne = SA == 1 && SB == 1;
  constexpr int kSlabs = SA * BM * kSlabRow + SB * BN * kSlabRow;
  constexpr int H = NW * 64 * P <= kSlabs ? 2 : 1;            // staging areas per wave, used in turn
  constexpr int kLds = kSlabs > H * NW * 32 * P ? kSlabs : H * NW * 32 * P;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && NW % 2 == 0, "whole loads per wave");
  static_assert(BM % (32 * WM) == 0 && BN % (16 * WN) == 0, "whole blocks per wave");
  static_assert(kOne || (SA >= 2 && SB >= 2 && SA - SB <= 1 && SB - SA <= 1), "stages");
  static_assert(kLds <= 163840, "LDS");
  __shared__ __attribute__((aligned(16))) char smem[kLds];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // Tile order: workgroups go to the 8 XCDs round-robin (blockIdx mod 8); XCD j
  // takes the j-th eighth of the tiles, in groups of 4 tile rows walked along
  // n, so that the rows of x and w in use at a time stay in its L2.
  const uint32_t tiles = g.tiles_m * g.tiles_n, xcd = blockIdx.x & 7u;
  const uint32_t id = xcd * (tiles >> 3) + min(xcd, tiles & 7u) + (blockIdx.x >> 3);
  const uint32_t gsz = 4u * g.tiles_n, first = id / gsz * 4u, in = id % gsz;
  const uint32_t rows = min(4u, g.tiles_m - first);
  const int row0 = (int)(first + in % rows) * BM, col0 = (int)(in / rows) * BN;

  // Slab loads: one instruction fills 8 LDS rows of 128 bytes, lane l slot
  // l mod 8 (16 bytes) of row l / 8. Slot s of row r holds k-vector s ^ (r / 2
  // mod 8) of the row, which makes the fragment reads below free of bank
  // conflicts. Rows past m (n) re-read the last row (never stored); k-vectors
  // past the end of k load zeros.
  const int kv = (lane & 7) ^ (4 * (wave & 1) + (lane >> 4));
  const char* pa[IA];
  const char* pb[IB];
#pragma unroll
  for (int i = 0; i < IA; ++i)
    pa[i] = reinterpret_cast<const char*>(
        g.x + (int64_t)min(row0 + 8 * (wave + NW * i) + (lane >> 3), g.m - 1) * g.ldx + 8 * kv);
#pragma unroll
  for (int i = 0; i < IB; ++i)
    pb[i] = reinterpret_cast<const char*>(
        g.w + (int64_t)min(col0 + 8 * (wave + NW * i) + (lane >> 3), g.n - 1) * g.ldw + 8 * kv);
  const int nk = (g.k + kBK - 1) / kBK;
  // before slab kt is loaded: lanes past the end of k to the zeros
  auto clip = [&](uint32_t kt, auto& p) {
    if (kBK * kt + kBK > (uint32_t)g.k) {
      const bool in_k = kBK * kt + 8 * kv < (uint32_t)g.k;
#pragma unroll
      for (auto& q : p) q = in_k ? q : reinterpret_cast<const char*>(&g_zero16);
    }
  };
  auto load_a = [&](uint32_t stage, int i) {
    lds_load16(lds0 + stage * kA + 1024 * (wave + NW * i), pa[i]);
    pa[i] += 2 * kBK;
  };
  auto load_b = [&](uint32_t stage, int i) {
    lds_load16(lds0 + kB0 + stage * kB + 1024 * (wave + NW * i), pb[i]);
    pb[i] += 2 * kBK;
  };
  // Loads are waited for in the order of issue, so of each slab the operand
  // with fewer stages, which is needed sooner, goes first.
  constexpr bool kAFirst = SA < SB;
  uint32_t fa = 0, fb = 0;   // the stages being refilled
  auto load = [&](int d) {   // d-th of the NV loads of a refill
    if (kAFirst) {
      if (d < IA) load_a(fa, d); else load_b(fb, d - IA);
    } else {
      if (d < IB) load_b(fb, d); else load_a(fa, d - IB);
    }
  };

  // Fragment reads: k-step ks (32 elements) of a slab, k-vector 4 ks + lane / 16
  // of row lane mod 16 of a block.
  const int fr = lane & 15, h = lane >> 4;
  const uint32_t kv0 = 16 * (h ^ (fr >> 1)), kv1 = 16 * ((4 + h) ^ (fr >> 1));
  const uint32_t oa = (wm * TM * 16 + fr) * kSlabRow, ob = kB0 + (wn * TN * 16 + fr) * kSlabRow;
  u32x4 af[TM], bf[2][TN];
  auto read_a = [&](uint32_t stage, int ks, int i) {
    af[i] = *reinterpret_cast<const u32x4*>(smem + (oa + stage * kA + (ks ? kv1 : kv0)) + 2048 * i);
  };
  auto read_b = [&](uint32_t stage, int ks, int j) {
    bf[ks][j] = *reinterpret_cast<const u32x4*>(smem + (ob + stage * kB + (ks ? kv1 : kv0)) + 2048 * j);
  };

  f32x4_t acc[TM][TN] = {};
  // the first SA / SB slabs, in the order their refills would have had
#pragma unroll
  for (int j = 0; j < (SA > SB ? SA : SB); ++j) {
    auto first_a = [&] {
      if (j < SA) {
        clip(j, pa);
#pragma unroll
        for (int i = 0; i < IA; ++i) load_a(j, i);
      }
    };
    if (kAFirst) first_a();
    if (j < SB) {
      clip(j, pb);
#pragma unroll
      for (int i = 0; i < IB; ++i) load_b(j, i);
    }
    if (!kAFirst) first_a();
  }
  wait_loads<(SA - 1) * IA + (SB - 1) * IB>();   // slab 0 is there
  lds_barrier();
  uint32_t ca = 0, cb = 0;   // the current slab's stages
#pragma unroll
  for (int i = 0; i < TM; ++i) read_a(0, 0, i);
#pragma unroll
  for (int j = 0; j < TN; ++j) read_b(0, 0, j);

  // One slab: TM TN products of its k-step 0, then of its k-step 1, row of
  // blocks by row of blocks. After the last product of a row the row's x
  // fragment is read again for the next k-step, in place; the w fragments have
  // two sets. The barrier stands after R1 rows of k-step 1: every wave's reads
  // of the slab are done there, the next slab has landed, and the slab's
  // stages are refilled from there until k-step 1 of the next slab.
  constexpr int M = TM * TN, R1 = TM >= 4 ? 2 : 1, Q1st = R1 * TN;
  constexpr int kWait = kOne ? 0 : (SA - 2) * IA + (SB - 2) * IB;   // loads that may still be in flight there
  constexpr int E = SA > SB ? IB : SA < SB ? IA : (NV + 1) / 2;   // loads of a refill beside k-step 1
  auto slab = [&](auto refill, int kt) {
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const int i = q / TN, j = q % TN;
      acc[i][j] = mfma16<DT>(bf[0][j], af[i], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
      if (j == TN - 1) read_a(ca, 1, i);
      if (q < TN) read_b(cb, 1, q);
      if (decltype(refill)::value) {
#pragma unroll
        for (int d = E; d < NV; ++d)
          if ((2 * (d - E) + 1) * M / (2 * (NV - E)) == q) load(d);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const int i = q / TN, j = q % TN;
      acc[i][j] = mfma16<DT>(bf[1][j], af[i], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
      const int p = q - (Q1st - 1);
      if (p == 0 && !kOne) {
        wait_loads<kWait>();
        lds_barrier();
        fa = ca;
        fb = cb;
        clip(kt + SA, pa);
        clip(kt + SB, pb);
        ca = ca + 1 == SA ? 0 : ca + 1;
        cb = cb + 1 == SB ? 0 : cb + 1;
      }
      if (p >= 0 && !kOne) {   // past the last slab: zeros, or what the stage last held; never used
        if (p < R1) read_a(ca, 0, p);
        else if (j == TN - 1) read_a(ca, 0, i);
        if (p < TN) read_b(cb, 0, p);
#pragma unroll
        for (int d = 0; d < E; ++d)
          if ((2 * d + 1) * (M - Q1st) / (2 * E) == p) load(d);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  slab(std::false_type{}, 0);   // the prologue filled every stage
  if constexpr (!kOne)
    for (int kt = 1; kt < nk; ++kt) slab(std::true_type{}, kt);
  wait_loads<0>();   // no load into LDS outlives its stage

  // Epilogue: GELU on the binary32 accumulators, rounded to the 16-bit format,
  // two rows of blocks (32 rows of y) at a time through this wave's own LDS
  // to whole rows. Accumulator r of block (i, j) in lane l is row 16 i + l mod 16,
  // column 16 j + 4 (l / 16) + r of the wave's part. All of a pass's LDS reads
  // stand before its first store (a store under the row guard ends a basic
  // block, so that a read after it would be waited for alone).
  __syncthreads();
  constexpr int CH = TN * 2;   // 16-byte vectors per row
  const int wrow = row0 + wm * TM * 16, wcol = col0 + wn * TN * 16;
  auto epilogue = [&](auto op) {
#pragma unroll
    for (int i = 0; i < TM; i += 2) {
      char* st = smem + (H * wave + (i >> 1) % H) * (32 * P);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          *reinterpret_cast<uint2*>(st + (16 * u + fr) * P + 32 * j + 8 * h) =
              gelu4<DT>(acc[i + u][j], g, decltype(op)::value);
      __builtin_amdgcn_wave_barrier();
      u32x4 v[TN];
#pragma unroll
      for (int q = 0; q < TN; ++q) {
        const int c = q * 64 + lane;
        v[q] = *reinterpret_cast<const u32x4*>(st + c / CH * P + 16 * (c % CH));
      }
#pragma unroll
      for (int q = 0; q < TN; ++q) {
        const int c = q * 64 + lane;
        const uint32_t row = wrow + 16 * i + c / CH, col = wcol + 8 * (c % CH);
        if (row >= (uint32_t)g.m || col >= (uint32_t)g.n) continue;
        uint16_t* yr = g.y + (int64_t)row * g.ldy + col;
        if (col + 8 > (uint32_t)g.n) store_head(yr, g.n - col, v[q]);
        else if (g.nt) __builtin_nontemporal_store(v[q], reinterpret_cast<u32x4*>(yr));
        else *reinterpret_cast<u32x4_any*>(yr) = v[q];
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  switch (g.op) {
    case EXACT: epilogue(std::integral_constant<int, EXACT>{}); break;
    case Q1: epilogue(std::integral_constant<int, Q1>{}); break;
    case Q2: epilogue(std::integral_constant<int, Q2>{}); break;
    case Q2M: epilogue(std::integral_constant<int, Q2M>{}); break;
    default: epilogue(std::integral_constant<int, -1>{}); break;
  }
}

template <int DT, int BM, int BN, int WM, int WN, int SA, int SB>
void launch_tile(GemmArgs g, hipStream_t s) {
  g.tiles_m = (uint32_t)(((int64_t)g.m + BM - 1) / BM);
  g.tiles_n = (uint32_t)(((int64_t)g.n + BN - 1) / BN);
  hipLaunchKernelGGL((gemm_kernel<DT, BM, BN, WM, WN, SA, SB>), dim3(g.tiles_m * g.tiles_n),
                     dim3(64 * WM * WN), 0, s, g);
}

// The tiles, and what a launch of each takes, in us:
//   first + s slab                  the first tile of the busiest CU (s slabs of 64 elements of k)
//   + (c - 1) (next + s next_slab)  c = ceil(tiles / CUs): the other tiles of that CU
//   + f (out + s load)              f = tiles / CUs: what all CUs share (L2 and memory);
//                                   out + gelu with the GELU, load + split where a row's
//                                   128 bytes of a slab lie on two lines
// Large tiles need the least operand traffic, small ones fill the chip where
// m n is small and overlap their first loads and their outputs where k is
// short; the estimate picks between them. k of one slab takes the tiles with one
// stage, longer k the others. Fitted to every tile's times on 1240 shapes (m to
// 16384, n to 4096, k to 4096, rows of x, w and y aligned and not, operands warm
// and cold; 300 shapes for one slab). On 880 others the picks took 0.4 % longer
// than the best tile measured on each, and 1.83x less time than the kernel of
// 128-wide tiles (2 of the 880 took over 5 % longer); the estimate before, of six
// tiles, took 1.51x less, but up to twice as long where k has few slabs. Whether
// the rows of y are aligned makes 0-4 % of difference and none to the pick. A
// launch takes fewer than 2^32 threads: a tile whose grid has more is passed over
// (only past 2^30 rows, where k of one slab takes the tiles for longer k).
struct Tile {
  uint32_t bm, bn, threads;
  float first, slab, next, next_slab, out, load, split, gelu;
};
constexpr int kFirstOne = 11;   // from here on one stage
constexpr Tile kTiles[] = {
    {256, 256, 512, 6.04f, 0.920f, 3.48f, 1.150f, 3.44f, 0.420f, 0.125f, 4.92f},
    {256, 192, 512, 5.55f, 0.860f, 4.85f, 0.776f, 1.83f, 0.224f, 0.160f, 4.93f},
    {128, 128, 512, 4.46f, 0.423f, 2.20f, 0.418f, 0.92f, 0.056f, 0.117f, 1.45f},
    {128, 128, 512, 3.82f, 0.364f, 0.94f, 0.216f, 0.50f, 0.208f, 0.113f, 1.06f},
    {128, 96, 256, 3.93f, 0.329f, 1.52f, 0.343f, 1.11f, 0.058f, 0.137f, 1.51f},
    {128, 64, 512, 3.18f, 0.306f, 0.12f, 0.157f, 0.71f, 0.101f, 0.092f, 0.39f},
    {128, 64, 256, 3.21f, 0.266f, 0.41f, 0.184f, 0.77f, 0.073f, 0.085f, 0.73f},
    {64, 64, 256, 3.02f, 0.202f, 0.41f, 0.133f, 0.40f, 0.031f, 0.045f, 0.29f},
    {64, 64, 256, 2.80f, 0.287f, 0.00f, 0.123f, 0.48f, 0.023f, 0.053f, 0.20f},
    {64, 32, 256, 2.72f, 0.165f, 0.10f, 0.080f, 0.38f, 0.009f, 0.034f, 0.13f},
    {64, 32, 256, 2.55f, 0.238f, 0.00f, 0.080f, 0.35f, 0.017f, 0.028f, 0.07f},
    {128, 128, 512, 3.38f, 0.0f, 0.00f, 0.0f, 1.26f, 0.0f, 0.0f, 1.08f},
    {64, 64, 256, 2.86f, 0.0f, 0.27f, 0.0f, 0.15f, 0.0f, 0.0f, 0.22f},
    {64, 32, 256, 2.55f, 0.0f, 0.18f, 0.0f, 0.17f, 0.0f, 0.0f, 0.08f},
};
constexpr int kTileCount = sizeof(kTiles) / sizeof(kTiles[0]);

// m, n < 2^31. About 0.1 us (32-bit divisions; a call's own time counts in the
// smallest products).
inline int pick_tile(uint32_t m, uint32_t n, uint32_t k, bool split, bool gelu, int cus) {
  const double slabs = (double)((k + kBK - 1) / kBK);
  auto grid = [&](const Tile& t) { return (uint64_t)((m - 1) / t.bm + 1) * ((n - 1) / t.bn + 1); };
  auto fits = [](const Tile& t, uint64_t tiles) { return tiles * t.threads <= UINT32_MAX; };
  const bool one = k <= kBK && fits(kTiles[kFirstOne], grid(kTiles[kFirstOne]));
  int best = 0;   // where no tile's grid can be launched: the launch reports it
  double best_us = -1;
  for (int i = one ? kFirstOne : 0; i < (one ? kTileCount : kFirstOne); ++i) {
    const Tile& t = kTiles[i];
    const uint64_t tiles = grid(t);
    if (!fits(t, tiles)) continue;
    const double share = (double)tiles / cus, others = std::ceil(share) - 1;
    const double us = t.first + slabs * t.slab + others * (t.next + slabs * t.next_slab) +
                      share * (t.out + (gelu ? t.gelu : 0.0) + slabs * (t.load + (split ? t.split : 0.0)));
    if (best_us < 0 || us < best_us) {
      best = i;
      best_us = us;
    }
  }
  return best;
}

template <int DT>
void launch_gemm(int tile, const GemmArgs& g, hipStream_t s) {
  switch (tile) {
    case 0: launch_tile<DT, 256, 256, 2, 4, 3, 2>(g, s); break;
    case 1: launch_tile<DT, 256, 192, 4, 2, 2, 3>(g, s); break;
    case 2: launch_tile<DT, 128, 128, 4, 2, 5, 5>(g, s); break;
    case 3: launch_tile<DT, 128, 128, 4, 2, 2, 3>(g, s); break;
    case 4: launch_tile<DT, 128, 96, 2, 2, 3, 3>(g, s); break;
    case 5: launch_tile<DT, 128, 64, 4, 2, 2, 2>(g, s); break;
    case 6: launch_tile<DT, 128, 64, 2, 2, 3, 3>(g, s); break;
    case 7: launch_tile<DT, 64, 64, 2, 2, 4, 4>(g, s); break;
    case 8: launch_tile<DT, 64, 64, 2, 2, 2, 2>(g, s); break;
    case 9: launch_tile<DT, 64, 32, 2, 2, 4, 4>(g, s); break;
    case 10: launch_tile<DT, 64, 32, 2, 2, 2, 2>(g, s); break;
    case 11: launch_tile<DT, 128, 128, 4, 2, 1, 1>(g, s); break;
    case 12: launch_tile<DT, 64, 64, 2, 2, 1, 1>(g, s); break;
    default: launch_tile<DT, 64, 32, 2, 2, 1, 1>(g, s); break;
  }
}

}  // namespace qk

using namespace qk;

extern "C" quake_status quake_linear_gelu(const void* x, const void* w, void* y, int64_t m,
                                          int64_t n, int64_t k, int64_t ldx, int64_t ldw,
                                          int64_t ldy, quake_dtype dtype, quake_mode mode,
                                          int gelu, void* stream) {
  if (dtype != QUAKE_BF16 && dtype != QUAKE_F16) return QUAKE_EDTYPE;
  if (!valid_mode(mode)) return QUAKE_EMODE;
  if (m < 0 || n < 0 || k < 0) return QUAKE_EINVAL;
  if (m == 0 || n == 0) return QUAKE_OK;
  if (k == 0 || k % 8 != 0 || x == nullptr || w == nullptr || y == nullptr) return QUAKE_EINVAL;
  if (ldx < k || ldw < k || ldy < n || ldx % 8 != 0 || ldw % 8 != 0) return QUAKE_EINVAL;
  if (!aligned16(x) || !aligned16(w)) return QUAKE_EINVAL;
  // 32-bit row, column and k arithmetic in the kernel: the largest row and
  // column formed are those of the last tile's last block
  if (m > INT32_MAX - 128 || n > INT32_MAX - 192 || k > INT32_MAX - 256) return QUAKE_EINVAL;
  if (((m + 127) / 128) * ((n + 127) / 128) > INT32_MAX) return QUAKE_EINVAL;
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  // a row's 128 bytes of a slab on two lines, for some rows
  const bool split = ldx % kBK != 0 || ldw % kBK != 0 || ((uintptr_t)x | (uintptr_t)w) % kSlabRow != 0;
  const int tile = pick_tile((uint32_t)m, (uint32_t)n, (uint32_t)k, split, gelu != 0, cus);
  const Affine af = gelu_affine(mode);
  // Non-temporal stores of y: whole aligned vectors of an output past 8 MB and
  // more than one slab. Smaller outputs fit L2 and are up to 12 % faster without
  // (2.6 MB, 743 x 1736 x 8: 3.9 against 4.3 us); with one slab nearly all of the
  // time is the write, and an output past 64 MB is 1.4-1.6x faster without. Past
  // 8 MB with more slabs 0-9 % slower without (14395 x 3872 x 240: 63.7 against
  // 58.7 us). Unaligned rows: their vectors share lines with the next tile's, so
  // that L2 has to merge them (8210 x 3081 x 16: 27.5 against 38.4 us).
  const bool nt = aligned16(y) && (ldy % 8 == 0 || m == 1) && k > kBK && m * n >= int64_t(1) << 22;
  const GemmArgs g{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w),
                   static_cast<uint16_t*>(y), (int32_t)m, (int32_t)n, (int32_t)k, ldx, ldw, ldy,
                   af.c0, af.c1, gelu_a(), 0, 0, gelu ? (int32_t)mode : -1, (uint32_t)nt};
  const hipStream_t s = static_cast<hipStream_t>(stream);
  if (dtype == QUAKE_BF16)
    launch_gemm<BF16>(tile, g, s);
  else
    launch_gemm<F16>(tile, g, s);
  return launch_status();
}
