// Narrow-level contraction tiles for gfx950: 16 or 32 rows per workgroup, K split over the workgroup's eight waves.
//
// A level of a few rows is a chain of latencies (launch, child index, operand rows, store) with little work in it.
// 128-row tiles multiplied padding, and their K had to be split over workgroups to fill the chip: partial sums through
// memory and a second launch (forward), or atomic adds into rows zeroed before (dz . W^T).  Here a workgroup owns its
// outputs: each wave contracts an eighth of K for the whole tile, with operands loaded straight into the fragments'
// registers (nothing is shared between waves, so LDS would only add a copy and a barrier), and the eight partial tiles
// meet in LDS.  16 x 16 MFMA tiles: row tiles of 16, and 4, 8 or 16 hidden units a workgroup, so that H = 1,024 gives 64
// to 256 workgroups a row tile.
//
// Fragments: lane l supplies row l % 16 of A and column l % 16 of B.  A step of K is 128 bytes of every row, read as two
// 16-byte pieces at 16 (l / 16) and 64 + 16 (l / 16): any order of K is right as long as both operands have the same.
// Result: lane l, register r holds row 4 (l / 16) + r, column l % 16.
#pragma once

#include "common.h"
#include "dma.h"
#include "mfma.h"

namespace fold {

namespace narrow {

constexpr int kThreads = 512, kWaves = 8;

// acc += 64 bytes of K
__device__ __forceinline__ f32x4 mma(float, uint4 a, uint4 b, f32x4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma(uint16_t, uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// One wave's share of K, steps wave, wave + 8, ... of np: arow(q, rt) and bcol(q, ct) give this lane's address of step q
// (arow with the piece 16 (l / 16), as `zero`).  PD steps are in flight; past the end they read the zero row.  The
// first weights go out before anything waits for a row index; ahead() issues the caller's own loads behind them.
template <typename T, int RT, int CT, int PD, class AROW, class BCOL, class AHEAD>
__device__ __forceinline__ void contract(int np, int wave, const char* zero, const AROW& arow, const BCOL& bcol,
                                         const AHEAD& ahead, f32x4 (&acc)[RT][CT]) {
  uint4 a[PD][RT][2], b[PD][CT][2];
  auto load_a = [&](int s, int i) {
    const int q = wave + kWaves * i;
    const bool in = q < np;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const char* p = in ? arow(q, rt) : zero;
      a[s][rt][0] = *reinterpret_cast<const uint4*>(p);
      a[s][rt][1] = *reinterpret_cast<const uint4*>(p + 64);
    }
  };
  auto load_b = [&](int s, int i) {
    const int q = wave + kWaves * i;
    const bool in = q < np;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const char* p = in ? bcol(q, ct) : zero;
      b[s][ct][0] = *reinterpret_cast<const uint4*>(p);
      b[s][ct][1] = *reinterpret_cast<const uint4*>(p + 64);
    }
  };
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int n = (np - wave + kWaves - 1) / kWaves;
#pragma unroll
  for (int s = 0; s < PD; ++s) load_b(s, s);
#pragma unroll
  for (int s = 0; s < PD; ++s) load_a(s, s);
  ahead();
  for (int i = 0; i < n; i += PD) {
#pragma unroll
    for (int s = 0; s < PD; ++s) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = mma(T(), a[s][rt][h], b[s][ct][h], acc[rt][ct]);
      load_b(s, i + s + PD);
      load_a(s, i + s + PD);
    }
  }
}

// A partial tile in LDS: four consecutive rows of a column are one 16-byte unit (a lane's registers); column c's units
// are at 4 c + (quad ^ c / 4), so that neither the writes (a wave: 1 KB) nor reads along a row collide.
__device__ __forceinline__ int unit_of(int col, int quad) { return 4 * col + (quad ^ (col >> 2)); }
__device__ __forceinline__ int float_of(int row, int col) { return 4 * unit_of(col, row >> 2) + (row & 3); }

// The eight waves' tiles, added up in wave order into red[0 .. RT * CT * 64).
template <int RT, int CT>
__device__ __forceinline__ void reduce(const f32x4 (&acc)[RT][CT], f32x4* red, int wave, int lane) {
  constexpr int N = RT * CT * 64;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      red[wave * N + (rt * CT + ct) * 64 + unit_of(lane & 15, lane >> 4)] = acc[rt][ct];
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += kThreads) {
    f32x4 s = red[i];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s += red[w * N + i];
    red[i] = s;
  }
  __syncthreads();
}

}  // namespace narrow

}  // namespace fold
