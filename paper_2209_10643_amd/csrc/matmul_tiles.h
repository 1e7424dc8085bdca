// Device pieces shared by the matmul tile kernels.
#pragma once
#include "upir.h"
#include "upir_launch.h"

namespace upir {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int WM, int WN>
__device__ inline void store_c(const MatmulP &p, int64_t row0, int64_t col0, const f32x16 (&acc)[BM / WM / 32][BN / WN / 32]) {
  constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int64_t col = col0 + wn * (BN / WN) + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = row0 + wm * (BM / WM) + i * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
        if (row < p.M && col < p.N) p.C[row * p.ldc + col] = acc[i][j][r];
      }
    }
}

// The same for KG wavefronts on each block: their sums meet in LDS (`red`,
// KG x BM x BN floats, free when this is called), and each thread adds and
// stores elements of C row by row.
template <int BM, int BN, int WM, int WN, int KG>
__device__ inline void store_c_sum(const MatmulP &p, int64_t row0, int64_t col0, const f32x16 (&acc)[BM / WM / 32][BN / WN / 32],
                                   float *red) {
  constexpr int FM = BM / WM / 32, FN = BN / WN / 32, NTH = WM * WN * KG * 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kg = wave / (WM * WN), wt = wave % (WM * WN), wm = wt / WN, wn = wt % WN;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wm * (BM / WM) + i * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
        red[(kg * BM + row) * BN + wn * (BN / WN) + j * 32 + (lane & 31)] = acc[i][j][r];
      }
  __syncthreads();
  for (int e = threadIdx.x; e < BM * BN; e += NTH) {
    float s = red[e];
#pragma unroll
    for (int h = 1; h < KG; ++h) s += red[h * BM * BN + e];
    const int64_t row = row0 + e / BN, col = col0 + e % BN;
    if (row < p.M && col < p.N) p.C[row * p.ldc + col] = s;
  }
}

// Tiles owned by this team under the tiled schedule.
template <class F>
__device__ inline void for_team_tiles(const SchedK &S, F &&f) {
  const int team = xcd_team(blockIdx.x, gridDim.x);
  if (S.policy == POL_STATIC) {
    int64_t lo, hi;
    block_range(S.ntiles, S.T, team, lo, hi);
    for (int64_t m = lo; m < hi; ++m) f(m);
  } else {
    const int64_t c = S.chunk;
    for (int64_t m0 = (int64_t)team * c; m0 < S.ntiles; m0 += (int64_t)S.T * c)
      for (int64_t m = m0; m < m0 + c && m < S.ntiles; ++m) f(m);
  }
}

template <auto K>
static hipError_t go_mm(const MatmulP &p, const SchedK &S, size_t lds, hipStream_t st) {
  const hipError_t e = raise_lds<K>(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(K, dim3(S.T), dim3(S.U), lds, st, p, S);
  return hipGetLastError();
}

}  // namespace upir
