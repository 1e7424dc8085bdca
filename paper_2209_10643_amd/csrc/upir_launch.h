// Host-side launchers of the HIP kernels (internal to libupir).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "once_per_device.h"
#include "upir_kern.h"

namespace upir {

// Raises kernel K's limit of dynamic LDS to `lds` bytes on the current device.
template <auto K>
inline hipError_t raise_lds(size_t lds) {
  static OncePerDevice once;
  int dev = -1;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return once.run(dev, [&] { return hipFuncSetAttribute((const void *)K, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); });
}

// Kernel variants a loop can run with, as upir_loop_resolve reports them. The
// tiled ones are reported for operands on 16-byte boundaries and rows of whole
// 16 bytes. V_GENERIC and V_DYNAMIC say that launch_generic chooses: tiles of
// the same schedules whose operands are not so aligned run the same strip,
// filter and float32 matrix kernels, AXPY and SUM under any policy but the
// chunk-4 stream's the team streams, and everything else the schedule-exact
// kernels.
enum Variant : int32_t {
  V_GENERIC = 0,      // chosen by launch_generic
  V_STREAM4 = 1,      // 1-D, static chunk 4, vectorised (AXPY, SUM f32, COVER)
  V_JACOBI_TILE = 2,  // tiled Jacobi, wavefront strips
  V_MATVEC_WAVE = 3,  // one wavefront per row
  V_MATMUL_MFMA = 4,  // MFMA tiles over C
  V_DYNAMIC = 5,      // dynamic / guided claims, chosen by launch_generic
  V_FILTER7_TILE = 6, // tiled 7 x 7 filter, wavefront strips
};

// Body payloads with device pointers already resolved.
struct AxpyP { float a; const float *x; float *y; };
struct SumP { const void *x; int32_t dtype; };
struct JacobiP { const float *src; float *dst; int64_t ld; };
struct MatmulP {
  const float *A, *B; float *C; int64_t M, N, K, lda, ldb, ldc;
  uint16_t *ah, *al, *bh, *bl;  // bfloat16 workspace (bh/bl stored transposed: N x K)
  int32_t kind;                 // 4 = f32, 5 = bf16, 6 = split3
  int32_t panel;                // workspace layout: 0 rows of K; 1 k-panels of 32; 2 rows of K rounded up to 32 (kernels_matmul.hip)
};
// Workspace k extent: K rounded up to the 32-wide k-panels.
__host__ __device__ inline int64_t mm_kpad(int64_t K) { return (K + 31) / 32 * 32; }
struct MatvecP { const float *A; const float *x; float *y; int64_t cols, lda; };
struct OwnerP { int32_t *out; };
struct CoverP { int32_t *count; };
struct Filter7P { const float *src; float *dst; const float *w; int64_t ld; };

hipError_t launch_generic(int32_t body, const void *payload, const LoopK &L, const SchedK &S,
                          const RedK &R, hipStream_t st);
hipError_t launch_stream4(int32_t body, const void *payload, const LoopK &L, const SchedK &S,
                          const RedK &R, hipStream_t st);
// AXPY and SUM under schedules whose units own runs of consecutive iterations.
hipError_t launch_team_stream(int32_t body, const void *payload, const LoopK &L, const SchedK &S,
                              const RedK &R, hipStream_t st);
bool team_stream_body(int32_t body, int32_t sum_dtype, int32_t op);
bool team_stream_supports(int32_t body, const void *payload, const LoopK &L, const SchedK &S, const RedK &R);
hipError_t launch_fold(const FoldK &F, hipStream_t st);
hipError_t launch_jacobi_tile(const JacobiP &p, const LoopK &L, const SchedK &S, const RedK &R,
                              hipStream_t st);
hipError_t launch_filter7_tile(const Filter7P &p, const LoopK &L, const SchedK &S, const RedK &R,
                               hipStream_t st);
hipError_t launch_matvec_wave(const MatvecP &p, const LoopK &L, const SchedK &S, const RedK &R,
                              hipStream_t st);
// MFMA matmul over tiles of C (tile[0] x tile[1]); S gives the team schedule over tiles.
hipError_t launch_matmul_mfma(const MatmulP &p, const LoopK &L, const SchedK &S, hipStream_t st);
bool matmul_mfma_supports(const MatmulP &p, const LoopK &L, const SchedK &S);
// float32 tiles for operands the above leaves out (any pitch and alignment); the schedule decides.
bool mm_f32_supports(const MatmulP &p, const LoopK &L, const SchedK &S);
hipError_t launch_mm_f32(const MatmulP &p, const SchedK &S, hipStream_t st);
// bfloat16 tiles that read the float32 operands themselves (no pre-pass).
bool matmul_direct(const MatmulP &p, const SchedK &S);
hipError_t launch_mm_direct(const MatmulP &p, const SchedK &S, hipStream_t st);
// BF16 pre-pass: A (M x K) -> ah, al; B (K x N) -> bh, bl transposed (N x K).
hipError_t launch_bf16_split(const MatmulP &p, bool need_lo, hipStream_t st);
// The 256 x 256 four-wavefront bfloat16 tile (it reads the k-panel workspace layout).
bool matmul_wide(const MatmulP &p, const SchedK &S);

// Tiled Jacobi and filter kernels: what they run at all, and what is
// reported as the tiled variant (16-byte aligned rows as well).
bool jacobi_strips_support(const JacobiP &p, const LoopK &L, const SchedK &S);
bool filter7_strips_support(const Filter7P &p, const LoopK &L, const SchedK &S);
bool jacobi_tile_supports(const JacobiP &p, const LoopK &L, const SchedK &S);
bool filter7_tile_supports(const Filter7P &p, const LoopK &L, const SchedK &S);

}  // namespace upir
