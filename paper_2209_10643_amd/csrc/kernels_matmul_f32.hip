// float32 matmul loop C = A B on MFMA tiles (gfx950), any sizes and pitches.
//
// Paper: sec. 6.2 names a matrix multiplication kernel among its four
// offloaded loops. v_mfma_f32_32x32x2f32 reads A (M x K) and B (K x N)
// directly.
#include "matmul_tiles.h"

namespace upir {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// One BM x BN tile of C by WM x WN x KG wavefronts: a WM x WN grid over the
// tile, KG of them deep. The KG wavefronts on the same block take different
// k of every step and their sums are added at the end (k group 0 first), so
// that a 64 x 64 or 32 x 32 tile still gives each SIMD two wavefronts; with
// one wavefront per SIMD every LDS and memory latency of the step is exposed.
//
// Operands go through registers into two LDS stages of BK (one barrier per
// step), fetched at least two steps ahead: a step of a small tile is too
// short to cover an L2 access. The loads of the full steps have no branch
// around them: with one, the compiler waited for every load in flight before
// a step's LDS writes (4096^3: 1,100 against 1,032 us, 133 TFLOP/s; 1,298 us
// with one step of prefetch). The limit is the matrix cores' float32 rate.
// Vectors of four are loaded at any alignment, so a pitch that is not a
// multiple of four needs no other kernel. Rows past M are read as row M - 1
// and columns past N as columns before N: they reach only elements of C that
// are not stored. k past K is read as zero (the last step alone tests it; its
// loads are issued first and wait in registers).
template <int BM, int BN, int WM, int WN, int KG, int BK>
__global__ void __launch_bounds__(WM * WN * KG * 64) k_mm_f32(MatmulP p, SchedK S) {
  constexpr int NTH = WM * WN * KG * 64;
  constexpr int PA = BK + 4;  // floats per A row in LDS
  constexpr int PB = BN + 8;  // floats per B row (k) in LDS
  constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
  constexpr int CA = BM * (BK / 4) / NTH, CB = BK * (BN / 4) / NTH;
  static_assert(BM * (BK / 4) % NTH == 0 && BK * (BN / 4) % NTH == 0, "chunk split");
  static_assert(BK % (8 * KG) == 0, "k groups");
  constexpr int STAGEF = BM * PA + BK * PB;  // floats per LDS stage (two stages)
  extern __shared__ __attribute__((aligned(16))) float ldsf[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kg = wave / (WM * WN), wt = wave % (WM * WN), wm = wt / WN, wn = wt % WN;
  const int64_t K = p.K;

  for_team_tiles(S, [&](int64_t m) {
    const int64_t mi = quot(m, S.nt[1]), row0 = (S.t0[0] + mi) * BM, col0 = (S.t0[1] + (m - mi * S.nt[1])) * BN;
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};
    // this thread's vectors: a row of A and four of its k; a k of B and four
    // columns, moved left by sh where they would pass column N - 1
    const float *pa[CA], *pb[CB];
    int sh[CB];
    const bool wide = p.N >= 4;
#pragma unroll
    for (int q = 0; q < CA; ++q) {
      const int c = tid + q * NTH, r = c / (BK / 4), kc = c % (BK / 4);
      const int64_t gr = row0 + r < p.M ? row0 + r : p.M - 1;
      pa[q] = p.A + gr * p.lda + kc * 4;
    }
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const int c = tid + q * NTH, r = c / (BN / 4), nc = c % (BN / 4);
      const int64_t gc = col0 + nc * 4, cc = wide && gc + 4 > p.N ? p.N - 4 : gc;
      sh[q] = gc - cc < 4 ? (int)(gc - cc) : 3;  // 0 unless the vector was moved
      pb[q] = p.B + r * p.ldb + (wide ? cc : 0);
    }
    auto shift = [](f32x4v v, int s) {
      return f32x4v{s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w, s == 0 ? v.y : s == 1 ? v.z : v.w,
                    s == 0 ? v.z : v.w, v.w};
    };
    // step i of the full ones: no branch, so that the compiler's count of
    // loads in flight stays exact and a step waits for its own loads only
    auto fetch = [&](int i, f32x4v (&ra)[CA], f32x4v (&rb)[CB]) {
      const int64_t k0 = (int64_t)i * BK;
#pragma unroll
      for (int q = 0; q < CA; ++q) ra[q] = *(const f32x4u *)(pa[q] + k0);
#pragma unroll
      for (int q = 0; q < CB; ++q) rb[q] = *(const f32x4u *)(pb[q] + k0 * p.ldb);
    };
    // the step at k0 when it passes K, or C has fewer than four columns
    auto fetch_tail = [&](int64_t k0, f32x4v (&ra)[CA], f32x4v (&rb)[CB]) {
#pragma unroll
      for (int q = 0; q < CA; ++q) {
        const int64_t gk = k0 + (tid + q * NTH) % (BK / 4) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) ra[q][e] = gk + e < K ? pa[q][k0 + e] : 0.0f;
      }
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        const int64_t gk = k0 + (tid + q * NTH) / (BN / 4);
        const int64_t gc = wide ? 0 : col0 + (tid + q * NTH) % (BN / 4) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          rb[q][e] = gk < K && (wide || gc + e < p.N) ? pb[q][k0 * p.ldb + gc + e] : 0.0f;
      }
    };
    auto stage = [&](int buf, f32x4v (&ra)[CA], f32x4v (&rb)[CB]) {
      float *sA = ldsf + buf * STAGEF, *sB = sA + BM * PA;
#pragma unroll
      for (int q = 0; q < CA; ++q) {
        const int c = tid + q * NTH, r = c / (BK / 4), kc = c % (BK / 4);
        *(f32x4v *)(sA + r * PA + kc * 4) = ra[q];
      }
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        const int c = tid + q * NTH, r = c / (BN / 4), nc = c % (BN / 4);
        *(f32x4v *)(sB + r * PB + nc * 4) = shift(rb[q], sh[q]);
      }
    };
    const int g = lane >> 5;
    // one wavefront's operands of a step, and its matrix instructions [lo, hi)
    constexpr int NU = BK / KG / 8;  // groups of eight k
    struct Frag {
      f32x4v a[NU][FM];
      float b[NU][4][FN];
    };
    auto read = [&](int buf, Frag &f) {
      const float *sA = ldsf + buf * STAGEF, *sB = sA + BM * PA;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int kk = kg * (BK / KG) + 8 * u;
#pragma unroll
        for (int i = 0; i < FM; ++i)
          f.a[u][i] = *(const f32x4v *)(sA + (wm * (BM / WM) + i * 32 + (lane & 31)) * PA + kk + 4 * g);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int j = 0; j < FN; ++j) f.b[u][s][j] = sB[(kk + 4 * g + s) * PB + wn * (BN / WN) + j * 32 + (lane & 31)];
      }
    };
    auto mfmas = [&](const Frag &f, int lo, int hi) {
#pragma unroll
      for (int q = lo; q < hi; ++q) {
        // group g takes k = kk + 4g + s at MFMA step s (same for A and B)
        const int u = q / 4, s = q % 4;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[u][i][s], f.b[u][s][j], acc[i][j], 0, 0, 0);
      }
    };
    // Full steps. Where wavefronts share a block (small tiles), software-
    // pipelined: in phase i the fragments of step i are in registers and feed
    // the matrix cores while those of step i + 1 are read from LDS, step
    // i + 2 goes from registers into the LDS stage that step i was read from,
    // and step i + 4 is fetched (1024^3 on 64 x 64 tiles: 25.4 against 27.5
    // us). The large tiles' fragments leave no registers for a second set:
    // there step i is read and used in one phase, step i + 1 is on its way in
    // registers and step i + 2 is fetched. Past the end the last full step is
    // loaded again and not used.
    const int nfull = wide ? (int)(K / BK) : 0, last = nfull - 1;
    int64_t kt = (int64_t)nfull * BK;
    f32x4v ta[CA], tb[CB];
    if (kt < K) fetch_tail(kt, ta, tb);
    __syncthreads();  // the previous tile's readers are done with both stages
    if (nfull > 0) {
      f32x4v ra0[CA], rb0[CB], ra1[CA], rb1[CB];
      Frag X, Y;
      auto at = [&](int i) { return i < last ? i : last; };
      fetch(0, ra0, rb0);
      fetch(at(1), ra1, rb1);
      stage(0, ra0, rb0);
      int i = 0;
      if constexpr (KG > 1) {
        auto phase = [&](int i, Frag &F, Frag &G, f32x4v (&ra)[CA], f32x4v (&rb)[CB]) {
          __syncthreads();  // step i + 1 is in LDS, everyone's reads of step i are done
          read((i + 1) & 1, G);
          __builtin_amdgcn_sched_barrier(0);
          mfmas(F, 0, 2 * NU);
          __builtin_amdgcn_sched_barrier(0);
          stage(i & 1, ra, rb);
          fetch(at(i + 4), ra, rb);
          __builtin_amdgcn_sched_barrier(0);
          mfmas(F, 2 * NU, 4 * NU);
        };
        fetch(at(2), ra0, rb0);
        stage(1, ra1, rb1);
        fetch(at(3), ra1, rb1);
        __syncthreads();
        read(0, X);
        for (; i + 2 <= nfull; i += 2) {
          phase(i, X, Y, ra0, rb0);
          phase(i + 1, Y, X, ra1, rb1);
        }
        if (i < nfull) mfmas(X, 0, 4 * NU);
      } else {
        auto phase = [&](int i, f32x4v (&ra)[CA], f32x4v (&rb)[CB], f32x4v (&na)[CA], f32x4v (&nb)[CB]) {
          __syncthreads();  // step i is in LDS, everyone's reads of step i - 1 are done
          fetch(at(i + 2), na, nb);
          read(i & 1, X);
          mfmas(X, 0, 4 * NU);
          stage((i + 1) & 1, ra, rb);
        };
        for (; i + 2 <= nfull; i += 2) {
          phase(i, ra1, rb1, ra0, rb0);
          phase(i + 1, ra0, rb0, ra1, rb1);
        }
        if (i < nfull) {
          __syncthreads();
          read(0, X);
          mfmas(X, 0, 4 * NU);
        }
      }
      __syncthreads();
    }
    while (kt < K) {
      stage(0, ta, tb);
      __syncthreads();
      Frag T;
      read(0, T);
      mfmas(T, 0, 4 * NU);
      kt += BK;
      if (kt < K) fetch_tail(kt, ta, tb);
      __syncthreads();
    }
    if constexpr (KG == 1) store_c<BM, BN, WM, WN>(p, row0, col0, acc);
    else store_c_sum<BM, BN, WM, WN, KG>(p, row0, col0, acc, ldsf);
  });
}

template <int BM, int BN, int WM, int WN, int KG, int BK>
static hipError_t go_f32(const MatmulP &p, const SchedK &S, hipStream_t st) {
  // two stages, or the k groups' sums at the end
  constexpr int stages = 2 * (BM * (BK + 4) + BK * (BN + 8)), sums = KG > 1 ? KG * BM * BN : 0;
  return go_mm<k_mm_f32<BM, BN, WM, WN, KG, BK>>(p, S, (stages > sums ? stages : sums) * 4, st);
}

bool mm_f32_supports(const MatmulP &p, const LoopK &L, const SchedK &S) {
  if (p.kind != UPIR_BODY_MATMUL_F32 || L.nd != 2 || !S.tiled || S.dist != DIST_TU) return false;
  if (S.policy != POL_STATIC && S.policy != POL_CHUNK) return false;
  if (L.lb[0] != 0 || L.lb[1] != 0) return false;
  const int bm = S.tile[0], bn = S.tile[1];
  return (bm == 256 && bn == 128 && S.U == 512) || (bm == 128 && bn == 128 && S.U == 256) ||
         (S.U == 512 && ((bm == 64 && (bn == 64 || bn == 128)) || (bm == 32 && bn == 32)));
}

hipError_t launch_mm_f32(const MatmulP &p, const SchedK &S, hipStream_t st) {
  if (S.tile[0] == 256) return go_f32<256, 128, 4, 2, 1, 32>(p, S, st);
  if (S.tile[0] == 128) return go_f32<128, 128, 2, 2, 1, 32>(p, S, st);
  if (S.tile[0] == 64) {
    if (S.tile[1] == 128) return go_f32<64, 128, 2, 2, 2, 32>(p, S, st);
    return go_f32<64, 64, 2, 1, 4, 32>(p, S, st);
  }
  return go_f32<32, 32, 1, 1, 8, 64>(p, S, st);
}

}  // namespace upir
