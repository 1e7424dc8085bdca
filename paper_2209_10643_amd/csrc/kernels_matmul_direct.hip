// bfloat16 and split-bfloat16 matmul loops straight from the float32
// operands (gfx950): small and middle sizes, any pitch and alignment.
//
// Paper: sec. 6.2 names a matrix multiplication kernel among its four
// offloaded loops; the bfloat16 forms are not in the paper.
#include "matmul_tiles.h"

namespace upir {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// One BM x BN tile of C by WM x WN x KG wavefronts (KG of them on the same
// block take different k of every step; their sums meet at the end, k group
// 0 first). A and B are loaded as float32, rounded to bfloat16 (and, for the
// split, into high and low parts) on the way from registers to LDS: the
// pre-pass that the large tiles read their operands from costs two launches
// and a round trip through memory, half or more of a product of this size
// (512^3: 16.9 us with it, most of them latency). What bounds these tiles is
// the operand traffic from L2, twice the bytes of bfloat16 operands, so the
// large products keep the pre-pass.
//
// A lane loads eight consecutive k of a row of A, and eight k of one column
// of B (64 neighbouring columns a wavefront), so that both reach LDS as
// 16-byte chunks of eight k, [row][k] and [column][k]. The tiles with most
// loads for their arithmetic (PAIR) take four k of A at a time, whole rows of
// the tile side by side, and two columns of B together, half the load
// instructions (bfloat16 128 x 128: 2000^3 42.9 -> 37.9 us; the 64 x 128 tile
// is slower with them in bfloat16, 36 against 29 us alone on the chip with K =
// 3072, and faster in the split, 50 against 54). Rows past M and columns past
// N repeat the last one (they reach only elements of C that are not stored);
// k past K is read as zero in the last step, whose loads are issued first and
// wait in registers. The full steps have no branch around their loads.
//
// In phase i the fragments of step i are in registers and feed the matrix
// cores while those of step i + 1 are read from LDS, step i + 2 goes from
// registers into the LDS stage that step i was read from, and step i + 4 is
// fetched. The conversions are dealt out between the matrix instructions, and
// the split takes its high parts' values from the packed words rather than
// converting twice: split, 1000 x 777 by 777 x 1300 24.0 -> 21.9 us, 2000^3
// 66 -> 62. Twice the steps in flight changed nothing.
template <int NPROD, int BM, int BN, int WM, int WN, int KG, int BK>
__global__ void __launch_bounds__(WM * WN * KG * 64) k_mm_direct(MatmulP p, SchedK S) {
  constexpr int NTH = WM * WN * KG * 64;
  constexpr int P = BK + 8;  // halfwords per LDS row
  constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
  // chunks per lane: KA k of a row of A, NB columns by KB k of B
  constexpr bool PAIR = BM == 128 || (BN == 128 && NPROD == 3);
  constexpr int KA = PAIR ? 4 : 8, NB = PAIR ? 2 : 1, KB = PAIR ? BN * BK / 2 / NTH : 8;
  constexpr int CA = BM * BK / KA / NTH, CB = BN * BK / (NB * KB) / NTH;
  static_assert(CA * KA * NTH == BM * BK && CB * NB * KB * NTH == BN * BK && (KB == 4 || KB == 8), "chunk split");
  static_assert(BK % (16 * KG) == 0, "k groups");
  constexpr int NL = NPROD == 3 ? 2 : 1;     // high parts, low parts
  constexpr int STAGE = NL * (BM + BN) * P;  // halfwords per LDS stage: A, B, then their low parts
  extern __shared__ __attribute__((aligned(16))) uint16_t ldsd[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kg = wave / (WM * WN), wt = wave % (WM * WN), wm = wt / WN, wn = wt % WN;
  const int g = lane >> 5;
  const int64_t K = p.K;

  for_team_tiles(S, [&](int64_t m) {
    const int64_t mi = quot(m, S.nt[1]), row0 = (S.t0[0] + mi) * BM, col0 = (S.t0[1] + (m - mi * S.nt[1])) * BN;
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};
    const float *pa[CA], *pb[CB];
#pragma unroll
    for (int q = 0; q < CA; ++q) {
      const int c = tid + q * NTH, r = c / (BK / KA), kc = c % (BK / KA);
      const int64_t gr = row0 + r < p.M ? row0 + r : p.M - 1;
      pa[q] = p.A + gr * p.lda + KA * kc;
    }
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const int c = tid + q * NTH, n = NB * (c % (BN / NB)), kc = c / (BN / NB);
      const int64_t gc = col0 + n < p.N ? col0 + n : p.N - 1;
      pb[q] = p.B + (int64_t)(KB * kc) * p.ldb + gc;
    }
    struct Regs {
      float a[CA][KA], b[CB][NB][KB];
    };
    auto fetch = [&](int i, Regs &r) {
      const int64_t k0 = (int64_t)i * BK;
#pragma unroll
      for (int q = 0; q < CA; ++q)
#pragma unroll
        for (int h = 0; h < KA; h += 4) {
          const f32x4v v = *(const f32x4u *)(pa[q] + k0 + h);
#pragma unroll
          for (int e = 0; e < 4; ++e) r.a[q][h + e] = v[e];
        }
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        const float *b = pb[q] + k0 * p.ldb;
#pragma unroll
        for (int e = 0; e < KB; ++e) {
          if constexpr (PAIR) {
            const f32x2u v = *(const f32x2u *)(b + e * p.ldb);
            r.b[q][0][e] = v[0];
            r.b[q][1][e] = v[1];
          } else {
            r.b[q][0][e] = b[e * p.ldb];
          }
        }
      }
    };
    auto fetch_tail = [&](int64_t k0, Regs &r) {
#pragma unroll
      for (int q = 0; q < CA; ++q) {
        const int64_t gk = k0 + KA * ((tid + q * NTH) % (BK / KA));
#pragma unroll
        for (int e = 0; e < KA; ++e) r.a[q][e] = gk + e < K ? pa[q][k0 + e] : 0.0f;
      }
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        const int c = tid + q * NTH;
        const int64_t gk = k0 + KB * (c / (BN / NB));
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          const int dx = col0 + NB * (c % (BN / NB)) + x < p.N ? x : 0;
#pragma unroll
          for (int e = 0; e < KB; ++e) r.b[q][x][e] = gk + e < K ? pb[q][(k0 + e) * p.ldb + dx] : 0.0f;
        }
      }
    };
    // consecutive k to LDS as bfloat16 (round to nearest even), and their
    // remainders as bfloat16 into the low part
    auto put = [&](uint16_t *hi, uint16_t *lo, const auto &x) {
      constexpr int KV = sizeof(x) / sizeof(x[0]);
      typedef uint32_t W __attribute__((ext_vector_type(KV / 2)));
      W h, l;
#pragma unroll
      for (int e = 0; e < KV; e += 2) {
        const bf16x2 w = {(__bf16)x[e], (__bf16)x[e + 1]};
        uint32_t u = __builtin_bit_cast(uint32_t, w);
        if (NPROD == 3) {
          __asm__("" : "+v"(u));  // the packed word's halves below, not two more conversions
          const float f0 = __builtin_bit_cast(float, u << 16), f1 = __builtin_bit_cast(float, u & 0xffff0000u);
          const bf16x2 v = {(__bf16)(x[e] - f0), (__bf16)(x[e + 1] - f1)};
          l[e / 2] = __builtin_bit_cast(uint32_t, v);
        }
        h[e / 2] = u;
      }
      *(W *)hi = h;
      if (NPROD == 3) *(W *)lo = l;
    };
    auto stage = [&](int buf, const Regs &r) {
      uint16_t *sA = ldsd + buf * STAGE, *sB = sA + BM * P;
      constexpr int LO = (BM + BN) * P;
#pragma unroll
      for (int q = 0; q < CA; ++q) {
        const int c = tid + q * NTH, o = c / (BK / KA) * P + KA * (c % (BK / KA));
        put(sA + o, sA + LO + o, r.a[q]);
      }
#pragma unroll
      for (int q = 0; q < CB; ++q)
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          const int c = tid + q * NTH, o = (NB * (c % (BN / NB)) + x) * P + KB * (c / (BN / NB));
          put(sB + o, sB + LO + o, r.b[q][x]);
        }
    };
    constexpr int NU = BK / KG / 16;  // groups of sixteen k per wavefront and step
    struct Frag {
      bf16x8 a[NL][NU][FM], b[NL][NU][FN];
    };
    auto read = [&](int buf, Frag &f) {
      const uint16_t *sA = ldsd + buf * STAGE, *sB = sA + BM * P;
#pragma unroll
      for (int h = 0; h < NL; ++h)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          const int kk = kg * (BK / KG) + 16 * u + 8 * g;
#pragma unroll
          for (int i = 0; i < FM; ++i)
            f.a[h][u][i] = *(const bf16x8 *)(sA + h * (BM + BN) * P + (wm * (BM / WM) + i * 32 + (lane & 31)) * P + kk);
#pragma unroll
          for (int j = 0; j < FN; ++j)
            f.b[h][u][j] = *(const bf16x8 *)(sB + h * (BM + BN) * P + (wn * (BN / WN) + j * 32 + (lane & 31)) * P + kk);
        }
    };
    auto mfmas = [&](const Frag &f) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            if constexpr (NPROD == 3) {
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[1][u][i], f.b[0][u][j], acc[i][j], 0, 0, 0);
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[0][u][i], f.b[1][u][j], acc[i][j], 0, 0, 0);
            }
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[0][u][i], f.b[0][u][j], acc[i][j], 0, 0, 0);
          }
    };
    // The second column of a pair may lie one element past the end of a row of
    // B, in a tile that crosses column N: such a tile takes the last row in its
    // last step, whose loads are guarded.
    const int nfull = (int)((PAIR && col0 + BN > p.N ? K - 1 : K) / BK), last = nfull - 1;
    const int64_t kt = (int64_t)nfull * BK;
    Regs t;
    if (kt < K) fetch_tail(kt, t);
    __syncthreads();  // the previous tile's readers are done with LDS
    if (nfull > 0) {
      Regs r0, r1;
      Frag X, Y;
      auto at = [&](int i) { return i < last ? i : last; };  // past the end: the last step again, not used
      auto phase = [&](int i, Frag &F, Frag &G, Regs &r) {
        __syncthreads();  // step i + 1 is in LDS, everyone's reads of step i are done
        read((i + 1) & 1, G);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(F);
        stage(i & 1, r);
        fetch(at(i + 4), r);
        // a matrix instruction, then what the vector pipe and LDS do beside it
        // (bfloat16 64 x 128 is 2% faster in the compiler's own order)
        if constexpr (PAIR || BN < 128) {
          constexpr int NM = NU * FM * FN * NPROD;
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, (NPROD == 3 ? 6 : 1) * (BM + BN) * BK / NTH / 2 / NM + 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x200, (NL * (CA + NB * CB) + NM - 1) / NM, 0);
          }
        }
      };
      fetch(0, r0);
      fetch(at(1), r1);
      stage(0, r0);
      fetch(at(2), r0);
      stage(1, r1);
      fetch(at(3), r1);
      __syncthreads();
      read(0, X);
      int i = 0;
      for (; i + 2 <= nfull; i += 2) {
        phase(i, X, Y, r0);
        phase(i + 1, Y, X, r1);
      }
      if (i < nfull) mfmas(X);
      __syncthreads();
    }
    if (kt < K) {
      Frag T;
      stage(0, t);
      __syncthreads();
      read(0, T);
      mfmas(T);
      __syncthreads();
    }
    if constexpr (KG == 1) store_c<BM, BN, WM, WN>(p, row0, col0, acc);
    else store_c_sum<BM, BN, WM, WN, KG>(p, row0, col0, acc, (float *)ldsd);
  });
}

template <int NPROD, int BM, int BN, int WM, int WN, int KG, int BK>
static hipError_t go_direct(const MatmulP &p, const SchedK &S, hipStream_t st) {
  // two stages, or the k groups' sums at the end
  constexpr int stages = 2 * (NPROD == 3 ? 2 : 1) * (BM + BN) * (BK + 8) * 2, sums = KG > 1 ? KG * BM * BN * 4 : 0;
  return go_mm<k_mm_direct<NPROD, BM, BN, WM, WN, KG, BK>>(p, S, stages > sums ? stages : sums, st);
}

// 128 x 128 on 512 units (on 256 units that tile reads the pre-pass workspace).
bool matmul_direct(const MatmulP &p, const SchedK &S) {
  const int bm = S.tile[0], bn = S.tile[1];
  return p.kind != UPIR_BODY_MATMUL_F32 && S.U == 512 &&
         ((bm == 128 && bn == 128) || (bm == 64 && (bn == 64 || bn == 128)) || (bm == 32 && bn == 32));
}

template <int NPROD>
static hipError_t go_direct_tile(const MatmulP &p, const SchedK &S, hipStream_t st) {
  if (S.tile[0] == 128) return go_direct<NPROD, 128, 128, 2, 4, 1, 32>(p, S, st);
  if (S.tile[0] == 64) {
    if (S.tile[1] == 128) return go_direct<NPROD, 64, 128, 2, 2, 2, 64>(p, S, st);
    return go_direct<NPROD, 64, 64, 2, 1, 4, 64>(p, S, st);
  }
  return go_direct<NPROD, 32, 32, 1, 1, 8, 128>(p, S, st);
}

hipError_t launch_mm_direct(const MatmulP &p, const SchedK &S, hipStream_t st) {
  return p.kind == UPIR_BODY_MATMUL_SPLIT3 ? go_direct_tile<3>(p, S, st) : go_direct_tile<1>(p, S, st);
}

}  // namespace upir
