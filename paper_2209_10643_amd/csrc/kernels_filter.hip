// 7 x 7 filter loop on tiles (gfx950).
//
// Paper: sec. 6.2's stencil kernel ("filter size 7" on N x N; its source is
// not printed).
#include "upir_launch.h"

namespace upir {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(4))) float const_float;  // read through the scalar cache

// Tiles of TH rows x 256 columns, anchored at multiples of (TH, 256), go to
// teams by the schedule. The team brings the tile's input, three more rows
// and columns on each side, into LDS with 16-byte loads (any pitch and
// alignment); wavefront w then computes a run of ceil(rows / wavefronts)
// rows and lane l columns 4l .. 4l+3, up to four rows together: each of the
// ten values an input row gives a lane is read from LDS once and feeds every
// output row it belongs to. An output receives filter row m = 0..6 in that
// order, and within a row n = 0..6, so its value is the definition's fused
// multiply-add chain.
//
// What bounds it: the 49 fused multiply-adds of a point (2048 x 2048: 5.2 us
// at the vector rate). The weights are scalars (an operand of each
// multiply-add, no vector registers), and there is no branch and no register
// move between the multiply-adds. The former kernel kept the weights and
// seven rotating output rows in vector registers, passed columns between
// lanes and waited for memory once per four input rows: 19.7 us for 2048 x
// 2048 and 9 us for any small grid, against 13.0 and 5 here (8192 x 8192: 156
// and 136).
constexpr int F7_W = 256;            // tile width (points)
constexpr int F7_PITCH = F7_W + 8;   // floats per LDS row: columns -3 .. 260 of the tile

template <int R>
__device__ __forceinline__ void f7_rows(const float *t, const float (&w)[49], float (&acc)[R][4]) {
#pragma unroll
  for (int o = 0; o < R; ++o)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[o][q] = 0.0f;
  // one input row ahead is read from LDS, no more: the fence keeps the
  // compiler from reading them all first (and spilling them)
  struct Row {
    f32x4 a, b;
    f32x2 c;
  };
  auto load = [&](int r) {
    const float *x = t + r * F7_PITCH;
    return Row{*(const f32x4 *)x, *(const f32x4 *)(x + 4), *(const f32x2 *)(x + 8)};
  };
  Row cur = load(0);
#pragma unroll
  for (int r = 0; r < R + 6; ++r) {
    const Row next = load(r < R + 5 ? r + 1 : r);
    const float s[10] = {cur.a.x, cur.a.y, cur.a.z, cur.a.w, cur.b.x, cur.b.y, cur.b.z, cur.b.w, cur.c.x, cur.c.y};
#pragma unroll
    for (int o = 0; o < R; ++o) {
      const int m = r - o;
      if (m < 0 || m > 6) continue;
#pragma unroll
      for (int n = 0; n < 7; ++n)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[o][q] = __builtin_fmaf(w[m * 7 + n], s[q + n], acc[o][q]);
    }
    cur = next;
    __builtin_amdgcn_sched_barrier(0);
  }
}

__global__ void __launch_bounds__(1024) k_filter7_tile(LoopK L, SchedK S, Filter7P p, RedK R) {
  extern __shared__ __attribute__((aligned(16))) float tile[];
  const int lane = threadIdx.x % WAVE, NW = blockDim.x / WAVE;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int TH = S.tile[0], ld = (int)p.ld;
  const int team = xcd_team(blockIdx.x, gridDim.x);
  const int64_t ilo = L.lb[0], ihi = L.lb[0] + L.cnt[0], jlo = L.lb[1], jhi = L.lb[1] + L.cnt[1];
  // first and last element that any tile reads
  const float *const gfirst = p.src + (ilo - 3) * p.ld + jlo - 3, *const glast = p.src + (ihi + 2) * p.ld + jhi + 2;
  // this team's tiles: runs of `run` from `m0` on, every `stride`
  int64_t m0, run, stride;
  if (S.policy == POL_STATIC) {
    block_range(S.ntiles, S.T, team, m0, run);
    run -= m0;
    stride = S.ntiles;
  } else {
    m0 = (int64_t)team * S.chunk;
    run = S.chunk;
    stride = (int64_t)S.T * S.chunk;
  }
  bool again = false;
#pragma nounroll
  for (; m0 < S.ntiles; m0 += stride)
#pragma nounroll
    for (int64_t m = m0; m < m0 + run && m < S.ntiles; ++m) {
      const int64_t mi = quot(m, S.nt[1]), ti = S.t0[0] + mi, tj = S.t0[1] + (m - mi * S.nt[1]);
      const int64_t i0 = ti * TH, j0 = tj * F7_W;
      const int64_t ra = i0 > ilo ? i0 : ilo, rb = i0 + TH < ihi ? i0 + TH : ihi;  // rows of the tile in the box
      const int n = (int)(rb - ra), nin = n + 6;
      // tile columns written [wlo, whi) and read [wlo - 3, whi + 2]
      const int wlo = (int)((j0 > jlo ? j0 : jlo) - j0), whi = (int)((j0 + F7_W < jhi ? j0 + F7_W : jhi) - j0);
      if (again) __syncthreads();  // the previous tile's readers are done
      again = true;
      // Input rows ra - 3 .. rb + 2, columns -3 .. 260 of the tile, in
      // vectors of four through a buffer resource that ends at glast and
      // starts at the tile's first element, or at gfirst if that is later:
      // nothing outside [gfirst, glast] is touched, and what lies inside it
      // is this array's. Columns that are not read hold whatever is there.
      const float *const t0 = p.src + (ra - 3) * p.ld + j0 - 3;
      const float *const base = t0 < gfirst ? gfirst : t0;
      const int shift = (int)(base - t0);
      const int64_t extent = 4 * (glast + 1 - base);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void *)base, (short)0, (int)(extent < 0x7FFFFFF0 ? extent : 0x7FFFFFF0), 0x00020000);
      constexpr int VR = F7_PITCH / 4;  // vectors per row
      constexpr int LG = 6;  // vectors in flight per thread: 22 input rows of a 16-row tile on 256 threads
      const int total = nin * VR;
#pragma nounroll
      for (int e0 = threadIdx.x; e0 < total; e0 += LG * (int)blockDim.x) {
        f32x4 v[LG];
#pragma unroll
        for (int u = 0; u < LG; ++u) {
          const int e = e0 + u * (int)blockDim.x, r = e / VR, c = e - r * VR;
          const uint32_t o = 4u * (uint32_t)(r * ld + 4 * c - shift);  // a vector that starts before base wraps: zero
          v[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, e < total ? o : 0x80000000u, 0, 0));
        }
#pragma unroll
        for (int u = 0; u < LG; ++u) {
          const int e = e0 + u * (int)blockDim.x;
          if (e < total) *(f32x4 *)(tile + 4 * e) = v[u];
        }
      }
      __syncthreads();
      // A vector that straddles gfirst or glast came back as zeros: its
      // elements that are read are in the first row from column wlo - 3 on or
      // in the last row up to column whi + 2, and are loaded one by one.
      const int ca = wlo / 4, cb = (whi + 5) / 4;  // vectors of columns wlo - 3 and whi + 2
      if (shift > 0 || t0 + (int64_t)(nin - 1) * p.ld + 4 * cb + 3 > glast) {
        if (threadIdx.x < 8) {
          const bool last = threadIdx.x >= 4;
          const int x = 4 * (last ? cb : ca) + (int)(threadIdx.x & 3), r = last ? nin - 1 : 0;
          if (x >= wlo && x <= whi + 5) tile[r * F7_PITCH + x] = t0[(int64_t)r * p.ld + x];
        }
        __syncthreads();
      }
      // the weights are read here, in the phase that uses them: kept from the
      // start of the kernel they and the loop's description do not fit the
      // scalar registers
      const_float *wp = (const_float *)p.w;
      __asm__ volatile("" : "+s"(wp));
      float wk[49];
#pragma unroll
      for (int i = 0; i < 49; ++i) wk[i] = wp[i];
      const int SH = (n + NW - 1) / NW, s1 = w * SH + SH < n ? w * SH + SH : n;
      const int c0 = 4 * lane;
      float *const out0 = p.dst + ra * p.ld + j0 + c0;
      const bool whole = c0 >= wlo && c0 + 3 < whi;
      auto rows = [&](auto rr, int s) {
        constexpr int RR = decltype(rr)::value;
        float acc[RR][4];
        f7_rows<RR>(tile + s * F7_PITCH + c0, wk, acc);
#pragma unroll
        for (int o = 0; o < RR; ++o) {
          float *out = out0 + (int64_t)(s + o) * p.ld;
          if (whole) {
            __builtin_nontemporal_store(f32x4{acc[o][0], acc[o][1], acc[o][2], acc[o][3]}, (f32x4u *)out);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (c0 + q >= wlo && c0 + q < whi) out[q] = acc[o][q];
          }
        }
      };
      int s = w * SH;
#pragma nounroll
      for (; s + 4 <= s1; s += 4) rows(std::integral_constant<int, 4>{}, s);
      if (s + 2 <= s1) {
        rows(std::integral_constant<int, 2>{}, s);
        s += 2;
      }
      if (s < s1) rows(std::integral_constant<int, 1>{}, s);
    }
  fold_hook(R);
}

// The schedules and boxes the tiles run, whatever the grid's pitch and
// alignment.
bool filter7_strips_support(const Filter7P &p, const LoopK &L, const SchedK &S) {
  if (L.nd != 2 || !S.tiled || S.dist != DIST_TU) return false;
  if (L.step[0] != 1 || L.step[1] != 1) return false;
  if (S.tile[1] != F7_W) return false;
  const int th = S.tile[0];
  if (th != 4 && th != 8 && th != 16 && th != 32 && th != 64) return false;
  if (S.U % WAVE != 0 || S.U < WAVE) return false;
  if (S.policy != POL_STATIC && S.policy != POL_CHUNK) return false;
  if (L.lb[1] < 3 || L.lb[0] < 3) return false;  // reads at lb-3 stay in the array
  if ((int64_t)(th + 8) * p.ld * 4 >= (1LL << 31)) return false;  // 32-bit byte offsets within a tile
  return true;
}
bool filter7_tile_supports(const Filter7P &p, const LoopK &L, const SchedK &S) {
  return filter7_strips_support(p, L, S) && (p.ld % 4) == 0 && ((uintptr_t)p.src % 16) == 0 && ((uintptr_t)p.dst % 16) == 0;
}

hipError_t launch_filter7_tile(const Filter7P &p, const LoopK &L, const SchedK &S, const RedK &R, hipStream_t st) {
  const size_t lds = (size_t)(S.tile[0] + 6) * F7_PITCH * 4;
  const hipError_t e = raise_lds<k_filter7_tile>((64 + 6) * F7_PITCH * 4);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_filter7_tile, dim3(S.T), dim3(S.U), lds, st, L, S, p, R);
  return hipGetLastError();
}

}  // namespace upir
