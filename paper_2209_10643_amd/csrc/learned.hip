// Schedule selection for schedule(auto): exhaustive tuner and a learned
// cost model.
//
// The paper's loop_parallel grammar (sec. 3.2) offers schedule(auto), which
// leaves the schedule to the implementation. Here AUTO resolves, in order,
// to the tuner's measured best for the loop's shape, to the cost model's
// choice, and to the library default.
//
//  * Tuner: every candidate (teams, units, chunk, tile) of a loop is timed
//    with HIP events on scratch copies of the loop's read-write outputs; one
//    row per (loop, candidate) goes into the context's timing table.
//  * Cost model: an MLP 32 -> 64 -> 64 -> 1 (float32) predicts log2(time in
//    microseconds) from 32 features of (loop, candidate). It is trained on
//    the timing table by this file's own kernels: one over the rows (forward
//    and backward, each wavefront summing its rows' gradients), one over the
//    parameters (sum over the wavefronts, Adam); forward passes of very many
//    rows have one of their own.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "runtime_internal.h"

using namespace upir;

namespace {

constexpr int F = 32, H1 = 64, H2 = 64;
constexpr int O_W1 = 0, O_B1 = O_W1 + H1 * F, O_W2 = O_B1 + H1, O_B2 = O_W2 + H2 * H1, O_W3 = O_B2 + H2,
              O_B3 = O_W3 + H2, NP = O_B3 + 1;
static_assert(NP == UPIR_MLP_PARAMS, "parameter count");
constexpr int MLP_PART = (NP + 1 + 63) / 64 * 64;  // floats per wavefront: gradients, squared error
constexpr int MLP_WAVES = 512;                     // wavefronts of a training step at most
constexpr int64_t MLP_MANY = 96 << 10;             // rows from which a forward pass takes one a thread
static_assert(H1 == 64 && H2 == 64 && O_W2 % 4 == 0, "a lane is a hidden unit; rows of weights are read by four");

// ------------------------------------------------------------------ kernels
// Rows of the network, forward and (TRAIN) backward. A workgroup is one
// wavefront and lane j is hidden unit j of both layers: it keeps row j of W1
// and W2 (and column j of W2) in registers and takes rows of X from a
// grid-strided loop, MLP_R at a time. A row's values, the first layer's
// activations and the second's deltas reach every lane through LDS, four per
// read. Pre-activations are sums over k in order, from
// the bias, as a thread per row computed them. TRAIN also sums this
// wavefront's gradients in registers (row j of both weight matrices) and
// leaves them, and its squared error, as row blockIdx.x of `part`.
//
// At these sizes (6,208 multiply-adds a row) time is latency: one thread per
// row, its activations indexed in scratch memory, took 41 us for the forward
// pass of 256 rows, 42 for the row deltas, and a thread per parameter walking
// the batch 68 us; this kernel takes 6 for the same rows.
constexpr int MLP_R = 4;
typedef float f32x4m __attribute__((ext_vector_type(4)));
typedef float f32x16m __attribute__((ext_vector_type(16)));

// z[q] = fma(w(k), rows[q][k], z[q]) over k in order, rows in LDS. The reads of
// the next eight k are under way while these eight are used; the fences keep
// the compiler from reading one value at a time, or all of them first.
template <int N, class W>
__device__ __forceinline__ void mlp_dot(const float (*rows)[N], float (&z)[MLP_R], W &&w) {
  f32x4m v[2][MLP_R][2];
  float wv[2][8];
  auto load = [&](int b, int k) {
#pragma unroll
    for (int q = 0; q < MLP_R; ++q) {
      v[b][q][0] = *(const f32x4m *)&rows[q][k];
      v[b][q][1] = *(const f32x4m *)&rows[q][k + 4];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) wv[b][e] = w(k + e);
  };
  load(0, 0);
#pragma unroll
  for (int k = 0; k < N; k += 8) {
    const int b = (k / 8) & 1;
    if (k + 8 < N) load(b ^ 1, k + 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int q = 0; q < MLP_R; ++q) z[q] = __builtin_fmaf(wv[b][e], v[b][q][e / 4][e % 4], z[q]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Sum over the 64 lanes of a workgroup that is one wavefront, in every lane.
__device__ __forceinline__ float mlp_sum(float v) {
  v += dpp_move<0xB1, 0xF>(v, 0.0f);
  v += dpp_move<0x4E, 0xF>(v, 0.0f);
  v += dpp_move<0x141, 0xF>(v, 0.0f);
  v += dpp_move<0x140, 0xF>(v, 0.0f);
  v += dpp_move<0x142, 0xA>(v, 0.0f);
  v += dpp_move<0x143, 0xC>(v, 0.0f);
  return read_lane63(v);
}

template <bool TRAIN, bool IDX>
__global__ void __launch_bounds__(64) k_mlp_rows(const float *__restrict__ X, const float *__restrict__ T,
                                                 const int32_t *__restrict__ idx, int64_t n,
                                                 const float *__restrict__ P, float *__restrict__ Y,
                                                 float *__restrict__ part) {
  __shared__ __attribute__((aligned(16))) float sx[MLP_R][F], sh[MLP_R][H1], sd[TRAIN ? MLP_R : 1][H2], s1[TRAIN ? MLP_R : 1][H1],
      sw[TRAIN ? H2 : 1][H1];  // W2, for its columns
  const int j = threadIdx.x, half = j >> 5, l32 = j & 31;
  float w1[F], w2[H1];
#pragma unroll
  for (int k = 0; k < F; k += 4) {
    const f32x4m v = *(const f32x4m *)(P + O_W1 + j * F + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) w1[k + e] = v[e];
  }
#pragma unroll
  for (int k = 0; k < H1; k += 4) {
    const f32x4m v = *(const f32x4m *)(P + O_W2 + j * H1 + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) w2[k + e] = v[e];
  }
  if constexpr (TRAIN) {
#pragma unroll
    for (int k = 0; k < H2; ++k) sw[k][j] = P[O_W2 + k * H1 + j];
  }
  const float b1 = P[O_B1 + j], b2 = P[O_B2 + j], w3 = P[O_W3 + j], b3 = P[O_B3];
  f32x16m g1[TRAIN ? 2 : 1] = {}, g2[TRAIN ? 2 : 1][TRAIN ? 2 : 1] = {};  // W1: 64 x 32, W2: 64 x 64, in 32 x 32 blocks
  // matrix operands: lane l holds element l mod 32 of row l / 32
  float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, se = 0.0f;
  // rows r0 .. r0 + MLP_R - 1 of the next iteration are loaded while this
  // one's are computed: lane l holds element l mod 32 of row 2 s + l / 32,
  // and the target of row l mod MLP_R. Past the end: the last row again, not
  // counted.
  float xv[MLP_R / 2], tv = 0.0f;
  auto fetch = [&](int64_t r0, float (&xn)[MLP_R / 2], float &tn) {
    auto row = [&](int64_t r) {
      r = r < n ? r : n - 1;
      return IDX ? (int64_t)idx[r] : r;
    };
#pragma unroll
    for (int s = 0; s < MLP_R / 2; ++s) xn[s] = X[row(r0 + 2 * s + half) * F + l32];
    if constexpr (TRAIN) tn = T[row(r0 + j % MLP_R)];
  };
  fetch((int64_t)blockIdx.x * MLP_R, xv, tv);
  for (int64_t r0 = (int64_t)blockIdx.x * MLP_R; r0 < n; r0 += (int64_t)gridDim.x * MLP_R) {
    float z1[MLP_R], z2[MLP_R], xn[MLP_R / 2], tn = 0.0f;
    __syncthreads();  // the previous rows' readers are done
#pragma unroll
    for (int s = 0; s < MLP_R / 2; ++s) sx[2 * s + half][l32] = xv[s];
    fetch(r0 + (int64_t)gridDim.x * MLP_R, xn, tn);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MLP_R; ++q) z1[q] = b1;
    mlp_dot<F>(sx, z1, [&](int k) { return w1[k]; });
#pragma unroll
    for (int q = 0; q < MLP_R; ++q) {
      sh[q][j] = z1[q] > 0.0f ? z1[q] : 0.0f;
      z2[q] = b2;
    }
    __syncthreads();
    mlp_dot<H1>(sh, z2, [&](int k) { return w2[k]; });
#pragma unroll
    for (int q = 0; q < MLP_R; ++q) {
      const float h2 = z2[q] > 0.0f ? z2[q] : 0.0f;
      const float y = b3 + mlp_sum(w3 * h2);
      const bool live = r0 + q < n;
      if constexpr (!TRAIN) {
        if (live && j == 0) Y[r0 + q] = y;
      } else {
        const float d = live ? y - __shfl(tv, q) : 0.0f, dy = 2.0f * d / (float)n;
        se += d * d;
        gb3 += dy;
        gw3 = __builtin_fmaf(dy, h2, gw3);
        z2[q] = z2[q] > 0.0f ? dy * w3 : 0.0f;  // the second layer's delta from here on
        gb2 += z2[q];
        sd[q][j] = z2[q];
      }
    }
    if constexpr (TRAIN) {
      __syncthreads();
      float d1[MLP_R] = {};
      mlp_dot<H2>(sd, d1, [&](int k) { return sw[k][j]; });
#pragma unroll
      for (int q = 0; q < MLP_R; ++q) {
        if (!(z1[q] > 0.0f)) d1[q] = 0.0f;
        gb1 += d1[q];
        s1[q][j] = d1[q];
      }
      __syncthreads();
#pragma unroll
      for (int s = 0; s < MLP_R / 2; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float a2 = sd[2 * s + half][32 * i + l32], a1 = s1[2 * s + half][32 * i + l32];
#pragma unroll
          for (int c = 0; c < 2; ++c)
            g2[i][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(a2, sh[2 * s + half][32 * c + l32], g2[i][c], 0, 0, 0);
          g1[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, xv[s], g1[i], 0, 0, 0);
        }
    }
#pragma unroll
    for (int s = 0; s < MLP_R / 2; ++s) xv[s] = xn[s];
    tv = tn;
  }
  if constexpr (TRAIN) {
    float *g = part + (int64_t)blockIdx.x * MLP_PART;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int u = 32 * i + 8 * (r / 4) + 4 * half + (r % 4);  // the unit whose weights these are
        g[O_W1 + u * F + l32] = g1[i][r];
        g[O_W2 + u * H1 + l32] = g2[i][0][r];
        g[O_W2 + u * H1 + 32 + l32] = g2[i][1][r];
      }
    g[O_B1 + j] = gb1;
    g[O_B2 + j] = gb2;
    g[O_W3 + j] = gw3;
    if (j == 0) {
      g[O_B3] = gb3;
      g[NP] = se;
    }
  }
}

// Forward pass of many rows, one per thread: without a lane's wait for the
// others' values the multiply-adds bound it (300,000 rows: 90 us, k_mlp_rows
// 129; 120,000: 50 and 59; 100,000: 50 and 51; up to 20,000 it takes 40, a thread's chain).
__global__ void __launch_bounds__(256) k_mlp_many(const float *__restrict__ X, int64_t n, const float *__restrict__ P,
                                                  float *__restrict__ Y) {
  __shared__ float sp[NP];
  for (int i = threadIdx.x; i < NP; i += blockDim.x) sp[i] = P[i];
  __syncthreads();
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  float x[F], h1[H1];
  for (int k = 0; k < F; ++k) x[k] = X[r * F + k];
  for (int j = 0; j < H1; ++j) {
    float z = sp[O_B1 + j];
    for (int k = 0; k < F; ++k) z = __builtin_fmaf(sp[O_W1 + j * F + k], x[k], z);
    h1[j] = z > 0.0f ? z : 0.0f;
  }
  float y = sp[O_B3];
  for (int j = 0; j < H2; ++j) {
    float z = sp[O_B2 + j];
    for (int k = 0; k < H1; ++k) z = __builtin_fmaf(sp[O_W2 + j * H1 + k], h1[k], z);
    y = __builtin_fmaf(sp[O_W3 + j], z > 0.0f ? z : 0.0f, y);
  }
  Y[r] = y;
}

// Sums the wavefronts' gradients in order (eight runs of every eighth, then
// the eight), writes them and the loss, and applies Adam with bias correction
// (Kingma & Ba 2015) when `adam`. 64 parameters per workgroup, eight threads
// each.
__global__ void __launch_bounds__(512) k_mlp_update(const float *__restrict__ part, int nw, int64_t n,
                                                    float *__restrict__ P, float *__restrict__ G,
                                                    float *__restrict__ loss, float *__restrict__ M,
                                                    float *__restrict__ V, bool adam, float lr, float b1, float b2,
                                                    float eps, float c1, float c2) {
  __shared__ float s8[8][64];
  const int t = threadIdx.x % 64, run = threadIdx.x / 64, p = blockIdx.x * 64 + t;
  float s = 0.0f;
  if (p <= NP) {
    constexpr int UN = 8;
    int w = run;
    for (; w + 8 * (UN - 1) < nw; w += 8 * UN) {
      float v[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) v[u] = part[(int64_t)(w + 8 * u) * MLP_PART + p];
#pragma unroll
      for (int u = 0; u < UN; ++u) s += v[u];
    }
    for (; w < nw; w += 8) s += part[(int64_t)w * MLP_PART + p];
  }
  s8[run][t] = s;
  __syncthreads();
  if (run != 0 || p > NP) return;
  float g = 0.0f;
#pragma unroll
  for (int q = 0; q < 8; ++q) g += s8[q][t];
  if (p == NP) {
    *loss = g / (float)n;
    return;
  }
  G[p] = g;
  if (!adam) return;
  const float m = b1 * M[p] + (1.0f - b1) * g;
  const float v = b2 * V[p] + (1.0f - b2) * g * g;
  M[p] = m;
  V[p] = v;
  const float mh = m / c1, vh = v / c2;
  P[p] = P[p] - lr * mh / (sqrtf(vh) + eps);
}

uint64_t mix64(uint64_t z) {  // SplitMix64 finalizer (Steele, Lea, Flood 2014)
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}
uint64_t hash_at(uint64_t seed, uint64_t stream, uint64_t i) {
  const uint64_t G = 0x9E3779B97F4A7C15ULL;
  return mix64(mix64(seed + stream * G) + (i + 1) * G);
}

}  // namespace

struct ModelState {
  float *P = nullptr, *M = nullptr, *V = nullptr, *G = nullptr;  // device, NP each
  int64_t step = 0;
  uint64_t seed = 0;
  int64_t epochs = 0;
  int64_t cap = 0;        // wavefronts `part` has room for
  float *part = nullptr;  // their gradients
  float *loss = nullptr;
};

void upir_model_free(upir_ctx *c) {
  ModelState *m = c->model;
  if (!m) return;
  for (float *p : {m->P, m->M, m->V, m->G, m->part, m->loss}) upir_dfree(c, p);
  delete m;
  c->model = nullptr;
}

#define HIPTRY(c, expr)                                      \
  do {                                                       \
    hipError_t e_ = (expr);                                  \
    if (e_ != hipSuccess) return upir_hipfail(c, e_, #expr); \
  } while (0)

// Gradient room for the `waves` wavefronts of a training step.
static upir_status model_buffers(upir_ctx *c, int64_t waves) {
  ModelState *m = c->model;
  if (waves <= m->cap) return UPIR_OK;
  float *np = (float *)upir_dalloc(c, (size_t)waves * MLP_PART * 4);
  if (!np) return upir_fail(c, UPIR_ENOMEM, "model work buffers");
  HIPTRY(c, hipStreamSynchronize(c->stream));  // earlier steps may still use the old one
  upir_dfree(c, m->part);
  m->part = np;
  m->cap = waves;
  return UPIR_OK;
}

static upir_status need_model(upir_ctx *c) {
  if (c->none) return upir_fail(c, UPIR_ESTATE, "host-only context");
  if (!c->model) return upir_fail(c, UPIR_ESTATE, "no model: call upir_model_init or upir_model_load");
  if (c->capturing) return upir_fail(c, UPIR_ESTATE, "model calls during graph capture");
  return UPIR_OK;
}

extern "C" upir_status upir_model_init(upir_ctx *c, uint64_t seed) {
  if (!c) return UPIR_EINVAL;
  if (c->none) return upir_fail(c, UPIR_ESTATE, "host-only context");
  upir_model_free(c);
  ModelState *m = new ModelState();
  c->model = m;
  m->seed = seed;
  m->P = (float *)upir_dalloc(c, NP * 4);
  m->M = (float *)upir_dalloc(c, NP * 4);
  m->V = (float *)upir_dalloc(c, NP * 4);
  m->G = (float *)upir_dalloc(c, NP * 4);
  m->loss = (float *)upir_dalloc(c, 64);
  if (!m->P || !m->M || !m->V || !m->G || !m->loss) {
    upir_model_free(c);
    return upir_fail(c, UPIR_ENOMEM, "model parameters");
  }
  // Kaiming-uniform weights U(-sqrt(6/fan_in), sqrt(6/fan_in)), zero biases
  std::vector<float> h(NP, 0.0f);
  auto fill = [&](int off, int count, int fan_in, uint64_t stream) {
    const double bound = sqrt(6.0 / fan_in);
    for (int i = 0; i < count; ++i) {
      const int64_t k = (int64_t)(hash_at(seed, stream, i) >> 40) - (1 << 23);  // [-2^23, 2^23)
      h[off + i] = (float)(bound * (double)k * 0x1p-23);
    }
  };
  fill(O_W1, H1 * F, F, 1);
  fill(O_W2, H2 * H1, H1, 2);
  fill(O_W3, H2, H2, 3);
  std::vector<float> zero(NP, 0.0f);
  HIPTRY(c, hipMemcpyAsync(m->P, h.data(), NP * 4, hipMemcpyHostToDevice, c->stream));
  HIPTRY(c, hipMemcpyAsync(m->M, zero.data(), NP * 4, hipMemcpyHostToDevice, c->stream));
  HIPTRY(c, hipMemcpyAsync(m->V, zero.data(), NP * 4, hipMemcpyHostToDevice, c->stream));
  HIPTRY(c, hipStreamSynchronize(c->stream));
  m->step = 0;
  return UPIR_OK;
}

extern "C" upir_status upir_model_set_params(upir_ctx *c, const float *host) {
  if (!c || !host) return UPIR_EINVAL;
  upir_status st = need_model(c);
  if (st) return st;
  HIPTRY(c, hipMemcpyAsync(c->model->P, host, NP * 4, hipMemcpyHostToDevice, c->stream));
  std::vector<float> zero(NP, 0.0f);
  HIPTRY(c, hipMemcpyAsync(c->model->M, zero.data(), NP * 4, hipMemcpyHostToDevice, c->stream));
  HIPTRY(c, hipMemcpyAsync(c->model->V, zero.data(), NP * 4, hipMemcpyHostToDevice, c->stream));
  HIPTRY(c, hipStreamSynchronize(c->stream));
  c->model->step = 0;
  return UPIR_OK;
}

extern "C" upir_status upir_model_get_params(upir_ctx *c, float *host) {
  if (!c || !host) return UPIR_EINVAL;
  upir_status st = need_model(c);
  if (st) return st;
  HIPTRY(c, hipMemcpyAsync(host, c->model->P, NP * 4, hipMemcpyDeviceToHost, c->stream));
  HIPTRY(c, hipStreamSynchronize(c->stream));
  return UPIR_OK;
}

// Predictions of rows idx[0 .. n) of X (idx == nullptr: rows 0 .. n).
static hipError_t fwd_launch(upir_ctx *c, const float *X, const int32_t *idx, int64_t n, float *Y) {
  if (n <= 0) return hipSuccess;
  if (!idx && n >= MLP_MANY) {
    hipLaunchKernelGGL(k_mlp_many, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, X, n, c->model->P, Y);
    return hipGetLastError();
  }
  // four wavefronts per SIMD at most: each brings the weights into its registers
  const int64_t waves = std::min<int64_t>((n + MLP_R - 1) / MLP_R, 16LL * c->num_cus);
  hipLaunchKernelGGL((idx ? k_mlp_rows<false, true> : k_mlp_rows<false, false>), dim3((unsigned)waves), dim3(64), 0, c->stream, X, (const float *)nullptr, idx,
                     n, c->model->P, Y, (float *)nullptr);
  return hipGetLastError();
}

extern "C" upir_status upir_model_forward(upir_ctx *c, const float *dev_x, int64_t n, float *dev_y) {
  if (!c) return UPIR_EINVAL;
  upir_status st = need_model(c);
  if (st) return st;
  if (n < 0 || (n > 0 && (!dev_x || !dev_y))) return upir_fail(c, UPIR_EINVAL, "model_forward arguments");
  HIPTRY(c, fwd_launch(c, dev_x, nullptr, n, dev_y));
  return UPIR_OK;
}

// One optimisation step on rows idx[0 .. n) (nullptr: 0 .. n) of X (rows of
// 32) and T, all on the device.
static upir_status step_dev(upir_ctx *c, const float *X, const float *T, const int32_t *idx, int64_t n, float lr,
                            bool adam, float *grad_out, float *loss_out) {
  ModelState *m = c->model;
  // every wavefront leaves 25 KB to be summed: from 1,024 rows on they take more
  // rows each (2,048 rows: 22.5 us with 256 of them, 23.8 with 512), from
  // 4,096 on the rows weigh more (8,192: 56 against 41 us)
  const int64_t waves = std::min<int64_t>((n + MLP_R - 1) / MLP_R, n > 4096 ? MLP_WAVES : MLP_WAVES / 2);
  upir_status st = model_buffers(c, waves);
  if (st) return st;
  hipLaunchKernelGGL((idx ? k_mlp_rows<true, true> : k_mlp_rows<true, false>), dim3((unsigned)waves), dim3(64), 0, c->stream, X, T, idx, n, m->P,
                     (float *)nullptr, m->part);
  float c1 = 1.0f, c2 = 1.0f;
  if (adam) {
    m->step++;
    c1 = (float)(1.0 - pow(0.9, (double)m->step));
    c2 = (float)(1.0 - pow(0.999, (double)m->step));
  }
  hipLaunchKernelGGL(k_mlp_update, dim3((NP + 1 + 63) / 64), dim3(512), 0, c->stream, m->part, (int)waves, n, m->P,
                     grad_out ? grad_out : m->G, m->loss, m->M, m->V, adam, lr, 0.9f, 0.999f, 1e-8f, c1, c2);
  HIPTRY(c, hipGetLastError());
  if (loss_out) {
    HIPTRY(c, hipMemcpyAsync(loss_out, m->loss, 4, hipMemcpyDeviceToHost, c->stream));
    HIPTRY(c, hipStreamSynchronize(c->stream));
  }
  return UPIR_OK;
}

extern "C" upir_status upir_model_step(upir_ctx *c, const float *dev_x, const float *dev_t, int64_t n, float lr,
                                       int32_t adam, float *dev_grad, float *loss_out) {
  if (!c) return UPIR_EINVAL;
  upir_status st = need_model(c);
  if (st) return st;
  if (n <= 0 || !dev_x || !dev_t) return upir_fail(c, UPIR_EINVAL, "model_step arguments");
  return step_dev(c, dev_x, dev_t, nullptr, n, lr, adam != 0, dev_grad, loss_out);
}

// ------------------------------------------------------------ timing table
extern "C" upir_status upir_tune_db_size(upir_ctx *c, int64_t *rows) {
  if (!c || !rows) return UPIR_EINVAL;
  *rows = (int64_t)c->db.size();
  return UPIR_OK;
}

extern "C" upir_status upir_tune_db_row(upir_ctx *c, int64_t row, float *feat, float *log2_us, int64_t *key) {
  if (!c) return UPIR_EINVAL;
  if (row < 0 || row >= (int64_t)c->db.size()) return upir_fail(c, UPIR_EINVAL, "row %lld", (long long)row);
  const TuneRow &r = c->db[row];
  if (feat) memcpy(feat, r.feat, sizeof r.feat);
  if (log2_us) *log2_us = r.log2_us;
  if (key) *key = r.loop_key;
  return UPIR_OK;
}

extern "C" upir_status upir_tune_db_save(upir_ctx *c, const char *path) {
  if (!c || !path) return UPIR_EINVAL;
  FILE *f = fopen(path, "w");
  if (!f) return upir_fail(c, UPIR_EINVAL, "cannot write %s", path);
  fprintf(f, "# upir timing table v1: loop_key log2_us f0..f31\n");
  for (const TuneRow &r : c->db) {
    fprintf(f, "%lld %.9g", (long long)r.loop_key, r.log2_us);
    for (int i = 0; i < F; ++i) fprintf(f, " %.9g", r.feat[i]);
    fputc('\n', f);
  }
  fclose(f);
  return UPIR_OK;
}

extern "C" upir_status upir_tune_db_load(upir_ctx *c, const char *path) {
  if (!c || !path) return UPIR_EINVAL;
  FILE *f = fopen(path, "r");
  if (!f) return upir_fail(c, UPIR_EINVAL, "cannot read %s", path);
  char line[4096];
  std::vector<TuneRow> rows;
  while (fgets(line, sizeof line, f)) {
    if (line[0] == '#' || line[0] == '\n') continue;
    TuneRow r{};
    long long key;
    int used = 0, off = 0;
    if (sscanf(line, "%lld %f%n", &key, &r.log2_us, &used) != 2) {
      fclose(f);
      return upir_fail(c, UPIR_EINVAL, "malformed row in %s", path);
    }
    off = used;
    for (int i = 0; i < F; ++i) {
      if (sscanf(line + off, "%f%n", &r.feat[i], &used) != 1) {
        fclose(f);
        return upir_fail(c, UPIR_EINVAL, "short row in %s", path);
      }
      off += used;
    }
    r.loop_key = key;
    rows.push_back(r);
  }
  fclose(f);
  c->db.insert(c->db.end(), rows.begin(), rows.end());
  return UPIR_OK;
}

// ----------------------------------------------------------------- training
extern "C" upir_status upir_model_train(upir_ctx *c, int32_t epochs, int32_t batch, float lr, int32_t holdout_mod,
                                        float *train_mse, float *holdout_mse) {
  if (!c) return UPIR_EINVAL;
  upir_status st = need_model(c);
  if (st) return st;
  if (epochs < 0 || batch < 1 || batch > 65536) return upir_fail(c, UPIR_EINVAL, "epochs / batch");
  std::vector<int32_t> train, hold;
  for (int32_t i = 0; i < (int32_t)c->db.size(); ++i) {
    const uint64_t k = (uint64_t)c->db[i].loop_key;
    if (holdout_mod >= 0 && (int32_t)(k % 5) == holdout_mod)
      hold.push_back(i);
    else
      train.push_back(i);
  }
  if (train.empty()) return upir_fail(c, UPIR_ESTATE, "no training rows");
  // the whole table on the device once
  const size_t nrow = c->db.size();
  std::vector<float> hx(nrow * F), ht(nrow);
  for (size_t i = 0; i < nrow; ++i) {
    memcpy(&hx[i * F], c->db[i].feat, F * 4);
    ht[i] = c->db[i].log2_us;
  }
  float *dX = (float *)upir_dalloc(c, nrow * F * 4), *dT = (float *)upir_dalloc(c, nrow * 4);
  int32_t *dIdx = (int32_t *)upir_dalloc(c, std::max(train.size(), hold.size()) * 4);
  auto cleanup = [&]() {
    upir_dfree(c, dX);
    upir_dfree(c, dT);
    upir_dfree(c, dIdx);
  };
  if (!dX || !dT || !dIdx) {
    cleanup();
    return upir_fail(c, UPIR_ENOMEM, "training buffers");
  }
  hipError_t e = hipMemcpyAsync(dX, hx.data(), nrow * F * 4, hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(dT, ht.data(), nrow * 4, hipMemcpyHostToDevice, c->stream);
  if (e != hipSuccess) {
    cleanup();
    return upir_hipfail(c, e, "training copy");
  }
  std::vector<int32_t> order = train;
  for (int32_t ep = 0; ep < epochs && st == UPIR_OK; ++ep) {
    // Fisher-Yates shuffle driven by SplitMix64 (seed, epoch)
    for (size_t i = order.size(); i > 1; --i) {
      const size_t j = (size_t)(hash_at(c->model->seed, 1000 + (uint64_t)(c->model->epochs + ep), i) % i);
      std::swap(order[i - 1], order[j]);
    }
    e = hipMemcpyAsync(dIdx, order.data(), order.size() * 4, hipMemcpyHostToDevice, c->stream);
    if (e != hipSuccess) {
      st = upir_hipfail(c, e, "index copy");
      break;
    }
    for (size_t b0 = 0; b0 < order.size(); b0 += batch) {
      const int64_t nb = (int64_t)std::min<size_t>(batch, order.size() - b0);
      st = step_dev(c, dX, dT, dIdx + b0, nb, lr, true, nullptr, nullptr);
      if (st) break;
    }
    // keep the index buffer alive until this epoch's kernels have read it
    e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess && st == UPIR_OK) st = upir_hipfail(c, e, "training epoch");
  }
  c->model->epochs += epochs;
  // final errors over the train / holdout rows
  auto mse = [&](const std::vector<int32_t> &rows, float *out) -> upir_status {
    if (!out) return UPIR_OK;
    if (rows.empty()) {
      *out = NAN;
      return UPIR_OK;
    }
    float *dY = (float *)upir_dalloc(c, rows.size() * 4);
    if (!dY) {
      return upir_fail(c, UPIR_ENOMEM, "evaluation buffers");
    }
    hipError_t e2 = hipMemcpyAsync(dIdx, rows.data(), rows.size() * 4, hipMemcpyHostToDevice, c->stream);
    const int64_t n = (int64_t)rows.size();
    if (e2 == hipSuccess) {
      e2 = fwd_launch(c, dX, dIdx, n, dY);
    }
    std::vector<float> y(n);
    if (e2 == hipSuccess) e2 = hipMemcpyAsync(y.data(), dY, n * 4, hipMemcpyDeviceToHost, c->stream);
    if (e2 == hipSuccess) e2 = hipStreamSynchronize(c->stream);
    upir_dfree(c, dY);
    if (e2 != hipSuccess) return upir_hipfail(c, e2, "evaluation");
    double s = 0;
    for (int64_t i = 0; i < n; ++i) {
      const double d = (double)y[i] - ht[rows[i]];
      s += d * d;
    }
    *out = (float)(s / n);
    return UPIR_OK;
  };
  if (st == UPIR_OK) st = mse(train, train_mse);
  if (st == UPIR_OK) st = mse(hold, holdout_mse);
  cleanup();
  return st;
}

extern "C" upir_status upir_model_enable(upir_ctx *c, int32_t on) {
  if (!c) return UPIR_EINVAL;
  if (on && !c->model) return upir_fail(c, UPIR_ESTATE, "no model");
  c->model_on = on != 0;
  return UPIR_OK;
}

extern "C" upir_status upir_model_save(upir_ctx *c, const char *path) {
  if (!c || !path) return UPIR_EINVAL;
  upir_status st = need_model(c);
  if (st) return st;
  std::vector<float> p(NP);
  st = upir_model_get_params(c, p.data());
  if (st) return st;
  uint64_t sum = 1469598103934665603ULL;
  for (float v : p) {
    uint32_t b;
    memcpy(&b, &v, 4);
    sum = (sum ^ b) * 1099511628211ULL;
  }
  FILE *f = fopen(path, "wb");
  if (!f) return upir_fail(c, UPIR_EINVAL, "cannot write %s", path);
  const int32_t hdr[4] = {0x52495055 /* "UPIR" */, F, H1, H2};
  const int64_t meta[3] = {(int64_t)c->model->seed, c->model->epochs, (int64_t)sum};
  bool ok = fwrite(hdr, sizeof hdr, 1, f) == 1 && fwrite(meta, sizeof meta, 1, f) == 1 &&
            fwrite(p.data(), 4, NP, f) == (size_t)NP;
  fclose(f);
  return ok ? UPIR_OK : upir_fail(c, UPIR_EINVAL, "short write %s", path);
}

extern "C" upir_status upir_model_load(upir_ctx *c, const char *path) {
  if (!c || !path) return UPIR_EINVAL;
  FILE *f = fopen(path, "rb");
  if (!f) return upir_fail(c, UPIR_EINVAL, "cannot read %s", path);
  int32_t hdr[4];
  int64_t meta[3];
  std::vector<float> p(NP);
  bool ok = fread(hdr, sizeof hdr, 1, f) == 1 && fread(meta, sizeof meta, 1, f) == 1 &&
            fread(p.data(), 4, NP, f) == (size_t)NP;
  fclose(f);
  if (!ok || hdr[0] != 0x52495055 || hdr[1] != F || hdr[2] != H1 || hdr[3] != H2)
    return upir_fail(c, UPIR_EINVAL, "%s is not a model file of this shape", path);
  uint64_t sum = 1469598103934665603ULL;
  for (float v : p) {
    uint32_t b;
    memcpy(&b, &v, 4);
    sum = (sum ^ b) * 1099511628211ULL;
  }
  if ((int64_t)sum != meta[2]) return upir_fail(c, UPIR_EINVAL, "%s: checksum mismatch", path);
  upir_status st = upir_model_init(c, (uint64_t)meta[0]);
  if (st) return st;
  st = upir_model_set_params(c, p.data());
  if (st == UPIR_OK) c->model->epochs = meta[1];
  return st;
}

// ----------------------------------------------------- candidates, features
namespace upir {

static double lg(double v) { return v > 0 ? log2(v) : 0.0; }

struct Cand {
  upir_spmd sp;
  upir_sched sc;
};

static bool is_mm(int32_t k) { return k >= UPIR_BODY_MATMUL_F32 && k <= UPIR_BODY_MATMUL_SPLIT3; }

// Candidate schedules of a loop. Candidate 0 is always the library default,
// so the table records what the default costs next to every alternative.
static std::vector<Cand> candidates(upir_ctx *c, const upir_loop_obj *lp) {
  std::vector<Cand> v;
  const int64_t n = lp->n;
  {
    Cand d{};
    default_choice(c, lp, d.sp, d.sc);
    v.push_back(d);
  }
  auto add = [&](int32_t T, int32_t U, int32_t pol, int64_t chunk, int t0 = 0, int t1 = 0) {
    Cand k{};
    k.sp = upir_spmd{T, U, UPIR_TARGET_GPU};
    k.sc.policy = pol;
    k.sc.chunk = chunk;
    k.sc.distribute = UPIR_DIST_TEAMS_UNITS;
    k.sc.tile[0] = t0;
    k.sc.tile[1] = t1;
    v.push_back(k);
  };
  const int64_t capT = 1 << 20;
  auto teams = [&](int64_t work, int64_t per) {
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(capT, (work + per - 1) / per));
  };
  switch (lp->kind) {
    case UPIR_BODY_AXPY:
    case UPIR_BODY_COVER:
    case UPIR_BODY_SUM:
      if (lp->loop.collapse == 1 && (lp->kind != UPIR_BODY_SUM || lp->sum_dtype == UPIR_DT_F32)) {
        for (int32_t U : {64, 256, 1024})
          for (int64_t per : {4, 16, 64, 256}) add(teams(n, U * per), U, UPIR_SCHED_STATIC_CHUNK, 4);
        for (int32_t U : {256, 512})  // one team per CU
          add((int32_t)std::min<int64_t>(c->num_cus, teams(n, U * 4)), U, UPIR_SCHED_STATIC_CHUNK, 4);
      } else {
        for (int32_t U : {64, 256, 1024})
          for (int64_t per : {1, 8, 64}) add(teams(n, U * per), U, UPIR_SCHED_STATIC, 0);
      }
      break;
    case UPIR_BODY_JACOBI5:
    case UPIR_BODY_FILTER7:
      for (int th : {8, 16, 32, 64, 128})
        for (int32_t U : {64, 128, 256, 512})
          if (U <= th * 64 && (th < 128 || lp->kind == UPIR_BODY_JACOBI5)) add(0, U, UPIR_SCHED_STATIC, 0, th, 256);
      break;
    case UPIR_BODY_MATVEC:
      for (int32_t U : {64, 256, 1024})
        for (int64_t rpw : {1, 4, 16}) add(teams(n, (U / 64) * rpw), U, UPIR_SCHED_STATIC_CHUNK, 1);
      break;
    case UPIR_BODY_MATMUL_F32:
      add(0, 256, UPIR_SCHED_STATIC, 0, 128, 128);
      add(0, 512, UPIR_SCHED_STATIC, 0, 256, 128);
      add(0, 512, UPIR_SCHED_STATIC, 0, 64, 128);
      add(0, 512, UPIR_SCHED_STATIC, 0, 64, 64);
      add(0, 512, UPIR_SCHED_STATIC, 0, 32, 32);
      break;
    case UPIR_BODY_MATMUL_BF16:
    case UPIR_BODY_MATMUL_SPLIT3:
      add(0, 256, UPIR_SCHED_STATIC, 0, 128, 128);
      add(0, 256, UPIR_SCHED_STATIC, 0, 256, 256);
      add(0, 512, UPIR_SCHED_STATIC, 0, 256, 256);
      for (int t : {128, 64, 32}) add(0, 512, UPIR_SCHED_STATIC, 0, t, t);
      add(0, 512, UPIR_SCHED_STATIC, 0, 64, 128);
      break;
    default:
      for (int32_t U : {64, 256}) add(teams(n, U * 4), U, UPIR_SCHED_STATIC, 0);
  }
  return v;
}

int candidate_count(upir_ctx *c, const upir_loop_obj *lp) { return (int)candidates(c, lp).size(); }

bool candidate_at(upir_ctx *c, const upir_loop_obj *lp, int idx, upir_spmd &sp, upir_sched &sc) {
  auto v = candidates(c, lp);
  if (idx < 0 || idx >= (int)v.size()) return false;
  sp = v[idx].sp;
  sc = v[idx].sc;
  return true;
}

// 32 features of (loop, candidate). Sizes enter as log2 / 32.
static void features(const upir_loop_obj *lp, const Cand &k, float f[32]) {
  for (int i = 0; i < 32; ++i) f[i] = 0.0f;
  const int kind = lp->kind;
  const int cls = kind == UPIR_BODY_AXPY || kind == UPIR_BODY_COVER ? 0
                  : kind == UPIR_BODY_SUM                           ? 1
                  : kind == UPIR_BODY_JACOBI5 || kind == UPIR_BODY_FILTER7 ? 2
                  : kind == UPIR_BODY_MATVEC                        ? 3
                                                                    : 4;
  f[cls] = 1.0f;
  const double n = (double)lp->n;
  double rows = (double)lp->cnt[0], cols = lp->loop.collapse > 1 ? (double)lp->cnt[1] : 1.0, K = 1.0;
  double bpi = 12, fpi = 2;
  if (kind == UPIR_BODY_SUM) bpi = 4, fpi = 1;
  if (kind == UPIR_BODY_COVER) bpi = 8, fpi = 0;
  if (kind == UPIR_BODY_JACOBI5) bpi = 8, fpi = 7;
  if (kind == UPIR_BODY_FILTER7) bpi = 8, fpi = 98;
  if (kind == UPIR_BODY_MATVEC) {
    cols = (double)((const upir_matvec_args *)lp->args)->cols;
    bpi = 4 * cols + 4, fpi = 2 * cols;
  }
  if (is_mm(kind)) {
    K = (double)((const upir_matmul_args *)lp->args)->K;
    bpi = 8.0 * K / 64.0, fpi = 2 * K;
  }
  f[5] = (float)(lg(n) / 32);
  f[6] = (float)(lg(rows) / 32);
  f[7] = (float)(lg(cols) / 32);
  f[8] = (float)(lg(K) / 32);
  f[9] = (float)(lg(bpi) / 32);
  f[10] = (float)(lg(fpi + 1) / 32);
  f[11] = lp->loop.dim[0].step == 1 ? 1.0f : 0.0f;
  f[12] = (float)lp->loop.collapse / 3.0f;
  f[13] = lp->has_red ? 1.0f : 0.0f;
  f[14] = lp->has_red && lp->red.op == UPIR_RED_SUM ? 1.0f : 0.0f;
  f[15] = lp->has_red && lp->red.op != UPIR_RED_SUM ? 1.0f : 0.0f;
  // candidate
  const double U = k.sp.num_units > 0 ? k.sp.num_units : 256;
  f[16] = (float)(lg(U) / 10);
  f[17] = (float)(lg(k.sc.tile[0] > 0 ? k.sc.tile[0] : 1) / 10);
  f[18] = (float)(lg(k.sc.tile[1] > 0 ? k.sc.tile[1] : 1) / 10);
  f[19] = (float)(lg(k.sc.chunk > 0 ? (double)k.sc.chunk : 1) / 10);
  double T = k.sp.num_teams;
  if (T <= 0 && k.sc.tile[0] > 0) {
    T = ceil(rows / k.sc.tile[0]) * (lp->loop.collapse > 1 ? ceil(cols / std::max(1, k.sc.tile[1])) : 1.0);
  }
  f[20] = (float)(lg(T) / 24);
  const double items = n / std::max(1.0, T);
  f[21] = (float)(lg(items) / 32);
  f[22] = (float)(lg(items / U) / 16);
  f[23] = (float)std::min(1.0, T / 2048.0);  // occupancy estimate: teams vs resident slots
  f[24] = k.sp.num_teams > 0 ? 0.0f : 1.0f;  // one team per tile
  f[25] = (float)(lg((double)(k.sc.tile[0] > 0 ? k.sc.tile[0] : 1) * (k.sc.tile[1] > 0 ? k.sc.tile[1] : 1)) / 24);
  const double ws = n * bpi;
  f[26] = (float)(lg(ws / 256e6 + 1e-9) / 32);
  // Jacobi: rows of a wavefront's strip (tile rows / wavefronts per team)
  f[27] = ((kind == UPIR_BODY_JACOBI5 || kind == UPIR_BODY_FILTER7) && k.sc.tile[0] > 0) ? (float)(k.sc.tile[0] / std::max(1.0, U / 64) / 64.0) : 0.0f;
  f[28] = (float)(lg(n * bpi) / 40);
  f[29] = (float)(lg(n * fpi + 1) / 48);
  f[30] = 0.0f;
  f[31] = 0.0f;
}

void candidate_features(upir_ctx *, const upir_loop_obj *lp, const upir_spmd &sp, const upir_sched &sc, float f[32]) {
  Cand k{sp, sc};
  features(lp, k, f);
}

// Cost model pick: batch every candidate through one forward pass and take
// the smallest predicted time. Returns false when the model is off.
bool model_pick(upir_ctx *c, upir_loop_obj *lp, upir_spmd &sp, upir_sched &sc) {
  if (!c->model || !c->model_on || c->capturing || c->no_alloc) return false;  // inference allocates
  auto cs = candidates(c, lp);
  if (cs.empty()) return false;
  std::vector<float> X(cs.size() * 32);
  for (size_t i = 0; i < cs.size(); ++i) features(lp, cs[i], &X[i * 32]);
  float *dX = (float *)upir_dalloc(c, X.size() * 4), *dY = (float *)upir_dalloc(c, cs.size() * 4);
  std::vector<float> y(cs.size());
  bool ok = dX && dY;
  if (ok) ok = hipMemcpyAsync(dX, X.data(), X.size() * 4, hipMemcpyHostToDevice, c->stream) == hipSuccess;
  if (ok) ok = fwd_launch(c, dX, nullptr, (int64_t)cs.size(), dY) == hipSuccess;
  if (ok) ok = hipMemcpyAsync(y.data(), dY, y.size() * 4, hipMemcpyDeviceToHost, c->stream) == hipSuccess;
  if (ok) ok = hipStreamSynchronize(c->stream) == hipSuccess;
  upir_dfree(c, dX);
  upir_dfree(c, dY);
  if (!ok) return false;
  size_t b = 0;
  for (size_t i = 1; i < y.size(); ++i)
    if (y[i] < y[b]) b = i;
  sp = cs[b].sp;
  sc = cs[b].sc;
  return true;
}

// ------------------------------------------------ engine schedules (batched)
std::vector<upir_engine_sched> engine_candidates() {
  std::vector<upir_engine_sched> v;
  v.push_back(upir_engine_sched{16384, 16384, 64});  // the default first
  for (int64_t a : {8192, 16384, 32768})
    for (int64_t s : {16384, 32768, 65536})
      for (int64_t m : {32, 64, 128})
        if (!(a == 16384 && s == 16384 && m == 64)) v.push_back(upir_engine_sched{a, s, m});
  return v;
}

namespace {
// engine class of a task: 0 AXPY / COVER, 1 SUM, 2 MATVEC
int engine_class(int32_t kind) { return kind == UPIR_BODY_SUM ? 1 : (kind == UPIR_BODY_MATVEC ? 2 : 0); }

int64_t task_len(const TaskRec &t) { return t.hi >= 0 ? t.hi - t.lo : t.loop->n; }

double task_bytes(const TaskRec &t) {
  const double n = (double)task_len(t);
  switch (t.loop->kind) {
    case UPIR_BODY_AXPY: return 12.0 * n;
    case UPIR_BODY_SUM: return 4.0 * n;
    case UPIR_BODY_MATVEC: return (4.0 * (double)((const upir_matvec_args *)t.loop->args)->cols + 4.0) * n;
    default: return 8.0 * n;
  }
}

// tile a candidate gives a task of class k (engine work items count rows for MATVEC)
int64_t class_tile(const upir_engine_sched &es, int k) {
  return k == 0 ? es.tile_axpy : (k == 1 ? es.tile_sum : es.rows_matvec);
}
}  // namespace

uint64_t batch_key(const upir_ctx *c) {
  // FNV-1a over the task count, each task's body and length, the edge count
  uint64_t h = 1469598103934665603ULL;
  auto mix = [&](uint64_t v) {
    for (int i = 0; i < 8; ++i) {
      h ^= (v >> (8 * i)) & 0xff;
      h *= 1099511628211ULL;
    }
  };
  mix(0xBA7C4ULL);
  mix((uint64_t)c->tasks.size());
  uint64_t edges = 0;
  for (const TaskRec &t : c->tasks) {
    mix((uint64_t)(t.loop ? t.loop->kind : 0));
    mix((uint64_t)(t.loop ? task_len(t) : 0));
    edges += t.preds.size();
  }
  mix(edges);
  return h;
}

// 32 features of (pending task graph, engine candidate). Slot 30 marks a
// graph row (loop rows leave it 0). The candidate enters as one one-hot per
// body over that body's three tile choices, weighted by the body's share of
// the graph's bytes, so that a choice's effect on the graph's relative cost
// is close to additive in the features; then the work items each body makes.
static const int64_t kEngineOpts[3][3] = {{8192, 16384, 32768}, {16384, 32768, 65536}, {32, 64, 128}};
static int choice_index(int k, int64_t tile) {
  for (int q = 0; q < 3; ++q)
    if (kEngineOpts[k][q] == tile) return q;
  return -1;
}
static int64_t choice_tile(int k, int q) { return kEngineOpts[k][q]; }

void batch_features(const upir_ctx *c, const upir_engine_sched &es, float f[32]) {
  for (int i = 0; i < 32; ++i) f[i] = 0.0f;
  const size_t n = c->tasks.size();
  double cnt[3] = {0, 0, 0}, bytes[3] = {0, 0, 0}, items[3] = {0, 0, 0}, lgsum = 0, lgmax = 0, edges = 0;
  std::vector<int32_t> depth(n, 0);
  int32_t dmax = 0;
  for (size_t j = 0; j < n; ++j) {
    const TaskRec &t = c->tasks[j];
    if (!t.loop) continue;
    const int k = engine_class(t.loop->kind);
    const int64_t len = std::max<int64_t>(task_len(t), 1);
    cnt[k] += 1;
    bytes[k] += task_bytes(t);
    const int64_t tile = std::max<int64_t>(1, class_tile(es, k));
    items[k] += (double)((len + tile - 1) / tile);
    lgsum += lg((double)len);
    lgmax = std::max(lgmax, lg((double)len));
    edges += (double)t.preds.size();
    int32_t d = 0;
    for (int64_t p : t.preds) d = std::max(d, depth[(size_t)p]);
    depth[j] = d + 1;
    dmax = std::max(dmax, depth[j]);
  }
  const double N = std::max<double>(1.0, (double)n), B = std::max(1.0, bytes[0] + bytes[1] + bytes[2]);
  const double I = std::max(1.0, items[0] + items[1] + items[2]), grid = 4.0 * c->num_cus;
  for (int k = 0; k < 3; ++k) {
    f[k] = (float)(cnt[k] / N);
    f[3 + k] = (float)(bytes[k] / B);
    const int q = choice_index(k, class_tile(es, k));
    if (q >= 0) f[12 + 3 * k + q] = (float)(bytes[k] / B);
    f[21 + k] = (float)(lg(items[k] + 1) / 24);
  }
  f[6] = (float)(lg(N) / 16);
  f[7] = (float)(lg(B) / 40);
  f[8] = (float)(lgsum / N / 32);
  f[9] = (float)(lgmax / 32);
  f[10] = (float)(edges / N / 8);
  f[11] = (float)(dmax / 64.0);
  f[24] = (float)(lg(I / grid) / 16);
  f[30] = 1.0f;
}

// Cost model pick of the engine schedule for the pending task graph: one
// forward pass over the 27 candidates, then the choice below. Returns false
// when the model is off.
bool model_pick_engine(upir_ctx *c, upir_engine_sched &es) {
  if (!c->model || !c->model_on || c->capturing || c->no_alloc || c->tasks.empty()) return false;
  const auto cs = engine_candidates();
  std::vector<float> X(cs.size() * 32), y(cs.size());
  for (size_t i = 0; i < cs.size(); ++i) batch_features(c, cs[i], &X[i * 32]);
  float *dX = (float *)upir_dalloc(c, X.size() * 4), *dY = (float *)upir_dalloc(c, cs.size() * 4);
  bool ok = dX && dY;
  if (ok) ok = hipMemcpyAsync(dX, X.data(), X.size() * 4, hipMemcpyHostToDevice, c->stream) == hipSuccess;
  if (ok) ok = fwd_launch(c, dX, nullptr, (int64_t)cs.size(), dY) == hipSuccess;
  if (ok) ok = hipMemcpyAsync(y.data(), dY, y.size() * 4, hipMemcpyDeviceToHost, c->stream) == hipSuccess;
  if (ok) ok = hipStreamSynchronize(c->stream) == hipSuccess;
  upir_dfree(c, dX);
  upir_dfree(c, dY);
  if (!ok) return false;
  // The choice is among the schedules the exhaustive batch tuner found best
  // on the (up to) ten tuned graphs most like this one, and the default.
  // Graphs are compared by their candidate-independent features (task and
  // byte shares per body, task count, bytes, lengths, edges, depth). Each
  // such schedule is scored by the model's prediction plus the mean of its
  // measured log2(time / default) over those graphs (the tuner timed every
  // candidate on them). On its own the model's error is of the order of the
  // differences it has to rank (the candidates of a large graph lie within
  // a few percent of each other): its argmin over all 27 sometimes took a
  // schedule that tuned graphs of another kind preferred (smaller graphs
  // favour smaller matvec tiles), and ranking only the nearest graphs' best
  // schedules by the prediction still flipped between two of them from one
  // trained model to the next. Without tuned graphs, each body takes the
  // tile whose candidates have the lowest mean prediction over the other
  // bodies' choices (nine predictions per mean).
  auto same = [](const upir_engine_sched &a, const upir_engine_sched &b) {
    return a.tile_axpy == b.tile_axpy && a.tile_sum == b.tile_sum && a.rows_matvec == b.rows_matvec;
  };
  struct Near {
    float d;
    upir_engine_sched best;
    const std::vector<float> *rel;
  };
  std::vector<Near> near;
  for (const auto &kv : c->tuned_engine) {
    auto g = c->tuned_engine_graph.find(kv.first);
    if (g == c->tuned_engine_graph.end()) continue;
    auto r = c->tuned_engine_rel.find(kv.first);
    float d = 0.0f;
    for (int q = 0; q < 12; ++q) d += (g->second[(size_t)q] - X[(size_t)q]) * (g->second[(size_t)q] - X[(size_t)q]);
    near.push_back(Near{d, kv.second.first,
                        r != c->tuned_engine_rel.end() && r->second.size() == cs.size() ? &r->second : nullptr});
  }
  const size_t kn = std::min<size_t>(10, near.size());
  std::partial_sort(near.begin(), near.begin() + (ptrdiff_t)kn, near.end(),
                    [](const Near &a, const Near &b) { return a.d < b.d; });
  int pick = -1, seen = 0;
  float pick_score = 0.0f;
  for (size_t i = 0; i < cs.size(); ++i) {
    bool in = i == 0;  // candidate 0, the default, always takes part
    for (size_t j = 0; j < kn && !in; ++j) in = same(near[j].best, cs[i]);
    if (!in) continue;
    seen += i > 0;
    double m = 0.0;
    int nm = 0;
    for (size_t j = 0; j < kn; ++j)
      if (near[j].rel) {
        m += (*near[j].rel)[i];
        ++nm;
      }
    const float score = y[i] + (nm ? (float)(m / nm) : 0.0f);
    if (pick < 0 || score < pick_score) {
      pick = (int)i;
      pick_score = score;
    }
  }
  if (seen > 0) {
    es = cs[(size_t)pick];
    return true;
  }
  double sum[3][3] = {}, cnt[3][3] = {};
  for (size_t i = 0; i < cs.size(); ++i)
    for (int k = 0; k < 3; ++k) {
      const int q = choice_index(k, class_tile(cs[i], k));
      if (q < 0) continue;
      sum[k][q] += y[i];
      cnt[k][q] += 1;
    }
  int best[3] = {0, 0, 0};
  for (int k = 0; k < 3; ++k)
    for (int q = 1; q < 3; ++q)
      if (cnt[k][q] > 0 && (cnt[k][best[k]] == 0 || sum[k][q] / cnt[k][q] < sum[k][best[k]] / cnt[k][best[k]])) best[k] = q;
  es = upir_engine_sched{choice_tile(0, best[0]), choice_tile(1, best[1]), choice_tile(2, best[2])};
  return true;
}

upir_status resolve_engine_sched(upir_ctx *c, upir_engine_sched &es, int32_t &source) {
  if (c->engine_set) {
    es = c->engine_sched;
    source = UPIR_ENGINE_FROM_CALLER;
    return UPIR_OK;
  }
  auto it = c->tuned_engine.find(batch_key(c));
  if (it != c->tuned_engine.end()) {
    es = it->second.first;
    source = UPIR_ENGINE_FROM_TUNER;
    return UPIR_OK;
  }
  if (model_pick_engine(c, es)) {
    source = UPIR_ENGINE_FROM_MODEL;
    return UPIR_OK;
  }
  es = engine_candidates()[0];
  source = UPIR_ENGINE_FROM_DEFAULT;
  return UPIR_OK;
}

}  // namespace upir

extern "C" upir_status upir_engine_sched_set(upir_ctx *c, const upir_engine_sched *es) {
  if (!c) return UPIR_EINVAL;
  if (!es) {
    c->engine_set = false;
    return UPIR_OK;
  }
  for (int64_t t : {es->tile_axpy, es->tile_sum, es->rows_matvec})
    if (t < 1 || t > (1 << 24)) return upir_fail(c, UPIR_EINVAL, "engine tile %lld", (long long)t);
  c->engine_sched = *es;
  c->engine_set = true;
  return UPIR_OK;
}

extern "C" upir_status upir_engine_sched_resolve(upir_ctx *c, upir_engine_sched *out, int32_t *source) {
  if (!c || !out) return UPIR_EINVAL;
  int32_t src = 0;
  upir_status st = resolve_engine_sched(c, *out, src);
  if (source) *source = src;
  return st;
}

extern "C" upir_status upir_engine_candidate(upir_ctx *c, int32_t idx, upir_engine_sched *out, float *feat) {
  if (!c || !out) return UPIR_EINVAL;
  const auto cs = engine_candidates();
  if (idx < 0 || idx >= (int)cs.size()) return upir_fail(c, UPIR_EINVAL, "engine candidate %d of %zu", idx, cs.size());
  *out = cs[idx];
  if (feat) batch_features(c, cs[idx], feat);
  return UPIR_OK;
}

// ------------------------------------------------------------------- tuner
extern "C" upir_status upir_candidates(upir_ctx *c, upir_loop_h lp, int32_t *count) {
  if (!c || !lp || !count || !c->loops.count(lp)) return UPIR_EINVAL;
  *count = candidate_count(c, lp);
  return UPIR_OK;
}

extern "C" upir_status upir_candidate_features(upir_ctx *c, upir_loop_h lp, int32_t idx, float *feat,
                                               upir_spmd *sp_out, upir_sched *sc_out) {
  if (!c || !lp || !c->loops.count(lp)) return UPIR_EINVAL;
  auto cs = candidates(c, lp);
  if (idx < 0 || idx >= (int)cs.size()) return upir_fail(c, UPIR_EINVAL, "candidate %d of %zu", idx, cs.size());
  if (feat) features(lp, cs[idx], feat);
  if (sp_out) *sp_out = cs[idx].sp;
  if (sc_out) *sc_out = cs[idx].sc;
  return UPIR_OK;
}

// Run `lp` under candidate k `reps` times; median time in microseconds.
static upir_status time_candidate(upir_ctx *c, upir_loop_obj *tmp, const Cand &k, int reps, double &us) {
  tmp->sched = k.sc;
  Plan pl;
  upir_status st = resolve_plan(c, &k.sp, tmp, pl);
  if (st) return st;
  if (tmp->has_red) {  // size the reduction slots first; the result slot moves with them
    st = ensure_scratch(c, tmp, pl.S.T);
    if (st) return st;
    tmp->red.result = tmp->scratch + SCR_RESULT;
  }
  st = launch_plan(c, tmp, pl, false);  // warm-up
  if (st) return st;
  std::vector<float> ms;
  hipEvent_t a, b;
  HIPTRY(c, hipEventCreate(&a));
  HIPTRY(c, hipEventCreate(&b));
  for (int r = 0; r < reps && st == UPIR_OK; ++r) {
    if (hipEventRecord(a, c->stream) != hipSuccess) {
      st = upir_fail(c, UPIR_EHIP, "event record");
      break;
    }
    st = launch_plan(c, tmp, pl, false);
    if (st) break;
    float t = 0;
    if (hipEventRecord(b, c->stream) != hipSuccess || hipEventSynchronize(b) != hipSuccess ||
        hipEventElapsedTime(&t, a, b) != hipSuccess)
      st = upir_fail(c, UPIR_EHIP, "event wait");
    ms.push_back(t);
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (st) return st;
  std::sort(ms.begin(), ms.end());
  us = 1e3 * ms[ms.size() / 2];
  return UPIR_OK;
}

extern "C" upir_status upir_tune(upir_ctx *c, const upir_spmd *spmd, upir_loop_h lp, int32_t reps, upir_sched *best,
                                 upir_spmd *best_spmd, double *best_us) {
  (void)spmd;
  if (!c || !lp || !c->loops.count(lp)) return UPIR_EINVAL;
  if (c->none) return upir_fail(c, UPIR_ESTATE, "host-only context");
  if (c->capturing) return upir_fail(c, UPIR_ESTATE, "tuning during graph capture");
  if (reps < 1 || reps > 1000) return upir_fail(c, UPIR_EINVAL, "reps");
  {
    upir_status s0 = settle(c);
    if (s0) return s0;
  }
  // scratch copies of read-write outputs, and an internal reduction result
  upir_loop_obj tmp = *lp;
  tmp.scratch = nullptr;
  tmp.part_cap = 0;
  tmp.ws = lp->ws;
  unsigned char pay[sizeof(MatmulP) + 16];
  upir_status st = resolve_payload(c, lp, pay);
  if (st) return st;
  tmp.args_dev = 1;
  std::vector<void *> owned;
  auto own = [&](size_t bytes) -> void * {
    void *p = upir_dalloc(c, bytes);
    if (p) owned.push_back(p);
    return p;
  };
  auto cleanup = [&]() {
    (void)settle(c);  // a deferred fold of the copy writes into its scratch
    (void)hipStreamSynchronize(c->stream);
    for (void *p : owned) upir_dfree(c, p);
    upir_dfree(c, tmp.scratch);
  };
  // extent (elements) of the index range a 1-D loop touches
  int64_t lo = lp->loop.dim[0].lb, hi = lo + (lp->n > 0 ? (lp->n - 1) * lp->loop.dim[0].step : 0);
  if (hi < lo) std::swap(lo, hi);
  const size_t span1 = (size_t)(hi + 1);
  switch (lp->kind) {
    case UPIR_BODY_AXPY: {  // y is read and written: time on a copy
      const AxpyP &p = *(const AxpyP *)pay;
      float *y2 = (float *)own(span1 * 4);
      if (!y2) break;
      if (lp->n > 0) (void)hipMemcpyAsync(y2, p.y, span1 * 4, hipMemcpyDeviceToDevice, c->stream);
      upir_axpy_args a{p.a, 0, p.x, y2};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    case UPIR_BODY_COVER: {
      int32_t *c2 = (int32_t *)own((size_t)std::max<int64_t>(lp->n, 1) * 4);
      if (!c2) break;
      upir_cover_args a{c2};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    case UPIR_BODY_SUM: {
      const SumP &p = *(const SumP *)pay;
      upir_sum_args a{p.x, p.dtype, 0};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    case UPIR_BODY_JACOBI5: {  // dst on a scratch grid of the same pitch
      const JacobiP &p = *(const JacobiP *)pay;
      const int64_t rows = lp->loop.dim[0].lb + lp->cnt[0] + 1;
      float *d2 = (float *)own((size_t)rows * p.ld * 4);
      if (!d2) break;
      upir_jacobi5_args a{p.src, d2, p.ld};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    case UPIR_BODY_FILTER7: {  // dst on a scratch grid of the same pitch
      const Filter7P &p = *(const Filter7P *)pay;
      const int64_t rows = lp->loop.dim[0].lb + lp->cnt[0] + 3;
      float *d2 = (float *)own((size_t)rows * p.ld * 4);
      if (!d2) break;
      upir_filter7_args a{p.src, d2, p.w, p.ld};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    case UPIR_BODY_MATVEC: {
      const MatvecP &p = *(const MatvecP *)pay;
      float *y2 = (float *)own(span1 * 4);
      if (!y2) break;
      upir_matvec_args a{p.A, p.x, y2, p.cols, p.lda};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    case UPIR_BODY_OWNER: {
      int32_t *o2 = (int32_t *)own((size_t)std::max<int64_t>(lp->n, 1) * 4);
      if (!o2) break;
      upir_owner_args a{o2};
      memcpy(tmp.args, &a, sizeof a);
      break;
    }
    default: {  // matmul: C on a scratch matrix, BF16 workspace of the loop
      const MatmulP &p = *(const MatmulP *)pay;
      float *c2 = (float *)own((size_t)std::max<int64_t>(p.M, 1) * p.ldc * 4);
      if (!c2) break;
      upir_matmul_args a = *(const upir_matmul_args *)lp->args;
      a.A = p.A;
      a.B = p.B;
      a.C = c2;
      a.workspace = p.ah;
      a.workspace_bytes = upir_matmul_workspace_bytes(lp->kind, p.M, p.N, p.K);
      memcpy(tmp.args, &a, sizeof a);
    }
  }
  if (owned.empty() && lp->kind != UPIR_BODY_SUM) {
    cleanup();
    return upir_fail(c, UPIR_ENOMEM, "tuner scratch");
  }
  if (lp->has_red) {
    tmp.red.result_on_host = 0;
    tmp.part_cap = 0;
  }
  tmp.part_cap = tmp.has_red ? 8192 : 0;
  tmp.scratch = (unsigned char *)upir_dalloc(c, scratch_bytes(tmp.part_cap));
  if (!tmp.scratch) {
    cleanup();
    return upir_fail(c, UPIR_ENOMEM, "tuner scratch");
  }
  st = clear_scratch(c, &tmp, tmp.scratch, tmp.part_cap);
  if (st) {
    cleanup();
    return st;
  }
  if (tmp.has_red) tmp.red.result = tmp.scratch + SCR_RESULT;
  auto cs = candidates(c, lp);
  double bus = 1e300;
  int bi = -1;
  for (int i = 0; i < (int)cs.size(); ++i) {
    double us = 0;
    st = time_candidate(c, &tmp, cs[i], reps, us);
    if (st) break;
    TuneRow row{};
    features(lp, cs[i], row.feat);
    row.log2_us = (float)log2(std::max(us, 1e-3));
    row.loop_key = (int64_t)(lp->key & 0x7FFFFFFFFFFFFFFFULL);
    c->db.push_back(row);
    if (us < bus) {
      bus = us;
      bi = i;
    }
  }
  cleanup();
  if (st) return st;
  if (bi < 0) return upir_fail(c, UPIR_EUNSUPPORTED, "no candidate schedules for this loop");
  c->tuned[lp->key] = TunedChoice{cs[bi].sp, cs[bi].sc, bus};
  if (best) *best = cs[bi].sc;
  if (best_spmd) *best_spmd = cs[bi].sp;
  if (best_us) *best_us = bus;
  return UPIR_OK;
}
