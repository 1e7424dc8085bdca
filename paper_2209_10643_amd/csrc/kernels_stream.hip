// One-dimensional streaming loops under schedules whose units own runs of
// consecutive iterations (gfx950): static blocks, static chunks, dynamic and
// guided claims.
//
// Paper: sec. 3.2 (worksharing with schedule inside an SPMD region), sec. 5
// (reduction).
//
// Under these schedules a team owns ranges of consecutive iterations: its
// block (static), every T-th run of U chunks (static, chunk) or what it
// claims (dynamic, guided). Each unit of the team owns a run inside the
// range, and a kernel that walks it unit by unit touches as many cache lines
// per load as there are lanes: AXPY over 102,400,000 elements under
// schedule(static) ran at 0.40 TB/s (3,045 us). The bodies here (AXPY, SUM)
// cannot observe which unit of a team runs an iteration, so the team goes
// through each of its ranges together, 16 bytes per lane side by side. The
// team's iterations stay what the schedule assigns.
//
// Only reductions whose value does not depend on the order (maximum,
// minimum, exact integers) or is carried in float64 take this path: a
// float32 sum keeps the order its schedule fixes (kernels_loop.hip).
#include "upir.h"
#include "upir_launch.h"

namespace upir {

template <class T> struct Vec16;  // 16 bytes of T, aligned like T
template <> struct Vec16<float> { typedef float V __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec16<double> { typedef double V __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct Vec16<int32_t> { typedef int32_t V __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec16<long long> { typedef long long V __attribute__((ext_vector_type(2), aligned(8))); };

// Ranges of a team, in order. Dynamic and guided claims are made by thread 0
// one ahead: the claim of the next range is in flight while the team runs
// the current one.
struct TeamRanges {
  const SchedK &S;
  const int64_t n;
  const int team;
  int64_t at = 0;                  // static: the next range's start
  int64_t step = 0, len = 0;
  long long nlo = 0, nhi = 0;      // thread 0: the claimed next range
  long long ticket = 0;            // thread 0: the claim's number
  long long first = 0, base = 0, glen = 0;  // guided: the round's first ticket, first iteration, length
  int par = 0;
  // Dynamic, guided: the claim queues and this team's. An atomic on one
  // address takes 10 ns of the whole launch, for 25,000 ranges and as many
  // again for the teams' last tickets more than the loop itself, so the
  // tickets are dealt over up to DYN_QUEUES counters, at least 32 teams to
  // each so that they still balance one another: ticket k of queue q is
  // ticket k nq + q of the sequence. Teams q, q + 8, ... share an XCD.
  // AXPY, dynamic, chunk 16, one counter against eight: 102,400,000 elements
  // 328 -> 218 us, 10,000,000 38 -> 24 us, 1,000,003 10.0 -> 6.0 us.
  const int nq, q;

  __device__ TeamRanges(const SchedK &S_, int64_t n_, int team_)
      : S(S_), n(n_), team(team_), nq(S_.T < 64 ? 1 : (S_.T / 32 < DYN_QUEUES ? S_.T / 32 : DYN_QUEUES)), q(team_ % nq) {
    if (S.policy == POL_STATIC) {
      int64_t hi;
      block_range(n, S.T, team, at, hi);
      len = hi - at;
      step = n + 1 - at;  // one range
      if (len <= 0) at = n;
      return;
    }
    // chunk x U, at most n
    const int64_t c = S.chunk < 1 ? 1 : S.chunk;
    const int64_t cu = c > quot(n, S.U) ? (n > 0 ? n : 1) : c * S.U;
    if (S.policy == POL_CHUNK) {
      len = cu;
      step = (int64_t)S.T * cu;
      at = (int64_t)team * cu;
      // cu is exact unless it exceeds n, and then team 0 owns everything
      if (cu == n && team > 0) at = n;
    } else {
      len = cu;
      if (threadIdx.x == 0) {
        glen = guided_len(n);
        claim();
      }
    }
  }

  __device__ long long guided_len(long long rem) const {
    const long long q = rem / (2LL * S.T);
    return q > len ? q : len;
  }

  __device__ long long *counter() const { return S.dyn_next + q * SLOT_WORDS; }

  // One fetch-add of a ticket; ticket k takes range k of a sequence that n, T
  // and the chunk fix. Dynamic: ranges of chunk U. Guided: rounds of T ranges
  // of max(chunk U, r / 2T) iterations, r = what remains when the round
  // begins, so that thread 0 reaches its ticket's range in about
  // log2(n / chunk U) steps; once the minimum is reached the rest is one
  // multiplication. (A compare-exchange on the position made 256 teams retry
  // against each other, 187 us for 1,772,561 iterations; the same sizes
  // recomputed for each of the tickets cost 0.2 us a ticket.)
  __device__ void claim() {
    ticket = (long long)atomicAdd((unsigned long long *)counter(), 1ULL) * nq + q;
    if (S.policy == POL_DYNAMIC) {
      glen = len;
    } else {
      while (glen > len && ticket - first >= S.T) {
        base += glen * S.T;
        first += S.T;
        glen = guided_len(n - base);
      }
    }
    const long long left = (n - base + glen - 1) / glen;  // ranges from the round's first on, at this length
    nlo = ticket - first < left ? base + (ticket - first) * glen : n;
    nhi = n - nlo > glen ? nlo + glen : n;
  }

  // The next range; false when there is none. All threads of the team call it.
  __device__ bool next(int64_t &lo, int64_t &hi) {
    if (S.policy == POL_STATIC || S.policy == POL_CHUNK) {
      if (at >= n) return false;
      lo = at;
      hi = n - at > len ? at + len : n;
      at = n - at > step ? at + step : n;
      return true;
    }
    __shared__ long long s_lo[2], s_hi[2];
    if (threadIdx.x == 0) {
      s_lo[par] = nlo < n ? nlo : n;
      s_hi[par] = nhi;
    }
    __syncthreads();  // the other pair is free again: its readers have passed this barrier
    lo = s_lo[par];
    hi = s_hi[par];
    par ^= 1;
    if (lo >= hi) {
      // A team stops at its first ticket past the last range, so a queue of
      // r ranges and t teams hands out r + t tickets and the last of them
      // re-arms the counter: no second counter of leaving teams.
      if (threadIdx.x == 0) {
        const long long R = ranges_total();
        const long long r = R > q ? (R - q + nq - 1) / nq : 0, t = (S.T - q + nq - 1) / nq;
        if (ticket == (r + t - 1) * nq + q)
          __hip_atomic_store(counter(), 0LL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      return false;
    }
    if (threadIdx.x == 0) claim();
    return true;
  }

  // Thread 0, after its last claim: the number of ranges.
  __device__ long long ranges_total() const {
    return first + (n - base + glen - 1) / glen;
  }
};

// By element type: a deduced vector type would lose its element alignment.
template <bool NT, class T>
__device__ __forceinline__ typename Vec16<T>::V ldv(const typename Vec16<T>::V *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, class T>
__device__ __forceinline__ void stv(typename Vec16<T>::V *p, typename Vec16<T>::V v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// x, y: the element of iteration 0. AXPY (y != null) or SUM.
template <bool AXPY, class T, class A, int OP, bool NT>
__global__ void __launch_bounds__(1024) k_team_stream(int64_t n, SchedK S, RedK R, float a, const T *x, T *y) {
  typedef typename Vec16<T>::V V;
  constexpr int W = 16 / sizeof(T);
  constexpr int UN = AXPY ? 4 : 8;  // vectors in flight per lane and array
  const int U = blockDim.x, tid = threadIdx.x;
  A acc = red_identity<A>(OP ? OP : RED_SUM);
  auto one = [&](int64_t i) {
    if constexpr (AXPY) {
      const float v = __builtin_fmaf(a, x[i], y[i]);
      y[i] = v;
      if (OP) acc = red_apply(OP, acc, v);
    } else {
      acc = red_apply(OP, acc, (A)x[i]);
    }
  };
  auto vec = [&](const V &xv, V yv, V *out) {
    if constexpr (AXPY) {
#pragma unroll
      for (int q = 0; q < W; ++q) yv[q] = __builtin_fmaf(a, xv[q], yv[q]);
      stv<NT, T>(out, yv);
      if (OP) {
#pragma unroll
        for (int q = 0; q < W; ++q) acc = red_apply(OP, acc, (A)yv[q]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < W; ++q) acc = red_apply(OP, acc, (A)xv[q]);
    }
  };
  TeamRanges ranges(S, n, blockIdx.x);
  int64_t lo, hi;
  while (ranges.next(lo, hi)) {
    // A range of no more elements than units: one each, in one access. In
    // vectors its ends would be accesses of their own, one after another
    // (AXPY, 65,000 elements in 1,024 static blocks: 3.4 us, 4.4 with them;
    // chunk 1 from element 1, 5,000,003 elements: 39 and 95).
    if (hi - lo <= U) {
      if (tid < hi - lo) one(lo + tid);
      continue;
    }
    // elements up to the first 16-byte boundary of the array that is written
    // (or read, for SUM), side by side (at most three, which a team of one or
    // two units takes in turn); x may stay unaligned beside y
    const uintptr_t at = (uintptr_t)(AXPY ? (const T *)y + lo : x + lo);
    int64_t head = ((0 - at) & 15) / sizeof(T);
    if (head > hi - lo) head = hi - lo;
    for (int64_t i = tid; i < head; i += U) one(lo + i);
    lo += head;
    const int64_t nv = (hi - lo) / W;
    const V *xv = (const V *)(x + lo);
    V *yv = AXPY ? (V *)(y + lo) : nullptr;
    int64_t m = tid;
    for (; m + (int64_t)(UN - 1) * U < nv; m += (int64_t)UN * U) {
      V xb[UN], yb[UN] = {};
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        xb[u] = ldv<NT, T>(&xv[m + u * U]);
        if constexpr (AXPY) yb[u] = ldv<NT, T>(&yv[m + u * U]);
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) vec(xb[u], yb[u], yv + m + u * U);
    }
    // what is left of the range, still loaded together
    if (m < nv) {
      V xb[UN - 1], yb[UN - 1] = {};
#pragma unroll
      for (int u = 0; u < UN - 1; ++u)
        if (m + (int64_t)u * U < nv) {
          xb[u] = ldv<NT, T>(&xv[m + u * U]);
          if constexpr (AXPY) yb[u] = ldv<NT, T>(&yv[m + u * U]);
        }
#pragma unroll
      for (int u = 0; u < UN - 1; ++u)
        if (m + (int64_t)u * U < nv) vec(xb[u], yb[u], yv + m + u * U);
    }
    for (int64_t i = lo + nv * W + tid; i < hi; i += U) one(i);  // at most three, as at the start
  }
  if constexpr (OP != RED_NONE) finish_reduction<A>(R, acc);
  fold_hook(R);
}

template <bool AXPY, class T, class A, int OP>
static hipError_t go_team(const LoopK &L, const SchedK &S, const RedK &R, float a, const T *x, T *y, hipStream_t st) {
  const bool nt = (uint64_t)L.n * sizeof(T) * (AXPY ? 2 : 1) >= (64ull << 20);  // as for the chunk-4 streams
  x += L.lb[0];
  if (AXPY) y += L.lb[0];
  if (nt)
    hipLaunchKernelGGL((k_team_stream<AXPY, T, A, OP, true>), dim3(S.T), dim3(S.U), 0, st, L.n, S, R, a, x, y);
  else
    hipLaunchKernelGGL((k_team_stream<AXPY, T, A, OP, false>), dim3(S.T), dim3(S.U), 0, st, L.n, S, R, a, x, y);
  return hipGetLastError();
}

template <class T, class A>
static hipError_t go_team_sum(const LoopK &L, const SchedK &S, const RedK &R, const void *x, hipStream_t st) {
  T *none = nullptr;
  if (R.op == RED_MAX) return go_team<false, T, A, RED_MAX>(L, S, R, 0.0f, (const T *)x, none, st);
  if (R.op == RED_MIN) return go_team<false, T, A, RED_MIN>(L, S, R, 0.0f, (const T *)x, none, st);
  if constexpr (std::is_same<T, float>::value) return hipErrorInvalidValue;
  else return go_team<false, T, A, RED_SUM>(L, S, R, 0.0f, (const T *)x, none, st);
}

// Bodies and reductions whose result does not depend on which unit of a team
// runs an iteration.
bool team_stream_body(int32_t body, int32_t sum_dtype, int32_t op) {
  if (body == UPIR_BODY_AXPY) return op != RED_SUM;
  return body == UPIR_BODY_SUM && op != RED_NONE && (sum_dtype != UPIR_DT_F32 || op != RED_SUM);
}

// Unit steps, untiled, iterations dealt over teams and units: the schedules
// above. distribute(teams) and distribute(units) run on few units by
// definition and keep the schedule-exact kernel, as do the float32 sums.
bool team_stream_supports(int32_t body, const void *payload, const LoopK &L, const SchedK &S, const RedK &R) {
  if (L.nd != 1 || L.step[0] != 1 || S.tiled || S.dist != DIST_TU) return false;
  return team_stream_body(body, body == UPIR_BODY_SUM ? ((const SumP *)payload)->dtype : 0, R.op);
}

hipError_t launch_team_stream(int32_t body, const void *payload, const LoopK &L, const SchedK &S, const RedK &R,
                              hipStream_t st) {
  if (body == UPIR_BODY_AXPY) {
    const AxpyP &p = *(const AxpyP *)payload;
    switch (R.op) {
      case RED_NONE: return go_team<true, float, float, RED_NONE>(L, S, R, p.a, p.x, p.y, st);
      case RED_MAX: return go_team<true, float, float, RED_MAX>(L, S, R, p.a, p.x, p.y, st);
      case RED_MIN: return go_team<true, float, float, RED_MIN>(L, S, R, p.a, p.x, p.y, st);
    }
    return hipErrorInvalidValue;
  }
  const SumP &p = *(const SumP *)payload;
  switch (p.dtype) {
    case UPIR_DT_F32: return go_team_sum<float, float>(L, S, R, p.x, st);
    case UPIR_DT_F64: return go_team_sum<double, double>(L, S, R, p.x, st);
    case UPIR_DT_I32: return go_team_sum<int32_t, long long>(L, S, R, p.x, st);
    case UPIR_DT_I64: return go_team_sum<long long, long long>(L, S, R, p.x, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace upir
