// Chunk arithmetic against 128-bit integers: sizes, chunks and launch shapes
// up to the largest that a caller may give.
#include "chunk_math.h"

#include <stdio.h>

#include <random>

typedef __int128 i128;

int main() {
  std::mt19937_64 rng(7);
  auto pick = [&](int64_t top) {  // spread over the logarithm, the ends often
    switch (rng() % 6) {
      case 0: return (int64_t)1;
      case 1: return top;
      default: {
        const int bits = 1 + (int)(rng() % 63);
        const int64_t v = (int64_t)(rng() >> (64 - bits)) + 1;
        return v < 1 || v > top ? top : v;
      }
    }
  };
  for (int it = 0; it < 2000000; ++it) {
    const int64_t n = rng() % 20 ? pick((int64_t)1 << 38) : 0, chunk = pick(INT64_MAX);
    const int64_t U = pick(1024), T = pick(1 << 24);
    const int64_t c = upir::bounded_chunk(chunk, n), k = upir::chunk_count(n, c);
    // the same items in each chunk: as many chunks, and all ends below n alike
    const i128 want = n ? ((i128)n + chunk - 1) / chunk : 0;
    bool ok = c >= 1 && c <= chunk && k == want && (n == 0 || (k - 1) * c < n) && (i128)k * c >= n;
    ok = ok && (i128)T * c < ((i128)1 << 63);                       // a team's first tile, a stride of tiles
    const int64_t len = upir::claim_length(n, c, U);
    const i128 full = (i128)chunk * U;
    ok = ok && len == (full < n ? (int64_t)full : len) && (full < n || len >= n || len == full) && len <= (n > 0 ? n : 0);
    ok = ok && (n == 0 || len >= 1);
    ok = ok && ((i128)T + 1) * len + n < ((i128)1 << 63);           // the counter after every team's last claim
    if (!ok) {
      printf("n %lld chunk %lld U %lld T %lld: c %lld k %lld len %lld\n", (long long)n, (long long)chunk, (long long)U,
             (long long)T, (long long)c, (long long)k, (long long)len);
      return 1;
    }
  }
  puts("ok");
  return 0;
}
