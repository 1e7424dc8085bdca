// Chunk arithmetic of the schedules for every chunk that a caller may give
// (1 .. 2^63 - 1): products with teams or units stay inside 64 bits.
#pragma once
#include <stdint.h>

namespace upir {

// The chunk of a schedule over `items` (iterations or tiles): one of as many
// items as there are, or of more, is the same schedule.
constexpr int64_t bounded_chunk(int64_t chunk, int64_t items) {
  return chunk <= items ? chunk : items > 0 ? items : 1;
}

// Chunks that `items` make.
constexpr int64_t chunk_count(int64_t items, int64_t chunk) { return items > 0 ? (items - 1) / chunk + 1 : 0; }

// Iterations of a team's claim, at least: a chunk for each of its units, or
// all n of them where that is less.
constexpr int64_t claim_length(int64_t n, int64_t chunk, int64_t units) {
  return chunk > n / units ? n : chunk * units;
}

}  // namespace upir
