// Launch rules that depend on sizes alone: plain host arithmetic without HIP, so that a test can compile it with the host
// compiler and walk the sizes at which a rule changes or a launch limit lies.
#pragma once
#include <algorithm>
#include <stddef.h>
#include <stdint.h>

namespace fq {

// Whether two ranges of memory share a byte.
inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes)
{
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return p < q + b_bytes && q < p + a_bytes;
}

// What one dimension of a launch can hold: the work items along it are counted in 32 bits.
inline bool launch_holds(long long workgroups, int threads) { return workgroups * threads < (1LL << 32); }

// The weight-streaming kernel for at most 4 rows has 512 threads per 16 columns.
constexpr int SKINNY_COLUMNS = 16, SKINNY_THREADS = 512;
inline bool skinny_holds(long long N) { return launch_holds((N + SKINNY_COLUMNS - 1) / SKINNY_COLUMNS, SKINNY_THREADS); }

// Grid of the absmax pass: `blocks` workgroups side by side cover the columns (64 * vec of them each), `strips` of
// rows_per_strip rows each cover the rows.  Every workgroup leaves one candidate.
struct AbsmaxGrid {
    int blocks, strips, rows_per_strip;
    int candidates() const { return blocks * strips; }
};

// Candidates that the workspace has room for: one per column block however wide the matrix, and enough strips of a narrow one.
constexpr int MAX_CANDIDATES = 1024;
inline long long candidate_capacity(long long K) { return std::max<long long>(MAX_CANDIDATES, (K + 63) / 64 * 64); }

// Strips of 64 rows (16 loads in flight for each of the four waves) while that gives at most 512 workgroups, then higher
// ones.  Odd multiples of 64: with a power-of-two row stride, strips that start a power-of-two number of rows apart hit
// the same memory channels (16384 x 8192 bf16: 54 us at 576 rows, 59 us at 512).  At most 1024 candidates, or one strip.
inline AbsmaxGrid absmax_grid(long long M, long long K, int vec)
{
    const long long bx = (K + 64 * vec - 1) / (64 * vec);
    long long rpb = (M * bx + 511) / 512;
    rpb = std::max(64LL, (rpb + 63) / 64 * 64);
    if (rpb > 64 && (rpb / 64) % 2 == 0) rpb += 64;
    while (rpb < M && (M + rpb - 1) / rpb * bx > MAX_CANDIDATES) rpb *= 2;
    rpb = std::min(rpb, M);
    return AbsmaxGrid{(int)bx, (int)((M + rpb - 1) / rpb), (int)rpb};
}

}  // namespace fq
