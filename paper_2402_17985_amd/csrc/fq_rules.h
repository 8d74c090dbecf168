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

// Integer products of few output tiles: which kernel takes one.  TILED: none of these, the large-tile kernels.
enum class FewTiles { TILED, SKINNY, STREAM, RING };
struct FewTilesChoice {
    FewTiles kernel;
    int bm, bn;      // tile of STREAM and RING
};

// The tiles in the order in which they are tried, and the shortest reduction (bytes of a quantized row) from which each is taken,
// for INT8, packed nibbles and E3M2, unbatched and batched (no batched E3M2).  Below it there is too little to split: the partial
// sums that meet in LDS (64 KiB of them for 64 x 64 tiles and eight waves) cost more than the latency that is hidden.
// Us, this tile / the 128 x 128 tiles (E3M2: 256 x 256) at half of it and from it on: INT8 512 x 2048, 64 x 64 tiles, 256 bytes
// 4.9 / 4.2, 640 5.5 / 6.3, 1024 5.7 / 8.4; 384 x 4096, 96 x 64 tiles, 512 bytes 6.9 / 6.6, 1024 7.9 / 9.1; nibbles 512 x 4096, 128 x 64
// tiles, 512 bytes 9.4 / 7.6, 1024 11.3 / 10.3, 2048 14.9 / 15.2; E3M2 the same 384 bytes 8.5 / 6.8, 1152 10.0 / 10.1, 1536 11.0 / 11.6;
// batched nibbles 12 x 256 x 512, 128 x 64 tiles, 512 bytes 9.3 / 8.1, 1024 11.8 / 12.5.
constexpr int NEVER = 1 << 30;
struct FewTilesRow {
    int bm, bn, from[2][3];
};
constexpr FewTilesRow FEW_TILES[] = {
    {32, 32, {{0, 0, 0}, {512, 512, NEVER}}},
    {32, 64, {{0, 0, 0}, {512, 512, NEVER}}},
    {64, 64, {{640, 384, 0}, {512, 512, NEVER}}},
    {32, 128, {{0, 0, 0}, {512, 512, NEVER}}},
    {96, 64, {{1024, 1024, 384}, {1024, 512, NEVER}}},
    {128, 64, {{0, 2048, 1152}, {512, 1024, NEVER}}},
    {64, 128, {{0, 1280, 768}, {512, 1024, NEVER}}},
    {128, 128, {{0, 0, NEVER}, {512, 512, NEVER}}},
};

//   - At most 4 rows, or 4-bit values, at most 16 and at most 64 columns per CU: the weights go straight into registers (gemm_skinny; INT8 at 8 and 16
//     rows, 6400 x 15360: 23.0, 24.3 us against 20.9, 21.0 for the stream kernel; nibbles 10.2, 10.4 against 11.6, 11.6).
//     Its 512 threads per 16 columns are more than a launch holds from 2^27 columns on; those go to the 128-column tiles.
//   - Otherwise the smallest tile with which one round of workgroups, one per CU, covers the output: a larger one leaves CUs
//     idle, a smaller one takes a second round and reads the operands more often (INT8 12544 x 4096, 256 rows: 32 x 64 30.6,
//     64 x 64 21.7, 96 x 64 25.2 us).  Up to 96 x 64 the reduction is split over the waves.  Beyond it INT8 goes through the
//     ring (4608 x 11008, 128 rows, 128 x 64: 16.3 us, by split waves 18.5), 4-bit values stay with split waves (12544 x 4096, 500
//     rows: nibbles 29.5 us, ring 37.6, 128 x 128 kernel 36.3; E3M2 27.3, its 256 x 256 kernel 46.2) up to 128 x 64; 128 x 128 tiles
//     through the ring for INT8 and nibbles (4608 x 11008, 200 rows: 19.4 and 20.7 us against 26.0 and 21.9).
//   - Batched products with a reduction of under 512 bytes stay with the tiled kernels throughout.
//   - Tall INT8 outputs of 128 x 64 tiles from 1024 bytes on (2048 x 1024, us, ring / 128 x 128 tiles: 640 bytes 6.2 / 5.5, 1024 7.6 /
//     8.0; wide 512 x 4096 of 640 bytes 6.1 / 7.6), batched nibbles of one 128-column tile not through the ring (64 x 512 x 128 of 1024
//     bytes 15.6 / 14.3, 40 x 512 x 128 13.0 / 13.2; 4 x 700 x 700 12.3 / 13.9).
inline FewTilesChoice few_tiles(long long M, long long N, int rowbytes, int bits, long long count, long long cus)
{
    const int batched = count > 1 ? 1 : 0, mode = bits == 8 ? 0 : bits == 4 ? 1 : 2;
    const FewTilesChoice tiled = {FewTiles::TILED, 0, 0};
    if (batched && rowbytes < 512) return tiled;
    if ((M <= 4 && skinny_holds(N)) || (mode != 0 && M <= 16 && N <= 64 * cus)) return {FewTiles::SKINNY, 0, 0};
    for (const FewTilesRow& t : FEW_TILES) {
        if ((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn) * count > cus) continue;
        if (rowbytes < t.from[batched][mode]) return tiled;
        const bool large = t.bm * t.bn == 128 * 128, middle = t.bm * t.bn == 128 * 64;
        if (mode == 0 && !batched && t.bm == 128 && t.bn == 64 && M > N && rowbytes < 1024) return tiled;
        if (mode == 1 && batched && large && N <= 128) return tiled;
        return {large || (mode == 0 && middle) ? FewTiles::RING : FewTiles::STREAM, t.bm, t.bn};
    }
    return tiled;
}

// Workgroups of the one-kernel quantizer, each of which walks a run of the M rows in strips of R: a row each while there are
// CUs for them, then strips, and no more than the CUs hold at once (`resident` per CU).
inline int direct_workgroups(int M, int R, int cus, int resident)
{
    return (int)std::min<long long>(std::max((M + (long long)R - 1) / R, (long long)std::min(M, cus)), (long long)cus * resident);
}

// ---- the kernel of the whole layer for a few rows (fq_linear_few.hip) ----
constexpr int FEW_WAVES = 16, FEW_PREP_WAVES = 8;             // four waves per SIMD: 128 registers each
constexpr int FEW_ROWS = 16, FEW_LDS = 160 * 1024;            // rows of an MFMA; LDS of a CU
constexpr int FEW_TABLE = 256, FEW_LDS_FIXED = (FEW_TABLE + FEW_WAVES + 4) * 4;   // multipliers m(n), wave maxima, a count
constexpr int FEW_PAD = 16;                                   // after a row in LDS
constexpr uint32_t few_row(uint32_t rowbytes) { return (rowbytes + 127) / 128 * 128 + FEW_PAD; }   // rows on different banks
constexpr int few_rows_held(int x_bytes) { return x_bytes == 4 ? 4 : 8; }         // per thread: 64 registers

struct FewShape {
    int M, K, ld, Kpad, N;
    int prep_waves, slots;     // waves that quantize; rows dealt over so many sets of them
    int cols;                  // columns of a workgroup and round
    int turns;                 // steps of the reduction less 1 where workgroups begin at different ones; else -1
};
struct FewPlan {
    FewShape sh;
    int fn, threads;           // fragments of 16 columns
    unsigned grid;
    size_t lds;
};

// One row.  The other choice is linear_decode_kernel or, for 4-bit weights beyond 16384 columns, the separate kernels.  linear_decode_kernel's
// preparation is shorter; from more than 16 columns per CU on (`wide`) it has several workgroups per CU, which repeat it, and while the
// second ones are few (up to `full`) the two kernels are near each other.  Us, bf16, dynamic scale where it says so, the other / this:
//   4-bit beyond 64 columns per CU   any K: nibbles 1 x 257 x 24576 12.9 / 9.7, 1803 x 24576 17.4 / 12.7, 4096 x 32000 20.8 / 18.1; E3M2 1024 x 24576 12.9 /
//                10.7, 5001 x 50000 7 % less; nibbles 4096 x 50000 (four rounds, three quarters full) 26.6 / 27.6, 4096 x 65536 32.0 / 31.3, 4096 x
//                100000 8 % more
//   whole K      INT8 2048 x 4096 7.3 / 7.4, 4096 x 1024 9.2 / 8.7, 2048 x 4112 8.4 / 7.2; 4096 x 36000 4 % less, 4096 x 40000 11 % more, 5120 x 50000 56.0 /
//                58.7, 7168 x 65536 3 % more, 3072 x 65536 7 % less, 8192 x 65536 102.2 / 101.8; nibbles 1024 x 4112 6.4 / 6.6, 1024 x 4300 6.6 / 6.5,
//                2048 x 4112 7.6 / 7.1; E3M2 4096 x 1024 9.1 / 9.2, 8192 x 1024 10.2 / 8.1, 1024 x 6000 7.0 / 7.0, 2048 x 4112 7.3 / 7.8, 2048 x 12288 9.5 /
//                8.9.  fp32: nibbles 1024 x 4300 6.0 / 6.6, 1024 x 12288 3-5 % less, 5120 x 2000 7.4 / 7.7, 8192 x 2000 14 % less; E3M2 2048 x 12288 static 4 %
//                more, 3072 x 4112 6.9 / 7.5, 4096 x 4300 4 % less
//   ragged K     (the last group is gathered, here by every CU too) dynamic: INT8 2507 x 4100 9.3 / 10.2, 2507 x 4300 10.3 / 10.1, 4090 x 4100 11.0 /
//                10.4, 6503 x 13000 equal, x 16384 26.9 / 28.2, 4090 x 24576 equal, x 32000 7 % more, fp32 less in all of these; nibbles 2507 x 4608
//                9.8 / 10.2, 2507 x 10000 equal, 3001 x 4608 10.6 / 10.5, 6503 x 4100 12.1 / 12.9, 8190 x 4100 16.1 / 13.0, fp32 3001 x 11008 10.7 /
//                11.3, 4503 x 4300 5 % less.  Static: INT8 2005 x 4100 8.1 / 7.7, nibbles 2005 x 5120 8.3 / 7.7, fp32 2005 x 8192 7.4 / 7.6, 2005 x
//                11008 6 % less, 2507 x 4100 6.9 / 7.7
inline bool few_takes_one_row(int N, int K, int bits, int x_bytes, bool dynamic, int cus)
{
    const long long n = N, per_cu = cus;
    const bool int8 = bits == 8, e3m2 = bits != 8 && bits != 4, fp32 = x_bytes == 4;
    const bool wide = n > 16 * per_cu, full = 2 * n > 33 * per_cu;
    if (!int8 && n > 64 * per_cu) {
        if (e3m2 || K < 2048) return true;
        return n <= 320 * per_cu && !(n > 192 * per_cu && n <= 224 * per_cu && K >= 3500);
    }
    if (K % 16 == 0) {
        if (e3m2) return K >= 8192 || (fp32 ? K >= 3072 && full : K >= 3072 ? wide : K >= 2048 && full);
        if (int8 && n > 144 * per_cu && K > 3328 && K < 7680) return false;
        if (!wide) return K >= (fp32 && !int8 ? 6144 : 4096);
        if (fp32 && !int8) return K >= 2560 || (K >= 1536 ? full : n > 32 * per_cu);
        return full || K >= 1536;
    }
    if (!wide || K < 2000 || e3m2) return false;
    if (int8) {
        if (!dynamic || fp32) return !dynamic || K >= 3200 || full;
        const bool many = n > 112 * per_cu ? K >= 2400 : n > 54 * per_cu && n <= 64 * per_cu && K >= 4000 && K < 7400;
        return !many && (K >= 3200 || full);
    }
    if (!dynamic) return !fp32 || K >= 3500 || (K >= 2300 ? full : n > 40 * per_cu);
    if (fp32) return K >= 4000 && full;
    return K >= 3000 ? full || K >= 7400 : n > 32 * per_cu;
}

// false: the layer is not for this kernel.  It takes up to 16 rows of up to 512 whole groups of 16 channels whose quantized form
// fits LDS, where a thread's registers hold its rows (2-byte types: 16 rows up to K = 4096, 8 up to 8192).
//   - E3M2 up to M K = 16384: its values are packed for LDS row by row.  Us, separate / this: 4 x 4096 x 4096 11.5 / 10.0, 8 x
//     2048 x 4096 10.6 / 9.6, but 8 x 4096 x 256 10.8 / 11.2, 16 x 4096 x 4096 12.6 / 15.5, 8 x 5120 x 4096 13.5 / 16.1.  (Within the line, over 2
//     to 16 rows of 512 to 8192 by 256 to 11008 columns, dynamic, 6 to 32 % less than the separate kernels everywhere.)
//   - One row: few_takes_one_row.
inline bool few_plan(int M, int N, int K, int ld, int Kpad, int bits, int x_bytes, bool dynamic, int cus, FewPlan* plan)
{
    const int NH = K >> 4;
    const bool e3m2 = bits != 8 && bits != 4;
    if (M < 1 || M > FEW_ROWS || NH < 1 || NH > 64 * FEW_PREP_WAVES || Kpad < NH * 16 || Kpad >= 65536) return false;
    if (e3m2 && (long long)M * K > 16384) return false;
    if (M == 1 && !few_takes_one_row(N, K, bits, x_bytes, dynamic, cus)) return false;
    const int head = (NH + 63) / 64 * 64, slots = std::max(1, std::min(64 * FEW_PREP_WAVES / head, M));
    if ((M + slots - 1) / slots > few_rows_held(x_bytes)) return false;
    // as few rounds as 64 columns per workgroup allow, all of the same width
    const long long rounds = ((long long)N + 64LL * cus - 1) / (64LL * cus), share = (N + cus * rounds - 1) / (cus * rounds);
    const int cols = (int)std::max(16LL, (share + 3) / 4 * 4);
    const int rowbytes = bits == 8 ? Kpad : bits == 4 ? Kpad / 2 : Kpad / 4 * 3, steps = e3m2 ? Kpad / 128 : (rowbytes + 127) / 128;
    const int prep = head * slots / 64, stream = std::min(FEW_WAVES - prep, std::max(steps, 4));
    plan->fn = (cols + 15) / 16;
    const size_t kq = (size_t)NH * 16, nt = (size_t)Kpad / 16 - NH, rows = (size_t)M;
    plan->lds = FEW_LDS_FIXED + kq + FEW_PAD + rows * (e3m2 ? (size_t)rowbytes : few_row(rowbytes)) + (bits == 8 ? 0 : rows * (kq + FEW_PAD)) +
                32 * nt + (nt + 15) / 16 * 16 + 2 * (((size_t)Kpad / 16 + 7) / 8 * 8) + (size_t)stream * plan->fn * 1024;
    if (plan->lds > FEW_LDS) return false;
    // Weight rows of 4, 8 or 16 KiB: workgroups that walk them in step meet on the same memory channels, so each begins at another step (5 w
    // modulo their number, a power of two).  INT8, us, all at step 0 / so: 1 x 8192 x 8192 20.1 / 14.3, x 16384 31.6 / 26.7, x 24576 39.9 / 37.4,
    // x 6144 12.3 / 12.4; nibbles 1 x 8192 x 24576 23.7 / 20.8.  On rows of 6 and 7 KiB it gave nothing or cost 1-2 %.  E3M2 rows are 96 bytes apart.
    const bool aliased = !e3m2 && rowbytes >= 4096 && (rowbytes & (rowbytes - 1)) == 0;
    plan->sh = FewShape{M, K, ld, Kpad, N, prep, slots, cols, aliased ? steps - 1 : -1};
    plan->threads = (prep + stream) * 64;
    plan->grid = (unsigned)std::min<long long>(((long long)N + cols - 1) / cols, cus);
    return true;
}

// Grid of the absmax pass: `blocks` workgroups side by side cover the columns (64 * vec of them each), `strips` of
// rows_per_strip rows each cover the rows.  Every workgroup leaves one candidate.
struct AbsmaxGrid {
    int blocks, strips, rows_per_strip;
    int candidates() const { return blocks * strips; }
};

// Candidates that the workspace has room for: one per column block however wide the matrix, and enough strips of a narrow one.
constexpr int MAX_CANDIDATES = 1024;
inline long long candidate_capacity(long long K) { return std::max<long long>(MAX_CANDIDATES, (K + 63) / 64 * 64); }

// A workgroup's four waves read 32 rows per round, eight loads in flight each; two to four workgroups per CU (at most 1024
// candidates), strips of whole rounds.  Of the three counts, and one round more, the one whose fullest CU has the fewest rounds, the
// lowest on a tie.  Strips of an even number of rounds count for a quarter more where rows are whole 4 KiB, or where they fill a
// stride of whole 8 KiB up to its padding: they start on the same memory channels.  (Of a wider stride taken in part that is not so:
// fp32 1000 x 7000 of 8192 6.0 us, with odd rounds 7.5; nor does it pay below 2048 rows, whole call, 1000 x 8184 of 8192 23.4, 24.2.)
// Whole quantizer call, fp32, us: 8192 x 4096 with strips of 128 rows 63.4, 256 63.6, 288 58.1, 342 59.1; 4096 x 8192 256 rows 63.0,
// 288 60.5; bf16 8192 x 4096 256 rows 37.8, 288 34.9; maxima alone, bf16 4096 x 4088 of 4096 64 rows 8.2, 32 6.8.  One workgroup per
// CU loses elsewhere: fp32 3000 x 5001 42.4, with two 35.7; weights 5120 x 20480 96.6, 92.4.
constexpr int ABSMAX_ROUND = 32;
inline AbsmaxGrid absmax_grid(long long M, long long K, long long ld, int vec, long long cus = 256)
{
    const long long bx = (K + 64 * vec - 1) / (64 * vec);
    const long long most = (M + ABSMAX_ROUND - 1) / ABSMAX_ROUND, row = K * (16 / vec), pitch = ld * (16 / vec);
    const bool aliased = row % 4096 == 0 || (M >= 2048 && pitch % 8192 == 0 && row > pitch - pitch / 16);
    long long rows = M, best = -1;
    for (int per_cu = 2; per_cu <= 4; ++per_cu) {
        const long long s = std::max(1LL, std::min(most, std::min<long long>(MAX_CANDIDATES, per_cu * cus) / bx));
        const long long least = ((M + s - 1) / s + ABSMAX_ROUND - 1) / ABSMAX_ROUND;
        for (long long rounds = least; rounds <= least + 1 && rounds <= most; ++rounds) {
            const long long wgs = bx * ((most + rounds - 1) / rounds);
            long long cost = 10 * ((wgs + cus - 1) / cus) * rounds;
            if (rounds % 2 == 0 && aliased) cost += cost / 4;
            if (best < 0 || cost < best) {
                best = cost;
                rows = rounds * ABSMAX_ROUND;
            }
        }
    }
    rows = std::min(rows, M);
    return AbsmaxGrid{(int)bx, (int)((M + rows - 1) / rows), (int)rows};
}

}  // namespace fq
