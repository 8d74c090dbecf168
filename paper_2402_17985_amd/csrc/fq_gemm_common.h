// What the GEMM translation units share: vector types, operand modes, the clock probe, the direct global -> LDS copy, the
// workgroup -> tile order and the epilogue (GPU code only; everything has internal linkage).
#pragma once
#include <type_traits>

#include "fq_internal.h"

namespace fq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));

enum { MODE_I8 = 0, MODE_I4 = 1, MODE_BF16 = 2, MODE_F6 = 3 };   // F6: 4-bit values stored as 6-bit E3M2 codes

// Clock probe (measurement hook): with a non-null counter pair, the first wave of the workgroup adds the shader-clock
// and the constant-rate ticks between construction and finish().  Both reads are scalar instructions.
struct ClockProbe {
    unsigned long long t0, r0;
    __device__ __forceinline__ explicit ClockProbe(const unsigned long long* ticks)
    {
        t0 = r0 = 0;
        if (ticks) {
            t0 = __builtin_amdgcn_s_memtime();
            r0 = __builtin_amdgcn_s_memrealtime();
        }
    }
    __device__ __forceinline__ void finish(unsigned long long* ticks) const
    {
        if (ticks) {
            const unsigned long long t1 = __builtin_amdgcn_s_memtime(), r1 = __builtin_amdgcn_s_memrealtime();
            if (threadIdx.x == 0) {
                atomicAdd(&ticks[0], t1 - t0);
                atomicAdd(&ticks[1], r1 - r0);
            }
        }
    }
};

template <int YDT> struct OutVec;
template <> struct OutVec<FQ_I32> { typedef int type __attribute__((ext_vector_type(4))); };
template <> struct OutVec<FQ_F32> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct OutVec<FQ_F16> { typedef _Float16 type __attribute__((ext_vector_type(4))); };
template <> struct OutVec<FQ_BF16> { typedef __bf16 type __attribute__((ext_vector_type(4))); };

// fp32 -> half of a value that has already been rounded to fp32.  The empty asm keeps the compiler from folding
// the preceding fp32 multiply (or bias add) into a mixed-precision instruction that rounds the exact product only
// once, straight to half: the interface defines the output as the fp32 result rounded again to the output type.
__device__ __forceinline__ _Float16 half_of_rounded_fp32(float f)
{
    asm("" : "+v"(f));
    return (_Float16)f;
}

// One output element: the accumulator scaled by s_x * s_w, plus (optionally) the column's bias, both
// in fp32 as two separately rounded operations, then rounded to the output type.
template <int MODE, int YDT, typename S>
__device__ __forceinline__ auto convert_value(S acc, float scale, bool has_bias = false, float b = 0.0f)
{
    if constexpr (MODE == MODE_BF16) {
        return (__bf16)acc;
    } else if constexpr (MODE == MODE_F6) {
        // the fp32 accumulator holds the integer result exactly (|acc| < 2^24): it is fl32(acc) already
        if constexpr (YDT == FQ_I32) {
            return (int)acc;
        } else {
            float f = acc * scale;
            if (has_bias) f += b;
            if constexpr (YDT == FQ_F32) return f;
            else if constexpr (YDT == FQ_BF16) return (__bf16)f;
            else return half_of_rounded_fp32(f);
        }
    } else {
        int v = acc;
        if (MODE == MODE_I4) v >>= 8;
        if constexpr (YDT == FQ_I32) {
            return v;
        } else {
            float f = (float)v * scale;
            if (has_bias) f += b;
            if constexpr (YDT == FQ_F32) return f;
            else if constexpr (YDT == FQ_BF16) return (__bf16)f;
            else return half_of_rounded_fp32(f);
        }
    }
}

// The four bias values of the columns col .. col + 3 (col a multiple of 4; zeros beyond column N).
__device__ __forceinline__ v4f bias4(const float* __restrict__ bias, int col, int N)
{
    v4f b = {0.0f, 0.0f, 0.0f, 0.0f};
    if (col + 3 < N) {
        b = *reinterpret_cast<const v4f*>(bias + col);
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (col + e < N) b[e] = bias[col + e];
    }
    return b;
}

// The product of the two per-tensor scales, read at the start of a tile so that the epilogue does not wait for two
// scalar loads (raw accumulator output passes null pointers: no scale).
template <int MODE> __device__ __forceinline__ float tile_scale(const float* __restrict__ s_x, const float* __restrict__ s_w)
{
    if constexpr (MODE == MODE_BF16) return 1.0f;
    else return (s_x && s_w) ? (*s_x) * (*s_w) : 1.0f;
}

#define FQ_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define FQ_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

// Direct global -> LDS copy of 16 bytes per lane (global_load_lds_dwordx4): lane i of the wave
// writes LDS bytes [lds_base + 16 i, +16).  lds_base is wave-uniform and travels in M0.
// Written as inline assembly so that the outstanding-copy count (vmcnt) is managed by the kernel
// itself: several stages stay in flight across barriers, which the compiler's conservative
// "wait for every LDS DMA before any LDS read" rule would forbid.
__device__ __forceinline__ void dma16(const uint8_t* uniform_base, uint32_t lane_offset, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                 :
                 : "s"(uniform_base), "v"(lane_offset), "s"(lds_base)
                 : "memory");
}
__device__ __forceinline__ void dma16_addr(const uint8_t* lane_address, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(lane_address), "s"(lds_base)
                 : "memory");
}

// 16 zero bytes in device memory: the source of DMA lanes that fall beyond the end of a row.
__device__ const int g_zero_chunk[4] = {0, 0, 0, 0};

template <int MODE> struct Acc { typedef v16i type; };
template <> struct Acc<MODE_BF16> { typedef v16f type; };
template <> struct Acc<MODE_F6> { typedef v16f type; };      // exact integers below 2^24 held in fp32

__device__ __forceinline__ void tile_of_logical(int logical, int tiles_m, int tiles_n, int& tile_m, int& tile_n);

// Workgroup id -> output tile.  Ids are dealt round-robin to the 8 XCDs; each XCD gets a contiguous
// band of the logical tile sequence, which walks GROUP_M tile-rows at a time.
__device__ __forceinline__ void tile_of_workgroup(int wg, int nwg, int tiles_m, int tiles_n, int& tile_m,
                                                  int& tile_n)
{
    const int q = nwg >> 3, rem = nwg & 7;
    const int xcd = wg & 7, idx = wg >> 3;
    const int logical = (xcd < rem) ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
    tile_of_logical(logical, tiles_m, tiles_n, tile_m, tile_n);
}
__device__ __forceinline__ void tile_of_logical(int logical, int tiles_m, int tiles_n, int& tile_m, int& tile_n)
{
    constexpr int GROUP_M = 8;     // 2, 4, 16, 32 measured 1-7 % slower on the 6-bit kernel
    const int group = GROUP_M * tiles_n;
    const int gidx = logical / group;
    const int first_m = gidx * GROUP_M;
    const int gsz = min(tiles_m - first_m, GROUP_M);
    const int in_group = logical - gidx * group;
    tile_m = first_m + in_group % gsz;
    tile_n = in_group / gsz;
}

// Batched launches: the grid's y dimension counts the problems, its x dimension their tiles.  Ids are dealt round-robin to
// the XCDs over the whole grid, so each XCD gets a contiguous band of (problem, tile) pairs: a problem's operands then pass
// through one L2, not through all eight.  Returns whether `id` is a logical tile of the problem already (tile_of_logical);
// otherwise it is a workgroup id within the problem (tile_of_workgroup).  With one tile per problem there is nothing to
// share.  (The sizes come as arguments: gridDim would be a load of its own before the first address, 0.12 us of a 3.4 us
// call.)
__device__ __forceinline__ bool place_of_workgroup(int tiles, int count, int& problem, int& id)
{
    problem = blockIdx.y;
    id = blockIdx.x;
    if (tiles == 1 || count == 1 || (unsigned long long)tiles * count >= (1ull << 31)) return false;
    const unsigned total = (unsigned)tiles * count, at = blockIdx.y * (unsigned)tiles + blockIdx.x;
    const unsigned q = total >> 3, rem = total & 7, xcd = at & 7, idx = at >> 3;
    const unsigned logical = (xcd < rem) ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
    problem = __builtin_amdgcn_readfirstlane((int)(logical / (unsigned)tiles));
    id = __builtin_amdgcn_readfirstlane((int)(logical - (unsigned)problem * tiles));
    return true;
}

// Epilogue of one wave.  The MFMAs are issued with the W fragment as the first operand and the X
// fragment as the second, so in the 32x32 accumulator block (i, j) lane l holds output row
// 32 i + l%32 and, in registers 4g..4g+3, the four consecutive output columns
// 32 j + 8 g + 4 (l/32) + 0..3: they are scaled, converted and written as one 8- or 16-byte store.
// One output element of a wave's accumulators.
template <int MODE, int YDT> __device__ __forceinline__ auto convert_out(typename Acc<MODE>::type const& acc, int r, float scale,
                                                                         bool has_bias = false, float b = 0.0f)
{
    return convert_value<MODE, YDT>(acc[r], scale, has_bias, b);
}

// The lane index as the epilogue sees it: an opaque copy, so that the per-lane addresses of the epilogue are computed
// after the main loop.  Derived from the plain lane index they are loop invariants the compiler computes at kernel
// start and keeps live across the main loop, where every register is taken: they were spilled, and their reloads
// (vector memory operations, waited for with vmcnt) had each tile's epilogue wait for everything in flight.
__device__ __forceinline__ int epilogue_lane()
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

template <int MODE, int YDT, int FM, int FN, bool hb = false, typename acc_t>
__device__ __forceinline__ void store_tile_as(acc_t (&acc)[FM][FN], int row0, int col0, int M, int N, float scale,
                                              void* __restrict__ Y, int ldy, bool fast,
                                              const float* __restrict__ bias = nullptr)
{
    typedef typename OutVec<YDT>::type vec_t;
    typedef decltype(convert_out<MODE, YDT>(acc[0][0], 0, scale)) elem_t;
    const int lane = epilogue_lane();
    const int frow = lane & 31, fhalf = lane >> 5;
    elem_t* Yt = static_cast<elem_t*>(Y);
    if (fast) {
        // whole wave tile inside the matrix, rows aligned for vector stores
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            elem_t* yrow = Yt + (size_t)(row0 + i * 32 + frow) * ldy + col0 + 4 * fhalf;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f b4 = hb ? bias4(bias, col0 + 4 * fhalf + j * 32 + 8 * g, N) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    vec_t v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = convert_out<MODE, YDT>(acc[i][j], 4 * g + e, scale, hb, b4[e]);
                    *reinterpret_cast<vec_t*>(yrow + j * 32 + 8 * g) = v;
                }
        }
    } else {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int row = row0 + i * 32 + frow;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int col = col0 + j * 32 + 8 * (r >> 2) + 4 * fhalf + (r & 3);
                    if (row < M && col < N)
                        Yt[(size_t)row * ldy + col] = convert_out<MODE, YDT>(acc[i][j], r, scale, hb, hb ? bias[col] : 0.0f);
                }
        }
    }
}

// 16 bytes of a row of 2- or 4-byte elements: the vector type of an unaligned store (global memory takes any alignment).
struct __attribute__((packed, aligned(2))) Bytes16 { v4i v; };

// A wave's tile goes out through a wave-private LDS staging area so that global memory sees row segments: the wave writes
// its accumulators as [row][column] (16-byte units XOR-swizzled with the row to spread banks), reads them back 16 bytes
// per lane, and stores 16 bytes per lane, 64/UNITS rows per instruction.  `stage` must hold CH*32 rows of FN*32
// elements.  Tiles that reach beyond the matrix drop what lies outside; rows may start at any element.  (Stored straight
// from the accumulator layout, a store instruction touches 32 rows: with an odd row length, element by element, an 8192
// x 4095 bf16 output took 75 us longer than an 8192 x 4096 one.)
template <int MODE, int YDT, int FM, int FN, bool hb, int CH, typename acc_t>
__device__ __forceinline__ void store_tile_via_lds(acc_t (&acc)[FM][FN], int row0, int col0, int M, int N, float scale,
                                                   void* __restrict__ Y, int ldy, uint8_t* stage,
                                                   const float* __restrict__ bias = nullptr)
{
    // CH = 32-row blocks staged at a time: `stage` holds CH*32 rows and is reused FM/CH times (the
    // LDS operations of one wave execute in order, so a chunk's reads precede the next chunk's writes)
    typedef typename OutVec<YDT>::type vec_t;
    constexpr int ES = sizeof(vec_t) / 4;                  // bytes per element
    constexpr int ROWB = FN * 32 * ES;                     // bytes per staged row
    constexpr int UNITS = ROWB / 16, PER = 16 / ES;        // 16-byte units per row, elements per unit
    constexpr int SW = (UNITS >= 8 ? 8 : UNITS) - 1;
    // the swizzle advances once per 256 bytes of staged rows, so that the 8- or 16-byte writes of 32 lanes (one
    // row each) spread over all 16-byte units of the 64 banks
    constexpr int SWS = (ROWB >= 256) ? 0 : (ROWB == 128 ? 1 : 2);
    constexpr int ROWS_PER_INSTR = 64 / UNITS;
    static_assert(UNITS <= 64 && (CH * 32) % ROWS_PER_INSTR == 0 && FM % CH == 0, "staging layout");
    const int lane = epilogue_lane();
    const int frow = lane & 31, fhalf = lane >> 5;
    uint8_t* Yb = static_cast<uint8_t*>(Y);
    const int mr = lane / UNITS, us = lane % UNITS;
    const bool whole_lines = row0 + FM * 32 <= M && col0 + FN * 32 <= N && (ldy * ES & 127) == 0 && (col0 * ES & 127) == 0 &&
                             (reinterpret_cast<uintptr_t>(Y) & 127) == 0;
#pragma unroll
    for (int c = 0; c < FM / CH; ++c) {
#pragma unroll
        for (int ic = 0; ic < CH; ++ic) {
            const int i = c * CH + ic;
            const int m = ic * 32 + frow;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f b4 = hb ? bias4(bias, col0 + 4 * fhalf + j * 32 + 8 * g, N) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    vec_t v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = convert_out<MODE, YDT>(acc[i][j], 4 * g + e, scale, hb, b4[e]);
                    const int u = ES == 2 ? g + 4 * j : 8 * j + 2 * g + fhalf;
                    *reinterpret_cast<vec_t*>(stage + m * ROWB + ((u ^ ((m >> SWS) & SW)) << 4) + (ES == 2 ? 8 * fhalf : 0)) = v;
                }
        }
        // The output is written once and not read by this kernel: a streaming store keeps it from
        // displacing the operand panels in L2 -- but only when the 128-byte row segments are whole cache
        // lines; partial-line streaming stores are several times slower than ordinary ones.  (Two loops
        // kept apart: merged, they become one ordinary store.)
        const int rbase = row0 + c * CH * 32;
        if (whole_lines) {
            uint8_t* ybase = Yb + ((size_t)rbase * ldy + col0) * ES;
            asm volatile("; streaming stores begin");    // the markers keep the two arms from being merged
#pragma unroll
            for (int t = 0; t < CH * 32 / ROWS_PER_INSTR; ++t) {
                const int m = t * ROWS_PER_INSTR + mr;
                const int u = us ^ ((m >> SWS) & SW);
                const v4i d = *reinterpret_cast<const v4i*>(stage + m * ROWB + (us << 4));
                __builtin_nontemporal_store(d, reinterpret_cast<v4i*>(ybase + (size_t)m * ldy * ES + (u << 4)));
            }
            asm volatile("; streaming stores end");
        } else {
            typedef decltype(convert_out<MODE, YDT>(acc[0][0], 0, scale)) elem_t;
#pragma unroll 4
            for (int t = 0; t < CH * 32 / ROWS_PER_INSTR; ++t) {
                const int m = t * ROWS_PER_INSTR + mr;
                const int row = rbase + m, col = col0 + (us ^ ((m >> SWS) & SW)) * PER;
                const uint8_t* sp = stage + m * ROWB + (us << 4);
                if (row < M && col < N) {
                    elem_t* y = reinterpret_cast<elem_t*>(Yb) + (size_t)row * ldy + col;
                    if (col + PER <= N) {
                        reinterpret_cast<Bytes16*>(y)->v = *reinterpret_cast<const v4i*>(sp);
                    } else {
                        for (int e = 0; col + e < N; ++e) y[e] = reinterpret_cast<const elem_t*>(sp)[e];
                    }
                }
            }
        }
    }
}

// ONLY = an output type: the caller guarantees y_dtype == ONLY and no bias, and only that path is compiled (a kernel
// that carries every output type keeps more live state across its main loop and spills in the epilogue).
constexpr int ANY_OUTPUT = -1;
template <int MODE, int FM, int FN, int CH = FM, int ONLY = ANY_OUTPUT, typename acc_t>
__device__ __forceinline__ void store_tile(acc_t (&acc)[FM][FN], int row0, int col0, int M, int N, float scale,
                                           void* __restrict__ Y, int y_dtype, int ldy, uint8_t* stage = nullptr,
                                           const float* __restrict__ bias = nullptr)
{
    // 2-byte outputs are staged CH blocks at a time, 4-byte ones half as many; without room for that (or without a
    // staging area) they leave straight from the accumulator layout
    auto put = [&](auto ydt, auto has_bias) {
        constexpr int YDT = decltype(ydt)::value;
        constexpr bool HB = decltype(has_bias)::value;
        constexpr int ES = sizeof(typename OutVec<YDT>::type) / 4, CHS = ES == 2 ? CH : CH / 2;
        const float sc = (MODE == MODE_BF16 || YDT == FQ_I32) ? 1.0f : scale;
        if constexpr (CHS >= 1) {
            if (stage) {
                store_tile_via_lds<MODE, YDT, FM, FN, HB, CHS>(acc, row0, col0, M, N, sc, Y, ldy, stage, bias);
                return;
            }
        }
        const bool fast = row0 + FM * 32 <= M && col0 + FN * 32 <= N && (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
        store_tile_as<MODE, YDT, FM, FN, HB>(acc, row0, col0, M, N, sc, Y, ldy, fast, bias);
    };
    typedef std::integral_constant<int, FQ_BF16> bf16_t;
    typedef std::integral_constant<int, FQ_F16> f16_t;
    typedef std::integral_constant<int, FQ_F32> f32_t;
    typedef std::integral_constant<int, FQ_I32> i32_t;
    if constexpr (MODE == MODE_BF16) {
        put(bf16_t{}, std::false_type{});
    } else if constexpr (ONLY != ANY_OUTPUT) {
        put(std::integral_constant<int, ONLY>{}, std::false_type{});
    } else if (y_dtype == FQ_I32) {
        put(i32_t{}, std::false_type{});
    } else if (bias) {
        // the biased epilogue is a separate instantiation so that the plain one carries none of it
        if (y_dtype == FQ_BF16) put(bf16_t{}, std::true_type{});
        else if (y_dtype == FQ_F16) put(f16_t{}, std::true_type{});
        else put(f32_t{}, std::true_type{});
    } else {
        if (y_dtype == FQ_BF16) put(bf16_t{}, std::false_type{});
        else if (y_dtype == FQ_F16) put(f16_t{}, std::false_type{});
        else put(f32_t{}, std::false_type{});
    }
}

// Four consecutive output elements of one row from their summed accumulators (vec: rows allow a vector store).
template <int MODE, int YDT, typename S>
__device__ __forceinline__ void store4_as(S const& acc, int row, int col, int N, float scale, void* __restrict__ Y, int ldy,
                                          const float* __restrict__ bias, bool vec)
{
    typedef typename OutVec<YDT>::type vec_t;
    typedef decltype(convert_value<MODE, YDT>(acc[0], scale)) elem_t;
    elem_t* y = static_cast<elem_t*>(Y) + (size_t)row * ldy + col;
    elem_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = convert_value<MODE, YDT>(acc[e], scale, bias != nullptr, bias && col + e < N ? bias[col + e] : 0.0f);
    if (vec && col + 3 < N) {
        *reinterpret_cast<vec_t*>(y) = vec_t{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (col + e < N) y[e] = v[e];
    }
}
template <int MODE, typename S>
__device__ __forceinline__ void store4(S const& acc, int row, int col, int N, float scale, void* __restrict__ Y, int y_dtype,
                                       int ldy, const float* __restrict__ bias, bool vec)
{
    if (y_dtype == FQ_BF16) store4_as<MODE, FQ_BF16>(acc, row, col, N, scale, Y, ldy, bias, vec);
    else if (y_dtype == FQ_F16) store4_as<MODE, FQ_F16>(acc, row, col, N, scale, Y, ldy, bias, vec);
    else if (y_dtype == FQ_F32) store4_as<MODE, FQ_F32>(acc, row, col, N, scale, Y, ldy, bias, vec);
    else store4_as<MODE, FQ_I32>(acc, row, col, N, 1.0f, Y, ldy, nullptr, vec);
}

}  // namespace
}  // namespace fq
