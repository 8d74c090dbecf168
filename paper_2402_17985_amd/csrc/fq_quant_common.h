// What the quantizing translation units share: element types, the map loads, the quantizer of one element and the packing of
// 16 quantized values (GPU code only; everything has internal linkage).
#pragma once
#include "fq_internal.h"

namespace fq {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
// 12 bytes at 4-byte alignment (a 3-element vector type would claim 16)
struct __attribute__((aligned(4))) u3 { uint32_t a, b, c; };

// 6-bit E3M2 code (sign, 3 exponent bits with bias 3, 2 mantissa bits) of an integer-valued float r in
// [-8, 8]: the fp32 form of |r| already holds the exponent and, in its top mantissa bits, the two
// mantissa bits (exponent field 127 + e -> 3 + e: subtract 124 << 2 after the shift); 0 -> 0.
__device__ __forceinline__ int e3m2_code_of_float(float r)
{
    const uint32_t bits = __float_as_uint(r + 0.0f);                   // -0 -> +0
    const int mag = max((int)((bits & 0x7fffffffu) >> 21) - (124 << 2), 0);
    return mag | (int)((bits >> 26) & 0x20u);
}
// 16 codes as a 96-bit little-endian bit stream (code i in bits 6 i .. 6 i + 5)
__device__ __forceinline__ u3 pack16_e3m2(const int (&c)[16])
{
    uint32_t g[4];                                                     // four codes = 24 bits
#pragma unroll
    for (int i = 0; i < 4; ++i)
        g[i] = (uint32_t)c[4 * i] | ((uint32_t)c[4 * i + 1] << 6) | ((uint32_t)c[4 * i + 2] << 12) | ((uint32_t)c[4 * i + 3] << 18);
    return u3{g[0] | (g[1] << 24), (g[1] >> 8) | (g[2] << 16), (g[2] >> 16) | (g[3] << 8)};
}

template <int DT> struct Elem;
template <> struct Elem<FQ_F32> {
    typedef float type;
    static constexpr int VEC = 4;   // elements per 16 bytes
    static __device__ __forceinline__ float widen(float v) { return v; }
};
template <> struct Elem<FQ_F16> {
    typedef _Float16 type;
    static constexpr int VEC = 8;
    static __device__ __forceinline__ float widen(_Float16 v) { return (float)v; }
};
template <> struct Elem<FQ_BF16> {
    typedef uint16_t type;
    static constexpr int VEC = 8;
    static __device__ __forceinline__ float widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
};

// Widen one 16-byte vector of storage elements to floats.
template <int DT> __device__ __forceinline__ void widen16(const v4u raw, float* out);
template <> __device__ __forceinline__ void widen16<FQ_F32>(const v4u raw, float* out)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = __uint_as_float(raw[i]);
}
template <> __device__ __forceinline__ void widen16<FQ_BF16>(const v4u raw, float* out)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        out[2 * i] = __uint_as_float(raw[i] << 16);
        out[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
    }
}
template <> __device__ __forceinline__ void widen16<FQ_F16>(const v4u raw, float* out)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        union { uint32_t u; _Float16 h[2]; } cv;
        cv.u = raw[i];
        out[2 * i] = (float)cv.h[0];
        out[2 * i + 1] = (float)cv.h[1];
    }
}

// Workgroup barrier that orders LDS only: global loads and stores stay in flight across it.
__device__ __forceinline__ void strip_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Eight consecutive map entries.  The entry points ask for 16-byte alignment of src only: a 4-byte aligned vector type
// keeps the loads wide for any rep (global memory needs no more than dword alignment).
struct __attribute__((packed, aligned(4))) i4a4 { int v[4]; };
__device__ __forceinline__ void load8(const int32_t* p, int* out)
{
    const i4a4 a = *reinterpret_cast<const i4a4*>(p), b = *reinterpret_cast<const i4a4*>(p + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { out[i] = a.v[i]; out[4 + i] = b.v[i]; }
}

// BITS = 8, 4, or 6 = the 4-bit quantizer with its values stored as 6-bit E3M2 codes (k-blocked layout);
// for 6 the result is the code itself, which is also what the row strip keeps in LDS
template <int BITS> __device__ __forceinline__ int quant1(float x, float m)
{
    constexpr int QB = (BITS == 6) ? 4 : BITS;
    constexpr float hi = (float)((1 << (QB - 1)) - 1);
    constexpr float lo = -(float)(1 << (QB - 1));
    float r = rintf(x * m);                 // one fp32 multiply, then round-half-even
    r = fminf(fmaxf(r, lo), hi);
    if constexpr (BITS == 6) return e3m2_code_of_float(r);
    else return (int)r;
}

// A gathered element, the largest finite value of its sign in place of an infinity (NaN counts as negative): the multiplier of
// a padding slot is 0, and 0 times what is not finite would be NaN, which clamps to qmin.  What other slots give is unchanged.
__device__ __forceinline__ float gathered(float x) { return __builtin_amdgcn_fmed3f(x, -3.402823466e38f, 3.402823466e38f); }

// 16 quantized values of a row, packed: 16 bytes of INT8 or 8 bytes of nibbles (even slot in the low nibble)
template <int BITS> __device__ __forceinline__ void pack16(const int (&q)[16], uint8_t* o)
{
    static_assert(BITS == 8 || BITS == 4, "E3M2 codes go through store16_e3m2");
    if constexpr (BITS == 8) {
        v4u w;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = (uint32_t)(q[4 * i] & 0xff) | ((uint32_t)(q[4 * i + 1] & 0xff) << 8) |
                   ((uint32_t)(q[4 * i + 2] & 0xff) << 16) | ((uint32_t)(q[4 * i + 3] & 0xff) << 24);
        *reinterpret_cast<v4u*>(o) = w;
    } else {
        v2u w;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t acc = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc |= (uint32_t)(q[8 * i + j] & 0xf) << (4 * j);
            w[i] = acc;
        }
        *reinterpret_cast<v2u*>(o) = w;
    }
}

// The 16 codes of group g of a row of a matrix of `rows` rows in E3M2 storage, blocked along k: block t (codes 128 t .. 128 t +
// 127) holds 96 bytes of every row in turn.  A row's 96 bytes are two 48-byte groups of 64 codes; the 24-byte bit stream of each
// 32-code unit a is split into its first 16 bytes X_a and last 8 bytes Y_a, and the group is stored X_a Y_a Y_b X_b with
// (a, b) = (0, 1) in rows whose index has bit 4 clear and (1, 0) in the others (what the GEMM's LDS reads want).  16 codes
// are half a unit: stream bytes 0..11 (e = 0) or 12..23 (e = 1).
__device__ __forceinline__ void store16_e3m2(const int (&q)[16], uint8_t* out, size_t rows, int row, int g)
{
    const u3 v = pack16_e3m2(q);
    const int gi = g & 7, e = gi & 1;
    uint8_t* grp = out + ((size_t)(g >> 3) * rows + (size_t)row) * 96 + 48 * (gi >> 2);
    const bool mirrored = (((gi >> 1) ^ (row >> 4)) & 1) != 0;
    if (!mirrored) {
        *reinterpret_cast<u3*>(grp + 12 * e) = v;                     // X at 0, Y at 16: the plain stream
    } else if (e == 0) {
        *reinterpret_cast<u3*>(grp + 32) = v;                         // X at 32
    } else {
        *reinterpret_cast<uint32_t*>(grp + 44) = v.a;                 // the last 4 bytes of X
        *reinterpret_cast<v2u*>(grp + 24) = v2u{v.b, v.c};            // Y at 24
    }
}

}  // namespace
}  // namespace fq
