// What the quantizing translation units share: element types, the map loads, the quantizer of 16 elements and the packing of
// its values (GPU code only; everything has internal linkage).
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

// Bytes of the result: those of a (selector 4..7) or b (0..3), 0x0c gives 0.
__device__ __forceinline__ uint32_t bytes_of(uint32_t a, uint32_t b, uint32_t sel) { return __builtin_amdgcn_perm(a, b, sel); }

// Four quantized values in [-8, 7], one per byte, to their 6-bit E3M2 codes (sign, 3 exponent bits with bias 3, 2 mantissa
// bits): byte tables for the values 0..7 and -8..-1, looked up by the low three bits, chosen by the sign.
__device__ __forceinline__ uint32_t e3m2_codes(uint32_t q)
{
    const uint32_t sel = q & 0x07070707u, neg = (q >> 3) & 0x01010101u, mask = (neg << 8) - neg;
    const uint32_t pos = bytes_of(0x17161514u, 0x12100c00u, sel), low = bytes_of(0x2c303234u, 0x35363738u, sel);
    return (low & mask) | (pos & ~mask);
}
// Four codes, one per byte, as 24 bits (code i in bits 6 i .. 6 i + 5)
__device__ __forceinline__ uint32_t e3m2_stream(uint32_t c)
{
    const uint32_t y = (c & 0x003f003fu) | ((c >> 2) & 0x0fc00fc0u);
    return (y & 0xfffu) | ((y >> 4) & 0xfff000u);
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

// 16 elements times their multipliers, quantized, one per byte: the product rounded to fp32, clamped, rounded half to even.
// BITS = 8, 4, or 6 = the 4-bit quantizer with its values as 6-bit E3M2 codes.
// The kernels for many rows spend about as long on these instructions as on memory.  Adding 1.5 * 2^23 rounds to an integer as
// rintf does and leaves it, in two's complement, in the low bits of the sum, from where a byte permute collects it: 4 to 5
// instructions per element with the widening, where rintf, clamp, conversion and packing by shifts take 8 or 9.
// (quantized_bits: one element, its value in two's complement in the low bits)
template <int BITS> __device__ __forceinline__ uint32_t quantized_bits(float x, float m)
{
    constexpr int QB = (BITS == 6) ? 4 : BITS;
    constexpr float hi = (float)((1 << (QB - 1)) - 1), lo = -(float)(1 << (QB - 1)), ROUND = 12582912.0f;
    return __float_as_uint(__builtin_amdgcn_fmed3f(x * m, lo, hi) + ROUND);
}
// (quantize4: four elements, one per byte of a word)
template <int BITS> __device__ __forceinline__ uint32_t quantize4(const float* x, const float* m)
{
    uint32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = quantized_bits<BITS>(x[i], m[i]);
    const uint32_t w = bytes_of(bytes_of(t[3], t[2], 0x0c0c0400u), bytes_of(t[1], t[0], 0x0c0c0400u), 0x05040100u);
    return BITS == 6 ? e3m2_codes(w) : w;
}
template <int BITS> __device__ __forceinline__ v4u quantize16(const float (&x)[16], const float (&m)[16])
{
    v4u w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = quantize4<BITS>(x + 4 * i, m + 4 * i);
    return w;
}

// A gathered element, the largest finite value of its sign in place of an infinity (NaN counts as negative): the multiplier of
// a padding slot is 0, and 0 times what is not finite would be NaN, which clamps to qmin.  What other slots give is unchanged.
__device__ __forceinline__ float gathered(float x) { return __builtin_amdgcn_fmed3f(x, -3.402823466e38f, 3.402823466e38f); }

// 16 quantized values of a row (one per byte) stored as INT8 (16 bytes) or nibbles (8 bytes, even slot in the low nibble)
template <int BITS> __device__ __forceinline__ void store16(const v4u& q, uint8_t* o)
{
    static_assert(BITS == 8 || BITS == 4, "E3M2 codes go through store16_e3m2");
    if constexpr (BITS == 8) {
        *reinterpret_cast<v4u*>(o) = q;
    } else {
        uint32_t y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = (q[i] & 0x000f000fu) | ((q[i] >> 4) & 0x00f000f0u);     // bytes 0 and 2: two values each
        *reinterpret_cast<v2u*>(o) = v2u{bytes_of(y[1], y[0], 0x06040200u), bytes_of(y[3], y[2], 0x06040200u)};
    }
}

// The 16 codes of group g of a row of a matrix of `rows` rows in E3M2 storage, blocked along k: block t (codes 128 t .. 128 t +
// 127) holds 96 bytes of every row in turn.  A row's 96 bytes are two 48-byte groups of 64 codes; the 24-byte bit stream of each
// 32-code unit a is split into its first 16 bytes X_a and last 8 bytes Y_a, and the group is stored X_a Y_a Y_b X_b with
// (a, b) = (0, 1) in rows whose index has bit 4 clear and (1, 0) in the others (what the GEMM's LDS reads want).  16 codes
// are half a unit: stream bytes 0..11 (e = 0) or 12..23 (e = 1).
__device__ __forceinline__ void store16_e3m2(const v4u& q, uint8_t* out, size_t rows, int row, int g)
{
    const uint32_t s0 = e3m2_stream(q[0]), s1 = e3m2_stream(q[1]), s2 = e3m2_stream(q[2]), s3 = e3m2_stream(q[3]);
    const u3 v = {s0 | (s1 << 24), (s1 >> 8) | (s2 << 16), (s2 >> 16) | (s3 << 8)};
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

// 16 quantized values of group g of a row in the storage of BITS; dense rows start at out + row * orow_bytes.
template <int BITS>
__device__ __forceinline__ void store_group(const v4u& q, uint8_t* out, size_t orow_bytes, size_t rows, int row, int g)
{
    if constexpr (BITS == 6) store16_e3m2(q, out, rows, row, g);
    else store16<BITS>(q, out + (size_t)row * orow_bytes + (size_t)g * (BITS == 8 ? 16 : 8));
}

// 16 bytes gathered from a row in LDS by 16-bit indexes
__device__ __forceinline__ v4u gather16(const uint8_t* row, const v4u& t0, const v4u& t1)
{
    v4u q;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = i < 2 ? t0[2 * i] : t1[2 * i - 4], b = i < 2 ? t0[2 * i + 1] : t1[2 * i - 3];
        q[i] = (uint32_t)row[a & 0xffffu] | ((uint32_t)row[a >> 16] << 8) | ((uint32_t)row[b & 0xffffu] << 16) | ((uint32_t)row[b >> 16] << 24);
    }
    return q;
}

}  // namespace
}  // namespace fq
