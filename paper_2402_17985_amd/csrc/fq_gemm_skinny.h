// The 16-row MFMA step that the weight-streaming kernels share: a lane's operands, where they lie in a row, and the product
// (GPU code only; everything has internal linkage).
#pragma once
#include "fq_gemm_common.h"

namespace fq {
namespace {

template <int MODE> struct Operand {           // a lane's share of a k-step of one row
    v4i a, b;                                  // 16-byte chunks c and c + 4 of the 128 bytes (c = lane / 16)
};
template <> struct Operand<MODE_F6> {
    v4i a;                                     // X and Y piece of the lane's 32-code unit
    v2i b;
};
template <int MODE> struct Sum { typedef v4i type; };
template <> struct Sum<MODE_F6> { typedef v4f type; };

template <int MODE>
__device__ __forceinline__ void multiply(const Operand<MODE>& w, const Operand<MODE>& x, typename Sum<MODE>::type& acc)
{
    if constexpr (MODE == MODE_I8) {
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(w.a, x.a, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(w.b, x.b, acc, 0, 0, 0);
    } else if constexpr (MODE == MODE_I4) {
        constexpr int HI = (int)0xf0f0f0f0;
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8((w.a << 4) & HI, (x.a << 4) & HI, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(w.a & HI, x.a & HI, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8((w.b << 4) & HI, (x.b << 4) & HI, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(w.b & HI, x.b & HI, acc, 0, 0, 0);
    } else {
        const v8i wo = {w.a[0], w.a[1], w.a[2], w.a[3], w.b[0], w.b[1], 0, 0};
        const v8i xo = {x.a[0], x.a[1], x.a[2], x.a[3], x.b[0], x.b[1], 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wo, xo, acc, 3, 3, 0, 127, 0, 127);   // 3 = E3M2, unit scales
    }
}

// Byte offsets of a lane's pieces of a row in k-step 0, and the distance between k-steps.
template <int MODE> struct RowPieces {
    uint32_t a, b;
    __device__ __forceinline__ void set(int row, int c, uint32_t rowbytes)
    {
        if constexpr (MODE == MODE_F6) {
            // 48-byte group c / 2 of the row's 96 bytes; unit c % 2 of it is stored X Y or, mirrored by row bit 4, Y X
            const uint32_t grp = (uint32_t)row * 96u + 48u * (c >> 1);
            const bool mirrored = (((c & 1) ^ (row >> 4)) & 1) != 0;
            a = grp + (mirrored ? 32u : 0u);
            b = grp + (mirrored ? 24u : 16u);
        } else {
            a = (uint32_t)row * rowbytes + 16u * c;
            b = a + 64u;
        }
    }
};

}  // namespace
}  // namespace fq
