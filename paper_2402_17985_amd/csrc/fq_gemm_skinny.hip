// Integer GEMM for few rows of X (decoding, short prompts): the weights are streamed once, straight into registers.
//
// arXiv 2402.17985 Sec. 5.1 (the quantized linear layer); the same product, storage and epilogue as the tiled kernels of
// fq_gemm.hip.  With at most 16 rows the product reads N * Kpad weight bytes for at most 16 multiply-adds each: it is bound
// by that stream, and by latency where the stream is short.  The tiled kernels lose there because a 128-column tile per
// workgroup leaves most CUs idle and two LDS stages keep too few bytes in flight (0.5-0.6 us per 128-byte stage at any M).
// One row, us before / now (rate of the weight stream): INT8 6400 x 15360 45.8 / 19.8 (5.0 TB/s), 12544 x 4096 52.0 / 9.9 (5.2
// TB/s), 8960 x 24576 86.7 / 37.7 (5.8 TB/s); nibbles 8960 x 24576 39.1 / 20.8; E3M2 51.4 / 30.1.
//
// A workgroup owns 16 FN columns and all rows; its NW waves split the reduction, wave w taking the 128-byte k-steps
// w, w + NW, ...  Nothing is shared between waves until the end, so the main loop has no barrier and no LDS: a lane loads
// its MFMA operands from global memory (16 rows x 64 contiguous bytes per instruction; X comes out of L2), D steps ahead.
// The partial accumulators meet in LDS; integer sums (and E3M2's fp32 sums of integers below 2^24) are exact in any
// order, so results equal the tiled kernels' bit for bit.
//   INT8  v_mfma_i32_16x16x64_i8          two per step and fragment pair
//   INT4  the same on the low and the high nibbles moved to the top of a byte (the accumulator holds 256 * sum)
//   E3M2  v_mfma_scale_f32_16x16x128_f8f6f4  one per step: a step is a block of 128 codes, 96 bytes per row
// The weights are the first MFMA operand: a lane's four accumulators are four consecutive columns of one row.
#include "fq_gemm_common.h"
#include "fq_gemm_skinny.h"
#include "fq_internal.h"

namespace fq {
namespace {

template <int MODE, int FN, int NW, int D>
__global__ __launch_bounds__(NW * 64) void gemm_skinny_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B,
                                                              int M, int N, uint32_t rowbytes, const float* __restrict__ s_x,
                                                              const float* __restrict__ s_w, void* __restrict__ Y, int y_dtype,
                                                              int ldy, Batch bt)
{
    typedef typename Sum<MODE>::type sum_t;
    typedef Operand<MODE> op_t;
    __shared__ sum_t part[NW][FN][64];
    const ClockProbe probe(bt.ticks);
    A += (size_t)blockIdx.y * bt.stride_a;
    B += (size_t)blockIdx.y * bt.stride_b;
    Y = static_cast<uint8_t*>(Y) + (size_t)blockIdx.y * bt.stride_y;
    const int lane = threadIdx.x & 63, r = lane & 15, c = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * (16 * FN);
    const float scale = tile_scale<MODE>(s_x, s_w);

    // rows beyond the matrices re-read the last one; what they give is never stored
    RowPieces<MODE> pw[FN], px;
#pragma unroll
    for (int j = 0; j < FN; ++j) pw[j].set(min(n0 + 16 * j + r, N - 1), c, rowbytes);
    px.set(min(r, M - 1), c, rowbytes);
    constexpr uint32_t STEP_BYTES = (MODE == MODE_F6) ? 96 : 128;
    const uint32_t stride_w = (MODE == MODE_F6) ? 96u * N : 128u, stride_x = (MODE == MODE_F6) ? 96u * M : 128u;
    const int steps = (int)((rowbytes + STEP_BYTES - 1) / STEP_BYTES);
    const int mine = __builtin_amdgcn_readfirstlane((steps - wave + NW - 1) / NW);   // this wave's steps: wave, wave + NW, ...

    op_t w[D][FN], x[D];
    auto load = [&](int d, int t) {
        const uint32_t s = (uint32_t)(wave + t * NW);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            w[d][j].a = *reinterpret_cast<const decltype(op_t::a)*>(B + (pw[j].a + s * stride_w));
            w[d][j].b = *reinterpret_cast<const decltype(op_t::b)*>(B + (pw[j].b + s * stride_w));
        }
        x[d].a = *reinterpret_cast<const decltype(op_t::a)*>(A + (px.a + s * stride_x));
        x[d].b = *reinterpret_cast<const decltype(op_t::b)*>(A + (px.b + s * stride_x));
    };
    // the row's last step may be partial: chunks beyond its end count as zeros (one operand of each product suffices)
    auto load_last = [&](int d, int t) {
        if constexpr (MODE == MODE_F6) {
            load(d, t);
        } else {
            const uint32_t s = (uint32_t)(wave + t * NW), at = s * 128u + 16u * c;
            const bool in_a = at < rowbytes, in_b = at + 64u < rowbytes;
            const v4i zero = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                w[d][j].a = zero;
                w[d][j].b = zero;
                if (in_a) w[d][j].a = *reinterpret_cast<const v4i*>(B + (pw[j].a + s * 128u));
                if (in_b) w[d][j].b = *reinterpret_cast<const v4i*>(B + (pw[j].b + s * 128u));
            }
            x[d].a = zero;
            x[d].b = zero;
            if (in_a) x[d].a = *reinterpret_cast<const v4i*>(A + (px.a + s * 128u));
            if (in_b) x[d].b = *reinterpret_cast<const v4i*>(A + (px.b + s * 128u));
        }
    };
    sum_t acc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[j] = sum_t{0, 0, 0, 0};
    auto compute = [&](int d) {
#pragma unroll
        for (int j = 0; j < FN; ++j) multiply<MODE>(w[d][j], x[d], acc[j]);
    };

    // Rounds of D steps without a branch while all of the next round's steps lie before this wave's last one; the rest
    // (at most 2 D steps) with a check per step.  The checks are made on scalars (readfirstlane): the MFMA ignores the
    // execution mask, so a condition that the compiler took for a per-lane one would not keep it from running.
    int t = 0;
    if (mine > D) {
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, d);
        for (; t + 2 * D < mine; t += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                compute(d);
                load(d, t + D + d);
            }
        }
        // steps t .. t + D - 1 are in registers, and more are left
        const int left = __builtin_amdgcn_readfirstlane(mine - t - D);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            compute(d);
            if (d < left) load_last(d, t + D + d);
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < left) compute(d);
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < mine) load_last(d, d);
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < mine) compute(d);
    }

    // ---- the waves' partial sums ----
#pragma unroll
    for (int j = 0; j < FN; ++j) part[wave][j][lane] = acc[j];
    __syncthreads();
    const bool vec = (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
    for (int p = threadIdx.x; p < FN * 64; p += NW * 64) {
        const int f = p >> 6, l = p & 63;
        sum_t s = part[0][f][l];
#pragma unroll
        for (int v = 1; v < NW; ++v) s += part[v][f][l];
        const int row = l & 15, col = n0 + 16 * f + 4 * (l >> 4);
        if (row < M && col < N) {
            store4<MODE>(s, row, col, N, scale, Y, y_dtype, ldy, bt.bias, vec);
        }
    }
    probe.finish(bt.ticks);
}

template <int MODE, int FN, int NW, int D>
int launch(const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w, void* Y, int y_dtype,
           int ldy, Batch bt, hipStream_t stream)
{
    const dim3 grid((unsigned)((N + 16 * FN - 1) / (16 * FN)), (unsigned)bt.count);
    gemm_skinny_kernel<MODE, FN, NW, D><<<grid, NW * 64, 0, stream>>>(
        static_cast<const uint8_t*>(A), static_cast<const uint8_t*>(B), M, N, (uint32_t)rowbytes, s_x, s_w, Y, y_dtype, ldy, bt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "GEMM launch failed: %s", hipGetErrorString(e));
    return FQ_OK;
}

template <int MODE>
int launch_mode(const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w, void* Y,
                int y_dtype, int ldy, Batch bt, hipStream_t stream)
{
    // Column fragments per workgroup: X is read once per workgroup, so wider is less traffic from L2, but the workgroups
    // should still number about the CUs: the smallest FN that makes them at most those.  Nibbles, 16 rows, us at FN = 1 / 2 / 4
    // on 256 CUs: 4608 x 11008 8.8 / 9.0 / 8.3, 6400 x 15360 13.6 / 11.3 / 10.6.  With a row or few (X is cached) FN = 1 is best
    // throughout (8960 x 24576 20.4 / 20.6 / 24.4); INT8 comes with at most 4 rows.
    if constexpr (MODE != MODE_I8) {
        const long long cus = compute_units();
        if (M > 4 && (N + 15) / 16 > cus) {
            if ((N + 31) / 32 <= cus) return launch<MODE, 2, 8, 2>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
            return launch<MODE, 4, 4, 2>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
        }
    }
    return launch<MODE, 1, 8, 2>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
}

}  // namespace

int launch_gemm_skinny(int bits, const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w,
                       void* Y, int y_dtype, int ldy, Batch bt, hipStream_t stream)
{
    if (bits == 8) return launch_mode<MODE_I8>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
    if (bits == FQ_BITS_I4_E3M2) return launch_mode<MODE_F6>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
    return launch_mode<MODE_I4>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
}

}  // namespace fq
