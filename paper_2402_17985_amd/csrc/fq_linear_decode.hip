// The whole layer for one row (decoding one sequence) in one kernel: every workgroup quantizes the row for itself, then
// streams its share of the weights.
//
// arXiv 2402.17985 Sec. 4.1 Eq. 3, Sec. 2.1 Eq. 1 (flatten and quantize) and Sec. 5.1 (the quantized linear layer); the
// values are those of the separate kernels, bit for bit.
// With one row the layer is the stream of its weights and two launches around it: a quantizer of one workgroup (6 us, all
// of it latency) and the product.  X and the map are a few tens of KiB and come out of L2, so each of up to 512
// workgroups (two per CU) forms the absmax (dynamic scale), the multipliers and the quantized row itself, into LDS,
// while the first weights are on their way; then it walks the 16-column tiles w, w + gridDim, ... as gemm_skinny_kernel
// does, with the X operand out of LDS.
// Us, this kernel / the two: INT8 20480 x 5120 39.3 / 43.5; E3M2 4096 x 4096 10.9 / 13.5; 512 x 512 11.2 / 13.3.  It serves one row where
// few_takes_one_row leaves it: short or narrow layers, INT8 layers of very many columns, ragged lengths of few columns.
#include <algorithm>
#include <atomic>

#include "fq_gemm_skinny.h"
#include "fq_internal.h"
#include "fq_quant_common.h"

namespace fq {
namespace {

constexpr int NW = 8, NTHR = NW * 64, D = 2, TABLE = 256;
// LDS: multipliers m(n), wave maxima, the waves' partial sums, then the quantized rows and slack for the last step's reads
constexpr int LDS_PART = (TABLE + NW) * 4, LDS_XQ = LDS_PART + NW * 64 * 16, LDS_SLACK = 128;

template <int DT, int MODE>
__global__ __launch_bounds__(NTHR, 4) void linear_decode_kernel(const void* __restrict__ Xv, int K,
                                                             const int32_t* __restrict__ src, const int32_t* __restrict__ rep,
                                                             int Kpad, const float* __restrict__ absmax_in,
                                                             const uint8_t* __restrict__ W, int N, const float* __restrict__ s_w,
                                                             const float* __restrict__ bias, void* __restrict__ Y, int y_dtype,
                                                             int ldy, unsigned long long* ticks)
{
    typedef typename Elem<DT>::type T;
    typedef typename Sum<MODE>::type sum_t;
    typedef Operand<MODE> op_t;
    constexpr int VEC = Elem<DT>::VEC, NV = 16 / VEC;
    constexpr int BITS = MODE == MODE_I8 ? 8 : MODE == MODE_I4 ? 4 : 6, QMAX = MODE == MODE_I8 ? 127 : 7;
    extern __shared__ __align__(16) uint8_t lds[];
    float* table = reinterpret_cast<float*>(lds);
    float* red = table + TABLE;
    sum_t* part = reinterpret_cast<sum_t*>(lds + LDS_PART);
    uint8_t* xq = lds + LDS_XQ;
    const ClockProbe probe(ticks);
    const T* X = static_cast<const T*>(Xv);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, c = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t rowbytes = MODE == MODE_I8 ? Kpad : MODE == MODE_I4 ? Kpad / 2 : Kpad / 4 * 3;

    // ---- the weight stream: steps wave, wave + NW, ... of a tile, D of them ahead ----
    RowPieces<MODE> pw, px;
    constexpr uint32_t STEP_BYTES = (MODE == MODE_F6) ? 96 : 128;
    const uint32_t stride_w = (MODE == MODE_F6) ? 96u * N : 128u, stride_x = STEP_BYTES;
    const int steps = (int)((rowbytes + STEP_BYTES - 1) / STEP_BYTES);
    const int mine = __builtin_amdgcn_readfirstlane((steps - wave + NW - 1) / NW);
    px.set(0, c, rowbytes);                                    // all 16 rows of the MFMA are the one row; the first is stored
    op_t w[D];
    auto load = [&](int d, int t) {
        const uint32_t s = (uint32_t)(wave + t * NW);
        w[d].a = *reinterpret_cast<const decltype(op_t::a)*>(W + (pw.a + s * stride_w));
        w[d].b = *reinterpret_cast<const decltype(op_t::b)*>(W + (pw.b + s * stride_w));
    };
    // the row's last step may be partial: weight chunks beyond its end count as zeros, whatever the X operand reads there
    auto load_last = [&](int d, int t) {
        if constexpr (MODE == MODE_F6) {
            load(d, t);
        } else {
            const uint32_t s = (uint32_t)(wave + t * NW), at = s * 128u + 16u * c;
            w[d].a = v4i{0, 0, 0, 0};
            w[d].b = v4i{0, 0, 0, 0};
            if (at < rowbytes) w[d].a = *reinterpret_cast<const v4i*>(W + (pw.a + s * 128u));
            if (at + 64u < rowbytes) w[d].b = *reinterpret_cast<const v4i*>(W + (pw.b + s * 128u));
        }
    };
    auto begin_tile = [&](int tile) {
        pw.set(min(tile * 16 + r, N - 1), c, rowbytes);
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < mine) load_last(d, d);
    };
    const int tiles = (N + 15) / 16;
    begin_tile(blockIdx.x);

    // ---- the activation: groups of 16 slots, one thread each ----
    const int G = Kpad >> 4;
    auto load_slots = [&](int g, int (&s)[16], int (&n)[16]) -> bool {
        load8(src + 16 * g, s);
        load8(src + 16 * g + 8, s + 8);
        load8(rep + 16 * g, n);
        load8(rep + 16 * g + 8, n + 8);
        bool plain = 16 * g + 15 < K;
#pragma unroll
        for (int i = 0; i < 16; ++i) plain = plain && s[i] == 16 * g + i;
        return plain;
    };
    // the group's 16 source elements (0 where a slot has none)
    auto load_x = [&](int g, const int (&s)[16], bool plain, float (&x)[16]) {
        if (plain) {
#pragma unroll
            for (int i = 0; i < NV; ++i) widen16<DT>(reinterpret_cast<const v4u*>(X + 16 * g)[i], x + i * VEC);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = (unsigned)s[i] < (unsigned)K ? Elem<DT>::widen(X[s[i]]) : 0.0f;
        }
    };
    // the thread's first group stays in registers, any others (more than 512 groups) are read again when they are needed
    int s0[16], n0[16];
    float x0[16];
    if (tid < G) load_x(tid, s0, load_slots(tid, s0, n0), x0);
    float a;
    if (absmax_in) {
        a = *absmax_in;
        if (!(a >= 0.0f) || a > 3.0e38f) a = 0.0f;             // negative / NaN / Inf static bound: treated as 0
    } else {
        // a' = max fl32(|x| / n): the largest exact quotient, compared by cross multiplication in float64 (exact for n <
        // 2^29), divided once per thread; rounding is monotonic.  (A branch for n = 1: 1 x 300 x 700 7.9 us, without 7.5.)
        float bc = 0.0f;
        int bn = 1;
        auto consider = [&](const int (&s)[16], const int (&n)[16], const float (&x)[16]) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float v = fabsf(x[i]);
                if ((unsigned)s[i] < (unsigned)K && n[i] > 0 && (double)v * (double)bn > (double)bc * (double)n[i]) {
                    bc = v;
                    bn = n[i];
                }
            }
        };
        if (tid < G) consider(s0, n0, x0);
        for (int g = tid + NTHR; g < G; g += NTHR) {
            int s[16], n[16];
            float x[16];
            load_x(g, s, load_slots(g, s, n), x);
            consider(s, n, x);
        }
        float best = (float)((double)bc / (double)bn);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) best = fmaxf(best, __shfl_xor(best, off, 64));
        if (lane == 0) red[wave] = best;
        __syncthreads();
        a = red[0];
#pragma unroll
        for (int v = 1; v < NW; ++v) a = fmaxf(a, red[v]);
    }
    const double ad = (double)a;
    auto multiplier = [&](int n) -> float { return (float)((double)QMAX / ((double)n * ad)); };
    if (tid < TABLE) table[tid] = (tid > 0 && a != 0.0f) ? multiplier(tid) : 0.0f;
    __syncthreads();
    const float s_x = (a == 0.0f) ? 1.0f : (float)(ad / (double)QMAX);
    const float scale = s_w ? s_x * *s_w : 1.0f;
    auto quantize = [&](int g, const int (&s)[16], const int (&n)[16], const float (&x)[16]) {
        float m[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            m[i] = 0.0f;
            if ((unsigned)s[i] < (unsigned)K && n[i] > 0) m[i] = n[i] < TABLE ? table[n[i]] : (a != 0.0f ? multiplier(n[i]) : 0.0f);
        }
        store_group<BITS>(quantize16<BITS>(x, m), xq, 0, 1, 0, g);      // a matrix of one row
    };
    if (tid < G) quantize(tid, s0, n0, x0);
    for (int g = tid + NTHR; g < G; g += NTHR) {
        int s[16], n[16];
        float x[16];
        load_x(g, s, load_slots(g, s, n), x);
        quantize(g, s, n, x);
    }
    __syncthreads();

    // ---- the product ----
    const bool vec = (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        sum_t acc = {0, 0, 0, 0};
        auto compute = [&](int d, int t) {
            const uint32_t s = (uint32_t)(wave + t * NW);
            op_t x;
            x.a = *reinterpret_cast<const decltype(op_t::a)*>(xq + (px.a + s * stride_x));
            x.b = *reinterpret_cast<const decltype(op_t::b)*>(xq + (px.b + s * stride_x));
            multiply<MODE>(w[d], x, acc);
        };
        // rounds of D steps, then the rest with scalar conditions: the MFMA ignores the execution mask
        int t = 0;
        for (; t + 2 * D < mine; t += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                compute(d, t + d);
                load(d, t + D + d);
            }
        }
        const int left = __builtin_amdgcn_readfirstlane(mine - t);     // at most 2 D, the first D of them loaded
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d < left) compute(d, t + d);
            if (D + d < left) load_last(d, t + D + d);
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (D + d < left) compute(d, t + D + d);
        // the next tile's first weights travel while this one's partial sums meet
        if (tile + (int)gridDim.x < tiles) begin_tile(tile + gridDim.x);
        part[wave * 64 + lane] = acc;
        strip_barrier();
        if (tid < 64) {
            sum_t sum = part[lane];
#pragma unroll
            for (int v = 1; v < NW; ++v) sum += part[v * 64 + lane];
            const int col = tile * 16 + 4 * c;
            if (r == 0 && col < N) store4<MODE>(sum, 0, col, N, scale, Y, y_dtype, ldy, bias, vec);
        }
        strip_barrier();
    }
    probe.finish(ticks);
}

int decode_lds(int Kpad, int bits) { return (bits == 8 ? Kpad : bits == 4 ? Kpad / 2 : Kpad / 4 * 3) + LDS_XQ + LDS_SLACK; }

template <int DT>
int launch(const void* X, int K, const int32_t* src, const int32_t* rep, int Kpad, int bits,
           const float* absmax_in, const void* W, int N, const float* s_w, const float* bias, void* Y, int y_dtype, int ldy,
           unsigned long long* ticks, int lds, hipStream_t stream)
{
    auto kern = bits == 8 ? linear_decode_kernel<DT, MODE_I8> : bits == 4 ? linear_decode_kernel<DT, MODE_I4> : linear_decode_kernel<DT, MODE_F6>;
    static std::atomic<unsigned long long> attr_set[3];
    if (int rc = set_lds_limit(reinterpret_cast<const void*>(kern), 80 * 1024, attr_set[bits == 8 ? 0 : bits == 4 ? 1 : 2])) return rc;
    const int tiles = (N + 15) / 16;
    kern<<<(unsigned)std::min(tiles, 2 * compute_units()), NTHR, lds, stream>>>(
        X, K, src, rep, Kpad, absmax_in, static_cast<const uint8_t*>(W), N, s_w, bias, Y, y_dtype, ldy, ticks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "layer launch failed: %s", hipGetErrorString(e));
    return FQ_OK;
}

}  // namespace

// One row whose quantized form leaves room for two workgroups per CU in LDS; for 4-bit weights up to 16384 columns and slots
// (beyond, the preparation weighs as much as the launch it saves: nibbles 8192 x 24576 dynamic 31.6 us against 30.6 by the
// separate kernels, 22016 x 8192 37.7 against 37.2).  E3M2 storage is for the layers that
// the quantizer takes; the others are left to it to refuse.
bool linear_decode_fits(int M, int N, int K, int Kpad, int bits)
{
    if (bits == FQ_BITS_I4_E3M2 && !quantizer_takes_e3m2(K, Kpad)) return false;
    return M == 1 && (bits == 8 || (N <= 16384 && Kpad <= 16384)) && decode_lds(Kpad, bits) <= 80 * 1024;
}

int launch_linear_decode(const void* X, int x_dtype, int K, const int32_t* src, const int32_t* rep, int Kpad, int bits,
                         const float* absmax_in, const void* W, int N, const float* s_w, const float* bias, void* Y, int y_dtype,
                         int ldy, hipStream_t stream)
{
    const int lds = decode_lds(Kpad, bits);
    unsigned long long* ticks = gemm_ticks_pointer();
    switch (x_dtype) {
    case FQ_F32: return launch<FQ_F32>(X, K, src, rep, Kpad, bits, absmax_in, W, N, s_w, bias, Y, y_dtype, ldy, ticks, lds, stream);
    case FQ_F16: return launch<FQ_F16>(X, K, src, rep, Kpad, bits, absmax_in, W, N, s_w, bias, Y, y_dtype, ldy, ticks, lds, stream);
    default: return launch<FQ_BF16>(X, K, src, rep, Kpad, bits, absmax_in, W, N, s_w, bias, Y, y_dtype, ldy, ticks, lds, stream);
    }
}

}  // namespace fq
