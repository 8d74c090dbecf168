// Integer GEMM for few output tiles: small tiles, the reduction split over the waves of a workgroup.
//
// arXiv 2402.17985 Sec. 5.1 (the quantized linear layer); operands, LDS layouts and values as in fq_gemm.hip.
// From a few rows of X up to a few hundred, a product has fewer 128 x 128 tiles than there are CUs, and a workgroup that
// walks its reduction stage by stage is bound by latency: copy a stage, barrier, read operands, multiply, barrier -- 0.3
// (64 x 64 tile) to 0.5 us (128 x 128) per 128-byte stage, with two stage buffers or with a ring of five to eight, against
// 0.06-0.25 us of MFMA.  Here every wave owns the whole tile (up to 96 x 64) for its share of the reduction: wave w takes
// the stages w, w + NW, ... through a private ring of S stages in LDS.  Waves share nothing until the end, so the main loop
// has no barrier: a wave waits for its own copies only, and the latencies of NW waves overlap.  An operand read feeds 32
// to 64 columns of MFMA, and no wave reads what another reads.  The partial accumulators meet in LDS (exact in any order:
// integers, or fp32 holding integers below 2^24).
// Us before / now: INT8 12544 x 4096, 64 rows 52.5 / 13.0, 128 rows 52.6 / 16.8, 256 rows 54.6 / 21.7, 384 rows 57.1 / 27.7;
// 6400 x 15360, 64 rows 44.9 / 24.5; nibbles 12544 x 4096, 64 rows 33.9 / 8.9, 256 rows 33.6 / 18.1; E3M2 42.3 / 10.4 and 40.3 / 17.4.
// What bounds it then, while the operands are near, is the traffic from L2 into the CUs, (BM + BN) * Kpad bytes per workgroup:
// 15.6-18.0 TB/s of L2 reads counted with all CUs busy (INT8 12544 x 4096, 64-384 rows; nibbles 12.5).  So the tile is the
// smallest for which one round of workgroups covers the output.  Weights that come from memory bound it first: INT8 77 x 15360
// x 5760 reads 211 MB from L2 at 7.2 TB/s, 100 MB of them past it at 3.4.  Batched products keep a
// problem's tiles on one XCD (place_of_workgroup): dealt over all of them, every L2 read every problem's operands, and 40 x
// 256 x 128 of 1024 bytes took 11.4 us against 9.0 so and 9.6 by the 128 x 128 tiles; 40 x 128 x 128 7.6 / 6.2 / 9.0.
#include <atomic>

#include "fq_gemm_common.h"
#include "fq_internal.h"

namespace fq {
namespace {

// s_waitcnt immediate: at most `vm` vector memory operations outstanding and no LDS operation
constexpr int wait_imm(int vm) { return (vm & 0xf) | ((vm >> 4) << 14) | 0x0070; }

// Bytes of a row in a stage, k-slices per stage (one MFMA, for packed nibbles two), a lane's operand and the vector in
// which four accumulators are summed
template <int MODE> struct Stage {
    static constexpr int SB = 128, KS = 4;
    typedef v4i operand;
    typedef v4i sum4;
};
template <> struct Stage<MODE_F6> {
    static constexpr int SB = 96, KS = 2;
    typedef v8i operand;
    typedef v4f sum4;
};

// Partial tiles of `bytes` that are summed through LDS at once: all waves', or half of them after folding the upper half
template <int NW> constexpr int partial_sums(int bytes) { return NW * bytes > 160 * 1024 ? NW / 2 : NW; }

template <int MODE, int BM, int BN, int NW, int S>
__global__ __launch_bounds__(NW * 64) void gemm_stream_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B,
                                                             int M, int N, int rowbytes, const float* __restrict__ s_x,
                                                             const float* __restrict__ s_w, void* __restrict__ Y,
                                                             int y_dtype, int ldy, int tiles_m, int tiles_n, Batch bt)
{
    typedef typename Acc<MODE>::type acc_t;
    typedef typename Stage<MODE>::operand op_t;
    typedef typename Stage<MODE>::sum4 sum4_t;
    constexpr int SB = Stage<MODE>::SB, KS = Stage<MODE>::KS, CPR = SB / 16;
    constexpr int A_BLOCKS = BM * SB / 1024, B_BLOCKS = BN * SB / 1024, LPS = A_BLOCKS + B_BLOCKS;   // 1 KiB copies
    constexpr int FM = BM / 32, FN = BN / 32;
    constexpr int STAGE = (BM + BN) * SB;
    static_assert(BM % 32 == 0 && BN % 32 == 0 && S * LPS < 64, "tiles of whole MFMA blocks; copies are counted in six bits");
    extern __shared__ __align__(16) uint8_t smem[];
    const ClockProbe probe(bt.ticks);
    int problem, id, tile_m, tile_n;
    if (place_of_workgroup(tiles_m * tiles_n, bt.count, problem, id)) tile_of_logical(id, tiles_m, tiles_n, tile_m, tile_n);
    else tile_of_workgroup(id, tiles_m * tiles_n, tiles_m, tiles_n, tile_m, tile_n);
    A += (size_t)problem * bt.stride_a;
    B += (size_t)problem * bt.stride_b;
    Y = static_cast<uint8_t*>(Y) + (size_t)problem * bt.stride_y;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const float scale = tile_scale<MODE>(s_x, s_w);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t* ring = smem + wave * (S * STAGE);

    // Copies: lane i of copy j fills the 16-byte chunk c = 64 j + i of the operand's stage, row c / CPR, position c % CPR,
    // which holds the row's chunk gc: bank swizzles, see the kernels of fq_gemm.hip (128-byte rows: position ^ (row / 2) %
    // 8; 96-byte rows: the halves exchanged in rows with bit 2 ^ bit 3 set).  Rows beyond the matrix re-read its last one.
    auto chunk_of = [&](int j) -> int {
        const int c = 64 * j + lane, row = c / CPR, pos = c % CPR;
        if constexpr (MODE == MODE_F6) return (((row >> 2) ^ (row >> 3)) & 1) ? (pos + 3) % CPR : pos;
        else return pos ^ ((row >> 1) & 7);
    };
    const uint32_t pitch = (MODE == MODE_F6) ? 96u : (uint32_t)rowbytes;     // between the rows of a stage
    uint32_t offA[A_BLOCKS], offB[B_BLOCKS];
#pragma unroll
    for (int j = 0; j < A_BLOCKS; ++j) offA[j] = (uint32_t)min(m0 + (64 * j + lane) / CPR, M - 1) * pitch + 16 * chunk_of(j);
#pragma unroll
    for (int j = 0; j < B_BLOCKS; ++j) offB[j] = (uint32_t)min(n0 + (64 * j + lane) / CPR, N - 1) * pitch + 16 * chunk_of(j);
    // between the stages of an operand
    const size_t next_a = (MODE == MODE_F6) ? (size_t)M * 96 : 128, next_b = (MODE == MODE_F6) ? (size_t)N * 96 : 128;
    const uint32_t lds0 = (uint32_t)(size_t)FQ_LDS_PTR(ring);
    const int nk = (rowbytes + SB - 1) / SB;
    const int mine = __builtin_amdgcn_readfirstlane((nk - wave + NW - 1) / NW);   // this wave's stages: wave, wave + NW, ...
    auto issue = [&](int t, int buf) {
        const uint32_t sA = lds0 + buf * STAGE, sB = sA + BM * SB;
        const int st = wave + t * NW;
        const uint8_t* gA = A + st * next_a;
        const uint8_t* gB = B + st * next_b;
        if (MODE == MODE_F6 || (st + 1) * SB <= rowbytes) {
#pragma unroll
            for (int j = 0; j < B_BLOCKS; ++j) dma16(gB, offB[j], sB + j * 1024);
#pragma unroll
            for (int j = 0; j < A_BLOCKS; ++j) dma16(gA, offA[j], sA + j * 1024);
        } else {
            // last, partial stage: chunks at or beyond the row end are zeros, the number of copies stays the same
            const uint8_t* z = reinterpret_cast<const uint8_t*>(g_zero_chunk);
#pragma unroll
            for (int j = 0; j < B_BLOCKS; ++j) dma16_addr(st * SB + 16 * chunk_of(j) < rowbytes ? gB + offB[j] : z, sB + j * 1024);
#pragma unroll
            for (int j = 0; j < A_BLOCKS; ++j) dma16_addr(st * SB + 16 * chunk_of(j) < rowbytes ? gA + offA[j] : z, sA + j * 1024);
        }
    };

    // a lane's operand: row lane % 32 of a block, k-half lane / 32 of the slice
    const int frow = lane & 31, fhalf = lane >> 5;
    const int a_rd = frow * SB, b_rd = BM * SB + frow * SB;
    int ofs[KS], ofs_y[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if constexpr (MODE == MODE_F6) {
            const int grp = 48 * (ks ^ (((frow >> 2) ^ (frow >> 3)) & 1)), mirrored = (fhalf ^ (frow >> 4)) & 1;
            ofs[ks] = grp + (mirrored ? 32 : 0);
            ofs_y[ks] = grp + (mirrored ? 24 : 16);
        } else {
            ofs[ks] = ((2 * ks + fhalf) ^ ((frow >> 1) & 7)) << 4;
        }
    }
    auto read = [&](const uint8_t* row, int ks) -> op_t {
        const v4i x = *reinterpret_cast<const v4i*>(row + ofs[ks]);
        if constexpr (MODE == MODE_F6) {
            const v2i y = *reinterpret_cast<const v2i*>(row + ofs_y[ks]);
            return op_t{x[0], x[1], x[2], x[3], y[0], y[1], 0, 0};
        } else {
            return x;
        }
    };

    acc_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    op_t a[2][FM], b[2][FN];
    auto read_slice = [&](const uint8_t* st, int buf, int ks) {
#pragma unroll
        for (int j = 0; j < FN; ++j) b[buf][j] = read(st + b_rd + j * 32 * SB, ks);
#pragma unroll
        for (int i = 0; i < FM; ++i) a[buf][i] = read(st + a_rd + i * 32 * SB, ks);
    };
    auto multiply = [&](const op_t (&x)[FM], const op_t (&w)[FN]) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if constexpr (MODE == MODE_F6) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[j], x[i], acc[i][j], 3, 3, 0, 127, 0, 127);
                else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[j], x[i], acc[i][j], 0, 0, 0);
            }
    };
    auto slice = [&](int cur) {
        if constexpr (MODE == MODE_I4) {
            constexpr int HI = (int)0xf0f0f0f0;
            op_t la[FM], lb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                la[i] = (a[cur][i] << 4) & HI;
                a[cur][i] = a[cur][i] & HI;
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                lb[j] = (b[cur][j] << 4) & HI;
                b[cur][j] = b[cur][j] & HI;
            }
            multiply(la, lb);
        }
        multiply(a[cur], b[cur]);
    };

#pragma unroll
    for (int st = 0; st < S; ++st)
        if (st < mine) issue(st, st);
    int buf = 0;
    for (int t = 0; t < mine; ++t) {
        // stage t has landed: of the stages issued after it (up to S - 1), all may be outstanding
        if (t + S <= mine) __builtin_amdgcn_s_waitcnt(wait_imm((S - 1) * LPS));
        else __builtin_amdgcn_s_waitcnt(wait_imm(0));
        asm volatile("" ::: "memory");
        const uint8_t* s = ring + buf * STAGE;
        read_slice(s, 0, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) {
                read_slice(s, (ks + 1) & 1, ks + 1);
            } else {
                // every operand of the stage is in registers: its buffer takes the stage S ahead
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (t + S < mine) issue(t + S, buf);
            }
            slice(ks & 1);
        }
        buf = buf + 1 == S ? 0 : buf + 1;
    }

    // ---- the waves' partial sums ----
    __syncthreads();
    sum4_t* part = reinterpret_cast<sum4_t*>(smem);             // [NP][FM FN][4][64]
    constexpr int NP = partial_sums<NW>(BM * BN * 4);
    constexpr bool FOLD = NP < NW;                              // too many for LDS: the upper half is added to the lower first
    static_assert(!FOLD || NW % 2 == 0, "waves are folded in pairs");
    auto write_part = [&](int slot) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    part[((slot * FM * FN + i * FN + j) * 4 + g) * 64 + lane] =
                        sum4_t{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
    };
    if constexpr (FOLD) {
        if (wave >= NP) write_part(wave - NP);
        __syncthreads();
        if (wave < NP) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const sum4_t o = part[((wave * FM * FN + i * FN + j) * 4 + g) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i][j][4 * g + e] += o[e];
                    }
        }
        __syncthreads();
    }
    if (!FOLD || wave < NP) write_part(wave);
    __syncthreads();
    const bool vec = (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
    for (int p = tid; p < FM * FN * 4 * 64; p += NW * 64) {
        sum4_t sum = part[p];
#pragma unroll
        for (int w = 1; w < NP; ++w) sum += part[w * (FM * FN * 256) + p];
        const int l = p & 63, g = (p >> 6) & 3, f = p >> 8;
        const int row = m0 + (f / FN) * 32 + (l & 31), col = n0 + (f % FN) * 32 + 8 * g + 4 * (l >> 5);
        if (row < M && col < N) store4<MODE>(sum, row, col, N, scale, Y, y_dtype, ldy, bt.bias, vec);
    }
    probe.finish(bt.ticks);
}

template <int MODE, int BM, int BN, int NW, int S>
int launch(const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w, void* Y, int y_dtype,
           int ldy, Batch bt, hipStream_t stream)
{
    auto kern = gemm_stream_kernel<MODE, BM, BN, NW, S>;
    constexpr int ring = NW * S * (BM + BN) * Stage<MODE>::SB;
    constexpr int parts = partial_sums<NW>(BM * BN * 4) * BM * BN * 4, smem = ring > parts ? ring : parts;
    static_assert(smem <= 160 * 1024, "LDS of a CU");
    static std::atomic<unsigned long long> attr_set{0};
    if (int rc = set_lds_limit(reinterpret_cast<const void*>(kern), smem, attr_set)) return rc;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    kern<<<dim3((unsigned)(tiles_m * tiles_n), (unsigned)bt.count), dim3(NW * 64), smem, stream>>>(
        static_cast<const uint8_t*>(A), static_cast<const uint8_t*>(B), M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, tiles_m,
        tiles_n, bt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "GEMM launch failed: %s", hipGetErrorString(e));
    return FQ_OK;
}

template <int MODE>
int launch_mode(int tile, const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w, void* Y,
                int y_dtype, int ldy, Batch bt, hipStream_t stream)
{
#define FQ_L(BM, BN, NW, S) launch<MODE, BM, BN, NW, S>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream)
    // Waves and stages per tile: many waves with one stage each, or fewer with two or three, whichever measured faster.  Eight
    // waves of one stage against four of two, 64 x 64: INT8 12544 x 4096, 256 rows 21.5 / 22.3 us, 4608 x 11008, 64 rows 13.5 / 13.0;
    // nibbles (twice the MFMA work per byte) 16.0 / 19.2, 9.8 / 11.3; at 96 x 64 nibbles 21.1 / 25.0 (384 rows), INT8 28.2 / 28.7 there
    // but 16.8 / 15.5 at 4608 x 11008, 96 rows; at 32 x 64 nibbles 8.2 / 8.9 (12 waves), INT8 11.9 / 11.1.
    constexpr bool I4 = MODE == MODE_I4;
    switch (tile) {
    case STREAM_32x32: return FQ_L(32, 32, 8, 2);
    case STREAM_32x64: return FQ_L(32, 64, I4 ? 12 : 4, I4 ? 1 : 3);
    case STREAM_64x64: return FQ_L(64, 64, 8, 1);
    case STREAM_32x128: return FQ_L(32, 128, 4, 2);
    case STREAM_96x64: return FQ_L(96, 64, I4 ? 8 : 4, I4 ? 1 : 2);
    default: break;
    }
    if constexpr (MODE != MODE_I8) {
        if (tile == STREAM_128x64) return FQ_L(128, 64, 6, 1);
        if (tile == STREAM_64x128) return FQ_L(64, 128, 6, 1);
    }
    return fail(FQ_ERR_RANGE, "unknown stream tile %d", tile);
#undef FQ_L
}

}  // namespace

int launch_gemm_stream(int tile, int bits, const void* A, const void* B, int M, int N, int rowbytes, const float* s_x,
                       const float* s_w, void* Y, int y_dtype, int ldy, Batch bt, hipStream_t stream)
{
    if (bits == 8) return launch_mode<MODE_I8>(tile, A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
    if (bits == FQ_BITS_I4_E3M2) return launch_mode<MODE_F6>(tile, A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
    return launch_mode<MODE_I4>(tile, A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
}

}  // namespace fq
