// Integer GEMM for problems with about as many tiles as CUs: small tiles, and all of LDS as a ring of stages.
//
// arXiv 2402.17985 Sec. 5.1 (the quantized linear layer); operands, swizzle, tile order and epilogue as in fq_gemm.hip.
// For outputs that one round of 64 x 128, 128 x 64 or 128 x 128 tiles covers, one tile per CU.  With two stage buffers a
// single 128-byte stage is then on its way while one is multiplied, and the kernel moves at the latency of memory.  Here
// the stage buffers form a ring of S that fills the 160 KiB of a CU (S = 5 at 128 x 128, else 6), S - 1 of them in flight.
// Us before / now: INT8 12544 x 4096, 1024 rows 65.7 / 54.8, 512 rows 61.7 / 37.3; 6400 x 15360, 256 rows 47.7 / 36.5, 128 rows
// 45.0 / 29.5; 4352 x 4096, 1024 rows 26.8 / 21.5; nibbles, whose stages multiply twice as long (128 x 128 tiles only), 51.9 / 50.6
// (12544 x 4096, 1024 rows), 28.2 / 28.1, 22.3 / 20.9.  Batched products keep a problem's tiles on one XCD (place_of_workgroup):
// INT8 40 x 768 x 128 of 2048 bytes 22.0 us dealt over all of them, 16.8 so; 40 x 384 x 128 17.9 / 11.2.
//
// The schedule of a stage: the MFMAs of k-slice s run while the operands of slice s + 1 are read from LDS
// into the other register buffer; before the last slice a barrier, which every wave reaches holding that slice in
// registers and having waited for its own copies of the next stage: it publishes the next stage and frees this one's
// buffer, whose refill is issued at once.
#include <atomic>
#include <type_traits>

#include "fq_gemm_common.h"
#include "fq_internal.h"

namespace fq {
namespace {

// s_waitcnt immediate: at most `vm` vector memory operations outstanding and no LDS operation
constexpr int wait_imm(int vm) { return (vm & 0xf) | ((vm >> 4) << 14) | 0x0070; }

template <int MODE, int BM, int BN, int WM, int WN, int S>
__global__ __launch_bounds__(WM * WN * 64) void gemm_ring_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B,
                                                                int M, int N, int rowbytes, const float* __restrict__ s_x,
                                                                const float* __restrict__ s_w, void* __restrict__ Y,
                                                                int y_dtype, int ldy, int tiles_m, int tiles_n, Batch bt)
{
    static_assert(MODE == MODE_I8 || MODE == MODE_I4, "16-byte operands per lane");
    constexpr int BKB = 128, NW = WM * WN, CPR = BKB / 16, RPB = 64 / CPR, KS = BKB / 32;
    constexpr int A_BLOCKS = BM / RPB / NW, B_BLOCKS = BN / RPB / NW, LPS = A_BLOCKS + B_BLOCKS;
    constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32, NR = FM + FN;
    constexpr int STAGE = (BM + BN) * BKB;
    static_assert(BM % (RPB * NW) == 0 && BN % (RPB * NW) == 0 && (RPB * NW) % 16 == 0, "copy blocks must tile the stage");
    static_assert((S - 1) * LPS < 64 && S >= 3, "outstanding copies are counted in six bits");
    static_assert(NW * TM * TN * 2 <= S * STAGE, "the output is staged through the ring");
    typedef typename Acc<MODE>::type acc_t;
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
    const int wm = wave / WN, wn = wave % WN;

    // Copies: block b of a stage operand covers its rows b RPB .. + RPB - 1; lane i lands at (row b RPB + i / CPR, stored
    // chunk i % CPR) and fetches global chunk (i % CPR) ^ swz(row).  Wave w owns blocks w, w + NW, ...  Rows beyond the
    // matrix re-read its last row.
    const int drow = lane / CPR;
    const int dchunk = (lane % CPR) ^ (((wave * RPB + drow) >> 1) & 7);
    const int nk_full = rowbytes / BKB, nk = nk_full + ((rowbytes % BKB) ? 1 : 0);
    uint32_t offA[A_BLOCKS], offB[B_BLOCKS];
#pragma unroll
    for (int j = 0; j < A_BLOCKS; ++j)
        offA[j] = (uint32_t)min(m0 + (wave + j * NW) * RPB + drow, M - 1) * (uint32_t)rowbytes + dchunk * 16;
#pragma unroll
    for (int j = 0; j < B_BLOCKS; ++j)
        offB[j] = (uint32_t)min(n0 + (wave + j * NW) * RPB + drow, N - 1) * (uint32_t)rowbytes + dchunk * 16;
    const uint32_t lds0 = (uint32_t)(size_t)FQ_LDS_PTR(smem) + wave * 1024;
    auto issue = [&](int stage, int buf) {
        const uint32_t sA = lds0 + buf * STAGE, sB = sA + BM * BKB;
        const int kb = stage * BKB;
        const uint8_t* gA = A + kb;
        const uint8_t* gB = B + kb;
        if (stage < nk_full) {
#pragma unroll
            for (int j = 0; j < A_BLOCKS; ++j) dma16(gA, offA[j], sA + j * NW * 1024);
#pragma unroll
            for (int j = 0; j < B_BLOCKS; ++j) dma16(gB, offB[j], sB + j * NW * 1024);
        } else {
            // last, partial stage: chunks at or beyond the row end are zeros, the number of copies stays the same
            const bool ok = kb + dchunk * 16 < rowbytes;
            const uint8_t* z = reinterpret_cast<const uint8_t*>(g_zero_chunk);
#pragma unroll
            for (int j = 0; j < A_BLOCKS; ++j) dma16_addr(ok ? gA + offA[j] : z, sA + j * NW * 1024);
#pragma unroll
            for (int j = 0; j < B_BLOCKS; ++j) dma16_addr(ok ? gB + offB[j] : z, sB + j * NW * 1024);
        }
    };

    const int frow = lane & 31, fhalf = lane >> 5, fsw = (frow >> 1) & 7;
    int kofs[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kofs[ks] = ((2 * ks + fhalf) ^ fsw) << 4;
    const int a_rd = (wm * TM + frow) * BKB, b_rd = BM * BKB + (wn * TN + frow) * BKB;

    acc_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // operands of a slice in the order the MFMA walk needs them: a0, b0 .. b(FN-1), a1 ..
    v4i a[2][FM], b[2][FN];
    auto read_op = [&](const uint8_t* st, int buf, int ks, int r) {
        if (r == 0) a[buf][0] = *reinterpret_cast<const v4i*>(st + a_rd + kofs[ks]);
        else if (r <= FN) b[buf][r - 1] = *reinterpret_cast<const v4i*>(st + b_rd + (r - 1) * 32 * BKB + kofs[ks]);
        else a[buf][r - FN] = *reinterpret_cast<const v4i*>(st + a_rd + (r - FN) * 32 * BKB + kofs[ks]);
    };
    // the MFMAs of the slice in buffer cur; two reads of slice rks of the stage at rs after each of the first ones
    auto slice = [&](int cur, const uint8_t* rs, int rks, bool rd) {
        constexpr int HI = (int)0xf0f0f0f0, NM = FM * FN, SLOTS = (MODE == MODE_I4) ? 2 * NM : NM;
        v4i lo_a[FM], lo_b[FN], hi_a[FM], hi_b[FN];
#pragma unroll
        for (int t = 0; t < SLOTS; ++t) {
            const int i = (t % NM) / FN, j = t % FN;
            if constexpr (MODE == MODE_I8) {
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b[cur][j], a[cur][i], acc[i][j], 0, 0, 0);
            } else if (t < NM) {                       // widen an operand the first time it is needed
                if (j == 0) lo_a[i] = (a[cur][i] << 4) & HI;
                if (i == 0) lo_b[j] = (b[cur][j] << 4) & HI;
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(lo_b[j], lo_a[i], acc[i][j], 0, 0, 0);
            } else {
                if (j == 0) hi_a[i] = a[cur][i] & HI;
                if (i == 0) hi_b[j] = b[cur][j] & HI;
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(hi_b[j], hi_a[i], acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (rd && 2 * t < NR) {
                read_op(rs, cur ^ 1, rks, 2 * t);
                if (2 * t + 1 < NR) read_op(rs, cur ^ 1, rks, 2 * t + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

#pragma unroll
    for (int st = 0; st < S; ++st)
        if (st < nk) issue(st, st);
    if (nk >= S) __builtin_amdgcn_s_waitcnt(wait_imm((S - 1) * LPS));
    else __builtin_amdgcn_s_waitcnt(wait_imm(0));
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) read_op(smem, 0, 0, r);
    __builtin_amdgcn_sched_barrier(0);
    int buf = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const int next = buf + 1 == S ? 0 : buf + 1;
        const uint8_t* s = smem + buf * STAGE;
        const uint8_t* sn = smem + next * STAGE;
#pragma unroll
        for (int ks = 0; ks < KS - 1; ++ks) slice(ks & 1, s, ks + 1, true);
        // my copies of stage kt + 1 have landed: of the stages issued after it (kt + 2 .. kt + S - 1), all may be outstanding
        if (kt + S - 1 < nk) __builtin_amdgcn_s_waitcnt(wait_imm((S - 2) * LPS));
        else __builtin_amdgcn_s_waitcnt(wait_imm(0));
        __syncthreads();
        if (kt + S < nk) issue(kt + S, buf);
        __builtin_amdgcn_sched_barrier(0);
        slice((KS - 1) & 1, sn, 0, kt + 1 < nk);
        buf = next;
    }
    // no wave reads the ring any more (the last slice's operands are in registers): each stages its output in its share
    store_tile<MODE, FM, FN>(acc, m0 + wm * TM, n0 + wn * TN, M, N, scale, Y, y_dtype, ldy, smem + wave * (TM * TN * 2), bt.bias);
    probe.finish(bt.ticks);
}

template <int MODE, int BM, int BN, int WM, int WN, int S>
int launch(const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w, void* Y, int y_dtype,
           int ldy, Batch bt, hipStream_t stream)
{
    auto kern = gemm_ring_kernel<MODE, BM, BN, WM, WN, S>;
    constexpr int smem = S * (BM + BN) * 128;
    static std::atomic<unsigned long long> attr_set{0};
    if (int rc = set_lds_limit(reinterpret_cast<const void*>(kern), smem, attr_set)) return rc;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    kern<<<dim3((unsigned)(tiles_m * tiles_n), (unsigned)bt.count), dim3(WM * WN * 64), smem, stream>>>(
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
#define FQ_L(BM, BN, WM, WN, S) launch<MODE, BM, BN, WM, WN, S>(A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream)
    if constexpr (MODE == MODE_I8) {
        if (tile == RING_64x128) return FQ_L(64, 128, 2, 2, 6);
        if (tile == RING_128x64) return FQ_L(128, 64, 2, 2, 6);
    }
    if (tile == RING_128x128) return FQ_L(128, 128, 2, 4, 5);
    return fail(FQ_ERR_RANGE, "unknown ring tile %d", tile);
#undef FQ_L
}

}  // namespace

int launch_gemm_ring(int tile, int bits, const void* A, const void* B, int M, int N, int rowbytes, const float* s_x, const float* s_w,
                     void* Y, int y_dtype, int ldy, Batch bt, hipStream_t stream)
{
    if (bits == 8) return launch_mode<MODE_I8>(tile, A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
    return launch_mode<MODE_I4>(tile, A, B, M, N, rowbytes, s_x, s_w, Y, y_dtype, ldy, bt, stream);
}

}  // namespace fq
