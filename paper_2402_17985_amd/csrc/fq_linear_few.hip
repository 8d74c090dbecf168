// The whole layer for a few rows (decoding a batch of sequences) in one kernel: every workgroup quantizes all rows for
// itself, into LDS, while its share of the weights is on its way into registers.
//
// arXiv 2402.17985 Sec. 4.1 Eq. 3, Sec. 2.1 Eq. 1 (flatten and quantize) and Sec. 5.1 (the quantized linear layer); the
// values are those of the separate kernels, bit for bit.
// With separate kernels such a layer is two launches in a row, neither of which fills the chip: a quantizer of a few
// workgroups (6-10 us, a chain of latencies) and then the stream of the weights.  X and the map come out of L2, so each
// workgroup (one per CU) quantizes everything, with one part of its waves, while the others ask for the weights:
//   quantize   up to 8 waves, a thread per group of 16 slots and up to 8 rows (4 of fp32) in registers: absmax (dynamic scale),
//              multipliers, quantized rows into LDS, appended slots copied there; groups that are neither plain nor such copies
//              are listed and gathered a slot per lane
//   stream     the rest of 16 waves: the reduction split over them, a step of 16 FN columns per wave and turn, the first
//              steps in registers before the rows are ready; then the product, whose partial sums meet in LDS
// The columns of a workgroup are a multiple of 4 and not of the 16 of an MFMA, so that all CUs get the same share (5120 columns: 20
// each, 12 of the second fragment's rows re-read the last one).
// What bounds it: at one row the weights' way from memory (5120 x 5120 INT8: 28 MB in 9.4 us, the launch and 6 us of loads at
// 4.7 TB/s); from 8 rows on the quantizer's instructions, which every CU repeats (16 x 4096: 2.6 us for 65536 elements, and 2 us for
// reading X, 128 KiB per CU).  Code that a call passes is fetched anew by every launch: the rare paths are loops, not unrolled
// (50 -> 30 KB per kernel: 1 x 5120 x 5120 9.9 -> 9.5 us, 16 x 256 x 256 8.4 -> 7.9), and a register spilled to scratch costs a
// round trip to memory at the end (16 x 4096 x 11008 nibbles: 1.5 us), hence the steps in flight per FN below.
// Us, separate kernels (one row: linear_decode_kernel) / this: INT8 1 x 5120 x 5120 static 12.4 / 9.4, 1 x 8192 x 8192 23.4 / 15.8,
// 4 x 5120 x 5120 dynamic 17.4 / 11.1, 8 x 4096 x 4096 13.0 / 9.9, 16 x 4096 x 12288 20.8 / 17.1; fp32 16 x 256 x 256 9.8 / 7.5;
// nibbles 1 x 4096 x 11008 14.0 / 10.2, 16 x 4096 x 11008 16.4 / 13.9; E3M2 2 x 4096 x 11008 15.9 / 11.8.
#include <algorithm>
#include <atomic>

#include "fq_gemm_skinny.h"
#include "fq_internal.h"
#include "fq_quant_common.h"
#include "fq_rules.h"

namespace fq {
namespace {

constexpr int TABLE = FEW_TABLE, RED = FEW_WAVES, MANY = 255, LDS_FIXED = FEW_LDS_FIXED, PAD = FEW_PAD;

// Maximum over a wave of non-negative floats, in lane 63: within rows of 16 lanes, then across them, without LDS.
__device__ __forceinline__ float wave_max(float v)
{
#define FQ_STEP(CTRL) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true)))
    FQ_STEP(0x111);                                           // row_shr:1, 2, 4, 8; lanes beyond a row count as 0
    FQ_STEP(0x112);
    FQ_STEP(0x114);
    FQ_STEP(0x118);
    FQ_STEP(0x142);                                           // row_bcast:15, 31
    FQ_STEP(0x143);
#undef FQ_STEP
    return v;
}

// Steps of the weights in flight per wave: what leaves the kernel without scratch
template <int MODE, int FN> constexpr int depth() { return FN == 1 ? 8 : FN == 2 ? (MODE == MODE_I4 ? 3 : 4) : FN == 3 && MODE == MODE_F6 ? 3 : 2; }

// Largest magnitude of the 16 columns over the rows that a thread holds.  Magnitudes of 2-byte types order as
// integers: a maximum takes two instructions for two elements.  NaN does not count, as in fmaxf: where the largest is not
// finite (the exponent's bits all set), the elements are looked at one by one.
template <int DT, int IT>
__device__ __forceinline__ void column_maxima(const v4u (&raw)[IT][16 / Elem<DT>::VEC], int held, float (&mx)[16])
{
    constexpr int VEC = Elem<DT>::VEC, NV = 16 / VEC;
    if constexpr (DT != FQ_F32) {
        typedef unsigned short v2s __attribute__((ext_vector_type(2)));
        constexpr uint32_t TOP = DT == FQ_BF16 ? 0x7f80u : 0x7c00u;
        v2s m[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) m[k] = v2s{0, 0};
#pragma unroll
        for (int i = 0; i < IT; ++i)
            if (i < held) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t u = raw[i][k >> 2][k & 3] & 0x7fff7fffu;
                    m[k] = __builtin_elementwise_max(m[k], __builtin_bit_cast(v2s, u));
                }
            }
        v2s top = m[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) top = __builtin_elementwise_max(top, m[k]);
        if (__builtin_expect(top[0] < TOP && top[1] < TOP, 1)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4u packed;
#pragma unroll
                for (int k = 0; k < 4; ++k) packed[k] = __builtin_bit_cast(uint32_t, m[4 * h + k]);
                widen16<DT>(packed, mx + 8 * h);
            }
            return;
        }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) mx[k] = 0.0f;
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (i < held) {
            float x[16];
#pragma unroll
            for (int v = 0; v < NV; ++v) widen16<DT>(raw[i][v], x + v * VEC);
#pragma unroll
            for (int k = 0; k < 16; ++k) mx[k] = fmaxf(mx[k], fabsf(x[k]));
        }
}

template <int DT, int MODE, int FN>
__global__ __launch_bounds__(FEW_WAVES * 64) void linear_few_kernel(const void* __restrict__ Xv, FewShape sh, const int32_t* __restrict__ src,
                                                          const int32_t* __restrict__ rep, const float* __restrict__ absmax_in,
                                                          const uint8_t* __restrict__ W, const float* __restrict__ s_w,
                                                          const float* __restrict__ bias, void* __restrict__ Y, int y_dtype,
                                                          int ldy, unsigned long long* ticks)
{
    typedef typename Elem<DT>::type T;
    typedef typename Sum<MODE>::type sum_t;
    typedef Operand<MODE> op_t;
    constexpr int VEC = Elem<DT>::VEC, NV = 16 / VEC, D = depth<MODE, FN>(), IT = few_rows_held(DT == FQ_F32 ? 4 : 2);
    constexpr int BITS = MODE == MODE_I8 ? 8 : MODE == MODE_I4 ? 4 : 6, QMAX = MODE == MODE_I8 ? 127 : 7;
    extern __shared__ __align__(16) uint8_t lds[];
    const ClockProbe probe(ticks);
    const T* X = static_cast<const T*>(Xv);
    const int M = sh.M, K = sh.K, Kpad = sh.Kpad, N = sh.N;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
    const int PW = sh.prep_waves, SW = waves - PW, nprep = PW << 6;
    const int NH = K >> 4, KQ = NH << 4, G = Kpad >> 4, NT = G - NH;       // groups of 16 slots: head, all, tail
    const uint32_t rowbytes = MODE == MODE_I8 ? Kpad : MODE == MODE_I4 ? Kpad / 2 : Kpad / 4 * 3;
    const uint32_t pitch = MODE == MODE_F6 ? 0 : few_row(rowbytes);
    // LDS: [fixed][counts8][xq: the quantized rows][qs: the head's values, a byte each; INT8: xq itself][ts][tf][list][part]
    float* table = reinterpret_cast<float*>(lds);
    float* red = table + TABLE;
    int* others = reinterpret_cast<int*>(red + RED);          // groups that are neither plain nor copies of plain ones
    uint8_t* counts8 = lds + LDS_FIXED;
    uint8_t* xq = counts8 + KQ + PAD;
    const uint32_t xq_bytes = MODE == MODE_F6 ? M * rowbytes : M * pitch;
    uint8_t* qs = MODE == MODE_I8 ? xq : xq + xq_bytes;
    const uint32_t qpitch = MODE == MODE_I8 ? pitch : (uint32_t)(KQ + PAD);
    // (INT8: the first of the zeros after a row)
    const uint32_t zero_at = MODE == MODE_I8 ? rowbytes : (uint32_t)KQ;    // a byte of every row of qs that is 0
    uint16_t* ts = reinterpret_cast<uint16_t*>(MODE == MODE_I8 ? xq + xq_bytes : qs + M * qpitch);
    uint8_t* tf = reinterpret_cast<uint8_t*>(ts + NT * 16);
    uint16_t* list = reinterpret_cast<uint16_t*>(tf + ((NT + 15) & ~15));    // those groups
    sum_t* part = reinterpret_cast<sum_t*>(list + ((G + 7) & ~7));

    const int round = gridDim.x * sh.cols;                    // columns of a round of all workgroups
    float a = 0.0f;                                            // the tensor's bound a'
    auto set_static = [&](float bound) { a = !(bound >= 0.0f) || bound > 3.0e38f ? 0.0f : bound; };   // negative / NaN / Inf: 0
    auto max_of_red = [&]() -> float {
        float v = red[0];
#pragma unroll
        for (int k = 1; k < RED; ++k) v = k < PW ? fmaxf(v, red[k]) : v;
        return v;
    };
    // The two kinds of waves share nothing but LDS and go through the same barriers: their registers are never live together.
    if (wave < PW) {
        // ---- quantization ----
        auto multiplier = [&](int n) -> float { return (float)((double)QMAX / ((double)n * (double)a)); };
        auto fill_table = [&]() {
            for (int n = tid; n < TABLE; n += nprep) table[n] = (n > 0 && a != 0.0f) ? multiplier(n) : 0.0f;
        };
        // a' from all of X: of several copies the largest exact quotient |x| / n, compared by cross multiplication in float64
        // (exact for n < 2^29) and divided once; rounding is monotonic
        float best = 0.0f, bc = 0.0f;
        int bn = 1;
        auto consider = [&](float v, int n) {
            if (n == 1) {
                best = fmaxf(best, v);
            } else if ((double)v * (double)bn > (double)bc * (double)n) {
                bc = v;
                bn = n;
            }
        };
        auto reduce_to_red = [&]() {
            if (bn != 1) best = fmaxf(best, (float)((double)bc / (double)bn));
            best = wave_max(best);
            if (lane == 63) red[wave] = best;
        };
        const int head = nprep / sh.slots;                     // threads that cover the head, a group each
        int slot = 0;
        for (int v = wave; v >= (head >> 6); v -= head >> 6) ++slot;
        // This thread's group.  16 elements of a 2-byte type are two 16-byte chunks: a wave loads its 128 chunks of a row 64 at a time,
        // whole lines per instruction (loaded pairwise by their owners, the lines cost twice the time), and adjacent lanes
        // exchange: even lanes own the groups of the first 64 chunks, odd lanes those of the others.
        constexpr bool PAIRS = NV == 2;
        const int w0 = (wave - slot * (head >> 6)) << 6;       // the wave's first group
        const int g = PAIRS ? w0 + (lane >> 1) + (lane & 1) * 32 : w0 + lane;
        float bound = 0.0f;
        if (absmax_in) bound = *absmax_in;
        // the head of the map, four slots per thread and pass (NH <= head: at most four passes)
        v4i sv[4];
        i4a4 nv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int at = (tid + k * nprep) * 4;
            if (at < KQ) {
                sv[k] = *reinterpret_cast<const v4i*>(src + at);
                nv[k] = *reinterpret_cast<const i4a4*>(rep + at);
            }
        }
        // rows slot, slot + slots, ... of the group, `held` of them
        const int held = (M - slot + sh.slots - 1) / sh.slots;
        auto row_of = [&](int i) -> int { return slot + sh.slots * i; };
        v4u raw[IT][NV];
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int row = row_of(i);
            if (i < held) {
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int chunk = PAIRS ? 2 * w0 + 64 * v + lane : g * NV + v;
                    if (chunk < NH * NV) raw[i][v] = reinterpret_cast<const v4u*>(X + (size_t)row * sh.ld)[chunk];
                }
            }
        }
        if (tid == 0) *others = 0;
        strip_barrier();                                       // (x) X is asked for before the weights
        // A head group is plain when its slots are the channels at the same indices with copies; its copy counts are left in LDS as
        // bytes, 0 in other groups.
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int at = (tid + k * nprep) * 4;
            if (at < KQ) {
                bool ok = true;
                uint32_t n = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ok = ok && sv[k][i] == at + i && nv[k].v[i] > 0;
                    n |= ((uint32_t)min(nv[k].v[i], MANY) & 0xffu) << (8 * i);
                }
                int all = ok ? 1 : 0;                          // of the group's four threads, the lanes of a quad
                all &= __builtin_amdgcn_update_dpp(0, all, 0xb1, 0xf, 0xf, true);
                all &= __builtin_amdgcn_update_dpp(0, all, 0x4e, 0xf, 0xf, true);
                if (!all && (lane & 3) == 0) list[atomicAdd(others, 1)] = (uint16_t)(at >> 4);
                *reinterpret_cast<uint32_t*>(counts8 + at) = all ? n : 0u;
            }
        }
        // the zeros after a row of xq, up to a whole step and the PAD that follows it, and the one after a row of qs
        if constexpr (MODE != MODE_F6) {
            const uint32_t words = (pitch - rowbytes) >> 2;
            for (uint32_t i = tid; i < M * words; i += nprep) *reinterpret_cast<uint32_t*>(xq + i / words * pitch + rowbytes + i % words * 4) = 0;
        }
        if (BITS != 8 && tid < M) qs[(size_t)tid * qpitch + zero_at] = 0;
        if (tid == 0) counts8[KQ] = 0;
        strip_barrier();                                       // (0) counts8
        uint32_t nb[4] = {0, 0, 0, 0};                         // the group's copy counts, if it is plain
        bool plain = false, many = false;
        if (g < NH) {
            const v4u n = *reinterpret_cast<const v4u*>(counts8 + (g << 4));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                nb[i] = n[i];
#pragma unroll
                for (int k = 0; k < 4; ++k) many = many || ((n[i] >> (8 * k)) & 0xff) == MANY;
            }
            plain = (nb[0] & 0xff) != 0;
        }
        if constexpr (PAIRS) {
#pragma unroll
            for (int i = 0; i < IT; ++i)
                if (i < held) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t a0 = raw[i][0][k], b0 = raw[i][1][k];
                        const uint32_t a1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a0, 0xb1, 0xf, 0xf, true);
                        const uint32_t b1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b0, 0xb1, 0xf, 0xf, true);
                        raw[i][0][k] = (lane & 1) ? b1 : a0;
                        raw[i][1][k] = (lane & 1) ? b0 : a1;
                    }
                }
        }
        if (!absmax_in) {
            if (plain) {
                float mx[16];
                column_maxima<DT, IT>(raw, held, mx);
                int n[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) n[i] = (nb[i >> 2] >> (8 * (i & 3))) & 0xff;
                if (many) {
                    load8(rep + (g << 4), n);
                    load8(rep + (g << 4) + 8, n + 8);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) consider(mx[i], n[i]);
            }
            reduce_to_red();
        }
        if (!absmax_in) strip_barrier();                       // (1) the wave maxima
        if (absmax_in) set_static(bound);
        else a = max_of_red();
        fill_table();
        strip_barrier();                                       // (2) the table, the tail's sources and flags
        const int nothers = *others;
        if (__builtin_expect(!absmax_in && nothers, 0)) {
            // the other groups, a slot of a row per thread
            best = a;
            bc = 0.0f;
            bn = 1;
            for (int q = tid; q < nothers * 16 * M; q += nprep) {
                const int row = (q >> 4) / nothers, at = list[(q >> 4) - row * nothers] * 16 + (q & 15);
                const int j = src[at], n = rep[at];
                if ((unsigned)j < (unsigned)K && n > 0) consider(fabsf(Elem<DT>::widen(X[(size_t)row * sh.ld + j])), n);
            }
            reduce_to_red();                                   // every wave has read the first maxima before barrier (2)
            strip_barrier();                                   // (2a)
            a = max_of_red();
            fill_table();
            strip_barrier();                                   // (2b)
        }
        if (plain) {
            float m[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) m[i] = table[(nb[i >> 2] >> (8 * (i & 3))) & 0xff];
            if (__builtin_expect(many && a != 0.0f, 0)) {      // beyond the table: one division at a time
#pragma unroll 1
                for (int k = 0; k < 16; ++k) {
                    const int n = rep[(g << 4) + k];
                    if (n < MANY) continue;
                    const float mk = multiplier(n);
#pragma unroll
                    for (int i = 0; i < 16; ++i) m[i] = i == k ? mk : m[i];
                }
            }
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int row = row_of(i);
                if (i < held) {
                    float x[16];
#pragma unroll
                    for (int v = 0; v < NV; ++v) widen16<DT>(raw[i][v], x + v * VEC);
                    const v4u q = quantize16<BITS>(x, m);
                    store_group<BITS>(q, xq, pitch, M, row, g);
                    if constexpr (BITS != 8) *reinterpret_cast<v4u*>(qs + row * qpitch + (g << 4)) = q;
                }
                __builtin_amdgcn_sched_barrier(0);             // rows one by one: mixed, they need more registers than there are
            }
        }
        strip_barrier();                                       // (3) the head's values
        for (int it = tid; it < M * NT; it += nprep) {
            const int row = it / NT, gt = it - row * NT;
            if (!tf[gt]) continue;
            const v4u* tp = reinterpret_cast<const v4u*>(ts + gt * 16);
            store_group<BITS>(gather16(qs + row * qpitch, tp[0], tp[1]), xq, pitch, M, row, NH + gt);
        }
        // the other groups: sixteen lanes gather a group of a row from global memory, a slot each
        for (int it = tid >> 4; it < nothers * M; it += nprep >> 4) {
            const int row = it / nothers, go = list[it - row * nothers], at = go * 16 + (lane & 15);
            const int j = src[at], n = rep[at];
            float x = 0.0f, m = 0.0f;                          // a slot without a channel: 0 whatever X holds
            if ((unsigned)j < (unsigned)K) {
                x = Elem<DT>::widen(X[(size_t)row * sh.ld + j]);
                if (n > 0) m = n < TABLE ? table[n] : (a != 0.0f ? multiplier(n) : 0.0f);
            }
            uint32_t v = (quantized_bits<BITS>(x, m) & 0xffu) << (8 * (lane & 3));
            v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);      // the four bytes of a quad
            v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true);
            if constexpr (BITS == 6) v = e3m2_codes(v);
            v4u q;
#pragma unroll
            for (int i = 0; i < 4; ++i) q[i] = __shfl(v, (lane & 48) + 4 * i, 64);
            if ((lane & 15) == 0) store_group<BITS>(q, xq, pitch, M, row, go);
        }
        strip_barrier();                                       // (4) the quantized rows
        for (int n0 = blockIdx.x * sh.cols; n0 < N; n0 += round) {
            strip_barrier();                                   // (5)
            if (n0 + round < N) strip_barrier();               // (6)
        }
    } else {
        // ---- the weight stream: steps sw, sw + SW, ... of the reduction for 16 FN columns, D ahead ----
        const int r = lane & 15, c = lane >> 4, sw = wave - PW, st = tid - nprep;
        constexpr uint32_t STEP_BYTES = (MODE == MODE_F6) ? 96 : 128;
        const uint32_t stride_w = (MODE == MODE_F6) ? 96u * N : 128u, stride_x = (MODE == MODE_F6) ? 96u * M : 128u;
        const int steps = (int)((rowbytes + STEP_BYTES - 1) / STEP_BYTES);
        const int mine = __builtin_amdgcn_readfirstlane((steps - sw + SW - 1) / SW);
        // The row's last step may be partial.  What a lane loads there is the next row's, or the matrix's last bytes, and meets the
        // zeros that follow a row of xq.  (E3M2 storage has whole steps only.)
        const uint32_t last_w = (uint32_t)((size_t)N * rowbytes - (MODE == MODE_F6 ? 8 : 16));
        RowPieces<MODE> pw[FN], px;
        op_t w[D][FN];
        // (turns: a mask, or all ones.  Wrapped by a comparison instead, layers of every pitch took 1-5 % longer.)
        const uint32_t turns = (uint32_t)sh.turns, from = sw + (sh.turns < 0 ? 0u : blockIdx.x * 5 & turns);
        auto step_of = [&](int t) -> uint32_t { return (from + (uint32_t)(t * SW)) & turns; };
        auto load = [&](int d, int t) {
            const uint32_t s = step_of(t);
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                w[d][j].a = *reinterpret_cast<const decltype(op_t::a)*>(W + min(pw[j].a + s * stride_w, last_w));
                w[d][j].b = *reinterpret_cast<const decltype(op_t::b)*>(W + min(pw[j].b + s * stride_w, last_w));
            }
        };
        auto begin_round = [&](int n0) {
#pragma unroll
            for (int j = 0; j < FN; ++j) pw[j].set(min(n0 + min(16 * j + r, sh.cols - 1), N - 1), c, rowbytes);
        };
        auto load_steps = [&](int from, int to) {
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (d >= from && d < to && d < mine) load(d, d);
        };
        // Before the weights, since loads return in order: the tail's map, eight slots per thread.  A slot's channel goes to 16
        // bits (KQ: none, the slot holds 0 whatever the input) and its copy count to a byte (0: none).
        struct { uint32_t j[4], n[2]; bool bad; } tail = {};
        auto load_tail = [&](int t) {
            int tj[8], tn[8];
            load8(src + KQ + t, tj);
            load8(rep + KQ + t, tn);
            tail.bad = false;
            tail.n[0] = tail.n[1] = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) tail.j[i] = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool none = (unsigned)tj[i] >= (unsigned)K;
                tail.bad = tail.bad || (!none && (tj[i] >= KQ || tn[i] <= 0));
                tail.j[i >> 1] |= min((uint32_t)tj[i], (uint32_t)KQ) << (16 * (i & 1));
                tail.n[i >> 2] |= (none ? 0u : (uint32_t)min(tn[i], MANY) & 0xffu) << (8 * (i & 3));
            }
        };
        // Places in a row of qs from which the slots can be copied; a group can when every slot has none or repeats a channel of
        // a plain group with that channel's own copy count.  The two threads of a group sit in adjacent lanes.
        auto finish_tail = [&](int t) {
            bool copyable = !tail.bad, big = false;
            uint32_t u[4];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t j = (tail.j[i >> 1] >> (16 * (i & 1))) & 0xffffu;
                const uint32_t own = counts8[j], n = (tail.n[i >> 2] >> (8 * (i & 3))) & 0xffu;
                copyable = copyable && own == n;
                big = big || own == MANY;
                const uint32_t at = j == (uint32_t)KQ ? zero_at : j;
                u[i >> 1] = (i & 1) ? u[i >> 1] | (at << 16) : at;
            }
            if (copyable && big) {                             // counts of MANY or more: compared in the map
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t j = (tail.j[i >> 1] >> (16 * (i & 1))) & 0xffffu;
                    copyable = copyable && (j == (uint32_t)KQ || rep[j] == rep[KQ + t + i]);
                }
            }
            *reinterpret_cast<v4u*>(ts + t) = v4u{u[0], u[1], u[2], u[3]};
            const int one = copyable ? 1 : 0, both = one & __shfl_xor(one, 1, 64);
            if ((tid & 1) == 0) {
                tf[t >> 4] = (uint8_t)both;
                if (!both) list[atomicAdd(others, 1)] = (uint16_t)((KQ + t) >> 4);
            }
        };
        if (st * 8 < NT * 16) load_tail(st * 8);
        float bound = 0.0f;
        if (absmax_in) bound = *absmax_in;
        const float sw_scale = s_w ? *s_w : 0.0f;
        // The waves that quantize wait for these at each barrier, and a load waits to be issued while those before it fill the
        // memory pipeline: the weights are asked for in three parts, each enough to keep it busy until the next.
        strip_barrier();                                       // (x)
        begin_round(blockIdx.x * sh.cols);
        constexpr int FIRST = D / 4 > 1 ? D / 4 : 1, SECOND = FIRST + D / 4;
        load_steps(0, FIRST);
        strip_barrier();                                       // (0)
        if (st * 8 < NT * 16) finish_tail(st * 8);
        for (int t = (st + SW * 64) * 8; t < NT * 16; t += SW * 512) {
            load_tail(t);
            finish_tail(t);
        }
        load_steps(FIRST, SECOND);
        if (!absmax_in) strip_barrier();                       // (1)
        load_steps(SECOND, D);
        strip_barrier();                                       // (2)
        if (!absmax_in && *others) {
            strip_barrier();                                   // (2a)
            strip_barrier();                                   // (2b)
        }
        if (absmax_in) set_static(bound);
        else a = max_of_red();
        strip_barrier();                                       // (3)
        strip_barrier();                                       // (4)

        // ---- the product ----
        const float s_x = (a == 0.0f) ? 1.0f : (float)((double)a / (double)QMAX);
        const float scale = s_w ? s_x * sw_scale : 1.0f;
        const bool vec = (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
        px.set(min(r, M - 1), c, MODE == MODE_F6 ? rowbytes : pitch);
        for (int n0 = blockIdx.x * sh.cols; n0 < N; n0 += round) {
            sum_t acc[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[j] = sum_t{0, 0, 0, 0};
            auto compute = [&](int d, int t) {
                const uint32_t s = step_of(t);
                op_t x;
                x.a = *reinterpret_cast<const decltype(op_t::a)*>(xq + (px.a + s * stride_x));
                x.b = *reinterpret_cast<const decltype(op_t::b)*>(xq + (px.b + s * stride_x));
#pragma unroll
                for (int j = 0; j < FN; ++j) multiply<MODE>(w[d][j], x, acc[j]);
            };
            // the conditions are on scalars: the MFMA ignores the execution mask
            for (int t = 0; t < mine; t += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    if (t + d < mine) compute(d, t + d);
                    if (t + D + d < mine) load(d, t + D + d);
                }
            }
            // the next round's first weights travel while this one's partial sums meet
            if (n0 + round < N) {
                begin_round(n0 + round);
                load_steps(0, D);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) part[(sw * FN + j) * 64 + lane] = acc[j];
            strip_barrier();                                   // (5)
            if (st < FN * 64) {
                sum_t sum = {0, 0, 0, 0};
                for (int v = 0; v < SW; v += 4) {
                    sum_t o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = part[min(v + q, SW - 1) * FN * 64 + st];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (v + q < SW) sum += o[q];
                }
                const int in = 16 * (st >> 6) + 4 * c, col = n0 + in;
                if (r < M && in < sh.cols && col < N) store4<MODE>(sum, r, col, N, scale, Y, y_dtype, ldy, bias, vec);
            }
            if (n0 + round < N) strip_barrier();               // (6)
        }
    }
    probe.finish(ticks);
}

typedef void (*few_kernel_t)(const void*, FewShape, const int32_t*, const int32_t*, const float*, const uint8_t*, const float*,
                             const float*, void*, int, int, unsigned long long*);

template <int DT, int MODE, int FN> int few_kernel(few_kernel_t* kern)
{
    static std::atomic<unsigned long long> raised{0};
    *kern = linear_few_kernel<DT, MODE, FN>;
    return set_lds_limit(reinterpret_cast<const void*>(*kern), 160 * 1024, raised);
}
template <int DT, int MODE> int few_kernel_of(int fn, few_kernel_t* kern)
{
    switch (fn) {
    case 1: return few_kernel<DT, MODE, 1>(kern);
    case 2: return few_kernel<DT, MODE, 2>(kern);
    case 3: return few_kernel<DT, MODE, 3>(kern);
    default: return few_kernel<DT, MODE, 4>(kern);
    }
}
template <int DT> int few_kernel_for(int bits, int fn, few_kernel_t* kern)
{
    if (bits == 8) return few_kernel_of<DT, MODE_I8>(fn, kern);
    if (bits == 4) return few_kernel_of<DT, MODE_I4>(fn, kern);
    return few_kernel_of<DT, MODE_F6>(fn, kern);
}

}  // namespace

bool linear_few_fits(int M, int N, int K, int Kpad, int bits, int x_dtype, bool dynamic)
{
    if (bits == FQ_BITS_I4_E3M2 && !quantizer_takes_e3m2(K, Kpad)) return false;
    FewPlan plan;
    return few_plan(M, N, K, 0, Kpad, bits, elem_size(x_dtype), dynamic, compute_units(), &plan);
}

int launch_linear_few(const void* X, int x_dtype, int M, int K, int ld, const int32_t* src, const int32_t* rep, int Kpad, int bits,
                      const float* absmax_in, const void* W, int N, const float* s_w, const float* bias, void* Y, int y_dtype,
                      int ldy, hipStream_t stream)
{
    FewPlan plan;
    if (!few_plan(M, N, K, ld, Kpad, bits, elem_size(x_dtype), absmax_in == nullptr, compute_units(), &plan)) return fail(FQ_ERR_RANGE, "layer not for the kernel for few rows");
    few_kernel_t kern = nullptr;
    const int rc = x_dtype == FQ_F32 ? few_kernel_for<FQ_F32>(bits, plan.fn, &kern)
                 : x_dtype == FQ_F16 ? few_kernel_for<FQ_F16>(bits, plan.fn, &kern) : few_kernel_for<FQ_BF16>(bits, plan.fn, &kern);
    if (rc) return rc;
    kern<<<plan.grid, plan.threads, plan.lds, stream>>>(X, plan.sh, src, rep, absmax_in, static_cast<const uint8_t*>(W), s_w, bias, Y,
                                                        y_dtype, ldy, gemm_ticks_pointer());
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "layer launch failed: %s", hipGetErrorString(e));
    return FQ_OK;
}

}  // namespace fq
