// Flatten + per-tensor quantize kernels (activation path at inference time, weight path offline).
//
// arXiv 2402.17985: Sec. 4.1 Eq. 3 (flatten, equal-split form: each of the n copies of a
// channel holds x/n), Eq. 4 (weight channel repeated), Sec. 2.1 Eq. 1 (per-tensor scale
// s = max|.| / qmax, round, here round-half-even, then clamp).
//
// The kernels, all bandwidth or latency bound:
//   colabsmax           per input channel max|x| over the rows for calibration (64-wide wave reads 1 KiB of a
//                       row per instruction; per-thread running max; one atomic max per column per block;
//                       the max of non-negative floats is taken on their bit patterns, so the
//                       result does not depend on the order of the updates)
//   tensor_absmax       the same pass over X, reduced to one candidate for the per-tensor absmax a' per workgroup
//   flatten_quant_direct  few rows: map, a', multipliers and the quantizer in one kernel (with tensor_absmax before
//                       it when the scale is dynamic and X more than a few rows)
//   scale               many rows: a' from the candidates, the scale s, the per-slot
//                       multiplier m_p = fl32(qmax / (n_p * a')) (float64 quotient), and two flags
//                       per group of 16 slots that tell the quantizer which path a group may take
//   flatten_quant_rows  the quantizer of the equal split: a workgroup owns a strip of rows, reads the
//                       head of the map with vector loads, keeps the quantized bytes in LDS and lets
//                       the appended copies take their values from there
//   flatten_quant       the general form (one thread per 16 slots and strip of rows, every slot
//                       gathered from global memory): the peel split of Eq. 3 as printed, and layers
//                       too wide for the row-strip kernel's LDS budget
#include <algorithm>
#include <atomic>

#include "fq_internal.h"
#include "fq_quant_common.h"
#include "fq_rules.h"

namespace fq {
namespace {

__global__ void fill_u32_kernel(uint32_t* p, int count, uint32_t v)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

// ---------------------------------------------------------------------------------------------
// per input channel absmax
// ---------------------------------------------------------------------------------------------
// Workgroup = 4 waves.  The 64 lanes of a wave cover 64 adjacent 16-byte column groups (1 KiB of a
// row per load); the 4 waves take interleaved rows of the block's row strip, each lane keeping
// eight loads in flight.  The 4 partial maxima
// of a column meet in LDS and one lane issues the atomic max, and only if its value exceeds what the
// column already holds (the stored value only grows, so a stale read can only cause a redundant
// atomic, never a missed one).
// NT: read with the streaming hint (1 GiB 6.4 -> 7.1 TB/s), which leaves nothing of X in the caches.
template <bool NT> __device__ __forceinline__ v4u load16(const void* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(static_cast<const v4u*>(p));
    else return *static_cast<const v4u*>(p);
}
// Running maxima of |X| over the rows r0 + wave, r0 + wave + 4, ... < r1 of the VEC columns from col0 on.
template <int DT, bool NT>
__device__ __forceinline__ void strip_colmax(const typename Elem<DT>::type* __restrict__ X, int K, int ld, int r0, int r1,
                                             int col0, int wave, float (&mx)[Elem<DT>::VEC])
{
    typedef typename Elem<DT>::type T;
    constexpr int VEC = Elem<DT>::VEC, U = ABSMAX_ROUND / 4;
#pragma unroll
    for (int v = 0; v < VEC; ++v) mx[v] = 0.0f;
    if (col0 + VEC <= K) {
        const T* p = X + (size_t)(r0 + wave) * ld + col0;
        const size_t step = (size_t)4 * ld;
        int left = (r1 - r0 - wave + 3) / 4;                     // rows of this wave
        auto round = [&](int n) {                                // n < U: the last one, beyond n the first row again
            v4u raw[U];
#pragma unroll
            for (int q = 0; q < U; ++q) raw[q] = load16<NT>(p + (q < n ? q : 0) * step);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                float f[VEC];
                widen16<DT>(raw[q], f);
#pragma unroll
                for (int v = 0; v < VEC; ++v) mx[v] = fmaxf(mx[v], fabsf(f[v]));
            }
        };
        for (; left >= U; left -= U, p += U * step) round(U);
        if (left > 0) round(left);
    } else if (col0 < K) {
        // Ragged last column group, element by element: a round of loads at once here too, or this lane's chain of single loads, which
        // grows with the strip's height, is what the pass takes (bf16 3000 x 3001 7.6 us, so 5.9; 8192 x 8190 135, so 46).
#pragma unroll 1
        for (int v = 0; v < K - col0; ++v) {
            const T* p = X + (size_t)(r0 + wave) * ld + col0 + v;
            const size_t step = (size_t)4 * ld;
            float m = 0.0f;
#pragma unroll 1
            for (int left = (r1 - r0 - wave + 3) / 4; left > 0; left -= U, p += U * step) {
                T e[U];
#pragma unroll
                for (int q = 0; q < U; ++q) e[q] = p[(q < left ? q : 0) * step];
#pragma unroll
                for (int q = 0; q < U; ++q) m = fmaxf(m, fabsf(Elem<DT>::widen(e[q])));
            }
#pragma unroll
            for (int i = 0; i < VEC; ++i) mx[i] = i == v ? m : mx[i];
        }
    }
}

template <int DT, bool NT>
__global__ __launch_bounds__(256) void colabsmax_kernel(const void* __restrict__ Xv, int M, int K, int ld,
                                                        int rows_per_block, uint32_t* __restrict__ cmax)
{
    constexpr int VEC = Elem<DT>::VEC;
    __shared__ float part[4][64 * VEC];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = blockIdx.y * rows_per_block;
    float mx[VEC];
    strip_colmax<DT, NT>(static_cast<const typename Elem<DT>::type*>(Xv), K, ld, r0, r0 + min(M - r0, rows_per_block),
                     (blockIdx.x * 64 + lane) * VEC, wave, mx);
#pragma unroll
    for (int v = 0; v < VEC; ++v) part[wave][lane * VEC + v] = mx[v];
    __syncthreads();
    // 256 threads finish 64*VEC columns
    for (int c = threadIdx.x; c < 64 * VEC; c += 256) {
        const int col = blockIdx.x * 64 * VEC + c;
        if (col < K) {
            const float m = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
            const uint32_t bits = __float_as_uint(m);
            if (bits > __hip_atomic_load(&cmax[col], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&cmax[col], bits);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// the map, prepared for the quantizer of few rows
// ---------------------------------------------------------------------------------------------
// What flatten_quant_direct_kernel needs of the map, worked out once instead of in each of its workgroups: copy counts of plain
// head groups as bytes (MANY: that many or more; 0 in other groups), sources of the tail's slots as 16-bit channel numbers (KQ:
// the slot holds 0), and per tail group whether each slot holds 0 whatever the input or repeats a channel of a plain group with
// that channel's own copy count.  Lies in the workspace where the general path keeps its multipliers.
constexpr int MANY = 255;
struct PreparedMap {
    uint8_t* counts;      // [KQ]
    uint16_t* sources;    // [16 NT]
    uint8_t* copies;      // [NT]
};
__host__ __device__ __forceinline__ PreparedMap prepared_map(float* mslot, int K, int Kpad)
{
    PreparedMap m;
    m.counts = reinterpret_cast<uint8_t*>(mslot);
    m.sources = reinterpret_cast<uint16_t*>(m.counts + (K & ~15));
    m.copies = reinterpret_cast<uint8_t*>(m.sources + (Kpad - (K & ~15)));
    return m;
}
// Workgroup w of n, 512 threads, a slot each.
__device__ void prepare_map(const int32_t* __restrict__ src, const int32_t* __restrict__ rep, int K, int Kpad, int w, int n, PreparedMap out)
{
    const int KQ = K & ~15, tid = threadIdx.x, lane = tid & 63;
    auto group_all = [&](bool ok) -> bool { return ((__ballot(ok) >> (lane & 48)) & 0xffffull) == 0xffffull; };
    for (int p = w * 512 + tid; p < Kpad; p += n * 512) {       // Kpad and KQ are multiples of 16: groups stay together
        const int j = src[p], c = rep[p];
        if (p < KQ) {
            const bool plain = group_all(j == p && c > 0);
            out.counts[p] = plain ? (uint8_t)min(c, MANY) : (uint8_t)0;
            continue;
        }
        bool ok = (unsigned)j >= (unsigned)K;
        out.sources[p - KQ] = (uint16_t)(ok ? KQ : min(j, KQ));
        if (!ok && j < KQ && c > 0 && rep[j] == c) {
            int sv[16], nv[16];
            const int g0 = j & ~15;
            load8(src + g0, sv);
            load8(src + g0 + 8, sv + 8);
            load8(rep + g0, nv);
            load8(rep + g0 + 8, nv + 8);
            ok = true;
#pragma unroll
            for (int i = 0; i < 16; ++i) ok = ok && sv[i] == g0 + i && nv[i] > 0;
        }
        const bool copies = group_all(ok);
        if ((lane & 15) == 0) out.copies[(p - KQ) >> 4] = copies ? 1 : 0;
    }
}

// ---------------------------------------------------------------------------------------------
// absmax of the flattened tensor, one candidate per workgroup
// ---------------------------------------------------------------------------------------------
// a' = max_p fl32(c_p / n_p) with c_p = max_i |X[i, src p]|.  The rounded quotient is monotonic in c, so the maximum
// over rows may be taken after it: a workgroup that has seen the columns [c0, c0 + 64 VEC) of some rows contributes
// max_j fl32(c_j / n_j), n_j = the smallest copy count of the valid slots that read channel j (channels that no slot reads
// contribute nothing).  Four waves stream X; four more scan the map for n_j meanwhile.  The candidate goes to
// cand[workgroup], and whoever needs a' takes the maximum of the candidates.
// What this replaces: a kernel that cleared K channel maxima, atomic maxima on them, and a gather of all channel maxima
// over the map in every workgroup of the kernel that forms the multipliers.
// ALL: a' = max |X| over all channels, whatever the map (weights, peel split).
// map: when not null, the grid's first row of workgroups prepares the map there and the strips follow.
template <int DT, bool ALL, bool NT>
__global__ __launch_bounds__(ALL ? 256 : 512) void tensor_absmax_kernel(const void* __restrict__ Xv, int M, int K, int ld,
                                                                        int rows_per_block, const int32_t* __restrict__ src,
                                                                        const int32_t* __restrict__ rep, int Kpad,
                                                                        float* __restrict__ cand, float* __restrict__ map)
{
    constexpr int VEC = Elem<DT>::VEC, COLS = 64 * VEC, NONE = 0x7fffffff, NTHR = ALL ? 256 : 512;
    __shared__ float part[4][COLS];
    __shared__ int copies[COLS];
    __shared__ float red[NTHR / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = blockIdx.x * COLS;
    int strip = blockIdx.y;
    if constexpr (!ALL) {
        if (map && strip-- == 0) {
            prepare_map(src, rep, K, Kpad, blockIdx.x, gridDim.x, prepared_map(map, K, Kpad));
            return;
        }
    }
    const int r0 = strip * rows_per_block;
    if constexpr (!ALL) {
        for (int c = tid; c < COLS; c += NTHR) copies[c] = NONE;
        __syncthreads();
    }
    float best = 0.0f;
    if (wave < 4) {
        float mx[VEC];
        strip_colmax<DT, NT>(static_cast<const typename Elem<DT>::type*>(Xv), K, ld, r0, r0 + min(M - r0, rows_per_block),
                         c0 + lane * VEC, wave, mx);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            if constexpr (ALL) best = fmaxf(best, mx[v]);
            else part[wave][lane * VEC + v] = mx[v];
        }
    } else if constexpr (!ALL) {
        // eight loads in flight; Kpad is a multiple of 32, a thread's four slots are inside or outside together
        for (int p = (tid - 256) * 4; p < Kpad; p += 8 * 1024) {
            v4i s[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                s[q] = p + q * 1024 < Kpad ? *reinterpret_cast<const v4i*>(src + p + q * 1024) : v4i{-1, -1, -1, -1};
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = s[q][i] - c0;
                    if ((unsigned)s[q][i] < (unsigned)K && (unsigned)c < (unsigned)COLS) {
                        const int n = rep[p + q * 1024 + i];
                        if (n > 0) atomicMin(&copies[c], n);
                    }
                }
        }
    }
    if constexpr (!ALL) {
        __syncthreads();
        for (int c = tid; c < COLS; c += NTHR) {
            const float m = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
            const int n = copies[c];
            // the float64 quotient rounded to fp32 is the correctly rounded fp32 quotient
            if (n == 1) best = fmaxf(best, m);
            else if (n != NONE) best = fmaxf(best, (float)((double)m / (double)n));
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) best = fmaxf(best, __shfl_xor(best, off, 64));
    if (lane == 0) red[wave] = best;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < NTHR / 64; ++w) best = fmaxf(best, red[w]);
        cand[strip * gridDim.x + blockIdx.x] = best;
    }
}

// ---------------------------------------------------------------------------------------------
// per-tensor absmax, scale and per-slot multipliers (a workgroup per 1024 slots)
// ---------------------------------------------------------------------------------------------
// Every workgroup takes the maximum of the candidates of tensor_absmax_kernel (one load per thread, unless the matrix has
// more than 1024 column blocks; none when the bound is static), tabulates the multipliers m(n) = fl32(qmax / (n * a')) for
// n < 256 in LDS (one float64 division per thread of four waves), and fills its own 1024 slots of mslot.  Workgroup 0 also writes the scale.
constexpr int SCALE_TABLE = 256;
__global__ __launch_bounds__(1024) void scale_kernel(const float* __restrict__ cand, int ncand, int K,
                                                     const int32_t* __restrict__ src,
                                                     const int32_t* __restrict__ rep, int Kpad, int qmax,
                                                     int mode, const float* __restrict__ absmax_in, float T,
                                                     float* __restrict__ mslot, float* __restrict__ scale_out,
                                                     float* __restrict__ scalars, uint8_t* __restrict__ gflag)
{
    __shared__ float red[16];
    __shared__ float table[SCALE_TABLE];
    const int tid = threadIdx.x;
    // the map first: its loads, and those that depend on them, travel while a' is formed
    const int p = blockIdx.x * 1024 + tid;
    const bool inside = p < Kpad, counted = mode != 2;
    const int s = inside ? src[p] : -1, n = inside ? (counted ? rep[p] : 1) : 0;
    // (A map may have fewer slots than there are channels: channel s then has no slot s.)
    const bool has_own = (unsigned)s < (unsigned)min((K >> 4) << 4, Kpad);
    const int own_src = has_own ? src[s] : -1, own_n = has_own ? (counted ? rep[s] : 1) : 0;
    float a;
    if (absmax_in) {
        a = *absmax_in;
        if (!(a >= 0.0f) || a > 3.0e38f) a = 0.0f;     // negative / NaN / Inf static bound: treated as 0
    } else {
        float best = 0.0f;
        for (int c = tid; c < ncand; c += 1024) best = fmaxf(best, cand[c]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) best = fmaxf(best, __shfl_xor(best, off, 64));
        if ((tid & 63) == 0) red[tid >> 6] = best;
        __syncthreads();
        a = red[0];
#pragma unroll
        for (int w = 1; w < 16; ++w) a = fmaxf(a, red[w]);
        if (mode == 3) a = fminf(a, T);
    }
    // Peel split (modes 3 dynamic / 4 static): `rep` carries the slot ordinals e; mslot[p] receives the
    // offset fl32(e * T) that the slot subtracts from |x| (+inf in padding, which clamps to 0), and the
    // single multiplier m = fl32(qmax / a') goes to scalars[2].  a' = min(T, max |X|) when dynamic.
    if (mode >= 3) {
        if (blockIdx.x == 0 && tid == 0) {
            *scale_out = (a == 0.0f) ? 1.0f : (float)((double)a / (double)qmax);
            scalars[0] = a;
            scalars[2] = (a == 0.0f) ? 0.0f : (float)((double)qmax / (double)a);
        }
        if (inside) mslot[p] = (unsigned)s < (unsigned)K && n >= 0 ? (float)n * T : __builtin_inff();      // n: the ordinal e
        return;
    }
    const double ad = (double)a;
    if (blockIdx.x == 0 && tid == 0) {
        *scale_out = (a == 0.0f) ? 1.0f : (float)(ad / (double)qmax);
        scalars[0] = a;
    }
    if (tid < SCALE_TABLE) table[tid] = (tid > 0 && a != 0.0f) ? (float)((double)qmax / ((double)tid * ad)) : 0.0f;
    __syncthreads();
    if (inside) {
        const bool valid = (unsigned)s < (unsigned)K && n > 0 && a != 0.0f;
        float m = 0.0f;
        if (valid) m = (n < SCALE_TABLE) ? table[n] : (float)((double)qmax / ((double)n * ad));
        mslot[p] = m;
    }
    // gflag[g] = 1 when the 16 slots of group g are the 16 channels at the same indices (the head of
    // the map): such a group is read with vector loads and its quantized values can be copied by the
    // appended slots that repeat its channels
    const bool ident = inside && p < K && s == p;
    const unsigned long long bal = __ballot(ident);
    if (p < Kpad && (tid & 15) == 0) gflag[p >> 4] = (((bal >> (tid & 48)) & 0xffffull) == 0xffffull) ? 1 : 0;
    // cflag[g] = 1 when every slot of group g either holds 0 whatever the input (padding) or repeats a
    // channel j < 16 * (K / 16) whose own slot j is the identity slot with the same copy count: the
    // slot's quantized value then equals slot j's and can be copied instead of recomputed.
    const bool copyable = inside && ((unsigned)s >= (unsigned)K || (own_src == s && n > 0 && own_n == n));
    const unsigned long long balc = __ballot(copyable);
    uint8_t* cflag = gflag + ((Kpad >> 4) + 1);
    if (p < Kpad && (tid & 15) == 0) cflag[p >> 4] = (((balc >> (tid & 48)) & 0xffffull) == 0xffffull) ? 1 : 0;
}

// ---------------------------------------------------------------------------------------------
// flatten + quantize
// ---------------------------------------------------------------------------------------------
// LDS of flatten_quant_direct_kernel before the strip itself: the table of multipliers and the wave maxima.  A plain group's
// copy counts are kept as bytes; MANY stands for MANY copies or more, whose count is read from the map where it matters.
constexpr int DIRECT_TABLE = 256, DIRECT_RED = 16;
constexpr int DIRECT_LDS_FIXED = (DIRECT_TABLE + DIRECT_RED) * 4;

// PEEL = false: slot value x * m_p (equal split; m_p from mslot).  PEEL = true: the printed split of
// Eq. 3, slot value sign(x) * clamp(|x| - t_p, 0, thr) times the single multiplier scalars[2], with the
// offsets t_p in mslot.
template <int DT, int BITS, bool PEEL = false>
__global__ __launch_bounds__(256) void flatten_quant_kernel(const void* __restrict__ Xv, int M, int K, int ld,
                                                            const int32_t* __restrict__ src,
                                                            const float* __restrict__ mslot, int Kpad,
                                                            int rows_per_thread, uint8_t* __restrict__ out,
                                                            const float* __restrict__ scalars = nullptr,
                                                            float thr = 0.0f)
{
    typedef typename Elem<DT>::type T;
    constexpr int VEC = Elem<DT>::VEC;
    const T* X = static_cast<const T*>(Xv);
    const int G = Kpad >> 4;                                   // groups of 16 slots per row
    // Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  Remap them so that
    // consecutive logical workgroups (the head and the gathered tail of the same rows) share an XCD:
    // the tail's gathers then hit the lines the head has just brought into that L2.
    const unsigned nwg = gridDim.x, wg = blockIdx.x;
    const unsigned q = nwg >> 3, rem = nwg & 7, xcd = wg & 7, idx = wg >> 3;
    const unsigned lwg = (xcd < rem) ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
    const long long gid = (long long)lwg * 256 + threadIdx.x;
    const int g = (int)(gid % G);
    const long long rt = gid / G;
    const long long r0l = rt * rows_per_thread;
    if (r0l >= M) return;
    const int r0 = (int)r0l;
    const int r1 = min(M, r0 + rows_per_thread);
    const int p0 = g << 4;

    int s[16];
    float m[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v4i sv = *reinterpret_cast<const v4i*>(src + p0 + 4 * i);
        v4f mv = *reinterpret_cast<const v4f*>(mslot + p0 + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) { s[4 * i + j] = sv[j]; m[4 * i + j] = mv[j]; }
    }
    bool contig = (s[0] >= 0) && (s[0] % VEC == 0) && (s[0] + 15 < K);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if ((unsigned)s[i] >= (unsigned)K) {
            s[i] = 0;
            m[i] = PEEL ? __builtin_inff() : 0.0f;
            contig = false;
        }
        if (s[i] != s[0] + i) contig = false;
    }

    float mq = 0.0f;
    if constexpr (PEEL) mq = scalars[2];
    const size_t orow_bytes = (BITS == 8) ? (size_t)Kpad : (size_t)(Kpad >> 1);
    uint8_t* o = out + (size_t)r0 * orow_bytes + ((BITS == 8) ? p0 : (p0 >> 1));
    const T* row = X + (size_t)r0 * ld;

#pragma unroll 4
    for (int r = r0; r < r1; ++r, row += ld, o += orow_bytes) {
        float x[16];
        if (contig) {
            const v4u* vp = reinterpret_cast<const v4u*>(row + s[0]);
#pragma unroll
            for (int i = 0; i < 16 / VEC; ++i) {
                v4u raw = vp[i];
                widen16<DT>(raw, x + i * VEC);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                x[i] = Elem<DT>::widen(row[s[i]]);
                if constexpr (!PEEL) x[i] = gathered(x[i]);
            }
        }
        if constexpr (PEEL) {
            float mult[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float mag = fminf(fmaxf(fabsf(x[i]) - m[i], 0.0f), thr);
                x[i] = x[i] < 0.0f ? -mag : mag;
                mult[i] = mq;
            }
            store16<BITS>(quantize16<BITS>(x, mult), o);
        } else {
            store16<BITS>(quantize16<BITS>(x, m), o);
        }
    }
}


// ---------------------------------------------------------------------------------------------
// flatten + quantize, row-strip form (the equal split)
// ---------------------------------------------------------------------------------------------
// A workgroup owns a strip of R rows.  Phase 1: each thread takes groups among the first K/16 (the
// head of the map): a group whose 16 slots are the 16 channels at the same indices (gflag) is read
// with vector loads, otherwise gathered; multiply, round, clamp, pack, store, and the quantized value
// of every identity slot also goes to LDS as a byte, q[row][channel].  Phase 2: the remaining groups
// (appended copies and padding), one (group, row) item at a time over all threads.  An appended slot
// with the same copy count as its channel's identity slot holds the same quantized value, so a group
// made of such slots and padding (cflag) is copied from LDS; any other group is gathered from global
// memory and quantized with its own multipliers.
// (ROW_PAD: a row in LDS is followed by a byte that is 0, the source of padding slots.)
constexpr int ROW_PAD = 16;

template <int DT, int BITS>
__global__ __launch_bounds__(512) void flatten_quant_rows_kernel(const void* __restrict__ Xv, int M, int K, int ld,
                                                                 const int32_t* __restrict__ src,
                                                                 const float* __restrict__ mslot,
                                                                 const uint8_t* __restrict__ gflag, int Kpad, int R,
                                                                 uint8_t* __restrict__ out)
{
    typedef typename Elem<DT>::type T;
    constexpr int VEC = Elem<DT>::VEC;
    extern __shared__ __align__(16) uint8_t lds[];
    const T* X = static_cast<const T*>(Xv);
    const int NH = K >> 4;                                     // groups of the head
    const int KQ = NH << 4;
    const int G = Kpad >> 4;
    const int NT = G - NH;                                     // groups of phase 2
    const int pitch = KQ + ROW_PAD;
    uint8_t* qs = lds;                                         // [R][pitch], a byte per value; byte KQ of a row is 0
    uint16_t* ts = reinterpret_cast<uint16_t*>(lds + (size_t)R * pitch);   // sources of the phase-2 slots
    uint8_t* tf = lds + (size_t)R * pitch + (size_t)NT * 32;               // copy flags of the phase-2 groups
    const uint8_t* cflag = gflag + (G + 1);
    const int r0 = blockIdx.x * R;
    const int nthr = blockDim.x;
    const int nr = min(M - r0, R);
    // bytes of an output row: 16 (INT8) or 8 (nibbles) per group of 16 slots (E3M2 has its own addressing, see store16_e3m2)
    const size_t orow_bytes = (size_t)G * (BITS == 8 ? 16 : 8);
    if ((int)threadIdx.x < R) qs[(size_t)threadIdx.x * pitch + KQ] = 0;

    // sources of the phase-2 slots as 16-bit channel numbers (KQ: the slot holds 0); eight slots per
    // thread and pass, loaded before any is stored, so that the passes do not each wait a round trip
    for (int t = threadIdx.x * 8; t < NT * 16; t += nthr * 8) {
        const v4i a = *reinterpret_cast<const v4i*>(src + KQ + t);
        const v4i b = *reinterpret_cast<const v4i*>(src + KQ + t + 4);
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j0 = (i < 2) ? a[2 * i] : b[2 * i - 4], j1 = (i < 2) ? a[2 * i + 1] : b[2 * i - 3];
            const uint32_t lo = min((uint32_t)j0, (uint32_t)KQ), hi = min((uint32_t)j1, (uint32_t)KQ);     // -1 is the largest
            w[i] = lo | (hi << 16);
        }
        *reinterpret_cast<v4u*>(ts + t) = v4u{w[0], w[1], w[2], w[3]};
    }
    for (int t = threadIdx.x; t < NT; t += nthr) tf[t] = cflag[NH + t];

    // the general form of one group over rows [ra, rb) of the strip: every slot's source element is
    // gathered from global memory; identity slots of the head also leave their value in LDS
    auto gather_group = [&](int g, int ra, int rb, bool to_lds) {
        const int p0 = g << 4;
        int s[16];
        float m[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v4i sv = *reinterpret_cast<const v4i*>(src + p0 + 4 * i);
            v4f mv = *reinterpret_cast<const v4f*>(mslot + p0 + 4 * i);
#pragma unroll
            for (int j = 0; j < 4; ++j) { s[4 * i + j] = sv[j]; m[4 * i + j] = mv[j]; }
        }
        bool ident[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            ident[i] = to_lds && s[i] == p0 + i;
            if ((unsigned)s[i] >= (unsigned)K) { s[i] = 0; m[i] = 0.0f; }
        }
        const T* row = X + (size_t)(r0 + ra) * ld;
        for (int r = ra; r < rb; ++r, row += ld) {
            float x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = gathered(Elem<DT>::widen(row[s[i]]));
            const v4u q = quantize16<BITS>(x, m);
            store_group<BITS>(q, out, orow_bytes, M, r0 + r, g);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (ident[i]) qs[(size_t)r * pitch + p0 + i] = (uint8_t)(q[i >> 2] >> (8 * (i & 3)));
        }
    };

    // ---- phase 1: the head ----
    for (int g = threadIdx.x; g < NH; g += nthr) {
        if (!gflag[g]) {
            gather_group(g, 0, nr, true);
            continue;
        }
        const int p0 = g << 4;
        float m[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v4f mv = *reinterpret_cast<const v4f*>(mslot + p0 + 4 * i);
#pragma unroll
            for (int j = 0; j < 4; ++j) m[4 * i + j] = mv[j];
        }
        const T* row = X + (size_t)r0 * ld + p0;
        uint8_t* ql = qs + p0;
#pragma unroll 4
        for (int r = 0; r < nr; ++r, row += ld, ql += pitch) {
            float x[16];
#pragma unroll
            for (int i = 0; i < 16 / VEC; ++i) widen16<DT>(*reinterpret_cast<const v4u*>(row + i * VEC), x + i * VEC);
            const v4u q = quantize16<BITS>(x, m);
            store_group<BITS>(q, out, orow_bytes, M, r0 + r, g);
            *reinterpret_cast<v4u*>(ql) = q;
        }
    }
    __syncthreads();

    // ---- phase 2: appended copies and padding, (group, row) items over all threads, two per thread
    //      and pass with the LDS reads of both issued before either is packed ----
    constexpr int U = 2;
    const int items = NT * nr;
    for (int it0 = threadIdx.x; it0 < items; it0 += nthr * U) {
        int gt[U], rr[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int it = it0 + u * nthr;
            const bool valid = it < items;
            gt[u] = valid ? it % NT : 0;
            rr[u] = valid ? it / NT : 0;
            const uint8_t cf = valid ? tf[gt[u]] : (uint8_t)1;
            ok[u] = valid && cf != 0;
            if (valid && cf == 0) gather_group(NH + gt[u], rr[u], rr[u] + 1, false);
        }
        v4u t0[U], t1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const v4u* tp = reinterpret_cast<const v4u*>(ts + gt[u] * 16);
            t0[u] = tp[0];
            t1[u] = tp[1];
        }
        v4u q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) q[u] = gather16(qs + (size_t)rr[u] * pitch, t0[u], t1[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ok[u]) store_group<BITS>(q[u], out, orow_bytes, M, r0 + rr[u], NH + gt[u]);
    }
}

// ---------------------------------------------------------------------------------------------
// flatten + quantize of an activation of few rows (the equal split)
// ---------------------------------------------------------------------------------------------
// The same two phases as the row-strip kernel, but nothing is prepared in kernels of their own: at these sizes a call is
// bound by its launches (each 4-8 us) and not by bytes.  A workgroup owns a run of rows, which it walks in strips of R,
// and has one thread per P head groups, so that a strip is one round of loads.
//   loads      X of the first strip, the map (head and tail) and the bound or the candidates are asked for at once: what
//              follows waits one round trip to memory for all of them.
//   the map    with a dynamic scale from the absmax pass, which prepares it (PreparedMap: a byte per slot instead of eight, and no checks;
//              500 x 11008 9.6 -> 7.8 us, 2048 x 4096 10.8 -> 9.5); else thread t reads the sources and copy counts of its groups t,
//              t + head threads, ... of the head.  A group is plain when its slots are the channels at the same indices with copies;
//              the counts of plain groups are left in LDS, and from them follows which appended groups only repeat their values.
//              (Counts beyond the table are rare and divide once per slot.  Gathering their groups and copies element by element
//              took 18.0 us for 1000 x 4096 static with one channel of 300 copies and 25.6 with 2000; this 8.7 and 11.8.)
//   a'         the static bound; or the maximum of the candidates that tensor_absmax_kernel left; or (few rows) taken
//              from all of X by every workgroup, which costs M * K reads from L2 against a launch: its threads then form
//              several slots of head threads, each with its share of the rows, so that the reads are one round trip.
//   strips     phase 1 quantizes the plain head groups from registers, phase 2 copies appended slots out of LDS; any
//              other group is gathered slot by slot.  The next strip is read before phase 2.
// A kernel that only loads and stores takes 2.0 us here; of the rest about half is loads, half the instructions of a wave that
// has its SIMD to itself (1.5 ns each).  Whole call before / with one round of loads, unconditional look-ups, divisions on the
// host and quantize16, us: 77 x 5120 fp16 static 6.3 / 5.1, 1000 x 4096 static 8.2 / 6.7, 16 x 4096 dynamic 8.3 / 7.7, 500 x
// 11008 dynamic 18.3 / 16.5, 1024 x 11008 22.7 / 20.3.  (The map by four slots per lane, whole lines per instruction, was slower:
// 1000 x 4096 7.8.)
template <int DT, int BITS, int P, int R>
__global__ __launch_bounds__(1024) void flatten_quant_direct_kernel(const void* __restrict__ Xv, int M, int K, int ld,
                                                                    const int32_t* __restrict__ src,
                                                                    const int32_t* __restrict__ rep, int Kpad,
                                                                    const float* __restrict__ absmax_in,
                                                                    const float* __restrict__ cand, int ncand,
                                                                    float* __restrict__ scale_out,
                                                                    float* __restrict__ scalars, uint8_t* __restrict__ out,
                                                                    int rows_each, int rows_more, int slots, float* __restrict__ map)
{
    typedef typename Elem<DT>::type T;
    constexpr int VEC = Elem<DT>::VEC, NV = 16 / VEC;
    constexpr int QMAX = (BITS == 8) ? 127 : 7;
    // the tail of the map is asked for with the rest where that fits the registers (fp32 2000 x 4096 static to INT8: with it, and scratch, 18.3 us;
    // without 13.1)
    constexpr bool TAIL_EARLY = DT != FQ_F32 && P == 1;
    const int nthr = blockDim.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = nthr >> 6;
    extern __shared__ __align__(16) uint8_t lds[];
    const T* X = static_cast<const T*>(Xv);
    const int NH = K >> 4;                                     // groups of the head
    const int KQ = NH << 4;
    const int G = Kpad >> 4;
    const int NT = G - NH;                                     // groups of phase 2
    const int pitch = KQ + ROW_PAD;
    float* table = reinterpret_cast<float*>(lds);              // [DIRECT_TABLE] m(n) = fl32(qmax / (n a'))
    float* red = table + DIRECT_TABLE;                         // [DIRECT_RED]
    uint8_t* counts8 = lds + DIRECT_LDS_FIXED;                 // [pitch] copy counts of the plain groups, 0 elsewhere
    uint8_t* qs = counts8 + pitch;                             // [R][pitch], a byte per value; byte KQ of a row is 0
    uint16_t* ts = reinterpret_cast<uint16_t*>(qs + (size_t)R * pitch);    // sources of the phase-2 slots
    uint8_t* tf = qs + (size_t)R * pitch + (size_t)NT * 32;                // copy flags of the phase-2 groups
    // rows_each rows per workgroup, one more in the first rows_more (from the host: a division here takes 0.3 us)
    const int wg = blockIdx.x, row_begin = wg * rows_each + min(wg, rows_more), row_end = row_begin + rows_each + (wg < rows_more ? 1 : 0);
    // the threads of one slot cover the head; slot 0 quantizes it, the others help with a' and with phase 2
    const int head_waves = (NH + 64 * P - 1) / (64 * P), head = head_waves << 6;
    int slot = 0;
    for (int w = wave; w >= head_waves; w -= head_waves) ++slot;
    const int t0 = tid - slot * head;
    const bool first = slot == 0;

    // the head groups of a strip of X; every row index is below row_end, every group inside the row
    v4u raw[P][R][NV];
    auto load_strip = [&](int rs) {
        if (!first) return;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int g = t0 + p * head;
            if (g < NH) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (rs + r < row_end) {
                        const v4u* vp = reinterpret_cast<const v4u*>(X + (size_t)(rs + r) * ld + (g << 4));
#pragma unroll
                        for (int i = 0; i < NV; ++i) raw[p][r][i] = vp[i];
                    }
            }
        }
    };

    // copy counts of eight slots (weights: no counts, every slot a plain copy)
    const int32_t* counts = rep ? rep : src;
    const bool counted = rep != nullptr;
    auto load_counts = [&](int p, int* n) {
        load8(counts + p, n);
#pragma unroll
        for (int i = 0; i < 8; ++i) n[i] = counted ? n[i] : 1;
    };
    // sources and copy counts of a group's 16 slots
    auto load_slots = [&](int p0, int (&sv)[16], int (&nv)[16]) {
        load8(src + p0, sv);
        load8(src + p0 + 8, sv + 8);
        load_counts(p0, nv);
        load_counts(p0 + 8, nv + 8);
    };

    // ---- the loads ----
    float best = 0.0f;
    if (absmax_in) best = *absmax_in;
    // With two head groups per thread what is live at once decides whether registers go to scratch (up to 80 bytes per lane): gathered
    // groups are taken in halves, fp32 rows two at a time for the maximum, and fp32 reads the map of its groups one after the other.
    // Static, us, before / so: fp32 to INT8 200 x 25000 15.5 / 12.5, 300 x 30000 24.0 / 18.1; bf16 to E3M2 400 x 20480 15.5 / 12.9.
    constexpr bool MAP_EARLY = DT != FQ_F32 || P == 1;
    int sv[MAP_EARLY ? P : 1][16], nv[MAP_EARLY ? P : 1][16];
    int tj[8], tn[8];
    uint32_t nb[P][4];                                         // copy counts of this thread's plain groups, as bytes
    const PreparedMap pm = prepared_map(map, K, Kpad);
    if (map) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            v4u n = {0, 0, 0, 0};
            if (t0 + p * head < NH) n = *reinterpret_cast<const v4u*>(pm.counts + ((t0 + p * head) << 4));
#pragma unroll
            for (int i = 0; i < 4; ++i) nb[p][i] = n[i];
        }
    } else {
        if constexpr (MAP_EARLY) {
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (t0 + p * head < NH) load_slots((t0 + p * head) << 4, sv[p], nv[p]);
        }
        // eight slots of the tail per thread and pass, the first pass now; the two threads of a group sit in adjacent lanes
        if (TAIL_EARLY && tid * 8 < NT * 16) {
            load8(src + KQ + tid * 8, tj);
            load_counts(KQ + tid * 8, tn);
        }
    }
    load_strip(row_begin);
    if (cand) {                                                // at most 1024 unless K is beyond 2^18: four per thread and pass
        for (int c = tid * 4; c < ncand; c += nthr * 16) {
            v4f v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = c + q * nthr * 4;
                v[q] = at < ncand ? *reinterpret_cast<const v4f*>(cand + at) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int i = 1; i < 4; ++i) v[q][i] = at + i < ncand ? v[q][i] : 0.0f;     // beyond the candidates: not written
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) best = fmaxf(fmaxf(best, fmaxf(v[q][0], v[q][1])), fmaxf(v[q][2], v[q][3]));
        }
    }
    if (tid <= R) counts8[(size_t)tid * pitch + KQ] = 0;       // also of the rows of qs, which follow
    float a = 0.0f;
    auto multiplier = [&](int n) -> float { return (float)((double)QMAX / ((double)n * (double)a)); };
    auto fill_table = [&]() {
        for (int n = tid; n < DIRECT_TABLE; n += nthr) table[n] = (n > 0 && a != 0.0f) ? multiplier(n) : 0.0f;
    };
    if (absmax_in) {
        a = best;
        if (!(a >= 0.0f) || a > 3.0e38f) a = 0.0f;             // negative / NaN / Inf static bound: treated as 0
        fill_table();
    }

    // ---- the map ----
    int plain = 0, many = 0;                                   // groups of this thread: plain; with a count of MANY
    bool other = false;                                        // a group that is neither plain nor copies of plain ones
    if (map) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if ((nb[p][0] & 0xff) == 0) continue;
            plain |= 1 << p;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (((nb[p][i >> 2] >> (8 * (i & 3))) & 0xff) == MANY) many |= 1 << p;
        }
        // the tail's sources and flags to LDS
        for (int t = tid * 8; t < NT * 16; t += nthr * 8) *reinterpret_cast<v4u*>(ts + t) = *reinterpret_cast<const v4u*>(pm.sources + t);
        for (int t = tid; t < NT; t += nthr) tf[t] = pm.copies[t];
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int g = t0 + p * head;
#pragma unroll
            for (int i = 0; i < 4; ++i) nb[p][i] = 0;
            if (g < NH) {
                const int e = MAP_EARLY ? p : 0;
                if constexpr (!MAP_EARLY) load_slots(g << 4, sv[0], nv[0]);
                int differ = 0, least = nv[e][0], most = nv[e][0];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    differ |= sv[e][i] ^ ((g << 4) + i);
                    least = min(least, nv[e][i]);
                    most = max(most, nv[e][i]);
                }
                if (differ == 0 && least > 0) {
                    plain |= 1 << p;
                    if (most >= MANY) many |= 1 << p;
#pragma unroll
                    for (int i = 0; i < 16; ++i) nb[p][i >> 2] |= (uint32_t)min(nv[e][i], MANY) << (8 * (i & 3));
                } else {
                    other = true;
                }
                if (first) *reinterpret_cast<v4u*>(counts8 + (g << 4)) = v4u{nb[p][0], nb[p][1], nb[p][2], nb[p][3]};
            }
        }
    }
    // a' from all of X (few rows): the plain groups' part.  Rounding is monotonic, so the largest element is divided.
    const bool self = !absmax_in && !cand;
    // Of several copies the largest exact quotient |x| / n, compared by cross multiplication in float64 (exact for n < 2^29)
    // and divided once; few channels have them, most waves none at a given place of their groups.
    float bc = 0.0f;
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
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) best = fmaxf(best, __shfl_xor(best, off, 64));
        if (lane == 0) red[wave] = best;
    };
    auto max_of_red = [&]() -> float {
        float v = red[0];
#pragma unroll
        for (int w = 1; w < DIRECT_RED; ++w) v = (w < waves) ? fmaxf(v, red[w]) : v;
        return v;
    };
    if (self) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (!((plain >> p) & 1)) continue;
            constexpr int U = DT == FQ_F32 && P == 2 ? 2 : 4;     // rows in flight
            float mx[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) mx[i] = 0.0f;
            const T* xp = X + ((t0 + p * head) << 4);
            auto take = [&](const v4u (&in)[NV]) {
                float x[16];
#pragma unroll
                for (int i = 0; i < NV; ++i) widen16<DT>(in[i], x + i * VEC);
#pragma unroll
                for (int i = 0; i < 16; ++i) mx[i] = fmaxf(mx[i], fabsf(x[i]));
            };
            // What is left over is read by itself: one row, of fp32 two, one after the other (read four at a time: fp32 1 x 20480 15.4 us,
            // so 12.9; 2 x 11008 10.1, so 8.9)
            constexpr int ALONE = DT == FQ_F32 && U == 4 ? 2 : 1;
            int r = slot;
            for (; r + ALONE * slots < M; r += U * slots) {
                v4u in[U][NV];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const T* xr = xp + (size_t)min(r + u * slots, M - 1) * ld;      // beyond the last row: that one again
#pragma unroll
                    for (int i = 0; i < NV; ++i) in[u][i] = reinterpret_cast<const v4u*>(xr)[i];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) take(in[u]);
            }
#pragma unroll 1
            for (; r < M; r += slots) {
                v4u in[NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) in[i] = reinterpret_cast<const v4u*>(xp + (size_t)r * ld)[i];
                take(in);
            }
            int n[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) n[i] = (nb[p][i >> 2] >> (8 * (i & 3))) & 0xff;
            if ((many >> p) & 1) {
                load_counts((t0 + p * head) << 4, n);
                load_counts(((t0 + p * head) << 4) + 8, n + 8);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) consider(mx[i], n[i]);
        }
        best = fmaxf(best, (float)((double)bc / (double)bn));
    }
    // A ragged head leaves channels that only a gathered group has: the maxima are reduced once, with that group's.  (Reduced before
    // and after it: 8 x 2500 bf16 dynamic 10.9 us, 40 x 2500 14.3; once 10.2 and 13.3.)
    const bool late = self && KQ != K;
    if (!absmax_in && !late) reduce_to_red();
    __syncthreads();
    if (!absmax_in && !late) {
        a = max_of_red();
        fill_table();
    }
    // Sources of the phase-2 slots as 16-bit channel numbers (KQ: the slot holds 0) and, per group, whether every
    // slot holds 0 whatever the input or repeats a channel of a plain group with that channel's own copy count.
    for (int t = tid * 8; !map && t < NT * 16; t += nthr * 8) {
        if (!TAIL_EARLY || t != tid * 8) {
            load8(src + KQ + t, tj);
            load_counts(KQ + t, tn);
        }
        bool copyable = true, big = false;
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t j = min((uint32_t)tj[i], (uint32_t)KQ);
            const int own = counts8[j];
            copyable = copyable && ((unsigned)tj[i] >= (unsigned)K || (own != 0 && min(tn[i], MANY) == own));
            big = big || own == MANY;
            w[i >> 1] |= j << (16 * (i & 1));
        }
        if (copyable && big) {                                     // counts of MANY or more: compared with the map's
            int c[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) c[i] = counts[(unsigned)tj[i] < (unsigned)KQ ? tj[i] : 0];
#pragma unroll
            for (int i = 0; i < 8; ++i) copyable = copyable && ((unsigned)tj[i] >= (unsigned)KQ || tn[i] == c[i]);
        }
        *reinterpret_cast<v4u*>(ts + t) = v4u{w[0], w[1], w[2], w[3]};
        const int mine = copyable ? 1 : 0, both = mine & __shfl_xor(mine, 1, 64);
        if ((tid & 1) == 0) tf[t >> 4] = (uint8_t)both;
        other = other || !both;
    }
    if (self) {
        // the slots of every other group (head groups that are not plain, appended groups that do not repeat plain
        // ones), one by one; plain groups and their copies have been seen above
        const bool others = __syncthreads_or(other ? 1 : 0) != 0;
        if (others || late) {
            bc = 0.0f;
            bn = 1;
            for (int q = tid; others && q < G * 16; q += nthr) {
                const int g = q >> 4;
                const bool seen = g < NH ? counts8[g << 4] != 0 : tf[g - NH] != 0;
                if (seen) continue;
                const int j = src[q], n = counted ? rep[q] : 1;
                if ((unsigned)j >= (unsigned)K || n <= 0) continue;
                float mx = 0.0f;
#pragma unroll 8
                for (int r = 0; r < M; ++r) mx = fmaxf(mx, fabsf(Elem<DT>::widen(X[(size_t)r * ld + j])));
                consider(mx, n);
            }
            best = fmaxf(best, (float)((double)bc / (double)bn));
            reduce_to_red();                                   // every thread has read the first maxima before the barrier above
            __syncthreads();
            a = max_of_red();
            fill_table();
            __syncthreads();
        }
    } else if (!absmax_in) {
        __syncthreads();
    }
    if (blockIdx.x == 0 && tid == 0) {
        *scale_out = (a == 0.0f) ? 1.0f : (float)((double)a / (double)QMAX);
        scalars[0] = a;
    }

    // ---- the multipliers ----
    float m[P][16];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < 16; ++i) m[p][i] = table[(nb[p][i >> 2] >> (8 * (i & 3))) & 0xff];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (!((many >> p) & 1) || a == 0.0f) continue;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (((nb[p][i >> 2] >> (8 * (i & 3))) & 0xff) == MANY) m[p][i] = multiplier(counts[((t0 + p * head) << 4) + i]);
    }

    // bytes of an output row: 16 (INT8) or 8 (nibbles) per group of 16 slots (E3M2 has its own addressing, see store16_e3m2)
    const size_t orow_bytes = (size_t)G * (BITS == 8 ? 16 : 8);
    // one group of one row in its general form: every slot's source element gathered from global memory
    auto gather_group = [&](int g, int row) {
        const T* xr = X + (size_t)row * ld;
        constexpr int U = P == 1 ? 16 : 8;                     // slots at a time
        v4u q = {0, 0, 0, 0};
#pragma unroll 1
        for (int h = 0; h < 16; h += U) {
            int s[U], n[U];
            float x[U], mult[U];
#pragma unroll
            for (int i = 0; i < U; i += 8) {
                load8(src + (g << 4) + h + i, s + i);
                load_counts((g << 4) + h + i, n + i);
            }
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const bool in = (unsigned)s[i] < (unsigned)K;         // a slot without a channel: 0 whatever X holds
                const float xs = Elem<DT>::widen(xr[in ? s[i] : 0]);
                x[i] = in ? xs : 0.0f;
                mult[i] = 0.0f;
                if (in && n[i] > 0) mult[i] = n[i] < DIRECT_TABLE ? table[n[i]] : (a != 0.0f ? multiplier(n[i]) : 0.0f);
            }
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (U == 16 || (w >> 1) == (h >> 3)) q[w] = quantize4<BITS>(x + 4 * w % U, mult + 4 * w % U);
        }
        store_group<BITS>(q, out, orow_bytes, M, row, g);
    };

    // head groups of this thread that are not plain
    int slow = 0;
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (first && t0 + p * head < NH && !((plain >> p) & 1)) slow |= 1 << p;

    // phase 2: a wave takes 64 groups of a row, or (few appended groups) all groups of two to eight rows, a batch.  The group with the
    // channels of a ragged head is gathered in every row.  Where waves have several batches a lane keeps what it is to gather for the
    // strip's end, and groups move on by a lane per row so that lanes differ: one gather and not one per batch.  Nibbles, fp16, 600 x
    // 1003 static 8.9 us, so 7.6; 4680 x 1003 11.7, 10.1; dynamic 18.5, 15.9.  With one batch per wave nothing is kept (INT8 600 x 1003 7.0,
    // kept 7.3).
    const int tail_waves = (NT + 63) >> 6, tail_log = NT <= 8 ? 3 : NT <= 16 ? 2 : NT <= 32 ? 1 : 0;
    const bool later = R == 4 && KQ != K && tail_waves * (R >> min(tail_log, 2)) > waves;
    for (int rs = row_begin; rs < row_end; rs += R) {
        const int nr = min(row_end - rs, R);
        // ---- phase 1: the head ----
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int g = t0 + p * head;
            if (first && ((plain >> p) & 1)) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (r < nr) {
                        float x[16];
#pragma unroll
                        for (int i = 0; i < NV; ++i) widen16<DT>(raw[p][r][i], x + i * VEC);
                        const v4u q = quantize16<BITS>(x, m[p]);
                        store_group<BITS>(q, out, orow_bytes, M, rs + r, g);
                        *reinterpret_cast<v4u*>(qs + (size_t)r * pitch + (g << 4)) = q;
                    }
            }
        }
        load_strip(rs + R);
        strip_barrier();

        // ---- this thread's head groups that are not plain; then phase 2, appended copies and padding (one row per
        //      wave whatever NT took 9000 x 300 static from 12.1 to 18.4 us) ----
        for (int k = 0; slow && k < P * nr; ++k)
            if ((slow >> (k / nr)) & 1) gather_group(t0 + (k / nr) * head, rs + k % nr);
        int kept = -1;                                         // group to be gathered: row << 20 | group
        for (int rb = 0, w = wave;; w += waves) {
            for (; rb < nr && w >= tail_waves; w -= tail_waves) rb += 1 << tail_log;
            if (rb >= nr) break;
            const int rr = rb + (lane >> (6 - tail_log)), gt = w * 64 + ((lane + (R == 4 ? rb : 0)) & ((64 >> tail_log) - 1));
            if (rr >= nr || gt >= NT) continue;
            if (!tf[gt]) {
                if (later && kept < 0) kept = rr << 20 | gt;
                else gather_group(NH + gt, rs + rr);
                continue;
            }
            const v4u* tp = reinterpret_cast<const v4u*>(ts + gt * 16);
            store_group<BITS>(gather16(qs + (size_t)rr * pitch, tp[0], tp[1]), out, orow_bytes, M, rs + rr, NH + gt);
        }
        if (kept >= 0) gather_group(NH + (kept & 0xfffff), rs + (kept >> 20));
        strip_barrier();
    }
}

// Whether X is larger than so many MiB: the eight L2s hold 32 together, the memory-side cache 256.
template <int DT> bool beyond_mib(int M, int K, int mib) { return (long long)M * K * (int)sizeof(typename Elem<DT>::type) > ((long long)mib << 20); }

// Per input channel max|x| into cmax (fp32 bit patterns, which order like the non-negative floats
// they hold); accumulate keeps what cmax holds on entry as the starting value.
template <int DT>
void launch_colabsmax(const void* X, int M, int K, int ld, bool accumulate, uint32_t* cmax, hipStream_t stream)
{
    constexpr int VEC = Elem<DT>::VEC;
    if (!accumulate) fill_u32_kernel<<<(K + 255) / 256, 256, 0, stream>>>(cmax, K, 0u);
    const AbsmaxGrid a = absmax_grid(M, K, ld, VEC, compute_units());
    // Streamed from 96 MiB on: smaller activations may still lie in the memory-side cache, from which the hint keeps nothing (fp32
    // 4096 x 4096, three such in turn: 15.1 us with it, 11.4 without; bf16 8192 x 11008 29.4 and 36.9).
    auto kern = beyond_mib<DT>(M, K, 96) ? colabsmax_kernel<DT, true> : colabsmax_kernel<DT, false>;
    kern<<<dim3((unsigned)a.blocks, (unsigned)a.strips), 256, 0, stream>>>(X, M, K, ld, a.rows_per_strip, cmax);
}

// Candidates for a' of the flattened tensor (or, all_channels, of the whole array) into cand, which has room for
// candidate_capacity(K) floats; their number goes to *ncand.
template <int DT>
int launch_tensor_absmax(const void* X, int M, int K, int ld, const int32_t* src, const int32_t* rep, int Kpad,
                         bool all_channels, float* cand, int* ncand, hipStream_t stream, float* map = nullptr)
{
    const AbsmaxGrid a = absmax_grid(M, K, ld, Elem<DT>::VEC, compute_units());
    const dim3 grid((unsigned)a.blocks, (unsigned)a.strips + (map ? 1 : 0));
    // The quantizer reads X again: what the memory-side cache can hold is left there (streamed past it, the pass itself gains,
    // the call loses: 8192 x 4096 bf16 to E3M2 37.5 -> 45.9 us; 8192 x 20480 to nibbles, 335 MB, gains, 168.2 -> 162.7).
    const bool nt = beyond_mib<DT>(M, K, 224);
    auto kern = all_channels ? (nt ? tensor_absmax_kernel<DT, true, true> : tensor_absmax_kernel<DT, true, false>)
                             : (nt ? tensor_absmax_kernel<DT, false, true> : tensor_absmax_kernel<DT, false, false>);
    kern<<<grid, all_channels ? 256 : 512, 0, stream>>>(X, M, K, ld, a.rows_per_strip, src, rep, Kpad, cand, map);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "absmax launch failed: %s", hipGetErrorString(e));
    *ncand = a.candidates();
    return FQ_OK;
}

typedef void (*direct_kernel_t)(const void*, int, int, int, const int32_t*, const int32_t*, int, const float*, const float*, int,
                                float*, float*, uint8_t*, int, int, int, float*);

// Rows per strip of flatten_quant_direct_kernel: what the registers hold in flight (fp32 takes twice as many).
template <int DT, int P> constexpr int direct_rows() { return DT == FQ_F32 ? (P == 1 ? 2 : 1) : (P == 1 ? 4 : 2); }

template <int DT, int BITS, int P>
int direct_kernel(direct_kernel_t* kern)
{
    static std::atomic<unsigned long long> raised{0};
    *kern = flatten_quant_direct_kernel<DT, BITS, P, direct_rows<DT, P>()>;
    return set_lds_limit(reinterpret_cast<const void*>(*kern), 144 * 1024, raised);
}

typedef void (*rows_kernel_t)(const void*, int, int, int, const int32_t*, const float*, const uint8_t*, int, int, uint8_t*);

template <int DT, int BITS>
int rows_kernel(rows_kernel_t* kern)
{
    static std::atomic<unsigned long long> raised{0};
    *kern = flatten_quant_rows_kernel<DT, BITS>;
    return set_lds_limit(reinterpret_cast<const void*>(*kern), 132 * 1024, raised);
}

// LDS of a strip kernel: K / 16 * 16 bytes per row, and per appended slot 2 bytes (its source), per appended group 1 (its
// flag).  Layers of which one row does not fit 64 KiB go to the general kernel.
size_t tail_bytes(int K, int Kpad)
{
    const size_t kq = (size_t)(K & ~15);
    return 2 * ((size_t)Kpad - kq) + ((size_t)Kpad - kq) / 16;
}
bool strip_fits(int K, int Kpad) { return K >= 16 && (size_t)(K & ~15) + tail_bytes(K, Kpad) <= 64u * 1024u; }

template <int DT>
int launch_for_dtype(const void* X, int M, int K, int ld, const int32_t* src_idx, const int32_t* rep,
                     int Kpad, int bits, int mode, const float* absmax_in, float T, void* out, float* scale_out,
                     const ActWorkspace& ws, hipStream_t stream)
{
    const int qmax = (bits == 6) ? 7 : (1 << (bits - 1)) - 1;       // 6: the 4-bit quantizer, E3M2 storage
    const bool peel = mode >= 3;
    uint8_t* o8 = static_cast<uint8_t*>(out);
    float* cand = ws.cmax;
    const bool dynamic = mode != 1 && mode != 4, all_channels = mode >= 2;
    const size_t kq = (size_t)(K & ~15), tail_src = tail_bytes(K, Kpad);
    const bool narrow = strip_fits(K, Kpad);
    if (bits == 6 && (peel || !narrow))                             // E3M2 storage exists in the strip kernels only
        return fail(FQ_ERR_DTYPE, "E3M2 storage (bits = 6) needs K >= 16 and a layer narrow enough for the "
                                  "row-strip kernel, and is not available for the peel split");
    const int NH = K >> 4, P = NH <= 1024 ? 1 : 2;
    // Up to 12 Mi elements the direct kernel, beyond it scale_kernel and the row-strip kernel (three or, static, two
    // launches, but no map work per workgroup).  Whole call, bf16, dynamic, direct against prepared: 16 x 4096 10.2 / 14.2
    // us, 500 x 11008 18.9 / 21.6, 2048 x 4096 18.4 / 18.7, 1024 x 11008 (11.3 M) 23.4 / 23.7; at 4096 x 4096 (16.8 M)
    // 25.5 / 24.7, 1024 x 20480 36.5 / 32.4, 8192 x 11008 98.9 / 87.0.
    if (out && !peel && narrow && NH <= 2048 && (long long)M * K <= (12ll << 20)) {
        const int R = P == 1 ? direct_rows<DT, 1>() : direct_rows<DT, 2>();
        // A few rows: every workgroup reads all of X for a' rather than a launch that does (16 x 4096 bf16: 10.2 against
        // 12.4 us for the call); at most 64 rows, since a slot that repeats no plain group walks them one by one.
        const bool self = mode == 0 && M <= 64 && (size_t)M * K * sizeof(typename Elem<DT>::type) <= 256u * 1024u;
        const int head = (int)round_up((size_t)(NH + P - 1) / P, 64);
        // several slots of head threads up to 256 threads (16 x 256: 7.8 us with one, 6.9 with four; 16 x 4096: 8.3, 9.8)
        const int slots = self ? std::max(1, std::min(256 / head, (M + 3) / 4)) : 1, nthr = head * slots;
        const size_t lds = DIRECT_LDS_FIXED + (size_t)(R + 1) * (kq + ROW_PAD) + tail_src;
        // what the CUs hold at once: 1024 threads (128 registers each) and 160 KiB of LDS
        const int occ = std::max(1, std::min((int)(160u * 1024u / lds), 1024 / nthr));
        const int nblk = direct_workgroups(M, R, compute_units(), occ);
        direct_kernel_t kern = nullptr;
        int rc;
        if (P == 1) rc = bits == 8 ? direct_kernel<DT, 8, 1>(&kern) : bits == 6 ? direct_kernel<DT, 6, 1>(&kern) : direct_kernel<DT, 4, 1>(&kern);
        else rc = bits == 8 ? direct_kernel<DT, 8, 2>(&kern) : bits == 6 ? direct_kernel<DT, 6, 2>(&kern) : direct_kernel<DT, 4, 2>(&kern);
        if (rc) return rc;
        int ncand = 0;
        // the absmax pass works the map out along the way (weights have no copy counts: theirs stays with the quantizer)
        float* map = mode == 0 && !self ? ws.mslot : nullptr;
        if (dynamic && !self)
            if ((rc = launch_tensor_absmax<DT>(X, M, K, ld, src_idx, rep, Kpad, all_channels, cand, &ncand, stream, map))) return rc;
        kern<<<(unsigned)nblk, nthr, lds, stream>>>(X, M, K, ld, src_idx, mode == 2 ? nullptr : rep, Kpad, absmax_in,
                                                    ncand ? cand : nullptr, ncand, scale_out, ws.scalars, o8, M / nblk, M % nblk, slots, map);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(FQ_ERR_HIP, "flatten-quantize launch failed: %s", hipGetErrorString(e));
        return FQ_OK;
    }
    rows_kernel_t rows = nullptr;
    if (!peel && narrow) {
        // the strip's rows in LDS, each with its padding, may come to a little more than 64 KiB (E3M2: 128): raised before anything
        // of this call is enqueued
        if (int rc = bits == 8 ? rows_kernel<DT, 8>(&rows) : bits == 6 ? rows_kernel<DT, 6>(&rows) : rows_kernel<DT, 4>(&rows)) return rc;
    }
    int ncand = 0;
    if (dynamic)
        if (int rc = launch_tensor_absmax<DT>(X, M, K, ld, src_idx, rep, Kpad, all_channels, cand, &ncand, stream)) return rc;
    scale_kernel<<<(Kpad + 1023) / 1024, 1024, 0, stream>>>(cand, ncand, K, src_idx, rep, Kpad, qmax, mode, absmax_in, T,
                                                            ws.mslot, scale_out, ws.scalars, ws.gflag);
    if (!out) {
        // scales only: the caller quantizes elsewhere (the GEMM that converts its A operand on the way into LDS)
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(FQ_ERR_HIP, "activation scale launch failed: %s", hipGetErrorString(e));
        return FQ_OK;
    }
    if (!peel && narrow) {
        // row-strip kernel: R rows per workgroup with R * K bytes of LDS plus 2 bytes per appended slot
        // (at most 64 KiB, so that two workgroups fit a CU); wider layers use the general kernel below
        int R = 8;
        while (R > 1 && (size_t)R * kq + tail_src > 64u * 1024u) R >>= 1;
        // 256 threads walk the strip's groups while the LDS lets four such workgroups share a CU (16 waves to hide the
        // loads).  Strips cut to two rows or one whose LDS admits only two or three get 512 threads.  Whole calls, us, 256 /
        // 512 threads: weight 5120 x 20480 to nibbles 111.1 / 104.3; activation, static, 8192 x 22016 to INT8 137.2 / 124.4, 8192
        // x 28672 188.0 / 155.8.  With four workgroups 512 threads lose: 8192 x 16384 91.4 / 95.0, 8192 x 36000 227.6 / 240.5,
        // weight 8192 x 28672 to INT8 278 / 291.  On higher strips it depends: 8192 x 11008 static 68.4 / 62.7, dynamic 97.0 /
        // 96.6, 8192 x 8192 static 45.8 / 46.4.
        int nthr = (R <= 2 && (size_t)R * kq + tail_src > 160u * 1024u / 4) ? 512 : 256;
        // Very wide layers (strips cut to two rows or one): the blocked E3M2 layout then gets runs of only
        // 192 or 96 bytes per block.  A strip twice as high in a 512-thread workgroup with up to 128 KiB of
        // LDS (one workgroup per CU) measured 11 % faster at K = 22016; at K = 11008 (four rows -> eight)
        // the same change was 16 % slower, so it stops there.
        if (bits == 6) {
            nthr = 256;
            if (R <= 2 && (size_t)(2 * R) * kq + tail_src <= 128u * 1024u) {
                R *= 2;
                nthr = 512;
            }
        }
        rows<<<(unsigned)((M + R - 1) / R), nthr, (size_t)R * (kq + ROW_PAD) + tail_src, stream>>>(X, M, K, ld, src_idx, ws.mslot, ws.gflag, Kpad,
                                                                                                   R, o8);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(FQ_ERR_HIP, "flatten-quantize launch failed: %s", hipGetErrorString(e));
        return FQ_OK;
    }
    const int G = Kpad / 16;
    // rows per thread: as many as 8 while the launch still has >= 2048 waves
    int rpt = 8;
    while (rpt > 1 && ((long long)G * ((M + rpt - 1) / rpt)) < 2048LL * 64) rpt >>= 1;
    const long long threads = (long long)G * ((M + rpt - 1) / rpt);
    const unsigned blocks = (unsigned)((threads + 255) / 256);
    if (peel && bits == 8)
        flatten_quant_kernel<DT, 8, true><<<blocks, 256, 0, stream>>>(X, M, K, ld, src_idx, ws.mslot, Kpad, rpt, o8, ws.scalars, T);
    else if (peel)
        flatten_quant_kernel<DT, 4, true><<<blocks, 256, 0, stream>>>(X, M, K, ld, src_idx, ws.mslot, Kpad, rpt, o8, ws.scalars, T);
    else if (bits == 8)
        flatten_quant_kernel<DT, 8><<<blocks, 256, 0, stream>>>(X, M, K, ld, src_idx, ws.mslot, Kpad, rpt, o8);
    else
        flatten_quant_kernel<DT, 4><<<blocks, 256, 0, stream>>>(X, M, K, ld, src_idx, ws.mslot, Kpad, rpt, o8);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "flatten-quantize launch failed: %s", hipGetErrorString(e));
    return FQ_OK;
}

}  // namespace

bool quantizer_takes_e3m2(int K, int Kpad) { return strip_fits(K, Kpad); }

ActWorkspace carve_act_workspace(void* base, int K, int Kpad)
{
    ActWorkspace ws;
    uint8_t* p = static_cast<uint8_t*>(base);
    size_t off = 0;
    ws.cmax = reinterpret_cast<float*>(p + off);
    off += round_up((size_t)candidate_capacity(K) * 4, 256);
    ws.mslot = reinterpret_cast<float*>(p + off);
    off += round_up((size_t)Kpad * 4, 256);
    ws.scalars = reinterpret_cast<float*>(p + off);
    off += 256;
    ws.gflag = p + off;
    off += round_up(2 * (size_t)(Kpad / 16 + 1), 256);       // gflag, then cflag
    ws.bytes = off;
    return ws;
}

int launch_flatten_quant(const void* X, int x_dtype, int M, int K, int ld, const int32_t* src_idx,
                         const int32_t* rep, int Kpad, int bits, int mode, const float* absmax_in,
                         void* out, float* scale_out, const ActWorkspace& ws, hipStream_t stream, float T)
{
    switch (x_dtype) {
    case FQ_F32:
        return launch_for_dtype<FQ_F32>(X, M, K, ld, src_idx, rep, Kpad, bits, mode, absmax_in, T, out, scale_out, ws, stream);
    case FQ_F16:
        return launch_for_dtype<FQ_F16>(X, M, K, ld, src_idx, rep, Kpad, bits, mode, absmax_in, T, out, scale_out, ws, stream);
    case FQ_BF16:
        return launch_for_dtype<FQ_BF16>(X, M, K, ld, src_idx, rep, Kpad, bits, mode, absmax_in, T, out, scale_out, ws, stream);
    default:
        return fail(FQ_ERR_DTYPE, "unsupported input dtype %d", x_dtype);
    }
}

int launch_channel_absmax(const void* X, int x_dtype, int M, int K, int ld, int accumulate, float* chmax,
                          hipStream_t stream)
{
    uint32_t* cmax = reinterpret_cast<uint32_t*>(chmax);
    switch (x_dtype) {
    case FQ_F32: launch_colabsmax<FQ_F32>(X, M, K, ld, accumulate != 0, cmax, stream); break;
    case FQ_F16: launch_colabsmax<FQ_F16>(X, M, K, ld, accumulate != 0, cmax, stream); break;
    case FQ_BF16: launch_colabsmax<FQ_BF16>(X, M, K, ld, accumulate != 0, cmax, stream); break;
    default: return fail(FQ_ERR_DTYPE, "unsupported input dtype %d", x_dtype);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FQ_ERR_HIP, "channel absmax launch failed: %s", hipGetErrorString(e));
    return FQ_OK;
}

}  // namespace fq
