// Base conversions of the key switch at N = 2^16 and 2^17, with the column passes on both sides of them.
//
// Bound by the arithmetic units (0.81 of their issue slots for eight rotations at N = 2^16, level 24) at the clock that the power
// limit leaves them.  Against a column pass of its own for the inverse transform and a ModUp pass that read a digit's sources through L2 for every two
// targets, 56 instead of 72 FP64 instructions per output: one rotation at level 13 7.5 + 24.4 -> 19.7 us, eight at level 24
// 41 + 290 -> 285 us, four at N = 2^17, level 30, 57 + 584 -> 490 us; 16 products with rescale 1827 -> 1695 us as a call (by this
// kernel alone; later steps took them further).
//
// ModDown's corrections, one rotation at level 13: 10.0 + 13.2 -> 19.4 us (inverse column pass of the special limbs and column pass of the
// corrections before), eight at level 24 32 + 142 -> 132, four at N = 2^17, level 30, 35 + 168 -> 186 (the centring and splitting of a digit
// is done once, not once per target).  A product with rescale at level 6 takes three launches fewer, 102 -> 95 us as a call.
//
// A conversion reads a few source limbs (a digit's, or the special ones) and makes many target limbs of them.  One work-group
// takes CONV_COLS columns of all rows: its waves run the inverse column pass of one source each and leave the scaled coefficients
// in LDS, then each wave makes one target after the other: conversion, forward column pass, store.  Sources are read once
// instead of once per two targets, they are converted to their arithmetic form once, the coefficients never travel to memory, and
// two launches are one.  A wave exchanges its values through LDS of its own, so that nothing but the sources' arrival
// takes a work-group barrier.
//
// Column passes that follow a conversion leave a limb with its rows interleaved by two (mid_at): a lane has both
// rows of a pair in hand, so it stores 16 bytes and a work-group's four columns fill segments of 64.
#pragma once
#include "kernels_ntt.h"

#define CONV_COLS 4
#define CONV_GROUPS (256 / CONV_COLS)
// 32-bit words per wave of the exchange: 16 groups of 16 rows x 4 columns, four pad words per group keep both patterns
// free of bank conflicts; the low and the high halves of the values go through it in turn
#define CONV_EXCH (16 * 68)

// SOURCES: the most that a conversion has (a tenth of the LDS of a compute unit each at N = 2^17, a twentieth at N = 2^16).
template <int LOGN, int SOURCES = 4> struct ConvGeom {
    static constexpr int ROWS = 1 << (LOGN - 8);
    static constexpr int HALVES = ROWS / 256;       // 16-element register steps per lane
    static constexpr int TILE = ROWS * CONV_COLS;   // words of one source
    // two work-groups per compute unit, four waves per SIMD; N = 2^17, with twice the values per lane and sources of twice the
    // size, one of three waves per SIMD (at four, 31 registers go to scratch memory), as with more than five sources at N = 2^16; ModDown, whose
    // inverse column pass is on the integer path as a rule, two waves per SIMD at N = 2^17
    static constexpr bool WIDE = SOURCES > 5;
    static constexpr int WAVES = LOGN == 16 && !WIDE ? 8 : 12, BOUND = LOGN == 16 && !WIDE ? 4 : 3;
    static constexpr int DOWN_WAVES = WIDE ? 12 : 8, DOWN_BOUND = WIDE ? 3 : LOGN == 16 ? 4 : 2;
};
// A lane's place: in the strided pattern it holds rows (lane >> 2) + 16 k of column lane & 3, in the consecutive one rows
// 16 (lane >> 2) + k.
// FWD: from the strided pattern to the consecutive one, else back.
template <bool FWD, class A> __device__ __forceinline__ void conv_exchange(typename A::V (&a)[16], const A &ar, unsigned *ex)
{
    const unsigned lane = threadIdx.x & 63u;
    unsigned *strided = ex + lane, *consec = ex + 68u * (lane >> 2) + (lane & 3u);
    unsigned *w = FWD ? strided : consec;
    const unsigned *r = FWD ? consec : strided;
    constexpr int WS = FWD ? 68 : 4, RS = FWD ? 4 : 68;
    unsigned lo[16];
#pragma unroll
    for (int k = 0; k < 16; k++) w[WS * k] = (unsigned)ar.store_mid(a[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) lo[k] = r[RS * k];
    block_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) w[WS * k] = (unsigned)(ar.store_mid(a[k]) >> 32);
    block_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) a[k] = ar.load_mid((u64)r[RS * k] << 32 | lo[k]);
    block_sync();
}

// Inverse column pass of CONV_COLS columns (col: this lane's column of the limb); v: rows (lane >> 2) + 16 k + 256 h, last stage with the
// arithmetic's 1/N factors.
template <int LOGN, class A>
__device__ __forceinline__ void conv_inverse(typename A::V (&v)[ConvGeom<LOGN>::HALVES][16], const u64 *col, const A &ar, unsigned *ex)
{
    constexpr int H = ConvGeom<LOGN>::HALVES;
    const unsigned g = (threadIdx.x & 63u) >> 2;
#pragma unroll
    for (int h = 0; h < H; h++)
#pragma unroll
        for (int k = 0; k < 16; k++) v[h][k] = ar.load_mid(col[(16 * (g + 16 * h) + k) * 256]);
    // written out: as a loop it is too large for the compiler to unroll, and the values, indexed by the half, go to scratch memory
    const auto half = [&](typename A::V (&a)[16], int h) __attribute__((always_inline)) {
        ar.template inv16<false>(a, H + 3, g + 16 * h);
        conv_exchange<false>(a, ar, ex);
        if (H == 1)
            ar.template inv16<true>(a, 0, 0);
        else
            ar.template inv16<false>(a, 1, h);
    };
    half(v[0], 0);
    if constexpr (H == 2) {
        half(v[1], 1);
        ar.inv_stage0_last(v[0], v[1]);
    }
}

// Forward column pass of the values of conv_inverse's pattern (floating point: within 1.5 q of zero; the first five stages then stay
// below 7.2 q), stored with the rows interleaved by two.
template <int LOGN, class A>
__device__ __forceinline__ void conv_forward(typename A::V (&v)[ConvGeom<LOGN>::HALVES][16], u64 *limb, unsigned col, const A &ar, unsigned *ex)
{
    constexpr int H = ConvGeom<LOGN>::HALVES;
    const unsigned g = (threadIdx.x & 63u) >> 2;
    if constexpr (H == 1)
        ar.fwd16(v[0], 0, 0, false);
    else {
        ar.fwd_stage0(v[0], v[1], false);
        ar.fwd16(v[0], 1, 0, false);
        ar.fwd16(v[1], 1, 1, false);
    }
    const auto half = [&](typename A::V (&a)[16], int h) __attribute__((always_inline)) {
        conv_exchange<true>(a, ar, ex);
        ar.fwd16(a, H + 3, g + 16 * h, true);
        u64 *o = limb + (size_t)(g + 16 * h) * 4096 + 2 * col;
#pragma unroll
        for (int p = 0; p < 8; p++) // read by a later kernel
            __builtin_nontemporal_store(u64x2{ar.store_mid(a[2 * p]), ar.store_mid(a[2 * p + 1])}, (u64x2 *)(o + 512 * p));
    };
    half(v[0], 0);
    if constexpr (H == 2) half(v[1], 1);
}

// Sum of up to five products y c modulo q, |y| <= 2^50 (of a fifth one 2^49), |c| <= q/2, q < 2^50: 21 instructions for four.  The
// running sum is kept on the grid of multiples of 2^50 (2^51 for five), the ulp of the bias; every step's rounding error, an integer of at most half
// a grid step, completes it exactly, and one quotient serves all products.  The result is within 1.25 q of zero (1.5 q for five).
template <int NS> __device__ __forceinline__ double conv_sum_fp(const double (&y)[NS], const double (&c)[NS], double q, double qinv)
{
    static_assert(NS <= 5, "the bias leaves room for five products");
    constexpr double BIAS = (NS <= 4 ? 1.0 : 2.0) * 7605903601369376408980219232256.0; // 1.5 * 2^102, 1.5 * 2^103
    double acc = BIAS, low = 0.0;
#pragma unroll
    for (int s = 0; s < NS; s++) {
        const double next = __builtin_fma(y[s], c[s], acc);
        const double l = __builtin_fma(y[s], c[s], acc - next);
        low = s == 0 ? l : low + l;
        acc = next;
    }
    const double h = acc - BIAS;
    const double quo = __builtin_rint(__builtin_fma(low, qinv, h * qinv));
    return __builtin_fma(-quo, q, h) + low;
}
// All sources of a conversion: up to five at once, more in two sums, reduced.
template <int NS> __device__ __forceinline__ double conv_value(const ArithFp &ar, const double (&y)[NS], const double (&c)[NS])
{
    if constexpr (NS <= 5)
        return conv_sum_fp(y, c, ar.q, ar.qinv);
    else {
        double y0[4], c0[4], y1[NS - 4], c1[NS - 4];
#pragma unroll
        for (int s = 0; s < 4; s++) y0[s] = y[s], c0[s] = c[s];
#pragma unroll
        for (int s = 4; s < NS; s++) y1[s - 4] = y[s], c1[s - 4] = c[s];
        return ar.reduce(conv_sum_fp(y0, c0, ar.q, ar.qinv) + conv_sum_fp(y1, c1, ar.q, ar.qinv));
    }
}
// The same on the integer path, 0 <= y < 2^50 - 1, rho[s] = c[s] / q: the quotient is summed in floating point (at most four off: half a
// unit for each of four roundings, less for the errors of rho) and the remainder modulo 2^64.  The result is in (0, 8q).
template <int NS> __device__ __forceinline__ u64 conv_sum_int(const double (&y)[NS], const u64 (&c)[NS], const double (&rho)[NS], u64 q4, u64 nq)
{
    static_assert(NS <= 4, "the quotient stays below 2^52");
    double quo = 4503599627370496.0;
    u64 r = q4;
#pragma unroll
    for (int s = 0; s < NS; s++) {
        quo = __builtin_fma(y[s], rho[s], quo);
        r += d2u(y[s]) * c[s];
    }
    return r + ((u64)__double_as_longlong(quo) & 0x000FFFFFFFFFFFFFull) * nq;
}

// Integer arithmetic of a limb that is the same for the whole wave (2457 instructions of a target become 2284).
template <int LOGN> __device__ __forceinline__ ArithInt conv_int(const DevTables &T, unsigned mi, ShoupConst extra = ShoupConst{0, 0})
{
    ArithInt ar = make_int(T, mi, LOGN, extra);
    ar.nq = negated_uniform(ar.q), ar.nq4 = negated_uniform(ar.q4);
    return ar;
}

template <int NS>
__device__ __forceinline__ u64 conv_value(const ArithInt &ar, const double (&y)[NS], const u64 (&c)[NS], const double (&rho)[NS])
{
    if constexpr (NS <= 4)
        return conv_sum_int(y, c, rho, ar.q4, ar.nq);
    else {
        static_assert(NS == 8, "two sums of four");
        double y0[4], y1[4], r0[4], r1[4];
        u64 c0[4], c1[4];
#pragma unroll
        for (int s = 0; s < 4; s++) y0[s] = y[s], c0[s] = c[s], r0[s] = rho[s], y1[s] = y[s + 4], c1[s] = c[s + 4], r1[s] = rho[s + 4];
        return csub(conv_sum_int(y0, c0, r0, ar.q4, ar.nq) + conv_sum_int(y1, c1, r1, ar.q4, ar.nq), 2 * ar.q4); // below 16q < 2^64
    }
}

// ModUp.  Operation o's scaled digits come from x + o * stride limbs, as the inverse block pass left them, and its raised
// digits go to raised + o * stride limbs, digit j's limb a (active index) at j * (level + K) + a.
struct ModUpArgs {
    const u64 *x;
    u64 *raised;
    int level, L, K, alpha, beta, chunks, stride;
    uint8_t op_level[HE_OPS_MAX]; // operations at levels of their own (0: level); the buffers are laid out for `level`
};

// grid: CONV_GROUPS * operations * beta * chunks, the column groups of an XCD adjacent (four of them share every line that is read).  A
// work-group makes every chunks'th target of its digit, the special limbs (the longest) first; its waves take them one by one.
template <int LOGN, int NS>
__global__ __launch_bounds__((64 * ConvGeom<LOGN, NS>::WAVES), (ConvGeom<LOGN, NS>::BOUND)) void k_ntt_fwd_cols_modup(ModUpArgs ua, DevTables T)
{
    typedef ConvGeom<LOGN, NS> G;
    constexpr int W = G::WAVES, H = G::HALVES;
    __shared__ double src[NS * G::TILE];
    __shared__ unsigned exch[W][CONV_EXCH];
    __shared__ int next;
    const unsigned s8 = blockIdx.x / XCDS, cg = blockIdx.x % XCDS * (CONV_GROUPS / XCDS) + s8 % (CONV_GROUPS / XCDS);
    unsigned unit = s8 / (CONV_GROUPS / XCDS);
    const int chunk = unit % (unsigned)ua.chunks;
    unit /= (unsigned)ua.chunks;
    const int j = unit % (unsigned)ua.beta;
    const unsigned op = unit / (unsigned)ua.beta;
    const int ol = op < HE_OPS_MAX ? ua.op_level[op] : 0, level = ol ? ol : ua.level;
    const int lo = j * ua.alpha, ns = min(ua.alpha, level - lo), M = ua.L + ua.K;
    if (ns <= 0) return; // an operation below the layout's level has fewer digits
    const unsigned lane = threadIdx.x & 63u, col = CONV_COLS * cg + (lane & 3u);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned *ex = exch[wave];
    const size_t slot0 = (size_t)j * ua.alpha + (ns - 1); // table slot of a digit of ns limbs
    if (threadIdx.x == 0) next = 0;
    if (wave < ns) {
        const ArithFp ar = make_fp(T, lo + wave, LOGN, T.up_inv_d[slot0 * ua.alpha + wave]);
        double v[H][16];
        conv_inverse<LOGN>(v, ua.x + (((size_t)op * ua.stride + lo + wave) << LOGN) + col, ar, ex);
#pragma unroll
        for (int h = 0; h < H; h++)
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const double r = ar.reduce(v[h][k]);
                src[wave * G::TILE + 1024 * h + 64 * k + lane] = r < 0.0 ? r + ar.q : r;
            }
    } else if (wave < NS) { // a shorter digit: sources of zero
#pragma unroll
        for (int k = 0; k < 16 * H; k++) src[wave * G::TILE + 64 * k + lane] = 0.0;
    }
    __syncthreads();
    const int targets = level + ua.K - ns;
    u64 *raised = ua.raised + (((size_t)op * ua.stride + (size_t)j * (ua.level + ua.K)) << LOGN);
    const double *sp = src + lane;
    for (;;) {
        int t = 0;
        if (lane == 0) t = atomicAdd(&next, 1);
        t = chunk + ua.chunks * __builtin_amdgcn_readfirstlane(t);
        if (t >= targets) break;
        const int i = t - ua.K < lo ? t - ua.K : t - ua.K + ns; // ciphertext limb, unless t < K
        const int a = t < ua.K ? ua.level + t : i, mi = t < ua.K ? ua.L + t : i;
        u64 *limb = raised + ((size_t)a << LOGN);
        if (T.mod[mi].qd != 0.0) {
            const ArithFp ar = make_fp(T, mi, LOGN);
            double c[NS], v[H][16];
#pragma unroll
            for (int s = 0; s < NS; s++) c[s] = s < ns ? T.up_hat_d[(slot0 * ua.alpha + s) * M + mi] : 0.0;
#pragma unroll
            for (int h = 0; h < H; h++)
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    double y[NS];
#pragma unroll
                    for (int s = 0; s < NS; s++) y[s] = sp[s * G::TILE + 1024 * h + 64 * k];
                    v[h][k] = conv_value(ar, y, c);
                }
            conv_forward<LOGN>(v, limb, col, ar, ex);
        } else {
            const ArithInt ar = conv_int<LOGN>(T, mi);
            u64 c[NS], v[H][16];
            double rho[NS];
#pragma unroll
            for (int s = 0; s < NS; s++) {
                c[s] = s < ns ? T.up_hat[(slot0 * ua.alpha + s) * M + mi] : 0;
                rho[s] = (double)c[s] * T.rq[mi];
            }
#pragma unroll
            for (int h = 0; h < H; h++)
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    double y[NS];
#pragma unroll
                    for (int s = 0; s < NS; s++) y[s] = sp[s * G::TILE + 1024 * h + 64 * k];
                    v[h][k] = conv_value(ar, y, c, rho);
                }
            conv_forward<LOGN>(v, limb, col, ar, ex);
        }
    }
}

// ModDown's corrections r of both components: operation o's special limbs come from u + o * stride limbs, component c's limb k at
// c * (level + K) + level + k, and the corrections go to r + o * stride limbs, component c's limb i at c * level + i.  For ciphertext limbs on
// the floating-point path and special primes below 2^50, or above with 2^50 mod q_i small for every i (DevTables.dn_fold).
struct ModDownArgs {
    u64 *u, *r;
    int level, L, K, chunks, stride;
    int first, limbs; // ciphertext limbs first .. first + limbs - 1 are made (of an operation at a lower level those that it has)
    int keep;         // the digits, as residues, replace the special limbs in u, for a second launch that takes them from there
    uint8_t op_level[HE_OPS_MAX];
};
// A centred digit y, |y| < 2^59, in LDS: y + 2^49.  Its low 50 bits are yl + 2^49 with |yl| <= 2^49, what is above them is yh = (y - yl) / 2^50, and
// y = yh (2^50 mod q) + yl modulo q, within 2^50 of zero.
#define CONV_HALF (1ull << 49)
__device__ __forceinline__ double conv_digit(u64 z, double r50)
{
    const double yl = __longlong_as_double((long long)((z & 0x3FFFFFFFFFFFFull) | 0x4330000000000000ull)) - (4503599627370496.0 + 562949953421312.0);
    return __builtin_fma((double)((int)(z >> 32) >> 18), r50, yl);
}

// grid: CONV_GROUPS * operations * 2 * chunks, work-groups and waves as in k_ntt_fwd_cols_modup; the digits come from the inverse column
// pass of the special limbs.  RS: with a rescale, after the dropped limb, level - 1, has been through ModDown: the digits are
// in u, and the dropped limb, as the inverse block pass left it in r, is one more source with P for its constant.
template <int LOGN, bool RS, int KMAX>
__global__ __launch_bounds__((64 * ConvGeom<LOGN, KMAX>::DOWN_WAVES), (ConvGeom<LOGN, KMAX>::DOWN_BOUND)) void k_ntt_fwd_cols_moddown(ModDownArgs da, DevTables T)
{
    typedef ConvGeom<LOGN, KMAX> G;
    constexpr int NS = KMAX + (RS ? 1 : 0), W = G::DOWN_WAVES, H = G::HALVES;
    __shared__ u64 src[NS * G::TILE];
    __shared__ unsigned exch[W][CONV_EXCH];
    __shared__ int next;
    const unsigned s8 = blockIdx.x / XCDS, cg = blockIdx.x % XCDS * (CONV_GROUPS / XCDS) + s8 % (CONV_GROUPS / XCDS);
    unsigned unit = s8 / (CONV_GROUPS / XCDS);
    const int chunk = unit % (unsigned)da.chunks;
    unit /= (unsigned)da.chunks;
    const int comp = unit & 1u;
    const unsigned op = unit >> 1;
    const int ol = op < HE_OPS_MAX ? da.op_level[op] : 0, level = ol ? ol : da.level;
    const unsigned lane = threadIdx.x & 63u, col = CONV_COLS * cg + (lane & 3u);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned *ex = exch[wave];
    u64 *special = da.u + (((size_t)op * da.stride + (size_t)comp * (da.level + da.K) + da.level) << LOGN);
    u64 *corr = da.r + (((size_t)op * da.stride + (size_t)comp * da.level) << LOGN);
    if (threadIdx.x == 0) next = 0;
    // row (lane >> 2) + 16 k + 256 h of this lane's column, in the limb; in LDS it sits at 1024 h + 64 k + lane
    const auto place = [&](int h, int k) { return ((lane >> 2) + 16 * k + 256 * h) * 256 + col; };
    u64 *mine = src + wave * G::TILE + lane;
    if (wave < da.K) {
        u64 *limb = special + ((size_t)wave << LOGN);
        const ModConst m = T.mod[da.L + wave];
        const u64 half = (m.q - 1) / 2;
        const auto put = [&](int h, int k, u64 y) { mine[1024 * h + 64 * k] = (y > half ? y - m.q : y) + CONV_HALF; };
        const auto put_keep = [&](int h, int k, u64 y) {
            put(h, k, y);
            if (da.keep) limb[place(h, k)] = y;
        };
        if (RS) {
#pragma unroll
            for (int h = 0; h < H; h++)
#pragma unroll
                for (int k = 0; k < 16; k++) put(h, k, limb[place(h, k)]);
        } else if (m.qd != 0.0) {
            const ArithFp ar = make_fp(T, da.L + wave, LOGN, T.dn_inv_d[wave]);
            double v[H][16];
            conv_inverse<LOGN>(v, limb + col, ar, ex);
#pragma unroll
            for (int h = 0; h < H; h++)
#pragma unroll
                for (int k = 0; k < 16; k++) put_keep(h, k, ar.store_final(v[h][k]));
        } else {
            const ArithInt ar = conv_int<LOGN>(T, da.L + wave, T.dn_inv[wave]);
            u64 v[H][16];
            conv_inverse<LOGN>(v, limb + col, ar, ex);
#pragma unroll
            for (int h = 0; h < H; h++)
#pragma unroll
                for (int k = 0; k < 16; k++) put_keep(h, k, ar.store_final(v[h][k]));
        }
    } else if (wave < KMAX) { // fewer special primes: digits of zero
#pragma unroll
        for (int k = 0; k < 16 * H; k++) mine[64 * k] = CONV_HALF;
    } else if (RS && wave == KMAX) {
        const ArithFp ar = make_fp(T, da.level - 1, LOGN);
        double v[H][16];
        conv_inverse<LOGN>(v, corr + ((size_t)(da.level - 1) << LOGN) + col, ar, ex);
        const double half = (ar.q - 1.0) * 0.5;
#pragma unroll
        for (int h = 0; h < H; h++)
#pragma unroll
            for (int k = 0; k < 16; k++) { // centred; the reduction may end on the wrong side of half by one
                const double r = ar.reduce(v[h][k]);
                mine[1024 * h + 64 * k] = ar.store_mid(r > half ? r - ar.q : r < -half ? r + ar.q : r);
            }
    }
    __syncthreads();
    const int end = min(da.first + da.limbs, level);
    const u64 *sp = src + lane;
    for (;;) {
        int t = 0;
        if (lane == 0) t = atomicAdd(&next, 1);
        const int i = da.first + chunk + da.chunks * __builtin_amdgcn_readfirstlane(t);
        if (i >= end) break;
        const ArithFp ar = make_fp(T, i, LOGN);
        const double r50 = T.dn_r50_d[i];
        double c[NS], v[H][16];
#pragma unroll
        for (int s = 0; s < KMAX; s++) c[s] = s < da.K ? T.dn_hat_d[s * da.L + i] : 0.0;
        if (RS) c[NS - 1] = T.dn_pmod_d[i];
#pragma unroll
        for (int h = 0; h < H; h++)
#pragma unroll
            for (int k = 0; k < 16; k++) {
                double y[NS];
#pragma unroll
                for (int s = 0; s < KMAX; s++) y[s] = conv_digit(sp[s * G::TILE + 1024 * h + 64 * k], r50);
                if (RS) y[NS - 1] = ar.load_mid(sp[(NS - 1) * G::TILE + 1024 * h + 64 * k]);
                v[h][k] = conv_value(ar, y, c);
            }
        conv_forward<LOGN>(v, corr + ((size_t)i << LOGN), col, ar, ex);
    }
}
