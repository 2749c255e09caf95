// Negacyclic NTT kernels with fused base-conversion prologues and ModDown/rescale epilogues.
//
// Forward transform = decimation in time with the powers of psi in bit-reversed order; stage s
// (s = 0 .. logN-1) pairs elements N/2^(s+1) apart and uses twiddle index 2^s + (j >> (logN-s)).
// A limb of N = 2^16 takes two kernels: the column pass (stages 0-7 on 16 columns x 256 rows, row stride 256 elements,
// 128-byte global segments; 16 elements per thread, four stages on them at a time, a radix-16 step, and one exchange through LDS between the
// 256 threads) and the block pass (stages 8-15 on contiguous blocks of 256, eight elements per lane, two blocks to a wave).
// N = 2^17 keeps the two kernels: its column pass runs nine stages on 512 rows (32 elements per thread).
// N = 2^12 has kernels of its own (kernels_n12.h).  The inverse runs the block pass first and the column pass last.
// The key switch's base conversions have column passes of their own (kernels_conv.h); the forms here serve what those leave out: the corrected
// conversions, primes of 2^50 and above among the sources, launches with few targets to a source.
//
// Fusions, all bit-identical to the unfused steps:
//  * the forward column pass can build its input on the fly: ModUp (sum over the digit's limbs of
//    y_i * (D/q_i mod t)), ModDown (sum over the special limbs of y_k * (P/p_k mod q_i)) or the
//    centred residue of a dropped limb (rescale);
//  * the inverse column pass can fold (D/q_i)^-1 or (P/p_k)^-1 into its 1/N scaling, so it emits
//    the y values those sums need;
//  * the forward block pass can finish a rescale, out = (u - ntt) * const, or the ModDown of the limb that a rescale drops, which goes
//    through its inverse block pass at once;
//  * ModDown followed by rescale takes one transform per limb instead of two: with t the centred dropped
//    limb of the ModDown result, NTT(r) P^-1 + NTT(t) = NTT(r + P t) P^-1, so the column pass transforms
//    r + P t and the inner product finishes out = (u - ntt) (P q_l)^-1.
#pragma once
#include "arith.h"

typedef u64 u64x2 __attribute__((ext_vector_type(2)));
typedef u64 u64x2u __attribute__((ext_vector_type(2), aligned(8))); // in buffers of a caller, which are aligned to words
// Work-groups go to the eight XCDs round-robin by index, and each XCD has its own L2.
#define XCDS 8u

// limbs per launch: the table below travels as a kernel argument (10 KiB); large launches matter, halving this
// costs the conversion passes 11-14 %
#ifndef HE_MAXB
#define HE_MAXB 2048
#endif
// operations per launch that can carry a key, a Galois element, a level and pointers of their own
#ifndef HE_OPS_MAX
#define HE_OPS_MAX 32
#endif
// A launch works on up to HE_MAXB limbs: limb b is written at dst + slot[b]*N, read (inverse block
// pass only) at src + src[b]*N, and uses modulus index mod[b].
struct LimbBatch {
    uint16_t slot[HE_MAXB];
    uint16_t src[HE_MAXB];
    uint8_t mod[HE_MAXB];
};

enum { PRO_LOAD = 0, PRO_MODUP = 1, PRO_MODDOWN = 2, PRO_RESCALE = 3, PRO_MODDOWN_RS = 4 };
__host__ __device__ constexpr bool pro_is_moddown(int pro) { return pro == PRO_MODDOWN || pro == PRO_MODDOWN_RS; }
// A column pass behind a conversion of the key switch (N = 2^16 and 2^17) leaves the limb with its rows, the blocks of 256 of the block pass,
// interleaved by two: element e of block b at mid_at<true>(b, e).  A plain transform works in place and cannot.
__host__ __device__ constexpr bool pro_pairs_rows(int pro) { return pro == PRO_MODUP || pro_is_moddown(pro); }
template <bool PAIR> __device__ __forceinline__ unsigned mid_at(unsigned b, unsigned e)
{
    return PAIR ? (b >> 1) * 512u + 2u * e + (b & 1u) : b * 256u + e;
}
enum { SCALE_NONE = 0, SCALE_MODUP = 1, SCALE_MODDOWN = 2 };
// Epilogues of the block pass: the transform; a finished rescale; the finished limb that a rescale drops, through its inverse block pass.
enum { EPI_STORE = 0, EPI_FIN = 1, EPI_FIN_INV = 2 };

// Batches: `count` independent ciphertexts are laid out with fixed strides (in limbs); a limb's slot
// is op * stride + local index, so op = slot / stride and the local index keeps its single-op meaning.
struct ConvArgs {
    const u64 *src; // ModUp: y limbs [level][N]; ModDown: u [2][level+K][N]; rescale: t [2][N]
    int level, L, K, alpha;
    int dst_stride; // limbs between two operations in the buffer being transformed
    int src_stride; // limbs between two operations in src
    // ModDown + rescale: the dropped limb of component c (coefficient domain) at src2 + (c*level + level-1) limbs
    const u64 *src2;
    int src2_stride;
    // centred-limb prologue (rescale, ModRaise): modulus index of the source limb, limbs per component in dst
    int rs_mod, rs_nl;
    // Corrected conversions selected: ModUp takes out floor(sum_i y_i / q_i) D, ModDown rint(sum_k y'_k / p_k) P,
    // the sums in double precision, one rounding per operation, sources in order.
    int exact;
    // Operations of one launch at different levels (mixed-level rotations): op_level[o] != 0 is the level of
    // operation o, while `level` stays the level the buffers are laid out for (the largest of the launch).
    uint8_t op_level[HE_OPS_MAX];
};
// level of the operation that owns destination slot `slot`
__device__ __forceinline__ int conv_op_level(const ConvArgs &cv, unsigned slot)
{
    const unsigned op = slot / (unsigned)cv.dst_stride;
    const int l = op < HE_OPS_MAX ? cv.op_level[op] : 0;
    return l ? l : cv.level;
}

// Finishing epilogue of the block pass: out = (u - ntt) * cst.  A limb's slot within its operation decodes
// as component c = slot / nl, limb i = slot % nl.
struct FinArgs {
    const u64 *u;   // minuend limbs, component stride u_cstride limbs
    u64 *out;       // component stride out_cstride limbs
    const ShoupConst *cst;
    const double *cst_d;
    int u_cstride, out_cstride, nl;
    int dst_stride, u_stride, out_stride; // limbs between two operations in each buffer
};

__device__ __forceinline__ int active_mod(int a, int level, int L) { return a < level ? a : L + (a - level); }

// NTT-domain index of the automorphism sigma_g: out[k] = in[k'] with
// 2 brv(k') + 1 = (2 brv(k) + 1) g mod 2N.
__device__ __forceinline__ unsigned galois_index(unsigned k, unsigned g, int logN)
{
    const unsigned b = __brev(k) >> (32 - logN);
    const unsigned e = ((2 * b + 1) * g) & ((2u << logN) - 1);
    return __brev((e - 1) >> 1) >> (32 - logN);
}

// ---- prologues: element `pos` of the limb the column pass is about to transform ----------------------

template <int NSMAX> struct ConvSetup {
    const u64 *sp[NSMAX];         // source limbs; entries past the real count repeat entry 0 with zero constants
    double cd[NSMAX], cdh[NSMAX]; // constants as balanced doubles (cdh: constant * 2^31)
    u64 ci[NSMAX], cp[NSMAX];     // constants as residues and their companions floor(c 2^64 / t) (integer targets)
    // ModDown: source digit s counts as y - p_s when y > hs[s]; each such digit subtracts P mod q_i
    u64 hs[NSMAX];
    u64 pm_i;
    double pm_d;
    double r50;  // ModDown, SPLIT 2: 2^50 mod q
    // rescale
    u64 ql, half;
    double qld;
    const u64 *tp; // ModDown + rescale: the dropped limb of this component
    // corrected conversions: 1.0 / (double)modulus of source s (0 past the real count), D mod t (ModUp)
    double rq[NSMAX];
    u64 dm_i;
    double dm_d;
};

// slot = position of the limb in the destination buffer; mi = its modulus index
template <int PRO, int NSMAX, int LOGN>
__device__ __forceinline__ ConvSetup<NSMAX> conv_setup(const ConvArgs &cv, const DevTables &T, unsigned slot, unsigned mi)
{
    ConvSetup<NSMAX> S;
    S.ql = S.half = 0;
    S.qld = 0.0;
    S.pm_i = 0;
    S.pm_d = 0.0;
    S.r50 = 0.0;
    S.tp = nullptr;
    S.dm_i = 0;
    S.dm_d = 0.0;
    const int M = cv.L + cv.K, Ma = cv.level + cv.K;
    const int op_level = conv_op_level(cv, slot);
    const unsigned op = slot / (unsigned)cv.dst_stride;
    slot -= op * (unsigned)cv.dst_stride;
    const u64 *src = cv.src + (((size_t)op * cv.src_stride) << LOGN);
#pragma unroll
    for (int s = 0; s < NSMAX; s++) {
        S.sp[s] = src;
        S.ci[s] = S.cp[s] = 0;
        S.cd[s] = S.cdh[s] = 0.0;
        S.hs[s] = ~(u64)0;
        S.rq[s] = 0.0;
    }
    if (PRO == PRO_MODUP) {
        const int j = slot / Ma;
        const int lo = j * cv.alpha, hi = min(lo + cv.alpha, op_level);
        const int ns = hi - lo;
        const size_t cs = ((size_t)j * cv.alpha + (ns - 1)) * cv.alpha;
#pragma unroll
        for (int s = 0; s < NSMAX; s++) {
            const bool on = s < ns;
            const size_t ci = (cs + (on ? s : 0)) * M + mi;
            S.sp[s] = src + ((size_t)(lo + (on ? s : 0)) << LOGN);
            S.ci[s] = on ? T.up_hat[ci] : 0;
            S.cp[s] = on ? T.up_hat_p[ci] : 0;
            S.cd[s] = on ? T.up_hat_d[ci] : 0.0;
            S.cdh[s] = on ? T.up_hat_dh[ci] : 0.0;
            S.rq[s] = on ? T.rq[lo + s] : 0.0;
        }
        S.dm_i = T.up_dmod[((size_t)j * cv.alpha + (ns - 1)) * M + mi];
        S.dm_d = T.up_dmod_d[((size_t)j * cv.alpha + (ns - 1)) * M + mi];
    } else if (pro_is_moddown(PRO)) {
        const int c = slot / cv.level, i = slot % cv.level;
#pragma unroll
        for (int s = 0; s < NSMAX; s++) {
            const bool on = s < cv.K;
            const size_t ci = (size_t)(on ? s : 0) * cv.L + i;
            S.sp[s] = src + (((size_t)c * Ma + cv.level + (on ? s : 0)) << LOGN);
            S.ci[s] = on ? T.dn_hat[ci] : 0;
            S.cd[s] = on ? T.dn_hat_d[ci] : 0.0;
            S.cdh[s] = on ? T.dn_hat_dh[ci] : 0.0;
            S.hs[s] = on ? (T.mod[cv.L + s].q - 1) / 2 : ~(u64)0;
            S.rq[s] = on ? T.rq[cv.L + s] : 0.0;
        }
        S.pm_i = T.dn_pmod[i];
        S.pm_d = T.dn_pmod_d[i];
        S.r50 = T.dn_r50_d[i];
        if (PRO == PRO_MODDOWN_RS) {
            S.tp = cv.src2 + (((size_t)op * cv.src2_stride + (size_t)c * cv.level + cv.level - 1) << LOGN);
            S.ql = T.mod[cv.level - 1].q;
            S.half = (S.ql - 1) / 2;
            S.qld = T.mod[cv.level - 1].qd;
        }
    } else if (PRO == PRO_RESCALE) {
        const int c = slot / cv.rs_nl;
        S.sp[0] = src + ((size_t)c << LOGN);
        S.ql = T.mod[cv.rs_mod].q;
        S.half = (S.ql - 1) / 2;
        S.qld = T.mod[cv.rs_mod].qd;
    }
    return S;
}

// SPLIT 1: the sources may be 2^50 or larger, so an FP64 target splits each at bit 31; SPLIT 2 (ModDown): it folds
// each at bit 50 instead, y = yh 2^50 + yl = yh r50 + yl modulo q with r50 = 2^50 mod q small (one product, not two).  TINT (ModDown + rescale):
// the dropped limb is 2^50 or larger and is reduced with integers first; a template parameter rather than a
// run-time branch, because the integer code would cost every launch 100 registers.
template <int PRO, int SPLIT, bool TINT, bool EX, int NSMAX>
__device__ __forceinline__ double conv_get(const ConvSetup<NSMAX> &S, const ArithFp &ar, const ModConst &m, unsigned pos)
{
    if (PRO == PRO_RESCALE) {
        const u64 tv = S.sp[0][pos];
        if (S.qld != 0.0) return u2d(tv) - (tv > S.half ? S.qld : 0.0); // centred value, |v| < q_last / 2
        const bool neg = tv > S.half; // q_last >= 2^50: reduce the magnitude with integers first
        const double w = u2d(reduce64(neg ? S.ql - tv : tv, m));
        return neg ? -w : w;
    }
    double acc = 0.0, sv = 0.0;
    int neg = 0; // ModDown: number of digits that stand for y - p
#pragma unroll
    for (int s = 0; s < NSMAX; s++) {
        const u64 y = S.sp[s][pos];
        const bool ng = pro_is_moddown(PRO) && y > S.hs[s];
        if (pro_is_moddown(PRO)) neg += ng ? 1 : 0;
        if (EX) { // the source as a fraction of its modulus (ModDown: of the centred digit)
            const double yd = !pro_is_moddown(PRO) ? (SPLIT ? (double)y : u2d(y))
                              : ng               ? -(double)(2 * S.hs[s] + 1 - y)
                                                 : (double)y;
            sv = sv + yd * S.rq[s];
        }
        if (!SPLIT)
            acc += ar.mulmod(u2d(y), S.cd[s]);
        else if (SPLIT == 2) {
            // y = yh 2^50 + yl = yh r50 + yl modulo q: below 2^50 + 2^10 2^40, exact, and one product instead of two
            const double yh = (double)(unsigned)(y >> 50), yl = u2d(y & 0x3FFFFFFFFFFFFull);
            acc += ar.mulmod(__builtin_fma(yh, S.r50, yl), S.cd[s]);
        } else {
            const double yh = (double)(unsigned)(y >> 31), yl = (double)(unsigned)(y & 0x7FFFFFFFu);
            acc += ar.mulmod(yh, S.cdh[s]) + ar.mulmod(yl, S.cd[s]);
        }
        if ((s & 3) == 3 && s + 1 < NSMAX) acc = ar.reduce(acc);
    }
    if (PRO == PRO_MODUP && EX) acc -= __builtin_floor(sv) * S.dm_d; // at most (sources - 1) D
    if (pro_is_moddown(PRO)) {
        if (NSMAX > 4) acc = ar.reduce(acc);
        // p_s * (P/p_s) = P for every centred digit; corrected: plus rint(sv) P, together between 0 and K times P
        acc -= ((double)neg + (EX ? __builtin_rint(sv) : 0.0)) * S.pm_d;
    }
    if (PRO == PRO_MODDOWN_RS) { // + P t with t the centred dropped limb
        const u64 tv = S.tp[pos];
        double tc;
        if (!TINT)
            tc = u2d(tv) - (tv > S.half ? S.qld : 0.0);
        else {
            const bool tneg = tv > S.half;
            const double w = u2d(reduce64(tneg ? S.ql - tv : tv, m));
            tc = tneg ? -w : w;
        }
        acc += ar.mulmod(tc, S.pm_d);
    }
    return acc;
}

template <int PRO, int SPLIT, bool TINT, bool EX, int NSMAX>
__device__ __forceinline__ u64 conv_get(const ConvSetup<NSMAX> &S, const ArithInt &ar, const ModConst &m, unsigned pos)
{
    if (PRO == PRO_RESCALE) {
        const u64 tv = S.sp[0][pos];
        const bool neg = tv > S.half;
        const u64 w = reduce64(neg ? S.ql - tv : tv, m);
        return neg ? (w ? m.q - w : 0) : w;
    }
    if (PRO == PRO_MODUP && NSMAX <= 4) {
        // up to four products in [0, 4q) each, summed without reduction: below 16q < 2^64
        u64 lazy = 0;
        double sv = 0.0;
#pragma unroll
        for (int s = 0; s < NSMAX; s++) {
            const u64 y = S.sp[s][pos];
            lazy += mul_shoup_sloppy(y, ShoupConst{S.ci[s], S.cp[s]}, ar.nq);
            if (EX) sv = sv + (double)y * S.rq[s];
        }
        lazy = csub(lazy, 8 * m.q); // the range the transform takes
        if (EX) {
            const u64 r = csub(csub(csub(lazy, 4 * m.q), 2 * m.q), m.q);
            return csub(r + m.q - mul_mod((u64)__builtin_floor(sv), S.dm_i, m), m.q);
        }
        return lazy;
    }
    U128 acc{0, 0};
    double sv = 0.0;
    u64 corr = 0; // ModDown: every digit that stands for y - p takes out one P
#pragma unroll
    for (int s = 0; s < NSMAX; s++) {
        const u64 y = S.sp[s][pos];
        mac128(acc, y, S.ci[s]);
        const bool ng = pro_is_moddown(PRO) && y > S.hs[s];
        if (pro_is_moddown(PRO)) corr = csub(corr + (ng ? S.pm_i : 0), m.q);
        if (EX) {
            const double yd = ng ? -(double)(2 * S.hs[s] + 1 - y) : (double)y;
            sv = sv + yd * S.rq[s];
        }
    }
    u64 r = reduce128(acc, m);
    if (PRO == PRO_MODUP && EX) r = csub(r + m.q - mul_mod((u64)__builtin_floor(sv), S.dm_i, m), m.q);
    if (pro_is_moddown(PRO)) {
        if (EX) { // the correction rint(sv), at most NSMAX / 2 in size, times P
            const int v = (int)__builtin_rint(sv);
#pragma unroll
            for (int t = 0; t < NSMAX / 2; t++) {
                if (t < v) corr = csub(corr + S.pm_i, m.q);
                if (t < -v) corr = csub(corr + m.q - S.pm_i, m.q);
            }
        }
        r = csub(r + m.q - corr, m.q);
    }
    if (PRO == PRO_MODDOWN_RS) {
        const u64 tv = S.tp[pos];
        const bool tneg = tv > S.half;
        const u64 pw = mul_mod(reduce64(tneg ? S.ql - tv : tv, m), S.pm_i, m);
        r = tneg ? csub(r + m.q - pw, m.q) : csub(r + pw, m.q);
    }
    return r;
}

// ---- epilogue: what the forward block pass does with a finished (canonical) NTT value ---------------------

// The limb of destination slot `slot`: where its minuend and its result lie (words), its modulus index (the limb within its component).
struct FinAt {
    size_t u, out;
    unsigned i;
};
template <int LOGN> __device__ __forceinline__ FinAt fin_at(const FinArgs &fa, unsigned slot)
{
    const unsigned op = slot / (unsigned)fa.dst_stride;
    slot -= op * (unsigned)fa.dst_stride;
    const unsigned c = slot / (unsigned)fa.nl, i = slot % (unsigned)fa.nl;
    return {(size_t)(op * fa.u_stride + c * fa.u_cstride + i) << LOGN, (size_t)(op * fa.out_stride + c * fa.out_cstride + i) << LOGN, i};
}
// The minuends of two neighbouring outputs: issued before the transform so that the load overlaps it.
__device__ __forceinline__ u64x2 fin_load(const FinArgs &fa, const FinAt &at, unsigned pos)
{
    return __builtin_nontemporal_load((const u64x2u *)(fa.u + at.u + pos));
}
// FP: the limb's modulus is on the floating-point path (known from the transform's arithmetic at compile time)
template <bool FP> __device__ __forceinline__ u64 fin_value(const FinArgs &fa, const DevTables &T, const FinAt &at, u64 rv, u64 uv)
{
    const ModConst m = T.mod[at.i];
    if (FP) return fp_canon(fp_mulmod(u2d(uv) - u2d(rv), fa.cst_d[at.i], m.qd, m.qinvd), m.qd, m.qinvd);
    return mul_shoup(uv + m.q - rv, fa.cst[at.i], m.q);
}
template <bool FP> __device__ __forceinline__ u64x2 fin_value(const FinArgs &fa, const DevTables &T, const FinAt &at, u64x2 rv, u64x2 uv)
{
    return u64x2{fin_value<FP>(fa, T, at, (u64)rv.x, (u64)uv.x), fin_value<FP>(fa, T, at, (u64)rv.y, (u64)uv.y)};
}
template <class Tv> __device__ __forceinline__ void fin_store(const FinArgs &fa, const FinAt &at, unsigned pos, Tv res) // Tv: u64 or u64x2u
{
    __builtin_nontemporal_store(res, (Tv *)(fa.out + at.out + pos)); // a result: nothing in this launch reads it
}

// LDS of the block pass, element i of block grp: one pad word per 16 elements and 16 per block keep all its patterns free of bank conflicts.
#define TILE_GROUP 272
__device__ __forceinline__ unsigned tile_at(unsigned grp, unsigned i) { return grp * TILE_GROUP + i + (i >> 4); }
// Exchange through LDS among the lanes of one wave.  A wave's LDS operations execute in order, so no work-group barrier is
// needed: only the compiler has to be kept from moving LDS accesses across this point.
__device__ __forceinline__ void block_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// column pass: row r of column c (0..15).  The 16 lanes of a column group always touch 16 consecutive words,
// so this tile needs no padding: 32 KiB at N = 2^16, five work-groups per compute unit.
#define COL_GROUP 256
__device__ __forceinline__ unsigned col_at(unsigned r, unsigned c) { return (r >> 4) * COL_GROUP + (r & 15) * 16 + c; }

// ---- block pass ---------------------------------------------------------------------------------------------
//
// A wave takes two blocks of 256 elements, eight per lane, 32 lanes a block, and runs their stages as three register steps, stages 0-2, 3-5
// and 6-7 of the block, with two exchanges through LDS among those lanes:
//   step 1: lane t holds e = t + 32 k;   step 2: lane (g = t & 7, r = t >> 3) holds e = 32 g + r + 4 k;
//   step 3: lane t holds e = 4 t + k' and 128 + 4 t + k' (k' < 4).
// With one pad word per 16 elements every 16 consecutive lanes of each pattern hit 16 different 8-byte banks.  The three patterns are
// one base each plus compile-time offsets (t + 32 k sits at t + (t >> 4) + 34 k, 32 g + r + 4 k at 34 g + r + 4 k + (k >> 2), and
// 128 h + 4 t + k' at 4 t + (t >> 2) + 136 h + k').
//
// Bound by memory in large launches, by the chain of one wave in small ones.  With 16 elements per lane, 16 lanes a block, two steps of four stages
// and one exchange, the kernels took 79 to 118 registers and four waves per SIMD; now 59 to 64 (with an epilogue 62 to 98, five to eight waves) and eight.  Transforms of
// 64 limbs at N = 2^16 34.0 -> 30.8 us, of 256 103 -> 101, of 34 at N = 2^17 40.5 -> 39.8.
#define WAVE_BLOCKS 2
#define BLK_THREADS 256
#define BLK_PER_WG (BLK_THREADS / 64 * WAVE_BLOCKS)
#define BLK_LDS (BLK_PER_WG * TILE_GROUP)
__device__ __forceinline__ unsigned wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
// This thread's place in the block pass and the LDS addresses of its three exchange patterns.
struct BlockLane {
    unsigned blk, t, g2;
    u64 *l1, *l2, *l3;
    const double *tw; // the block's 255 twiddles in LDS
};
__device__ __forceinline__ BlockLane block_lane(u64 *lds, const double *tws)
{
    BlockLane b;
    b.blk = (threadIdx.x >> 5) & 1u, b.t = threadIdx.x & 31, b.g2 = b.t & 7;
    b.l1 = lds + b.blk * TILE_GROUP + b.t + (b.t >> 4);
    b.l2 = lds + b.blk * TILE_GROUP + 34 * b.g2 + (b.t >> 3);
    b.l3 = lds + b.blk * TILE_GROUP + 4 * b.t + (b.t >> 2);
    b.tw = tws + b.blk * 256;
    return b;
}
// This thread's eight values, t + 32 k of its block, from the two blocks at `pair` (in LDS or in memory) as the column pass left them, rows
// interleaved.  A lane reads four elements of both rows, 16 bytes at a time, the lower half of the wave k < 4 and the upper one k >= 4, and
// the halves swap what belongs to the other's row: read one row at a time, every access would hit half of the banks only.
template <class A> __device__ __forceinline__ void mid_pairs8(const A &ar, typename A::V (&dv)[8], const u64 *pair, const BlockLane &b)
{
    const u64x2 *p = (const u64x2 *)pair + b.t + 128 * b.blk;
    u64x2 v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = p[32 * k];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const auto l = __builtin_amdgcn_permlane32_swap((unsigned)v[k].x, (unsigned)v[k].y, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(v[k].x >> 32), (unsigned)(v[k].y >> 32), false, false);
        dv[k] = ar.load_mid((u64)h[0] << 32 | l[0]);
        dv[k + 4] = ar.load_mid((u64)h[1] << 32 | l[1]);
    }
}
// Block pass of the eight values dv of this thread (pattern of step 1); the result is left in the wave's LDS, element e
// of block b at tile_at(b, e), for the caller to read after a block_sync.  tw(m, i): twiddle of local stage m, group i of the block.
// Ranges (in units of q): floating point: the column pass leaves up to 5.8; reduced, step 1 ends below 2.7 and step 2 below 6.3;
// reduced again, step 3 ends below 1.9, small enough for exact products.  Integer: in [0, 8) throughout.
template <class A, class F> __device__ __forceinline__ void block_pass8(const A &ar, typename A::V (&dv)[8], const BlockLane &b, F tw)
{
    ar.fwd8_with(dv, true, [&](int sp, int gg) { return tw(sp, (unsigned)gg); });
#pragma unroll
    for (int k = 0; k < 8; k++) b.l1[34 * k] = ar.store_mid(dv[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load_mid(b.l2[4 * k + (k >> 2)]);
    ar.fwd8_with(dv, false, [&](int sp, int gg) { return tw(3 + sp, (b.g2 << sp) + gg); });
#pragma unroll
    for (int k = 0; k < 8; k++) b.l2[4 * k + (k >> 2)] = ar.store_mid(dv[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load_mid(b.l3[136 * (k >> 2) + (k & 3)]);
    ar.fwd4x2_with(dv, true, [&](int h, int sp, int gg) { return tw(6 + sp, ((b.t + 32 * h) << sp) + gg); });
#pragma unroll
    for (int k = 0; k < 8; k++) b.l3[136 * (k >> 2) + (k & 3)] = ar.store_mid(dv[k]);
}
// The inverse block pass of canonical residues in the wave's LDS (element e of block b at tile_at(b, e)), which it leaves as the inverse column pass
// takes them; dv: elements t + 32 k.
template <class A, class F> __device__ __forceinline__ void inv_block_pass8(const A &ar, typename A::V (&dv)[8], const BlockLane &b, F tw)
{
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load(b.l3[136 * (k >> 2) + (k & 3)]);
    ar.inv4x2_with(dv, [&](int h, int sp, int gg) { return tw(6 + sp, ((b.t + 32 * h) << sp) + gg); });
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) b.l3[136 * (k >> 2) + (k & 3)] = ar.store_mid(dv[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load_mid(b.l2[4 * k + (k >> 2)]);
    ar.template inv8_with<false>(dv, [&](int sp, int gg) { return tw(3 + sp, (b.g2 << sp) + gg); });
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) b.l2[4 * k + (k >> 2)] = ar.store_mid(dv[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load_mid(b.l1[34 * k]);
    ar.template inv8_with<false>(dv, [&](int sp, int gg) { return tw(sp, (unsigned)gg); });
}
// the same as block_pass8 with the twiddles in LDS
__device__ __forceinline__ void block_pass8(const ArithFp &ar, double (&dv)[8], const BlockLane &b)
{
    block_pass8(ar, dv, b, [&](int m, unsigned i) { return b.tw[(1u << m) - 1 + i]; });
}

// Twiddles of local stage m, group i of block G, forward or inverse.
template <int LOGN, class Tv> __device__ __forceinline__ Tv block_twiddle(const Tv *tw, unsigned G, int m, unsigned i)
{
    return tw[(1u << (LOGN - 8 + m)) + (G << m) + i];
}

// block_pass8 with the twiddles requested ahead: those of the first two steps before the values are waited for (`first`), those of the third behind the
// first step.  For the epilogues, which take more than 64 registers in any case: launches whose waves are all resident at once run the three waits in
// step (a rescale of 46 limbs at N = 2^16: 17.9 -> 16.5 us); the plain pass, eight waves per SIMD without, loses by it (34 limbs 21.6 -> 22.8 with the column pass).
template <int LOGN> struct BlockTwiddles {
    double w1[7], w2[7], w3[6];
    __device__ __forceinline__ void first(const double *tw, const BlockLane &b, unsigned G)
    {
#pragma unroll
        for (int sp = 0; sp < 3; sp++)
#pragma unroll
            for (int g = 0; g < (1 << sp); g++) {
                w1[(1 << sp) - 1 + g] = block_twiddle<LOGN>(tw, G, sp, (unsigned)g);
                w2[(1 << sp) - 1 + g] = block_twiddle<LOGN>(tw, G, 3 + sp, (b.g2 << sp) + g);
            }
    }
    __device__ __forceinline__ void third(const double *tw, const BlockLane &b, unsigned G)
    {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int sp = 0; sp < 2; sp++)
#pragma unroll
                for (int g = 0; g < (1 << sp); g++) w3[3 * h + (1 << sp) - 1 + g] = block_twiddle<LOGN>(tw, G, 6 + sp, ((b.t + 32 * h) << sp) + g);
    }
};
template <int LOGN> __device__ __forceinline__ void block_pass8(const ArithFp &ar, double (&dv)[8], const BlockLane &b, unsigned G, BlockTwiddles<LOGN> &w)
{
    ar.fwd8_with(dv, true, [&](int sp, int g) { return w.w1[(1 << sp) - 1 + g]; });
    w.third(ar.twf, b, G);
    __builtin_amdgcn_sched_barrier(0); // or the compiler asks for them where they are used
#pragma unroll
    for (int k = 0; k < 8; k++) b.l1[34 * k] = ar.store_mid(dv[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load_mid(b.l2[4 * k + (k >> 2)]);
    ar.fwd8_with(dv, false, [&](int sp, int g) { return w.w2[(1 << sp) - 1 + g]; });
#pragma unroll
    for (int k = 0; k < 8; k++) b.l2[4 * k + (k >> 2)] = ar.store_mid(dv[k]);
    block_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) dv[k] = ar.load_mid(b.l3[136 * (k >> 2) + (k & 3)]);
    ar.fwd4x2_with(dv, true, [&](int h, int sp, int g) { return w.w3[3 * h + (1 << sp) - 1 + g]; });
#pragma unroll
    for (int k = 0; k < 8; k++) b.l3[136 * (k >> 2) + (k & 3)] = ar.store_mid(dv[k]);
}

// Product of two residues, canonical.
__device__ __forceinline__ u64 mul_residues(u64 x, u64 y, const ModConst &m, const ArithFp &)
{
    return fp_canon(fp_mulmod(u2d(x), u2d(y), m.qd, m.qinvd), m.qd, m.qinvd);
}
__device__ __forceinline__ u64 mul_residues(u64 x, u64 y, const ModConst &m, const ArithInt &) { return mul_mod(x, y, m); }

// Where a wave's pairs of neighbouring elements, 128 i + 2 lane and + 1 of its 512, i < 4, sit in its LDS.
__device__ __forceinline__ unsigned wave_pair_at(int i)
{
    const unsigned p = 128u * i + 2u * (threadIdx.x & 63u);
    return tile_at(p >> 8, p & 255u);
}
// The wave's inverse block pass from canonical residues in its LDS, stored to `limb` as the inverse column pass takes them.  stream: out of place, as
// part of a conversion, whose batch is far larger than the caches as a rule (the few limbs of a single call are stored past them too); in place (a plain
// inverse transform) the column pass that follows finds the stores in the last-level cache
template <int LOGN, class A> __device__ __forceinline__ void inv_blocks_wave(u64 *limb, unsigned bg, const A &ar, const BlockLane &b, bool stream)
{
    typename A::V v[8];
    inv_block_pass8(ar, v, b, [&](int m, unsigned i) { return block_twiddle<LOGN>(ar.twi, bg, m, i); });
    u64 *o = limb + bg * 256 + b.t;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        if (stream)
            __builtin_nontemporal_store(ar.store_mid(v[k]), o + 32 * k);
        else
            o[32 * k] = ar.store_mid(v[k]);
    }
}
// PAIR: the column pass has interleaved the rows; a wave's two blocks are a pair, so that the result may still go in their place.
// AHEAD (with an epilogue): twiddles and minuends are requested ahead of where they are used, which takes 88 registers, five waves per SIMD.  A rescale's
// launch that needs more waves than that to be resident at once asks for the minuends behind the transform, in 62 registers, eight waves.  N = 2^16, the
// kernel and a rescale that is waited for: 24 limbs 8.5 us ahead, 9.9 behind (43.8, 45.0), 38 13.4 and 13.3 (48.7, 48.8), 42 15.0 and 15.0 (50.4, 50.3), 48
// 17.4 and 15.3 (53.7, 52.2), 56 19.4 and 17.4 (56.7, 54.0), 736 193.5 and 191.3 (341, 339).  (16 elements per lane, four waves: 24 limbs 9.9, 48 14.1, 56 19.4, 736 195.)
#define FIN_AHEAD_GROUPS (5 * 256)
template <int LOGN, int EPI, bool PAIR, bool AHEAD, class A>
__device__ __forceinline__ void fwd_blocks_body(u64 *__restrict__ limb, const A &ar, u64 *lds, unsigned tile,
                                                const FinArgs &fa, const DevTables &T, unsigned slot)
{
    u64 *wlds = lds + wave_id() * WAVE_BLOCKS * TILE_GROUP;
    const BlockLane b = block_lane(wlds, nullptr);
    const unsigned b0 = tile * BLK_PER_WG + wave_id() * WAVE_BLOCKS, bg = b0 + b.blk; // block index within the limb
    BlockTwiddles<LOGN> tw;
    if constexpr (A::IS_FP && AHEAD) tw.first(ar.twf, b, bg);
    typename A::V a[8];
    u64x2 uv[EPI == EPI_STORE ? 1 : 4];
    const unsigned pos = b0 * 256 + 2u * (threadIdx.x & 63u); // of the first of this lane's pairs, 128 apart
    if (PAIR)
        mid_pairs8(ar, a, limb + b0 * 256, b);
    else {
#pragma unroll
        for (int k = 0; k < 8; k++) a[k] = ar.load_mid(__builtin_nontemporal_load(limb + bg * 256 + b.t + 32 * k)); // read once: the column pass wrote it
    }
    FinAt at = {0, 0, 0};
    const auto minuends = [&] {
        at = fin_at<LOGN>(fa, slot);
#pragma unroll
        for (int i = 0; i < 4; i++) uv[i] = fin_load(fa, at, pos + 128 * i);
    };
    if (EPI != EPI_STORE && AHEAD) minuends();
    if constexpr (A::IS_FP && AHEAD) {
        __builtin_amdgcn_sched_barrier(0);
        block_pass8(ar, a, b, bg, tw);
    } else
        block_pass8(ar, a, b, [&](int m, unsigned i) { return block_twiddle<LOGN>(ar.twf, bg, m, i); });
    if (EPI != EPI_STORE && !AHEAD) {
        __builtin_amdgcn_sched_barrier(0);
        minuends();
    }
    block_sync();
#pragma unroll
    for (int i = 0; i < 4; i++) {
        u64 *w = wlds + wave_pair_at(i);
        const u64x2 v = {ar.store_final(ar.load_mid(w[0])), ar.store_final(ar.load_mid(w[1]))};
        if (EPI == EPI_STORE)
            __builtin_nontemporal_store((u64x2u)v, (u64x2u *)(limb + pos + 128 * i));
        else {
            const u64x2 res = fin_value<A::IS_FP>(fa, T, at, v, uv[i]);
            if (EPI == EPI_FIN)
                fin_store<u64x2u>(fa, at, pos + 128 * i, res);
            else
                w[0] = res.x, w[1] = res.y;
        }
    }
    if constexpr (EPI == EPI_FIN_INV) {
        block_sync();
        inv_blocks_wave<LOGN>(fa.out + at.out, bg, ar, b, false);
    }
}

// PROD: the input is the product of `in` and `in2` (d2 = a1 b1 of a Mult, which is stored nowhere)
template <int LOGN, bool PROD, class A>
__device__ __forceinline__ void inv_blocks_body(const u64 *in, const u64 *in2, u64 *limb, const ModConst &m, const A &ar,
                                                u64 *lds, unsigned tile)
{
    u64 *wlds = lds + wave_id() * WAVE_BLOCKS * TILE_GROUP;
    const BlockLane b = block_lane(wlds, nullptr);
    const unsigned b0 = tile * BLK_PER_WG + wave_id() * WAVE_BLOCKS, pos = b0 * 256 + 2u * (threadIdx.x & 63u);
    u64x2 x[4], y[PROD ? 4 : 1];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        x[i] = __builtin_nontemporal_load((const u64x2u *)(in + pos + 128 * i)); // read once
        if (PROD) y[i] = __builtin_nontemporal_load((const u64x2u *)(in2 + pos + 128 * i));
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (PROD) x[i] = u64x2{mul_residues(x[i].x, y[i].x, m, ar), mul_residues(x[i].y, y[i].y, m, ar)};
        u64 *w = wlds + wave_pair_at(i);
        w[0] = x[i].x, w[1] = x[i].y;
    }
    block_sync();
    inv_blocks_wave<LOGN>(limb, b0 + b.blk, ar, b, in != limb);
}

// grid.x = (N / (256 BLK_PER_WG)) * batch
template <int LOGN, int EPI, bool PAIR, bool AHEAD>
__global__ __launch_bounds__(BLK_THREADS, 4) void k_ntt_fwd_blocks(u64 *__restrict__ data, DevTables T, LimbBatch lb, FinArgs fa)
{
    __shared__ __align__(16) u64 lds[BLK_LDS];
    constexpr unsigned TILES = (1u << LOGN) / (256 * BLK_PER_WG);
    const unsigned tile = blockIdx.x % TILES, b = blockIdx.x / TILES;
    const unsigned mi = lb.mod[b], slot = lb.slot[b];
    u64 *limb = data + ((size_t)slot << LOGN);
    if (T.mod[mi].qd != 0.0)
        fwd_blocks_body<LOGN, EPI, PAIR, AHEAD>(limb, make_fp(T, mi, LOGN), lds, tile, fa, T, slot);
    else
        fwd_blocks_body<LOGN, EPI, PAIR, AHEAD>(limb, make_int(T, mi, LOGN), lds, tile, fa, T, slot);
}

// src2: with PROD, the second factor, at the same limbs as src
template <int LOGN, bool PROD>
__global__ __launch_bounds__(BLK_THREADS, 4) void k_ntt_inv_blocks(const u64 *src, const u64 *src2, u64 *dst,
                                                        DevTables T, LimbBatch lb)
{
    __shared__ __align__(16) u64 lds[BLK_LDS];
    constexpr unsigned TILES = (1u << LOGN) / (256 * BLK_PER_WG);
    const unsigned tile = blockIdx.x % TILES, b = blockIdx.x / TILES;
    const unsigned mi = lb.mod[b];
    const ModConst m = T.mod[mi];
    const u64 *in = src + ((size_t)lb.src[b] << LOGN), *in2 = PROD ? src2 + ((size_t)lb.src[b] << LOGN) : nullptr;
    u64 *limb = dst + ((size_t)lb.slot[b] << LOGN);
    if (m.qd != 0.0)
        inv_blocks_body<LOGN, PROD>(in, in2, limb, m, make_fp(T, mi, LOGN), lds, tile);
    else
        inv_blocks_body<LOGN, PROD>(in, in2, limb, m, make_int(T, mi, LOGN), lds, tile);
}

// ---- column pass, N = 2^16 and 2^17: all rows x 16 columns per work-group (element (r, c) at r*256 + c) ---------
//
// N = 2^16: 256 rows, 16 elements per thread, stages 0-3 then 4-7.  N = 2^17: 512 rows, 32 elements per thread:
// stage 0 pairs the two halves of the rows, each half then takes stages 1-4 as a 16-element step, and after
// the exchange every thread runs stages 5-8 on two groups of 16 consecutive rows.

template <int LOGN> struct ColsGeom {
    static constexpr int ROWS = 1 << (LOGN - 8);
    static constexpr int HALVES = ROWS / 256;          // 16-element register steps per thread and phase
    static constexpr int LDS_WORDS = 16 * COL_GROUP;   // one half of the rows at a time: 32 KiB at either size
};

// the 16 inputs of one thread in rows rl + 16 k + 256 h (plain load or base conversion)
template <int PRO, int SPLIT, bool TINT, bool EX, int NSMAX, class A>
__device__ __forceinline__ void cols_inputs(typename A::V (&a)[16], const u64 *__restrict__ limb, unsigned col0, int h,
                                            const A &ar, const ConvSetup<NSMAX> &S, const ModConst &m)
{
    const unsigned rl = threadIdx.x >> 4, c = threadIdx.x & 15;
#pragma unroll
    for (int k = 0; k < 16; k++) {
        const unsigned pos = (rl + 16 * k + 256 * h) * 256 + col0 + c;
        a[k] = PRO == PRO_LOAD ? ar.load(__builtin_nontemporal_load(limb + pos)) : conv_get<PRO, SPLIT, TINT, EX>(S, ar, m, pos);
    }
}
// second phase of the forward column pass for rows 16 g .. 16 g + 15, held in LDS as group gl.  With a prologue the
// output is a new buffer that a later kernel reads, so it is stored past the sources that stay in L2
template <int S_BASE, int PRO, class A>
__device__ __forceinline__ void cols_finish_group(typename A::V (&a)[16], u64 *__restrict__ limb, unsigned col0, unsigned g,
                                                  unsigned gl, const A &ar, const u64 *lds)
{
    const unsigned c = threadIdx.x & 15;
#pragma unroll
    for (int k = 0; k < 16; k++) a[k] = ar.load_mid(lds[col_at(16 * gl + k, c)]);
    ar.fwd16(a, S_BASE, g, true);
    if constexpr (pro_pairs_rows(PRO)) {
#pragma unroll
        for (int k = 0; k < 16; k += 2)
            __builtin_nontemporal_store(u64x2{ar.store_mid(a[k]), ar.store_mid(a[k + 1])}, (u64x2 *)(limb + mid_at<true>(16 * g + k, col0 + c)));
        return;
    }
#pragma unroll
    for (int k = 0; k < 16; k++) { // the block pass finishes
        u64 *dst = limb + (16 * g + k) * 256 + col0 + c;
        if (PRO != PRO_LOAD)
            __builtin_nontemporal_store(ar.store_mid(a[k]), dst);
        else
            *dst = ar.store_mid(a[k]);
    }
}

template <int LOGN, int PRO, int SPLIT, bool TINT, bool EX, int NSMAX, class A>
__device__ __forceinline__ void fwd_cols_body(u64 *__restrict__ limb, unsigned col0, const A &ar, u64 *lds,
                                              const ConvSetup<NSMAX> &S, const ModConst &m)
{
    constexpr int H = ColsGeom<LOGN>::HALVES;
    const unsigned rl = threadIdx.x >> 4, c = threadIdx.x & 15;
    typename A::V a0[16];
    cols_inputs<PRO, SPLIT, TINT, EX>(a0, limb, col0, 0, ar, S, m);
    if (H == 1) {
        ar.fwd16(a0, 0, 0, PRO != PRO_LOAD);
#pragma unroll
        for (int k = 0; k < 16; k++) lds[col_at(rl + 16 * k, c)] = ar.store_mid(a0[k]);
        __syncthreads();
        cols_finish_group<4, PRO>(a0, limb, col0, rl, rl, ar, lds);
    } else {
        typename A::V a1[16];
        // one half's source loads at a time: 32 outputs x up to 8 sources in flight would not fit the registers
        if (PRO != PRO_LOAD) __builtin_amdgcn_sched_barrier(0);
        cols_inputs<PRO, SPLIT, TINT, EX>(a1, limb, col0, 1, ar, S, m);
        ar.fwd_stage0(a0, a1, PRO != PRO_LOAD);
        ar.fwd16(a0, 1, 0, true);
        ar.fwd16(a1, 1, 1, true);
        // after stage 0 the two halves of the rows are independent: they go through the same 32 KiB of LDS in turn
#pragma unroll
        for (int k = 0; k < 16; k++) lds[col_at(rl + 16 * k, c)] = ar.store_mid(a0[k]);
        __syncthreads();
        cols_finish_group<5, PRO>(a0, limb, col0, rl, rl, ar, lds);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k++) lds[col_at(rl + 16 * k, c)] = ar.store_mid(a1[k]);
        __syncthreads();
        cols_finish_group<5, PRO>(a1, limb, col0, rl + 16, rl, ar, lds);
    }
}

// CACHED: a plain transform of at most INV_CACHED bytes, whose values the block pass has left in the last-level cache; a plain load keeps them
// there for the stores.  Larger launches stream through it (64 limbs of N = 2^16 32.8 us with plain loads, 34.0 with nontemporal ones, 150 66.2 and
// 64.8, 256 115 and 106; 34 of N = 2^17 40.3 and 42.0, 80 78.7 and 77.2; on buffers in turn, 1.5 GiB of them, 28 limbs of N = 2^16 22.3 and 22.8,
// 64 34.3 and 35.4, 120 57.2 and 58.0, 34 of N = 2^17 43.0 and 43.6, 60 62.4 and 63.4, 20 and fewer the same; limbs met for the first time, waited
// for, 34 of N = 2^17 60.8 and 63.1).
#define INV_CACHED (64ull << 20)
template <int LOGN, bool CACHED, class A>
__device__ __forceinline__ void inv_cols_body(u64 *__restrict__ limb, unsigned col0, const A &ar, u64 *lds)
{
    constexpr int H = ColsGeom<LOGN>::HALVES;
    const unsigned rl = threadIdx.x >> 4, c = threadIdx.x & 15;
    typedef typename A::V V;
    V a[H][16];
    // each half of the rows: stages logN-9 .. logN-12 on 16 consecutive rows, exchange through the same 32 KiB of
    // LDS, then stages 3 .. 0 (N = 2^16) or 4 .. 1 (N = 2^17: stage 0 pairs the halves afterwards).  Written as two calls:
    // as a loop it is too large for the compiler to unroll, and the values, indexed by the half, go to scratch memory.
    // N = 2^17 (two or three work-groups per compute unit): a step's twiddles are loaded by themselves, ahead of the values, else they come
    // late, and the limbs on the integer path with them; the second half's values are on their way behind the first half's first
    // step.  34 limbs, both passes: 40.0 us (41.6 with the values of both halves ahead of everything, 40.7 with the second half's in its
    // turn); 4 limbs: 16.3 (16.8 in its turn)
    const auto values = [&](V (&v)[16], int h) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const u64 *src = limb + (16 * (rl + 16 * h) + k) * 256 + col0 + c;
            v[k] = ar.load_mid(CACHED ? *src : __builtin_nontemporal_load(src)); // the block pass wrote it
        }
    };
    const auto half = [&](V (&v)[16], int h) __attribute__((always_inline)) {
        const unsigned g = rl + 16 * h;
        typename A::W tw[15];
        if (H == 2) {
#pragma unroll
            for (int t = 0; t < 15; t++) tw[t] = ar.twi[step16_twiddle(H + 3, g, (unsigned)t)];
        }
        if (h == 0) values(v, 0);
        if (H == 2)
            ar.template inv16_with<false>(v, [&](int t) { return tw[t]; });
        else
            ar.template inv16<false>(v, H + 3, g);
        if (H == 2 && h == 0) {
            values(a[H - 1], 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (h > 0) __syncthreads(); // the previous half has been read back by every thread
#pragma unroll
        for (int k = 0; k < 16; k++) lds[col_at(16 * rl + k, c)] = ar.store_mid(v[k]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] = ar.load_mid(lds[col_at(rl + 16 * k, c)]);
        if (H == 1)
            ar.template inv16<true>(v, 0, 0);
        else
            ar.template inv16<false>(v, 1, h);
    };
    half(a[0], 0);
    if constexpr (H == 2) half(a[H - 1], 1);
    if (H == 2) ar.inv_stage0_last(a[0], a[H - 1]);
#pragma unroll
    for (int h = 0; h < H; h++)
#pragma unroll
        for (int k = 0; k < 16; k++) limb[(rl + 16 * k + 256 * h) * 256 + col0 + c] = ar.store_final(a[h][k]);
}

// column pass of limb b of the launch (the arithmetic path and the prologue's variant follow from its modulus)
template <int LOGN, int PRO, int NSMAX, bool EX>
__device__ __forceinline__ void fwd_cols_limb(u64 *__restrict__ data, const DevTables &T, const LimbBatch &lb,
                                              const ConvArgs &cv, unsigned tile, unsigned b, u64 *lds)
{
    const unsigned mi = lb.mod[b], slot = lb.slot[b];
    u64 *limb = data + ((size_t)slot << LOGN);
    const ModConst m = T.mod[mi];
    const ConvSetup<NSMAX> S = conv_setup<PRO, NSMAX, LOGN>(cv, T, slot, mi);
    const bool split = PRO == PRO_MODUP ? T.up_split != 0 : pro_is_moddown(PRO) ? T.dn_split != 0 : false;
    const bool fold = pro_is_moddown(PRO) && !EX && NSMAX <= 4 && T.dn_fold != 0; // the common case only: each variant costs code
    const bool tint = PRO == PRO_MODDOWN_RS && S.qld == 0.0; // dropped limb on the integer path
    if (m.qd == 0.0)
        fwd_cols_body<LOGN, PRO, 0, false, EX>(limb, tile * 16, make_int(T, mi, LOGN), lds, S, m);
    else if (PRO == PRO_MODDOWN_RS && tint) {
        if (split)
            fwd_cols_body<LOGN, PRO, 1, PRO == PRO_MODDOWN_RS, EX>(limb, tile * 16, make_fp(T, mi, LOGN), lds, S, m);
        else
            fwd_cols_body<LOGN, PRO, 0, PRO == PRO_MODDOWN_RS, EX>(limb, tile * 16, make_fp(T, mi, LOGN), lds, S, m);
    } else if (fold)
        fwd_cols_body<LOGN, PRO, pro_is_moddown(PRO) && !EX && NSMAX <= 4 ? 2 : 0, false, EX>(limb, tile * 16, make_fp(T, mi, LOGN), lds, S, m);
    else if (split)
        fwd_cols_body<LOGN, PRO, 1, false, EX>(limb, tile * 16, make_fp(T, mi, LOGN), lds, S, m);
    else
        fwd_cols_body<LOGN, PRO, 0, false, EX>(limb, tile * 16, make_fp(T, mi, LOGN), lds, S, m);
}
template <int LOGN, int PRO, int NSMAX, bool EX>
__device__ __forceinline__ void fwd_cols_kernel(u64 *__restrict__ data, const DevTables &T, const LimbBatch &lb,
                                                const ConvArgs &cv)
{
    __shared__ u64 lds[ColsGeom<LOGN>::LDS_WORDS];
    fwd_cols_limb<LOGN, PRO, NSMAX, EX>(data, T, lb, cv, blockIdx.x & 15, blockIdx.x >> 4, lds);
}

// ModUp column pass of the corrected conversion for two limbs per work-group (N = 2^16; grid.x = 16 * ceil(batch / 2)): limbs 2i and 2i+1 of
// the launch.  When both are floating-point targets of the same digit of the same operation (the usual case:
// the targets of a digit follow each other in a launch), the digit's source limbs are read and converted to
// doubles once and both base conversions are formed from them, term by term as in conv_get; every target
// otherwise re-reads the same source tile through L2.  Any other pair is processed one limb after the other.
template <int NSMAX>
__global__ __launch_bounds__(256) void k_ntt_fwd_cols16_modup2(u64 *__restrict__ data, DevTables T, LimbBatch lb,
                                                                ConvArgs cv, int nb)
{
    __shared__ u64 lds[ColsGeom<16>::LDS_WORDS];
    const unsigned tile = blockIdx.x & 15, b0 = (blockIdx.x >> 4) * 2, b1 = b0 + 1;
    if (b1 >= (unsigned)nb) {
        fwd_cols_limb<16, PRO_MODUP, NSMAX, true>(data, T, lb, cv, tile, b0, lds);
        return;
    }
    const unsigned mi0 = lb.mod[b0], mi1 = lb.mod[b1], slot0 = lb.slot[b0], slot1 = lb.slot[b1];
    const ConvSetup<NSMAX> S0 = conv_setup<PRO_MODUP, NSMAX, 16>(cv, T, slot0, mi0);
    const ConvSetup<NSMAX> S1 = conv_setup<PRO_MODUP, NSMAX, 16>(cv, T, slot1, mi1);
    bool same = T.up_split == 0 && T.mod[mi0].qd != 0.0 && T.mod[mi1].qd != 0.0;
#pragma unroll
    for (int s = 0; s < NSMAX; s++) same = same && S0.sp[s] == S1.sp[s];
    if (!same) {
        fwd_cols_limb<16, PRO_MODUP, NSMAX, true>(data, T, lb, cv, tile, b0, lds);
        __syncthreads(); // the first limb's second phase has read the tile
        fwd_cols_limb<16, PRO_MODUP, NSMAX, true>(data, T, lb, cv, tile, b1, lds);
        return;
    }
    const ArithFp ar0 = make_fp(T, mi0, 16), ar1 = make_fp(T, mi1, 16);
    const unsigned rl = threadIdx.x >> 4, c = threadIdx.x & 15, col0 = tile * 16;
    double a0[16], a1[16];
#pragma unroll
    for (int k = 0; k < 16; k++) {
        const unsigned pos = (rl + 16 * k) * 256 + col0 + c;
        double acc0 = 0.0, acc1 = 0.0, sv = 0.0;
#pragma unroll
        for (int s = 0; s < NSMAX; s++) {
            const double y = u2d(S0.sp[s][pos]);
            sv = sv + y * S0.rq[s];
            acc0 += ar0.mulmod(y, S0.cd[s]);
            acc1 += ar1.mulmod(y, S1.cd[s]);
            if ((s & 3) == 3 && s + 1 < NSMAX) acc0 = ar0.reduce(acc0), acc1 = ar1.reduce(acc1);
        }
        const double v = __builtin_floor(sv); // one estimate of the multiple of D for both targets
        a0[k] = acc0 - v * S0.dm_d, a1[k] = acc1 - v * S1.dm_d;
    }
    u64 *limb0 = data + ((size_t)slot0 << 16), *limb1 = data + ((size_t)slot1 << 16);
    ar0.fwd16(a0, 0, 0, true);
#pragma unroll
    for (int k = 0; k < 16; k++) lds[col_at(rl + 16 * k, c)] = ar0.store_mid(a0[k]);
    __syncthreads();
    cols_finish_group<4, PRO_MODUP>(a0, limb0, col0, rl, rl, ar0, lds);
    __syncthreads();
    ar1.fwd16(a1, 0, 0, true);
#pragma unroll
    for (int k = 0; k < 16; k++) lds[col_at(rl + 16 * k, c)] = ar1.store_mid(a1[k]);
    __syncthreads();
    cols_finish_group<4, PRO_MODUP>(a1, limb1, col0, rl, rl, ar1, lds);
}
// grid.x = 16 * batch
// EX: the corrected conversions (a kernel of its own: their extra registers would cost the default form waves)
template <int PRO, int NSMAX, bool EX>
__global__ __launch_bounds__(256) void k_ntt_fwd_cols16(u64 *__restrict__ data, DevTables T, LimbBatch lb, ConvArgs cv)
{
    fwd_cols_kernel<16, PRO, NSMAX, EX>(data, T, lb, cv);
}
template <int PRO, int NSMAX, bool EX>
__global__ __launch_bounds__(256) void k_ntt_fwd_cols17(u64 *__restrict__ data, DevTables T, LimbBatch lb, ConvArgs cv)
{
    fwd_cols_kernel<17, PRO, NSMAX, EX>(data, T, lb, cv);
}

// extra constant of the inverse column pass for modulus index mi
__device__ __forceinline__ void scale_consts(int scale, const ConvArgs &cv, const DevTables &T, unsigned mi, unsigned slot,
                                             ShoupConst &ci, double &cd)
{
    ci = ShoupConst{0, 0};
    cd = 0.0;
    if (scale == SCALE_MODUP) {
        const int j = mi / cv.alpha, ii = mi - j * cv.alpha;
        const int na = min(cv.alpha, conv_op_level(cv, slot) - j * cv.alpha);
        const size_t idx = ((size_t)j * cv.alpha + (na - 1)) * cv.alpha + ii;
        ci = T.up_inv[idx];
        cd = T.up_inv_d[idx];
    } else if (scale == SCALE_MODDOWN) {
        ci = T.dn_inv[mi - cv.L];
        cd = T.dn_inv_d[mi - cv.L];
    }
}

template <int LOGN, int SCALE, bool CACHED>
__device__ __forceinline__ void inv_cols_kernel(u64 *__restrict__ data, const DevTables &T, const LimbBatch &lb,
                                                const ConvArgs &cv)
{
    __shared__ u64 lds[ColsGeom<LOGN>::LDS_WORDS];
    const unsigned tile = blockIdx.x & 15, b = blockIdx.x >> 4;
    const unsigned mi = lb.mod[b];
    u64 *limb = data + ((size_t)lb.slot[b] << LOGN);
    ShoupConst ci;
    double cd;
    scale_consts(SCALE, cv, T, mi, lb.slot[b], ci, cd);
    if (T.mod[mi].qd != 0.0)
        inv_cols_body<LOGN, CACHED>(limb, tile * 16, make_fp(T, mi, LOGN, cd), lds);
    else
        inv_cols_body<LOGN, CACHED>(limb, tile * 16, make_int(T, mi, LOGN, ci), lds);
}
template <int SCALE, bool CACHED>
__global__ __launch_bounds__(256) void k_ntt_inv_cols16(u64 *__restrict__ data, DevTables T, LimbBatch lb, ConvArgs cv)
{
    inv_cols_kernel<16, SCALE, CACHED>(data, T, lb, cv);
}
template <int SCALE, bool CACHED>
__global__ __launch_bounds__(256, 3) void k_ntt_inv_cols17(u64 *__restrict__ data, DevTables T, LimbBatch lb, ConvArgs cv)
{
    inv_cols_kernel<17, SCALE, CACHED>(data, T, lb, cv);
}
