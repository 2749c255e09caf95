// Kernels of the ring size N = 2^12: a limb is 32 KiB and fits the LDS of one compute unit, so one work-group of 512
// threads, 8 elements each, runs a whole transform (four steps of three stages), and a key switch is four launches:
//   1. inverse transform of the input limbs, scaled                                  (k_ntt_inv12<SCALE_MODUP>)
//   2. ModUp and forward transform of every raised limb                                 (k_ntt_fwd12<PRO_MODUP>)
//   3. per active limb (and component, but for a rotation's ciphertext limbs): inner product u, for special limbs its inverse transform, scaled (k_inner12)
//   4. per ciphertext limb and component: ModDown correction, its forward transform, (u - r) * const + addend (k_fin12)
// and one more for Mult with rescale, which finishes the dropped limb between 3 and 4 (k_fin12 with DROP).
//
// Single calls are bound neither by memory nor by instructions: a launch is a chain of dependent steps on few
// work-groups, so what counts is the number of launches and the length of the chain in each.  With two launches per
// transform (column pass, block pass) and the digits finished inside the inner product, one rotation (three primes, one
// special prime) took seven launches of 4 to 10 us, 46 us in all; it takes 28 now, and eight
// transforms 7.3 to 8.4 us, the host's time for one call, instead of 11.5.  The chain is kept short by fetching a step's
// twiddles before the step ahead of it is worked on, by giving every component that is transformed a work-group of its own, and by short
// code: a launch runs it once, and with 256 threads of 16 elements, twice the instructions, it took 37 us (the
// finishing kernel 14.9).  Batches are bound by memory and by how many work-groups are resident: at most 128 registers keep two
// per compute unit (64 rotations of 24 primes, with k_fin12 at 137 and the digits read once per component, took 572 us against
// 510 in two passes per transform; 511 now.  1024 of three primes: 778, 685 and 659).
#pragma once
#include "kernels_ks.h"

#define N12_THREADS 512
#define N12_LDS (4096 + 256)
// Word of element e in LDS: one pad word per 16 keeps the patterns below free of most bank conflicts.
__device__ __forceinline__ unsigned at12(unsigned e) { return e + (e >> 4); }
// A thread's elements in step i (stages 3 i .. 3 i + 2): base + k * 2^SH, k < 8, with SH = 9 - 3 i.  From step 1 on the 64
// lanes of a wave own an aligned group of 512 elements, so that only the exchange behind step 0 crosses waves.
template <int SH> __device__ __forceinline__ unsigned base12()
{
    return (threadIdx.x >> SH) << (SH + 3) | (threadIdx.x & ((1u << SH) - 1u));
}
// offset of element k from the base, in LDS words: linear in k but for SH = 3, where every second k passes a pad word
template <int SH> __device__ __forceinline__ constexpr unsigned step12(int k)
{
    return SH >= 4 ? (unsigned)k * ((1u << SH) + (1u << SH >> 4)) : SH == 3 ? 8u * k + (k >> 1) : (unsigned)k;
}
// A thread's elements where limbs are read and written in the NTT domain: step 1's.
#define N12_BASE base12<6>()

// twiddles of the 8-element step that starts at stage s_base in group G
template <class A> struct Step8 {
    typename A::W w[7];
    __device__ __forceinline__ Step8(const typename A::W *tw, unsigned s_base, unsigned G)
    {
#pragma unroll
        for (int c = 0; c < 7; c++) w[c] = tw[step16_twiddle(s_base, G, (unsigned)c)];
    }
    __device__ __forceinline__ typename A::W operator()(int sp, int g) const { return w[(1 << sp) - 1 + g]; }
};
template <int SH, class A> __device__ __forceinline__ void put12(const typename A::V (&a)[8], const A &ar, u64 *lds)
{
    u64 *p = lds + at12(base12<SH>());
#pragma unroll
    for (int k = 0; k < 8; k++) p[step12<SH>(k)] = ar.store_mid(a[k]);
}
template <int SH, class A> __device__ __forceinline__ void get12(typename A::V (&a)[8], const A &ar, const u64 *lds)
{
    const u64 *p = lds + at12(base12<SH>());
#pragma unroll
    for (int k = 0; k < 8; k++) a[k] = ar.load_mid(p[step12<SH>(k)]);
}

// Forward transform: a[k] = element 512 k + thread (of the range that fwd8_with takes); v: the canonical result at
// elements N12_BASE + 64 k.
template <class A> __device__ __forceinline__ void fwd12(typename A::V (&a)[8], u64 (&v)[8], const A &ar, u64 *lds, bool reduce_first)
{
    const unsigned t = threadIdx.x;
    const Step8<A> w0(ar.twf, 0, 0), w1(ar.twf, 3, t >> 6);
    ar.fwd8_with(a, reduce_first, w0);
    put12<9>(a, ar, lds);
    const Step8<A> w2(ar.twf, 6, t >> 3);
    __syncthreads();
    get12<6>(a, ar, lds);
    ar.fwd8_with(a, true, w1);
    const Step8<A> w3(ar.twf, 9, t);
    block_sync();
    put12<6>(a, ar, lds);
    block_sync();
    get12<3>(a, ar, lds);
    ar.fwd8_with(a, true, w2);
    block_sync();
    put12<3>(a, ar, lds);
    block_sync();
    get12<0>(a, ar, lds);
    ar.fwd8_with(a, true, w3);
    block_sync();
    u64 *p = lds + at12(base12<0>());
#pragma unroll
    for (int k = 0; k < 8; k++) p[k] = ar.store_final(a[k]);
    block_sync();
    const u64 *r = lds + at12(N12_BASE);
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = r[step12<6>(k)];
}

// Inverse transform of canonical values v[k] = element N12_BASE + 64 k; stores the finished limb.
template <class A> __device__ __forceinline__ void inv12(const u64 (&v)[8], u64 *limb, const A &ar, u64 *lds)
{
    const unsigned t = threadIdx.x;
    const Step8<A> w3(ar.twi, 9, t), w2(ar.twi, 6, t >> 3);
    typename A::V a[8];
    block_sync(); // the wave has read what it overwrites
    u64 *p = lds + at12(N12_BASE);
#pragma unroll
    for (int k = 0; k < 8; k++) p[step12<6>(k)] = v[k];
    block_sync();
    const u64 *r = lds + at12(base12<0>());
#pragma unroll
    for (int k = 0; k < 8; k++) a[k] = ar.load(r[k]);
    ar.template inv8_with<false>(a, w3);
    const Step8<A> w1(ar.twi, 3, t >> 6), w0(ar.twi, 0, 0);
    block_sync();
    put12<0>(a, ar, lds);
    block_sync();
    get12<3>(a, ar, lds);
    ar.template inv8_with<false>(a, w2);
    block_sync();
    put12<3>(a, ar, lds);
    block_sync();
    get12<6>(a, ar, lds);
    ar.template inv8_with<false>(a, w1);
    block_sync();
    put12<6>(a, ar, lds);
    __syncthreads();
    get12<9>(a, ar, lds);
    ar.template inv8_with<true>(a, w0);
#pragma unroll
    for (int k = 0; k < 8; k++) limb[k * 512 + t] = ar.store_final(a[k]);
}

// Calls f(arithmetic, split, tint) with the variant of the prologue that modulus and tables ask for (split, tint: types
// whose `value` is the template argument of conv_get).  INTS false: no limb of the launch, nor one that is dropped, is on the integer path.
template <int PRO, int NSMAX, bool EX, bool INTS, class F>
__device__ __forceinline__ void conv_variant12(const DevTables &T, unsigned mi, const ModConst &m, double qld, F f)
{
    constexpr bool MD = pro_is_moddown(PRO), FOLD = MD && !EX && NSMAX <= 4;
    const bool split = PRO == PRO_MODUP ? T.up_split != 0 : MD ? T.dn_split != 0 : false;
    if (INTS && m.qd == 0.0) {
        if constexpr (INTS) f(make_int(T, mi, 12), std::integral_constant<int, 0>{}, std::false_type{});
    } else if (INTS && PRO == PRO_MODDOWN_RS && qld == 0.0) { // dropped limb on the integer path
        if (split)
            f(make_fp(T, mi, 12), std::integral_constant<int, 1>{}, std::integral_constant<bool, INTS && PRO == PRO_MODDOWN_RS>{});
        else
            f(make_fp(T, mi, 12), std::integral_constant<int, 0>{}, std::integral_constant<bool, INTS && PRO == PRO_MODDOWN_RS>{});
    } else if (FOLD && T.dn_fold != 0)
        f(make_fp(T, mi, 12), std::integral_constant<int, FOLD ? 2 : 0>{}, std::false_type{});
    else if (split)
        f(make_fp(T, mi, 12), std::integral_constant<int, 1>{}, std::false_type{});
    else
        f(make_fp(T, mi, 12), std::integral_constant<int, 0>{}, std::false_type{});
}

// Column inputs of the forward transform of the limb at `limb` / of the conversion S.
template <int PRO, int SPLIT, bool TINT, bool EX, int NSMAX, class A>
__device__ __forceinline__ void inputs12(typename A::V (&a)[8], const u64 *limb, const A &ar, const ConvSetup<NSMAX> &S,
                                         const ModConst &m)
{
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const unsigned pos = k * 512 + threadIdx.x;
        a[k] = PRO == PRO_LOAD ? ar.load(limb[pos]) : conv_get<PRO, SPLIT, TINT, EX>(S, ar, m, pos);
    }
}

// grid.x = limbs
template <int PRO, int NSMAX, bool EX, int EPI>
__global__ __launch_bounds__(N12_THREADS, EPI == EPI_FIN ? 4 : 1) void k_ntt_fwd12(u64 *data, DevTables T, LimbBatch lb, ConvArgs cv, FinArgs fa)
{
    __shared__ u64 lds[N12_LDS];
    const unsigned mi = lb.mod[blockIdx.x], slot = lb.slot[blockIdx.x], nb = N12_BASE;
    u64 *limb = data + ((size_t)slot << 12);
    const ModConst m = T.mod[mi];
    const ConvSetup<NSMAX> S = conv_setup<PRO, NSMAX, 12>(cv, T, slot, mi);
    u64 uv[EPI == EPI_FIN ? 8 : 1];
    FinAt at = {0, 0, 0};
    if (EPI == EPI_FIN) {
        at = fin_at<12>(fa, slot);
#pragma unroll
        for (int k = 0; k < 8; k++) uv[k] = __builtin_nontemporal_load(fa.u + at.u + nb + 64 * k);
    }
    conv_variant12<PRO, NSMAX, EX, true>(T, mi, m, S.qld, [&](auto ar, auto split, auto tint) {
        typedef decltype(ar) A;
        typename A::V a[8];
        inputs12<PRO, decltype(split)::value, decltype(tint)::value, EX>(a, limb, ar, S, m);
        u64 v[8];
        fwd12(a, v, ar, lds, PRO != PRO_LOAD);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const unsigned pos = nb + 64 * k;
            if (EPI == EPI_FIN)
                fin_store(fa, at, pos, fin_value<A::IS_FP>(fa, T, at, v[k], uv[k]));
            else
                limb[pos] = v[k];
        }
    });
}

// grid.x = limbs; in place where src and dst are the same buffer and slots (a work-group has read its limb before it stores)
// src2: null, or a second factor of the input
template <int SCALE>
__global__ __launch_bounds__(N12_THREADS) void k_ntt_inv12(const u64 *src, const u64 *src2, u64 *dst, DevTables T, LimbBatch lb, ConvArgs cv)
{
    __shared__ u64 lds[N12_LDS];
    const unsigned mi = lb.mod[blockIdx.x], slot = lb.slot[blockIdx.x], nb = N12_BASE;
    const u64 *in = src + ((size_t)lb.src[blockIdx.x] << 12);
    u64 *limb = dst + ((size_t)slot << 12);
    u64 v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = in[nb + 64 * k];
    ShoupConst ci;
    double cd;
    scale_consts(SCALE, cv, T, mi, slot, ci, cd);
    const ModConst m = T.mod[mi];
    const auto run = [&](auto ar) {
        if (src2) {
            const u64 *in2 = src2 + ((size_t)lb.src[blockIdx.x] << 12);
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] = mul_residues(v[k], in2[nb + 64 * k], m, ar);
        }
        inv12(v, limb, ar, lds);
    };
    if (m.qd != 0.0)
        run(make_fp(T, mi, 12, cd));
    else
        run(make_int(T, mi, 12, ci));
}

// What a work-group of the inner product works on: active limb a of operation op, from component c on.
struct Inner12 {
    unsigned op, g;
    int a, c, level, beta;
    bool none;
};
__device__ __forceinline__ Inner12 inner12_of(const InnerArgs &ia, const OpArgs &oa, unsigned op, int a, int c)
{
    Inner12 w;
    w.op = op, w.c = c, w.a = a;
    w.g = ia.per_op ? oa.g[w.op] : ia.g;
    w.level = ia.per_op && oa.level[w.op] ? oa.level[w.op] : ia.level;
    w.beta = (w.level + ia.alpha - 1) / ia.alpha;
    w.none = w.a < ia.level && w.a >= w.level; // an operation below the layout's level
    return w;
}
// Element n of d2 (g = 1) and of d0, d1 for Mult, of the C components from w.c on, canonical residues.
template <int C, class A>
__device__ __forceinline__ void tensor12(const InnerArgs &ia, const Inner12 &w, unsigned n, const ModConst &m, const A &ar, u64 (&d)[C], u64 &d2)
{
    const size_t c0 = (((size_t)w.op * ia.t_stride + w.a) << 12) + n, c1 = c0 + ((size_t)ia.level << 12);
    d2 = mul_residues(ia.ta[c1], ia.tb[c1], m, ar);
#pragma unroll
    for (int c = 0; c < C; c++) {
        if (w.c + c == 0)
            d[c] = mul_residues(ia.ta[c0], ia.tb[c0], m, ar);
        else
            d[c] = csub(mul_residues(ia.ta[c0], ia.tb[c1], m, ar) + mul_residues(ia.ta[c1], ia.tb[c0], m, ar), m.q);
    }
}
// u of the C components from w.c on at elements N12_BASE + 64 k, for Mult with P times d0 or d1: on the floating-point path within 4.3 q of
// zero (not canonical), as a double; canonical residues on the integer path.
template <int C, bool MULT, class A>
__device__ __forceinline__ void inner12(typename A::V (&r)[C][8], const InnerArgs &ia, const OpArgs &oa, const DevTables &T, const Inner12 &w, unsigned mi,
                                        const A &ar, const ModConst &m)
{
    const unsigned nb = N12_BASE;
    constexpr int PART = 8 / C; // elements at a time: as many loads in flight and 128-bit sums with two components as with one
    const int own = w.a < ia.level ? w.a / ia.alpha : -1, M = ia.L + ia.K, Ma = ia.level + ia.K;
    const u64 *key0 = (ia.per_op ? oa.evk[w.op] : ia.evk) + (((size_t)w.c * M + mi) << 12);
    const size_t comp_words = (size_t)M << 12;
    const u64 *dig0 = ia.raised + (((size_t)w.op * ia.raised_stride + w.a) << 12);
    const u64 *d_limb = (ia.per_op && oa.d[w.op] ? oa.d[w.op] : ia.d + (((size_t)w.op * ia.d_stride) << 12)) + ((size_t)w.a << 12);
    unsigned sr[8];
#pragma unroll
    for (int k = 0; k < 8; k++) sr[k] = MULT || w.g == 1 ? nb + 64 * k : galois_index(nb + 64 * k, w.g, 12); // a Mult's g is 1
    if constexpr (A::IS_FP) {
#pragma unroll
        for (int c = 0; c < C; c++)
#pragma unroll
            for (int k = 0; k < 8; k++) r[c][k] = 0.0;
        if (MULT && own >= 0) { // the digit's own limb: few elements in flight, each takes four factors
            const u64 *kj = key0 + (((size_t)own * 2 * M) << 12);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                u64 d[C], x;
                tensor12<C>(ia, w, nb + 64 * k, m, ar, d, x);
#pragma unroll
                for (int c = 0; c < C; c++)
                    r[c][k] = ar.mulmod(u2d(d[c]), T.dn_pmod_d[w.a]) + ar.mulmod(u2d(x), ar.load_mid(kj[c * comp_words + nb + 64 * k]));
            }
        }
        for (int j = 0; j < w.beta; j++) {
            const u64 *dj = j == own ? d_limb : dig0 + (((size_t)j * Ma) << 12), *kj = key0 + (((size_t)j * 2 * M) << 12);
            if (!(MULT && j == own)) {
#pragma unroll
                for (int p = 0; p < 8; p += PART) {
                    u64 x[PART], e[C][PART];
#pragma unroll
                    for (int c = 0; c < C; c++)
#pragma unroll
                        for (int k = 0; k < PART; k++) e[c][k] = kj[c * comp_words + nb + 64 * (p + k)];
#pragma unroll
                    for (int k = 0; k < PART; k++) x[k] = dj[sr[p + k]];
#pragma unroll
                    for (int c = 0; c < C; c++)
#pragma unroll
                        for (int k = 0; k < PART; k++) r[c][p + k] += ar.mulmod(u2d(x[k]), ar.load_mid(e[c][k])); // key words are balanced doubles
                }
            }
            if ((j & 3) == 3) {
#pragma unroll
                for (int c = 0; c < C; c++)
#pragma unroll
                    for (int k = 0; k < 8; k++) r[c][k] = ar.reduce(r[c][k]);
            }
        }
    } else {
        static_assert(C == 1, "128-bit sums: one component at a time");
        U128 acc[8];
#pragma unroll
        for (int k = 0; k < 8; k++) acc[k] = U128{0, 0};
        for (int j = 0; j < w.beta; j++) {
            const u64 *dj = j == own ? d_limb : dig0 + (((size_t)j * Ma) << 12), *kj = key0 + (((size_t)j * 2 * M) << 12);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                u64 x;
                if (MULT && j == own) {
                    u64 d[1];
                    tensor12<1>(ia, w, nb + 64 * k, m, ar, d, x);
                    mac128(acc[k], d[0], T.dn_pmod[w.a]);
                } else
                    x = dj[sr[k]];
                mac128(acc[k], x, kj[nb + 64 * k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 8; k++) r[0][k] = reduce128(acc[k], m);
    }
}

// u of the ciphertext limbs, and of the special ones (the longest work, first) the inverse transform, scaled by (P/p_k)^-1.  All
// limbs in one launch: formed in k_fin12, u would add its chain of loads, a round per digit, to the longest kernel.
// Rotations: grid (level + 2 K, 1, operations); a work-group makes both components of a ciphertext limb, so that its digits are read
// once, or one of a special limb.  With one component per work-group everywhere, 1024 rotations of three primes took 715 us instead of 667,
// 128 of 24 primes 1025 instead of 997, a single one of 24 primes 50.3 instead of 47.8 (three primes: the same within 0.5 us).
// MULT (the switched polynomial is a product, InnerArgs.ta): grid (level + K, 2, operations), one component per work-group: with the factors
// of both components the registers of two work-groups per compute unit do not suffice (16 products of three primes 41.3 -> 45.5 us).
template <bool MULT> __global__ __launch_bounds__(N12_THREADS, 4) void k_inner12(InnerArgs ia, DevTables T, OpArgs oa)
{
    constexpr bool BOTH = !MULT;
    __shared__ u64 lds[N12_LDS];
    const unsigned nb = N12_BASE;
    unsigned unit = blockIdx.x, c0 = blockIdx.y;
    if constexpr (BOTH) {
        c0 = unit < 2u * ia.K ? unit & 1u : 0;
        unit = unit < 2u * ia.K ? unit >> 1 : unit - ia.K;
    }
    Inner12 w = inner12_of(ia, oa, blockIdx.z, (int)unit < ia.K ? ia.level + (int)unit : (int)unit - ia.K, (int)c0);
    if (w.none) return;
    const bool special = w.a >= ia.level;
    const unsigned mi = active_mod(w.a, ia.level, ia.L), k_sp = special ? w.a - ia.level : 0;
    const ModConst m = T.mod[mi];
    const size_t comp_words = (size_t)(ia.level + ia.K) << 12;
    u64 *limb = ia.u + (((size_t)w.op * ia.u_stride + w.a) << 12) + w.c * comp_words;
    const auto store = [&](const u64 (&v)[8], u64 *out) {
#pragma unroll
        for (int k = 0; k < 8; k++) out[nb + 64 * k] = v[k];
    };
    if (BOTH && !special) {
        if (m.qd != 0.0) {
            double r[2][8];
            inner12<2, MULT>(r, ia, oa, T, w, mi, make_fp(T, mi, 12), m);
#pragma unroll
            for (int c = 0; c < 2; c++)
#pragma unroll
                for (int k = 0; k < 8; k++) limb[c * comp_words + nb + 64 * k] = fp_canon(r[c][k], m.qd, m.qinvd);
        } else {
#pragma unroll 1
            for (w.c = 0; w.c < 2; w.c++) {
                u64 v[1][8];
                inner12<1, MULT>(v, ia, oa, T, w, mi, make_int(T, mi, 12), m);
                store(v[0], limb + w.c * comp_words);
            }
        }
    } else if (m.qd != 0.0) {
        const ArithFp ar = make_fp(T, mi, 12, special ? T.dn_inv_d[k_sp] : 0.0);
        double r[1][8];
        inner12<1, MULT>(r, ia, oa, T, w, mi, ar, m);
        u64 v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = fp_canon(r[0][k], m.qd, m.qinvd);
        if (special)
            inv12(v, limb, ar, lds);
        else
            store(v, limb);
    } else {
        const ArithInt ar = make_int(T, mi, 12, special ? T.dn_inv[k_sp] : ShoupConst{0, 0});
        u64 v[1][8];
        inner12<1, MULT>(v, ia, oa, T, w, mi, ar, m);
        if (special)
            inv12(v[0], limb, ar, lds);
        else
            store(v[0], limb);
    }
}

// grid (ciphertext limbs, components, operations).  DROP: the limb that a rescale drops (limb level - 1 alone); its
// finished value goes through the inverse transform and is left, in the coefficient domain, in its slot of the
// correction buffer.  INTS: some ciphertext limb is on the integer path, whose conversion takes up to 256 registers; without it every form
// stays within 128 and two work-groups fit a compute unit (128 products with rescale, digits of six primes: 649 -> 476 us).
template <int PRO, int NSMAX, bool EX, bool DROP, bool INTS>
__global__ __launch_bounds__(N12_THREADS, INTS && (EX || DROP) ? 1 : 4) void k_fin12(InnerArgs ia, FinishArgs fa, DevTables T, OpArgs oa, ConvArgs cv, int mode)
{
    __shared__ u64 lds[N12_LDS];
    const unsigned nb = N12_BASE;
    const Inner12 w = inner12_of(ia, oa, blockIdx.z, DROP ? ia.level - 1 : (int)blockIdx.x, (int)blockIdx.y);
    if (w.none) return;
    const ModConst m = T.mod[w.a];
    const unsigned slot = w.op * (unsigned)cv.dst_stride + (unsigned)(w.c * ia.level + w.a);
    const ConvSetup<NSMAX> S = conv_setup<PRO, NSMAX, 12>(cv, T, slot, w.a);
    // u and the addends (canonical residues) are on their way while the corrections are transformed
    const u64 *u = ia.u + (((size_t)w.op * ia.u_stride + (size_t)w.c * (ia.level + ia.K) + w.a) << 12);
    u64 uv[8], v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) uv[k] = u[nb + 64 * k], v[k] = 0;
    if (mode != FIN_MULT) {
        const u64 *add = ia.per_op && oa.add[w.op] ? oa.add[w.op] : fa.add + (((size_t)w.op * fa.add_stride) << 12);
        const u64 *add_same = add + (((size_t)w.c * fa.add_cstride + w.a) << 12), *add_rot = add + ((size_t)w.a << 12);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const unsigned n = nb + 64 * k;
            if (mode == FIN_ROTSUM) v[k] = add_same[n];
            if (w.c == 0) v[k] = csub(v[k] + add_rot[w.g == 1 ? n : galois_index(n, w.g, 12)], m.q);
        }
    }
    conv_variant12<PRO, NSMAX, EX, INTS>(T, w.a, m, S.qld, [&](auto ar, auto split, auto tint) {
        typedef decltype(ar) A;
        typename A::V a[8];
        inputs12<PRO, decltype(split)::value, decltype(tint)::value, EX>(a, nullptr, ar, S, m);
        u64 rv[8];
        fwd12(a, rv, ar, lds, true);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            if constexpr (A::IS_FP) {
                const double x = ar.mulmod(u2d(uv[k]) - u2d(rv[k]), fa.cst_d[w.a]) + u2d(v[k]);
                v[k] = fp_canon(x, m.qd, m.qinvd);
            } else
                v[k] = csub(mul_shoup(uv[k] + m.q - rv[k], fa.cst[w.a], m.q) + v[k], m.q);
        }
        if constexpr (DROP)
            inv12(v, const_cast<u64 *>(fa.r) + ((size_t)slot << 12), ar, lds);
        else {
            const unsigned out_cstride = ia.per_op && oa.level[w.op] ? oa.level[w.op] : (unsigned)fa.out_cstride;
            u64 *o = (ia.per_op ? oa.out[w.op] : fa.out + (((size_t)w.op * fa.out_stride) << 12)) + (((size_t)w.c * out_cstride + w.a) << 12);
#pragma unroll
            for (int k = 0; k < 8; k++) o[nb + 64 * k] = v[k];
        }
    });
}
