// The inner product of key switching with the evaluation key.
#pragma once
#include "kernels_conv.h"

// ---- inner product with the evaluation key, fused with the transforms on both sides of it -----------------------
//
// u[c][a][n] = sum_j D_j[a][pi_g(n)] * evk[j][c][mod(a)][n] on every active limb a, where D_j[a] is the
// raised digit outside digit j and the NTT-domain input d[a] inside it.
// One work-group produces INNER_TILE consecutive outputs (a few blocks of 256) of one active limb.  The index map of
// sigma_g sends aligned groups of 2^m consecutive NTT-domain indices to aligned groups (the low bits of
// (2 brv(k) + 1) g depend only on the low bits of brv(k), i.e. on the high bits of k), so the sources of
// these outputs are the indices of one input tile of that size.  For a limb on the floating-point path the raised
// digits arrive as the column pass left them; each is finished here (stages logN-8 .. logN-1) into LDS
// and read back through the index map, so the transformed digits never travel to memory.  Ciphertext limbs on
// the integer path read digits that the block-pass kernel has finished.
//
// Two launches make a key switch's inner product.  The first (k_inner_special, k_inner_finished) takes the special limbs, whose
// results leave it with the block pass of their inverse transform already applied.  The second (k_inner_fin) runs
// after the ModDown corrections r have been through their column pass: it forms u on the ciphertext limbs, finishes
// the transform of r the way it finishes a digit, and writes (u - r) * const + addend, so that u never travels to
// memory either.  As one inner product over all limbs and a finishing block pass, u was written and read back:
// 4 level limbs of traffic per operation, a tenth of a key switch's total.

typedef double f64x2 __attribute__((ext_vector_type(2)));

struct InnerArgs {
    const u64 *raised, *d, *evk;
    // Mult (g = 1): the two factors, operation z at z * t_stride limbs.  The polynomial that is switched is d2 = a1 b1, and
    // d0 = a0 b0, d1 = a0 b1 + a1 b0 join the result as u + P d (P: the product of the special primes), so that
    // the finishing step's (u - r) * const adds them; d is not used.  Null: no Mult.
    const u64 *ta, *tb;
    u64 *u;
    int level, L, K, alpha;
    int first; // the lowest active limb of the first launch (level: the special limbs alone)
    unsigned g;
    int raised_stride, u_stride, d_stride, t_stride; // limbs between two operations of a batch in each buffer
    int per_op; // operation z uses entry z of the OpArgs argument
    int finished; // the raised limbs from `first` on have been through their block pass: k_inner_finished in place of k_inner_special
    int count;  // operations in this launch
};
// What differs between the operations of one launch, when anything but their place in the buffers does.
struct OpArgs {
    const u64 *evk[HE_OPS_MAX];
    // the operation's NTT-domain input polynomial and its addend (null: InnerArgs.d + operation * d_stride,
    // FinishArgs.add + operation * add_stride), its output
    const u64 *d[HE_OPS_MAX];
    const u64 *add[HE_OPS_MAX];
    u64 *out[HE_OPS_MAX];
    unsigned g[HE_OPS_MAX];
    // mixed-level rotations: the operation's level (0: InnerArgs.level, which always gives the buffer layout)
    uint8_t level[HE_OPS_MAX];
};
// The finishing step on ciphertext limb i, component c: out = (u - NTT(r)) * cst + addend.
// FIN_MULT: no addend (u holds it, InnerArgs.ta); FIN_ROT: sigma_g of limb i
// of `add` (c0 of the rotated ciphertext) on component 0; FIN_ROTSUM: as FIN_ROT plus limb i of component c of `add`.
enum { FIN_MULT = 0, FIN_ROT = 1, FIN_ROTSUM = 2 };
struct FinishArgs {
    const u64 *r; // [2][level] limbs per operation, as the column pass left them
    u64 *out;
    const u64 *add;
    const ShoupConst *cst;
    const double *cst_d;
    int nl; // output limbs per component (level, or level - 1 when a rescale is folded in)
    int r_stride, out_stride, out_cstride, add_stride, add_cstride;
};

// One-dimensional grid of inner_grid() work-groups; every buffer is 16-byte aligned.  Work-groups go to the
// eight XCDs round-robin by index, and each XCD has its own L2: index 8 s + x runs on XCD x, and the `count`
// operations of one (tile, limb) take consecutive s there, so the key slice they share is fetched from
// memory once per XCD visit instead of once per operation.
__host__ __device__ inline unsigned inner_grid(unsigned tiles, unsigned limbs, unsigned count)
{
    return (tiles * limbs + XCDS - 1) / XCDS * XCDS * count;
}

// A wave works alone: it produces 512 consecutive outputs, eight per lane, and the sources of an aligned group of 512
// are an aligned group of 512, so the wave transforms the very blocks that its outputs read and nothing is exchanged
// between waves: no work-group barrier anywhere.  With the sources of a tile of 1024 shared between two waves, two barriers
// per digit, the special limbs of 32 mixed rotations (N = 2^16, levels 8 .. 24) took 228 us instead of 186, a whole
// rotation 113.9 us instead of 110.4 at N = 2^16, level 13, and 47.9 instead of 44.7 at N = 2^12.  Two waves per work-group
// (one: the same within 0.7 %),
// 25 KiB of LDS (exchange tile, twiddles, the next digit: 12.25 KiB per wave) allow three waves per SIMD, at up to
// 170 registers.  A 256-element
// block belongs to 32 lanes (half a wave) and its block pass runs as three register steps, stages 0-2, 3-5 and
// 6-7 of the block, with two exchanges through LDS among those lanes:
//   step 1: lane t holds e = t + 32 k;   step 2: lane (g = t & 7, r = t >> 3) holds e = 32 g + r + 4 k;
//   step 3: lane t holds e = 4 t + k' and 128 + 4 t + k' (k' < 4).
// With one pad word per 16 elements every 16 consecutive lanes of each pattern hit 16 different 8-byte banks.
// All 255 twiddles of a block's eight stages sit in LDS, the one of local stage m and group i at 2^m - 1 + i.
// In the product phase lane t of wave v owns the pairs (INNER_TILE tile + 512 v + 128 i + 2 t, + 1), i < 4.
// The 128 twiddles of a block's last stage, like all others, are contiguous in the block-major table (twd_blk), so a
// wave's 4 KiB of twiddles are fetched straight into LDS.

#define INNER_THREADS 128
#define INNER_TILE (INNER_THREADS * 8)      // outputs per work-group
#define INNER_TLOG 10
#define WAVE_OUT 512u                       // outputs per wave
#define WAVE_LOG 9
#define WAVE_LDS (WAVE_BLOCKS * (TILE_GROUP + 512)) // LDS words per wave: exchange tile, twiddles, the next digit
__device__ __forceinline__ unsigned pair8_at(unsigned i) { return WAVE_OUT * wave_id() + 128u * i + 2u * (threadIdx.x & 63u); }

// Addresses are formed as a wave-uniform base plus a 32-bit lane offset so that they stay in scalar registers;
// the three LDS patterns of the block pass are one base each plus compile-time offsets (with the pad word per
// 16 elements: t + 32 k sits at t + (t >> 4) + 34 k, 32 g + r + 4 k at 34 g + r + 4 k + (k >> 2), and
// 128 h + 4 t + k' at 4 t + (t >> 2) + 136 h + k').
template <class Tv> __device__ __forceinline__ Tv ld_at(const void *base, unsigned byte_off)
{
    return *(const Tv *)((const char *)base + byte_off);
}

// Copies of 4 KiB (the two blocks that a wave owns) from global memory into LDS by loads that write to LDS directly:
// lane i's 16 bytes land at dst + 16 i, and no registers are needed while they are in flight.  src: this lane's
// address.  NT: cache policy 2, nontemporal.
template <bool NT> __device__ __forceinline__ void wave_copy_4k(const char *src, char *dst)
{
#pragma unroll
    for (int c = 0; c < 4; c++)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + 1024 * c),
                                         (__attribute__((address_space(3))) void *)(dst + 1024 * c), 16, 0, NT ? 2 : 0);
}

// What one work-group works on.
struct InnerTile {
    unsigned op, tile, g;
    unsigned grp, grp_in; // this wave's group of 512 outputs within the limb, and the group its sources lie in
    int a; // active limb
    int level, beta; // of the operation
    bool none;
};
template <int LOGN, int TLOG>
__device__ __forceinline__ InnerTile inner_tile(const InnerArgs &ia, const OpArgs &oa, int limbs, int first)
{
    InnerTile w;
    const unsigned ntile = 1u << (LOGN - TLOG);
    const unsigned slot = blockIdx.x / XCDS;
    w.op = slot % (unsigned)ia.count;
    const unsigned tl = slot / (unsigned)ia.count * XCDS + blockIdx.x % XCDS;
    w.tile = tl % ntile;
    w.a = first + limbs - 1 - (int)(tl / ntile); // special limbs (the slowest) first
    w.g = ia.per_op ? oa.g[w.op] : ia.g;
    w.grp = w.tile * (INNER_TILE / WAVE_OUT) + wave_id();
    w.grp_in = w.g == 1 ? w.grp : galois_index(w.grp << WAVE_LOG, w.g, LOGN) >> WAVE_LOG;
    w.level = ia.per_op && oa.level[w.op] ? oa.level[w.op] : ia.level;
    w.beta = (w.level + ia.alpha - 1) / ia.alpha;
    // padding of the last group of eight; an operation below the layout's level has no limbs a in [its level, level)
    w.none = tl >= ntile * (unsigned)limbs || (w.a < ia.level && w.a >= w.level);
    return w;
}

// The pair of NTT-domain indices (pos, pos + 1) of limb a of both components of both factors of a Mult.
struct TensorPair {
    u64x2 a0, a1, b0, b1;
};
template <int LOGN> __device__ __forceinline__ TensorPair tensor_pair(const InnerArgs &ia, unsigned op, int a, unsigned pos)
{
    const size_t c0 = ((size_t)op * ia.t_stride + a) << LOGN, c1 = c0 + ((size_t)ia.level << LOGN);
    TensorPair p;
    p.a0 = ld_at<u64x2>(ia.ta + c0, pos * 8u), p.a1 = ld_at<u64x2>(ia.ta + c1, pos * 8u);
    p.b0 = ld_at<u64x2>(ia.tb + c0, pos * 8u), p.b1 = ld_at<u64x2>(ia.tb + c1, pos * 8u);
    return p;
}
// d2 is returned; d0 P and d1 P are added to the sums.  Floating point: |d2| below 0.9 q, the sums grow by less than 0.9 q.
__device__ __forceinline__ double tensor_mac(const ArithFp &ar, u64 a0, u64 a1, u64 b0, u64 b1, double P, double &acc0, double &acc1)
{
    const double x0 = u2d(a0), x1 = u2d(a1), y0 = u2d(b0), y1 = u2d(b1);
    acc0 += ar.mulmod(ar.mulmod(x0, y0), P);
    acc1 += ar.mulmod(ar.mulmod(x0, y1) + ar.mulmod(x1, y0), P);
    return ar.mulmod(x1, y1);
}
__device__ __forceinline__ u64 tensor_mac(const ModConst &m, u64 a0, u64 a1, u64 b0, u64 b1, u64 P, U128 &acc0, U128 &acc1)
{
    U128 d1{0, 0};
    mac128(d1, a0, b1);
    mac128(d1, a1, b0);
    mac128(acc0, mul_mod(a0, b0, m), P);
    mac128(acc1, reduce128(d1, m), P);
    return mul_mod(a1, b1, m);
}

// The products of one floating-point limb: acc0, acc1 = sums over the digits, within 3.5 q (MULT: 4.9 q, with d0 and d1), for
// this thread's pairs.
// If `then` is not null, the 4 KiB that it points at (this lane's address) are on their way into `pre` when
// the function returns.
template <int LOGN, bool MULT>
__device__ __forceinline__ void inner_products8(const InnerArgs &ia, const OpArgs &oa, const DevTables &T, const InnerTile &w,
                                                unsigned mi, const ArithFp &ar, const BlockLane &b, u64 *lds, double *tws, u64 *pre,
                                                const char *then, double (&acc0)[8], double (&acc1)[8])
{
    const int a = w.a, own = a < ia.level ? a / ia.alpha : -1, M = ia.L + ia.K, Ma = ia.level + ia.K;
    const unsigned lane16 = (threadIdx.x & 63) * 16u; // this lane's pair within a row of 64 pairs
    // wave-uniform bases (bytes): raised digit 0 and key component 0 of digit 0 for this limb and group; digit j is
    // raised_step / key_step further on, key component 1 comp_step after component 0
    const char *raised0 = (const char *)(ia.raised + ((((size_t)w.op * ia.raised_stride + a) << LOGN) + ((size_t)w.grp_in << WAVE_LOG)));
    const char *key0 = (const char *)((ia.per_op ? oa.evk[w.op] : ia.evk) + (((size_t)mi << LOGN) + ((size_t)w.grp << WAVE_LOG)));
    const size_t raised_step = ((size_t)Ma << LOGN) * 8, comp_step = ((size_t)M << LOGN) * 8, key_step = 2 * comp_step;
    // The raised digit after the one being worked on is already on its way into LDS.  A digit that only this operation
    // reads is streamed past the key slices that the batch shares in L2.
    auto prefetch = [&](int j) {
        const char *src = raised0 + (size_t)j * raised_step + lane16;
        if (ia.raised_stride != 0)
            wave_copy_4k<true>(src, (char *)pre);
        else
            wave_copy_4k<false>(src, (char *)pre);
    };
    wave_copy_4k<false>((const char *)(T.twd_blk + (((size_t)mi << LOGN) + ((size_t)w.grp_in << WAVE_LOG))) + lane16, (char *)tws);
    const int j0 = own == 0 ? 1 : 0;
    if (j0 < w.beta)
        prefetch(j0);
    else if (then)
        wave_copy_4k<true>(then, (char *)pre);
    // pair i of the product phase: LDS words of the sources of its even and odd element (an aligned pair, in
    // either order), and whether the pair arrives swapped
    unsigned lsx[4], lsy[4], swm = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const unsigned pos = (w.tile << INNER_TLOG) + pair8_at(i);
        const unsigned sr = w.g == 1 ? pos : galois_index(pos, w.g, LOGN);
        const unsigned sl = sr & (WAVE_OUT - 2u), sw = sr & 1u;
        const unsigned wd = (sl >> 8) * TILE_GROUP + (sl & 255u) + ((sl & 255u) >> 4);
        lsx[i] = wd + sw, lsy[i] = wd + 1 - sw;
        swm |= sw << i;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) acc0[k] = acc1[k] = 0.0;
    for (int j = 0; j < w.beta; j++) {
        double dv[8];
        f64x2 e0[4], e1[4]; // key words of a floating-point limb are balanced doubles
        const char *kj = key0 + (size_t)j * key_step;
        if (MULT && j == own) {
            const double P = T.dn_pmod_d[a];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const TensorPair p = tensor_pair<LOGN>(ia, w.op, a, (w.tile << INNER_TLOG) + pair8_at(i));
                dv[2 * i] = tensor_mac(ar, p.a0.x, p.a1.x, p.b0.x, p.b1.x, P, acc0[2 * i], acc1[2 * i]);
                dv[2 * i + 1] = tensor_mac(ar, p.a0.y, p.a1.y, p.b0.y, p.b1.y, P, acc0[2 * i + 1], acc1[2 * i + 1]);
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
                e0[i] = ld_at<f64x2>(kj + 1024 * i, lane16), e1[i] = ld_at<f64x2>(kj + comp_step + 1024 * i, lane16);
        } else if (!MULT && j == own) {
            const char *d_limb = (const char *)((ia.per_op && oa.d[w.op] ? oa.d[w.op] : ia.d + (((size_t)w.op * ia.d_stride) << LOGN)) + ((size_t)a << LOGN));
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const unsigned pos = (w.tile << INNER_TLOG) + pair8_at(i);
                const unsigned sr = w.g == 1 ? pos : galois_index(pos, w.g, LOGN);
                const u64x2 v = ld_at<u64x2>(d_limb, (sr & ~1u) * 8u);
                const bool sw = (swm >> i) & 1u;
                dv[2 * i] = u2d(sw ? v.y : v.x), dv[2 * i + 1] = u2d(sw ? v.x : v.y);
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
                e0[i] = ld_at<f64x2>(kj + 1024 * i, lane16), e1[i] = ld_at<f64x2>(kj + comp_step + 1024 * i, lane16);
        } else {
            // this digit has arrived (nothing else of this wave is in flight here); once it is in registers the
            // buffer is free for the next one
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            mid_pairs8(ar, dv, pre, b);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            {
                const int jn = j + 1 == own ? j + 2 : j + 1;
                if (jn < w.beta)
                    prefetch(jn);
                else if (then)
                    wave_copy_4k<true>(then, (char *)pre);
            }
            // the key loads are issued before the block pass and complete behind it
#pragma unroll
            for (int i = 0; i < 4; i++)
                e0[i] = ld_at<f64x2>(kj + 1024 * i, lane16), e1[i] = ld_at<f64x2>(kj + comp_step + 1024 * i, lane16);
            block_pass8(ar, dv, b);
            block_sync();
#pragma unroll
            for (int i = 0; i < 4; i++) dv[2 * i] = ar.load_mid(lds[lsx[i]]), dv[2 * i + 1] = ar.load_mid(lds[lsy[i]]);
            block_sync();
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            acc0[2 * i] += ar.mulmod(dv[2 * i], e0[i].x);
            acc0[2 * i + 1] += ar.mulmod(dv[2 * i + 1], e0[i].y);
            acc1[2 * i] += ar.mulmod(dv[2 * i], e1[i].x);
            acc1[2 * i + 1] += ar.mulmod(dv[2 * i + 1], e1[i].y);
        }
        if ((j & 3) == 3) {
#pragma unroll
            for (int k = 0; k < 8; k++) acc0[k] = ar.reduce(acc0[k]), acc1[k] = ar.reduce(acc1[k]);
        }
    }
}

// Pair h of the product phase (h < 2: pairs 2 h and 2 h + 1) on the integer path: the raised digits arrive finished
// (NTT domain) and are read through the index map.
template <int LOGN, bool MULT>
__device__ __forceinline__ void inner_products_int(const InnerArgs &ia, const OpArgs &oa, const DevTables &T, const InnerTile &w, unsigned mi,
                                                   const ModConst &m, int h, u64 (&r0)[4], u64 (&r1)[4])
{
    const int a = w.a, own = a < ia.level ? a / ia.alpha : -1, M = ia.L + ia.K, Ma = ia.level + ia.K;
    const char *key0 = (const char *)((ia.per_op ? oa.evk[w.op] : ia.evk) + (((size_t)mi << LOGN) + ((size_t)w.grp << WAVE_LOG)));
    const char *d_limb = (const char *)((ia.per_op && oa.d[w.op] ? oa.d[w.op] : ia.d + (((size_t)w.op * ia.d_stride) << LOGN)) + ((size_t)a << LOGN));
    const char *fin0 = (const char *)(ia.raised + (((size_t)w.op * ia.raised_stride + a) << LOGN));
    const size_t raised_step = ((size_t)Ma << LOGN) * 8, comp_step = ((size_t)M << LOGN) * 8, key_step = 2 * comp_step;
    const unsigned lane16 = (threadIdx.x & 63) * 16u;
    unsigned sr[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const unsigned pos = (w.tile << INNER_TLOG) + pair8_at(2 * h + i);
        sr[i] = w.g == 1 ? pos : galois_index(pos, w.g, LOGN);
    }
    U128 acc0[4], acc1[4];
#pragma unroll
    for (int k = 0; k < 4; k++) acc0[k] = acc1[k] = U128{0, 0};
    for (int j = 0; j < w.beta; j++) {
        const char *dj = j == own ? d_limb : fin0 + (size_t)j * raised_step;
        const char *kj = key0 + (size_t)j * key_step;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int ii = 2 * h + i;
            u64 x, y;
            if (MULT && j == own) {
                const TensorPair p = tensor_pair<LOGN>(ia, w.op, a, sr[i]); // g = 1: the pair itself
                const u64 P = T.dn_pmod[a];
                x = tensor_mac(m, p.a0.x, p.a1.x, p.b0.x, p.b1.x, P, acc0[2 * i], acc1[2 * i]);
                y = tensor_mac(m, p.a0.y, p.a1.y, p.b0.y, p.b1.y, P, acc0[2 * i + 1], acc1[2 * i + 1]);
            } else {
                const u64x2 v = ld_at<u64x2>(dj, (sr[i] & ~1u) * 8u);
                const bool sw = sr[i] & 1u;
                x = sw ? v.y : v.x, y = sw ? v.x : v.y;
            }
            const u64x2 ka = ld_at<u64x2>(kj + 1024 * ii, lane16), kb = ld_at<u64x2>(kj + comp_step + 1024 * ii, lane16);
            mac128(acc0[2 * i], x, ka.x);
            mac128(acc0[2 * i + 1], y, ka.y);
            mac128(acc1[2 * i], x, kb.x);
            mac128(acc1[2 * i + 1], y, kb.y);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; k++) r0[k] = reduce128(acc0[k], m), r1[k] = reduce128(acc1[k], m);
}

// ---- first launch: the special limbs ------------------------------------------------------------------------------------
//
// Few limbs (K per operation) with the most work per word: the special primes are on the integer path, whose block pass
// takes about three times the instructions of the floating-point one.  Two forms, chosen by special_finished() in device.hip:
//
// k_inner_special, for launches that leave the chip part empty: what a wave of k_inner_fin does alone is shared
// out: a work-group of four waves makes SPECIAL_TILE outputs of both components, and in each round every wave finishes
// the transform of another digit (the steps of k_inner_fin's block pass) into LDS;
// then all threads multiply the digits of the round, read through the index map, with the key.  One operation
// alone then has four digits in work at a time, and the finished digits never travel to memory.
// Bound by the chain of a round (load, three steps with their twiddles, exchanges, products): one rotation at N = 2^16, level 13, takes
// 15.3 us, with tiles of 1024 outputs and 16 elements per lane 18.3; eight at level 24 128 us, 137 (105 registers instead of 148, four waves per
// SIMD instead of three).
//
// k_inner_finished, for launches that fill it and for digits that several operations share: k_ntt_fwd_blocks finishes the
// digits, each thread reads them through the index map straight into its sums, without LDS and without a barrier.
//
// The result leaves either with the block pass of its inverse transform applied.
#define SPECIAL_THREADS 256
#define SPECIAL_WAVES (SPECIAL_THREADS / 64)
#define SPECIAL_TLOG 9
#define SPECIAL_TILE (1 << SPECIAL_TLOG)           // outputs per work-group: two blocks, 8 elements per lane of a wave
#define SPECIAL_DIGIT (WAVE_BLOCKS * TILE_GROUP)   // LDS words of 512 elements
#define FINISHED_TLOG 10

// The pair of digit values at `key`-order position: floating point, within 1.9 q of zero; integer, below 8q.
__device__ __forceinline__ void special_mac(const ArithFp &ar, double x, u64 k0, u64 k1, double &s0, double &s1)
{
    s0 += ar.mulmod(x, ar.load_mid(k0)), s1 += ar.mulmod(x, ar.load_mid(k1)); // key words are balanced doubles
}
__device__ __forceinline__ void special_mac(const ArithInt &, u64 x, u64 k0, u64 k1, U128 &s0, U128 &s1) { mac128(s0, x, k0), mac128(s1, x, k1); }
template <class A> struct SpecialSum;
template <> struct SpecialSum<ArithFp> {
    typedef double S;
    static __device__ __forceinline__ double zero() { return 0.0; }
    static __device__ __forceinline__ double fold(const ModConst &m, double s) { return fp_reduce(s, m.qd, m.qinvd); }
    static __device__ __forceinline__ u64 result(const ArithFp &ar, const ModConst &, double s) { return ar.store_final(s); }
    static __device__ __forceinline__ double product(const DevTables &T, const ModConst &, const ArithFp &ar, int a, u64 a0, u64 a1, u64 b0, u64 b1, double &s0, double &s1)
    {
        return tensor_mac(ar, a0, a1, b0, b1, T.dn_pmod_d[a], s0, s1);
    }
};
template <> struct SpecialSum<ArithInt> {
    typedef U128 S;
    static __device__ __forceinline__ U128 zero() { return U128{0, 0}; }
    static __device__ __forceinline__ U128 fold(const ModConst &m, U128 s) { return U128{reduce128(s, m), 0}; }
    static __device__ __forceinline__ u64 result(const ArithInt &, const ModConst &m, U128 s) { return reduce128(s, m); }
    static __device__ __forceinline__ u64 product(const DevTables &T, const ModConst &m, const ArithInt &, int a, u64 a0, u64 a1, u64 b0, u64 b1, U128 &s0, U128 &s1)
    {
        return tensor_mac(m, a0, a1, b0, b1, T.dn_pmod[a], s0, s1);
    }
};

// limb w.a of one operation; the results of the thread's pair (2 thread, + 1) of both components
template <int LOGN, bool MULT, class A>
__device__ __forceinline__ void special_products(const InnerArgs &ia, const OpArgs &oa, const DevTables &T, const InnerTile &w, unsigned mi,
                                                 const ModConst &m, const A &ar, u64 *lds, u64 (&r0)[2], u64 (&r1)[2])
{
    typedef SpecialSum<A> Sum;
    const int a = w.a, own = MULT && a < ia.level ? a / ia.alpha : -1, M = ia.L + ia.K, Ma = ia.level + ia.K; // own: the dropped limb of a Mult
    const unsigned tile_in = w.g == 1 ? w.tile : galois_index(w.tile << SPECIAL_TLOG, w.g, LOGN) >> SPECIAL_TLOG;
    const char *key0 = (const char *)((ia.per_op ? oa.evk[w.op] : ia.evk) + (((size_t)mi << LOGN) + ((size_t)w.tile << SPECIAL_TLOG)));
    const u64 *raised0 = ia.raised + ((((size_t)w.op * ia.raised_stride + a) << LOGN) + ((size_t)tile_in << SPECIAL_TLOG));
    const size_t raised_step = (size_t)Ma << LOGN, comp_step = ((size_t)M << LOGN) * 8, key_step = 2 * comp_step;
    const int wave = wave_id();
    // an integer-path ciphertext limb (the one a rescale drops) has been finished with the other ciphertext limbs
    const bool finished = MULT && !A::IS_FP && a < ia.level;
    // source of the pair: index in the limb, LDS words of the even and the odd element
    const unsigned pos = (w.tile << SPECIAL_TLOG) + 2u * threadIdx.x, sr = w.g == 1 ? pos : galois_index(pos, w.g, LOGN);
    const unsigned sl = sr & (SPECIAL_TILE - 2u), sw = sr & 1u, wd = tile_at(sl >> 8, sl & 255u);
    typename Sum::S s0[2], s1[2];
#pragma unroll
    for (int e = 0; e < 2; e++) s0[e] = s1[e] = Sum::zero();
    // the key words of the digit after the one at hand are on their way, those of a round's first through the transforms
    u64x2 ka, kb;
    const auto load_key = [&](int j) {
        const char *kj = key0 + (size_t)j * key_step;
        ka = ld_at<u64x2>(kj, threadIdx.x * 16u), kb = ld_at<u64x2>(kj + comp_step, threadIdx.x * 16u);
    };
    load_key(0);
    for (int j0 = 0; j0 < w.beta; j0 += SPECIAL_WAVES) {
        const int jw = j0 + wave;
        if (jw < w.beta && jw != own) {
            const u64 *in = raised0 + (size_t)jw * raised_step;
            u64 *dig = lds + wave * SPECIAL_DIGIT;
            const BlockLane b = block_lane(dig, nullptr);
            if (finished) {
#pragma unroll
                for (int k = 0; k < 8; k++) b.l1[34 * k] = in[b.blk * 256 + b.t + 32 * k];
            } else {
                typename A::V v[8];
                mid_pairs8(ar, v, in, b);
                const unsigned G = tile_in * WAVE_BLOCKS + b.blk;
                block_pass8(ar, v, b, [&](int st, unsigned i) { return block_twiddle<LOGN>(ar.twf, G, st, i); });
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int jj = 0; jj < SPECIAL_WAVES && j0 + jj < w.beta; jj++) {
            const int j = j0 + jj;
            const u64 *dig = lds + jj * SPECIAL_DIGIT;
            const u64x2 ca = ka, cb = kb;
            if (j + 1 < w.beta) load_key(j + 1);
            typename A::V x, y;
            if (MULT && j == own) { // g = 1: the pair itself
                const TensorPair p = tensor_pair<LOGN>(ia, w.op, a, sr);
                x = Sum::product(T, m, ar, a, p.a0.x, p.a1.x, p.b0.x, p.b1.x, s0[0], s1[0]);
                y = Sum::product(T, m, ar, a, p.a0.y, p.a1.y, p.b0.y, p.b1.y, s0[1], s1[1]);
            } else
                x = ar.load_mid(dig[wd + sw]), y = ar.load_mid(dig[wd + 1 - sw]);
            special_mac(ar, x, ca.x, cb.x, s0[0], s1[0]);
            special_mac(ar, y, ca.y, cb.y, s0[1], s1[1]);
        }
        if (A::IS_FP || w.beta > 28) { // floating point: after at most four products; integer: 28 below 2^123 fit, with the two of d0 and d1
#pragma unroll
            for (int e = 0; e < 2; e++) s0[e] = Sum::fold(m, s0[e]), s1[e] = Sum::fold(m, s1[e]);
        }
        __syncthreads(); // the digits have been read
    }
#pragma unroll
    for (int e = 0; e < 2; e++) r0[e] = Sum::result(ar, m, s0[e]), r1[e] = Sum::result(ar, m, s1[e]);
}

// What both forms do with their sums, PAIRS pairs (512 i + 2 thread, + 1) of a thread and component, groups of 512 outputs from `tile` on: the inverse block
// pass on a special limb, one group of one component per wave, through LDS (which nothing reads any more); u on a ciphertext limb (MULT: the dropped one).
template <int LOGN, bool MULT, int PAIRS, class A>
__device__ __forceinline__ void special_result(const InnerArgs &ia, const InnerTile &w, const u64 (&r0)[2 * PAIRS], const u64 (&r1)[2 * PAIRS], const A &ar, u64 *lds)
{
    u64 *u0 = ia.u + (((size_t)w.op * ia.u_stride + w.a) << LOGN);
    const size_t comp_words = (size_t)(ia.level + ia.K) << LOGN;
    const unsigned group0 = w.tile * PAIRS;
    if (MULT && w.a < ia.level) {
#pragma unroll
        for (int i = 0; i < PAIRS; i++) {
            char *o = (char *)(u0 + ((size_t)(group0 + i) << WAVE_LOG)) + threadIdx.x * 16u;
            __builtin_nontemporal_store(u64x2{r0[2 * i], r0[2 * i + 1]}, (u64x2 *)o);
            __builtin_nontemporal_store(u64x2{r1[2 * i], r1[2 * i + 1]}, (u64x2 *)(o + comp_words * 8));
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < PAIRS; i++) {
        const unsigned p = 2u * threadIdx.x, wd = tile_at(p >> 8, p & 255u);
        u64 *d0 = lds + (2 * i) * SPECIAL_DIGIT + wd, *d1 = d0 + SPECIAL_DIGIT;
        d0[0] = r0[2 * i], d0[1] = r0[2 * i + 1];
        d1[0] = r1[2 * i], d1[1] = r1[2 * i + 1];
    }
    __syncthreads();
    const unsigned wave = wave_id(), comp = wave & 1u, group = group0 + (wave >> 1);
    if (wave >= 2 * PAIRS) return;
    const BlockLane b = block_lane(lds + wave * SPECIAL_DIGIT, nullptr);
    const unsigned G = group * WAVE_BLOCKS + b.blk;
    typename A::V v[8];
    inv_block_pass8(ar, v, b, [&](int st, unsigned i) { return block_twiddle<LOGN>(ar.twi, G, st, i); });
    u64 *o = u0 + comp * comp_words + (size_t)G * 256 + b.t;
#pragma unroll
    for (int k = 0; k < 8; k++) o[32 * k] = ar.store_mid(v[k]);
}

// Active limbs ia.first .. level + K - 1 of every operation.  The same order of work-groups as k_inner_fin.
// MULT: of a Mult with rescale, whose dropped limb takes d0, d1 and d2 (a kernel of its own: with their code in every launch
// 32 mixed rotations at N = 2^16 took 2388 us instead of 2342)
template <int LOGN, bool MULT> __global__ __launch_bounds__(SPECIAL_THREADS, MULT ? 3 : 4) void k_inner_special(InnerArgs ia, DevTables T, OpArgs oa)
{
    __shared__ __align__(16) u64 lds[SPECIAL_WAVES * SPECIAL_DIGIT];
    const InnerTile w = inner_tile<LOGN, SPECIAL_TLOG>(ia, oa, ia.level + ia.K - ia.first, ia.first);
    if (w.none) return;
    const int mi = active_mod(w.a, ia.level, ia.L);
    const ModConst m = T.mod[mi];
    u64 r0[2], r1[2];
    if (m.qd != 0.0) {
        const ArithFp ar = make_fp(T, mi, LOGN);
        special_products<LOGN, MULT>(ia, oa, T, w, mi, m, ar, lds, r0, r1);
        special_result<LOGN, MULT, 1>(ia, w, r0, r1, ar, lds);
    } else {
        const ArithInt ar = make_int(T, mi, LOGN);
        special_products<LOGN, MULT>(ia, oa, T, w, mi, m, ar, lds, r0, r1);
        special_result<LOGN, MULT, 1>(ia, w, r0, r1, ar, lds);
    }
}

// The sums of a thread's pairs (512 i + 2 thread, + 1), i < 2, from digits in the NTT domain.
template <int LOGN, bool MULT, class A>
__device__ __forceinline__ void finished_products(const InnerArgs &ia, const OpArgs &oa, const DevTables &T, const InnerTile &w, unsigned mi,
                                                  const ModConst &m, const A &ar, u64 (&r0)[4], u64 (&r1)[4])
{
    typedef SpecialSum<A> Sum;
    const int own = MULT && w.a < ia.level ? w.a / ia.alpha : -1, M = ia.L + ia.K, Ma = ia.level + ia.K;
    const char *key0 = (const char *)((ia.per_op ? oa.evk[w.op] : ia.evk) + (((size_t)mi << LOGN) + ((size_t)w.tile << FINISHED_TLOG)));
    const char *dig0 = (const char *)(ia.raised + (((size_t)w.op * ia.raised_stride + w.a) << LOGN));
    const size_t dig_step = ((size_t)Ma << LOGN) * 8, comp_step = ((size_t)M << LOGN) * 8, key_step = 2 * comp_step;
    unsigned sr[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const unsigned pos = (w.tile << FINISHED_TLOG) + 512u * i + 2u * threadIdx.x;
        sr[i] = w.g == 1 ? pos : galois_index(pos, w.g, LOGN);
    }
    typename Sum::S s0[4], s1[4];
#pragma unroll
    for (int k = 0; k < 4; k++) s0[k] = s1[k] = Sum::zero();
    for (int j = 0; j < w.beta; j++) {
        const char *kj = key0 + (size_t)j * key_step;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const u64x2 ka = ld_at<u64x2>(kj + 4096 * i, threadIdx.x * 16u), kb = ld_at<u64x2>(kj + comp_step + 4096 * i, threadIdx.x * 16u);
            typename A::V x, y;
            if (MULT && j == own) { // g = 1: the pair itself
                const TensorPair p = tensor_pair<LOGN>(ia, w.op, w.a, sr[i]);
                x = Sum::product(T, m, ar, w.a, p.a0.x, p.a1.x, p.b0.x, p.b1.x, s0[2 * i], s1[2 * i]);
                y = Sum::product(T, m, ar, w.a, p.a0.y, p.a1.y, p.b0.y, p.b1.y, s0[2 * i + 1], s1[2 * i + 1]);
            } else {
                const u64x2 v = ld_at<u64x2>(dig0 + (size_t)j * dig_step, (sr[i] & ~1u) * 8u);
                x = ar.load(sr[i] & 1u ? v.y : v.x), y = ar.load(sr[i] & 1u ? v.x : v.y);
            }
            special_mac(ar, x, ka.x, kb.x, s0[2 * i], s1[2 * i]);
            special_mac(ar, y, ka.y, kb.y, s0[2 * i + 1], s1[2 * i + 1]);
        }
        if (A::IS_FP && (j & 3) == 3) {
#pragma unroll
            for (int k = 0; k < 4; k++) s0[k] = Sum::fold(m, s0[k]), s1[k] = Sum::fold(m, s1[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; k++) r0[k] = Sum::result(ar, m, s0[k]), r1[k] = Sum::result(ar, m, s1[k]);
}
// The limbs of k_inner_special, in the same order.
template <int LOGN, bool MULT> __global__ __launch_bounds__(SPECIAL_THREADS, 5) void k_inner_finished(InnerArgs ia, DevTables T, OpArgs oa)
{
    __shared__ __align__(16) u64 lds[4 * SPECIAL_DIGIT];
    const InnerTile w = inner_tile<LOGN, FINISHED_TLOG>(ia, oa, ia.level + ia.K - ia.first, ia.first);
    if (w.none) return;
    const int mi = active_mod(w.a, ia.level, ia.L);
    const ModConst m = T.mod[mi];
    u64 r0[4], r1[4];
    if (m.qd != 0.0) {
        const ArithFp ar = make_fp(T, mi, LOGN);
        finished_products<LOGN, MULT>(ia, oa, T, w, mi, m, ar, r0, r1);
        special_result<LOGN, MULT, 2>(ia, w, r0, r1, ar, lds);
    } else {
        const ArithInt ar = make_int(T, mi, LOGN);
        finished_products<LOGN, MULT>(ia, oa, T, w, mi, m, ar, r0, r1);
        special_result<LOGN, MULT, 2>(ia, w, r0, r1, ar, lds);
    }
}

// ---- second launch: the ciphertext limbs ------------------------------------------------------------------------------------

// Addend of pair i of component c of a rotation, as canonical residues.
template <int LOGN, int MODE>
__device__ __forceinline__ u64x2 fin_addend(const FinishArgs &fa, const OpArgs &oa, const InnerArgs &ia, const InnerTile &w, int c,
                                            int i, u64 q)
{
    u64x2 v = {0, 0};
    if (MODE == FIN_MULT) return v;
    const u64 *add = ia.per_op && oa.add[w.op] ? oa.add[w.op] : fa.add + (((size_t)w.op * fa.add_stride) << LOGN);
    const unsigned pos = (w.tile << INNER_TLOG) + pair8_at(i);
    if (MODE == FIN_ROTSUM) v = ld_at<u64x2>(add + (((size_t)c * fa.add_cstride + w.a) << LOGN), pos * 8u);
    if (c == 0) {
        const unsigned sr = w.g == 1 ? pos : galois_index(pos, w.g, LOGN);
        u64x2 s = ld_at<u64x2>(add + ((size_t)w.a << LOGN), (sr & ~1u) * 8u);
        if (sr & 1u) s = u64x2{s.y, s.x};
        v = MODE == FIN_ROT ? s : u64x2{csub(v.x + s.x, q), csub(v.y + s.y, q)};
    }
    return v;
}

// Second launch: the ciphertext limbs.  PATH: the arithmetic of the limbs of this launch; FIN_BOTH where a chain mixes them, one launch for
// all rather than one per path: half a grid's work-groups would return at once, and the second launch waited for the first (primes
// of 55 and 50 bits in turn at N = 2^16, one rotation at level 12: 170 -> 148 us, 150 as one inner product and a finishing pass; eight
// 55-bit primes, eight rotations: 382 -> 343, 370).
// Bound by memory for batches with one key (the digits, r, the addend and the result once each); a call as a whole
// takes less than the inner product over the same limbs and the finishing block pass took together: at N = 2^16, level 24,
// 15 hoisted rotations 1200 -> 1061 us, 16 products 2120 -> 2017 us, 32 rotations of mixed levels 2515 -> 2362 us.
enum { FIN_FP = 0, FIN_INT = 1, FIN_BOTH = 2 };

// One integer-path limb: both corrections through their block pass first, the twiddles from the table (the wave keeps both, in
// [0, 8q), in its LDS), then pair by pair the products and the finishing step.
template <int LOGN, int MODE>
__device__ __forceinline__ void inner_fin_int(const InnerArgs &ia, const FinishArgs &fa, const DevTables &T, const OpArgs &oa, const InnerTile &w,
                                              const ModConst &m, const u64 *r_grp, char *o, size_t o_step, u64 *lds)
{
    const unsigned lane16 = (threadIdx.x & 63) * 16u;
    const ArithInt ar = make_int(T, w.a, LOGN);
#pragma unroll 1
    for (int c = 0; c < 2; c++) {
        const BlockLane b = block_lane(lds + c * WAVE_BLOCKS * TILE_GROUP, nullptr);
        const u64 *in = r_grp + c * ((size_t)ia.level << LOGN) + mid_at<true>(b.blk, b.t);
        u64 v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = __builtin_nontemporal_load(in + 64 * k);
        const unsigned G = w.grp * WAVE_BLOCKS + b.blk;
        block_pass8(ar, v, b, [&](int st, unsigned i) { return ar.twf[(1u << (LOGN - 8 + st)) + (G << st) + i]; });
    }
    block_sync();
#pragma unroll
    for (int h = 0; h < 2; h++) {
        u64 x[2][4];
        inner_products_int<LOGN, MODE == FIN_MULT>(ia, oa, T, w, w.a, m, h, x[0], x[1]);
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const int ii = 2 * h + i;
                const unsigned p = 128u * ii + 2u * (threadIdx.x & 63);
                const u64 *rv = lds + c * WAVE_BLOCKS * TILE_GROUP + tile_at(p >> 8, p & 255u);
                const u64x2 av = fin_addend<LOGN, MODE>(fa, oa, ia, w, c, ii, m.q);
                u64x2 res; // u - r + 8q stays below 9q < 2^64
                res.x = mul_shoup(x[c][2 * i] + 8 * m.q - rv[0], fa.cst[w.a], m.q);
                res.y = mul_shoup(x[c][2 * i + 1] + 8 * m.q - rv[1], fa.cst[w.a], m.q);
                res.x = csub(res.x + av.x, m.q);
                res.y = csub(res.y + av.y, m.q);
                __builtin_nontemporal_store(res, (u64x2 *)(o + c * o_step + 1024 * ii + lane16));
            }
    }
}

// One floating-point limb.
template <int LOGN, int MODE>
__device__ __forceinline__ void inner_fin_fp(const InnerArgs &ia, const FinishArgs &fa, const DevTables &T, const OpArgs &oa, const InnerTile &w,
                                             const ModConst &m, const u64 *r_grp, char *o, size_t o_step, u64 *lds)
{
    const unsigned lane16 = (threadIdx.x & 63) * 16u;
    const size_t r_step = ((size_t)ia.level << LOGN) * 8;
    double *tws = (double *)(lds + WAVE_BLOCKS * TILE_GROUP);
    u64 *pre = lds + WAVE_BLOCKS * (TILE_GROUP + 256);
    const ArithFp ar = make_fp(T, w.a, LOGN);
    const BlockLane b = block_lane(lds, tws);
    const char *r_lane = (const char *)r_grp + lane16;
    double acc[2][8];
    inner_products8<LOGN, MODE == FIN_MULT>(ia, oa, T, w, w.a, ar, b, lds, tws, pre, r_lane, acc[0], acc[1]);
    // the corrections are transformed in the output's own blocks: other twiddles where a rotation maps the group
    // elsewhere (the wave's own reads of the old ones have returned, and what it still has in flight was issued
    // before the last key words and has arrived with them)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (w.grp_in != w.grp)
        wave_copy_4k<false>((const char *)(T.twd_blk + (((size_t)w.a << LOGN) + ((size_t)w.grp << WAVE_LOG))) + lane16, (char *)tws);
    const double k1 = fa.cst_d[w.a];
#pragma unroll
    for (int c = 0; c < 2; c++) {
        double dv[8];
        u64x2 av[4];
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        mid_pairs8(ar, dv, pre, b);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (c == 0) wave_copy_4k<true>(r_lane + r_step, (char *)pre);
#pragma unroll
        for (int i = 0; i < 4; i++) av[i] = fin_addend<LOGN, MODE>(fa, oa, ia, w, c, i, m.q);
        block_pass8(ar, dv, b);
        block_sync();
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const unsigned p = 128u * i + 2u * (threadIdx.x & 63), wd = tile_at(p >> 8, p & 255u);
            dv[2 * i] = ar.load_mid(lds[wd]), dv[2 * i + 1] = ar.load_mid(lds[wd + 1]);
        }
        block_sync();
#pragma unroll
        for (int i = 0; i < 4; i++) {
            u64x2 res;
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const double v = ar.mulmod(acc[c][2 * i + e] - dv[2 * i + e], k1);
                res[e] = fp_canon(MODE == FIN_MULT ? v : v + u2d(av[i][e]), m.qd, m.qinvd);
            }
            __builtin_nontemporal_store(res, (u64x2 *)(o + c * o_step + 1024 * i + lane16));
        }
    }
}

template <int LOGN, int MODE, int PATH>
__global__ __launch_bounds__(INNER_THREADS, PATH != FIN_INT ? 6 : MODE == FIN_MULT ? 3 : 4) void k_inner_fin(InnerArgs ia, FinishArgs fa, DevTables T, OpArgs oa)
{
    __shared__ __align__(16) u64 wave_lds[INNER_THREADS / 64][PATH == FIN_INT ? 2 * WAVE_BLOCKS * TILE_GROUP : WAVE_LDS];
    const InnerTile w = inner_tile<LOGN, INNER_TLOG>(ia, oa, fa.nl, 0);
    if (w.none) return;
    const ModConst m = T.mod[w.a];
    const u64 *r_grp = fa.r + (((size_t)w.op * fa.r_stride + w.a) << LOGN) + ((size_t)w.grp << WAVE_LOG);
    const unsigned out_cstride = ia.per_op && oa.level[w.op] ? oa.level[w.op] : (unsigned)fa.out_cstride;
    char *o = (char *)((ia.per_op ? oa.out[w.op] : fa.out + (((size_t)w.op * fa.out_stride) << LOGN)) + (((size_t)w.a << LOGN) + ((size_t)w.grp << WAVE_LOG)));
    const size_t o_step = ((size_t)out_cstride << LOGN) * 8;
    u64 *lds = wave_lds[wave_id()];
    if (PATH == FIN_INT || (PATH == FIN_BOTH && m.qd == 0.0)) {
        if constexpr (PATH != FIN_FP) inner_fin_int<LOGN, MODE>(ia, fa, T, oa, w, m, r_grp, o, o_step, lds);
    } else {
        if constexpr (PATH != FIN_INT) inner_fin_fp<LOGN, MODE>(ia, fa, T, oa, w, m, r_grp, o, o_step, lds);
    }
}
