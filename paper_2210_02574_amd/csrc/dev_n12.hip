// Kernels of the ring size N = 2^12 and their launchers.  Compiled twice: with HE_FEW the default conversions of one and two sources, which are an
// object of their own, else everything else.  The launches of a call are short and fetch their code anew, and where in memory it lies shows: with
// those in the one object, between the others, one rotation at level 24 (24 primes in digits of four) took 47.0 us instead of 46.2, 16 at level 12
// 71.1 instead of 70.0.
#include "launch.h"
#include "kernels_n12.h"

// The conversions, but for the corrected ones, are instantiated for up to one, two, four and eight sources: a source past the real count costs its
// product, and single calls are as long as one work-group's chain (one rotation of three primes, digits and special primes of one:
// 30.0 us, 32.5 with four sources everywhere; two digits of two primes 47.8 -> 45.0).
void fwd12_modup_few(he_ctx *c, hipStream_t st, double bytes, u64 *data, const LimbBatch &lb, int nb, const ConvArgs &cv);
void fin12_few(he_ctx *c, hipStream_t st, double bytes, int pro, bool drop, bool ints, int mode, const InnerArgs &ia, const FinishArgs &fa,
               const OpArgs &oa, const ConvArgs &cv);

template <int PRO, int NSMAX, bool EX>
static void launch_fwd12(he_ctx *c, hipStream_t st, double bytes, u64 *data, const LimbBatch &lb, int nb, const ConvArgs &cv,
                         const FinArgs *fin)
{
    constexpr int kid = PRO == PRO_MODUP ? KID_FWD12_MODUP : PRO == PRO_RESCALE ? KID_FWD12_RESCALE : KID_FWD12;
    if constexpr (PRO == PRO_RESCALE) { // the one prologue that the finishing epilogue follows here
        if (fin) {
            KLAUNCH_T(c, st, kid, bytes, (k_ntt_fwd12<PRO, NSMAX, EX, EPI_FIN>), nb, N12_THREADS, data, c->dev, lb, cv, *fin);
            return;
        }
    }
    KLAUNCH_T(c, st, kid, bytes, (k_ntt_fwd12<PRO, NSMAX, EX, EPI_STORE>), nb, N12_THREADS, data, c->dev, lb, cv, FinArgs{});
}
// one instance of the finishing kernel
template <int PRO, int NSMAX, bool EX, bool DROP, bool INTS>
static void launch_fin12(he_ctx *c, hipStream_t st, double bytes, int mode, const InnerArgs &ia, const FinishArgs &fa, const OpArgs &oa, const ConvArgs &cv)
{
    const dim3 grid(DROP ? 1 : fa.nl, 2, ia.count);
    KLAUNCH_T(c, st, KID_FIN12, bytes, (k_fin12<PRO, NSMAX, EX, DROP, INTS>), grid, N12_THREADS, ia, fa, c->dev, oa, cv, mode);
}
#if HE_FEW
void fwd12_modup_few(he_ctx *c, hipStream_t st, double bytes, u64 *data, const LimbBatch &lb, int nb, const ConvArgs &cv)
{
    (c->alpha > 1 ? launch_fwd12<PRO_MODUP, 2, false> : launch_fwd12<PRO_MODUP, 1, false>)(c, st, bytes, data, lb, nb, cv, nullptr);
}
template <int PRO, bool DROP>
static void fin12_of(he_ctx *c, hipStream_t st, double bytes, bool ints, int mode, const InnerArgs &ia, const FinishArgs &fa, const OpArgs &oa,
                     const ConvArgs &cv)
{
    if (c->K > 1)
        (ints ? launch_fin12<PRO, 2, false, DROP, true> : launch_fin12<PRO, 2, false, DROP, false>)(c, st, bytes, mode, ia, fa, oa, cv);
    else
        (ints ? launch_fin12<PRO, 1, false, DROP, true> : launch_fin12<PRO, 1, false, DROP, false>)(c, st, bytes, mode, ia, fa, oa, cv);
}
void fin12_few(he_ctx *c, hipStream_t st, double bytes, int pro, bool drop, bool ints, int mode, const InnerArgs &ia, const FinishArgs &fa,
               const OpArgs &oa, const ConvArgs &cv)
{
    (drop ? fin12_of<PRO_MODDOWN, true> : pro == PRO_MODDOWN_RS ? fin12_of<PRO_MODDOWN_RS, false> : fin12_of<PRO_MODDOWN, false>)(c, st, bytes, ints, mode, ia, fa, oa, cv);
}
#else
template <int PRO>
static void fwd12(he_ctx *c, hipStream_t st, double bytes, bool wide, u64 *data, const LimbBatch &lb, int nb,
                  const ConvArgs &cv, const FinArgs *fin)
{
    if constexpr (PRO == PRO_MODUP) {
        if (!cv.exact && !wide && c->alpha <= 2)
            fwd12_modup_few(c, st, bytes, data, lb, nb, cv);
        else if (cv.exact)
            (wide ? launch_fwd12<PRO, 8, true> : launch_fwd12<PRO, 4, true>)(c, st, bytes, data, lb, nb, cv, fin);
        else
            (wide ? launch_fwd12<PRO, 8, false> : launch_fwd12<PRO, 4, false>)(c, st, bytes, data, lb, nb, cv, fin);
    } else
        launch_fwd12<PRO, 4, false>(c, st, bytes, data, lb, nb, cv, fin);
}
static void inv12(he_ctx *c, hipStream_t st, double bytes, int scale, const u64 *src, const u64 *src2, u64 *dst, const LimbBatch &lb, int nb,
                  const ConvArgs &cv)
{
    switch (scale) { // special limbs are scaled where they are produced
    case SCALE_NONE: KLAUNCH_T(c, st, KID_INV12, bytes, (k_ntt_inv12<SCALE_NONE>), nb, N12_THREADS, src, src2, dst, c->dev, lb, cv); break;
    default: KLAUNCH_T(c, st, KID_INV12, bytes, (k_ntt_inv12<SCALE_MODUP>), nb, N12_THREADS, src, src2, dst, c->dev, lb, cv); break;
    }
}
static void inner12(he_ctx *c, hipStream_t st, double bytes, const InnerArgs &ia, const OpArgs &oa)
{
    if (ia.ta)
        KLAUNCH_T(c, st, KID_INNER12, bytes, (k_inner12<true>), dim3(ia.level + ia.K, 2, ia.count), N12_THREADS, ia, c->dev, oa);
    else
        KLAUNCH_T(c, st, KID_INNER12, bytes, (k_inner12<false>), dim3(ia.level + 2 * ia.K, 1, ia.count), N12_THREADS, ia, c->dev, oa);
}
template <int PRO, bool DROP, bool INTS>
static void fin12_of(he_ctx *c, hipStream_t st, double bytes, bool wide, int mode, const InnerArgs &ia, const FinishArgs &fa, const OpArgs &oa,
                     const ConvArgs &cv)
{
    if (cv.exact)
        (wide ? launch_fin12<PRO, 8, true, DROP, INTS> : launch_fin12<PRO, 4, true, DROP, INTS>)(c, st, bytes, mode, ia, fa, oa, cv);
    else
        (wide ? launch_fin12<PRO, 8, false, DROP, INTS> : launch_fin12<PRO, 4, false, DROP, INTS>)(c, st, bytes, mode, ia, fa, oa, cv);
}
static void fin12(he_ctx *c, hipStream_t st, double bytes, bool wide, int pro, bool drop, int mode, const InnerArgs &ia,
                  const FinishArgs &fa, const OpArgs &oa, const ConvArgs &cv)
{
    bool ints = false;
    for (int i = 0; i < ia.level; i++) ints |= c->modc[i].qd == 0.0;
    if (!cv.exact && !wide && c->K <= 2)
        fin12_few(c, st, bytes, pro, drop, ints, mode, ia, fa, oa, cv);
    else if (drop)
        (ints ? fin12_of<PRO_MODDOWN, true, true> : fin12_of<PRO_MODDOWN, true, false>)(c, st, bytes, wide, mode, ia, fa, oa, cv);
    else if (pro == PRO_MODDOWN_RS)
        (ints ? fin12_of<PRO_MODDOWN_RS, false, true> : fin12_of<PRO_MODDOWN_RS, false, false>)(c, st, bytes, wide, mode, ia, fa, oa, cv);
    else
        (ints ? fin12_of<PRO_MODDOWN, false, true> : fin12_of<PRO_MODDOWN, false, false>)(c, st, bytes, wide, mode, ia, fa, oa, cv);
}
void dev_launch_n12(DevLaunch &t)
{
    t.fwd_limb[PRO_LOAD] = fwd12<PRO_LOAD>;
    t.fwd_limb[PRO_MODUP] = fwd12<PRO_MODUP>;
    t.fwd_limb[PRO_RESCALE] = fwd12<PRO_RESCALE>;
    t.inv_limb = inv12;
    t.inner_limb = inner12;
    t.fin_limb = fin12;
}
#endif
