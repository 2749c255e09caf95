// Kernel launch plumbing shared by the translation units of the device library.
//
// The kernels are templates over the ring size; each ring size is instantiated in a translation unit of
// its own (dev_n12.hip twice, dev_n16_blocks.hip, dev_n17_blocks.hip, dev_conv.hip once per larger ring size, and dev_cols.hip once per larger
// ring size and prologue) so that the library builds in parallel, and device.hip reaches them through one table of launchers per ring size.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "kernels_ks.h"

// ---- optional per-kernel timing with HIP events on the launch stream (he_profile_start/stop)
enum KernelId {
    KID_FWD_COLS, KID_FWD_COLS_MODUP, KID_FWD_COLS_MODDOWN, KID_FWD_COLS_RESCALE, KID_FWD_COLS_MODDOWN_RS, KID_FWD_BLOCKS,
    KID_FWD_BLOCKS_FIN,
    KID_INV_BLOCKS, KID_INV_COLS, KID_LIMBWISE, KID_CMULT, KID_COPY, KID_INNER_SPECIAL, KID_INNER_FINISHED, KID_INNER_FIN,
    KID_FWD12, KID_FWD12_MODUP, KID_FWD12_RESCALE, KID_INV12, KID_INNER12, KID_FIN12, // N = 2^12
    KID_COUNT
};

// Creates the event pair of one profiled launch and appends it to the context's record list.
bool prof_events(he_ctx *c, int kid, double bytes, ProfRecord &r);

// Launch wrapper: `bytes` = bytes the launch has to move by the definition of its step.  While profiling,
// the launch carries a start and a stop event that take the kernel's own begin and end timestamps.
#define KLAUNCH_T(c, st, kid, bytes, kernel, grid, threads, ...)                                                    \
    do {                                                                                                             \
        ProfRecord pr_;                                                                                              \
        if ((c)->prof_on && prof_events((c), (kid), (double)(bytes), pr_))                                           \
            hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, (st), (hipEvent_t)pr_.a, (hipEvent_t)pr_.b,   \
                                  0, __VA_ARGS__);                                                                   \
        else                                                                                                         \
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, (st), __VA_ARGS__);                             \
    } while (0)
#define KLAUNCH(c, st, kid, bytes, kernel, grid, ...) KLAUNCH_T(c, st, kid, bytes, kernel, grid, 256, __VA_ARGS__)
// work-groups per limb of the block pass
#define BLK_TILES(c) ((int)((c)->N / (256 * BLK_PER_WG)))

// Launchers of one ring size.  `wide`: a base conversion has more than four source limbs.
struct DevLaunch {
    // Ring sizes whose limbs fit one work-group (N = 2^12; null otherwise) have whole transforms and key-switch halves in
    // place of the passes below: fwd_limb, with the finishing epilogue if fin is not null; inv_limb; the inner product, with
    // the special limbs' inverse transform; the finishing of the first fa.nl limbs (rescale: with the dropped limb's
    // share in the corrections; drop: of the dropped limb alone, into fa.r).
    void (*fwd_limb[5])(he_ctx *c, hipStream_t st, double bytes, bool wide, u64 *data, const LimbBatch &lb, int nb,
                        const ConvArgs &cv, const FinArgs *fin);
    void (*inv_limb)(he_ctx *c, hipStream_t st, double bytes, int scale, const u64 *src, const u64 *src2, u64 *dst, const LimbBatch &lb, int nb,
                     const ConvArgs &cv);
    void (*inner_limb)(he_ctx *c, hipStream_t st, double bytes, const InnerArgs &ia, const OpArgs &oa);
    void (*fin_limb)(he_ctx *c, hipStream_t st, double bytes, bool wide, int pro, bool drop, int mode, const InnerArgs &ia,
                     const FinishArgs &fa, const OpArgs &oa, const ConvArgs &cv);
    // forward column pass of the nb limbs of lb, one launcher per prologue (PRO_*)
    void (*fwd_cols[5])(he_ctx *c, hipStream_t st, int kid, double bytes, bool wide, u64 *data, const LimbBatch &lb, int nb,
                        const ConvArgs &cv);
    // the same with the corrected base conversions (entries of prologues without a conversion stay null)
    void (*fwd_cols_ex[5])(he_ctx *c, hipStream_t st, int kid, double bytes, bool wide, u64 *data, const LimbBatch &lb, int nb,
                           const ConvArgs &cv);
    // forward block pass of the first nb limbs of lb with epilogue epi; pairs: their rows are interleaved (EPI_FIN: never, EPI_FIN_INV: always)
    void (*fwd_blocks)(he_ctx *c, hipStream_t st, double bytes, int epi, bool pairs, u64 *data, const LimbBatch &lb, int nb,
                       const FinArgs &fa);
    // src2: null, or a second factor of the transform's input
    void (*inv_blocks)(he_ctx *c, hipStream_t st, double bytes, const u64 *src, const u64 *src2, u64 *dst, const LimbBatch &lb, int nb);
    void (*inv_cols)(he_ctx *c, hipStream_t st, double bytes, int scale, u64 *dst, const LimbBatch &lb, int nb,
                     const ConvArgs &cv);
    // ModUp of `count` operations with the inverse column pass ahead of it: digits of up to eight limbs (N = 2^17: four) on the floating-point path
    void (*modup)(he_ctx *c, hipStream_t st, double bytes, int count, const ModUpArgs &ua);
    // ModDown's corrections of `count` operations with the inverse column pass ahead of it; rs: with a rescale
    void (*moddown)(he_ctx *c, hipStream_t st, double bytes, bool rs, int count, const ModDownArgs &da);
    // inner product on the limbs ia.first .. level + K - 1, and the finishing one on the first fa.nl limbs (path: FIN_FP, ..)
    void (*inner)(he_ctx *c, hipStream_t st, double bytes, unsigned grid, const InnerArgs &ia, const OpArgs &oa);
    void (*inner_fin)(he_ctx *c, hipStream_t st, double bytes, unsigned grid, int mode, int path, const InnerArgs &ia, const FinishArgs &fa,
                      const OpArgs &oa);
};
// Each translation unit fills its part of a ring size's table: dev_launch_cols<logN>_<p> the forward
// column pass with prologue p (p = 5: the inverse column pass).
void dev_launch_n12(DevLaunch &t);
void dev_launch_n16_blocks(DevLaunch &t);
void dev_launch_n17_blocks(DevLaunch &t);
void dev_launch_conv16(DevLaunch &t);
void dev_launch_conv17(DevLaunch &t);
#define HE_DECL_COLS(n)                                                                                              \
    void dev_launch_cols##n##_0(DevLaunch &t);                                                                       \
    void dev_launch_cols##n##_1(DevLaunch &t);                                                                       \
    void dev_launch_cols##n##_2(DevLaunch &t);                                                                       \
    void dev_launch_cols##n##_3(DevLaunch &t);                                                                       \
    void dev_launch_cols##n##_4(DevLaunch &t);                                                                       \
    void dev_launch_cols##n##_5(DevLaunch &t);                                                                       \
    void dev_launch_cols_ex##n##_1(DevLaunch &t);                                                                    \
    void dev_launch_cols_ex##n##_2(DevLaunch &t);                                                                    \
    void dev_launch_cols_ex##n##_4(DevLaunch &t);
HE_DECL_COLS(16)
HE_DECL_COLS(17)
#undef HE_DECL_COLS

// ---- launcher bodies, instantiated by the per-ring-size translation units ------------------------------

template <int LOGN>
static void launch_fwd_blocks(he_ctx *c, hipStream_t st, double bytes, int epi, bool pairs, u64 *data, const LimbBatch &lb, int nb, const FinArgs &fa)
{
    const int grid = BLK_TILES(c) * nb;
    if (epi == EPI_FIN_INV) // of a Mult's dropped limb, behind its ModDown
        KLAUNCH_T(c, st, KID_FWD_BLOCKS_FIN, bytes, (k_ntt_fwd_blocks<LOGN, EPI_FIN_INV, true, true>), grid, BLK_THREADS, data, c->dev, lb, fa);
    else if (epi == EPI_FIN && grid <= FIN_AHEAD_GROUPS) // of a rescale
        KLAUNCH_T(c, st, KID_FWD_BLOCKS_FIN, bytes, (k_ntt_fwd_blocks<LOGN, EPI_FIN, false, true>), grid, BLK_THREADS, data, c->dev, lb, fa);
    else if (epi == EPI_FIN)
        KLAUNCH_T(c, st, KID_FWD_BLOCKS_FIN, bytes, (k_ntt_fwd_blocks<LOGN, EPI_FIN, false, false>), grid, BLK_THREADS, data, c->dev, lb, fa);
    else if (pairs)
        KLAUNCH_T(c, st, KID_FWD_BLOCKS, bytes, (k_ntt_fwd_blocks<LOGN, EPI_STORE, true, false>), grid, BLK_THREADS, data, c->dev, lb, fa);
    else
        KLAUNCH_T(c, st, KID_FWD_BLOCKS, bytes, (k_ntt_fwd_blocks<LOGN, EPI_STORE, false, false>), grid, BLK_THREADS, data, c->dev, lb, fa);
}
template <int LOGN>
static void launch_inv_blocks(he_ctx *c, hipStream_t st, double bytes, const u64 *src, const u64 *src2, u64 *dst,
                              const LimbBatch &lb, int nb)
{
    if (src2)
        KLAUNCH_T(c, st, KID_INV_BLOCKS, bytes, (k_ntt_inv_blocks<LOGN, true>), BLK_TILES(c) * nb, BLK_THREADS, src, src2, dst, c->dev, lb);
    else
        KLAUNCH_T(c, st, KID_INV_BLOCKS, bytes, (k_ntt_inv_blocks<LOGN, false>), BLK_TILES(c) * nb, BLK_THREADS, src, src2, dst, c->dev, lb);
}
template <int LOGN>
static void launch_inner(he_ctx *c, hipStream_t st, double bytes, unsigned grid, const InnerArgs &ia, const OpArgs &oa)
{
    const bool mult = ia.ta && ia.first < ia.level; // the dropped limb of a Mult is among them
    if (ia.finished) {
        if (mult)
            KLAUNCH_T(c, st, KID_INNER_FINISHED, bytes, (k_inner_finished<LOGN, true>), grid, SPECIAL_THREADS, ia, c->dev, oa);
        else
            KLAUNCH_T(c, st, KID_INNER_FINISHED, bytes, (k_inner_finished<LOGN, false>), grid, SPECIAL_THREADS, ia, c->dev, oa);
    } else {
        if (mult)
            KLAUNCH_T(c, st, KID_INNER_SPECIAL, bytes, (k_inner_special<LOGN, true>), grid, SPECIAL_THREADS, ia, c->dev, oa);
        else
            KLAUNCH_T(c, st, KID_INNER_SPECIAL, bytes, (k_inner_special<LOGN, false>), grid, SPECIAL_THREADS, ia, c->dev, oa);
    }
}
template <int LOGN, int MODE>
static void launch_inner_fin_mode(he_ctx *c, hipStream_t st, double bytes, unsigned grid, int path, const InnerArgs &ia, const FinishArgs &fa,
                                  const OpArgs &oa)
{
    if (path == FIN_FP)
        KLAUNCH_T(c, st, KID_INNER_FIN, bytes, (k_inner_fin<LOGN, MODE, FIN_FP>), grid, INNER_THREADS, ia, fa, c->dev, oa);
    else if (path == FIN_INT)
        KLAUNCH_T(c, st, KID_INNER_FIN, bytes, (k_inner_fin<LOGN, MODE, FIN_INT>), grid, INNER_THREADS, ia, fa, c->dev, oa);
    else
        KLAUNCH_T(c, st, KID_INNER_FIN, bytes, (k_inner_fin<LOGN, MODE, FIN_BOTH>), grid, INNER_THREADS, ia, fa, c->dev, oa);
}
template <int LOGN>
static void launch_inner_fin(he_ctx *c, hipStream_t st, double bytes, unsigned grid, int mode, int path, const InnerArgs &ia, const FinishArgs &fa,
                             const OpArgs &oa)
{
    if (mode == FIN_MULT)
        launch_inner_fin_mode<LOGN, FIN_MULT>(c, st, bytes, grid, path, ia, fa, oa);
    else if (mode == FIN_ROT)
        launch_inner_fin_mode<LOGN, FIN_ROT>(c, st, bytes, grid, path, ia, fa, oa);
    else
        launch_inner_fin_mode<LOGN, FIN_ROTSUM>(c, st, bytes, grid, path, ia, fa, oa);
}
