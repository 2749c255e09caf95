// Conversion kernels of the ring size N = 2^HE_LOGN (16 or 17) and their launchers.
#include "launch.h"

template <int NS> static void modup_sources(he_ctx *c, hipStream_t st, double bytes, int count, const ModUpArgs &ua)
{
    KLAUNCH_T(c, st, KID_FWD_COLS_MODUP, bytes, (k_ntt_fwd_cols_modup<HE_LOGN, NS>), CONV_GROUPS * count * ua.beta * ua.chunks,
              (64 * ConvGeom<HE_LOGN, NS>::WAVES), ua, c->dev);
}
template <int K> static void moddown_sources(he_ctx *c, hipStream_t st, double bytes, bool rs, int count, const ModDownArgs &da)
{
    const int grid = CONV_GROUPS * 2 * count * da.chunks, threads = 64 * ConvGeom<HE_LOGN, K>::DOWN_WAVES;
    if (rs)
        KLAUNCH_T(c, st, KID_FWD_COLS_MODDOWN_RS, bytes, (k_ntt_fwd_cols_moddown<HE_LOGN, true, K>), grid, threads, da, c->dev);
    else
        KLAUNCH_T(c, st, KID_FWD_COLS_MODDOWN, bytes, (k_ntt_fwd_cols_moddown<HE_LOGN, false, K>), grid, threads, da, c->dev);
}
static void modup(he_ctx *c, hipStream_t st, double bytes, int count, const ModUpArgs &ua)
{
#if HE_LOGN == 16
    if (ua.alpha > 4) return modup_sources<8>(c, st, bytes, count, ua);
#endif
    modup_sources<4>(c, st, bytes, count, ua); // more are refused at N = 2^17 when the context is created
}
static void moddown(he_ctx *c, hipStream_t st, double bytes, bool rs, int count, const ModDownArgs &da)
{
#if HE_LOGN == 16
    if (da.K > 4) return moddown_sources<8>(c, st, bytes, rs, count, da);
#endif
    moddown_sources<4>(c, st, bytes, rs, count, da);
}

#define PASTE_(a, b) a##b
#define PASTE(a, b) PASTE_(a, b)
void PASTE(dev_launch_conv, HE_LOGN)(DevLaunch &t) { t.modup = modup, t.moddown = moddown; }
