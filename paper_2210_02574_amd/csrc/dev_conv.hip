// Conversion kernels of the ring size N = 2^HE_LOGN (16 or 17) and their launchers.
#include "launch.h"

static void modup(he_ctx *c, hipStream_t st, double bytes, int count, const ModUpArgs &ua)
{
    KLAUNCH_T(c, st, KID_FWD_COLS_MODUP, bytes, (k_ntt_fwd_cols_modup<HE_LOGN>), CONV_GROUPS * count * ua.beta * ua.chunks, 64 * ConvGeom<HE_LOGN>::WAVES, ua, c->dev);
}

static void moddown(he_ctx *c, hipStream_t st, double bytes, bool rs, int count, const ModDownArgs &da)
{
    const int grid = CONV_GROUPS * 2 * count * da.chunks, threads = 64 * ConvGeom<HE_LOGN>::DOWN_WAVES;
    if (rs)
        KLAUNCH_T(c, st, KID_FWD_COLS_MODDOWN_RS, bytes, (k_ntt_fwd_cols_moddown<HE_LOGN, true>), grid, threads, da, c->dev);
    else
        KLAUNCH_T(c, st, KID_FWD_COLS_MODDOWN, bytes, (k_ntt_fwd_cols_moddown<HE_LOGN, false>), grid, threads, da, c->dev);
}

#define PASTE_(a, b) a##b
#define PASTE(a, b) PASTE_(a, b)
void PASTE(dev_launch_conv, HE_LOGN)(DevLaunch &t) { t.modup = modup, t.moddown = moddown; }
