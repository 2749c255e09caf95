// Device-side entry points of the RNS-CKKS library: table upload, kernel launch sequences of
// NTT, Mult (tensor product + relinearisation), Rotate (hybrid key switching), rescale and
// rotate-and-sum.  The kernels are in kernels_ntt.h, kernels_conv.h, kernels_ks.h, kernels_n12.h and kernels_elem.h.
//
// Key switch of a polynomial d (NTT domain, `level` limbs) with key evk, Galois element g:
//   1. inverse NTT of d, its column pass also multiplying limb i by (D/q_i)^-1      -> y  (ws.x)
//   2. forward NTT of every raised limb (digit j, modulus t outside the digit), the
//      column pass summing y_i (D/q_i mod t) on the fly (ModUp)                     -> raised
//   3. inner product with the key on the special limbs, reading the digits through the index map of g -> u
//   4. inverse NTT of these, scaled by (P/p_k)^-1                                    (in place)
//   5. column pass of the forward NTT of the 2*level ModDown corrections, summing
//      y_k (P/p_k mod q_i) over centred digits y_k                                     -> r
//   6. inner product on the ciphertext limbs (the digit's own limbs straight from d), block pass of r and
//      out = (u - r) P^-1 + addend, in one kernel                                      -> out
// N = 2^16 and 2^17: the inverse column passes of steps 1 and 4 are part of the kernels of steps 2 and 5 (kernels_conv.h) where conv_pays() says
// so, five launches in all; the coefficients then stay in LDS.
// Hoisted rotations share steps 1-2.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <functional>
#include <mutex>
#include <vector>

#include "kernels_elem.h"
#include "launch.h"

#define HIP_TRY(ctx, expr)                                                                                           \
    do {                                                                                                             \
        hipError_t e_ = (expr);                                                                                      \
        if (e_ != hipSuccess) {                                                                                      \
            (ctx)->hip_err = std::string(#expr) + ": " + hipGetErrorString(e_);                                      \
            return HE_EHIP;                                                                                          \
        }                                                                                                            \
    } while (0)

// Scratch array of he_hrot_noalloc: the workspace of one rotation for callers that cannot allocate and pass
// none.  Every GPU the library runs on holds its own copy at its own address; in host code the name below is
// only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned long long scratch[HE_STATIC_SCRATCH_BYTES / sizeof(unsigned long long)];

// Address of `scratch` on the context's device, asked for once per device (the caller has made that device
// current) and kept: kernels and copies take this pointer, never the array's name.
static int32_t static_scratch_address(he_ctx *c)
{
    static std::mutex mu;
    static u64 *per_device[64] = {};
    std::lock_guard<std::mutex> lock(mu);
    if (c->device < 0 || c->device >= 64) return HE_EINVAL;
    if (!per_device[c->device]) {
        void *p = nullptr;
        HIP_TRY(c, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) {
            c->hip_err = "hipGetSymbolAddress(scratch) returned a null address";
            return HE_EHIP;
        }
        per_device[c->device] = (u64 *)p;
    }
    c->static_scratch = per_device[c->device];
    return HE_OK;
}

template <class Tv> static int32_t upload(he_ctx *c, const std::vector<Tv> &v, const Tv **out)
{
    void *p = nullptr;
    const size_t bytes = std::max<size_t>(v.size() * sizeof(Tv), 16);
    HIP_TRY(c, hipMalloc(&p, bytes));
    c->dev_allocs.push_back(p);
    if (!v.empty()) HIP_TRY(c, hipMemcpy(p, v.data(), v.size() * sizeof(Tv), hipMemcpyHostToDevice));
    *out = (const Tv *)p;
    return HE_OK;
}

int32_t dev_upload_tables(he_ctx *c)
{
    if (c->logN != 12 && c->logN != 16 && c->logN != 17) return HE_EINVAL;
    if (c->alpha > 8 || c->K > 8 || c->M > 64) return HE_EINVAL; // conversion kernels are built for up to 8 sources
    if (c->logN == 17 && (c->alpha > 4 || c->K > 4)) return HE_EINVAL; // ... and for up to 4 at N = 2^17
    HIP_TRY(c, hipSetDevice(c->device));
    int32_t rc;
    if ((rc = static_scratch_address(c)) != HE_OK) return rc; // once per context, with its device current
    HIP_TRY(c, hipGetFuncBySymbol((hipFunction_t *)&c->copy_kernel, (const void *)k_copy_limbs));
#define UP(field)                                                                                                    \
    if ((rc = upload(c, c->field, &c->dev.field)) != HE_OK) return rc;
    if ((rc = upload(c, c->modc, &c->dev.mod)) != HE_OK) return rc;
    UP(tw_fwd) UP(tw_inv) UP(ninv) UP(twd_fwd) UP(twd_blk) UP(twd_inv) UP(ninvd)
    UP(up_inv) UP(up_hat) UP(up_inv_d) UP(up_hat_d) UP(up_hat_dh) UP(rq) UP(up_dmod) UP(up_dmod_d) UP(up_hat_p) UP(dn_r50_d)
    UP(dn_inv) UP(dn_hat) UP(dn_pinv) UP(dn_inv_d) UP(dn_hat_d) UP(dn_hat_dh) UP(dn_pinv_d) UP(dn_pmod) UP(dn_pmod_d)
    UP(rs_inv) UP(rs_inv_d) UP(rsp_inv) UP(rsp_inv_d)
#undef UP
    c->dev.up_split = c->up_split ? 1 : 0;
    c->dev.dn_split = c->dn_split ? 1 : 0;
    c->dev.dn_fold = c->dn_fold ? 1 : 0;
    return HE_OK;
}

void dev_free_tables(he_ctx *c)
{
    for (void *p : c->dev_allocs) (void)hipFree(p);
    c->dev_allocs.clear();
}

// Device form of a key: limbs of a modulus below 2^50 (the floating-point path) hold balanced residues as
// doubles (v, or v - q above (q-1)/2), the other limbs the residues themselves.  The inner product then
// multiplies key words without converting them, and products with |word| <= q/2 are exact for wider inputs.
int32_t dev_upload_evk(he_evk *k)
{
    he_ctx *c = const_cast<he_ctx *>(k->ctx);
    const size_t N = c->N, limbs = (size_t)c->dnum * 2 * c->M;
    std::vector<u64> img;
    try {
        img.resize(limbs * N);
    } catch (...) {
        return HE_ENOMEM;
    }
    std::atomic<bool> bad(false);
    hostmath::parallel_for((int)limbs, [&](int l) {
        const ModConst &m = c->modc[l % c->M];
        const u64 *src = k->host.data() + (size_t)l * N, half = (m.q - 1) / 2;
        u64 *dst = img.data() + (size_t)l * N;
        bool b = false;
        for (size_t n = 0; n < N; n++) {
            const u64 v = src[n];
            b |= v >= m.q;
            if (m.qd != 0.0) {
                const double d = v > half ? -(double)(m.q - v) : (double)v;
                memcpy(&dst[n], &d, sizeof(d));
            } else
                dst[n] = v;
        }
        if (b) bad = true;
    });
    if (bad) return HE_EINVAL; // a residue that is not below its modulus
    HIP_TRY(c, hipSetDevice(c->device));
    HIP_TRY(c, hipMalloc((void **)&k->dev, img.size() * sizeof(u64)));
    hipError_t e = hipMemcpy(k->dev, img.data(), img.size() * sizeof(u64), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        c->hip_err = std::string("hipMemcpy (key upload): ") + hipGetErrorString(e);
        (void)hipFree(k->dev);
        k->dev = nullptr;
        return HE_EHIP;
    }
    return HE_OK;
}

void dev_free_evk(he_evk *k)
{
    if (k->dev) (void)hipFree(k->dev);
    k->dev = nullptr;
}

extern "C" int32_t he_evk_to_host(const he_evk *evk, uint64_t *h_out)
{
    if (!evk || !h_out) return HE_EINVAL;
    const he_ctx *c = evk->ctx;
    const size_t N = c->N, limbs = (size_t)c->dnum * 2 * c->M, words = limbs * N;
    if (!evk->dev) {
        memcpy(h_out, evk->host.data(), words * sizeof(u64));
        return HE_OK;
    }
    he_ctx *cm = const_cast<he_ctx *>(c);
    HIP_TRY(cm, hipMemcpy(h_out, evk->dev, words * sizeof(u64), hipMemcpyDeviceToHost));
    hostmath::parallel_for((int)limbs, [&](int l) { // back from the device form to residues
        const ModConst &m = c->modc[l % c->M];
        if (m.qd == 0.0) return;
        u64 *w = h_out + (size_t)l * N;
        for (size_t n = 0; n < N; n++) {
            double d;
            memcpy(&d, &w[n], sizeof(d));
            w[n] = d < 0.0 ? m.q - (u64)(-d) : (u64)d;
        }
    });
    return HE_OK;
}

// ---- optional per-kernel timing with HIP events on the launch stream (he_profile_start/stop)
static const char *const kKernelNames[KID_COUNT] = {
    "k_ntt_fwd_cols", "k_ntt_fwd_cols_modup", "k_ntt_fwd_cols_moddown", "k_ntt_fwd_cols_rescale", "k_ntt_fwd_cols_moddown_rescale",
    "k_ntt_fwd_blocks",
    "k_ntt_fwd_blocks_fin", "k_ntt_inv_blocks", "k_ntt_inv_cols", "k_limbwise", "k_cmult", "k_copy_limbs", "k_inner_special", "k_inner_finished",
    "k_inner_fin", "k_ntt_fwd12", "k_ntt_fwd12_modup", "k_ntt_fwd12_rescale", "k_ntt_inv12", "k_inner12", "k_fin12"};

bool prof_events(he_ctx *c, int kid, double bytes, ProfRecord &r)
{
    r.kid = kid;
    r.bytes = bytes;
    r.a = r.b = nullptr;
    if (hipEventCreate((hipEvent_t *)&r.a) != hipSuccess) return false;
    if (hipEventCreate((hipEvent_t *)&r.b) != hipSuccess) {
        (void)hipEventDestroy((hipEvent_t)r.a);
        return false;
    }
    c->prof.push_back(r);
    return true;
}

// launchers of the context's ring size (dev_upload_tables has checked that it is one of the three)
static const DevLaunch &dev_launch(const he_ctx *c)
{
    static const DevLaunch tables[3] = {
        [] { DevLaunch t{}; dev_launch_n12(t); return t; }(),
        [] {
            DevLaunch t{};
            dev_launch_cols16_0(t), dev_launch_cols16_1(t), dev_launch_cols16_2(t), dev_launch_cols16_3(t);
            dev_launch_cols16_4(t), dev_launch_cols16_5(t), dev_launch_n16_blocks(t), dev_launch_conv16(t);
            dev_launch_cols_ex16_1(t), dev_launch_cols_ex16_2(t), dev_launch_cols_ex16_4(t);
            return t;
        }(),
        [] {
            DevLaunch t{};
            dev_launch_cols17_0(t), dev_launch_cols17_1(t), dev_launch_cols17_2(t), dev_launch_cols17_3(t);
            dev_launch_cols17_4(t), dev_launch_cols17_5(t), dev_launch_n17_blocks(t), dev_launch_conv17(t);
            dev_launch_cols_ex17_1(t), dev_launch_cols_ex17_2(t), dev_launch_cols_ex17_4(t);
            return t;
        }(),
    };
    return tables[c->logN == 12 ? 0 : c->logN == 16 ? 1 : 2];
}

extern "C" int32_t he_profile_start(he_ctx *ctx)
{
    if (!ctx) return HE_EINVAL;
    if (ctx->device < 0) return HE_ENODEV;
    ctx->prof_on = true;
    return HE_OK;
}

extern "C" int32_t he_profile_stop(he_ctx *ctx, he_kernel_stat *out, int32_t max_out, int32_t *n_out)
{
    if (!ctx || !out || !n_out || max_out < 0) return HE_EINVAL;
    ctx->prof_on = false;
    double ms[KID_COUNT] = {0}, bytes[KID_COUNT] = {0};
    int64_t cnt[KID_COUNT] = {0};
    int32_t rc = HE_OK;
    for (ProfRecord &r : ctx->prof) {
        float t = 0.f;
        if (r.a && r.b && hipEventSynchronize((hipEvent_t)r.b) == hipSuccess &&
            hipEventElapsedTime(&t, (hipEvent_t)r.a, (hipEvent_t)r.b) == hipSuccess) {
            ms[r.kid] += t;
            bytes[r.kid] += r.bytes;
            cnt[r.kid]++;
        } else
            rc = HE_EHIP;
        if (r.a) (void)hipEventDestroy((hipEvent_t)r.a);
        if (r.b) (void)hipEventDestroy((hipEvent_t)r.b);
    }
    ctx->prof.clear();
    int32_t n = 0;
    for (int k = 0; k < KID_COUNT; k++) {
        if (!cnt[k]) continue;
        if (n < max_out) {
            memset(&out[n], 0, sizeof(out[n]));
            strncpy(out[n].name, kKernelNames[k], sizeof(out[n].name) - 1);
            out[n].launches = cnt[k];
            out[n].total_ms = ms[k];
            out[n].bytes = bytes[k];
        }
        n++;
    }
    *n_out = n;
    if (n > max_out && rc == HE_OK) rc = HE_EINVAL; // the caller's array is too small: n_out says how many are needed
    return rc;
}

static inline int32_t launch_ok(he_ctx *c)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        c->hip_err = std::string("kernel launch: ") + hipGetErrorString(e);
        return HE_EHIP;
    }
    return HE_OK;
}

// ---- limb lists -----------------------------------------------------------------------------------

struct LimbList {
    std::vector<int> slot, src, mod;
    void add(int s, int m) { slot.push_back(s), src.push_back(s), mod.push_back(m); }
    void add(int s, int from, int m) { slot.push_back(s), src.push_back(from), mod.push_back(m); }
    void reserve(int n) { slot.reserve(n), src.reserve(n), mod.reserve(n); }
    int size() const { return (int)slot.size(); }
};

// calls launch(batch, count) for chunks of at most HE_MAXB limbs; within a chunk the limbs on the integer path
// (moduli of 2^50 and above) take about three times longer and are scheduled first, so that the others fill in
// behind them
template <class F> static int32_t for_batches(he_ctx *c, const LimbList &l, F launch)
{
    const int total = l.size();
    std::vector<int> order(HE_MAXB);
    // chunks of equal size (even, so that pairs of limbs stay together) rather than full ones and a small rest
    const int nchunks = (total + HE_MAXB - 1) / HE_MAXB;
    const int per = nchunks ? std::min(HE_MAXB, ((total + nchunks - 1) / nchunks + 1) & ~1) : 0;
    for (int off = 0; off < total; off += per) {
        const int nb = std::min(per, total - off);
        for (int b = 0; b < nb; b++) order[b] = off + b;
        std::stable_partition(order.begin(), order.begin() + nb, [&](int b) { return c->modc[l.mod[b]].qd == 0.0; });
        LimbBatch lb;
        for (int b = 0; b < nb; b++) {
            const int o = order[b];
            lb.slot[b] = (uint16_t)l.slot[o];
            lb.src[b] = (uint16_t)l.src[o];
            lb.mod[b] = (uint8_t)l.mod[o];
        }
        launch(lb, nb);
        int32_t rc = launch_ok(c);
        if (rc != HE_OK) return rc;
    }
    return HE_OK;
}

static ConvArgs conv_args(const he_ctx *c, const u64 *src, int level, int dst_stride = 1 << 30, int src_stride = 0)
{
    ConvArgs cv;
    cv.src = src;
    cv.level = level;
    cv.L = c->L;
    cv.K = c->K;
    cv.alpha = c->alpha;
    cv.dst_stride = dst_stride;
    cv.src_stride = src_stride;
    cv.src2 = nullptr;
    cv.src2_stride = 0;
    cv.rs_mod = level - 1;
    cv.rs_nl = level - 1;
    cv.exact = c->exact_conv;
    memset(cv.op_level, 0, sizeof(cv.op_level));
    return cv;
}

static const FinArgs kNoFin = {nullptr, nullptr, nullptr, nullptr, 0, 0, 1, 1 << 30, 0, 0};
static const OpArgs kNoOps = {};

// Forward NTT of the listed limbs of `data`.  pro selects what the column pass transforms (the
// limb's own content, or a base conversion of cv.src); with fin != nullptr the block pass writes
// (u - ntt) * const to fin->out instead of the transform itself.
// src_limbs = number of source limbs the prologue reads in total (for the byte count).
// blocks: the limbs whose block pass runs here (the others are finished by the kernel that consumes them): all, none, or
// the ciphertext limbs on the integer path and every limb with a modulus index from finish_from on.
enum { BLOCKS_ALL, BLOCKS_SOME, BLOCKS_NONE };
static int32_t ntt_forward(he_ctx *c, hipStream_t st, u64 *data, const LimbList &l, int pro, const ConvArgs &cv,
                           const FinArgs *fin, int src_limbs, int blocks = BLOCKS_ALL, int finish_from = 0)
{
    const bool wide = std::max(c->alpha, c->K) > 4;
    const double N8 = (double)c->N * 8.0;
    const DevLaunch &dl = dev_launch(c);
    int32_t rc = for_batches(c, l, [&](const LimbBatch &lb, int nb) {
        const double cols_bytes = pro == PRO_LOAD ? 2.0 * nb * N8 : (double)(src_limbs + nb) * N8;
        const int kid_cols = pro == PRO_LOAD      ? KID_FWD_COLS
                             : pro == PRO_MODUP   ? KID_FWD_COLS_MODUP
                             : pro == PRO_MODDOWN ? KID_FWD_COLS_MODDOWN
                             : pro == PRO_MODDOWN_RS ? KID_FWD_COLS_MODDOWN_RS
                                                  : KID_FWD_COLS_RESCALE;
        if (dl.fwd_limb[pro]) { // the whole transform in one launch, on every limb
            dl.fwd_limb[pro](c, st, cols_bytes + (fin ? (double)nb * N8 : 0.0), wide, data, lb, nb, cv, fin);
            return;
        }
        (cv.exact && dl.fwd_cols_ex[pro] ? dl.fwd_cols_ex[pro] : dl.fwd_cols[pro])(c, st, kid_cols, cols_bytes, wide, data, lb, nb, cv);
        if (fin) {
            // reads the transform's input and the minuend, writes the result
            dl.fwd_blocks(c, st, 3.0 * nb * N8, EPI_FIN, false, data, lb, nb, *fin);
        } else if (blocks == BLOCKS_ALL)
            dl.fwd_blocks(c, st, 2.0 * nb * N8, EPI_STORE, pro_pairs_rows(pro), data, lb, nb, kNoFin);
    });
    if (rc != HE_OK || blocks != BLOCKS_SOME || dl.fwd_limb[pro]) return rc;
    // after all column passes: few launches, each as large as possible
    LimbList li;
    for (int b = 0; b < l.size(); b++)
        if (l.mod[b] >= finish_from || (c->modc[l.mod[b]].qd == 0.0 && l.mod[b] < c->L)) li.add(l.slot[b], l.src[b], l.mod[b]);
    return for_batches(c, li, [&](const LimbBatch &lb, int nb) {
        dl.fwd_blocks(c, st, 2.0 * nb * N8, EPI_STORE, pro_pairs_rows(pro), data, lb, nb, kNoFin);
    });
}

// Inverse NTT: limb b read at src + l.src[b]*N, result at dst + l.slot[b]*N; scale folds a base
// conversion constant into the final 1/N.
// blocks_done: the block pass has already been applied (by the inner-product kernel), in place in dst.
// src2: the transform's input is the limb-wise product of src and src2.
static int32_t ntt_inverse(he_ctx *c, hipStream_t st, const u64 *src, u64 *dst, const LimbList &l, int scale,
                           const ConvArgs &cv, bool blocks_done = false, const u64 *src2 = nullptr)
{
    const double N8 = (double)c->N * 8.0;
    const DevLaunch &dl = dev_launch(c);
    return for_batches(c, l, [&](const LimbBatch &lb, int nb) {
        const double bytes = 2.0 * nb * N8;
        if (dl.inv_limb) {
            dl.inv_limb(c, st, src2 ? 1.5 * bytes : bytes, scale, src, src2, dst, lb, nb, cv);
            return;
        }
        if (!blocks_done) dl.inv_blocks(c, st, src2 ? 1.5 * bytes : bytes, src, src2, dst, lb, nb);
        dl.inv_cols(c, st, bytes, scale, dst, lb, nb, cv);
    });
}

static int32_t dev_guard(he_ctx *c)
{
    if (!c) return HE_EINVAL;
    if (c->device < 0) return HE_ENODEV;
    return HE_OK;
}

static int32_t ntt_api(he_ctx *ctx, uint64_t *d_limbs, const int32_t *h_mod_idx, int32_t batch, void *stream, bool inv)
{
    int32_t rc = dev_guard(ctx);
    if (rc != HE_OK) return rc;
    if (!d_limbs || !h_mod_idx || batch < 0) return HE_EINVAL;
    for (int b = 0; b < batch; b++)
        if (h_mod_idx[b] < 0 || h_mod_idx[b] >= ctx->M) return HE_EINVAL;
    const ConvArgs cv = conv_args(ctx, nullptr, 1);
    // limb slots are 16-bit: walk the buffer in windows
    const int WIN = 32768;
    for (int off = 0; off < batch; off += WIN) {
        const int nb = std::min(WIN, batch - off);
        LimbList l;
        for (int b = 0; b < nb; b++) l.add(b, h_mod_idx[off + b]);
        u64 *base = d_limbs + (size_t)off * ctx->N;
        rc = inv ? ntt_inverse(ctx, (hipStream_t)stream, base, base, l, SCALE_NONE, cv)
                 : ntt_forward(ctx, (hipStream_t)stream, base, l, PRO_LOAD, cv, nullptr, 0);
        if (rc != HE_OK) return rc;
    }
    return HE_OK;
}

extern "C" int32_t he_ntt(he_ctx *ctx, uint64_t *d_limbs, const int32_t *h_mod_idx, int32_t batch, void *stream)
{
    return ntt_api(ctx, d_limbs, h_mod_idx, batch, stream, false);
}
extern "C" int32_t he_intt(he_ctx *ctx, uint64_t *d_limbs, const int32_t *h_mod_idx, int32_t batch, void *stream)
{
    return ntt_api(ctx, d_limbs, h_mod_idx, batch, stream, true);
}

static int32_t level_guard(he_ctx *c, int level)
{
    int32_t rc = dev_guard(c);
    if (rc != HE_OK) return rc;
    if (level < 1 || level > c->L) return HE_ELEVEL;
    return HE_OK;
}

// a, b, out: [count] operations of `limbs` limbs each, strides sa / sb / so limbs between operations
static int32_t limbwise(he_ctx *c, const u64 *a, const u64 *b, u64 *out, int level, int op, int limbs, int b_limbs,
                        void *stream, int count = 1, int sa = 0, int sb = 0, int so = 0)
{
    int32_t rc = level_guard(c, level);
    if (rc != HE_OK) return rc;
    if (!a || !b || !out || count < 1 || limbs > 65535 || count > 65535) return HE_EINVAL;
    dim3 grid((unsigned)(c->N / 256), (unsigned)limbs, (unsigned)count);
    KLAUNCH(c, (hipStream_t)stream, KID_LIMBWISE, (double)count * (2 * limbs + b_limbs) * c->N * 8.0, (k_limbwise), grid, a,
            b, out, c->dev, op, level, b_limbs, c->logN, sa, sb, so);
    return launch_ok(c);
}

static bool count_ok(int level, int count) { return count >= 1 && (long)count * 2 * level <= 65535; }

extern "C" int32_t he_add_batch(he_ctx *ctx, const uint64_t *d_a, const uint64_t *d_b, uint64_t *d_out, int32_t level,
                                int32_t count, void *stream)
{
    if (!count_ok(level, count)) return HE_EINVAL;
    return limbwise(ctx, d_a, d_b, d_out, level, 0, count * 2 * level, count * 2 * level, stream);
}
extern "C" int32_t he_sub_batch(he_ctx *ctx, const uint64_t *d_a, const uint64_t *d_b, uint64_t *d_out, int32_t level,
                                int32_t count, void *stream)
{
    if (!count_ok(level, count)) return HE_EINVAL;
    return limbwise(ctx, d_a, d_b, d_out, level, 1, count * 2 * level, count * 2 * level, stream);
}
extern "C" int32_t he_pmult_batch(he_ctx *ctx, const uint64_t *d_ct, const uint64_t *d_pt, uint64_t *d_out,
                                  int32_t level, int32_t count, void *stream)
{
    if (!count_ok(level, count)) return HE_EINVAL;
    return limbwise(ctx, d_ct, d_pt, d_out, level, 2, count * 2 * level, level, stream);
}
extern "C" int32_t he_add(he_ctx *ctx, const uint64_t *d_a, const uint64_t *d_b, uint64_t *d_out, int32_t level,
                          void *stream)
{
    return he_add_batch(ctx, d_a, d_b, d_out, level, 1, stream);
}
extern "C" int32_t he_sub(he_ctx *ctx, const uint64_t *d_a, const uint64_t *d_b, uint64_t *d_out, int32_t level,
                          void *stream)
{
    return he_sub_batch(ctx, d_a, d_b, d_out, level, 1, stream);
}
extern "C" int32_t he_pmult(he_ctx *ctx, const uint64_t *d_ct, const uint64_t *d_pt, uint64_t *d_out, int32_t level,
                            void *stream)
{
    return he_pmult_batch(ctx, d_ct, d_pt, d_out, level, 1, stream);
}

extern "C" int32_t he_pmult_sum(he_ctx *ctx, const uint64_t *const *h_d_cts, const uint64_t *const *h_d_pts,
                                int32_t count, uint64_t *d_out, int32_t level, void *stream)
{
    int32_t rc = level_guard(ctx, level);
    if (rc != HE_OK) return rc;
    if (!h_d_cts || !h_d_pts || !d_out || count < 1 || count > PMULT_SUM_MAX) return HE_EINVAL;
    PmultSumArgs a;
    memset(&a, 0, sizeof(a));
    for (int k = 0; k < count; k++) {
        if (!h_d_cts[k] || !h_d_pts[k]) return HE_EINVAL;
        a.ct[k] = h_d_cts[k];
        a.pt[k] = h_d_pts[k];
    }
    a.count = count;
    dim3 grid((unsigned)(ctx->N / 256), (unsigned)(2 * level));
    KLAUNCH(ctx, (hipStream_t)stream, KID_LIMBWISE, (double)(3 * count + 2) * level * ctx->N * 8.0, (k_pmult_sum), grid, a,
            d_out, ctx->dev, level, ctx->logN);
    return launch_ok(ctx);
}

static int32_t scalar_args(he_ctx *ctx, const uint64_t *h_scalar, int level, bool with_companion, ScalarArgs &sc)
{
    memset(&sc, 0, sizeof(sc));
    for (int i = 0; i < level; i++) {
        if (h_scalar[i] >= ctx->mod[i]) return HE_EINVAL;
        if (with_companion)
            sc.s[i] = hostmath::shoup(h_scalar[i], ctx->mod[i]);
        else
            sc.s[i].w = h_scalar[i];
    }
    return HE_OK;
}

extern "C" int32_t he_cmult_batch(he_ctx *ctx, const uint64_t *d_ct, const uint64_t *h_scalar, uint64_t *d_out,
                                  int32_t level, int32_t count, void *stream)
{
    int32_t rc = level_guard(ctx, level);
    if (rc != HE_OK) return rc;
    if (!d_ct || !h_scalar || !d_out || !count_ok(level, count)) return HE_EINVAL;
    ScalarArgs sc;
    if ((rc = scalar_args(ctx, h_scalar, level, true, sc)) != HE_OK) return rc;
    dim3 grid((unsigned)(ctx->N / 256), (unsigned)(count * 2 * level));
    KLAUNCH(ctx, (hipStream_t)stream, KID_CMULT, 4.0 * count * level * ctx->N * 8.0, (k_cmult), grid, d_ct, d_out, ctx->dev,
            sc, level, ctx->logN);
    return launch_ok(ctx);
}
extern "C" int32_t he_cmult(he_ctx *ctx, const uint64_t *d_ct, const uint64_t *h_scalar, uint64_t *d_out, int32_t level,
                            void *stream)
{
    return he_cmult_batch(ctx, d_ct, h_scalar, d_out, level, 1, stream);
}

extern "C" int32_t he_add_const_batch(he_ctx *ctx, const uint64_t *d_ct, const uint64_t *h_scalar, uint64_t *d_out,
                                      int32_t level, int32_t count, void *stream)
{
    int32_t rc = level_guard(ctx, level);
    if (rc != HE_OK) return rc;
    if (!d_ct || !h_scalar || !d_out || !count_ok(level, count)) return HE_EINVAL;
    ScalarArgs sc;
    if ((rc = scalar_args(ctx, h_scalar, level, false, sc)) != HE_OK) return rc;
    dim3 grid((unsigned)(ctx->N / 256), (unsigned)(count * 2 * level));
    KLAUNCH(ctx, (hipStream_t)stream, KID_LIMBWISE, 4.0 * count * level * ctx->N * 8.0, (k_addconst), grid, d_ct, d_out,
            ctx->dev, sc, level, ctx->logN);
    return launch_ok(ctx);
}
extern "C" int32_t he_add_const(he_ctx *ctx, const uint64_t *d_ct, const uint64_t *h_scalar, uint64_t *d_out,
                                int32_t level, void *stream)
{
    return he_add_const_batch(ctx, d_ct, h_scalar, d_out, level, 1, stream);
}

// Rows of `width` limbs, src_stride and dst_stride limbs apart.  Launched by the kernel's handle: small copies take as long as their call, and by the
// kernel's name that is 0.3 us more (3.8 us of host time, 3.4 by the handle and for the runtime's two-dimensional copy).
static int32_t copy_limbs(he_ctx *c, const u64 *src, int src_stride, u64 *dst, int dst_stride, int width, int rows, hipStream_t st)
{
    const dim3 grid((unsigned)(c->N / 512), (unsigned)width, (unsigned)std::min(rows, 65535));
    if (!c->prof_on) {
        void *args[] = {&src, &dst, &src_stride, &dst_stride, &rows, &c->logN};
        HIP_TRY(c, hipModuleLaunchKernel((hipFunction_t)c->copy_kernel, grid.x, grid.y, grid.z, 256, 1, 1, 0, st, args, nullptr));
        return HE_OK;
    }
    KLAUNCH(c, st, KID_COPY, 2.0 * rows * width * c->N * 8.0, (k_copy_limbs), grid, src, dst, src_stride, dst_stride, rows, c->logN);
    return launch_ok(c);
}

extern "C" int32_t he_moddrop_batch(he_ctx *ctx, const uint64_t *d_ct, int32_t in_level, uint64_t *d_out,
                                    int32_t out_level, int32_t count, void *stream)
{
    int32_t rc = level_guard(ctx, in_level);
    if (rc != HE_OK) return rc;
    if (out_level < 1 || out_level > in_level) return HE_ELEVEL;
    if (!d_ct || !d_out || d_ct == d_out || count < 1) return HE_EINVAL;
    // one row per (operation, component): the first out_level limbs of in_level
    return copy_limbs(ctx, d_ct, in_level, d_out, out_level, out_level, count * 2, (hipStream_t)stream);
}
extern "C" int32_t he_moddrop(he_ctx *ctx, const uint64_t *d_ct, int32_t in_level, uint64_t *d_out, int32_t out_level,
                              void *stream)
{
    return he_moddrop_batch(ctx, d_ct, in_level, d_out, out_level, 1, stream);
}

// the key-switch kernels read and write 16-byte pairs
static inline bool misaligned16(const void *p) { return ((uintptr_t)p & 15u) != 0; }

// ---- workspace layout (in limbs of N words), per operation of a batch
struct WsLayout {
    size_t x, raised, u, r, tmp, total;
};
static WsLayout ws_layout(const he_ctx *c, int level)
{
    const size_t Ma = level + c->K, beta = (level + c->alpha - 1) / c->alpha;
    WsLayout w;
    size_t o = 0;
    w.x = o, o += std::max(level, 2); // y: inverse transform of the switched polynomial, scaled
    o += level;                       // spare: the size that callers have been told stays as it was
    w.raised = o, o += beta * Ma;     // raised digits (slots of a digit's own limbs stay unused)
    w.u = o, o += 2 * Ma;             // inner products
    w.r = o, o += 2 * level;          // ModDown / rescale corrections
    w.tmp = o, o += 2 * level;        // rotate_sum: the rotated ciphertext; Mult: a result that overlaps a factor
    w.total = o;
    return w;
}

extern "C" int32_t he_workspace_bytes(const he_ctx *ctx, int32_t level, int32_t count, size_t *out)
{
    if (!ctx || !out || count < 1) return HE_EINVAL;
    if (level < 1 || level > ctx->L) return HE_ELEVEL;
    *out = ws_layout(ctx, level).total * (size_t)count * ctx->N * sizeof(u64);
    return HE_OK;
}

// limb slots are 16-bit offsets from a buffer's base
static bool batch_fits(const WsLayout &w, int count) { return count >= 1 && w.total * (size_t)count <= 65535; }

// Whether the block pass of the raised limbs from active limb `first` on runs ahead of the first inner-product launch
// (k_inner_finished), rather than inside it (k_inner_special).  Digits that three or more rotations share: yes (N = 2^16, 15 rotations at
// level 24 983 us, not 1048, 4 at level 12 155, not 158).  Otherwise k_inner_special is the faster one as long as its launch leaves
// the chip part empty or more than half of its four waves have a digit in every round: 16 products with rescale at level 24 (six digits) take
// 1676 us, not 1693, 4 take 460, not 467.  It loses in launches of four and more work-groups per compute unit where half of the waves
// have none (one or two digits: 8 rotations at level 4 144 us, not 151, 8 products with rescale at level 6 253, not 260, 4 rotations at
// level 4 of N = 2^17 175, not 182).
// Special limbs on the floating-point path (none of 2^50 or above) are cheap to finish: k_inner_special (8 rotations 267 us, not 282).
static bool special_finished(const he_ctx *c, int level, int first, int count, bool shared)
{
    if (dev_launch(c).inner_limb) return false; // N = 2^12: every raised limb is finished
    if (shared) return count > 2;
    bool ints = false;
    for (int k = 0; k < c->K; k++) ints |= c->modc[c->L + k].qd == 0.0;
    const size_t groups = (size_t)(level + c->K - first) * count * (c->N >> FINISHED_TLOG);
    const int beta = (level + c->alpha - 1) / c->alpha, rounds = (beta + SPECIAL_WAVES - 1) / SPECIAL_WAVES, idle = rounds * SPECIAL_WAVES - beta;
    return ints && groups >= 1024 && idle * 2 >= rounds * SPECIAL_WAVES;
}
// the modulus index from which on ks_raise finishes raised limbs
static int finish_from(const he_ctx *c, int level, int first, bool finished) { return !finished ? c->M : first < level ? first : c->L; }

// What a launch of conversions has to do: units (a digit, or a component's special limbs), their source limbs and the limbs made of them, over
// operations that may be at levels of their own.
struct ConvWork {
    int units = 0, sources = 0, targets = 0;
};
enum ConvKind { CONV_UP, CONV_DOWN, CONV_DOWN_RS };
// Whether a conversion goes through the kernels with the inverse column pass ahead of it (kernels_conv.h) or through passes of their own.  A work-group
// of those kernels waits for the inverse pass of its sources, the waves that have none without work, so its unit has to have some targets to make:
// the more, the fewer sources each of them reads.  Where all work-groups are resident at once what counts is that there is one launch less.  With one
// work-group per compute unit, a last round that is nearly empty counts against it too.  Gain of the call as a whole, in per cent, N = 2^16 unless stated:
//   digits of one limb, 16 to 64 of them, 4 targets each: -5 to 0, 6: +1 to +2, 12: +6 to +11; of two, 4: -3 to +2, 6: +2 to +4; of three,
//   4: -1 to +4; of four, 4: 0 to +5, 24: +9 to +14; of five and more, 5: -2 to +1, 8: 0 to +5; N = 2^17, four limbs, 8: -3, 10: +1 to +2 (12 units),
//   -3 to -4 (6, a round and a half), 30: +5 to +8; two limbs, 8: -3 to -8, 12: -1 to +2
//   corrections of one special limb, 32 units, 6 targets: -3, 8: -1 to 0, 12: +1 to +2; of two, 4: -1, 8: +2; of three, 3: -1, 4: 0; of four,
//   2: +1, 24: +3; of five, 16 units, 8: -1, 10: +2, 32 units, 9: -3, 11: +2; N = 2^17, four, 8 units, 6: -1, 8: +2, 16 units, 12: 0, 16: 0;
//   two, 8 to 16 units, 8: -1 to -3, 12: -1
//   with a rescale, 32 units, 3 targets -1 to -2 (one to four special limbs), 5: 0, 7: +1 to +4; N = 2^17, 8 units, 5: -1 to +1, 7: +2 to +4.
//   Where digits or special primes are more than four, its pass apart is the one for eight sources: with one target +7, with more +20 to +85.
static bool conv_pays(const he_ctx *c, ConvKind kind, const ConvWork &w)
{
    const bool two = c->logN == 16 && (kind == CONV_UP ? c->alpha : c->K) <= 4; // work-groups per compute unit
    const int units = std::max(w.units, 1), groups = CONV_GROUPS * units;
    if (groups <= (two ? 512 : 256)) return true;
    if (kind == CONV_DOWN_RS && std::max(c->alpha, c->K) > 4) return true;
    const int s = (w.sources + units - 1) / units; // per unit
    const int up = c->logN == 17 ? 13 - s : two ? std::max(4, 7 - s) : 6;
    const int down = c->logN == 17 ? (s >= 3 && units < 16 ? 8 : 14) : two ? 10 - 2 * s : 12 + std::min(units, 32) / 8 - s;
    const int rs = c->logN == 17 ? 7 : 5;
    const int need = kind == CONV_UP ? up : kind == CONV_DOWN ? down : rs;
    const int rounds = two ? units : (groups + 255) / 256 * (256 / CONV_GROUPS); // in units: of whole rounds
    return w.targets >= need * rounds;
}
// ModUp so (k_ntt_fwd_cols_modup): N = 2^16 and 2^17, digits whose limbs are all on the floating-point path, without the correction of the
// overshoot.
static bool modup_fused(const he_ctx *c, const ConvWork &w) { return dev_launch(c).modup && !c->up_split && !c->exact_conv && conv_pays(c, CONV_UP, w); }
// The same for ModDown's corrections of both components of `count` operations, `limbs` of each component in all (k_ntt_fwd_cols_moddown): ciphertext limbs
// on the floating-point path.
static bool moddown_fused(const he_ctx *c, int limbs, int count, bool rs)
{
    ConvWork w;
    w.units = 2 * count, w.sources = w.units * c->K, w.targets = 2 * limbs;
    return dev_launch(c).moddown && !c->up_split && (!c->dn_split || c->dn_fold) && !c->exact_conv && conv_pays(c, rs ? CONV_DOWN_RS : CONV_DOWN, w);
}
// The targets of a digit are shared out among so many work-groups that a launch of few operations puts one on every compute unit, and no
// more, for each repeats the inverse column pass (N = 2^16: one rotation at level 13 93.5 us, with two on every unit 96.4; one product at level 6
// 103.5 and 104.9).
static int conv_chunks(int units, int targets) { return std::max(1, std::min(256 / (CONV_GROUPS * units), targets)); }

// Steps 1-2 of the key switch for `count` polynomials (d_ntt2: products of two): operation o reads its NTT-domain input at
// d_ntt + from(o) limbs and works in ws + o*w.total limbs, laid out for `level`; levels: null, or the operations' own.  Raised ciphertext
// limbs on the floating-point path and special ones are left as the column pass wrote them (the inner-product kernels finish
// them), but for those of modulus index finish_at and above.
template <class F>
static int32_t ks_raise(he_ctx *c, const u64 *d_ntt, F from, u64 *ws, const WsLayout &w, int level, const int32_t *levels, int count,
                        hipStream_t st, int finish_at, const u64 *d_ntt2 = nullptr)
{
    const size_t N = c->N;
    const int K = c->K, Ma = level + K, W = (int)w.total;
    const auto level_of = [&](int o) { return levels ? (int)levels[o] : level; };
    LimbList l;
    ConvWork cw;
    for (int o = 0; o < count; o++) {
        const int lo = level_of(o), beta = (lo + c->alpha - 1) / c->alpha;
        for (int i = 0; i < lo; i++) l.add(o * W + i, from(o) + i, i);
        cw.units += beta, cw.sources += lo, cw.targets += beta * (lo + K) - lo;
    }
    ConvArgs cv = conv_args(c, ws + w.x * N, level, W, W);
    for (int o = 0; levels && o < count; o++) cv.op_level[o] = (uint8_t)levels[o];
    const bool fused = modup_fused(c, cw);
    // limbs that go through a column pass or a block pass of their own; listed once the first launches are on their way
    LimbList r;
    const auto list_raised = [&] {
        const int from = fused ? finish_at : 0; // modulus index
        if (from < c->M) r.reserve(cw.targets);
        for (int o = 0; o < count; o++) {
            const int lo = level_of(o), beta = (lo + c->alpha - 1) / c->alpha;
            for (int j = 0; j < beta; j++) {
                const int dlo = j * c->alpha, dhi = std::min(dlo + c->alpha, lo), slot = o * W + j * Ma;
                for (int i = from; i < dlo; i++) r.add(slot + i, i);
                for (int i = std::max(from, dhi); i < lo; i++) r.add(slot + i, i);
                for (int k = std::max(from - c->L, 0); k < K; k++) r.add(slot + level + k, c->L + k);
            }
        }
    };
    int32_t rc;
    if (!fused) {
        if ((rc = ntt_inverse(c, st, d_ntt, ws + w.x * N, l, SCALE_MODUP, cv, false, d_ntt2)) != HE_OK) return rc;
        list_raised();
        return ntt_forward(c, st, ws + w.raised * N, r, PRO_MODUP, cv, nullptr, cw.sources, BLOCKS_SOME, finish_at);
    }
    const double N8 = (double)N * 8.0;
    const DevLaunch &dl = dev_launch(c);
    rc = for_batches(c, l, [&](const LimbBatch &lb, int nb) { dl.inv_blocks(c, st, (d_ntt2 ? 3.0 : 2.0) * nb * N8, d_ntt, d_ntt2, ws + w.x * N, lb, nb); });
    if (rc != HE_OK) return rc;
    ModUpArgs ua;
    ua.x = ws + w.x * N, ua.raised = ws + w.raised * N;
    ua.level = level, ua.L = c->L, ua.K = K, ua.alpha = c->alpha, ua.beta = (level + c->alpha - 1) / c->alpha, ua.stride = W;
    ua.chunks = conv_chunks(ua.beta * count, Ma - c->alpha);
    memcpy(ua.op_level, cv.op_level, sizeof(ua.op_level));
    dl.modup(c, st, (double)(cw.sources + cw.targets) * N8, count, ua);
    if ((rc = launch_ok(c)) != HE_OK) return rc;
    list_raised();
    return for_batches(c, r, [&](const LimbBatch &lb, int nb) { dl.fwd_blocks(c, st, 2.0 * nb * N8, EPI_STORE, true, ws + w.raised * N, lb, nb, kNoFin); });
}

// limb offset of operation o's input where inputs are `stride` limbs apart
static auto every(int stride)
{
    return [stride](int o) { return o * stride; };
}

static InnerArgs inner_args(const he_ctx *c, const he_evk *evk, const u64 *d_ntt, int d_stride, u64 *ws, const WsLayout &w,
                            int level, int count, const OpArgs *oa, bool shared_raised, bool finished)
{
    InnerArgs ia;
    ia.raised = ws + w.raised * c->N, ia.d = d_ntt, ia.evk = evk->dev, ia.u = ws + w.u * c->N;
    ia.level = level, ia.L = c->L, ia.K = c->K, ia.alpha = c->alpha, ia.first = level;
    ia.g = (unsigned)evk->galois;
    ia.raised_stride = shared_raised ? 0 : (int)w.total, ia.u_stride = (int)w.total, ia.d_stride = d_stride;
    ia.per_op = oa ? 1 : 0, ia.count = count, ia.finished = finished ? 1 : 0;
    ia.ta = ia.tb = nullptr, ia.t_stride = 0;
    return ia;
}
// Words per index that the inner product has to move on the active limbs [lo, hi), by the definition of the step and
// each operand once per launch: per operation its digits (once for all if they share them), and 2 key words per digit
// for each distinct key, up to the highest level it is used at.
static double inner_words(const he_ctx *c, const InnerArgs &ia, const OpArgs *oa, int lo, int hi)
{
    auto limbs = [&](int level) { // active limbs of an operation at `level` within [lo, hi)
        return std::max(0, std::min(hi, level) - lo) + std::max(0, hi - std::max(lo, ia.level));
    };
    double words = 0.0;
    std::vector<std::pair<const u64 *, int>> keys;
    for (int o = 0; o < ia.count; o++) {
        const int level = oa && oa->level[o] ? oa->level[o] : ia.level, beta = (level + c->alpha - 1) / c->alpha;
        const u64 *key = oa ? oa->evk[o] : ia.evk;
        if (o == 0 || ia.raised_stride != 0) words += (double)beta * limbs(level);
        auto k = std::find_if(keys.begin(), keys.end(), [&](const std::pair<const u64 *, int> &e) { return e.first == key; });
        if (k == keys.end())
            keys.push_back({key, level});
        else
            k->second = std::max(k->second, level);
    }
    for (const auto &k : keys) words += 2.0 * ((k.second + c->alpha - 1) / c->alpha) * limbs(k.second);
    return words;
}

// Steps 3 and 4: the scaled coefficient-domain digits of the special limbs, in u (cols false: what the inverse block pass leaves, for a kernel that
// makes them itself).  ia.first < level: also u on the limbs from there on.
static int32_t ks_special(he_ctx *c, const InnerArgs &ia, const OpArgs *oa, const WsLayout &w, bool cols, hipStream_t st)
{
    const size_t N = c->N;
    const int K = c->K, Ma = ia.level + K, W = (int)w.total;
    if (misaligned16(ia.raised) || misaligned16(ia.d) || misaligned16(ia.evk)) return HE_EINVAL; // entry points check first
    if (dev_launch(c).inner_limb) { // u on every limb
        dev_launch(c).inner_limb(c, st, (inner_words(c, ia, oa, 0, Ma) + 2.0 * ia.count * Ma) * N * 8.0, ia, oa ? *oa : kNoOps);
        return launch_ok(c);
    }
    const double bytes = (inner_words(c, ia, oa, ia.first, Ma) + 2.0 * ia.count * (Ma - ia.first)) * N * 8.0;
    const unsigned tile = ia.finished ? 1u << FINISHED_TLOG : SPECIAL_TILE;
    dev_launch(c).inner(c, st, bytes, inner_grid((unsigned)N / tile, (unsigned)(Ma - ia.first), (unsigned)ia.count), ia,
                        oa ? *oa : kNoOps);
    int32_t rc = launch_ok(c);
    if (rc != HE_OK || !cols) return rc;
    LimbList sp;
    for (int o = 0; o < ia.count; o++)
        for (int cc = 0; cc < 2; cc++)
            for (int k = 0; k < K; k++) sp.add(o * W + cc * Ma + ia.level + k, c->L + k);
    const ConvArgs cv = conv_args(c, ia.u, ia.level, W, W);
    return ntt_inverse(c, st, ia.u, ia.u, sp, SCALE_MODDOWN, cv, true);
}

// ModDown's corrections of the ciphertext limbs [first, first + limbs) into ws, step 5 with the inverse column pass of step 4.
static int32_t ks_corrections(he_ctx *c, const InnerArgs &ia, const OpArgs *oa, const WsLayout &w, u64 *ws, int first, int limbs, bool rs, bool keep,
                              hipStream_t st)
{
    ModDownArgs da;
    da.u = ia.u, da.r = ws + w.r * c->N;
    da.level = ia.level, da.L = c->L, da.K = c->K, da.stride = (int)w.total;
    da.first = first, da.limbs = limbs, da.keep = keep ? 1 : 0;
    da.chunks = conv_chunks(2 * ia.count, limbs);
    memset(da.op_level, 0, sizeof(da.op_level));
    double moved = (2.0 * c->K + (rs ? 2.0 : keep ? 2.0 * c->K : 0.0)) * ia.count;
    for (int o = 0; o < ia.count; o++) {
        const int level = oa && oa->level[o] ? oa->level[o] : ia.level;
        if (oa) da.op_level[o] = oa->level[o];
        moved += 2.0 * std::max(0, std::min(first + limbs, level) - first);
    }
    dev_launch(c).moddown(c, st, moved * c->N * 8.0, rs, ia.count, da);
    return launch_ok(c);
}

// Steps 5 and 6 on the first fa.nl limbs of every operation (those that it has): pro is the prologue of the
// corrections' column pass, `extra` the source limbs it reads besides the special ones; fused: k_ntt_fwd_cols_moddown makes them.
static int32_t ks_finish(he_ctx *c, const InnerArgs &ia, const OpArgs *oa, const WsLayout &w, u64 *ws, FinishArgs fa, int mode, int pro,
                         const ConvArgs &cv, int extra, bool fused, hipStream_t st)
{
    const size_t N = c->N;
    const int W = (int)w.total;
    u64 *r = ws + w.r * N;
    LimbList l;
    double words = inner_words(c, ia, oa, 0, fa.nl);
    for (int o = 0; o < ia.count; o++) {
        const int limbs = std::min(oa && oa->level[o] ? oa->level[o] : ia.level, fa.nl);
        for (int cc = 0; cc < 2; cc++)
            for (int i = 0; i < limbs; i++) l.add(o * W + cc * ia.level + i, i);
        words += limbs * (4.0 + (mode == FIN_ROT ? 1.0 : 3.0)); // r, results, addends (FIN_MULT: four inputs in place of d)
    }
    fa.r = r, fa.r_stride = W;
    if (dev_launch(c).fin_limb) { // reads u and the special limbs in place of digits, keys and r
        words += 2.0 * c->K * ia.count + extra - l.size() - inner_words(c, ia, oa, 0, fa.nl);
        dev_launch(c).fin_limb(c, st, words * N * 8.0, std::max(c->alpha, c->K) > 4, pro, false, mode, ia, fa, oa ? *oa : kNoOps, cv);
        return launch_ok(c);
    }
    int32_t rc = fused ? ks_corrections(c, ia, oa, w, ws, 0, fa.nl, pro == PRO_MODDOWN_RS, false, st)
                                  : ntt_forward(c, st, r, l, pro, cv, nullptr, 2 * c->K * ia.count + extra, BLOCKS_NONE);
    if (rc != HE_OK) return rc;
    const unsigned grid = inner_grid((unsigned)(N / INNER_TILE), (unsigned)fa.nl, (unsigned)ia.count);
    int n_int = 0;
    for (int i = 0; i < fa.nl; i++) n_int += c->modc[i].qd == 0.0 ? 1 : 0;
    dev_launch(c).inner_fin(c, st, words * N * 8.0, grid, mode, n_int == 0 ? FIN_FP : n_int == fa.nl ? FIN_INT : FIN_BOTH, ia, fa, oa ? *oa : kNoOps);
    return launch_ok(c);
}

static FinishArgs finish_args(const he_ctx *c, u64 *out, int out_stride, const u64 *add, int add_stride, int add_cstride, int level)
{
    FinishArgs fa;
    fa.r = nullptr, fa.out = out, fa.add = add;
    fa.cst = c->dev.dn_pinv, fa.cst_d = c->dev.dn_pinv_d;
    fa.nl = level, fa.r_stride = 0, fa.out_stride = out_stride, fa.out_cstride = level;
    fa.add_stride = add_stride, fa.add_cstride = add_cstride;
    return fa;
}

// Steps 3-6 of one or more key switches that keep their level.
static int32_t ks_apply(he_ctx *c, const InnerArgs &ia, const OpArgs *oa, u64 *ws, const WsLayout &w, const FinishArgs &fa, int mode,
                        hipStream_t st)
{
    const int W = (int)w.total;
    int limbs = 0;
    for (int o = 0; o < ia.count; o++) limbs += std::min(oa && oa->level[o] ? (int)oa->level[o] : ia.level, fa.nl);
    const bool fused = moddown_fused(c, limbs, ia.count, false);
    int32_t rc = ks_special(c, ia, oa, w, !fused, st);
    if (rc != HE_OK) return rc;
    const ConvArgs cv = conv_args(c, ws + w.u * c->N, ia.level, W, W);
    return ks_finish(c, ia, oa, w, ws, fa, mode, PRO_MODDOWN, cv, 0, fused, st);
}

static int32_t ks_guard(he_ctx *c, const he_evk *evk, int level, int count, void *ws, size_t ws_bytes)
{
    int32_t rc = level_guard(c, level);
    if (rc != HE_OK) return rc;
    if (!evk || evk->ctx != c || !evk->dev) return HE_ENOKEY;
    if (!ws || misaligned16(ws) || misaligned16(evk->dev)) return HE_EINVAL;
    const WsLayout w = ws_layout(c, level);
    if (!batch_fits(w, count)) return HE_EINVAL;
    if (ws_bytes < w.total * (size_t)count * c->N * sizeof(u64)) return HE_EWORKSPACE;
    return HE_OK;
}

// Where a Mult writes its result: d_out itself, or the workspace, to be copied, where d_out overlaps a factor that
// work-groups of the same launch still read (where a limb is one work-group's, the launch that writes reads no factor).  A
// result that replaces a whole factor, limb for limb, needs no copy: the thread that writes a position has read it.
struct MultOut {
    u64 *out;
    int stride; // limbs between two operations
    bool copy;
};
static MultOut mult_out(const he_ctx *c, const u64 *a, const u64 *b, u64 *out, u64 *tmp, int W, int in_limbs, int out_limbs, int count)
{
    if (dev_launch(c).fin_limb) return {out, out_limbs, false};
    const size_t limb = c->N * sizeof(u64);
    const auto clash = [&](const u64 *x) {
        const uintptr_t x0 = (uintptr_t)x, x1 = x0 + (size_t)count * in_limbs * limb;
        const uintptr_t o0 = (uintptr_t)out, o1 = o0 + (size_t)count * out_limbs * limb;
        return x0 < o1 && o0 < x1 && !(x == out && in_limbs == out_limbs);
    };
    if (clash(a) || clash(b)) return {tmp, W, true};
    return {out, out_limbs, false};
}
static int32_t mult_copy(he_ctx *c, const MultOut &mo, u64 *out, int out_limbs, int count, hipStream_t st)
{
    if (!mo.copy) return HE_OK;
    return copy_limbs(c, mo.out, mo.stride, out, out_limbs, out_limbs, count, st);
}
static InnerArgs mult_args(const he_ctx *c, const he_evk *relin, const u64 *a, const u64 *b, u64 *ws, const WsLayout &w, int level, int count,
                           bool finished)
{
    InnerArgs ia = inner_args(c, relin, a, 0, ws, w, level, count, nullptr, false, finished);
    ia.ta = a, ia.tb = b, ia.t_stride = 2 * level;
    return ia;
}

extern "C" int32_t he_hmult_relin_batch(he_ctx *ctx, const he_evk *relin, const uint64_t *d_a, const uint64_t *d_b,
                                        uint64_t *d_out, int32_t level, int32_t count, void *d_ws, size_t ws_bytes,
                                        void *stream)
{
    int32_t rc = ks_guard(ctx, relin, level, count, d_ws, ws_bytes);
    if (rc != HE_OK) return rc;
    if (relin->galois != 1) return HE_ENOKEY;
    if (!d_a || !d_b || !d_out || misaligned16(d_a) || misaligned16(d_b) || misaligned16(d_out)) return HE_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const WsLayout w = ws_layout(ctx, level);
    const size_t N = ctx->N;
    const MultOut mo = mult_out(ctx, d_a, d_b, d_out, ws + w.tmp * N, (int)w.total, 2 * level, 2 * level, count);
    const bool finished = special_finished(ctx, level, level, count, false);
    if ((rc = ks_raise(ctx, d_a + (size_t)level * N, every(2 * level), ws, w, level, nullptr, count, st, finish_from(ctx, level, level, finished),
                       d_b + (size_t)level * N)) != HE_OK)
        return rc;
    if ((rc = ks_apply(ctx, mult_args(ctx, relin, d_a, d_b, ws, w, level, count, finished), nullptr, ws, w,
                       finish_args(ctx, mo.out, mo.stride, nullptr, 0, 0, level), FIN_MULT, st)) != HE_OK)
        return rc;
    return mult_copy(ctx, mo, d_out, 2 * level, count, st);
}

extern "C" int32_t he_hmult_relin(he_ctx *ctx, const he_evk *relin, const uint64_t *d_a, const uint64_t *d_b,
                                  uint64_t *d_out, int32_t level, void *d_ws, size_t ws_bytes, void *stream)
{
    return he_hmult_relin_batch(ctx, relin, d_a, d_b, d_out, level, 1, d_ws, ws_bytes, stream);
}

// Mult followed by rescale with one forward transform per output limb.  The inner product gives u + P d (d: the
// limb of d0 or d1).  After it: ModDown of the last limb alone (c_last = (u + P d - ntt(r)) P^-1), its inverse transform t,
// then for every other limb the column pass transforms r + P t_centred and the block pass finishes
// (u + P d - ntt) (P q_l)^-1.
extern "C" int32_t he_hmult_relin_rescale_batch(he_ctx *ctx, const he_evk *relin, const uint64_t *d_a,
                                                const uint64_t *d_b, uint64_t *d_out, int32_t level, int32_t count,
                                                void *d_ws, size_t ws_bytes, void *stream)
{
    int32_t rc = ks_guard(ctx, relin, level, count, d_ws, ws_bytes);
    if (rc != HE_OK) return rc;
    if (relin->galois != 1) return HE_ENOKEY;
    if (level < 2) return HE_ELEVEL;
    if (!d_a || !d_b || !d_out || misaligned16(d_a) || misaligned16(d_b) || misaligned16(d_out)) return HE_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const WsLayout w = ws_layout(ctx, level);
    const size_t N = ctx->N;
    const int W = (int)w.total, K = ctx->K, Ma = level + K, L = ctx->L;
    const MultOut mo = mult_out(ctx, d_a, d_b, d_out, ws + w.tmp * N, W, 2 * level, 2 * (level - 1), count);
    const int first = level - 1; // the dropped limb goes with the special ones
    const bool finished = special_finished(ctx, level, first, count, false);
    if ((rc = ks_raise(ctx, d_a + (size_t)level * N, every(2 * level), ws, w, level, nullptr, count, st, finish_from(ctx, level, first, finished),
                       d_b + (size_t)level * N)) != HE_OK)
        return rc;
    InnerArgs ia = mult_args(ctx, relin, d_a, d_b, ws, w, level, count, finished);
    ia.first = first;
    const bool fused_drop = moddown_fused(ctx, count, count, false), fused = moddown_fused(ctx, (level - 1) * count, count, true);
    if ((rc = ks_special(ctx, ia, nullptr, w, !fused_drop, st)) != HE_OK) return rc;
    u64 *rbuf = ws + w.r * N;
    ConvArgs cv = conv_args(ctx, ws + w.u * N, level, W, W);
    cv.src2 = rbuf;
    cv.src2_stride = W;
    // ModDown of the last limb of both components, in place in the correction buffer, and its inverse transform
    FinishArgs fa = finish_args(ctx, mo.out, mo.stride, nullptr, 0, 0, level);
    fa.r = rbuf, fa.r_stride = W;
    if (dev_launch(ctx).fin_limb) {
        const double bytes = (2.0 * K + 6.0) * count * N * 8.0;
        dev_launch(ctx).fin_limb(ctx, st, bytes, std::max(ctx->alpha, K) > 4, PRO_MODDOWN, true, FIN_MULT, ia, fa, kNoOps, cv);
        if ((rc = launch_ok(ctx)) != HE_OK) return rc;
    } else {
        LimbList last;
        for (int o = 0; o < count; o++)
            for (int cc = 0; cc < 2; cc++) last.add(o * W + cc * level + level - 1, level - 1);
        const FinArgs fl = {ws + w.u * N, rbuf, ctx->dev.dn_pinv, ctx->dev.dn_pinv_d, Ma, level, level, W, W, W};
        if (fused_drop) {
            if ((rc = ks_corrections(ctx, ia, nullptr, w, ws, first, 1, false, true, st)) != HE_OK) return rc;
        } else if ((rc = ntt_forward(ctx, st, rbuf, last, PRO_MODDOWN, cv, nullptr, 2 * K * count, BLOCKS_NONE)) != HE_OK)
            return rc;
        const double N8 = (double)N * 8.0;
        const DevLaunch &dl = dev_launch(ctx);
        rc = for_batches(ctx, last, [&](const LimbBatch &lb, int nb) {
            dl.fwd_blocks(ctx, st, 3.0 * nb * N8, EPI_FIN_INV, true, rbuf, lb, nb, fl);
            if (!fused) dl.inv_cols(ctx, st, 2.0 * nb * N8, SCALE_NONE, rbuf, lb, nb, cv); // else part of the last conversion
        });
        if (rc != HE_OK) return rc;
    }
    // every other limb: ModDown and rescale corrections in one transform
    fa.nl = fa.out_cstride = level - 1;
    fa.cst = ctx->dev.rsp_inv + (size_t)(level - 1) * L, fa.cst_d = ctx->dev.rsp_inv_d + (size_t)(level - 1) * L;
    if ((rc = ks_finish(ctx, ia, nullptr, w, ws, fa, FIN_MULT, PRO_MODDOWN_RS, cv, 2 * count, fused, st)) != HE_OK) return rc;
    return mult_copy(ctx, mo, d_out, 2 * (level - 1), count, st);
}

extern "C" int32_t he_hmult_relin_rescale(he_ctx *ctx, const he_evk *relin, const uint64_t *d_a, const uint64_t *d_b,
                                          uint64_t *d_out, int32_t level, void *d_ws, size_t ws_bytes, void *stream)
{
    return he_hmult_relin_rescale_batch(ctx, relin, d_a, d_b, d_out, level, 1, d_ws, ws_bytes, stream);
}

extern "C" int32_t he_hrot_many(he_ctx *ctx, const he_evk *const *rots, int32_t count, const uint64_t *d_ct,
                                uint64_t *const *h_d_outs, int32_t level, void *d_ws, size_t ws_bytes, void *stream)
{
    if (!rots || count < 1 || !h_d_outs) return HE_EINVAL;
    int32_t rc;
    for (int r = 0; r < count; r++) {
        if ((rc = ks_guard(ctx, rots[r], level, 1, d_ws, ws_bytes)) != HE_OK) return rc;
        if (rots[r]->galois == 1) return HE_ENOKEY;
        if (!h_d_outs[r] || h_d_outs[r] == d_ct || misaligned16(h_d_outs[r])) return HE_EINVAL;
    }
    if (!d_ct || misaligned16(d_ct)) return HE_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const WsLayout w = ws_layout(ctx, level);
    const u64 *c1 = d_ct + (size_t)level * ctx->N;
    const bool finished = special_finished(ctx, level, level, count, true);
    if ((rc = ks_raise(ctx, c1, every(0), ws, w, level, nullptr, 1, st, finish_from(ctx, level, level, finished))) != HE_OK) return rc;
    // With workspace for several operations the rotations share every launch: operation o keeps its inner
    // products and ModDown corrections in workspace o, all read the raised digits of workspace 0.
    int fit = (int)std::min<size_t>(ws_bytes / (w.total * ctx->N * sizeof(u64)), HE_OPS_MAX);
    while (fit > 1 && !batch_fits(w, fit)) fit--;
    for (int r = 0; r < count;) {
        const int nb = std::min(fit, count - r);
        OpArgs oa = {};
        for (int o = 0; o < nb; o++) {
            oa.evk[o] = rots[r + o]->dev, oa.g[o] = (unsigned)rots[r + o]->galois;
            oa.d[o] = c1, oa.add[o] = d_ct, oa.out[o] = h_d_outs[r + o];
        }
        if ((rc = ks_apply(ctx, inner_args(ctx, rots[r], c1, 0, ws, w, level, nb, &oa, true, finished), &oa, ws, w,
                           finish_args(ctx, nullptr, 0, d_ct, 0, level, level), FIN_ROT, st)) != HE_OK)
            return rc;
        r += nb;
    }
    return HE_OK;
}

// in: operation o at d_ct + o*in_stride limbs; out: operation o at d_out + o*out_stride limbs.
// plus_input: the result is ct + Rotate(ct) instead of Rotate(ct).
static int32_t hrot_batch_to(he_ctx *ctx, const he_evk *rot, const u64 *d_ct, int in_stride, u64 *d_out, int out_stride,
                             int level, int count, void *d_ws, size_t ws_bytes, hipStream_t st, bool plus_input = false)
{
    int32_t rc = ks_guard(ctx, rot, level, count, d_ws, ws_bytes);
    if (rc != HE_OK) return rc;
    if (rot->galois == 1) return HE_ENOKEY;
    if (!d_ct || !d_out || d_ct == d_out || misaligned16(d_ct) || misaligned16(d_out)) return HE_EINVAL;
    u64 *ws = (u64 *)d_ws;
    const WsLayout w = ws_layout(ctx, level);
    const u64 *c1 = d_ct + (size_t)level * ctx->N;
    const bool finished = special_finished(ctx, level, level, count, false);
    if ((rc = ks_raise(ctx, c1, every(in_stride), ws, w, level, nullptr, count, st, finish_from(ctx, level, level, finished))) != HE_OK) return rc;
    return ks_apply(ctx, inner_args(ctx, rot, c1, in_stride, ws, w, level, count, nullptr, false, finished), nullptr, ws, w,
                    finish_args(ctx, d_out, out_stride, d_ct, in_stride, level, level), plus_input ? FIN_ROTSUM : FIN_ROT, st);
}

extern "C" int32_t he_hrot_batch(he_ctx *ctx, const he_evk *rot, const uint64_t *d_ct, uint64_t *d_out, int32_t level,
                                 int32_t count, void *d_ws, size_t ws_bytes, void *stream)
{
    return hrot_batch_to(ctx, rot, d_ct, 2 * level, d_out, 2 * level, level, count, d_ws, ws_bytes, (hipStream_t)stream);
}

extern "C" int32_t he_hrot(he_ctx *ctx, const he_evk *rot, const uint64_t *d_ct, uint64_t *d_out, int32_t level,
                           void *d_ws, size_t ws_bytes, void *stream)
{
    return he_hrot_batch(ctx, rot, d_ct, d_out, level, 1, d_ws, ws_bytes, stream);
}

// he_hrot on the library's own scratch array: no workspace argument, no allocation.
extern "C" int32_t he_hrot_noalloc(he_ctx *ctx, const he_evk *rot, const uint64_t *d_ct, uint64_t *d_out, int32_t level,
                                   void *stream)
{
    int32_t rc = level_guard(ctx, level);
    if (rc != HE_OK) return rc;
    if (!ctx->static_scratch) return HE_EHIP;
    if (ws_layout(ctx, level).total * ctx->N * sizeof(u64) > HE_STATIC_SCRATCH_BYTES) return HE_ESCRATCH;
    return hrot_batch_to(ctx, rot, d_ct, 2 * level, d_out, 2 * level, level, 1, ctx->static_scratch, HE_STATIC_SCRATCH_BYTES,
                         (hipStream_t)stream);
}

extern "C" int32_t he_hrot_batch_keys(he_ctx *ctx, const he_evk *const *rots, const uint64_t *d_ct, uint64_t *d_out,
                                      int32_t level, int32_t count, void *d_ws, size_t ws_bytes, void *stream)
{
    if (!rots || count < 1) return HE_EINVAL;
    int32_t rc;
    for (int r = 0; r < count; r++) {
        if ((rc = ks_guard(ctx, rots[r], level, 1, d_ws, ws_bytes)) != HE_OK) return rc;
        if (rots[r]->galois == 1) return HE_ENOKEY;
    }
    if (!d_ct || !d_out || d_ct == d_out || misaligned16(d_ct) || misaligned16(d_out)) return HE_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const WsLayout w = ws_layout(ctx, level);
    const size_t N = ctx->N;
    const int ct_limbs = 2 * level;
    int fit = (int)std::min<size_t>(ws_bytes / (w.total * N * sizeof(u64)), HE_OPS_MAX);
    while (fit > 1 && !batch_fits(w, fit)) fit--;
    for (int r = 0; r < count;) {
        const int nb = std::min(fit, count - r);
        const u64 *in = d_ct + (size_t)r * ct_limbs * N, *c1 = in + (size_t)level * N;
        const bool finished = special_finished(ctx, level, level, nb, false);
        if ((rc = ks_raise(ctx, c1, every(ct_limbs), ws, w, level, nullptr, nb, st, finish_from(ctx, level, level, finished))) != HE_OK) return rc;
        OpArgs oa = {};
        for (int o = 0; o < nb; o++) {
            oa.evk[o] = rots[r + o]->dev, oa.g[o] = (unsigned)rots[r + o]->galois;
            oa.out[o] = d_out + (size_t)(r + o) * ct_limbs * N;
        }
        if ((rc = ks_apply(ctx, inner_args(ctx, rots[r], c1, ct_limbs, ws, w, level, nb, &oa, false, finished), &oa, ws, w,
                           finish_args(ctx, nullptr, 0, in, ct_limbs, level, level), FIN_ROT, st)) != HE_OK)
            return rc;
        r += nb;
    }
    return HE_OK;
}

// Rotations at mixed levels in shared launches.  The buffers of every operation are laid out for the largest
// level of its group (workspace stride, limbs per raised digit and per component), an operation below that
// level simply has no limbs between its own level and the layout's, and fewer digits.
extern "C" int32_t he_hrot_batch_levels(he_ctx *ctx, const he_evk *const *rots, const int32_t *h_levels, const uint64_t *d_ct,
                                        uint64_t *d_out, int32_t count, void *d_ws, size_t ws_bytes, void *stream)
{
    if (!rots || !h_levels || count < 1) return HE_EINVAL;
    int32_t rc;
    int lmax_all = 0;
    for (int r = 0; r < count; r++) {
        if ((rc = level_guard(ctx, h_levels[r])) != HE_OK) return rc;
        lmax_all = std::max(lmax_all, (int)h_levels[r]);
    }
    for (int r = 0; r < count; r++) {
        if ((rc = ks_guard(ctx, rots[r], lmax_all, 1, d_ws, ws_bytes)) != HE_OK) return rc;
        if (rots[r]->galois == 1) return HE_ENOKEY;
    }
    if (!d_ct || !d_out || d_ct == d_out || misaligned16(d_ct) || misaligned16(d_out)) return HE_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const size_t N = ctx->N;
    size_t done_limbs = 0; // limbs of the operations already processed (inputs and outputs are packed alike)
    for (int r = 0; r < count;) {
        // group: as many operations as the workspace holds at the layout of their largest level
        int nb = 0, lmax = 0;
        while (r + nb < count && nb < HE_OPS_MAX) {
            const int lm = std::max(lmax, (int)h_levels[r + nb]);
            const WsLayout wl = ws_layout(ctx, lm);
            if (!batch_fits(wl, nb + 1) || wl.total * (size_t)(nb + 1) * N * sizeof(u64) > ws_bytes) break;
            lmax = lm, nb++;
        }
        if (nb == 0) return HE_EWORKSPACE;
        const WsLayout w = ws_layout(ctx, lmax);
        const u64 *in0 = d_ct + done_limbs * N;
        u64 *out0 = d_out + done_limbs * N;
        std::vector<size_t> off(nb + 1, 0); // limb offset of operation o within the group
        for (int o = 0; o < nb; o++) off[o + 1] = off[o] + 2 * (size_t)h_levels[r + o];
        if (off[nb] > 65535) return HE_EINVAL;
        OpArgs oa = {};
        for (int o = 0; o < nb; o++) {
            const int lo = h_levels[r + o];
            oa.level[o] = (uint8_t)lo;
            oa.evk[o] = rots[r + o]->dev, oa.g[o] = (unsigned)rots[r + o]->galois;
            oa.d[o] = in0 + (off[o] + lo) * N; // c1
            oa.add[o] = in0 + off[o] * N;      // c0
            oa.out[o] = out0 + off[o] * N;
        }
        // 1 - 2
        const bool finished = special_finished(ctx, lmax, lmax, nb, false);
        if ((rc = ks_raise(ctx, in0, [&](int o) { return (int)off[o] + h_levels[r + o]; }, ws, w, lmax, h_levels + r, nb, st,
                           finish_from(ctx, lmax, lmax, finished))) != HE_OK)
            return rc;
        // 3 - 6
        if (misaligned16(ws)) return HE_EINVAL;
        if ((rc = ks_apply(ctx, inner_args(ctx, rots[r], in0, 0, ws, w, lmax, nb, &oa, false, finished), &oa, ws, w,
                           finish_args(ctx, nullptr, 0, in0, 0, lmax, lmax), FIN_ROT, st)) != HE_OK)
            return rc;
        done_limbs += off[nb];
        r += nb;
    }
    return HE_OK;
}

extern "C" int32_t he_rotate_sum_batch(he_ctx *ctx, const he_evk *const *rots, int32_t n_rot, uint64_t *d_ct,
                                       int32_t level, int32_t count, void *d_ws, size_t ws_bytes, void *stream)
{
    if (!rots || n_rot < 0) return HE_EINVAL;
    int32_t rc = level_guard(ctx, level);
    if (rc != HE_OK) return rc;
    if (!d_ws || !d_ct) return HE_EINVAL;
    const WsLayout w = ws_layout(ctx, level);
    if (!batch_fits(w, count)) return HE_EINVAL;
    if (ws_bytes < w.total * (size_t)count * ctx->N * sizeof(u64)) return HE_EWORKSPACE;
    if (misaligned16(d_ct)) return HE_EINVAL;
    for (int k = 0; k < n_rot; k++) { // every key is checked before the first launch
        if ((rc = ks_guard(ctx, rots[k], level, count, d_ws, ws_bytes)) != HE_OK) return rc;
        if (rots[k]->galois == 1) return HE_ENOKEY;
    }
    // ct + Rotate(ct) is written by the key switch itself, alternately into the workspace (operation o at
    // tmp + o*w.total limbs) and back into d_ct
    u64 *tmp = (u64 *)d_ws + w.tmp * ctx->N;
    const int W = (int)w.total;
    hipStream_t st = (hipStream_t)stream;
    bool in_tmp = false;
    for (int k = 0; k < n_rot; k++) {
        rc = in_tmp ? hrot_batch_to(ctx, rots[k], tmp, W, d_ct, 2 * level, level, count, d_ws, ws_bytes, st, true)
                    : hrot_batch_to(ctx, rots[k], d_ct, 2 * level, tmp, W, level, count, d_ws, ws_bytes, st, true);
        if (rc != HE_OK) return rc;
        in_tmp = !in_tmp;
    }
    return in_tmp ? copy_limbs(ctx, tmp, W, d_ct, 2 * level, 2 * level, count, st) : HE_OK;
}

extern "C" int32_t he_rotate_sum(he_ctx *ctx, const he_evk *const *rots, int32_t count, uint64_t *d_ct, int32_t level,
                                 void *d_ws, size_t ws_bytes, void *stream)
{
    return he_rotate_sum_batch(ctx, rots, count, d_ct, level, 1, d_ws, ws_bytes, stream);
}

extern "C" int32_t he_rescale_batch(he_ctx *ctx, const uint64_t *d_ct, uint64_t *d_out, int32_t level, int32_t count,
                                    void *d_ws, size_t ws_bytes, void *stream)
{
    int32_t rc = level_guard(ctx, level);
    if (rc != HE_OK) return rc;
    if (level < 2) return HE_ELEVEL;
    if (!d_ct || !d_out || !d_ws || d_ct == d_out) return HE_EINVAL;
    const WsLayout w = ws_layout(ctx, level);
    if (!batch_fits(w, count)) return HE_EINVAL;
    if (ws_bytes < w.total * (size_t)count * ctx->N * sizeof(u64)) return HE_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const size_t N = ctx->N;
    const int W = (int)w.total;
    u64 *t = ws + w.x * N; // per operation two limbs: the dropped limb of each component, coefficient domain
    u64 *r = ws + w.r * N; // per operation [2][level-1][N]
    LimbList last;
    for (int o = 0; o < count; o++)
        for (int c = 0; c < 2; c++) last.add(o * W + c, o * 2 * level + c * level + level - 1, level - 1);
    const ConvArgs cv = conv_args(ctx, t, level, W, W);
    if ((rc = ntt_inverse(ctx, st, d_ct, t, last, SCALE_NONE, cv)) != HE_OK) return rc;
    LimbList l;
    for (int o = 0; o < count; o++)
        for (int c = 0; c < 2; c++)
            for (int i = 0; i < level - 1; i++) l.add(o * W + c * (level - 1) + i, i);
    const FinArgs fa = {d_ct, d_out, ctx->dev.rs_inv + (size_t)(level - 1) * ctx->L, ctx->dev.rs_inv_d + (size_t)(level - 1) * ctx->L,
                        level, level - 1, level - 1, W, 2 * level, 2 * (level - 1)};
    return ntt_forward(ctx, st, r, l, PRO_RESCALE, cv, &fa, 2 * count);
}

// ModRaise, the first step of bootstrapping: the centred coefficients of a level-1 ciphertext reduced modulo
// every q_i, i < level_out.
extern "C" int32_t he_modraise(he_ctx *ctx, const uint64_t *d_ct, uint64_t *d_out, int32_t level_out, void *d_ws,
                               size_t ws_bytes, void *stream)
{
    int32_t rc = level_guard(ctx, level_out);
    if (rc != HE_OK) return rc;
    if (level_out < 2) return HE_ELEVEL;
    if (!d_ct || !d_out || !d_ws || d_ct == d_out) return HE_EINVAL;
    const WsLayout w = ws_layout(ctx, level_out);
    if (ws_bytes < w.total * ctx->N * sizeof(u64)) return HE_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    u64 *ws = (u64 *)d_ws;
    const size_t N = ctx->N;
    u64 *t = ws + w.x * N; // two limbs: the coefficient-domain components
    LimbList in;
    in.add(0, 0, 0);
    in.add(1, 1, 0);
    ConvArgs cv = conv_args(ctx, t, level_out, 1 << 30, 0);
    cv.rs_mod = 0;
    cv.rs_nl = level_out;
    if ((rc = ntt_inverse(ctx, st, d_ct, t, in, SCALE_NONE, cv)) != HE_OK) return rc;
    LimbList l;
    for (int c = 0; c < 2; c++)
        for (int i = 1; i < level_out; i++) l.add(c * level_out + i, i);
    if ((rc = ntt_forward(ctx, st, d_out, l, PRO_RESCALE, cv, nullptr, 2)) != HE_OK) return rc;
    // limb 0 of both components is the input itself
    return copy_limbs(ctx, d_ct, 1, d_out, level_out, 1, 2, st);
}

extern "C" int32_t he_rescale(he_ctx *ctx, const uint64_t *d_ct, uint64_t *d_out, int32_t level, void *d_ws,
                              size_t ws_bytes, void *stream)
{
    return he_rescale_batch(ctx, d_ct, d_out, level, 1, d_ws, ws_bytes, stream);
}
