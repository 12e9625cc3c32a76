// Full SFSeg operator (Eq. 7 with alpha > 0 and a unary map distinct from the
// pairwise feature): kernel instantiations and the C ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "../../include/stpi.h"
#include "chain.hpp"
#include "host_internal.hpp"
#include "sfseg.hpp"

namespace stpi {
namespace {

#define STPI_SFSEG_ENTRY(ST, RS, RT, TH, TW, NTHR, RY, QX) \
    {RS, RT, TH, TW, NTHR, 0, &launch_sfseg<ST, RS, RT, TH, TW, NTHR, RY, QX>, &sfseg_blocks_per_cu<ST, RS, RT, TH, TW, NTHR, RY, QX>}
// matrix-core spatial passes, slab margin RS (8 or 16)
#define STPI_SFSEG_MFMA(RS, RT, TH, TW, NTHR) \
    {RS, RT, TH, TW, NTHR, 1, &launch_sfseg_mfma<RT, TH, TW, NTHR, RS>, &sfseg_mfma_blocks_per_cu<RT, TH, TW, NTHR, RS>}

// Compiled (RS, RT) pairs: the smallest one covering the problem's radii is
// used, in its matrix-core form for the steps of an iteration where that pays
// (see sfseg_variant).
const SfsegVariant kSfsegF32[] = {
    STPI_SFSEG_ENTRY(float, 4, 2, 16, 64, 256, 8, 4),
    STPI_SFSEG_ENTRY(float, 8, 3, 16, 64, 256, 8, 4),
    STPI_SFSEG_ENTRY(float, 16, 5, 32, 64, 512, 8, 4),
    STPI_SFSEG_MFMA(8, 3, 32, 64, 512),
    STPI_SFSEG_MFMA(16, 5, 32, 64, 512),
};
const SfsegVariant kSfsegF64[] = {
    STPI_SFSEG_ENTRY(double, 4, 2, 16, 64, 256, 8, 4),
};

// chain: for the steps of an iteration. There the matrix-core form is taken
// beyond r = (8, 3), and at (8, 3) on volumes whose arithmetic and not their
// frame-by-frame latency counts. Chain step in us, vector / matrix cores, r =
// (15, 5): 8x64x112 58 / 45, 5x233x347 43 / 43, 32x240x432 126 / 84, 64x480x854 485
// / 347; r = (8, 3): 5x233x347 20 / 26, 16x240x432 36 / 41, 32x240x432 59 / 50,
// 64x480x854 280 / 247 (1.7 and 3.3 M voxels lie on either side); r = (4, 2), no
// matrix-core form: 64x480x854 220 against 237 with the one of (8, 3). A single
// step runs the vector form: there a value that is not finite reaches the
// outputs whose window holds it and no others, as its products with the zeros
// of a band would.
const SfsegVariant *sfseg_variant(const stpi_problem *p, bool chain) {
    const SfsegVariant *list = p->dtype == STPI_F64 ? kSfsegF64 : kSfsegF32;
    const int n = p->dtype == STPI_F64 ? (int)(sizeof(kSfsegF64) / sizeof(kSfsegF64[0]))
                                       : (int)(sizeof(kSfsegF32) / sizeof(kSfsegF32[0]));
    const SfsegVariant *v = nullptr;
    for (int i = 0; i < n && !v; ++i)
        if (list[i].RS >= p->r_s && list[i].RT >= p->r_t && !list[i].mfma) v = &list[i];
    if (!v || !chain) return v;
    const bool pays = v->RS > 8 || (int64_t)p->T * p->H * p->W >= (int64_t)5 << 19;
    for (int i = 0; i < n; ++i)
        if (list[i].mfma && list[i].RS == v->RS && list[i].RT == v->RT && pays) return &list[i];
    return v;
}

int sfseg_tiles(const SfsegVariant &v, const stpi_problem *p) {
    return ((p->W + v.TW - 1) / v.TW) * ((p->H + v.TH - 1) / v.TH);
}

// Frame segments per tile: enough work units to fill the resident slots when
// the frame has few tiles, each segment at least 4 r_t frames long, and further
// ones on idle CUs as the single-field step has them (split_short_tiles).
int sfseg_segments(const SfsegVariant &v, const stpi_problem *p) {
    const int tiles = sfseg_tiles(v, p);
    const int resident = device_cus() * v.blocks_per_cu();
    const int rt = std::max(v.RT, 1);
    int nseg = std::min(std::min(resident / std::max(tiles, 1), p->T / (4 * rt)), STPI_NSEG_MAX);
    if (nseg < 1) nseg = 1;
    return split_short_tiles(std::max(tiles, 1), p->T, v.RT, nseg);
}

// Workspace as the single-field chain's (WsLayout), without maxima: state
// slots, two sets of partial sums (the range check's partials share the first
// set's room), the ping-pong volume. One size for steps and iterations.
WsLayout sfseg_layout(const stpi_problem *p) {
    WsLayout L;
    const size_t elem = p->dtype == STPI_F64 ? 8 : 4;
    L.state_off = 0;
    L.partials_off = (FINAL_SLOT + 1) * STATE_SLOT;
    const int tiles = std::max(sfseg_tiles(*sfseg_variant(p, false), p), sfseg_tiles(*sfseg_variant(p, true), p));
    L.partials_cap = std::max((size_t)tiles * STPI_NSEG_MAX, (size_t)std::max(NORM_BLOCKS_HOST, 2 * SFSEG_RANGE_BLOCKS));
    L.wmax_off = L.partials_off;
    const size_t off = L.partials_off + 2 * L.partials_cap * 2 * sizeof(double);
    L.buf_off = (off + 255) & ~(size_t)255;
    L.total = L.buf_off + (((size_t)p->T * p->H * p->W * elem + 255) & ~(size_t)255);
    return L;
}

int sfseg_check(const stpi_problem *p, bool chain, const SfsegVariant **v) {
    int rc = validate_problem(p);
    if (rc) return rc;
    if (p->dtype != STPI_F32 && p->dtype != STPI_F64) return fail(STPI_EUNSUPPORTED, "sfseg: float or double only");
    *v = sfseg_variant(p, chain);
    if (!*v) return fail(STPI_EUNSUPPORTED, "sfseg: no compiled kernel for radii (%d, %d)", p->r_s, p->r_t);
    return STPI_OK;
}

void sfseg_fill(SfsegLaunch &L, const stpi_problem *p, const void *s, const void *f, double alpha) {
    std::memset(&L, 0, sizeof(L));
    L.s = s;
    L.f = f;
    L.ainv = 1.0 / alpha;
    L.T = p->T;
    L.H = p->H;
    L.W = p->W;
    make_taps(p, L.gs, L.gt);
}

// The chain's check from the range partials: flags |= FLAG_AFFINITY and done
// when some affinity of Eq. 2 can be negative (alpha (max f - min f)^2 > 1, a
// negative s, or a NaN).
__global__ __launch_bounds__(256) void sfseg_range_check_kernel(const double *partials, int n, double alpha, DevState *s) {
    __shared__ SfsegRange rw[256 / 64];
    SfsegRange r = SFSEG_RANGE_EMPTY;
    for (int b = threadIdx.x; b < n; b += 256)
        r.take(SfsegRange{partials[3 * b], partials[3 * b + 1], partials[3 * b + 2]});
    r.wave();
    if ((threadIdx.x & 63) == 0) rw[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < 256 / 64; ++w) r.take(rw[w]);
    const double d = r.fmx - r.fmn;
    const bool nan = r.fmn != r.fmn || r.fmx != r.fmx || r.smn != r.smn;
    if (nan || r.smn < 0.0 || alpha * d * d > 1.0) {
        s->flags |= FLAG_AFFINITY;
        s->done = 1;
    }
}

template <class ST>
hipError_t sfseg_range(size_t n, const void *s, const void *f, double *partials, double alpha, DevState *state,
                       hipStream_t st) {
    hipLaunchKernelGGL(sfseg_range_kernel<ST>, dim3(SFSEG_RANGE_BLOCKS), dim3(256), 0, st, n, (const ST *)s,
                       (const ST *)f, partials);
    hipLaunchKernelGGL(sfseg_range_check_kernel, dim3(1), dim3(256), 0, st, partials, SFSEG_RANGE_BLOCKS, alpha,
                       state);
    return hipGetLastError();
}

}  // namespace
}  // namespace stpi

using namespace stpi;

extern "C" {

int stpi_sfseg_unary(int64_t n, int dtype, const void *S, double p, void *s, void *stream) {
    clear_error();
    if (n < 1 || !S || !s) return fail(STPI_EINVAL, "sfseg_unary: empty volume or NULL buffer");
    if (!std::isfinite(p) || p < 0.0) return fail(STPI_EINVAL, "sfseg_unary: p must be finite and >= 0");
    hipStream_t st = (hipStream_t)stream;
    if (dtype == STPI_F32)
        hipLaunchKernelGGL(sfseg_unary_kernel<float>, dim3(1024), dim3(256), 0, st, (size_t)n, (const float *)S, p,
                           (float *)s);
    else if (dtype == STPI_F64)
        hipLaunchKernelGGL(sfseg_unary_kernel<double>, dim3(1024), dim3(256), 0, st, (size_t)n, (const double *)S,
                           p, (double *)s);
    else
        return fail(STPI_EUNSUPPORTED, "sfseg_unary: float or double only");
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? STPI_OK : hip_fail(e, "sfseg_unary launch");
}

size_t stpi_sfseg_workspace_bytes(const stpi_problem *p) {
    const SfsegVariant *v = nullptr;
    if (sfseg_check(p, false, &v) != STPI_OK) return 0;
    return sfseg_layout(p).total;
}

int stpi_sfseg_step(const stpi_problem *p, const void *s, const void *f, double alpha, const void *x,
                    double x_scale, void *z, double *d_sums, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    const SfsegVariant *v = nullptr;
    int rc = sfseg_check(p, false, &v);
    if (rc) return rc;
    if (!s || !f || !x || !z || !d_sums) return fail(STPI_EINVAL, "NULL buffer");
    if (z == s || z == f || z == x) return fail(STPI_EINVAL, "z must not alias s, f or x");
    if (!(alpha > 0.0) || !std::isfinite(alpha)) return fail(STPI_EINVAL, "alpha must be finite and > 0");
    if (!std::isfinite(x_scale)) return fail(STPI_EINVAL, "x_scale must be finite");
    const WsLayout L = sfseg_layout(p);
    if (!ws || ws_bytes < L.total) return fail(STPI_EWORKSPACE, "sfseg workspace needs %zu bytes", L.total);
    hipStream_t st = (hipStream_t)stream;
    SfsegLaunch SL;
    sfseg_fill(SL, p, s, f, alpha);
    SL.buf0 = const_cast<void *>(x);
    SL.buf1 = z;
    SL.x_scale = x_scale;
    SL.partials = (double *)((char *)ws + L.partials_off);
    SL.nseg = sfseg_segments(*v, p);
    hipError_t e = v->launch(SL, st);
    if (e != hipSuccess) return hip_fail(e, "sfseg step launch");
    e = launch_step_sums(SL.partials, sfseg_tiles(*v, p) * SL.nseg, x_scale, d_sums, st);
    return e == hipSuccess ? STPI_OK : hip_fail(e, "step sums launch");
}

int stpi_sfseg_iterate(const stpi_problem *p, const void *s, const void *f, double alpha, void *x, int init,
                       int max_iters, double tol, void *ws, size_t ws_bytes, stpi_result *out, void *stream) {
    clear_error();
    const SfsegVariant *v = nullptr;
    int rc = sfseg_check(p, true, &v);
    if (rc) return rc;
    if (!s || !f || !x || !out) return fail(STPI_EINVAL, "NULL buffer or result");
    if (x == s || x == f) return fail(STPI_EINVAL, "x must not alias s or f");
    if (!(alpha > 0.0) || !std::isfinite(alpha)) return fail(STPI_EINVAL, "alpha must be finite and > 0");
    if (max_iters < 0) return fail(STPI_EINVAL, "max_iters must be >= 0");
    if (init != 0 && init != 1) return fail(STPI_EINVAL, "init must be 0 (use x) or 1 (uniform)");
    if (!std::isfinite(tol)) return fail(STPI_EINVAL, "tol must be finite");
    const WsLayout L = sfseg_layout(p);
    if (!ws || ws_bytes < L.total) return fail(STPI_EWORKSPACE, "sfseg workspace needs %zu bytes", L.total);
    std::memset(out, 0, sizeof(*out));
    hipStream_t st = (hipStream_t)stream;
    const DtypeOps *ops = ops_for(p->dtype);
    const size_t N = (size_t)p->T * p->H * p->W;
    const ChainMem m = chain_mem(L, ws);
    DevState *state = m.state;
    hipError_t e;
    // start vector and state (as stpi_iterate's plain form)
    if (init == 1) {
        if ((e = ops->uniform_start(x, N, state, tol, max_iters, st)) != hipSuccess) return hip_fail(e, "init");
    } else {
        if ((e = launch_state_init(state, 1.0, tol, max_iters, 0, 0, st)) != hipSuccess) return hip_fail(e, "init");
        if ((e = ops->sumsq(x, N, m.partials, st)) != hipSuccess) return hip_fail(e, "norm");
        if ((e = launch_state_from_norm(m.partials, NORM_BLOCKS_HOST, state, st)) != hipSuccess)
            return hip_fail(e, "init norm");
    }
    e = p->dtype == STPI_F64 ? sfseg_range<double>(N, s, f, m.partials, alpha, state, st)
                             : sfseg_range<float>(N, s, f, m.partials, alpha, state, st);
    if (e != hipSuccess) return hip_fail(e, "affinity range check");
    SfsegLaunch SL;
    sfseg_fill(SL, p, s, f, alpha);
    SL.buf0 = x;
    SL.buf1 = m.buf1;
    SL.nseg = sfseg_segments(*v, p);
    const int nunits = sfseg_tiles(*v, p) * SL.nseg;
    const bool defer = nunits <= DEFER_MAX_UNITS && !fusion_disabled();
    // steps in chunks; a tolerance run checks the stop flag after each chunk
    // (its last step not yet finalised)
    DevState hs;
    int done = 0;
    while (done < max_iters) {
        const int n = tol > 0.0 ? std::min(CHAIN_CHUNK, max_iters - done) : max_iters;
        for (int k = 0; k < n; ++k) {
            const int kk = done + k, slot = defer ? kk & 1 : 0;
            SL.no_prev = tol <= 0.0 && kk >= 2 && kk < max_iters - 1 ? 1 : 0;
            SL.state = m.slot(slot);
            SL.state_out = defer ? m.slot(slot ^ 1) : nullptr;
            SL.partials = m.set(slot).sums;
            SL.prev_part = {m.set(slot ^ 1).sums, nullptr};
            if ((e = v->launch(SL, st)) != hipSuccess) return hip_fail(e, "sfseg step launch");
            if (!defer && (e = launch_finalize({SL.partials, nullptr}, nunits, state, st)) != hipSuccess)
                return hip_fail(e, "finalize launch");
        }
        done += n;
        if (done < max_iters) {
            if ((e = hipMemcpyAsync(&hs, m.slot(defer ? done & 1 : 0), sizeof(hs), hipMemcpyDeviceToHost, st)) !=
                    hipSuccess ||
                (e = hipStreamSynchronize(st)) != hipSuccess)
                return hip_fail(e, "stop check");
            if (hs.done) break;
        }
    }
    const bool pend = defer && done > 0;
    const StepPartials last = {m.set((done + 1) & 1).sums, nullptr};
    if ((e = ops->normalize(x, m.buf1, N, m.slot(pend ? done & 1 : 0), last, pend ? nunits : 0, m.slot(FINAL_SLOT),
                            st)) != hipSuccess)
        return hip_fail(e, "normalize");
    if ((e = hipMemcpyAsync(&hs, m.slot(FINAL_SLOT), sizeof(hs), hipMemcpyDeviceToHost, st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
        return hip_fail(e, "state readback");
    out->iters = hs.iters;
    out->converged = hs.converged;
    out->flags = hs.flags;
    out->residual = hs.residual;
    out->lambda = hs.lambda;
    out->rayleigh = hs.rayleigh;
    out->first_residuals[0] = hs.first_res[0];
    out->first_residuals[1] = hs.first_res[1];
    if (hs.flags & FLAG_AFFINITY) {
        out->status = STPI_EINVAL;
        return fail(STPI_EINVAL, "sfseg: an affinity 1 - alpha (f_i - f_j)^2 can be negative (alpha (max f - min f)^2 "
                                 "> 1), or s has a negative or NaN value");
    }
    out->status = (hs.flags & FLAG_NONFINITE) ? STPI_ENONFINITE : (hs.flags & FLAG_ZERO) ? STPI_EZERO_NORM : 0;
    if (out->status) return fail(out->status, "iteration stopped after %d steps: %s", hs.iters,
                                 stpi_status_string(out->status));
    return STPI_OK;
}

}  // extern "C"
