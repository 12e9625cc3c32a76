// Grid transfer for the two-level start: box-average restriction of a volume
// to a coarse grid and its prolongation back (nearest cell or cell-centred
// trilinear), optionally multiplied by a fine field. One thread per output
// voxel; arithmetic in float (double for double storage).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/stpi.h"
#include "common.hpp"
#include "host_internal.hpp"

namespace stpi {

struct CoarseDims {
    int T, H, W;     // fine
    int Tc, Hc, Wc;  // coarse: ceil(T / st), ceil(H / sy), ceil(W / sy)
    int sy, st;
};

template <class ST>
__global__ void downsample_kernel(CoarseDims d, const ST *in, ST *out) {
    using CT = typename Compute<ST>::type;
    const size_t nc = (size_t)d.Tc * d.Hc * d.Wc;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += (size_t)gridDim.x * blockDim.x) {
        const int xc = (int)(i % d.Wc);
        const int yc = (int)((i / d.Wc) % d.Hc);
        const int tc = (int)(i / ((size_t)d.Wc * d.Hc));
        const int t1 = min(d.T, (tc + 1) * d.st), y1 = min(d.H, (yc + 1) * d.sy), x1 = min(d.W, (xc + 1) * d.sy);
        CT s = CT(0);
        int cnt = 0;
        for (int t = tc * d.st; t < t1; ++t)
            for (int y = yc * d.sy; y < y1; ++y) {
                const ST *row = in + ((size_t)t * d.H + y) * d.W;
                for (int x = xc * d.sy; x < x1; ++x) {
                    s += ld(row + x);
                    ++cnt;
                }
            }
        st(out + i, s / CT(cnt));
    }
}

// Cell-centred linear coordinate of fine index i on an axis of coarse size n
// and scale s: c = (i + 1/2) / s - 1/2, clamped to [0, n - 1], as its whole part
// i0 and the rest w (in whole numbers up to the last division, so that w is
// rounded once: a coordinate in CT loses the bits of its whole part).
template <class CT>
__device__ __forceinline__ void lin_axis(int i, int s, int n, int &i0, int &i1, CT &w) {
    const uint32_t num = 2u * (uint32_t)i + 1u, den = 2u * (uint32_t)s;
    const uint32_t up = num > (uint32_t)s ? num - (uint32_t)s : 0u;
    const uint32_t q = up / den;
    const bool last = q >= (uint32_t)(n - 1);
    i0 = last ? n - 1 : (int)q;
    i1 = last ? n - 1 : i0 + 1;
    w = last ? CT(0) : CT(up - q * den) / CT(den);
}

// A workgroup keeps one span of UP_SPAN columns, whose places between the coarse
// columns it finds once, and each of its wavefronts takes every so many rows.
// Linear mode: all outputs of a row lie between the same two coarse rows of the
// same two coarse frames, so the wavefront first blends those four rows into one
// in LDS (y, then t), and an output is one blend of two neighbours there. Bound
// by memory (the multiplier read, the output written): 32x480x854 from
// 16x120x214 with a multiplier 35 us, 66 with eight reads and three divisions
// of an index per output, 42 with the places found again for every row.
constexpr int UP_SPAN = 256, UP_WAVES = 4, UP_GROUPS = 2048;
template <class ST>
__global__ __launch_bounds__(64 * UP_WAVES) void upsample_kernel(CoarseDims d, int mode, const ST *in, const ST *mul,
                                                                 ST *out) {
    using CT = typename Compute<ST>::type;
    constexpr int PER = UP_SPAN / 64;  // outputs per lane
    __shared__ CT row[UP_WAVES][UP_SPAN + 2];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xb = blockIdx.x * UP_SPAN, xe = min(d.W, xb + UP_SPAN);
    int near[PER], cx0[PER], cx1[PER], cb, ce, unused;
    CT wx[PER], wu;
    lin_axis<CT>(xb, d.sy, d.Wc, cb, unused, wu);      // coarse columns cb ..
    lin_axis<CT>(xe - 1, d.sy, d.Wc, unused, ce, wu);  // .. ce
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int x = min(xb + lane + 64 * k, xe - 1);
        near[k] = x / d.sy;
        lin_axis<CT>(x, d.sy, d.Wc, cx0[k], cx1[k], wx[k]);
        cx0[k] -= cb;
        cx1[k] -= cb;
    }
    const int64_t lines = (int64_t)d.T * d.H, step = (int64_t)gridDim.y * UP_WAVES;
    const int64_t first = (int64_t)blockIdx.y * UP_WAVES + wid;
    int t = (int)(first / d.H), y = (int)(first % d.H);
    const int dt = (int)(step / d.H), dy = (int)(step % d.H);
    // every wavefront makes the rounds of the first (the barriers)
    for (int64_t line = first; line - wid < lines; line += step) {
        const bool live = line < lines;
        CT m[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int x = xb + lane + 64 * k;
            m[k] = mul && live && x < xe ? (CT)ld(mul + (size_t)line * d.W + x) : CT(1);
        }
        ST *orow = out + (size_t)line * d.W;
        if (mode == 0) {
            const ST *r = in + (live ? ((size_t)(t / d.st) * d.Hc + y / d.sy) * d.Wc : 0);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int x = xb + lane + 64 * k;
                if (live && x < xe) st(orow + x, (CT)ld(r + near[k]) * m[k]);
            }
        } else {
            if (live) {
                int t0, t1, y0, y1;
                CT wt, wy;
                lin_axis<CT>(t, d.st, d.Tc, t0, t1, wt);
                lin_axis<CT>(y, d.sy, d.Hc, y0, y1, wy);
                const ST *a0 = in + ((size_t)t0 * d.Hc + y0) * d.Wc, *a1 = in + ((size_t)t0 * d.Hc + y1) * d.Wc;
                const ST *b0 = in + ((size_t)t1 * d.Hc + y0) * d.Wc, *b1 = in + ((size_t)t1 * d.Hc + y1) * d.Wc;
                for (int c = cb + lane; c <= ce; c += 64) {
                    const CT a = (CT)ld(a0 + c) + wy * ((CT)ld(a1 + c) - (CT)ld(a0 + c));
                    const CT b = (CT)ld(b0 + c) + wy * ((CT)ld(b1 + c) - (CT)ld(b0 + c));
                    row[wid][c - cb] = a + wt * (b - a);
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int x = xb + lane + 64 * k;
                const CT r0 = row[wid][cx0[k]], r1 = row[wid][cx1[k]];
                if (live && x < xe) st(orow + x, (r0 + wx[k] * (r1 - r0)) * m[k]);
            }
            __syncthreads();  // the row is rewritten
        }
        t += dt;
        y += dy;
        if (y >= d.H) {
            y -= d.H;
            ++t;
        }
    }
}

// One output per thread, for narrow volumes, whose rows would fill a fraction of
// a span: the same blends in the same order. us, spans / this, linear: 32x4096x8
// 41 / 9.2, 4000x16x16 23 / 9.1, 64x512x16 14 / 8.8, but 1000x64x64 23.9 / 26.6.
constexpr int UP_NARROW = 48;
template <class ST>
__global__ void upsample_narrow_kernel(CoarseDims d, int mode, const ST *in, const ST *mul, ST *out) {
    using CT = typename Compute<ST>::type;
    const size_t n = (size_t)d.T * d.H * d.W;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int x = (int)(i % d.W);
        const int y = (int)((i / d.W) % d.H);
        const int t = (int)(i / ((size_t)d.W * d.H));
        CT v;
        if (mode == 0) {
            v = ld(in + ((size_t)(t / d.st) * d.Hc + y / d.sy) * d.Wc + x / d.sy);
        } else {
            int t0, t1, y0, y1, x0, x1;
            CT wt, wy, wx;
            lin_axis<CT>(t, d.st, d.Tc, t0, t1, wt);
            lin_axis<CT>(y, d.sy, d.Hc, y0, y1, wy);
            lin_axis<CT>(x, d.sy, d.Wc, x0, x1, wx);
            auto column = [&](int c) {
                auto at = [&](int tt, int yy) { return (CT)ld(in + ((size_t)tt * d.Hc + yy) * d.Wc + c); };
                const CT a = at(t0, y0) + wy * (at(t0, y1) - at(t0, y0));
                const CT b = at(t1, y0) + wy * (at(t1, y1) - at(t1, y0));
                return a + wt * (b - a);
            };
            const CT r0 = column(x0), r1 = column(x1);
            v = r0 + wx * (r1 - r0);
        }
        st(out + i, v * (mul ? (CT)ld(mul + i) : CT(1)));
    }
}

template <class ST>
static hipError_t launch_down(const CoarseDims &d, const void *in, void *out, hipStream_t s) {
    const size_t nc = (size_t)d.Tc * d.Hc * d.Wc;
    const int blocks = (int)std::min<size_t>((nc + 255) / 256, 4096);
    hipLaunchKernelGGL(downsample_kernel<ST>, dim3(blocks), dim3(256), 0, s, d, (const ST *)in, (ST *)out);
    return hipGetLastError();
}

template <class ST>
static hipError_t launch_up(const CoarseDims &d, int mode, const void *in, const void *mul, void *out,
                            hipStream_t s) {
    if (d.W <= UP_NARROW) {
        const size_t n = (size_t)d.T * d.H * d.W;
        const int blocks = (int)std::min<size_t>((n + 255) / 256, 8192);
        hipLaunchKernelGGL(upsample_narrow_kernel<ST>, dim3(blocks), dim3(256), 0, s, d, mode, (const ST *)in,
                           (const ST *)mul, (ST *)out);
        return hipGetLastError();
    }
    const int nspan = (d.W + UP_SPAN - 1) / UP_SPAN;
    const int64_t groups = ((int64_t)d.T * d.H + UP_WAVES - 1) / UP_WAVES;
    const dim3 grid((unsigned)nspan, (unsigned)std::min<int64_t>(groups, std::max(1, UP_GROUPS / nspan)));
    hipLaunchKernelGGL(upsample_kernel<ST>, grid, dim3(64 * UP_WAVES), 0, s, d, mode, (const ST *)in, (const ST *)mul,
                       (ST *)out);
    return hipGetLastError();
}

// y[i] = x[i] * s (times *s_dev when given), formed in double and rounded to
// the storage type once.
template <class ST>
__global__ void scale_kernel(size_t n, const ST *x, double s, const double *s_dev, ST *y) {
    const double m = s_dev ? s * *s_dev : s;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        st(y + i, (typename Compute<ST>::type)((double)ld(x + i) * m));
}

template <class ST>
hipError_t launch_scale(size_t n, const void *x, double s, const double *s_dev, void *y, hipStream_t st_) {
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(scale_kernel<ST>, dim3(blocks), dim3(256), 0, st_, n, (const ST *)x, s, s_dev, (ST *)y);
    return hipGetLastError();
}

static int coarse_dims(int T, int H, int W, int sy, int st, int dtype, CoarseDims &d) {
    if (T < 1 || H < 1 || W < 1) return fail(STPI_EINVAL, "volume must be at least 1x1x1 (got %dx%dx%d)", T, H, W);
    if (sy < 1 || st < 1) return fail(STPI_EINVAL, "factors must be >= 1 (got sy %d, st %d)", sy, st);
    if (dtype != STPI_F32 && dtype != STPI_BF16 && dtype != STPI_F64) return fail(STPI_EINVAL, "unknown dtype %d", dtype);
    d.T = T;
    d.H = H;
    d.W = W;
    d.sy = sy;
    d.st = st;
    d.Tc = (T + st - 1) / st;
    d.Hc = (H + sy - 1) / sy;
    d.Wc = (W + sy - 1) / sy;
    return STPI_OK;
}

}  // namespace stpi

using namespace stpi;

extern "C" {

int stpi_downsample(int T, int H, int W, int sy, int st, int dtype, const void *in, void *out, void *stream) {
    clear_error();
    CoarseDims d;
    int rc = coarse_dims(T, H, W, sy, st, dtype, d);
    if (rc) return rc;
    if (!in || !out) return fail(STPI_EINVAL, "NULL buffer");
    if (in == out) return fail(STPI_EINVAL, "out must not alias in");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = dtype == STPI_F32    ? launch_down<float>(d, in, out, s)
                   : dtype == STPI_BF16 ? launch_down<bf16>(d, in, out, s)
                                        : launch_down<double>(d, in, out, s);
    return e == hipSuccess ? STPI_OK : hip_fail(e, "downsample");
}

int stpi_upsample(int T, int H, int W, int sy, int st, int mode, int dtype, const void *in, const void *mul, void *out,
                  void *stream) {
    clear_error();
    CoarseDims d;
    int rc = coarse_dims(T, H, W, sy, st, dtype, d);
    if (rc) return rc;
    if (mode != 0 && mode != 1) return fail(STPI_EINVAL, "mode must be 0 (nearest) or 1 (linear)");
    if (!in || !out) return fail(STPI_EINVAL, "NULL buffer");
    if (in == out || mul == out) return fail(STPI_EINVAL, "out must not alias in or mul");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = dtype == STPI_F32    ? launch_up<float>(d, mode, in, mul, out, s)
                   : dtype == STPI_BF16 ? launch_up<bf16>(d, mode, in, mul, out, s)
                                        : launch_up<double>(d, mode, in, mul, out, s);
    return e == hipSuccess ? STPI_OK : hip_fail(e, "upsample");
}

int stpi_coarse_problem(const stpi_problem *fine, int sy, int st, stpi_problem *coarse) {
    clear_error();
    if (!fine || !coarse) return fail(STPI_EINVAL, "NULL problem");
    CoarseDims d;
    int rc = coarse_dims(fine->T, fine->H, fine->W, sy, st, fine->dtype, d);
    if (rc) return rc;
    if (fine->r_s < 0 || fine->r_t < 0 || !(fine->sigma_s > 0.f) || !(fine->sigma_t > 0.f))
        return fail(STPI_EINVAL, "kernel needs sigmas > 0 and radii >= 0");
    stpi_problem c = *fine;
    c.T = d.Tc;
    c.H = d.Hc;
    c.W = d.Wc;
    c.sigma_s = (float)((double)fine->sigma_s / sy);
    c.sigma_t = (float)((double)fine->sigma_t / st);
    c.r_s = (fine->r_s + sy - 1) / sy;
    c.r_t = (fine->r_t + st - 1) / st;
    *coarse = c;
    return STPI_OK;
}

int stpi_scale(int64_t n, int dtype, const void *x, double s, const double *s_dev, void *y, void *stream) {
    clear_error();
    if (n < 0) return fail(STPI_EINVAL, "negative length");
    if (dtype != STPI_F32 && dtype != STPI_BF16 && dtype != STPI_F64) return fail(STPI_EINVAL, "unknown dtype %d", dtype);
    if (n == 0) return STPI_OK;
    if (!x || !y) return fail(STPI_EINVAL, "NULL buffer");
    hipStream_t sm = (hipStream_t)stream;
    hipError_t e = dtype == STPI_F32    ? launch_scale<float>((size_t)n, x, s, s_dev, y, sm)
                   : dtype == STPI_BF16 ? launch_scale<bf16>((size_t)n, x, s, s_dev, y, sm)
                                        : launch_scale<double>((size_t)n, x, s, s_dev, y, sm);
    return e == hipSuccess ? STPI_OK : hip_fail(e, "scale");
}

}  // extern "C"
