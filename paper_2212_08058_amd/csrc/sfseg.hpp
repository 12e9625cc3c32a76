// Full SFSeg step (Sec. 3, Eq. 7 / Eq. 10): the update with the first-order
// Taylor affinity of Eq. 2,
//
//   z = s (1/alpha - f^2) G*(s x) - s G*(f^2 s x) + 2 s f G*(f s x),
//
// i.e. z_i = s_i sum_j s_j [1/alpha - (f_i - f_j)^2] G_ij x_j, with s the unary
// map raised to p and f the pairwise feature. The three filtered fields go
// through one separable stencil pass: a workgroup owns a TH x TW output tile
// and streams its frames; per frame it stages u1 = s x, u2 = f^2 s x and
// u3 = f s x on the halo-extended tile into three LDS planes (one load of s,
// f and x per element, issued a frame ahead), runs the y-pass and the x-pass
// on each plane, scatters the three results into three register rings of
// 2 RT + 1 output frames (the t-pass), and recombines them per output voxel
// with that voxel's own s and f. Zero padding comes from out-of-range buffer
// loads, as in the single-field step. The reduction partials (sum z^2 and
// sum z x_stored) and their finalisation by the next launch are those of the
// single-field step kernel. At larger radii the two spatial passes run on the
// matrix cores (sfseg_mfma_kernel).
#pragma once

#include "stencil.hpp"
#include "stencil_mfma.hpp"

namespace stpi {

template <class ST>
struct SfsegArgs {
    using CT = typename Compute<ST>::type;
    const ST *s;  // unary map to the power p
    const ST *f;  // pairwise feature
    ST *buf0;
    ST *buf1;
    const DevState *state;  // null: single step (src = buf0, dst = buf1, scale x_scale)
    DevState *state_out;    // as FwdArgs
    StepPartials prev_part;
    double *partials;
    int no_prev;  // the previous iterate is not read at the outputs (sum z x_stored = 0)
    double x_scale;
    CT ainv;  // 1 / alpha
    int T, H, W;
    int nseg;
    int rs;  // the problem's space radius
    Taps<CT> taps;
};

// The launch's view of the iteration: buffers and scale. False: nothing to do.
template <int NTHR, class ST>
__device__ __forceinline__ bool sfseg_begin(const SfsegArgs<ST> &a, int nunits, DevState &st, double *red,
                                            const ST *&src, ST *&dst, double &scale) {
    if (!a.state) {
        src = a.buf0;
        dst = a.buf1;
        scale = a.x_scale;
        return true;
    }
    if (a.state_out) {
        resolve_state<NTHR>(a.state, a.prev_part, nunits, &st, red, a.state_out, 1);
    } else {
        if (threadIdx.x == 0) st = *a.state;
        __syncthreads();
    }
    if (__builtin_amdgcn_readfirstlane(st.done)) return false;
    const int cur = __builtin_amdgcn_readfirstlane(st.cur);
    src = cur ? a.buf1 : a.buf0;
    dst = cur ? a.buf0 : a.buf1;
    scale = st.scale;
    return true;
}
template <int NTHR>
constexpr int sfseg_red() {
    return 3 * (NTHR > FINAL_THREADS ? NTHR : FINAL_THREADS) / 64;
}

template <int RS, int RT, int TH, int TW, int NTHR, int RY, int QX>
struct SfsegGeometry {
    using G = Geometry<RS, RT, TH, TW, NTHR, RY, QX>;
    static constexpr int PLANE = G::LDS_ELEMS;  // one field: staged tile, then the y-pass output
    static constexpr int LDS_ELEMS = 3 * PLANE;
};

template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX>
__global__ __launch_bounds__(NTHR) void sfseg_step_kernel(SfsegArgs<ST> a) {
    using CT = typename Compute<ST>::type;
    using IO = BufIO<ST>;
    using G = Geometry<RS, RT, TH, TW, NTHR, RY, QX>;
    using SG = SfsegGeometry<RS, RT, TH, TW, NTHR, RY, QX>;
    constexpr int NC = G::NC, NU = G::NU, NPF = G::NPF, LW = G::LW, RSA = G::RSA;
    constexpr int NYI = G::NYI, NQ = G::NQ, NXI = G::NXI, IPT = G::IPT, NTS = G::NTS;
    constexpr uint32_t ESZ = IO::SZ;
    __shared__ CT lds[SG::LDS_ELEMS];
    __shared__ double red[sfseg_red<NTHR>()];
    __shared__ DevState st;

    const int nbx = (a.W + TW - 1) / TW, nby = (a.H + TH - 1) / TH;
    const int unit = xcd_tile(blockIdx.x, nbx * nby * a.nseg);
    if (unit < 0) return;
    const int tile = unit / a.nseg, seg = unit % a.nseg;
    const int t0 = (int)((int64_t)seg * a.T / a.nseg), t1 = (int)((int64_t)(seg + 1) * a.T / a.nseg);
    const ST *src;
    ST *dst;
    double scale;
    if (!sfseg_begin<NTHR>(a, nbx * nby * a.nseg, st, red, src, dst, scale)) return;
    const CT sc = (CT)scale;
    const size_t plane = (size_t)a.H * a.W;
    const uint32_t pbytes = (uint32_t)(plane * ESZ);
    const int x0 = (tile % nbx) * TW, y0 = (tile / nbx) * TH;
    const int tid = threadIdx.x;
    const Taps<CT> &tp = a.taps;

    // staged-element offsets, as in the single-field plain tile loop
    uint32_t poff[NPF];
#pragma unroll
    for (int k = 0; k < NPF; ++k) {
        const int e = tid + k * NTHR;
        const int r = e / NC, c = e % NC;
        const int gy = y0 - RS + r, gx = x0 - RS + c;
        const bool ok = e < NU && (unsigned)gy < (unsigned)a.H && (unsigned)gx < (unsigned)a.W;
        poff[k] = ok ? (uint32_t)(gy * a.W + gx) * ESZ : OOB;
    }
    uint32_t ooff[IPT][QX];
    int orow[IPT], ocol[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int item = tid + i * NTHR;
        const bool live = item < NXI;
        orow[i] = live ? item / NQ : 0;
        ocol[i] = live ? (item % NQ) * QX : 0;
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            const int gy = y0 + orow[i], gx = x0 + ocol[i] + q;
            ooff[i][q] = (live && gy < a.H && gx < a.W) ? (uint32_t)(gy * a.W + gx) * ESZ : OOB;
        }
    }

    CT acc[3][NTS][IPT][QX];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int s = 0; s < NTS; ++s)
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int q = 0; q < QX; ++q) acc[m][s][i][q] = CT(0);

    const FrameWalk<RT> fw(a.T, t0, t1);  // frame order (the last segment walks backward)
    CT ps[NPF], pfv[NPF], px[NPF];
    // ok = false issues the same loads on an empty range (they return 0 and
    // touch no memory): both load groups below are issued in every frame, so
    // the compiler's memory-counter waits before each use allow for the
    // younger group instead of draining it
    auto fetch = [&](int t, bool ok) __attribute__((always_inline)) {
        const size_t tt = ok ? (size_t)t : 0;
        const uint32_t pb = ok ? pbytes : 0u;
        const auto rs = make_rsrc(a.s + tt * plane, pb);
        const auto rf = make_rsrc(a.f + tt * plane, pb);
        const auto rx = make_rsrc(src + tt * plane, pb);
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            ps[k] = IO::load(rs, poff[k]);
            pfv[k] = IO::load(rf, poff[k]);
            px[k] = IO::load(rx, poff[k]);
        }
    };
    fetch(fw.in(0), true);
    CT os[IPT][QX], of[IPT][QX], ox[IPT][QX];
    double d1 = 0.0, d2 = 0.0;

    ring_loop<NTS, 0>(fw.nstep, [&](auto ring_pos, int i) __attribute__((always_inline)) {
        constexpr int J = decltype(ring_pos)::value;
        CT v[3][IPT][QX];
        const bool live = i < fw.nin;
        const int tout = fw.out(i);
        const bool emit = tout >= t0 && tout < t1;
        {
            // the epilogue's operands (empty range when the frame is not emitted)
            const size_t to = emit ? (size_t)tout : 0;
            const uint32_t pb = emit ? pbytes : 0u;
            const auto rs = make_rsrc(a.s + to * plane, pb);
            const auto rf = make_rsrc(a.f + to * plane, pb);
            const auto rx = make_rsrc(src + to * plane, a.no_prev ? 0u : pb);
#pragma unroll
            for (int ii = 0; ii < IPT; ++ii)
#pragma unroll
                for (int q = 0; q < QX; ++q) {
                    os[ii][q] = IO::load(rs, ooff[ii][q]);
                    of[ii][q] = IO::load(rf, ooff[ii][q]);
                    ox[ii][q] = IO::load(rx, ooff[ii][q]);
                }
        }
        if (live) {
            // stage the three fields of this frame
#pragma unroll
            for (int k = 0; k < NPF; ++k) {
                const int e = tid + k * NTHR;
                if (NU % NTHR == 0 || k < NPF - 1 || e < NU) {
                    const CT u1 = (ps[k] * px[k]) * sc;
                    const CT u3 = pfv[k] * u1;
                    lds[e] = u1;
                    lds[SG::PLANE + e] = pfv[k] * u3;
                    lds[2 * SG::PLANE + e] = u3;
                }
            }
        }
        fetch(fw.in(i + 1), i + 1 < fw.nin);
        if (live) {
            __syncthreads();
            // y-pass of each field: RY rows of one halo column per item
            for (int it = tid; it < NYI; it += NTHR) {
                const int c = it % NC;
                const int g = it / NC;
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    const CT *col = lds + m * SG::PLANE + (g * RY) * NC + c;
                    CT u[RY + 2 * RS];
#pragma unroll
                    for (int k = 0; k < RY + 2 * RS; ++k) u[k] = col[k * NC];
                    CT *dstp = lds + m * SG::PLANE + G::NUP + (g * RY) * LW + c + (RSA - RS);
#pragma unroll
                    for (int r = 0; r < RY; ++r) {
                        CT sum = CT(0);
#pragma unroll
                        for (int d = 0; d <= 2 * RS; ++d) sum = fma(tp.gs[d], u[r + d], sum);
                        dstp[r * LW] = sum;
                    }
                }
            }
            __syncthreads();
            // x-pass of each field: QX outputs of a row per item, 16-byte LDS reads
#pragma unroll
            for (int ii = 0; ii < IPT; ++ii) {
                using V4 = LdsVec<CT>;
                constexpr int NV = (QX + 2 * RSA) / V4::N;
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    const typename V4::type *rowp = reinterpret_cast<const typename V4::type *>(
                        __builtin_assume_aligned(lds + m * SG::PLANE + G::NUP + orow[ii] * LW + ocol[ii], 16));
                    CT w[QX + 2 * RSA];
#pragma unroll
                    for (int k = 0; k < NV; ++k) {
                        const typename V4::type t = rowp[k];
#pragma unroll
                        for (int e = 0; e < V4::N; ++e) w[k * V4::N + e] = t[e];
                    }
#pragma unroll
                    for (int q = 0; q < QX; ++q) {
                        CT sum = CT(0);
#pragma unroll
                        for (int d = 0; d <= 2 * RS; ++d) sum = fma(tp.gs[d], w[q + d + RSA - RS], sum);
                        v[m][ii][q] = sum;
                    }
                }
            }
            // t-pass: each field's ring
#pragma unroll
            for (int m = 0; m < 3; ++m) ring_scatter<J, -RT, RT>(acc[m], v[m], tp);
        }
        constexpr int es = ((J - RT) % NTS + NTS) % NTS;
        if (emit) {
            const auto rz = make_rsrc(dst + (size_t)tout * plane, pbytes);
#pragma unroll
            for (int ii = 0; ii < IPT; ++ii)
#pragma unroll
                for (int q = 0; q < QX; ++q) {
                    const CT fo = of[ii][q];
                    const CT A = acc[0][es][ii][q], B = acc[1][es][ii][q], C = acc[2][es][ii][q];
                    const CT z = os[ii][q] * (fma(a.ainv - fo * fo, A, -B) + CT(2) * fo * C);
                    const double zs = (double)IO::rounded(z);
                    d2 = fma(zs, zs, d2);
                    d1 = fma(zs, (double)ox[ii][q], d1);
                    IO::store(rz, ooff[ii][q], z);
                }
        }
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int ii = 0; ii < IPT; ++ii)
#pragma unroll
                for (int q = 0; q < QX; ++q) acc[m][es][ii][q] = CT(0);
    });

    float unused = 0.f;
    block_reduce<NTHR>(d1, d2, unused, red);
    if (threadIdx.x == 0) {
        a.partials[2 * unit] = d1;
        a.partials[2 * unit + 1] = d2;
    }
}

// g v + c with a result register of its own: the compiler forms the two-operand
// multiply-add, which needs a copy of c first when c stays live or moves.
__device__ __forceinline__ float fma3(float g, float v, float c) {
    float d;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "s"(g), "v"(v), "v"(c));
    return d;
}

// The same step with both spatial passes of the three fields on the matrix
// cores, in float (v_mfma_f32_16x16x4_f32, whose products and sums round as the
// vector form's multiply-adds do): a 1D pass over 16 outputs is a product with a
// banded matrix of 16 + 2 PAD columns, as in stencil_tile_mfma. The order of a
// product's K index is free, so the four lane groups each take a quarter of the
// band's columns in a row: a lane reads its operands of all products of a block
// as 16-byte pieces. (Half-precision parts run at four times the rate: 286 us a
// step at 64x480x854, r = (15, 5), against 347 here and 485 in the vector form.
// But they keep a value to 2^-34 of the volume's largest only, so a region far
// below it came out with few bits, or as 0.)
// Per frame a workgroup (TH x TW outputs) stages the three fields of its slab
// once, y-filters 3 MB NYC blocks into the Y planes, and x-filters one block
// per field and wavefront. The planes are single-buffered and a frame has two
// barriers:
//   region 1: x-pass of frame k, staging of frame k + 1, the loads of frame
//             k + 2 (as early as their registers are free), t-pass, epilogue
//             and stores of frame k;
//   region 2: y-pass of frame k + 1.
// The t-pass is a transposed filter: the sums of the output frames still open
// move down one slot as a tap is added (acc[i] = acc[i + 1] + g v, one
// multiply-add with another destination), so the ring needs no index and the
// frame loop no unrolling (3 x 11 slots would unroll to more than the
// instruction cache).
// Bound by the matrix cores and by what does not run beside them: on the 210
// occupied CUs (r = (15, 5), 117 KB of LDS each) they are busy 50% of the time,
// the vector ALU 22% and the LDS 20%, and two barriers a frame with one workgroup
// per CU leave the loads, staging and t-pass little of the y-pass to hide behind.
template <int RT, int TH, int TW, int NTHR, int PAD>
struct SfsegMfma {
    static constexpr int MB = TH / 16, NB = TW / 16;            // output blocks down / across
    static constexpr int SR = TH + 2 * PAD, SC = TW + 2 * PAD;  // staged slab rows / columns
    static constexpr int NK = (16 + 2 * PAD) / 4;               // products per block = operands per lane
    // floats per line: an odd number of 16-byte pieces, so that the pieces of 16 lanes lie in different banks
    static constexpr int pitch(int n) { return ((n + 3) / 4 | 1) * 4; }
    static constexpr int UP = pitch(SR), YP = pitch(SC);
    static constexpr int UF = SC * UP, YF = TH * YP;  // a field's planes: staged [column][row], y-filtered [row][column]
    static constexpr int NG4 = SR / 4;                // staging items: 4 rows of a slab column
    static constexpr int NITEM = SC * NG4;
    static constexpr int IPS = (NITEM + NTHR - 1) / NTHR;
    static constexpr int NPF = 4 * IPS;
    static constexpr int NWAVE = NTHR / 64;
    static constexpr int NYC = SC / 16, NYB1 = MB * NYC, NYB = 3 * NYB1;  // y-pass blocks
    static constexpr int YPW = (NYB + NWAVE - 1) / NWAVE;
    static_assert(3 * (UF + YF) * 4 + 2048 <= 160 * 1024, "LDS");
    static_assert(SR % 4 == 0 && NK % 4 == 0 && MB * NB == NWAVE, "one output block per wavefront and field");
};

template <int RT, int TH, int TW, int NTHR, int PAD>
__global__ __launch_bounds__(NTHR) void sfseg_mfma_kernel(SfsegArgs<float> a) {
    using S = SfsegMfma<RT, TH, TW, NTHR, PAD>;
    using IO = BufIO<float>;
    constexpr int NTS = 2 * RT + 1, NPF = S::NPF, IPS = S::IPS, NK = S::NK;
    __shared__ __align__(16) float lds[3 * (S::UF + S::YF)];
    __shared__ double red[sfseg_red<NTHR>()];
    __shared__ DevState st;
    __shared__ float tapl[2 * 16 + 1];
    const int nbx = (a.W + TW - 1) / TW, nby = (a.H + TH - 1) / TH, ntiles = nbx * nby;
    const int unit = xcd_tile(blockIdx.x, ntiles * a.nseg);
    if (unit < 0) return;
    const int tile = unit % ntiles, seg = unit / ntiles;
    const int t0 = (int)((int64_t)seg * a.T / a.nseg), t1 = (int)((int64_t)(seg + 1) * a.T / a.nseg);
    const float *src;
    float *dst;
    double scale;
    if (!sfseg_begin<NTHR>(a, ntiles * a.nseg, st, red, src, dst, scale)) return;
    const float sc = (float)scale;
    if (threadIdx.x < 2 * 16 + 1) {
        float g = 0.f;
#pragma unroll
        for (int i = 0; i < 2 * 16 + 1; ++i) g = (int)threadIdx.x == i ? a.taps.gs[i] : g;
        tapl[threadIdx.x] = g;
    }
    __syncthreads();

    const size_t plane = (size_t)a.H * a.W;
    const uint32_t pbytes = (uint32_t)(plane * 4);
    const int x0 = (tile % nbx) * TW, y0 = (tile / nbx) * TH;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *const U = lds, *const Y = lds + 3 * S::UF;
    // band taps: product k of a block takes band column NK lg + k
    float tap[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int d = NK * lg + k - PAD - li;
        tap[k] = (d >= -16 && d <= 16) ? tapl[d + 16] : 0.f;
    }
    uint32_t poff[NPF];
#pragma unroll
    for (int m = 0; m < IPS; ++m) {
        const int it = tid + m * NTHR, c = it % S::SC, g = it / S::SC, gx = x0 - PAD + c;
        const bool colok = it < S::NITEM && c >= PAD - a.rs && c < TW + PAD + a.rs && (unsigned)gx < (unsigned)a.W;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 4 * g + j, gy = y0 - PAD + r;
            const bool ok = colok && r >= PAD - a.rs && r < TH + PAD + a.rs && (unsigned)gy < (unsigned)a.H;
            poff[4 * m + j] = ok ? (uint32_t)(gy * a.W + gx) * 4 : OOB;
        }
    }
    // this lane's outputs: row li, columns 4 lg .. + 3 of the wavefront's block
    const int orow = y0 + 16 * (wid / S::NB) + li, ocol = x0 + 16 * (wid % S::NB) + 4 * lg;
    const int nout = orow < a.H ? (a.W - ocol < 0 ? 0 : (a.W - ocol < 4 ? a.W - ocol : 4)) : 0;
    const uint32_t ooff = nout > 0 ? (uint32_t)(orow * a.W + ocol) * 4 : OOB;

    float acc[3][NTS][4];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int i = 0; i < NTS; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[m][i][q] = 0.f;
    const FrameWalk<RT> fw(a.T, t0, t1);
    const int nin = fw.nin;
    float ps[NPF], pf[NPF], px[NPF];
    // an empty range when !ok (see FwdOp::fetch)
    auto fetch = [&](int t, bool ok) __attribute__((always_inline)) {
        const size_t o = (size_t)(ok ? t : 0) * plane;
        const uint32_t pb = ok ? pbytes : 0u;
        const auto rs = make_rsrc(a.s + o, pb), rf = make_rsrc(a.f + o, pb), rx = make_rsrc(src + o, pb);
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            ps[k] = IO::load(rs, poff[k]);
            px[k] = IO::load(rx, poff[k]);
            pf[k] = IO::load(rf, poff[k]);
        }
    };
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < IPS; ++m) {
            const int it = tid + m * NTHR;
            if (S::NITEM % NTHR == 0 || m < IPS - 1 || it < S::NITEM) {
                float *q = U + (it % S::SC) * S::UP + 4 * (it / S::SC);
                float4_t u[3];  // the three fields: u, u f^2, u f
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = 4 * m + j;
                    u[0][j] = (ps[k] * px[k]) * sc;
                    u[2][j] = pf[k] * u[0][j];
                    u[1][j] = pf[k] * u[2][j];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) *reinterpret_cast<float4_t *>(q + c * S::UF) = u[c];
            }
        }
    };
    auto operands = [&](const float *p, float (&w)[NK]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NK / 4; ++j) {
            const float4_t t = reinterpret_cast<const float4_t *>(p + NK * lg)[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[4 * j + e] = t[e];
        }
    };
    auto ypass = [&]() __attribute__((always_inline)) {
        float4_t ya[S::YPW];
#pragma unroll
        for (int m = 0; m < S::YPW; ++m) {
            const int b = wid + m * S::NWAVE, f = b / S::NYB1, rb = b % S::NYB1 / S::NYC, cb = b % S::NYC;
            if (S::NYB % S::NWAVE == 0 || m < S::YPW - 1 || b < S::NYB) {
                float w[NK];
                operands(U + f * S::UF + (16 * cb + li) * S::UP + 16 * rb, w);
                ya[m] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < NK; ++k) ya[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[k], tap[k], ya[m], 0, 0, 0);
            }
        }
#pragma unroll
        for (int m = 0; m < S::YPW; ++m) {
            const int b = wid + m * S::NWAVE, f = b / S::NYB1, rb = b % S::NYB1 / S::NYC, cb = b % S::NYC;
            if (S::NYB % S::NWAVE == 0 || m < S::YPW - 1 || b < S::NYB)
                *reinterpret_cast<float4_t *>(Y + f * S::YF + (16 * rb + li) * S::YP + 16 * cb + 4 * lg) = ya[m];
        }
    };
    double d1 = 0.0, d2 = 0.0;
    fetch(fw.in(0), true);
    stage();
    __syncthreads();
    fetch(fw.in(1), 1 < nin);
    ypass();
    __syncthreads();
    for (int k = 0; k < fw.nstep; ++k) {
        const int tout = fw.out(k);
        const bool emit = tout >= t0 && tout < t1;
        const size_t to = (size_t)(emit ? tout : 0) * plane;
        const uint32_t ob = emit ? pbytes : 0u;
        float os[4], of[4], ox[4];
        IO::load4(make_rsrc(a.s + to, ob), ooff, os);
        IO::load4(make_rsrc(a.f + to, ob), ooff, of);
        IO::load4(make_rsrc(src + to, a.no_prev ? 0u : ob), ooff, ox);
        float4_t v[3];
        // without branches, as the single-field loop: past the last input frame
        // the loads return 0, and with them the staged fields and the products
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            float w[NK];
            operands(Y + m * S::YF + (16 * (wid / S::NB) + li) * S::YP + 16 * (wid % S::NB), w);
            v[m] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < NK; ++i) v[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(tap[i], w[i], v[m], 0, 0, 0);
        }
        stage();
        fetch(fw.in(k + 2), k + 2 < nin);
        // fma3 is inline assembly, for which the compiler inserts no wait states
        // after the products that made v
        asm volatile("s_nop 15\n\ts_nop 7" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]));
        // t-pass: slot i holds the output frame i steps ahead of out(k)
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int i = 0; i < NTS - 1; ++i) acc[m][i][q] = fma3(a.taps.gt[i], v[m][q], acc[m][i + 1][q]);
                acc[m][NTS - 1][q] = a.taps.gt[NTS - 1] * v[m][q];
            }
        if (emit) {
            const auto rz = make_rsrc(dst + to, pbytes);
            float z[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // columns past the right edge: the 4-wide loads read the next row there
                const float fo = of[q];
                const float A = acc[0][0][q], B = acc[1][0][q], C = acc[2][0][q];
                z[q] = q < nout ? os[q] * (fmaf(a.ainv - fo * fo, A, -B) + 2.f * fo * C) : 0.f;
                const double zs = (double)z[q];
                d2 = fma(zs, zs, d2);
                d1 = fma(zs, (double)ox[q], d1);
            }
            if (nout == 4) {
                IO::store4(rz, ooff, z);
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (q < nout) IO::store(rz, ooff + 4 * q, z[q]);
            }
        }
        __syncthreads();
        ypass();
        __syncthreads();
    }
    float unused = 0.f;
    block_reduce<NTHR>(d1, d2, unused, red);
    if (threadIdx.x == 0) {
        a.partials[2 * unit] = d1;
        a.partials[2 * unit + 1] = d2;
    }
}

// The range check of the affinity (Eq. 2's Taylor term): every entry of M is
// >= 0 when s >= 0 and alpha (max f - min f)^2 <= 1. Per-block min f, max f,
// min s into partials[3 b .. 3 b + 2]; a NaN anywhere gives NaNs.
// One read of both volumes, 16-byte chunks with two of each in flight per
// thread (196 us element by element on 256 workgroups at 64x480x854, 42 us now).
constexpr int SFSEG_RANGE_BLOCKS = 1024;
struct SfsegRange {
    double fmn, fmx, smn;
    __device__ __forceinline__ void take(double f, double s) {
        fmn = (f < fmn || f != f) ? f : fmn;
        fmx = (f > fmx || f != f) ? f : fmx;
        smn = (s < smn || s != s) ? s : smn;
    }
    // minima with minima, maxima with maxima: an empty range changes nothing
    __device__ __forceinline__ void take(const SfsegRange &o) {
        fmn = (o.fmn < fmn || o.fmn != o.fmn) ? o.fmn : fmn;
        fmx = (o.fmx > fmx || o.fmx != o.fmx) ? o.fmx : fmx;
        smn = (o.smn < smn || o.smn != o.smn) ? o.smn : smn;
    }
    __device__ __forceinline__ void wave() {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const SfsegRange o = {__shfl_xor(fmn, off, 64), __shfl_xor(fmx, off, 64), __shfl_xor(smn, off, 64)};
            take(o);
        }
    }
};
constexpr SfsegRange SFSEG_RANGE_EMPTY = {INFINITY, -INFINITY, INFINITY};

template <class ST>
__global__ __launch_bounds__(256) void sfseg_range_kernel(size_t n, const ST *s, const ST *f, double *partials) {
    __shared__ SfsegRange rw[256 / 64];
    constexpr int VEC = 16 / (int)sizeof(ST);
    SfsegRange r = SFSEG_RANGE_EMPTY;
    const size_t stride = (size_t)gridDim.x * 256, tid = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t head = 0;
    if ((((uintptr_t)s | (uintptr_t)f) & 15) == 0) {
        const size_t nv = n / VEC;
        const uint4 *s4 = reinterpret_cast<const uint4 *>(s), *f4 = reinterpret_cast<const uint4 *>(f);
        // minima and maxima in the storage type (exact), widened at the end; a NaN sticks
        ST fmn = (ST)INFINITY, fmx = -(ST)INFINITY, smn = (ST)INFINITY;
        bool nan = false;
        for (size_t i = tid; i < nv; i += 2 * stride) {
            union {
                uint4 u;
                ST e[VEC];
            } cs[2], cf[2];
            const size_t i1 = i + stride < nv ? i + stride : i;
            cs[0].u = s4[i];
            cf[0].u = f4[i];
            cs[1].u = s4[i1];
            cf[1].u = f4[i1];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const ST fv = cf[k].e[e], sv = cs[k].e[e];
                    nan |= fv != fv || sv != sv;
                    fmn = fv < fmn ? fv : fmn;
                    fmx = fv > fmx ? fv : fmx;
                    smn = sv < smn ? sv : smn;
                }
        }
        r.take(SfsegRange{(double)fmn, (double)fmx, (double)smn});
        if (nan) r.take((double)NAN, (double)NAN);
        head = nv * VEC;
    }
    for (size_t i = head + tid; i < n; i += stride) r.take((double)f[i], (double)s[i]);
    r.wave();
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) rw[wid] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / 64; ++w) r.take(rw[w]);
        partials[3 * blockIdx.x] = r.fmn;
        partials[3 * blockIdx.x + 1] = r.fmx;
        partials[3 * blockIdx.x + 2] = r.smn;
    }
}

template <class ST>
__global__ void sfseg_unary_kernel(size_t n, const ST *S, double p, ST *s) {
    using CT = typename Compute<ST>::type;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const CT v = ld(S + i);
        // S^p for S >= 0 (0^p = 0 for p > 0, 1 for p = 0); NaN for negative S
        st(s + i, (CT)pow((double)v, p));
    }
}

struct SfsegLaunch {
    const void *s, *f;
    void *buf0, *buf1;
    const DevState *state;
    DevState *state_out;
    StepPartials prev_part;
    double *partials;
    int no_prev;
    double x_scale;
    double ainv;
    int T, H, W, nseg;
    double gs[2 * 16 + 1];
    double gt[2 * 8 + 1];
};

using SfsegLaunchFn = hipError_t (*)(const SfsegLaunch &, hipStream_t);

struct SfsegVariant {
    int RS, RT, TH, TW, NTHR;
    int mfma;  // 1: matrix-core spatial passes
    SfsegLaunchFn launch;
    int (*blocks_per_cu)();
};

// CENTRE: where the kernel wants the centre space tap.
template <class ST, int CENTRE, int RT>
SfsegArgs<ST> sfseg_args(const SfsegLaunch &L) {
    using CT = typename Compute<ST>::type;
    SfsegArgs<ST> a;
    a.s = (const ST *)L.s;
    a.f = (const ST *)L.f;
    a.buf0 = (ST *)L.buf0;
    a.buf1 = (ST *)L.buf1;
    a.state = L.state;
    a.state_out = L.state_out;
    a.prev_part = L.prev_part;
    a.partials = L.partials;
    a.no_prev = L.state && L.no_prev ? 1 : 0;
    a.x_scale = L.x_scale;
    a.ainv = (CT)L.ainv;
    a.T = L.T;
    a.H = L.H;
    a.W = L.W;
    a.nseg = L.nseg > 0 ? L.nseg : 1;
    a.rs = 0;
    for (int d = 1; d <= 16; ++d)
        if (L.gs[16 + d] != 0.0) a.rs = d;
    for (int i = 0; i < 2 * 16 + 1; ++i) a.taps.gs[i] = CT(0);
    for (int i = 0; i < 2 * 8 + 1; ++i) a.taps.gt[i] = CT(0);
    for (int d = -CENTRE; d <= CENTRE; ++d) a.taps.gs[d + CENTRE] = (CT)L.gs[d + 16];
    for (int d = -RT; d <= RT; ++d) a.taps.gt[d + RT] = (CT)L.gt[d + 8];
    return a;
}

template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX>
hipError_t launch_sfseg(const SfsegLaunch &L, hipStream_t stream) {
    if (L.state && L.state_out == L.state) return hipErrorInvalidValue;
    const SfsegArgs<ST> a = sfseg_args<ST, RS, RT>(L);
    const int nunits = ((L.W + TW - 1) / TW) * ((L.H + TH - 1) / TH) * a.nseg;
    const int per = (nunits + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((sfseg_step_kernel<ST, RS, RT, TH, TW, NTHR, RY, QX>), dim3(per * NUM_XCD), dim3(NTHR), 0,
                       stream, a);
    return hipGetLastError();
}

template <int RT, int TH, int TW, int NTHR, int PAD>
hipError_t launch_sfseg_mfma(const SfsegLaunch &L, hipStream_t stream) {
    if (L.state && L.state_out == L.state) return hipErrorInvalidValue;
    const SfsegArgs<float> a = sfseg_args<float, 16, RT>(L);
    const int nunits = ((L.W + TW - 1) / TW) * ((L.H + TH - 1) / TH) * a.nseg;
    const int per = (nunits + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((sfseg_mfma_kernel<RT, TH, TW, NTHR, PAD>), dim3(per * NUM_XCD), dim3(NTHR), 0, stream, a);
    return hipGetLastError();
}

template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX>
int sfseg_blocks_per_cu() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sfseg_step_kernel<ST, RS, RT, TH, TW, NTHR, RY, QX>, NTHR,
                                                     0) != hipSuccess)
        n = 1;
    return n > 0 ? n : 1;
}

template <int RT, int TH, int TW, int NTHR, int PAD>
int sfseg_mfma_blocks_per_cu() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sfseg_mfma_kernel<RT, TH, TW, NTHR, PAD>, NTHR, 0) !=
        hipSuccess)
        n = 1;
    return n > 0 ? n : 1;
}

}  // namespace stpi
