// Forward power-iteration step and the small kernels of the iteration chain.
#pragma once

#include <type_traits>

#include "stencil.hpp"
#include "stencil_mfma.hpp"

namespace stpi {

// Launch description shared by every storage type (host side).
struct FwdLaunch {
    const void *f;
    void *buf0;          // the caller's x (iterate mode: ping-pong buffer 0)
    void *buf1;          // z (iterate mode: ping-pong buffer 1)
    DevState *state;     // null: single step with x_scale, src = buf0, dst = buf1
    double x_scale;
    const double *norm_in;  // single step: if set, x_scale = 1 / *norm_in (read on the device)
    void *vout;             // if set, also store v = G (f x) (x unit) for the adjoint
    double *partials;    // [tiles * nseg][2] doubles
    uint32_t *wpart;     // iterate mode: [tiles * nseg] maxima (see StepPartials)
    // iterate mode: the slot this step's state goes to and the previous step's
    // partials (resolve_state); state_out null: the state is already final
    // (a separate kernel finalises every step)
    DevState *state_out;
    StepPartials prev_part;
    int T, H, W;
    int nseg;            // frame segments per tile (0 is read as 1)
    int no_prev;         // iterate mode: the step's inner product with the previous iterate is not formed
    // matrix-core variants: float bits of a bound on |f x_stored scale| (iterate
    // mode: on |f|, the iterate being unit; single step: on |f x_stored|, scaled
    // by |x_scale| in the kernel)
    const uint32_t *ubound;
    double gs[2 * 16 + 1];
    double gt[2 * 8 + 1];
};

// One variant of the step kernel: compiled radii and tile.
using FwdLaunchFn = hipError_t (*)(const FwdLaunch &, hipStream_t);

struct Variant {
    int RS, RT, TH, TW, NTHR, RY, QX, OCC, PIPE;
    FwdLaunchFn launch;
    int (*blocks_per_cu)();  // resident workgroups per CU (occupancy query)
    FwdLaunchFn launch_p;    // product-form chain step (see FwdOpP); null where not compiled
};

template <class ST>
struct FwdArgs {
    using CT = typename Compute<ST>::type;
    const ST *f;
    ST *buf0;
    ST *buf1;
    const DevState *state;
    DevState *state_out;       // see FwdLaunch
    StepPartials prev_part;
    double *partials;
    uint32_t *wpart;
    int no_prev;  // 1: the previous iterate is not read at the outputs (p1 = 0; see FwdOp::prev)
    double x_scale;
    const double *norm_in;
    ST *vout;
    int T, H, W;
    int nseg;  // frame segments per tile: workgroup (tile, seg) owns frames [seg T / nseg, (seg + 1) T / nseg)
    const uint32_t *ubound;  // matrix-core variants (see FwdLaunch)
    int rs;                  // the problem's space radius
    Taps<CT> taps;
};

// A 4-wide load of bfloat16 values reads words of two. Where a frame's last
// voxel has no partner (a frame of an odd number of voxels), its word reaches
// past the frame's range and reads as 0 whole: the workgroup that owns the voxel
// loads it by itself as well and puts it in place. Kernels of their own (ODD)
// do so, as the two loads and registers cost the others 3% (20 iterations of
// 64x480x854 1765 -> 1818 us).
template <class ST, int QX, int PIPE>
constexpr bool odd_frames_apart() {
    return std::is_same<ST, bf16>::value && QX == 4 && PIPE != 2 && PIPE != 4;
}
constexpr uint32_t NO_LAST = 1u;  // no element's offset: the voxel is in another tile
inline __device__ uint32_t last_of_odd_frame(int H, int W, int x0, int y0, int TH, int TW) {
    if ((H & W & 1) == 0 || x0 + TW < W || y0 + TH < H) return NO_LAST;
    return (uint32_t)((size_t)H * W - 1) * (uint32_t)sizeof(bf16);
}
// Two operand arrays of the epilogue, and with ODD the last voxel's two values.
template <class CT, int IPT, int QX, bool ODD>
struct LastVoxel {
    __device__ __forceinline__ void place(uint32_t, const uint32_t (&)[IPT][QX], CT (&)[IPT][QX], CT (&)[IPT][QX]) const {}
};
template <class CT, int IPT, int QX>
struct LastVoxel<CT, IPT, QX, true> {
    CT a, b;
    __device__ __forceinline__ void place(uint32_t last, const uint32_t (&off)[IPT][QX], CT (&va)[IPT][QX],
                                          CT (&vb)[IPT][QX]) const {
        if (last == NO_LAST) return;
#pragma unroll
        for (int i = 0; i < IPT; ++i)
#pragma unroll
            for (int q = 0; q < QX; q += 2) {  // a group starts on a multiple of 4, the voxel's index is even
                va[i][q] = off[i][q] == last ? a : va[i][q];
                vb[i][q] = off[i][q] == last ? b : vb[i][q];
            }
    }
};

// u = f * x_stored; z = s f acc with s the scale that makes x unit;
// p1 += z * x_stored, p2 += z^2 on the values as stored. The products are
// formed in double, where they are exact for float and bfloat16 operands, so
// the residual sqrt(2 - 2 cos) keeps its accuracy near convergence.
template <class ST, bool ODD = false>
struct FwdOp {
    using CT = typename Compute<ST>::type;
    using IO = BufIO<ST>;
    static constexpr uint32_t ESZ = IO::SZ;
    const ST *f;
    const ST *src;
    ST *dst;
    ST *vout;         // optional: v = s * acc = G (f x_unit)
    CT scale;
    size_t plane;     // elements per frame
    uint32_t pbytes;  // bytes per frame
    bool cut = false;  // epilogue operands came from 4-wide loads that groups cut by the right edge extend past it
    uint32_t last = NO_LAST;  // ODD: see last_of_odd_frame
    // false: the epilogue reads the previous iterate on an empty range (as 0),
    // so p1 is 0. A chain of a fixed count of steps uses p1 (the cosine with
    // the previous iterate: the residual and the Rayleigh quotient) only on
    // its first two steps and its last; the other steps save that read.
    bool prev = true;

    template <int NPF>
    struct Raw {
        CT f[NPF], x[NPF];
    };
    // live = false issues the same loads on an empty range (they return 0 and
    // touch no memory): the matrix-core tile loop fetches every phase, so the
    // compiler's memory-counter waits count a fixed number of younger loads
    template <int NPF>
    __device__ __forceinline__ void fetch(int t, const uint32_t (&off)[NPF], Raw<NPF> &raw, bool live = true) const {
        const auto rf = make_rsrc(f + (size_t)(live ? t : 0) * plane, live ? pbytes : 0u);
        const auto rx = make_rsrc(src + (size_t)(live ? t : 0) * plane, live ? pbytes : 0u);
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            raw.f[k] = IO::load(rf, off[k]);
            raw.x[k] = IO::load(rx, off[k]);
        }
    }
    template <int NPF>
    __device__ __forceinline__ CT input(const Raw<NPF> &raw, int k) const {
        return raw.f[k] * raw.x[k];
    }
    template <int IPT, int QX>
    struct OutRaw {
        CT f[IPT][QX], x[IPT][QX];
        LastVoxel<CT, IPT, QX, ODD> last;
    };
    // Epilogue operands, in a fixed count of memory instructions whatever the
    // lanes: with QX = 4 each group moves with one 4-wide access at its first
    // offset (a group cut by the right edge of the frame then reads into the
    // next row, and the epilogue, told by cut, takes f there as 0); otherwise
    // element by element. live = false issues the loads on an empty range.
    template <int IPT, int QX>
    __device__ __forceinline__ void fetch_out(int t, const uint32_t (&off)[IPT][QX], OutRaw<IPT, QX> &raw,
                                              bool live = true) const {
        const auto rf = make_rsrc(f + (size_t)(live ? t : 0) * plane, live ? pbytes : 0u);
        const auto rx = make_rsrc(src + (size_t)(live ? t : 0) * plane, live && prev ? pbytes : 0u);
        if constexpr (ODD) {
            if (last != NO_LAST) {
                raw.last.a = IO::load(rf, last);
                raw.last.b = IO::load(rx, last);
            }
        }
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            if constexpr (QX == 4) {
                IO::load4(rf, off[i][0], raw.f[i]);
                IO::load4(rx, off[i][0], raw.x[i]);
            } else {
#pragma unroll
                for (int q = 0; q < QX; ++q) {
                    raw.f[i][q] = IO::load(rf, off[i][q]);
                    raw.x[i][q] = IO::load(rx, off[i][q]);
                }
            }
        }
    }
    // Fixed-count forms for the straight-line tile loop: every call issues the
    // same memory instructions (one per element), whatever the tile position
    // and whether the frame is emitted, so the compiler's memory-counter waits
    // never have to cover a path with fewer operations. Elements outside the
    // frame and non-emitted frames use out-of-range offsets (loads give 0,
    // stores are dropped) and add nothing to the sums.
    template <int IPT, int QX>
    __device__ __forceinline__ void fetch_out_fixed(int t, const uint32_t (&off)[IPT][QX],
                                                    OutRaw<IPT, QX> &raw) const {
        const auto rf = make_rsrc(f + (size_t)t * plane, pbytes);
        const auto rx = make_rsrc(src + (size_t)t * plane, prev ? pbytes : 0u);
#pragma unroll
        for (int i = 0; i < IPT; ++i)
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                raw.f[i][q] = IO::load(rf, off[i][q]);
                raw.x[i][q] = IO::load(rx, off[i][q]);
            }
    }
    template <int IPT, int QX>
    __device__ __forceinline__ void emit_frame_fixed(int t, bool emit, const CT (&acc)[IPT][QX],
                                                     const OutRaw<IPT, QX> &raw, const uint32_t (&off)[IPT][QX],
                                                     double &d1, double &d2) const {
        const auto rz = make_rsrc(dst + (size_t)t * plane, pbytes);
        if (vout) {
            const auto rv = make_rsrc(vout + (size_t)t * plane, pbytes);
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int q = 0; q < QX; ++q) IO::store(rv, emit ? off[i][q] : OOB, scale * acc[i][q]);
        }
        double p1 = 0.0, p2 = 0.0;
#pragma unroll
        for (int i = 0; i < IPT; ++i)
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                const CT z = scale * (raw.f[i][q] * acc[i][q]);
                const double zs = (double)IO::rounded(z);
                p2 = fma(zs, zs, p2);
                p1 = fma(zs, (double)raw.x[i][q], p1);
                IO::store(rz, emit ? off[i][q] : OOB, z);
            }
        d1 += emit ? p1 : 0.0;
        d2 += emit ? p2 : 0.0;
    }
    template <int IPT, int QX>
    __device__ __forceinline__ void emit_frame(int t, const CT (&acc)[IPT][QX], const OutRaw<IPT, QX> &loaded,
                                               const uint32_t (&off)[IPT][QX], double &d1, double &d2) const {
        OutRaw<IPT, QX> raw = loaded;
        raw.last.place(last, off, raw.f, raw.x);
        const auto rz = make_rsrc(dst + (size_t)t * plane, pbytes);
        if (vout) {
            const auto rv = make_rsrc(vout + (size_t)t * plane, pbytes);
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int q = 0; q < QX; ++q) IO::store(rv, off[i][q], scale * acc[i][q]);
        }
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            CT z[QX];
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                const CT fv = cut && off[i][q] == OOB ? CT(0) : raw.f[i][q];
                z[q] = scale * (fv * acc[i][q]);
                const double zs = (double)IO::rounded(z[q]);
                d2 = fma(zs, zs, d2);
                d1 = fma(zs, (double)raw.x[i][q], d1);
            }
            if constexpr (QX == 4) {
                if (off[i][3] != OOB) {
                    IO::store4(rz, off[i][0], z);
                    continue;
                }
            }
#pragma unroll
            for (int q = 0; q < QX; ++q) IO::store(rz, off[i][q], z[q]);
        }
    }
};

// 1 / f from the hardware reciprocal (about one ulp); 0 for f = 0 and for
// subnormal f (whose outputs are negligible).
__device__ __forceinline__ float recip_or_zero(float fv) {
    return fabsf(fv) >= 1.17549435e-38f ? __builtin_amdgcn_rcpf(fv) : 0.f;
}

// Product form of a chain step (matrix-core tile loop only). The buffers hold
// w = f x g instead of the iterate x, with g = 2^-2e a power of two from the
// bound max |f| < 2^e (so w stays in range whatever the scale of f). A step
// then stages one array, w (times a power of two: w scale 2^(10 + e) =
// f x_unit 2^(10 - e)), instead of f and x, and its epilogue reads f and w at
// the outputs as the plain form reads f and x. It stores
// w_new = acc f^2 2^-S g; the iterate is w / (f g) (0 where f = 0). The
// sums are taken on its float image x~ = fl(w rcp(f)) / g: p2 = sum x~_new^2
// and p1 = sum x~_prev x~_new, products exact in double. The next step forms
// x~_prev from the same stored w and f, so it is bitwise this step's x~_new:
// the scale, the cosine and the norm all refer to one vector, which differs
// from the staged iterate by float rounding per element (the residual keeps
// float-level accuracy near convergence). The emitted sums leave out the
// powers of two 1/g: the caller multiplies d1 by ginv_in ginv_out and d2 by
// ginv_out^2. ginv_in = 1 / g of the input: 1 on the first step of a uniform
// start, whose input is f itself (w of the constant 1, up to g).
// Staging range: the staged values are w s ginv_in 2^(10 - e_in) with e_in the
// exponent of a bound on |w s ginv_in| taken from max |w| of the input buffer
// (collected by the step that wrote it; max |f| for the uniform start), so
// the largest staged value lies in [2^9, 2^10) whatever the scale of the
// iterate, and the split's half-precision parts keep their full precision
// for every value within 2^14 of it.

template <class ST, bool ODD = false>
struct FwdOpP {
    using CT = float;
    using IO = BufIO<ST>;
    static constexpr uint32_t ESZ = IO::SZ;
    const ST *f;
    const ST *src;  // w of the current iterate (or f)
    ST *dst;        // w of the next
    CT gout;        // g
    CT sg;          // 2^-S g (2^-S undoes the staging prescale): w_new = acc f^2 sg
    double ginv_in, ginv_out;
    size_t plane;
    uint32_t pbytes;
    mutable float wmax = 0.f;  // max |w_new| stored by this thread (the next step's staging bound)
    bool cut = false;          // as FwdOp::cut
    bool prev = true;          // as FwdOp::prev
    uint32_t last = NO_LAST;   // as FwdOp::last

    template <int NPF>
    struct Raw {
        CT u[NPF];
    };
    template <int NPF>
    __device__ __forceinline__ void fetch(int t, const uint32_t (&off)[NPF], Raw<NPF> &raw, bool live = true) const {
        const auto ru = make_rsrc(src + (size_t)(live ? t : 0) * plane, live ? pbytes : 0u);
#pragma unroll
        for (int k = 0; k < NPF; ++k) raw.u[k] = IO::load(ru, off[k]);
    }
    template <int NPF>
    __device__ __forceinline__ CT input(const Raw<NPF> &raw, int k) const {
        return raw.u[k];
    }
    template <int IPT, int QX>
    struct OutRaw {
        CT f[IPT][QX], u[IPT][QX];
        LastVoxel<CT, IPT, QX, ODD> last;
    };
    template <int IPT, int QX>  // as FwdOp::fetch_out
    __device__ __forceinline__ void fetch_out(int t, const uint32_t (&off)[IPT][QX], OutRaw<IPT, QX> &raw,
                                              bool live = true) const {
        const auto rf = make_rsrc(f + (size_t)(live ? t : 0) * plane, live ? pbytes : 0u);
        const auto ru = make_rsrc(src + (size_t)(live ? t : 0) * plane, live && prev ? pbytes : 0u);
        if constexpr (ODD) {
            if (last != NO_LAST) {
                raw.last.a = IO::load(rf, last);
                raw.last.b = IO::load(ru, last);
            }
        }
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            if constexpr (QX == 4) {
                IO::load4(rf, off[i][0], raw.f[i]);
                IO::load4(ru, off[i][0], raw.u[i]);
            } else {
#pragma unroll
                for (int q = 0; q < QX; ++q) {
                    raw.f[i][q] = IO::load(rf, off[i][q]);
                    raw.u[i][q] = IO::load(ru, off[i][q]);
                }
            }
        }
    }
    template <int IPT, int QX>
    __device__ __forceinline__ void emit_frame(int t, const CT (&acc)[IPT][QX], const OutRaw<IPT, QX> &loaded,
                                               const uint32_t (&off)[IPT][QX], double &d1, double &d2) const {
        OutRaw<IPT, QX> raw = loaded;
        raw.last.place(last, off, raw.f, raw.u);
        const auto rw = make_rsrc(dst + (size_t)t * plane, pbytes);
        CT wr[IPT][QX], r[IPT][QX];  // what the stores leave in memory, 1/f
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            CT w[QX];
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                const CT fv = cut && off[i][q] == OOB ? CT(0) : raw.f[i][q];
                w[q] = (acc[i][q] * (fv * fv)) * sg;
                r[i][q] = recip_or_zero(fv);
            }
            bool whole = false;
            if constexpr (QX == 4) {
                if (off[i][3] != OOB) {
                    IO::store4_rounded(rw, off[i][0], w, wr[i]);
                    whole = true;
                }
            }
            if (!whole) {
#pragma unroll
                for (int q = 0; q < QX; ++q) wr[i][q] = IO::store_rounded(rw, off[i][q], w[q]);
            }
        }
        // The sums after every store of the frame: the branch on prev (uniform)
        // then holds no memory operation, so the waits that follow count the
        // same younger operations on both paths.
        if (prev) {
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int q = 0; q < QX; ++q) {
                    wmax = fmaxf(wmax, fabsf(wr[i][q]));
                    const double xn = (double)(wr[i][q] * r[i][q]);
                    const double xp = (double)(raw.u[i][q] * r[i][q]);
                    d2 = fma(xn, xn, d2);
                    d1 = fma(xp, xn, d1);
                }
        } else {
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int q = 0; q < QX; ++q) {
                    wmax = fmaxf(wmax, fabsf(wr[i][q]));
                    const double xn = (double)(wr[i][q] * r[i][q]);
                    d2 = fma(xn, xn, d2);
                }
        }
    }
};

// OCC: minimum waves per SIMD the register allocation must allow (1 = no limit;
// with NTHR = 512, OCC = 4 lets two workgroups share a CU).
// PIPE: 1 selects the software-pipelined tile loop (stencil_tile_pipe), 2 its
// straight-line form (stencil_tile_flat), 3 the matrix-core tile loop
// (stencil_tile_mfma; RS = 16, any space radius up to 16), 4 the output frames of
// a segment one by one with all their input frames at once (stencil_tile_gather;
// segments of one frame while that is at most four workgroups per CU).
// ALT: the kernel for frames of an odd number of voxels (odd_frames_apart); with
// PIPE 4 the one for segments of several frames (the loop over them costs the
// others 0.3 us of 6).
// PF: product-form chain step (PIPE 3, iterate mode only).
template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX, int OCC, int PIPE, bool PF, bool ALT>
__global__ __launch_bounds__(NTHR, OCC) void fwd_step_kernel(FwdArgs<ST> a) {
    using CT = typename Compute<ST>::type;
    constexpr bool ODD = ALT && PIPE != 4;
    using G = Geometry<RS, RT, TH, TW, NTHR, RY, QX>;
    using PG = PipeGeometry<RS, RT, TH, TW, NTHR, RY, QX>;
    static_assert(PIPE != 3 || ((RS == 16 || RS == 8) && sizeof(CT) == 4),
                  "matrix-core variants: RS 8 or 16 (the slab margin), float arithmetic");
    static_assert(!PF || PIPE == 3, "the product form runs on the matrix-core tile loop");
    constexpr int PAD = RS <= 8 ? 8 : 16;
    // bfloat16 product-form chains stage their raw bfloat16 values (one U plane)
    constexpr bool EXACT = PF && std::is_same<ST, bf16>::value;
    __shared__ CT lds[PIPE == 3 ? MfmaLds<PIPE, TH, TW, NTHR, PAD, EXACT ? 1 : 2>::value
                                : (PIPE == 1 || PIPE == 2 ? PG::LDS_ELEMS : G::LDS_ELEMS)];
    constexpr int RED = 3 * (NTHR > FINAL_THREADS ? NTHR : FINAL_THREADS) / 64;
    __shared__ double red[RED];

    const int nbx = (a.W + TW - 1) / TW, nby = (a.H + TH - 1) / TH;
    // consecutive units share an XCD: neighbouring tiles of one frame segment
    // (they stage overlapping slabs of the same frames at about the same time,
    // so halo lines fetched by one are L2 hits for the other)
    const int ntiles = nbx * nby;
    const int unit = xcd_tile(blockIdx.x, ntiles * a.nseg);
    if (unit < 0) return;
    const int tile = unit % ntiles, seg = unit / ntiles;
    const int t0 = (int)((int64_t)seg * a.T / a.nseg), t1 = (int)((int64_t)(seg + 1) * a.T / a.nseg);
    FwdOp<ST, ODD> op;
    op.f = a.f;
    double scale;
    __shared__ DevState st;  // iterate mode: the state this step works on
    if (a.state) {
        if (a.state_out)
            resolve_state<NTHR>(a.state, a.prev_part, ntiles * a.nseg, &st, red, a.state_out, 1);
        else {
            if (threadIdx.x == 0) st = *a.state;
            __syncthreads();
        }
        if (__builtin_amdgcn_readfirstlane(st.done)) return;
        const int cur = __builtin_amdgcn_readfirstlane(st.cur);
        op.src = cur ? a.buf1 : a.buf0;
        op.dst = cur ? a.buf0 : a.buf1;
        scale = st.scale;
    } else {
        op.src = a.buf0;
        op.dst = a.buf1;
        scale = a.norm_in ? 1.0 / *a.norm_in : a.x_scale;
    }
    op.scale = (CT)scale;
    op.vout = a.vout;
    op.plane = (size_t)a.H * a.W;
    op.pbytes = (uint32_t)(op.plane * sizeof(ST));
    double d1 = 0.0, d2 = 0.0;
    float wm = 0.f;  // product form: max |w| stored by this thread
    const int x0 = (tile % nbx) * TW, y0 = (tile / nbx) * TH;
    op.cut = x0 + TW > a.W;  // 4-wide epilogue loads read past the right edge here
    if (ODD) op.last = last_of_odd_frame(a.H, a.W, x0, y0, TH, TW);
    op.prev = !a.no_prev;
    if constexpr (PIPE == 3) {
        // space taps centred at 16 (the kernel's are centred at RS)
        __shared__ float tapl[2 * 16 + 1];
        if (threadIdx.x < 2 * 16 + 1) {
            float g = 0.f;
#pragma unroll
            for (int i = 0; i < 2 * RS + 1; ++i) g = (int)threadIdx.x == i + 16 - RS ? (float)a.taps.gs[i] : g;
            tapl[threadIdx.x] = g;
        }
        __syncthreads();
        constexpr bool YACC_OUT = sizeof(ST) == 4 || TW == 64;
        constexpr MfmaTail TAIL = sizeof(ST) == 4 ? TAIL_APART : !PF && TW == 64 ? TAIL_BY_LENGTH : TAIL_WHOLE;
        // staging multiplier umul = scale 2^S with |f x scale 2^S| < 2^10, output scale 2^-S
        float bound = __uint_as_float(a.state ? st.ubound : *a.ubound);
        if constexpr (PF) {
            const int e = bound_exponent(bound, PRODUCT_ELIM);
            const bool first = __builtin_amdgcn_readfirstlane(st.pform) == 2;
            const int cur = __builtin_amdgcn_readfirstlane(st.cur);
            FwdOpP<ST, ODD> pp;
            pp.f = a.f;
            pp.src = first ? a.f : op.src;
            pp.dst = op.dst;
            pp.gout = ldexpf(1.f, -2 * e);
            pp.ginv_out = ldexp(1.0, 2 * e);
            pp.ginv_in = first ? 1.0 : pp.ginv_out;
            pp.plane = op.plane;
            pp.pbytes = op.pbytes;
            pp.cut = x0 + TW > a.W;
            pp.prev = op.prev;
            pp.last = op.last;
            // staging power of two from the input's own maximum
            const float win = first ? bound : __uint_as_float(st.wmax[cur]);
            float umul;
            if constexpr (EXACT) {
                // the y-pass multiplies the staged bfloat16 w by ginv_in
                // 2^(10 - ein) (a power of two, folded into its taps); the scale
                // moves to the epilogue
                const int ein = bound_exponent((float)((double)win * pp.ginv_in), 100);
                pp.sg = (float)(scale * ldexp(1.0, ein - 10 - 2 * e));
                umul = (float)ldexp(pp.ginv_in, 10 - ein);
            } else {
                const int ein = bound_exponent((float)((double)win * scale * pp.ginv_in), 100);
                pp.sg = ldexpf(1.f, ein - 10 - 2 * e);
                umul = (float)(scale * ldexp(1.0, 10 - ein) * pp.ginv_in);
            }
            stencil_tile_mfma<CT, RT, TH, TW, NTHR, PAD, TAIL, YACC_OUT, EXACT>(
                pp, a.taps, tapl, umul, a.rs, a.T, t0, t1, a.H, a.W, x0, y0, lds, d1, d2);
            d1 *= pp.ginv_in * pp.ginv_out;
            d2 *= pp.ginv_out * pp.ginv_out;
            wm = pp.wmax;
        } else {
            if (!a.state) bound *= (float)fabs(scale);
            const int e = bound_exponent(bound, 100);
            const float umul = (float)(scale * ldexp(1.0, 10 - e));
            op.scale = ldexpf(1.f, e - 10);
            stencil_tile_mfma<CT, RT, TH, TW, NTHR, PAD, TAIL, YACC_OUT>(op, a.taps, tapl, umul, a.rs, a.T, t0, t1, a.H,
                                                                         a.W, x0, y0, lds, d1, d2);
        }
    } else if constexpr (PIPE == 4) {
        int t = t0;
        do
            stencil_tile_gather<CT, RS, RT, TH, TW, NTHR, RY>(op, a.taps, a.T, t, a.H, a.W, x0, y0, lds, d1, d2);
        while (ALT && ++t < t1);
    } else if constexpr (PIPE == 2)
        stencil_tile_flat<CT, RS, RT, TH, TW, NTHR, RY, QX>(op, a.taps, a.T, t0, t1, a.H, a.W, x0, y0, lds, d1, d2);
    else if constexpr (PIPE == 1)
        stencil_tile_pipe<CT, RS, RT, TH, TW, NTHR, RY, QX>(op, a.taps, a.T, t0, t1, a.H, a.W, x0, y0, lds, d1, d2);
    else
        stencil_tile<CT, RS, RT, TH, TW, NTHR, RY, QX>(op, a.taps, a.T, t0, t1, a.H, a.W, x0, y0, lds, d1, d2);
    block_reduce<NTHR>(d1, d2, wm, red);
    if (threadIdx.x == 0) {
        a.partials[2 * unit] = d1;
        a.partials[2 * unit + 1] = d2;
        if (PF) a.wpart[unit] = __float_as_uint(wm);
    }
}

template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX, int OCC, int PIPE, bool PF = false>
hipError_t launch_fwd(const FwdLaunch &L, hipStream_t stream) {
    using CT = typename Compute<ST>::type;
    FwdArgs<ST> a;
    a.f = (const ST *)L.f;
    a.buf0 = (ST *)L.buf0;
    a.buf1 = (ST *)L.buf1;
    a.state = L.state;
    a.state_out = L.state_out;
    a.prev_part = L.prev_part;
    if (!PF) a.prev_part.wmax = nullptr;
    a.partials = L.partials;
    a.wpart = L.wpart;
    a.no_prev = L.state && L.no_prev ? 1 : 0;
    a.x_scale = L.x_scale;
    a.norm_in = L.norm_in;
    a.vout = (ST *)L.vout;
    a.T = L.T;
    a.H = L.H;
    a.W = L.W;
    a.nseg = L.nseg > 0 ? L.nseg : 1;
    a.ubound = L.ubound;
    a.rs = 0;
    for (int d = 1; d <= 16; ++d)
        if (L.gs[16 + d] != 0.0) a.rs = d;
    if (PIPE == 3 && !L.ubound) return hipErrorInvalidValue;
    if (PF && (!L.state || L.vout || !L.wpart)) return hipErrorInvalidValue;
    if (L.state && L.state_out == L.state) return hipErrorInvalidValue;
    // L holds taps centred at index 16 (space) and 8 (time), zero beyond the
    // problem's radii; the kernel wants them centred at its compiled RS, RT.
    for (int i = 0; i < 2 * 16 + 1; ++i) a.taps.gs[i] = CT(0);
    for (int i = 0; i < 2 * 8 + 1; ++i) a.taps.gt[i] = CT(0);
    for (int d = -RS; d <= RS; ++d) a.taps.gs[d + RS] = (CT)L.gs[d + 16];
    for (int d = -RT; d <= RT; ++d) a.taps.gt[d + RT] = (CT)L.gt[d + 8];
    const int nunits = ((L.W + TW - 1) / TW) * ((L.H + TH - 1) / TH) * a.nseg;
    const int per = (nunits + NUM_XCD - 1) / NUM_XCD;
    if constexpr (odd_frames_apart<ST, QX, PIPE>() || PIPE == 4) {
        if (PIPE == 4 ? a.nseg < L.T : (L.H & L.W & 1) != 0) {
            hipLaunchKernelGGL((fwd_step_kernel<ST, RS, RT, TH, TW, NTHR, RY, QX, OCC, PIPE, PF, true>),
                               dim3(per * NUM_XCD), dim3(NTHR), 0, stream, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((fwd_step_kernel<ST, RS, RT, TH, TW, NTHR, RY, QX, OCC, PIPE, PF, false>), dim3(per * NUM_XCD),
                       dim3(NTHR), 0, stream, a);
    return hipGetLastError();
}

// Matrix-core variants report the occupancy of their product-form kernel,
// the one an iteration chain runs (with bfloat16 storage it stages a single
// half plane and may fit more workgroups per CU than the plain step).
template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX, int OCC, int PIPE>
int fwd_blocks_per_cu() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, fwd_step_kernel<ST, RS, RT, TH, TW, NTHR, RY, QX, OCC, PIPE, PIPE == 3, false>, NTHR, 0) != hipSuccess)
        n = 1;
    return n > 0 ? n : 1;
}

// The product-form launcher of a variant (matrix-core variants only).
template <class ST, int RS, int RT, int TH, int TW, int NTHR, int RY, int QX, int OCC, int PIPE>
constexpr FwdLaunchFn product_launcher() {
    if constexpr (PIPE == 3)
        return &launch_fwd<ST, RS, RT, TH, TW, NTHR, RY, QX, OCC, PIPE, true>;
    else
        return nullptr;
}

}  // namespace stpi
