// Shared device-side types for the stpi kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace stpi {

// bfloat16 storage: the upper 16 bits of an IEEE binary32 value.
struct bf16 {
    uint16_t bits;
};

__device__ __forceinline__ float ld(const float *p) { return *p; }
__device__ __forceinline__ double ld(const double *p) { return *p; }
__device__ __forceinline__ float ld(const bf16 *p) {
    return __uint_as_float(((uint32_t)p->bits) << 16);
}

// Round-to-nearest-even float -> bfloat16 (NaN stays NaN): the hardware
// conversion, one instruction per pair.
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
__device__ __forceinline__ uint32_t f32x2_to_bf16x2_bits(float a, float b) {
    typedef float f2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    const f2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2_t));
}

__device__ __forceinline__ void st(float *p, float v) { *p = v; }
__device__ __forceinline__ void st(double *p, double v) { *p = v; }
__device__ __forceinline__ void st(bf16 *p, float v) { p->bits = f32_to_bf16_bits(v); }

// The value a store of v would leave in memory, read back in compute precision.
__device__ __forceinline__ float stored_value(const float *, float v) { return v; }
__device__ __forceinline__ double stored_value(const double *, double v) { return v; }
__device__ __forceinline__ float stored_value(const bf16 *, float v) {
    return __uint_as_float(((uint32_t)f32_to_bf16_bits(v)) << 16);
}

// Compute type for a storage type.
template <class ST> struct Compute { using type = float; };
template <> struct Compute<double> { using type = double; };

// Iteration state kept in device memory so that a whole iteration chain runs
// without host round trips. The stored iterate is unnormalised; the unit
// iterate is scale * stored.
struct DevState {
    double scale;      // 1 / ||stored iterate||
    double residual;   // ||x_k - x_{k-1}|| of the last step
    double lambda;     // ||A x_{k-1}||
    double rayleigh;   // <x_{k-1}, A x_{k-1}>
    double tol;        // <= 0: run a fixed number of steps
    int32_t iters;     // applications of A done
    int32_t done;      // 1: converged or stopped, further steps are no-ops
    int32_t cur;       // 0: iterate lives in buffer 0 (the caller's x), 1: in buffer 1
    uint32_t flags;    // bit 0 zero norm, bit 1 non-finite
    int32_t max_iters;
    int32_t converged;
    uint32_t ubound;   // float bits of max |f| (matrix-core step variants)
    double first_res[2];  // residuals after the chain's first and second steps
    int32_t check_rise;   // 1: stop after the second step if its residual is above the first's
    // 0: the buffers hold the iterate itself. Product form (matrix-core chain
    // steps): 1: the current buffer holds w = f x g (see FwdOpP), 2: uniform
    // start, no step taken yet (the iterate is the constant 1, w = f itself).
    int32_t pform;
    // Product form: float bits of max |w| over buffer 0 / buffer 1, set for
    // the buffer a step wrote by that step's finalisation.
    uint32_t wmax[2];
    // Batched chains, plain form: 1 after a rejected warm start until the
    // clip's buffer has been refilled with the uniform start.
    int32_t refill;
    // Single-clip chains: 1 while the last step's finalisation is still to be
    // formed from its partial sums (see resolve_state).
    int32_t pending;
};

static_assert(sizeof(DevState) <= 256, "the iteration state lives in a 256-byte workspace slot");

constexpr uint32_t FLAG_ZERO = 1u;
constexpr uint32_t FLAG_NONFINITE = 2u;
constexpr uint32_t FLAG_ROSE = 4u;  // the check_rise rule fired (not an error): single clip stops, batched clip restarts

// Exponent e of a bound (bound < 2^e, from frexp), clamped to [-lim, lim];
// 0 for a zero or non-finite bound.
__device__ __forceinline__ int bound_exponent(float bound, int lim) {
    int e = 0;
    if (bound > 0.f && bound <= 3.0e38f) (void)frexpf(bound, &e);
    return e < -lim ? -lim : (e > lim ? lim : e);
}
// Product-form chains keep 2^(+-2e) normal floats.
constexpr int PRODUCT_ELIM = 60;

constexpr uint32_t FLAG_AFFINITY = 16u;  // full operator: a Taylor affinity could be negative (see sfseg.hip)

// Workgroup size and summation order of the per-step reduction of partial
// sums: thread i < FINAL_THREADS adds entries i, i + FINAL_THREADS, ... in
// turn, then the workgroup tree of block_sum.
constexpr int FINAL_THREADS = 256;

// Step finalisation from the reduced sums P1 = sum z * x_stored and
// P2 = sum z^2: n = ||z||, x_{k+1} = z / n (Eq. 8), cos = <x_{k+1}, x_k> =
// scale * P1 / n, residual = sqrt(2 - 2 cos), and the stopping rules.
// wm: float bits of max |w| of the buffer the step wrote (product form).
__device__ __forceinline__ void step_finalize(DevState *s, double p1, double p2, uint32_t wm = 0u) {
    const double scale = s->scale;
    const double nz = sqrt(p2);
    if (!isfinite(nz) || !isfinite(p1)) {
        s->flags |= FLAG_NONFINITE;
        s->done = 1;
        return;
    }
    if (nz == 0.0) {
        s->flags |= FLAG_ZERO;
        s->done = 1;
        return;
    }
    const double c = scale * p1 / nz;
    s->rayleigh = scale * p1;
    s->lambda = nz;
    s->residual = sqrt(fmax(0.0, 2.0 - 2.0 * c));
    s->scale = 1.0 / nz;
    s->cur ^= 1;
    s->wmax[s->cur] = wm;
    s->iters += 1;
    if (s->pform == 2) s->pform = 1;
    if (s->iters <= 2) s->first_res[s->iters - 1] = s->residual;
    if (s->check_rise && s->iters == 2 && !(s->first_res[1] <= s->first_res[0])) {
        s->flags |= FLAG_ROSE;
        s->done = 1;
        return;
    }
    if (s->tol > 0.0 && s->residual < s->tol) {
        s->converged = 1;
        s->done = 1;
    }
    if (s->iters >= s->max_iters) s->done = 1;
}

// Sum of a double over a workgroup (fixed shuffle/LDS tree: deterministic).
template <int NTHR>
__device__ __forceinline__ double block_sum(double v, double *lds) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    constexpr int NW = NTHR / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NW; ++i) s += lds[i];
    }
    return s;  // valid in thread 0 only
}

// Maximum of a non-negative float over a workgroup (valid in thread 0).
template <int NTHR>
__device__ __forceinline__ float block_max(float v, float *lds) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    constexpr int NW = NTHR / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    float m = 0.f;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NW; ++i) m = fmaxf(m, lds[i]);
    }
    return m;
}

// Partial results of a step's workgroups: [n][2] sums, [n] float bits of max |w|.
struct StepPartials {
    double *sums;
    uint32_t *wmax;
};

// The sums of n workgroups' partial pairs, and the largest of their maxima, in
// the order of one FINAL_THREADS workgroup (thread i adds entries i, i +
// FINAL_THREADS, ..., then the tree of block_sum) whatever NTHR is. Valid in
// thread 0. sh: 3 * FINAL_THREADS / 64 doubles.
template <int NTHR>
__device__ __forceinline__ void sum_partials(const double *sums, const uint32_t *wmax, int n, double *sh, double &p1,
                                             double &p2, uint32_t &wm) {
    constexpr int NW = FINAL_THREADS / 64;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v0 = 0; v0 < FINAL_THREADS; v0 += NTHR) {
        const int v = v0 + (int)threadIdx.x;
        if (v < FINAL_THREADS) {  // whole wavefronts
            double a = 0.0, b = 0.0;
            uint32_t m = 0u;
            for (int i = v; i < n; i += FINAL_THREADS) {
                a += sums[2 * i];
                b += sums[2 * i + 1];
                const uint32_t w = wmax ? wmax[i] : 0u;
                m = w > m ? w : m;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                a += __shfl_xor(a, off, 64);
                b += __shfl_xor(b, off, 64);
                const uint32_t w = (uint32_t)__shfl_xor((int)m, off, 64);
                m = w > m ? w : m;
            }
            if (lane == 0) {
                sh[v >> 6] = a;
                sh[NW + (v >> 6)] = b;
                sh[2 * NW + (v >> 6)] = (double)m;  // exact
            }
        }
    }
    __syncthreads();
    p1 = p2 = 0.0;
    wm = 0u;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            p1 += sh[i];
            p2 += sh[NW + i];
            const uint32_t w = (uint32_t)sh[2 * NW + i];
            wm = w > wm ? w : wm;
        }
    }
}

// The chain's state as a launch finds it. A step does not finalise itself: its
// workgroups leave partial sums, and every workgroup of the next launch (the
// next step, or the final pass) forms the finalisation from them for itself, at
// its start, all with the same result; workgroup 0 writes it to the other
// state slot for the launch after. So a step needs no counter that its
// workgroups raise one after the other (16 ns each: 14 us for 840), no last
// workgroup that polls for the others' sums, and no launch of its own. `in` and `out` are
// different slots, as the launch's own partials are another set than the ones
// read here. After the call *st holds the state (LDS); pend is the value of
// its `pending` written to `out` (the launch leaves partial sums itself).
template <int NTHR>
__device__ __forceinline__ void resolve_state(const DevState *in, StepPartials part, int n, DevState *st, double *sh,
                                              DevState *out, int pend) {
    constexpr int NWORD = (int)(sizeof(DevState) / 4);
    static_assert(NWORD <= 64 && NTHR >= 64, "one wavefront copies the state");
    if (threadIdx.x < NWORD) reinterpret_cast<uint32_t *>(st)[threadIdx.x] = reinterpret_cast<const uint32_t *>(in)[threadIdx.x];
    double p1, p2;
    uint32_t wm;
    sum_partials<NTHR>(part.sums, part.wmax, n, sh, p1, p2, wm);
    if (threadIdx.x == 0) {
        if (st->pending) {
            st->pending = 0;
            if (!st->done) step_finalize(st, p1, p2, wm);
        }
        if (out && blockIdx.x == 0) {
            *out = *st;
            out->pending = pend && !st->done ? 1 : 0;
        }
    }
    __syncthreads();
}

// Sums of two values and the maximum of a third over a workgroup, valid in
// thread 0 (the order of block_sum). sh: 3 * NTHR / 64 doubles.
template <int NTHR>
__device__ __forceinline__ void block_reduce(double &a, double &b, float &m, double *sh) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
        m = fmaxf(m, __shfl_xor(m, off, 64));
    }
    constexpr int NW = NTHR / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) {
        sh[wid] = a;
        sh[NW + wid] = b;
        sh[2 * NW + wid] = (double)m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a = b = 0.0;
        m = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            a += sh[i];
            b += sh[NW + i];
            m = fmaxf(m, (float)sh[2 * NW + i]);
        }
    }
}

}  // namespace stpi
