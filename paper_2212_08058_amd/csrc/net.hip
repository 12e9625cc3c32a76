// Warm-start network: four 'same' 3x3x3 convolutions (1 -> 16 -> 16 -> 16 -> 1
// channels, zero padding, bias, ReLU between layers) mapping the feature
// volume f to a start vector for the power iteration.
//
// Weights and activations are bfloat16, accumulation is FP32. Hidden
// activations are stored channels-last ([voxel][16], 32 bytes per voxel).
// All layers and their gradients run on the matrix cores: the two 16 -> 16
// layers as implicit GEMMs (conv16_kernel: per wavefront a 16-channel x 16-voxel
// output block accumulates 27 taps of (16 out x 16 in) weights times (16 in x 16
// voxels) inputs, one tap an instruction in the forward pass, two in the input
// gradient); their weight gradients as sums over voxels of 16 x 16 outer products
// per tap, 32 voxels an instruction (wgrad16_kernel); the one-channel layers with
// their 27 taps as the K dimension or as output rows (one_channel_kernel,
// conv_out_kernel, wgrad1_kernel).
//
// Parameter layout (FP32 masters, PyTorch conv3d order [Cout][Cin][3][3][3]):
//   w1[16][1][27] b1[16] w2[16][16][27] b2[16] w3[16][16][27] b3[16] w4[1][16][27] b4[1]
#include <hip/hip_runtime.h>

#include <algorithm>

#include <cmath>
#include <cstring>

#include "../../include/stpi.h"
#include "common.hpp"
#include "host_internal.hpp"

namespace stpi {

namespace net {

constexpr int C = 16;
constexpr int NT = 27;
constexpr int OFF_W1 = 0, OFF_B1 = 432, OFF_W2 = 448, OFF_B2 = 448 + 6912, OFF_W3 = OFF_B2 + 16,
              OFF_B3 = OFF_W3 + 6912, OFF_W4 = OFF_B3 + 16, OFF_B4 = OFF_W4 + 432, NPARAM = OFF_B4 + 1;
static_assert(NPARAM == 14737, "parameter count");

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Prepared weights (device): float copies, rounded to bfloat16 values, for the
// one-channel layers and the per-lane MFMA operand blocks of the 16 -> 16 layers,
// forward and transposed/flipped (input gradient).
struct Prep {
    float w1[C][NT];       // [co][tap]
    float b1[C];
    bf16x4 a2[NT][64];     // forward A operand of layer 2: lane l -> W2[co=l%16][ci=4(l/16)+j][tap]
    bf16x4 a2d[NT][64];    // input-gradient A operand:     lane l -> W2[co=4(l/16)+j][ci=l%16][26-tap]
    float b2[C];
    bf16x4 a3[NT][64];
    bf16x4 a3d[NT][64];
    float b3[C];
    float w4[C][NT];       // [ci][tap]
    float b4;
};

__device__ __forceinline__ float bfr(float v) { return __uint_as_float(((uint32_t)f32_to_bf16_bits(v)) << 16); }
__device__ __forceinline__ short bfbits(float v) { return (short)f32_to_bf16_bits(v); }
__device__ __forceinline__ float bf2f(short b) { return __uint_as_float(((uint32_t)(uint16_t)b) << 16); }

__global__ void prepare_kernel(const float *m, Prep *p) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int nth = gridDim.x * blockDim.x;
    for (int i = tid; i < C * NT; i += nth) {
        const int co = i / NT, tap = i % NT;
        p->w1[co][tap] = bfr(m[OFF_W1 + i]);
        p->w4[co][tap] = bfr(m[OFF_W4 + i]);  // w4[0][ci=co][tap]
    }
    for (int i = tid; i < NT * 64; i += nth) {
        const int tap = i / 64, l = i % 64;
        bf16x4 f2, d2, f3, d3;
        for (int j = 0; j < 4; ++j) {
            const int co = l % 16, ci = 4 * (l / 16) + j;          // forward
            f2[j] = bfbits(m[OFF_W2 + (co * C + ci) * NT + tap]);
            f3[j] = bfbits(m[OFF_W3 + (co * C + ci) * NT + tap]);
            const int co2 = 4 * (l / 16) + j, ci2 = l % 16;        // transposed, flipped
            d2[j] = bfbits(m[OFF_W2 + (co2 * C + ci2) * NT + (NT - 1 - tap)]);
            d3[j] = bfbits(m[OFF_W3 + (co2 * C + ci2) * NT + (NT - 1 - tap)]);
        }
        p->a2[tap][l] = f2;
        p->a2d[tap][l] = d2;
        p->a3[tap][l] = f3;
        p->a3d[tap][l] = d3;
    }
    if (tid < C) {
        p->b1[tid] = m[OFF_B1 + tid];
        p->b2[tid] = m[OFF_B2 + tid];
        p->b3[tid] = m[OFF_B3 + tid];
    }
    if (tid == 0) p->b4 = m[OFF_B4];
}

struct Dims {
    int T, H, W;
};

// Work unit of a workgroup: consecutive units share an XCD (workgroups are
// dealt round-robin over the 8 XCDs), so neighbours find each other's rows in
// the same L2. -1 for workgroups past the last unit.
constexpr int XCDS = 8;
__device__ __forceinline__ int net_unit(int block, int n) {
    const int per = (n + XCDS - 1) / XCDS;
    const int u = (block % XCDS) * per + block / XCDS;
    return u < n ? u : -1;
}
inline int net_grid(int n) { return (n + XCDS - 1) / XCDS * XCDS; }

// Raw buffer loads over a channels-last activation volume: an out-of-range
// byte offset reads 0, so the loads of the zero padding need no branch (and
// the compiler no full memory wait where branches join). The host limits
// activation volumes to 2^31 bytes.
constexpr uint32_t OOB_OFF = 0xFFFFFFF0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t act_rsrc(const short *base, const Dims &d) {
    const int bytes = (int)((size_t)d.T * d.H * d.W * C * sizeof(short));
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<short *>(base), (short)0, bytes, 0x00020000);
}
__device__ __forceinline__ short load_b16(__amdgpu_buffer_rsrc_t r, uint32_t boff) {
    return (short)__builtin_amdgcn_raw_buffer_load_b16(r, boff, 0, 0);
}

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));

// A 16 x 16 accumulator and its products, of one K for its whole life. A product
// that follows one of another K on the same accumulator has to come 4 wait
// states later: with 0 to 3 between them, half of the sums lacked the earlier
// product (v_mfma_f32_16x16x16_bf16 and v_mfma_f32_16x16x32_bf16, in either
// order, small integers; with 4 or more all were right), and the compiler (clang
// 22 of ROCm 7.2.0) puts none. The build's device-code check looks for such pairs.
template <int K>
struct Acc {
    static_assert(K == 16 || K == 32, "bfloat16 products of 16 x 16 outputs");
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    __device__ __forceinline__ void add(const bf16x4 &a, const bf16x4 &b) {
        static_assert(K == 16, "operands of a K = 16 product");
        v = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, v, 0, 0, 0);
    }
    __device__ __forceinline__ void add(const bf16v8 &a, const bf16v8 &b) {
        static_assert(K == 32, "operands of a K = 32 product");
        v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, v, 0, 0, 0);
    }
};

// The exact split of a float into three bfloat16 parts: each part is the rest
// rounded to bfloat16. A finite value that rounds past the largest bfloat16
// takes that as its first part; an infinite one is its own first part, with
// nothing left.
constexpr float SPLIT_CARE = 0x1.ffp127f;
__device__ __forceinline__ short first_part(float v) {
    const short b = bfbits(v);
    const bool over = fabsf(v) >= SPLIT_CARE && fabsf(v) < INFINITY;
    return over ? (short)(b - 1) : b;
}
__device__ __forceinline__ float split_rest(float v, float part) { return fabsf(v) == INFINITY ? 0.f : v - part; }

// Tile of the layer kernels that stream a tile's frames: CT_H x CT_W voxels,
// staged with the one-voxel rim their taps reach. A unit is a range of frames
// of one tile ("segment"); neighbouring tiles of a segment share an XCD.
constexpr int CT_H = 16, CT_W = 32, CT_C = CT_W + 2, CT_V = (CT_H + 2) * CT_C;
struct TileUnit {
    int x0, y0, t0, t1;
};
__device__ __forceinline__ bool tile_unit(const Dims &d, int nseg, TileUnit &u) {
    const int nbx = (d.W + CT_W - 1) / CT_W, ntiles = nbx * ((d.H + CT_H - 1) / CT_H);
    const int k = net_unit(blockIdx.x, ntiles * nseg);
    if (k < 0) return false;
    const int tile = k % ntiles, seg = k / ntiles;
    u.x0 = (tile % nbx) * CT_W;
    u.y0 = (tile / nbx) * CT_H;
    u.t0 = (int)((int64_t)seg * d.T / nseg);
    u.t1 = (int)((int64_t)(seg + 1) * d.T / nseg);
    return true;
}
// One frame of a channels-last volume (an empty range outside the clip: loads return 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frame_rsrc(const short *base, const Dims &d, int t) {
    const bool ok = t >= 0 && t < d.T;
    const size_t plane = (size_t)d.H * d.W * C;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<short *>(base + (ok ? t : 0) * plane), (short)0,
                                             ok ? (int)(plane * sizeof(short)) : 0, 0x00020000);
}

// The layers with one input channel. MODE 0: layer 1, act = relu(conv(f) + b1),
// f rounded to bfloat16. MODE 1: the input gradient of layer 4 masked by layer
// 3's ReLU, g3[v][ci] = (act3[v][ci] > 0) sum_tap w4[ci][tap] g_y[v - off(tap)],
// g_y in float: split exactly into three bfloat16 parts, one product each.
// One v_mfma_f32_16x16x32_bf16 per 16 voxels of a row: A = weights [channel]
// [tap] with the 27 taps padded to K = 32 (lane l holds channel l % 16, taps
// 8 (l / 16) .. + 7), B = the voxels' 27 neighbours in the same order. A
// workgroup streams the frames of a tile as the 16 -> 16 layers do; a staged
// element is the pair (f[x], f[x + 1]), so any two neighbours of a row are one
// aligned 4-byte read, and a lane's 8 taps (8 consecutive of the row triples
// in tap order) are four such pairs, some made of two reads by a byte permute.
// Bound by the 32 bytes a voxel written. The gathers they replace (8 element
// loads per lane and 16 voxels; a scalar sum of 27 x 16 terms per voxel) took
// 296 us at 32x480x854 (layer 1) and 127 us at 16x240x432 (the gradient; layer
// 1 there 46); these take 121 and 42 us (20).
template <int MODE>
__global__ __launch_bounds__(256) void one_channel_kernel(Dims d, const float *f, const Prep *p, const short *mask,
                                                          short *out, int nseg) {
    constexpr int PARTS = MODE == 0 ? 1 : 3;
    __shared__ uint32_t lds[4 * PARTS * CT_V];  // [frame ring 4][part][row][column]
    TileUnit u;
    if (!tile_unit(d, nseg, u)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane % 16, kq = lane / 16;
    bf16x8 aw;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int tap = 8 * kq + j;  // MODE 1 reads v - off(tap) = v + off(26 - tap)
        const float w = tap >= NT ? 0.f : (MODE == 0 ? p->w1[n][tap] : p->w4[n][NT - 1 - tap]);
        aw[j] = bfbits(w);  // the prepared weights are already bfloat16 values
    }
    float bv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bv[j] = MODE == 0 ? p->b1[4 * kq + j] : 0.f;
    // This lane's taps 8 kq .. + 7 as four pairs: pair i is (element a) alone, or
    // the low halves of elements a and b. An element is named by its row R =
    // 3 (dt + 1) + (dy + 1) and its column offset from the voxel's left neighbour.
    constexpr uint32_t WHOLE = 0x03020100u, LOWS = 0x05040100u, LOW0 = 0x0c0c0100u, ZERO = 0x0c0c0c0cu;
    constexpr int RA[4][4] = {{0, 0, 1, 2}, {2, 3, 4, 4}, {5, 6, 6, 7}, {8, 8, 8, 8}};
    constexpr int CA[4][4] = {{0, 2, 1, 0}, {2, 1, 0, 2}, {1, 0, 2, 1}, {0, 2, 0, 0}};
    constexpr int RB[4][4] = {{0, 1, 1, 2}, {3, 3, 4, 5}, {5, 6, 7, 7}, {8, 8, 8, 8}};  // column offset 0
    constexpr uint32_t SEL[4][4] = {{WHOLE, LOWS, WHOLE, WHOLE},
                                    {LOWS, WHOLE, WHOLE, LOWS},
                                    {WHOLE, WHOLE, LOWS, WHOLE},
                                    {WHOLE, LOW0, ZERO, ZERO}};
    const int r0 = 8 * (wid >> 1), c0 = 16 * (wid & 1);
    int fa[4], fb[4], oa[4], ob[4];
    uint32_t sel[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int ra = 0, ca = 0, rb = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (kq == q) {
                ra = RA[q][i];
                ca = CA[q][i];
                rb = RB[q][i];
                sel[i] = SEL[q][i];
            }
        fa[i] = ra / 3;
        oa[i] = (r0 + ra % 3) * CT_C + c0 + n + ca;
        fb[i] = rb / 3;
        ob[i] = (r0 + rb % 3) * CT_C + c0 + n;
    }
    constexpr int NST = (CT_V + 255) / 256;
    uint32_t s0[NST], s1[NST];  // byte offsets of f[x], f[x + 1] in a frame
#pragma unroll
    for (int m = 0; m < NST; ++m) {
        const int v = tid + 256 * m, gy = u.y0 - 1 + v / CT_C, gx = u.x0 - 1 + v % CT_C;
        const bool ok = v < CT_V && (unsigned)gy < (unsigned)d.H;
        s0[m] = ok && (unsigned)gx < (unsigned)d.W ? (uint32_t)(gy * d.W + gx) * 4 : OOB_OFF;
        s1[m] = ok && (unsigned)(gx + 1) < (unsigned)d.W ? (uint32_t)(gy * d.W + gx + 1) * 4 : OOB_OFF;
    }
    float e0[3][NST], e1[3][NST];  // up to three frames' loads in flight
    auto fetch = [&](int t, int slot) __attribute__((always_inline)) {
        const bool ok = t >= 0 && t < d.T;
        const size_t plane = (size_t)d.H * d.W;
        const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(f + (ok ? t : 0) * plane), (short)0,
                                                         ok ? (int)(plane * sizeof(float)) : 0, 0x00020000);
#pragma unroll
        for (int m = 0; m < NST; ++m) {
            e0[slot][m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, s0[m], 0, 0));
            e1[slot][m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, s1[m], 0, 0));
        }
    };
    auto stage = [&](int t, int slot) __attribute__((always_inline)) {
        uint32_t *q = lds + (t & 3) * PARTS * CT_V;
#pragma unroll
        for (int m = 0; m < NST; ++m) {
            const int v = tid + 256 * m;
            if (CT_V % 256 == 0 || m < NST - 1 || v < CT_V) {
                float a = e0[slot][m], b = e1[slot][m];
#pragma unroll
                for (int k = 0; k < PARTS; ++k) {
                    uint32_t h = f32x2_to_bf16x2_bits(a, b);
                    if (PARTS > 1 && k == 0 && fmaxf(fabsf(a), fabsf(b)) >= SPLIT_CARE)
                        h = (uint32_t)(uint16_t)first_part(a) | (uint32_t)(uint16_t)first_part(b) << 16;
                    q[k * CT_V + v] = h;
                    a = split_rest(a, __uint_as_float(h << 16));
                    b = split_rest(b, __uint_as_float(h & 0xffff0000u));
                }
            }
        }
    };
    const int x = u.x0 + c0 + n;
#pragma unroll
    for (int k = 0; k < 3; ++k) fetch(u.t0 - 1 + k, k);
#pragma unroll
    for (int k = 0; k < 3; ++k) stage(u.t0 - 1 + k, k);
    __syncthreads();
    for (int t = u.t0; t < u.t1; ++t) {
        const bool more = t + 1 < u.t1;
        if (more) fetch(t + 2, 0);
        bf16x4 mk[MODE == 0 ? 1 : 8];  // the mask of the step's outputs, in flight beside the products
        if constexpr (MODE == 1) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int y = u.y0 + r0 + r;
                mk[r] = bf16x4{0, 0, 0, 0};
                if (y < d.H && x < d.W)
                    mk[r] = *reinterpret_cast<const bf16x4 *>(mask + (((size_t)t * d.H + y) * d.W + x) * C + 4 * kq);
            }
        }
        const uint32_t *qa[4], *qb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            qa[i] = lds + ((t - 1 + fa[i]) & 3) * PARTS * CT_V + oa[i];
            qb[i] = lds + ((t - 1 + fb[i]) & 3) * PARTS * CT_V + ob[i];
        }
        Acc<32> acc[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
#pragma unroll
            for (int k = PARTS - 1; k >= 0; --k) {  // smallest part first
                uint4 b;
                const int at = k * CT_V + r * CT_C;
                b.x = __builtin_amdgcn_perm(qb[0][at], qa[0][at], sel[0]);
                b.y = __builtin_amdgcn_perm(qb[1][at], qa[1][at], sel[1]);
                b.z = __builtin_amdgcn_perm(qb[2][at], qa[2][at], sel[2]);
                b.w = __builtin_amdgcn_perm(qb[3][at], qa[3][at], sel[3]);
                acc[r].add(__builtin_bit_cast(bf16v8, aw), __builtin_bit_cast(bf16v8, b));
            }
        }
        // lane holds out[channel 4 kq + j][column n] of each row
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int y = u.y0 + r0 + r;
            if (y >= d.H || x >= d.W) continue;
            const size_t v = ((size_t)t * d.H + y) * d.W + x;
            bf16x4 o;
            if (MODE == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = bfbits(fmaxf(acc[r].v[j] + bv[j], 0.0f));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = bf2f(mk[r][j]) > 0.0f ? bfbits(acc[r].v[j]) : (short)0;
            }
            *reinterpret_cast<bf16x4 *>(out + v * C + 4 * kq) = o;
        }
        if (more) stage(t + 2, 0);
        __syncthreads();
    }
}

// 16 -> 16 convolution on the matrix cores. MODE 0: out = relu(conv + bias);
// MODE 1 (input gradient of a ReLU layer): out = conv(g, flipped W^T) masked
// by mask > 0. A workgroup streams the frames of a CT_H x CT_W tile through a
// ring of four staged frames (the rim included; the frame after the next is
// loaded while one is computed, one barrier per frame). In LDS the two channel
// halves of a voxel lie in planes of their own, so what a lane reads is next to
// its neighbours'. Each wavefront owns 8 rows x 16 columns; a staged fragment
// feeds up to three output rows, and the weights stay in registers.
// MODE 0 takes one tap an instruction (v_mfma_f32_16x16x16_bf16) in the taps'
// order: its results are rounded to bfloat16 and feed three further layers, so
// the order of its float sums is part of the network's arithmetic. MODE 1
// takes two taps an instruction (K = 32): the nine (frame, x) taps of an input
// row make four pairs and one single, whose upper half is zero in both
// operands (no product of another K is mixed in: see Acc).
// Bound by memory (32 bytes a voxel read, 1.2 times with the rims, and 32
// written) beside the matrix cores. The form it replaces (a wavefront per 16 x
// 4 voxels, every row loaded from memory three times and shifted by lane
// moves) took 502 us at 32x480x854 and 64 (MODE 0) and 67 us (MODE 1) at
// 16x240x432; this takes 302, 44 and 42 us.
constexpr int CV_PLANE = CT_V * 8;     // halves of one channel half of a staged frame
constexpr int CV_FRAME = 2 * CV_PLANE;
constexpr int CV_ROWS = 8;             // output rows per wavefront

template <int MODE>
__global__ __launch_bounds__(256, MODE == 0 ? 4 : 2) void conv16_kernel(Dims d, const short *in, const bf16x4 (*A)[64],
                                                        const float *bias, const short *mask, short *out, int nseg) {
    __shared__ __align__(16) short lds[4 * CV_FRAME];
    TileUnit u;
    if (!tile_unit(d, nseg, u)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane % 16, kq = lane / 16;
    // MODE 0: tap operands as prepared (channels 4 kq .. + 3 of one tap).
    // MODE 1: tap order of an input row q = 3 (dt + 1) + (dx + 1). Pair p holds
    // taps 2 p (lanes kq 0, 1) and 2 p + 1 (kq 2, 3), channels 8 (kq % 2) .. + 7;
    // pair 4 is the single q = 8 (kq 0, 1).
    constexpr bool PAIR = MODE == 1;
    const bool lower = kq < 2;
    bf16x4 a1[PAIR ? 1 : NT];
    bf16v8 ap[3][5];
    if constexpr (PAIR) {
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int p = 0; p < 5; ++p) {
                const int q = p < 4 ? 2 * p + kq / 2 : 8, tap = (q / 3) * 9 + dy * 3 + q % 3;
                union {
                    bf16x4 h[2];
                    bf16v8 v;
                } w;
                w.h[0] = A[tap][n + 32 * (kq % 2)];
                w.h[1] = A[tap][n + 32 * (kq % 2) + 16];
                if (p == 4 && !lower) w.h[0] = w.h[1] = bf16x4{0, 0, 0, 0};
                ap[dy][p] = w.v;
            }
    } else {
#pragma unroll
        for (int tap = 0; tap < NT; ++tap) a1[tap] = A[tap][lane];
    }
    float bv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bv[j] = MODE == 0 ? bias[4 * kq + j] : 0.f;
    // staging: item it = 16 bytes (voxel it / 2 of the rimmed tile, channel half it % 2)
    constexpr int NIT = 2 * CT_V, NST = (NIT + 255) / 256;
    uint32_t soff[NST];
#pragma unroll
    for (int m = 0; m < NST; ++m) {
        const int it = tid + 256 * m, v = it >> 1;
        const int gy = u.y0 - 1 + v / CT_C, gx = u.x0 - 1 + v % CT_C;
        const bool ok = it < NIT && (unsigned)gy < (unsigned)d.H && (unsigned)gx < (unsigned)d.W;
        soff[m] = ok ? (uint32_t)(gy * d.W + gx) * (C * 2) + 16 * (it & 1) : OOB_OFF;
    }
    uint4 st[3][NST];  // up to three frames' loads in flight
    auto fetch = [&](int t, int slot) __attribute__((always_inline)) {
        const auto r = frame_rsrc(in, d, t);
#pragma unroll
        for (int m = 0; m < NST; ++m) st[slot][m] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, soff[m], 0, 0));
    };
    auto stage = [&](int t, int slot) __attribute__((always_inline)) {
        short *f = lds + (t & 3) * CV_FRAME;
#pragma unroll
        for (int m = 0; m < NST; ++m) {
            const int it = tid + 256 * m;
            if (NIT % 256 == 0 || m < NST - 1 || it < NIT)
                *reinterpret_cast<uint4 *>(f + (it & 1) * CV_PLANE + (it >> 1) * 8) = st[slot][m];
        }
    };
    const int r0 = CV_ROWS * (wid >> 1), c0 = 16 * (wid & 1);  // the wavefront's rows and columns of the tile
    // fragment addresses within a staged frame, row r0 - 1 of the tile (pairs: by this lane's tap)
    int poff[5], pdt[5];
#pragma unroll
    for (int p = 0; p < 5; ++p) {
        const int q = p < 4 ? 2 * p + kq / 2 : 8;
        pdt[p] = q / 3;
        poff[p] = (kq % 2) * CV_PLANE + (r0 * CT_C + c0 + n + q % 3) * 8;
    }
    const int off1 = (kq / 2) * CV_PLANE + (r0 * CT_C + c0 + n) * 8 + 4 * (kq % 2);
    const int x = u.x0 + c0 + n;
#pragma unroll
    for (int k = 0; k < 3; ++k) fetch(u.t0 - 1 + k, k);
#pragma unroll
    for (int k = 0; k < 3; ++k) stage(u.t0 - 1 + k, k);
    __syncthreads();
    for (int t = u.t0; t < u.t1; ++t) {
        const bool more = t + 1 < u.t1;
        if (more) fetch(t + 2, 0);
        bf16x4 mk[MODE == 0 ? 1 : CV_ROWS];  // the mask of the step's outputs, in flight beside the products
        if constexpr (MODE == 1) {
#pragma unroll
            for (int r = 0; r < CV_ROWS; ++r) {
                const int y = u.y0 + r0 + r;
                mk[r] = bf16x4{0, 0, 0, 0};
                if (y < d.H && x < d.W)
                    mk[r] = *reinterpret_cast<const bf16x4 *>(mask + (((size_t)t * d.H + y) * d.W + x) * C + 4 * kq);
            }
        }
        Acc<PAIR ? 32 : 16> acc[CV_ROWS];
        if constexpr (PAIR) {
            const short *pp[5];
#pragma unroll
            for (int p = 0; p < 5; ++p) pp[p] = lds + ((t - 1 + pdt[p]) & 3) * CV_FRAME + poff[p];
#pragma unroll
            for (int ry = 0; ry < CV_ROWS + 2; ++ry) {  // input row r0 - 1 + ry of the tile
                bf16v8 b[5];
#pragma unroll
                for (int p = 0; p < 5; ++p) {
                    uint4 w = *reinterpret_cast<const uint4 *>(pp[p] + ry * CT_C * 8);
                    if (p == 4) {
                        w.x = lower ? w.x : 0u;
                        w.y = lower ? w.y : 0u;
                        w.z = lower ? w.z : 0u;
                        w.w = lower ? w.w : 0u;
                    }
                    b[p] = __builtin_bit_cast(bf16v8, w);
                }
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int r = ry - dy;  // output row fed through tap row dy
                    if (r < 0 || r >= CV_ROWS) continue;
#pragma unroll
                    for (int p = 0; p < 5; ++p)
                        acc[r].add(ap[dy][p], b[p]);
                }
            }
        } else {
#pragma unroll
            for (int dt = 0; dt < 3; ++dt) {
                const short *q = lds + ((t - 1 + dt) & 3) * CV_FRAME + off1;
#pragma unroll
                for (int ry = 0; ry < CV_ROWS + 2; ++ry) {
                    bf16x4 b[3];
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) b[dx] = *reinterpret_cast<const bf16x4 *>(q + (ry * CT_C + dx) * 8);
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) {
                        const int r = ry - dy;
                        if (r < 0 || r >= CV_ROWS) continue;
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx)
                            acc[r].add(a1[dt * 9 + dy * 3 + dx], b[dx]);
                    }
                }
            }
        }
        // lane holds out[co = 4 kq + j][column n] of each row
#pragma unroll
        for (int r = 0; r < CV_ROWS; ++r) {
            const int y = u.y0 + r0 + r;
            if (y >= d.H || x >= d.W) continue;
            const size_t v = ((size_t)t * d.H + y) * d.W + x;
            bf16x4 o;
            if (MODE == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = bfbits(fmaxf(acc[r].v[j] + bv[j], 0.0f));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = bf2f(mk[r][j]) > 0.0f ? bfbits(acc[r].v[j]) : (short)0;
            }
            *reinterpret_cast<bf16x4 *>(out + v * C + 4 * kq) = o;
        }
        if (more) stage(t + 2, 0);
        __syncthreads();
    }
}

// Layer 4 (16 -> 1), no activation: y = b4 + sum w4 * act3. One output channel
// leaves an output-by-voxel product 15 of 16 rows empty, so the product is
// turned around: v_mfma_f32_32x32x16_bf16 forms, for 32 voxels u at a time,
// P[tap][u] = sum_ci w4[ci][tap] act3[u][ci] (27 of 32 rows used), and every
// output adds the 27 entries P[tap][v + off(tap)] in float. A workgroup streams
// the frames of a tile: per frame the P of its 612 voxels goes through LDS, and
// each thread adds 9 entries to each of the three output frames in flight.
// Bound by the read of act3 (32 bytes a voxel, 1.2 times with the rims): the
// per-voxel gather of 432 products it replaces took 651 us at 32x480x854;
// this takes 148 us.
constexpr int CO_PV = 616;  // floats per tap: 4 * CO_PV is half the banks, so a wavefront's two tap rows do not collide
static_assert(CO_PV >= CT_V && CO_PV % 16 == 8, "P row pitch");
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256, 2) void conv_out_kernel(Dims d, const short *act, const Prep *p, float *y, int nseg) {
    __shared__ float P[NT * CO_PV];
    TileUnit u;
    if (!tile_unit(d, nseg, u)) return;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int n = lane % 32, hf = lane / 32;
    // A operand: lane holds tap n, channels 8 hf .. + 7; B: voxel n of the block, the same channels
    bf16x8 aw;
#pragma unroll
    for (int j = 0; j < 8; ++j) aw[j] = n < NT ? bfbits(p->w4[8 * hf + j][n]) : (short)0;
    const float b4 = p->b4;
    constexpr int NB = (CT_V + 127) / 128;  // 32-voxel blocks per wavefront
    uint32_t off[NB];
#pragma unroll
    for (int m = 0; m < NB; ++m) {
        const int v = 32 * (wid + 4 * m) + n;
        const int gy = u.y0 - 1 + v / CT_C, gx = u.x0 - 1 + v % CT_C;
        const bool ok = v < CT_V && (unsigned)gy < (unsigned)d.H && (unsigned)gx < (unsigned)d.W;
        off[m] = ok ? (uint32_t)(gy * d.W + gx) * (C * 2) + 16 * hf : OOB_OFF;
    }
    uint4 b[NB];
    auto fetch = [&](int t) __attribute__((always_inline)) {
        const auto r = frame_rsrc(act, d, t);
#pragma unroll
        for (int m = 0; m < NB; ++m) b[m] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off[m], 0, 0));
    };
    fetch(u.t0 - 1);
    constexpr int NO = CT_H * CT_W / 256;  // outputs per thread
    float a1[NO], a2[NO];                  // frames t and t - 1 in flight
#pragma unroll
    for (int k = 0; k < NO; ++k) a1[k] = a2[k] = b4;
    for (int t = u.t0 - 1; t <= u.t1; ++t) {
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            f32x16 z;
#pragma unroll
            for (int i = 0; i < 16; ++i) z[i] = 0.f;
            const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16v8, aw),
                                                                       __builtin_bit_cast(bf16v8, b[m]), z, 0, 0, 0);
            const int v = 32 * (wid + 4 * m) + n;
            if (v < CT_V) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int tap = i % 4 + 8 * (i / 4) + 4 * hf;  // D row of element i
                    if (tap < NT) P[tap * CO_PV + v] = acc[i];
                }
            }
        }
        if (t < u.t1) fetch(t + 1);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NO; ++k) {
            const int o = tid + 256 * k, row = o / CT_W, col = o % CT_W;
            const float *q = P + row * CT_C + col;
            float a0 = b4;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int at = (i / 3) * CT_C + i % 3;
                a0 += q[i * CO_PV + at];
                a1[k] += q[(9 + i) * CO_PV + at];
                a2[k] += q[(18 + i) * CO_PV + at];
            }
            const int gy = u.y0 + row, gx = u.x0 + col;
            if (t - 1 >= u.t0 && gy < d.H && gx < d.W) y[((size_t)(t - 1) * d.H + gy) * d.W + gx] = a2[k];
            a2[k] = a1[k];
            a1[k] = a0;
        }
        __syncthreads();
    }
}

// Loss MSE(y, x* sqrt(V)) and g_y = 2 (y - x* sqrt(V)) / V; partials[2b] = sum of squares.
__global__ void mse_kernel(size_t V, const float *y, const float *xs, double scale, float *gy, double *partials) {
    __shared__ double red[256 / 64];
    double s = 0.0;
    const double inv = 1.0 / (double)V;
    for (size_t v = (size_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (size_t)gridDim.x * 256) {
        const double dlt = (double)y[v] - (double)xs[v] * scale;
        s += dlt * dlt;
        gy[v] = (float)(2.0 * dlt * inv);
    }
    const double t = block_sum<256>(s, red);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = t;
        partials[2 * blockIdx.x + 1] = 0.0;
    }
}

__global__ __launch_bounds__(256) void mse_finalize(int nb, size_t V, const double *partials, double *loss) {
    __shared__ double red[256 / 64];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) s += partials[2 * b];
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) *loss = s / (double)V;
}

// Weight and bias gradients of a 16 -> 16 layer on the matrix cores. For each
// tap, dW_tap[co][ci] = sum_v g[v][co] a[v + tap][ci] is a (16 x V) x (V x 16)
// product: v_mfma_f32_16x16x32_bf16 takes 32 voxels of a row per instruction,
// lane l holding 8 consecutive voxels of channel l % 16 of g (A) and of a (B).
// The volumes are channels-last, so rows are transposed on their way into LDS
// (blocks of 4 voxels x 8 channels per thread, byte permutes in registers).
// A workgroup walks down a WG_XC-voxel wide strip of one frame: per row step
// it stages one row of a of the three frames t - 1 .. t + 1 (a ring of four
// rows per frame) and one row of g, and each wavefront forms all 27 taps of
// 32 voxels: the three x shifts are taken on g (12 fragment reads for 27
// products), the nine (t, y) shifts are the staged rows of a. Rows, columns
// and frames outside the volume are staged as zeros. The strips' row steps
// are dealt out as equal contiguous ranges, one per workgroup.
// Operands are the stored bfloat16 values, products are exact, sums FP32. Each
// workgroup writes its partial sums ([co][ci * 27 + tap], then the bias of
// co); wgrad_reduce sums them.
// Bound by the matrix cores and the LDS reads (27 products per 12 reads). The
// form with one 16-bit load per (voxel, tap) and K = 4 float products it
// replaces took 606 us at 16x240x432; this takes 51.5 us (two reads of 53 MB).
constexpr int WG_XC = 128;              // strip width: 32 voxels per wavefront
constexpr int WG_AP = WG_XC + 8;        // halves per transposed row of a (conflict-free 16-byte reads)
constexpr int WG_GP = WG_XC + 24;       // the same for g, with its neighbours at x - 1 and x + WG_XC
constexpr int WG_GO = 8;                // index of the strip's first voxel in a row of g
constexpr int WG_ROW_A = C * WG_AP, WG_ROW_G = C * WG_GP;

__device__ __forceinline__ uint4 load_b128(__amdgpu_buffer_rsrc_t r, uint32_t boff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, boff, 0, 0));
}

// One thread's block of a channels-last row: 4 consecutive voxels (from byte
// offset row + 32 x of the volume) x 8 channels (half 0 or 1).
struct Block4x8 {
    uint4 v[4];
};
__device__ __forceinline__ void load_block(Block4x8 &b, __amdgpu_buffer_rsrc_t r, bool rowok, uint32_t row, int x,
                                           int W, int half) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
        b.v[j] = load_b128(r, rowok && x + j < W ? row + (uint32_t)(x + j) * (C * 2) + 16 * half : OOB_OFF);
}
// Writes it transposed: channel 8 half + c at dst + (8 half + c) * pitch.
__device__ __forceinline__ void store_block(const Block4x8 &b, short *dst, int pitch, int half) {
    const uint32_t w[4][4] = {{b.v[0].x, b.v[0].y, b.v[0].z, b.v[0].w},
                              {b.v[1].x, b.v[1].y, b.v[1].z, b.v[1].w},
                              {b.v[2].x, b.v[2].y, b.v[2].z, b.v[2].w},
                              {b.v[3].x, b.v[3].y, b.v[3].z, b.v[3].w}};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
        uint2 o;
        o.x = __builtin_amdgcn_perm(w[1][c / 2], w[0][c / 2], sel);
        o.y = __builtin_amdgcn_perm(w[3][c / 2], w[2][c / 2], sel);
        *reinterpret_cast<uint2 *>(dst + (8 * half + c) * pitch) = o;
    }
}

// Row steps of the weight-gradient strips: index r is row y of strip xc of
// frame t, r = (t * nxc + xc) * H + y; workgroup `unit` of n owns an equal share.
__device__ __forceinline__ int strip_count(const Dims &d) { return (d.W + WG_XC - 1) / WG_XC; }
__device__ __forceinline__ int share_begin(const Dims &d, int unit, int n) {
    return (int)((int64_t)unit * d.T * strip_count(d) * d.H / n);
}

// Fragment of 8 consecutive voxels shifted by one: elements -1 .. 6 or 1 .. 8
// around the aligned block m (prev and next hold the neighbouring pairs).
__device__ __forceinline__ bf16v8 shift_up(const uint4 &m, uint32_t prev) {
    const uint4 r = {__builtin_amdgcn_alignbit(m.x, prev, 16), __builtin_amdgcn_alignbit(m.y, m.x, 16),
                     __builtin_amdgcn_alignbit(m.z, m.y, 16), __builtin_amdgcn_alignbit(m.w, m.z, 16)};
    return __builtin_bit_cast(bf16v8, r);
}
__device__ __forceinline__ bf16v8 shift_down(const uint4 &m, uint32_t next) {
    const uint4 r = {__builtin_amdgcn_alignbit(m.y, m.x, 16), __builtin_amdgcn_alignbit(m.z, m.y, 16),
                     __builtin_amdgcn_alignbit(m.w, m.z, 16), __builtin_amdgcn_alignbit(next, m.w, 16)};
    return __builtin_bit_cast(bf16v8, r);
}
__device__ __forceinline__ bf16v8 ones_frag() {
    const uint4 r = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    return __builtin_bit_cast(bf16v8, r);
}

__global__ __launch_bounds__(256, 2) void wgrad16_kernel(Dims d, const short *a, const short *g, int nunits,
                                                         float *partials) {
    constexpr int NP = C * (C * NT + 1);
    constexpr int STAGE = 12 * WG_ROW_A + 2 * WG_ROW_G;  // halves
    constexpr int LDS_BYTES = STAGE * 2 > NP * 4 ? STAGE * 2 : NP * 4;
    __shared__ __align__(16) char lds[LDS_BYTES];
    short *const La = reinterpret_cast<short *>(lds);  // [frame 3][row ring 4][C][WG_AP]
    short *const Lg = La + 12 * WG_ROW_A;              // [2][C][WG_GP]
    const int unit = net_unit(blockIdx.x, nunits);
    if (unit < 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ch = lane % 16, kv = lane / 16;
    const auto ra = act_rsrc(a, d), rg = act_rsrc(g, d);
    // staging: wavefront 0 .. 2 the row of frame t - 1 .. t + 1 of a, wavefront 3 the row of g
    const int half = lane & 1, bx = 4 * (lane >> 1);
    Acc<32> acc[NT], bacc;
    const int nxc = strip_count(d);
    const int rend = share_begin(d, unit + 1, nunits);
    int r = share_begin(d, unit, nunits);
    while (r < rend) {
        const int strip = r / d.H, ys = r - strip * d.H;
        const int t = strip / nxc, X0 = (strip - t * nxc) * WG_XC;
        const int ye = ys + (rend - r) < d.H ? ys + (rend - r) : d.H;
        Block4x8 blk[3];  // up to three rows' loads in flight
        short edge[3] = {0, 0, 0};
        // loads of row ya of a (three frames) and row yg of g
        auto load_rows = [&](int ya, int yg, int slot) __attribute__((always_inline)) {
            const int tt = wid < 3 ? t + wid - 1 : t, yy = wid < 3 ? ya : yg;
            const bool ok = tt >= 0 && tt < d.T && yy >= 0 && yy < d.H;
            const uint32_t row = (uint32_t)(((size_t)(ok ? tt : 0) * d.H + (ok ? yy : 0)) * d.W) * (C * 2);
            load_block(blk[slot], wid < 3 ? ra : rg, ok, row, X0 + bx, d.W, half);
            if (wid == 3) {  // the strip's neighbours of g: lanes 0 .. 15 x - 1, 16 .. 31 x + WG_XC
                const int xe = lane < 16 ? X0 - 1 : X0 + WG_XC;
                edge[slot] = load_b16(rg, ok && lane < 32 && xe >= 0 && xe < d.W ? row + (uint32_t)xe * (C * 2) + 2 * ch
                                                                            : OOB_OFF);
            }
        };
        auto store_rows = [&](int ya, int yg, int slot) __attribute__((always_inline)) {
            if (wid < 3) {
                store_block(blk[slot], La + (wid * 4 + (ya & 3)) * WG_ROW_A + bx, WG_AP, half);
            } else {
                short *dst = Lg + (yg & 1) * WG_ROW_G;
                store_block(blk[slot], dst + WG_GO + bx, WG_GP, half);
                if (lane < 32) dst[ch * WG_GP + (lane < 16 ? WG_GO - 1 : WG_GO + WG_XC)] = edge[slot];
            }
        };
        // rows ys - 1, ys, ys + 1 of a and row ys of g (rows of g outside the range are never read)
#pragma unroll
        for (int k = 0; k < 3; ++k) load_rows(ys - 1 + k, ys, k);
#pragma unroll
        for (int k = 0; k < 3; ++k) store_rows(ys - 1 + k, ys, k);
        __syncthreads();
        for (int y = ys; y < ye; ++y) {
            const bool more = y + 1 < ye;
            if (more) load_rows(y + 2, y + 1, 0);
            if (X0 + 32 * wid < d.W) {
                const short *gp = Lg + (y & 1) * WG_ROW_G + ch * WG_GP + WG_GO + 32 * wid + 8 * kv;
                const uint4 m = *reinterpret_cast<const uint4 *>(gp);
                const uint32_t prev = *reinterpret_cast<const uint32_t *>(gp - 2);
                const uint32_t next = *reinterpret_cast<const uint32_t *>(gp + 8);
                // a at u = v + off: for x shift dx the voxel of g is u - dx
                const bf16v8 gf[3] = {shift_down(m, next), __builtin_bit_cast(bf16v8, m), shift_up(m, prev)};
                bacc.add(gf[1], ones_frag());
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    const int slot = (k / 3) * 4 + ((y + k % 3 - 1) & 3);
                    const bf16v8 af = *reinterpret_cast<const bf16v8 *>(La + slot * WG_ROW_A + ch * WG_AP +
                                                                        32 * wid + 8 * kv);
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        acc[3 * k + dx].add(gf[dx], af);
                }
            }
            if (more) store_rows(y + 2, y + 1, 0);
            __syncthreads();
        }
        r += ye - ys;
    }
    // the workgroup's four wavefronts add into LDS in turn (lane holds
    // dW_tap[co = 4 kv + j][ci = ch]), then one partial per workgroup
    float *red = reinterpret_cast<float *>(lds);
    for (int w = 0; w < 4; ++w) {
        if (wid == w) {
#pragma unroll
            for (int tap = 0; tap < NT; ++tap)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = (4 * kv + j) * (C * NT + 1) + ch * NT + tap;
                    red[k] = (w == 0 ? 0.0f : red[k]) + acc[tap].v[j];
                }
            if (ch == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = (4 * kv + j) * (C * NT + 1) + C * NT;
                    red[k] = (w == 0 ? 0.0f : red[k]) + bacc.v[j];
                }
            }
        }
        __syncthreads();
    }
    float *out = partials + (size_t)unit * NP;
    for (int k = tid; k < NP; k += 256) out[k] = red[k];
}

// Weight and bias gradients of the one-channel layers on the matrix cores:
//   MODE 1 (layer 1): D[co][tap] = sum_v g[v][co] bf16(f[v + off(tap)]),
//                     db1[co] = sum_v g[v][co]; X = g (channels-last), Z = f;
//   MODE 4 (layer 4): D[ci][tap] = sum_u act3[u][ci] g_y[u - off(tap)]
//                     (the same sum as over v = u - off), db4 = sum_v g_y[v];
//                     X = act3, Z = g_y, split exactly into three bfloat16 parts.
// Strips, row steps and shares as wgrad16_kernel: X rows are staged transposed,
// 32 voxels of a row per instruction, the 27 taps as two blocks of 16 columns.
// Z rows of the three frames lie in LDS three times, shifted by x = -1, 0, 1, so
// that a lane's 8 consecutive voxels at its own tap are one aligned read.
// Bound by the read of X (32 bytes a voxel) and the row steps' latency. The
// element-wise gathers with K = 4 float products it replaces took 104 (layer 1)
// and 102 us (layer 4) at 16x240x432; this takes 22 and 28 us.
template <int MODE>
__global__ __launch_bounds__(256) void wgrad1_kernel(Dims d, const short *x16, const float *z1, int nunits,
                                                     float *partials) {
    constexpr int PARTS = MODE == 1 ? 1 : 3;
    constexpr int NPR = MODE == 1 ? C * (NT + 1) : C * NT + 1;
    constexpr int ZROWS = 3 * 3 * 4;  // [x shift][frame][row ring]
    __shared__ __align__(16) short lds[2 * WG_ROW_A + PARTS * ZROWS * WG_AP];
    __shared__ float red[NPR];
    short *const Lx = lds;                 // [2][C][WG_AP]
    short *const Lz = lds + 2 * WG_ROW_A;  // [part][shift][frame][4][WG_AP]
    const int unit = net_unit(blockIdx.x, nunits);
    if (unit < 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane % 16, kv = lane / 16;
    const auto rx = act_rsrc(x16, d);
    const auto rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(z1), (short)0,
                                                      (int)((size_t)d.T * d.H * d.W * sizeof(float)), 0x00020000);
    // this lane's tap columns: Z at off(tap) (MODE 1) or at -off(tap) = off(26 - tap) (MODE 4)
    bool tapok[2];
    int zoff[2], zdy[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        const int tap = 16 * blk + c;
        tapok[blk] = tap < NT;
        const int s = !tapok[blk] ? 0 : (MODE == 1 ? tap : NT - 1 - tap);
        zoff[blk] = ((s % 3) * 3 + s / 9) * 4 * WG_AP + 32 * wid + 8 * kv;
        zdy[blk] = (s / 3) % 3 - 1;
    }
    Acc<32> acc[2], bacc;
    const int nxc = strip_count(d);
    const int rend = share_begin(d, unit + 1, nunits);
    int r = share_begin(d, unit, nunits);
    while (r < rend) {
        const int strip = r / d.H, ys = r - strip * d.H;
        const int t = strip / nxc, X0 = (strip - t * nxc) * WG_XC;
        const int ye = ys + (rend - r) < d.H ? ys + (rend - r) : d.H;
        Block4x8 blk[3];  // up to three rows' loads in flight
        float z[3][3];
        // wavefront 0 stages a row of X, wavefronts 1 .. 3 a row of Z of the
        // frames t - 1 .. t + 1 (columns X0 - 1 .. X0 + WG_XC)
        auto load_rows = [&](int yx, int yz, int slot) __attribute__((always_inline)) {
            const int tt = wid == 0 ? t : t + wid - 2, yy = wid == 0 ? yx : yz;
            const bool ok = tt >= 0 && tt < d.T && yy >= 0 && yy < d.H;
            const size_t row = ((size_t)(ok ? tt : 0) * d.H + (ok ? yy : 0)) * d.W;
            if (wid == 0) {
                load_block(blk[slot], rx, ok, (uint32_t)row * (C * 2), X0 + 4 * (lane >> 1), d.W, lane & 1);
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const int e = lane + 64 * k, xe = X0 - 1 + e;
                    z[slot][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        rz, ok && e < WG_XC + 2 && xe >= 0 && xe < d.W ? (uint32_t)(row + xe) * 4 : OOB_OFF, 0, 0));
                }
            }
        };
        auto store_rows = [&](int yx, int yz, int slot) __attribute__((always_inline)) {
            if (wid == 0) {
                store_block(blk[slot], Lx + (yx & 1) * WG_ROW_A + 4 * (lane >> 1), WG_AP, lane & 1);
            } else {
                short *dst = Lz + ((wid - 1) * 4 + (yz & 3)) * WG_AP;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const int e = lane + 64 * k;  // column X0 - 1 + e: index e - s of the plane shifted by s - 1
                    float rest = z[slot][k];
#pragma unroll
                    for (int q = 0; q < PARTS; ++q) {
                        const short b = PARTS > 1 && q == 0 ? first_part(rest) : bfbits(rest);
                        rest = split_rest(rest, bf2f(b));
#pragma unroll
                        for (int s = 0; s < 3; ++s)
                            if (e >= s && e - s < WG_XC) dst[(q * 9 + s * 3) * 4 * WG_AP + e - s] = b;
                    }
                }
            }
        };
#pragma unroll
        for (int k = 0; k < 3; ++k) load_rows(ys, ys - 1 + k, k);
#pragma unroll
        for (int k = 0; k < 3; ++k) store_rows(ys, ys - 1 + k, k);
        __syncthreads();
        for (int y = ys; y < ye; ++y) {
            const bool more = y + 1 < ye;
            if (more) load_rows(y + 1, y + 2, 0);
            if (X0 + 32 * wid < d.W) {
                const bf16v8 xf =
                    *reinterpret_cast<const bf16v8 *>(Lx + (y & 1) * WG_ROW_A + c * WG_AP + 32 * wid + 8 * kv);
                if constexpr (MODE == 1) bacc.add(xf, ones_frag());
#pragma unroll
                for (int q = PARTS - 1; q >= 0; --q) {  // smallest part first
                    bf16v8 zf[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        zf[b] = *reinterpret_cast<const bf16v8 *>(Lz + q * ZROWS * WG_AP + zoff[b] +
                                                                  ((y + zdy[b]) & 3) * WG_AP);
                    acc[0].add(xf, zf[0]);
                    acc[1].add(xf, zf[1]);
                    // column 13 of block 0 is the centre tap
                    if constexpr (MODE == 4)
                        bacc.add(ones_frag(), zf[0]);
                }
            }
            if (more) store_rows(y + 1, y + 2, 0);
            __syncthreads();
        }
        r += ye - ys;
    }
    // lane holds D[channel 4 kv + j][tap 16 blk + c]; the four wavefronts add into LDS in turn
    for (int w = 0; w < 4; ++w) {
        if (wid == w) {
#pragma unroll
            for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (!tapok[blk]) continue;
                    const int ch = 4 * kv + j, tap = 16 * blk + c;
                    const int k = MODE == 1 ? ch * (NT + 1) + tap : ch * NT + tap;
                    red[k] = (w == 0 ? 0.0f : red[k]) + acc[blk].v[j];
                }
            if (MODE == 1 ? c == 0 : lane == 13) {
#pragma unroll
                for (int j = 0; j < (MODE == 1 ? 4 : 1); ++j) {
                    const int k = MODE == 1 ? (4 * kv + j) * (NT + 1) + NT : C * NT;
                    red[k] = (w == 0 ? 0.0f : red[k]) + bacc.v[j];
                }
            }
        }
        __syncthreads();
    }
    float *out = partials + (size_t)unit * NPR;
    for (int k = tid; k < NPR; k += 256) out[k] = red[k];
}

constexpr int WG16_BLOCKS = 512;  // x 4 wavefronts (two per SIMD): one partial per workgroup

// Sums the workgroup partials of one layer into the gradient buffer (same
// layout as the masters): dW[co][ci][tap] at w_off, db[co] at b_off. A
// workgroup takes 64 consecutive entries (the partials are read in whole
// lines; one workgroup per entry read 4 bytes of each line and took 20 us for
// 512 partials of a 16 -> 16 layer, this 4.8 us): each of its 16 wavefronts adds
// every 16th partial in double, then the 16 sums are added in order.
template <int CI, int CO>
__global__ __launch_bounds__(1024) void wgrad_reduce(int nblocks, const float *partials, float *grad, int w_off,
                                                     int b_off) {
    constexpr int NP = CO * (CI * NT + 1);
    __shared__ double red[16][64];
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    double s = 0.0;
    if (i < NP) {
#pragma unroll 8
        for (int b = part; b < nblocks; b += 16) s += (double)partials[(size_t)b * NP + i];
    }
    red[part][lane] = s;
    __syncthreads();
    if (part == 0 && i < NP) {
        for (int k = 1; k < 16; ++k) s += red[k][lane];
        const int co = i / (CI * NT + 1), r = i % (CI * NT + 1);
        if (r < CI * NT)
            grad[w_off + co * CI * NT + r] = (float)s;
        else
            grad[b_off + co] = (float)s;
    }
}

// Start vector from the net output: x0 = max(y, 0) + eps (normalised by the
// iteration), 16 bytes at a time where the arrays allow it (32x480x854 19 us,
// 33 by single elements on a fixed 1024 workgroups).
__global__ void warm_x0_kernel(size_t V, const float *y, float eps, float *x0) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    const size_t nv = (((uintptr_t)y | (uintptr_t)x0) & 15) == 0 ? V / 4 : 0;
    for (size_t i = i0; i < nv; i += stride) {
        float4 v = reinterpret_cast<const float4 *>(y)[i];
        v.x = fmaxf(v.x, 0.0f) + eps;
        v.y = fmaxf(v.y, 0.0f) + eps;
        v.z = fmaxf(v.z, 0.0f) + eps;
        v.w = fmaxf(v.w, 0.0f) + eps;
        reinterpret_cast<float4 *>(x0)[i] = v;
    }
    for (size_t v = 4 * nv + i0; v < V; v += stride) x0[v] = fmaxf(y[v], 0.0f) + eps;
}

constexpr int WG1_BLOCKS = 1024;  // x 4 wavefronts: wgrad1_kernel's partial sums (448 floats each)

}  // namespace net

}  // namespace stpi

using namespace stpi;
using namespace stpi::net;

extern "C" {

int stpi_net_param_count(void) { return NPARAM; }

size_t stpi_net_prep_bytes(void) { return sizeof(Prep); }

size_t stpi_net_workspace_bytes(const stpi_problem *p) {
    if (validate_problem(p) != STPI_OK) return 0;
    const size_t V = (size_t)p->T * p->H * p->W;
    // 3 activation volumes + 2 gradient volumes (bf16 x 16 channels), g_y, loss partials,
    // weight-gradient partials.
    size_t b = 5 * ((V * C * 2 + 255) & ~(size_t)255);
    b += (V * 4 + 255) & ~(size_t)255;
    b += 4096 * 8;
    b += std::max((size_t)WG1_BLOCKS * C * (NT + 1), (size_t)WG16_BLOCKS * C * (C * NT + 1)) * sizeof(float);
    return b;
}

int stpi_net_prepare(const float *master, void *prep, void *stream) {
    clear_error();
    if (!master || !prep) return fail(STPI_EINVAL, "NULL buffer");
    hipLaunchKernelGGL(prepare_kernel, dim3(8), dim3(256), 0, (hipStream_t)stream, master, (Prep *)prep);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? STPI_OK : hip_fail(e, "net prepare");
}

static int net_check(const stpi_problem *p, const void *ws, size_t ws_bytes) {
    int rc = validate_problem(p);
    if (rc) return rc;
    if ((size_t)p->T * p->H * p->W * C * sizeof(short) >= ((size_t)1 << 31))
        return fail(STPI_EUNSUPPORTED, "net volumes are limited to 2^31 bytes of activations (%d x %d x %d)", p->T,
                    p->H, p->W);
    if (!ws || ws_bytes < stpi_net_workspace_bytes(p))
        return fail(STPI_EWORKSPACE, "net workspace needs %zu bytes", stpi_net_workspace_bytes(p));
    return STPI_OK;
}

struct NetWs {
    short *act1, *act2, *act3, *g_a, *g_b;
    float *gy;
    double *lpart;
    float *wpart;
};

static NetWs net_ws(const stpi_problem *p, void *ws) {
    const size_t V = (size_t)p->T * p->H * p->W;
    const size_t vb = (V * C * 2 + 255) & ~(size_t)255;
    char *w = (char *)ws;
    NetWs n;
    n.act1 = (short *)w;
    n.act2 = (short *)(w + vb);
    n.act3 = (short *)(w + 2 * vb);
    n.g_a = (short *)(w + 3 * vb);
    n.g_b = (short *)(w + 4 * vb);
    char *q = w + 5 * vb;
    n.gy = (float *)q;
    q += (V * 4 + 255) & ~(size_t)255;
    n.lpart = (double *)q;
    q += 4096 * 8;
    n.wpart = (float *)q;
    return n;
}

static int net_tiles(const stpi_problem *p) { return ((p->W + CT_W - 1) / CT_W) * ((p->H + CT_H - 1) / CT_H); }

// Frame segments of the streamed layer kernels (two workgroups per CU): a
// segment costs its frames plus three (two rim frames and the start), and the
// chip takes the units in rounds of its resident workgroups, so the split with
// the fewest frame steps over all rounds (4000x8x8, one tile: 512 segments, forward
// 498 us with at most 64 of them, 110 now; 1000x16x32 145 and 56).
static int tile_segments(const stpi_problem *p) {
    const int64_t tiles = net_tiles(p), slots = 2 * (int64_t)device_cus();
    int64_t best = 1, cost = INT64_MAX;
    auto take = [&](int64_t k) {
        const int64_t c = (tiles * k + slots - 1) / slots * ((p->T + k - 1) / k + 3);
        if (c < cost) {
            cost = c;
            best = k;
        }
    };
    const int few = std::min(p->T, 64);
    for (int k = 1; k <= few; ++k) take(k);
    for (int rounds = 1; rounds <= 8; ++rounds) {  // long clips of few tiles: whole rounds
        const int64_t k = std::min<int64_t>(p->T, rounds * slots / tiles);
        if (k > few) take(k);
    }
    return (int)best;
}

// Workgroups of a weight-gradient launch: as many as fit at once (two per CU
// of wgrad16_kernel, four of wgrad1_kernel), and at least six row steps each (a
// share starts by staging three rows), or two where not every CU would have one
// (4x64x80: wgrad16 22.7 -> 18.7 us, wgrad1 12.3 -> 6.5 and 8.6 -> 4.7, with
// the first three rows' loads in flight together).
static int wgrad_units(const stpi_problem *p, int most) {
    const int64_t rows = (int64_t)p->T * ((p->W + WG_XC - 1) / WG_XC) * p->H;
    return (int)std::min<int64_t>(most, std::max<int64_t>(1, std::max(rows / 6, std::min<int64_t>(rows / 2, device_cus()))));
}

int stpi_net_forward(const stpi_problem *p, const float *f, const void *prep, float *y, void *ws, size_t ws_bytes,
                     void *stream) {
    clear_error();
    int rc = net_check(p, ws, ws_bytes);
    if (rc) return rc;
    if (!f || !prep || !y) return fail(STPI_EINVAL, "NULL buffer");
    const Prep *P = (const Prep *)prep;
    NetWs n = net_ws(p, ws);
    hipStream_t s = (hipStream_t)stream;
    const Dims d{p->T, p->H, p->W};
    const int nseg = tile_segments(p), grid = net_grid(net_tiles(p) * nseg);
    hipLaunchKernelGGL(one_channel_kernel<0>, dim3(grid), dim3(256), 0, s, d, f, P, (const short *)nullptr, n.act1, nseg);
    hipLaunchKernelGGL(conv16_kernel<0>, dim3(grid), dim3(256), 0, s, d, (const short *)n.act1, P->a2, P->b2,
                       (const short *)nullptr, n.act2, nseg);
    hipLaunchKernelGGL(conv16_kernel<0>, dim3(grid), dim3(256), 0, s, d, (const short *)n.act2, P->a3, P->b3,
                       (const short *)nullptr, n.act3, nseg);
    hipLaunchKernelGGL(conv_out_kernel, dim3(grid), dim3(256), 0, s, d,
                       (const short *)n.act3, P, y, nseg);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? STPI_OK : hip_fail(e, "net forward");
}

int stpi_net_backward(const stpi_problem *p, const float *f, const void *prep, const float *y, const float *x_star,
                      double *loss, float *grad, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    int rc = net_check(p, ws, ws_bytes);
    if (rc) return rc;
    if (!f || !prep || !y || !x_star || !loss || !grad) return fail(STPI_EINVAL, "NULL buffer");
    const Prep *P = (const Prep *)prep;
    NetWs n = net_ws(p, ws);
    hipStream_t s = (hipStream_t)stream;
    const Dims d{p->T, p->H, p->W};
    const size_t V = (size_t)p->T * p->H * p->W;
    const int nw = wgrad_units(p, WG16_BLOCKS), nw1 = wgrad_units(p, WG1_BLOCKS), nseg = tile_segments(p), grid = net_grid(net_tiles(p) * nseg);
    hipLaunchKernelGGL(mse_kernel, dim3(2048), dim3(256), 0, s, V, y, x_star, std::sqrt((double)V), n.gy, n.lpart);
    hipLaunchKernelGGL(mse_finalize, dim3(1), dim3(256), 0, s, 2048, V, n.lpart, loss);
    // layer 4
    hipLaunchKernelGGL(wgrad1_kernel<4>, dim3(net_grid(nw1)), dim3(256), 0, s, d, (const short *)n.act3,
                       (const float *)n.gy, nw1, n.wpart);
    hipLaunchKernelGGL((wgrad_reduce<C, 1>), dim3((C * NT + 1 + 63) / 64), dim3(1024), 0, s, nw1, n.wpart, grad, OFF_W4, OFF_B4);
    hipLaunchKernelGGL(one_channel_kernel<1>, dim3(grid), dim3(256), 0, s, d, (const float *)n.gy, P,
                       (const short *)n.act3, n.g_a, nseg);  // g at pre3
    // layer 3
    hipLaunchKernelGGL(wgrad16_kernel, dim3(net_grid(nw)), dim3(256), 0, s, d, (const short *)n.act2,
                       (const short *)n.g_a, nw, n.wpart);
    hipLaunchKernelGGL((wgrad_reduce<C, C>), dim3((C * (C * NT + 1) + 63) / 64), dim3(1024), 0, s, nw,
                       n.wpart, grad, OFF_W3, OFF_B3);
    hipLaunchKernelGGL(conv16_kernel<1>, dim3(grid), dim3(256), 0, s, d, (const short *)n.g_a, P->a3d,
                       (const float *)nullptr, (const short *)n.act2, n.g_b, nseg);  // g at pre2
    // layer 2
    hipLaunchKernelGGL(wgrad16_kernel, dim3(net_grid(nw)), dim3(256), 0, s, d, (const short *)n.act1,
                       (const short *)n.g_b, nw, n.wpart);
    hipLaunchKernelGGL((wgrad_reduce<C, C>), dim3((C * (C * NT + 1) + 63) / 64), dim3(1024), 0, s, nw,
                       n.wpart, grad, OFF_W2, OFF_B2);
    hipLaunchKernelGGL(conv16_kernel<1>, dim3(grid), dim3(256), 0, s, d, (const short *)n.g_b, P->a2d,
                       (const float *)nullptr, (const short *)n.act1, n.g_a, nseg);  // g at pre1
    // layer 1
    hipLaunchKernelGGL(wgrad1_kernel<1>, dim3(net_grid(nw1)), dim3(256), 0, s, d, (const short *)n.g_a, f, nw1, n.wpart);
    hipLaunchKernelGGL((wgrad_reduce<1, C>), dim3((C * (NT + 1) + 63) / 64), dim3(1024), 0, s, nw1, n.wpart, grad, OFF_W1, OFF_B1);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? STPI_OK : hip_fail(e, "net backward");
}

int stpi_net_warm_start(int64_t n, const float *y, float eps, float *x0, void *stream) {
    clear_error();
    if (n < 1 || !y || !x0) return fail(STPI_EINVAL, "bad arguments");
    hipLaunchKernelGGL(warm_x0_kernel, dim3(2048), dim3(256), 0, (hipStream_t)stream, (size_t)n, y, eps, x0);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? STPI_OK : hip_fail(e, "warm start");
}

}  // extern "C"
