// Fitting one sine MLP per image on the GPU (Eq. 1): full-batch gradient of the squared error by forward and backward
// passes on the matrix cores, Adam update fused into the same kernel.  This file: the handle, the fp32 kernels described
// next, the host side of both families; the split-precision kernels (fp16 hi/lo operand pairs) are rinr_fit16.hip.h.
//
// One workgroup per image and one launch per step; with few images, several workgroups share an image's pixels and a second
// launch adds their gradients up (plan_splits).  The image's weights live in LDS (bias folded in as an
// extra input column that multiplies a row of ones), pixels are taken in chunks of PC, and every
// contraction of a chunk is a set of 16x16 output tiles computed with v_mfma_f32_16x16x4_f32 from LDS
// operands:
//     forward        Z_l [d_out x PC]  = W_l [d_out x d_in+1] . H_l [d_in+1 x PC]        H_{l+1} = sin(w0 Z_l)
//     weight grads   dW_l [d_out x d_in+1] += D_l [d_out x PC] . H_l^T                   (contraction over pixels)
//     backward       D_{l-1} = (W_l^T . D_l) * w0 cos(w0 Z_{l-1})
// In LDS the sine layers' weights and biases are held times w0 / 2pi, so that Z comes out in revolutions, the unit of
// the hardware sine and cosine, and the error is carried as E_l = c_l D_l with c_{L-1} = 1, c_{L-2} = 1 / w0,
// c_{l-1} = c_l / 2pi below that: then E_{l-1} = (W_l^T . E_l) * cos(2pi Z'_{l-1}) with the LDS weights, one multiply per
// element, and the accumulated sum over pixels of E_l H_l^T is c_l times the gradient: the factor 1 / c_l is applied
// once per parameter at the end.
// The weight-gradient tiles stay in registers for the whole step (each wavefront owns a fixed set of
// tiles of every layer): at the end of the step the owner of an entry applies Adam to it in place, or
// hands it to the second launch.  Nothing is allocated and nothing else leaves the workgroup except the
// parameters, the moments and one loss value.
#include "../../include/rinr_fit.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxL = RINR_FIT_MAX_LAYERS;
// The kernels are built per hidden width rounded up to a multiple of 8 (WQ) and per depth bucket.
// Row tiles of a hidden layer: MT = ceil(WQ / 16).
constexpr int fit_tiles(int wq) { return (wq + 15) / 16; }
// Wavefronts per workgroup (= per image).  Every phase between two barriers is a short dependent chain per
// wavefront, so what fills the matrix pipe is other wavefronts: 4 at widths <= 16, whose 4 tiles per layer do not feed
// more, and several images per CU; 8 at widths <= 32, two images per CU; 12 at widths <= 48, one wavefront per tile of
// their 12-tile layers (LDS holds one image); 16 above, one per forward tile, so that the 20 gradient tiles of a
// width-64 layer take two rounds instead of three (+3 %, a few spilled registers notwithstanding).
constexpr int fit_waves(int wq) { return fit_tiles(wq) == 1 ? 4 : (fit_tiles(wq) == 2 ? 8 : (fit_tiles(wq) == 3 ? 12 : 16)); }
// Wavefronts per SIMD the kernel is compiled for (the register budget follows): at widths <= 32 two workgroups
// share a CU (10 x 32 at 224 x 224, 512 images: 26.8 -> 20.3 ms per step).
constexpr int fit_waves_per_simd(int wq) { return fit_tiles(wq) == 1 ? 3 : (fit_tiles(wq) == 3 ? 3 : 4); }
// Layer counts the kernels are built for: the accumulators of all layers stay in registers, so the depth
// is a compile-time bound and a shallow model takes the kernel with the smaller one.
constexpr int fit_depth_lo(int wq) { return fit_tiles(wq) == 1 ? 4 : (fit_tiles(wq) == 4 ? 7 : 10); }
constexpr int fit_depth_hi(int wq) { return fit_tiles(wq) <= 2 ? kMaxL : fit_depth_lo(wq); }
constexpr uint32_t kLdsLimit = 160 * 1024;

thread_local int g_fit_last_hip = 0;
inline bool hip_fail(hipError_t e) {
    if (e == hipSuccess) return false;
    g_fit_last_hip = (int)e;
    return true;
}
#define FIT_HIP(call) do { if (hip_fail(call)) return RINR_E_HIP; } while (0)

// Shapes for hidden widths <= WQ (a multiple of 8) and the LDS layout in floats.  Padding is with zero weights, which
// leaves values and gradients of the real entries unchanged (a padded unit outputs sin(0) = 0 and receives no
// error), so every hidden layer has the same compile-time shape whatever its true width.  Pixels are taken 64 at a time.
// A layer's input is a block of four rows (ones, and three rows whose weights are zero) followed by the activations:
// the bias is the weight of the row of ones, the contraction over the inputs takes 1 + WQ / 4 k-steps of four rows, and
// what lies beyond row 4 + WQ is never read.  The first layer's block is (ones, x, y, zero) and is its whole input.
// LDS has 32 banks and serves a wavefront's 4-byte accesses in two halves of 32 lanes; a half that hits a bank
// twice takes a second cycle.  The MFMA operands are read in two patterns, lane (m, kq) -> (row m, column kq) and
// -> (row kq, column m), so a half covers 16 rows x 2 columns or 2 rows x 16 columns.  Weight rows have stride
// LD = 2 * odd, which makes the first pattern conflict-free.  Pixel-buffer rows come in pairs: row r starts at
// prow(r) = (r / 2) * PAIR + (r % 2) * ODD with PAIR = 2 * odd and ODD = 16 (mod 32), so that 16 consecutive rows
// start in 16 different even banks and the two rows of a pair are 16 banks apart: both patterns conflict-free
// (ODD = 80 is the first such value that holds 64 pixels, PAIR = 146 the first that holds two rows).
//   W0  [RO][6]        first layer: columns bias, x, y, 0
//   Wh  [RO][LD] each  layers 1..L-2: columns bias, 0, 0, 0, then the weights (RO = 16 MT rows, zero beyond the width)
//   Wl  [16][LD]       last layer (3 real rows)
//   B0, B1, B2 [KR rows] three pixel buffers.  Forward: the input of layer l is B[l & 1] (row 0 ones, rows 4.. the
//       activations; B0 rows 1..3 hold x, y, 0).  Backward: B0 holds the restored input of the layer at hand; B1 / B2
//       the back-propagated error with row = unit, ping-pong (so B1's row of ones is written again for every chunk).
//   B3 [KR rows]       with PIPE: the restored layer inputs alternate between B0 and B3.
// Pre-activations are not stashed in LDS: the wavefront that computed a tile keeps it in registers until the
// backward pass has used it (sine again for the weight gradient's operand, cosine for the error).
template <int WQ> struct Shape {
    static constexpr int PC = 64, PT = PC / 16;
    static constexpr int MT = fit_tiles(WQ), RO = 16 * MT, LD = RO + 6, KR = RO + 4;
    static constexpr int KSF = 1 + WQ / 4;                          // k-steps of a hidden layer's forward contraction
    static constexpr int KSB = WQ / 4;                              // ... of the backward one (over the layer's outputs)
    static constexpr int NIT = (4 + WQ + 15) / 16;                  // column tiles of a hidden weight gradient (block of four + inputs)
    static constexpr int PAIR = 146, ODD = 80;
    static __host__ __device__ constexpr int prow(int r) { return (r >> 1) * PAIR + (r & 1) * ODD; }
    static constexpr int ML = fit_depth_hi(WQ);                     // deepest model: register budget (and LDS at width 64)
    static constexpr int NW = fit_waves(WQ), NTHREADS = NW * 64;
    static constexpr int ZSLOTS = (MT * PT + NW - 1) / NW;  // forward tiles a wavefront owns per layer
    static constexpr int GSLOTS = (MT * NIT + NW - 1) / NW; // gradient tiles a wavefront owns per layer
    static __host__ __device__ constexpr int w_off(int l) { return l == 0 ? 0 : RO * 6 + (l - 1) * RO * LD; }
    static __host__ __device__ constexpr int w_end(int L) { return RO * 6 + (L - 2) * RO * LD + 16 * LD; }
    static __host__ __device__ constexpr int buf(int b, int L) { return w_end(L) + b * prow(KR); }
    // A fourth buffer, where LDS has room for it (one image per CU at widths 33..48, small models at widths <= 16):
    // the backward pass then restores the next layer's input while it works on this one, one barrier less per layer.
    static constexpr bool PIPE = MT == 1 || MT == 3;
    static __host__ __device__ constexpr int total(int L) { return buf(PIPE ? 4 : 3, L); }
};

// Adam steps one launch takes at most, and chunks of pixels a workgroup has in it if there is more than one step (a step of more is long enough by itself)
constexpr int kStepsAtOnce = 32, kChunksAtOnce = 1024;
struct FitStep { float lr, c1inv, c2inv; };

struct FitArgs {
    float *params, *m, *v;        // [n_images][n_params]
    const uint8_t *keep;          // [n_images][n_params] or null
    const float *target;          // [n_images][3][HW]
    float *loss;                  // [n_images]
    float *emag;                  // [n_images] root-mean-square output error the last step saw (split-precision kernel's error scale); may be null
    float *grad_out;              // null: Adam update; else the gradient is written here and nothing is updated
    float *part;                  // splits > 1: [n_images][splits][n_params + 1] partial gradients, and the squared error behind them
    int32_t splits;               // workgroups per image
    int64_t n_params;
    uint32_t HW, W;
    uint32_t wmagic, wshift;      // p / W == umulhi(p, wmagic) >> wshift for p < 2^31; wmagic == 0 means W == 1
    float inv2W, inv2H, lo, span, w0rev;        // w0rev = w0 / 2pi
    float loss_scale;
    float neg1;                   // -1, as data: keeps x - float(half) a single mixed-precision fma in the split kernels
    float b1, b2, eps;
    int32_t L;
    int32_t d[kMaxL + 1];         // true widths
    int32_t p_off[kMaxL];         // offset of W_l in the parameter vector
    float gscale[kMaxL];          // what the accumulated weight gradient of layer l is multiplied by (see the kernel)
    int32_t steps;                // Adam steps of this launch: one, or more of a kernel that takes several (fit16_many_steps)
    FitStep step[kStepsAtOnce];
};

// The chunks of an image's pixels that this workgroup takes: all of them, or its share where `splits` workgroups have one image.
struct FitShare { size_t img; uint32_t c0, c1; float *part; };
template <class Args> __device__ __forceinline__ FitShare fit_share(const Args &a, uint32_t nchunks) {
    const uint32_t img = blockIdx.x / (uint32_t)a.splits, sp = blockIdx.x - img * (uint32_t)a.splits;
    FitShare w;
    w.img = img;
    w.c0 = (uint32_t)((uint64_t)nchunks * sp / (uint32_t)a.splits);
    w.c1 = (uint32_t)((uint64_t)nchunks * (sp + 1) / (uint32_t)a.splits);
    w.part = a.splits > 1 ? a.part + (size_t)blockIdx.x * (size_t)(a.n_params + 1) : nullptr;
    return w;
}

// Squared error of the workgroup's pixels (`s`, one thread): the image's loss and error size, or this share's part of them.
template <class Args> __device__ __forceinline__ void fit_put_loss(const Args &a, const FitShare &w, float s) {
    if (w.part) {
        w.part[a.n_params] = s;
    } else {
        a.loss[w.img] = a.loss_scale * s;
        if (a.emag && !a.grad_out) a.emag[w.img] = sqrtf(s / (3.0f * (float)a.HW));
    }
}

// Adam's two moments.  Which product of a sum goes unrounded is written out: the compiler's choice differs from kernel to kernel, and with it a fit's bits.
template <class Args> __device__ __forceinline__ float adam_m(const Args &a, float m, float gr) { return fmaf(1.0f - a.b1, gr, a.b1 * m); }
template <class Args> __device__ __forceinline__ float adam_v(const Args &a, float v, float gr) { return fmaf((1.0f - a.b2) * gr, gr, a.b2 * v); }

// One gradient entry of an image: handed out, or Adam on the parameter in place (a pruned one stays 0).
template <class Args> __device__ __forceinline__ void fit_apply(const Args &a, size_t img, int at, float gr, int step) {
    const size_t q = img * (size_t)a.n_params + (size_t)at;
    const bool kept = !a.keep || a.keep[q];
    if (a.grad_out) {
        a.grad_out[q] = kept ? gr : 0.0f;
    } else if (kept) {
        const float mm = adam_m(a, a.m[q], gr);
        const float vv = adam_v(a, a.v[q], gr);
        a.m[q] = mm;
        a.v[q] = vv;
        a.params[q] -= a.step[step].lr * (mm * a.step[step].c1inv) / (sqrtf(vv * a.step[step].c2inv) + a.eps);
    } else {
        a.params[q] = 0.0f;
    }
}
template <class Args> __device__ __forceinline__ void fit_put_grad(const Args &a, const FitShare &w, int at, float gr, int step) {
    if (w.part) w.part[at] = gr;
    else fit_apply(a, w.img, at, gr, step);
}

// Four entries of an image at once (at < 0: none).  A share's part goes out first and waits for nothing.  For Adam, what it reads of all four is
// under way together (an entry at a time waits for memory twice for each, since the stores may be to what the next one loads), and all of it is used
// whether an entry is there or not: a load that some lanes leave unused is still under way where the ways meet again, and the wait for it there was a
// wait for the last tile's stores on every way, the share's too.  With that, and Adam's code five times behind every tile, us a step, before -> now:
// 4 images of 32 x 32, 5 x 64 39.1 -> 37.2, 30 of 64 x 64, 6 x 40 59.4 -> 57.6, one of 224 x 224, 10 x 32 43.5 -> 42.1, 2 of 128 x 128, 5 x 56 46.9
// -> 45.0; 8 of 171 x 219, 10 x 40 170.2 -> 168.0, 10 x 32 102.6 -> 100.9; unshared, 256 of 96 x 96: 9 x 48 974 -> 935, 8 x 40 736 -> 720, 7 x 24 523
// -> 523, 10 x 40 909 -> 914, 9 x 24 417 -> 423, 12 x 32 668 -> 676 and, where the compiler orders the code over the pixels the worse way for it, 9 x
// 40 810 -> 822, 5 x 64 705 -> 726.
template <class Args> __device__ __forceinline__ void fit_put_grads(const Args &a, const FitShare &w, const int (&at)[4], const float (&gr)[4], int step) {
    if (w.part) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (at[v] >= 0) w.part[at[v]] = gr[v];
        return;
    }
    const size_t first = w.img * (size_t)a.n_params;
    if (a.grad_out) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (at[v] >= 0) a.grad_out[first + (size_t)at[v]] = !a.keep || a.keep[first + (size_t)at[v]] ? gr[v] : 0.0f;
        return;
    }
    float m[4], s[4], p[4];
    bool kept[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const size_t q = first + (size_t)(at[v] < 0 ? 0 : at[v]);
        kept[v] = !a.keep || a.keep[q];
        m[v] = a.m[q];
        s[v] = a.v[q];
        p[v] = a.params[q];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        m[v] = adam_m(a, m[v], gr[v]);
        s[v] = adam_v(a, s[v], gr[v]);
        p[v] -= a.step[step].lr * (m[v] * a.step[step].c1inv) / (sqrtf(s[v] * a.step[step].c2inv) + a.eps);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (at[v] < 0) continue;
        const size_t q = first + (size_t)at[v];
        if (kept[v]) {
            a.m[q] = m[v];
            a.v[q] = s[v];
        }
        a.params[q] = kept[v] ? p[v] : 0.0f;
    }
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// acc += sum over KSTEPS k-steps of A(ks) x B(ks): one float per lane from LDS at ap[ks * AS], bp[ks * BS].
// Trip count and strides are compile-time, so the loads become immediate-offset reads issued ahead of the MFMAs
// (in groups of eight, which bounds the registers held).
// ZERO: the sum starts at 0 (as the first MFMA's inline-constant C operand: no registers are cleared).
template <int KSTEPS, int AS, int BS, bool ZERO>
__device__ __forceinline__ f32x4 contract(const float *ap, const float *bp, f32x4 acc) {
#pragma unroll
    for (int k0 = 0; k0 < KSTEPS; k0 += 8) {
        constexpr int G = 8;
        float av[G], bv[G];
#pragma unroll
        for (int u = 0; u < G; ++u)
            if (k0 + u < KSTEPS) {
                av[u] = ap[(k0 + u) * AS];
                bv[u] = bp[(k0 + u) * BS];
            }
#pragma unroll
        for (int u = 0; u < G; ++u)
            if (k0 + u < KSTEPS) acc = mfma4(av[u], bv[u], (ZERO && k0 + u == 0) ? (f32x4){0.0f, 0.0f, 0.0f, 0.0f} : acc);
    }
    return acc;
}

}  // namespace
#include "rinr_fit16.hip.h"
namespace {

// Where entry (o, i) of layer l's weight-gradient tile lives in the parameter vector, or -1 (padding).
// Column 0 is the bias; input j is column 1 + j of the first layer and column 4 + j of the others.
__device__ __forceinline__ int param_index(const FitArgs &a, int l, int o, int i) {
    const int din = a.d[l], dout = a.d[l + 1];
    if (o >= dout) return -1;
    if (i == 0) return a.p_off[l] + dout * din + o;
    const int j = i - (l == 0 ? 1 : 4);
    if (j >= 0 && j < din) return a.p_off[l] + o * din + j;
    return -1;
}

template <int WQ, int ML>
__global__ __launch_bounds__(Shape<WQ>::NTHREADS, fit_waves_per_simd(WQ)) void fit_step_kernel(const FitArgs a) {
    typedef Shape<WQ> S;
    constexpr int MT = S::MT, LD = S::LD, KR = S::KR, KSF = S::KSF, KSB = S::KSB, PC = S::PC, PT = S::PT, NIT = S::NIT;
    constexpr int PSTEP = 2 * S::PAIR;       // prow(r + 4) - prow(r): one k-step down a pixel buffer
    constexpr int ZSLOTS = S::ZSLOTS, GSLOTS = S::GSLOTS, kWaves = S::NW, kThreads = S::NTHREADS;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ float red[kWaves];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, m = lane & 15, kq = lane >> 4;
    // fit_share divides on the vector ALU; its results, the same in every lane, are taken out of the vector registers, where they
    // would stay over the whole kernel: 8 more of the deepest kernels' registers spilled (us a step, 256 images of 128 x 128:
    // 12 layers x 24 3732 -> 3709, 12 x 32 4597 -> 4562).  The split-precision kernels are not the better for it (10 x 32: 6010 -> 6090).
    FitShare share = fit_share(a, (a.HW + PC - 1) / PC);
    share.img = __builtin_amdgcn_readfirstlane((uint32_t)share.img);
    share.c0 = __builtin_amdgcn_readfirstlane(share.c0);
    share.c1 = __builtin_amdgcn_readfirstlane(share.c1);
    const size_t img = share.img;
    const float *P = a.params + img * a.n_params;
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr bool PIPE = S::PIPE;
    float *const B0 = lds + S::buf(0, a.L), *const B1 = lds + S::buf(1, a.L), *const B2 = lds + S::buf(2, a.L);
    float *const B3 = PIPE ? lds + S::buf(3, a.L) : B0;

    // ---- set up: zero everything, then the weights (sine layers times w0 / 2pi) behind their bias column
    for (int q = tid; q < S::total(a.L); q += kThreads) lds[q] = 0.0f;
    __syncthreads();
    for (int l = 0; l < a.L; ++l) {
        const int din = a.d[l], dout = a.d[l + 1], ld = l == 0 ? 6 : LD, first = l == 0 ? 1 : 4;
        float *Wt = lds + S::w_off(l);
        const float *src = P + a.p_off[l];
        const float sc = l < a.L - 1 ? a.w0rev : 1.0f;
        for (int e = tid; e < dout * din; e += kThreads) Wt[(e / din) * ld + first + e % din] = src[e] * sc;
        for (int o = tid; o < dout; o += kThreads) Wt[o * ld] = src[dout * din + o] * sc;
    }
    if (PIPE && tid < PC) B3[S::prow(0) + tid] = 1.0f;       // its row of ones; nothing else ever writes its rows 0..3
    __syncthreads();

    f32x4 acc[ML][GSLOTS];          // weight-gradient tiles, whole step
    f32x4 zst[ML][ZSLOTS];          // pre-activation tiles of the chunk at hand
#pragma unroll
    for (int l = 0; l < ML; ++l) {
#pragma unroll
        for (int s = 0; s < GSLOTS; ++s) acc[l][s] = zero4;
#pragma unroll
        for (int s = 0; s < ZSLOTS; ++s) zst[l][s] = zero4;
    }
    float loss_part = 0.0f;

    // rows ones, x, y, zero of B0: the first layer's input at the chunk's pixel centres (a ragged last chunk
    // repeats the last pixel; its error is zeroed)
    auto put_coords = [&](uint32_t c) {
        if (tid < PC) {
            uint32_t p = c * PC + tid;
            p = p < a.HW ? p : a.HW - 1;
            const uint32_t row = p / a.W, col = p - row * a.W;
            B0[S::prow(0) + tid] = 1.0f;
            B0[S::prow(1) + tid] = fmaf(a.span, (float)(2 * col + 1) * a.inv2W, a.lo);
            B0[S::prow(2) + tid] = fmaf(a.span, (float)(2 * row + 1) * a.inv2H, a.lo);
            B0[S::prow(3) + tid] = 0.0f;
        }
    };

    for (uint32_t c = share.c0; c < share.c1; ++c) {
        // the layer count is read afresh per chunk: otherwise every "l < L" and "l == L - 1" of the unrolled layers is
        // kept as a lane mask across the loop, and the masks spill out of the scalar registers
        int L = a.L;
        asm volatile("" : "+s"(L));
        put_coords(c);
        if (tid >= kThreads - PC) B1[S::prow(0) + tid - (kThreads - PC)] = 1.0f;     // the backward pass kept errors here
        __syncthreads();
        // ---- forward: Z_l = W_l H_l, one 16x16 tile (rows mt, pixels nt) per task; H_{l+1} = sin(2pi Z_l)
#pragma unroll
        for (int l = 0; l < ML; ++l) {
            if (l < L) {
                const bool last = l == L - 1;
                const float *in = (l & 1) ? B1 : B0;
                float *out = (l & 1) ? B0 : B1;
                const int ntasks = (last ? 1 : MT) * PT;
#pragma unroll
                for (int s = 0; s < ZSLOTS; ++s) {
                    const int task = wave + s * kWaves;
                    if (task < ntasks) {
                        const int mt = task / PT, nt = task - mt * PT, col = nt * 16 + m;
                        f32x4 z;
                        if (l == 0)
                            z = contract<1, 4, PSTEP, true>(lds + S::w_off(0) + (mt * 16 + m) * 6 + kq, in + S::prow(kq) + col, zero4);
                        else
                            z = contract<KSF, 4, PSTEP, true>(lds + S::w_off(l) + (mt * 16 + m) * LD + kq, in + S::prow(kq) + col, zero4);
                        if (!last) {
                            zst[l][s] = z;
#pragma unroll
                            for (int v = 0; v < 4; ++v) out[S::prow(4 + mt * 16 + 4 * kq + v) + col] = __builtin_amdgcn_sinf(z[v]);
                        } else {
                            const uint32_t pix = c * PC + col;
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int o = 4 * kq + v;
                                float e = 0.0f;
                                if (o < 3 && pix < a.HW) e = z[v] - a.target[(img * 3 + o) * a.HW + pix];
                                loss_part = fmaf(e, e, loss_part);
                                B2[S::prow(o) + col] = 2.0f * a.loss_scale * e;
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
        // ---- backward, layer by layer: restore H_l (the layer's input); then dW_l += E_l H_l^T into this wavefront's
        //      accumulators (tile rows ot, columns it) and E_{l-1} = (W_l^T E_l) * cos(2pi z_{l-1}) (tile rows it, pixels nt).
        //      With PIPE only the first of these layers restores its own input ahead; every layer restores the next one's
        //      into the other H buffer while it computes.
        auto restore = [&](int l, float *H) {          // l is a constant after unrolling
            if (l == 0) {
                put_coords(c);                         // B0, which is where layer 0's input is expected
            } else {
#pragma unroll
                for (int s = 0; s < ZSLOTS; ++s) {
                    const int task = wave + s * kWaves;
                    if (task < MT * PT) {
                        const int mt = task / PT, nt = task - mt * PT, col = nt * 16 + m;
#pragma unroll
                        for (int v = 0; v < 4; ++v) H[S::prow(4 + mt * 16 + 4 * kq + v) + col] = __builtin_amdgcn_sinf(zst[l - 1][s][v]);
                    }
                }
            }
        };
        float *Dc = B2, *Dn = B1;
#pragma unroll
        for (int l = ML - 1; l >= 0; --l) {
            if (l < L) {
                const bool last = l == L - 1;
                float *const Hc = (PIPE && (l & 1)) ? B3 : B0;      // holds H_l
                float *const Hn = (PIPE && !(l & 1)) ? B3 : B0;     // PIPE: receives H_{l-1}
                if (!PIPE || last) {
                    restore(l, Hc);
                    __syncthreads();
                }
                if (l == 0) {
#pragma unroll
                    for (int s = 0; s < GSLOTS; ++s) {
                        const int ot = wave + s * kWaves;        // columns ones, x, y; the other lanes read the zero row
                        if (ot < MT) acc[0][s] = contract<PC / 4, 4, 4, false>(Dc + S::prow(ot * 16 + m) + kq, Hc + S::prow(m < 4 ? m : 3) + kq, acc[0][s]);
                    }
                } else {
                    const int ntasks = (last ? 1 : MT) * NIT;
#pragma unroll
                    for (int s = 0; s < GSLOTS; ++s) {
                        const int task = wave + s * kWaves;
                        if (task < ntasks) {
                            const int ot = task / NIT, it = task - ot * NIT, i = it * 16 + m;
                            // columns beyond the buffer's rows read the buffer's zero row
                            acc[l][s] = contract<PC / 4, 4, 4, false>(Dc + S::prow(ot * 16 + m) + kq, Hc + S::prow(i < KR ? i : 3) + kq, acc[l][s]);
                        }
                    }
                    const float *Wt = lds + S::w_off(l);
#pragma unroll
                    for (int s = 0; s < ZSLOTS; ++s) {
                        const int task = wave + s * kWaves;
                        if (task < MT * PT) {
                            const int it = task / PT, nt = task - it * PT, col = nt * 16 + m;
                            const float *ap = Wt + kq * LD + 4 + it * 16 + m, *bp = Dc + S::prow(kq) + col;
                            const f32x4 g = last ? contract<1, 4 * LD, PSTEP, true>(ap, bp, zero4) : contract<KSB, 4 * LD, PSTEP, true>(ap, bp, zero4);
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                Dn[S::prow(it * 16 + 4 * kq + v) + col] = g[v] * __builtin_amdgcn_cosf(zst[l - 1][s][v]);
                        }
                    }
                    if (PIPE) restore(l - 1, Hn);
                }
                __syncthreads();
                float *t = Dc;
                Dc = Dn;
                Dn = t;
            }
        }
    }
    const int L = a.L;

    // ---- loss of this step's parameters
    for (int off = 32; off > 0; off >>= 1) loss_part += __shfl_xor(loss_part, off, 64);
    if (lane == 0) red[wave] = loss_part;
    __syncthreads();
    if (tid == 0) {
        float s = 0.0f;
        for (int w = 0; w < kWaves; ++w) s += red[w];
        fit_put_loss(a, share, s);
    }

    // ---- every gradient entry is in exactly one lane: Adam in place, or the entry handed out
#pragma unroll
    for (int l = 0; l < ML; ++l) {
        if (l < L) {
            const int nit = l == 0 ? 1 : NIT, ntasks = (l == L - 1 ? 1 : MT) * nit;
#pragma unroll
            for (int s = 0; s < GSLOTS; ++s) {
                const int task = wave + s * kWaves;
                if (task < ntasks) {
                    const int ot = task / nit, it = task - ot * nit;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int at = param_index(a, l, ot * 16 + 4 * kq + v, it * 16 + m);
                        if (at >= 0) fit_put_grad(a, share, at, acc[l][s][v] * a.gscale[l], 0);
                    }
                }
            }
        }
    }
}

// Where an image's pixels are shared by several workgroups: the sum of their partial gradients and squared errors (in a
// fixed order, so that a step is reproducible), then the update.  GROUPS threads share a parameter's sum (each takes every
// GROUPS-th share), so that a long sum is not one thread's chain of loads.  Bound by reading the partial gradients once.
constexpr int kReduceParams = 64;       // parameters per workgroup
template <int GROUPS>
__global__ __launch_bounds__(kReduceParams *GROUPS) void fit_reduce_kernel(const FitArgs a) {
    __shared__ float red[GROUPS][kReduceParams];
    const int lane = threadIdx.x % kReduceParams, grp = threadIdx.x / kReduceParams;
    const size_t img = blockIdx.y, stride = (size_t)a.n_params + 1;
    const int64_t at = (int64_t)blockIdx.x * kReduceParams + lane;              // n_params is the squared error's place
    const float *src = a.part + img * (size_t)a.splits * stride;
    float s0 = 0.0f, s1 = 0.0f;
    if (at <= a.n_params) {
        int k = grp;
        for (; k + GROUPS < a.splits; k += 2 * GROUPS) {
            s0 += src[(size_t)k * stride + at];
            s1 += src[(size_t)(k + GROUPS) * stride + at];
        }
        if (k < a.splits) s0 += src[(size_t)k * stride + at];
    }
    red[grp][lane] = s0 + s1;
    __syncthreads();
    if (grp == 0 && at <= a.n_params) {
        float g = 0.0f;
#pragma unroll
        for (int w = 0; w < GROUPS; ++w) g += red[w][lane];
        if (at < a.n_params) {
            fit_apply(a, img, (int)at, g, 0);
        } else {
            a.loss[img] = a.loss_scale * g;
            if (!a.grad_out) a.emag[img] = sqrtf(g / (3.0f * (float)a.HW));
        }
    }
}

typedef void (*fit_fn)(const FitArgs);

template <int WQ> fit_fn kernel_of(int L) {
    if (L <= fit_depth_lo(WQ)) return fit_step_kernel<WQ, fit_depth_lo(WQ)>;
    return fit_step_kernel<WQ, fit_depth_hi(WQ)>;
}
// wq: the widest hidden layer rounded up to a multiple of 8
fit_fn kernel_for(int wq, int L) {
    switch (wq) {
        case 8: return kernel_of<8>(L);
        case 16: return kernel_of<16>(L);
        case 24: return kernel_of<24>(L);
        case 32: return kernel_of<32>(L);
        case 40: return kernel_of<40>(L);
        case 48: return kernel_of<48>(L);
        case 56: return kernel_of<56>(L);
        default: return kernel_of<64>(L);
    }
}
template <int WQ> int lds_floats_of(int L) { return L <= Shape<WQ>::ML ? Shape<WQ>::total(L) : 0; }
// LDS floats of a model of L linear layers at rounded width wq, or 0 if no kernel is built that deep
int lds_floats(int wq, int L) {
    switch (wq) {
        case 8: return lds_floats_of<8>(L);
        case 16: return lds_floats_of<16>(L);
        case 24: return lds_floats_of<24>(L);
        case 32: return lds_floats_of<32>(L);
        case 40: return lds_floats_of<40>(L);
        case 48: return lds_floats_of<48>(L);
        case 56: return lds_floats_of<56>(L);
        default: return lds_floats_of<64>(L);
    }
}


// ---- the split-precision kernels (rinr_fit16.hip.h): built per hidden width rounded up to a multiple of 16 and per depth
constexpr int fit16_depth(int wp) { return wp <= 32 ? kMaxL : (wp == 48 ? 10 : 6); }
// 16-pixel tiles a wavefront takes at a time: one where that leaves registers for a second wavefront per SIMD and two do not,
// else two where the registers hold them (a lone wavefront has only its own two tiles to fill the gaps between dependent instructions).
constexpr int fit16_tiles(int wp, int ml) {
    const int one = fit16::fit16_waves_per_simd(wp, ml, 1), two = fit16::fit16_waves_per_simd(wp, ml, 2);
    return (one > 1 && two == 1) || fit16::fit16_registers(wp, ml, 2) > 512 ? 1 : 2;
}
// The kernel, and the one that takes several steps a launch (or null); LDS bytes and pixels a workgroup takes at a time of either
struct Fit16 { fit_fn fn, many; uint32_t lds; int pixels; };
template <int WP, bool HALF, int L, int NT> constexpr fit_fn many_of() {
    if constexpr (fit16::fit16_many_steps(WP, L, NT)) return fit16::fit16_step_kernel<WP, HALF, L, NT, true>;
    else return nullptr;
}
template <int WP, bool HALF, int L = 2> Fit16 kernel16_of(int n) {
    if constexpr (L > fit16_depth(WP)) {
        return Fit16{nullptr, nullptr, 0, 0};
    } else {
        constexpr int nt = fit16_tiles(WP, L);
        if constexpr (WP == 64 && HALF && L <= 3) return kernel16_of<WP, HALF, L + 1>(n);
        else if (n != L) return kernel16_of<WP, HALF, L + 1>(n);
        else return Fit16{fit16::fit16_step_kernel<WP, HALF, L, nt, false>, many_of<WP, HALF, L, nt>(), fit16::Shape<WP, HALF>::total(L, nt), fit16::kThreads / 4 * nt};
    }
}
// width: of the widest hidden layer.  Half of the last tile empty: the kernels that do not compute it (fit16::Shape), but for one that spills and is
// the slower for it (256 images of 96 x 96, 3 layers x 56: 318 us a step instead of 310).
bool half_filled(int width, int L) {
    const int wp = (width + 15) / 16 * 16;
    return width <= wp - 8 && !(wp == 64 && L <= 3);
}
// Pixels of a workgroup's share from which they pay: a step's start and end, the same for any share, are longer in them.  us a step of one image
// of 25 x 17, all units of the last tile -> the half-filled tile's kernel: 10 layers x 24 29.3 -> 32.4, 4 x 40 19.2 -> 21.3, 6 x 49 39.5 -> 45.0,
// and of 300 of 32 x 32 (512 pixels a share): 163 -> 161, 92.9 -> 90.0, 259 -> 273; 8 of 171 x 219 (1216), 4 x 56: 97.9 -> 94.1, 6 x 56:
// 162.8 -> 165.8.  Up to 8 units they are the faster ones from 8 x 8 pixels.  1024 images, one share each, of 256 pixels: 2 layers x 40 26.1 -> 24.4, 4 x 40
// 85.6 -> 83.4, 10 x 40 446 -> 405, 3 x 24 34.4 -> 31.9, 7 x 24 90.0 -> 85.5.  Models of 17 to 24 units and 8 layers or more leave no registers for
// a wavefront more than whole tiles do, and gain later: 8 x 24 at 256, 384, 448, 512 pixels 103.3 -> 104.3, 122.8 -> 123.5, 133.1 -> 132.3, 143.6 -> 141.7;
// 9, 10 and 11 layers at 256 171.5 -> 173.3, 192.3 -> 195.6, 211.9 -> 214.1, at 320 198.7 -> 195.7, 221.9 -> 220.3, 245.0 -> 242.2.
int64_t half_pays_from(int width, int L) {
    if (width <= 8) return 0;
    if (width <= 24 && L >= 8) return L == 8 ? 448 : 257;
    return width <= 40 ? 256 : 832 * (L - 3);
}
Fit16 kernel16_for(int width, int L, bool half) {
    const int wp = (width + 15) / 16 * 16;
    const Fit16 k = half ? (wp == 16 ? kernel16_of<16, true>(L) : (wp == 32 ? kernel16_of<32, true>(L) : (wp == 48 ? kernel16_of<48, true>(L) : kernel16_of<64, true>(L))))
                         : (wp == 16 ? kernel16_of<16, false>(L) : (wp == 32 ? kernel16_of<32, false>(L) : (wp == 48 ? kernel16_of<48, false>(L) : kernel16_of<64, false>(L))));
    return k.lds <= kLdsLimit - 256 ? k : Fit16{nullptr, nullptr, 0, 0};
}

}  // namespace

struct rinr_fit {
    rinr_fit_arch arch;
    int64_t n_images, n_params;
    int32_t H, W;
    int wq, lds_floats;         // wq: widest hidden layer rounded up to a multiple of 8 (fp32 kernels); lds_floats 0 = no fp32 kernel fits
    int family;                 // RINR_FIT_KERNEL_FP32 or RINR_FIT_KERNEL_SPLIT16: the kernels this handle's steps run
    Fit16 k16;                  // their kernels; null = none is built for the shape
    int most;                   // Adam steps that a launch takes; more than one: of k16.many
    int units;                  // of a hidden layer that the handle's kernel computes (rinr_fit_kernel_units)
    float *emag;                // [n_images] error size seen by the last step (split kernels' error scale); 0 = none yet
    int32_t p_off[kMaxL];
    float *params, *m, *v, *loss, *scratch_grad;
    float *part;              // partial gradients, where an image's pixels are shared by several workgroups
    int splits;               // ... that many
    uint8_t *keep;            // null until set
    bool has_keep;
    int64_t t;                // Adam steps taken
    int device;               // where all of it is
};

namespace {
// Adam steps that a launch takes of an image that one workgroup has
int most_steps(const rinr_fit *f) {
    if (f->family != RINR_FIT_KERNEL_SPLIT16 || !f->k16.many) return 1;
    const int64_t chunks = ((int64_t)f->H * f->W + f->k16.pixels - 1) / f->k16.pixels;
    return (int)std::max<int64_t>(1, std::min<int64_t>(kStepsAtOnce, kChunksAtOnce / chunks));
}
// Dynamic LDS beyond the default for a handle's kernels
bool may_use_lds(const Fit16 &k) {
    const int most = (int)kLdsLimit - 256;
    return !hip_fail(hipFuncSetAttribute((const void *)k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, most)) &&
           (!k.many || !hip_fail(hipFuncSetAttribute((const void *)k.many, hipFuncAttributeMaxDynamicSharedMemorySize, most)));
}
// Workgroups per image.  One workgroup per image updates it in the same launch; where the images alone leave the machine
// idle (few of them, or a last round that is nearly empty), an image's pixels are shared by several, and a second kernel
// adds their partial gradients up.  The model: rounds of workgroups x (a share's chunks + what a workgroup costs before its
// first chunk, about two chunks' time), and for more than one share the second launch, about one chunk more.  Measured
// (8 images of 171 x 219, 10 layers x 32): 3241 us a step with one workgroup per image, 101 with 30.
// Where a launch takes several steps of an unshared image, and no second launch, the second launch of a shared one weighs more: it takes 5 to 11 us,
// and a chunk of 128 pixels 1.1 us at 2 layers x 15, 1.6 at 3 x 15, 1.8 at 2 x 32, 2.3 at 3 x 32, 2.5 at 4 and 5 x 15, 3.6 at 8 x 15.  That gives
// what it weighs in chunks.  us a step, shared -> a workgroup an image in launches of 32 steps, and one step a call: 300 images of 32 x 32, 2 x 8
// 13.6 -> 10.8, 13.4; 64 of 24 x 24, 2 x 15 10.7 -> 7.7, 10.0; 1000 of 40 x 40, 7 x 15 147 -> 120, 123; 700, 3 x 32 92.5 -> 72.9, 75.0; 600 of 32 x
// 32, 8 x 15 83.7 -> 74.0, 76.7.  Five chunks for all of them are too much for deeper models: 64 of 24 x 24, 4 x 15 13.8 -> 14.2, 16.5, 5 x 15 15.5
// -> 17.1, 19.5, 8 x 15 20.8 -> 24.9, 27.4; 128 of 28 x 28, 6 x 15 21.8 -> 24.5, 27.1, 3 x 32 19.5 -> 20.6, 22.8; 800 of 64 x 64, 8 x 15 288 -> 312,
// 307.  The plan is the handle's, whatever the steps of a call, so that a fit's bits do not depend on how its steps are cut into calls; one step a
// call loses most at 700 of 64 x 64, 2 x 15: 57.0 -> 58.9, in launches of 32 56.5.  What the rule leaves shared although launches of 32 are the
// faster: 1100 of 48 x 48, 3 x 32 160 -> 155, 154; 300 of 32 x 32, 5 x 8 23.0 -> 22.2, 25.3.
int plan_splits(const rinr_fit *f) {
    const bool split16 = f->family == RINR_FIT_KERNEL_SPLIT16;
    const int waves = split16 ? fit16::kWaves : fit_waves(f->wq);
    const size_t lds = split16 ? (size_t)f->k16.lds : (size_t)f->lds_floats * 4;
    const int64_t pc = split16 ? f->k16.pixels : 64, chunks = ((int64_t)f->H * f->W + pc - 1) / pc;
    int device = 0, cus = 256;
    if (hip_fail(hipGetDevice(&device)) || hip_fail(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device)) || cus < 1) cus = 256;
    // workgroups that run side by side without slowing each other much: four wavefronts per SIMD
    auto side_by_side = [&](const void *fn) {
        int resident = 1;
        if (hip_fail(hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, fn, 64 * waves, lds)) || resident < 1) resident = 1;
        return (int64_t)cus * std::min(resident, std::max(1, 16 / waves));
    };
    const bool many = most_steps(f) > 1;
    const int64_t shared = side_by_side(split16 ? (const void *)f->k16.fn : (const void *)kernel_for(f->wq, f->arch.n_layers));
    const int64_t alone = many ? side_by_side((const void *)f->k16.many) : shared;
    const int L = f->arch.n_layers;
    const int64_t second = !many ? 1 : (L >= 8 ? 2 : (L >= 4 ? 3 : (L == 3 && f->wq > 16 ? 4 : 5)));
    if (f->n_images >= 16 * alone) return 1;           // many rounds: the last one's idle part does not matter
    int64_t best = 1, best_t = INT64_MAX;
    for (int64_t s = 1; s <= chunks && s <= 1024; ++s) {
        const int64_t slots = s > 1 ? shared : alone, rounds = (f->n_images * s + slots - 1) / slots;
        const int64_t t = rounds * ((chunks + s - 1) / s + 2) + (s > 1 ? second : 0);
        if (t < best_t) { best_t = t; best = s; }
        if (f->n_images * s > 8 * slots) break;
    }
    return (int)best;
}
}  // namespace

extern "C" int rinr_fit_create_ex(const rinr_fit_arch *arch, int64_t n_images, int32_t H, int32_t W, uint32_t flags, rinr_fit **out) {
    if (!arch || !out) return RINR_E_NULL;
    *out = nullptr;
    if (arch->n_layers < 2 || arch->n_layers > kMaxL || n_images < 0 || H <= 0 || W <= 0) return RINR_E_ARG;
    if (flags & ~(uint32_t)RINR_FIT_FLAG_FP32_MFMA) return RINR_E_ARG;
    if ((int64_t)H * W >= ((int64_t)1 << 31) || n_images > ((int64_t)1 << 31) - 1) return RINR_E_SIZE;
    if (arch->widths[0] != 2 || arch->widths[arch->n_layers] != 3) return RINR_E_ARG;
    for (int l = 1; l < arch->n_layers; ++l)
        if (arch->widths[l] < 1 || arch->widths[l] > RINR_MAX_WIDTH) return RINR_E_ARG;
    if (!(arch->coord_hi > arch->coord_lo) || !std::isfinite(arch->w0) || !std::isfinite(arch->coord_lo) ||
        !std::isfinite(arch->coord_hi))
        return RINR_E_ARG;
    rinr_fit *f = new (std::nothrow) rinr_fit();
    if (!f) return RINR_E_SIZE;
    f->arch = *arch;
    if (hip_fail(hipGetDevice(&f->device))) f->device = 0;       // no GPU: the allocations below say so
    f->n_images = n_images;
    f->H = H;
    f->W = W;
    int wmax = 1;
    for (int l = 1; l < arch->n_layers; ++l) wmax = arch->widths[l] > wmax ? arch->widths[l] : wmax;
    f->wq = (wmax + 7) / 8 * 8;
    f->lds_floats = lds_floats(f->wq, arch->n_layers);
    if ((size_t)f->lds_floats * 4 + 256 > kLdsLimit) f->lds_floats = 0;
    const bool half = half_filled(wmax, arch->n_layers);
    f->k16 = kernel16_for(wmax, arch->n_layers, half);
    // the split-precision kernels where they are built for the shape, the fp32 ones otherwise or on request
    f->family = (f->k16.fn && !(flags & RINR_FIT_FLAG_FP32_MFMA)) ? RINR_FIT_KERNEL_SPLIT16 : RINR_FIT_KERNEL_FP32;
    if (f->family == RINR_FIT_KERNEL_FP32 && f->lds_floats == 0) { delete f; return RINR_E_UNSUPPORTED; }
    f->units = f->family == RINR_FIT_KERNEL_FP32 || half ? f->wq : (wmax + 15) / 16 * 16;
    f->n_params = 0;
    for (int l = 0; l < arch->n_layers; ++l) {
        f->p_off[l] = (int32_t)f->n_params;
        f->n_params += (int64_t)arch->widths[l + 1] * (arch->widths[l] + 1);
    }
    const size_t ni = (size_t)(n_images > 0 ? n_images : 1);
    const size_t np = ni * (size_t)f->n_params;
    f->params = f->m = f->v = f->loss = f->scratch_grad = f->emag = f->part = nullptr;
    f->keep = nullptr;
    f->has_keep = false;
    f->t = 0;
    if (hip_fail(hipMalloc((void **)&f->params, np * 4)) || hip_fail(hipMalloc((void **)&f->m, np * 4)) ||
        hip_fail(hipMalloc((void **)&f->v, np * 4)) || hip_fail(hipMalloc((void **)&f->keep, np)) ||
        hip_fail(hipMalloc((void **)&f->loss, ni * 4)) || hip_fail(hipMalloc((void **)&f->emag, ni * 4)) ||
        hip_fail(hipMemset(f->params, 0, np * 4)) || hip_fail(hipMemset(f->m, 0, np * 4)) ||
        hip_fail(hipMemset(f->v, 0, np * 4)) || hip_fail(hipMemset(f->loss, 0, ni * 4)) || hip_fail(hipMemset(f->emag, 0, ni * 4)) ||
        !may_use_lds(f->family == RINR_FIT_KERNEL_SPLIT16 ? f->k16 : Fit16{kernel_for(f->wq, arch->n_layers), nullptr, 0, 0})) {
        rinr_fit_destroy(f);
        return RINR_E_HIP;
    }
    f->splits = plan_splits(f);
    if (half && f->family == RINR_FIT_KERNEL_SPLIT16 && ((int64_t)H * W + f->splits - 1) / f->splits < half_pays_from(wmax, arch->n_layers)) {
        const Fit16 k = kernel16_for(wmax, arch->n_layers, false);
        if (k.fn && may_use_lds(k)) {
            f->k16 = k;
            f->units = (wmax + 15) / 16 * 16;
            f->splits = plan_splits(f);
        }
    }
    // no memory for the partial gradients: a workgroup takes a whole image, and the refusal is not left for the first launch's check
    if (f->splits > 1 && hip_fail(hipMalloc((void **)&f->part, ni * (size_t)f->splits * (size_t)(f->n_params + 1) * 4))) {
        f->part = nullptr;
        f->splits = 1;
        (void)hipGetLastError();
    }
    f->most = f->splits == 1 ? most_steps(f) : 1;
    *out = f;
    return RINR_OK;
}

extern "C" int rinr_fit_create(const rinr_fit_arch *arch, int64_t n_images, int32_t H, int32_t W, rinr_fit **out) {
    return rinr_fit_create_ex(arch, n_images, H, W, 0u, out);
}

extern "C" int rinr_fit_kernel_family(const rinr_fit *f) { return f ? f->family : RINR_E_NULL; }
extern "C" int rinr_fit_kernel_units(const rinr_fit *f) { return f ? f->units : RINR_E_NULL; }

extern "C" int rinr_fit_destroy(rinr_fit *f) {
    if (!f) return RINR_OK;
    (void)hipFree(f->params);
    (void)hipFree(f->m);
    (void)hipFree(f->v);
    (void)hipFree(f->keep);
    (void)hipFree(f->loss);
    (void)hipFree(f->scratch_grad);
    (void)hipFree(f->emag);
    (void)hipFree(f->part);
    delete f;
    return RINR_OK;
}

extern "C" int64_t rinr_fit_n_params(const rinr_fit *f) { return f ? f->n_params : -1; }

namespace {
// Start of a fit or of a round of it: pruned parameters are zero (`keep`, may be null), the moments (`m`, `v`, may be null) and the
// error's history are cleared.  One pass over the handle's state where there were three fills and, with a mask, a way to the host and
// back for mask and parameters (8 images, 10 layers x 32, masked: 8 steps with their upload and read-back 1019 -> 942 us).
__global__ __launch_bounds__(256) void fit_start_kernel(float *params, float *m, float *v, float *emag, const uint8_t *keep, int64_t np, int64_t n_images) {
    const int64_t stride = (int64_t)gridDim.x * 256, first = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float4 none = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int64_t q = first; q < np / 4; q += stride) {              // the arrays are whole allocations: aligned
        if (m) {
            ((float4 *)m)[q] = none;
            ((float4 *)v)[q] = none;
        }
        if (keep) {
            const uchar4 k = ((const uchar4 *)keep)[q];
            float4 p = ((float4 *)params)[q];
            p.x = k.x ? p.x : 0.0f;
            p.y = k.y ? p.y : 0.0f;
            p.z = k.z ? p.z : 0.0f;
            p.w = k.w ? p.w : 0.0f;
            ((float4 *)params)[q] = p;
        }
    }
    for (int64_t i = np / 4 * 4 + first; i < np; i += stride) {
        if (m) m[i] = v[i] = 0.0f;
        if (keep && !keep[i]) params[i] = 0.0f;
    }
    for (int64_t i = first; i < n_images; i += stride) emag[i] = 0.0f;
}
// Makes a GPU the current one for the calls that follow, and the one before it again at the end
struct OnDevice {
    int was = -1;
    bool switched = false;
    int to(int device) {
        FIT_HIP(hipGetDevice(&was));
        if (was == device) return RINR_OK;
        FIT_HIP(hipSetDevice(device));
        switched = true;
        return RINR_OK;
    }
    ~OnDevice() { if (switched) (void)hipSetDevice(was); }
};
// Called with the handle's GPU current, as its uploads are; complete when it returns, whatever stream the next call is given.
int fit_start(rinr_fit *f, bool moments, bool mask) {
    const int64_t np = f->n_images * f->n_params;
    if (f->n_images == 0) return RINR_OK;
    const uint32_t blocks = (uint32_t)std::min<int64_t>((np / 4 + 255) / 256 + 1, 2048);
    hipLaunchKernelGGL(fit_start_kernel, dim3(blocks), dim3(256), 0, (hipStream_t) nullptr, f->params, moments ? f->m : nullptr,
                       moments ? f->v : nullptr, f->emag, mask ? f->keep : nullptr, np, f->n_images);
    FIT_HIP(hipGetLastError());
    FIT_HIP(hipStreamSynchronize(nullptr));
    return RINR_OK;
}
}  // namespace

// The three calls that overwrite a handle's state wait for all work on its GPU first, whatever GPU is current: a caller that holds handles
// on several need not switch to upload.
extern "C" int rinr_fit_reset_optimizer(rinr_fit *f) {
    if (!f) return RINR_E_NULL;
    OnDevice on;
    if (const int rc = on.to(f->device)) return rc;
    FIT_HIP(hipDeviceSynchronize());
    const int rc = fit_start(f, true, false);      // a new round: no moments, no error history
    if (rc) return rc;
    f->t = 0;
    return RINR_OK;
}

extern "C" int rinr_fit_set_params(rinr_fit *f, const float *params) {
    if (!f || (!params && f->n_images > 0)) return RINR_E_NULL;
    const size_t np = (size_t)f->n_images * (size_t)f->n_params;
    OnDevice on;
    if (const int rc = on.to(f->device)) return rc;
    FIT_HIP(hipDeviceSynchronize());
    if (np) FIT_HIP(hipMemcpy(f->params, params, np * 4, hipMemcpyHostToDevice));
    const int rc = fit_start(f, true, f->has_keep);
    if (rc) return rc;
    f->t = 0;
    return RINR_OK;
}

extern "C" int rinr_fit_set_keep(rinr_fit *f, const uint8_t *keep) {
    if (!f) return RINR_E_NULL;
    const size_t np = (size_t)f->n_images * (size_t)f->n_params;
    OnDevice on;
    if (const int rc = on.to(f->device)) return rc;
    FIT_HIP(hipDeviceSynchronize());
    if (np && keep) FIT_HIP(hipMemcpy(f->keep, keep, np, hipMemcpyHostToDevice));
    f->has_keep = keep != nullptr;
    return fit_start(f, false, f->has_keep);
}

extern "C" int rinr_fit_get_params(const rinr_fit *f, float *params, void *stream) {
    if (!f || (!params && f->n_images > 0)) return RINR_E_NULL;
    const size_t np = (size_t)f->n_images * (size_t)f->n_params;
    FIT_HIP(hipStreamSynchronize((hipStream_t)stream));
    if (np) FIT_HIP(hipMemcpy(params, f->params, np * 4, hipMemcpyDeviceToHost));
    return RINR_OK;
}

namespace {
// The steps `steps` at rates lr[0 ..], the first of them the handle's `t`-th
int launch(rinr_fit *f, const float *targets, float loss_scale, const float *lr, int steps, int64_t t, float b1, float b2, float eps,
           float *grad_out, hipStream_t stream) {
    FitArgs a;
    a.params = f->params; a.m = f->m; a.v = f->v;
    a.keep = f->has_keep ? f->keep : nullptr;
    a.target = targets;
    a.loss = f->loss;
    a.emag = f->emag;
    a.grad_out = grad_out;
    a.part = f->part;
    a.splits = f->splits;
    a.n_params = f->n_params;
    a.HW = (uint32_t)(f->H * f->W);
    a.W = (uint32_t)f->W;
    uint32_t bits = 0;
    while ((1ull << bits) < (uint64_t)f->W) ++bits;
    a.wmagic = bits ? (uint32_t)((((uint64_t)1 << (31 + bits)) + (uint64_t)f->W - 1) / (uint64_t)f->W) : 0u;
    a.wshift = bits ? bits - 1 : 0u;
    a.inv2W = 1.0f / (2.0f * (float)f->W);
    a.inv2H = 1.0f / (2.0f * (float)f->H);
    a.lo = f->arch.coord_lo;
    a.span = f->arch.coord_hi - f->arch.coord_lo;
    a.w0rev = (float)((double)f->arch.w0 / (2.0 * 3.14159265358979323846));
    a.loss_scale = loss_scale;
    a.neg1 = -1.0f;
    {
        const int L = f->arch.n_layers;
        double c = 1.0;                                   // 1 / c_l
        for (int l = L - 1; l >= 0; --l) {
            a.gscale[l] = (float)c;
            c = l == L - 1 ? (double)f->arch.w0 : c * 2.0 * 3.14159265358979323846;
        }
    }
    a.steps = steps;
    for (int k = 0; k < steps; ++k)
        a.step[k] = FitStep{lr[k], (float)(1.0 / (1.0 - std::pow((double)b1, (double)(t + k)))), (float)(1.0 / (1.0 - std::pow((double)b2, (double)(t + k))))};
    a.b1 = b1; a.b2 = b2; a.eps = eps;
    a.L = f->arch.n_layers;
    for (int l = 0; l <= a.L; ++l) a.d[l] = f->arch.widths[l];
    for (int l = 0; l < a.L; ++l) a.p_off[l] = f->p_off[l];
    if (f->family == RINR_FIT_KERNEL_SPLIT16)
        hipLaunchKernelGGL(f->most > 1 ? f->k16.many : f->k16.fn, dim3((uint32_t)(f->n_images * f->splits)), dim3(fit16::kThreads), (size_t)f->k16.lds, stream, a);
    else
        hipLaunchKernelGGL(kernel_for(f->wq, f->arch.n_layers), dim3((uint32_t)(f->n_images * f->splits)), dim3(64 * fit_waves(f->wq)), (size_t)f->lds_floats * 4, stream, a);
    FIT_HIP(hipGetLastError());
    if (f->splits > 1) {
        const dim3 grid((uint32_t)(f->n_params / kReduceParams + 1), (uint32_t)f->n_images);
        if (f->splits <= 16) hipLaunchKernelGGL(fit_reduce_kernel<4>, grid, dim3(kReduceParams * 4), 0, stream, a);
        else hipLaunchKernelGGL(fit_reduce_kernel<16>, grid, dim3(kReduceParams * 16), 0, stream, a);
        FIT_HIP(hipGetLastError());
    }
    return RINR_OK;
}
}  // namespace

extern "C" int rinr_fit_steps(rinr_fit *f, const float *targets, int32_t n_steps, const rinr_fit_opts *o, void *stream) {
    if (!f || !o || (!targets && f->n_images > 0)) return RINR_E_NULL;
    if (n_steps < 0 || !(o->lr >= 0.0f) || o->t0 < 0) return RINR_E_ARG;
    if (((uintptr_t)targets & 3) != 0) return RINR_E_ALIGN;
    const float b1 = o->beta1 != 0.0f ? o->beta1 : 0.9f, b2 = o->beta2 != 0.0f ? o->beta2 : 0.999f;
    const float eps = o->eps != 0.0f ? o->eps : 1e-8f;
    if (!(b1 > 0.0f && b1 < 1.0f && b2 > 0.0f && b2 < 1.0f && eps > 0.0f) || !(o->loss_scale >= 0.0f)) return RINR_E_ARG;
    const float ls = o->loss_scale != 0.0f ? o->loss_scale : (float)(1.0 / (3.0 * (double)f->H * (double)f->W));
    if (f->n_images == 0) { f->t += n_steps; return RINR_OK; }
    for (int32_t i = 0; i < n_steps;) {
        float rates[kStepsAtOnce];
        int32_t k = 0;
        for (; k < f->most && i + k < n_steps; ++k) {
            double lr = o->lr;
            if (o->T > 0) lr = 0.5 * lr * (1.0 + std::cos(3.14159265358979323846 * (double)(o->t0 + i + k) / (double)o->T));
            rates[k] = (float)lr;
        }
        const int rc = launch(f, targets, ls, rates, k, f->t + 1, b1, b2, eps, nullptr, (hipStream_t)stream);
        f->t += rc ? 1 : k;
        if (rc) return rc;
        i += k;
    }
    return RINR_OK;
}

extern "C" int rinr_fit_loss_grad(rinr_fit *f, const float *targets, float loss_scale, float *loss, float *grad, void *stream) {
    if (!f || !loss || (!targets && f->n_images > 0)) return RINR_E_NULL;
    if (((uintptr_t)targets & 3) != 0) return RINR_E_ALIGN;
    if (!(loss_scale >= 0.0f)) return RINR_E_ARG;
    if (f->n_images == 0) return RINR_OK;
    const size_t np = (size_t)f->n_images * (size_t)f->n_params;
    if (!f->scratch_grad) FIT_HIP(hipMalloc((void **)&f->scratch_grad, np * 4));
    const float ls = loss_scale != 0.0f ? loss_scale : (float)(1.0 / (3.0 * (double)f->H * (double)f->W));
    const float none = 0.0f;
    const int rc = launch(f, targets, ls, &none, 1, 1, 0.9f, 0.999f, 1e-8f, f->scratch_grad, (hipStream_t)stream);
    if (rc) return rc;
    FIT_HIP(hipStreamSynchronize((hipStream_t)stream));
    FIT_HIP(hipMemcpy(loss, f->loss, (size_t)f->n_images * 4, hipMemcpyDeviceToHost));
    if (grad) FIT_HIP(hipMemcpy(grad, f->scratch_grad, np * 4, hipMemcpyDeviceToHost));
    return RINR_OK;
}

extern "C" int rinr_fit_last_loss(const rinr_fit *f, float *loss, void *stream) {
    if (!f || (!loss && f->n_images > 0)) return RINR_E_NULL;
    FIT_HIP(hipStreamSynchronize((hipStream_t)stream));
    if (f->n_images) FIT_HIP(hipMemcpy(loss, f->loss, (size_t)f->n_images * 4, hipMemcpyDeviceToHost));
    return RINR_OK;
}

// ---- PSNR per image: a streaming reduction, bound by HBM (8 bytes read per element) where there are images enough to fill the GPU.  A workgroup
// reads about 0.1 TB/s, so fewer than 128 images of 131072 elements or more are shared by several workgroups each, which leave their sums in the
// caller's workspace, where there is one, and a second small kernel adds them up.  us a call, before -> now, images of 224 x 224: 1 14.8 -> 12.2, 64
// 26.8 -> 16.9, 300 82.0 -> 74.2; of 512 x 512: 1 67.6 -> 12.1, 8 117 -> 16.0; rows that begin anywhere in a 16-byte word: 100 of 333 x 211 105.8 ->
// 34.2, 2000 of 73 x 73 50.3 -> 43.7; 4096 of 16 x 16 15.8 -> 7.7.  Sharing takes the host 12 us for a call instead of 7: below 131072 elements, or
// from 128 images on (200 of 224 x 224: 41.1 alone, 45.3 shared), it does not pay.  Inside that it always does for images that no cache holds; the
// same images again, one call after the other, are up to 3 us slower for it where they are small and few, or 80 and more.  One workgroup each
// -> shared, new images, and the same again: 1 of 210 x 210 13.6 -> 12.5, 9.3 -> 12.5; of 224 x 224 15.2 -> 12.5, 10.3 -> 12.4; 16 25.8 -> 12.8, 10.6 -> 12.6; 1 of 256 x 256 19.2 ->
// 12.6, 12.6 -> 12.6; 64 37.3 -> 21.1, 21.6 -> 18.1; 100 37.3 -> 32.0, 23.5 -> 25.5; 110 38.1 -> 36.2, 25.2 -> 28.5; 127 of 512 x 512 152 -> 144, 152
// -> 143.
namespace {
constexpr int kPsnrThreads = 1024;
constexpr int64_t kPsnrSmall = 4096, kPsnrShared = 131072, kPsnrShare = 16384;      // elements of an image for 256 threads; to share; of a share, at least
// workgroups per image, with a workspace
int64_t psnr_splits(int64_t n_images, int64_t elems) {
    if (n_images < 1 || n_images >= 128 || elems < kPsnrShared) return 1;
    return std::min((512 + n_images - 1) / n_images, elems / kPsnrShare);
}

// Sum of squared differences of `elems` elements over the workgroup; thread 0 has it.  AHEAD pairs of loads are under way in a thread: one where each
// workgroup has a CU to itself (256 images of 224 x 224: 51.4 us, with two 52.3), else two (300: 82.0 and 74.2; 512 of 128 x 128: 37.0 and 35.2).
template <int THREADS, int AHEAD> __device__ __forceinline__ double psnr_sum(const float *pa, const float *pb, int64_t elems) {
    __shared__ double red[THREADS / 64];
    const int tid = threadIdx.x;
    double acc = 0.0;
    float part = 0.0f;
    int since = 0;
    auto flush = [&] { acc += (double)part; part = 0.0f; since = 0; };         // keeps the fp32 partial sums short
    // groups of 4 floats where both have the same place in a 16-byte word (but for the elements before the first whole one), singly otherwise
    const bool vec = ((((uintptr_t)pa) ^ ((uintptr_t)pb)) & 15) == 0;
    const int64_t head = vec ? min((int64_t)(-(((uintptr_t)pa) >> 2) & 3), elems) : 0, nv = vec ? (elems - head) / 4 : 0;
    const float4 *const va = (const float4 *)(pa + head), *const vb = (const float4 *)(pb + head);
    auto add = [&](float4 x, float4 y) {
        const float d0 = x.x - y.x, d1 = x.y - y.y, d2 = x.z - y.z, d3 = x.w - y.w;
        part += d0 * d0 + d1 * d1 + d2 * d2 + d3 * d3;
        if (++since == 64) flush();
    };
    int64_t q = tid;
    if (AHEAD > 1) {
        for (; q + (AHEAD - 1) * THREADS < nv; q += AHEAD * THREADS) {
            float4 x[AHEAD], y[AHEAD];
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {
                x[k] = va[q + k * THREADS];
                y[k] = vb[q + k * THREADS];
            }
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) add(x[k], y[k]);
        }
    }
    for (; q < nv; q += THREADS) add(va[q], vb[q]);
    flush();
    if (tid < head) {
        const float d = pa[tid] - pb[tid];
        part += d * d;
    }
    for (int64_t k = head + nv * 4 + tid; k < elems; k += THREADS) {
        const float d = pa[k] - pb[k];
        part += d * d;
        if (++since == 256) flush();
    }
    flush();
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    double s = 0.0;
    if (tid == 0)
        for (int w = 0; w < THREADS / 64; ++w) s += red[w];
    return s;
}
__device__ __forceinline__ float psnr_of(double s, int64_t elems, float peak) {
    return s == 0.0 ? INFINITY : (float)(10.0 * log10((double)peak * (double)peak * (double)elems / s));         // (not a number stays one)
}
template <int THREADS, int AHEAD>
__global__ __launch_bounds__(THREADS) void psnr_kernel(const float *a, const float *b, int64_t elems, float peak, float *out) {
    const size_t at = (size_t)blockIdx.x * (size_t)elems;
    const double s = psnr_sum<THREADS, AHEAD>(a + at, b + at, elems);
    if (threadIdx.x == 0) out[blockIdx.x] = psnr_of(s, elems, peak);
}
// One share of an image: `share` elements, the last one's to the image's end
__global__ __launch_bounds__(kPsnrThreads) void psnr_share_kernel(const float *a, const float *b, int64_t elems, int64_t share, double *sums) {
    const int64_t from = (int64_t)blockIdx.x * share;
    const size_t at = (size_t)blockIdx.y * (size_t)elems + (size_t)from;
    const double s = psnr_sum<kPsnrThreads, 2>(a + at, b + at, blockIdx.x + 1 == gridDim.x ? elems - from : share);
    if (threadIdx.x == 0) sums[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}
__global__ __launch_bounds__(256) void psnr_finish_kernel(const double *sums, int32_t splits, int64_t elems, float peak, float *out, int32_t n) {
    const int i = threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int k = 0; k < splits; ++k) s += sums[(size_t)i * splits + k];
    out[i] = psnr_of(s, elems, peak);
}
}  // namespace

extern "C" size_t rinr_psnr_workspace_bytes(int64_t n_images, int64_t elems) {
    const int64_t s = psnr_splits(n_images, elems);
    return s > 1 ? (size_t)(n_images * s) * sizeof(double) : 0;
}

extern "C" int rinr_psnr_batch_ex(const float *a, const float *b, int64_t n_images, int64_t elems, float peak, float *psnr, void *workspace,
                                  size_t workspace_bytes, void *stream) {
    if (n_images < 0 || elems < 0 || !(peak > 0.0f) || n_images > ((int64_t)1 << 31) - 1) return RINR_E_ARG;
    if (n_images == 0) return RINR_OK;
    if (!psnr || (elems > 0 && (!a || !b))) return RINR_E_NULL;
    if ((((uintptr_t)a) | ((uintptr_t)b) | ((uintptr_t)psnr)) & 3) return RINR_E_ALIGN;
    if (workspace && ((uintptr_t)workspace & 7)) return RINR_E_ALIGN;
    const hipStream_t st = (hipStream_t)stream;
    const int64_t splits = psnr_splits(n_images, elems);
    if (splits > 1 && workspace && workspace_bytes >= rinr_psnr_workspace_bytes(n_images, elems)) {
        const int64_t share = elems / splits / 4 * 4;
        hipLaunchKernelGGL(psnr_share_kernel, dim3((uint32_t)splits, (uint32_t)n_images), dim3(kPsnrThreads), 0, st, a, b, elems, share, (double *)workspace);
        FIT_HIP(hipGetLastError());
        hipLaunchKernelGGL(psnr_finish_kernel, dim3(1), dim3(256), 0, st, (const double *)workspace, (int32_t)splits, elems, peak, psnr, (int32_t)n_images);
    } else if (elems <= kPsnrSmall) {           // a small image leaves most of 1024 threads idle
        hipLaunchKernelGGL((psnr_kernel<256, 2>), dim3((uint32_t)n_images), dim3(256), 0, st, a, b, elems, peak, psnr);
    } else if (n_images <= 256) {
        hipLaunchKernelGGL((psnr_kernel<kPsnrThreads, 1>), dim3((uint32_t)n_images), dim3(kPsnrThreads), 0, st, a, b, elems, peak, psnr);
    } else {
        hipLaunchKernelGGL((psnr_kernel<kPsnrThreads, 2>), dim3((uint32_t)n_images), dim3(kPsnrThreads), 0, st, a, b, elems, peak, psnr);
    }
    FIT_HIP(hipGetLastError());
    return RINR_OK;
}

extern "C" int rinr_psnr_batch(const float *a, const float *b, int64_t n_images, int64_t elems, float peak, float *psnr, void *stream) {
    return rinr_psnr_batch_ex(a, b, n_images, elems, peak, psnr, nullptr, 0, stream);
}

// ---- Sec. IV as one call: fit, prune (fixed round, then the PSNR-driven one), re-fit, quantise, pack -------------
namespace {

struct EncodeModels {                       // host-side model descriptions of every image, in rinr_pack's terms
    std::vector<float> params;              // [n][n_params]
    std::vector<uint8_t> keep;              // [n][n_params] (biases: 1)
    std::vector<uint8_t> maskbits, codes8;
    std::vector<uint16_t> codes16;
    std::vector<rinr_layer_desc> layers;
    std::vector<rinr_model_desc> models;
};

// keep flags of every weight matrix of every image after pruning `ratio[i]` of image i's entries by magnitude
int prune_round(const rinr_fit *f, const std::vector<float> &params, const std::vector<double> &ratio, std::vector<uint8_t> &keep,
                bool have_keep) {
    const int L = f->arch.n_layers;
    std::vector<uint8_t> out;
    for (int64_t i = 0; i < f->n_images; ++i) {
        const float *p = params.data() + (size_t)i * (size_t)f->n_params;
        uint8_t *k = keep.data() + (size_t)i * (size_t)f->n_params;
        for (int l = 0; l < L; ++l) {
            const int64_t nw = (int64_t)f->arch.widths[l] * f->arch.widths[l + 1];
            out.resize((size_t)nw);
            const int rc = rinr_l1_mask(p + f->p_off[l], nw, ratio[(size_t)i], have_keep ? k + f->p_off[l] : nullptr, out.data());
            if (rc) return rc;
            std::memcpy(k + f->p_off[l], out.data(), (size_t)nw);
        }
    }
    return RINR_OK;
}

int psnr_now(rinr_fit *f, const float *targets, std::vector<double> &psnr, void *stream) {
    std::vector<float> loss((size_t)f->n_images);
    const int rc = rinr_fit_loss_grad(f, targets, 0.0f, loss.data(), nullptr, stream);      // mean squared error
    if (rc) return rc;
    psnr.resize(loss.size());
    for (size_t i = 0; i < loss.size(); ++i) psnr[i] = loss[i] == 0.0f ? INFINITY : -10.0 * std::log10((double)loss[i]);
    return RINR_OK;
}

int check_encode_opts(const rinr_encode_opts *o) {
    if (!o) return RINR_E_NULL;
    if (o->schedule < 0 || o->schedule > 2 || o->fit_steps < 0 || o->refit_steps < 0) return RINR_E_ARG;
    if (!(o->first_ratio >= 0.0f && o->first_ratio <= 1.0f) || !(o->lr > 0.0f) || !(o->refit_lr > 0.0f)) return RINR_E_ARG;
    if (!(o->hidden_bits == 0 || (o->hidden_bits >= 2 && o->hidden_bits <= 8) || o->hidden_bits == 16)) return RINR_E_ARG;
    return RINR_OK;
}

// descriptions for rinr_pack: hidden layers as codes of `bits` bits, first and last layer fp32 (Sec. IV-B)
int describe(const rinr_fit *f, int bits, EncodeModels &e) {
    const int L = f->arch.n_layers;
    const int64_t n = f->n_images;
    size_t wtot = 0, mtot = 0;
    for (int l = 0; l < L; ++l) {
        const size_t nw = (size_t)f->arch.widths[l] * (size_t)f->arch.widths[l + 1];
        wtot += nw;
        mtot += (nw + 7) / 8;
    }
    e.maskbits.assign((size_t)n * mtot, 0);
    if (bits && bits <= 8) e.codes8.assign((size_t)n * wtot, 0);
    if (bits == 16) e.codes16.assign((size_t)n * wtot, 0);
    e.layers.resize((size_t)n * (size_t)L);
    e.models.resize((size_t)n);
    std::vector<uint16_t> codes;
    for (int64_t i = 0; i < n; ++i) {
        const float *p = e.params.data() + (size_t)i * (size_t)f->n_params;
        const uint8_t *k = e.keep.data() + (size_t)i * (size_t)f->n_params;
        size_t woff = 0, moff = 0;
        for (int l = 0; l < L; ++l) {
            const int din = f->arch.widths[l], dout = f->arch.widths[l + 1];
            const size_t nw = (size_t)din * (size_t)dout;
            uint8_t *mb = e.maskbits.data() + (size_t)i * mtot + moff;
            for (size_t q = 0; q < nw; ++q)
                if (k[f->p_off[l] + q]) mb[q >> 3] |= (uint8_t)(1u << (q & 7));
            rinr_layer_desc &d = e.layers[(size_t)i * (size_t)L + (size_t)l];
            d.in = din;
            d.out = dout;
            d.bits = 0;
            d.scale = 1.0f;
            d.zp = 0;
            d.weights = p + f->p_off[l];
            d.mask = mb;
            d.bias = p + f->p_off[l] + nw;
            if (bits && l > 0 && l < L - 1) {
                codes.resize(nw);
                const int rc = rinr_quantize_layer(p + f->p_off[l], k + f->p_off[l], (int64_t)nw, bits, &d.scale, &d.zp, codes.data());
                if (rc) return rc;
                d.bits = bits;
                if (bits <= 8) {
                    uint8_t *c8 = e.codes8.data() + (size_t)i * wtot + woff;
                    for (size_t q = 0; q < nw; ++q) c8[q] = (uint8_t)codes[q];
                    d.weights = c8;
                } else {
                    uint16_t *c16 = e.codes16.data() + (size_t)i * wtot + woff;
                    std::memcpy(c16, codes.data(), nw * 2);
                    d.weights = c16;
                }
            }
            woff += nw;
            moff += (nw + 7) / 8;
        }
        e.models[(size_t)i].n_layers = L;
        e.models[(size_t)i].layers = e.layers.data() + (size_t)i * (size_t)L;
    }
    return RINR_OK;
}

}  // namespace

extern "C" int rinr_encode_blob_bound(const rinr_fit *f, int32_t hidden_bits, size_t *bytes) {
    if (!f || !bytes) return RINR_E_NULL;
    if (!(hidden_bits == 0 || (hidden_bits >= 2 && hidden_bits <= 8) || hidden_bits == 16)) return RINR_E_ARG;
    try {
        EncodeModels e;
        e.params.assign((size_t)f->n_images * (size_t)f->n_params, 0.0f);
        e.keep.assign((size_t)f->n_images * (size_t)f->n_params, 1);     // masks present, everything kept: the largest record
        const int rc = describe(f, hidden_bits, e);
        if (rc) return rc;
        const rinr_store_opts so = {f->arch.w0, f->arch.coord_lo, f->arch.coord_hi};
        return rinr_pack_size(e.models.data(), f->n_images, &so, bytes);
    } catch (const std::bad_alloc &) {
        return RINR_E_SIZE;
    }
}

extern "C" int rinr_encode_images(rinr_fit *f, const float *targets, const rinr_encode_opts *o, float *psnr_out, void *blob,
                                  size_t capacity, size_t *blob_bytes, void *stream) {
    if (!f || !blob_bytes || (!targets && f->n_images > 0)) return RINR_E_NULL;
    int rc = check_encode_opts(o);
    if (rc) return rc;
    try {
        const int64_t n = f->n_images;
        EncodeModels e;
        e.params.resize((size_t)n * (size_t)f->n_params);
        e.keep.assign((size_t)n * (size_t)f->n_params, 1);
        std::vector<double> psnr, ratio((size_t)n);
        bool have_keep = false;
        // the fit itself (Eq. 1; cosine decay over the stage)
        rinr_fit_opts fo = {o->lr, 0, o->fit_steps, 0.0f, 0.0f, 0.0f, 0.0f};
        if ((rc = rinr_fit_set_keep(f, nullptr)) || (rc = rinr_fit_steps(f, targets, o->fit_steps, &fo, stream))) return rc;
        // pruning rounds (Sec. IV-A): a fixed ratio first (large images only), then the ratio chosen from each image's PSNR;
        // after each, the mask is applied and the model re-fitted from a fresh optimiser at the smaller rate
        for (int round = 0; round < 2; ++round) {
            if (round == 0 && !(o->first_ratio > 0.0f)) continue;
            if (round == 0) {
                std::fill(ratio.begin(), ratio.end(), (double)o->first_ratio);
            } else {
                if ((rc = psnr_now(f, targets, psnr, stream))) return rc;
                // (an image whose error is no number does not end the others' encoding)
                for (int64_t i = 0; i < n; ++i) ratio[(size_t)i] = rinr_prune_ratio(o->schedule, std::isnan(psnr[(size_t)i]) ? INFINITY : psnr[(size_t)i]);
            }
            if ((rc = rinr_fit_get_params(f, e.params.data(), stream))) return rc;
            if ((rc = prune_round(f, e.params, ratio, e.keep, have_keep))) return rc;
            have_keep = true;
            fo.lr = o->refit_lr;
            fo.T = o->refit_steps;
            if ((rc = rinr_fit_set_keep(f, e.keep.data())) || (rc = rinr_fit_reset_optimizer(f)) ||
                (rc = rinr_fit_steps(f, targets, o->refit_steps, &fo, stream)))
                return rc;
        }
        if ((rc = psnr_now(f, targets, psnr, stream))) return rc;
        if (psnr_out)
            for (int64_t i = 0; i < n; ++i) psnr_out[i] = (float)psnr[(size_t)i];
        if ((rc = rinr_fit_get_params(f, e.params.data(), stream))) return rc;
        // hidden layers to codes, first and last layer fp32 (Sec. IV-B); one blob for the decode side
        if ((rc = describe(f, o->hidden_bits, e))) return rc;
        const rinr_store_opts so = {f->arch.w0, f->arch.coord_lo, f->arch.coord_hi};
        if ((rc = rinr_pack_size(e.models.data(), n, &so, blob_bytes))) return rc;
        if (!blob || capacity < *blob_bytes) return RINR_E_SIZE;
        return rinr_pack(e.models.data(), n, &so, blob, *blob_bytes);
    } catch (const std::bad_alloc &) {
        return RINR_E_SIZE;
    }
}
