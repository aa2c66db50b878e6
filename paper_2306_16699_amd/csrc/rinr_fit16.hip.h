// Fitting step (Eq. 1) on the fp16 matrix cores: the three contractions of a layer (forward, backward, weight
// gradient) run as v_mfma_f32_16x16x32_f16 with every fp32 operand carried as an exact-sum pair of halfs,
// hi = fp16(x), lo = fp16(x - hi), three terms per product (hi*hi + hi*lo + lo*hi, fp32 accumulate): ~22 significant
// bits per product at a third of the fp32 matrix instruction's time, and the fp16 matrix pipe runs beside the vector ALU
// that does the sines, cosines and splits.
//
// A workgroup has four wavefronts, and nothing passes between them until the end of the step: a wavefront takes NT x 16
// pixels at a time through all layers forward and backward with activations, pre-activations and errors in registers, and
// accumulates the weight gradients of all layers over its own pixels in registers as well (deep and wide models take all
// 512 registers of a lone wavefront per SIMD for it).  The only barriers are before the first pixel, when the weights are
// in LDS, and after the last, when the wavefronts' gradients are added up.  The version before this shared the gradient tiles
// among eight wavefronts: fewer registers, but every layer's errors and inputs went through LDS between two barriers.
//
// What bounds it is instruction issue: a matrix instruction takes 8 clocks of it (and 16 of the matrix unit), a sine or cosine 8, any other
// instruction 4, s_nop 4 a wait state; an LDS read is back after 64 (measured in streams of them and on pieces of this kernel, one wavefront
// per SIMD; a sum over the instructions of a piece in order, with those latencies, gives its measured time to 3 %).  A hidden
// layer of 48 units takes 48 matrix and 169 vector slots per 16 pixels backward, 15 and 52 forward.  So a lone wavefront loses what it waits
// in order: for operand words from LDS and for matrix results (see kDownFirst).  At 10 layers x 40, with a half-filled last tile, the
// matrix unit is busy 50 % of the time and vector issue 59 % (the matrix instructions' included), 31 % of the matrix time has
// vector instructions beside it, and a wavefront waits 12 % of its time for loads and barriers and 19 % to issue.
// Measured, ms a step, gradient tiles shared -> a wavefront's own -> layers interleaved (see the kernel) -> half-filled tiles, inputs in LDS
// (Shape) -> words loaded ahead (kDownFirst): 256 images of 224 x 224, 10 layers x 40: 8.91 -> 6.83 -> 6.29 -> 5.00 -> 4.69; 10 x 32: 4.54 -> 3.50 ->
// 3.00, no more from the half-filled tiles, -> 2.88; 2048 of 32 x 32, 3 x 15: 0.0934 -> 0.0738 -> 0.0675 -> 0.0655.
//
// Two orientations.  P: lane (n, g) holds pixel n and, per 16-row tile of a layer's units, the quad of units 4 g + v.  That is
// what a matrix instruction leaves with the units as its rows, and two tiles' quads side by side are exactly the B operand
// of one 32-deep step of the next layer, so nothing moves between lanes from one layer to the next, in either direction.
// U: lane (n, g) holds unit n and the pixels 4 g + v: the operand of the weight gradient, which contracts over pixels.  From P
// to U goes a matrix step with the unit matrix (the data as A, the unit matrix as B), which is exact for halfs, or, where
// several wavefronts share a SIMD, a write to LDS and a transposing read (Shape::areas).
// With NT = 2 the two tiles' quads make a 32-deep step over pixels; with NT = 1 the hi and the lo part of one tile do
// ([Eh | El] x [Hh | Hh], then x [Hl | Hl]: two steps instead of three, and the term lo*lo comes along).  The odd last tile of
// a layer's units is treated the same way in the forward and backward products ([Wh | Wl] x [Hh | Hh], x [Hl | Hl]).
//
// LDS holds the weights of the hidden layers twice, once with the outputs and once with the inputs as rows (those times the
// factor that the error is multiplied by going down, where it is above 1, see below), in operand order: per pair of 16-unit tiles a hi and a lo
// plane of 64-byte rows, 16 bytes per lane group: the quads of both tiles; an odd last tile's plane has the hi and the lo quad
// side by side.  A lane reads an operand as one 16-byte word at a fixed place
// in its row; rows 4..7 of every eight have their two pairs of words exchanged, which makes that read free of bank conflicts
// (measured: 4.8 clocks per wavefront instead of 8.7).  Plain 8-byte reads of row-major planes, as before, were merged
// by the compiler into two-address reads at 8.6 clocks or more.
//
// Range of the error in fp16: the error of layer l is carried times a power of two T_l.  T of the output layer is
// chosen from the root-mean-square error the previous step saw (kept per image; 0.25 if there was none), so that the
// scaled error is around 2^4 and at most 2^15 for errors up to 4; going down, each layer multiplies by the power of two
// nearest to the inverse of its estimated gain (0.7 * sqrt(sum of squared weights / inputs), from the weights at hand),
// which keeps the scaled error's magnitude level through deep models.  The split of the error rounds toward zero, which
// saturates at the largest half instead of producing infinities; 1 / T_l goes into the factor that the accumulated
// gradient is multiplied by at the end.
// A layer's factor above 1 (the usual case) is in its transposed weights: times a power of two both halves stay exact.  Below 1
// (an estimated gain above 1.4) the low half would go into fp16's subnormals, 1.1e-7 of the weights' size instead of 4.6e-8
// (64 units, factor 1/64), so such a factor multiplies the cosine in fp32.  One more multiply per unit costs up to 5 %,
// so the code over the pixels is there twice, and a model takes the form with the multiply only if one
// of its factors is below 1.  us a step, without and with: 256 images of 224 x 224, 10 layers x 40 4690 and 4900; 512, 10 x 32 5730 and 5890; of 96 x 96,
// 5 x 24 364 and 366; 256, 4 x 56 430 and 445; 1024 of 64 x 64, 3 x 8 79 and 82; 2048 of 32 x 32, 3 x 15 66.0 and 68.2.  Having both costs the other form
// nothing (10 x 40, whole last tile: 6.27 -> 6.24 ms).
#pragma once

namespace fit16 {

typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4, kThreads = 64 * kWaves;

// Registers: gradient tiles and pre-activations of all layers, and what a layer in progress takes.
constexpr int fit16_registers(int wp, int ml, int nt) {
    const int mt = wp / 16;
    return 4 * (2 * mt + (ml - 2) * mt * mt) + 4 * nt * mt * (ml - 1) + 40 + 16 * nt * mt;
}
// Wavefronts per SIMD a kernel is compiled for: as many as its estimate leaves.  The estimate does not count the addresses and operands of
// the inputs in LDS, and so some kernels spill: 4 layers x 16 at four wavefronts (23 registers; half-filled 8), 7 x 16 at three (17; 1), 5 x 32 (4), 8 x 32 (16)
// and 8 x 24 (15) at two.  With
// the inputs in LDS and these spills against the kernels before (of them 7 x 16 alone spilled, 24): 512 images of 96 x 96, 5 x 32 500 -> 459, 256 of 96 x 96, 8 x 32 475 -> 478 and 8 x 24 (half-filled
// tile) 441 -> 396, 1024 of 64 x 64, 7 x 16 343 -> 312.  Measured, us a step, spilled -> as chosen:
//   four instead of three, 48 x 48, width 16, 2048 images: 4 layers 198 -> 189, 5 layers 249 -> 241; 6144 images: 561 -> 555, 692 -> 691
//   two instead of three: 8 layers x 16: 243 -> 232; 3 x 32: 150 -> 144
//   three (spilling) instead of two at 7 layers x 16, 48 x 48: 6144 images 1063 -> 1001; against it 1024 of 64 x 64: 319 -> 328
// Four (spilling) is as chosen too at 4 layers x 16 where a launch takes several steps: 1024 images of 64 x 64, width 8, three 110, four 94.1.  Where
// images are shared, three: 20 of 128 x 128, 4 x 15 24.2, four 26.3.
// many: of the kernel that takes several steps a launch, where there is one
constexpr int fit16_waves_per_simd(int wp, int ml, int nt, bool many = true) {
    const int r = fit16_registers(wp, ml, nt);
    return r <= (many ? 112 : 100) ? 4 : (r <= 156 ? 3 : (r <= 256 ? 2 : 1));
}

// Whether a launch takes several steps of an image that one workgroup has.  A launch of its own costs a step its gap, the last round's idle part and
// instructions that are fetched again; a kernel that loops takes more registers, which small ones have.  Images that are shared, or so large that a
// launch takes one step, have the kernel without the loop (with it -> without: 8 images of 128 x 128, 3 x 24 18.1 -> 17.4; 20, 4 x 15 26.3 -> 24.2;
// 256 of 362 x 362, 2 x 15 556 -> 545).  us a step, a launch each -> 32 steps a launch, 2048 images of 32 x 32: 2 layers x 15 43.0 -> 39.6, 3 x 15
// 64.8 -> 60.5, 5 x 15 107.7 -> 104.6, 8 x 15 187.9 -> 181.3, 8 x 8 129.1 -> 122.5, 2 x 32 71.2 -> 69.1, 3 x 32 132.3 -> 127.8; 1024 of 64 x 64: 4 x
// 15 158.1 -> 146.7, 5 x 15 194.3 -> 195.7, 3 x 32 214.2 -> 209.5.  Beyond: 512 of 96 x 96, 4 x 32 322 -> 331, 5 x 24 338 -> 352.
constexpr bool fit16_many_steps(int wp, int ml, int nt) { return fit16_registers(wp, ml, nt) <= 168; }

// Shapes and the LDS layout (bytes) for hidden widths <= WP (a multiple of 16).
// HALF: the widths are at most WP - 8, so half of the last tile is padding.  A lane then holds two real units of it
// instead of four (units 16 t + 2 g + v sit in rows 4 g + v, v < 2), which takes half the sines, cosines and splits, and the two
// halfs of both go into one quad (h0 h1 l0 l1).  As an operand that quad meets (W0 W1 W0 W1) and (w0 w1 0 0), w the weights' low parts: an odd last
// tile has both side by side and takes all three terms in one matrix step instead of two; in a pair of tiles they are the halves of its two
// planes.  Turned in one step instead of two, its rows are the units' hi and lo parts side by side, and a gradient tile that it makes as
// either operand takes fewer steps likewise; the parts' rows and columns are added up at the end of the step.
// A hidden layer of 40 units takes 52 matrix steps per 16 pixels instead of 63, and 10 sines instead of 12 each way.  us a step, before ->
// now: 256 images of 224 x 224, 10 x 40: 6230 -> 5120; of 96 x 96, 3 x 40: 190 -> 166, 7 x 40: 709 -> 584, 4 x 56: 506 -> 467; 1024 of 64 x 64, 3 x 8: 114 -> 79,
// 10 x 8: 394 -> 244; 512 of 96 x 96, 3 x 24: 237 -> 198, 6 x 24: 541 -> 502, 10 x 24: 1149 -> 968.  Against fp64 the gradient is as far off as before
// (10 x 40: 2.73e-6, 10 x 24: 1.94e-6 and 1.92e-6, 3 x 8: 7.8e-7).
template <int WP, bool HALF> struct Shape {
    static constexpr int MT = WP / 16;                  // 16-unit tiles of a hidden layer
    static constexpr int NP = MT / 2, TAIL = MT % 2;    // pairs of them, and an odd last one
    static constexpr int NPL = 2 * NP + TAIL;           // planes of one operand matrix
    static __device__ __forceinline__ bool mixed(int t) { return HALF && t == MT - 1; }          // tile t's quads hold hi and lo
    static __device__ __forceinline__ int row(int unit) {
        const int j = unit & 15;
        return mixed(unit >> 4) ? (unit & ~15) + 4 * ((j >> 1) & 3) + (j & 1) + ((j & 8) >> 2) : unit;
    }
    static constexpr uint32_t PLANE = WP * 64;          // bytes of a plane of WP rows
    static constexpr uint32_t HID = NPL * PLANE;        // one hidden layer in one orientation
    static constexpr int GT = MT == 1 ? 4 : 16;         // gradient tiles that go through LDS at a time at the end
    // All offsets but the end are compile-time, so a lane's address is one register plus an immediate.
    static constexpr uint32_t MISC = 0;                                                          // see Misc
    static constexpr uint32_t W0 = 1024;                                                         // float [WP][4]: x weight, y weight, bias, 0
    static constexpr uint32_t BIAS = W0 + WP * 16;                                               // float [16] output layer, then [kMaxL - 2][WP], per step (see the kernel)
    static constexpr uint32_t LASTF = BIAS + 64 + (kMaxL - 2) * WP * 4;                          // 16 rows, channel c in row 4 c
    static constexpr uint32_t LASTT = LASTF + NPL * 16 * 64;                                     // WP rows, one tile of outputs
    static constexpr uint32_t HID0 = LASTT + PLANE;                                              // hidden layers: outputs as rows, inputs as rows
    static __host__ __device__ constexpr uint32_t weights(int L) { return HID0 + (uint32_t)(L - 2) * 2 * HID; }
    static constexpr uint32_t INPUT = kWaves * MT * 1024;                                        // one layer's input, hi and lo, per 16 pixels of a wavefront
    // How many areas of that size fit beside the weights, with as many workgroups on a CU as its registers hold.  In them the inputs of
    // the first hidden layers stay from the forward pass for the weight gradient, which then takes neither their sines and splits again
    // nor the steps that turn them, and an error is turned through one more: fewer instructions, and LDS latency instead of
    // the matrix unit's.  It pays where another wavefront of the SIMD fills that latency.  us a step, before -> now: 2048 of 32 x 32, 3 x 15:
    // 68.0 -> 64.6; 1024 of 64 x 64, 5 x 15: 227 -> 196, 8 x 15: 360 -> 309; 512 of 96 x 96, 5 x 24: 457 -> 416, 6 x 30: 628 -> 570; 256 of 96 x 96,
    // 3 x 46: 212 -> 200.  A lone wavefront, which waits for LDS with nothing else to do, gets slower (10 x 32: 6000 -> 6360, all turning
    // through LDS 7190), and so does an SIMD that loses a wavefront to the areas (8 x 30: 865 -> 1084).  The error turned through LDS as well:
    // 8 x 15: 325 -> 309, but 3 x 15: 64.7 -> 65.7, 5 x 30: 430 -> 530.  One area of several layers: 8 x 30: 863 -> 869.
    static __host__ __device__ constexpr int areas(int L, int NT) {
        const int waves = fit16_waves_per_simd(WP, L, NT), room = (int)kLdsLimit / waves - 256 - (int)weights(L);
        return waves == 1 || room < 0 ? 0 : room / (int)(NT * INPUT);
    }
    static __host__ __device__ constexpr bool turned(int L, int NT) { return WP == 16 && L > 3 && areas(L, NT) > 0; }
    static __host__ __device__ constexpr int kept(int L, int NT) {
        const int n = areas(L, NT) - turned(L, NT);
        return n >= L - 2 ? L - 2 : (n >= 2 ? n : 0);
    }
    static __host__ __device__ constexpr uint32_t total(int L, int NT) {
        const uint32_t w = weights(L) + (kept(L, NT) + turned(L, NT)) * NT * INPUT, r = W0 + kWaves * GT * 1024;
        return w > r ? w : r;
    }
};
struct Misc {              // small tables at the start of LDS; everything behind is reused when the gradients are added up
    float grad[16];        // factor of the accumulated gradient, per layer
    float scale[kMaxL];    // per layer: what the error is multiplied by going down through it
    float out;             // the output difference's factor
    int32_t below;         // a factor in `scale` is below 1
    float ss[kMaxL][kWaves];
    float red[kWaves];
    int32_t d[16], p_off[kMaxL];
};
static_assert(sizeof(Misc) <= 1024, "Misc");

__device__ __forceinline__ h8v cat(h4v a, h4v b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
// One matrix step: lane group g supplies k = 8 g .. 8 g + 7, as two quads; both operands of a product are built the same
// way, so the order within the 32 is immaterial.
__device__ __forceinline__ f32x4 mfma32(h8v a, h8v b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
// exact hi/lo split of a quad, round to nearest (activations, |x| <= 1).  neg1 is -1.0f passed as data, so that
// x - float(hi) stays one mixed-precision fma instead of a conversion and a subtraction.
__device__ __forceinline__ void split_rne(f32x4 x, float neg1, h4v &hi, h4v &lo) {
    const f2v p0 = {x[0], x[1]}, p1 = {x[2], x[3]};
    const h2v a0 = __builtin_convertvector(p0, h2v), a1 = __builtin_convertvector(p1, h2v);
    const f2v r0 = {__builtin_fmaf((float)a0[0], neg1, x[0]), __builtin_fmaf((float)a0[1], neg1, x[1])};
    const f2v r1 = {__builtin_fmaf((float)a1[0], neg1, x[2]), __builtin_fmaf((float)a1[1], neg1, x[3])};
    const h2v b0 = __builtin_convertvector(r0, h2v), b1 = __builtin_convertvector(r1, h2v);
    hi = (h4v){a0[0], a0[1], a1[0], a1[1]};
    lo = (h4v){b0[0], b0[1], b1[0], b1[1]};
}
__device__ __forceinline__ h4v to_h4(f32x4 x) {
    const auto a0 = __builtin_amdgcn_cvt_pkrtz(x[0], x[1]), a1 = __builtin_amdgcn_cvt_pkrtz(x[2], x[3]);
    return (h4v){(_Float16)a0[0], (_Float16)a0[1], (_Float16)a1[0], (_Float16)a1[1]};
}
// hi/lo split of a quad, round toward zero: values beyond the largest half saturate there instead of becoming infinite
__device__ __forceinline__ void split_rtz(f32x4 x, float neg1, h4v &hi, h4v &lo) {
    hi = to_h4(x);
    lo = to_h4((f32x4){__builtin_fmaf((float)hi[0], neg1, x[0]), __builtin_fmaf((float)hi[1], neg1, x[1]),
                       __builtin_fmaf((float)hi[2], neg1, x[2]), __builtin_fmaf((float)hi[3], neg1, x[3])});
}
// the same of two values, both parts in one quad
__device__ __forceinline__ h4v split2_rne(float x0, float x1, float neg1) {
    const f2v p = {x0, x1};
    const h2v a = __builtin_convertvector(p, h2v);
    const f2v r = {__builtin_fmaf((float)a[0], neg1, x0), __builtin_fmaf((float)a[1], neg1, x1)};
    const h2v b = __builtin_convertvector(r, h2v);
    return (h4v){a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ h4v split2_rtz(float x0, float x1, float neg1) {
    const auto a = __builtin_amdgcn_cvt_pkrtz(x0, x1);
    const auto b = __builtin_amdgcn_cvt_pkrtz(__builtin_fmaf((float)a[0], neg1, x0), __builtin_fmaf((float)a[1], neg1, x1));
    return (h4v){(_Float16)a[0], (_Float16)a[1], (_Float16)b[0], (_Float16)b[1]};
}
__device__ __forceinline__ f32x4 sin4(f32x4 z) {
    return (f32x4){__builtin_amdgcn_sinf(z[0]), __builtin_amdgcn_sinf(z[1]), __builtin_amdgcn_sinf(z[2]), __builtin_amdgcn_sinf(z[3])};
}
__device__ __forceinline__ f32x4 cos4(f32x4 z) {
    return (f32x4){__builtin_amdgcn_cosf(z[0]), __builtin_amdgcn_cosf(z[1]), __builtin_amdgcn_cosf(z[2]), __builtin_amdgcn_cosf(z[3])};
}

// A quad of tile t: the sines, split; the error, split
template <class S> __device__ __forceinline__ void sine_split(f32x4 z, int t, float neg1, h4v &hi, h4v &lo) {
    if (S::mixed(t)) {
        hi = split2_rne(__builtin_amdgcn_sinf(z[0]), __builtin_amdgcn_sinf(z[1]), neg1);
        lo = S::TAIL ? hi : (h4v)((_Float16)0.0f);              // in a pair, the second term's step takes nothing more of this tile
    } else {
        split_rne(sin4(z), neg1, hi, lo);
    }
}
template <class S> __device__ __forceinline__ void error_split(f32x4 e, int t, float neg1, h4v &hi, h4v &lo) {
    if (S::mixed(t)) {
        hi = split2_rtz(e[0], e[1], neg1);
        lo = S::TAIL ? hi : (h4v)((_Float16)0.0f);
    } else {
        split_rtz(e, neg1, hi, lo);
    }
}

// Entry (row r, contraction index k) of an operand matrix whose planes have `plane` bytes, as a hi/lo pair
template <int WP, bool HALF> __device__ __forceinline__ void put_operand(char *m, uint32_t plane, int r, int k, float w) {
    typedef Shape<WP, HALF> S;
    const _Float16 h = (_Float16)w, l = (_Float16)(w - (float)h);
    const int t = k >> 4;
    if (HALF) k = S::row(k);
    const int q = (k >> 2) & 3;
    const uint32_t at = (uint32_t)r * 64 + 16 * (q ^ ((r >> 1) & 2)) + 2 * (k & 3);
    if (HALF && t == S::MT - 1) {
        _Float16 *p = (_Float16 *)(m + (S::TAIL ? 2 * S::NP : 2 * (S::NP - 1)) * plane + at + (S::TAIL ? 0 : 8));
        p[0] = p[2] = h;
        p[S::TAIL ? 4 : plane / 2] = l;             // beside them, or in the pair's plane of low parts
    } else if (S::TAIL && t == S::MT - 1) {
        _Float16 *p = (_Float16 *)(m + 2 * S::NP * plane + at);
        p[0] = h;
        p[4] = l;
    } else {
        _Float16 *p = (_Float16 *)(m + (t >> 1) * 2 * plane + at + 8 * (t & 1));
        p[0] = h;
        p[plane / 2] = l;
    }
}

// The operand words of R row tiles of a matrix, all planes: this lane's word of each row tile is at `m` + 1024 t
template <int WP, bool HALF, int R> struct Words {
    typedef Shape<WP, HALF> S;
    h8v w[S::NPL][R];
    __device__ __forceinline__ void load(const char *m, uint32_t plane) {
#pragma unroll
        for (int p = 0; p < S::NPL; ++p)
#pragma unroll
            for (int t = 0; t < R; ++t) w[p][t] = *(const h8v *)(m + p * plane + t * 1024);
    }
    // acc += rows x B, contraction block k: a pair of tiles (three terms) or an odd last tile (two); the row tiles take turns, so
    // that a matrix step does not wait for the one before it
    template <int NT> __device__ __forceinline__ void block(int k, const h4v (&Bh)[NT][S::MT], const h4v (&Bl)[NT][S::MT], f32x4 (&acc)[NT][R]) const {
        const bool tail = k == S::NP;
        const int p = 2 * k, b0 = 2 * k, b1 = tail ? b0 : b0 + 1;
#pragma unroll
        for (int term = 0; term < (tail ? (HALF ? 1 : 2) : 3); ++term)
#pragma unroll
            for (int t = 0; t < R; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[nt][t] = mfma32(w[term == 2 ? p + 1 : p][t], term == 1 ? cat(Bl[nt][b0], Bl[nt][b1]) : cat(Bh[nt][b0], Bh[nt][b1]), acc[nt][t]);
    }
};

// Ends a basic block between two layers: `stop` is 0, which the compiler cannot see.  A whole chunk as one block has its
// registers assigned badly (10 layers x 40: 78 to 219 spilled; with these edges none), and code moves across too far.
// A kernel that takes more than 256 registers must not spill: the compiler's pass that puts matrix results into the upper half
// then loses reloads of parts of a quad (seen in the assembly of a 7 x 48 kernel whose gradients were wrong in that quad).
#define FIT16_EDGE                         \
    do {                                   \
        asm volatile("" : "+s"(stop));     \
        if (stop) return;                  \
    } while (0)

// Weights and tables of image `img` into LDS.  Returns whether some layer's factor of the error is below 1 (the same in every lane).
template <int WP, bool HALF, int L, class Args> __device__ __forceinline__ bool fit16_set_up(const Args &a, char *lds, size_t img, int tid, int wave) {
    typedef Shape<WP, HALF> S;
    constexpr int MT = S::MT;
    Misc *const misc = (Misc *)(lds + S::MISC);
    const int lane = tid & 63;
    const float *P = a.params + img * a.n_params;

    // ---- set up: zero everything; weights as hi/lo operands (sine layers times w0 / 2pi: Z comes out in revolutions), biases;
    //      per layer the sum of squared weights (for the error's scale), summed in a fixed order.  A thread has all its weights
    //      of a layer under way at once, and the next layer's while it places this one's: one memory latency, not one per weight.
    constexpr int kOwn = MT * MT;                       // WP * WP / kThreads
    float cur[kOwn], next[kOwn];
    auto fetch = [&](int l, float (&w)[kOwn]) {
        const int cnt = l < L ? a.d[l] * a.d[l + 1] : 0;
        const float *src = P + a.p_off[l < L ? l : 0];
#pragma unroll
        for (int k = 0; k < kOwn; ++k) w[k] = tid + k * kThreads < cnt ? src[tid + k * kThreads] : 0.0f;
    };
    fetch(0, cur);
    for (uint32_t q = tid; q < S::weights(L) / 16; q += kThreads) ((uint4 *)lds)[q] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    for (int l = 0; l < L; ++l) {
        const int din = a.d[l], dout = a.d[l + 1];
        const bool last = l == L - 1;
        const uint32_t per = (1u << 20) / (uint32_t)din + 1u;               // e / din == e * per >> 20 for e < 4096
        const float sc = last ? 1.0f : a.w0rev;
        const float bias = tid < dout ? P[a.p_off[l] + dout * din + tid] : 0.0f;
        fetch(l + 1, next);
        char *const F = lds + S::HID0 + (uint32_t)(l > 0 ? l - 1 : 0) * 2 * S::HID;
        float ss = 0.0f;
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
            const int e = tid + k * kThreads;
            if (e < dout * din) {
                const int o = (int)((uint32_t)e * per >> 20), i = e - o * din;
                const float w = cur[k] * sc;
                ss = fmaf(w, w, ss);
                if (l == 0) {
                    ((float *)(lds + S::W0))[o * 4 + i] = w;
                } else if (last) {
                    put_operand<WP, HALF>(lds + S::LASTF, 16 * 64, 4 * o, i, w);
                    put_operand<16, false>(lds + S::LASTT, S::PLANE, S::row(i), 4 * o, w);
                } else {
                    put_operand<WP, HALF>(F, S::PLANE, S::row(o), i, w);
                    put_operand<WP, HALF>(F + S::HID, S::PLANE, S::row(i), o, w);
                }
            }
            cur[k] = next[k];
        }
        if (tid < dout) {
            float *const B = (float *)(lds + S::BIAS) + (last ? 4 * tid : 16 + (l - 1) * WP + S::row(tid));
            *(l == 0 ? (float *)(lds + S::W0) + tid * 4 + 2 : B) = bias * sc;
        }
        for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
        if (lane == 0) misc->ss[l][wave] = ss;
    }
    if (tid < 16) misc->d[tid] = tid <= L ? a.d[tid] : 0;
    if (tid < L) misc->p_off[tid] = a.p_off[tid];
    __syncthreads();
    if (tid == 0) {
        // scale of the output layer's error from the error the previous step saw; then down the layers by the estimated gains
        float rms = a.emag ? a.emag[img] : 0.0f;
        rms = rms > 0.0f ? fminf(fmaxf(rms, 0.001953125f), 4.0f) : 0.25f;
        const float raw = 2.0f * a.loss_scale * rms;                        // error of the output layer before scaling, typical size
        float T = exp2f(4.0f - ceilf(log2f(raw)));
        T = fminf(fmaxf(T, 1e-30f), 1e30f);
        misc->out = T * 2.0f * a.loss_scale;                                // what the output difference is multiplied by
        misc->grad[L - 1] = a.gscale[L - 1] / T;
        bool below = false;
        for (int l = L - 1; l >= 1; --l) {
            float ss = 0.0f;
            for (int w = 0; w < kWaves; ++w) ss += misc->ss[l][w];
            const float gain = 0.7f * sqrtf(ss / (float)a.d[l]);
            float r = gain > 0.0f ? exp2f(rintf(-log2f(gain))) : 1.0f;
            r = fminf(fmaxf(r, 0.015625f), 256.0f);
            if (!(T * r < 1e30f && T * r > 1e-30f)) r = 1.0f;
            T *= r;
            misc->scale[l] = r;                                             // E_{l-1} = r (W_l^T E_l) cos(.)
            below |= r < 1.0f;
            misc->grad[l - 1] = a.gscale[l - 1] / T;
        }
        misc->below = below;
    }
    __syncthreads();
    const bool below = __builtin_amdgcn_readfirstlane(misc->below) != 0;
    // the transposed weights carry that factor where it is above 1
    for (int l = 1; l < L; ++l) {
        const _Float16 r = (_Float16)fmaxf(misc->scale[l], 1.0f);
        h8v *const T = (h8v *)(lds + (l == L - 1 ? S::LASTT : S::HID0 + (uint32_t)(2 * l - 1) * S::HID));
        for (uint32_t q = tid; q < (l == L - 1 ? S::PLANE : S::HID) / 16; q += kThreads) T[q] *= r;
    }
    __syncthreads();

    return below;
}

// One kernel per depth L: the hidden layers are steps u = 0 .. L - 3 of unrolled code without conditions, so that what one
// layer's end and the next one's start have to do runs side by side.  Forward, a piece of code between two edges takes the last
// block of a layer's contraction (its odd last tile, or last pair of tiles), the sines and splits of its tiles as they come
// out, and the next layer's other blocks, whose operand words it has loaded first; the row tiles take turns at the matrix
// unit.  With a layer a piece of its own, as before, a layer's matrix steps waited for each other and for every load, and its
// sines came after them.  Measured, ms a step, before -> now: 256 images of 224 x 224, 10 layers x 40: 6.83 -> 6.29; 512 of
// 224 x 224, 10 x 32: 6.98 -> 6.00; 512 of 96 x 96, 5 x 24: 0.532 -> 0.457; 64 of 128 x 128, 6 x 64: 0.500 -> 0.450.  Forcing one
// matrix step per two to four vector instructions backward (scheduling groups) was slower: 7.8 ms at 10 x 40.
// kBelow: some layer's factor of the error is below 1 and is applied here, on the cosine (see the file header).
template <int WP, bool HALF, int L, int NT, bool kBelow, class Args> __device__ __forceinline__ void fit16_pixels(const Args &a, char *lds, const FitShare &share, int number, int tid, int wave) {
    typedef Shape<WP, HALF> S;
    constexpr int MT = S::MT, NH = L - 2, kPC = kWaves * 16 * NT;
    constexpr int kColOut = 11, kColFirst = 12;         // columns of acc_b: step u's biases in column u, the output layer's, the first layer's bias, x and y
    constexpr int kRegisters = fit16_registers(WP, L, NT);
    // The order of a lone wavefront's work, which nothing else hides the waits of.  Everywhere: the first layer's words are loaded before the
    // coordinates are formed, the output layer's before its last contraction, and the way down's (kAhead tiles of them) at the layer's start, where
    // the split of the error covers them.  kDownFirst: all of the way down's words at once, the contraction with nothing else beside it, and the output
    // layer's input is turned before the output is there.  That is the faster one with four tiles, and with three where registers are
    // scarcest and a half tile spares some; else two tiles' words ahead and the compiler's own order are.  Clocks per 16 NT
    // pixels of a wavefront as the compiler orders them, before -> two tiles ahead, kDownFirst: 10 layers x 32 16500 -> 15600, 19900; 10 x 40 14540 ->
    // 14140 with spills, 13090; 8 x 40 11610 -> 10460, 11020; 8 x 48 13530 -> 12020, 12990; 6 x 56 13500 -> 13390, 12680; 6 x 64 13740 -> 13950, 13340.  us a step,
    // 256 images of 96 x 96, before -> now: 5 x 40 389 -> 372, 8 x 40 793 -> 722, 6 x 48 564 -> 554, 8 x 48 908 -> 822, 10 x 48 1221 -> 1128, 4 x 56 458 -> 430, 6 x 56 892 ->
    // 848, 4 x 64 510 -> 469, 6 x 64 932 -> 898, 10 x 24 488 -> 474, 12 x 32 726 -> 687; against it 12 x 24 589 -> 593 (since the end of a step is another, 583).  The form with the multiply (kBelow): 10 x 24 570 ->
    // 494, 10 x 48 1320 -> 1121, 6 x 64 1019 -> 921.
    // kTight: the one kernel (10 layers x 48) that spills (see FIT16_EDGE) where the first layer's words are ahead or the contraction is not first.
    constexpr bool kAlone = fit16_waves_per_simd(WP, L, NT) == 1, kTight = !HALF && kRegisters > 500;
    constexpr bool kDownFirst = kAlone && !kTight && (MT == 4 || (MT == 3 && (kBelow ? HALF || kRegisters <= 480 : HALF && kRegisters > 480)));
    constexpr bool kFirstAhead = kAlone && !kTight;
    constexpr int kAhead = !kAlone ? 1 : (kDownFirst || MT < 2 ? MT : 2);          // row tiles whose operand words the way down loads ahead
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    const h4v zh = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
    Misc *const misc = (Misc *)(lds + S::MISC);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    const size_t img = share.img;
    const float neg1 = a.neg1;

    f32x4 acc[NH > 0 ? NH : 1][MT][MT];                         // weight gradients of the hidden layers: rows are outputs, columns inputs
    f32x4 acc_last[MT], acc_b[MT];                 // output layer (channel c in row 4 c); biases and first layer
    f32x4 zst[NH + 1][NT][MT];                     // pre-activations (revolutions) of the pixels at hand: what goes into step u, into the output layer
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        acc_last[t] = acc_b[t] = zero4;
#pragma unroll
        for (int u = 0; u < NH; ++u)
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[u][t][i] = zero4;
    }
#pragma unroll
    for (int u = 0; u <= NH; ++u)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int t = 0; t < MT; ++t) zst[u][nt][t] = zero4;
    float loss_part = 0.0f;
    // the unit matrix as B operand, in the first quad (for the even tile of a pair) and in the second
    const h4v id = {(_Float16)(4 * g == n ? 1.0f : 0.0f), (_Float16)(4 * g + 1 == n ? 1.0f : 0.0f), (_Float16)(4 * g + 2 == n ? 1.0f : 0.0f),
                    (_Float16)(4 * g + 3 == n ? 1.0f : 0.0f)};
    const h8v I0 = cat(id, zh), I1 = cat(zh, id);
    // P -> U: tile t of a hi/lo pair of quads.  An odd last tile's quads go side by side into one operand, of which either unit
    // matrix takes one half.
    auto turn = [&](const h4v (&Xh)[MT], const h4v (&Xl)[MT], int t, h4v &hi, h4v &lo) {
        if (HALF && !S::TAIL && t == MT - 1) {
            hi = lo = to_h4(mfma32(cat(Xh[t & ~1], Xh[t | 1]), I1, zero4));
        } else if (t < 2 * S::NP) {
            hi = to_h4(mfma32(cat(Xh[t & ~1], Xh[t | 1]), (t & 1) ? I1 : I0, zero4));
            lo = to_h4(mfma32(cat(Xl[t & ~1], Xl[t | 1]), (t & 1) ? I1 : I0, zero4));
        } else {
            const h8v x = cat(Xh[t], Xl[t]);
            hi = to_h4(mfma32(x, I0, zero4));
            lo = HALF ? hi : to_h4(mfma32(x, I1, zero4));      // (a half tile's quad holds both)
        }
    };
    auto turn1 = [&](h4v xh, h4v xl, h4v &hi, h4v &lo) {
        const h8v x = cat(xh, xl);
        hi = to_h4(mfma32(x, I0, zero4));
        lo = to_h4(mfma32(x, I1, zero4));
    };
    // P -> U through LDS: a quad is written as it is, 32 bytes of a tile's units to a pixel, and read back by the transposing read, in which
    // the 16 lanes of a group take four rows of 16 halfs and get a column each; places exchanged in half of the rows, for the banks.
    constexpr int kKept = S::kept(L, NT);               // steps u < kKept: the input stays in area u
    constexpr bool kTurned = S::turned(L, NT);          // the error goes through area kKept
    char *const areas = lds + S::weights(L) + wave * (NT * MT * 1024);
    char *const put_at = areas + (n * 32 + 8 * (g ^ ((n >> 2) & 2)));
    const char *const get_at = areas + ((4 * g + (n >> 2)) * 32 + 8 * ((n & 3) ^ (g & 2)));
    auto put = [&](int area, const h4v (&Xh)[NT][MT], const h4v (&Xl)[NT][MT]) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                char *const p = put_at + area * (NT * S::INPUT) + (nt * MT + t) * 1024;
                *(h4v *)p = Xh[nt][t];
                if (!S::mixed(t)) *(h4v *)(p + 512) = Xl[nt][t];
            }
    };
    auto get = [&](int area, int nt, int t, int part) -> h4v {
        typedef __fp16 f4v __attribute__((ext_vector_type(4)));
        const char *const p = get_at + area * (NT * S::INPUT) + (nt * MT + t) * 1024 + part * 512;
        return __builtin_bit_cast(h4v, __builtin_amdgcn_ds_read_tr16_b64_v4f16((__attribute__((address_space(3))) f4v *)p));
    };
    auto column = [&](int k, uint32_t c) -> h8v {                           // ones in column k
        int m = n;
        asm("" : "+v"(m) : "s"(c));         // made again where it is used: eight steps' columns are not held across the loop
        const uint32_t two = m == k ? 0x3C003C00u : 0u;
        const u4v w = {two, two, two, two};
        return __builtin_bit_cast(h8v, w);
    };
    const char *const base = lds + (n * 64 + 16 * (g ^ ((n >> 1) & 2)));    // this lane's word of an operand's row
    auto step = [&](int u, uint32_t c, uint32_t at) {                       // ... in step u's layer: one addition per step, the rest immediates
        uint32_t s = S::HID0 + at + (uint32_t)u * 2 * S::HID;
        asm("" : "+s"(s) : "s"(c));        // formed per chunk: not held across the loop in a register per layer
        return base + s;
    };

    auto pixel = [&](uint32_t c, int nt) { return c * kPC + (uint32_t)(wave * 16 * NT + nt * 16 + n); };
    auto target = [&](uint32_t c, int nt) {                                 // lane group g: channel g
        const uint32_t p = pixel(c, nt);
        return a.target[(img * 3 + (g < 3 ? g : 2)) * a.HW + (p < a.HW ? p : a.HW - 1)];
    };
    float tgt[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tgt[nt] = share.c0 < share.c1 ? target(share.c0, nt) : 0.0f;

    for (uint32_t c = share.c0; c < share.c1; ++c) {
        int stop = 0;                      // see FIT16_EDGE

        // ---- forward.  First layer on the vector ALU (two inputs); hidden layers: Z = W H + b
        h4v Bh[NT][MT], Bl[NT][MT];
        float x[NT], y[NT], want[NT];
        float4 w0[MT][4];
        auto first_word = [&](int t, int v) { w0[t][v] = ((const float4 *)(lds + S::W0))[16 * t + (S::mixed(t) ? 2 : 4) * g + v]; };
        auto first = [&](f32x4 (&z)[NT][MT], bool ahead) {             // ahead: its words are loaded
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int v = 0; v < (S::mixed(t) ? 2 : 4); ++v) {
                    if (!ahead) first_word(t, v);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) z[nt][t][v] = fmaf(w0[t][v].x, x[nt], fmaf(w0[t][v].y, y[nt], w0[t][v].z));
                }
        };
        Words<WP, HALF, MT> W;
        Words<WP, HALF, 1> WL;
        f32x4 zo[NT][1];                   // output layer: channel g of pixel n in the first register of lane (n, g)
        // What the contraction into step u's layer, or the output layer, starts from: its operand words, and the biases
        auto begin = [&](int u) {
            if (u < NH) {
                const f32x4 *B = (const f32x4 *)(lds + S::BIAS + 64 + u * WP * 4);
                W.load(step(u, c, 0), S::PLANE);
#pragma unroll
                for (int t = 0; t < MT; ++t)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) zst[u + 1][nt][t] = B[4 * t + g];
            } else {
                WL.load(base + S::LASTF, 16 * 64);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) zo[nt][0] = ((const f32x4 *)(lds + S::BIAS))[g];
            }
        };
        constexpr int kBlocks = S::NP + S::TAIL;
        auto blocks = [&](int u, int k0, int k1) {
#pragma unroll
            for (int k = k0; k < k1; ++k) {
                if (u < NH) W.template block<NT>(k, Bh, Bl, zst[u + 1]);
                else WL.template block<NT>(k, Bh, Bl, zo);
            }
        };
        {
            f32x4 z0[NT][MT];
            if (kFirstAhead) {
#pragma unroll
                for (int t = 0; t < MT; ++t)
#pragma unroll
                    for (int v = 0; v < (S::mixed(t) ? 2 : 4); ++v) first_word(t, v);
            }
            if (kDownFirst) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const uint32_t p = min(pixel(c, nt), a.HW - 1);
                const uint32_t row = a.wmagic ? (__umulhi(p, a.wmagic) >> a.wshift) : p, col = p - row * a.W;
                x[nt] = fmaf(a.span, (float)(2 * col + 1) * a.inv2W, a.lo);
                y[nt] = fmaf(a.span, (float)(2 * row + 1) * a.inv2H, a.lo);
                want[nt] = tgt[nt];
                tgt[nt] = target(c + 1 < share.c1 ? c + 1 : c, nt);             // the next pixels' targets are under way during this chunk
            }
            first(z0, kFirstAhead);
            begin(0);
            if (kDownFirst) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    if (NH == 0) zst[NH][nt][t] = z0[nt][t];
                    sine_split<S>(z0[nt][t], t, neg1, Bh[nt][t], Bl[nt][t]);
                }
            if (kKept > 0) put(0, Bh, Bl);
            blocks(0, 0, kBlocks - 1);
        }
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            FIT16_EDGE;
            blocks(u, kBlocks - 1, kBlocks);
            begin(u + 1);
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) sine_split<S>(zst[u + 1][nt][t], t, neg1, Bh[nt][t], Bl[nt][t]);
            if (u + 1 < kKept) put(u + 1, Bh, Bl);
            blocks(u + 1, 0, kBlocks - 1);
        }
        FIT16_EDGE;
        h8v out_words[MT];
        h4v inh[NT][MT], inl[NT][MT];      // the output layer's input, turned
        if (kAlone) {
#pragma unroll
            for (int t = 0; t < MT; ++t) out_words[t] = *(const h8v *)(base + S::LASTT + t * 1024);
        }
        blocks(NH, kBlocks - 1, kBlocks);
        if (kDownFirst) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) turn(Bh[nt], Bl[nt], i, inh[nt][i], inl[nt][i]);
        }

        // ---- output layer
        f32x4 E[NT][MT];                   // the error at hand, scaled (see the file header)
        h4v Eh[NT][MT], El[NT][MT];
        // Its split belongs to the end of the layer that leaves it, beside that layer's weight gradient (10 layers x 32: 6.08 ->
        // 6.00 ms a step); where registers are scarce, to the start of the next.
        constexpr bool kLate = kRegisters > 480;
        auto slope = [&](f32x4 z, int l) { return kBelow ? cos4(z) * fminf(misc->scale[l], 1.0f) : cos4(z); };
        auto leave = [&](int nt, int t, f32x4 e, f32x4 z, int l) {
            if (HALF) {
                f32x4 c = zero4;
                if (S::mixed(t)) {
                    c[0] = __builtin_amdgcn_cosf(z[0]);
                    c[1] = __builtin_amdgcn_cosf(z[1]);
                } else {
                    c = cos4(z);
                }
                if (kBelow) c *= fminf(misc->scale[l], 1.0f);
#pragma unroll
                for (int v = 0; v < (S::mixed(t) ? 2 : 4); ++v) E[nt][t][v] = e[v] * c[v];
            } else {
                E[nt][t] = e * slope(z, l);
            }
            if (!kLate) error_split<S>(E[nt][t], t, neg1, Eh[nt][t], El[nt][t]);
        };
        auto take = [&] {
            if (kLate)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int t = 0; t < MT; ++t) error_split<S>(E[nt][t], t, neg1, Eh[nt][t], El[nt][t]);
        };
        {
            if (!kAlone || kDownFirst) FIT16_EDGE;
            const float eo = misc->out;
            h4v eh[NT], el[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float e = g < 3 && pixel(c, nt) < a.HW ? zo[nt][0][0] - want[nt] : 0.0f;
                loss_part = fmaf(e, e, loss_part);
                split_rtz((f32x4){e * eo, 0.0f, 0.0f, 0.0f}, neg1, eh[nt], el[nt]);
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const h8v at = kAlone ? out_words[t] : *(const h8v *)(base + S::LASTT + t * 1024);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) E[nt][t] = mfma32(at, cat(el[nt], el[nt]), mfma32(at, cat(eh[nt], eh[nt]), zero4));
            }
            h8v A0, A1;
            h4v uh[NT], ul[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) turn1(eh[nt], el[nt], uh[nt], ul[nt]);
            A0 = cat(uh[0], NT == 2 ? uh[NT - 1] : ul[0]);
            A1 = cat(ul[0], ul[NT - 1]);
            const h8v ones = column(kColOut, c);
            acc_b[0] = mfma32(A0, ones, acc_b[0]);
            if (NT == 2) acc_b[0] = mfma32(A1, ones, acc_b[0]);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (!kDownFirst) turn(Bh[nt], Bl[nt], i, inh[nt][i], inl[nt][i]);
                }
                const h8v b0 = cat(inh[0][i], inh[NT - 1][i]), b1 = cat(inl[0][i], inl[NT - 1][i]);
                acc_last[i] = mfma32(A0, b0, acc_last[i]);
                if (!S::mixed(i)) acc_last[i] = mfma32(A0, b1, acc_last[i]);
                if (NT == 2) acc_last[i] = mfma32(A1, b0, acc_last[i]);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < MT; ++t) leave(nt, t, E[nt][t], zst[NH][nt][t], L - 1);
        }

        // ---- backward: the error goes down through the hidden layers, each layer's weight gradient takes these pixels
        h8v A0[MT], A1[MT];                // the error turned: NT = 2: hi, lo; NT = 1: [hi | lo], unused
        auto turn_error = [&](const h4v (&Eh)[NT][MT], const h4v (&El)[NT][MT]) {
            if (kTurned) put(kKept, Eh, El);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                h4v uh[NT], ul[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (!kTurned) turn(Eh[nt], El[nt], t, uh[nt], ul[nt]);
                    else if (S::mixed(t)) uh[nt] = ul[nt] = get(kKept, nt, t, 0);
                    else { uh[nt] = get(kKept, nt, t, 0); ul[nt] = get(kKept, nt, t, 1); }
                }
                A0[t] = cat(uh[0], NT == 2 ? uh[NT - 1] : ul[0]);
                A1[t] = cat(ul[0], ul[NT - 1]);
            }
        };
#pragma unroll
        for (int u = NH - 1; u >= 0; --u) {
            if (u == 0) {                              // not kept from the forward pass: cheaper to form again than to hold
                FIT16_EDGE;
                first(zst[0], false);
            }
            h4v Hh[NT][MT], Hl[NT][MT];
            FIT16_EDGE;
            Words<WP, HALF, 1> V[kAhead];
            const char *const down_at = step(u, c, S::HID);
            if (kAlone) {
#pragma unroll
                for (int t = 0; t < kAhead; ++t) V[t].load(down_at + t * 1024, S::PLANE);
                if (kDownFirst || kTight) __builtin_amdgcn_sched_barrier(0);
            }
            take();
            f32x4 down[NT][MT];
            auto contract = [&] {
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    if (!kAlone) V[0].load(step(u, c, S::HID + t * 1024), S::PLANE);
                    else if (t > 0 && t + kAhead - 1 < MT) V[(t + kAhead - 1) % kAhead].load(down_at + (t + kAhead - 1) * 1024, S::PLANE);
                    f32x4 d[NT][1];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) d[nt][0] = zero4;
#pragma unroll
                    for (int k = 0; k < kBlocks; ++k) V[t % kAhead].template block<NT>(k, Eh, El, d);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) down[nt][t] = d[nt][0];
                }
            };
            // (the contraction first: fewer registers; with the multiply, kBelow, where they are scarce, and where several wavefronts share a SIMD)
            constexpr bool kContractFirst = kDownFirst || kTight || (kBelow && (!kAlone || kLate));
            if (kContractFirst) contract();
            if (kDownFirst) __builtin_amdgcn_sched_barrier(0);
            turn_error(Eh, El);
            if (u >= kKept)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int t = 0; t < MT; ++t) sine_split<S>(zst[u][nt][t], t, neg1, Hh[nt][t], Hl[nt][t]);
            if (!kContractFirst) contract();
            const h8v ones = column(u, c);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                acc_b[t] = mfma32(A0[t], ones, acc_b[t]);
                if (NT == 2 && !S::mixed(t)) acc_b[t] = mfma32(A1[t], ones, acc_b[t]);
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                h4v uh[NT], ul[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (u >= kKept) turn(Hh[nt], Hl[nt], i, uh[nt], ul[nt]);
                    else if (S::mixed(i)) uh[nt] = ul[nt] = get(u, nt, i, 0);
                    else { uh[nt] = get(u, nt, i, 0); ul[nt] = get(u, nt, i, 1); }
                }
                const h8v b0 = cat(uh[0], uh[NT - 1]), b1 = cat(ul[0], ul[NT - 1]);
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    acc[u][t][i] = mfma32(A0[t], b0, acc[u][t][i]);
                    if (!S::mixed(i)) acc[u][t][i] = mfma32(A0[t], b1, acc[u][t][i]);
                    if (NT == 2 && !S::mixed(t)) acc[u][t][i] = mfma32(A1[t], b0, acc[u][t][i]);
                }
            }
            // E_{l-1} = r (W_l^T E_l) cos(2 pi z_{l-1})
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < MT; ++t) leave(nt, t, down[nt][t], zst[u][nt][t], u + 1);
        }
        // ---- first layer: its input's columns are one, x, y
        {
            FIT16_EDGE;
            h4v h[NT], lo[NT];
            take();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                h4v xh, xl;
                split_rne((f32x4){1.0f, x[nt], y[nt], 0.0f}, neg1, xh, xl);
                turn1(g == kColFirst / 4 ? xh : zh, g == kColFirst / 4 ? xl : zh, h[nt], lo[nt]);
            }
            if (MT == 4 && NT == 2) __builtin_amdgcn_sched_barrier(0);          // (256 images of 96 x 96, 4 x 64 461 -> 455 us a step, 4 x 56 423 -> 420)
            turn_error(Eh, El);
            const h8v b0 = cat(h[0], h[NT - 1]), b1 = cat(lo[0], lo[NT - 1]);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                acc_b[t] = mfma32(A0[t], b0, acc_b[t]);
                acc_b[t] = mfma32(A0[t], b1, acc_b[t]);
                if (NT == 2 && !S::mixed(t)) acc_b[t] = mfma32(A1[t], b0, acc_b[t]);
            }
        }
    }

    // ---- loss of this step's parameters, and the error's size for the next step's scale
    for (int off = 32; off > 0; off >>= 1) loss_part += __shfl_xor(loss_part, off, 64);
    if (lane == 0) misc->red[wave] = loss_part;
    __syncthreads();
    if (tid == 0) {
        float s = 0.0f;
        for (int w = 0; w < kWaves; ++w) s += misc->red[w];
        fit_put_loss(a, share, s);
    }

    // ---- the wavefronts' gradients are added up, GT tiles at a time through LDS (in a fixed order), and each entry handed out.  Where
    //      wavefronts share a SIMD, what comes after the tiles are written is one piece of code for all of them: instructions that a launch meets for the
    //      first time cost it more than their issue (with a lone wavefront's registers that makes the pixels' code the worse one: 10 layers x 40 4690 -> 5060).
    //      us a step with that and four entries of Adam at once (fit_put_grads), before -> now: 256 images of 96 x 96, 4 x 64 469 -> 449, 7 x 40 560 -> 546, 6 x 56 843 -> 824,
    //      10 x 24 478 -> 465; 512 of 96 x 96, 6 x 30 558 -> 552; of 224 x 224, 10 x 40 4690 -> 4650.
    f32x4 *const R = (f32x4 *)(lds + S::W0);
    constexpr int kTiles = 2 * MT + NH * MT * MT;
#pragma unroll (kAlone ? kTiles : 1)
    for (int b0 = 0; b0 < kTiles; b0 += S::GT) {
#pragma unroll
        for (int c = 0; c < kTiles; c += S::GT)
            if (b0 == c) {
#pragma unroll
                for (int q = 0; q < S::GT; ++q) {
                    const int at = c + q, h = at - 2 * MT;
                    if (at < kTiles)
                        R[(wave * S::GT + q) * 64 + lane] = at < MT ? acc_b[at] : (at < 2 * MT ? acc_last[at - MT] : acc[h / (MT * MT)][h / MT % MT][h % MT]);
                }
            }
        __syncthreads();
        for (int q = wave; q < S::GT && b0 + q < kTiles; q += kWaves) {
            const int at = b0 + q, h = at - 2 * MT;
            f32x4 s = R[q * 64 + lane];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) s += R[(w * S::GT + q) * 64 + lane];
            // layer, row tile, and which column of its matrix this lane's column is (din: the bias, -1: none)
            int l = L - 1, ot = 0, col;
            if (at < MT) {
                ot = at;
                l = n < NH ? n + 1 : (n == kColOut ? L - 1 : 0);
                col = n < NH ? misc->d[l] : (n == kColOut ? misc->d[l] : (n >= kColFirst && n < kColFirst + 3 ? (n + 2 - kColFirst) % 3 : -1));
                if (col < 0) l = 0;
            } else if (at < 2 * MT) {
                col = (at - MT) * 16 + n;
            } else {
                l = h / (MT * MT) + 1;
                ot = h / MT % MT;
                col = h % MT * 16 + n;
            }
            const int din = misc->d[l], dout = misc->d[l + 1], off = misc->p_off[l];
            float gs = misc->grad[l];
            // a half tile's hi and lo parts: columns n and n + 2, rows v and v + 2; those rows came in twice where a step has 16 pixels
            if (HALF && at >= MT && (at < 2 * MT ? at - MT : h % MT) == MT - 1) {
#pragma unroll
                for (int v = 0; v < 4; ++v) s[v] += __shfl_xor(s[v], 2, 64);
                col = (n & 2) ? -1 : (MT - 1) * 16 + 2 * (n >> 2) + (n & 1);
            }
            const bool half_rows = HALF && (at < MT || at >= 2 * MT) && l < L - 1 && ot == MT - 1;
            if (half_rows) {
                s[0] += s[2];
                s[1] += s[3];
                gs *= NT == 1 ? 0.5f : 1.0f;
            }
            if (at >= MT && col >= din) col = -1;
            const bool bias = col == din;                               // entry (o, col) of the layer is at from + o * by
            const int from = off + (bias ? dout * din : col), by = bias ? 1 : din;
            int to[4];
            float gr[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = ot * 16 + (half_rows ? 2 : 4) * g + v, o = l == L - 1 ? (ot == 0 && v == 0 ? g : dout) : row;
                to[v] = col >= 0 && o < dout && !(half_rows && v >= 2) ? from + o * by : -1;
                gr[v] = s[v] * gs;
            }
            if (!kTight) {
                fit_put_grads(a, share, to, gr, number);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (to[v] >= 0) fit_put_grad(a, share, to[v], gr[v], number);
            }
        }
        __syncthreads();
    }
}

// kMany: several steps of an image that one workgroup has
template <int WP, bool HALF, int L, int NT, bool kMany>
__global__ __launch_bounds__(kThreads, fit16_waves_per_simd(WP, L, NT, kMany)) void fit16_step_kernel(const FitArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds16[];
    const uint32_t pixels = kWaves * 16 * NT;
    auto step = [&](const auto &args, int s, int tid) {
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const uint32_t nchunks = (args.HW + pixels - 1) / pixels;
        const FitShare share = kMany ? FitShare{blockIdx.x, 0u, nchunks, nullptr} : fit_share(args, nchunks);
        if (!fit16_set_up<WP, HALF, L>(args, lds16, share.img, tid, wave)) fit16_pixels<WP, HALF, L, NT, false>(args, lds16, share, s, tid, wave);
        else fit16_pixels<WP, HALF, L, NT, true>(args, lds16, share, s, tid, wave);
    };
    if constexpr (kMany) {
        // The arguments and the lane are made unknown again for every step: what a step derives from them would be held across the loop, and spill.
        typedef const __attribute__((address_space(4))) FitArgs *ConstArgs;
        for (int s = 0; s < a.steps; ++s) {
            ConstArgs args = (ConstArgs)__builtin_amdgcn_kernarg_segment_ptr();
            int tid = threadIdx.x;
            asm volatile("" : "+s"(args), "+v"(tid));
            step(*args, s, tid & (kThreads - 1));       // (its range is known again)
        }
    } else {
        step(a, 0, threadIdx.x);
    }
}

}  // namespace fit16
