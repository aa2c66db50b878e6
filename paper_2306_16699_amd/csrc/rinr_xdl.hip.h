// Split-precision decode kernel: the layers' contractions run on the fp16 matrix cores
// (v_mfma_f32_32x32x16_f16 / 16x16x32_f16 / 16x16x16_f16, fp32 accumulate) with every fp32
// operand carried as an exact-sum pair of halfs, hi = fp16(x), lo = fp16(x - hi), so a product
// keeps ~22 significant bits:  W*h ~= Wh*hh + Wh*hl + Wl*hh   (the dropped Wl*hl is 2^-22 relative).
// A hidden layer stored as 2..8-bit codes (Sec. IV-B) needs no low part at all: its integers
// q - zp are exact in fp16, so W*h = scale * (Q*hh + Q*hl) and the scale moves into the sine
// epilogue.  Unlike fp32 MFMA, the fp16 matrix pipe runs concurrently with the vector ALU on
// this chip, so the sine + split work hides the matrix work; the method and its results
// (Sec. III-B decode) are unchanged.
//
// Same structure as the fp32 kernel: workgroup = (slot, range of 64-pixel tiles), model
// expanded once into LDS, activations register-resident across layers.  Tile = TM rows x TM
// pixels (xdl_tile_rows; 32 above 48 units in the all-class kernel), lane = (n = lane % TM, g = lane / TM).
// A lane's accumulator registers come in quads of four consecutive rows; quad Q (counted over
// all row tiles of the layer) holds rows
//     TM = 16:  16 Q + 4 g + b            TM = 32:  32 (Q / 4) + 8 (Q % 4) + 4 g + b,   b = 0..3.
// One MFMA k-step takes 8 halfs per lane = quads 2j and 2j+1 of every lane group, i.e. exactly the
// activations the lanes already hold, so again nothing crosses lanes between layers.  An odd last quad takes a step of its own,
// full-depth, with the hi and the lo parts side by side, or half-depth, v_mfma_f32_16x16x16_f16, on the same accumulators (XLayout::TAIL).
// Two MFMAs of different depth must not follow each other closely on one accumulator: with a 16x16x16 step issued
// right behind a 16x16x32 step that writes its C operand (one vector instruction between them, no wait states
// added by the compiler) the second read the accumulator before the first had written it, and the first step's
// contribution was lost.  So all full-depth steps of a layer are issued first, then 20 idle cycles of this wavefront
// (one more than the longest wait the instruction set documents between dependent matrix instructions of different
// kinds; the SIMD's other wavefronts issue meanwhile), then all half-depth steps,
// the order being forced through the accumulators themselves (xdl_touch).  tests/test_gpu_parity.py pins it with a
// model whose output must contain a term that only the full-depth step supplies.
#pragma once
#include "rinr_kernels.hip.h"

namespace rinr {

typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef float f2v __attribute__((ext_vector_type(2)));

// A hidden layer takes the two-term integer form when its codes are exact in fp16 and the
// scale is a usable multiplier; otherwise its dequantised fp32 weights are split hi/lo.
__host__ __device__ inline bool xdl_int_layer(uint32_t bits, float scale_pre) {
    const float a = scale_pre < 0 ? -scale_pre : scale_pre;
    return bits >= 2 && bits <= 8 && a >= 1e-12f && a <= 1e12f;
}

// What kinds of hidden layer the models served by a launch have (the host knows it from the store): a kernel
// for one kind runs a layer loop without a branch on the kind.  With the branch inside, the compiler hoists and
// sinks the two halves' common epilogue code out of the branches, away from the MFMAs it is meant to run under.
enum { kHiddenAllInt = 0, kHiddenAllRaw = 1, kHiddenMixed = 2 };
// Added to the kind: activations travel as one fp16 value instead of a hi+lo pair (RINR_FLAG_FP16_ACT): one MFMA
// term less per layer and a two-instruction epilogue, at 2^-12 relative rounding per activation.
enum { kAct16 = 4 };
// Added to kAct16 (the kind is then irrelevant): the hidden layers' weights are single fp16 values too, fp16(w * w0 / 2pi)
// whether the layer is stored as codes or as fp32, so every hidden layer is one MFMA term and its epilogue is
// sine + conversion (RINR_FLAG_FP16_ALL): fp16 operands with fp32 accumulation throughout the hidden layers.
enum { kWeight16 = 8 };

// MFMA tile rows the split-precision kernels use for widths up to WQ (a multiple of 8).  A matrix step delays the vector instructions
// beside it by a clock per operand register, so a 32-row step, which does twice the work of a 16-row one on as many, delays
// less; but it takes more energy for it, and these kernels run at the card's power limit (a stream of 32-row steps on random operands runs at
// 1.73 GHz, of 16-row ones at 1.9, on zeros both at 2.4), and its accumulators are harder to place.  us, 32 -> 16 rows, on two cards: 256 images
// of 160 x 160, 4 x 32: 154.5 -> 147.7 and 148.6 -> 144.7, of fp32 weights 171 -> 159 and 161 -> 152; 4 x 64: 349.5 -> 337.5.  The reduced modes (one
// term, the lightest on the matrix unit) keep 32 rows there: all in fp16 16 are no better on either card (114 -> 114, 111.8 -> 113.5), with fp16
// activations on one of them only (110 -> 104, 103.0 -> 103.5).  At 24 units a 32-row tile has three
// quads a lane and the odd one's terms take one step, while 16-row ones make a pair of a full and a half-filled tile: 126.9 against 128.2.
__host__ __device__ constexpr int xdl_tile_rows(int wq, int mode) {
    return wq == 24 || (wq == 32 && (mode & (kAct16 | kWeight16))) ? 32 : 16;
}
// ... and the one grid's: with 32-row tiles above 48 units 122 registers leave room for 16 wavefronts a CU; with 16-row ones 64 ragged images
// of 300 x 300 take 236 us instead of 209
__host__ __device__ constexpr int xdl_any_tile_rows(int wq, int mode) { return wq > 48 ? 32 : xdl_tile_rows(wq, mode); }

struct XLayer {            // one entry per linear layer, built in LDS by the workgroup
    uint32_t off_hi;       // byte offset of the fp16 operand block
    uint32_t off_lo;       // byte offset of the low-part block, 0 = none (integer layer)
    float scale;           // multiplies the accumulator before the sine (1 unless integer layer)
    uint32_t off_bias;     // byte offset of the fp32 bias tile(s)
};

// How the last quad of a layer's rows enters the next layer's contraction where the quads do not pair up, or are not full.
//   kTailHalf  an odd last quad by half-depth steps, a step per term
//   kTailFull  an odd last quad by full-depth steps: [hi | lo] of the activations against the weights twice over (and against their
//              low parts twice over where the layer has them: two steps instead of three)
//   kTailTwo   an odd last quad of which two rows are real: (h0 h1 l0 l1 | h0 h1 l0 l1) against (W0 W1 W0 W1 | w0 w1 0 0), w the weights' low
//              parts: one step for all terms, whatever the kind of layer
enum { kTailNone = 0, kTailHalf = 1, kTailFull = 2, kTailTwo = 3 };

// WQ: the widest hidden layer rounded up to a multiple of 8.  Rows are padded to WP, but what is not computed for the padding is half a
// tile: where WQ is an odd multiple of 8, a lane holds two real rows of the last 16-row tile (units 16 t + 2 g + b sit in rows 4 g + b,
// b < 2, and the padding in b = 2, 3), or one quad less of a 32-row tile.  A padded unit would cost a sine and its split like a real one:
// us a call, width padded to 16 -> to 8: 64 images of 224 x 224, 9 x 40: 269 -> 240; 256 of 160 x 160, 4 sine layers of 8 units: 83.0 -> 64.9, 24:
// 142.6 -> 122.3, 40: 234 -> 212, 56: 325 -> 313, of fp32 weights 152 -> 137 (24), 279 -> 236 (40).  kTailFull instead of kTailHalf, a step where
// two half-depth ones and their wait were: 1024 of 64 x 64, 5 x 48: 196 -> 187; 256 of 160 x 160, 4 x 48: 244.6 -> 233.9, 4 x 16: 83.0 -> 81.7.
// Where activations are single halfs (one term: one step either way) or the layer has a low part, wide odd last quads stay with kTailHalf.
// INT: every hidden layer of the models served is integer-coded, and activations are hi/lo pairs.
template <int TM, int WQ_, bool INT> struct XLayout {
    static constexpr int WQ = WQ_, WP = (WQ + 15) / 16 * 16;
    static constexpr bool INTS = INT;
    static constexpr int G = 64 / TM;              // lane groups
    static constexpr int RV = TM * TM / 64;        // accumulator registers per tile
    static constexpr int MT = WP / TM;             // row tiles per layer
    static constexpr bool HALF = TM == 16 && WQ != WP;   // two real rows per lane in the last tile
    static constexpr int NQ = TM == 16 ? WP / 16 : WQ / 8;   // quads per lane over the layer's rows
    static constexpr int KJ = NQ / 2;              // full k-steps (8 halfs per lane) of two quads
    static constexpr int TAIL = NQ % 2 == 0 ? kTailNone : (HALF ? kTailTwo : (TM == 32 || INT ? kTailFull : kTailHalf));
    static constexpr int SELECT = 16 * 16;         // bytes: one XLayer per linear layer, 16 at most; then the 16 byte selectors of expand_hidden
    static constexpr int TABLE = SELECT + 16 * 4;
    static constexpr int TAILB = TAIL == kTailNone ? 0 : (TAIL == kTailHalf ? 512 : 1024);       // bytes of the last quad's step, per row tile
    static constexpr int HID = KJ * MT * 1024 + MT * TAILB;                                      // bytes of one hidden operand block
    static constexpr int HIDLO = KJ * MT * 1024 + (TAIL == kTailTwo ? 0 : MT * TAILB);           // ... of the low parts (kTailTwo has them with the others)
    static constexpr int FIRST = G * MT * 64 * 16; // bytes: [pixel tile q][mt][lane][8 halfs], hi and lo in one k-step; variant q has the
                                                   // weights in lane group q's k-slots only, so that group q's coordinates alone count
    static constexpr int OUT = KJ * 1024 + TAILB, OUTLO = KJ * 1024 + (TAIL == kTailTwo ? 0 : TAILB);   // bytes: one TM-row tile
    static constexpr int OUTB = TM * 4;            // bytes of the output layer's bias tile
    static_assert(WP % TM == 0 && WQ % 8 == 0, "layout");

    // unit r of the layer -> (quad, lane group, position in the quad)
    static __device__ __forceinline__ void locate(int r, int &q, int &g, int &b) {
        b = r & 3;
        if (TM == 32) { q = r >> 3; g = (r >> 2) & 1; return; }
        q = r >> 4; g = (r >> 2) & 3;
        if (HALF && q == MT - 1) { g = (r >> 1) & 3; b = (r & 1) + ((r & 8) >> 2); }
    }
    // ... -> row
    static __device__ __forceinline__ int row(int r) {
        if (!HALF) return r;
        int q, g, b;
        locate(r, q, g, b);
        return 16 * q + 4 * g + b;
    }
    // half index inside an operand block of `mts` row tiles: k-step's row tile mt, lane, input (q, g, b); kTailFull has the weight at + 4 too,
    // kTailTwo at + 2, and its low part at + 4
    static __device__ __forceinline__ int idx(int mts, int mt, int m, int q, int g, int b) {
        if (q < 2 * KJ) return (((q >> 1) * mts + mt) * 64 + g * TM + m) * 8 + (q & 1) * 4 + b;
        return KJ * mts * 512 + (mt * 64 + g * TM + m) * (TAIL == kTailHalf ? 4 : 8) + b;
    }
    static __device__ __forceinline__ bool in_tail(int i) { return TAIL != kTailNone && i >= (TM == 16 ? 32 * KJ : 16 * KJ); }
    static __device__ __forceinline__ int idx_input(int i) {      // input i of row 0 in a hidden layer's block
        int q, g, b;
        locate(i, q, g, b);
        return idx(MT, 0, 0, q, g, b);
    }
    // hidden weight (o, i)
    static __device__ __forceinline__ int idx_hidden(int o, int i) {
        const int r = row(o);
        int q, g, b;
        locate(i, q, g, b);
        return idx(MT, r / TM, r % TM, q, g, b);
    }
    static __device__ __forceinline__ int idx_first(int q, int o, int e) { const int r = row(o); return (((q * MT + r / TM) * 64) + q * TM + (r % TM)) * 8 + e; }
    // output channel c sits in row 4c of the single output tile
    static __device__ __forceinline__ int idx_out(int c, int i) {
        int q, g, b;
        locate(i, q, g, b);
        return idx(1, 0, 4 * c, q, g, b);
    }
    // bias tiles are accumulator shaped: [row tile][lane group][register]; `o` a row for the output layer's tile
    static __device__ __forceinline__ int idx_bias_row(int r) {
        const int v = TM == 16 ? r & 3 : ((r >> 3 & 3) << 2) | (r & 3), g = TM == 16 ? (r >> 2) & 3 : (r >> 2) & 1;
        return ((r / TM) * G + g) * RV + v;
    }
    static __device__ __forceinline__ int idx_bias(int o) { return idx_bias_row(row(o)); }
};

// Bytes of LDS of an expanded model (without the staging copy of the record): base + (L - 2) * layer, in layout XLayout<tm, wq, ints>
struct XBytes { uint32_t base, layer; };
__host__ __device__ constexpr XBytes xdl_bytes(uint32_t tm, uint32_t wq, bool ints, bool two_blocks) {
    const uint32_t wp = (wq + 15u) / 16u * 16u, g = 64u / tm, mt = wp / tm, nq = tm == 16u ? wp / 16u : wq / 8u, kj = nq / 2u;
    const bool odd = nq % 2u != 0u, two_rows = odd && tm == 16u && wq != wp;                              // kTailTwo
    const uint32_t tail = !odd ? 0u : (two_rows || tm == 32u || ints ? 1024u : 512u), low = two_rows ? 0u : tail;
    const uint32_t hidden = mt * (kj * 1024u + tail), hidden_low = mt * (kj * 1024u + low);
    return XBytes{16u * 16u + 16u * 4u + 4u * wp + 4u * tm + g * mt * 1024u + 2u * kj * 1024u + tail + low,
                  4u * wp + hidden + (two_blocks ? hidden_low : 0u)};
}
// ... of one of `width` units and L linear layers in the layout that `form` (kFit...) names
__host__ __device__ inline uint32_t xdl_model_bytes(uint32_t form, uint32_t width, uint32_t L) {
    const uint32_t cls = width == 0u ? 1u : (width + 15u) >> 4, own = width == 0u ? 8u : (width + 7u) & ~7u;
    const uint32_t wq = form & kFitAny ? own : 16u * cls - (form & (uint32_t)kFitNarrow << (cls - 1u) ? 8u : 0u);
    const uint32_t tm = form & kFitAny ? (uint32_t)xdl_any_tile_rows((int)wq, form & kFitOneTerm ? kAct16 : 0)
                                       : (uint32_t)xdl_tile_rows((int)wq, form & kFitOneTerm ? kAct16 : 0);
    const XBytes b = xdl_bytes(tm, wq, (form & kFitPairs) != 0u, (form & kFitKind) == kFitXdlTwo);
    return b.base + (L - 2u) * b.layer;
}
// Whether xdl_bytes has layout LY's
template <int TM, class LY> constexpr bool xdl_bytes_hold() {
    constexpr XBytes one = xdl_bytes(TM, LY::WQ, LY::INTS, false), two = xdl_bytes(TM, LY::WQ, LY::INTS, true);
    return one.base == LY::TABLE + 4 * LY::WP + LY::OUTB + LY::FIRST + LY::OUT + LY::OUTLO && two.base == one.base &&
           one.layer == 4 * LY::WP + LY::HID && two.layer == one.layer + LY::HIDLO;
}

// Builds the operand blocks of layers [l0, l1) in LDS and their XLayer entries tab[l].  `rec` is the model record:
// the staged copy in LDS, or the record itself in global memory; `t` its layer records in the lanes.
//   SLOTTED == false (resident model, l0 = 0, l1 = L): table, all bias tiles, then the blocks back to back.
//   SLOTTED == true  (streamed model): table, then one fixed-size slot per layer of the group: bias tile, blocks.
// Ends with a barrier.
template <class LY> struct XSlot {
    static constexpr int HID = LY::HID + LY::HIDLO, OUT = LY::OUT + LY::OUTLO;
    static constexpr int BLOCKS = HID > LY::FIRST ? (HID > OUT ? HID : OUT) : (LY::FIRST > OUT ? LY::FIRST : OUT);
    static constexpr int BIAS = LY::WP * 4 > LY::OUTB ? LY::WP * 4 : LY::OUTB;
    static constexpr int BYTES = BIAS + BLOCKS;
};

// This wavefront's part of a hidden layer, four consecutive inputs of one output per lane: one 8-byte word of the operand block (PutFour: in
// a last quad more),
// written whole, pruned weights and the padding of a row included, so only rows of padding have to be cleared first.  A lane has a nibble
// of the mask; the ranks of all lanes' first kept weights come from the counts' three bits (ballots and masked bit counts), and
// the codes of a lane's kept weights follow each other, so two words of the stream hold them.  For 2..8-bit codes the four bytes
// go to their places by one byte permute, whose selector is a table's (pruned: the zero point), and to halfs by another:
// 1024 + code is a half with the code as its low byte, and subtracting 1024 + zp is exact.
// About 35 vector instructions for up to 256 weights, where one weight per lane took 30 for up to 64 (10 layers x 40: from the
// workgroup's start to the end of this phase 25 -> 14.5 thousand clocks).
template <int WQ> struct XExpand {
    static constexpr int LANES = WQ <= 16 ? 4 : (WQ <= 32 ? 8 : 16), ROWS = 64 / LANES;      // lanes per row, rows per pass
    static constexpr int PASSES = (WQ + ROWS - 1) / ROWS;
};
// Byte selector of a nibble of keep bits: byte b is the rank of weight b among the kept ones, or 4 (the zero point) if pruned.
__device__ __forceinline__ uint32_t nibble_selector(uint32_t bits) {
    uint32_t s = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) s |= ((bits >> b & 1u) ? (uint32_t)__popc(bits & ((1u << b) - 1u)) : 4u) << (8 * b);
    return s;
}
// Where a lane's four consecutive inputs of one output go in an operand block: one word of it, two where the step has it twice (kTailFull),
// or, in a last tile with two rows a lane, half of the words of two lane groups.  A pass's rows are in one row tile, so what
// depends on the pass is the scalar unit's, and what depends on the lane is known before the first pass; the half tile's inputs take no branch
// of their own but for the second word.  Expansion of 8 x 40 and 8 x 56, us a call with nothing decoded behind it: 515 images of 146 x 17 (2575
// workgroups) 61.4 -> 53.7 and 59.1 -> 53.3 against two branches that find their places in every pass (and passes for rows of padding),
// 57 of 23 x 38 (228) 11.6 -> 10.1 and 13.2 -> 12.0; whole calls, 515 of 146 x 17 149.0 -> 140.6, 57 of 23 x 38 17.3 -> 15.8 and 21.1 -> 19.9.
template <class LY, int TM> struct PutFour {
    static constexpr int LANES = XExpand<LY::WQ>::LANES, ROWS = XExpand<LY::WQ>::ROWS;
    static constexpr int NEXT = 16 * 16;            // bytes to the next lane group's word
    uint32_t at, at_half;                           // bytes: the word of the lane's row in a pass that begins a row tile; ... the half tile
    uint32_t narrow;                                // 1: rows are 8 bytes apart (kTailHalf), not 16
    bool tail, split, has;                          // in the last quad; ... shared with the next lane group; there is such an input
    __device__ __forceinline__ PutFour(uint32_t lane) {
        const uint32_t i = 4u * (lane % LANES), r = lane / LANES;
        const bool last = LY::in_tail((int)i);
        tail = last;
        narrow = LY::TAIL == kTailHalf && last ? 1u : 0u;
        split = LY::HALF && i >= 16u * (LY::MT - 1);
        has = i < (uint32_t)LY::WQ;
        const uint32_t word = 2u * (uint32_t)LY::idx_input((int)i);
        at = word + (16u * r >> narrow);
        at_half = word + 16u * ((r & 7u) + (r & 6u) + (r >> 3) * 2u);     // row(16 t + j); j above 7 are rows of padding
    }
    // bytes of the lane's word in pass p
    __device__ __forceinline__ uint32_t place(uint32_t p) const {
        // with whole tiles and four of them the compiler's schedule is the better one where the place is worked out anew: 515 images of 146 x 17,
        // 8 x 64 of 16-bit weights, 419 us as below and 411 so (of 8-bit codes 253 either way); at 25 to 32 units as below 19.3 and 21.3 so
        if (!LY::HALF && TM == 16 && LY::MT == 4) {
            const uint32_t lane = (uint32_t)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
            return 2u * (uint32_t)LY::idx_hidden((int)(p * ROWS + lane / LANES), (int)(4u * (lane % LANES)));
        }
        const uint32_t row = p * ROWS, t = row / TM, in = row % TM;
        const bool half = LY::HALF && t == (uint32_t)LY::MT - 1u;
        const uint32_t pass = t * 1024u + 16u * in * (half ? 2u : 1u);
        return (half ? at_half : at) + (LY::TAIL == kTailHalf ? pass >> narrow : pass);
    }
    __device__ __forceinline__ void put(char *block, uint32_t place, h4v w, h4v low) const {
        typedef uint32_t u2v __attribute__((ext_vector_type(2)));
        typedef uint32_t u4v __attribute__((ext_vector_type(4)));
        char *const p = block + place;
        const u2v x = __builtin_bit_cast(u2v, w), y = __builtin_bit_cast(u2v, low);
        if (LY::HALF && LY::TAIL == kTailTwo) {
            *(u2v *)p = (u2v){x[0], split ? x[0] : x[1]};
            if (split) {
                *(u2v *)(p + 8) = (u2v){y[0], 0u};
                *(u4v *)(p + NEXT) = (u4v){x[1], x[1], y[1], 0u};
            }
        } else if (LY::HALF) {
            *(u2v *)p = (u2v){x[0], split ? 0u : x[1]};
            if (split) *(u2v *)(p + NEXT) = (u2v){x[1], 0u};
        } else {
            *(u2v *)p = x;
            if (LY::TAIL == kTailFull && tail) *(u2v *)(p + 8) = x;
        }
    }
};
template <class LY, int TM, bool W16, int KIND, int U>
__device__ __forceinline__ void expand_hidden(const uint32_t *rec, const LaneLayers &t, int l, int lane, char *lds, char *hi, char *lo, float *bt,
                                              float bias_factor, bool whole, float pre) {
    typedef XExpand<LY::WQ> X;
    const uint32_t last = lane_value(t.upto, l), first = last - lane_value(t.passes, l);
    if (t.g1 <= first || t.g0 >= last) return;
    const uint32_t io = lane_value(t.io, l), kind = lane_value(t.kind, l), n_in = io & 0xFFFFu, n_out = io >> 16;
    const bool has_mask = (kind >> 8 & 0xFFu) != 0, coded = (kind & 0xFFu) != 0;
    const uint32_t cb = coded ? kind & 0xFFu : 32u;
    const float scale = __uint_as_float(lane_value(__float_as_uint(t.scale), l));
    const int32_t zp = (int32_t)lane_value((uint32_t)t.zp, l);
    const uint32_t *mw = rec + (lane_value(t.mask_off, l) >> 2);
    const uint32_t *cs = rec + (lane_value(t.code_off, l) >> 2);
    const uint32_t p0 = t.g0 > first ? t.g0 - first : 0u, p1 = (t.g1 < last ? t.g1 : last) - first;
    const uint32_t i = 4u * ((uint32_t)lane % X::LANES);
    const uint32_t real = i >= n_in ? 0u : (n_in - i >= 4u ? 15u : (1u << (n_in - i)) - 1u);    // the lane's inputs that exist
    const uint32_t last_word = (n_in * n_out - 1u) >> 5;
    const uint32_t *select = (const uint32_t *)(lds + LY::SELECT);
    const PutFour<LY, TM> to((uint32_t)lane);
    const uint32_t zp4 = (uint32_t)zp * 0x01010101u;
    const h2v less = {(_Float16)(float)(-1024 - zp), (_Float16)(float)(-1024 - zp)};
    const uint32_t k0 = min(p0 * X::ROWS, n_out) * n_in;                        // weights before the wavefront's first pass
    uint32_t running = k0;
    if (has_mask && p0) {
        uint32_t part = 0;
        for (uint32_t wi = lane; wi <= min(k0 >> 5, last_word); wi += 64) part += __popc(mw[wi] & (wi == k0 >> 5 ? (1u << (k0 & 31u)) - 1u : 0xFFFFFFFFu));
        running = wave_sum(part);
    }
    for (uint32_t p = p0; p < p1; p += U) {
        uint32_t o[U], bits[U], rank[U];
        const uint32_t before = running;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            o[j] = (p + j) * X::ROWS + (uint32_t)lane / X::LANES;
            bits[j] = 15u;
            if (has_mask) {
                const uint32_t k = __umul24(o[j], n_in) + i, w = min(k >> 5, last_word);
                bits[j] = __builtin_amdgcn_alignbit(mw[min(w + 1u, last_word)], mw[w], k & 31u);
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            bits[j] &= o[j] < n_out ? real : 0u;
            const uint32_t c = (uint32_t)__popc(bits[j]);
            const uint64_t c0 = __ballot(c & 1u), c1 = __ballot(c & 2u), c2 = __ballot(c & 4u);
            const uint32_t r1 = __builtin_amdgcn_mbcnt_hi((uint32_t)(c1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)c1, 0u));
            const uint32_t r2 = __builtin_amdgcn_mbcnt_hi((uint32_t)(c2 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)c2, 0u));
            rank[j] = __builtin_amdgcn_mbcnt_hi((uint32_t)(c0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)c0, running)) + 2u * r1 + 4u * r2;
            rank[j] = bits[j] ? rank[j] : 0u;               // a lane without weights reads the first code and drops it
            running += (uint32_t)(__popcll(c0) + 2 * __popcll(c1) + 4 * __popcll(c2));
        }
        const bool some = running != before;                // no code kept: there may be none to read
        if (KIND == kHiddenAllInt || (KIND == kHiddenMixed && whole)) {
            uint32_t x[U], sel[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                sel[j] = select[bits[j]];
                x[j] = 0u;
            }
            if (some) {
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const uint32_t bit = __umul24(rank[j], cb);
                    x[j] = __builtin_amdgcn_alignbit(cs[(bit >> 5) + 1u], cs[bit >> 5], bit & 31u);
                }
                if (cb != 8u) {
                    const uint32_t m = (1u << cb) - 1u;
#pragma unroll
                    for (int j = 0; j < U; ++j)
                        x[j] = (x[j] & m) | (x[j] >> cb & m) << 8 | (x[j] >> 2u * cb & m) << 16 | (x[j] >> 3u * cb & m) << 24;
                }
            }
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t y = __builtin_amdgcn_perm(zp4, x[j], sel[j]);
                const h2v h01 = __builtin_bit_cast(h2v, __builtin_amdgcn_perm(0x64646464u, y, 0x04010400u)) + less;
                const h2v h23 = __builtin_bit_cast(h2v, __builtin_amdgcn_perm(0x64646464u, y, 0x04030402u)) + less;
                if (to.has && p + j < p1) to.put(hi, to.place(p + j), (h4v){h01[0], h01[1], h23[0], h23[1]}, (h4v)((_Float16)0.0f));
            }
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                h4v wh, wl;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const bool kept = bits[j] >> b & 1u;
                    const uint32_t rk = kept ? rank[j] + (uint32_t)__popc(bits[j] & ((1u << b) - 1u)) : 0u;
                    uint32_t code = 0u;
                    if (some) {
                        if (cb == 32u) code = cs[rk];
                        else if (cb == 16u) code = ((const uint16_t *)cs)[rk];
                        else if (W16 || KIND == kHiddenMixed || KIND == kHiddenAllRaw) code = take_code(cs, rk, cb);
                    }
                    const float v = coded ? scale * (float)((int32_t)code - zp) : __uint_as_float(code);
                    const float w = kept ? v * pre : 0.0f;
                    wh[b] = (_Float16)w;
                    wl[b] = (_Float16)(w - (float)wh[b]);
                }
                if (to.has && p + j < p1) {
                    const uint32_t place = to.place(p + j);
                    to.put(hi, place, wh, W16 ? (h4v)((_Float16)0.0f) : wl);
                    if (!W16 && !(LY::TAIL == kTailTwo && to.tail)) to.put(lo, place, wl, wl);
                }
            }
        }
    }
    if (p0 == 0) {
        const float *bias = (const float *)(rec + (lane_value(t.bias_off, l) >> 2));
        if ((uint32_t)lane < n_out) bt[LY::idx_bias(lane)] = bias[lane] * pre * bias_factor;
    }
}

// KIND says which kinds of hidden layer there can be (kHidden...), U how many passes of a hidden layer a wavefront has under way.
template <class LY, int TM, bool W16, bool SLOTTED, int KIND, int U>
__device__ __forceinline__ void xdl_expand_layers(char *lds, const uint32_t *rec, const LaneLayers &t, int L, int l0, int l1, float pre, int tid,
                                                  int nthreads) {
    constexpr int WP = LY::WP;
    const int lane = tid & 63;
    // lane l: layer l's entry; the offsets are sums over the lanes
    XLayer mine;
    {
        const bool last = lane == L - 1, in_group = lane >= l0 && lane < l1;
        const bool whole = !W16 && lane > 0 && !last && xdl_int_layer(t.kind & 0xFFu, t.scale * pre);
        const uint32_t one = lane == 0 ? LY::FIRST : (last ? LY::OUT : LY::HID), two = last ? LY::OUTLO : (lane > 0 && !W16 && !whole ? LY::HIDLO : 0u);
        const uint32_t size = one + two;
        const uint32_t upto = row_incl_sum(lane < L ? size : 0u);
        mine.off_bias = LY::TABLE + (SLOTTED ? (uint32_t)(lane - l0) * XSlot<LY>::BYTES : (uint32_t)lane * WP * 4u);
        mine.off_hi = SLOTTED ? mine.off_bias + XSlot<LY>::BIAS : LY::TABLE + (uint32_t)(L - 1) * WP * 4u + LY::OUTB + upto - size;
        mine.off_lo = last || (lane > 0 && !W16 && !whole) ? mine.off_hi + one : 0u;
        mine.scale = whole ? t.scale * pre : 1.0f;
        if (tid < 16) {
            if (in_group) ((XLayer *)lds)[lane] = mine;
            ((uint32_t *)(lds + LY::SELECT))[lane] = nibble_selector((uint32_t)lane);
        }
    }
    // cleared: the biases, the first layer's and the output layer's blocks (the hidden layers' are written whole)
    auto clear = [&](uint32_t from, uint32_t to) {
        for (uint32_t q = (from >> 4) + tid; q < (to >> 4); q += nthreads) ((uint4 *)lds)[q] = make_uint4(0u, 0u, 0u, 0u);
    };
    if (SLOTTED) {
        for (int l = l0; l < l1; ++l) {
            const uint32_t at = LY::TABLE + (uint32_t)(l - l0) * XSlot<LY>::BYTES;
            clear(at, at + (l == 0 || l == L - 1 ? XSlot<LY>::BYTES : XSlot<LY>::BIAS));
        }
    } else {
        const uint32_t out = lane_value(mine.off_hi, L - 1);
        clear(LY::TABLE, lane_value(mine.off_hi, 0) + LY::FIRST);
        clear(out, out + LY::OUT + LY::OUTLO);
    }
    // Rows of hidden layers' last tiles that are only padding: nothing reads what they make, but with whatever LDS held before in them the
    // matrix unit takes more energy (256 images of 160 x 160, 4 x 40 of 16-bit weights, fp16 activations: 172.3 us instead of 166.6).
    if (XExpand<LY::WQ>::PASSES * XExpand<LY::WQ>::ROWS < WP) {
        constexpr int STEPS = LY::KJ + (LY::TAIL != kTailNone ? 1 : 0), LOW = LY::KJ + (LY::TAIL == kTailFull ? 1 : 0), PER = 8 * LY::G;       // words of 16 bytes a step
        const int nwaves = nthreads >> 6;
        for (int l = max(l0, 1) + __builtin_amdgcn_readfirstlane(tid >> 6); l < min(l1, L - 1); l += nwaves) {
            const uint32_t hi = lane_value(mine.off_hi, l), lo = lane_value(mine.off_lo, l);
            for (int e = lane; e < STEPS * PER; e += 64) {
                const int j = e / PER, g = e / 8 % LY::G, m = LY::HALF ? (e & 6) * 2 + 2 + (e & 1) : TM - 8 + (e & 7);
                const uint32_t at = (uint32_t)(((j + 1) * LY::MT - 1) * 64 + g * TM + m) * 16u;
                *(uint4 *)(lds + hi + at) = make_uint4(0u, 0u, 0u, 0u);
                if (lo && j < LOW) *(uint4 *)(lds + lo + at) = make_uint4(0u, 0u, 0u, 0u);
            }
        }
    }
    __syncthreads();
    // only the layers that have passes of this wavefront (from the lanes: those whose passes end behind its first, and begin before its end)
    const uint64_t at = __ballot(t.passes != 0u && t.upto > t.g0 && t.upto - t.passes < t.g1) & 0xFFFFull;
    const int la = at ? __ffsll((unsigned long long)at) - 1 : 0, lb = at ? la + __popcll(at) : 0;
    for (int l = la; l < lb; ++l) {
        const uint32_t off_lo = lane_value(mine.off_lo, l);
        _Float16 *hi = (_Float16 *)(lds + lane_value(mine.off_hi, l)), *lo = (_Float16 *)(lds + off_lo);
        float *bt = (float *)(lds + lane_value(mine.off_bias, l));
        if (l == L - 1) {
            expand_layer<1>(rec, t, l, lane,
                         [=](int o, int i, float v, int) {
                             const _Float16 h = (_Float16)v, w = (_Float16)(v - (float)h);
                             const int at = LY::idx_out(o, i);
                             hi[at] = h;
                             if (LY::TAIL == kTailTwo && LY::in_tail(i)) {
                                 hi[at + 2] = h;
                                 hi[at + 4] = w;
                             } else {
                                 lo[at] = w;
                                 if (LY::TAIL == kTailFull && LY::in_tail(i)) {
                                     hi[at + 4] = h;
                                     lo[at + 4] = w;
                                 }
                             }
                         },
                         [=](int o, float v) { bt[LY::idx_bias_row(4 * o)] = v; });
        } else if (l == 0) {
            expand_layer<1>(rec, t, l, lane,
                         [=](int o, int i, float v, int) {
                             const float w = v * pre;
                             const _Float16 h = (_Float16)w, lw = (_Float16)(w - (float)h);
                             for (int q = 0; q < LY::G; ++q) {
                                 hi[LY::idx_first(q, o, i)] = h;          // pairs with the coordinate's high half
                                 hi[LY::idx_first(q, o, 2 + i)] = h;      // ... with its low half
                                 hi[LY::idx_first(q, o, 4 + i)] = lw;     // low weight part x high coordinate half
                             }
                         },
                         [=](int o, float v) { bt[LY::idx_bias(o)] = v * pre; });
        } else {
            const bool whole = !W16 && off_lo == 0;
            const float s = whole ? __uint_as_float(lane_value(__float_as_uint(mine.scale), l)) : 1.0f;
            expand_hidden<LY, TM, W16, KIND, U>(rec, t, l, lane, lds, (char *)hi, (char *)lo, bt, whole ? 1.0f / s : 1.0f, whole, pre);
        }
    }
    __syncthreads();
}

// Values every lane holds alike, moved to scalar registers
__device__ __forceinline__ float uniform_f(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ __forceinline__ XLayer uniform_layer(const XLayer e) {
    XLayer u;
    u.off_hi = __builtin_amdgcn_readfirstlane(e.off_hi);
    u.off_lo = __builtin_amdgcn_readfirstlane(e.off_lo);
    u.scale = uniform_f(e.scale);
    u.off_bias = __builtin_amdgcn_readfirstlane(e.off_bias);
    return u;
}

// ---- MFMA wrappers per tile shape -------------------------------------------------------------------
template <int TM> struct XTile;
template <> struct XTile<16> {
    typedef f32x4 acc_t;
    static __device__ __forceinline__ acc_t mfma(h8v a, h8v b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ acc_t mfma_half(h4v a, h4v b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0); }
};
template <> struct XTile<32> {
    typedef f32x16 acc_t;
    static __device__ __forceinline__ acc_t mfma(h8v a, h8v b, acc_t c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

// sine of four accumulator values (one quad), then the exact hi/lo split of the results: hi = fp16(h), lo = fp16(h - hi).
// The four differences come from one small matrix step, v_mfma_f32_4x4x4_16b_f16, C operand h, B operand hi, A operand minus the
// unit matrix (`neg_unit`): its 16 blocks are four lanes each, and with that A a lane gets its own C less its own B back.
// One product per sum and a difference that 32 bits hold: exact, and for finite activations the outputs are those of the
// four mixed-precision subtractions (v_fma_mix_f32) that it replaces, byte for byte.  (A sine is NaN only for a pre-activation that is no finite
// number; the step's products by zero then make the low parts of its whole quad NaN, which in a half-filled last tile is two pixels'.)  Those took 4.9 clocks each beside matrix work,
// this step takes about 4.2 (a matrix step delays vector instructions by a clock per operand register of A and B, and has two
// of each here, against four of each in a 16x16x32 step).  us before -> now: 256 images of 224 x 224, 6 x 64: 986 -> 955; 4096 of
// 32 x 32, 4 x 32: 109.3 -> 104.0; 64 of 224 x 224, 9 x 40: 283 -> 268; 256 of 160 x 160, 4 x 16: 88.2 -> 83.1, 4 x 64 of fp32 weights: 415 -> 408.
__device__ __forceinline__ void sine_split(float d0, float d1, float d2, float d3, float scale, h4v neg_unit, h4v &hi, h4v &lo) {
    const f2v p0 = {sin_rev(d0 * scale), sin_rev(d1 * scale)};
    const f2v p1 = {sin_rev(d2 * scale), sin_rev(d3 * scale)};
    const h2v a0 = __builtin_convertvector(p0, h2v), a1 = __builtin_convertvector(p1, h2v);
    hi = (h4v){a0[0], a0[1], a1[0], a1[1]};
    const f32x4 r = __builtin_amdgcn_mfma_f32_4x4x4f16(neg_unit, hi, (f32x4){p0[0], p0[1], p1[0], p1[1]}, 0, 0, 0);
    const f2v r0 = {r[0], r[1]}, r1 = {r[2], r[3]};
    const h2v b0 = __builtin_convertvector(r0, h2v), b1 = __builtin_convertvector(r1, h2v);
    lo = (h4v){b0[0], b0[1], b1[0], b1[1]};
}
// Row l % 4 of minus the unit matrix, the A operand of that step
__device__ __forceinline__ h4v xdl_neg_unit(int lane) {
    const _Float16 one = (_Float16)-1.0f, z = (_Float16)0.0f;
    const int r = lane & 3;
    return (h4v){r == 0 ? one : z, r == 1 ? one : z, r == 2 ? one : z, r == 3 ? one : z};
}

// sine of four accumulator values rounded to fp16 (single-term activations)
__device__ __forceinline__ void sine_hi(float d0, float d1, float d2, float d3, float scale, h4v &hi) {
    const f2v p0 = {sin_rev(d0 * scale), sin_rev(d1 * scale)};
    const f2v p1 = {sin_rev(d2 * scale), sin_rev(d3 * scale)};
    const h2v a0 = __builtin_convertvector(p0, h2v), a1 = __builtin_convertvector(p1, h2v);
    hi = (h4v){a0[0], a0[1], a1[0], a1[1]};
}

// Between the full-depth and the half-depth MFMAs of one set of accumulators: 20 wait states that no MFMA of the set
// can cross.  The empty asm statements make every accumulator an operand: the full-depth steps that produce it must
// come before the first, the half-depth steps that consume it after the last, and volatile asm statements keep their
// order, so the idle cycles sit between the two groups whatever the scheduler does with the rest.
template <class Acc> __device__ __forceinline__ void xdl_touch(Acc &acc) { asm volatile("" : "+v"(acc)); }
__device__ __forceinline__ void xdl_wait_states() { asm volatile("s_nop 15\n\ts_nop 3"); }

// ---- per-wavefront state of one half (32 pixels) of a 64-pixel tile ------------------------------------
template <int TM, class LY_> struct XHalf {
    typedef LY_ LY;
    static constexpr int NTH = 32 / TM;            // pixel tiles in a half: two of 16 pixels, or one of 32
    static constexpr int KJA = LY::KJ ? LY::KJ : 1;
    h8v Hh[NTH][KJA], Hl[NTH][KJA];                // activations as fp16 hi / lo, one entry per full k-step
    h4v Hh4[NTH], Hl4[NTH];                        // ... of the last quad (kTailHalf)
    h8v Ht[NTH];                                   // ... or of its full-depth step (kTailFull, kTailTwo)
    typename XTile<TM>::acc_t D[NTH][LY::MT];      // accumulators
};

// sine + split of all accumulators of a half: WQ/2 activations per lane, 3 VALU instructions and a quarter of a small matrix step each
template <int TM, class LY, bool A16>
__device__ __forceinline__ void xdl_epilogue(XHalf<TM, LY> &H, float scale, h4v neg_unit) {
    constexpr int QT = LY::RV / 4;                 // quads per tile
    constexpr int NTH = XHalf<TM, LY>::NTH;
    const h4v none = (h4v)((_Float16)0.0f);
#pragma unroll
    for (int nt = 0; nt < NTH; ++nt)
#pragma unroll
        for (int q = 0; q < LY::NQ - (LY::HALF ? 1 : 0); ++q) {
            const int t = q / QT, v0 = q % QT * 4;
            h4v hi, lo = none;
            if (A16) sine_hi(H.D[nt][t][v0], H.D[nt][t][v0 + 1], H.D[nt][t][v0 + 2], H.D[nt][t][v0 + 3], scale, hi);
            else sine_split(H.D[nt][t][v0], H.D[nt][t][v0 + 1], H.D[nt][t][v0 + 2], H.D[nt][t][v0 + 3], scale, neg_unit, hi, lo);
            if (q < 2 * LY::KJ) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    H.Hh[nt][q >> 1][(q & 1) * 4 + v] = hi[v];
                    if (!A16) H.Hl[nt][q >> 1][(q & 1) * 4 + v] = lo[v];
                }
            } else if (LY::TAIL == kTailHalf) {
                H.Hh4[nt] = hi;
                if (!A16) H.Hl4[nt] = lo;
            } else {
                H.Ht[nt] = __builtin_shufflevector(hi, lo, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
    if constexpr (LY::HALF) {                      // two rows a lane of the last tile: the two pixel tiles make one quad for the split
        constexpr int t = LY::MT - 1;
        h4v hi, lo = none;
        if (A16) sine_hi(H.D[0][t][0], H.D[0][t][1], H.D[1][t][0], H.D[1][t][1], scale, hi);
        else sine_split(H.D[0][t][0], H.D[0][t][1], H.D[1][t][0], H.D[1][t][1], scale, neg_unit, hi, lo);
        if (LY::TAIL == kTailTwo) {
            H.Ht[0] = __builtin_shufflevector(hi, lo, 0, 1, 4, 5, 0, 1, 4, 5);
            H.Ht[1] = __builtin_shufflevector(hi, lo, 2, 3, 6, 7, 2, 3, 6, 7);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    H.Hh[nt][LY::KJ - 1][4 + v] = v < 2 ? hi[2 * nt + v] : (_Float16)0.0f;
                    if (!A16) H.Hl[nt][LY::KJ - 1][4 + v] = v < 2 ? lo[2 * nt + v] : (_Float16)0.0f;
                }
        }
    }
}

// MFMAs of one hidden layer for a half.  LO: the layer has a low weight part (one more term).  A16: no low activation part.
template <int TM, class LY, bool LO, bool A16>
__device__ __forceinline__ void xdl_hidden(XHalf<TM, LY> &H, const char *lds, const XLayer el, uint32_t lane, uint32_t g) {
    typedef XTile<TM> T;
    typedef typename T::acc_t acc_t;
    constexpr int KJ = LY::KJ, MT = LY::MT, NTH = XHalf<TM, LY>::NTH;
    const h8v *ah = (const h8v *)(lds + el.off_hi) + lane;
    const h8v *al = (const h8v *)(lds + el.off_lo) + lane;
    const acc_t *bt = (const acc_t *)(lds + el.off_bias) + g;
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const h8v av = ah[(j * MT + mt) * 64];
            h8v aw;
            if (LO) aw = al[(j * MT + mt) * 64];
            acc_t c;
            if (j == 0) c = bt[mt * LY::G];
#pragma unroll
            for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma(av, H.Hh[nt][j], j == 0 ? c : H.D[nt][mt]);
            if (!A16) {
#pragma unroll
                for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma(av, H.Hl[nt][j], H.D[nt][mt]);
            }
            if (LO) {
#pragma unroll
                for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma(aw, H.Hh[nt][j], H.D[nt][mt]);
            }
        }
    if constexpr (LY::TAIL == kTailFull || LY::TAIL == kTailTwo) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const h8v av = ah[(KJ * MT + mt) * 64];
            acc_t c;
            if (KJ == 0) c = bt[mt * LY::G];
#pragma unroll
            for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma(av, H.Ht[nt], KJ == 0 ? c : H.D[nt][mt]);
            if (LO && LY::TAIL == kTailFull) {
                const h8v aw = al[(KJ * MT + mt) * 64];
#pragma unroll
                for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma(aw, H.Ht[nt], H.D[nt][mt]);
            }
        }
    }
    if constexpr (LY::TAIL == kTailHalf) {
        const h4v *ah4 = (const h4v *)(lds + el.off_hi + KJ * MT * 1024) + lane;
        const h4v *al4 = (const h4v *)(lds + el.off_lo + KJ * MT * 1024) + lane;
        if (KJ) {
#pragma unroll
            for (int nt = 0; nt < NTH; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) xdl_touch(H.D[nt][mt]);
            xdl_wait_states();
#pragma unroll
            for (int nt = 0; nt < NTH; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) xdl_touch(H.D[nt][mt]);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const h4v av = ah4[mt * 64];
            h4v aw;
            if (LO) aw = al4[mt * 64];
            acc_t c;
            if (KJ == 0) c = bt[mt * LY::G];
#pragma unroll
            for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma_half(av, H.Hh4[nt], KJ == 0 ? c : H.D[nt][mt]);
            if (!A16) {
#pragma unroll
                for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma_half(av, H.Hl4[nt], H.D[nt][mt]);
            }
            if (LO) {
#pragma unroll
                for (int nt = 0; nt < NTH; ++nt) H.D[nt][mt] = T::mfma_half(aw, H.Hh4[nt], H.D[nt][mt]);
            }
        }
    }
}

// One hidden layer for both halves of a 64-pixel tile, software-pipelined: the matrix work of X(l) is issued
// together with the sine/split of Y(l-1), then the matrix work of Y(l) with the sine/split of X(l).
template <int TM, class LY, bool LO, bool A16>
__device__ __forceinline__ void xdl_layer(XHalf<TM, LY> &X, XHalf<TM, LY> &Y, const char *lds, const XLayer el, uint32_t lane, uint32_t g,
                                          float scale_prev, float scale, h4v neg_unit) {
    xdl_hidden<TM, LY, LO, A16>(X, lds, el, lane, g);
    xdl_epilogue<TM, LY, A16>(Y, scale_prev, neg_unit);
    __builtin_amdgcn_sched_barrier(0);
    xdl_hidden<TM, LY, LO, A16>(Y, lds, el, lane, g);
    xdl_epilogue<TM, LY, A16>(X, scale, neg_unit);
}

// The slot's augmentation map (every lane holds it alike), in scalar registers.
struct XUniform {
    float af0, af1, af2, af3, af4, af5;
};
__device__ __forceinline__ XUniform xdl_uniform(const DecodeArgs &a, uint32_t slot) {
    XUniform u;
    u.af0 = 1.0f; u.af1 = 0.0f; u.af2 = 0.0f; u.af3 = 0.0f; u.af4 = 1.0f; u.af5 = 0.0f;   // augmentation: this slot's map of the sampling grid
    if (a.affine) {
        const float *m = a.affine + (size_t)slot * 6;
        u.af0 = uniform_f(m[0]); u.af1 = uniform_f(m[1]); u.af2 = uniform_f(m[2]);
        u.af3 = uniform_f(m[3]); u.af4 = uniform_f(m[4]); u.af5 = uniform_f(m[5]);
    }
    return u;
}

// ---- first layer: every lane forms the coordinates of one pixel of the tile as hi/lo halfs in
//      k slots (xh, yh, xl, yl, xh, yh, 0, 0); the MFMA of pixel tile q uses the weight variant whose
//      non-zero k slots are lane group q's, so one operand register set serves all pixel tiles.
//      Per-lane values that only the first and the last layer use are derived again for every tile
//      (the empty asm keeps them from being hoisted): held across the hidden layers they would
//      push the kernel over its register budget.
template <int TM, class LY>
__device__ __forceinline__ void xdl_first(XHalf<TM, LY> &X, XHalf<TM, LY> &Y, const DecodeArgs &a, const XUniform &u, const char *lds,
                                          const XLayer e0, uint32_t tile, uint32_t lane) {
    typedef XTile<TM> T;
    typedef typename T::acc_t acc_t;
    constexpr int MT = LY::MT, G = LY::G, NTH = XHalf<TM, LY>::NTH;
    const uint32_t g = lane / TM;
    float lo_v = a.lo, af2 = u.af2, af5 = u.af5;        // second uniform operand of an fma: copied to a vector register at the use
    asm volatile("" : "+s"(lo_v), "+s"(af2), "+s"(af5));
    const h8v *a0 = (const h8v *)(lds + e0.off_hi) + lane;
    const acc_t *bt = (const acc_t *)(lds + e0.off_bias) + g;
    // lane (pixel tile q = lane / TM, column n = lane % TM) feeds pixel n * (64 / TM) + q of the 64: a lane's columns of the
    // pixel tiles are then consecutive pixels, which the output layer stores as one vector.  The tile's first pixel's row and column are the
    // scalar unit's; a lane is at most 63 pixels on, which is one row at most, or, where rows are shorter, a small quotient.
    const uint32_t p0 = tile << 6, row0 = a.wmagic ? (__umulhi(p0, a.wmagic) >> a.wshift) : p0;
    uint32_t col = p0 - row0 * a.W + min(lane % TM * (64 / TM) + lane / TM, a.HW - 1 - p0), row;
    if (a.wsmall) {
        const uint32_t q = __umul24(col, a.wsmall) >> 16;
        col -= __umul24(q, a.W);
        row = row0 + q;
    } else {
        const bool next = col >= a.W;
        col -= next ? a.W : 0u;
        row = row0 + next;
    }
    const float x0 = fmaf(a.span, (float)(2 * col + 1) * a.inv2W, lo_v);
    const float y0 = fmaf(a.span, (float)(2 * row + 1) * a.inv2H, lo_v);
    float x = x0, y = y0;
    if (a.affine) {
        asm volatile("");                               // a branch, not selects
        x = fmaf(u.af0, x0, fmaf(u.af1, y0, af2));
        y = fmaf(u.af3, x0, fmaf(u.af4, y0, af5));
    }
    const _Float16 xh = (_Float16)x, yh = (_Float16)y;
    const _Float16 xl = (_Float16)(x - (float)xh), yl = (_Float16)(y - (float)yh);
    const _Float16 z = (_Float16)0.0f;
    const h8v b0 = {xh, yh, xl, yl, xh, yh, z, z};
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const acc_t c = bt[mt * G];
#pragma unroll
        for (int nt = 0; nt < NTH; ++nt) {
            X.D[nt][mt] = T::mfma(a0[(nt * MT + mt) * 64], b0, c);
            Y.D[nt][mt] = T::mfma(a0[((NTH + nt) * MT + mt) * 64], b0, c);
        }
    }
}

// ---- output layer width -> 3: one TM-row tile with channel c in row 4c.  At TM = 16 that is
//      register 0 of lane group c; at TM = 32 registers 0 (R) and 4 (B) of group 0, register 0 (G) of group 1.
//      Then clamp, optional normalisation and the NCHW store.
template <int TM, class LY, bool A16>
__device__ __forceinline__ void xdl_output(const XHalf<TM, LY> &X, const XHalf<TM, LY> &Y, const DecodeArgs &a, float ns0, float ns1,
                                           float ns2, float nb0, float nb1, float nb2, const char *lds, const XLayer eo,
                                           uint32_t tile, uint32_t lane, uint32_t chan, size_t plane0) {
    typedef XTile<TM> T;
    typedef typename T::acc_t acc_t;
    constexpr int KJ = LY::KJ, NTH = XHalf<TM, LY>::NTH;
    const uint32_t go = lane / TM, no = lane % TM;
    const h8v *ah = (const h8v *)(lds + eo.off_hi) + lane;
    const h8v *al = (const h8v *)(lds + eo.off_lo) + lane;
    const acc_t c = ((const acc_t *)(lds + eo.off_bias))[go];
    acc_t O[2 * NTH];
#pragma unroll
    for (int nt = 0; nt < 2 * NTH; ++nt) O[nt] = c;
#pragma unroll
    for (int j = 0; j < KJ; ++j) {
        const h8v av = ah[j * 64], aw = al[j * 64];
#pragma unroll
        for (int nt = 0; nt < 2 * NTH; ++nt) {
            const h8v bh = nt < NTH ? X.Hh[nt % NTH][j] : Y.Hh[nt % NTH][j];
            O[nt] = T::mfma(av, bh, O[nt]);
            if (!A16) O[nt] = T::mfma(av, nt < NTH ? X.Hl[nt % NTH][j] : Y.Hl[nt % NTH][j], O[nt]);
            O[nt] = T::mfma(aw, bh, O[nt]);
        }
    }
    if constexpr (LY::TAIL == kTailFull || LY::TAIL == kTailTwo) {
        const h8v av = ah[KJ * 64];
        h8v aw;
        if (LY::TAIL == kTailFull) aw = al[KJ * 64];
#pragma unroll
        for (int nt = 0; nt < 2 * NTH; ++nt) {
            const h8v bt = nt < NTH ? X.Ht[nt % NTH] : Y.Ht[nt % NTH];
            O[nt] = T::mfma(av, bt, O[nt]);
            if (LY::TAIL == kTailFull) O[nt] = T::mfma(aw, bt, O[nt]);
        }
    }
    if constexpr (LY::TAIL == kTailHalf) {
        const h4v *ah4 = (const h4v *)(lds + eo.off_hi + KJ * 1024) + lane;
        const h4v *al4 = (const h4v *)(lds + eo.off_lo + KJ * 1024) + lane;
        if (KJ) {
#pragma unroll
            for (int nt = 0; nt < 2 * NTH; ++nt) xdl_touch(O[nt]);
            xdl_wait_states();
#pragma unroll
            for (int nt = 0; nt < 2 * NTH; ++nt) xdl_touch(O[nt]);
        }
        const h4v av = ah4[0], aw = al4[0];
#pragma unroll
        for (int nt = 0; nt < 2 * NTH; ++nt) {
            const h4v bh = nt < NTH ? X.Hh4[nt % NTH] : Y.Hh4[nt % NTH];
            O[nt] = T::mfma_half(av, bh, O[nt]);
            if (!A16) O[nt] = T::mfma_half(av, nt < NTH ? X.Hl4[nt % NTH] : Y.Hl4[nt % NTH], O[nt]);
            O[nt] = T::mfma_half(aw, bh, O[nt]);
        }
    }
    // lane (go, no) holds column `no` of every pixel tile: pixels p0 .. p0 + NT - 1 of the image, NT = 64 / TM
    constexpr int NT = 2 * NTH;
    constexpr int NS = TM == 16 ? 1 : 2;         // channels a lane stores: TM = 16: channel go; TM = 32: R and B (group 0), G (group 1)
    const uint32_t p0 = (tile << 6) + (uint32_t)no * NT;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const uint32_t ch = TM == 16 ? go : (go == 0 ? 2 * k : 1);
        const bool live = TM == 16 ? go < 3 : (go == 0 || k == 0);
        float r[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            r[nt] = O[nt][TM == 16 ? 0 : 4 * k];
        }
        if (!a.no_clamp) {
            asm volatile("");                               // branches, not selects
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) r[nt] = fminf(fmaxf(r[nt], 0.0f), 1.0f);
        }
        if (a.normalize) {
            asm volatile("");
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) r[nt] = fmaf(r[nt], ch == 0 ? ns0 : (ch == 1 ? ns1 : ns2), ch == 0 ? nb0 : (ch == 1 ? nb1 : nb2));
        }
        const uint32_t at = (TM == 16 ? chan : (k ? 2u * a.HW : chan)) + p0;    // within the slot's three planes: 3 HW < 2^32 is checked by the host
        // A lane's pixels go out as one vector wherever its plane begins: global memory takes vectors at any float's address, and words at any
        // byte's.  Only the lane that has the image's last pixels takes them singly, where they are fewer.  us, a pixel at a
        // time in odd sizes -> so: 300 images of 129 x 127, 3 x 8 58.1 -> 53.2; 4096 of 31 x 33, 2 x 15, fp16 activations 34.0 -> 32.3; 64 of 223 x 225, 3 x 24, bytes 50.5 -> 48.9,
        // 6 x 40 164.7 -> 164.2; 2 of 1021 x 1363, 9 x 32 of 16-bit weights, bytes 152.3 -> 150.3.
        if (live && p0 + NT <= a.HW) {
            if (a.out_f32) {
                typedef float vec_t __attribute__((ext_vector_type(NT), aligned(4)));
                float *dst = a.out_f32 + plane0 + at;
                vec_t w;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) w[nt] = r[nt];
                *(vec_t *)dst = w;
            }
            if (a.out_u8) {
                uint32_t pk = 0u;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) pk = __builtin_amdgcn_cvt_pk_u8_f32(255.0f * r[nt], nt, pk);   // round to nearest even, packed
                uint8_t *dst = a.out_u8 + plane0 + at;
                if constexpr (NT == 4) {
                    typedef uint32_t word_t __attribute__((aligned(1)));
                    *(word_t *)dst = pk;
                } else {
                    typedef uint16_t word_t __attribute__((aligned(1)));
                    *(word_t *)dst = (uint16_t)pk;
                }
            }
        }
        if (!a.vec_store && live && p0 < a.HW && p0 + NT > a.HW) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (p0 + nt < a.HW) {
                    if (a.out_f32) (a.out_f32 + plane0)[at + nt] = r[nt];
                    if (a.out_u8) (a.out_u8 + plane0)[at + nt] = (uint8_t)rintf(255.0f * r[nt]);
                }
        }
    }
}

// Resident form: the model is expanded once per workgroup; a wavefront takes one 64-pixel tile at a time through all
// layers.  What a tile costs beside its layers counts at small models (3 x 15: 108 of 188 vector instructions): pixel indices come from
// the scalar unit and an addition per lane, the augmentation map, the clamp and the normalisation are branches that a launch without
// them skips, where a layer's blocks are is arithmetic.  us a call, before -> now: 4096 images of 32 x 32, fp16 activations, 2 x 15: 34.3 ->
// 31.4; 4 x 32: 100.2 -> 96.1; 1024 of 64 x 64, 5 x 48: 180.2 -> 176.3; 256 of 224 x 224, 6 x 64: 914 -> 905; 256 of 160 x 160, 4 x 8: 65.1 -> 58.3.
template <int TM, int WQ, int MODE_>
__device__ __forceinline__ void xdl_body(const DecodeArgs &a, const Work &w, float *lds_f) {
    constexpr bool W16 = (MODE_ & kWeight16) != 0;
    constexpr int MODE = W16 ? (int)kHiddenAllRaw : (MODE_ & 3);      // all-fp16: one form for every hidden layer, no scale
    constexpr bool A16 = (MODE_ & kAct16) != 0 || W16;
    typedef XLayout<TM, WQ, MODE_ == kHiddenAllInt> LY;
    typedef XHalf<TM, LY> Half;
    constexpr int WP = LY::WP;
    static_assert(xdl_bytes_hold<TM, LY>(), "what the host sizes LDS for");
    char *lds = (char *)lds_f;
    const int tid = threadIdx.x, nthreads = blockDim.x;
    const uint32_t tile0 = w.tile0, tile1 = w.tile1;
    const size_t plane0 = w.plane0;
    const IndexEntry e = w.e;
    const int L = e.n_layers;

    // the packed record is staged at the end of the workgroup's LDS, the operand blocks are built at the start
    const uint8_t *record = a.blob + e.off;
    const uint32_t room = a.lds_bytes - 16u;                     // behind it: the tile counter
    // Tiles are handed out through a counter in LDS: the SIMD arbiter favours its older wavefront, so
    // with a fixed split the favoured waves would finish early and leave the others running alone.
    uint32_t *next_tile = (uint32_t *)(lds + room);
    if (tid == 0) *next_tile = tile0 + (nthreads >> 6);
    {
        const LaneLayers t = lane_layers<XExpand<LY::WQ>::PASSES>(record, L, 0, L, tid & 63, __builtin_amdgcn_readfirstlane(tid >> 6), nthreads >> 6);
        constexpr XBytes bytes = xdl_bytes(TM, WQ, LY::INTS, true);
        const uint32_t need = bytes.base + (uint32_t)(L - 2) * bytes.layer;
        if (MODE == kHiddenAllInt || W16 || need + e.nbytes <= room) {     // (in one-block form a model fits with its record)
            uint32_t *stage = (uint32_t *)(lds + (room - e.nbytes));
            for (uint32_t q = tid; q < (e.nbytes >> 4); q += nthreads) ((uint4 *)stage)[q] = ((const uint4 *)record)[q];
            xdl_expand_layers<LY, TM, W16, false, MODE, (WP <= 32 ? 1 : 2)>(lds, stage, t, L, 0, L, a.pre, tid, nthreads);
        } else {
            xdl_expand_layers<LY, TM, W16, false, MODE, 1>(lds, (const uint32_t *)record, t, L, 0, L, a.pre, tid, nthreads);
        }
    }

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const XLayer *tab = (const XLayer *)lds;
    const h4v neg_unit = xdl_neg_unit(tid & 63);
    const XLayer e0 = uniform_layer(tab[0]), eo = uniform_layer(tab[L - 1]);
    const XUniform u = xdl_uniform(a, w.slot);
    // per-channel normalisation constants as values (not as an address chosen per lane)
    const float ns0 = uniform_f(a.ns[0]), ns1 = uniform_f(a.ns[1]), ns2 = uniform_f(a.ns[2]);
    const float nb0 = uniform_f(a.nb[0]), nb1 = uniform_f(a.nb[1]), nb2 = uniform_f(a.nb[2]);

    uint32_t chan = (uint32_t)(tid & 63) / TM * a.HW;            // the first plane this lane stores to
    asm volatile("" : "+v"(chan));
    // Where a layer's blocks are: known from its number where all hidden layers are of one kind, else from the table
    const uint32_t hidden0 = e0.off_hi + LY::FIRST;
    auto layer = [&](int l) -> XLayer {
        if (MODE == kHiddenMixed) return uniform_layer(tab[l]);
        XLayer el;
        el.off_hi = hidden0 + (uint32_t)(l - 1) * (MODE == kHiddenAllInt || W16 ? LY::HID : LY::HID + LY::HIDLO);
        el.off_lo = MODE == kHiddenAllInt || W16 ? 0u : el.off_hi + LY::HID;
        el.scale = MODE == kHiddenAllInt ? uniform_f(tab[l].scale) : 1.0f;
        el.off_bias = LY::TABLE + (uint32_t)l * WP * 4u;
        return el;
    };
    for (uint32_t tile = tile0 + wave; tile < tile1;) {
        Half X, Y;
        uint32_t ones = ~0u;
        asm volatile("" : "+s"(ones));
        uint32_t lane = __builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0u));
        xdl_first<TM, LY>(X, Y, a, u, lds, e0, tile, lane);
        xdl_epilogue<TM, LY, A16>(X, 1.0f, neg_unit);
        // ---- hidden layers, software-pipelined over the two halves:
        //      matrix work of X(l) with the sine/split of Y(l-1), then matrix work of Y(l) with the sine/split of X(l)
        float scale_prev = 1.0f;
        int l = 1;
        if (MODE == kHiddenAllInt && L > 2) {      // first hidden layer on its own: the first layer's outputs carry no scale
            const XLayer el = layer(1);
            uint32_t ll = lane;
            asm volatile("" : "+v"(ll));
            xdl_layer<TM, LY, false, A16>(X, Y, lds, el, ll, ll / TM, 1.0f, el.scale, neg_unit);
            scale_prev = el.scale;
            l = 2;
        }
        for (; l < L - 1; ++l) {
            const XLayer el = layer(l);
            uint32_t ll = lane;                       // the lane group is derived from the lane index per layer, not kept
            asm volatile("" : "+v"(ll));
            if constexpr (MODE == kHiddenAllInt) {
                xdl_layer<TM, LY, false, A16>(X, Y, lds, el, ll, ll / TM, scale_prev, el.scale, neg_unit);
            } else if constexpr (MODE == kHiddenAllRaw) {
                xdl_layer<TM, LY, !W16, A16>(X, Y, lds, el, ll, ll / TM, 1.0f, 1.0f, neg_unit);
            } else {
                if (el.off_lo == 0) xdl_layer<TM, LY, false, A16>(X, Y, lds, el, ll, ll / TM, scale_prev, el.scale, neg_unit);
                else xdl_layer<TM, LY, true, A16>(X, Y, lds, el, ll, ll / TM, scale_prev, el.scale, neg_unit);
            }
            scale_prev = el.scale;
        }
        xdl_epilogue<TM, LY, A16>(Y, scale_prev, neg_unit);
        asm volatile("" : "+s"(ones));           // pixel indices and addresses: derived again rather than kept
        lane = __builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0u));
        xdl_output<TM, LY, A16>(X, Y, a, ns0, ns1, ns2, nb0, nb1, nb2, lds, eo, tile, lane, chan, plane0);
        uint32_t nt_ = 0;
        if (lane == 0) nt_ = atomicAdd(next_tile, 1u);
        tile = __builtin_amdgcn_readfirstlane(nt_);
    }
}

// Streamed form, for a model whose operand blocks do not fit LDS: the layers go through LDS in groups of as many
// slots as fit.  Every wavefront keeps one tile in registers (both halves, mid-pipeline: X holds activations, Y
// accumulators awaiting their sine); for each group the workgroup builds the group's blocks straight from the
// packed record in global memory, then every wavefront takes its tile through the group's layers.
template <int TM, int WQ, int MODE_>
__device__ __forceinline__ void xdl_stream_body(const DecodeArgs &a, const Work &w, float *lds_f) {
    constexpr bool W16 = (MODE_ & kWeight16) != 0;
    constexpr bool A16 = (MODE_ & kAct16) != 0 || W16;
    typedef XLayout<TM, WQ, MODE_ == kHiddenAllInt> LY;
    typedef XHalf<TM, LY> Half;
    char *lds = (char *)lds_f;
    const int tid = threadIdx.x, nthreads = blockDim.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthreads >> 6;
    const IndexEntry e = w.e;
    const int L = e.n_layers;
    const int K = (int)((a.lds_bytes - LY::TABLE) / (uint32_t)XSlot<LY>::BYTES);   // layers per group (>= 1 by the host's launch size)
    const uint32_t *rec = (const uint32_t *)(a.blob + e.off);
    const XLayer *tab = (const XLayer *)lds;
    const h4v neg_unit = xdl_neg_unit(tid & 63);
    const XUniform u = xdl_uniform(a, w.slot);
    // per-channel normalisation constants as values (not as an address chosen per lane)
    const float ns0 = uniform_f(a.ns[0]), ns1 = uniform_f(a.ns[1]), ns2 = uniform_f(a.ns[2]);
    const float nb0 = uniform_f(a.nb[0]), nb1 = uniform_f(a.nb[1]), nb2 = uniform_f(a.nb[2]);

    for (uint32_t t0 = w.tile0; t0 < w.tile1; t0 += (uint32_t)nwaves) {
        const uint32_t tile = t0 + (uint32_t)wave;
        const bool active = tile < w.tile1;                            // the same for a whole wavefront
        Half X, Y;
        float scale_prev = 1.0f;
        for (int l0 = 0; l0 < L; l0 += K) {
            const int l1 = l0 + K < L ? l0 + K : L;
            __syncthreads();                                           // every wavefront is done with the previous group
            const LaneLayers t = lane_layers<XExpand<LY::WQ>::PASSES>((const uint8_t *)rec, L, l0, l1, lane, wave, nwaves);
            xdl_expand_layers<LY, TM, W16, true, kHiddenMixed, 1>(lds, rec, t, L, l0, l1, a.pre, tid, nthreads);
            if (!active) continue;
            for (int l = l0; l < l1; ++l) {
                const XLayer el = uniform_layer(tab[l]);
                if (l == 0) {
                    xdl_first<TM, LY>(X, Y, a, u, lds, el, tile, lane);
                    xdl_epilogue<TM, LY, A16>(X, 1.0f, neg_unit);
                } else if (l < L - 1) {
                    if (W16) xdl_layer<TM, LY, false, A16>(X, Y, lds, el, lane, lane / TM, 1.0f, 1.0f, neg_unit);
                    else if (el.off_lo == 0) xdl_layer<TM, LY, false, A16>(X, Y, lds, el, lane, lane / TM, scale_prev, el.scale, neg_unit);
                    else xdl_layer<TM, LY, true, A16>(X, Y, lds, el, lane, lane / TM, scale_prev, el.scale, neg_unit);
                    scale_prev = W16 ? 1.0f : el.scale;
                } else {
                    xdl_epilogue<TM, LY, A16>(Y, scale_prev, neg_unit);
                    xdl_output<TM, LY, A16>(X, Y, a, ns0, ns1, ns2, nb0, nb1, nb2, lds, el, tile, lane, (uint32_t)lane / TM * a.HW, w.plane0);
                }
            }
        }
    }
}

// One width class per launch (a.cls != 0): WQ is the class's padded width, or 8 less where the store has no wider model of the class.
// (One kernel with both bodies, chosen per model, takes more registers than either, and 2048 ragged images of 32 x 32, decoded class by
// class, went from 135 to 141 us.) ...
template <int WQ, int NTHREADS, int MODE>
__global__ __launch_bounds__(NTHREADS) void decode_xdl_kernel(const DecodeArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    Work w;
    if (!decode_prologue(a, w)) return;
    xdl_body<xdl_tile_rows(WQ, MODE), WQ, MODE>(a, w, lds_f);
}

// ... or every width class in one launch (a.cls == 0)
template <int NTHREADS, int MODE>
__global__ __launch_bounds__(NTHREADS) void decode_xdl_any_kernel(const DecodeArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    Work w;
    if (!decode_prologue(a, w)) return;
    switch ((w.e.width + 7u) >> 3) {
        case 0: case 1: xdl_body<xdl_any_tile_rows(8, MODE), 8, MODE>(a, w, lds_f); break;
        case 2: xdl_body<xdl_any_tile_rows(16, MODE), 16, MODE>(a, w, lds_f); break;
        case 3: xdl_body<xdl_any_tile_rows(24, MODE), 24, MODE>(a, w, lds_f); break;
        case 4: xdl_body<xdl_any_tile_rows(32, MODE), 32, MODE>(a, w, lds_f); break;
        case 5: xdl_body<xdl_any_tile_rows(40, MODE), 40, MODE>(a, w, lds_f); break;
        case 6: xdl_body<xdl_any_tile_rows(48, MODE), 48, MODE>(a, w, lds_f); break;
        case 7: xdl_body<xdl_any_tile_rows(56, MODE), 56, MODE>(a, w, lds_f); break;
        default: xdl_body<xdl_any_tile_rows(64, MODE), 64, MODE>(a, w, lds_f); break;
    }
}

// The streamed form: one width class per launch, one wavefront per SIMD.  MODE: kHiddenAllInt or kHiddenMixed (hi+lo activations; the
// resident kernels' layout for such models, so that the bytes are the same), kHiddenMixed | kAct16, or kHiddenMixed | kAct16 | kWeight16.
template <int WQ, int MODE>
__global__ __launch_bounds__(kStreamThreads) void decode_xdl_stream_kernel(const DecodeArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    Work w;
    if (!decode_prologue(a, w)) return;
    xdl_stream_body<xdl_tile_rows(WQ, MODE), WQ, MODE>(a, w, lds_f);
}

// ... in a store of several width classes: the bodies of the all-class kernel, for the same bytes (a launch still serves one class)
template <int MODE>
__global__ __launch_bounds__(kStreamThreads) void decode_xdl_stream_any_kernel(const DecodeArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    Work w;
    if (!decode_prologue(a, w)) return;
    switch ((w.e.width + 7u) >> 3) {
        case 0: case 1: xdl_stream_body<xdl_any_tile_rows(8, MODE), 8, MODE>(a, w, lds_f); break;
        case 2: xdl_stream_body<xdl_any_tile_rows(16, MODE), 16, MODE>(a, w, lds_f); break;
        case 3: xdl_stream_body<xdl_any_tile_rows(24, MODE), 24, MODE>(a, w, lds_f); break;
        case 4: xdl_stream_body<xdl_any_tile_rows(32, MODE), 32, MODE>(a, w, lds_f); break;
        case 5: xdl_stream_body<xdl_any_tile_rows(40, MODE), 40, MODE>(a, w, lds_f); break;
        case 6: xdl_stream_body<xdl_any_tile_rows(48, MODE), 48, MODE>(a, w, lds_f); break;
        case 7: xdl_stream_body<xdl_any_tile_rows(56, MODE), 56, MODE>(a, w, lds_f); break;
        default: xdl_stream_body<xdl_any_tile_rows(64, MODE), 64, MODE>(a, w, lds_f); break;
    }
}

// ---- debug export of the split-precision operand blocks (see rinr_debug_dequant_split) ----------------------------
template <int TM, int WQ, int KIND, bool W16>
__global__ __launch_bounds__(256) void xdl_debug_kernel(const uint8_t *blob, int64_t id, int layer, uint32_t lds_bytes,
                                                        float *hi_out, float *lo_out, float *bias_out, float *scale_out) {
    typedef XLayout<TM, WQ, !W16 && KIND == kHiddenAllInt> LY;
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    char *lds = (char *)lds_f;
    const IndexEntry e = *(const IndexEntry *)(blob + sizeof(StoreHeader) + (size_t)id * sizeof(IndexEntry));
    const int tid = threadIdx.x, nthreads = blockDim.x;
    const int L = e.n_layers;
    const uint32_t *rec = (const uint32_t *)(blob + e.off);
    // one layer at a time in the slotted layout, straight from global memory: any depth fits
    const LaneLayers t = lane_layers<XExpand<LY::WQ>::PASSES>((const uint8_t *)rec, L, layer, layer + 1, tid & 63, __builtin_amdgcn_readfirstlane(tid >> 6), nthreads >> 6);
    xdl_expand_layers<LY, TM, W16, true, kHiddenMixed, 1>(lds, rec, t, L, layer, layer + 1, 1.0f, tid, nthreads);
    const XLayer el = ((const XLayer *)lds)[layer];
    const LayerRec r = *(const LayerRec *)(rec + layer * (sizeof(LayerRec) / 4));
    const _Float16 *hi = (const _Float16 *)(lds + el.off_hi), *lo = (const _Float16 *)(lds + el.off_lo);
    const float *bt = (const float *)(lds + el.off_bias);
    const int n_in = r.n_in, cnt = r.n_in * r.n_out;
    const float nan = __uint_as_float(0x7FC00000u);
    for (int k = tid; k < cnt; k += nthreads) {
        const int o = k / n_in, i = k - o * n_in;
        float h, l;
        if (layer == 0) {
            h = (float)hi[LY::idx_first(0, o, i)];
            l = (float)hi[LY::idx_first(0, o, 4 + i)];
            for (int q = 0; q < LY::G; ++q) {          // every copy must agree
                if ((float)hi[LY::idx_first(q, o, i)] != h || (float)hi[LY::idx_first(q, o, 2 + i)] != h) h = nan;
                if ((float)hi[LY::idx_first(q, o, 4 + i)] != l) l = nan;
            }
        } else {
            const int at = layer == L - 1 ? LY::idx_out(o, i) : LY::idx_hidden(o, i);
            const bool two = LY::TAIL == kTailTwo && LY::in_tail(i), full = LY::TAIL == kTailFull && LY::in_tail(i);
            h = (float)hi[at];
            l = el.off_lo ? (float)(two ? hi[at + 4] : lo[at]) : 0.0f;
            if ((two && (float)hi[at + 2] != h) || (full && (float)hi[at + 4] != h)) h = nan;
            if (full && el.off_lo && (float)lo[at + 4] != l) l = nan;
        }
        hi_out[k] = h;
        lo_out[k] = l;
    }
    if (bias_out)
        for (int o = tid; o < r.n_out; o += nthreads) bias_out[o] = bt[layer == L - 1 ? LY::idx_bias_row(4 * o) : LY::idx_bias(o)];
    if (scale_out && tid == 0) *scale_out = el.scale;
}

}  // namespace rinr
