// Backward products of small and middling layers, formed directly from the operands where they lie.
//
// The limb products of cdl_qgemm.hip need the largest |g|, transposed copies of the index operands and a plan before
// their first multiplication: seven launches and 30 to 60 us for a layer whose products are a microsecond or two of arithmetic.
// Here both products run in one launch.  One wave forms 16 x 64 outputs (or 16 x 16, 64 x 16 where there are few columns): per 16
// contraction entries a lane loads four entries of one row of the fp32 operand and, for each of them, four neighbouring
// index bytes of the other; the order of the entries inside a step is the same on both sides and otherwise free.  The waves of
// a block split the contraction and add their tiles through LDS in a fixed order.
//   The smallest: in double (v_mfma_f64_16x16x4_f64, 69 TFLOP/s measured).  A product of a float and a level index is exact in
// double, and a sum of n of them is off by at most n 2^-53 of the sum of their magnitudes, far below the rounding of the fp32 result.
//   The others: on six int8 digits of every entry, scaled by row (digit_tile).
#include "cdl_internal.h"
#include "cdl_finish.h"
#include "cdl_bwd_plan.h"
#include "cdl_div.h"
#include "cdl_limbs.h"

#include <cmath>
#include <type_traits>

namespace cdl {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef uint32_t u32_any __attribute__((aligned(1)));

constexpr int kDirThreads = 512, kDirWaves = 8;

// A convolution's part of a product.
//   windows (weight gradient): contraction entry m is output pixel (b, p, q), column k entry (tap row, tap column, channel) of
//     its window, read from x [B][H][W][C]; outside the image the stored byte of level index 0
//   gathered (activation gradient): output row m is pixel (b, i, j) of a grid of gh x gw pixels per image, contraction entry
//     k = (tap (r, s) of .. x st, output channel n of gn) is g[b, i + ph - r, j + pw - s, n] where that lies inside; grid pixel
//     (b, i, j) is input pixel (b, step i + oa, step j + oc), its tap (r, s) tap (r0 + step r, s0 + step s) of the kernel (one
//     grid for stride 1, one per parity class of the input pixels for stride 2)
struct ConvPart {
    int H, W, C, S, stride, pad, P, Q, pad_byte;
    DivBy by_pq, by_q;
    int end_w, end_h, next_w, next_h, next_b;      // Q and P strides; from a window to the next: in a row, over its end, over an image's
    int gh, gw, gn, st, ph, pw, step, oa, oc, r0, s0;
    DivBy by_ghw, by_gw, by_gn, by_st;
    int taps_c;            // entries of one output channel's kernel: R S C
};

// One product: `rows` x `cols` outputs over `kc` contraction entries.
struct DirectProduct {
    const float *g;        // fp32 operand
    const int8_t *idx;     // index operand
    int rows, cols, kc;
    int64_t ldg, ldi;      // row lengths of g and idx as matrices
    int offset;            // added to every stored index
    int vec;               // four neighbouring entries of g in one 16-byte load
    int ksp;               // waves that split a contraction piece (1, 2, 4 or 8)
    int narrow;            // tiles of 16 x 16 outputs per wave instead of 16 x 64
    int tiles_r, tiles_c, splits, steps, steps_per_split;      // steps: of 64 contraction entries, narrow and thin tiles: 16
    int rounds_to;         // on digits: biased exponent up to which a row's scale may round entries far below it (-1: never)
    double delta;
    float *out;            // [rows][cols]
    double *partial;       // [splits][rows][cols], unscaled, when splits > 1
};

// ---- where the operands of one lane come from.  load: contraction entries e0 + 4 (lane / 16) .. + 3, as they lie in memory (what is
// done to them waits until they are multiplied, so that the loads of the next step stay in flight); WHOLE: e0 .. e0 + 15 all
// exist.  e0 is the same for the wave, so a whole load takes a base in scalar registers and a lane offset that stays. ----
// (ends a branch that must keep its loads: alike in both branches, they would be moved behind them, with addresses in vector registers)
#define KEEP_APART(TEXT) asm volatile("; " TEXT)

template <class T>
__device__ __forceinline__ T load_at(const void *base, uint32_t offset) { return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + offset); }

// the index bytes of four columns of a row-major index matrix, in as many rows as the step has entries
struct IndexColumns {
    int at, q4, sh;        // column; sh: the last columns of a matrix whose width is no multiple of four: a word that ends with the row, shifted
    uint32_t off[4];
    template <int TN>
    __device__ __forceinline__ void init_index(const DirectProduct &p, int col0, int lane)
    {
        // TN = 1: one column per lane, a byte
        const int c = col0 + TN * (lane & 15);
        at = min(c, p.cols - TN);      // (host: cols >= 4)
        sh = 8 * min(c - at, 3);
        q4 = 4 * (lane >> 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) off[j] = (uint32_t)(q4 + j) * (uint32_t)p.ldi + (uint32_t)at;      // (ldi < 2^26)
    }
    template <int TN, bool WHOLE>
    __device__ __forceinline__ void load_index(const DirectProduct &p, int e0, uint32_t (&b)[4]) const
    {
        const int8_t *whole = p.idx + (int64_t)e0 * p.ldi;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int8_t *base = WHOLE ? whole : p.idx + (int64_t)min(e0 + q4 + j, p.kc - 1) * p.ldi;
            const uint32_t o = WHOLE ? off[j] : (uint32_t)at;
            if (TN == 4) b[j] = load_at<u32_any>(base, o);
            else b[j] = load_at<uint8_t>(base, o);
        }
    }
};

// rows of g: dL/dQ(a)[m][k] = sum_n g[m][n] b[n][k]
struct RowsOfG : IndexColumns {
    static constexpr int kMask = 0, kAhead = 2;
    int row0;
    uint32_t goff[4];
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int first_row, int col0, int lane)
    {
        row0 = min(first_row, p.rows - 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) goff[i] = (uint32_t)min(16 * i + (lane & 15), p.rows - 1 - row0) * (uint32_t)p.ldg * 4u;      // (64 ldg < 2^30)
        init_index<TN>(p, col0, lane);
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e0, float (&a)[TM][4], uint32_t (&b)[4], int &) const
    {
        const float *base = p.g + (int64_t)row0 * p.ldg + (WHOLE ? e0 : 0);
        const int e = WHOLE ? q4 : e0 + q4;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (p.vec) {
                const float4 v = load_at<float4>(base, goff[i] + 4u * (uint32_t)(WHOLE ? e : min(e, p.kc - 4)));
                a[i][0] = v.x; a[i][1] = v.y; a[i][2] = v.z; a[i][3] = v.w;
                KEEP_APART("one load");
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) a[i][j] = load_at<float>(base, goff[i] + 4u * (uint32_t)(WHOLE ? e + j : min(e + j, p.kc - 1)));
            }
        }
        load_index<TN, WHOLE>(p, e0, b);
    }
};

// columns of g: dL/dQ(b)[n][k] = sum_m g[m][n] a[m][k]
struct ColumnsOfG {
    int gat[4], gq4;
    uint32_t goff[4][4];
    template <int TM>
    __device__ __forceinline__ void init_g(const DirectProduct &p, int row0, int lane)
    {
        gq4 = 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            gat[i] = min(row0 + 16 * i + (lane & 15), p.rows - 1);
#pragma unroll
            for (int j = 0; j < 4; ++j) goff[i][j] = ((uint32_t)(gq4 + j) * (uint32_t)p.ldg + (uint32_t)gat[i]) * 4u;      // (16 ldg < 2^30)
        }
    }
    template <int TM, bool WHOLE>
    __device__ __forceinline__ void load_g(const DirectProduct &p, int e0, float (&a)[TM][4]) const
    {
        const float *whole = p.g + (int64_t)e0 * p.ldg;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float *base = WHOLE ? whole : p.g + (int64_t)min(e0 + gq4 + j, p.kc - 1) * p.ldg;
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i][j] = load_at<float>(base, WHOLE ? goff[i][j] : (uint32_t)gat[i] * 4u);
        }
    }
};

struct ColumnsOfGMatrix : ColumnsOfG, IndexColumns {
    static constexpr int kMask = 0, kAhead = 2;
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int row0, int col0, int lane)
    {
        init_g<TM>(p, row0, lane);
        init_index<TN>(p, col0, lane);
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e0, float (&a)[TM][4], uint32_t (&b)[4], int &) const
    {
        load_g<TM, WHOLE>(p, e0, a);
        load_index<TN, WHOLE>(p, e0, b);
    }
};

// columns of g against the windows of a convolution.  kMask = 1: bit j of `ok` says whether entry j lies inside the image.
// A lane's four output pixels follow each other: the first one is found by division, the others by steps.
struct ColumnsOfGWindows : ColumnsOfG {
    static constexpr int kMask = 1, kAhead = 2;
    const ConvPart *cv;
    int tr, ts, chan, sh;      // the column's tap, less the padding, and channel
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int row0, int col0, int lane)
    {
        init_g<TM>(p, row0, lane);
        const int c = min(col0 + TN * (lane & 15), p.cols - TN), t = c / cv->C;      // (cols a multiple of 16, a word inside one tap)
        tr = t / cv->S - cv->pad;
        ts = t - t / cv->S * cv->S - cv->pad;
        chan = c - t * cv->C;
        sh = 0;
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e0, float (&a)[TM][4], uint32_t (&b)[4], int &ok) const
    {
        load_g<TM, WHOLE>(p, e0, a);
        ok = 0;
        int h = 0, w = 0, at = 0;
        auto place = [&](int m) {
            const int bb = div_by(m, cv->by_pq), rem = m - bb * (cv->P * cv->Q), pp = div_by(rem, cv->by_q);
            h = pp * cv->stride + tr;
            w = (rem - pp * cv->Q) * cv->stride + ts;
            at = ((bb * cv->H + h) * cv->W + w) * cv->C + chan;      // (fewer than 2^31 entries where these products serve)
        };
        place(WHOLE ? e0 + gq4 : min(e0 + gq4, p.kc - 1));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!WHOLE && j > 0) place(min(e0 + gq4 + j, p.kc - 1));
            const bool in = (unsigned)h < (unsigned)cv->H && (unsigned)w < (unsigned)cv->W;
            ok |= in ? 1 << j : 0;
            const uint32_t o = in ? (uint32_t)at : 0u;
            if (TN == 4) b[j] = load_at<uint32_t>(p.idx, o);
            else b[j] = load_at<uint8_t>(p.idx, o);
            if (WHOLE && j < 3) {
                w += cv->stride;
                at += cv->next_w;
                const bool row_end = w == cv->end_w + ts;
                w = row_end ? ts : w;
                h += row_end ? cv->stride : 0;
                at += row_end ? cv->next_h : 0;
                const bool image_end = h == cv->end_h + tr;
                h = image_end ? tr : h;
                at += image_end ? cv->next_b : 0;
            }
        }
        asm volatile("" : "+v"(ok));      // (four bits of a register, not four masks in scalar ones)
    }
};

// g gathered tap by tap against the kernels as they lie.  kMask = 2: bit i of `ok` says whether row i's pixel is there.
struct GatheredG {
    static constexpr int kMask = 2, kAhead = 2;
    const ConvPart *cv;
    const int8_t *col;
    int gi[4], gj[4], base[4], sh, q4;
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int row0, int col0, int lane)
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = min(row0 + 16 * i + (lane & 15), p.rows - 1);
            const int bb = div_by(m, cv->by_ghw), rem = m - bb * (cv->gh * cv->gw);
            gi[i] = div_by(rem, cv->by_gw);
            gj[i] = rem - gi[i] * cv->gw;
            base[i] = bb * cv->P * cv->Q;
        }
        col = p.idx + min(col0 + TN * (lane & 15), p.cols - TN);       // (cols a multiple of 4)
        sh = 0;
        q4 = 4 * (lane >> 4);
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e0, float (&a)[TM][4], uint32_t (&b)[4], int &ok) const
    {
        const int k = WHOLE ? e0 + q4 : min(e0 + q4, p.kc - 4);                     // (gn a multiple of 4: four entries share a tap)
        const int t = div_by(k, cv->by_gn), n = k - t * cv->gn, r = div_by(t, cv->by_st), s = t - r * cv->st;
        const int dh = cv->ph - r, dw = cv->pw - s;
        ok = 0;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int h = gi[i] + dh, w = gj[i] + dw;
            const bool in = (unsigned)h < (unsigned)cv->P && (unsigned)w < (unsigned)cv->Q;
            ok |= in ? 1 << i : 0;
            const float4 v = *reinterpret_cast<const float4 *>(p.g + (in ? (int64_t)(base[i] + h * cv->Q + w) * cv->gn + n : 0));
            a[i][0] = v.x; a[i][1] = v.y; a[i][2] = v.z; a[i][3] = v.w;
        }
        const int8_t *at = col + (int64_t)n * cv->taps_c + ((cv->r0 + cv->step * r) * cv->S + cv->s0 + cv->step * s) * cv->C;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (TN == 4) b[j] = *reinterpret_cast<const uint32_t *>(at + (int64_t)j * cv->taps_c);
            else b[j] = *reinterpret_cast<const uint8_t *>(at + (int64_t)j * cv->taps_c);
        }
    }
};

// four neighbouring outputs of a row
__device__ __forceinline__ void store_outputs(const DirectProduct &p, int64_t row, int col, const double (&v)[4])
{
    float *o = p.out + row * p.cols + col;
    if ((p.cols & 3) == 0) {
        if (col < p.cols) *reinterpret_cast<float4 *>(o) = make_float4((float)(v[0] * p.delta), (float)(v[1] * p.delta), (float)(v[2] * p.delta), (float)(v[3] * p.delta));
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (col + c < p.cols) o[c] = (float)(v[c] * p.delta);
    }
}

// The products of a tile over steps [s0, s1) of 16 contraction entries, wave ks of p.ksp, into the wave's part of LDS
// (`mine`), or to memory where there is nothing to add (null).
// TM x TN: 16 x 16 MFMA tiles; TN = 4: the tiles' columns are the four bytes of a word, 64 columns in all.
template <int TM, int TN, class Src, class RowMap>
__device__ __forceinline__ void direct_tile(const DirectProduct &p, Src &src, int row0, int col0, int s0, int s1, int ks, double *mine, RowMap out_row,
                                            uint32_t pad_word = 0u)
{
    const int lane = threadIdx.x & 63, q4 = (lane >> 4) * 4;
    src.template init<TM, TN>(p, row0, col0, lane);
    v4d acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][t][r] = 0.0;
    // kAhead steps are in flight: a step is 256 TM TN cycles of one SIMD's matrix pipe, a load from memory one to four thousand
    constexpr int kAhead = TM * TN >= 4 ? 2 : 4;
    float a[kAhead][TM][4];
    uint32_t b[kAhead][4];
    int ok[kAhead];
    auto load = [&](int u, int s) {
        if (16 * s + 16 <= p.kc) {
            src.template load<TM, TN, true>(p, 16 * s, a[u], b[u], ok[u]);
            KEEP_APART("whole step");
        } else src.template load<TM, TN, false>(p, 16 * s, a[u], b[u], ok[u]);
    };
    auto multiply = [&](int u, int s) {
        const int e = 16 * s + q4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double av[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const float v = e + j < p.kc && (Src::kMask != 2 || (ok[u] >> i & 1)) ? a[u][i][j] : 0.0f;
                av[i] = (double)v;
            }
            const uint32_t w = Src::kMask == 1 && !(ok[u] >> j & 1) ? pad_word : b[u][j] >> src.sh;
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const int x = (int)(w << (24 - 8 * t)) >> 24;
                const double bv = (double)(x + p.offset);
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv, acc[i][t], 0, 0, 0);
            }
        }
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (s0 + ks + u * p.ksp < s1) load(u, s0 + ks + u * p.ksp);
    for (int s = s0 + ks; s < s1; s += kAhead * p.ksp) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int su = s + u * p.ksp, next = su + kAhead * p.ksp;
            if (su < s1) multiply(u, su);
            if (next < s1) load(u, next);
        }
    }
    // register r of a tile: row lane / 16 + 4 r, column lane % 16 (of 16), i.e. TN (lane % 16) + t of 16 TN
    if (!mine) {
        // the tile is complete in this wave's registers: straight to memory, 256 bytes of a row per 16 lanes
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = row0 + 16 * i + (lane >> 4) + 4 * r, col = col0 + (lane & 15) * TN;
                if (row >= p.rows) continue;
                float v[TN];
#pragma unroll
                for (int t = 0; t < TN; ++t) v[t] = (float)(acc[i][t][r] * p.delta);
                float *o = p.out + out_row(row) * p.cols + col;
                if (TN == 4 && (p.cols & 3) == 0) {
                    if (col < p.cols) *reinterpret_cast<float4 *>(o) = make_float4(v[0], v[1 % TN], v[2 % TN], v[3 % TN]);
                } else {
#pragma unroll
                    for (int t = 0; t < TN; ++t)
                        if (col + t < p.cols) o[t] = v[t];
                }
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double *d = mine + (16 * i + (lane >> 4) + 4 * r) * (16 * TN) + (lane & 15) * TN;
#pragma unroll
            for (int t = 0; t < TN; ++t) d[t] = acc[i][t][r];
        }
}

// the largest of three; a NaN if there is one
__device__ __forceinline__ float largest(float a, float b, float c)
{
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

__device__ __forceinline__ float smallest(float a, float b, float c)
{
    return __builtin_elementwise_minimum(__builtin_elementwise_minimum(a, b), c);
}

__device__ __forceinline__ unsigned int max_over_groups(unsigned int v)      // over lanes that agree mod 16
{
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const unsigned int m = max(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return max(b[0], b[1]);
}

// The products of a 16 x 64 tile as direct_tile forms them, on the int8 matrix cores: steps of 64 contraction entries, the
// lane's 16 entries of a row of g as six balanced base-256 digits of g 2^s, s from the largest exponent in the row.
//
// What is exact.  A row's scale leaves the entry that set it at 2^43 .. 2^44 and holds entries up to 2^46, so digits give an entry within 2^-20 of the
// row's largest in full (24 bits of mantissa) and smaller ones to 2^-44 of it; digit sums are exact in int32 and are added up in
// double.  What they leave of the smaller ones is multiplied in double, the 4 contraction entries of an instruction at a time
// where there is something left: with entries N(0, 1) one step in 600 has such an entry, so that every product is exact, as it is in
// double, at 0.2 - 0.6 us of 9 - 20.  A step with many of them is formed in double as a whole, as one with an infinity or a NaN, which shows in
// the same outputs as before (256 x 1000 x 512  N(0, 1) 12.4 us; times e^2N 18; spread over 2^60 28, in double 29).  Beyond the sizes where double is
// the alternative what is left is left out where that is harmless (rounds_to).  A row whose entries grow beyond its scale has its sums
// moved to double and gets a new scale.
//
// Why.  In double a step of 64 entries is 64 matrix instructions of 64 cycles; here 24 of 16 and about 245 others, of which 104
// make the digits.  What bounds it is that wave's chain of instructions, two waves to a SIMD: 1 us a step, of 4 us + 2 us a step for a
// block (load 1.5, the last sums and their addition over waves 2.5).  Both products, in double / so: 256 x 1000 x 512  29 / 12 us,
// 512 x 512 x 256  20 / 10, 700 x 700 x 700 (limbs before)  48 / 21, dL/dQ(w) of 16 images of 28 x 28 x 64 -> 64, 3 x 3  32 / 18.
// (Tiles of 16 columns would need as long for the digits as double takes in all: those stay with direct_tile.)
// SHORT: the contraction may have fewer than 64 entries (whose loads, one by one with their bounds, would cost the others registers).
constexpr int kDigits = 6, kDigitStep = 64;

struct Diag { float amax; int colabs[4]; };      // of a lane: largest |g|, sums of |index| of its columns

template <bool DIAG, bool SHORT, class Src, class RowMap>
__device__ __forceinline__ void digit_tile(const DirectProduct &p, Src &src, int row0, int col0, int s0, int s1, int ks, double *mine, bool alone, Diag &dg,
                                           RowMap out_row, uint32_t pad_word = 0u)
{
    const int lane = threadIdx.x & 63, q = lane >> 4;
    src.template init<1, 4>(p, row0, col0, lane);
    const bool shifted = (p.cols & 3) != 0;
    v4i acc[kDigits][4];
    int row_sum[kDigits];
#pragma unroll
    for (int l = 0; l < kDigits; ++l) {
        row_sum[l] = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[l][t] = v4i{0, 0, 0, 0};
    }
    int cap = -1;              // biased exponent that the row's scale holds: s = 172 - cap
    int since = 0;             // steps in acc
    bool folded = false;       // `mine` holds sums

    // Value of tile element (row 4 q + r, column 4 (lane % 16) + t) in acc.  In LDS it lies at (4 t + r) 64 + lane.
    double unit[4], offset_part[4];
    auto scales = [&]() {
        double sum = 0.0;
        if (p.offset) {
            sum = (double)row_sum[kDigits - 1];
#pragma unroll
            for (int l = kDigits - 2; l >= 0; --l) sum = __builtin_fma(sum, 256.0, (double)row_sum[l]);
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            sum *= (double)p.offset;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            unit[r] = __hiloint2double((1023 - 172 + __shfl(cap, 4 * q + r, 64)) << 20, 0);      // 2^-s
            offset_part[r] = p.offset ? __shfl(sum, 4 * q + r, 64) : 0.0;
        }
    };
    // (a sum of at most seven steps and 256 times another fit an int32: two limbs at a time)
    auto value = [&](int t, int r, bool few) {
        double run;
        if (few) {
            run = (double)(256 * acc[5][t][r] + acc[4][t][r]);
            run = __builtin_fma(run, 65536.0, (double)(256 * acc[3][t][r] + acc[2][t][r]));
            run = __builtin_fma(run, 65536.0, (double)(256 * acc[1][t][r] + acc[0][t][r]));
        } else {
            run = (double)acc[kDigits - 1][t][r];
#pragma unroll
            for (int l = kDigits - 2; l >= 0; --l) run = __builtin_fma(run, 256.0, (double)acc[l][t][r]);
        }
        return (run + offset_part[r]) * unit[r];
    };
    auto fold = [&]() {
        scales();
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double *m = mine + (4 * t + r) * 64 + lane;
                const double v = value(t, r, false);
                *m = folded ? *m + v : v;
            }
#pragma unroll
        for (int l = 0; l < kDigits; ++l) {
            row_sum[l] = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[l][t] = v4i{0, 0, 0, 0};
        }
        folded = true;
        since = 0;
    };

    constexpr int kAhead = Src::kAhead;
    float a[kAhead][4][1][4];
    uint32_t b[kAhead][4][4];
    int ok[kAhead][4];
    // A step's entries: the last one of a contraction that is no multiple of 64 starts earlier, where 64 are there, and leaves out
    // (as zeros) what the step before it has.  Quarter u: entries 16 u + 4 q .. + 3 of it.
    auto start = [&](int s) { return max(min(kDigitStep * s, p.kc - kDigitStep), 0); };
    auto quarter_empty = [&](int s, int u) { return start(s) + 16 * u + 16 <= kDigitStep * s || start(s) + 16 * u >= p.kc; };
    auto load = [&](int buf, int s) {
        const int e0 = start(s);
        if (!SHORT || p.kc >= kDigitStep) {
#pragma unroll
            for (int u = 0; u < 4; ++u) src.template load<1, 4, true>(p, e0 + 16 * u, a[buf][u], b[buf][u], ok[buf][u]);
            KEEP_APART("whole step");
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (16 * u < p.kc) src.template load<1, 4, false>(p, 16 * u, a[buf][u], b[buf][u], ok[buf][u]);
        }
    };
    auto step = [&](int buf, int s) {
        const int e0 = start(s);
        const bool whole = kDigitStep * s + kDigitStep <= p.kc;
        float (&g)[4][1][4] = a[buf];
        if (!whole) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int e = e0 + 16 * u + 4 * q + j;
                    g[u][0][j] = e >= kDigitStep * s && e < p.kc ? g[u][0][j] : 0.0f;
                }
        }
        // smallest magnitude (of what lies inside the image), largest, a NaN stays one, and the biased exponent of the row's largest
        float m = 0.0f, least = INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float two = __builtin_elementwise_minimum(fabsf(g[u][0][0]), fabsf(g[u][0][1]));
            const float four = smallest(two, fabsf(g[u][0][2]), fabsf(g[u][0][3]));
            least = __builtin_elementwise_minimum(least, Src::kMask == 2 && !(ok[buf][u] & 1) ? INFINITY : four);
        }
        if (Src::kMask == 2) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) g[u][0][j] = (ok[buf][u] & 1) ? g[u][0][j] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            m = largest(m, fabsf(g[u][0][0]), fabsf(g[u][0][1]));
            m = largest(m, fabsf(g[u][0][2]), fabsf(g[u][0][3]));
        }
        if (DIAG) dg.amax = fmaxf(dg.amax, m);
        const int E = (int)(max_over_groups(__float_as_uint(m)) >> 23);
        const uint32_t sh = shifted ? src.sh : 0;
        auto word = [&](int u, int j) {
            return Src::kMask == 1 && !(ok[buf][u] >> j & 1) ? pad_word : b[buf][u][j] >> sh;
        };
        // what the row's scale holds with this step, and the exponent from which on its unit divides an entry (0: rounding is allowed)
        const int to = E > cap ? min(E + 2, 254) : cap, whole_from = to <= p.rounds_to ? 0 : max(to - 22, 0);
        if (__ballot(E > cap || !(least >= __int_as_float(whole_from << 23))) != 0 || since == 1024) {      // (an int32 holds 2048 steps of 64 products of 128 and 128)
            // bits without the sign, one less, so that zeros are the largest
            auto ordered = [&](int k) { return 2u * __float_as_uint(g[k >> 2][0][k & 3]) - 1u; };
            const uint32_t limit = whole_from > 0 ? ((uint32_t)whole_from << 24) - 1u : 0u;
            uint32_t small = ~0u;
#pragma unroll
            for (int k = 0; k < 16; ++k) small = min(small, ordered(k));
            // the contraction entries (quarter u, place j: bit 4 u + j) where the digits would round one
            uint32_t groups = 0u;
            if (__ballot(small < limit) != 0)
#pragma unroll
                for (int k = 0; k < 16; ++k) groups |= __ballot(ordered(k) < limit) != 0 ? 1u << k : 0u;
            // Where most are, or with an infinity or a NaN, the step is formed in double without digits; otherwise what the digits leave is.
            const bool all = __ballot(E == 255) != 0 || __popc(groups) > 12;
            if (all) groups = 0xffffu;
            if (since == 1024 || (since > 0 && !all && __ballot(E > cap) != 0)) fold();
            if (!all) cap = to;
            if (groups && !folded) {
#pragma unroll
                for (int i = 0; i < 16; ++i) mine[i * 64 + lane] = 0.0;
                folded = true;
            }
            if (groups) {
                const double unit_of = __hiloint2double((1023 - 172 + cap) << 20, 0), per_unit = __hiloint2double((1023 + 172 - cap) << 20, 0);
#pragma unroll 1
                for (int t0 = 0; t0 < 4; t0 += 2) {      // (two columns of a word at a time: registers)
                    v4d sum[2] = {v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}};
#pragma unroll 1
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if (!(groups >> (4 * u + j) & 1)) continue;
                            double v = (double)(u == 0 ? g[0][0][j] : u == 1 ? g[1][0][j] : u == 2 ? g[2][0][j] : g[3][0][j]);
                            if (!all) {
                                v *= per_unit;
                                v = (v - __builtin_rint(v)) * unit_of;
                            }
                            const uint32_t w = (u == 0 ? word(0, j) : u == 1 ? word(1, j) : u == 2 ? word(2, j) : word(3, j)) >> (8 * t0);
#pragma unroll
                            for (int t = 0; t < 2; ++t)
                                sum[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, (double)(((int)(w << (24 - 8 * t)) >> 24) + p.offset), sum[t], 0, 0, 0);
                        }
                    // (element (row q + 4 r, ...) of that tile)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) mine[(4 * (t0 + t) + q) * 64 + 16 * r + (lane & 15)] += sum[t][r];
                }
            }
            if (all) {
                if (!DIAG) return;
#pragma unroll
                for (int k = 0; k < 16; ++k) g[k >> 2][0][k & 3] = 0.0f;      // (on for the sums of |index|)
            }
        }
        const double scale = __hiloint2double((1023 + 172 - cap) << 20, 0);
        v4i fa[kDigits], fb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!whole && quarter_empty(s, u)) {
#pragma unroll
                for (int l = 0; l < kDigits; ++l) fa[l][u] = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) fb[t][u] = 0;
                continue;
            }
            uint32_t d[kDigits], w[4], c[4];
            limbs_of4_wide<kDigits>(g[u][0], scale, d);
#pragma unroll
            for (int l = 0; l < kDigits; ++l) fa[l][u] = (int)d[l];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = word(u, j);
            transpose4(w, c);
#pragma unroll
            for (int t = 0; t < 4; ++t) fb[t][u] = (int)c[t];
        }
        if (p.offset) {
#pragma unroll
            for (int l = 0; l < kDigits; ++l)
#pragma unroll
                for (int u = 0; u < 4; ++u) row_sum[l] = __builtin_amdgcn_sdot4(fa[l][u], 0x01010101, row_sum[l], false);
        }
        if (DIAG) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                uint32_t there = ~0u;
                if (!whole) {
                    there = 0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int e = e0 + 16 * u + 4 * q + j;
                        there |= e >= kDigitStep * s && e < p.kc ? 0xffu << (8 * j) : 0u;
                    }
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    dg.colabs[t] = (int)__builtin_amdgcn_sad_u8(((uint32_t)fb[t][u] & there) ^ 0x80808080u, 0x80808080u, (unsigned int)dg.colabs[t]);
            }
        }
#pragma unroll
        for (int l = 0; l < kDigits; ++l)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[l][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[l], fb[t], acc[l][t], 0, 0, 0);
        ++since;
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (s0 + ks + u * p.ksp < s1) load(u, s0 + ks + u * p.ksp);
    for (int s = s0 + ks; s < s1; s += kAhead * p.ksp) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int su = s + u * p.ksp, next = su + kAhead * p.ksp;
            if (su < s1) step(u, su);
            if (next < s1) load(u, next);
        }
    }
    scales();
    auto finish = [&](bool few) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[t] = value(t, r, few);
                if (folded) v[t] += mine[(4 * t + r) * 64 + lane];
            }
            if (alone) {
                const int row = row0 + 4 * q + r;
                if (row < p.rows) store_outputs(p, out_row(row), col0 + 4 * (lane & 15), v);
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) mine[(4 * t + r) * 64 + lane] = v[t];
            }
        }
    };
    if (since <= 7) finish(true);
    else finish(false);
}

// The sums of the waves that share a digit_tile; after a barrier.
template <class RowMap>
__device__ __forceinline__ void digit_store(const DirectProduct &p, const double *lds, int row0, int col0, int split, RowMap out_row)
{
    const int wave = threadIdx.x >> 6, grp = wave / p.ksp;
    const double *base = lds + (size_t)grp * p.ksp * 1024;
    for (int i = (int)threadIdx.x - grp * p.ksp * 64; i < 256; i += 64 * p.ksp) {
        const int r = i >> 6, l = i & 63;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int w = 0; w < p.ksp; ++w)
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] += base[w * 1024 + (4 * t + r) * 64 + l];
        const int row = row0 + 4 * (l >> 4) + r, col = col0 + 4 * (l & 15);
        if (row >= p.rows) continue;
        if (p.splits > 1) {
            double *o = p.partial + ((int64_t)split * p.rows + row) * p.cols + col;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < p.cols) o[c] = v[c];
        } else {
            store_outputs(p, out_row(row), col, v);
        }
    }
}

// Adds the waves' tiles and writes the outputs; after a barrier.  row0: of the wave group's tile.
template <int TM, int TN, class RowMap>
__device__ __forceinline__ void direct_store(const DirectProduct &p, const double *lds, int row0, int col0, int split, RowMap out_row)
{
    const int wave = threadIdx.x >> 6, grp = wave / p.ksp, t0 = (int)threadIdx.x - grp * p.ksp * 64;
    constexpr int kTile = 256 * TM * TN;
    const double *base = lds + (size_t)grp * p.ksp * kTile;
    for (int quad = t0; quad < kTile / 4; quad += 64 * p.ksp) {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int w = 0; w < p.ksp; ++w)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] += base[w * kTile + 4 * quad + c];
        const int row = row0 + 4 * quad / (16 * TN), col = col0 + 4 * quad % (16 * TN);
        if (row >= p.rows) continue;
        if (p.splits > 1) {
            double *o = p.partial + ((int64_t)split * p.rows + row) * p.cols + col;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < p.cols) o[c] = v[c];
        } else {
            store_outputs(p, out_row(row), col, v);
        }
    }
}

struct DirectArgs {
    DirectProduct p[2];            // dL/dQ(a), dL/dQ(b) or the other way round
    int first;                     // blocks of p[0]
    int a_at;                      // which of them is dL/dQ(a)
    BwdPlan *plan;                 // for the diagnostic words
    // DIAG: the limb rule's inputs
    unsigned long long *records;   // [gridDim.x][2]
    unsigned long long tag;
    float delta_a, delta_b;
    int *column_sums;              // [splits][cols] of dL/dQ(b), where that is cut into pieces: direct_reduce_kernel finishes then; else null
    const unsigned int *col_abs_b; // the largest sum of |index| of dL/dQ(a), where that was formed before; else null
};

struct DirectItem {
    int split, row0, col0, s0, s1;
    __device__ __forceinline__ DirectItem(const DirectProduct &p, int item, int wave)
    {
        const int tc = item % p.tiles_c;
        item /= p.tiles_c;
        const int tr = item % p.tiles_r;
        split = item / p.tiles_r;
        row0 = (tr * (kDirWaves / p.ksp) + wave / p.ksp) * 16;
        col0 = tc * (p.narrow ? 16 : 64);
        s0 = split * p.steps_per_split;
        s1 = min(s0 + p.steps_per_split, p.steps);
    }
};

// Small products, in double (plan_double).  The diagnostic words say that there are no limbs.
__global__ __launch_bounds__(kDirThreads)
void bwd_double_kernel(DirectArgs a)
{
    __shared__ double lds[kDirWaves * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), which = (int)blockIdx.x >= a.first;
    const DirectProduct &p = a.p[which];
    const DirectItem it(p, (int)blockIdx.x - (which ? a.first : 0), wave);
    if (blockIdx.x == 0 && threadIdx.x == 0) no_limbs(a.plan);
    auto product = [&](auto &&src, auto tn_c) {
        constexpr int TN = decltype(tn_c)::value;
        const auto same = [](int row) { return (int64_t)row; };
        const bool alone = p.ksp == 1 && p.splits == 1;
        direct_tile<1, TN>(p, src, it.row0, it.col0, it.s0, it.s1, wave % p.ksp, alone ? nullptr : lds + wave * 256 * TN, same);
        if (alone) return;
        __syncthreads();
        direct_store<1, TN>(p, lds, it.row0, it.col0, it.split, same);
    };
    constexpr auto wide = std::integral_constant<int, 4>{};
    constexpr auto thin = std::integral_constant<int, 1>{};
    if (which == a.a_at) { if (p.narrow) product(RowsOfG{}, thin); else product(RowsOfG{}, wide); }
    else { if (p.narrow) product(ColumnsOfGMatrix{}, thin); else product(ColumnsOfGMatrix{}, wide); }
}

// The others, on digits (plan_digits).  DIAG: leaves in the workspace the limb counts and bounds that the limb products would have
// had (the documented diagnostic words): every block publishes the largest |g| and the largest column sum of |index| it has seen,
// the last block takes the maxima; where a contraction is cut into pieces the column sums of the pieces go to memory and the kernel
// that adds the pieces up takes them.  Otherwise: that there are none.
template <bool DIAG, bool SHORT>
__global__ __launch_bounds__(kDirThreads)
void bwd_direct_kernel(DirectArgs a)
{
    __shared__ double lds[kDirWaves * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), which = (int)blockIdx.x >= a.first;
    const DirectProduct &p = a.p[which];
    const DirectItem it(p, (int)blockIdx.x - (which ? a.first : 0), wave);
    Diag dg = {0.0f, {0, 0, 0, 0}};
    if (!DIAG && blockIdx.x == 0 && threadIdx.x == 0) no_limbs(a.plan);
    auto product = [&](auto &&src) {
        const auto same = [](int row) { return (int64_t)row; };
        const bool alone = p.ksp == 1 && p.splits == 1;
        digit_tile<DIAG, SHORT>(p, src, it.row0, it.col0, it.s0, it.s1, wave % p.ksp, lds + wave * 1024, alone, dg, same);
        if (alone) return;
        __syncthreads();
        digit_store(p, lds, it.row0, it.col0, it.split, same);
    };
    if (which == a.a_at) product(RowsOfG{});
    else product(ColumnsOfGMatrix{});

    if (DIAG) {
        // the waves of group 0 walk the whole contraction piece of the block's columns between them
        int *colabs = reinterpret_cast<int *>(lds);                                  // [kDirWaves][64]
        unsigned int *amax = reinterpret_cast<unsigned int *>(lds) + kDirWaves * 64, *red = amax + kDirWaves;      // [kDirWaves], [3][kDirWaves]
        const int lane = threadIdx.x & 63;
        auto wave_max = [](unsigned int v) {
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) v = max(v, (unsigned int)__shfl_xor((int)v, off, 64));
            return max_over_groups(v);
        };
        const unsigned int wave_amax = wave_max(__float_as_uint(dg.amax));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            dg.colabs[t] += __shfl_xor(dg.colabs[t], 16, 64);
            dg.colabs[t] += __shfl_xor(dg.colabs[t], 32, 64);
        }
        __syncthreads();
        if (lane == 0) amax[wave] = wave_amax;
        if (lane < 16)
#pragma unroll
            for (int t = 0; t < 4; ++t) colabs[wave * 64 + 4 * lane + t] = dg.colabs[t];
        __syncthreads();
        if (wave == 0) {
            int sum = 0;
            if (it.col0 + lane < p.cols)
                for (int w = 0; w < p.ksp; ++w) sum += colabs[w * 64 + lane];
            const bool piece = p.splits > 1;
            if (piece && it.row0 == 0 && it.col0 + lane < p.cols) a.column_sums[(int64_t)it.split * p.cols + it.col0 + lane] = sum;
            const unsigned int m = piece ? 0u : wave_max((unsigned int)sum), g = wave_max(lane < kDirWaves ? amax[lane] : 0u);
            if (lane == 0) {
                const unsigned long long v = ((unsigned long long)g << 32) | m;
                unsigned long long *r = a.records + 2 * (size_t)blockIdx.x;
                device_store(r, v);
                device_store(r + 1, v ^ a.tag);
            }
        }
        if (a.column_sums || blockIdx.x != gridDim.x - 1) return;
        unsigned int gm = 0u, sa = 0u, sb = 0u;
        for (int i = threadIdx.x; i < (int)gridDim.x; i += kDirThreads) {
            unsigned long long *r = a.records + 2 * (size_t)i;
            unsigned long long v, c;
            do {
                v = device_load(r);
                c = device_load(r + 1);
            } while ((v ^ c) != a.tag);
            device_store(r + 1, v);
            gm = max(gm, (unsigned int)(v >> 32));
            if ((i >= a.first) == (a.a_at != 0)) sb = max(sb, (unsigned int)v);
            else sa = max(sa, (unsigned int)v);
        }
        gm = wave_max(gm);
        sa = wave_max(sa);
        sb = wave_max(sb);
        if (lane == 0) { red[wave] = gm; red[kDirWaves + wave] = sa; red[2 * kDirWaves + wave] = sb; }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < kDirWaves; ++w) {
                gm = max(gm, red[w]);
                sa = max(sa, red[kDirWaves + w]);
                sb = max(sb, red[2 * kDirWaves + w]);
            }
            if (a.col_abs_b) sb = *a.col_abs_b;
            choose_limbs(a.plan, gm, sa, sb, a.delta_a, a.delta_b);
        }
    }
}

// The weight gradient of a convolution: a product over output pixels whose index operand is the windows.
template <bool DIGITS>
__global__ __launch_bounds__(kDirThreads)
void conv_dw_direct_kernel(DirectProduct p, ConvPart cv)
{
    __shared__ double lds[kDirWaves * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const DirectItem it(p, blockIdx.x, wave);
    const auto same = [](int row) { return (int64_t)row; };
    ColumnsOfGWindows src;
    src.cv = &cv;
    const uint32_t pad_word = (uint32_t)cv.pad_byte * 0x01010101u;
    if constexpr (DIGITS) {
        Diag dg;
        digit_tile<false, false>(p, src, it.row0, it.col0, it.s0, it.s1, wave % p.ksp, lds + wave * 1024, false, dg, same, pad_word);
        __syncthreads();
        digit_store(p, lds, it.row0, it.col0, it.split, same);
    } else if (p.narrow) {
        direct_tile<1, 1>(p, src, it.row0, it.col0, it.s0, it.s1, wave % p.ksp, lds + wave * 256, same, pad_word);
        __syncthreads();
        direct_store<1, 1>(p, lds, it.row0, it.col0, it.split, same);
    } else {
        direct_tile<1, 4>(p, src, it.row0, it.col0, it.s0, it.s1, wave % p.ksp, lds + wave * 1024, same, pad_word);
        __syncthreads();
        direct_store<1, 4>(p, lds, it.row0, it.col0, it.split, same);
    }
}

// ---- weight gradients over long contractions: the columns of a block share the digits ----
//
// A wave of digit_tile makes the digits of 16 columns of g for its 64 columns of the index operand, and each wave reads g again (131072 x 16 x 144: 80 MB
// fetched where the operands are 27).  Here a block goes through up to six tiles of 64 columns at once, in rounds of eight steps of 64
// contraction entries: every wave makes the digits of one step, scaled by the round's largest entry in a row, and multiplies the steps of its part of the round by its own
// 64 columns.  What is exact, and how, is as in digit_tile; the remainders of a step are multiplied by each wave for its columns, g read once more.
// What bounds it: the chain of a round - g, the exchange of the rows' largest exponents, the digits through LDS, a wave's steps one after the other - 4.5 us and 1.4 us for
// each tile beyond two (a block has one compute unit to itself).  dL/dQ(b) by digit_tile / so, with the kernel that adds up the pieces, us: 131072 x 16 x 144  21.9 / 15.7,
// 131072 x 32 x 144  38.9 / 23.2, 400000 x 24 x 263  158 / 72, 239609 x 29 x 199  88 / 39, 84130 x 21 x 1382  106 / 68.
// (With a convolution's windows as the operand slower: finding their pixels is on six of eight waves then, 128 x 32 x 32 x 16 -> 16 19.2 / 20.9.  All columns on one wave to
// a SIMD, without barriers: 288 registers of digit sums and 846 spilled.)
constexpr int kSharedTiles = 6;
__host__ __device__ constexpr int shared_parts(int tiles) { return tiles <= 2 ? 4 : tiles <= 4 ? 2 : 1; }      // waves to a tile; at most eight (two to a SIMD, the registers of the digit sums)
constexpr int kSharedSteps = 8;       // of a round: each of eight waves makes the digits of one

template <int TC>
__device__ __forceinline__ void shared_tiles(const DirectProduct &p, int row0, int col0, int s0, int s1, double *sums, int8_t *digits)
{
    ColumnsOfGMatrix src;
    constexpr int KS = shared_parts(TC), kMine = kSharedSteps / KS;      // kMine: steps of a round that a wave multiplies
    __shared__ int exponents[kSharedSteps][16];
    __shared__ unsigned int rest[kSharedSteps];      // groups of a step that have remainders; bit 16: the whole step in double
    const int lane = threadIdx.x & 63, q = lane >> 4, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave / TC, tc = wave - ks * TC;
    double *const mine = sums + wave * 1024;
    const bool multiplies = ks < KS;
    src.init<1, 4>(p, row0, col0 + 64 * tc, lane);
    const uint32_t sh = (p.cols & 3) != 0 ? src.sh : 0;
    v4i acc[kDigits][4];
    int row_sum[kDigits];
#pragma unroll
    for (int l = 0; l < kDigits; ++l) {
        row_sum[l] = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[l][t] = v4i{0, 0, 0, 0};
    }
    int cap = -1, since = 0;
    bool folded = false;
    double unit[4], offset_part[4];
    auto scales = [&]() {
        double sum = 0.0;
        if (p.offset) {
            sum = (double)row_sum[kDigits - 1];
#pragma unroll
            for (int l = kDigits - 2; l >= 0; --l) sum = __builtin_fma(sum, 256.0, (double)row_sum[l]);
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            sum *= (double)p.offset;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            unit[r] = __hiloint2double((1023 - 172 + __shfl(cap, 4 * q + r, 64)) << 20, 0);      // 2^-s
            offset_part[r] = p.offset ? __shfl(sum, 4 * q + r, 64) : 0.0;
        }
    };
    auto value = [&](int t, int r) {
        double run = (double)acc[kDigits - 1][t][r];
#pragma unroll
        for (int l = kDigits - 2; l >= 0; --l) run = __builtin_fma(run, 256.0, (double)acc[l][t][r]);
        return (run + offset_part[r]) * unit[r];
    };
    auto fold = [&]() {
        scales();
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double *m = mine + (4 * t + r) * 64 + lane;
                const double v = value(t, r);
                *m = folded ? *m + v : v;
            }
        folded = true;
    };

    auto start = [&](int s) { return max(min(kDigitStep * s, p.kc - kDigitStep), 0); };      // (host: kc >= kDigitStep)
    float g[4][1][4];
    uint32_t b[2][4][4];      // two of its steps under way
    auto load_gradient = [&](int s) {
#pragma unroll
        for (int u = 0; u < 4; ++u) src.load_g<1, true>(p, start(s) + 16 * u, g[u]);
    };
    auto load_columns = [&](int k, int s) {
#pragma unroll
        for (int u = 0; u < 4; ++u) src.load_index<4, true>(p, start(s) + 16 * u, b[k & 1][u]);
    };
    // what a step before it has, of the last one of a contraction that is no multiple of 64, left out
    auto mask = [&](int s) {
        if (kDigitStep * s + kDigitStep <= p.kc) return;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) g[u][0][j] = start(s) + 16 * u + 4 * q + j >= kDigitStep * s ? g[u][0][j] : 0.0f;
    };

    if (s0 + wave < s1) load_gradient(s0 + wave);
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (multiplies && s0 + ks + k * KS < s1) load_columns(k, s0 + ks + k * KS);
    for (int s = s0; s < s1; s += kSharedSteps) {
        const bool makes = s + wave < s1;
        float m = 0.0f;
        if (makes) {
            mask(s + wave);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                m = largest(m, fabsf(g[u][0][0]), fabsf(g[u][0][1]));
                m = largest(m, fabsf(g[u][0][2]), fabsf(g[u][0][3]));
            }
        }
        const int E = (int)(max_over_groups(__float_as_uint(m)) >> 23);
        if (lane < 16) exponents[wave][lane] = E < 255 ? E : 0;      // (a step with an infinity or a NaN has no digits)
        __syncthreads();
        int most = 0;
#pragma unroll
        for (int w = 0; w < kSharedSteps; ++w) most = max(most, exponents[w][lane & 15]);
        // (all waves alike)
        const bool grows = __ballot(most > cap) != 0;
        if (since > 0 && (grows || since + kSharedSteps > 1024)) {      // (an int32 holds 2048 steps of 64 products of 128 and 128)
            fold();
#pragma unroll
            for (int l = 0; l < kDigits; ++l) {
                row_sum[l] = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[l][t] = v4i{0, 0, 0, 0};
            }
            since = 0;
        }
        cap = most > cap ? min(most + 2, 254) : cap;
        if (makes) {
            // (see digit_tile)
            const int whole_from = cap <= p.rounds_to ? 0 : max(cap - 22, 0);
            auto ordered = [&](int k) { return 2u * __float_as_uint(g[k >> 2][0][k & 3]) - 1u; };
            const uint32_t limit = whole_from > 0 ? ((uint32_t)whole_from << 24) - 1u : 0u;
            uint32_t small = ~0u, groups = 0u;
#pragma unroll
            for (int k = 0; k < 16; ++k) small = min(small, ordered(k));
            if (__ballot(small < limit) != 0)
#pragma unroll
                for (int k = 0; k < 16; ++k) groups |= __ballot(ordered(k) < limit) != 0 ? 1u << k : 0u;
            const bool all = __ballot(E == 255) != 0 || __popc(groups) > 12;
            if (all) groups = 0x1ffffu;
            if (lane == 0) rest[wave] = groups;
            const double scale = __hiloint2double((1023 + 172 - cap) << 20, 0);
            v4i f[kDigits];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                uint32_t d[kDigits];
                limbs_of4_wide<kDigits>(g[u][0], scale, d);
#pragma unroll
                for (int l = 0; l < kDigits; ++l) f[l][u] = all ? 0 : (int)d[l];
            }
#pragma unroll
            for (int l = 0; l < kDigits; ++l) *reinterpret_cast<v4i *>(digits + ((wave * kDigits + l) * 64 + lane) * 16) = f[l];
        }
        if (s + kSharedSteps + wave < s1) load_gradient(s + kSharedSteps + wave);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kMine; ++k) {
            const int w = ks + k * KS, step = s + w;
            if (!multiplies || step >= s1) break;
            auto word = [&](int u, int j) { return b[k & 1][u][j] >> sh; };
            v4i fb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                uint32_t x[4], c[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = word(u, j);
                transpose4(x, c);
#pragma unroll
                for (int t = 0; t < 4; ++t) fb[t][u] = (int)c[t];
            }
#pragma unroll
            for (int l = 0; l < kDigits; ++l) {
                const v4i fa = *reinterpret_cast<const v4i *>(digits + ((w * kDigits + l) * 64 + lane) * 16);
                if (p.offset)
#pragma unroll
                    for (int u = 0; u < 4; ++u) row_sum[l] = __builtin_amdgcn_sdot4(fa[u], 0x01010101, row_sum[l], false);
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[l][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb[t], acc[l][t], 0, 0, 0);
            }
            ++since;
            const unsigned int groups = (unsigned int)__builtin_amdgcn_readfirstlane((int)rest[w]);
            if (groups) {
                if (!folded) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) mine[i * 64 + lane] = 0.0;
                    folded = true;
                }
                const bool all = groups >> 16;
                const double unit_of = __hiloint2double((1023 - 172 + cap) << 20, 0), per_unit = __hiloint2double((1023 + 172 - cap) << 20, 0);
#pragma unroll 1
                for (int u = 0; u < 4; ++u) {
                    if (!(groups >> (4 * u) & 15u)) continue;
                    float v4[1][4];
                    src.load_g<1, true>(p, start(step) + 16 * u, v4);
#pragma unroll 1
                    for (int j = 0; j < 4; ++j) {
                        if (!(groups >> (4 * u + j) & 1u)) continue;
                        const float gj = j == 0 ? v4[0][0] : j == 1 ? v4[0][1] : j == 2 ? v4[0][2] : v4[0][3];
                        double v = start(step) + 16 * u + 4 * q + j >= kDigitStep * step ? (double)gj : 0.0;
                        if (!all) {
                            v *= per_unit;
                            v = (v - __builtin_rint(v)) * unit_of;
                        }
                        uint32_t x = 0u;
#pragma unroll
                        for (int i = 0; i < 16; ++i) x = 4 * u + j == i ? word(i >> 2, i & 3) : x;
#pragma unroll 1
                        for (int t = 0; t < 4; ++t) {
                            const v4d sum = __builtin_amdgcn_mfma_f64_16x16x4f64(v, (double)(((int)(x << (24 - 8 * t)) >> 24) + p.offset), v4d{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
                            // (element (row q + 4 r, ...) of that tile)
#pragma unroll
                            for (int r = 0; r < 4; ++r) mine[(4 * t + q) * 64 + 16 * r + (lane & 15)] += sum[r];
                        }
                    }
                }
            }
            if (k + 2 < kMine && step + 2 * KS < s1) load_columns(k, step + 2 * KS);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (multiplies && s + kSharedSteps + ks + k * KS < s1) load_columns(k, s + kSharedSteps + ks + k * KS);
    }
    if (multiplies) fold();
}

constexpr size_t shared_lds(int tiles) { return (size_t)tiles * shared_parts(tiles) * 1024 * sizeof(double) + kSharedSteps * kDigits * 1024; }

template <int TC>
__global__ __launch_bounds__(kDirThreads)
void dw_shared_kernel(DirectProduct p, BwdPlan *plan)
{
    extern __shared__ __attribute__((aligned(16))) char shared_area[];
    double *const sums = reinterpret_cast<double *>(shared_area);      // [waves that multiply][1024], then the digits
    constexpr int KS = shared_parts(TC);
    if (blockIdx.x == 0 && threadIdx.x == 0) no_limbs(plan);
    int item = blockIdx.x;
    const int col0 = item % p.tiles_c * (TC * 64);
    item /= p.tiles_c;
    const int row0 = item % p.tiles_r * 16, split = item / p.tiles_r;
    const int s0 = split * p.steps_per_split, s1 = min(s0 + p.steps_per_split, p.steps);
    shared_tiles<TC>(p, row0, col0, s0, s1, sums, reinterpret_cast<int8_t *>(sums + TC * KS * 1024));
    __syncthreads();
    for (int i = threadIdx.x; i < TC * 256; i += kDirThreads) {
        const int tc = i >> 8, r = i >> 6 & 3, l = i & 63;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] += sums[(k * TC + tc) * 1024 + (4 * t + r) * 64 + l];
        const int row = row0 + 4 * (l >> 4) + r, col = col0 + 64 * tc + 4 * (l & 15);
        if (row >= p.rows) continue;
        if (p.splits > 1) {
            double *o = p.partial + ((int64_t)split * p.rows + row) * p.cols + col;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < p.cols) o[c] = v[c];
        } else store_outputs(p, row, col, v);
    }
}

// The activation gradient of a convolution; one product per class of input pixels.  THIN: few channels, tiles of 64 pixels
// x 16 channels (a tile of 16 x 64 would be padding), else 16 x 64.
struct ConvDxArgs {
    DirectProduct p[4];
    ConvPart cv[4];
    int first[5];          // blocks of class c: first[c] .. first[c + 1]
};

enum DxForm { kThin, kWide, kWideDigits };
template <DxForm FORM>
__global__ __launch_bounds__(kDirThreads)
void conv_dx_direct_kernel(ConvDxArgs a)
{
    constexpr int TM = FORM == kThin ? 4 : 1, TN = FORM == kThin ? 1 : 4;
    __shared__ double lds[kDirWaves * 1024];
    int c = 0;
    while ((int)blockIdx.x >= a.first[c + 1]) ++c;
    const DirectProduct &p = a.p[c];
    const ConvPart &cv = a.cv[c];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), item = (int)blockIdx.x - a.first[c];
    const int tc = item % p.tiles_c, tr = item / p.tiles_c;
    const int row0 = (tr * (kDirWaves / p.ksp) + wave / p.ksp) * 16 * TM, col0 = tc * 16 * TN;
    const auto scattered = [&](int m) {
        const int bb = div_by(m, cv.by_ghw), rem = m - bb * (cv.gh * cv.gw), i = div_by(rem, cv.by_gw), j = rem - i * cv.gw;
        return ((int64_t)bb * cv.H + cv.step * i + cv.oa) * cv.W + cv.step * j + cv.oc;
    };
    GatheredG src;
    src.cv = &cv;
    const bool alone = p.ksp == 1;
    if constexpr (FORM == kWideDigits) {
        Diag dg;
        digit_tile<false, false>(p, src, row0, col0, 0, p.steps, wave % p.ksp, lds + wave * 1024, alone, dg, scattered);
        if (alone) return;
        __syncthreads();
        digit_store(p, lds, row0, col0, 0, scattered);
    } else {
        direct_tile<TM, TN>(p, src, row0, col0, 0, p.steps, wave % p.ksp, alone ? nullptr : lds + wave * 1024, scattered);
        if (alone) return;
        __syncthreads();
        direct_store<TM, TN>(p, lds, row0, col0, 0, scattered);
    }
}

// What the diagnostic words of a product cut into pieces take.
struct ReduceDiag {
    const int *column_sums;            // [splits][cols]
    int cols;
    const unsigned long long *records; // [blocks][2] of the products' kernel
    int blocks, first_b, end_b;        // blocks first_b .. end_b - 1: dL/dQ(b), which have no column sums
    unsigned long long *own;           // [ceil(cols / 32)][2]
    unsigned long long tag;
    float delta_a, delta_b;
    BwdPlan *plan;
    const unsigned int *col_abs_b;     // as in DirectArgs
};

// out[i] = delta * sum over splits of partial[split][i], eight splits side by side per output.  DIAG: the first ceil(cols / 32) blocks
// also add up the pieces' sums of |index| of 32 columns each, and the last of these makes the plan.
template <bool DIAG>
__global__ __launch_bounds__(256)
void direct_reduce_kernel(const double *__restrict__ partial, int splits, int64_t n, double delta, float *__restrict__ out, ReduceDiag dg)
{
    __shared__ double part[8][33];
    const int e = threadIdx.x & 31, sub = threadIdx.x >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + e;
    double s = 0.0;
    if (i < n) {
#pragma unroll 8
        for (int q = sub; q < splits; q += 8) s += partial[(int64_t)q * n + i];
    }
    part[sub][e] = s;
    __syncthreads();
    if (sub == 0 && i < n) {
#pragma unroll
        for (int q = 1; q < 8; ++q) s += part[q][e];
        out[i] = (float)(s * delta);
    }
    if (DIAG) {
        const int owners = (dg.cols + 31) / 32;
        if ((int)blockIdx.x >= owners) return;
        __shared__ unsigned int sums[8][32], red[3][4];
        unsigned int c = 0u;
        if (i < dg.cols)
            for (int q = sub; q < splits; q += 8) c += (unsigned int)dg.column_sums[(int64_t)q * dg.cols + i];
        sums[sub][e] = c;
        __syncthreads();
        auto wave_max = [](unsigned int v) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned int)__shfl_xor((int)v, off, 64));
            return v;
        };
        if (threadIdx.x < 64) {
            c = 0u;
            if (threadIdx.x < 32)
#pragma unroll
                for (int q = 0; q < 8; ++q) c += sums[q][threadIdx.x];
            const unsigned int m = wave_max(c);
            if (threadIdx.x == 0) {
                unsigned long long *r = dg.own + 2 * (size_t)blockIdx.x;
                device_store(r, m);
                device_store(r + 1, m ^ dg.tag);
            }
        }
        if ((int)blockIdx.x != owners - 1) return;
        unsigned int gm = 0u, sa = 0u, sb = 0u;
        for (int k = threadIdx.x; k < dg.blocks; k += 256) {
            const unsigned long long v = dg.records[2 * (size_t)k];
            gm = max(gm, (unsigned int)(v >> 32));
            if (k < dg.first_b || k >= dg.end_b) sb = max(sb, (unsigned int)v);
        }
        for (int k = threadIdx.x; k < owners; k += 256) {
            unsigned long long *r = dg.own + 2 * (size_t)k;
            unsigned long long v, w;
            do {
                v = device_load(r);
                w = device_load(r + 1);
            } while ((v ^ w) != dg.tag);
            device_store(r + 1, v);
            sa = max(sa, (unsigned int)v);
        }
        gm = wave_max(gm);
        sa = wave_max(sa);
        sb = wave_max(sb);
        if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = gm; red[1][threadIdx.x >> 6] = sa; red[2][threadIdx.x >> 6] = sb; }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < 4; ++w) { gm = max(gm, red[0][w]); sa = max(sa, red[1][w]); sb = max(sb, red[2][w]); }
            if (dg.col_abs_b) sb = *dg.col_abs_b;
            choose_limbs(dg.plan, gm, sa, sb, dg.delta_a, dg.delta_b);
        }
    }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Cycles per SIMD that a product takes in double on all of them (a step of 16 entries of a 16 x 64 tile: 1024), and where digits
// are the faster way: from kDigitsFrom on, all products of a launch together.  Both products by cdl_qgemm_bwd, us, in double / on digits:
//   60 x 128 x 448 (400)  4.4 / 8.2    79 x 128 x 1536 (1920)  6.4 / 8.4    256 x 256 x 256 (2048)  6.8 / 8.1
//   2048 x 64 x 256 (4096)  13.2 / 10.8    512 x 512 x 256 (8192)  20 / 10.6
constexpr int64_t kDigitsFrom = 4000;
constexpr int kDirRecords = (int)(kBwdDirectRecordBytes / (2 * sizeof(unsigned long long)));
int64_t double_cycles(const DirectProduct &p) { return ceil_div(p.rows, 16) * ceil_div(p.cols, 64) * ceil_div(p.kc, 16); }

// In double: tiles of 16 x 64 outputs per wave, 16 x 16 where even with eight waves to a tile those would leave half of the
// SIMDs without one; a tile over the waves of a block until there are about two per SIMD; over blocks (max_splits) where the
// contraction is long and the tiles are still few.
void plan_double(DirectProduct &p, int max_splits)
{
    const int64_t steps = ceil_div(p.kc, 16), rows = ceil_div(p.rows, 16);
    p.narrow = rows * ceil_div(p.cols, 64) * (steps < kDirWaves ? steps : kDirWaves) * max_splits < 512;
    p.tiles_c = (int)ceil_div(p.cols, p.narrow ? 16 : 64);
    p.steps = (int)steps;
    p.ksp = 1;
    while (p.ksp < kDirWaves && 2 * p.ksp <= steps && rows * p.tiles_c * p.ksp < 2048) p.ksp *= 2;
    p.tiles_r = (int)ceil_div(rows, kDirWaves / p.ksp);
    int64_t splits = 768 / ((int64_t)p.tiles_r * p.tiles_c);
    if (splits > steps / (4 * p.ksp)) splits = steps / (4 * p.ksp);
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    p.steps_per_split = (int)ceil_div(steps, splits);
    p.splits = (int)ceil_div(steps, p.steps_per_split);
}

// On digits: tiles of 16 x 64.  A compute unit holds one block of eight waves (two to a SIMD, the registers of the digit sums).  What
// is chosen: how many waves of a block share a tile's contraction (ksp) for each product, and, where the outputs may be cut into
// pieces over blocks (partial), how many.  A block takes about 4 us and 2 us for each step of its waves; the choice is the one
// whose blocks, the longer ones first, are done soonest on 256 compute units (256 x 1000 x 512, both products: 254 blocks in one
// round, 12 us; 384 in two, 18).  Pieces cost another launch and their traffic.  Returns that time, us.
constexpr int kDigitBlocks = 256;
double plan_digits(DirectProduct **ps, int n, int max_splits)
{
    struct Choice { int64_t tiles, blocks; int ksp, splits; double us; };
    auto choice = [](const DirectProduct &p, int ksp, int64_t splits) {
        Choice c;
        c.ksp = ksp;
        c.tiles = ceil_div(ceil_div(p.rows, 16), kDirWaves / ksp) * p.tiles_c;
        const int64_t per = ceil_div(p.steps, splits);
        c.splits = (int)ceil_div(p.steps, per);
        c.blocks = c.tiles * c.splits;
        c.us = 4.0 + 2.0 * (double)ceil_div(per, ksp);
        return c;
    };
    // blocks of x, which take longer, spread over the compute units; then those of y, where one is free
    auto makespan = [](const Choice &x, const Choice &y) {
        const int64_t rounds = x.blocks / kDigitBlocks, rest = x.blocks % kDigitBlocks;
        const double early = (double)rounds * x.us, late = rest ? early + x.us : early;
        for (int64_t k = 0;; ++k)
            for (int half = 0; half < 2; ++half) {
                const double t = (half ? late : early) + (double)k * y.us;
                if (t < late) continue;
                const int64_t room = (kDigitBlocks - rest) * (int64_t)((t - early) / y.us + 1e-9) + rest * (int64_t)((t - late) / y.us + 1e-9);
                if (room >= y.blocks) return t;
            }
    };
    Choice best[2] = {}, some[2][16];
    int count[2] = {1, 1};
    some[1][0] = Choice{0, 0, 1, 1, 1.0};
    for (int i = 0; i < n; ++i) {
        DirectProduct &p = *ps[i];
        p.narrow = 0;
        p.tiles_c = (int)ceil_div(p.cols, 64);
        p.steps = (int)ceil_div(p.kc, kDigitStep);
        count[i] = 0;
        for (int ksp = 1; ksp <= kDirWaves; ksp *= 2) {
            if (ksp > 1 && ksp > p.steps) break;
            some[i][count[i]++] = choice(p, ksp, 1);
            const int64_t tiles = some[i][count[i] - 1].tiles;
            for (int rounds = 1; rounds <= 3 && p.partial; ++rounds) {
                int64_t splits = rounds * kDigitBlocks / tiles;
                if (splits > max_splits) splits = max_splits;
                if (splits > p.steps / ksp) splits = p.steps / ksp;
                if (splits > 1) some[i][count[i]++] = choice(p, ksp, splits);
            }
        }
    }
    double least = -1.0;
    for (int i = 0; i < count[0]; ++i)
        for (int j = 0; j < count[1]; ++j) {
            const Choice &x = some[0][i], &y = some[1][j];
            if (least >= 0.0 && ((double)x.blocks * x.us + (double)y.blocks * y.us >= least * kDigitBlocks || x.us >= least || y.us >= least)) continue;
            double t = x.us >= y.us ? makespan(x, y) : makespan(y, x);
            for (int k = 0; k < n; ++k) {
                const Choice &c = k ? y : x;
                if (c.splits > 1) t += 5.0 + (double)c.splits * ps[k]->rows * ps[k]->cols * 16.0 / 5e6;
            }
            if (least < 0.0 || t < least) { least = t; best[0] = x; best[1] = y; }
        }
    for (int i = 0; i < n; ++i) {
        DirectProduct &p = *ps[i];
        p.ksp = best[i].ksp;
        p.tiles_r = (int)(best[i].tiles / p.tiles_c);
        p.splits = best[i].splits;
        p.steps_per_split = (int)ceil_div(p.steps, p.splits);
        p.splits = (int)ceil_div(p.steps, p.steps_per_split);
    }
    return least;
}

// Blocks that share digits (dw_shared_kernel): column groups of equal numbers of tiles, pieces of whole rounds; the number of pieces whose time is the least.  Returns that time, us
// (fitted to 52 layers of 17 to 308 rows, 80 to 2000 columns and 2 to 400 thousand contraction entries).
double plan_shared(DirectProduct &p, int max_splits, int &tiles)
{
    const int64_t all = ceil_div(p.cols, 64);
    tiles = (int)ceil_div(all, ceil_div(all, kSharedTiles));
    p.tiles_c = (int)ceil_div(all, tiles);
    p.tiles_r = (int)ceil_div(p.rows, 16);
    p.steps = (int)ceil_div(p.kc, kDigitStep);
    p.narrow = 0;
    const int64_t per_split = (int64_t)p.tiles_r * p.tiles_c;
    double least = -1.0;
    for (int blocks = 1; blocks <= 4; ++blocks) {      // of a compute unit
        int64_t splits = blocks * kDigitBlocks / per_split;
        if (splits > max_splits) splits = max_splits;
        if (splits < 1) splits = 1;
        const int64_t rounds = ceil_div(ceil_div(p.steps, splits), kSharedSteps);
        splits = ceil_div(p.steps, rounds * kSharedSteps);
        double t = (double)ceil_div(splits * per_split, kDigitBlocks) * (3.0 + (4.5 + 1.4 * (tiles - 2)) * (double)rounds);
        if (splits > 1) t += 5.0 + (double)splits * p.rows * p.cols * 16.0 / 5e6;
        if (least >= 0.0 && t >= least) continue;
        least = t;
        p.steps_per_split = (int)(rounds * kSharedSteps);
        p.splits = (int)splits;
    }
    return least;
}

// Where they serve: by the two plans' times.  That of plan_digits does not count what is read several times: it is up to 2.2 times too short where the operands are long, and about right up to 5120 contraction
// entries, or 20480 against groups of five and six tiles, whose waves have the longest rounds.  Of 530 layers of 1000 to 450000 entries, 20 to 360 rows and 80 to 1600 columns, each measured both ways, 209 are served, in 0.78 of
// the time of digit_tile, ten of them more than 2 % slower (by one margin of 1.15 for all 34 of 237: 7259 x 320 x 608 30.4 / 37.1, 12354 x 120 x 528 24.6 / 29.6; left 99871 x 56 x 480 54.2 / 64.0, 13763 x 56 x 496 16.3 / 19.2).
// A second tile of a few columns is not worth its padding (270320 x 19 x 69 30.5 / 31.7).
bool shared_serves(const DirectProduct &p, int max_splits)
{
    if (p.cols < 80 || p.kc < kDigitStep) return false;
    DirectProduct now = p, shared = p, *one = &now;
    int tiles;
    const double us = plan_shared(shared, max_splits, tiles);
    return us < (p.kc < (tiles >= 5 ? 20480 : 5120) ? 0.95 : 1.15) * plan_digits(&one, 1, max_splits);
}

int launch_shared(DirectProduct &p, int max_splits, BwdPlan *plan, hipStream_t stream)
{
    int tiles = 0;
    plan_shared(p, max_splits, tiles);
    const dim3 grid((unsigned)(p.tiles_r * p.tiles_c * p.splits)), threads(kDirThreads);
    const size_t lds = shared_lds(tiles);
#define CDL_SHARED(TC) \
    do { \
        const hipError_t e = hipFuncSetAttribute((const void *)dw_shared_kernel<TC>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        if (e != hipSuccess) return hip_failed(e); \
        CDL_LAUNCH("dw_shared_kernel", stream, dw_shared_kernel<TC>, grid, threads, lds, p, plan); \
    } while (0)
    switch (tiles) {
        case 2: CDL_SHARED(2); break;
        case 3: CDL_SHARED(3); break;
        case 4: CDL_SHARED(4); break;
        case 5: CDL_SHARED(5); break;
        default: CDL_SHARED(6); break;
    }
#undef CDL_SHARED
    const int rc = check_launch();
    if (rc != CDL_OK || p.splits == 1) return rc;
    const int64_t n = (int64_t)p.rows * p.cols;
    CDL_LAUNCH("direct_reduce_kernel", stream, direct_reduce_kernel<false>, dim3((unsigned)ceil_div(n, 32)), dim3(256), 0, p.partial, p.splits, n, p.delta, p.out, ReduceDiag{});
    return check_launch();
}

}  // namespace

static int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// multiply-adds of one product, counted in whole tiles
static double padded_macs(int64_t rows, int64_t kc, int64_t cols) { return (double)round_up(rows, 16) * (double)round_up(kc, 16) * (double)round_up(cols, 64); }

// Up to kBwdDirectNoDiag the diagnostic words say that neither product has limbs.
constexpr int64_t kBwdDirectNoDiag = 1ll << 25;

bool bwd_direct_diag(int32_t M, int32_t N, int32_t K) { return N > 32 && (int64_t)M * N * K > kBwdDirectNoDiag; }

// DirectProduct::rounds_to.  Where sums in double are the alternative (`exact`) nothing is rounded.  Beyond, the alternative are limbs, whose
// rounding may change an output by kLimbBoundTarget, and digits may round (entries 2^-20 of their row's largest and smaller, by half a unit,
// 2^(cap - 173)) where that changes an output by a 512th of it at most, whatever the indices.  That is never more than limbs round an entry: up to five
// leave 2^-40 of the largest |g| of all at least, digits 2^-44 of the row's; six leave 2^-48 of it, but serve only where five miss the target,
// hence for a |g| beyond 2^(cap - 125).
static int digits_round_to(const DirectProduct &p, bool exact)
{
    if (exact) return -1;
    const int e = 173 + std::ilogb(kLimbBoundTarget / 512.0 / (p.delta * (128.0 + std::abs(p.offset)) * (double)p.kc));
    return e < -1 ? -1 : (e > 254 ? 254 : e);
}

// Products of `macs` multiply-adds in all that sums in double serve as fast as limbs (both, us, in double / on limbs: 2000 x 300 x 1000 67 / 70;  1000 x 1000 x 1000
// 88 / 65), with the diagnostic words as far as a contraction in one piece is.
static bool exact_serves(double macs, int32_t M, int32_t N, bool diag) { return macs <= 7e8 && (!diag || (M <= 5120 && N <= 5120)); }

// The products of a call as a launch: in double or on digits, and the plan.
struct BwdDirectPlan {
    DirectProduct a, b;
    DirectProduct *ps[2];
    int n;
    bool digits;
    double us;             // on digits: what it takes
};

// (by the layer's sizes alone: an output that is formed here is formed in the same order whether or not the other one is asked for too; whether dL/dQ(a) of a short contraction is, and
// what is served here between 0.35 and 0.7 G multiply-adds, depends on that: da_direct_preferred, bwd_direct_serves)
static void plan_bwd_direct(BwdDirectPlan &d, int32_t M, int32_t N, int32_t K, bool only_b, bool diag, double *partial, int max_splits)
{
    d.a = d.b = DirectProduct{};
    d.n = 0;
    int64_t cycles = 0;
    if (!only_b) {
        d.a.rows = M; d.a.cols = K; d.a.kc = N;
        cycles += double_cycles(d.a);
        d.ps[d.n++] = &d.a;
    }
    d.b.rows = N; d.b.cols = K; d.b.kc = M; d.b.partial = partial;
    cycles += double_cycles(d.b);
    d.ps[d.n++] = &d.b;
    d.digits = diag || cycles >= kDigitsFrom;
    if (!d.digits) {
        for (int i = 0; i < d.n; ++i) plan_double(*d.ps[i], d.ps[i]->partial ? max_splits : 1);
        return;
    }
    // (the column sums of the pieces take the place of the last piece's partial results)
    int pieces = max_splits;
    if (diag) pieces = (int)(max_splits - 1 < 2 * (int64_t)N ? max_splits - 1 : 2 * (int64_t)N);
    if (pieces < 1 || (diag && ceil_div(K, 32) > kDirRecords / 2)) pieces = 1;
    d.us = plan_digits(d.ps, d.n, pieces);
    // the longer waves first
    if (d.n == 2 && ceil_div(d.b.steps_per_split, d.b.ksp) > ceil_div(d.a.steps_per_split, d.a.ksp)) { d.ps[0] = &d.b; d.ps[1] = &d.a; }
}

// Where the products are formed directly: the small ones, what double serves (exact_serves), and of the others those whose plan takes less time than the limb products
// with their helpers, 27 us + 4.8 us for a thousand million multiply-adds in whole tiles + 0.36 us a megabyte (fitted to 54 shapes of
// 30 M to 2.6 G multiply-adds, off by 17 %; the plan's time is 0.9 of the measured one, hence 1.25).  Both products, limbs / directly, us:
//   307 x 1257 x 83  39 / 14     700 x 700 x 700  48 / 20      3914 x 1024 x 128  46 / 25    1092 x 1172 x 785  42 / 43
//   12425 x 64 x 192  42 / 21    152 x 2252 x 928  43 / 24     9020 x 2048 x 128  116 / 93   2934 x 384 x 1152  47 / 61
bool bwd_direct_serves(int32_t M, int32_t N, int32_t K, bool only_b, double *partial, int max_splits, bool words, int asked)
{
    if (K < 4) return false;
    const double macs = ((only_b ? 0.0 : (double)round_up(M, 32) * (double)round_up(N, 128)) + (double)round_up(N, 32) * (double)round_up(M, 128)) * (double)round_up(K, 128);
    const double bytes = 4.0 * M * N * (only_b ? 2 : 3) + (double)K * (M + 4.0 * N + (only_b ? 0.0 : N + 4.0 * M));
    if (macs > 1e10) return false;
    BwdDirectPlan d;
    plan_bwd_direct(d, M, N, K, only_b, words && bwd_direct_diag(M, N, K), partial, max_splits);
    int64_t blocks = 0;
    for (int i = 0; i < d.n; ++i) blocks += (int64_t)d.ps[i]->tiles_r * d.ps[i]->tiles_c * d.ps[i]->splits;
    // (what double serves goes directly in any case: exact products.  24 layers of 0.36 - 0.7 G multiply-adds a product that limbs would serve, one product a call, us
    // in all, dL/dQ(a) / dL/dQ(b): on limbs 1052 / 874, directly 832 / 773; a few are slower, 2208 x 64 x 4672 28 / 34 and 41 / 37)
    if (asked > 0 && blocks <= kDirRecords / 2 && exact_serves(asked * padded_macs(M, N, K), M, N, words && bwd_direct_diag(M, N, K))) return true;
    return !d.digits || (blocks <= kDirRecords / 2 && 1.25 * d.us < 27.0 + 4.8e-9 * macs + 0.36e-6 * bytes);
}

int launch_bwd_direct(const float *g, const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float delta_a, float delta_b,
                      int32_t a_offset, int32_t b_offset, float *d_a_hat, float *d_b_hat, BwdPlan *plan, void *records, double *partial, int max_splits,
                      bool only_b, bool words, const unsigned int *col_abs_b, hipStream_t stream)
{
    const bool diag = words && bwd_direct_diag(M, N, K);
    BwdDirectPlan d;
    plan_bwd_direct(d, M, N, K, only_b, diag, partial, max_splits);
    d.a.g = g; d.a.idx = b_idx; d.a.ldg = N; d.a.ldi = K; d.a.offset = b_offset; d.a.vec = N % 4 == 0; d.a.delta = (double)delta_b; d.a.out = d_a_hat;
    d.b.g = g; d.b.idx = a_idx; d.b.ldg = N; d.b.ldi = K; d.b.offset = a_offset; d.b.delta = (double)delta_a; d.b.out = d_b_hat;
    // (by what is asked for: only outputs next to entries of g more than 2^20 times as large can show it)
    const int asked = (d.a.out && !only_b ? 1 : 0) + (d.b.out ? 1 : 0);
    const bool exact = exact_serves(asked * padded_macs(M, N, K), M, N, diag);
    d.a.rounds_to = digits_round_to(d.a, exact);
    d.b.rounds_to = digits_round_to(d.b, exact);
    if (only_b && d.digits && !diag && d_b_hat && shared_serves(d.b, max_splits)) return launch_shared(d.b, max_splits, plan, stream);
    DirectArgs a{};
    a.plan = plan;
    a.records = reinterpret_cast<unsigned long long *>(records);
    a.delta_a = delta_a; a.delta_b = delta_b;
    unsigned grid = 0;
    int at = 0;
    a.a_at = 1;
    for (int i = 0; i < d.n; ++i) {
        if (!d.ps[i]->out) continue;
        if (d.ps[i] == &d.a) a.a_at = at;
        a.p[at] = *d.ps[i];
        grid += (unsigned)(a.p[at].tiles_r * a.p[at].tiles_c * a.p[at].splits);
        if (at++ == 0) a.first = (int)grid;
    }
    const int splits = d_b_hat ? d.b.splits : 1;
    if (diag) {
        a.tag = next_finish_tag();
        a.col_abs_b = col_abs_b;
        if (splits > 1) a.column_sums = reinterpret_cast<int *>(partial + (int64_t)splits * N * K);
    }
#define CDL_DIRECT(KERNEL) CDL_LAUNCH("bwd_direct_kernel", stream, (KERNEL), dim3(grid), dim3(kDirThreads), 0, a)
    const bool is_short = M < kDigitStep || N < kDigitStep;
    if (!d.digits) CDL_DIRECT(bwd_double_kernel);
    else if (diag) { if (is_short) CDL_DIRECT((bwd_direct_kernel<true, true>)); else CDL_DIRECT((bwd_direct_kernel<true, false>)); }
    else { if (is_short) CDL_DIRECT((bwd_direct_kernel<false, true>)); else CDL_DIRECT((bwd_direct_kernel<false, false>)); }
#undef CDL_DIRECT
    int rc = check_launch();
    if (rc == CDL_OK && splits > 1) {
        const int64_t n_out = (int64_t)N * K;
        const dim3 blocks((unsigned)ceil_div(n_out, 32));
        if (diag) {
            const int b_first = a.a_at == 0 ? a.first : 0, b_end = a.a_at == 0 ? (int)grid : a.first;
            const ReduceDiag dg{a.column_sums, K, a.records, (int)grid, b_first, b_end, a.records + kDirRecords, next_finish_tag(), delta_a, delta_b, plan, col_abs_b};
            CDL_LAUNCH("direct_reduce_kernel", stream, direct_reduce_kernel<true>, blocks, dim3(256), 0, partial, splits, n_out, (double)delta_a, d_b_hat, dg);
        } else {
            CDL_LAUNCH("direct_reduce_kernel", stream, direct_reduce_kernel<false>, blocks, dim3(256), 0, partial, splits, n_out, (double)delta_a, d_b_hat, ReduceDiag{});
        }
        rc = check_launch();
    }
    return rc;
}

// The gradients of a convolution, directly / on limbs, us: weights, 16 x 28 x 28 x 64 -> 64, 3 x 3 (0.5 G in whole tiles)  16 / 32;
// 24 x 32 x 32 x 48 -> 84 (1.0 G)  28 / 39;  31 x 30 x 30 x 80 -> 56 (1.3 G)  36 / 41;  25 x 33 x 33 x 288 -> 112, stride 2 (1.7 G)  51 / 40;
// activations, on digits  58 x 19 x 19 x 80 -> 32 (0.8 G)  28 / 29;  72 x 17 x 17 x 272 -> 64, stride 2 (1.0 G)  35 / 37;
// 17 x 9 x 9 x 368 -> 204 (1.0 G)  40 / 39;  31 x 30 x 30 x 80 -> 56 (1.8 G)  45 / 40.
constexpr double kConvDwDirectMaxMacs = 1.2e9, kConvDxDirectMaxMacs = 1e9, kConvDxDoubleMaxMacs = 5e8;
constexpr double kConvExactMacs = 5e8;      // (digits_round_to: as far as sums in double are as fast as limbs)

bool conv_dw_direct_serves(int64_t M, int32_t N, int32_t K) { return padded_macs(N, M, K) <= kConvDwDirectMaxMacs; }

int launch_conv_dw_direct(const float *g, const int8_t *x_idx, const ConvWindows &w, int32_t N, float delta_x, int32_t x_offset, float *d_w_hat,
                          double *partial, int max_splits, hipStream_t stream)
{
    DirectProduct p{};
    p.g = g; p.idx = x_idx; p.rows = N; p.cols = w.R * w.S * w.C; p.kc = w.B * w.P * w.Q; p.ldg = N;
    p.offset = x_offset; p.delta = (double)delta_x; p.out = d_w_hat; p.partial = partial;
    p.rounds_to = digits_round_to(p, padded_macs(p.rows, p.kc, p.cols) <= kConvExactMacs);
    DirectProduct *one = &p;
    const bool digits = p.kc >= kDigitStep && double_cycles(p) >= kDigitsFrom / 2;
    if (digits) plan_digits(&one, 1, max_splits);
    else plan_double(p, max_splits);
    ConvPart cv{};
    cv.H = w.H; cv.W = w.W; cv.C = w.C; cv.S = w.S; cv.stride = w.stride; cv.pad = w.pad; cv.P = w.P; cv.Q = w.Q;
    cv.pad_byte = (int)(uint8_t)(int8_t)(-x_offset);
    cv.by_pq = make_div_by((uint32_t)(w.P * w.Q));
    cv.by_q = make_div_by((uint32_t)w.Q);
    cv.end_w = w.Q * w.stride; cv.end_h = w.P * w.stride;
    cv.next_w = w.stride * w.C; cv.next_h = (w.stride * w.W - cv.end_w) * w.C; cv.next_b = (w.H - cv.end_h) * w.W * w.C;
    const unsigned grid = (unsigned)(p.tiles_r * p.tiles_c * p.splits);
    if (digits) CDL_LAUNCH("conv_dw_direct_kernel", stream, conv_dw_direct_kernel<true>, dim3(grid), dim3(kDirThreads), 0, p, cv);
    else CDL_LAUNCH("conv_dw_direct_kernel", stream, conv_dw_direct_kernel<false>, dim3(grid), dim3(kDirThreads), 0, p, cv);
    int rc = check_launch();
    if (rc == CDL_OK && p.splits > 1) {
        const int64_t n = (int64_t)p.rows * p.cols;
        CDL_LAUNCH("direct_reduce_kernel", stream, direct_reduce_kernel<false>, dim3((unsigned)ceil_div(n, 32)), dim3(256), 0, partial, p.splits, n, p.delta, d_w_hat, ReduceDiag{});
        rc = check_launch();
    }
    return rc;
}

// The form of an activation gradient.  On digits where every class of input pixels has 64 contraction entries and the product is not
// tiny; few channels take tiles of 16 in double: up to 16, and up to 32 where the contraction is short (us, thin / digits:
// 128 x 32 x 32 x 16 -> 16, 3 x 3  24 / 46;  ... x 32 -> 16  38 / 45;  189 x 19 x 19 x 32 -> 32  66 / 45;  64 x 14 x 14 x 48 -> 48  27 / 17).
static DxForm conv_dx_form(int64_t pixels, int32_t N, int32_t C, int32_t R, int32_t S, int32_t stride)
{
    if (C <= 16 || (C <= 32 && (int64_t)R * S * N < 256 * stride * stride)) return kThin;
    const int64_t least = stride == 1 ? (int64_t)R * S : (int64_t)(R > 1 ? R / 2 : 1) * (S > 1 ? S / 2 : 1);      // taps of a class
    const int64_t cycles = ceil_div(pixels, 16) * ceil_div(C, 64) * ceil_div((int64_t)R * S * N, 16) / (stride * stride);
    return least * N >= kDigitStep && cycles >= kDigitsFrom / 2 ? kWideDigits : kWide;
}

// what sums in double serve, in tiles of 16 columns up to 48 channels; macs: multiply-adds of a column
static bool conv_dx_exact(double macs, int32_t C) { return macs * (double)round_up(C, C <= 48 ? 16 : 64) <= kConvExactMacs; }

bool conv_dx_direct_serves(int64_t pixels, int32_t N, int32_t C, int32_t R, int32_t S, int32_t stride)
{
    if (C <= 32 && (int64_t)R * S * N <= 288) return true;      // (any number of pixels: most of a limb tile would be padding)
    const DxForm form = conv_dx_form(pixels, N, C, R, S, stride);
    const double macs = (double)pixels * (double)round_up((int64_t)R * S * N, 16) / (stride * stride);      // a column
    return macs * (double)round_up(C, form == kThin ? 16 : 64) <= (form == kWideDigits ? kConvDxDirectMaxMacs : kConvDxDoubleMaxMacs) || conv_dx_exact(macs, C);
}

int launch_conv_dx_direct(const float *g, const int8_t *w_idx, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                          int32_t R, int32_t S, int32_t P, int32_t Q, int32_t stride, float delta_w, float *d_x_hat, hipStream_t stream)
{
    const DxForm form = conv_dx_form((int64_t)B * H * W, N, C, R, S, stride);
    const bool thin = form == kThin;
    ConvDxArgs a{};
    int blocks = 0;
    for (int c = 0; c < n_grids; ++c) {
        const ConvDxGrid &k = grids[c];
        DirectProduct &p = a.p[c];
        p.g = g; p.idx = w_idx; p.rows = B * k.Hc * k.Wc; p.cols = C; p.kc = k.Rc * k.Sc * N;
        p.delta = (double)delta_w; p.out = d_x_hat; p.splits = 1;
        p.rounds_to = digits_round_to(p, conv_dx_exact((double)B * H * W * (double)round_up((int64_t)R * S * N, 16) / (stride * stride), C));
        const int64_t steps = ceil_div(p.kc, form == kWideDigits ? kDigitStep : 16), rows = ceil_div(p.rows, thin ? 64 : 16);
        p.steps = (int)steps;
        p.tiles_c = (int)ceil_div(C, thin ? 16 : 64);
        p.ksp = 1;
        while (p.ksp < kDirWaves && 2 * p.ksp <= steps && rows * p.tiles_c * p.ksp < (form == kWideDigits ? kDigitBlocks * kDirWaves / 2 : 2048)) p.ksp *= 2;
        p.tiles_r = (int)ceil_div(rows, kDirWaves / p.ksp);
        ConvPart &cv = a.cv[c];
        cv.H = H; cv.W = W; cv.C = C; cv.S = S; cv.P = P; cv.Q = Q;
        cv.gh = k.Hc; cv.gw = k.Wc; cv.gn = N; cv.st = k.Sc; cv.ph = k.pad_h; cv.pw = k.pad_w;
        cv.step = stride; cv.oa = k.oa; cv.oc = k.oc; cv.r0 = k.r0; cv.s0 = k.s0;
        cv.by_ghw = make_div_by((uint32_t)(k.Hc * k.Wc)); cv.by_gw = make_div_by((uint32_t)k.Wc);
        cv.by_gn = make_div_by((uint32_t)N); cv.by_st = make_div_by((uint32_t)k.Sc);
        cv.taps_c = R * S * C;
        a.first[c] = blocks;
        blocks += p.tiles_r * p.tiles_c;
    }
    for (int c = n_grids; c <= 4; ++c) a.first[c] = blocks;
    if (blocks == 0) return CDL_OK;
    if (form == kThin) CDL_LAUNCH("conv_dx_direct_kernel", stream, conv_dx_direct_kernel<kThin>, dim3((unsigned)blocks), dim3(kDirThreads), 0, a);
    else if (form == kWide) CDL_LAUNCH("conv_dx_direct_kernel", stream, conv_dx_direct_kernel<kWide>, dim3((unsigned)blocks), dim3(kDirThreads), 0, a);
    else CDL_LAUNCH("conv_dx_direct_kernel", stream, conv_dx_direct_kernel<kWideDigits>, dim3((unsigned)blocks), dim3(kDirThreads), 0, a);
    return check_launch();
}

}  // namespace cdl
