// Backward products of small layers, formed directly in double on the matrix cores (v_mfma_f64_16x16x4_f64).
//
// The limb products of cdl_qgemm.hip need the largest |g|, transposed copies of the index operands and a plan before
// their first multiplication: seven launches and 45 us for a layer whose products are a microsecond of arithmetic.  A
// product of a float and a level index is exact in double, and a sum of n of them is off by at most n 2^-53 of the sum of
// their magnitudes, far below the rounding of the fp32 result; so where the contraction is small enough for the double
// rate (69 TFLOP/s measured, against 2 POP/s of a limb) both products run here in one launch, straight from the
// operands where they lie.  One wave forms 16 x 64 outputs (or 64 x 16 where there are few columns): per step of 16
// contraction entries a lane loads four entries of one row of the fp32 operand and, for each of them, four neighbouring
// index bytes of the other, enough for 16 MFMAs of 64 cycles; the order of the entries inside a step is the same on both
// sides and otherwise free.  The waves of a block split the contraction and add their tiles through LDS in a fixed order.
#include "cdl_internal.h"
#include "cdl_finish.h"
#include "cdl_bwd_plan.h"
#include "cdl_div.h"

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
    int tiles_r, tiles_c, splits, steps_per_split;
    double delta;
    float *out;            // [rows][cols]
    double *partial;       // [splits][rows][cols], unscaled, when splits > 1
};

// ---- where the operands of one lane come from.  load: contraction entries e .. e + 3, as they lie in memory (what is done
// to them waits until they are multiplied, so that the loads of the next step stay in flight); WHOLE: all four exist. ----

// the index bytes of four columns of a row-major index matrix, in as many rows as the step has entries
struct IndexColumns {
    const int8_t *col;
    int sh;                // the last columns of a matrix whose width is no multiple of four: a word that ends with the row, shifted
    template <int TN>
    __device__ __forceinline__ void init_index(const DirectProduct &p, int col0, int lane)
    {
        // TN = 1: one column per lane, a byte
        const int c = col0 + TN * (lane & 15), cc = min(c, p.cols - TN);      // (host: cols >= 4)
        col = p.idx + cc;
        sh = 8 * min(c - cc, 3);
    }
    template <int TN, bool WHOLE>
    __device__ __forceinline__ void load_index(const DirectProduct &p, int e, uint32_t (&b)[4]) const
    {
        const int8_t *q = col + (int64_t)e * p.ldi;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int8_t *at = WHOLE ? q + j * p.ldi : col + (int64_t)min(e + j, p.kc - 1) * p.ldi;
            if (TN == 4) b[j] = *reinterpret_cast<const u32_any *>(at);
            else b[j] = *reinterpret_cast<const uint8_t *>(at);
        }
    }
};

// rows of g: dL/dQ(a)[m][k] = sum_n g[m][n] b[n][k]
struct RowsOfG : IndexColumns {
    static constexpr int kMask = 0;
    const float *row[4];
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int row0, int col0, int lane)
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) row[i] = p.g + (int64_t)min(row0 + 16 * i + (lane & 15), p.rows - 1) * p.ldg;
        init_index<TN>(p, col0, lane);
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e, float (&a)[TM][4], uint32_t (&b)[4], int &) const
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (p.vec) {
                const float4 v = *reinterpret_cast<const float4 *>(row[i] + (WHOLE ? e : min(e, p.kc - 4)));
                a[i][0] = v.x; a[i][1] = v.y; a[i][2] = v.z; a[i][3] = v.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) a[i][j] = row[i][WHOLE ? e + j : min(e + j, p.kc - 1)];
            }
        }
        load_index<TN, WHOLE>(p, e, b);
    }
};

// columns of g: dL/dQ(b)[n][k] = sum_m g[m][n] a[m][k]
struct ColumnsOfG {
    const float *at[4];
    template <int TM>
    __device__ __forceinline__ void init_g(const DirectProduct &p, int row0, int lane)
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) at[i] = p.g + min(row0 + 16 * i + (lane & 15), p.rows - 1);
    }
    template <int TM, bool WHOLE>
    __device__ __forceinline__ void load_g(const DirectProduct &p, int e, float (&a)[TM][4]) const
    {
        const int64_t o = (int64_t)e * p.ldg;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i][j] = at[i][WHOLE ? o + j * p.ldg : (int64_t)min(e + j, p.kc - 1) * p.ldg];
    }
};

struct ColumnsOfGMatrix : ColumnsOfG, IndexColumns {
    static constexpr int kMask = 0;
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int row0, int col0, int lane)
    {
        init_g<TM>(p, row0, lane);
        init_index<TN>(p, col0, lane);
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e, float (&a)[TM][4], uint32_t (&b)[4], int &) const
    {
        load_g<TM, WHOLE>(p, e, a);
        load_index<TN, WHOLE>(p, e, b);
    }
};

// columns of g against the windows of a convolution.  kMask = 1: bit j of `ok` says whether entry j lies inside the image.
struct ColumnsOfGWindows : ColumnsOfG {
    static constexpr int kMask = 1;
    const ConvPart *cv;
    const int8_t *tap;     // x shifted by the column's tap and channel
    int tr, ts, sh;
    template <int TM, int TN>
    __device__ __forceinline__ void init(const DirectProduct &p, int row0, int col0, int lane)
    {
        init_g<TM>(p, row0, lane);
        const int c = min(col0 + TN * (lane & 15), p.cols - TN), t = c / cv->C;      // (cols a multiple of 16, a word inside one tap)
        tr = t / cv->S - cv->pad;
        ts = t - t / cv->S * cv->S - cv->pad;
        tap = p.idx + ((int64_t)tr * cv->W + ts) * cv->C + (c - t * cv->C);
        sh = 0;
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e, float (&a)[TM][4], uint32_t (&b)[4], int &ok) const
    {
        load_g<TM, WHOLE>(p, e, a);
        ok = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = WHOLE ? e + j : min(e + j, p.kc - 1);
            const int bb = div_by(m, cv->by_pq), rem = m - bb * (cv->P * cv->Q), pp = div_by(rem, cv->by_q), qq = rem - pp * cv->Q;
            const int h = pp * cv->stride, w = qq * cv->stride;
            const bool in = (unsigned)(h + tr) < (unsigned)cv->H && (unsigned)(w + ts) < (unsigned)cv->W;
            ok |= in ? 1 << j : 0;
            const int8_t *at = in ? tap + ((int64_t)(bb * cv->H + h) * cv->W + w) * cv->C : p.idx;
            if (TN == 4) b[j] = *reinterpret_cast<const uint32_t *>(at);
            else b[j] = *reinterpret_cast<const uint8_t *>(at);
        }
    }
};

// g gathered tap by tap against the kernels as they lie.  kMask = 2: bit i of `ok` says whether row i's pixel is there.
struct GatheredG {
    static constexpr int kMask = 2;
    const ConvPart *cv;
    const int8_t *col;
    int gi[4], gj[4], base[4], sh;
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
    }
    template <int TM, int TN, bool WHOLE>
    __device__ __forceinline__ void load(const DirectProduct &p, int e, float (&a)[TM][4], uint32_t (&b)[4], int &ok) const
    {
        const int k = WHOLE ? e : min(e, p.kc - 4);                     // (gn a multiple of 4: four entries share a tap)
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

// The products of a tile over steps [s0, s1) of 16 contraction entries, wave ks of p.ksp, into the wave's part of LDS
// (`mine`), or to memory where there is nothing to add (null).
// TM x TN: 16 x 16 MFMA tiles; TN = 4: the tiles' columns are the four bytes of a word, 64 columns in all.
struct Diag { float amax; int colabs[4]; };

template <int TM, int TN, bool DIAG, class Src, class RowMap>
__device__ __forceinline__ void direct_tile(const DirectProduct &p, Src &src, int row0, int col0, int s0, int s1, int ks, double *mine, Diag &dg, RowMap out_row,
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
        const int e = 16 * s + q4;
        if (16 * s + 16 <= p.kc) src.template load<TM, TN, true>(p, e, a[u], b[u], ok[u]);
        else src.template load<TM, TN, false>(p, e, a[u], b[u], ok[u]);
    };
    auto multiply = [&](int u, int s) {
        const int e = 16 * s + q4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double av[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const float v = e + j < p.kc && (Src::kMask != 2 || (ok[u] >> i & 1)) ? a[u][i][j] : 0.0f;
                if (DIAG) dg.amax = fmaxf(dg.amax, fabsf(v));
                av[i] = (double)v;
            }
            const uint32_t w = Src::kMask == 1 && !(ok[u] >> j & 1) ? pad_word : b[u][j] >> src.sh;
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const int x = (int)(w << (24 - 8 * t)) >> 24;
                const double bv = (double)(x + p.offset);
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv, acc[i][t], 0, 0, 0);
                if (DIAG) dg.colabs[t] += e + j < p.kc ? abs(x) : 0;
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
            float *o = p.out + out_row(row) * p.cols + col;
            if ((p.cols & 3) == 0) {
                if (col < p.cols) *reinterpret_cast<float4 *>(o) = make_float4((float)(v[0] * p.delta), (float)(v[1] * p.delta), (float)(v[2] * p.delta), (float)(v[3] * p.delta));
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (col + c < p.cols) o[c] = (float)(v[c] * p.delta);
            }
        }
    }
}

struct DirectArgs {
    DirectProduct a, b;            // dL/dQ(a), dL/dQ(b); rows = 0: not asked for
    int blocks_a, blocks_b;
    BwdPlan *plan;                 // for the diagnostic words
    // DIAG: the limb rule's inputs
    unsigned long long *records;   // [gridDim.x][2]
    unsigned long long tag;
    float delta_a, delta_b;
};

// DIAG: leaves in the workspace the limb counts and bounds that the limb products would have had (the documented
// diagnostic words): every block publishes the largest |g| and the largest column sum of |index| it has seen, the last
// block takes the maxima.  Otherwise: that there are none.
template <bool DIAG>
__global__ __launch_bounds__(kDirThreads)
void bwd_direct_kernel(DirectArgs a)
{
    __shared__ double lds[kDirWaves * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool is_a = (int)blockIdx.x < a.blocks_a;
    const DirectProduct &p = is_a ? a.a : a.b;
    int item = is_a ? (int)blockIdx.x : (int)blockIdx.x - a.blocks_a;
    const int tc = item % p.tiles_c;
    item /= p.tiles_c;
    const int tr = item % p.tiles_r, split = item / p.tiles_r;
    const int row0 = (tr * (kDirWaves / p.ksp) + wave / p.ksp) * 16, col0 = tc * (p.narrow ? 16 : 64);
    const int s0 = split * p.steps_per_split, s1 = min(s0 + p.steps_per_split, (p.kc + 15) / 16);
    Diag dg = {0.0f, {0, 0, 0, 0}};
    if (!DIAG && blockIdx.x == 0 && threadIdx.x == 0) no_limbs(a.plan);
    auto product = [&](auto &&src, auto tn_c) {
        constexpr int TN = decltype(tn_c)::value;
        const auto same = [](int row) { return (int64_t)row; };
        const bool alone = p.ksp == 1 && p.splits == 1;
        direct_tile<1, TN, DIAG>(p, src, row0, col0, s0, s1, wave % p.ksp, alone ? nullptr : lds + wave * 256 * TN, dg, same);
        if (alone) return;
        __syncthreads();
        direct_store<1, TN>(p, lds, row0, col0, split, same);
    };
    constexpr auto wide = std::integral_constant<int, 4>{};
    constexpr auto thin = std::integral_constant<int, 1>{};
    if (is_a) { if (p.narrow) product(RowsOfG{}, thin); else product(RowsOfG{}, wide); }
    else { if (p.narrow) product(ColumnsOfGMatrix{}, thin); else product(ColumnsOfGMatrix{}, wide); }

    if (DIAG) {
        // every wave group walks the whole contraction piece of its columns: the column sums of group 0
        int *colabs = reinterpret_cast<int *>(lds);
        unsigned int &amax = reinterpret_cast<unsigned int *>(lds)[64];
        __syncthreads();
        if (threadIdx.x < 64) colabs[threadIdx.x] = 0;
        if (threadIdx.x == 0) amax = 0u;
        __syncthreads();
        const int lane = threadIdx.x & 63;
        atomicMax(&amax, __float_as_uint(dg.amax));
        if (wave / p.ksp == 0)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (!p.narrow || t == 0) atomicAdd(&colabs[(p.narrow ? 1 : 4) * (lane & 15) + t], dg.colabs[t]);
        __syncthreads();
        // (a contraction cut into pieces over blocks is not used together with the diagnostics)
        unsigned int m = threadIdx.x < 64 && col0 + (int)threadIdx.x < p.cols ? (unsigned int)colabs[threadIdx.x & 63] : 0u;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned int)__shfl_xor((int)m, off, 64));
        if (threadIdx.x == 0) {
            const unsigned long long v = ((unsigned long long)amax << 32) | m;
            unsigned long long *r = a.records + 2 * (size_t)blockIdx.x;
            device_store(r, v);
            device_store(r + 1, v ^ a.tag);
        }
        if (blockIdx.x != gridDim.x - 1) return;
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
            if (i < a.blocks_a) sb = max(sb, (unsigned int)v);
            else sa = max(sa, (unsigned int)v);
        }
        unsigned int *red = reinterpret_cast<unsigned int *>(lds) + 65;
        if (threadIdx.x < 3) red[threadIdx.x] = 0u;
        __syncthreads();
        atomicMax(&red[0], gm);
        atomicMax(&red[1], sa);
        atomicMax(&red[2], sb);
        __syncthreads();
        if (threadIdx.x == 0) choose_limbs(a.plan, red[0], red[1], red[2], a.delta_a, a.delta_b);
    }
}

// The weight gradient of a convolution: a product over output pixels whose index operand is the windows.
__global__ __launch_bounds__(kDirThreads)
void conv_dw_direct_kernel(DirectProduct p, ConvPart cv)
{
    __shared__ double lds[kDirWaves * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int item = blockIdx.x;
    const int tc = item % p.tiles_c;
    item /= p.tiles_c;
    const int tr = item % p.tiles_r, split = item / p.tiles_r;
    const int row0 = (tr * (kDirWaves / p.ksp) + wave / p.ksp) * 16, col0 = tc * (p.narrow ? 16 : 64);
    const int s0 = split * p.steps_per_split, s1 = min(s0 + p.steps_per_split, (p.kc + 15) / 16);
    Diag dg = {0.0f, {0, 0, 0, 0}};
    const auto same = [](int row) { return (int64_t)row; };
    ColumnsOfGWindows src;
    src.cv = &cv;
    const uint32_t pad_word = (uint32_t)cv.pad_byte * 0x01010101u;
    if (p.narrow) {
        direct_tile<1, 1, false>(p, src, row0, col0, s0, s1, wave % p.ksp, lds + wave * 256, dg, same, pad_word);
        __syncthreads();
        direct_store<1, 1>(p, lds, row0, col0, split, same);
    } else {
        direct_tile<1, 4, false>(p, src, row0, col0, s0, s1, wave % p.ksp, lds + wave * 1024, dg, same, pad_word);
        __syncthreads();
        direct_store<1, 4>(p, lds, row0, col0, split, same);
    }
}

// The activation gradient of a convolution; one product per class of input pixels.  THIN: few channels, tiles of 64 pixels
// x 16 channels (a tile of 16 x 64 would be padding), else 16 x 64.
struct ConvDxArgs {
    DirectProduct p[4];
    ConvPart cv[4];
    int first[5];          // blocks of class c: first[c] .. first[c + 1]
};

template <bool THIN>
__global__ __launch_bounds__(kDirThreads)
void conv_dx_direct_kernel(ConvDxArgs a)
{
    constexpr int TM = THIN ? 4 : 1, TN = THIN ? 1 : 4;
    __shared__ double lds[kDirWaves * 1024];
    int c = 0;
    while ((int)blockIdx.x >= a.first[c + 1]) ++c;
    const DirectProduct &p = a.p[c];
    const ConvPart &cv = a.cv[c];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), item = (int)blockIdx.x - a.first[c];
    const int tc = item % p.tiles_c, tr = item / p.tiles_c;
    const int row0 = (tr * (kDirWaves / p.ksp) + wave / p.ksp) * 16 * TM, col0 = tc * 16 * TN;
    Diag dg = {0.0f, {0, 0, 0, 0}};
    const auto scattered = [&](int m) {
        const int bb = div_by(m, cv.by_ghw), rem = m - bb * (cv.gh * cv.gw), i = div_by(rem, cv.by_gw), j = rem - i * cv.gw;
        return ((int64_t)bb * cv.H + cv.step * i + cv.oa) * cv.W + cv.step * j + cv.oc;
    };
    GatheredG src;
    src.cv = &cv;
    const bool alone = p.ksp == 1;
    direct_tile<TM, TN, false>(p, src, row0, col0, 0, (p.kc + 15) / 16, wave % p.ksp, alone ? nullptr : lds + wave * 1024, dg, scattered);
    if (alone) return;
    __syncthreads();
    direct_store<TM, TN>(p, lds, row0, col0, 0, scattered);
}

// out[i] = delta * sum over splits of partial[split][i], eight splits side by side per output
__global__ __launch_bounds__(256)
void direct_reduce_kernel(const double *__restrict__ partial, int splits, int64_t n, double delta, float *__restrict__ out)
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
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Splits the work of a product: tiles of 16 x 64 outputs per wave, 16 x 16 where even with eight waves to a tile those would
// leave half of the SIMDs without one; a tile over the waves of a block until there are about two per SIMD; over blocks (max_splits)
// where the contraction is long and the tiles are still few.
void plan_product(DirectProduct &p, int max_splits)
{
    const int64_t steps = ceil_div(p.kc, 16), rows = ceil_div(p.rows, 16);
    p.narrow = rows * ceil_div(p.cols, 64) * (steps < kDirWaves ? steps : kDirWaves) * max_splits < 512;
    p.tiles_c = (int)ceil_div(p.cols, p.narrow ? 16 : 64);
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

}  // namespace

// multiply-adds of one product, counted in whole tiles
static double padded_macs(int64_t rows, int64_t kc, int64_t cols) { return (double)(ceil_div(rows, 16) * 16) * (double)(ceil_div(kc, 16) * 16) * (double)(ceil_div(cols, 64) * 64); }

// Where the products are formed directly: both products, against the limb path with its helpers (us):
//   32 x 128 x 256          36 ->  4      1988 x 225 x  752 (0.34 G multiply-adds each)  63 ->  44
//   256 x 1000 x 512        45 -> 18      2000 x 300 x 1000 (0.6 G)                      70 ->  67
//   131072 x 16 x 144, dL/dQ(b) 43 -> 26  1000 x 1000 x 1000 (1 G)                       65 ->  88
// so up to 0.7 G multiply-adds in whole tiles, both products together.
// Up to kBwdDirectNoDiag the diagnostic words say that neither product has limbs.
constexpr int64_t kBwdDirectNoDiag = 1ll << 25;
constexpr double kBwdDirectMaxMacs = 7e8, kConvDwDirectMaxMacs = 5e8, kConvDxDirectMaxMacs = 5e8;

static bool bwd_direct_diag(int32_t M, int32_t N, int32_t K) { return N > 32 && (int64_t)M * N * K > kBwdDirectNoDiag; }

bool bwd_direct_serves(int32_t M, int32_t N, int32_t K, bool want_a, bool want_b)
{
    const double work = (want_a ? padded_macs(M, N, K) : 0.0) + (want_b ? padded_macs(N, M, K) : 0.0);
    if (K < 4 || work > kBwdDirectMaxMacs) return false;
    // (with the diagnostics a contraction is not cut into pieces: no longer than 40 steps per wave)
    return !bwd_direct_diag(M, N, K) || (M <= 5120 && N <= 5120);
}

int launch_bwd_direct(const float *g, const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float delta_a, float delta_b,
                      int32_t a_offset, int32_t b_offset, float *d_a_hat, float *d_b_hat, BwdPlan *plan, void *records, double *partial, int max_splits,
                      hipStream_t stream)
{
    DirectArgs a{};
    const bool diag = bwd_direct_diag(M, N, K);
    a.plan = plan;
    a.records = reinterpret_cast<unsigned long long *>(records);
    a.delta_a = delta_a; a.delta_b = delta_b;
    if (d_a_hat) {
        DirectProduct &p = a.a;
        p.g = g; p.idx = b_idx; p.rows = M; p.cols = K; p.kc = N; p.ldg = N; p.ldi = K;
        p.offset = b_offset; p.vec = N % 4 == 0; p.delta = (double)delta_b; p.out = d_a_hat;
        plan_product(p, 1);
        a.blocks_a = p.tiles_r * p.tiles_c;
    }
    if (d_b_hat) {
        DirectProduct &p = a.b;
        p.g = g; p.idx = a_idx; p.rows = N; p.cols = K; p.kc = M; p.ldg = N; p.ldi = K;
        p.offset = a_offset; p.delta = (double)delta_a; p.out = d_b_hat; p.partial = partial;
        plan_product(p, diag ? 1 : max_splits);
        a.blocks_b = p.tiles_r * p.tiles_c * p.splits;
    }
    const unsigned grid = (unsigned)(a.blocks_a + a.blocks_b);
    if (diag) {
        a.tag = next_finish_tag();
        CDL_LAUNCH("bwd_direct_kernel", stream, bwd_direct_kernel<true>, dim3(grid), dim3(kDirThreads), 0, a);
    } else {
        CDL_LAUNCH("bwd_direct_kernel", stream, bwd_direct_kernel<false>, dim3(grid), dim3(kDirThreads), 0, a);
    }
    int rc = check_launch();
    if (rc == CDL_OK && a.b.splits > 1) {
        const int64_t n = (int64_t)N * K;
        CDL_LAUNCH("direct_reduce_kernel", stream, direct_reduce_kernel, dim3((unsigned)ceil_div(n, 32)), dim3(256), 0, partial, a.b.splits, n,
                   (double)delta_a, d_b_hat);
        rc = check_launch();
    }
    return rc;
}

bool conv_dw_direct_serves(int64_t M, int32_t N, int32_t K) { return padded_macs(N, M, K) <= kConvDwDirectMaxMacs; }

int launch_conv_dw_direct(const float *g, const int8_t *x_idx, const ConvWindows &w, int32_t N, float delta_x, int32_t x_offset, float *d_w_hat,
                          double *partial, int max_splits, hipStream_t stream)
{
    DirectProduct p{};
    p.g = g; p.idx = x_idx; p.rows = N; p.cols = w.R * w.S * w.C; p.kc = w.B * w.P * w.Q; p.ldg = N;
    p.offset = x_offset; p.delta = (double)delta_x; p.out = d_w_hat; p.partial = partial;
    plan_product(p, max_splits);
    ConvPart cv{};
    cv.H = w.H; cv.W = w.W; cv.C = w.C; cv.S = w.S; cv.stride = w.stride; cv.pad = w.pad; cv.P = w.P; cv.Q = w.Q;
    cv.pad_byte = (int)(uint8_t)(int8_t)(-x_offset);
    cv.by_pq = make_div_by((uint32_t)(w.P * w.Q));
    cv.by_q = make_div_by((uint32_t)w.Q);
    CDL_LAUNCH("conv_dw_direct_kernel", stream, conv_dw_direct_kernel, dim3((unsigned)(p.tiles_r * p.tiles_c * p.splits)), dim3(kDirThreads), 0, p, cv);
    int rc = check_launch();
    if (rc == CDL_OK && p.splits > 1) {
        const int64_t n = (int64_t)p.rows * p.cols;
        CDL_LAUNCH("direct_reduce_kernel", stream, direct_reduce_kernel, dim3((unsigned)ceil_div(n, 32)), dim3(256), 0, partial, p.splits, n, p.delta, d_w_hat);
        rc = check_launch();
    }
    return rc;
}

static bool conv_dx_thin(int32_t C) { return C <= 48; }

bool conv_dx_direct_serves(int64_t pixels, int32_t N, int32_t C, int32_t R, int32_t S, int32_t stride)
{
    if (C <= 32 && (int64_t)R * S * N <= 288) return true;      // (any number of pixels: most of a limb tile would be padding)
    const double cols = conv_dx_thin(C) ? ceil_div(C, 16) * 16 : ceil_div(C, 64) * 64;
    return (double)pixels * cols * (double)(ceil_div((int64_t)R * S * N, 16) * 16) / (stride * stride) <= kConvDxDirectMaxMacs;
}

int launch_conv_dx_direct(const float *g, const int8_t *w_idx, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                          int32_t R, int32_t S, int32_t P, int32_t Q, int32_t stride, float delta_w, float *d_x_hat, hipStream_t stream)
{
    const bool thin = conv_dx_thin(C);
    ConvDxArgs a{};
    int blocks = 0;
    for (int c = 0; c < n_grids; ++c) {
        const ConvDxGrid &k = grids[c];
        DirectProduct &p = a.p[c];
        p.g = g; p.idx = w_idx; p.rows = B * k.Hc * k.Wc; p.cols = C; p.kc = k.Rc * k.Sc * N;
        p.delta = (double)delta_w; p.out = d_x_hat; p.splits = 1;
        const int64_t steps = ceil_div(p.kc, 16), rows = ceil_div(p.rows, thin ? 64 : 16);
        p.tiles_c = (int)ceil_div(C, thin ? 16 : 64);
        p.ksp = 1;
        while (p.ksp < kDirWaves && 2 * p.ksp <= steps && rows * p.tiles_c * p.ksp < 2048) p.ksp *= 2;
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
    if (thin) CDL_LAUNCH("conv_dx_direct_kernel", stream, conv_dx_direct_kernel<true>, dim3((unsigned)blocks), dim3(kDirThreads), 0, a);
    else CDL_LAUNCH("conv_dx_direct_kernel", stream, conv_dx_direct_kernel<false>, dim3((unsigned)blocks), dim3(kDirThreads), 0, a);
    return check_launch();
}

}  // namespace cdl
