// dL/dQ(x) of a convolutional layer on limbs, from patches of g that stay in LDS: d_x_hat[b,h,w,c] = delta_w sum_{r,s,n}
// g[b,p,q,n] w[n,r,s,c] over the taps that reach pixel (h, w), without a matrix of windows.
//
// The pixels of g that a run of output pixels needs are one contiguous range of g, [lo, lo + count) x N, of about the run's length
// and R - 1 image rows.  A block takes such a range, scales its digits by the range's largest entry, and writes them into LDS once,
// one byte per limb and entry; every tap then reads its fragments there, row by row at an offset that depends on the tap.  The limb
// count is that of the whole tensor, so no output is further from the exact sum than with one scale for all of g: the launch that rearranges the weights
// also takes, in a pass over g beside that, the largest entry of every pixel and of every block of the pass, and the columns' sums of |w|.
// g is read from memory once more, or found in the last-level cache, about once per 256 channels.
// The weights' fragments go from L2 straight to registers: a wave's columns are its own, LDS would be written and read for one use.
//
// What bounds it: the matrix cores while both blocks of a compute unit are in their k-steps (pipes 55 % busy over the whole kernel at 14 x 14 x 256; LDS
// and the vector cache at half their rates); the rest of a block - digits 5 us, outputs 3 of 30 - hides only behind the other block.
// Stride 2: 18 %, digits of 62 pixels for 32 of the grid, and waves of one to four taps.  (The largest entry taken by every block from g itself, with no
// pass before, and a limb count of its own: 87 - 87, 97 - 89, 130 - 129 us the call at 28 x 28 x 128, stride 2, 14 x 14 x 256.)  Before, a pass
// that made the digits ran first and the product read them tap by tap through L2 into LDS, where
// reads and writes together took longer than the matrix instructions.  The whole call, us, with uniform indices: 256 images of
// 14 x 14 x 256 -> 256, 3 x 3  216 -> 149;  128 x 28 x 28 x 128 -> 128  123 -> 94;  128 x 7 x 7 x 512 -> 512  139 -> 82;
// 128 x 56 x 56 x 64 -> 128, stride 2  119 -> 88.
#include "cdl_bwd_plan.h"
#include "cdl_limbs.h"

#include <type_traits>

namespace cdl {

namespace {

struct PatchClass {
    int oa, oc, Hc, Wc, pad_h, pad_w, Rc, Sc;
    const int8_t *wr;
    DivBy by_s;
};

// The classes of output pixels (one; stride 2: up to four) share a grid of Hm x Wm pixels an image, the smaller ones with pixels that
// are not there; grid pixel (i, j) reads g at rows i + lo_h .. i + hi_h and columns j + lo_w .. j + hi_w, over all classes.
struct PatchArgs {
    PatchClass c[4];
    int n_classes;
    const float *g;
    float *out;
    int N, Np, C, C32, P, Q, oH, oW, step, tiles_c, share, pixels;      // C32: C padded to 32; share: row tiles of an XCD; pixels: of g
    int Hm, Wm, rows, row_tiles, lo_h, hi_h, lo_w, hi_w;
    DivBy by_hw, by_w;
    int px_max;                              // pixels of a patch, at most
    int nc[kMaxLimbs + 1];                   // channels of a patch that fit, by limbs
    int taps;                                // of a class, at most
    PatchMaxima maxima;
    double delta_w;
};
// (read where the launch put them: indexing a by-value argument by the class would copy it to scratch memory)
typedef const PatchArgs __attribute__((address_space(4))) *patch_args_t;

struct PatchTile { int row0, col0, lo, count; };

template <int L, int WN>
__device__ __forceinline__ void patch_body(patch_args_t args, const PatchTile t, int8_t *lds, double out_scale, float gscale, bool few)
{
    constexpr int TN = 2, ROWS = patch_rows(WN);
    // The digits and the outputs go before the other block's matrix instructions, which leave issue slots enough: 53 x 19 x 53 x 288 -> 412, 3 x 3 359 -> 353 us, 26 x 55 x 55 x 48 -> 468 170 -> 164.
    // (A block's k-steps before the other's: 5 - 15 % slower.  Four classes: 97 -> 99.)
    if (WN != 0) __builtin_amdgcn_s_setprio(2);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));      // (what the limb counts' code has in common is not moved in front of all of it, where registers are short)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = WN == 0 ? 0 : wave / (WN ? WN : 1), wn = WN == 0 ? 0 : wave % (WN ? WN : 1), cls = WN == 0 ? wave : 0;
    const bool idle = WN == 0 && cls >= args->n_classes;
    const auto &k = args->c[idle ? 0 : cls];
    const int P = args->P, Q = args->Q, Np = args->Np, N = args->N, C = args->C, Wm = args->Wm, hw = args->Hm * Wm, rows = args->rows, Sc = k.Sc, taps = k.Rc * Sc;
    const DivBy by_hw{args->by_hw.mul, args->by_hw.sh}, by_w{args->by_w.mul, args->by_w.sh};
    // (rows an odd multiple of 16 bytes apart: conflicts only where lanes read the row of zeros or pixels that do not follow each other, 0.28 of the
    // LDS cycles at 14 x 14 x 256, 0.07 at stride 2)
    const int nc = args->nc[L], stride = nc + 16, px_max = args->px_max;
    const int plane = (px_max + 1) * stride;                                  // (row px_max of a plane: zeros)
    // [class][taps + 1][ROWS]: the row of a plane where a tap's pixel lies
    uint16_t *table = reinterpret_cast<uint16_t *>(lds + kPatchFixed) + (idle ? 0 : cls) * (args->taps + 1) * ROWS;
    int8_t *planes = lds + kPatchFixed + 2 * (WN == 0 ? args->n_classes : 1) * (args->taps + 1) * ROWS;

    for (int i = tid; i < L * (stride / 4); i += kPatchThreads) {
        const int l = i / (stride / 4), w = i - l * (stride / 4);
        reinterpret_cast<uint32_t *>(planes + l * plane + px_max * stride)[w] = 0u;
    }
    // digits of channels n0 .. n0 + nc of the patch: a thread keeps its four channels and goes through the pixels
    const int words = nc >> 2, px_step = kPatchThreads / words;      // (plan_patch: words <= kPatchThreads)
    const int px0 = tid / words, n_own = 4 * (tid - px0 * words);
    auto make_digits = [&](int n0) {
        if (px0 >= px_step) return;
        const bool there = n0 + n_own < N;
        const float *src = args->g + (int64_t)t.lo * N + (there ? n0 + n_own : 0);
        constexpr int U = 8;
        // (behind the last pixel: the last one again, with what its own thread writes; count N and count stride < 2^22)
        const int src_step = px_step * N, src_last = (t.count - 1) * N, dst_step = px_step * stride, dst_last = (t.count - 1) * stride;
        int from = px0 * N, to = px0 * stride;
        for (int px = px0; px < t.count; px += U * px_step) {
            float4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4 *>(src + min(from + u * src_step, src_last));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float g4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                uint32_t w[L];
                limbs_of4<L>(g4, gscale, w);
                if (!there)
#pragma unroll
                    for (int l = 0; l < L; ++l) w[l] = 0u;
                int8_t *d = planes + min(to + u * dst_step, dst_last) + n_own;
#pragma unroll
                for (int l = 0; l < L; ++l) *reinterpret_cast<uint32_t *>(d + l * plane) = w[l];
            }
            from += U * src_step;
            to += U * dst_step;
        }
    };
    // weights: 1 KB a k-step of 32 entries and tile of 32 columns, in the order of the lanes
    uint32_t bo[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bo[j] = (uint32_t)min((t.col0 >> 5) + wn * TN + j, (args->C32 >> 5) - 1) * 1024u + (uint32_t)lane * 16u;
    const int half = (lane >> 5) * 16;
    constexpr int NA = L <= 5 ? 2 : 1, NB = patch_ahead(L);
    v4i fb[NB][TN];
    const int nk = idle ? 0 : taps * (nc / 32);
    PatchWeights weights(0, nc, Np, args->C32, nk);
    auto load_b = [&](int buf) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[buf][j] = *reinterpret_cast<const v4i *>(k.wr + weights.at + bo[j]);
        weights.next();
    };
    // (the first ones on their way while the digits are made: 128 x 7 x 7 x 512 -> 512 82.6 -> 80.7 us, 41 x 51 x 49 x 128 -> 20 51.7 -> 48.7)
#pragma unroll
    for (int u = 0; u < NB; ++u) load_b(u);
    if (nc == Np) make_digits(0);      // all channels at once, for all classes

    // (WN = 0: a wave makes its own table)
    for (int i = WN == 0 ? lane : tid; i < (idle ? 0 : taps + 1) * ROWS; i += WN == 0 ? 64 : kPatchThreads) {
        const int tap = i / ROWS, row = i - tap * ROWS, m = t.row0 + row;
        const int b = div_by(m, by_hw), rem = m - b * hw, ii = div_by(rem, by_w), jj = rem - ii * Wm;
        const int tr = div_by(tap, k.by_s.mul, k.by_s.sh), ts = tap - tr * Sc;
        const int p = ii + k.pad_h - tr, q = jj + k.pad_w - ts;
        const bool inside = tap < taps && m < rows && (unsigned)p < (unsigned)P && (unsigned)q < (unsigned)Q;
        const int px = (b * P + p) * Q + q - t.lo;
        table[i] = (uint16_t)(inside ? min(max(px, 0), px_max - 1) : px_max);
    }
    v16i acc[L][TN];
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[l][j][r] = 0;
    const int arow = wm * 32 + (lane & 31);

    for (int n0 = 0; n0 < Np; n0 += nc) {
        if (n0 > 0) {
            weights = PatchWeights(n0, nc, Np, args->C32, nk);
#pragma unroll
            for (int u = 0; u < NB; ++u) load_b(u);
            __syncthreads();
        }
        if (nc < Np) make_digits(n0);
        __syncthreads();

        // k-steps of 32 entries, tap after tap.  The weights of a step are asked for four steps ahead, the row of LDS two, the digits
        // one (more than four limbs leave registers for less).
        v4i fa[NA][L];
        int row[2], at[2];      // a lane's row of a plane, and the step's first channel (put together where they are used: no wait for the table before)
        int rt = 0, rn = 0;
        auto load_row = [&](int buf) {
            row[buf] = table[rt * ROWS + arow];
            at[buf] = rn;
            rn += 32;
            rt = min(rn == nc ? rt + 1 : rt, taps);
            rn = rn == nc ? 0 : rn;
        };
        auto load_a = [&](int buf, int rbuf) {
            const int8_t *p = planes + (row[rbuf] * stride + (at[rbuf] + half));
#pragma unroll
            for (int l = 0; l < L; ++l) fa[buf][l] = *reinterpret_cast<const v4i *>(p + l * plane);
        };
        auto mfma_all = [&](int abuf, int bbuf) {
#pragma unroll
            for (int l = 0; l < L; ++l)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[l][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[abuf][l], fb[bbuf][j], acc[l][j], 0, 0, 0);
        };
        load_row(0);
        load_row(1);
        if (NA == 2) load_a(0, 0);
        // (a step behind the last one multiplies rows of zeros)
        if (WN != 0) __builtin_amdgcn_s_setprio(0);
        for (int it = 0; it < nk; it += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (u == 2 && it + 2 >= nk) break;
                if (NA == 2) load_a((u + 1) & 1, (u + 1) & 1);
                else load_a(0, u & 1);
                load_row(u & 1);
                mfma_all(NA == 2 ? u & 1 : 0, u % NB);
                load_b(u % NB);
#pragma unroll
                for (int i = 0; i < L * TN; ++i) {      // behind each matrix instruction a part of the rest
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x006, 5, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (WN != 0) __builtin_amdgcn_s_setprio(2);
    }

    if (idle) return;
    // the limbs of an output: the integers are exact, the Horner steps round at 2^-53 relative
    int elane = lane;
    asm volatile("" : "+v"(elane));      // (addresses formed here, not kept in registers through the loop)
    const int m = t.row0 + wm * 32 + (elane & 31);
    const int b = div_by(m, by_hw), rem = m - b * hw, i = div_by(rem, by_w), jj = rem - i * Wm;
    const int pixel = m < rows && i < k.Hc && jj < k.Wc ? (b * args->oH + args->step * i + k.oa) * args->oW + args->step * jj + k.oc : -1;
    float *out = args->out;
    const int ecol = t.col0 + wn * TN * 32 + (elane & 31);
    auto outputs = [&](auto pairs) {
#pragma unroll
        for (int rr = 0; rr < 16; ++rr) {
            const int pix = __shfl(pixel, 4 * (elane >> 5) + 8 * (rr >> 2) + (rr & 3), 64);      // (layout of an accumulator)
            float *p = out + (int64_t)pix * C + ecol;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                double run;
                if (L == 4 && pairs.value) {
                    run = __builtin_fma((double)(256 * acc[L - 1][j][rr] + acc[L - 2][j][rr]), 65536.0, (double)(256 * acc[1][j][rr] + acc[0][j][rr]));
                } else {
                    run = (double)acc[L - 1][j][rr];
#pragma unroll
                    for (int l = L - 2; l >= 0; --l) run = __builtin_fma(run, 256.0, (double)acc[l][j][rr]);
                }
                if (pix >= 0 && ecol + j * 32 < C) p[j * 32] = (float)(run * out_scale);
            }
        }
    };
    // (two limbs as one integer: five instructions in double instead of nine.  Not with four classes, whose blocks then all store at a time: 128 x 56 x 56 x 64 -> 128 at stride 2
    // 95.4 us so, 98.6 with pairs)
    if (WN != 0 && L == 4 && few) outputs(std::true_type{});
    else outputs(std::false_type{});
}

template <int WN>
__global__ __launch_bounds__(kPatchThreads, 2)
void limb_conv_patch_kernel(PatchArgs a)
{
    constexpr int ROWS = patch_rows(WN), COLS = patch_cols(WN);
    extern __shared__ __attribute__((aligned(16))) int8_t patch_lds[];
    const patch_args_t args = (patch_args_t)__builtin_amdgcn_kernarg_segment_ptr();
    // Blocks go to the eight XCDs round-robin; XCD x takes the x-th eighth of the row tiles, all columns of one after the
    // other (they read the same g through one L2).
    const int xcd = (int)blockIdx.x & 7, q = (int)blockIdx.x >> 3, r = q / args->tiles_c;
    PatchTile t;
    t.col0 = (q - r * args->tiles_c) * COLS;
    const int tile = xcd * args->share + r;
    if (r >= args->share || tile >= args->row_tiles) return;
    t.row0 = tile * ROWS;
    // the range of g
    {
        const int m1 = min(t.row0 + ROWS, args->rows) - 1, Wm = args->Wm, hw = args->Hm * Wm, P = args->P, Q = args->Q;
        const DivBy by_hw{args->by_hw.mul, args->by_hw.sh}, by_w{args->by_w.mul, args->by_w.sh};
        const int b0 = div_by(t.row0, by_hw), rem0 = t.row0 - b0 * hw, i0 = div_by(rem0, by_w), j0 = rem0 - i0 * Wm;
        const int b1 = div_by(m1, by_hw), rem1 = m1 - b1 * hw, i1 = div_by(rem1, by_w), j1 = rem1 - i1 * Wm;
        const int p0 = i0 + args->lo_h, q0 = j0 + args->lo_w, p1 = i1 + args->hi_h, q1 = j1 + args->hi_w;
        // (above the image: from its first pixel on; below it: to its last one)
        const int lo = (b0 * P + min(max(p0, 0), P - 1)) * Q + (p0 < 0 ? 0 : min(max(q0, 0), Q - 1));
        const int hi = (b1 * P + min(max(p1, 0), P - 1)) * Q + (p1 > P - 1 ? Q - 1 : min(max(q1, 0), Q - 1));
        t.lo = __builtin_amdgcn_readfirstlane(lo);
        t.count = __builtin_amdgcn_readfirstlane(min(max(hi - lo + 1, 1), min(args->px_max, args->pixels - lo)));
    }
    // largest |g| of the range and of all (an infinity or a NaN is larger than any number), largest sum of |w| of a column.  Every block takes the
    // maxima by itself, in the trip to memory for its pixels' (by the last block of the launch before: 4 us).
    unsigned int *red = reinterpret_cast<unsigned int *>(patch_lds);
    {
        const unsigned int *block_max = args->maxima.block_max;
        const int n_max = args->maxima.n_max, n_abs = args->maxima.n_abs;
        unsigned int v[3] = {0u, 0u, 0u};
        // (the first of each, which are all for most layers, in one trip)
        const unsigned int *pixel_max = args->maxima.pixel_max + t.lo, *col_abs = args->maxima.col_abs;
        v[0] = pixel_max[min((int)threadIdx.x, t.count - 1)];
        v[2] = col_abs[min((int)threadIdx.x, n_abs - 1)];
#pragma unroll
        for (int u = 0; u < kPatchMaxima / kPatchThreads; ++u) v[1] = max(v[1], block_max[min(u * kPatchThreads + (int)threadIdx.x, n_max - 1)]);
        for (int i = kPatchThreads + threadIdx.x; i < n_abs; i += kPatchThreads) v[2] = max(v[2], col_abs[i]);
        for (int i = kPatchThreads + threadIdx.x; i < t.count; i += kPatchThreads) v[0] = max(v[0], pixel_max[i]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v[k] = max(v[k], (unsigned int)__shfl_xor((int)v[k], off, 64));
            if ((threadIdx.x & 63) == 0) red[4 * k + (threadIdx.x >> 6)] = v[k];
        }
    }
    __syncthreads();
    auto maximum = [&](int k) { return max(max(red[4 * k], red[4 * k + 1]), max(red[4 * k + 2], red[4 * k + 3])); };
    const unsigned int amax_bits = maximum(0), all_bits = maximum(1), inf_bits = 0x7f800000u;
    const float amax = __uint_as_float(amax_bits), all = __uint_as_float(all_bits);
    // The fewest limbs, four to six, whose bound for the whole tensor, delta_w sigma 2^-8L sum|w| with sigma = 2^e > 1.01 max|g|, is under the
    // target (choose_limbs; six with an infinity or a NaN), and the scale of the range
    int e_all = 0;
    if (all > 0.0f) frexpf(all * 1.01f, &e_all);
    e_all = max(min(e_all, 127), -80);
    const double unit = args->delta_w * (double)maximum(2);
    int L = all_bits < inf_bits ? kPatchMinLimbs : kMaxLimbs;
    while (L < kMaxLimbs && unit * ldexp(1.0, e_all - 8 * L) > kLimbBoundTarget) ++L;
    L = __builtin_amdgcn_readfirstlane(L);
    int e = 0;
    if (amax > 0.0f) frexpf(amax * 1.01f, &e);
    e = __builtin_amdgcn_readfirstlane(max(min(e, 127), -80));
    // (an infinity or a NaN in the range: NaN for the tile)
    const bool finite = amax_bits < inf_bits;
    // (in scalar registers: kept in memory, their loads among the stores of the outputs would wait for every store before them)
    const long long scale_bits = finite ? __double_as_longlong(args->delta_w * ldexp(1.0, e + 1 - 8 * L)) : 0x7ff8000000000000ll;
    const double out_scale = __hiloint2double(__builtin_amdgcn_readfirstlane((int)(scale_bits >> 32)), __builtin_amdgcn_readfirstlane((int)scale_bits));
    const float gscale = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ldexpf(1.0f, 8 * L - 1 - e))));
    // a limb of an output is 128 sum|w| at most: two of them as one integer, 257 times that
    const bool few = maximum(2) < 65024u;
    switch (L) {
        case 4: patch_body<4, WN>(args, t, patch_lds, out_scale, gscale, few); break;
        case 5: patch_body<5, WN>(args, t, patch_lds, out_scale, gscale, few); break;
        default: patch_body<6, WN>(args, t, patch_lds, out_scale, gscale, few); break;
    }
}

template <int WN>
int launch_patch(PatchArgs a, hipStream_t stream)
{
    constexpr int ROWS = patch_rows(WN), COLS = patch_cols(WN);
    a.tiles_c = (a.C + COLS - 1) / COLS;
    a.row_tiles = (a.rows + ROWS - 1) / ROWS;
    a.share = (a.row_tiles + 7) / 8;
    const int64_t blocks = 8ll * a.share * a.tiles_c;
    if (blocks > 2147483647LL) return CDL_ERR_PARAM;
    const hipError_t e = hipFuncSetAttribute((const void *)limb_conv_patch_kernel<WN>, hipFuncAttributeMaxDynamicSharedMemorySize, kPatchLds);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("limb_conv_patch_kernel", stream, (limb_conv_patch_kernel<WN>), dim3((unsigned)blocks), dim3(kPatchThreads), kPatchLds, a);
    return check_launch();
}

}  // namespace

bool conv_dx_patch_serves(const ConvDxGrid *grids, int n_grids, int32_t B, int32_t C, int32_t N, int32_t P, int32_t Q)
{
    return plan_patch(grids, n_grids, B, P, Q, C, (N + 31) / 32 * 32).served;
}

int launch_conv_dx_patch(const float *g, const int8_t *wr, const PatchMaxima &maxima, int64_t ld, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H,
                         int32_t W, int32_t C, int32_t N, int32_t Np, int32_t P, int32_t Q, int32_t stride, float delta_w, float *d_x_hat, hipStream_t stream)
{
    const PatchPlan p = plan_patch(grids, n_grids, B, P, Q, C, Np);
    const PatchGrid grid = patch_grid(grids, n_grids);
    PatchArgs a{};
    a.n_classes = n_grids;
    a.g = g; a.out = d_x_hat;
    a.N = N; a.Np = Np; a.C = C; a.C32 = (C + 31) / 32 * 32; a.P = P; a.Q = Q; a.oH = H; a.oW = W; a.step = stride;
    a.pixels = B * P * Q;
    a.Hm = grid.Hm; a.Wm = grid.Wm; a.rows = B * grid.Hm * grid.Wm;
    a.lo_h = grid.lo_h; a.hi_h = grid.hi_h; a.lo_w = grid.lo_w; a.hi_w = grid.hi_w;
    a.by_hw = make_div_by((uint32_t)grid.Hm * (uint32_t)grid.Wm);
    a.by_w = make_div_by((uint32_t)grid.Wm);
    a.px_max = p.px_max; a.taps = p.taps;
    for (int l = kPatchMinLimbs; l <= kMaxLimbs; ++l) a.nc[l] = p.nc[l];
    a.maxima = maxima;
    a.delta_w = (double)delta_w;
    for (int i = 0; i < n_grids; ++i) {
        const ConvDxGrid &s = grids[i];
        PatchClass &d = a.c[i];
        d.oa = s.oa; d.oc = s.oc; d.Hc = s.Hc; d.Wc = s.Wc; d.pad_h = s.pad_h; d.pad_w = s.pad_w; d.Rc = s.Rc; d.Sc = s.Sc;
        d.wr = wr + (int64_t)i * a.C32 * ld;
        d.by_s = make_div_by((uint32_t)s.Sc);
    }
    if (p.wn == 0) return launch_patch<0>(a, stream);
    if (p.wn == 4) return launch_patch<4>(a, stream);
    if (p.wn == 2) return launch_patch<2>(a, stream);
    return launch_patch<1>(a, stream);
}

}  // namespace cdl
