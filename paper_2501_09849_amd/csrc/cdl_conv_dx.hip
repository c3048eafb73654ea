// dL/dQ(x) of a convolutional layer on limbs: d_x_hat[b,h,w,c] = delta_w sum_{r,s,n} g[b,p,q,n] w[n,r,s,c] over the taps
// that reach pixel (h, w), without a matrix of windows.
//
// g is read by every tap (nine times for 3 x 3) and by every tile of channels, and its digits (see limbs_of4) cost more
// instructions than the matrix cores take for them when few channels share them.  So the digits are made once, into
// planes[pixel][channels / 64][limb][64] (a pass over g of 4 bytes read and one byte per limb written for each entry), and the product is an int8 product with
// L left operands and one right one: the planes come into LDS by direct loads, 16-byte chunks each inside one tap, the
// chunks of taps outside the image from a page of zeros.  (K-tiles are 64 bytes, half a cache line: the limbs of 64 channels
// lie side by side, and the weights K-tile by K-tile, so that a K-tile takes whole lines.)
//
// Stride 2: input pixel (h, w) is reached only by the taps r = h + pad, s = w + pad (mod 2), so the pixels of each of the
// four parities form a product of their own; all of them share one launch, the blocks numbered class after class.
#include "cdl_bwd_plan.h"
#include "cdl_limbs.h"

#include <type_traits>

namespace cdl {

namespace {

constexpr int kDxThreads = 256;
constexpr int kDxLds = 80 << 10;        // two blocks share a compute unit and fill each other's waits

struct DxClass {
    int oa, oc, Hc, Wc, pad_h, pad_w, Rc, Sc;
    int rows, tiles;                    // output rows, tiles
    const int8_t *wr;
    float inv_s;                        // 1 / Sc
    DivBy by_hw, by_w;
};

struct DxArgs {
    DxClass c[4];
    int n_classes;
    const int8_t *planes, *zeros;
    int Np, C, P, Q, oH, oW, step, tiles_c;
    float inv_np;                       // 1 / Np
    const BwdPlan *plan;
    float *out;
};

// ---- digits of g ----
constexpr int kPlaneUnroll = 4;
template <int L>
__device__ __forceinline__ void planes_body(const float *__restrict__ g, int64_t words, int N, int Np, float gscale, int8_t *__restrict__ planes)
{
    // a word: four consecutive channels of one pixel
    const int wn = Np >> 2;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < words; i0 += kPlaneUnroll * stride) {
        float4 v[kPlaneUnroll];
        int64_t row[kPlaneUnroll];
        int n[kPlaneUnroll];
#pragma unroll
        for (int u = 0; u < kPlaneUnroll; ++u) {
            const int64_t i = i0 + u * stride < words ? i0 + u * stride : words - 1;
            row[u] = (int64_t)((uint64_t)i / (uint32_t)wn);
            n[u] = 4 * (int)(i - row[u] * wn);
            v[u] = n[u] < N ? *reinterpret_cast<const float4 *>(g + row[u] * N + n[u]) : float4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int u = 0; u < kPlaneUnroll; ++u) {
            const float g4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            uint32_t w[L];
            limbs_of4<L>(g4, gscale, w);
            const int first = n[u] & ~63, width = min(64, Np - first);
            int8_t *d = planes + row[u] * ((int64_t)L * Np) + L * first + (n[u] & 63);
#pragma unroll
            for (int l = 0; l < L; ++l) *reinterpret_cast<uint32_t *>(d + l * width) = w[l];
        }
    }
}

__global__ __launch_bounds__(256)
void g_planes_kernel(const float *__restrict__ g, int64_t words, int N, int Np, const BwdPlan *__restrict__ plan, int8_t *__restrict__ planes)
{
    const float gscale = plan->gscale_da;
    switch (plan->limbs_da) {
        case 3: planes_body<3>(g, words, N, Np, gscale, planes); break;
        case 4: planes_body<4>(g, words, N, Np, gscale, planes); break;
        case 5: planes_body<5>(g, words, N, Np, gscale, planes); break;
        default: planes_body<6>(g, words, N, Np, gscale, planes); break;
    }
}

// ---- the product ----
// (read where the launch put them: indexing a by-value argument by the class would copy it to scratch memory)
typedef const DxArgs __attribute__((address_space(4))) *dx_args_t;

// Four waves as (4 / WN) x WN, a wave 32 pixels by TN tiles of 32 channels by L limbs; K-tiles of KT bytes.
template <int WN, int TN>
struct DxTile {
    static constexpr int kRows = 32 * (4 / WN), kCols = 32 * WN * TN;
};
template <int L, int WN, int TN>
constexpr int dx_kt() { return L > 4 && WN == 1 ? 32 : 64; }      // (so that two stages fit kDxLds)
template <int L, int WN, int TN>
constexpr int dx_stage() { return (L * DxTile<WN, TN>::kRows + DxTile<WN, TN>::kCols) * dx_kt<L, WN, TN>(); }

template <int L, int WN, int TN>
__device__ __forceinline__ void conv_dx_body(dx_args_t args, int8_t *lds, double out_scale)
{
    constexpr int ROWS = DxTile<WN, TN>::kRows, COLS = DxTile<WN, TN>::kCols, KT = dx_kt<L, WN, TN>(), STAGE = dx_stage<L, WN, TN>();
    constexpr int NS = kDxLds / STAGE >= 4 ? 4 : kDxLds / STAGE;
    static_assert(NS >= 2, "two stages");
    constexpr int CH = KT / 16, LINE = 8 / CH;              // chunks of a row; rows of a 128-byte line
    constexpr int NR = ROWS * CH / kDxThreads > 0 ? ROWS * CH / kDxThreads : 1;      // rows of a plane a thread loads a chunk of
    constexpr int NB = COLS * CH / kDxThreads > 0 ? COLS * CH / kDxThreads : 1;
    constexpr int LOADS = L * NR + NB;                      // direct loads of a thread for one K-tile
    // a row's chunk q lies at chunk q ^ swz(row): the rows of a fragment read then take all banks of their lines
    auto swz = [](int row) { return (row / LINE) & (CH - 1); };

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // Tiles.  Blocks go to the eight XCDs round-robin; XCD x takes the x-th eighth of every class's tiles (so that the rows that
    // neighbouring tiles share are read through one L2), class after class, block `slot` of it every slots-th.
    struct Tile { int q, cls, row0, col0, nk; };
    const int xcd = (int)blockIdx.x & 7, slot_x = (int)blockIdx.x >> 3, slots = (int)gridDim.x >> 3;
    auto tile_at = [&](int q) {
        Tile t{q, 0, 0, 0, 0};
        int r = q;
        for (int c = 0; c < args->n_classes; ++c) {
            const int share = (args->c[c].tiles + 7) >> 3, mine = min(max(args->c[c].tiles - xcd * share, 0), share);
            if (r < mine) {
                const int at = xcd * share + r, tr = (int)((uint32_t)at / (uint32_t)args->tiles_c);
                t.cls = c;
                t.row0 = tr * ROWS;
                t.col0 = (at - tr * args->tiles_c) * COLS;
                t.nk = (args->c[c].Rc * args->c[c].Sc * args->Np + KT - 1) / KT;
                return t;
            }
            r -= mine;
        }
        return t;      // nk = 0: no such tile
    };
    Tile now = tile_at(slot_x);
    if (now.nk == 0) return;

    // ---- loads: the tile and K-tile that `issue` is called for next ----
    // left operand: this thread's chunk of its rows (ROWS / NR apart, alike in their swizzle)
    Tile ld_tile = now;
    int ld_k = 0;                        // K-tile
    int kc = 0;                          // contraction entry of this thread's chunk
    int hi[NR], wi[NR], img[NR];
    int nP = 0, nQ = 0, Rc = 0, Sc = 1;
    float inv_s = 1.0f;
    const int slot = NR * kDxThreads > ROWS * CH ? tid % (ROWS * CH) : tid, chunk = (slot % CH) ^ swz(slot / CH);
    // right operand
    const int8_t *wr = nullptr;
    uint32_t gb[NB];
    const int bslot = NB * kDxThreads > COLS * CH ? tid % (COLS * CH) : tid, bchunk = (bslot % CH) ^ swz(bslot / CH);
    auto open_tile = [&]() {
        const auto &k = args->c[ld_tile.cls];
        const int rows = k.rows, Hc = k.Hc, Wc = k.Wc, pad_h = k.pad_h, pad_w = k.pad_w;
        const DivBy by_hw{k.by_hw.mul, k.by_hw.sh}, by_w{k.by_w.mul, k.by_w.sh};
        Rc = k.Rc; Sc = k.Sc; inv_s = k.inv_s; wr = k.wr;
        nP = args->P; nQ = args->Q;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int m = min(ld_tile.row0 + i * (ROWS / NR) + slot / CH, rows - 1);
            const int b = div_by(m, by_hw.mul, by_hw.sh), rem = m - b * (Hc * Wc);
            const int h = div_by(rem, by_w.mul, by_w.sh);
            hi[i] = h + pad_h;
            wi[i] = rem - h * Wc + pad_w;
            img[i] = b * nP;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) gb[i] = (uint32_t)min(ld_tile.col0 + i * (COLS / NB) + bslot / CH, args->C - 1) * 64u + (uint32_t)bchunk * 16u;
        ld_k = 0;
        kc = chunk * 16;
    };
    open_tile();
    // where that chunk lies (limb 0), and how far apart its limbs are
    const int8_t *src[NR];
    int step[NR];
    const int8_t *srcb = nullptr;
    auto prepare = [&]() {
        // (kc < 2^17 + a few K-tiles: (kc + 1/2) / Np in fp32 is far enough from a whole number to truncate to the quotient)
        const int tap = (int)(((float)kc + 0.5f) * args->inv_np), n = kc - tap * args->Np;
        const int tr = (int)(((float)tap + 0.5f) * inv_s), ts = tap - tr * Sc;
        const int first = n & ~63;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int hh = hi[i] - tr, ww = wi[i] - ts;
            const bool inside = tr < Rc && (unsigned)hh < (unsigned)nP && (unsigned)ww < (unsigned)nQ;
            const int64_t at = (int64_t)((img[i] + hh) * nQ + ww) * (L * args->Np) + (L * first + (n & 63));
            src[i] = inside ? args->planes + at : args->zeros;
            step[i] = inside ? min(64, args->Np - first) : 0;
        }
        const int kb = ld_k * KT;
        srcb = wr + ((int64_t)(kb >> 6) * args->C * 64 + (kb & 63));
    };
    // (behind the last tile the last K-tile is loaded again and again: the number of loads in flight is then always the same)
    auto advance = [&]() {
        if (ld_k + 1 < ld_tile.nk) { ++ld_k; kc += KT; }
        else {
            const Tile t = tile_at(ld_tile.q + slots);
            if (t.nk != 0) { ld_tile = t; open_tile(); }
        }
    };
    int ahead = 0;                       // stage
    auto issue = [&]() {
        int8_t *base = lds + ahead * STAGE;
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int l = 0; l < L; ++l)
                __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + l * step[i]), (lptr_t)(base + (l * ROWS + i * (ROWS / NR)) * KT + (wave * 1024) % (ROWS * KT)), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(srcb + gb[i]), (lptr_t)(base + (L * ROWS + i * (COLS / NB)) * KT + (wave * 1024) % (COLS * KT)), 16, 0, 0);
        ahead = ahead + 1 == NS ? 0 : ahead + 1;
    };

    const int frow = lane & 31, fa0 = (wm * 32 + frow) * KT, fb0 = (L * ROWS + wn * TN * 32 + frow) * KT, fsw = swz(frow);
    v16i acc[L][TN];
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[l][j][r] = 0;

    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    v4i fa[2][L], fb[2][TN];
    auto read_frags = [&](int buf, int stage, int ks) {
        const int8_t *base = lds + stage * STAGE + (((2 * ks + (lane >> 5)) ^ fsw) << 4);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[buf][j] = *reinterpret_cast<const v4i *>(base + fb0 + j * 32 * KT);
#pragma unroll
        for (int l = 0; l < L; ++l) fa[buf][l] = *reinterpret_cast<const v4i *>(base + fa0 + l * ROWS * KT);
    };
    auto mfma_all = [&](int buf) {
#pragma unroll
        for (int l = 0; l < L; ++l)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[l][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[buf][l], fb[buf][j], acc[l][j], 0, 0, 0);
    };
    // the limbs of an output: the integers are exact, the Horner steps round at 2^-53 relative
    auto write_tile = [&]() {
        int elane = lane;
        asm volatile("" : "+v"(elane));      // (addresses formed here, not kept in registers through the loop)
        const auto &k = args->c[now.cls];
        // output pixel of row lane % 32 of the wave's rows, passed from lane to lane below
        const int rows = k.rows, m = now.row0 + wm * 32 + (elane & 31);
        const int b = div_by(m, k.by_hw.mul, k.by_hw.sh), rem = m - b * (k.Hc * k.Wc);
        const int i = div_by(rem, k.by_w.mul, k.by_w.sh), jj = rem - i * k.Wc;
        const int pixel = m < rows ? (b * args->oH + args->step * i + k.oa) * args->oW + args->step * jj + k.oc : -1;
        float *out = args->out;
        const int C = args->C, ecol = now.col0 + wn * TN * 32 + (elane & 31);
#pragma unroll
        for (int rr = 0; rr < 16; ++rr) {
            const int pix = __shfl(pixel, 4 * (elane >> 5) + 8 * (rr >> 2) + (rr & 3), 64);      // (layout of an accumulator)
            float *p = out + (int64_t)pix * C + ecol;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                double run = (double)acc[L - 1][j][rr];
#pragma unroll
                for (int l = L - 2; l >= 0; --l) run = __builtin_fma(run, 256.0, (double)acc[l][j][rr]);
                if (pix >= 0 && ecol + j * 32 < C) p[j * 32] = (float)(run * out_scale);
            }
        }
#pragma unroll
        for (int l = 0; l < L; ++l)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[l][j][r] = 0;
    };
    int stage = 0, kt = 0;
    if constexpr (KT == 64 && L <= 4) {
        // A K-tile is two k-steps; each reads the fragments of the next one while its own MFMAs run, and the hand-over to
        // the next K-tile lies between them: all fragments of the old one are in registers then, so its stage can be filled again.
#pragma unroll
        for (int s = 0; s < NS; ++s) { prepare(); issue(); advance(); }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 1) * LOADS));
        barrier();
        read_frags(0, 0, 0);
        for (;;) {
            const int next = stage + 1 == NS ? 0 : stage + 1;
            read_frags(1, stage, 1);
            prepare();
            mfma_all(0);
#pragma unroll
            for (int i = 0; i < L * TN; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // the next K-tile has landed (younger: the NS - 2 behind it), this wave's fragment reads are done
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * LOADS));
            __builtin_amdgcn_s_waitcnt(kLgkmcnt0);
            barrier();
            read_frags(0, next, 0);
            issue();
            mfma_all(1);
#pragma unroll
            for (int i = 0; i < L * TN; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            stage = next;
            advance();
            if (++kt == now.nk) {
                write_tile();
                now = tile_at(now.q + slots);
                if (now.nk == 0) break;
                kt = 0;
            }
        }
    } else {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) { prepare(); issue(); advance(); }
        for (;;) {
            // this K-tile has landed (younger: the NS - 2 behind it), for every wave, and every wave has left the stage that is filled next
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * LOADS));
            barrier();
            prepare();
            issue();
            advance();
#pragma unroll
            for (int ks = 0; ks < KT / 32; ++ks) {
                read_frags(0, stage, ks);
                mfma_all(0);
            }
            stage = stage + 1 == NS ? 0 : stage + 1;
            if (++kt == now.nk) {
                write_tile();
                now = tile_at(now.q + slots);
                if (now.nk == 0) break;
                kt = 0;
            }
        }
    }
    // loads behind the last K-tile write LDS: they must be done before this wave ends
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

template <int WN, int TN>
__global__ __launch_bounds__(kDxThreads, 2)
void limb_conv_dx_kernel(DxArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t dx_lds[];
    const dx_args_t args = (dx_args_t)__builtin_amdgcn_kernarg_segment_ptr();
    const double out_scale = a.plan->out_scale_da;
    switch (a.plan->limbs_da) {
        case 3: conv_dx_body<3, WN, TN>(args, dx_lds, out_scale); break;
        case 4: conv_dx_body<4, WN, TN>(args, dx_lds, out_scale); break;
        case 5: conv_dx_body<5, WN, TN>(args, dx_lds, out_scale); break;
        default: conv_dx_body<6, WN, TN>(args, dx_lds, out_scale); break;
    }
}

template <int WN, int TN>
int launch_dx(DxArgs a, hipStream_t stream)
{
    constexpr int ROWS = DxTile<WN, TN>::kRows, COLS = DxTile<WN, TN>::kCols;
    a.tiles_c = (a.C + COLS - 1) / COLS;
    int64_t per_xcd = 0, longest = 0;
    for (int c = 0; c < a.n_classes; ++c) {
        const int64_t tiles = (int64_t)((a.c[c].rows + ROWS - 1) / ROWS) * a.tiles_c;
        if (tiles > 2147483640LL) return CDL_ERR_PARAM;
        a.c[c].tiles = (int)tiles;
        per_xcd += (tiles + 7) / 8;
        const int64_t kt = ((int64_t)a.c[c].Rc * a.c[c].Sc * a.Np + 63) / 64;
        if (kt > longest) longest = kt;
    }
    if (per_xcd > 268435455LL) return CDL_ERR_PARAM;
    // Short contractions: two blocks per compute unit go through all tiles, the loads of a tile under way while the last one is
    // written (3 x 3 stride 2 from 128 channels, eight K-tiles at most: 94 -> 81 us; 1 x 1 from 432, seven: 136 -> 127).  Long
    // ones: a block per tile, handed out as compute units get free (3 x 3 from 256 channels, 36 K-tiles: 140 us against 147; from
    // 100, sixteen: 130 against 152).
    const int slots = (int)(per_xcd < 64 || longest >= 12 ? per_xcd : 64);
    const hipError_t e = hipFuncSetAttribute((const void *)limb_conv_dx_kernel<WN, TN>, hipFuncAttributeMaxDynamicSharedMemorySize, kDxLds);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("limb_conv_dx_kernel", stream, (limb_conv_dx_kernel<WN, TN>), dim3((unsigned)(8 * slots)), dim3(kDxThreads), kDxLds, a);
    return check_launch();
}

}  // namespace

int launch_conv_dx_planes(const float *g, const int8_t *wr, int64_t ld, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H, int32_t W,
                          int32_t C, int32_t N, int32_t Np, int32_t P, int32_t Q, int32_t stride, const BwdPlan *plan, int8_t *planes,
                          const int8_t *zeros, float *d_x_hat, hipStream_t stream)
{
    const int64_t words = (int64_t)B * P * Q * (Np / 4);
    const int64_t blocks = (words + 256 * kPlaneUnroll - 1) / (256 * kPlaneUnroll);
    CDL_LAUNCH("g_planes_kernel", stream, g_planes_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, g, words, N, Np, plan, planes);
    int rc = check_launch();
    if (rc != CDL_OK) return rc;
    DxArgs a{};
    a.n_classes = n_grids;
    a.planes = planes; a.zeros = zeros;
    a.Np = Np; a.inv_np = 1.0f / (float)Np; a.C = C; a.P = P; a.Q = Q; a.oH = H; a.oW = W; a.step = stride;
    a.plan = plan; a.out = d_x_hat;
    for (int i = 0; i < n_grids; ++i) {
        const ConvDxGrid &s = grids[i];
        DxClass &d = a.c[i];
        d.oa = s.oa; d.oc = s.oc; d.Hc = s.Hc; d.Wc = s.Wc; d.pad_h = s.pad_h; d.pad_w = s.pad_w; d.Rc = s.Rc; d.Sc = s.Sc;
        d.rows = B * s.Hc * s.Wc;
        d.wr = wr + (int64_t)i * C * ld;
        d.inv_s = 1.0f / (float)s.Sc;
        d.by_hw = make_div_by((uint32_t)s.Hc * (uint32_t)s.Wc);
        d.by_w = make_div_by((uint32_t)s.Wc);
    }
    // the tile that pads the channels least; 128 x 64 of those that pad equally, unless 64 x 128 halves the reading of the planes
    if (C <= 32) return launch_dx<1, 1>(a, stream);
    // (fewer of those than two per compute unit: half of it)
    int64_t pixels = 0;
    for (int i = 0; i < n_grids; ++i) pixels += a.c[i].rows;
    if ((pixels + 127) / 128 * ((C + 63) / 64) < 512) return launch_dx<2, 1>(a, stream);
    if ((C + 63) / 64 % 2 == 0) return launch_dx<2, 2>(a, stream);
    return launch_dx<1, 2>(a, stream);
}

}  // namespace cdl
