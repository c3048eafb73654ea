// Layer products over quantized operands on the int8 matrix cores of gfx950
// (v_mfma_i32_32x32x32_i8, int32 accumulation), rescaled by the step sizes only in the epilogue.
//
// Forward (Sec. IV-A; Algorithm 1, forward step): C[r, s] = sum_k A[r, k] * B[s, k] on the index
// tensors, both with the contraction index contiguous.
//
// Backward (Algorithm 1, backward step): the fp32 upstream gradient G is contracted with an index
// matrix.  The entries of G are written, inside the GEMM kernel, as L balanced base-256 digits
// ("limbs") of q = rint(g * 2^(8L-1) / sigma) for one power-of-two sigma > max|g|: the product
// g * 2^k is exact, so every entry is represented to within sigma * 2^-8L.  Each limb plane is an
// int8 matrix; the limb planes of 32 output rows form L x 32 rows of one int8 MFMA tile, the limb
// products are exact in int32 and are recombined in double in the epilogue.  L (3..6) is chosen on
// the device so that the rounding of q stays well below the parity tolerance.
#include "cdl_internal.h"
#include "cdl_bwd_plan.h"
#include "cdl_limbs.h"
#include "cdl_finish.h"
#include "cdl_rows.h"

#include <mutex>
#include "cdl_quantizer_math.h"

#include <math.h>

#include <type_traits>

namespace cdl {

namespace {


constexpr int kGemmThreads = 256;
constexpr int kKT = 64;          // forward: contraction bytes staged per pipeline step

struct GemmArgs {
    const int8_t *A;      // [rowsA][lda]
    const int8_t *B;      // [rowsB][ldb]
    int64_t lda, ldb;
    int rowsA, rowsB, Kc;  // Kc: contraction length in bytes, multiple of 16 unless the kernel is for any
    int tiles_m, tiles_n;
    int32_t *acc_out;     // [rowsA][ldc] or null
    float *y_out;         // [rowsA][ldc] or null
    int64_t ldc;
    float scale;          // delta_a * delta_b
    // Operands stored as index - offset (level sets that reach beyond 127): what the stored product lacks,
    //   sum_k (a' + oa)(b' + ob) - sum_k a' b' = oa sum_k b'[s,k] + ob sum_k a'[r,k] + K oa ob,
    // as one int32 per output column (corr_col, includes the constant) and one per output row (corr_row); null = 0.
    const int32_t *corr_col;
    const int32_t *corr_row;
};

// The sum of a row of K index bytes, in lane 0 of the wave that reads it (16 bytes a lane and trip: the sums of 52 x 4032 weights byte by byte 15 us, so 4.7).
__device__ __forceinline__ int row_sum(const int8_t *row, int K, int lane)
{
    int s = 0;
    if (K >= 16) {
#pragma unroll 4
        for (int k = 16 * lane; k < K; k += 1024) {
            const cdl_v4i w = tail_chunk(row, k, K);
#pragma unroll
            for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_sdot4(w[i], 0x01010101, s, false);
        }
    } else if (lane < K) {
        s = (int)row[lane];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    return s;
}

__device__ __forceinline__ int swz(int row, int q) { return q ^ ((row >> 1) & 3); }

// TM x TN: 32x32 MFMA tiles per wave; the block's four waves form a 2 x 2 grid.
// RAGGED: Kc is any length from 16 on, rows start where they start, and the chunk that a row ends in is shifted into place (cdl_rows.h).  That costs
// less than the copies of both operands with padded rows that aligned loads need: 24773 x 73 x 2646, us, copies and product 77 + 30, so 35.
template <int TM, int TN, bool RAGGED>
__global__ __launch_bounds__(kGemmThreads, 2)
void qgemm_kernel(GemmArgs a)
{
    constexpr int BM = 2 * TM * 32, BN = 2 * TN * 32;
    constexpr int LA = BM / 64, LB = BN / 64;   // 16-byte chunks each thread stages per step
    __shared__ __attribute__((aligned(16))) int8_t lds[2][(BM + BN) * kKT];

    // Workgroups are handed to the eight XCDs round-robin; give each XCD a contiguous run of
    // tiles so that tiles sharing an A row-block meet in one L2.
    const int total = a.tiles_m * a.tiles_n;
    const int per_xcd = (int)gridDim.x >> 3;
    const int logical = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (logical >= total) return;
    const int tile_m = logical / a.tiles_n, tile_n = logical % a.tiles_n;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // staging assignment: chunk s = tid + 256 i  ->  LDS byte offset 16 s; row s/4, physical chunk s%4
    const int8_t *ga[LA];
    const int8_t *gb[LB];
    int qa[LA], qb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int s = tid + kGemmThreads * i, row = s >> 2;
        qa[i] = swz(row, s & 3) * 16;
        const int grow = min(tile_m * BM + row, a.rowsA - 1);
        ga[i] = a.A + (int64_t)grow * a.lda + qa[i];
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int s = tid + kGemmThreads * i, row = s >> 2;
        qb[i] = swz(row, s & 3) * 16;
        const int grow = min(tile_n * BN + row, a.rowsB - 1);
        gb[i] = a.B + (int64_t)grow * a.ldb + qb[i];
    }

    // fragment read offsets (bytes inside one stage), per k-step ks: chunk q = 2 ks + lane/32
    int ra[TM][2], rb[TN][2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int row = wm * TM * 32 + i * 32 + (lane & 31);
            ra[i][ks] = row * kKT + swz(row, 2 * ks + (lane >> 5)) * 16;
        }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int row = wn * TN * 32 + j * 32 + (lane & 31);
            rb[j][ks] = BM * kKT + row * kKT + swz(row, 2 * ks + (lane >> 5)) * 16;
        }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    const int steps = (a.Kc + kKT - 1) / kKT;
    const v4i zero4 = {0, 0, 0, 0};

    // 64-row tiles, which run where tiles are fewer than compute units, have two sets of staging registers: a step's chunks are
    // asked for two steps ahead (with one set a step took a whole trip to memory; 10000 x 128 x 1024: 25.4 -> 20.4 us with the
    // index quantizer, 1500 x 1500 x 1500: 38.4 -> 30.5).  Larger tiles fill each other's waits, two sets cost them 1 - 3 %.
    constexpr bool DEEP = TM == 1;
    v4i pa0[LA], pb0[LB], pa1[DEEP ? LA : 1], pb1[DEEP ? LB : 1];
    auto fetch = [&](int kt, v4i (&pa)[LA], v4i (&pb)[LB]) {
        const int64_t off = (int64_t)kt * kKT;
        if constexpr (RAGGED) {
            if (kt * kKT + kKT <= a.Kc) {
#pragma unroll
                for (int i = 0; i < LA; ++i) pa[i] = load_any16(ga[i] + off);
#pragma unroll
                for (int i = 0; i < LB; ++i) pb[i] = load_any16(gb[i] + off);
            } else {
#pragma unroll
                for (int i = 0; i < LA; ++i) pa[i] = tail_chunk(ga[i] - qa[i], kt * kKT + qa[i], a.Kc);
#pragma unroll
                for (int i = 0; i < LB; ++i) pb[i] = tail_chunk(gb[i] - qb[i], kt * kKT + qb[i], a.Kc);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < LA; ++i)
            pa[i] = (kt * kKT + qa[i] < a.Kc) ? *reinterpret_cast<const v4i *>(ga[i] + off) : zero4;
#pragma unroll
        for (int i = 0; i < LB; ++i)
            pb[i] = (kt * kKT + qb[i] < a.Kc) ? *reinterpret_cast<const v4i *>(gb[i] + off) : zero4;
    };
    auto stash = [&](int stage, const v4i (&pa)[LA], const v4i (&pb)[LB]) {
#pragma unroll
        for (int i = 0; i < LA; ++i)
            *reinterpret_cast<v4i *>(&lds[stage][(tid + kGemmThreads * i) * 16]) = pa[i];
#pragma unroll
        for (int i = 0; i < LB; ++i)
            *reinterpret_cast<v4i *>(&lds[stage][BM * kKT + (tid + kGemmThreads * i) * 16]) = pb[i];
    };

    auto compute = [&](int stage) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            v4i fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const v4i *>(&lds[stage][ra[i][ks]]);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = *reinterpret_cast<const v4i *>(&lds[stage][rb[j][ks]]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    };
    fetch(0, pa0, pb0);
    if constexpr (DEEP) fetch(1, pa1, pb1);
    stash(0, pa0, pb0);
    __syncthreads();
    if constexpr (DEEP) {
        for (int step = 0; step < steps; step += 2) {
            fetch(step + 2, pa0, pb0);
            compute(0);
            stash(1, pa1, pb1);
            __syncthreads();
            if (step + 1 >= steps) break;
            fetch(step + 3, pa1, pb1);
            compute(1);
            stash(0, pa0, pb0);
            __syncthreads();
        }
    } else {
        for (int step = 0; step < steps; ++step) {
            if (step + 1 < steps) fetch(step + 1, pa0, pb0);
            compute(step & 1);
            if (step + 1 < steps) stash((step & 1) ^ 1, pa0, pb0);
            __syncthreads();
        }
    }

    // epilogue: lane holds column (lane%32) of each 32x32 tile; register r holds row 8(r/4) + 4(lane/32) + r%4.
    // CORR: operands stored with an offset, corrections per column and row (a branch of its own: a test per
    // element in the common path cost a third of the kernel's time)
    auto epilogue = [&](auto corr_c) {
        constexpr bool CORR = decltype(corr_c)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = tile_n * BN + wn * TN * 32 + j * 32 + (lane & 31);
                if (col >= a.rowsB) continue;
                const int cc = (CORR && a.corr_col) ? a.corr_col[col] : 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = tile_m * BM + wm * TM * 32 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    if (row >= a.rowsA) continue;
                    const int64_t o = (int64_t)row * a.ldc + col;
                    const int v = CORR ? acc[i][j][r] + cc + (a.corr_row ? a.corr_row[row] : 0) : acc[i][j][r];
                    if (a.acc_out) a.acc_out[o] = v;
                    if (a.y_out) a.y_out[o] = a.scale * (float)v;
                }
            }
    };
    if (a.corr_col || a.corr_row) epilogue(std::true_type{});
    else epilogue(std::false_type{});
}

template <int TM, int TN>
int launch_gemm(GemmArgs a, bool ragged, hipStream_t stream)
{
    constexpr int BM = 2 * TM * 32, BN = 2 * TN * 32;
    a.tiles_m = (a.rowsA + BM - 1) / BM;
    a.tiles_n = (a.rowsB + BN - 1) / BN;
    const int64_t total = (int64_t)a.tiles_m * a.tiles_n;
    if (total == 0) return CDL_OK;
    const int64_t grid = (total + 7) / 8 * 8;
    if (ragged) CDL_LAUNCH("qgemm_kernel(fwd)", stream, (qgemm_kernel<TM, TN, true>), dim3((unsigned)grid), dim3(kGemmThreads), 0, a);
    else CDL_LAUNCH("qgemm_kernel(fwd)", stream, (qgemm_kernel<TM, TN, false>), dim3((unsigned)grid), dim3(kGemmThreads), 0, a);
    return check_launch();
}

// ---- backward: limb GEMM ---------------------------------------------------------------------

struct LimbArgs {
    const float *G;       // [M][N] fp32 upstream gradient
    int M, N;
    const int8_t *Bt;     // [cols][ldb] int8 index matrix, contraction index contiguous, zero-filled up to nk * kLBK
    int64_t ldb;          // row stride in bytes: an odd multiple of kLBK, so that rows start in different memory channels
    int nk;               // K-tiles covering the contraction: ceil(kc / kLBK)
    int rows, cols, kc;   // output rows / columns, contraction length
    int tiles_r, splits, kt_per_split;
    int units_per_block;  // consecutive row tiles one block works through
    const BwdPlan *plan;
    int which;            // 0 = d_a_hat, 1 = d_b_hat
    float *out;           // [rows][cols] (splits == 1)
    double *partial;      // [splits][rows][cols] (splits > 1)
    // forward product with the quantizer in its prologue
    QConst fq_k;
    float fq_scale;           // delta_a * delta_b
    const double *row_corr;   // [rows] or null: added to every entry of an output row (the index operand is stored with an offset:
                              // the missing part of the product is offset * step * sum of g over the contraction); splits == 1 only
};

constexpr int kLBK = 128;     // contraction bytes per K-tile
constexpr int kLRows = 32;    // output rows per block
constexpr int kLPlane = kLRows * kLBK;
constexpr int kLThreads = 256;

constexpr int limb_tn(int L) { return L <= 5 ? 3 : 2; }          // 32-column tiles per wave
constexpr int limb_cols(int L) { return 4 * limb_tn(L) * 32; }   // output columns per block
constexpr int limb_stage_bytes(int L) { return L * kLPlane + limb_cols(L) * kLBK; }
constexpr int kLimbLdsBytes = 2 * limb_stage_bytes(5);
static_assert(limb_stage_bytes(3) <= limb_stage_bytes(5) && limb_stage_bytes(4) <= limb_stage_bytes(5) &&
              limb_stage_bytes(6) <= limb_stage_bytes(5), "LDS sized for five limbs");

__device__ __forceinline__ int lswz(int row) { return (row >> 1) & 7; }


// Forward product, fast path for contraction lengths that are multiples of 64: 512 threads = 2 x 4 waves, 256 x 256 tiles
// (wave tile 128 x 64: eight 32x32 accumulators).  One block per compute unit takes tile after tile as ONE sequence of K-tiles of 64
// bytes, brought in by direct global->LDS loads (no staging registers) through a ring of five stages of 32 KiB, four of them under way;
// 16-byte chunks XOR-swizzled over the four chunks of a row so that the fragment reads are free of bank conflicts.  The
// barrier is a bare s_barrier with the one wait it needs written out.
// What bounds it: for large outputs the stores (65536 x 3072 x 768: 805 MB in 219 us, the matrix cores 28 % busy), otherwise the trips of a
// K-tile's loads.  With a block for each tile and one K-tile under way every tile began with an empty pipeline and a K-tile
// took a trip to memory (that size 286 us, without its stores still 252; 100000 x 512 x 128 51 -> 37, 60000 x 1500 x 1024 about 200 -> 160,
// 65536 x 1024 x 256 63 -> 54).  A step's first fragments are read behind the products of the step before (8192 x 3072 x 3072
// 101 -> 93).
constexpr int kRingBK = 64;
// A block of WM x WN waves of TM x TN accumulators each, a ring of RING stages, PER_CU blocks to a compute unit.
template <int WM_, int WN_, int TM_, int TN_, int RING_, int PER_CU_>
struct RingShape {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, RING = RING_, PER_CU = PER_CU_;
    static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves, kRows = WM * TM * 32, kCols = WN * TN * 32;
    static constexpr int kStage = (kRows + kCols) * kRingBK, kLds = RING * kStage;
    static constexpr int kLoadsA = kRows / 16 / kWaves, kLoadsB = kCols / 16 / kWaves;      // of a wave and K-tile, 1 KB each
    static_assert(kLoadsA * 16 * kWaves == kRows && kLoadsB * 16 * kWaves == kCols && PER_CU * kLds <= 160 << 10, "a wave's loads; LDS");
};
using RingWide = RingShape<2, 4, 4, 2, 5, 1>;       // 256 x 256
// The others, four waves, two blocks to a compute unit: less padding and more blocks where outputs are few or narrow (choose_tiles).
using RingTall = RingShape<2, 2, 4, 2, 3, 2>;       // 256 x 128
using RingNarrow = RingShape<4, 1, 2, 2, 4, 2>;     // 256 x 64
using RingSquare = RingShape<2, 2, 2, 2, 5, 2>;     // 128 x 128
using RingLow = RingShape<4, 1, 1, 2, 6, 2>;        // 128 x 64
constexpr int kFTile = RingWide::kRows;

// load i of `loads` of a wave and operand fills LDS slots (wave * loads + i) * 64 + lane: row slot / 4, chunk slot % 4
__device__ __forceinline__ int ring_row(int wave, int lane, int i, int loads) { return (wave * loads + i) * 16 + (lane >> 2); }
// (sixteen rows read at the same chunk q lie in all sixteen chunks of the 64 banks; with (row >> 1) half the cycles of the reads
// were conflicts; up to 1 % of the kernel's time)
__device__ __forceinline__ int ring_swz(int row, int q) { return q ^ ((row >> 2) & 3); }
__device__ __forceinline__ int ring_chunk(int lane) { return ring_swz(lane >> 2, lane & 3) * 16; }      // (rows 16 apart swizzle alike)

// SOURCE: where a wave's loads come from - tile(m, n, ...) the first K-tile of a tile, issue() the loads of a K-tile and on to the next
template <class SHAPE, bool STREAM, class SOURCE>
__device__ __forceinline__ void ring_tiles(const GemmArgs &a, SOURCE &source, int nk)
{
    constexpr int WN = SHAPE::WN, TM = SHAPE::TM, TN = SHAPE::TN, KS = kRingBK / 32, AHEAD = SHAPE::RING - 1;
    constexpr int kLoads = SHAPE::kLoadsA + SHAPE::kLoadsB, kStores = TM * TN * 16;      // of a wave: per K-tile, per tile
    extern __shared__ __attribute__((aligned(16))) int8_t flds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // Workgroups go to the eight XCDs round-robin; XCD x takes the x-th eighth of the tiles, its blocks side by side through them
    // (tiles of one A row-block meet in one L2).
    const int total = a.tiles_m * a.tiles_n, share = (total + 7) >> 3, xcd = (int)blockIdx.x & 7, each = (int)gridDim.x >> 3;
    const int first = xcd * share + ((int)blockIdx.x >> 3), end = min(total, (xcd + 1) * share);
    if (first >= end) return;
    const int tiles = (end - 1 - first) / each + 1, steps = tiles * nk;

    int load_tile = first, load_kt = 0;
    auto tile_sources = [&]() {
        const int m = load_tile / a.tiles_n, n = load_tile - m * a.tiles_n;
        source.tile(m, n, wave, lane);
    };
    auto issue = [&](int stage) {
        source.issue(flds + stage * SHAPE::kStage, wave);
        if (++load_kt == nk) {
            load_kt = 0;
            load_tile = min(load_tile + each, total - 1);
            tile_sources();
        }
    };
    const int frow = lane & 31;
    int fr[KS];                               // (rows 32 apart swizzle alike)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fr[ks] = frow * kRingBK + ring_swz(frow, 2 * ks + (lane >> 5)) * 16;
    const int fa_at = wm * TM * 32 * kRingBK, fb_at = (SHAPE::kRows + wn * TN * 32) * kRingBK;

    static_assert(KS == 2, "fragments of two k-steps");
    v16i acc[TM][TN];
    v4i fa[2][TM], fb[2][TN];
    auto read = [&](int stage, int ks) {
        const int8_t *base = flds + stage * SHAPE::kStage;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[ks][i] = *reinterpret_cast<const v4i *>(base + fa_at + i * 32 * kRingBK + fr[ks]);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[ks][j] = *reinterpret_cast<const v4i *>(base + fb_at + j * 32 * kRingBK + fr[ks]);
    };
    auto multiply = [&](int ks, auto first_c) {
        constexpr bool FIRST = decltype(first_c)::value;
        const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks][i], fb[ks][j], FIRST ? zero : acc[i][j], 0, 0, 0);
    };
    // CORR: operands stored with an offset, corrections per column and row, loaded before the first store (a load between the stores makes every store wait for the one before it): a lane
    // has its columns' and those of the rows 32 i + (its number in its half), which the others get from it
    // (us, rows x columns x contraction, staged tiles / loads between the stores / so: 6617 x 480 x 448 13.8 / 21.2 / 12.8, 46255 x 608 x 192 52 / 69 / 29.2, 934088 x 288 x 128 461 / 580 / 258; the kernels without corrections are as they were)
    auto emit = [&](auto full_c, auto corr_c, auto *out, int row0, int col0) {
        constexpr bool FULL = decltype(full_c)::value, CORR = decltype(corr_c)::value;
        using T = std::remove_pointer_t<decltype(out)>;
        typedef T __attribute__((address_space(1))) *out_t;
        typedef char __attribute__((address_space(1))) *byte_t;
        int elane = lane;
        asm volatile("" : "+v"(elane));      // (addresses formed here, not kept in registers through the loop)
        const int half4 = 4 * (elane >> 5), ecol = elane & 31;
        const uint32_t off = 4u * (uint32_t)(half4 * (int)a.ldc + ecol);
        const out_t base = (out_t)out + (int64_t)row0 * a.ldc + col0;
        int row_corr[TM], col_corr[TN];
        if (CORR) {
#pragma unroll
            for (int j = 0; j < TN; ++j) col_corr[j] = a.corr_col && (FULL || col0 + ecol + 32 * j < a.rowsB) ? a.corr_col[col0 + ecol + 32 * j] : 0;
#pragma unroll
            for (int i = 0; i < TM; ++i) row_corr[i] = a.corr_row && (FULL || row0 + 32 * i + ecol < a.rowsA) ? a.corr_row[row0 + 32 * i + ecol] : 0;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = i * 32 + 8 * (r >> 2) + (r & 3);
                const int rc = CORR ? __shfl(row_corr[i], 8 * (r >> 2) + (r & 3) + half4, 64) : 0;      // (all lanes, also those beyond the rows)
                out_t at = base + (int64_t)dr * a.ldc;
                asm("" : "+s"(at));          // (a base in scalar registers and the lane's offset)
                const out_t p = (out_t)((byte_t)at + off);
                const bool row_ok = FULL || row0 + dr + half4 < a.rowsA;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const bool ok = FULL || (row_ok && col0 + ecol + 32 * j < a.rowsB);
                    if (!ok) continue;
                    const int v = CORR ? acc[i][j][r] + rc + col_corr[j] : acc[i][j][r];
                    const T x = std::is_same<T, float>::value ? (T)(a.scale * (float)v) : (T)v;
                    if (FULL && STREAM) __builtin_nontemporal_store(x, p + 32 * j);
                    else p[32 * j] = x;
                }
            }
    };
    auto epilogue = [&](int tile) {
        const int m = tile / a.tiles_n, n = tile - m * a.tiles_n, row0 = m * SHAPE::kRows + wm * TM * 32, col0 = n * SHAPE::kCols + wn * TN * 32;
        const bool full = row0 + TM * 32 <= a.rowsA && col0 + TN * 32 <= a.rowsB, corr = a.corr_col || a.corr_row;
        auto all = [&](auto full_c, auto corr_c) {
            if (a.acc_out) emit(full_c, corr_c, a.acc_out, row0, col0);
            if (a.y_out) emit(full_c, corr_c, a.y_out, row0, col0);
        };
        if (full && !corr) {
            all(std::true_type{}, std::false_type{});
        } else {
            if (corr) all(std::false_type{}, std::true_type{});
            else all(std::false_type{}, std::false_type{});
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // (fewer than kStores stores, see below)
        }
    };

    tile_sources();
    for (int s = 0; s < AHEAD; ++s) issue(s);              // (past the last step: the last tile again, which nobody reads)
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((AHEAD - 1) * kLoads));
    barrier();
    read(0, 0);
    int stage = 0, kt = 0, tile = first;
    for (int s = 0; s < steps; ++s) {
        // The next step's loads have landed, so that its first fragments are read behind this one's products; younger are those of AHEAD - 2
        // steps, and where a tile ended since they were asked for its kStores stores or more: loads and stores are counted together, up to 63, in order.
        if (s >= nk && kt < AHEAD - 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kStores < 63 ? kStores : 63));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm((AHEAD - 2) * kLoads));
        barrier();                                         // ... for every wave, and every wave has left the stage before
        const int next = stage + 1 == SHAPE::RING ? 0 : stage + 1;
        issue(stage == 0 ? SHAPE::RING - 1 : stage - 1);
        read(stage, 1);
        if (kt == 0) multiply(0, std::true_type{});
        else multiply(0, std::false_type{});
        read(next, 0);
        multiply(1, std::false_type{});
        stage = next;
        if (++kt == nk) {
            epilogue(tile);
            kt = 0;
            tile += each;
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));              // the loads behind the last step write LDS: done before this wave ends
}

template <class SHAPE>
struct MatrixSource {
    const GemmArgs &a;
    const int8_t *src_a, *src_b;             // of the next K-tile (uniform)
    uint32_t off_a[SHAPE::kLoadsA], off_b[SHAPE::kLoadsB];
    __device__ __forceinline__ void tile(int m, int n, int wave, int lane)
    {
        src_a = a.A + (int64_t)m * SHAPE::kRows * a.lda;
        src_b = a.B + (int64_t)n * SHAPE::kCols * a.ldb;
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsA; ++i)
            off_a[i] = (uint32_t)min(ring_row(wave, lane, i, SHAPE::kLoadsA), a.rowsA - 1 - m * SHAPE::kRows) * (uint32_t)a.lda + (uint32_t)ring_chunk(lane);
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsB; ++i)
            off_b[i] = (uint32_t)min(ring_row(wave, lane, i, SHAPE::kLoadsB), a.rowsB - 1 - n * SHAPE::kCols) * (uint32_t)a.ldb + (uint32_t)ring_chunk(lane);
    }
    __device__ __forceinline__ void issue(int8_t *stage, int wave)
    {
        int8_t *const to_a = stage + wave * SHAPE::kLoadsA * 1024, *const to_b = stage + SHAPE::kRows * kRingBK + wave * SHAPE::kLoadsB * 1024;
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsA; ++i) __builtin_amdgcn_global_load_lds((gptr_t)(src_a + off_a[i]), (lptr_t)(to_a + i * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsB; ++i) __builtin_amdgcn_global_load_lds((gptr_t)(src_b + off_b[i]), (lptr_t)(to_b + i * 1024), 16, 0, 0);
        src_a += kRingBK;
        src_b += kRingBK;
    }
};

template <class SHAPE, bool STREAM>
__global__ __launch_bounds__(SHAPE::kThreads, SHAPE::PER_CU)
void qgemm_dma_kernel(GemmArgs a)
{
    MatrixSource<SHAPE> source{a};
    ring_tiles<SHAPE, STREAM>(a, source, a.Kc / kRingBK);
}

// Contraction lengths that are whole K-tiles, and enough rows: where the rounds of 256 x 256 tiles, one a compute unit, take no longer
// than those of 256 x 128 tiles, two a compute unit - a round 1.25 times as long, 0.85 with one.  us, this kernel / that one, K = 1024: 24000 rows x
// 640 columns 41.5 / 30.6, x 512 24.3 / 29.4, x 256 21.0 / 19.4; 9000 x 640 23.2 / 19.5, x 1000 25.0 / 28.6; 60000 x 1000 104 / 133.
bool dma_serves(int64_t M, int64_t N, int64_t K)
{
    // (32-bit offsets inside a tile)
    if (K % kRingBK != 0 || M * N < (int64_t)kFTile * kFTile * 64 || N <= 128 || K >= 1 << 23 || N >= 1 << 27) return false;
    const int64_t rows = (M + 255) / 256, here = (rows * ((N + 255) / 256) + 255) / 256, other = rows * ((N + 127) / 128), rest = other % 512;
    return here * 100 <= other / 512 * 125 + (rest == 0 ? 0 : rest <= 256 ? 85 : 125);
}

// Which tiles a product of M x N outputs over nk K-tiles of 64 bytes takes.  A form's time, us: its start, its K-tiles through every round of blocks (half: a last round with a block
// to a compute unit at most), a share for every round, and what its output adds, per megabyte.  Fitted to 260 convolutions and 130 matrix products, each run in every form (off by 5 - 12 %; of the staged tiles of 256 x 64
// those terms that choose best for 673 layers and 105 products of up to 64 columns).  No term for the operands' bytes: where those bound a product the rules of choose_tiles hold.  Of 1672 convolutions (1 to 512 images and more, 16 to 640 channels -> 20 to 800) and 1033 matrix products (200 to 3 M rows, 33 to 1500
// columns, 1 to 64 K-tiles), each run in every form, the choices take 0.91 and 0.95 of the time of the staged or wide form that they replace; 48 are more than 3 % slower than that, the worst 9 and 7 %.  us, staged / the choice: convolutions 56 x 56 x 64 -> 64 on 128 images 48.4 / 32.8
// (narrow), 28 x 28 x 128 -> 128 33.5 / 25.9 (tall), 29 x 18 x 48 -> 148 on 185 36.1 / 24.9 (narrow), 25 x 25 x 448 -> 52 at stride 2 on 138 33.3 / 21.0 (low), 19 x 53 x 288 -> 412 on 53 110 / 89.6 (wide), 26 x 26 x 32 -> 84, 5 x 5,
// on 229 45.9 / 33.3 (square); matrices 60000 x 128 x 1152 23.7 / 19.1 (square), 982 x 1408 x 1280 11.4 / 8.5 (low), 100352 x 128 x 1152 34.8 / 28.7 (tall).
enum TileForm { kTileStaged, kTileWide, kTileTall, kTileNarrow, kTileSquare, kTileLow };
struct TileTime { int rows, cols, per_cu; double start, round, half, share, per_mb; };
constexpr TileTime kRingTimes[2][5] = {      // matrices, windows; in the order of the forms
    {{256, 256, 1, 7.1, 0.696, 0.0, 0.0, 0.130}, {256, 128, 2, 5.7, 0.837, 0.549, 0.0, 0.123}, {256, 64, 2, 4.2, 0.675, 0.338, 0.0, 0.113}, {128, 128, 2, 4.6, 0.537, 0.286, 0.0, 0.114}, {128, 64, 2, 4.1, 0.381, 0.207, 0.0, 0.103}},
    {{256, 256, 1, 8.3, 0.774, 0.0, 0.0, 0.153}, {256, 128, 2, 8.0, 0.870, 0.637, 0.0, 0.130}, {256, 64, 2, 6.5, 0.652, 0.474, 0.0, 0.121}, {128, 128, 2, 6.2, 0.541, 0.424, 0.0, 0.130}, {128, 64, 2, 5.5, 0.406, 0.321, 0.0, 0.129}}};
constexpr TileTime kStagedTimes[2][2][3] = {      // up to 64 columns, more; 64, 128, 256 rows
    {{{64, 64, 2, 1.9, 0.386, 0.284, 1.9, 0.025}, {128, 64, 2, 1.4, 0.540, 0.4, 1.4, 0.24}, {256, 64, 2, 0.0, 1.798, 0.667, 0.0, 0.216}}, {{64, 128, 2, 2.1, 0.441, 0.329, 2.1, 0.175}, {128, 128, 2, 3.0, 0.671, 0.49, 3.0, 0.133}, {256, 128, 2, 2.0, 1.075, 0.7, 12.1, 0.003}}},
    {{{64, 64, 2, 1.9, 0.386, 0.284, 1.9, 0.025}, {128, 64, 2, 2.3, 0.468, 0.35, 2.3, 0.153}, {256, 64, 2, 2.1, 0.818, 0.597, 3.8, 0.132}}, {{64, 128, 2, 2.3, 0.463, 0.367, 2.3, 0.156}, {128, 128, 2, 3.4, 0.726, 0.485, 3.4, 0.094}, {256, 128, 2, 4.2, 1.062, 0.641, 9.1, 0.037}}}};

// least: K-tiles that a block takes the time of in any case (a ring is filled first)
double tile_time(const TileTime &t, int64_t M, int64_t N, int64_t nk, int least)
{
    const int64_t tiles = ((M + t.rows - 1) / t.rows) * ((N + t.cols - 1) / t.cols), places = 256ll * t.per_cu, rest = tiles % places;
    const bool half = t.per_cu == 2 && rest > 0 && rest <= 256;
    const double whole = (double)(tiles / places + (rest > 0 && !half ? 1 : 0)), rounds = whole + (half ? 1.0 : 0.0);
    const double steps = rounds * (double)nk < least ? least / rounds : (double)nk;
    return t.start + (whole * t.round + (half ? t.half : 0.0)) * steps + rounds * t.share + 4e-6 * (double)M * (double)N * t.per_mb;
}

// Rows of a staged tile: as few as give every compute unit one.
int staged_rows(int64_t M, int64_t N)
{
    const int64_t cols = (N + (N <= 64 ? 63 : 127)) / (N <= 64 ? 64 : 128);
    const bool few = (M + 255) / 256 * cols < 256 && M > 128;
    return !few ? 256 : (M + 127) / 128 * cols < 256 ? 64 : 128;
}

// whole: contractions of whole K-tiles (windows: of taps of whole K-tiles), which the widest tiles take where they are no worse than staged ones.
TileForm choose_tiles(bool windows, bool whole, int64_t M, int64_t N, int64_t K)
{
    // (32-bit offsets inside a tile)
    if (K >= 1 << 23 || N >= 1 << 27 || (!windows && !whole)) return kTileStaged;
    constexpr int kRingLeast = 6;
    const int64_t nk = (K + kRingBK - 1) / kRingBK;
    const bool wide = whole && dma_serves(M, N, K);
    const int rows = staged_rows(M, N);
    // Bound by memory, which the times do not tell apart.  Outputs beyond the memory-side cache over few K-tiles: whole rows of 256 columns (us, wide / what the times would choose: 252312 x 1189 x 64 287 / 384, 522648 x 574 x 64
    // 304 / 356, 478895 x 192 x 128 74 / 67).  Up to 64 columns over few K-tiles: staged, whose stores do not wait where the columns end inside a tile (us, staged / so: 662125 x 63 x 128 41.8 / 52.6, 240573 x 43 x 128 16.6 / 20.8,
    // 147875 x 36 x 448 20.2 / 22.4, 73034 x 46 x 512 15.8 / 14.3; up to 128 rows to a tile 23877 x 38 x 576 6.4 / 7.0, with 64 columns 16514 x 64 x 960 8.5 / 7.5).
    if (wide && nk <= 8 && M * N > 64 << 20) return kTileWide;
    if (!windows && N <= 64 && nk < (rows == 256 || N == 64 ? 8 : 17)) return kTileStaged;
    TileForm best = wide ? kTileWide : kTileStaged;
    // (staged tiles of 64 rows, a last round of which is mostly short, are often better than that for windows: 7 x 49 x 49 x 240 -> 24, 5 x 5  35 us, low 42)
    const double margin = windows && rows == 64 ? 0.85 : 0.92;
    double least = margin * (wide ? tile_time(kRingTimes[windows][0], M, N, nk, kRingLeast) : tile_time(kStagedTimes[windows][N > 64][rows == 64 ? 0 : rows == 128 ? 1 : 2], M, N, nk, 0));
    for (int f = 0; f < 5; ++f) {
        if (f == 4 && !windows && nk < 8) continue;      // (1825 x 694 x 128: staged 5.4, low 8.2)
        const double t = tile_time(kRingTimes[windows][f], M, N, nk, kRingLeast);
        if (t < least) { least = t; best = (TileForm)(kTileWide + f); }
    }
    return best;
}

int64_t ring_grid(int64_t tiles, int per_cu)
{
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0)
        n_cu = 256;
    const int64_t places = (int64_t)per_cu * n_cu;
    return tiles < places ? (tiles + 7) / 8 * 8 : places / 8 * 8;
}

template <class SHAPE>
int launch_gemm_ring(GemmArgs a, hipStream_t stream)
{
    a.tiles_m = (a.rowsA + SHAPE::kRows - 1) / SHAPE::kRows;
    a.tiles_n = (a.rowsB + SHAPE::kCols - 1) / SHAPE::kCols;
    const int64_t total = (int64_t)a.tiles_m * a.tiles_n;
    if (total == 0) return CDL_OK;
    const int64_t grid = ring_grid(total, SHAPE::PER_CU);
    const auto kernel = stream_output((int64_t)a.rowsA * a.rowsB, a.rowsB, a.y_out) && !a.acc_out ? qgemm_dma_kernel<SHAPE, true> : qgemm_dma_kernel<SHAPE, false>;
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SHAPE::kLds);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("qgemm_kernel(fwd)", stream, kernel, dim3((unsigned)grid), dim3(SHAPE::kThreads), SHAPE::kLds, a);
    return check_launch();
}

// ---- forward product of a convolutional layer, without an im2col matrix ---------------------------------
//
// acc[b,p,q,n] = sum_{r,s,c} x[b, p*stride + r - pad, q*stride + s - pad, c] * w[n,r,s,c]  (Sec. IV-A for a
// convolutional layer): the product of the [B*P*Q, R*S*C] matrix of input windows with w^T, where row m of that
// matrix is never stored - its 16-byte chunks are read from the NHWC tensor where they lie (C is a multiple of
// 16, so a chunk lies inside one tap), and chunks of taps that fall outside the image come from a page of
// padding bytes (the stored value of level index 0).
struct ConvArgs {
    const int8_t *X;       // [B][H][W][C]
    const int8_t *Wt;      // [N][R*S*C]
    const int8_t *pad_page;   // 128 bytes of the padding value (direct-load kernel)
    int pad_word;          // the padding value in all four bytes (register-staged kernel)
    int B, H, W, C, N, R, S, stride, pad, P, Q;
    int M, Kc;             // B*P*Q, R*S*C
    int tiles_m, tiles_n;
    int32_t *acc_out;      // [M][N] or null
    float *y_out;          // [M][N] or null
    float scale;
    const int32_t *corr_col;   // [N] or null: x stored with an offset, x_offset * sum over the window of w[n]
    // ChunkSource: zeros (16 bytes); chunks of a tap, and a K-tile's four chunks in whole taps and chunks
    const int8_t *zero_page;
    int c16, step_taps, step_in;
    DivBy by_c16, by_s, by_pq, by_q;
};

// where output pixel m looks: first input row and column of its window, and the offset of that (possibly
// virtual) pixel in X
struct ConvRow { int h0, w0; int64_t off; };
// BY: with the launch's multipliers (the kernels with direct loads: 2 - 4 % of small layers; the staged one is 3 % slower with them)
template <bool BY>
__device__ __forceinline__ ConvRow conv_row(const ConvArgs &a, int m)
{
    const int pq = a.P * a.Q;
    const int b = BY ? div_by(m, a.by_pq) : m / pq, rem = m - b * pq, p = BY ? div_by(rem, a.by_q) : rem / a.Q, q = rem - p * a.Q;
    ConvRow r;
    r.h0 = p * a.stride - a.pad;
    r.w0 = q * a.stride - a.pad;
    r.off = (((int64_t)b * a.H + r.h0) * a.W + r.w0) * a.C;
    return r;
}

__device__ __forceinline__ void conv_store(const ConvArgs &a, int row, int col, int v)
{
    const int64_t o = (int64_t)row * a.N + col;
    if (a.acc_out) a.acc_out[o] = v;
    if (a.y_out) a.y_out[o] = a.scale * (float)v;
}

// C a multiple of 64: the tiles of qgemm_dma_kernel, a K-tile being 64 channels of one tap.  Where a row's chunk lies is worked out when the tap
// changes; inside a tap it moves on by 64 channels, or stays on the padding.  us, against a block for every tile with K-tiles of 128 channels: 256 images of
// 14 x 14 x 320 -> 320, 3 x 3  102 -> 81;  128 x 28 x 28 x 192 -> 192  76 -> 59;  256 x 14 x 14 x 256 -> 256  44.6 -> 43.0.
template <class SHAPE>
struct WindowSource {
    static constexpr int kLoads = SHAPE::kLoadsA;
    const ConvArgs &a;
    const int8_t *src_b;                     // of the next K-tile (uniform)
    uint32_t off_b[SHAPE::kLoadsB];
    int h0[kLoads], w0[kLoads];              // first input row and column of a row's window, and its first chunk
    int64_t off[kLoads];
    int tr, ts, left;                        // tap of the next K-tile, and K-tiles left in it
    const int8_t *at[kLoads];                // a row's chunk of the next K-tile, or the padding
    uint32_t on[kLoads];
    __device__ __forceinline__ void tap()
    {
        const int64_t tap_off = ((int64_t)tr * a.W + ts) * a.C;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const bool inside = (unsigned)(h0[i] + tr) < (unsigned)a.H && (unsigned)(w0[i] + ts) < (unsigned)a.W;
            at[i] = inside ? a.X + (off[i] + tap_off) : a.pad_page;
            on[i] = inside ? kRingBK : 0;
        }
        left = a.C / kRingBK;
    }
    __device__ __forceinline__ void tile(int m, int n, int wave, int lane)
    {
        src_b = a.Wt + (int64_t)n * SHAPE::kCols * a.Kc;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const ConvRow r = conv_row<true>(a, min(m * SHAPE::kRows + ring_row(wave, lane, i, kLoads), a.M - 1));
            h0[i] = r.h0;
            w0[i] = r.w0;
            off[i] = r.off + ring_chunk(lane);
        }
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsB; ++i)
            off_b[i] = (uint32_t)min(ring_row(wave, lane, i, SHAPE::kLoadsB), a.N - 1 - n * SHAPE::kCols) * (uint32_t)a.Kc + (uint32_t)ring_chunk(lane);
        tr = ts = 0;
        tap();
    }
    __device__ __forceinline__ void issue(int8_t *stage, int wave)
    {
        int8_t *const to_a = stage + wave * kLoads * 1024, *const to_b = stage + SHAPE::kRows * kRingBK + wave * SHAPE::kLoadsB * 1024;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) __builtin_amdgcn_global_load_lds((gptr_t)at[i], (lptr_t)(to_a + i * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsB; ++i) __builtin_amdgcn_global_load_lds((gptr_t)(src_b + off_b[i]), (lptr_t)(to_b + i * 1024), 16, 0, 0);
        src_b += kRingBK;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) at[i] += on[i];
        if (--left == 0) {
            if (++ts == a.S) { ts = 0; ++tr; }
            tap();                           // (behind the last tap: the next tile follows, or nobody loads from there)
        }
    }
};

// Any C that is a multiple of 16: a lane's chunk of a K-tile, the same of all its rows, lies in a tap of its own.  What lies behind the contraction in the
// last K-tile reads as zeros of x and any weights.
template <class SHAPE>
struct ChunkSource {
    static constexpr int kLoads = SHAPE::kLoadsA;
    const ConvArgs &a;
    const int8_t *src_b;                     // (uniform)
    uint32_t row_b[SHAPE::kLoadsB];
    int h0[kLoads], w0[kLoads];
    int64_t off[kLoads];
    int chunk, tap, in_tap;                  // a lane's chunk of the contraction, its tap and place in it
    __device__ __forceinline__ void tile(int m, int n, int wave, int lane)
    {
        src_b = a.Wt + (int64_t)n * SHAPE::kCols * a.Kc;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const ConvRow r = conv_row<true>(a, min(m * SHAPE::kRows + ring_row(wave, lane, i, kLoads), a.M - 1));
            h0[i] = r.h0;
            w0[i] = r.w0;
            off[i] = r.off;
        }
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsB; ++i) row_b[i] = (uint32_t)min(ring_row(wave, lane, i, SHAPE::kLoadsB), a.N - 1 - n * SHAPE::kCols) * (uint32_t)a.Kc;
        chunk = ring_chunk(lane) / 16;
        tap = div_by(chunk, a.by_c16);
        in_tap = chunk - tap * a.c16;
    }
    __device__ __forceinline__ void issue(int8_t *stage, int wave)
    {
        int8_t *const to_a = stage + wave * kLoads * 1024, *const to_b = stage + SHAPE::kRows * kRingBK + wave * SHAPE::kLoadsB * 1024;
        const int tr = div_by(tap, a.by_s), ts = tap - tr * a.S;
        const bool there = tap < a.R * a.S;
        const int64_t tap_off = (int64_t)(tr * a.W + ts) * a.C + in_tap * 16;
        const int8_t *const outside = there ? a.pad_page : a.zero_page;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const bool inside = there && (unsigned)(h0[i] + tr) < (unsigned)a.H && (unsigned)(w0[i] + ts) < (unsigned)a.W;
            __builtin_amdgcn_global_load_lds((gptr_t)(inside ? a.X + (off[i] + tap_off) : outside), (lptr_t)(to_a + i * 1024), 16, 0, 0);
        }
        const uint32_t at_b = there ? (uint32_t)chunk * 16u : 0u;
#pragma unroll
        for (int i = 0; i < SHAPE::kLoadsB; ++i) __builtin_amdgcn_global_load_lds((gptr_t)(src_b + (row_b[i] + at_b)), (lptr_t)(to_b + i * 1024), 16, 0, 0);
        chunk += kRingBK / 16;
        tap += a.step_taps;
        in_tap += a.step_in;
        const bool over = in_tap >= a.c16;
        tap += over ? 1 : 0;
        in_tap -= over ? a.c16 : 0;
    }
};

template <class SHAPE, bool STREAM, bool CHUNKS>
__global__ __launch_bounds__(SHAPE::kThreads, SHAPE::PER_CU)
void qconv_dma_kernel(ConvArgs a)
{
    GemmArgs out{};
    out.rowsA = a.M; out.rowsB = a.N; out.ldc = a.N;
    out.tiles_m = a.tiles_m; out.tiles_n = a.tiles_n;
    out.acc_out = a.acc_out; out.y_out = a.y_out; out.scale = a.scale; out.corr_col = a.corr_col;
    if constexpr (CHUNKS) {
        ChunkSource<SHAPE> source{a};
        ring_tiles<SHAPE, STREAM>(out, source, (a.Kc + kRingBK - 1) / kRingBK);
    } else {
        WindowSource<SHAPE> source{a};
        ring_tiles<SHAPE, STREAM>(out, source, a.Kc / kRingBK);
    }
}

// Any C that is a multiple of 16: the structure of qgemm_kernel (256 x 128 tile, 64-byte K steps staged through
// registers), every 16-byte chunk of the window matrix looked up on its own: a table in LDS gives, per chunk of the
// contraction, its tap and its offset from the window's first pixel.
constexpr int kConvMaxChunks = 2048;     // contraction lengths up to 32768

template <int TM, int TN>
__global__ __launch_bounds__(kGemmThreads, 2)
void qconv_kernel(ConvArgs a)
{
    constexpr int BM = 2 * TM * 32, BN = 2 * TN * 32;
    constexpr int LA = BM / 64, LB = BN / 64;
    __shared__ __attribute__((aligned(16))) int8_t lds[2][(BM + BN) * kKT];
    __shared__ int2 taps[kConvMaxChunks];    // .x: offset of the chunk from the window's first pixel, .y: tap row << 16 | tap column

    const int total = a.tiles_m * a.tiles_n;
    const int per_xcd = (int)gridDim.x >> 3;
    const int logical = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (logical >= total) return;
    const int tile_m = logical / a.tiles_n, tile_n = logical % a.tiles_n;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    for (int c16 = tid; c16 < a.Kc / 16; c16 += kGemmThreads) {
        const int k = c16 * 16, tap = k / a.C, c = k - tap * a.C, r = tap / a.S, s = tap - r * a.S;
        taps[c16] = make_int2((r * a.W + s) * a.C + c, (r << 16) | s);
    }

    ConvRow xr[LA];
    const int8_t *gb[LB];
    int qa[LA], qb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int s = tid + kGemmThreads * i, row = s >> 2;
        qa[i] = swz(row, s & 3);
        xr[i] = conv_row<false>(a, min(tile_m * BM + row, a.M - 1));
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int s = tid + kGemmThreads * i, row = s >> 2;
        qb[i] = swz(row, s & 3) * 16;
        const int grow = min(tile_n * BN + row, a.N - 1);
        gb[i] = a.Wt + (int64_t)grow * a.Kc + qb[i];
    }

    int ra[TM][2], rb[TN][2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int row = wm * TM * 32 + i * 32 + (lane & 31);
            ra[i][ks] = row * kKT + swz(row, 2 * ks + (lane >> 5)) * 16;
        }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int row = wn * TN * 32 + j * 32 + (lane & 31);
            rb[j][ks] = BM * kKT + row * kKT + swz(row, 2 * ks + (lane >> 5)) * 16;
        }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    const int steps = (a.Kc + kKT - 1) / kKT;
    const int chunks = a.Kc / 16;
    const v4i zero4 = {0, 0, 0, 0};
    const v4i pad4 = {a.pad_word, a.pad_word, a.pad_word, a.pad_word};
    __syncthreads();        // the tap table is complete

    // Two sets of staging registers where the tile leaves room for them: a step's chunks are asked for two steps ahead, and taps
    // outside the image read the page of padding instead of branching round the load (a convolution 5 x 5 x 272 -> 24 on 176
    // images of 11 x 11, with its 64-row tiles: whole step 275 -> 253 us).  The largest tile was 2 % slower that way.
    constexpr bool DEEP = TM * TN < 8;
    v4i pa0[LA], pb0[LB], pa1[DEEP ? LA : 1], pb1[DEEP ? LB : 1];
    auto fetch = [&](int kt, v4i (&pa)[LA], v4i (&pb)[LB]) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int c16 = kt * (kKT / 16) + qa[i];
            // (beyond the contraction: multiplies zeros of the other operand)
            const int2 t = taps[min(c16, chunks - 1)];
            const bool inside = (unsigned)(xr[i].h0 + (t.y >> 16)) < (unsigned)a.H && (unsigned)(xr[i].w0 + (t.y & 0xffff)) < (unsigned)a.W;
            if constexpr (DEEP) pa[i] = *reinterpret_cast<const v4i *>(inside ? a.X + (xr[i].off + t.x) : a.pad_page);
            else pa[i] = inside ? *reinterpret_cast<const v4i *>(a.X + (xr[i].off + t.x)) : pad4;
        }
        const int64_t off = (int64_t)kt * kKT;
#pragma unroll
        for (int i = 0; i < LB; ++i)
            pb[i] = (kt * kKT + qb[i] < a.Kc) ? *reinterpret_cast<const v4i *>(gb[i] + off) : zero4;
    };
    auto stash = [&](int stage, const v4i (&pa)[LA], const v4i (&pb)[LB]) {
#pragma unroll
        for (int i = 0; i < LA; ++i)
            *reinterpret_cast<v4i *>(&lds[stage][(tid + kGemmThreads * i) * 16]) = pa[i];
#pragma unroll
        for (int i = 0; i < LB; ++i)
            *reinterpret_cast<v4i *>(&lds[stage][BM * kKT + (tid + kGemmThreads * i) * 16]) = pb[i];
    };

    auto compute = [&](int stage) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            v4i fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const v4i *>(&lds[stage][ra[i][ks]]);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = *reinterpret_cast<const v4i *>(&lds[stage][rb[j][ks]]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    };
    fetch(0, pa0, pb0);
    if constexpr (DEEP) fetch(1, pa1, pb1);
    stash(0, pa0, pb0);
    __syncthreads();
    if constexpr (DEEP) {
        for (int step = 0; step < steps; step += 2) {
            fetch(step + 2, pa0, pb0);
            compute(0);
            stash(1, pa1, pb1);
            __syncthreads();
            if (step + 1 >= steps) break;
            fetch(step + 3, pa1, pb1);
            compute(1);
            stash(0, pa0, pb0);
            __syncthreads();
        }
    } else {
        for (int step = 0; step < steps; ++step) {
            if (step + 1 < steps) fetch(step + 1, pa0, pb0);
            compute(step & 1);
            if (step + 1 < steps) stash((step & 1) ^ 1, pa0, pb0);
            __syncthreads();
        }
    }

    auto epilogue = [&](auto corr_c) {
        constexpr bool CORR = decltype(corr_c)::value;
        int cc[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = tile_n * BN + wn * TN * 32 + j * 32 + (lane & 31);
            cc[j] = (CORR && col < a.N) ? a.corr_col[col] : 0;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = tile_n * BN + wn * TN * 32 + j * 32 + (lane & 31);
                if (col >= a.N) continue;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = tile_m * BM + wm * TM * 32 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    if (row < a.M) conv_store(a, row, col, CORR ? acc[i][j][r] + cc[j] : acc[i][j][r]);
                }
            }
    };
    if (a.corr_col) epilogue(std::true_type{});
    else epilogue(std::false_type{});
}

// 128 bytes that read as level index 0 of an operand stored with offset `off` and 128 zeros, and (with an offset) the
// correction per output channel: off * sum of w[n] over the whole window (a padded tap holds -off + off = 0)
__global__ __launch_bounds__(256)
void conv_prep_kernel(int8_t *page, int off, const int8_t *w, int N, int Kc, int32_t *corr)
{
    if (blockIdx.x == 0) page[threadIdx.x] = threadIdx.x < 128 ? (int8_t)(-off) : (int8_t)0;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int n = blockIdx.x * 4 + wave; n < N; n += gridDim.x * 4) {
        const int s = row_sum(w + (int64_t)n * Kc, Kc, lane);
        if (lane == 0) corr[n] = off * s;
    }
}

// a page of zeros that belongs to the library's device code (one copy per GPU): the padding of operands stored
// without an offset, so that such calls need no workspace
static __device__ __align__(256) int8_t conv_zero_page[256];

// One output tile is 32 rows x (4 waves x TN x 32) columns; every wave holds all L limb tiles of the
// 32 rows for its TN column tiles (one wave per SIMD, accumulators in the AGPRs).  A block takes
// `units_per_block` consecutive row tiles of one column tile (and one piece of the contraction) and
// runs them as ONE sequence of K-tile steps: the loads and conversions for the first K-tiles of the
// next row tile are already under way while the last K-tile of the current one is multiplied, so the
// start-up of a block (plan and argument loads, first G latency from HBM, LDS fill: about 9 us,
// measured) is paid once per block instead of once per output tile.  Per K-tile of 128 contraction
// entries:
//   A side: 16 entries of G per thread -> registers -> digits -> L planes [32][128] int8 in LDS;
//   B side: direct global->LDS loads of the index matrix rows (16-byte chunks, XOR-swizzled).
// Two LDS stages and two register sets for G.  While the MFMAs of step s run (four k-steps of L*TN
// MFMAs), the same wave
//   k-steps 0, 1: turns G(s+1), loaded two steps ago, into digit words (VALU only) and issues the second
//                 half of the direct loads of B(s+1),
//   k-step 2:     writes the digits to the other stage and issues the loads of G(s+3),
//   barrier       (step s+1 complete in LDS for everyone, every read of step s issued and done),
//   k-step 3:     reads the first fragments of step s+1 and issues the first half of the direct loads of
//                 B(s+2) into the stage step s has just left;
//   after the last K-tile of a row tile: recombination of the limbs and the stores of that tile.
// A wave runs its instructions in order: an MFMA occupies the matrix pipe for 32 cycles and about seven
// VALU or LDS instructions issued behind it are free (measured), more are not.  Hence the recipe per
// k-step below, which hands the scheduler the numbers of LDS, memory and VALU instructions per MFMA.
// Every k-step is one basic block: loads never branch (addresses are clamped, the index matrix is
// zero beyond the contraction length, so whatever G value is read there multiplies a zero), which
// lets the scheduler put the VALU and LDS work into the shadow of the MFMAs.
// TRANS: G is read transposed (rows of the product are columns of G).  VEC: 16-byte loads of G
// (N % 4 == 0).
template <int L, int TN, bool TRANS, bool VEC, bool LONG_RUNS, bool QUANT = false>
__device__ __forceinline__ void limb_gemm_body(const LimbArgs &a, int8_t *lds, float gscale, double out_scale, int block)
{
    constexpr int NB = 4 * TN * 32;
    constexpr int STAGE = L * kLPlane + NB * kLBK;
    constexpr int WLB = NB / 32;          // direct loads per wave per K-tile
    constexpr int GL = VEC ? 4 : 16;      // G load instructions per thread per K-tile
    constexpr int NM = L * TN;            // MFMAs per k-step

    // RUNS: a block takes `units_per_block` consecutive row tiles and, for each of them, every column tile
    // in turn (the rows of G just read for one column tile are still in L2 for the next).  With five or six
    // limbs the accumulators fill the AGPRs and a write-out inside the loop makes the register allocator
    // spill in the k-steps: then, and when the launcher does not ask for runs, a block takes one row tile
    // and one column tile and writes it after the loop.
    constexpr bool RUNS = LONG_RUNS && L <= 4;
    const int tiles_c = (a.cols + NB - 1) / NB;
    const int R = RUNS ? a.units_per_block : 1;
    const int runs = (a.tiles_r + R - 1) / R;        // runs of row tiles per contraction piece
    const int c_per_block = RUNS ? tiles_c : 1;
    // Workgroups go to the eight XCDs round-robin: XCD x takes the x-th eighth of the work items, so that
    // neighbouring items (neighbouring rows of G, same K-tiles of the index matrix) share an L2.  The grid
    // may hold more blocks than items (it is sized before the limb count is known).
    const int64_t items = (int64_t)runs * (tiles_c / c_per_block) * a.splits;
    const int64_t per_xcd = (items + 7) >> 3;
    const int64_t slot = (int64_t)(block >> 3);
    const int64_t logical = (int64_t)(block & 7) * per_xcd + slot;
    if (slot >= per_xcd || logical >= items) return;
    const int c_begin = RUNS ? 0 : (int)(logical % tiles_c);
    const int64_t rest = RUNS ? logical : logical / tiles_c;
    const int run = (int)(rest % runs);
    const int split = (int)(rest / runs);
    const int nk_total = a.nk;
    const int kt0 = split * a.kt_per_split;
    const int nk = min(nk_total, kt0 + a.kt_per_split) - kt0;   // K-tiles per output tile (at least one)
    const int tile_r0 = run * R;
    const int U = min(R, a.tiles_r - tile_r0);                   // row tiles of this block
    const int S = U * c_per_block * nk;                          // steps

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- A side ----
    // Each thread owns four groups q = 0..3 of four consecutive contraction entries (one float4 of G, or
    // one column of a 4 x 4 patch of G^T), laid out so that one load instruction of a wave covers whole
    // 128-byte lines of G:
    // !TRANS: group q is row 8 q + tid / 32, entries 4 (tid % 32) .. +3
    //  TRANS: the patch is rows 4 t .. +3 by entries 4 j .. +3 with t = 0..7 and j = 0..7 inside the wave, j + 8 * wave in the
    //         block; group q is its row q.  t takes tid bits 0, 1 and 5, j bits 2..4: a half-wave then holds four values of
    //         t (four different swizzles) and all eight j (two chunks x four words), i.e. 32 different LDS banks when the
    //         digits are stored (with t in bits 0..2 rows t and t + 4 met in every bank: 19 % conflict cycles, measured).
    float gbuf[2][16];
    const int tr_t = (tid & 3) | ((tid >> 3) & 4), tr_j = ((tid >> 2) & 7) + 8 * (tid >> 6);
    const int ar = TRANS ? 4 * tr_t : (tid >> 5);            // row of group 0
    const int ak = TRANS ? 4 * tr_j : 4 * (tid & 31);        // first contraction entry inside the K-tile
    // (every address inside a tile is clamped to the matrix)
    // (r, kt): row tile inside the block and K-tile inside the contraction piece, both valid
    auto load_g = [&](float (&g)[16], int r, int kt) {
        const int row0 = (tile_r0 + r) * kLRows;
        const int k0 = (kt0 + kt) * kLBK + ak;
        if (!TRANS) {
            // g[4 q + e] = G[row0 + ar + 8 q][k0 + e]
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float *p = a.G + (int64_t)min(row0 + ar + 8 * q, a.rows - 1) * a.N;
                if (VEC) {
                    const float4 v = *reinterpret_cast<const float4 *>(p + min(k0, a.kc - 4));
                    g[4 * q] = v.x; g[4 * q + 1] = v.y; g[4 * q + 2] = v.z; g[4 * q + 3] = v.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) g[4 * q + e] = p[min(k0 + e, a.kc - 1)];
                }
            }
        } else {
            // g[4 e + q] = G[k0 + e][row0 + ar + q]
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float *p = a.G + (int64_t)min(k0 + e, a.kc - 1) * a.N;
                if (VEC) {
                    const float4 v = *reinterpret_cast<const float4 *>(p + min(row0 + ar, a.rows - 4));
                    g[4 * e] = v.x; g[4 * e + 1] = v.y; g[4 * e + 2] = v.z; g[4 * e + 3] = v.w;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) g[4 * e + q] = p[min(row0 + ar + q, a.rows - 1)];
                }
            }
        }
    };
    // digit words of the four groups, w[q][l] = digit l of the group's four entries; two groups at a time
    uint32_t w[4][L];
    auto convert_half = [&](const float (&g)[16], int h) {
#pragma unroll
        for (int q = 2 * h; q < 2 * h + 2; ++q) {
            if constexpr (QUANT) {
                // the "digits" are the level indices of the quantizer (one plane): the forward product with the
                // quantizer in its prologue
                w[q][0] = pack_indices((int)anchor_level<true>(g[4 * q], a.fq_k), (int)anchor_level<true>(g[4 * q + 1], a.fq_k),
                                       (int)anchor_level<true>(g[4 * q + 2], a.fq_k), (int)anchor_level<true>(g[4 * q + 3], a.fq_k),
                                       a.fq_k.idx_off);
            } else if constexpr (!TRANS) {
                const float g4[4] = {g[4 * q], g[4 * q + 1], g[4 * q + 2], g[4 * q + 3]};
                limbs_of4<L>(g4, gscale, w[q]);
            } else {
                const float g4[4] = {g[q], g[4 + q], g[8 + q], g[12 + q]};
                limbs_of4<L>(g4, gscale, w[q]);
            }
        }
    };
    // where the word of group q goes inside a plane: row * 128 + (swizzled 16-byte chunk) + word in chunk.
    // The rows of a thread's groups are 8 apart from a row below 8 (!TRANS: the swizzle of rows +8, +24 is
    // that of row +0 with bit 2 flipped) or consecutive from a multiple of 4 (TRANS: rows +2, +3 flip bit 0).
    const int aw_row = ar * kLBK + ((ak >> 2) & 3) * 4;
    const int aw_chunk = ((ak >> 4) ^ lswz(ar)) << 4;
    auto store_digits = [&](int stage) {
        int8_t *base = lds + stage * STAGE + aw_row;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int8_t *d = TRANS ? base + (q >> 1 ? aw_chunk ^ 16 : aw_chunk) + q * kLBK
                              : base + (q & 1 ? aw_chunk ^ 64 : aw_chunk) + q * 8 * kLBK;
#pragma unroll
            for (int l = 0; l < L; ++l) *reinterpret_cast<uint32_t *>(d + l * kLPlane) = w[q][l];
        }
    };

    // ---- B side: a uniform base per (column tile, K-tile) and a 32-bit offset per lane.  Load i of a wave
    // covers rows brow + 8 i of the column tile (clamped to the matrix), lane % 8 picks the 16-byte chunk,
    // XOR-swizzled with the row: the swizzle of row brow + 8 i is that of brow with bit 2 flipped for odd i. ----
    const int brow = wave * (WLB * 8) + (lane >> 3);
    const int bq16 = ((lane & 7) ^ lswz(brow)) << 4;
    const uint32_t ldb32 = (uint32_t)a.ldb;
    // half h of the direct loads of K-tile kt of column tile c: a wave that issues all of them back to back
    // outruns the address unit (1 KiB per instruction, 64 bytes per cycle per CU) and stalls behind its own loads
    auto issue_b = [&](int stage, int c, int kt, int h) {
        int8_t *base = lds + stage * STAGE + L * kLPlane + wave * (WLB * 1024);
        const int col0 = (c_begin + c) * NB;
        const int8_t *src = a.Bt + (int64_t)col0 * a.ldb + (int64_t)(kt0 + kt) * kLBK;
        const int lim = a.cols - 1 - col0;
#pragma unroll
        for (int i = h * (WLB / 2); i < (h + 1) * (WLB / 2); ++i) {
            const uint32_t off = (uint32_t)min(brow + 8 * i, lim) * ldb32 + (uint32_t)(i & 1 ? bq16 ^ 64 : bq16);
            __builtin_amdgcn_global_load_lds((gptr_t)(src + off), (lptr_t)(base + i * 1024), 16, 0, 0);
        }
    };

    // ---- fragments ----
    const int frow = lane & 31;
    const int fsw = lswz(frow);
    const int fa_off = frow * kLBK;
    const int fb_off = L * kLPlane + (wave * TN * 32 + frow) * kLBK;   // row 32 t + frow swizzles like frow
    int fc[4];                                                         // the 32-byte slice of k-step ks, per lane half
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) fc[ks] = ((2 * ks + (lane >> 5)) ^ fsw) << 4;

    v4i fa[2][L], fb[2][TN];
    auto read_frags = [&](int buf, int stage, int ks) {
        const int8_t *base = lds + stage * STAGE + fc[ks];
#pragma unroll
        for (int l = 0; l < L; ++l) fa[buf][l] = *reinterpret_cast<const v4i *>(base + l * kLPlane + fa_off);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[buf][j] = *reinterpret_cast<const v4i *>(base + fb_off + j * 32 * kLBK);
    };

    v16i acc[L][TN];
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[l][j][r] = 0;
    auto mfma_all = [&](int buf) {
#pragma unroll
        for (int l = 0; l < L; ++l)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[l][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[buf][l], fb[buf][j], acc[l][j], 0, 0, 0);
    };

    // a bare s_barrier: the waits it needs are spelled out next to it, so that loads of later tiles stay in flight
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // Scheduling recipe for one k-step: after every MFMA, up to `ds` LDS accesses, `vm` memory loads and
    // `va` VALU instructions go into its shadow.
#define CDL_INTERLEAVE(ds, vm, va)                                                          \
    _Pragma("unroll") for (int i_ = 0; i_ < NM; ++i_) {                                     \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                  \
        if ((ds) > 0) __builtin_amdgcn_sched_group_barrier(0x080, (ds), 0);                 \
        if ((vm) > 0) __builtin_amdgcn_sched_group_barrier(0x020, (vm), 0);                 \
        if ((va) > 0) __builtin_amdgcn_sched_group_barrier(0x002, (va), 0);                 \
    }
    constexpr int kDs2 = (L + TN + 4 * L + NM - 1) / NM;    // k-step 2: fragment reads + digit writes
    constexpr int kVm2 = (GL + NM - 1) / NM;
    // VALU instructions per MFMA: enough slots for the k-step's conversion work, spread as evenly as the
    // count allows (12 MFMAs and about 30 VALU instructions with up to four limbs: three each measured 2-3 %
    // faster than five, two slower; 15 MFMAs and the longer conversion of five limbs: five, four in the
    // k-steps that convert nothing)
    constexpr int kVaConv = L <= 4 ? 3 : 5, kVaRest = L <= 4 ? 3 : 4;

    // ---- recombination of the limbs of row tile u: the integers are exact, the Horner steps round at
    // 2^-53 relative.  (The lane index passes through an empty asm so that the output addresses are formed
    // here instead of being kept in registers all the way through the loop.) ----
    auto write_tile = [&](int r, int c) {
        int elane = lane;
        asm volatile("" : "+v"(elane));
        const int row0 = (tile_r0 + r) * kLRows, col0 = (c_begin + c) * NB;
        const int erow = row0 + 4 * (elane >> 5), ecol = col0 + wave * TN * 32 + (elane & 31);
        const bool full = row0 + kLRows <= a.rows && col0 + NB <= a.cols;
        // register rr of an accumulator is row 8 (rr / 4) + rr % 4 (+ 4 for the upper half of the lanes)
        auto combined = [&](int j, int rr) {
            double run = (double)acc[L - 1][j][rr];
#pragma unroll
            for (int l = L - 2; l >= 0; --l) run = __builtin_fma(run, 256.0, (double)acc[l][j][rr]);   // run * 256 is exact
            return run;
        };
        // one address per row, the TN column tiles of a wave at fixed distances from it; tiles that do not reach
        // the edge of the matrix (FULL) store without a test
        const int64_t first = (int64_t)erow * a.cols + ecol;
        const bool direct = a.splits == 1;                       // the block writes the finished fp32 output itself
        const bool corr = a.row_corr != nullptr && direct;
        // CORR: row corrections of an operand stored with an offset, in a copy of the write-out of their own.  A load
        // between the stores - even one that a branch skips - makes the compiler wait for every earlier store at each
        // row (loads and stores share one counter) and a store takes microseconds to complete: the common path must
        // not contain one (it cost dL/dQ(x) 5 %).  The copy with corrections loads one per row and pays for it; holding
        // all sixteen in registers instead pushed the five-limb kernels into spilling.
        auto emit = [&](auto full_c, auto corr_c, auto *base) {
            constexpr bool FULL = decltype(full_c)::value;
            constexpr bool CORR = decltype(corr_c)::value;
            using T = std::remove_pointer_t<decltype(base)>;
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                const int dr = 8 * (rr >> 2) + (rr & 3);
                T *p = base + (int64_t)dr * a.cols;
                const bool row_ok = FULL || erow + dr < a.rows;
                const double rc = (CORR && row_ok) ? a.row_corr[erow + dr] : 0.0;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if (FULL || (row_ok && ecol + j * 32 < a.cols)) {
                        if (QUANT) p[j * 32] = (T)(a.fq_scale * (float)acc[0][j][rr]);      // as the forward product rounds
                        else if (std::is_same<T, float>::value) p[j * 32] = (T)__builtin_fma(combined(j, rr), out_scale, rc);
                        else p[j * 32] = (T)combined(j, rr);
                    }
                }
            }
        };
        if (direct) {
            if (corr) {
                if (full) emit(std::true_type{}, std::true_type{}, a.out + first);
                else emit(std::false_type{}, std::true_type{}, a.out + first);
            } else {
                if (full) emit(std::true_type{}, std::false_type{}, a.out + first);
                else emit(std::false_type{}, std::false_type{}, a.out + first);
            }
        } else {
            double *base = a.partial + (int64_t)split * a.rows * a.cols + first;
            if (full) emit(std::true_type{}, std::false_type{}, base);
            else emit(std::false_type{}, std::false_type{}, base);
        }
    };

    // positions of the steps s, s+1, s+2, s+3 in the block's sequence: (row tile, column tile, K-tile), the
    // K-tile running fastest; past the end they stay on the last valid step (such loads go to registers or
    // to an LDS stage nobody reads)
    struct Pos { int r, c, kt; };
    auto advance = [&](Pos &q) {
        if (q.kt < nk - 1) { ++q.kt; }
        else if (q.c < c_per_block - 1) { q.kt = 0; ++q.c; }
        else if (q.r < U - 1) { q.kt = 0; q.c = 0; ++q.r; }
    };
    Pos p0{0, 0, 0}, p1 = p0;
    advance(p1);
    Pos p2 = p1;
    advance(p2);
    Pos p3 = p2;
    advance(p3);

    // k-step 0 of a step; FIRST: the first K-tile of a row tile starts from zero accumulators
    auto kstep0 = [&](auto parity, auto first) {
        constexpr int P = decltype(parity)::value;
        constexpr bool FIRST = decltype(first)::value;
        read_frags(1, P, 1);
        issue_b(P ^ 1, p1.c, p1.kt, 1);
        convert_half(gbuf[P ^ 1], 0);
        if (FIRST) {
            const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int l = 0; l < L; ++l)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[l][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[0][l], fb[0][j], zero, 0, 0, 0);
        } else {
            mfma_all(0);
        }
        CDL_INTERLEAVE(1, 1, kVaConv)
        __builtin_amdgcn_sched_barrier(0);
    };
    // one step (its parity P picks the LDS stage and the register set of G) under the schedule above
    auto step = [&](auto parity) {
        constexpr int P = decltype(parity)::value;
        // k-step 0
        if (RUNS && p0.kt == 0) kstep0(parity, std::true_type{});
        else kstep0(parity, std::false_type{});
        // k-step 1
        read_frags(0, P, 2);
        convert_half(gbuf[P ^ 1], 1);
        mfma_all(1);
        CDL_INTERLEAVE(1, 0, kVaConv)
        __builtin_amdgcn_sched_barrier(0);
        // k-step 2
        store_digits(P ^ 1);
        read_frags(1, P, 3);
        load_g(gbuf[P ^ 1], p3.r, p3.kt);
        mfma_all(0);
        CDL_INTERLEAVE(kDs2, kVm2, kVaRest)
        __builtin_amdgcn_sched_barrier(0);
        // B(s+1) has landed (younger loads: G(s+3)); own LDS writes and fragment reads are done
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(GL));
        __builtin_amdgcn_s_waitcnt(kLgkmcnt0);
        barrier();
        // k-step 3
        read_frags(0, P ^ 1, 0);
        issue_b(P, p2.c, p2.kt, 0);
        mfma_all(1);
        CDL_INTERLEAVE(1, 1, kVaRest)
        __builtin_amdgcn_sched_barrier(0);
        if (RUNS && p0.kt == nk - 1) write_tile(p0.r, p0.c);
        advance(p0);
        advance(p1);
        advance(p2);
        advance(p3);
    };

    load_g(gbuf[0], p0.r, p0.kt);
    load_g(gbuf[1], p1.r, p1.kt);
    issue_b(0, p0.c, p0.kt, 0);
    issue_b(0, p0.c, p0.kt, 1);
    convert_half(gbuf[0], 0);
    convert_half(gbuf[0], 1);
    store_digits(0);
    asm volatile("" ::: "memory");
    load_g(gbuf[0], p2.r, p2.kt);
    issue_b(1, p1.c, p1.kt, 0);
    asm volatile("" ::: "memory");
    // B(0) has landed (younger loads: G(2), the first half of B(1)); own LDS writes are done
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(GL + WLB / 2));
    __builtin_amdgcn_s_waitcnt(kLgkmcnt0);
    barrier();
    read_frags(0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    int st = 0;
    for (; st + 1 < S; st += 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
    if (st < S) step(std::integral_constant<int, 0>{});
    // the loads issued for steps past the end write LDS: they must be done before this wave ends
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#undef CDL_INTERLEAVE
    if (!RUNS) write_tile(0, 0);
}

template <bool TRANS, bool LONG_RUNS>
__global__ __launch_bounds__(kLThreads, 1)
void limb_gemm_kernel(LimbArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t limb_lds[];
    const bool vec = (a.N & 3) == 0;
    const int limbs = a.which == 0 ? a.plan->limbs_da : a.plan->limbs_db;
    const float gscale = a.which == 0 ? a.plan->gscale_da : a.plan->gscale_db;
    const double out_scale = a.which == 0 ? a.plan->out_scale_da : a.plan->out_scale_db;
    switch (limbs) {
        case 3: if (vec) limb_gemm_body<3, 3, TRANS, true, LONG_RUNS>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); else limb_gemm_body<3, 3, TRANS, false, LONG_RUNS>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
        case 4: if (vec) limb_gemm_body<4, 3, TRANS, true, LONG_RUNS>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); else limb_gemm_body<4, 3, TRANS, false, LONG_RUNS>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
        case 5: if (vec) limb_gemm_body<5, 3, TRANS, true, false>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); else limb_gemm_body<5, 3, TRANS, false, false>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
        default: if (vec) limb_gemm_body<6, 2, TRANS, true, false>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); else limb_gemm_body<6, 2, TRANS, false, false>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
    }
}

// Output matrices of few columns: tiles of 128 (TN = 1) or 256 columns (TN = 2) instead of 384, for N % 4 == 0.  The
// conversion of g costs the same whatever the width, 0.55 and 0.73 of a K-tile's time in all (limb_tile_width).  With one column tile per wave
// a K-tile has only 4 L MFMAs per wave, fewer cycles than a load takes to come back, so that kernel is held to 256
// registers and 80 KiB of LDS: two blocks share a compute unit and fill each other's waits.
constexpr int limb_narrow_lds_bytes(int tn) { return 2 * (kMaxLimbs * kLPlane + 4 * tn * 32 * kLBK); }

template <int TN, bool TRANS, bool LONG_RUNS>
__global__ __launch_bounds__(kLThreads, TN == 1 ? 2 : 1)
void limb_narrow_kernel(LimbArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t limb_lds[];
    const int limbs = a.which == 0 ? a.plan->limbs_da : a.plan->limbs_db;
    const float gscale = a.which == 0 ? a.plan->gscale_da : a.plan->gscale_db;
    const double out_scale = a.which == 0 ? a.plan->out_scale_da : a.plan->out_scale_db;
    switch (limbs) {
        case 3: limb_gemm_body<3, TN, TRANS, true, LONG_RUNS>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
        case 4: limb_gemm_body<4, TN, TRANS, true, LONG_RUNS>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
        case 5: limb_gemm_body<5, TN, TRANS, true, false>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
        default: limb_gemm_body<6, TN, TRANS, true, false>(a, limb_lds, gscale, out_scale, (int)blockIdx.x); break;
    }
}

// Both products of a small layer in one launch, one tile per block: neither fills the chip, and side by side they take the
// time of the longer one.
__global__ __launch_bounds__(kLThreads, 1)
void limb_pair_kernel(LimbArgs a, LimbArgs b, int blocks_a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t limb_lds[];
    const bool vec = (a.N & 3) == 0, first = (int)blockIdx.x < blocks_a;
    const BwdPlan *plan = a.plan;
    const int limbs = first ? plan->limbs_da : plan->limbs_db, block = first ? (int)blockIdx.x : (int)blockIdx.x - blocks_a;
    const float gscale = first ? plan->gscale_da : plan->gscale_db;
    const double out_scale = first ? plan->out_scale_da : plan->out_scale_db;
#define CDL_PAIR(L, TN)                                                                                                        \
    if (first) { if (vec) limb_gemm_body<L, TN, false, true, false>(a, limb_lds, gscale, out_scale, block);                    \
                 else limb_gemm_body<L, TN, false, false, false>(a, limb_lds, gscale, out_scale, block); }                     \
    else { if (vec) limb_gemm_body<L, TN, true, true, false>(b, limb_lds, gscale, out_scale, block);                           \
           else limb_gemm_body<L, TN, true, false, false>(b, limb_lds, gscale, out_scale, block); }
    switch (limbs) {
        case 3: CDL_PAIR(3, 3) break;
        case 4: CDL_PAIR(4, 3) break;
        case 5: CDL_PAIR(5, 3) break;
        default: CDL_PAIR(6, 2) break;
    }
#undef CDL_PAIR
}

// The plan of a backward call, made by the last block of the launch that forms the column sums (a launch of its own
// took 5 us).  The flag of a block goes up when its sums have arrived; see cdl_finish.h.
struct PlanArgs {
    BwdPlan *plan;
    const unsigned int *block_max;
    int n_max;
    const unsigned int *col_abs_a, *col_abs_b;
    int n_abs_a, n_abs_b;
    float delta_a, delta_b;
    unsigned long long *flags;     // [blocks]
    unsigned long long tag;
};
constexpr int kPlanMaxBlocks = 4096;

// all 256 threads of block `self` of `blocks`
__device__ __forceinline__ void plan_at_end(const PlanArgs &a, int self, int blocks)
{
    if (!a.plan) return;      // (more blocks than flags: a launch of its own follows)
    __shared__ unsigned int red[3][4];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (self != blocks - 1) {
        if (threadIdx.x == 0) device_store(a.flags + self, a.tag);
        return;
    }
    for (int base = 0; base < blocks - 1; base += 8 * 256) {
        bool waiting = true;
        while (waiting) {
            waiting = false;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = base + u * 256 + (int)threadIdx.x;
                if (i < blocks - 1 && device_load(a.flags + i) != a.tag) waiting = true;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * 256 + (int)threadIdx.x;
            if (i < blocks - 1) device_store(a.flags + i, 0ull);
        }
    }
    asm volatile("" ::: "memory");
    __syncthreads();
    unsigned int v[3] = {0u, 0u, 0u};
#pragma unroll 8
    for (int i = threadIdx.x; i < a.n_max; i += 256) v[0] = max(v[0], a.block_max[i]);
    auto sums = [&](const unsigned int *p, int n, unsigned int &m) {
#pragma unroll 8
        for (int i = threadIdx.x; i < n; i += 256) m = max(m, __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    sums(a.col_abs_a, a.n_abs_a, v[1]);
    sums(a.col_abs_b, a.n_abs_b, v[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[q] = max(v[q], (unsigned int)__shfl_xor((int)v[q], off, 64));
        if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = v[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = max(max(red[q][0], red[q][1]), max(red[q][2], red[q][3]));
        choose_limbs(a.plan, v[0], v[1], v[2], a.delta_a, a.delta_b);
    }
}

// dL/dQ(x) of a convolutional layer (cdl_conv_dx.hip): the weights [N][R][S][C] rearranged as its index operand
// Wr[(r', s', n) / 64][c][64], every tap's channels padded with zeros to Np (zero beyond the contraction length, up to ld) and the sum of |w| over the contraction per
// channel c (the limb rule's column sums).  One rearrangement per class of taps (blockIdx.y): the taps
// (r0 + tstep r', s0 + tstep s') with r' < Rc, s' < Sc - all of them for stride 1 (one class, tstep = 1), those of one
// parity for stride 2.
struct ConvDxClass { int r0, s0, Rc, Sc; };
struct ConvDxClasses { ConvDxClass c[4]; int tstep; };

struct ConvDxWeights {
    const int8_t *w;
    int N, Np, R, S, C;
    ConvDxClasses cls;
    int8_t *wr;
    int64_t ld;
};

// A block turns 64 contraction entries (bx) x 64 channels (by) of one class (bz): rows of 64 channels are contiguous in w, 64 entries of a channel in
// wr (PATCH: 1 KB for 32 contraction entries of 32 channels, [half of the entries][channel][16]).  Returns, to four threads each, the sum of |w| over the entries of
// channel 64 by + threadIdx.x / 4.
template <bool PATCH>
__device__ __forceinline__ unsigned int rearrange_weights(const ConvDxWeights &a, int bx, int by, int bz)
{
    __shared__ int8_t tile[64][68];
    const int N = a.N, Np = a.Np, R = a.R, S = a.S, C = a.C;
    const int8_t *w = a.w;
    const ConvDxClass k_ = a.cls.c[bz];
    const int kc = k_.Rc * k_.Sc * Np, k0 = bx * 64, c0 = by * 64;
    const float inv_np = 1.0f / (float)Np, inv_s = 1.0f / (float)k_.Sc;
    {
        const int c = threadIdx.x & 63, part = threadIdx.x >> 6;
        int8_t v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            // (k < 2^17: (k + 1/2) / Np in fp32 is far enough from a whole number to truncate to the quotient)
            const int k = k0 + 4 * e + part, kk = min(k, kc - 1), tap = (int)(((float)kk + 0.5f) * inv_np), nn = kk - tap * Np, n = min(nn, N - 1);
            const int tr = (int)(((float)tap + 0.5f) * inv_s), ts = tap - tr * k_.Sc;
            const int r = k_.r0 + a.cls.tstep * tr, sx = k_.s0 + a.cls.tstep * ts;
            const int8_t x = w[(((int64_t)n * R + r) * S + sx) * C + min(c0 + c, C - 1)];
            v[e] = k < kc && nn < N ? x : (int8_t)0;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) tile[c][4 * e + part] = v[e];
    }
    __syncthreads();
    const int c = threadIdx.x >> 2, q = threadIdx.x & 3;
    unsigned int s_abs = 0u;
    uint32_t word[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        word[i] = *reinterpret_cast<const uint32_t *>(&tile[c][16 * q + 4 * i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int x = (int)(int8_t)(word[i] >> (8 * e));
            s_abs += (unsigned int)(x < 0 ? -x : x);
        }
    }
    s_abs += (unsigned int)__shfl_xor((int)s_abs, 1, 64);
    s_abs += (unsigned int)__shfl_xor((int)s_abs, 2, 64);
    if (c0 + c < C) {
        const int C32 = (C + 31) & ~31, ch = c0 + c;
        int8_t *dst = PATCH ? a.wr + (int64_t)bz * C32 * a.ld + (((int64_t)(2 * bx + (q >> 1)) * (C32 >> 5) + (ch >> 5)) * 64 + (q & 1) * 32 + (ch & 31)) * 16
                            : a.wr + (int64_t)bz * C * a.ld + ((int64_t)bx * C + ch) * 64 + 16 * q;
        *reinterpret_cast<uint4 *>(dst) = uint4{word[0], word[1], word[2], word[3]};
    }
    return s_abs;
}

__global__ __launch_bounds__(256)
void conv_dx_prep_kernel(ConvDxWeights a, unsigned int *col_abs /* zeroed */, PlanArgs plan)
{
    const unsigned int s_abs = rearrange_weights<false>(a, blockIdx.x, blockIdx.y, blockIdx.z);
    const int ch = blockIdx.y * 64 + (threadIdx.x >> 2);
    if ((threadIdx.x & 3) == 0 && ch < a.C) __hip_atomic_fetch_add(&col_abs[blockIdx.z * a.C + ch], s_abs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    plan_at_end(plan, (int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x), (int)(gridDim.x * gridDim.y * gridDim.z));
}

// What the kernel on patches needs (cdl_conv_patch.hip), in one launch: blocks 0 .. nx ny nz - 1 rearrange the weights, and the last block of every 64
// channels of a class adds up the column sums of |w| of its blocks and leaves the largest; the others take the largest |g| of every
// pixel (as the bits of a float), and of all their pixels.  Waiting is for lower blocks only (cdl_finish.h).  15 us for
// 51 MB of g and 0.6 MB of weights; in two launches 11 + 8.
struct PatchPrep {
    ConvDxWeights weights;
    int nx, ny, nz;
    unsigned int *part;                // [nz][nx][C]
    unsigned long long *flags;         // [nz][ny][nx]
    unsigned long long tag;
    unsigned int *col_max;             // [nz][ny]
    const float *g;
    int pixels, N, log_t;              // N a multiple of 4; 2^log_t lanes to a pixel
    unsigned int *pixel_max, *block_max;
};

__global__ __launch_bounds__(256)
void conv_patch_prep_kernel(PatchPrep a)
{
    __shared__ unsigned int red[4];
    const int prep = a.nx * a.ny * a.nz;
    auto block_largest = [&](unsigned int v) {      // thread 0 has it
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned int)__shfl_xor((int)v, off, 64));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        return max(max(red[0], red[1]), max(red[2], red[3]));
    };
    if ((int)blockIdx.x < prep) {
        const int bx = blockIdx.x % a.nx, bg = blockIdx.x / a.nx, by = bg % a.ny, bz = bg / a.ny, C = a.weights.C;
        const unsigned int s_abs = rearrange_weights<true>(a.weights, bx, by, bz);
        const int ch = by * 64 + (threadIdx.x >> 2);
        if ((threadIdx.x & 3) == 0 && ch < C) __hip_atomic_store(&a.part[((int64_t)bz * a.nx + bx) * C + ch], s_abs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        unsigned long long *flags = a.flags + (int64_t)bg * a.nx;
        if (bx != a.nx - 1) {
            if (threadIdx.x == 0) device_store(flags + bx, a.tag);
            return;
        }
        for (int i = threadIdx.x; i < a.nx - 1; i += 256) {
            while (device_load(flags + i) != a.tag) {}
            device_store(flags + i, 0ull);
        }
        asm volatile("" ::: "memory");
        __syncthreads();
        // four threads to a channel
        unsigned int sum = 0u;
        if (ch < C)
#pragma unroll 8
            for (int i = threadIdx.x & 3; i < a.nx; i += 4) sum += __hip_atomic_load(&a.part[((int64_t)bz * a.nx + i) * C + ch], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sum += (unsigned int)__shfl_xor((int)sum, 1, 64);
        sum += (unsigned int)__shfl_xor((int)sum, 2, 64);
        const unsigned int most = block_largest(sum);
        if (threadIdx.x == 0) a.col_max[bg] = most;
        return;
    }
    // four pixels at a time, two trips of loads under way
    constexpr int U = 4;
    const int self = blockIdx.x - prep, blocks = gridDim.x - prep, log_t = a.log_t;
    const int quads = a.N >> 2, own = threadIdx.x & ((1 << log_t) - 1), group = threadIdx.x >> log_t, per = 256 >> log_t;
    unsigned int all = 0u;
    for (int p0 = self * per * U + group; p0 < a.pixels; p0 += blocks * per * U) {
        const float4 *src[U];
        unsigned int m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            src[u] = reinterpret_cast<const float4 *>(a.g + (int64_t)min(p0 + u * per, a.pixels - 1) * a.N);
            m[u] = 0u;
        }
#pragma unroll 2
        for (int q = own; q < quads; q += 1 << log_t) {
            float4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = src[u][q];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                m[u] = max(m[u], max(__float_as_uint(fabsf(v[u].x)), __float_as_uint(fabsf(v[u].y))));
                m[u] = max(m[u], max(__float_as_uint(fabsf(v[u].z)), __float_as_uint(fabsf(v[u].w))));
            }
        }
        for (int off = 1 << log_t >> 1; off > 0; off >>= 1)
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = max(m[u], (unsigned int)__shfl_xor((int)m[u], off, 64));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (own == 0 && p0 + u * per < a.pixels) a.pixel_max[p0 + u * per] = m[u];
            all = max(all, m[u]);
        }
    }
    const unsigned int most = block_largest(all);
    if (threadIdx.x == 0) a.block_max[self] = most;
}

// The forward product with the quantizer of the activations in its prologue: y = delta_a delta_b (Q_idx(X) . Wi^T)
// where Q_idx(X) - the level indices cdl_quantize_fwd would store - exists only as one int8 plane per K-tile in LDS.
// The limb kernel's loop with the conversion to digits replaced by the nearest-level rule, one plane, four column
// tiles per wave (512 columns per block), runs of row tiles per block.
constexpr int kQuantFwdTN = 4;
static_assert(2 * (kLPlane + 4 * kQuantFwdTN * 32 * kLBK) <= kLimbLdsBytes, "LDS of the limb kernels serves");

__global__ __launch_bounds__(kLThreads, 1)
void qgemm_quantize_fwd_kernel(LimbArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t limb_lds[];
    limb_gemm_body<1, kQuantFwdTN, false, true, true, true>(a, limb_lds, 0.0f, 0.0, (int)blockIdx.x);
}

// out = out_scale * sum over the contraction splits.  Four partial sums per lane, combined in a fixed order,
// keep four loads in flight: with a few hundred splits a single dependent chain is all latency.  LANES lanes
// share one output (lane j takes the splits j, j + LANES, ...; butterfly over the lanes at the end): used
// when there are few outputs and many splits, where one lane per output leaves most of the chip idle.
template <int LANES>
__global__ __launch_bounds__(256)
void limb_reduce_kernel(const double *__restrict__ partial, int splits, int64_t n, const BwdPlan *plan, float *__restrict__ out,
                        const double *__restrict__ row_corr /* [n / cols] or null */, int cols)
{
    const double out_scale = plan->out_scale_db;
    const int sub = threadIdx.x % LANES;
    const int64_t per_block = 256 / LANES;
    // whole groups of LANES run every trip (the index is clamped), so that the shuffles see all their lanes
    const int64_t n_round = (n + per_block - 1) / per_block * per_block;
    for (int64_t i = (int64_t)blockIdx.x * per_block + threadIdx.x / LANES; i < n_round; i += (int64_t)gridDim.x * per_block) {
        const int64_t ii = i < n ? i : n - 1;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        int p = sub;
        for (; p + 3 * LANES < splits; p += 4 * LANES) {
            s0 += partial[(int64_t)p * n + ii];
            s1 += partial[(int64_t)(p + LANES) * n + ii];
            s2 += partial[(int64_t)(p + 2 * LANES) * n + ii];
            s3 += partial[(int64_t)(p + 3 * LANES) * n + ii];
        }
        for (; p < splits; p += LANES) s0 += partial[(int64_t)p * n + ii];
        double s = (s0 + s1) + (s2 + s3);
#pragma unroll
        for (int off = LANES / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (sub == 0 && i < n) out[i] = (float)__builtin_fma(s, out_scale, row_corr ? row_corr[i / cols] : 0.0);
    }
}

// dL/dQ(a) for a very short contraction (N <= 32: the first stages of a small CNN have 16 or 32 output
// channels; up to 64 in long layers of few columns): d_a_hat[m][k] = delta_b * sum_n g[m][n] * b_idx[n][k].  One K-tile of the limb kernel would be
// at least three quarters padding there; here every output is a chain of N multiply-adds in double on the matrix cores: products of a
// float and an int8 are exact in double and N additions round at 2^-53 relative.
// A wave keeps the index values of up to C tiles of 16 columns in registers as doubles and goes over tiles of 16 rows, the entries of g of the next one
// under way.  Quarter q of the wave holds the contraction entries 4 q to 4 q + 3 (and 16 more on), so that a lane's part of a row of g is one load of 16 bytes
// and nothing of the operands passes through LDS.
// Bound by the stores.  us, a thread per two or four columns with the rows of g in LDS, whose reads took as long as the additions / this: 131072 x 16 x 144 (rows, contraction, columns) 26.1 / 20.7,
// 131072 x 32 x 288 136 / 50, 500000 x 32 x 64 186 / 44, 60000 x 16 x 576 53 / 32, 1000 x 16 x 8000 36 / 16, 262144 x 16 x 16 16.1 / 9.5.
constexpr int kDirectMaxN = 32, kDirectWideN = 64;
// Where it serves before bwd_direct_kernel, whose waves take one step of a short contraction each: many outputs, and long ones from fewer on.  us, that / this, alone: 16 entries, 4096 x 256 (rows x columns) 5.3 / 6.9, 16384 x 144 12.6 / 8.0,
// 2048 x 1500 12.9 / 10.7, 65536 x 16 11.9 / 5.0, 32768 x 36 7.0 / 5.4, 131072 x 27 23.6 / 9.2; 32 entries, 8192 x 200 7.9 / 8.2, 16384 x 144 13.1 / 9.5.  With the weight gradient, which that kernel makes in the same launch: 16 entries, 16384 x 144
// 15.9 / 20.2, 50000 x 64 17.3 / 21.3, 2048 x 1500 13.6 / 22.2, 65536 x 16 20.2 / 14.3, 65536 x 60 21.4 / 19.7, 131072 x 9 32.9 / 18.4; 32 entries, 65536 x 36 21.0 / 19.6, 65536 x 60 22.7 / 25.2, 100000 x 40 33.4 / 31.6, 200000 x 9 54.8 / 32.3.
// 33 to 64 entries in long layers of few columns (one wave has all columns; the other kernels' steps are as short, and more of them), us, that / this with the diagnostic words (1.3 - 1.8 us of it alone): alone 64 entries, 65536 x 27 17.7 / 14.6, 131072 x 9 32.2 / 16.3, 400000 x 32 90 / 48.7,
// 65536 x 64 16.6 / 19.0 (without words), 32768 x 36 9.6 / 11.0 (without); 48 entries, 65536 x 64 18.0 / 16.6, 131072 x 144 44.3 / 47.3 (without); 33 entries, 3 M x 32 1633 / 208; both products, 64 entries, 65536 x 27 35.2 / 33.7, 65536 x 48 34.7 / 37.7, 32768 x 27 24.5 / 27.0;
// 48 entries, 65536 x 27 35.3 / 30.7, 65536 x 64 35.9 / 37.1, 400000 x 32 136 / 79.
bool da_direct_preferred(int M, int N, int K, bool both)
{
    if (N > kDirectMaxN) return N <= kDirectWideN && M >= 1 << 16 && (K <= 32 || (N <= 48 && K <= 64 && !both));
    const int64_t outputs = (int64_t)M * K;
    if (outputs >= 1 << 22) return true;
    if (!both) return outputs >= 1 << 21 || (M >= 1 << 15 && outputs >= 1 << 20);
    return M >= 1 << 16 && outputs >= 1 << 20 && (N <= 16 || K <= 40);
}
constexpr int direct_tiles(int nn) { return nn == 16 ? 10 : 4; }     // tiles of 16 columns per wave: 80 and 64 registers of index values, 96 and 128 beyond 32 entries (two waves per SIMD: with four they spill)

// How the outputs are stored.  kDaWords (rows of whole words of four columns; the entry points take aligned tensors only): the index operand comes first in the product and column 4 (i & 3) + (i >> 2) of a tile is its row i, a lane then has
// four neighbouring outputs.  kDaScalars: g first, 16 neighbouring columns per store.  Both write pieces of 64 bytes.  kDaRows, kDaFlat: through LDS and from there as they lie in memory (kDaFlat: rows of any
// length, where a wave has all columns); serial in a wave, but results that don't fit the memory-side cache of 256 MB are written at 4 instead of 2.6 TB/s.
// us, pieces / through LDS: 16 entries, 144 columns, 131072 rows 20.7 / 24.9, 400000 (58 M outputs) 47 / 57, 460000 (66 M) 94 / 72, 1048576 222 / 144; 32 entries, 64 columns, 1 M rows (64 M) 88 / 98; 16 entries, 576 columns, 120000 rows (69 M) 71 / 64;
// rows of any length: 130 columns, 33333 rows (4.3 M) 15.0 / 16.1, 147, 131072 (19 M) 27.3 / 24.7, 75, 600000 (45 M) 50 / 45, 2 M rows 231 / 161.
enum DaStore { kDaWords, kDaScalars, kDaRows, kDaFlat };
bool direct_staged(int64_t outputs, bool words) { return outputs >= (words ? 65000000 : 1 << 24); }
// Waves: two per SIMD (four: 131072 x 16 x 144 20.7 / 21.5, 460000 rows through LDS 72 / 74), four where their tiles in LDS leave room and a trip is short (1 M x 32 x 48 82 / 74, 3 M x 16 x 27 112 / 98).
int direct_waves(bool staged, int col_tiles) { return staged && col_tiles <= 5 ? 4096 : 2048; }

// The diagnostic words of a call whose dL/dQ(a) is formed here.  (The last block waits for the others, all of lower numbers: cdl_finish.h.)
struct DaWords {
    BwdPlan *plan;                 // null: another product follows, and tells
    // beyond 32 entries, where the words tell the limb counts and bounds that limbs would have had (bwd_direct_diag):
    unsigned long long *records;   // [gridDim.x][2]: the blocks' largest |g|, and the first one's of the next line, from which the last block makes the plan; null: no limbs
    unsigned long long tag;
    float delta_a, delta_b;
    unsigned int *col_abs;         // [1]: the largest sum of |index| of a column, for the product that follows; null: none does
};

template <int NN, DaStore STORE>
__global__ __launch_bounds__(256, NN <= 32 ? 4 : 2)
void da_direct_kernel(const float *__restrict__ g, const int8_t *__restrict__ b_idx, int M, int N, int K, int col_tiles /* per wave */, int blocks /* per group of them */,
                      double delta_b, double b_offset, float *__restrict__ out, DaWords words)
{
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int C = direct_tiles(NN), H = NN / 16;
    constexpr bool VEC = STORE == kDaWords || STORE == kDaRows, STAGED = STORE == kDaRows || STORE == kDaFlat;
    extern __shared__ __align__(16) float da_lds[];
    if (words.plan && (NN <= 32 || !words.records) && blockIdx.x == 0 && threadIdx.x == 0) no_limbs(words.plan);
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    const int group = (int)blockIdx.x / blocks, k0 = group * col_tiles * 16;
    const int tiles = min(col_tiles, (K - k0 + 15) / 16);
    const int row_tiles = (M - 1) / 16 + 1, step = blocks * 4;
    int rt = ((int)blockIdx.x - group * blocks) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (NN <= 32 && rt >= row_tiles) return;

    const bool whole = N % 4 == 0;
    unsigned int amax = 0u;
    auto load = [&](int tile, float (&v)[H][4]) {
        const int row = tile * 16 + i;
        const float *src = g + (int64_t)row * N;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int n = 16 * h + 4 * q;
            if (whole) {
                const float4 x = row < M && n < N ? *reinterpret_cast<const float4 *>(src + n) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                v[h][0] = x.x; v[h][1] = x.y; v[h][2] = x.z; v[h][3] = x.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[h][j] = row < M && n + j < N ? src[n + j] : 0.0f;
            }
        }
    };
    float next[H][4];
    load(rt, next);
    double b[C][H][4];
#pragma unroll
    for (int t = 0; t < C; ++t) {
        const int k = k0 + 16 * t + (VEC ? 4 * (i & 3) + (i >> 2) : i);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = 16 * h + 4 * q + j;
                b[t][h][j] = t < tiles && n < N && k < K ? (double)b_idx[(int64_t)n * K + k] + b_offset : 0.0;     // (the level index itself)
            }
    }
    // the largest sum of |index| of a column, from the registers: in the first block's first wave, before its loop (at the end, where the last block waits, 1 us)
    unsigned int columns = 0u;
    if (NN > 32 && blockIdx.x == 0 && threadIdx.x < 64) {
#pragma unroll
        for (int t = 0; t < C; ++t) {
            double sum = 0.0;
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) sum += 16 * h + 4 * q + j < N ? fabs(b[t][h][j] - b_offset) : 0.0;
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            const int k = k0 + 16 * t + (VEC ? 4 * (i & 3) + (i >> 2) : i);
            columns = max(columns, t < tiles && k < K ? (unsigned int)sum : 0u);
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) columns = max(columns, (unsigned int)__shfl_xor((int)columns, off, 64));
        if (words.col_abs && lane == 0) *words.col_abs = columns;
    }
    // the wave's tile of outputs on its way to stores of neighbouring addresses: kDaRows rows of `pitch` words, kDaFlat as in memory (all columns)
    const int pitch = col_tiles * 16 + 4;
    float *const mine = da_lds + (threadIdx.x >> 6) * 16 * pitch;
    int width = 0, row_first = 0, col_first = 0, row_step = 0, col_step = 0;
    if constexpr (STORE == kDaRows) {      // (rows of whole words: every group has one at least)
        width = min(col_tiles * 4, (K - k0) >> 2);
        row_first = lane / width; col_first = lane - row_first * width;
        row_step = 64 / width; col_step = 64 - row_step * width;
    }
    for (; rt < row_tiles; rt += step) {
        double gv[H][4];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                gv[h][j] = (double)next[h][j];
                if (NN > 32) amax = max(amax, __float_as_uint(next[h][j]) & 0x7fffffffu);
            }
        if (rt + step < row_tiles) load(rt + step, next);
#pragma unroll
        for (int t = 0; t < C; ++t) {
            if (t < tiles) {
                v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc = VEC ? __builtin_amdgcn_mfma_f64_16x16x4f64(b[t][h][j], gv[h][j], acc, 0, 0, 0) : __builtin_amdgcn_mfma_f64_16x16x4f64(gv[h][j], b[t][h][j], acc, 0, 0, 0);
                if (VEC) {
                    const float4 v = make_float4((float)(acc[0] * delta_b), (float)(acc[1] * delta_b), (float)(acc[2] * delta_b), (float)(acc[3] * delta_b));
                    const int row = rt * 16 + i, k = k0 + 16 * t + 4 * q;
                    if (STAGED) *reinterpret_cast<float4 *>(mine + i * pitch + 16 * t + 4 * q) = v;
                    else if (row < M && k < K) *reinterpret_cast<float4 *>(out + (int64_t)row * K + k) = v;
                } else {
                    const int k = k0 + 16 * t + i;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = rt * 16 + q + 4 * r;
                        const float v = (float)(acc[r] * delta_b);
                        if (STAGED) { if (k < K) mine[(q + 4 * r) * K + k] = v; }
                        else if (row < M && k < K) out[(int64_t)row * K + k] = v;
                    }
                }
            }
        }
        if (!STAGED) continue;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int rows = min(16, M - rt * 16);
        if (STORE == kDaRows) {
            int row = row_first, col = col_first;
            float *dst = out + (int64_t)rt * 16 * K + k0;
            while (row < rows) {
                *reinterpret_cast<float4 *>(dst + (int64_t)row * K + 4 * col) = *reinterpret_cast<const float4 *>(mine + row * pitch + 4 * col);
                row += row_step;
                col += col_step;
                if (col >= width) { col -= width; ++row; }
            }
        } else {
            float *dst = out + (int64_t)rt * 16 * K;
            const int count = rows * K;
            for (int f = lane; f < count >> 2; f += 64) reinterpret_cast<float4 *>(dst)[f] = reinterpret_cast<const float4 *>(mine)[f];
            if (lane < (count & 3)) dst[(count & ~3) + lane] = mine[(count & ~3) + lane];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (NN > 32) {      // (host: one group of columns)
        if (!words.records) return;
        __shared__ unsigned int red[2][4];
        auto block_max = [&](unsigned int v, int which) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned int)__shfl_xor((int)v, off, 64));
            if (lane == 0) red[which][threadIdx.x >> 6] = v;
            __syncthreads();
            return max(max(red[which][0], red[which][1]), max(red[which][2], red[which][3]));
        };
        amax = block_max(amax, 0);
        if (blockIdx.x != gridDim.x - 1) {
            if (threadIdx.x == 0) {
                const unsigned long long v = (unsigned long long)amax << 32 | columns;
                device_store(words.records + 2 * (size_t)blockIdx.x, v);
                device_store(words.records + 2 * (size_t)blockIdx.x + 1, v ^ words.tag);
            }
            return;
        }
        for (int k = threadIdx.x; k < (int)gridDim.x - 1; k += 256) {
            unsigned long long *r = words.records + 2 * (size_t)k;
            unsigned long long v, c;
            do {
                v = device_load(r);
                c = device_load(r + 1);
            } while ((v ^ c) != words.tag);
            device_store(r + 1, v);
            amax = max(amax, (unsigned int)(v >> 32));
            columns = max(columns, (unsigned int)v);
        }
        __syncthreads();
        amax = block_max(amax, 0);
        columns = block_max(columns, 1);
        if (threadIdx.x == 0) choose_limbs(words.plan, amax, 0u, columns, words.delta_a, words.delta_b);
    }
}

// The same up to 16 entries for results well beyond the memory-side cache whose rows, of more columns than a wave holds, are no whole pieces of 64 bytes: a thread has four neighbouring columns, their index values in
// registers, and goes over rows of g in LDS, so that the threads of a block write one row behind the other without a gap.  There the pieces of a row that waves of da_direct_kernel store apart begin and end inside lines of
// memory.  us, da_direct_kernel / this (rows, contraction, columns): 271171 x 12 x 508 204 / 133, 319776 x 7 x 504 206 / 142, 142331 x 10 x 972 172 / 131, 590091 x 8 x 300 224 / 187, 339174 x 6 x 324 153 / 113; of 60 layers 48 with such rows 1.14 times as
// long, 12 with rows of whole pieces 0.91 (117855 x 9 x 656 0.78, 683073 x 8 x 224 1.0); below 90 M outputs: 128872 x 6 x 572 (74 M) 72 / 95, 257589 x 7 x 276 (71 M) 72 / 84.  (The groups of the same rows side by side on an XCD in da_direct_kernel: no faster
// here, 5 - 15 % slower elsewhere.)  Bound by its reads of LDS and the stores.
constexpr int kDaColumnsRows = 128;
bool da_columns_serves(int64_t M, int N, int K) { return N <= 16 && K % 4 == 0 && K % 16 != 0 && K > 16 * direct_tiles(16) && K <= 1 << 25 /* blocks in y */ && M * K >= 90000000; }

__global__ __launch_bounds__(256)
void da_columns_kernel(const float *__restrict__ g, const int8_t *__restrict__ b_idx, int M, int N, int K, double delta_b, double b_offset, float *__restrict__ out, BwdPlan *plan /* null: another product follows */)
{
    constexpr int NN = 16, C = 4;
    __shared__ double gs[kDaColumnsRows][NN];
    if (plan && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) no_limbs(plan);
    const int row0 = blockIdx.x * kDaColumnsRows, rows = min(kDaColumnsRows, M - row0);
    const int words = K / C, per_block = min(words, 256), row_groups = 256 / per_block;
    const int word = blockIdx.y * per_block + (int)threadIdx.x % per_block, first = (int)threadIdx.x / per_block;
    for (int i = threadIdx.x; i < kDaColumnsRows * NN; i += 256) {
        const int r = i / NN, n = i - r * NN;
        gs[r][n] = r < rows && n < N ? (double)g[(int64_t)(row0 + r) * N + n] : 0.0;
    }
    const bool active = word < words && first < row_groups;
    double b[C][NN];
#pragma unroll
    for (int n = 0; n < NN; ++n) {
        const uint32_t w = active && n < N ? *reinterpret_cast<const uint32_t *>(b_idx + (int64_t)n * K + C * word) : 0u;
#pragma unroll
        for (int c = 0; c < C; ++c) b[c][n] = active && n < N ? (double)(int8_t)(w >> (8 * c)) + b_offset : 0.0;      // (the level index itself)
    }
    __syncthreads();
    if (!active) return;
    for (int r = first; r < rows; r += row_groups) {
        double acc[C] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int n = 0; n < NN; ++n) {
            const double v = gs[r][n];
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = fma(v, b[c][n], acc[c]);
        }
        *reinterpret_cast<float4 *>(out + (int64_t)(row0 + r) * K + C * word) =
            make_float4((float)(acc[0] * delta_b), (float)(acc[1] * delta_b), (float)(acc[2] * delta_b), (float)(acc[3] * delta_b));
    }
}

// out[r] = mult * sum_k idx[r][k] + add for an int8 matrix [rows][K]: the corrections of a product whose
// other operand is stored with an offset.  As many lanes a row as it has chunks of 16 bytes, up to a wave (with a wave for every row most lanes of short ones are idle: forward
// product of 130000 x 16 x 64 with an offset 31.3 us, byte by byte 26.2, so 17.5; x 1024 58).
__host__ __device__ __forceinline__ int rowsum_lanes_log2(int K)
{
    int l = 0;
    while (l < 6 && (16 << l) < K) ++l;
    return l;
}

__global__ __launch_bounds__(256) void index_rowsum_kernel(const int8_t *__restrict__ idx, int rows, int K, int mult, int add,
                                                           int32_t *__restrict__ out)
{
    const int lanes_log2 = rowsum_lanes_log2(K), lanes = 1 << lanes_log2, lane = threadIdx.x & 63, own = lane & (lanes - 1);
    if (lanes_log2 == 6) {      // (a wave: its row's address in scalar registers, 82753 x 569 3 us less)
        for (int64_t r = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); r < rows; r += (int64_t)gridDim.x * 4) {
            const int s = row_sum(idx + r * K, K, lane);
            if (lane == 0) out[r] = mult * s + add;
        }
        return;
    }
    for (int64_t first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) << (6 - lanes_log2); first < rows; first += (int64_t)gridDim.x * 4 << (6 - lanes_log2)) {
        const int64_t r = first + (lane >> lanes_log2);
        const int8_t *row = idx + (r < rows ? r : rows - 1) * K;
        int s = 0;
        if (K >= 16) {
            const cdl_v4i w = tail_chunk(row, 16 * own, K);
#pragma unroll
            for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_sdot4(w[i], 0x01010101, s, false);
        } else {
            for (int k = 0; k < K; ++k) s += (int)row[k];
        }
        for (int o = lanes >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (own == 0 && r < rows) out[r] = mult * s + add;
    }
}

// Row sums of the fp32 gradient g [M][N] in double, times `mult`: out[m] = mult * sum_n g[m][n].  One wave per row.
__global__ __launch_bounds__(256) void g_rowsum_kernel(const float *__restrict__ g, int M, int N, double mult, double *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    for (int m = blockIdx.x * 4 + (threadIdx.x >> 6); m < M; m += gridDim.x * 4) {
        const float *p = g + (int64_t)m * N;
        double s = 0.0;
        for (int n = lane; n < N; n += 64) s += (double)p[n];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if (lane == 0) out[m] = mult * s;
    }
}

// Column sums of g [M][N], and of the same pass max |g| per block (what absmax_kernel leaves): block b adds rows b * rows_per .. of every column into
// partial[b][N].  A thread takes V neighbouring columns (V = 4 where rows stay aligned) and, where there are fewer such groups than threads, every
// subs-th row of them, four rows' loads in flight; the subs are added through LDS.  g_colsum_finish adds the blocks.  All in double and in a fixed order.
// What bounds it is memory: 96570 x 148, us, as two passes with a column and four loads of 4 bytes a thread 10 + 29, so 12 (4.9 TB/s); 10669 x 64 4.3 + 5.0, so 4.4.
// A thread of g_colsum_finish adds 16 of 512 blocks' sums (64 of them: 6.6 us instead of 4.6).
constexpr int kColsumBlocks = 512;

template <int V>
__global__ __launch_bounds__(256) void g_colsum_kernel(const float *__restrict__ g, int M, int N, int rows_per, double *__restrict__ partial,
                                                       unsigned int *__restrict__ block_max, unsigned int *__restrict__ clear, int n_clear)
{
    __shared__ double sums[256][V];
    __shared__ unsigned int wave_max[4];
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_clear; i += 256) clear[i] = 0u;      // (absmax_kernel)
    const int groups = N / V, subs = groups < 256 ? 256 / groups : 1, per_pass = groups < 256 ? groups : 256;
    const int sub = (int)threadIdx.x / per_pass, at = (int)threadIdx.x - sub * per_pass;
    const int m0 = blockIdx.x * rows_per, m1 = min(M, m0 + rows_per);
    unsigned int largest = 0u;
    for (int base = 0; base < groups; base += per_pass) {
        const int c = V * (base + at);
        const bool mine = sub < subs && base + at < groups;
        double s[V];
#pragma unroll
        for (int e = 0; e < V; ++e) s[e] = 0.0;
        if (mine) {
            auto rows = [&](int m, auto count) {
                constexpr int R = decltype(count)::value;
                float x[R][V];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float *p = g + (int64_t)(m + r * subs) * N + c;
                    if (V == 4) {
                        const float4 t = load_stream4(p);
                        x[r][0] = t.x; x[r][1 % V] = t.y; x[r][2 % V] = t.z; x[r][3 % V] = t.w;
                    } else {
                        x[r][0] = *p;
                    }
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        s[e] += (double)x[r][e];
                        largest = max(largest, __float_as_uint(fabsf(x[r][e])));
                    }
            };
            int m = m0 + sub;
            for (; m + 3 * subs < m1; m += 4 * subs) rows(m, std::integral_constant<int, 4>{});
            for (; m < m1; m += subs) rows(m, std::integral_constant<int, 1>{});
        }
        if (subs > 1) {
#pragma unroll
            for (int e = 0; e < V; ++e) sums[threadIdx.x][e] = s[e];
            __syncthreads();
            if (sub == 0 && mine)
                for (int q = 1; q < subs; ++q)
#pragma unroll
                    for (int e = 0; e < V; ++e) s[e] += sums[q * per_pass + at][e];
        }
        if (sub == 0 && mine)
#pragma unroll
            for (int e = 0; e < V; ++e) partial[(int64_t)blockIdx.x * N + c + e] = s[e];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) largest = max(largest, (unsigned int)__shfl_down((int)largest, off, 64));
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = largest;
    __syncthreads();
    if (threadIdx.x == 0) block_max[blockIdx.x] = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
}

__global__ __launch_bounds__(256) void g_colsum_finish_kernel(const double *__restrict__ partial, int blocks, int N, double mult, double *__restrict__ out)
{
    // 8 columns per block, 32 threads to a column, eight loads in flight each (one thread per column is one chain of
    // memory latencies: 60 us for 512 blocks' sums of 1000 columns)
    __shared__ double part[32][9];
    const int e = threadIdx.x & 7, sub = threadIdx.x >> 3, n = blockIdx.x * 8 + e;
    double s = 0.0;
    if (n < N) {
#pragma unroll 8
        for (int b = sub; b < blocks; b += 32) s += partial[(int64_t)b * N + n];
    }
    part[sub][e] = s;
    __syncthreads();
    if (sub == 0 && n < N) {
#pragma unroll
        for (int q = 1; q < 32; ++q) s += part[q][e];
        out[n] = mult * s;
    }
}

// ---- helpers -------------------------------------------------------------------------------

// dst[r][0..ldd) = src[r][0..cols) followed by zeros.
__global__ void pad_rows_kernel(const int8_t *__restrict__ src, int64_t rows, int cols, int8_t *__restrict__ dst, int ldd)
{
    const int64_t total = rows * (int64_t)ldd;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / ldd;
        const int c = (int)(i - r * ldd);
        dst[i] = c < cols ? src[r * cols + c] : (int8_t)0;
    }
}

// max |g| per block (as fp32 bits: non-negative floats order like unsigned ints): each block streams
// contiguous pieces, eight independent 16-byte loads per thread and trip.  One plain store per block -
// thousands of atomics on one address would take longer than the pass itself.
__global__ __launch_bounds__(256) void absmax_kernel(const float *__restrict__ g, int64_t n, unsigned int *__restrict__ block_max,
                                                     unsigned int *__restrict__ clear, int n_clear)
{
    // (the transposition kernels that follow on the stream add into these words)
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_clear; i += 256) clear[i] = 0u;
    __shared__ unsigned int wave_max[4];
    unsigned int m = 0u;
    const int64_t n4 = n >> 2;
    const float4 *g4 = reinterpret_cast<const float4 *>(g);
    for (int64_t base = (int64_t)blockIdx.x * 2048; base < n4; base += (int64_t)gridDim.x * 2048) {
        float4 t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t v = base + j * 256 + threadIdx.x;
            t[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (v < n4) {
                // streaming loads (183 -> 122 us on 805 MB): g is far larger than the last-level cache, and the
                // index matrices that the products read next should stay there
                t[j] = load_stream4(reinterpret_cast<const float *>(g4 + v));
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            m = max(m, __float_as_uint(fabsf(t[j].x)));
            m = max(m, __float_as_uint(fabsf(t[j].y)));
            m = max(m, __float_as_uint(fabsf(t[j].z)));
            m = max(m, __float_as_uint(fabsf(t[j].w)));
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
        for (int64_t e = n4 << 2; e < n; ++e) m = max(m, __float_as_uint(fabsf(g[e])));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned int)__shfl_down((int)m, off, 64));
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) block_max[blockIdx.x] = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
}

// dst[c][r] = src[r][c] for an int8 matrix [rows][cols]; dst rows are ldd bytes apart and are
// zero-filled from `rows` up to the next multiple of 128.  Also adds, for every column c of src, the sum of
// |src[r][c]| over the block's rows to col_abs[c] (one atomic per column and block; the array is cleared by the
// max|g| kernel that runs first): the largest of these sums bounds what the rounding of g can do to one output of
// the product that contracts over r, see choose_limbs.
// One block moves tiles of 128 rows x 128 columns: 16-byte loads along the rows (those of the next tile under way while this one is
// stored), four to a thread, into LDS; then every thread takes 16 rows of 4 columns, transposes their 4 x 4 byte blocks in
// registers and stores 16 bytes of four output rows, so that 8 lanes write 128 contiguous bytes.  LDS rows are 33 words apart and
// rows from 64 on 8 words further: the 32 lanes of a read (8 groups of 16 rows, 4 columns) then lie in different banks.
// Limited by memory: 50176 windows of 2304 entries 65 -> 28 us (4.6 TB/s), a matrix of that size 70 -> 44.
// ALIGNED: the rows are, cols % 16 == 0.  Otherwise they are read in the same 16-byte loads from where they start (cdl_rows.h; 24773 x 2646 byte by
// byte 84 us, so 46), and a chunk that they end in is shifted into place on its way to LDS, when all loads of a tile are under way (89744 x 200 in loads of 4 bytes 18.0 us, shifted
// behind its own load 21.4, so 16.6; x 150 byte by byte 27.3, 19.6, 16.1).
// CONV: src is not a matrix but the activations of a convolutional layer, [B][H][W][C] with C a multiple of 16, and
// "src[r][c]" is entry c = (tap row, tap column, channel) of the window of output pixel r = (b, p, q) - the matrix of
// input windows, which is never stored the right way round: only its transpose is written, as the product that
// contracts over the pixels needs it.  Taps outside the image read as geom.pad_word (the stored byte of level index 0).
struct ConvGeom {
    int B, H, W, C, R, S, stride, pad, P, Q;
    int pad_word;
    DivBy by_pq, by_q;
};

struct TransposeJob {
    const int8_t *src;
    int rows, cols;
    int8_t *dst;
    int64_t ldd;
    unsigned int *col_abs;
    int tiles_per_block;
    int blocks_r, blocks;      // blocks along the rows, and in all
    bool fragments;            // 1 KB for 32 rows of 32 columns, [half of the rows][column][16], those of 32 columns one after the other (ldd * 32 bytes)
};

constexpr int kTrRows = 128, kTrCols = 128;

template <bool ALIGNED, bool CONV>
__device__ __forceinline__ void transpose_tiles(const TransposeJob &job, int block, const ConvGeom &geom)
{
    const int8_t *__restrict__ src = job.src;
    int8_t *__restrict__ dst = job.dst;
    const int rows = job.rows, cols = job.cols, tiles_per_block = job.tiles_per_block;
    const int64_t ldd = job.ldd;
    const int block_x = block % job.blocks_r, block_y = block / job.blocks_r;   // neighbouring blocks write neighbouring 128-byte pieces
    __shared__ uint32_t tile[kTrRows * 33 + 8];
    auto at = [](int row, int word) { return row * 33 + (row >> 6) * 8 + word; };
    const int c0 = block_y * kTrCols, tid = threadIdx.x;
    const int row_tiles = (rows + kTrRows - 1) / kTrRows;
    const int t0 = block_x * tiles_per_block, t_end = min(row_tiles, t0 + tiles_per_block);

    // load j: row tid / 8 + 32 j of the tile, 16-byte chunk tid % 8
    const int lrow = tid >> 3, c = c0 + 16 * (tid & 7);
    // CONV: the chunk as a tap and an offset from the window's origin (C % 16 == 0: it lies inside one tap)
    int tap_r = 0, tap_s = 0, tap_off = 0;
    if (CONV) {
        const int cc = min(c, cols - 16), tap = cc / geom.C;
        tap_r = tap / geom.S;
        tap_s = tap - tap_r * geom.S;
        tap_off = (tap_r * geom.W + tap_s) * geom.C + (cc - tap * geom.C);
    }
    // (a chunk that the rows end in is read from their last 16 bytes: this many lie before it)
    const int over = !ALIGNED && !CONV && cols >= 16 && c < cols ? max(c + 16 - cols, 0) : 0;
    uint4 v[4];
    auto load = [&](int rt) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = rt * kTrRows + lrow + 32 * j;
            v[j] = uint4{0u, 0u, 0u, 0u};
            if (CONV) {
                const int m = min(r, rows - 1), pq = geom.P * geom.Q;
                const int b = div_by(m, geom.by_pq.mul, geom.by_pq.sh), rem = m - b * pq, p = div_by(rem, geom.by_q.mul, geom.by_q.sh), q = rem - p * geom.Q;
                const int h0 = p * geom.stride - geom.pad, w0 = q * geom.stride - geom.pad;
                const bool inside = (unsigned)(h0 + tap_r) < (unsigned)geom.H && (unsigned)(w0 + tap_s) < (unsigned)geom.W;
                if (r < rows && c < cols) {
                    const uint32_t pw = (uint32_t)geom.pad_word;
                    v[j] = uint4{pw, pw, pw, pw};
                    // (host: B*H*W*C < 2^31)
                    if (inside) v[j] = *reinterpret_cast<const uint4 *>(src + (((b * geom.H + h0) * geom.W + w0) * geom.C + tap_off));
                }
            } else if (r < rows) {
                const int8_t *p = src + (int64_t)r * cols;
                if (ALIGNED) {
                    if (c < cols) v[j] = *reinterpret_cast<const uint4 *>(p + c);
                } else if (cols >= 16) {
                    if (c < cols) {
                        const cdl_v4i w = load_any16(p + min(c, cols - 16));
                        v[j] = uint4{(uint32_t)w[0], (uint32_t)w[1], (uint32_t)w[2], (uint32_t)w[3]};
                    }
                } else if (c == 0) {
                    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (i < cols) w[i >> 2] |= (uint32_t)(uint8_t)p[i] << (8 * (i & 3));
                    v[j] = uint4{w[0], w[1], w[2], w[3]};
                }
            }
        }
    };
    // A block takes `tiles_per_block` consecutive row tiles of its columns and keeps the column sums of |x| in
    // registers across them: one atomic per column and BLOCK on col_abs (with one per tile the 512 row tiles of
    // workload 5's activations queued 512 atomics on every address and doubled the kernel's time).
    unsigned int part[4] = {};
    const int rg = tid & 7, cg = tid >> 3;      // rows 16 rg .. + 15, columns 4 cg .. + 3
    if (t0 < t_end) load(t0);
    for (int rt = t0; rt < t_end; ++rt) {
        if (!ALIGNED && over > 0)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const cdl_v4i w = without_first(cdl_v4i{(int)v[j].x, (int)v[j].y, (int)v[j].z, (int)v[j].w}, over);
                v[j] = uint4{(uint32_t)w[0], (uint32_t)w[1], (uint32_t)w[2], (uint32_t)w[3]};
            }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t *d = tile + at(lrow + 32 * j, 4 * (tid & 7));
            d[0] = v[j].x; d[1] = v[j].y; d[2] = v[j].z; d[3] = v[j].w;
        }
        __syncthreads();
        if (rt + 1 < t_end) load(rt + 1);
        uint32_t o[4][4];                       // [column][group of four rows]
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t d0 = tile[at(16 * rg + 4 * g, cg)], d1 = tile[at(16 * rg + 4 * g + 1, cg)];
            const uint32_t d2 = tile[at(16 * rg + 4 * g + 2, cg)], d3 = tile[at(16 * rg + 4 * g + 3, cg)];
            const uint32_t x0 = bperm(d1, d0, 0x05010400u), x2 = bperm(d3, d2, 0x05010400u);
            const uint32_t x1 = bperm(d1, d0, 0x07030602u), x3 = bperm(d3, d2, 0x07030602u);
            o[0][g] = bperm(x2, x0, 0x05040100u);
            o[1][g] = bperm(x2, x0, 0x07060302u);
            o[2][g] = bperm(x3, x1, 0x05040100u);
            o[3][g] = bperm(x3, x1, 0x07060302u);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int col = c0 + 4 * cg + b;
            const int64_t at_col = job.fragments ? (int64_t)(col >> 5) * 32 * ldd + (rt * kTrRows + 16 * (rg & 6)) * 32 + (rg & 1) * 512 + (col & 31) * 16
                                                 : (int64_t)col * ldd + rt * kTrRows + 16 * rg;
            if (col < cols) *reinterpret_cast<uint4 *>(dst + at_col) = uint4{o[b][0], o[b][1], o[b][2], o[b][3]};
            // sum of |x| over the four int8 of a word: |x| = |(x + 128) - 128| on the biased bytes
#pragma unroll
            for (int g = 0; g < 4; ++g) part[b] = __builtin_amdgcn_sad_u8(o[b][g] ^ 0x80808080u, 0x80808080u, part[b]);
        }
        __syncthreads();   // the tile is overwritten by the next trip
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        unsigned int sum = part[b];
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) sum += (unsigned int)__shfl_xor((int)sum, off, 64);
        if (rg == 0) tile[4 * cg + b] = sum;
    }
    // (one atomic instruction over neighbouring words: from the lanes that have the sums it would be four with eight words each,
    // and L2 takes the atomics of one line one after the other - 347 blocks of 128 columns: 33 us instead of 14)
    __syncthreads();
    if (tid < kTrCols && c0 + tid < cols && tile[tid] != 0u) atomicAdd(&job.col_abs[c0 + tid], tile[tid]);
}

// Blocks 0 .. a.blocks - 1 do job a, the rest job b; the last of all makes the plan.
template <bool ALIGNED, bool CONV>
__global__ __launch_bounds__(256) void transpose_i8_kernel(TransposeJob a, TransposeJob b, ConvGeom geom, PlanArgs plan)
{
    if ((int)blockIdx.x < a.blocks) transpose_tiles<ALIGNED, CONV>(a, blockIdx.x, geom);
    else if (!CONV) transpose_tiles<ALIGNED, false>(b, (int)blockIdx.x - a.blocks, geom);
    plan_at_end(plan, blockIdx.x, gridDim.x);
}

// The plan as a launch of its own (more blocks than plan_at_end has flags for).
__global__ __launch_bounds__(1024)
void plan_kernel(BwdPlan *plan, const unsigned int *__restrict__ block_max, int n_max,
                 const unsigned int *__restrict__ col_abs_a, int n_abs_a, const unsigned int *__restrict__ col_abs_b, int n_abs_b,
                 float delta_a, float delta_b)
{
    __shared__ unsigned int red_m[1024], red_a[1024], red_b[1024];
    // one block of 1024 threads, four independent loads per thread and trip (the first array holds up to a few
    // thousand per-block results; a single dependent chain per thread is all latency)
    const int t = threadIdx.x;
    unsigned int m = 0u, sa = 0u, sb = 0u;
    for (int i = t; i < n_max; i += 4096) {
        const unsigned int v0 = block_max[i], v1 = i + 1024 < n_max ? block_max[i + 1024] : 0u;
        const unsigned int v2 = i + 2048 < n_max ? block_max[i + 2048] : 0u, v3 = i + 3072 < n_max ? block_max[i + 3072] : 0u;
        m = max(max(m, v0), max(max(v1, v2), v3));
    }
    for (int i = t; i < n_abs_a; i += 1024) sa = max(sa, col_abs_a[i]);
    for (int i = t; i < n_abs_b; i += 1024) sb = max(sb, col_abs_b[i]);
    red_m[t] = m; red_a[t] = sa; red_b[t] = sb;
    __syncthreads();
    for (int off = 512; off > 0; off >>= 1) {
        if (t < off) {
            red_m[t] = max(red_m[t], red_m[t + off]);
            red_a[t] = max(red_a[t], red_a[t + off]);
            red_b[t] = max(red_b[t], red_b[t + off]);
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    choose_limbs(plan, red_m[0], red_a[0], red_b[0], delta_a, delta_b);
}

__global__ void zero_f32_kernel(float *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0.0f;
}

__global__ void zero_i32_kernel(int32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

// ---- measurement aid: register-resident int8 MFMA issue rate ----------------------------------
// Eight independent accumulators per wave, no memory traffic.  random_operands = 0: the two operand
// registers never change (the least switching activity the matrix cores can see); 1: every MFMA of
// the body gets its own pseudo-random operand bits, as dense random int8 data would present them.
__global__ __launch_bounds__(256)
void mfma_probe_kernel(int iters, int random_operands, int *sink)
{
    v4i xs[8], ys[8];
    unsigned h = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            h = h * 1664525u + 1013904223u;
            xs[t][c] = random_operands ? (int)h : 0x01020304;
            h = h * 1664525u + 1013904223u;
            ys[t][c] = random_operands ? (int)h : 0x04030201;
        }
    v16i acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs[t], ys[t], acc[t], 0, 0, 0);
    }
    int x = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) x ^= acc[t][r];
    if (x == 0x7fffffff) *sink = x;   // keeps the MFMAs alive; practically never true
}

inline int64_t pad_to(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

inline unsigned blocks_for(int64_t n, int per_block, int cap = 65536)
{
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// workspace layout of a backward call

// 32-column tiles per wave: the width whose tiles take the least time in all (see limb_narrow_kernel)
int limb_tile_width(int N, int cols)
{
    if (N % 4 != 0) return 3;
    const int64_t cost[4] = {0, 55, 73, 100};
    int best = 3;
    for (int tn = 2; tn >= 1; --tn) {
        auto time = [&](int t) { return ((int64_t)cols + 128 * t - 1) / (128 * t) * cost[t]; };
        if (time(tn) < time(best)) best = tn;
    }
    return best;
}

struct BwdLayout {
    size_t plan, records, block_max, ss_a, ss_b, scalars, bt, at, partial, corr_da, corr_db, colsum_partial, total;
    int n_max;                    // per-block partial results of the absmax launch
    int64_t ldn, ldm;             // row strides of the transposed index copies (odd multiples of kLBK)
    int nk_n, nk_m;               // K-tiles of the two contractions
    int splits, kt_per_split;     // d_b_hat: splits of the contraction over M
    int direct_splits;            // the same for the direct products, at most
};

BwdLayout bwd_layout(int32_t M, int32_t N, int32_t K)
{
    BwdLayout L;
    L.nk_n = (int)((N + kLBK - 1) / kLBK);
    L.nk_m = (int)((M + kLBK - 1) / kLBK);
    L.ldn = (int64_t)(L.nk_n | 1) * kLBK;
    L.ldm = (int64_t)(L.nk_m | 1) * kLBK;
    // d_b_hat has few output tiles and a long contraction: cut the contraction into pieces of at least four K-tiles and (int32
    // accumulators of products up to 2^14) at most 1023 of them.  More pieces fill the last round of blocks better but
    // each is written and read again in double.  Of the numbers of pieces that just fill one to six rounds, the one with the
    // least rounds x K-tiles of a piece (1.8 us each) + traffic of the partial results (5 TB/s).  Against three blocks per compute
    // unit throughout: 1344 x 448 over 11924 rows 82 -> 51 us with the reduction, 576 x 128 over 100352 79 -> 55, 2304 x 256 over 50176 148 -> 140.
    const int tn = limb_tile_width(N, K);
    const int64_t base = (int64_t)((N + kLRows - 1) / kLRows) * ((K + 128 * tn - 1) / (128 * tn)), slots = tn == 1 ? 512 : 256;
    const int64_t nk = L.nk_m;
    int64_t splits = 1, per = nk;
    double least = -1.0;
    for (int rounds = 1; rounds <= 6; ++rounds) {
        int64_t s = rounds * slots / base;
        if (s > nk / 4) s = nk / 4;
        if (s < 1) s = 1;
        int64_t p = (nk + s - 1) / s;
        if (p > 1023) p = 1023;
        s = (nk + p - 1) / p;
        const double t = 1.8 * (double)((base * s + slots - 1) / slots * p) + (s > 1 ? (double)s * N * K * 16.0 / 5e6 : 0.0);
        if (least < 0.0 || t < least) { least = t; splits = s; per = p; }
    }
    // (the direct products: room for about three blocks per compute unit)
    L.direct_splits = (int)((768 + base - 1) / base < nk / 4 ? (768 + base - 1) / base : nk / 4);
    if (L.direct_splits < 1) L.direct_splits = 1;
    L.splits = (int)splits;
    L.kt_per_split = (int)per;
    L.n_max = (int)blocks_for(((int64_t)M * N) >> 2, 2048, 2048);
    size_t off = 0;
    L.plan = off;    off += align_up(sizeof(BwdPlan), 256);
    L.records = off; off += kBwdDirectRecordBytes;
    L.block_max = off; off += align_up((size_t)L.n_max * sizeof(unsigned int), 256);
    L.ss_a = off;    off += align_up((size_t)K * sizeof(unsigned int), 256);   // sums of |a_idx| per column, directly followed by
    L.ss_b = off;    off += align_up((size_t)K * sizeof(unsigned int), 256);   // sums of |b_idx| per column (cleared together)
    const int64_t na = (int64_t)M * K, nb = (int64_t)N * K;
    L.scalars = off; off += align_up(quantize_scalar_bytes(na > nb ? na : nb), 256);     // the quantizers' backward passes that follow in the same call
    L.bt = off;      off += align_up((size_t)pad_to(K, 32) * (size_t)L.ldn, 256);           // b_idx^T: [K][ldn], or in fragments (limb_by_rows)
    L.at = off;      off += align_up((size_t)K * (size_t)L.ldm, 256);           // a_idx^T: [K][ldm]
    L.partial = off; off += align_up((size_t)(L.splits > L.direct_splits ? L.splits : L.direct_splits) * (size_t)N * (size_t)K * sizeof(double), 256);
    // operands stored with an offset: one correction per output row of either product, and the per-block column sums of g
    L.corr_da = off; off += align_up((size_t)M * sizeof(double), 256);
    L.corr_db = off; off += align_up((size_t)N * sizeof(double), 256);
    L.colsum_partial = off; off += align_up((size_t)kColsumBlocks * (size_t)N * sizeof(double), 256);
    L.total = off;
    return L;
}

int launch_limb_gemm(LimbArgs a, bool trans, hipStream_t stream)
{
    // About one block per compute unit: each works through a run of consecutive row tiles.  The limb count,
    // hence the column tile, is only known on the device: the run length is chosen for the wide tile, the
    // grid is sized for the narrowest.
    if (a.tiles_r <= 0 || a.cols <= 0) return CDL_OK;
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0)
        n_cu = 256;
    const int tn = limb_tile_width(a.N, a.cols), narrowest = tn == 3 ? limb_cols(6) : 128 * tn;
    const int64_t slots = tn == 1 ? 2 * n_cu : n_cu, runs_wanted = slots / a.splits > 0 ? slots / a.splits : 1;
    a.units_per_block = (int)((a.tiles_r + runs_wanted - 1) / runs_wanted);
    // (five and six limbs: one row tile per block, and six limbs have the narrower column tile)
    const int64_t items = (int64_t)a.tiles_r * ((a.cols + narrowest - 1) / narrowest) * a.splits;
    if (items > 2147483640LL) return CDL_ERR_PARAM;
    // the kernel addresses the rows of one column tile of the index matrix with 32-bit offsets
    if ((int64_t)limb_cols(3) * a.ldb > 0xffffffffLL) return CDL_ERR_RANGE;
    const unsigned grid = (unsigned)((items + 7) / 8 * 8);
    // Runs pay off for short contractions (measured against one tile per block: -12 % at two K-tiles, -20 % at
    // one, +10 % at 24, where the start-up they save is small and the blocks, all in the same phase for the
    // whole launch, ask L2 for the same lines at the same moments).
    // But a block does every column tile of its row tiles: where that leaves four compute units in ten without work, one tile per
    // block is better (142 row tiles x 2432 columns, two K-tiles: 60 -> 41 us; 94 x 3000, four: 87 -> 42; runs of two over
    // 324 row tiles x 832 columns, 63 % of the units busy: 29 us against 44).
    const bool long_runs = a.kt_per_split <= 4 && (int64_t)a.tiles_r * 10 >= a.units_per_block * runs_wanted * 6;
    const char *name = trans ? "limb_gemm_kernel(d_b_hat)" : "limb_gemm_kernel(d_a_hat)";
    if (tn < 3) {
        const int lds = limb_narrow_lds_bytes(tn);
#define CDL_NARROW(T, TR, LR)                                                                                                            \
    do {                                                                                                                                 \
        const hipError_t e_ = hipFuncSetAttribute((const void *)limb_narrow_kernel<T, TR, LR>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); \
        if (e_ != hipSuccess) return hip_failed(e_);                                                                                     \
        CDL_LAUNCH(name, stream, (limb_narrow_kernel<T, TR, LR>), dim3(grid), dim3(kLThreads), lds, a);                                  \
    } while (0)
        if (trans) { if (tn == 1) CDL_NARROW(1, true, false); else CDL_NARROW(2, true, false); }
        else if (long_runs) { if (tn == 1) CDL_NARROW(1, false, true); else CDL_NARROW(2, false, true); }
        else { if (tn == 1) CDL_NARROW(1, false, false); else CDL_NARROW(2, false, false); }
#undef CDL_NARROW
        return check_launch();
    }
    const void *fn = trans ? (long_runs ? (const void *)limb_gemm_kernel<true, true> : (const void *)limb_gemm_kernel<true, false>)
                           : (long_runs ? (const void *)limb_gemm_kernel<false, true> : (const void *)limb_gemm_kernel<false, false>);
    // more than 64 KiB of dynamic LDS has to be allowed per function (and per device: set it every time)
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLimbLdsBytes);
    if (e != hipSuccess) return hip_failed(e);
    if (trans && long_runs) CDL_LAUNCH(name, stream, (limb_gemm_kernel<true, true>), dim3(grid), dim3(kLThreads), kLimbLdsBytes, a);
    else if (trans) CDL_LAUNCH(name, stream, (limb_gemm_kernel<true, false>), dim3(grid), dim3(kLThreads), kLimbLdsBytes, a);
    else if (long_runs) CDL_LAUNCH(name, stream, (limb_gemm_kernel<false, true>), dim3(grid), dim3(kLThreads), kLimbLdsBytes, a);
    else CDL_LAUNCH(name, stream, (limb_gemm_kernel<false, false>), dim3(grid), dim3(kLThreads), kLimbLdsBytes, a);
    return check_launch();
}

// Whether the two products go into one launch: their blocks (in tiles of 384 columns) are at most four for every compute
// unit, and those of the first product too few for runs of tiles to pay.
bool limb_pair_serves(int64_t M, int32_t N, int32_t K, int splits)
{
    const int64_t tiles_c = (K + limb_cols(5) - 1) / limb_cols(5);
    const int64_t na = (M + kLRows - 1) / kLRows * tiles_c, nb = (int64_t)((N + kLRows - 1) / kLRows) * tiles_c * splits;
    return na <= 512 && na + nb <= 1024;
}

// Whether dL/dQ(a) goes through limb_rows_kernel where that serves (by sizes alone, whatever is asked for): not where both products fit
// one launch in one or two tiles of 384 columns with little padding, us a call: 9000 x 384 x 384 51.1 / 46.1, 4000 x 320 x 768 45.5 / 42.8,
// 8000 x 128 x 384 38.4 / 36.2; but 9000 x 384 x 512 51.0 / 54.3, 3000 x 384 x 1500 57.1 / 64.5, 3000 x 256 x 2304 51.9 / 62.2.
bool limb_by_rows(int64_t M, int32_t N, int32_t K, int splits)
{
    const int padded = (K + limb_cols(5) - 1) / limb_cols(5) * limb_cols(5);
    return limb_rows_serves(M, N, K) && !(padded <= 2 * limb_cols(5) && padded * 10 <= K * 11 && limb_pair_serves(M, N, K, splits));
}

int launch_limb_pair(LimbArgs a, LimbArgs b, hipStream_t stream)
{
    const int64_t tiles_c = (a.cols + limb_cols(6) - 1) / limb_cols(6);
    if ((int64_t)limb_cols(3) * a.ldb > 0xffffffffLL || (int64_t)limb_cols(3) * b.ldb > 0xffffffffLL) return CDL_ERR_RANGE;
    a.units_per_block = b.units_per_block = 1;
    const unsigned ga = (unsigned)((a.tiles_r * tiles_c + 7) / 8 * 8), gb = (unsigned)((b.tiles_r * tiles_c * b.splits + 7) / 8 * 8);
    const hipError_t e = hipFuncSetAttribute((const void *)limb_pair_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLimbLdsBytes);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("limb_pair_kernel(d_a_hat, d_b_hat)", stream, limb_pair_kernel, dim3(ga + gb), dim3(kLThreads), kLimbLdsBytes, a, b, (int)ga);
    return check_launch();
}

// about a thousand blocks where the matrix has that many tiles, each with up to 16 row tiles of its columns
TransposeJob transpose_job(const int8_t *src, int rows, int cols, int8_t *dst, int64_t ldd, unsigned int *col_abs, bool fragments = false)
{
    const int row_tiles = (rows + kTrRows - 1) / kTrRows, col_tiles = (cols + kTrCols - 1) / kTrCols;
    int per = (int)(((int64_t)row_tiles * col_tiles + 1023) / 1024);
    per = per < 1 ? 1 : (per > 16 ? 16 : per);
    const int blocks_r = (row_tiles + per - 1) / per;
    return TransposeJob{src, rows, cols, dst, ldd, col_abs, per, blocks_r, blocks_r * col_tiles, fragments};
}

// Column sums and transposed copies of the operands, and from them the plan (whatever `p` asks for).
int launch_transposes(const TransposeJob &a, const TransposeJob &b, const ConvGeom *windows, PlanArgs p, void *flags, hipStream_t stream)
{
    const int blocks = a.blocks + b.blocks;
    const PlanArgs here = p;
    p.flags = reinterpret_cast<unsigned long long *>(flags);
    p.tag = next_finish_tag();
    if (blocks > kPlanMaxBlocks) p.plan = nullptr;
    if (windows) CDL_LAUNCH("transpose_i8_kernel(windows)", stream, (transpose_i8_kernel<true, true>), dim3((unsigned)blocks), dim3(256), 0, a, b, *windows, p);
    else if (a.cols % 16 == 0) CDL_LAUNCH("transpose_i8_kernel", stream, (transpose_i8_kernel<true, false>), dim3((unsigned)blocks), dim3(256), 0, a, b, ConvGeom{}, p);
    else CDL_LAUNCH("transpose_i8_kernel", stream, (transpose_i8_kernel<false, false>), dim3((unsigned)blocks), dim3(256), 0, a, b, ConvGeom{}, p);
    if (!p.plan)
        CDL_LAUNCH("plan_kernel", stream, plan_kernel, dim3(1), dim3(1024), 0, here.plan, here.block_max, here.n_max, here.col_abs_a, here.n_abs_a,
                   here.col_abs_b, here.n_abs_b, here.delta_a, here.delta_b);
    return check_launch();
}

}  // namespace

int launch_mfma_probe(int iters, int random_operands, int blocks, int *sink, hipStream_t stream)
{
    CDL_LAUNCH("mfma_probe_kernel", stream, mfma_probe_kernel, dim3(blocks), dim3(256), 0, iters, random_operands, sink);
    return check_launch();
}

// Whether a product of rows of K % 16 != 0 entries goes through zero-padded copies of both operands: fewer than a chunk; and results that stream past the last-level cache, where
// the copies let the kernel of direct loads serve (K up to 15 below a multiple of 64) and N is so large that they are little beside the product.  us, as they are / in copies:
// 72595 x 1102 x 377 155 / 134, 60000 x 1500 x 377 173 / 136, x 764 220 / 204, x 1020 248 / 243, x 2040 378 / 415, 20000 x 3072 x 505 99 / 82, x 124 53 / 50, but 60000 x 900 x 377 78 / 87;
// 155000 x 400 x 57 74 / 62, 180232 x 344 x 57 71 / 78.  (Copies for short rows of odd lengths and the other tiles: 0.82 - 1.16, 1.0 in the mean.)
static bool copies_pay(int32_t M, int32_t N, int32_t K)
{
    if (K % 16 == 0) return false;
    if (K < 16) return true;
    return (int64_t)M * N >= 60000000 && N >= (K < 64 ? 384 : K < 1024 ? 1024 : 2048) && dma_serves(M, N, pad_to(K, 16));
}

// forward workspace: [when K % 16 != 0: room for operand copies with padded rows; not every product makes them, see copies_pay][with offsets: corrections per output column: int32 N][per output row: int32 M]
size_t qgemm_fwd_workspace_bytes(int32_t M, int32_t N, int32_t K, bool with_offsets)
{
    size_t b = 0;
    if (K % 16 != 0) {
        const int64_t kp = pad_to(K, 16);
        b += align_up((size_t)M * (size_t)kp, 256) + align_up((size_t)N * (size_t)kp, 256);
    }
    if (with_offsets) b += align_up((size_t)N * sizeof(int32_t), 256) + align_up((size_t)M * sizeof(int32_t), 256);
    return b;
}

size_t qgemm_bwd_workspace_bytes(int32_t M, int32_t N, int32_t K)
{
    if ((int64_t)M * N * K == 0) return 0;
    return bwd_layout(M, N, K).total;
}

int launch_qgemm_fwd(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K,
                     float delta_a, float delta_b, int32_t a_offset, int32_t b_offset,
                     int32_t *acc, float *y, void *ws, hipStream_t stream)
{
    if ((int64_t)M * N == 0) return CDL_OK;
    if (K == 0) {
        if (acc) CDL_LAUNCH("zero_i32_kernel", stream, zero_i32_kernel, dim3(blocks_for((int64_t)M * N, 256, 4096)), dim3(256), 0, acc, (int64_t)M * N);
        if (y) CDL_LAUNCH("zero_f32_kernel", stream, zero_f32_kernel, dim3(blocks_for((int64_t)M * N, 256, 4096)), dim3(256), 0, y, (int64_t)M * N);
        return check_launch();
    }
    if (qgemm_small_serves(M, N, K, a_offset, b_offset))
        return launch_qgemm_small(a_idx, b_idx, M, N, K, delta_a * delta_b, a_offset, b_offset, acc, y, stream);
    if (qgemm_thin_serves(M, N, K, a_offset, b_offset)) return launch_qgemm_thin(a_idx, b_idx, M, N, K, delta_a * delta_b, a_offset, acc, y, stream);
    GemmArgs g{};
    g.A = a_idx; g.B = b_idx; g.lda = K; g.ldb = K;
    g.rowsA = M; g.rowsB = N; g.Kc = K;
    char *corr_base = reinterpret_cast<char *>(ws) + qgemm_fwd_workspace_bytes(M, N, K, false);
    int32_t *corr_col = reinterpret_cast<int32_t *>(corr_base);
    int32_t *corr_row = reinterpret_cast<int32_t *>(corr_base + align_up((size_t)N * sizeof(int32_t), 256));
    if (a_offset != 0) {
        // per output column s: oa * sum_k b'[s][k] + K oa ob
        CDL_LAUNCH("index_rowsum_kernel", stream, index_rowsum_kernel, dim3(blocks_for(N, 256 >> rowsum_lanes_log2(K), 4096)), dim3(256), 0, b_idx, N, K, a_offset,
                   K * a_offset * b_offset, corr_col);
        g.corr_col = corr_col;
    }
    if (b_offset != 0) {
        // per output row r: ob * sum_k a'[r][k] (plus the constant if no column correction carries it)
        CDL_LAUNCH("index_rowsum_kernel", stream, index_rowsum_kernel, dim3(blocks_for(M, 256 >> rowsum_lanes_log2(K), 4096)), dim3(256), 0, a_idx, M, K, b_offset,
                   a_offset != 0 ? 0 : K * a_offset * b_offset, corr_row);
        g.corr_row = corr_row;
    }
    const bool copies = copies_pay(M, N, K), ragged = K % 16 != 0 && !copies;
    if (copies) {
        const int kp = (int)pad_to(K, 16);
        int8_t *ap = reinterpret_cast<int8_t *>(ws);
        int8_t *bp = ap + align_up((size_t)M * (size_t)kp, 256);
        CDL_LAUNCH("pad_rows_kernel", stream, pad_rows_kernel, dim3(blocks_for((int64_t)M * kp, 256, 8192)), dim3(256), 0, a_idx, (int64_t)M, K, ap, kp);
        CDL_LAUNCH("pad_rows_kernel", stream, pad_rows_kernel, dim3(blocks_for((int64_t)N * kp, 256, 8192)), dim3(256), 0, b_idx, (int64_t)N, K, bp, kp);
        int rc = check_launch();
        if (rc != CDL_OK) return rc;
        g.A = ap; g.B = bp; g.lda = kp; g.ldb = kp; g.Kc = kp;
    }
    g.acc_out = acc; g.y_out = y; g.ldc = N;
    g.scale = delta_a * delta_b;
    switch (choose_tiles(false, !ragged && g.Kc % kRingBK == 0, M, N, g.Kc)) {
        case kTileWide: return launch_gemm_ring<RingWide>(g, stream);
        case kTileTall: return launch_gemm_ring<RingTall>(g, stream);
        case kTileNarrow: return launch_gemm_ring<RingNarrow>(g, stream);
        case kTileSquare: return launch_gemm_ring<RingSquare>(g, stream);
        case kTileLow: return launch_gemm_ring<RingLow>(g, stream);
        case kTileStaged: break;
    }
    // (up to 64 output columns: tiles 64 columns wide, so that half of a wider one is not padding)
    const int rows = staged_rows(M, N);
    if (N <= 64) return rows == 64 ? launch_gemm<1, 1>(g, ragged, stream) : rows == 128 ? launch_gemm<2, 1>(g, ragged, stream) : launch_gemm<4, 1>(g, ragged, stream);
    return rows == 64 ? launch_gemm<1, 2>(g, ragged, stream) : rows == 128 ? launch_gemm<2, 2>(g, ragged, stream) : launch_gemm<4, 2>(g, ragged, stream);
}

int launch_qgemm_quantize_fwd(const float *x, const cdl_qparams &p, const int8_t *b_idx, int32_t M, int32_t N, int32_t K,
                              float delta_b, float *y, hipStream_t stream)
{
    if ((int64_t)M * N == 0) return CDL_OK;
    LimbArgs a{};
    a.G = x; a.M = M; a.N = K;            // the fp32 operand: [M][K], contraction along its rows
    a.Bt = b_idx; a.ldb = K;              // [N][K]: the contraction index is contiguous as it is
    a.rows = M; a.cols = N; a.kc = K;
    a.nk = K / kLBK;
    a.tiles_r = (M + kLRows - 1) / kLRows; a.splits = 1; a.kt_per_split = a.nk;
    a.out = y;
    a.fq_k = make_const(p);
    a.fq_scale = p.delta * delta_b;
    constexpr int NB = 4 * kQuantFwdTN * 32;
    if ((int64_t)NB * a.ldb > 0xffffffffLL) return CDL_ERR_RANGE;
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0)
        n_cu = 256;
    a.units_per_block = (a.tiles_r + n_cu - 1) / n_cu;
    const int64_t items = (a.tiles_r + a.units_per_block - 1) / a.units_per_block;      // runs; each takes every column tile
    const unsigned grid = (unsigned)((items + 7) / 8 * 8);
    const hipError_t e = hipFuncSetAttribute((const void *)qgemm_quantize_fwd_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLimbLdsBytes);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("qgemm_kernel(quantize + fwd)", stream, qgemm_quantize_fwd_kernel, dim3(grid), dim3(kLThreads), kLimbLdsBytes, a);
    return check_launch();
}

// address of conv_zero_page on the current device (taken once per device)
static int conv_zero_page_ptr(const int8_t **ptr)
{
    constexpr int kMaxDevices = 64;
    static const int8_t *cached[kMaxDevices];
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_failed(e);
    if (dev < 0 || dev >= kMaxDevices) return CDL_ERR_PARAM;
    std::lock_guard<std::mutex> lock(mu);
    if (!cached[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(conv_zero_page));
        if (e != hipSuccess) return hip_failed(e);
        if (!p) return hip_failed(hipErrorInvalidSymbol);
        cached[dev] = reinterpret_cast<const int8_t *>(p);
    }
    *ptr = cached[dev];
    return CDL_OK;
}

constexpr int kConvDxMaxBlocks = 2048;      // of the pass for max |g|
struct ConvDxLayout {
    size_t plan, flags, block_max, ss_b, wr, planes, total;      // (patches: see patch_scratch)
    int n_max, Np, classes;
    int64_t ld;
};

ConvDxLayout conv_dx_layout(int64_t M_out, int32_t N, int32_t C, int32_t R, int32_t S, int32_t stride, int32_t pad_n)
{
    ConvDxLayout L;
    // stride 2: four classes of taps, each with at most ceil(R / 2) x ceil(S / 2) of them
    L.classes = stride == 2 ? 4 : 1;
    L.Np = (N + pad_n - 1) / pad_n * pad_n;
    const int64_t kc = (stride == 2 ? (int64_t)((R + 1) / 2) * ((S + 1) / 2) : (int64_t)R * S) * L.Np;
    L.ld = (kc + 63) / 64 * 64;
    L.n_max = (int)blocks_for((M_out * N) >> 2, 2048, kConvDxMaxBlocks);
    size_t off = 0;
    L.plan = off;      off += align_up(sizeof(BwdPlan), 256);
    L.flags = off;     off += kPlanMaxBlocks * sizeof(unsigned long long);
    L.block_max = off; off += align_up((size_t)L.n_max * sizeof(unsigned int), 256);
    L.ss_b = off;      off += align_up((size_t)L.classes * C * sizeof(unsigned int), 256);
    L.wr = off;        off += align_up((size_t)((C + 31) / 32 * 32) * (size_t)L.classes * (size_t)L.ld, 256);
    L.planes = off;    off += align_up((size_t)M_out * (size_t)L.Np * kMaxLimbs, 256);
    L.total = off;
    return L;
}

// What the kernel on patches has in the place of the planes.
struct PatchScratch { size_t pixel_max, part, flags, total; int nx, ny; };
PatchScratch patch_scratch(const ConvDxLayout &L, int64_t M_out, int32_t C)
{
    PatchScratch p;
    p.nx = (int)(L.ld / 64);
    p.ny = (C + 63) / 64;
    size_t off = L.planes;
    p.pixel_max = off; off += align_up((size_t)M_out * sizeof(unsigned int), 256);
    p.part = off;      off += align_up((size_t)L.classes * (size_t)p.nx * (size_t)C * sizeof(unsigned int), 256);
    p.flags = off;     off += align_up((size_t)L.classes * (size_t)p.nx * (size_t)p.ny * sizeof(unsigned long long), 256);
    p.total = off;
    return p;
}

// (a 1 x 1 convolution of stride 1 is a linear layer)
bool conv_dx_is_linear(int32_t R, int32_t S, int32_t stride) { return R == 1 && S == 1 && stride == 1; }

size_t qconv_bwd_activations_workspace_bytes(int32_t B, int32_t H, int32_t W, int32_t C, int32_t N, int32_t R, int32_t S, int32_t stride, int32_t pad)
{
    const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1;
    const int64_t M_out = (int64_t)B * P * Q;
    ConvDxGrid grids[4];
    bool unreached;
    const int n_cls = conv_dx_classes(H, W, R, S, stride, pad, grids, unreached);
    const bool patch = conv_dx_patch_serves(grids, n_cls, B, C, N, P, Q);
    const ConvDxLayout L = conv_dx_layout(M_out, N, C, R, S, stride, patch ? 32 : 16);
    // Room for digit planes from half a G multiply-adds on: the digits of a patch lie in LDS, but what a size asks for does not depend on
    // which of the kernels serves it.  None for a linear layer, nor for few channels on both sides (the direct product at any size).
    const bool is_linear = conv_dx_is_linear(R, S, stride), few = C <= 32 && (int64_t)R * S * N <= 288;
    const double cols = C <= 48 ? (C + 15) / 16 * 16 : (C + 63) / 64 * 64;
    const double work = (double)B * H * W * cols * (double)(((int64_t)R * S * N + 15) / 16 * 16) / (stride * stride);
    size_t own = is_linear || few || work <= 5e8 ? L.planes : L.total;
    if (!conv_dx_direct_serves((int64_t)B * H * W, N, C, R, S, stride) && !is_linear) {
        const size_t least = patch ? patch_scratch(L, M_out, C).total : L.total;
        if (least > own) own = least;
    }
    const size_t linear = is_linear ? bwd_layout((int32_t)M_out, N, C).total : 0;
    return own > linear ? own : linear;
}

int launch_qconv_bwd_activations(const float *g, const int8_t *w_idx, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                                 int32_t R, int32_t S, int32_t stride, int32_t pad, float delta_w, float *d_x_hat, void *ws,
                                 hipStream_t stream)
{
    const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1;
    const int64_t M_out = (int64_t)B * P * Q;
    ConvDxGrid grids[4];
    bool zero_first;
    const int n_cls = conv_dx_classes(H, W, R, S, stride, pad, grids, zero_first);
    if (zero_first)
        CDL_LAUNCH("zero_f32_kernel", stream, zero_f32_kernel, dim3(blocks_for((int64_t)B * H * W * C, 256, 4096)), dim3(256), 0, d_x_hat, (int64_t)B * H * W * C);
    if (n_cls == 0) return check_launch();
    if (conv_dx_thin_serves(grids, B, H, W, C, N, R, S, P, Q, stride)) return launch_conv_dx_thin(g, w_idx, grids[0], B, C, N, P, Q, delta_w, d_x_hat, stream);
    if (conv_dx_direct_serves((int64_t)B * H * W, N, C, R, S, stride))
        return launch_conv_dx_direct(g, w_idx, grids, n_cls, B, H, W, C, N, R, S, P, Q, stride, delta_w, d_x_hat, stream);
    if (conv_dx_is_linear(R, S, stride))      // (the padding is smaller than the kernel: none)
        return launch_qgemm_bwd(g, nullptr, w_idx, (int32_t)M_out, N, C, 1.0f, delta_w, 0, 0, d_x_hat, nullptr, ws, stream);

    const bool patch = conv_dx_patch_serves(grids, n_cls, B, C, N, P, Q);
    const ConvDxLayout L = conv_dx_layout(M_out, N, C, R, S, stride, patch ? 32 : 16);
    char *base = reinterpret_cast<char *>(ws);
    BwdPlan *plan = reinterpret_cast<BwdPlan *>(base + L.plan);
    unsigned int *block_max = reinterpret_cast<unsigned int *>(base + L.block_max);
    unsigned int *ss_b = reinterpret_cast<unsigned int *>(base + L.ss_b);
    int8_t *wr = reinterpret_cast<int8_t *>(base + L.wr);
    ConvDxClasses taps{};
    taps.tstep = stride;
    for (int c = 0; c < n_cls; ++c) taps.c[c] = ConvDxClass{grids[c].r0, grids[c].s0, grids[c].Rc, grids[c].Sc};
    const ConvDxWeights weights{w_idx, N, L.Np, R, S, C, taps, wr, L.ld};
    if (patch) {
        static_assert(kPatchMaxima >= kConvDxMaxBlocks, "maxima that a block of the patch kernel reads");
        const PatchScratch at = patch_scratch(L, M_out, C);
        PatchPrep p{};
        p.weights = weights;
        p.nx = at.nx; p.ny = at.ny; p.nz = n_cls;
        p.part = reinterpret_cast<unsigned int *>(base + at.part);
        p.flags = reinterpret_cast<unsigned long long *>(base + at.flags);
        p.tag = next_finish_tag();
        p.col_max = ss_b;
        p.g = g; p.pixels = (int)M_out; p.N = N;
        while (p.log_t < 6 && 2 << p.log_t <= N / 4) ++p.log_t;
        p.pixel_max = reinterpret_cast<unsigned int *>(base + at.pixel_max);
        p.block_max = block_max;
        const int64_t blocks = (int64_t)at.nx * at.ny * n_cls;
        if (blocks > 1 << 30) return CDL_ERR_RANGE;
        CDL_LAUNCH("conv_patch_prep_kernel", stream, conv_patch_prep_kernel, dim3((unsigned)blocks + (unsigned)L.n_max), dim3(256), 0, p);
        const int rc = check_launch();
        if (rc != CDL_OK) return rc;
        return launch_conv_dx_patch(g, wr, PatchMaxima{p.pixel_max, block_max, ss_b, L.n_max, (int)(at.ny * n_cls)}, L.ld, grids, n_cls, B, H, W, C, N, L.Np, P, Q, stride, delta_w, d_x_hat, stream);
    }
    CDL_LAUNCH("absmax_kernel", stream, absmax_kernel, dim3(L.n_max), dim3(256), 0, g, M_out * N, block_max, ss_b, n_cls * C);
    // (one limb count for all classes: the largest column sum of any of them)
    PlanArgs pa{plan, block_max, L.n_max, nullptr, ss_b, 0, n_cls * C, 1.0f, delta_w, reinterpret_cast<unsigned long long *>(base + L.flags), next_finish_tag()};
    const dim3 prep((unsigned)(L.ld / 64), (unsigned)((C + 63) / 64), (unsigned)n_cls);
    const bool plan_apart = (int64_t)prep.x * prep.y * prep.z > kPlanMaxBlocks;
    if (plan_apart) pa.plan = nullptr;
    CDL_LAUNCH("conv_dx_prep_kernel", stream, conv_dx_prep_kernel, prep, dim3(256), 0, weights, ss_b, pa);
    if (plan_apart)
        CDL_LAUNCH("plan_kernel", stream, plan_kernel, dim3(1), dim3(1024), 0, plan, block_max, L.n_max,
                   (const unsigned int *)nullptr, 0, ss_b, n_cls * C, 1.0f, delta_w);
    const int8_t *zeros = nullptr;
    int rc = check_launch();
    if (rc == CDL_OK) rc = conv_zero_page_ptr(&zeros);
    if (rc != CDL_OK) return rc;
    return launch_conv_dx_planes(g, wr, L.ld, grids, n_cls, B, H, W, C, N, L.Np, P, Q, stride, plan, reinterpret_cast<int8_t *>(base + L.planes), zeros, d_x_hat, stream);
}

size_t qconv_fwd_workspace_bytes(int32_t N, int32_t x_offset)
{
    return x_offset != 0 ? 256 + align_up((size_t)N * sizeof(int32_t), 256) : 0;
}

template <class SHAPE>
static int launch_conv_ring(ConvArgs a, hipStream_t stream)
{
    a.tiles_m = (a.M + SHAPE::kRows - 1) / SHAPE::kRows;
    a.tiles_n = (a.N + SHAPE::kCols - 1) / SHAPE::kCols;
    const int64_t grid = ring_grid((int64_t)a.tiles_m * a.tiles_n, SHAPE::PER_CU);
    const bool stream_out = stream_output((int64_t)a.M * a.N, a.N, a.y_out) && !a.acc_out, chunks = a.C % kRingBK != 0;
    if (chunks) {
        a.step_taps = kRingBK / 16 / a.c16;
        a.step_in = kRingBK / 16 % a.c16;
    }
    const auto kernel = chunks ? (stream_out ? qconv_dma_kernel<SHAPE, true, true> : qconv_dma_kernel<SHAPE, false, true>)
                               : (stream_out ? qconv_dma_kernel<SHAPE, true, false> : qconv_dma_kernel<SHAPE, false, false>);
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SHAPE::kLds);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("qconv_kernel(fwd)", stream, kernel, dim3((unsigned)grid), dim3(SHAPE::kThreads), SHAPE::kLds, a);
    return check_launch();
}

int launch_qconv_fwd(const int8_t *x_idx, const int8_t *w_idx, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                     int32_t R, int32_t S, int32_t stride, int32_t pad, float delta_x, float delta_w, int32_t x_offset,
                     int32_t *acc, float *y, void *ws, hipStream_t stream)
{
    ConvArgs a{};
    a.X = x_idx; a.Wt = w_idx;
    a.B = B; a.H = H; a.W = W; a.C = C; a.N = N; a.R = R; a.S = S; a.stride = stride; a.pad = pad;
    a.P = (H + 2 * pad - R) / stride + 1;
    a.Q = (W + 2 * pad - S) / stride + 1;
    a.M = B * a.P * a.Q;
    a.Kc = R * S * C;
    a.by_pq = make_div_by((uint32_t)a.P * (uint32_t)a.Q);
    a.by_q = make_div_by((uint32_t)a.Q);
    a.c16 = C / 16;
    a.by_c16 = make_div_by((uint32_t)a.c16);
    a.by_s = make_div_by((uint32_t)S);
    a.acc_out = acc; a.y_out = y;
    a.scale = delta_x * delta_w;
    if ((int64_t)a.M * N == 0) return CDL_OK;
    if (qconv_thin_serves(a.M, N, a.Kc, x_offset))
        return launch_qconv_thin(x_idx, w_idx, ConvWindows{B, H, W, C, R, S, stride, pad, a.P, a.Q}, N, a.scale, x_offset, acc, y, stream);
    if (x_offset != 0) {
        int8_t *page = reinterpret_cast<int8_t *>(ws);
        int32_t *corr = reinterpret_cast<int32_t *>(page + 256);
        CDL_LAUNCH("conv_prep_kernel", stream, conv_prep_kernel, dim3((unsigned)blocks_for(N, 4, 1024)), dim3(256), 0, page, x_offset, w_idx, N, a.Kc, corr);
        int rc = check_launch();
        if (rc != CDL_OK) return rc;
        a.pad_page = page;
        a.zero_page = page + 128;      // (no look-up of the library's own page: a call with an offset may be the first on a GPU, and captured)
        a.corr_col = corr;
    } else {
        int rc = conv_zero_page_ptr(&a.pad_page);
        if (rc != CDL_OK) return rc;
        a.zero_page = a.pad_page;
    }
    const uint32_t pb = (uint32_t)(uint8_t)(int8_t)(-x_offset);
    a.pad_word = (int)(pb | (pb << 8) | (pb << 16) | (pb << 24));
    switch (choose_tiles(true, C % kRingBK == 0, a.M, N, a.Kc)) {
        case kTileWide: return launch_conv_ring<RingWide>(a, stream);
        case kTileTall: return launch_conv_ring<RingTall>(a, stream);
        case kTileNarrow: return launch_conv_ring<RingNarrow>(a, stream);
        case kTileSquare: return launch_conv_ring<RingSquare>(a, stream);
        case kTileLow: return launch_conv_ring<RingLow>(a, stream);
        case kTileStaged: break;
    }
    const int BN = N <= 64 ? 64 : 128, BM = staged_rows(a.M, N);
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (N + BN - 1) / BN;
    const int64_t grid = ((int64_t)a.tiles_m * a.tiles_n + 7) / 8 * 8;
    const auto kernel = N <= 64 ? (BM == 64 ? qconv_kernel<1, 1> : BM == 128 ? qconv_kernel<2, 1> : qconv_kernel<4, 1>)
                                : (BM == 64 ? qconv_kernel<1, 2> : BM == 128 ? qconv_kernel<2, 2> : qconv_kernel<4, 2>);
    CDL_LAUNCH("qconv_kernel(fwd)", stream, kernel, dim3((unsigned)grid), dim3(kGemmThreads), 0, a);
    return check_launch();
}

int qconv_max_chunks() { return kConvMaxChunks; }

int launch_qgemm_bwd(const float *gr, const int8_t *a_idx, const int8_t *b_idx,
                     int32_t M, int32_t N, int32_t K, float delta_a, float delta_b, int32_t a_offset, int32_t b_offset,
                     float *d_a_hat, float *d_b_hat, void *ws, hipStream_t stream, const ConvWindows *cw)
{
    const bool want_db = d_b_hat != nullptr;
    if (cw && d_a_hat) return CDL_ERR_PARAM;                       // (windows: a_idx is not a matrix; only the product over its rows is served)
    if (d_a_hat && ((int64_t)M * K > 0) && N == 0)
        CDL_LAUNCH("zero_f32_kernel", stream, zero_f32_kernel, dim3(blocks_for((int64_t)M * K, 256, 4096)), dim3(256), 0, d_a_hat, (int64_t)M * K);
    if (d_b_hat && ((int64_t)N * K > 0) && M == 0)
        CDL_LAUNCH("zero_f32_kernel", stream, zero_f32_kernel, dim3(blocks_for((int64_t)N * K, 256, 4096)), dim3(256), 0, d_b_hat, (int64_t)N * K);
    if ((int64_t)M * N * K == 0) return check_launch();

    const BwdLayout L = bwd_layout(M, N, K);
    char *base = reinterpret_cast<char *>(ws);
    BwdPlan *plan = reinterpret_cast<BwdPlan *>(base + L.plan);
    double *partial = reinterpret_cast<double *>(base + L.partial);
    // (the windows of a 1 x 1 kernel of stride 1 are the activations as they lie)
    const bool is_conv_weights = cw != nullptr;
    if (cw && cw->R == 1 && cw->S == 1 && cw->stride == 1 && cw->pad == 0) cw = nullptr;
    if (cw && conv_dw_direct_serves(M, N, K)) return launch_conv_dw_direct(gr, a_idx, *cw, N, delta_a, a_offset, d_b_hat, partial, L.direct_splits, stream);
    // (many outputs of few multiplications each: see da_direct_kernel)
    const bool only_b = is_conv_weights || da_direct_preferred(M, N, K, want_db) || (N <= kDirectMaxN && !bwd_direct_serves(M, N, K, false, partial, L.direct_splits, true, 0));
    const unsigned int *col_abs_b = nullptr;      // the largest sum of |b_idx| of a column, for the words, where dL/dQ(a) is formed before the plan is made
    if (d_a_hat && only_b) {
        // (blocks of four waves per group of columns: as many as the chip holds, at most one wave per tile of rows)
        const int most = direct_tiles((N + 15) / 16 * 16), all = (K + 15) / 16, groups = (all + most - 1) / most;
        const int col_tiles = (all + groups - 1) / groups;
        const bool staged = N <= 32 && direct_staged((int64_t)M * K, K % 4 == 0);
        const int64_t row_blocks = ((int64_t)M + 63) / 64, fill = std::max<int64_t>(direct_waves(staged, col_tiles) / 4 / groups, 1), trips = (row_blocks + fill - 1) / fill;
        const int blocks = (int)((row_blocks + trips - 1) / trips);
        const int used = (all + col_tiles - 1) / col_tiles;
        const dim3 grid(used * blocks);
        const size_t lds = (size_t)4 * 16 * (col_tiles * 16 + 4) * sizeof(float);
        // (the words: all of them here, or what another product's cannot know)
        DaWords words{want_db ? nullptr : plan, nullptr, 0ull, delta_a, delta_b, nullptr};
        if (N > 32 && want_db) col_abs_b = words.col_abs = reinterpret_cast<unsigned int *>(base + L.ss_b);
        if (!want_db && bwd_direct_diag(M, N, K)) {
            words.records = reinterpret_cast<unsigned long long *>(base + L.records);
            words.tag = next_finish_tag();
            if (grid.x > kBwdDirectRecordBytes / (2 * sizeof(unsigned long long))) return CDL_ERR_PARAM;      // (at most 512 blocks)
        }
#define CDL_DA_N(NN, STORE) CDL_LAUNCH("da_direct_kernel", stream, (da_direct_kernel<NN, STORE>), grid, dim3(256), STORE == kDaRows || STORE == kDaFlat ? lds : 0, gr, b_idx, M, N, K, col_tiles, blocks, (double)delta_b, (double)b_offset, d_a_hat, words)
#define CDL_DA(STORE) do { if (N <= 16) CDL_DA_N(16, STORE); else CDL_DA_N(32, STORE); } while (0)
#define CDL_DA_WIDE(STORE) do { if (N <= 48) CDL_DA_N(48, STORE); else CDL_DA_N(64, STORE); } while (0)
        if (da_columns_serves(M, N, K))
            CDL_LAUNCH("da_direct_kernel", stream, da_columns_kernel, dim3((unsigned)(((int64_t)M + kDaColumnsRows - 1) / kDaColumnsRows), (unsigned)((K / 4 + 255) / 256)), dim3(256), 0, gr, b_idx, M, N, K, (double)delta_b, (double)b_offset, d_a_hat, words.plan);
        else if (N > 32) { if (K % 4 == 0) CDL_DA_WIDE(kDaWords); else CDL_DA_WIDE(kDaScalars); }
        else if (K % 4 == 0) { if (staged) CDL_DA(kDaRows); else CDL_DA(kDaWords); }
        else if (used == 1 && staged) CDL_DA(kDaFlat);
        else CDL_DA(kDaScalars);
#undef CDL_DA_WIDE
#undef CDL_DA_N
#undef CDL_DA
        d_a_hat = nullptr;           // done; what follows is for the other product only
        if (!want_db) return check_launch();
    }

    const int asked = (d_a_hat ? 1 : 0) + (want_db ? 1 : 0);
    if (!cw && bwd_direct_serves(M, N, K, only_b, partial, L.direct_splits, !is_conv_weights, asked))
        return launch_bwd_direct(gr, a_idx, b_idx, M, N, K, delta_a, delta_b, a_offset, b_offset, d_a_hat, d_b_hat, plan, base + L.records, partial, L.direct_splits, only_b, !is_conv_weights, col_abs_b, stream);

    const bool by_rows = d_a_hat && limb_by_rows(M, N, K, L.splits);
    int8_t *bt = reinterpret_cast<int8_t *>(base + L.bt);
    int8_t *at = reinterpret_cast<int8_t *>(base + L.at);

    unsigned int *block_max = reinterpret_cast<unsigned int *>(base + L.block_max);
    unsigned int *ss_a = reinterpret_cast<unsigned int *>(base + L.ss_a);
    unsigned int *ss_b = reinterpret_cast<unsigned int *>(base + L.ss_b);
    // the column sums that the weight gradient needs besides (below) are of the same pass over g as its largest entry
    int n_max = L.n_max;
    const int n_clear = (int)((L.ss_b - L.ss_a) / sizeof(unsigned int)) + (col_abs_b ? 0 : K);
    if (want_db && a_offset != 0) {
        double *cp = reinterpret_cast<double *>(base + L.colsum_partial);
        const int most = L.n_max < kColsumBlocks ? L.n_max : kColsumBlocks, rows_per = (M + most - 1) / most;
        n_max = (M + rows_per - 1) / rows_per;
        if (N % 4 == 0) CDL_LAUNCH("g_colsum_kernel", stream, g_colsum_kernel<4>, dim3(n_max), dim3(256), 0, gr, M, N, rows_per, cp, block_max, ss_a, n_clear);
        else CDL_LAUNCH("g_colsum_kernel", stream, g_colsum_kernel<1>, dim3(n_max), dim3(256), 0, gr, M, N, rows_per, cp, block_max, ss_a, n_clear);
    } else {
        CDL_LAUNCH("absmax_kernel", stream, absmax_kernel, dim3(L.n_max), dim3(256), 0, gr, (int64_t)M * N, block_max, ss_a, n_clear);
    }
    {
        // the larger operand first: what is left when its blocks run out is the smaller one's
        TransposeJob ja{}, jb{};
        if (want_db) ja = transpose_job(a_idx, M, K, at, L.ldm, ss_a);
        if (d_a_hat) (want_db ? jb : ja) = transpose_job(b_idx, N, K, bt, L.ldn, ss_b, by_rows);
        const PlanArgs pa{plan, block_max, n_max, ss_a, ss_b, want_db ? K : 0, d_a_hat ? K : col_abs_b ? 1 : 0, delta_a, delta_b, nullptr, 0ull};
        ConvGeom g{};
        if (cw) {
            g = ConvGeom{cw->B, cw->H, cw->W, cw->C, cw->R, cw->S, cw->stride, cw->pad, cw->P, cw->Q, 0, make_div_by((uint32_t)cw->P * (uint32_t)cw->Q), make_div_by((uint32_t)cw->Q)};
            const uint32_t pb = (uint32_t)(uint8_t)(int8_t)(-a_offset);
            g.pad_word = (int)(pb | (pb << 8) | (pb << 16) | (pb << 24));
        }
        const int rc = launch_transposes(ja, jb, cw ? &g : nullptr, pa, base + L.records, stream);
        if (rc != CDL_OK) return rc;
    }
    // operands stored as index - offset: d_a_hat lacks delta_b * ob * sum_n g[m][n] in row m, d_b_hat lacks
    // delta_a * oa * sum_m g[m][n] in row n; both sums are taken of the unrounded g, in double
    double *corr_da = nullptr, *corr_db = nullptr;
    if (d_a_hat && b_offset != 0) {
        corr_da = reinterpret_cast<double *>(base + L.corr_da);
        CDL_LAUNCH("g_rowsum_kernel", stream, g_rowsum_kernel, dim3(blocks_for(M, 4, 8192)), dim3(256), 0, gr, M, N,
                   (double)delta_b * (double)b_offset, corr_da);
    }
    if (want_db && a_offset != 0) {
        corr_db = reinterpret_cast<double *>(base + L.corr_db);
        CDL_LAUNCH("g_colsum_finish_kernel", stream, g_colsum_finish_kernel, dim3((N + 7) / 8), dim3(256), 0,
                   reinterpret_cast<const double *>(base + L.colsum_partial), n_max, N,
                   (double)delta_a * (double)a_offset, corr_db);
    }
    int rc = check_launch();
    if (rc != CDL_OK) return rc;

    LimbArgs pa{}, pb{};
    pa.G = pb.G = gr;
    pa.M = pb.M = M;
    pa.N = pb.N = N;
    pa.cols = pb.cols = K;
    pa.plan = pb.plan = plan;
    pa.Bt = bt; pa.ldb = L.ldn;
    pa.rows = M; pa.kc = N;
    pa.nk = L.nk_n;
    pa.tiles_r = (M + kLRows - 1) / kLRows; pa.splits = 1; pa.kt_per_split = L.nk_n;
    pa.which = 0;
    pa.out = d_a_hat;
    pa.row_corr = corr_da;
    pb.Bt = at; pb.ldb = L.ldm;
    pb.rows = N; pb.kc = M;
    pb.nk = L.nk_m;
    pb.tiles_r = (N + kLRows - 1) / kLRows; pb.splits = L.splits; pb.kt_per_split = L.kt_per_split;
    pb.which = 1;
    pb.out = d_b_hat; pb.partial = partial;
    pb.row_corr = corr_db;
    if (by_rows) {
        rc = launch_limb_rows(gr, bt, 32 * L.ldn, M, N, K, plan, corr_da, d_a_hat, stream);
        if (rc == CDL_OK && want_db) rc = launch_limb_gemm(pb, true, stream);
    } else if (d_a_hat && want_db && limb_pair_serves(M, N, K, L.splits)) {
        rc = launch_limb_pair(pa, pb, stream);
    } else {
        if (d_a_hat) rc = launch_limb_gemm(pa, false, stream);
        if (rc == CDL_OK && want_db) rc = launch_limb_gemm(pb, true, stream);
    }
    if (rc != CDL_OK) return rc;
    if (want_db) {
        if (L.splits > 1) {
            if ((int64_t)N * K <= 65536 && L.splits >= 32)
                CDL_LAUNCH("limb_reduce_kernel", stream, limb_reduce_kernel<16>, dim3(blocks_for((int64_t)N * K * 16, 256, 4096)), dim3(256), 0,
                           partial, L.splits, (int64_t)N * K, plan, d_b_hat, corr_db, K);
            else
                CDL_LAUNCH("limb_reduce_kernel", stream, limb_reduce_kernel<1>, dim3(blocks_for((int64_t)N * K, 256, 4096)), dim3(256), 0,
                           partial, L.splits, (int64_t)N * K, plan, d_b_hat, corr_db, K);
            rc = check_launch();
        }
    }
    return rc;
}

int launch_qgemm_bwd_quantize_bwd(const float *g, const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K,
                                  int32_t a_offset, int32_t b_offset, float delta_b, const float *theta_a, const cdl_qparams &p_a,
                                  float *d_theta_a, float *d_delta_a, float *d_alpha_a, float *d_b_hat, const float *theta_b,
                                  const cdl_qparams *p_b, float *d_theta_b, float *d_delta_b, float *d_alpha_b, void *ws, hipStream_t stream)
{
    float *b_hat = d_b_hat ? d_b_hat : d_theta_b;      // (null: the weight gradient is not asked for)
    int rc = launch_qgemm_bwd(g, a_idx, b_idx, M, N, K, p_a.delta, delta_b, a_offset, b_offset, d_theta_a, b_hat, ws, stream);
    if (rc != CDL_OK) return rc;
    void *scalars = reinterpret_cast<char *>(ws) + bwd_layout(M, N, K).scalars;
    rc = launch_quantize_bwd(theta_a, d_theta_a, (int64_t)M * K, p_a, d_theta_a, d_delta_a, d_alpha_a, scalars, stream);
    if (rc == CDL_OK && d_theta_b)
        rc = launch_quantize_bwd(theta_b, b_hat, (int64_t)N * K, *p_b, d_theta_b, d_delta_b, d_alpha_b, scalars, stream);
    return rc;
}

}  // namespace cdl
