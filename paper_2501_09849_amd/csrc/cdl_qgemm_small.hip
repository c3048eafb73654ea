// Forward layer product over quantized operands (Sec. IV-A) for problems with few output tiles.
//
// The kernels of cdl_qgemm.hip give a block a 128 - 256 row tile and walk the contraction one K-tile after the other:
// with fewer tiles than compute units a launch is one chain of memory latencies (16 x 3072 x 768: 24 blocks, twelve
// steps, 14.4 us for 3 MB).  Here a tile is small and the contraction of a tile is split over the waves of its block,
// whose int32 sums are exact and are added through LDS at the end.  Operand fragments go from memory straight to
// registers: a lane reads 64 consecutive bytes of its row as four 16-byte loads, so that the two lanes of a row share a
// 128-byte line and all of it is used at once; the order of the contraction inside a block of 128 does not matter as
// long as both operands share it.  Rows need no alignment and K any multiple: the last, partial block is shifted into
// place in registers.  What bounds it is the L2: a wave's tile of 64 x 64 reads 16 KB for 16 MFMAs.
#include "cdl_internal.h"
#include "cdl_rows.h"

#include <type_traits>

namespace cdl {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

struct SmallArgs {
    const int8_t *A;      // [M][K]
    const int8_t *B;      // [N][K]
    int M, N, K;
    int tiles_m, tiles_n;
    int32_t *acc_out;     // [M][N] or null
    float *y_out;         // [M][N] or null
    float scale;
    int oa, ob;           // offsets the operands were stored with
};

// 32 x 32 MFMA tiles of a block, and its waves
constexpr int TM = 1, TN = 1, KS = 4;

// OFF: operands stored with an offset.
template <bool OFF>
__global__ __launch_bounds__(64 * KS)
void qgemm_small_kernel(SmallArgs a)
{
    constexpr int R = TM * TN * 16;
    __shared__ int red[KS][R][64];

    const int total = a.tiles_m * a.tiles_n;
    const int per_xcd = (int)gridDim.x >> 3;
    const int logical = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (logical >= total) return;
    const int tile_m = logical / a.tiles_n, tile_n = logical % a.tiles_n;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h64 = (lane >> 5) * 64;

    const int8_t *pa[TM];
    const int8_t *pb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) pa[i] = a.A + (int64_t)min((tile_m * TM + i) * 32 + (lane & 31), a.M - 1) * a.K;
#pragma unroll
    for (int j = 0; j < TN; ++j) pb[j] = a.B + (int64_t)min((tile_n * TN + j) * 32 + (lane & 31), a.N - 1) * a.K;

    v16i acc[TM][TN], rs[TM], cs[TN];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            rs[i][r] = 0;
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j][r] = 0;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) cs[j][r] = 0;
    }

    const int full = a.K >> 7, nkb = (a.K + 127) >> 7;
    v4i fa[2][TM][4], fb[2][TN][4];
    auto load = [&](auto buf_c, int kb) {
        constexpr int buf = decltype(buf_c)::value;
        const int k0 = kb * 128 + h64;
        if (kb < full) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[buf][i][c] = load_any16(pa[i] + k0 + 16 * c);
#pragma unroll
                for (int j = 0; j < TN; ++j) fb[buf][j][c] = load_any16(pb[j] + k0 + 16 * c);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[buf][i][c] = tail_chunk(pa[i], k0 + 16 * c, a.K);
#pragma unroll
                for (int j = 0; j < TN; ++j) fb[buf][j][c] = tail_chunk(pb[j], k0 + 16 * c, a.K);
            }
        }
    };
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    auto multiply = [&](auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[buf][i][c], fb[buf][j][c], acc[i][j], 0, 0, 0);
            if (OFF) {
                // sums of the stored indices along the contraction, in the layout of the product
#pragma unroll
                for (int i = 0; i < TM; ++i) rs[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[buf][i][c], ones, rs[i], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < TN; ++j) cs[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ones, fb[buf][j][c], cs[j], 0, 0, 0);
            }
        }
    };
    constexpr auto b0 = std::integral_constant<int, 0>{};
    constexpr auto b1 = std::integral_constant<int, 1>{};
    int kb = wave;
    if (kb < nkb) load(b0, kb);
    while (kb < nkb) {
        if (kb + KS < nkb) load(b1, kb + KS);
        multiply(b0);
        kb += KS;
        if (kb >= nkb) break;
        if (kb + KS < nkb) load(b0, kb + KS);
        multiply(b1);
        kb += KS;
    }

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                red[wave][(i * TN + j) * 16 + r][lane] = OFF ? (int)((unsigned)acc[i][j][r] + (unsigned)a.oa * (unsigned)cs[j][r] + (unsigned)a.ob * (unsigned)rs[i][r]) : acc[i][j][r];
    __syncthreads();
    // wave w finishes registers w, w + KS, ...: lane holds column lane % 32, register r row 8 (r / 4) + 4 (lane / 32) + r % 4
    const int constant = OFF ? a.K * a.oa * a.ob : 0;
    for (int q = wave; q < R; q += KS) {
        unsigned int sum = (unsigned int)constant;        // (the waves' parts may wrap where the sum does not)
#pragma unroll
        for (int w = 0; w < KS; ++w) sum += (unsigned int)red[w][q][lane];
        const int v = (int)sum;
        const int r = q & 15, j = (q >> 4) % TN, i = (q >> 4) / TN;
        const int row = (tile_m * TM + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), col = (tile_n * TN + j) * 32 + (lane & 31);
        if (row < a.M && col < a.N) {
            const int64_t o = (int64_t)row * a.N + col;
            if (a.acc_out) a.acc_out[o] = v;
            if (a.y_out) a.y_out[o] = a.scale * (float)v;
        }
    }
}

int launch_tiles(SmallArgs a, hipStream_t stream)
{
    a.tiles_m = (a.M + 32 * TM - 1) / (32 * TM);
    a.tiles_n = (a.N + 32 * TN - 1) / (32 * TN);
    const int64_t grid = ((int64_t)a.tiles_m * a.tiles_n + 7) / 8 * 8;
    if (a.oa || a.ob) CDL_LAUNCH("qgemm_kernel(fwd)", stream, qgemm_small_kernel<true>, dim3((unsigned)grid), dim3(64 * KS), 0, a);
    else CDL_LAUNCH("qgemm_kernel(fwd)", stream, qgemm_small_kernel<false>, dim3((unsigned)grid), dim3(64 * KS), 0, a);
    return check_launch();
}

}  // namespace

// Where this kernel serves, measured against the other forward kernels (us, y only):
//   16 x 3072 x 768     13.9 ->  3.3      384 x  320 x 1664   18.0 -> 5.3     10366 x 128 x  832  12.9 -> 9.2
//   256 x 1000 x 512    10.0 ->  3.4     1988 x  225 x  752   11.9 -> 4.2      1024 x 1024 x 1024 14.1 -> 10.1
//   512 x 512 x 4096    35.1 ->  9.6       85 x  747 x 2951   52.7 -> 15.4    20000 x  64 x  512   7.4 -> 8.0
// i.e. up to about a thousand tiles of 32 x 32.  Twice as many at most where contractions are no multiple of 16, by what the others lack there: their tiles shift a row's end into
// place, they take a launch for each operand's sums beside an offset (those of the rows most), and the kernel for few columns has no offset of the weights.  Here a lane's 16 bytes take far
// longer at addresses that are no multiples of four.  us, here / there, at 1040 | 1600 | 2040 tiles: 16 columns x 300 6.5 / 5.9 | 9.2 / 7.1 | 10.6 / 8.1, x 1468 13 / 18 | 21 / 24 | 25 / 27, x 301 8.9 / 9
// | 15.5 / 11 | 18 / 13; offset of the weights, x 300 8.8 / 17 | 10 / 19 | 13 / 22, x 3001 55 / 57 | 70 / 73; 300 columns x 300 8.0 / 8.5 | 11.4 / 9.9, x 700 7.4 / 9.3 | 12.5 / 11; both offsets x 75
// 8.4 / 14.4 | 11.8 / 15.9 | 12 / 16.  Over 5 K shapes this rule is 0.6 % in the mean from the better of both, and 20 % better than 2048 tiles for all of them.
static int64_t most_tiles(int32_t N, int32_t K, int32_t a_offset, int32_t b_offset)
{
    if (K % 16 == 0) return 1024;
    const bool words = K % 4 == 0;
    if (b_offset != 0) {
        if (words) return N <= 512 || K < 1536 ? 2048 : 1664;
        if (N > 32) return K < 192 ? 2048 : K < 384 ? 1536 : 1024;
        return N <= 12 || K < 1024 || (N <= 24 && K < 1536) ? 2048 : K < 1536 ? 1408 : N <= 16 ? 1280 : 1024;
    }
    if (a_offset != 0) {
        if (N <= 32) return words ? (K < 1024 ? 1024 : N <= 16 && K < 1536 ? 1280 : 1792) : K >= 512 && K < 1024 ? 1280 : 1024;
        return words || K < 256 ? 1536 : 1024;
    }
    if (!words) return N > 32 && K >= 64 && K < 128 ? 1536 : 1024;
    if (N <= 16) return K < 640 ? 1024 : K < 1100 ? 1664 : 2048;
    if (N <= 32) return K < 128 ? 1024 : K < 640 ? 1536 : 1664;
    return N > 512 && K < 768 ? 1536 : K < 384 || K >= 1024 ? 1280 : 1200;
}

bool qgemm_small_serves(int32_t M, int32_t N, int32_t K, int32_t a_offset, int32_t b_offset)
{
    return K >= 16 && (int64_t)((M + 31) / 32) * ((N + 31) / 32) <= most_tiles(N, K, a_offset, b_offset);
}

int launch_qgemm_small(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float scale, int32_t a_offset,
                       int32_t b_offset, int32_t *acc, float *y, hipStream_t stream)
{
    SmallArgs a{};
    a.A = a_idx; a.B = b_idx;
    a.M = M; a.N = N; a.K = K;
    a.acc_out = acc; a.y_out = y;
    a.scale = scale;
    a.oa = a_offset; a.ob = b_offset;
    return launch_tiles(a, stream);
}

}  // namespace cdl
