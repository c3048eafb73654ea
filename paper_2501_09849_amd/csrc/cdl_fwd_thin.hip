// Forward products with few output columns: rows of indices, or the windows of a convolution, times up to 32 columns.
//
// Tiles of 64 columns and more are padding here, and staging operands in LDS, tile after tile, is a chain of trips to memory around a handful of matrix
// instructions.  A wave forms 64 rows x 16 (32) columns on its own: a lane reads 16 bytes of a row (of one tap of a window's pixel) and of a
// column of weights straight into the fragments of v_mfma_i32_16x16x64_i8, kAhead steps of 64 contraction entries under way, with no LDS and no
// barrier.  The weights are the rows of the result's tile, so that a lane has four neighbouring columns of a row and a wave stores whole lines.
// Sums are exact int32; those of the weights that an offset of the other operand needs come from one more product with ones.
//
// What bounds it: memory for long rows, the launch and two trips to memory for short ones.  us, in tiles of
// 256 x 64 / so: 131072 rows of 144, 16 columns 9.6 / 6.3 (4.3 TB/s), of unsigned indices 16.3 / 6.2; 65536 of 3072 46.6 / 33.6; 128 x 32 x 32 x 16 -> 16, 3 x 3  10.5 / 5.8.
#include "cdl_internal.h"
#include "cdl_div.h"
#include "cdl_limbs.h"
#include "cdl_rows.h"

namespace cdl {

namespace {

constexpr int kThinFwdWaves = 4, kThinFwdRows = 64 * kThinFwdWaves;

struct ThinFwdArgs {
    const int8_t *X, *W;      // rows (or activations [B][H][W][C]), weights [N][K]
    int64_t M;
    int N, K, off;            // off: what was subtracted from the indices of X
    int32_t *acc;             // [M][N] or null
    float *y;                 // [M][N] or null
    float scale;
    int vec;                  // outputs in 16-byte stores
    int64_t share;            // blocks of an XCD
    // windows: M = B P Q of them
    int H, Wd, C, S, stride, pad, P, Q, pad_word;
    DivBy by_pq, by_q, by_cu, by_s;      // by_cu: C / 16
};

template <bool CONV, int TN>
__global__ __launch_bounds__(64 * kThinFwdWaves)
void fwd_thin_kernel(ThinFwdArgs a)
{
    constexpr int kAhead = 3;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, own = lane & 15, g4 = lane >> 4;
    // XCD x takes the x-th eighth of the rows (neighbouring windows share rows of the image)
    const int64_t block = (blockIdx.x & 7) * a.share + (blockIdx.x >> 3), row0 = block * kThinFwdRows + wave * 64;
    if ((int64_t)(blockIdx.x >> 3) >= a.share || row0 >= a.M) return;
    const int K = a.K, steps = (K + 63) >> 6;
    const int8_t *row[4], *col[TN];
    int h0[4], w0[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t at = row0 + 16 * i + own, m = at < a.M ? at : a.M - 1;
        if (CONV) {
            const int mi = (int)m, b = div_by(mi, a.by_pq), rem = mi - b * (a.P * a.Q), p = div_by(rem, a.by_q), q = rem - p * a.Q;
            h0[i] = p * a.stride - a.pad;
            w0[i] = q * a.stride - a.pad;
            row[i] = a.X + (int64_t)b * a.H * a.Wd * a.C;      // the image
        } else {
            row[i] = a.X + m * K;
        }
    }
#pragma unroll
    for (int c = 0; c < TN; ++c) col[c] = a.W + (int64_t)min(16 * c + own, a.N - 1) * K;

    v4i fa[kAhead][4], fb[kAhead][TN];
    int inside[kAhead];       // CONV: bit i, whether the pixel is there
    auto load = [&](int buf, int s) {
        const int k0 = 64 * s + 16 * g4;
        inside[buf] = 0;
        if (CONV) {
            const int u = min(4 * s + g4, (K >> 4) - 1), t = div_by(u, a.by_cu), r = div_by(t, a.by_s), sx = t - r * a.S, c = 16 * (u - t * (a.C >> 4));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int h = h0[i] + r, w = w0[i] + sx;
                const bool in = (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.Wd;
                inside[buf] |= in ? 1 << i : 0;
                fa[buf][i] = *reinterpret_cast<const v4i *>(row[i] + (in ? (h * a.Wd + w) * a.C + c : 0));      // (an image has fewer than 2^31 entries)
            }
#pragma unroll
            for (int c16 = 0; c16 < TN; ++c16) {
                fb[buf][c16] = *reinterpret_cast<const v4i *>(col[c16] + 16 * u);
                if (k0 >= K) fb[buf][c16] = v4i{0, 0, 0, 0};
            }
        } else if (64 * s + 64 <= K) {
#pragma unroll
            for (int i = 0; i < 4; ++i) fa[buf][i] = load_any16(row[i] + k0);
#pragma unroll
            for (int c = 0; c < TN; ++c) fb[buf][c] = load_any16(col[c] + k0);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) fa[buf][i] = tail_chunk(row[i], k0, K);
#pragma unroll
            for (int c = 0; c < TN; ++c) fb[buf][c] = tail_chunk(col[c], k0, K);
        }
    };
    v4i acc[4][TN], sums[TN];
#pragma unroll
    for (int c = 0; c < TN; ++c) {
        sums[c] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][c] = v4i{0, 0, 0, 0};
    }
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101}, padding = {a.pad_word, a.pad_word, a.pad_word, a.pad_word};
    auto multiply = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v4i x = fa[buf][i];
            if (CONV && !(inside[buf] >> i & 1)) x = padding;
#pragma unroll
            for (int c = 0; c < TN; ++c) acc[i][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[buf][c], x, acc[i][c], 0, 0, 0);
        }
        if (a.off)
#pragma unroll
            for (int c = 0; c < TN; ++c) sums[c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[buf][c], ones, sums[c], 0, 0, 0);
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (u < steps) load(u, u);
    for (int s = 0; s < steps; s += kAhead)
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (s + u < steps) multiply(u);
            if (s + u + kAhead < steps) load(u, s + u + kAhead);
        }

    // register r: row of the weights 4 (lane / 16) + r, column lane % 16
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = row0 + 16 * i + own;
        if (m >= a.M) continue;
#pragma unroll
        for (int c = 0; c < TN; ++c) {
            const int n = 16 * c + 4 * g4;
            const int64_t at = m * a.N + n;
            int v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (int)((unsigned)acc[i][c][r] + (unsigned)a.off * (unsigned)sums[c][r]);
            if (a.vec) {
                if (n >= a.N) continue;
                if (a.acc) *reinterpret_cast<int4 *>(a.acc + at) = make_int4(v[0], v[1], v[2], v[3]);
                if (a.y) *reinterpret_cast<float4 *>(a.y + at) = make_float4(a.scale * (float)v[0], a.scale * (float)v[1], a.scale * (float)v[2], a.scale * (float)v[3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (n + r >= a.N) continue;
                    if (a.acc) a.acc[at + r] = v[r];
                    if (a.y) a.y[at + r] = a.scale * (float)v[r];
                }
            }
        }
    }
}

int launch_thin(ThinFwdArgs a, bool conv, hipStream_t stream)
{
    a.vec = a.N % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.acc) | reinterpret_cast<uintptr_t>(a.y)) & 15) == 0;
    a.share = ((a.M + kThinFwdRows - 1) / kThinFwdRows + 7) / 8;
    const dim3 grid((unsigned)(8 * a.share)), block(64 * kThinFwdWaves);
    const char *name = conv ? "fwd_thin_kernel(windows)" : "fwd_thin_kernel";
    if (conv && a.N <= 16) CDL_LAUNCH(name, stream, (fwd_thin_kernel<true, 1>), grid, block, 0, a);
    else if (conv) CDL_LAUNCH(name, stream, (fwd_thin_kernel<true, 2>), grid, block, 0, a);
    else if (a.N <= 16) CDL_LAUNCH(name, stream, (fwd_thin_kernel<false, 1>), grid, block, 0, a);
    else CDL_LAUNCH(name, stream, (fwd_thin_kernel<false, 2>), grid, block, 0, a);
    return check_launch();
}

}  // namespace

// Where this kernel serves, us, tiles of 64 columns / so, beyond qgemm_small_serves.
// Rows of up to 1664 entries, up to 2048 for 8 columns, the more so with an offset, whose sums cost the others a launch: 65536 x 16 x 144 8.2 / 4.6 (15.1 / 4.6), 100000 x 16 x 1024 23.4 / 22.8, 131072 x 32 x
// 144 12.4 / 9.6; two tiles of columns 65536 x 32 x 1024 22.1 / 15.8, 70001 x 32 x 768
// 19.9 / 21.4, x 400 14.6 / 13.2, 131072 x 32 x 768 24.9 / 24.0, x 1024 29.3 / 31.4 (36.4 / 31.5).  Longer ones, up to 16 columns, while
// all waves fit the chip at once: 65536 x 16 x 2048 33 / 25, 100000 x 16 x 2048 44.8 / 51.9 (51.8 / 51.7), 98000 x 16 x 1600 40 / 38, x 2000 58 / 60, x 8 x 1600 40 / 37, 190000 x 8 x 1376 77 / 65.  Rows that start at odd addresses: 100000 x 16 x 147
// 10.6 / 10.2, x 577 20.3 / 27.3 (26.7 / 27.2), 65536 x 1 x 577 17.8 / 13.7, 33000 x 1 x 577 11.0 / 12.7; 70001 x 26 x 250 (18.9 / 16.4).  Rows of the result that are no
// multiple of four wide are stored word by word, which the second tile of 16 columns does not pay for: 70001 x 17 x 144 8.7 / 6.6, x 22 8.8 / 9.0,
// x 31 9.2 / 10.2, 131072 x 31 x 144 12.2 / 15.8 (20 / 17).
bool qgemm_thin_serves(int32_t M, int32_t N, int32_t K, int32_t a_offset, int32_t b_offset)
{
    if (N > 32 || K < 16 || b_offset != 0) return false;
    const bool words = K % 4 == 0, at_once = M <= 65536, offset = a_offset != 0;
    if (N <= 16) return words ? K <= (N <= 8 ? 2048 : 1664) || at_once || offset : K <= (offset || (N <= 4 && M > 49152) ? 640 : 256);
    if (offset) return K <= (words ? 1024 : 512);
    const int64_t rounds = ((int64_t)M + 65535) / 65536;      // of resident waves; the last one may be nearly empty
    return (N % 4 == 0 || N < 20) && K <= (!words ? 160 : at_once ? 1024 : 8 * (int64_t)M >= 7 * 65536 * rounds ? 768 : 448);
}

int launch_qgemm_thin(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float scale, int32_t a_offset, int32_t *acc, float *y,
                      hipStream_t stream)
{
    ThinFwdArgs a{};
    a.X = a_idx; a.W = b_idx;
    a.M = M; a.N = N; a.K = K; a.off = a_offset;
    a.acc = acc; a.y = y; a.scale = scale;
    return launch_thin(a, false, stream);
}

// Windows are read again tap by tap, by each wave for itself.  30720 windows of 16 channels, 3 x 3, 16 columns 5.0 / 4.8 (8.6 / 4.9), 32 columns 5.2 / 5.6 (9 / 5.6), 32805 6.6 / 5.5;
// 30720 of 32 channels, 16 columns 5.7 / 5.7, 32 5.9 / 6.6 (9.6 / 6.7); 61 K 7.9 / 6.0 and 8.3 / 7.2; 102459 x 20 x 1152 21.8 / 25.5, but 401408 x 32 x 288 36.8 / 21.9.
bool qconv_thin_serves(int64_t M, int32_t N, int32_t K, int32_t x_offset)
{
    if (N > 32 || K > 320) return false;
    if (x_offset != 0) return M >= 16384;
    return N <= 16 ? M >= (K <= 160 ? 16384 : 32768) : (N % 4 == 0 || N < 20) && M > 32768;
}

int launch_qconv_thin(const int8_t *x_idx, const int8_t *w_idx, const ConvWindows &w, int32_t N, float scale, int32_t x_offset, int32_t *acc, float *y,
                      hipStream_t stream)
{
    ThinFwdArgs a{};
    a.X = x_idx; a.W = w_idx;
    a.M = (int64_t)w.B * w.P * w.Q; a.N = N; a.K = w.R * w.S * w.C; a.off = x_offset;
    a.acc = acc; a.y = y; a.scale = scale;
    a.H = w.H; a.Wd = w.W; a.C = w.C; a.S = w.S; a.stride = w.stride; a.pad = w.pad; a.P = w.P; a.Q = w.Q;
    a.pad_word = (int)(0x01010101u * (uint32_t)(uint8_t)(int8_t)(-x_offset));
    a.by_pq = make_div_by((uint32_t)w.P * (uint32_t)w.Q);
    a.by_q = make_div_by((uint32_t)w.Q);
    a.by_cu = make_div_by((uint32_t)(w.C / 16));
    a.by_s = make_div_by((uint32_t)w.S);
    return launch_thin(a, true, stream);
}

}  // namespace cdl
