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

// Where this kernel serves, us, tiles / so.  Rows beyond qgemm_small_serves: 33000 x 32 x 2048 23.1 / 24.5, 65536 x 32 x 1024 22.0 / 15.9, 60000 x 27 x 147 9.9 / 10.1.
// Windows of a long contraction are read again tap by tap, by each wave for itself: 102459 x 20 x 1152 21.8 / 25.5, 25088 x 32 x 512 6.4 / 9.5, but 401408 x 32 x 288
// 36.8 / 21.9; 16384 x 16 x 144 4.3 / 4.3.
bool qgemm_thin_serves(int32_t N, int32_t K, int32_t b_offset) { return N <= 32 && K >= 16 && (N <= 16 || K <= 1024) && b_offset == 0; }

int launch_qgemm_thin(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float scale, int32_t a_offset, int32_t *acc, float *y,
                      hipStream_t stream)
{
    ThinFwdArgs a{};
    a.X = a_idx; a.W = b_idx;
    a.M = M; a.N = N; a.K = K; a.off = a_offset;
    a.acc = acc; a.y = y; a.scale = scale;
    return launch_thin(a, false, stream);
}

bool qconv_thin_serves(int64_t M, int32_t N, int32_t K) { return N <= 32 && K <= 320 && M >= 16384; }

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
