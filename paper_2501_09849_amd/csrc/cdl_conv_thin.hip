// dL/dQ(x) of convolutional layers of stride 1 with up to 32 channels on both sides, exactly, from digits of g that stay in LDS.
//
// Few channels leave a limb tile mostly padding.  conv_dx_direct_kernel forms such layers in double, and gathers an entry of g once per tap: loaded, tested
// against the image's edge, addressed in 64 bits, converted.  Here a block loads the contiguous range of g that its run of pixels
// needs once (as cdl_conv_patch.hip does), turns it into six int8 digits scaled by the range's largest entry, and a table says where each tap's
// pixel lies in LDS (outside the image: a row of zeros).  A wave forms 64 pixels x 16 channels, for 32 channels one 16 after the other.
//
// Every product is exact, as it is in double: digits hold entries down to 2^-22 of the largest in full.  If there are smaller ones the block makes digits
// of those, scaled by the largest of them, and so on; digit sums are exact in int32 and added up in double.  A range with an infinity or a NaN is
// formed in double as a whole.
//
// What bounds it: a wave's instructions (digits, table, putting the digit sums together; the matrix instructions, 1152 cycles a wave at 3 x 3 x 16, are a
// seventh of it), two waves to a SIMD, and the trips to memory before them.
#include "cdl_internal.h"
#include "cdl_div.h"
#include "cdl_limbs.h"

namespace cdl {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kThinWaves = 4, kThinPixels = 64 * kThinWaves, kThinDigits = 6;
constexpr int kThinKeep = 6, kThinKept = kThinKeep * kThinPixels / 4;      // quads of channels that a thread keeps in registers, pixels of up to 16 channels that so are kept
constexpr int kThinLds = 160 << 10;      // (two blocks share a compute unit where they fit)
constexpr int kThinUnits = 25;           // most units of 16 contraction entries
static_assert(257ll * 128 * 128 * 16 * kThinUnits < (1ll << 31), "a digit sum, times 256 and another added, fits an int32");

struct ThinArgs {
    const float *g;
    const int8_t *w;                 // [N][R][S][C]
    float *out;
    int N, C, P, Q, S, taps;
    int Hc, Wc, pad_h, pad_w;
    int rows, tiles, share;          // pixels, runs of them, and those of an XCD
    int lo_h, hi_h, lo_w, hi_w;      // rows and columns of g that a pixel reads, from its own
    DivBy by_hw, by_w;
    int pixels;                      // of g
    int px_max, patch_bytes;         // pixels of a patch, at most (row px_max: zeros)
    double delta;
};

// TN: tiles of 16 input channels; NU: units of 16 output channels.
// LDS: the patch - digit planes [kThinDigits][px_max + 1][kPlaneStride] bytes, or floats [px_max + 1][16 NU + 4] -, then the weights [units of 16
// contraction entries][16 TN][16], then the table [taps + 1][waves][16][4], then the reductions.
template <int TN, int NU>
__global__ __launch_bounds__(kThinPixels, 2)
void conv_dx_thin_kernel(ThinArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t thin_lds[];
    constexpr int T = kThinPixels, NQ = 4 * NU, kPlaneStride = 16 * NU, kStride = 16 * NU + 4;
    // XCD x takes the x-th eighth of the runs (neighbours share rows of g)
    const int tile = ((int)blockIdx.x & 7) * a.share + ((int)blockIdx.x >> 3);
    if (tile >= a.tiles || ((int)blockIdx.x >> 3) >= a.share) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g4 = lane >> 4;
    const int N = a.N, C = a.C, P = a.P, Q = a.Q, Wc = a.Wc, hw = a.Hc * Wc, rows = a.rows, taps = a.taps, px_max = a.px_max;
    const int row0 = tile * T, plane = (px_max + 1) * kPlaneStride, units = taps * NU, steps = (units + 3) >> 2;
    int8_t *const planes = thin_lds;
    float *const floats = reinterpret_cast<float *>(thin_lds);
    int8_t *const weights = thin_lds + a.patch_bytes;
    uint16_t *const table = reinterpret_cast<uint16_t *>(weights + 4 * steps * 256 * TN);
    uint32_t *const red = reinterpret_cast<uint32_t *>(table + (taps + 1) * T);

    // the range of g
    int lo, count;
    {
        const int m1 = min(row0 + T, rows) - 1;
        const int b0 = div_by(row0, a.by_hw), rem0 = row0 - b0 * hw, i0 = div_by(rem0, a.by_w), j0 = rem0 - i0 * Wc;
        const int b1 = div_by(m1, a.by_hw), rem1 = m1 - b1 * hw, i1 = div_by(rem1, a.by_w), j1 = rem1 - i1 * Wc;
        const int p0 = i0 + a.lo_h, q0 = j0 + a.lo_w, p1 = i1 + a.hi_h, q1 = j1 + a.hi_w;
        // (above the image: from its first pixel on; below it: to its last one)
        const int from = (b0 * P + min(max(p0, 0), P - 1)) * Q + (p0 < 0 ? 0 : min(max(q0, 0), Q - 1));
        const int to = (b1 * P + min(max(p1, 0), P - 1)) * Q + (p1 > P - 1 ? Q - 1 : min(max(q1, 0), Q - 1));
        lo = __builtin_amdgcn_readfirstlane(from);
        count = __builtin_amdgcn_readfirstlane(min(max(to - from + 1, 1), min(px_max, a.pixels - from)));
    }
    const float *const src = a.g + (int64_t)lo * N;
    const int quads = count * NQ;      // of four channels; those beyond N are zeros
    constexpr int kKeep = kThinKeep;
    float4 kept[kKeep];
    const bool keeps = NU == 1 && quads <= kKeep * T;      // g is read once (32 channels: never so few)
    auto load = [&](int base, float4 (&v)[kKeep]) {
#pragma unroll
        for (int u = 0; u < kKeep; ++u) {
            const int i = min(base + u * T, quads - 1), n = 4 * (i % NQ);
            v[u] = *reinterpret_cast<const float4 *>(src + (i / NQ * N + min(n, N - 4)));      // (count N < 2^20)
            if (n >= N) v[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    // f(pixel, quad of channels, its four entries)
    auto each = [&](auto &&f) {
        for (int base = tid; base < quads; base += kKeep * T) {
            float4 v[kKeep];
            if (keeps)
#pragma unroll
                for (int u = 0; u < kKeep; ++u) v[u] = kept[u];
            else load(base, v);
#pragma unroll
            for (int u = 0; u < kKeep; ++u)
                if (base + u * T < quads) f((base + u * T) / NQ, (base + u * T) % NQ, v[u]);
        }
    };
    // where channel n of a pixel lies in a plane (32 channels: halves change places every eight pixels, no bank conflicts between neighbours)
    auto in_plane = [&](int px, int n) { return px * kPlaneStride + (NU == 2 ? n ^ ((px & 8) << 1) : n); };
    // largest of the threads' values
    int turn = 0;
    auto block_max = [&](uint32_t v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
        uint32_t *r = red + (turn & 1) * kThinWaves;
        ++turn;
        if (lane == 0) r[wave] = v;
        __syncthreads();
        v = max(max(r[0], r[1]), max(r[2], r[3]));
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    };

    if (keeps) load(tid, kept);
    {      // a word of the weights: four output channels
        constexpr int kWords = 4;
        const int words = 4 * steps * 64 * TN;
        for (int base = tid; base < words; base += kWords * T) {
            uint8_t b[kWords][4];
#pragma unroll
            for (int x = 0; x < kWords; ++x) {
                const int i = min(base + x * T, words - 1), c = min((i >> 2) & (16 * TN - 1), C - 1), u = min(i / (64 * TN), units - 1);
                const int t = u / NU, n = min(16 * (u - t * NU) + 4 * (i & 3), N - 4);
                const int8_t *p = a.w + ((n * taps + t) * C + c);
#pragma unroll
                for (int q = 0; q < 4; ++q) b[x][q] = (uint8_t)p[q * taps * C];
            }
#pragma unroll
            for (int x = 0; x < kWords; ++x) {
                const int i = min(base + x * T, words - 1), c = (i >> 2) & (16 * TN - 1), u = i / (64 * TN), n = 16 * (u % NU) + 4 * (i & 3);
                const uint32_t w = b[x][0] | (uint32_t)b[x][1] << 8 | (uint32_t)b[x][2] << 16 | (uint32_t)b[x][3] << 24;
                reinterpret_cast<uint32_t *>(weights)[i] = u < units && c < C && n < N ? w : 0u;
            }
        }
    }
    {      // pixel tid of the run: one place per tap
        const int m = row0 + tid, b = div_by(m, a.by_hw), rem = m - b * hw, ii = div_by(rem, a.by_w), jj = rem - ii * Wc;
        uint16_t *at = table + wave * 64 + (lane & 15) * 4 + g4;
        int r = 0, s = 0;
        for (int t = 0; t <= taps; ++t) {
            const int p = ii + a.pad_h - r, q = jj + a.pad_w - s;
            const bool inside = t < taps && m < rows && (unsigned)p < (unsigned)P && (unsigned)q < (unsigned)Q;
            const int px = (b * P + p) * Q + q - lo;
            at[t * T] = (uint16_t)(inside ? min(max(px, 0), px_max - 1) : px_max);
            if (++s == a.S) { s = 0; ++r; }
        }
    }
    for (int i = tid; i < kThinDigits * (kPlaneStride / 4); i += T) {
        const int l = i / (kPlaneStride / 4);
        reinterpret_cast<uint32_t *>(planes + l * plane + px_max * kPlaneStride)[i - l * (kPlaneStride / 4)] = 0u;
    }
    uint32_t largest = 0u;
    each([&](int, int, const float4 &v) {
        largest = max(largest, max(max(__float_as_uint(fabsf(v.x)), __float_as_uint(fabsf(v.y))), max(__float_as_uint(fabsf(v.z)), __float_as_uint(fabsf(v.w)))));
    });
    largest = block_max(largest);
    const uint16_t *const my_table = table + wave * 64 + (lane & 15) * 4;

    if (largest < 0x7f800000u) {
        double total[4][TN][4];      // [tile of 16 pixels][tile of channels][register]
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < TN; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) total[i][c][r] = 0.0;
        while (largest > 0u) {
            const int E = (int)(largest >> 23);
            const uint32_t least = (uint32_t)max(E - 22, 0) << 23;
            const double scale = __hiloint2double((1023 + 172 - E) << 20, 0), unit = __hiloint2double((1023 - 172 + E) << 20, 0);
            uint32_t rest = 0u;
            each([&](int px, int q, const float4 &v) {
                float g[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t bits = __float_as_uint(fabsf(g[e]));
                    rest = max(rest, bits < least ? bits : 0u);
                    g[e] = bits >= least && bits <= largest ? g[e] : 0.0f;      // (larger ones went before)
                }
                uint32_t d[kThinDigits];
                limbs_of4_wide<kThinDigits>(g, scale, d);
                int8_t *to = planes + in_plane(px, 4 * q);
#pragma unroll
                for (int l = 0; l < kThinDigits; ++l) *reinterpret_cast<uint32_t *>(to + l * plane) = d[l];
            });
            rest = block_max(rest);      // (and the planes are there)
#pragma unroll
            for (int c = 0; c < TN; ++c) {
                v4i acc[kThinDigits][4];
#pragma unroll
                for (int l = 0; l < kThinDigits; ++l)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[l][i] = v4i{0, 0, 0, 0};
                // (a step ahead: where the taps' pixels lie, and the weights; behind the last step the last one's)
                int at, next_at;
                ushort4 px4, next_px4;
                v4i fb, next_fb;
                auto ahead = [&](int s) {
                    const int u = 4 * min(s, steps - 1) + g4, t = min(u / NU, taps);
                    next_at = t < taps ? 16 * (u % NU) : 0;
                    next_px4 = *reinterpret_cast<const ushort4 *>(my_table + t * T);
                    next_fb = *reinterpret_cast<const v4i *>(weights + ((u * TN + c) * 16 + (lane & 15)) * 16);
                };
                ahead(0);
                for (int s = 0; s < steps; ++s) {
                    at = next_at; px4 = next_px4; fb = next_fb;
                    ahead(s + 1);
                    const int px[4] = {px4.x, px4.y, px4.z, px4.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int8_t *p = planes + in_plane(px[i], at);
#pragma unroll
                        for (int l = 0; l < kThinDigits; ++l)
                            acc[l][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(*reinterpret_cast<const v4i *>(p + l * plane), fb, acc[l][i], 0, 0, 0);
                    }
                }
                // (two digits at a time as integers)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double run = (double)(256 * acc[5][i][r] + acc[4][i][r]);
                        run = __builtin_fma(run, 65536.0, (double)(256 * acc[3][i][r] + acc[2][i][r]));
                        run = __builtin_fma(run, 65536.0, (double)(256 * acc[1][i][r] + acc[0][i][r]));
                        total[i][c][r] = __builtin_fma(run, unit, total[i][c][r]);
                    }
            }
            largest = rest;
            if (largest > 0u) __syncthreads();      // the planes are written again
        }
        // register r of a tile: row 4 (lane / 16) + r, column lane % 16
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = row0 + wave * 64 + 16 * i + 4 * g4 + r;
                if (m >= rows) continue;
                float *p = a.out + (int64_t)m * C + (lane & 15);
#pragma unroll
                for (int c = 0; c < TN; ++c)
                    if (16 * c + (lane & 15) < C) p[16 * c] = (float)(total[i][c][r] * a.delta);
            }
        return;
    }
    // An infinity or a NaN in the patch: in double as a whole, 16 contraction entries (a unit) a step, so that it shows where it is multiplied.
    __syncthreads();
    each([&](int px, int q, const float4 &v) { *reinterpret_cast<float4 *>(floats + px * kStride + 4 * q) = v; });
    for (int i = tid; i < kStride; i += T) floats[px_max * kStride + i] = 0.0f;
    __syncthreads();
#pragma unroll 1
    for (int c = 0; c < TN; ++c) {
        v4d sum[4] = {v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}};
        const int col = 16 * c + (lane & 15);
#pragma unroll 1
        for (int u = 0; u < units; ++u) {
            const int t = u / NU, n = 16 * (u % NU) + 4 * g4;
            const bool there = n < N;
            const ushort4 px4 = *reinterpret_cast<const ushort4 *>(my_table + t * T);
            const int px[4] = {px4.x, px4.y, px4.z, px4.w};
            const uint32_t w = *reinterpret_cast<const uint32_t *>(weights + (u * 16 * TN + col) * 16 + 4 * g4);
            float4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const float4 *>(floats + (there ? px[i] * kStride + n : px_max * kStride));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double b = (double)((int)(w << (24 - 8 * j)) >> 24);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    sum[i] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(j == 0 ? v[i].x : j == 1 ? v[i].y : j == 2 ? v[i].z : v[i].w), b, sum[i], 0, 0, 0);
            }
        }
        // register r: row lane / 16 + 4 r
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = row0 + wave * 64 + 16 * i + g4 + 4 * r;
                if (m < rows && col < C) a.out[(int64_t)m * C + col] = (float)(sum[i][r] * a.delta);
            }
    }
}

struct ThinPlan { int px_max, patch, lds; };

// LDS of a block, 0 if its patch does not fit.
ThinPlan plan_thin(const ConvDxGrid &grid, int64_t B, int32_t C, int32_t N, int P, int Q)
{
    const int nu = (N + 15) / 16, tn = (C + 15) / 16, taps = grid.Rc * grid.Sc;
    const int64_t px = patch_pixels(patch_grid(&grid, 1), kThinPixels, P, Q, B * P * Q);
    const int64_t digits = kThinDigits * (px + 1) * 16 * nu, floats = (px + 1) * (16 * nu + 4) * 4, patch = digits > floats ? digits : floats;
    const int64_t lds = patch + (int64_t)(taps * nu + 3) / 4 * 4 * 256 * tn + (int64_t)(taps + 1) * kThinPixels * 2 + 2 * kThinWaves * 4;
    return lds > kThinLds ? ThinPlan{} : ThinPlan{(int)px, (int)patch, (int)lds};
}

}  // namespace

// Pixels from which this kernel is the faster one; 0: from no number on.  It makes digits of 16 or 32 output channels and forms 16 or 32 input channels whatever there are, and the digits
// are for all taps.  us of the call, before (in double gathered from memory, on digits or limbs) / so, entries N(0, 1), and in brackets entries times 2^(2 N(0, 1)), of which a range has
// some below 2^-22 of its largest, so that its digits are made twice; 3 x 3 if not said:
//   128 x 32 x 32 x 16 -> 16   24.5 / 12.4 (24.6 / 15.3)     128 x 32 x 32 x 32 -> 16  37.9 / 16.6 (38.2 / 22.6)     32 x 32 x 32 x 16 -> 16  9.3 / 8.4
//   128 x 28 x 28 x 32 -> 32   60.5 / 31.1 (78.8 / 33.9)     100 x 24 x 24 x 28 -> 16, 5 x 5  28 / 19
// and so / before, images of 28 x 28 | 56 x 56 | 96 x 96, 80 K pixels, then 200 K, where * is what the rule leaves to the other paths:
//   16 -> 4    1.0* 1.0* 1.6* (1.3 1.4 1.8)      1.0* 1.1* 1.3* (1.1 1.2 1.6)           32 -> 4    1.1* 1.1* 1.3* (1.5 1.5 1.7)     1.4* 1.4* 2.0* (1.5 1.5 2.2)
//   16 -> 8    0.86 0.81 1.0* (1.03 1.08 1.4)    0.79 0.81 0.98* (0.92 0.97 1.25)       32 -> 8    0.86* 0.87* 1.3* (1.2 1.2 1.4)   0.97* 0.98* 1.5* (1.15 1.2 1.7)
//   16 -> 12   0.73 0.75 0.82* (0.86 0.90 1.2)   0.64 0.66 0.80 (0.77 0.78 1.06)        32 -> 12   0.69 0.79 0.79* (0.96 0.96 1.1)  0.81 0.85 1.1* (0.93 0.93 1.4)
//   16 -> 16   0.55 0.52 0.69 (0.70 0.73 0.89)   0.50 0.51 0.59 (0.62 0.63 0.78)        32 -> 16   0.54 0.54 0.76 (0.77 0.77 0.86)  0.64 0.60 0.81 (0.78 0.83 1.1)
//   16 -> 20   0.77 0.82 1.3* (1.03 1.07 1.7)    0.73 0.79 1.2* (0.95 1.01 1.7)         32 -> 20   0.81 1.1* 1.2* (1.09 1.4 1.5)    0.78 1.1* 1.5* (1.08 1.5 2.0)
//   16 -> 24   0.71 0.73 1.2* (0.92 0.96 1.6)    0.68 0.70 1.1* (0.88 0.92 1.5)         32 -> 24   0.62 0.97* 1.0* (0.97 1.4 1.3)   0.74 1.0* 1.3* (0.96 1.3 1.7)
//   16 -> 28   0.63 0.70 1.2* (0.82 0.86 1.5)    0.60 0.67 0.98* (0.79 0.83 1.3)        32 -> 28   0.74 0.86* 0.92* (0.87 1.3 1.3)  0.67 0.90* 1.2* (0.87 1.2 1.5)
//   16 -> 32   0.54 0.51 0.79* (0.65 0.67 1.2)   0.45 0.46 0.68 (0.61 0.63 0.94)        32 -> 32   0.72 1.2* 1.0* (0.74 1.2 1.25)   0.55 0.89 0.93 (0.65 0.93 0.96)
//   and 5 x 5:
//   16 -> 4    0.89* 1.0* 1.7* (1.1 1.4 2.1)     0.87* 1.0* 1.5* (1.0 1.2 1.8)          32 -> 4    0.89* 1.0* 1.7* (1.3 1.5 2.2)    1.0* 1.1* 1.8* (1.2 1.4 2.4)
//   16 -> 8    0.64 0.69 1.1* (0.81 0.98 1.4)    0.57 0.67 0.91* (0.68 0.82 1.3)        32 -> 8    0.58 0.77 1.1* (0.84 0.95 1.4)   0.65 0.71 1.2* (0.78 0.91 1.7)
//   16 -> 12   0.47 0.52 0.87* (0.61 0.74 1.1)   0.44 0.19 0.78* (0.49 0.23 1.06)       32 -> 12   0.91* 0.42 1.5* (1.1 0.58 1.7)   0.92* 0.37 1.6* (1.1 0.50 2.0)
//   16 -> 16   0.42 0.21 0.61 (0.55 0.28 0.77)   0.43 0.19 0.80 (0.50 0.22 0.96)        32 -> 16   0.89* 0.54 1.3* (1.1 0.54 1.5)   0.96* 0.37 1.5* (1.1 0.46 1.9)
// With fewer pixels (40 K): 16 -> 12 0.97 (1.13), 16 -> 8 1.1 (1.3), 32 -> 16 0.89 (1.28), 32 -> 28 0.84 (1.3), but 16 -> 16 0.7 - 0.9 (0.96), 32 -> 32 0.6 - 0.85 (0.88).  Few taps do not
// pay for the digits (256 x 14 x 14 x 16, 1 x 1  8.3 / 11.6), classes of stride 2 make them four times (64 x 28 x 28 x 16 -> 16  8.3 / 13.7), fewer pixels
// are faster where the waves of a block share a contraction (16 x 32 x 32 x 16 -> 16  6.5), and longer contractions leave a compute unit one block whose
// k-steps hide nothing (60 x 27 x 27 x 32 -> 20, 5 x 5  27 / 48).
static int64_t thin_from(int32_t C, int32_t N, int taps, const ThinPlan &plan)
{
    const int64_t few = 32768, more = 65536, many = 131072;
    // (a patch: two blocks share a compute unit; its range of g is kept in registers, px_max being two more than an aligned run of whole rows reads)
    const bool two = plan.lds <= kThinLds / 2, kept = plan.px_max - 2 <= kThinKept;
    if (taps >= 16) return N < 8 || !(two || (C <= 16 && N == 16)) ? 0 : N < 12 && C > 16 ? more : few;
    if (N < 8 || (C > 16 && N < 12)) return 0;
    if (N > 16) return two ? (N == 32 ? few : more) : N == 32 ? many : 0;
    if (N == 16) return C <= 16 ? few : more;
    return kept ? more : C <= 16 && N == 12 ? many : 0;
}

bool conv_dx_thin_serves(const ConvDxGrid *grids, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N, int32_t R, int32_t S, int32_t P, int32_t Q, int32_t stride)
{
    const int taps = grids->Rc * grids->Sc;
    if (stride != 1 || C > 32 || N > 32 || N % 4 != 0 || taps < 9 || taps * ((N + 15) / 16) > kThinUnits) return false;
    const ThinPlan plan = plan_thin(*grids, B, C, N, P, Q);
    const int64_t from = plan.lds > 0 ? thin_from(C, N, taps, plan) : 0;
    if (from == 0 || (int64_t)B * grids->Hc * grids->Wc < from) return false;
    // (many taps of more than 16 input channels: limbs of a patch of 128 pixels in LDS have them for less, and so have digits made beforehand for wider images; a patch of fewer
    // pixels has a tile of 128 and more channels, most of them for nothing)
    if (taps < 16 || C <= 16 || N < 12 || conv_dx_direct_serves((int64_t)B * H * W, N, C, R, S, stride)) return true;
    const PatchPlan other = plan_patch(grids, 1, B, P, Q, C, 32);
    return other.served && other.wn > 1;
}

int launch_conv_dx_thin(const float *g, const int8_t *w_idx, const ConvDxGrid &grid, int32_t B, int32_t C, int32_t N, int32_t P, int32_t Q, float delta_w,
                        float *d_x_hat, hipStream_t stream)
{
    const ThinPlan plan = plan_thin(grid, B, C, N, P, Q);
    const PatchGrid range = patch_grid(&grid, 1);
    ThinArgs a{};
    a.g = g; a.w = w_idx; a.out = d_x_hat;
    a.N = N; a.C = C; a.P = P; a.Q = Q; a.S = grid.Sc; a.taps = grid.Rc * grid.Sc;
    a.Hc = grid.Hc; a.Wc = grid.Wc; a.pad_h = grid.pad_h; a.pad_w = grid.pad_w;
    a.rows = B * grid.Hc * grid.Wc;
    a.tiles = (a.rows + kThinPixels - 1) / kThinPixels;
    a.share = (a.tiles + 7) / 8;
    a.lo_h = range.lo_h; a.hi_h = range.hi_h; a.lo_w = range.lo_w; a.hi_w = range.hi_w;
    a.by_hw = make_div_by((uint32_t)grid.Hc * (uint32_t)grid.Wc);
    a.by_w = make_div_by((uint32_t)grid.Wc);
    a.pixels = B * P * Q;
    a.px_max = plan.px_max; a.patch_bytes = plan.patch;
    a.delta = (double)delta_w;
#define CDL_THIN(TN, NU)                                                                                                                        \
    do {                                                                                                                                        \
        const hipError_t e_ = hipFuncSetAttribute((const void *)conv_dx_thin_kernel<TN, NU>, hipFuncAttributeMaxDynamicSharedMemorySize, kThinLds); \
        if (e_ != hipSuccess) return hip_failed(e_);                                                                                            \
        CDL_LAUNCH("conv_dx_thin_kernel", stream, (conv_dx_thin_kernel<TN, NU>), dim3((unsigned)(8 * a.share)), dim3(kThinPixels), plan.lds, a);   \
    } while (0)
    if (C <= 16) { if (N <= 16) CDL_THIN(1, 1); else CDL_THIN(1, 2); }
    else { if (N <= 16) CDL_THIN(2, 1); else CDL_THIN(2, 2); }
#undef CDL_THIN
    return check_launch();
}

}  // namespace cdl
