// dL/dQ(a) on limbs for a contraction short enough for the digits of a few rows of g to stay in LDS: d_a_hat[m][k] = delta_b
// sum_n g[m][n] b_idx[n][k], N <= 384, the widths of the layers of a CNN in window-matrix form.
//
// A block writes the digits of 64 rows of g (32 where 64 do not fit) into LDS once and goes through the columns, 128 (256) in a pass; the
// weights' fragments go from L2 straight to registers, a whole pass ahead where N is 64, 128, 192 or 256.  The passes of all row tiles in order are
// dealt out evenly over two blocks a compute unit, so no last round is part empty, and 32 x 64 outputs of one wave are put together and
// stored while the other wave of its SIMD multiplies.
//
// What bounds it: N = 256 the matrix cores at their power-limited rate (without the stores 15 % less time), N = 64 the stores (3.9 TB/s; without
// them 40 % less).  Before, a tile of the general limb kernel had two or three K-tiles between write-outs of 32 x 384 outputs by the one
// wave of a SIMD: nine instructions in double an output, as long as the products, and then loads that waited for the stores.  The whole
// call with max |g| and the transposition, us: 50176 x 256 x 2304 217 -> 150;  200000 x 64 x 576 313 -> 133;  60000 x 192 x 288 101 -> 55;
// 30000 x 384 x 3000 252 -> 190;  9000 x 320 x 1000 60 -> 39;  3136 x 256 x 2304 34 -> 28.
#include "cdl_bwd_plan.h"
#include "cdl_limbs.h"

namespace cdl {

namespace {

constexpr int kRowsThreads = 256;
constexpr int kRowsLds = 80 << 10;           // two blocks share a compute unit
constexpr int kRowsFixed = 64 * 8;           // corrections of the rows
constexpr int kRowsTN = 2;
constexpr int kLimbRowsMaxN = 384;           // 32 rows on six limbs fit

struct RowsArgs {
    const float *g;
    int M, N, K;
    const int8_t *frag;                      // [K / 32][tile_bytes]: 1 KB for 32 contraction entries of 32 columns, [half of the entries][column][16]
    int64_t tile_bytes;
    int nk;                                  // k-steps of 32 entries: even
    const BwdPlan *plan;
    const double *row_corr;                  // [M] or null
    float *out;
};

// rows of g whose digits fit: 64, or 32
constexpr int rows_row_bytes(int nk) { return 32 * nk + 16; }      // (an odd multiple of 16: no bank conflicts)
constexpr bool rows_fit(int rows, int nk, int limbs) { return kRowsFixed + rows * rows_row_bytes(nk) * limbs <= kRowsLds; }

// NB: steps that the weights are asked for ahead (four where the steps of a pass are a multiple of it; fewer where registers are short)
template <int L, int WN, int NB, bool STREAM>
__device__ __forceinline__ void rows_body(const RowsArgs &a, int8_t *lds, float gscale, double out_scale)
{
    constexpr int TN = kRowsTN, WM = 4 / WN, ROWS = 32 * WM, COLS = 32 * TN * WN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const int N = a.N, K = a.K, nk = a.nk, stride = rows_row_bytes(nk), plane = ROWS * stride;
    double *corr = reinterpret_cast<double *>(lds);
    int8_t *planes = lds + kRowsFixed;

    // this block's part of the passes (row tile, COLS columns), in order of the rows; neighbours share an XCD
    const int passes = (K + COLS - 1) / COLS, per_xcd = (int)gridDim.x >> 3, self = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    const int all = (a.M + ROWS - 1) / ROWS * passes, share = all / (int)gridDim.x, more = all - share * (int)gridDim.x;
    int left = __builtin_amdgcn_readfirstlane(share + (self < more ? 1 : 0));
    if (left == 0) return;
    const int begin = self * share + min(self, more);
    int tile = __builtin_amdgcn_readfirstlane(begin / passes), pass = __builtin_amdgcn_readfirstlane(begin - begin / passes * passes);

    // digits: a thread keeps its four entries of a row and goes through the rows
    auto make_digits = [&](int row0) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));      // (formed here, not kept in registers through the passes)
        const int words = 8 * nk, row_step = kRowsThreads / words, own_row = tid / words, own_n = 4 * (tid - own_row * words);
        const int count = min(ROWS, a.M - row0);
        if (a.row_corr && tid < count) corr[tid] = a.row_corr[row0 + tid];
        if (!a.row_corr && tid < ROWS) corr[tid] = 0.0;
        if (own_row >= row_step) return;
        const bool there = own_n < N;
        const float *src = a.g + (int64_t)row0 * N + (there ? own_n : 0);
        constexpr int U = 8;
        const int src_step = row_step * N, src_last = (count - 1) * N, dst_step = row_step * stride, dst_last = (count - 1) * stride;
        int from = own_row * N, to = own_row * stride;
        for (int r = own_row; r < count; r += U * row_step) {      // (behind the last row: the last one again, with what its own thread writes)
            float4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4 *>(src + min(from + u * src_step, src_last));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float g4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                uint32_t w[L];
                limbs_of4<L>(g4, gscale, w);
                int8_t *d = planes + min(to + u * dst_step, dst_last) + own_n;
#pragma unroll
                for (int l = 0; l < L; ++l) *reinterpret_cast<uint32_t *>(d + l * plane) = there ? w[l] : 0u;
            }
            from += U * src_step;
            to += U * dst_step;
        }
    };

    constexpr int NA = L <= 5 ? 2 : 1;
    v4i fa[NA][L], fb[NB][TN];
    v16i acc[L][TN];
    const int last_tile = (K + 31) / 32 - 1;
    const uint32_t lane16 = (uint32_t)lane * 16u;
    struct Columns { const int8_t *p[TN]; };      // where the weights of the next NB steps lie (uniform)
    auto columns = [&](int ps) {
        Columns c;
#pragma unroll
        for (int j = 0; j < TN; ++j) c.p[j] = a.frag + (int64_t)min((ps * WN + wn) * TN + j, last_tile) * a.tile_bytes;
        return c;
    };
    auto load_b = [&](const Columns &c, int u) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int8_t __attribute__((address_space(1))) *p = (const int8_t __attribute__((address_space(1))) *)c.p[j] + u / 4 * 4096;
            asm("" : "+s"(p));      // (a base in scalar registers and the lane's offset: no address a lane)
            fb[u][j] = *(const v4i __attribute__((address_space(1))) *)(p + (uint32_t)(u % 4 * 1024 + lane16));
        }
    };
    const int8_t *a_rows = planes + (wm * 32 + (lane & 31)) * stride + (lane >> 5) * 16;
    int a_n = 0;
    auto load_a = [&](int buf) {
#pragma unroll
        for (int l = 0; l < L; ++l) fa[buf][l] = *reinterpret_cast<const v4i *>(a_rows + a_n + l * plane);
        a_n = a_n + 32 == 32 * nk ? 0 : a_n + 32;
    };
    auto steps = [&](auto first_c, const Columns &next) {
        constexpr bool FIRST = decltype(first_c)::value;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if (NA == 2) load_a((u + 1) & 1);
            else load_a(0);
            const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int l = 0; l < L; ++l)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[l][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[NA == 2 ? u & 1 : 0][l], fb[u][j], FIRST && u == 0 ? zero : acc[l][j], 0, 0, 0);
            load_b(next, u);
#pragma unroll
            for (int i = 0; i < L * TN; ++i) {      // behind each matrix instruction a part of the rest
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x006, 5, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    Columns at = columns(pass);
    auto following = [&](int it) {      // of the steps NB behind `it`
        if (it + NB < nk) {
#pragma unroll
            for (int j = 0; j < TN; ++j) at.p[j] += NB * 1024;
        } else {
            at = columns(pass + 1 == passes ? 0 : pass + 1);
        }
    };
    auto all_steps = [&]() {
        following(0);
        steps(std::true_type{}, at);
        for (int it = NB; it < nk; it += NB) {
            following(it);
            steps(std::false_type{}, at);
        }
    };

    // 32 x 64 outputs of the wave.  Two limbs are put together as integers: |acc| <= 384 128 128, and 257 times that is under 2^31;
    // the rest in double (at 2^-53 relative).
    auto write = [&](auto full_c, int row0, int col0) {
        constexpr bool FULL = decltype(full_c)::value;
        int elane = lane;
        asm volatile("" : "+v"(elane));      // (addresses formed here, not kept in registers through the loop)
        const int half4 = 4 * (elane >> 5), ecol = elane & 31;
        typedef float __attribute__((address_space(1))) *out_t;
        const out_t base = (out_t)a.out + (int64_t)row0 * K + col0;
        const uint32_t off = 4u * (uint32_t)(half4 * K + ecol);
#pragma unroll
        for (int rr = 0; rr < 16; ++rr) {
            const int dr = 8 * (rr >> 2) + (rr & 3);
            out_t row = base + (int64_t)dr * K;
            asm("" : "+s"(row));
            const out_t p = (out_t)((char __attribute__((address_space(1))) *)row + off);
            const double rc = FULL ? 0.0 : corr[wm * 32 + dr + half4];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                double run = 0.0;
#pragma unroll
                for (int l = (L - 1) / 2; l >= 0; --l) {
                    const int two = 2 * l + 1 < L ? acc[2 * l + 1 < L ? 2 * l + 1 : 0][j][rr] * 256 + acc[2 * l][j][rr] : acc[2 * l][j][rr];
                    run = l == (L - 1) / 2 ? (double)two : __builtin_fma(run, 65536.0, (double)two);
                }
                if (FULL && STREAM) __builtin_nontemporal_store((float)(run * out_scale), p + 32 * j);
                else if (FULL) p[32 * j] = (float)(run * out_scale);
                else if (row0 + dr + half4 < a.M && col0 + ecol + 32 * j < K) p[32 * j] = (float)__builtin_fma(run, out_scale, rc);
            }
        }
    };

#pragma unroll
    for (int u = 0; u < NB; ++u) load_b(at, u);
    while (true) {
        const int row0 = tile * ROWS + wm * 32;
        make_digits(tile * ROWS);
        __syncthreads();
        a_n = 0;
        if (NA == 2) load_a(0);
        const int last = min(passes, pass + left);
        left -= last - pass;
        // passes that this wave writes without a test
        const int full = row0 + 32 <= a.M && !a.row_corr ? min(last, (K - wn * 32 * TN) / COLS + ((K - wn * 32 * TN) % COLS >= 32 * TN ? 1 : 0)) : pass;
        // A wave's loads and stores are counted together, in order: weights wait for every store before them, and a store takes
        // microseconds.  With the next pass's weights under way before the stores, the second loop waits only for what is older than the
        // stores of the pass before - as long as every way to it has the same stores behind it, hence the first pass apart.
        if (pass < full) {
            all_steps();
            write(std::true_type{}, row0, pass * COLS + wn * 32 * TN);
            for (++pass; pass < full; ++pass) {
                all_steps();
                write(std::true_type{}, row0, pass * COLS + wn * 32 * TN);
            }
        }
        for (; pass < last; ++pass) {
            all_steps();
            write(std::false_type{}, row0, pass * COLS + wn * 32 * TN);
        }
        if (left == 0) break;
        ++tile;
        pass = 0;
        __syncthreads();
    }
}

template <int NB, bool STREAM>
__global__ __launch_bounds__(kRowsThreads, 2)
void limb_rows_kernel(RowsArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t rows_lds[];
    const int limbs = a.plan->limbs_da;
    const float gscale = a.plan->gscale_da;
    const double out_scale = a.plan->out_scale_da;
#define CDL_ROWS(L, NB)                                                                          \
    if (rows_fit(64, a.nk, L)) rows_body<L, 2, NB, STREAM>(a, rows_lds, gscale, out_scale);              \
    else rows_body<L, 4, NB, STREAM>(a, rows_lds, gscale, out_scale);                                    \
    break;
    switch (limbs) {
        case 3: CDL_ROWS(3, NB)
        case 4: CDL_ROWS(4, NB)
        case 5: CDL_ROWS(5, 2)
        default: CDL_ROWS(6, 1)
    }
#undef CDL_ROWS
}

}  // namespace

bool limb_rows_serves(int64_t M, int32_t N, int32_t K)
{
    return N % 4 == 0 && N <= kLimbRowsMaxN && (M + 31) / 32 * ((K + 127) / 128) <= 2147483647LL;
}

int launch_limb_rows(const float *g, const int8_t *frag, int64_t tile_bytes, int32_t M, int32_t N, int32_t K, const BwdPlan *plan, const double *row_corr, float *out, hipStream_t stream)
{
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0)
        n_cu = 256;
    RowsArgs a{};
    a.g = g; a.M = M; a.N = N; a.K = K;
    a.frag = frag; a.tile_bytes = tile_bytes;
    a.nk = (N + 63) / 64 * 2;
    a.plan = plan; a.row_corr = row_corr; a.out = out;
    const bool stream_out = stream_output((int64_t)M * K, K, out);      // (50176 x 256 x 2304 160 -> 150 us)
#define CDL_PICK(NB) (stream_out ? limb_rows_kernel<NB, true> : limb_rows_kernel<NB, false>)
    const auto kernel = a.nk % 8 == 0 ? CDL_PICK(8) : a.nk % 6 == 0 ? CDL_PICK(6) : a.nk % 4 == 0 ? CDL_PICK(4) : CDL_PICK(2);
#undef CDL_PICK
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLds);
    if (e != hipSuccess) return hip_failed(e);
    CDL_LAUNCH("limb_rows_kernel(d_a_hat)", stream, kernel, dim3((unsigned)(2 * n_cu / 8 * 8)), dim3(kRowsThreads), kRowsLds, a);
    return check_launch();
}

}  // namespace cdl
