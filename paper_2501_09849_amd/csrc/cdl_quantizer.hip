// Probabilistic quantizer of CDL on gfx950: forward (hard index, soft value, marginal PMF,
// entropy) and analytic backward (Lemma 1) as single-pass streaming kernels.
//
// The conditional PMF of one entry theta over the levels i*delta is
//     P_i = softmax_i(-alpha (theta - i delta)^2)                       (eq. CPMF, Sec. III-A).
// Let c be a level next to theta (the nearest one, clamped to the set), u = theta - c*delta and
// kappa = alpha*delta^2.  Relative to level c the weight of level c+j is
//     w_j = exp(alpha*delta * j * (2u - j*delta)),          w_0 = 1,
// which is exp(-kappa j^2 + 2 alpha delta u j) written so that nothing large cancels.  For
// |u| <= delta/2 it is at most exp(-kappa |j| (|j|-1)), so only a band of W levels on each side
// of c carries weight above fp32 resolution; W depends on kappa alone and is fixed per launch.
// All moments are taken of the offset j, which keeps fp32 free of the cancellation that raw
// powers of the index would suffer:
//     Q_d = delta (c + mu),  Var = delta^2 var_j,  third central moment = delta^3 c3_j.
// Lemma 1 in these terms (Skew_u = c3 + 2 E Var):
//     dQd/dtheta = 2 kappa var_j
//     dQd/ddelta = (c + mu) + 2 kappa ((r - c - 2 mu) var_j - c3_j),   r = u/delta
//     dQd/dalpha = delta^3 (2 (r - mu) var_j - c3_j)
//
// These kernels are bound by plain fp32 ALU work as much as by HBM (one wave instruction costs
// four cycles, exp and rcp sixteen), so the band is evaluated with as few instructions as the
// accuracy allows:
//   W = 1 (kappa > 10.9): two exponentials whose arguments are formed without rounding error;
//   W = 2 (3.8 < kappa <= 10.9): one exponential t = exp(2 alpha delta u); the five weights are
//          t^(j) exp(-kappa j^2), all multiplied by t^2 so that they are a polynomial in t;
//   W = 3, 4: one exponential per level;  larger W (soft regime): a table (cdl_soft.hip), kernels on a common centre or a
//          loop over the band.
#include "cdl_internal.h"
#include "cdl_one_trip.h"
#include "cdl_finish.h"
#include "cdl_marginal.h"
#include "cdl_quantizer_math.h"
#include "cdl_soft.h"

#include <math.h>

#include <mutex>
#include <type_traits>

namespace cdl {

namespace {

constexpr int one_trip_threads(int u) { return u > 1 ? kOneTripThreads : kQuantThreads; }
constexpr int64_t kOneTripEntries = 4ll * kMaxQuantBlocks * kQuantThreads;

// f(std::true_type) or f(std::false_type): a switch of the launch taken once, so that no load waits at a branch for another
template <typename F>
__device__ __forceinline__ void with_constant(bool yes, F f)
{
    if (yes) f(std::true_type{});
    else f(std::false_type{});
}

// group(v, N, RAGGED): N vectors of four entries v, v + T, .. of the first `vectors`, of which `whole` have four.  U > 1: U vectors a thread in the block's one trip (without a branch
// around any: it would take the loads with it, behind the stores), in the last block one at a time.  U == 1: a loop over the tensor (of the first `blocks` blocks, where that is not 0).
// RAGGED: the last vector may have fewer entries, which puts a branch around the loads of a loop.  Whole tensors go without where all blocks are short (quantizer gradient, 0.5 M entries of 31 levels, two
// on each side 6.1 us, with it 6.5; 2.1 M, four 11.5 / 12.1), but the loops of larger ones are faster with it (2.1 M, four on each side without scalars 9.4 / 8.8; 24 M, gradient of the entropy added 57 / 53).
template <int T, int U, typename F>
__device__ __forceinline__ void one_trip_or_loop(int64_t whole, int64_t vectors, F group, int blocks = 0)
{
    const int64_t v0 = (int64_t)blockIdx.x * T * U;
    if (U > 1 && v0 + T * U <= whole) group(v0 + threadIdx.x, std::integral_constant<int, U>{}, std::false_type{});
    else {
        const int64_t end = U > 1 ? (v0 + T * U < vectors ? v0 + T * U : vectors) : vectors;
        auto loop = [&](auto ragged) {
#pragma unroll 1
            for (int64_t v = v0 + threadIdx.x; v < end; v += U > 1 ? T : (int64_t)(blocks ? blocks : gridDim.x) * T) group(v, std::integral_constant<int, 1>{}, ragged);
        };
        if (U > 1 || vectors > whole || whole > (int64_t)kMaxQuantBlocks * T) loop(std::true_type{});
        else loop(std::false_type{});
    }
}

// The first cnt of four entries, zeros behind them
__device__ __forceinline__ float4 load_first(const float *p, int cnt)
{
    return make_float4(p[0], cnt > 1 ? p[1] : 0.0f, cnt > 2 ? p[2] : 0.0f, 0.0f);
}

constexpr int kPad = 4;   // spare histogram bins on each side, so that band offsets never leave the array

// Fixed-point histogram: a block of kMargThreads threads (8 waves) makes at most kMaxHistTrips trips of
// its loop, each lane adds 4 entries per trip, and the 2 * 8 lanes with the same lane % 32 share one
// copy of a bin: at most 16 * 4 * 16 = 2^10 adds of at most 2^s each reach one cell, so s = 21 keeps
// every cell at or below 2^31.
constexpr int kMaxHistTrips = 16;
constexpr int kMargThreads = 512;   // threads of a block that builds a histogram

// The rows of a large grid.  Grid: (ceil(levels / 8), chunks), about 64 blocks in all: a block adds its chunk of the
// rows for eight levels (32 rows at a time, 64 contiguous bytes per row); the last block adds the chunks.  (A block for
// all levels of every 32nd row instead: 5.4 us for 1024 rows of 31 levels, but 9.8 for 255, where the last block then
// polls 8 K records.)
constexpr int kFinChunks = 16;
constexpr int kFinThreads = 256, kFinGroups = kFinThreads / 8;

__global__ __launch_bounds__(kFinThreads)
void marginal_finalize_kernel(const unsigned long long *__restrict__ rows, int n_rows, int n_levels, MargFinish fin)
{
    __shared__ unsigned long long red[kFinGroups][8];
    const int b8 = threadIdx.x & 7, grp = threadIdx.x >> 3;
    const int level = blockIdx.x * 8 + b8;
    const int rows_per = (n_rows + (int)gridDim.y - 1) / (int)gridDim.y;
    const int r0 = blockIdx.y * rows_per, r1 = min(n_rows, r0 + rows_per);
    unsigned long long s = 0ull;
    if (level < n_levels) {
#pragma unroll 8
        for (int row = r0 + grp; row < r1; row += kFinGroups) s += rows[(size_t)row * n_levels + level];
    }
    red[grp][b8] = s;
    __syncthreads();
    if (threadIdx.x < 8 && level < n_levels) {
        unsigned long long tot = 0ull;
        for (int q = 0; q < kFinGroups; ++q) tot += red[q][threadIdx.x];
        marginal_publish(tot, (size_t)blockIdx.y * n_levels + level, fin);
    }
    if (blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1)
        marginal_collect<kFinThreads, 4>(0ull, (int)gridDim.y, n_levels, fin);
}

// ------------------------------------------------------------------------------------------
// Forward kernel.  One thread handles four consecutive entries per trip of a grid-stride loop
// (one 16-byte load, one 16-byte store of soft values, one 4-byte store of indices).
//
// MARG: the CPMF of every entry is added into a histogram in LDS, in fixed point: a probability
// p is added as the integer floor(p * 2^s + 1/2), so that a level's share is off by half a unit of 2^-s and the rounding of p at most, also where
// all entries are equal.  (LDS integer atomics run at ~10 lane updates
// per clock per CU on this chip, fp32 LDS atomics at a thirtieth of that; integer sums are also
// independent of the order of the adds, so the result is reproducible.)  The block keeps 32 copies of
// the histogram, bin-major and copy-minor, and lane l uses copy l mod 32: the copy is the LDS bank, so
// the lanes of one instruction never meet in a bank except lane l with lane l + 32 (measured against
// 4 or 16 copies per wave, where different bins fall into the same bank: -8 % on the whole forward
// kernel at 255 levels, -22 % on the pass that only builds the histogram).  s comes from
// kHistScaleBits: with at most kMaxHistTrips trips of the loop a cell never exceeds 2^31.
// kPad spare bins on each side take the zero weights of levels that do not exist.  At the end
// the block adds the copies into 64-bit sums, and marginal_end adds these over all blocks.
// (Levels c + j and c - j as the halves of one 64-bit cell of level c, that of c from the number of entries: W atomics an entry instead of 2 W + 1, but more
// cells to clear and to add up, and a share of the nearest level that takes the roundings of all others.  us with indices, bins / pairs:
// 25.6 M entries of 31 levels, W = 2 41.0 / 40.4, of 63 41.8 / 44.1, W = 3 of 47 60.3 / 63.1; 2.5 M of 63 12.7 / 15.5, 1.5 M of 72 11.1 / 18.1.)
// ------------------------------------------------------------------------------------------
constexpr int kHistCopies = 32;

// Quantizes four entries: soft values, level indices, and (MARG) their CPMFs into the histogram.
// my_hist: this lane's copy of the bin of level 0, whether it is in the set or not
template <int W, bool IDX, bool MARG>
__device__ __forceinline__ void forward4(const float (&th)[4], int cnt, const QConst &k, unsigned int *my_hist,
                                         float (&sv)[4], int (&ci)[4])
{
    constexpr int R = kHistCopies;
    constexpr float kScale = (float)(1u << kHistScaleBits);
    float cf[4];
    if (W > 0) anchor_levels<IDX>(th, k, cf);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (W > 0) {
            Band<W> b;
            band_weights<W, 1>(th[e], cf[e], k, b);
            const float inv = fast_rcp(b.Z);
            sv[e] = fmaf(b.S1 * inv, k.delta, b.cf * k.delta);
            ci[e] = (int)b.cf;
            if (MARG && e < cnt) {
                unsigned int *h = my_hist + (ci[e] + kPad - W) * R;   // bin of level c-W
                const float invs = inv * kScale;
                atomicAdd(h + W * R, (unsigned int)fmaf(b.ctr, invs, 0.5f));
#pragma unroll
                for (int j = 1; j <= W; ++j) {
                    atomicAdd(h + (W + j) * R, (unsigned int)fmaf(b.up[j - 1], invs, 0.5f));
                    atomicAdd(h + (W - j) * R, (unsigned int)fmaf(b.dn[j - 1], invs, 0.5f));
                }
                // (the pass that only builds the histogram: the atomics of an entry stay in front of the next one's arithmetic, else those of four
                // go out in one burst.  us without / so: 25.6 M entries of 31 levels 39.1 / 36.9, 47 levels, three on each side 53.2 / 51.9)
                if (!IDX && W <= 3) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            GenericSums g;
            generic_sums<IDX>(th[e], k, g);
            const float inv = fast_rcp(g.Z);
            sv[e] = fmaf(g.S1 * inv, k.delta, g.cf * k.delta);
            ci[e] = (int)g.cf;
            if (MARG && e < cnt) {
                unsigned int *h = my_hist + (ci[e] + kPad) * R;
                const float two_u = 2.0f * g.u, invs = inv * kScale;
                for (int j = g.jlo; j <= g.jhi; ++j)
                    atomicAdd(h + j * R, (unsigned int)fmaf(generic_weight(j, two_u, k), invs, 0.5f));
            }
        }
    }
}

// U: vectors of four entries a thread takes per trip.  U > 1: with MARG the loads of a trip (hist_ahead) are issued before the trip before it is
// computed and stored, without MARG there is one trip.
template <int W, bool IDX, bool SOFT, bool MARG, int FORM, int U>
__global__ __launch_bounds__(MARG ? kMargThreads : one_trip_threads(U))
void quantize_fwd_kernel(const float *__restrict__ theta, int64_t n, QConst k,
                         int8_t *__restrict__ idx, float *__restrict__ soft,
                         MargFinish fin)
{
    extern __shared__ __attribute__((aligned(16))) unsigned int lds_hist[];  // [n_levels + 2 kPad][copies] when MARG
    constexpr int R = kHistCopies;
    constexpr int T = MARG ? kMargThreads : one_trip_threads(U);
    unsigned int *my_hist = lds_hist + (int)(threadIdx.x & (R - 1)) - k.lo * R;
    constexpr bool SLICES = MARG && FORM == kMargSlices;
    if constexpr (SLICES) {
        if (fin.roles.collects((int)blockIdx.x)) {
            rows_collect<T, 8>(k.n_levels, fin);
            return;
        }
    }
    if (MARG) {
        const int cells = (k.n_levels + 2 * kPad) * R;
        for (int i = 4 * threadIdx.x; i < cells; i += 4 * T) *reinterpret_cast<uint4 *>(lds_hist + i) = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    }

    const int64_t n4 = n >> 2;
    float sv[4];
    int ci[4];
    with_constant(k.stream != 0, [&](auto streams) {
        auto vec = [&](const float4 &t, int64_t w) {
            const float th[4] = {t.x, t.y, t.z, t.w};
            forward4<W, IDX, MARG>(th, 4, k, my_hist, sv, ci);
            if (SOFT) store_stream4(soft + 4 * w, sv[0], sv[1], sv[2], sv[3], streams.value);
            if (IDX) {
                const uint32_t packed = pack_indices(ci[0], ci[1], ci[2], ci[3], k.idx_off);
                reinterpret_cast<uint32_t *>(idx)[w] = packed;   // (ordinary store: the products read the indices next)
            }
        };
        if (MARG && U > 1) {
            float4 t[U];
            auto load = [&](int64_t v) {
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] = load_stream4(theta + 4 * (v + u * T < n4 ? v + u * T : 0), streams.value);
            };
            const int64_t stride = (int64_t)gridDim.x * T * U;
            int64_t v = (int64_t)blockIdx.x * T * U + threadIdx.x;
            load(v);
            for (; v < n4; v += stride) {
                float4 now[U];
#pragma unroll
                for (int u = 0; u < U; ++u) now[u] = t[u];
                load(v + stride);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u == 0 || v + u * T < n4) vec(now[u], v + u * T);
            }
        } else {
            auto group = [&](int64_t v, auto count, auto ragged) {
                constexpr int N = decltype(count)::value;
                float4 t[N];
#pragma unroll
                for (int u = 0; u < N; ++u) t[u] = load_stream4(theta + 4 * (v + u * T), streams.value);
#pragma unroll
                for (int u = 0; u < N; ++u) vec(t[u], v + u * T);
            };
            one_trip_or_loop<T, U>(n4, n4, group, SLICES ? fin.roles.workers : 0);      // (the tail is below)
        }
    });
    // ragged tail: the last 1..3 entries, one thread of the last block that has entries
    const int cnt = (int)(n - (n4 << 2));
    if (cnt > 0 && blockIdx.x == (SLICES ? (unsigned int)fin.roles.workers : gridDim.x) - 1 && threadIdx.x == 0) {
        float th[4];
        for (int e = 0; e < 4; ++e) th[e] = (e < cnt) ? theta[(n4 << 2) + e] : 0.0f;
        forward4<W, IDX, MARG>(th, cnt, k, my_hist, sv, ci);
        for (int e = 0; e < cnt; ++e) {
            if (SOFT) soft[(n4 << 2) + e] = sv[e];
            if (IDX) idx[(n4 << 2) + e] = (int8_t)(ci[e] - k.idx_off);
        }
    }

    if (MARG) {
        __syncthreads();
        unsigned long long own = 0ull;
        if ((int)threadIdx.x < k.n_levels) {
            const unsigned int *row = lds_hist + ((int)threadIdx.x + kPad) * R;
#pragma unroll
            for (int r = 0; r < R; ++r) own += row[(r + (int)threadIdx.x) & (R - 1)];   // rotated start: no bank conflicts
        }
        marginal_end<T, FORM>(own, k.n_levels, fin);
    }
}

// ------------------------------------------------------------------------------------------
// Backward kernel: recomputes the band, forms the central moments and multiplies by the
// upstream gradient.  The two scalar sums are accumulated per thread in double and added up over
// threads and blocks in a fixed order.
// ------------------------------------------------------------------------------------------
template <int W, bool DTHETA, bool SCALARS, int U>
__global__ __launch_bounds__(one_trip_threads(U))
void quantize_bwd_kernel(const float *__restrict__ theta, const float *g, int64_t n, QConst k,
                         float *dtheta /* may be g */, ScalarFinish fin)
{
    constexpr int T = one_trip_threads(U);
    double acc_d = 0.0, acc_a = 0.0;
    const int64_t n4 = n >> 2;
    auto four = [&](const float (&th)[4], const float (&ge)[4], float (&dv)[4]) {
        float sum_d = 0.0f, sum_a = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float d_th, t_d, t_a;
            quantizer_bwd_terms<W, SCALARS>(th[e], k, d_th, t_d, t_a);
            dv[e] = ge[e] * d_th;
            if (SCALARS) {
                sum_d = fmaf(ge[e], t_d, sum_d);
                sum_a = fmaf(ge[e], t_a, sum_a);
            }
        }
        if (SCALARS) { acc_d += (double)sum_d; acc_a += (double)sum_a; }
    };
    with_constant(k.stream != 0, [&](auto streams) {
        // vectors v, v + T, ..  (a last one of 1 to 3 entries is a thread's vector like all others: by itself behind them it is one more chain at the end of the launch, 1003 entries of
        // 128 levels in the soft regime 18.3 us, so 10.9)
        auto group = [&](int64_t v, auto count, auto ragged) {
            constexpr int N = decltype(count)::value;
            const int cnt = !ragged.value || v < n4 ? 4 : (int)(n - (n4 << 2));
            float4 t[N], q[N];
            if (!ragged.value || cnt == 4) {
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    t[u] = load_stream4(theta + 4 * (v + u * T), streams.value);
                    q[u] = load_stream4(g + 4 * (v + u * T), streams.value);
                }
            } else {
                t[0] = load_first(theta + 4 * v, cnt);
                q[0] = load_first(g + 4 * v, cnt);
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float th[4] = {t[u].x, t[u].y, t[u].z, t[u].w}, ge[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
                float dv[4];
                four(th, ge, dv);
                if (DTHETA) {
                    if (!ragged.value || cnt == 4) store_stream4(dtheta + 4 * (v + u * T), dv[0], dv[1], dv[2], dv[3], streams.value);
                    else for (int e = 0; e < cnt; ++e) dtheta[4 * v + e] = dv[e];
                }
            }
        };
        one_trip_or_loop<T, U>(n4, (n + 3) >> 2, group);
    });
    if (SCALARS) scalar_finish<T>(acc_d, acc_a, fin);
}

// ------------------------------------------------------------------------------------------
// Soft regime on a small level set (at most 33 levels, kappa small enough that every level carries weight:
// the paper starts training at alpha = 500, Sec. V-B, where kappa is 0.01 - 0.5 for 2 - 5 bit weights).
// Here the band is the whole set for every entry, so nothing is gained by anchoring at the nearest level, and
// a common centre makes the loop over the levels the same for every lane.  With c0 the centre of the set
// (a level for an odd number of levels, a midpoint for an even one), r = theta / delta - c0 and offsets
// o_j = j - eps (eps = 0 or 1/2), the weight of the level at c0 +- o_j is
//     exp(-kappa o_j^2) T^(+-o_j),      T = exp(2 kappa r),
// a launch constant times a power of one exponential per entry.  The even and odd parts
//     s_j = T^o_j + T^-o_j,   d_j = T^o_j - T^-o_j
// obey s_(j+1) = (T + 1/T) s_j - s_(j-1) (the same for d): one fused multiply-add each per pair of levels,
// and the power sums take one more each (Z += E_j s_j, S1 += o_j E_j d_j, S2 += o_j^2 E_j s_j, S3 += o_j^3 E_j d_j)
// against an exponential and five instructions per single level in the generic loop.
// Everything is in double: an error of T is raised to the power o_j and hits all levels alike (it acts like a
// shift of theta by var_j * eps * delta, 5e-6 delta for fp32 with 31 live levels - too much next to the
// tolerance), moments about a centre that may be 16 levels away from the mean would cancel in fp32, and with
// packed fp32 arithmetic switched off a double fused multiply-add issues at the same rate as a single one.
// theta far outside the set: r is held at +-r_safe = JH + 15 / kappa, beyond which the CPMF is one level to
// 1e-13, so that T^JH stays finite.  The host uses these kernels when kappa * JH^2 <= 72.
// Marginal PMF: sum_e P = sum_e (E_j / 2Z_e)(s_j +- d_j): every thread keeps sum_e s_j / Z_e and sum_e d_j / Z_e
// for all j in registers (the loop is unrolled, JH is a template parameter, level sets in between are padded
// with E_j = 0), the block adds them up in a fixed order through LDS and writes one fixed-point row like the
// histogram kernels do - no atomics at all, where the generic kernel issues one per entry and level.
// ------------------------------------------------------------------------------------------
constexpr int kUniMaxJH = 16;
constexpr int kUniThreads = 256;

struct UniConst {
    double delta, c0;          // step; centre of the level set in units of the step
    double inv_delta;
    double x_per_r;            // log2(e) * kappa: T^(1/2) = exp2(x_per_r * r)
    double two_kappa;
    double r_safe;
    double e[kUniMaxJH][4];    // E_j, o_j E_j, o_j^2 E_j, o_j^3 E_j (zero for offsets beyond the set)
    int odd;                   // number of levels is odd: offsets are integers and the centre is a level
    int pairs;                 // pairs of levels: n_levels / 2
};

template <int JH>
struct UniSums {
    double Z, S1, S2, S3, r;
};

// 1 / a for a positive normal double well inside the exponent range: the hardware's reciprocal estimate and two
// Newton steps (each squares the relative error: full precision), without the scaling and fix-up code that a
// general division carries for subnormal and infinite operands - a fifth of its instructions.
__device__ __forceinline__ double uni_rcp(double a)
{
    double y = __builtin_amdgcn_rcp(a);
    y = fma(fma(-a, y, 1.0), y, y);
    y = fma(fma(-a, y, 1.0), y, y);
    return y;
}

// 2^x for |x| < 1000: x = n + f with |f| <= 1/2, e^(f ln 2) by its Taylor polynomial of degree 12 (remainder
// (ln 2 / 2)^13 / 13! = 1.7e-16) in Horner form, scaled by 2^n.  No special cases: the callers clamp x.
__device__ __forceinline__ double uni_exp2(double x)
{
    const double n = rint(x);
    const double t = (x - n) * 0.6931471805599453094;
    double p = 1.0 / 479001600.0;
    p = fma(p, t, 1.0 / 39916800.0);
    p = fma(p, t, 1.0 / 3628800.0);
    p = fma(p, t, 1.0 / 362880.0);
    p = fma(p, t, 1.0 / 40320.0);
    p = fma(p, t, 1.0 / 5040.0);
    p = fma(p, t, 1.0 / 720.0);
    p = fma(p, t, 1.0 / 120.0);
    p = fma(p, t, 1.0 / 24.0);
    p = fma(p, t, 1.0 / 6.0);
    p = fma(p, t, 0.5);
    p = fma(p, t, 1.0);
    p = fma(p, t, 1.0);
    return ldexp(p, (int)n);
}

// NMOM: how many of S1, S2, S3 are needed.  HIST: also adds s_j / Z and d_j / Z (and 1 / Z for the centre) to acc.
template <int JH, int NMOM, bool HIST>
__device__ __forceinline__ void uni_sums(float th, const UniConst &u, UniSums<JH> &o, double (&acc_s)[JH], double (&acc_d)[JH], double &acc_0)
{
    double r = fma((double)th, u.inv_delta, -u.c0);
    r = fmin(fmax(r, -u.r_safe), u.r_safe);
    o.r = r;
    const double half = uni_exp2(u.x_per_r * r);      // T^(1/2)
    const double half_inv = uni_rcp(half);
    const double T = half * half, Tinv = half_inv * half_inv;
    const double c = T + Tinv;
    const double a = u.odd ? T : half, b = u.odd ? Tinv : half_inv;
    const double s1 = a + b, d1 = a - b;
    double s_prev = u.odd ? 2.0 : s1, d_prev = u.odd ? 0.0 : -d1;
    double s = s1, d = d1;
    double Z = u.odd ? 1.0 : 0.0, S1 = 0.0, S2 = 0.0, S3 = 0.0;
#pragma unroll
    for (int j = 0; j < JH; ++j) {
        Z = fma(u.e[j][0], s, Z);
        S1 = fma(u.e[j][1], d, S1);
        if (NMOM >= 2) S2 = fma(u.e[j][2], s, S2);
        if (NMOM >= 3) S3 = fma(u.e[j][3], d, S3);
        const double s_next = fma(c, s, -s_prev), d_next = fma(c, d, -d_prev);
        s_prev = s; d_prev = d; s = s_next; d = d_next;
    }
    o.Z = Z; o.S1 = S1; o.S2 = S2; o.S3 = S3;
    if (HIST) {
        const double inv = uni_rcp(Z);
        acc_0 += inv;
        s_prev = u.odd ? 2.0 : s1; d_prev = u.odd ? 0.0 : -d1;
        s = s1 * inv; d = d1 * inv;
        s_prev *= inv; d_prev *= inv;
#pragma unroll
        for (int j = 0; j < JH; ++j) {
            acc_s[j] += s;
            acc_d[j] += d;
            const double s_next = fma(c, s, -s_prev), d_next = fma(c, d, -d_prev);
            s_prev = s; d_prev = d; s = s_next; d = d_next;
        }
    }
}

// The same sums for the backward pass, which needs all four.  Four launch constants per offset would be 128
// scalar registers at JH = 16, more than a wave has (the compiler then parks them in vector registers and
// fetches each with two extra instructions: measured twice the time).  So only E_j comes from the table and the
// powers of o_j = j - eps are literals, which costs two more multiplications per pair of levels; ODD (the
// number of levels is odd, eps = 0) is a template parameter for that reason.
template <int JH, int NMOM, bool ODD>
__device__ __forceinline__ void uni_sums_literal(float th, const UniConst &u, UniSums<JH> &o)
{
    double r = fma((double)th, u.inv_delta, -u.c0);
    r = fmin(fmax(r, -u.r_safe), u.r_safe);
    o.r = r;
    const double half = uni_exp2(u.x_per_r * r);      // T^(1/2)
    const double half_inv = uni_rcp(half);
    const double T = half * half, Tinv = half_inv * half_inv;
    const double c = T + Tinv;
    const double a = ODD ? T : half, b = ODD ? Tinv : half_inv;
    const double s1 = a + b, d1 = a - b;
    double s_prev = ODD ? 2.0 : s1, d_prev = ODD ? 0.0 : -d1;
    double s = s1, d = d1;
    double Z = ODD ? 1.0 : 0.0, S1 = 0.0, S2 = 0.0, S3 = 0.0;
#pragma unroll
    for (int j = 0; j < JH; ++j) {
        constexpr double kEps = ODD ? 0.0 : 0.5;
        const double off = (double)(j + 1) - kEps;
        const double es = u.e[j][0] * s, ed = u.e[j][0] * d;
        Z += es;
        S1 = fma(off, ed, S1);
        if (NMOM >= 2) S2 = fma(off * off, es, S2);
        if (NMOM >= 3) S3 = fma(off * off * off, ed, S3);
        const double s_next = fma(c, s, -s_prev), d_next = fma(c, d, -d_prev);
        s_prev = s; d_prev = d; s = s_next; d = d_next;
    }
    o.Z = Z; o.S1 = S1; o.S2 = S2; o.S3 = S3;
}

template <int JH, bool IDX, bool SOFT, bool MARG, int FORM>
__global__ __launch_bounds__(kUniThreads)
void quantize_fwd_uniform_kernel(const float *__restrict__ theta, int64_t n, QConst k, UniConst u,
                                 int8_t *__restrict__ idx, float *__restrict__ soft,
                                 MargFinish fin)
{
    extern __shared__ double uni_lds[];   // [kUniThreads][2 JH + 1] when MARG
    double acc_s[JH], acc_d[JH], acc_0 = 0.0;
#pragma unroll
    for (int j = 0; j < JH; ++j) { acc_s[j] = 0.0; acc_d[j] = 0.0; }

    const int64_t n4 = n >> 2;
    const int64_t stride = (int64_t)gridDim.x * kUniThreads;
    const int tail = (int)(n - (n4 << 2));
    for (int64_t v = (int64_t)blockIdx.x * kUniThreads + threadIdx.x; v < n4 + (tail ? 1 : 0); v += stride) {
        float th[4];
        int cnt = 4;
        if (v < n4) {
            const float4 t = load_stream4(theta + 4 * v, k.stream);
            th[0] = t.x; th[1] = t.y; th[2] = t.z; th[3] = t.w;
        } else {
            cnt = tail;
            for (int e = 0; e < 4; ++e) th[e] = (e < cnt) ? theta[(n4 << 2) + e] : 0.0f;
        }
        float sv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        int ci[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (IDX) ci[e] = (int)anchor_level<true>(th[e], k);
        if (MARG) {
            // (one entry after the other in a loop that stays a loop, see the backward kernel; entries past the end
            // of the tensor are not visited)
#pragma unroll 1
            for (int e = 0; e < cnt; ++e) {
                const float th_e = e == 0 ? th[0] : (e == 1 ? th[1] : (e == 2 ? th[2] : th[3]));
                UniSums<JH> q;
                uni_sums<JH, 1, true>(th_e, u, q, acc_s, acc_d, acc_0);
                const float sv_e = (float)(u.delta * (u.c0 + q.S1 * uni_rcp(q.Z)));
                sv[0] = e == 0 ? sv_e : sv[0]; sv[1] = e == 1 ? sv_e : sv[1];
                sv[2] = e == 2 ? sv_e : sv[2]; sv[3] = e == 3 ? sv_e : sv[3];
            }
        } else if (SOFT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                UniSums<JH> q;
                uni_sums<JH, 1, false>(th[e], u, q, acc_s, acc_d, acc_0);
                sv[e] = (float)(u.delta * (u.c0 + q.S1 * uni_rcp(q.Z)));
            }
        }
        if (v < n4) {
            if (SOFT) store_stream4(soft + 4 * v, sv[0], sv[1], sv[2], sv[3], k.stream);
            if (IDX) reinterpret_cast<uint32_t *>(idx)[v] = pack_indices(ci[0], ci[1], ci[2], ci[3], k.idx_off);
        } else {
            for (int e = 0; e < cnt; ++e) {
                if (SOFT) soft[(n4 << 2) + e] = sv[e];
                if (IDX) idx[(n4 << 2) + e] = (int8_t)(ci[e] - k.idx_off);
            }
        }
    }

    if (MARG) {
        // per thread: the sums over its entries of P(level) for every level; row stride 2 JH + 1 doubles
        constexpr int LS = 2 * JH + 1;
        double *mine = uni_lds + (size_t)threadIdx.x * LS;
        // level index (from the lowest level) of the offsets +o_j and -o_j: odd sets pairs + j and pairs - j around the
        // centre level `pairs`; even sets pairs - 1 + j and pairs - j
        if (u.odd) mine[u.pairs] = acc_0;
#pragma unroll
        for (int j = 1; j <= JH; ++j) {
            if (j <= u.pairs) {
                const double up = 0.5 * u.e[j - 1][0] * (acc_s[j - 1] + acc_d[j - 1]);
                const double dn = 0.5 * u.e[j - 1][0] * (acc_s[j - 1] - acc_d[j - 1]);
                mine[u.odd ? u.pairs + j : u.pairs - 1 + j] = up;
                mine[u.pairs - j] = dn;
            }
        }
        __syncthreads();
        unsigned long long own = 0ull;
        // Every thread adds up one level over every kParts-th row (a wave reads consecutive words) into the first of them, which
        // nobody else reads; then a thread per level, the kParts sums.  One thread per level over all rows is a chain of 256 reads
        // and additions.  us, forward pass at alpha step^2 of 0.008 (31 levels), 0.037 (15) and 0.2 (7), that / this: 1000 entries of 31 levels 7.3 / 6.2, 8000 10.9 / 9.6, 131072 11.9 / 10.6,
        // 2 M 28.4 / 26.5; of 15 levels 131072 9.5 / 8.5; of 7 levels 9.0 / 8.0.
        constexpr int kParts = kUniThreads / LS;
        if ((int)threadIdx.x < kParts * LS) {
            double part = 0.0;
#pragma unroll 4
            for (int t = threadIdx.x; t < kUniThreads * LS; t += kParts * LS) part += uni_lds[t];
            uni_lds[threadIdx.x] = part;
        }
        __syncthreads();
        if ((int)threadIdx.x < k.n_levels) {
            double tot = 0.0;
#pragma unroll
            for (int t = 0; t < kParts; ++t) tot += uni_lds[(size_t)t * LS + threadIdx.x];
            own = (unsigned long long)__double2ll_rn(tot * (double)(1u << kHistScaleBits));
        }
        marginal_end<kUniThreads, FORM>(own, k.n_levels, fin);
    }
}

template <int JH, bool ODD, bool DTHETA, bool SCALARS>
__global__ __launch_bounds__(kUniThreads)
void quantize_bwd_uniform_kernel(const float *__restrict__ theta, const float *g, int64_t n, QConst k, UniConst u,
                                 float *dtheta /* may be g */, ScalarFinish fin)
{
    double acc_d = 0.0, acc_a = 0.0;
    const int64_t n4 = n >> 2;
    const int64_t stride = (int64_t)gridDim.x * kUniThreads;
    const int tail = (int)(n - (n4 << 2));
    for (int64_t v = (int64_t)blockIdx.x * kUniThreads + threadIdx.x; v < n4 + (tail ? 1 : 0); v += stride) {
        float th[4], ge[4];
        int cnt = 4;
        if (v < n4) {
            const float4 t = load_stream4(theta + 4 * v, k.stream);
            const float4 q = load_stream4(g + 4 * v, k.stream);
            th[0] = t.x; th[1] = t.y; th[2] = t.z; th[3] = t.w;
            ge[0] = q.x; ge[1] = q.y; ge[2] = q.z; ge[3] = q.w;
        } else {
            cnt = tail;
            for (int e = 0; e < 4; ++e) {
                th[e] = (e < cnt) ? theta[(n4 << 2) + e] : 0.0f;
                ge[e] = (e < cnt) ? g[(n4 << 2) + e] : 0.0f;
            }
        }
        float dv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        // One entry after the other, in a loop that stays a loop: four interleaved entries of this much double
        // arithmetic need more registers than four waves per SIMD leave (the compiler took 234, or spilled).
        // th_e, g_e and the outputs move through selects on the loop counter, which is uniform.
#pragma unroll 1
        for (int e = 0; e < 4; ++e) {
            const float th_e = e == 0 ? th[0] : (e == 1 ? th[1] : (e == 2 ? th[2] : th[3]));
            const float g_e = e == 0 ? ge[0] : (e == 1 ? ge[1] : (e == 2 ? ge[2] : ge[3]));
            UniSums<JH> q;
            uni_sums_literal<JH, SCALARS ? 3 : 2, ODD>(th_e, u, q);
            const double inv = uni_rcp(q.Z);
            const double mu = q.S1 * inv, m2 = q.S2 * inv;
            const double var = fma(-mu, mu, m2);
            const double gd = (double)g_e;
            const float dv_e = (float)(gd * (u.two_kappa * var));
            dv[0] = e == 0 ? dv_e : dv[0]; dv[1] = e == 1 ? dv_e : dv[1];
            dv[2] = e == 2 ? dv_e : dv[2]; dv[3] = e == 3 ? dv_e : dv[3];
            if (SCALARS) {
                const double m3 = q.S3 * inv;
                const double c3 = fma(-mu, fma(-2.0 * mu, mu, 3.0 * m2), m3);   // m3 - 3 mu m2 + 2 mu^3
                // Lemma 1 in offsets from the centre c0 (the derivation holds for any origin of the level index)
                const double t_d = (u.c0 + mu) + u.two_kappa * fma(q.r - u.c0 - 2.0 * mu, var, -c3);
                const double t_a = fma(2.0 * (q.r - mu), var, -c3);
                acc_d = fma(gd, t_d, acc_d);
                acc_a = fma(gd, t_a, acc_a);
            }
        }
        if (DTHETA) {
            if (v < n4) store_stream4(dtheta + 4 * v, dv[0], dv[1], dv[2], dv[3], k.stream);
            else for (int e = 0; e < cnt; ++e) dtheta[(n4 << 2) + e] = dv[e];
        }
    }
    if (SCALARS) scalar_finish<kUniThreads>(acc_d, acc_a, fin);
}

// The pairs of sums that the blocks of a large grid left.  Fixed summation order: thread t of all takes the pairs t, t + threads, ... (four
// independent chains, so that four loads are in flight: with a few thousand pairs one chain per thread is nothing but memory
// latency), then scalar_finish.  56448 pairs: one block 12.2 us, sixteen 6; 12501 pairs: one 5.0, four 5.8.
constexpr int kScalarFinThreads = 1024;

__global__ __launch_bounds__(kScalarFinThreads)
void scalar_finalize_kernel(const double *__restrict__ partial, int n_pairs, ScalarFinish fin)
{
    const int T = kScalarFinThreads * (int)gridDim.x;
    const double2 *pairs = reinterpret_cast<const double2 *>(partial);
    double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
    int i = blockIdx.x * kScalarFinThreads + threadIdx.x;
    for (; i + 3 * (int64_t)T < n_pairs; i += 4 * T) {
#pragma unroll
        for (int u = 0; u < 4; ++u) { const double2 v = pairs[i + u * T]; a[u] += v.x; b[u] += v.y; }
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)
        if (i + u * (int64_t)T < n_pairs) { const double2 v = pairs[i + u * T]; a[u] += v.x; b[u] += v.y; }
    scalar_finish<kScalarFinThreads>((a[0] + a[1]) + (a[2] + a[3]), (b[0] + b[1]) + (b[2] + b[3]), fin);
}

// ------------------------------------------------------------------------------------------
// The probabilistic quantizer Q_p (eq. Qprob, Sec. III-A) by inversion: with one uniform number
// u in [0,1) per entry the draw is the first level, in increasing order, whose cumulative
// probability exceeds u.  The comparison is made on un-normalised weights (cumulative weight against
// u * Z), which spares the division.  Reads theta and u, writes one index byte per entry.
// ------------------------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ int draw_one(float th, float u, const QConst &k)
{
    if (W > 0) {
        Band<W> b;
        band_weights<W, 1>(th, anchor_level<false>(th, k), k, b);
        const float target = u * b.Z;
        float cum = 0.0f;
        int pick = -W - 1, last = 0;
#pragma unroll
        for (int i = 0; i <= 2 * W; ++i) {
            const int j = i - W;
            const float w = j < 0 ? b.dn[-j - 1] : (j == 0 ? b.ctr : b.up[j - 1]);
            cum += w;
            if (w > 0.0f) last = j;
            if (pick < -W && cum > target) pick = j;
        }
        if (pick < -W) pick = last;
        return (int)b.cf + pick;
    } else {
        GenericSums g;
        generic_sums<false>(th, k, g);
        const float target = u * g.Z, two_u = 2.0f * g.u;
        float cum = 0.0f;
        int pick = g.jlo - 1, last = g.jlo;
        for (int j = g.jlo; j <= g.jhi; ++j) {
            const float w = generic_weight(j, two_u, k);
            cum += w;
            if (w > 0.0f) last = j;
            if (pick < g.jlo && cum > target) pick = j;
        }
        if (pick < g.jlo) pick = last;
        return (int)g.cf + pick;
    }
}

template <int W, int U>
__global__ __launch_bounds__(one_trip_threads(U), W == 1 || W == 2 ? 8 : 1)      // (W = 2, 13 M entries: eight waves 20.3, six 21.0 us)
void quantize_draw_kernel(const float *__restrict__ theta, const float *__restrict__ u, int64_t n, QConst k,
                          int8_t *__restrict__ idx)
{
    constexpr int T = one_trip_threads(U);
    const int64_t n4 = n >> 2;
    with_constant(k.stream != 0, [&](auto streams) {
        auto group = [&](int64_t v, auto count, auto ragged) {
            constexpr int N = decltype(count)::value;
            float4 t[N], r[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                t[i] = load_stream4(theta + 4 * (v + i * T), streams.value);
                r[i] = load_stream4(u + 4 * (v + i * T), streams.value);
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int c0 = draw_one<W>(t[i].x, r[i].x, k), c1 = draw_one<W>(t[i].y, r[i].y, k);
                const int c2 = draw_one<W>(t[i].z, r[i].z, k), c3 = draw_one<W>(t[i].w, r[i].w, k);
                reinterpret_cast<uint32_t *>(idx)[v + i * T] = pack_indices(c0, c1, c2, c3, k.idx_off);
            }
        };
        one_trip_or_loop<T, U>(n4, n4, group);      // (the tail is below)
    });
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        for (int64_t e = n4 << 2; e < n; ++e) idx[e] = (int8_t)(draw_one<W>(theta[e], u[e], k) - k.idx_off);
}

// ------------------------------------------------------------------------------------------
// Gradient of the entropy term (Sec. IV-D; Algorithm 1, the step that forms the partials of H).
// With l_k = log2 of the marginal PMF (0 where the marginal is 0), for one entry
//     dH/dtheta = -(2 alpha delta / n) Cov_P(k, l_k)
//     dH/dq     = -(2 alpha / n) (theta Cov_P(k, l) - delta Cov_P(k^2, l))
//     dH/dalpha =  (1 / n) (-2 theta delta Cov_P(k, l) + delta^2 Cov_P(k^2, l))
// (differentiate H = -sum m log2 m through m_k = mean of P_k, with the CPMF derivatives of App. B).
// In band offsets j = k - c, lam_j = l_(c+j) - l_c:  C1 = Cov(j, lam),  C2 = Cov(j^2, lam),
// Cov(k^2, l) = 2 c C1 + C2, so with r = u / delta
//     dH/dq     = -(2 alpha delta / n) sum_e ((r - c) C1 - C2)
//     dH/dalpha =  (delta^2 / n)       sum_e (C2 - 2 r C1)
// The table of l_k sits in LDS with kPad zeros on both sides.  dtheta = g_in + scale * dH/dtheta.
// ------------------------------------------------------------------------------------------
// (bands: registers for eight waves.  Without the scalar sums the compiler takes up to 127 for three and four levels on each side, and four waves: 25 M entries 85.7, so 76.3 us)
template <int W, bool DTHETA, bool SCALARS, bool ADD, int U>
__global__ __launch_bounds__(one_trip_threads(U), W > 0 ? 8 : 1)
void entropy_bwd_kernel(const float *__restrict__ theta, const float *__restrict__ marg, const float *__restrict__ g_in,
                        int64_t n, QConst k, float dtheta_mul /* scale * (-2 alpha delta / n) */,
                        float *__restrict__ dtheta, ScalarFinish fin)
{
    // l_k as a sum of two floats: only differences of l enter, between levels a few apart, and the scalar
    // sums multiply them by the anchor index - with a level set around index 100 the 2^-24 of a single float
    // l_k (about -5) showed as 2e-4 of dH/dq
    __shared__ float ell[256 + 2 * kPad], ell_fine[256 + 2 * kPad];
    constexpr int T = one_trip_threads(U);
    for (int i = threadIdx.x; i < k.n_levels + 2 * kPad; i += T) {
        const int lv = i - kPad;
        double v = 0.0;
        if (lv >= 0 && lv < k.n_levels) { const float m = marg[lv]; v = m > 0.0f ? log2((double)m) : 0.0; }
        const float hi = (float)v;
        ell[i] = hi;
        ell_fine[i] = (float)(v - (double)hi);
    }
    __syncthreads();
    const float *ell0 = ell + kPad - k.lo;    // ell0[level] for level in [lo - kPad, hi + kPad]
    const float *fine0 = ell_fine + kPad - k.lo;

    double acc_d = 0.0, acc_a = 0.0;
    const int64_t n4 = n >> 2;
    auto four = [&](const float (&th)[4], const float (&ge)[4], int cnt, float (&dv)[4]) {
        float sum_d = 0.0f, sum_a = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float cf, u, Z, S1, S2, B0 = 0.0f, B1 = 0.0f, B2 = 0.0f;
            if (W > 0) {
                Band<W> b;
                band_weights<W, 2>(th[e], anchor_level<false>(th[e], k), k, b);
                cf = b.cf; u = b.u; Z = b.Z; S1 = b.S1; S2 = b.S2;
                const float *lp = ell0 + (int)cf, *fp = fine0 + (int)cf;
                const float l0 = lp[0], f0 = fp[0];
#pragma unroll
                for (int j = 1; j <= W; ++j) {
                    const float jf = (float)j;
                    const float xu = b.up[j - 1] * ((lp[j] - l0) + (fp[j] - f0)), xd = b.dn[j - 1] * ((lp[-j] - l0) + (fp[-j] - f0));
                    B0 += xu + xd;
                    B1 = fmaf(jf, xu - xd, B1);
                    B2 = fmaf(jf * jf, xu + xd, B2);
                }
            } else {
                GenericSums s;
                generic_sums<false>(th[e], k, s);
                cf = s.cf; u = s.u; Z = s.Z; S1 = s.S1; S2 = s.S2;
                const float *lp = ell0 + (int)cf, *fp = fine0 + (int)cf;
                const float l0 = lp[0], f0 = fp[0], two_u = 2.0f * u;
                for (int j = s.jlo; j <= s.jhi; ++j) {
                    const float jf = (float)j;
                    const float x = generic_weight(j, two_u, k) * ((lp[j] - l0) + (fp[j] - f0));
                    B0 += x;
                    B1 = fmaf(jf, x, B1);
                    B2 = fmaf(jf * jf, x, B2);
                }
            }
            const float inv = fast_rcp(Z);
            const float mu = S1 * inv, m2 = S2 * inv, b0 = B0 * inv;
            const float C1 = fmaf(-mu, b0, B1 * inv), C2 = fmaf(-m2, b0, B2 * inv);
            dv[e] = ADD ? fmaf(dtheta_mul, C1, ge[e]) : dtheta_mul * C1;
            if (SCALARS && e < cnt) {
                const float r = u * k.inv_delta;
                sum_d += fmaf(r - cf, C1, -C2);
                sum_a += fmaf(-2.0f * r, C1, C2);
            }
        }
        if (SCALARS) { acc_d += (double)sum_d; acc_a += (double)sum_a; }
    };
    with_constant(k.stream != 0, [&](auto streams) {
        auto group = [&](int64_t v, auto count, auto ragged) {
            constexpr int N = decltype(count)::value;
            const int cnt = !ragged.value || v < n4 ? 4 : (int)(n - (n4 << 2));      // (the last vector as in quantize_bwd_kernel: 256 K entries of 127 levels in the soft regime 37.6 us by itself, so 22.0)
            float4 t[N], q[N];
            if (!ragged.value || cnt == 4) {
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    t[u] = load_stream4(theta + 4 * (v + u * T), streams.value);
                    q[u] = ADD ? load_stream4(g_in + 4 * (v + u * T), streams.value) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
            } else {
                t[0] = load_first(theta + 4 * v, cnt);
                q[0] = ADD ? load_first(g_in + 4 * v, cnt) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float th[4] = {t[u].x, t[u].y, t[u].z, t[u].w}, ge[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
                float dv[4];
                four(th, ge, cnt, dv);
                if (DTHETA) {
                    if (!ragged.value || cnt == 4) store_stream4(dtheta + 4 * (v + u * T), dv[0], dv[1], dv[2], dv[3], streams.value);
                    else for (int e = 0; e < cnt; ++e) dtheta[4 * v + e] = dv[e];
                }
            }
        };
        one_trip_or_loop<T, U>(n4, (n + 3) >> 2, group);
    });
    if (SCALARS) scalar_finish<T>(acc_d, acc_a, fin);
}

__global__ void zero_floats_kernel(float *a, int na, float *b, int nb, float *c, int nc)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (a && i < na) a[i] = 0.0f;
    if (b && i < nb) b[i] = 0.0f;
    if (c && i < nc) c[i] = 0.0f;
}

}  // namespace

// Which unrolled band kernel serves these parameters (0: the generic loop).
int band_template(const QConst &k) { return (!k.slide && k.wgen <= 4) ? k.wgen : 0; }

QConst make_const(const cdl_qparams &p)
{
    QConst k;
    const double delta = (double)p.delta, alpha = (double)p.alpha;
    const double kappa = alpha * delta * delta;
    k.delta = p.delta;
    k.inv_delta = (float)(1.0 / delta);
    k.c1 = (float)(alpha * delta * 1.4426950408889634);
    k.b2 = (float)(2.0 * alpha * delta * 1.4426950408889634);
    k.k1 = (float)exp(-kappa);
    k.k4 = (float)exp(-4.0 * kappa);
    k.two_kappa = (float)(2.0 * kappa);
    k.lo = p.lo;
    k.idx_off = index_offset(p);
    k.n_levels = p.n_levels;
    k.lo_f = (float)p.lo;
    k.hi_f = (float)(p.lo + p.n_levels - 1);
    k.lo1_f = k.lo_f + 1.0f;
    k.hi1_f = k.hi_f - 1.0f;
    k.near = (float)(0.5 * delta * (1.0 - 1.0 / (1 << 20)));
    k.wgen = quantizer_window(kappa, p.n_levels);
    k.slide = 0;
    k.stream = 0;
    k.u_clamp = INFINITY;
    if (p.top_k > 0 && p.top_k < p.n_levels) {
        // Truncated CPMF.  Where the band that kappa asks for is no wider than the top_k nearest levels the
        // truncation drops nothing above fp32 resolution and the ordinary kernels serve; otherwise the generic
        // kernels run on exactly the top_k nearest levels.
        const int wt = (p.top_k - 1) / 2;
        if (k.wgen > wt) { k.wgen = wt; k.slide = 1; }
    }
    if (band_template(k) == 2) k.u_clamp = (float)(30.0 / (2.0 * alpha * delta * 1.4426950408889634));
    return k;
}

namespace {

int grid_for(int64_t n)
{
    const int64_t vecs = (n >> 2) + 1;
    int64_t blocks = (vecs + kQuantThreads - 1) / kQuantThreads;
    if (blocks > kMaxQuantBlocks) blocks = kMaxQuantBlocks;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

// Whether the kernels that take a large tensor in one trip serve: the unrolled bands (the loop over the levels is bound by arithmetic).
bool one_trip_serves(int64_t n, const QConst &k) { return n > kOneTripEntries && band_template(k) != 0 && one_trip_fits(n); }

// Gradients of the quantizer.  Wider bands: a loop's waits hide behind the arithmetic up to twice as many entries.  us without scalars, loop / one trip, one to four levels on each side: 3.2 M entries
// 9.5 / 9.3, 9.4 / 9.1, 10.0 / 10.6, 10.7 / 11.7; 4.5 M 12.0 / 11.6, 11.8 / 11.4, 13.0 / 12.8, 14.3 / 14.4.
bool gradient_one_trip(int64_t n, const QConst &k) { return one_trip_serves(n, k) && (band_template(k) <= 2 || n >= 2 * kOneTripEntries); }

// Gradient of the entropy: every block makes the logarithms of all levels first, and with the scalar gradients a looping grid finishes their sums itself where blocks of one trip that stream leave them for a
// second launch.  There one trip pays only for very large tensors that are added to a gradient as well, with up to two levels on each side.  us with the scalars, loop / one trip, 64 levels, two on each side:
// 3.2 M entries 13.4 / 13.1, 6 M 18.7 / 18.7, 24 M 50.1 / 54.9, 60 M 114 / 121, added to a gradient 24 M 56.6 / 57.5, 60 M 135 / 131 (one on each side 130 / 120); four on each side 3.2 M 17.3 / 19.1, 24 M 81 / 89;
// 255 levels, two on each side 3.2 M 14.7 / 14.6, 24 M 54 / 66, 60 M 126 / 146, added 134 / 147.  Without them, added to a gradient, 255 levels, two on each side: 25 M 57.7 / 50.2, 50 M 115.6 / 97.3.
bool entropy_one_trip(int64_t n, const QConst &k, bool scalars, bool add)
{
    if (!gradient_one_trip(n, k)) return false;
    if (!scalars) return true;
    const int w = band_template(k);
    return w <= 2 && (n < kStreamFrom || (add && n >= 4 * kStreamFrom && (w == 1 || k.n_levels <= 64)));
}

// Draws (two streams of floats read) and forward passes without PMF (with soft values: one read, one written).  Indices alone leave a loop nearly no stores to wait for.  us, loop / one trip, two levels on each side: draws 4.3 M
// entries 9.5 / 9.9, 6.5 M 13.0 / 13.1, 8.8 M 16.0 / 14.9, 24 M 41 / 35; index and soft value 10.9 / 11.5 (5.3 M), 12.6 / 12.9, 15.4 / 14.8, 38.3 / 34.1; four on each side 5.3 M 15.6 / 15.3, 6.5 M 18.2 / 17.1;
// indices alone 4.3 M 5.3 / 5.8, 8.8 M 8.6 / 9.2, 16 M 14.4 / 14.5, 24 M 21.0 / 20.6, 48 M 39.7 / 37.7.
bool forward_one_trip(int64_t n, const QConst &k, bool two_streams)
{
    return one_trip_serves(n, k) && n >= (!two_streams ? 2 * kStreamFrom : band_template(k) <= 2 ? kStreamFrom : 3 * kOneTripEntries);
}

// Up to four times as many blocks as can finish the job themselves: that many, of more trips each.  A second launch costs more
// (forward + backward of 0.3 M entries, 15 levels: 13.8 -> 12.3 us, 255 levels 17.3 -> 14.1; 0.9 M, 15 levels 17.0 -> 16.1) - not in
// the soft regime, whose kernels are bound by arithmetic.
int finishing_grid(int64_t blocks)
{
    if (blocks > 4 * kFinishMaxBlocks) return (int)blocks;
    const int64_t trips = (blocks + kFinishMaxBlocks - 1) / kFinishMaxBlocks;
    return (int)((blocks + trips - 1) / trips);
}

// Grid of the histogram kernels: half of grid_for, but never more than kMaxHistTrips trips per block, and - once
// the chip is full - a whole number of rounds: 256 CUs hold four 512-thread blocks each (2048 threads; the
// histogram of 256 levels takes 33 KB of the 160 KB of LDS), and a last round that fills half of them
// cost 10-18 % on 50 M entries.
constexpr int64_t kHistResident = 256 * 4;
constexpr int64_t kHistFullFrom = 16ll << 20;

int64_t hist_grid_for(int64_t n, bool half)
{
    const int64_t vecs = (n >> 2) + 1;
    const int64_t need = (vecs + (int64_t)kMargThreads * kMaxHistTrips - 1) / ((int64_t)kMargThreads * kMaxHistTrips);
    const int64_t full = (grid_for(n) + 1) / 2, g = half && full > kHistResident / 2 ? kHistResident / 2 : full;
    return need > g ? (need + kHistResident - 1) / kHistResident * kHistResident : g;
}

// Where half of them are better: large sets in tensors that four blocks of a compute unit take in few trips, since every block clears its bins first and adds them up
// last, 2 - 3 us in which it loads and stores nothing; and the kernel of 17 to 33 levels on a common centre, of which a compute unit holds two blocks.
// us, index, soft value and PMF, on 1024 / 512 blocks: 2.36 M entries of 255 levels, two on each side 14.5 / 13.5, 5 M 18.5 / 18.4, 12.8 M 30.2 / 30.2 (without soft values
// 27.0 / 26.3), of 200 levels 14.0 / 12.9, of 127 13.6 / 13.5, 12.8 M of 127 29.1 / 30.3, of 15 29.0 / 29.5; four on each side 9 M of 255 33.7 / 36.0; on a common
// centre 2.5 M of 31 levels 32.9 / 30.2, 13 M of 7 60.8 / 70.4; the nearest five of 15 levels 16 M 61.3 / 69.6.
bool hist_half(int64_t n, const QConst &k, int uniform_half)
{
    if (n <= kOneTripEntries || n >= kHistFullFrom) return false;
    const int w = band_template(k);
    return uniform_half == kUniMaxJH || ((w == 1 || w == 2) && k.n_levels >= 192);
}

// Whether a trip takes kHistVectors vectors a thread and their loads go ahead of the stores of the trip before: where soft values are stored as well and the arithmetic of
// an entry is short.  us, index, soft value and PMF, a vector a trip / so: 25.6 M entries of 31 levels, two on each side 47.7 / 47.1, 50.3 M 81.1 / 79.2, 12.8 M 28.8 / 29.8;
// index and PMF 25.6 M 39.6 / 40.6, 36 M 48.8 / 51.4; three on each side 25.6 M of 15 levels 61.5 / 65.8.
constexpr int kHistVectors = 2;
bool hist_ahead(int64_t n, const QConst &k) { return n >= kHistFullFrom && (band_template(k) == 1 || band_template(k) == 2); }

// Who adds up the blocks' histograms.  Up to 256 blocks finish the job themselves: the last one where they have 4096 records (of a level) at most, beyond, blocks of their own behind them, a slice of the
// levels each (cdl_marg_slices.h; the unrolled bands only, the others keep the last block up to 16384).  Blocks of one trip and more than 16384 records, and larger grids, leave rows for a second launch.
// us of the forward pass, second launch / slices: 65536 entries of 255 levels (33 blocks) 10.0 / 7.7, 131068 (64 blocks, 16320 records) 9.9 / 8.3, 262144 of 63 (129) 9.9 / 8.2, 700 K of 255 (171, two trips) 10.0 / 10.1, 2.1 M (256, four) 13.1 / 13.2;
// beyond the line 131072 of 255 (65 blocks) 9.9 / 8.5, 524284 (256) 9.8 / 9.7, of 200 with four levels on each side 10.1 / 11.1 (the line is older than the collectors; up to 128 blocks it could go); 1024 blocks (the last ones with entries of their own): 6 M of 63 17.7 / 18.7, 25.6 M of 31 46.0 / 46.9.
// Last block / slices: 65536 of 255 10.1 / 8.1;  63 levels 520 K (254) 15.4 / 9.2, 1 M (245, two) 16.9 / 10.0, 2.1 M 18.4 / 13.0.
MargForm marg_form(int64_t blocks, int64_t n, const cdl_qparams &p, const QConst &k)
{
    if (blocks > kFinishMaxBlocks) return kMargRows;
    const int64_t records = blocks * p.n_levels;
    if (band_template(k) == 0) return records <= 16384 ? kMargLast : kMargRows;
    const bool one_trip = n <= blocks * (4 * kMargThreads);
    return records <= 4096 ? kMargLast : records <= 16384 || !one_trip ? kMargSlices : kMargRows;
}

// workspace layout: [rows of the histogram kernel's blocks][records of the finishing blocks][scalar partials or records]
// (or the table and the rows of moments of the soft regime)
// (never less than a smaller tensor has: callers keep one workspace for several)
size_t hist_row_bytes(int64_t n, int32_t n_levels) { return align_up((size_t)hist_grid_for(n, false) * (size_t)n_levels * sizeof(unsigned long long), 256); }
size_t hist_bytes(int64_t n, int32_t n_levels)
{
    const size_t rows = hist_row_bytes(n, n_levels);
    const size_t soft = n >= kSoftFrom ? align_up(soft_fwd_bytes(n, n_levels), 256) : 0;
    return rows > soft ? rows : soft;
}
constexpr size_t kRecordBytes = 16384 * 2 * sizeof(unsigned long long);      // (marginal_finalize_kernel: at most 16 chunks of 256 levels)

// Whether the blocks' sums are left for a second launch (cdl_finish.h), and where: [records of the launch that adds up][partial sums or records]
bool scalars_in_two_launches(int64_t n, int grid) { return n >= kStreamFrom && grid > kMaxQuantBlocks; }
constexpr int kScalarFinBlocks = 16;
constexpr size_t kScalarFinBytes = kScalarFinBlocks * 4 * sizeof(unsigned long long);

ScalarFinish scalar_finish_args(void *scalars, int64_t n, int grid, double mul_d, double mul_a, float *d_delta, float *d_alpha)
{
    ScalarFinish f{};
    char *const area = reinterpret_cast<char *>(scalars) + kScalarFinBytes;
    if (scalars_in_two_launches(n, grid)) f.partial = reinterpret_cast<double *>(area);
    else { f.records = reinterpret_cast<unsigned long long *>(area); f.tag = next_finish_tag(); }
    f.mul_d = mul_d; f.mul_a = mul_a; f.d_delta = d_delta; f.d_alpha = d_alpha;
    return f;
}

int launch_scalar_end(const ScalarFinish &f, void *scalars, int grid, hipStream_t stream)
{
    const int rc = check_launch();
    if (rc != CDL_OK || !f.partial) return rc;
    ScalarFinish last = f;
    last.partial = nullptr;
    last.records = reinterpret_cast<unsigned long long *>(scalars);
    last.tag = next_finish_tag();
    const int blocks = grid <= 16384 ? 1 : kScalarFinBlocks;
    CDL_LAUNCH("scalar_finalize_kernel", stream, scalar_finalize_kernel, dim3(blocks), dim3(kScalarFinThreads), 0, f.partial, grid, last);
    return check_launch();
}

template <int W>
void launch_fwd(bool want_idx, bool want_soft, bool want_marg, bool one_trip, MargForm form, int grid, hipStream_t s,
                  const float *theta, int64_t n, const QConst &k, int8_t *idx, float *soft,
                  const MargFinish &fin)
{
    const size_t lds = (size_t)(k.n_levels + 2 * kPad) * kHistCopies * sizeof(unsigned int);
#define CDL_FWD(I, S, M, F, U)                                                                            \
    CDL_LAUNCH((I) ? "quantize_fwd_kernel" : "quantize_fwd_kernel(marginal only)", s,                     \
               (quantize_fwd_kernel<W, I, S, M, F, U>), dim3(grid), dim3((M) ? kMargThreads : one_trip_threads(U)), \
               (M) ? lds : 0, theta, n, k, idx, soft, fin)
#define CDL_FWD_MARG(I, S)                                                                                \
    do {                                                                                                  \
        if (form == kMargLast) CDL_FWD(I, S, true, kMargLast, 1);                                         \
        else if (form == kMargRows) CDL_FWD(I, S, true, kMargRows, 1);                                    \
        else if constexpr (W > 0) CDL_FWD(I, S, true, kMargSlices, 1);                                    \
    } while (0)
    constexpr int UM = W == 1 || W == 2 ? kHistVectors : 1, UN = W > 0 ? kOneTripVectors : 1;
    if (want_idx && want_soft && want_marg && form == kMargRows && hist_ahead(n, k)) CDL_FWD(true, true, true, kMargRows, UM);
    else if (want_idx && want_soft && want_marg) CDL_FWD_MARG(true, true);
    else if (want_idx && want_soft && one_trip) CDL_FWD(true, true, false, kMargRows, UN);
    else if (want_idx && want_soft) CDL_FWD(true, true, false, kMargRows, 1);
    else if (want_idx && want_marg) CDL_FWD_MARG(true, false);
    else if (want_idx && one_trip) CDL_FWD(true, false, false, kMargRows, UN);
    else if (want_idx) CDL_FWD(true, false, false, kMargRows, 1);
    else CDL_FWD_MARG(false, false);
#undef CDL_FWD_MARG
#undef CDL_FWD
}

// The soft-regime kernels on a common centre serve: the full CPMF, 6 to 33 levels (smaller sets always fall to
// the unrolled band kernels), and kappa * JH^2 <= 72 with JH the padded half-width, so that T^JH stays finite
// at +-r_safe.  Returns the padded half-width (4, 8 or 16), or 0 when the other kernels serve.
int uniform_half_width(const cdl_qparams &p, const QConst &k)
{
    if (k.slide || band_template(k) != 0) return 0;
    if (p.n_levels < 6 || p.n_levels > 2 * kUniMaxJH + 1) return 0;
    const int pairs = p.n_levels / 2;
    const int jh = pairs <= 4 ? 4 : (pairs <= 8 ? 8 : 16);
    const double kappa = (double)p.alpha * (double)p.delta * (double)p.delta;
    // only where (nearly) every level is live anyway: a band much narrower than the set is cheaper in the generic loop
    if (2 * k.wgen + 1 < p.n_levels - 2) return 0;
    if (kappa * jh * jh > 72.0) return 0;
    return jh;
}

// Where the table of cdl_soft.hip is faster than these kernels although it takes two small launches more (us, table against
// loop over the levels, at n * (n_levels / 2) = 1, 2, 3 times 2^24):
//   forward   31 levels  27.0/23.5  30.3/29.9  33.4/36.6     15 levels  30.1/22.6  37.0/34.3  42.2/45.6     7 levels  38.5/31.7  53.4/53.4  69.0/77.1 (4)
//   backward             16.0/14.6  19.8/21.9  22.4/28.5                19.1/18.3  26.8/30.3  32.7/40.2               28.1/28.5  43.1/48.2  58.8/71.6
// The loop over the levels, forward only for sets that it serves, is left for the
// table from kSoftFrom on (63 levels, 65 K entries: 24 against 50 us; 255 levels: 36 against 156, 1 M entries 39 against 245).
// The backward pass of those larger sets stays with the loop: in the soft regime the scalar gradients' sums cancel
// almost completely, and what is left there are the roundings of the loop's own arithmetic.
bool soft_fwd_from_uniform(const cdl_qparams &p, int64_t n) { return n * (p.n_levels / 2) >= (5ll << 23); }
bool soft_bwd_from_uniform(const cdl_qparams &p, int64_t n) { return n * (p.n_levels / 2) >= (3ll << 23); }

UniConst make_uniform(const cdl_qparams &p, int jh)
{
    UniConst u{};
    const double delta = (double)p.delta, alpha = (double)p.alpha;
    const double kappa = alpha * delta * delta;
    u.delta = delta;
    u.inv_delta = 1.0 / delta;
    u.odd = p.n_levels & 1;
    u.pairs = p.n_levels / 2;
    u.c0 = (double)p.lo + 0.5 * (double)(p.n_levels - 1);
    u.x_per_r = kappa * 1.4426950408889634;
    u.two_kappa = 2.0 * kappa;
    u.r_safe = (double)jh + 15.0 / kappa;
    for (int j = 1; j <= kUniMaxJH; ++j) {
        const double o = u.odd ? (double)j : (double)j - 0.5;
        const double E = j <= u.pairs ? exp(-kappa * o * o) : 0.0;
        u.e[j - 1][0] = E;
        u.e[j - 1][1] = o * E;
        u.e[j - 1][2] = o * o * E;
        u.e[j - 1][3] = o * o * o * E;
    }
    return u;
}

template <int JH>
int launch_fwd_uniform(bool want_idx, bool want_soft, bool want_marg, MargForm form, int grid, hipStream_t s, const float *theta, int64_t n,
                       const QConst &k, const UniConst &u, int8_t *idx, float *soft, const MargFinish &fin)
{
    const size_t lds = want_marg ? (size_t)kUniThreads * (2 * JH + 1) * sizeof(double) : 0;
#define CDL_UNI(I, S, M)                                                                                        \
    do {                                                                                                        \
        if (lds > 65536) {                                                                                      \
            const hipError_t e_ = hipFuncSetAttribute((const void *)quantize_fwd_uniform_kernel<JH, I, S, (M) != 0, (M) == 2 ? kMargLast : kMargRows>,   \
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);    \
            if (e_ != hipSuccess) return hip_failed(e_);                                                        \
        }                                                                                                       \
        CDL_LAUNCH((I) ? "quantize_fwd_kernel" : "quantize_fwd_kernel(marginal only)", s,                       \
                   (quantize_fwd_uniform_kernel<JH, I, S, (M) != 0, (M) == 2 ? kMargLast : kMargRows>), dim3(grid), dim3(kUniThreads), lds,              \
                   theta, n, k, u, idx, soft, fin);                                                 \
    } while (0)
    const bool few = form == kMargLast;
    if (want_idx && want_soft && want_marg && few) CDL_UNI(true, true, 2);
    else if (want_idx && want_soft && want_marg) CDL_UNI(true, true, 1);
    else if (want_idx && want_soft) CDL_UNI(true, true, 0);
    else if (want_idx && want_marg && few) CDL_UNI(true, false, 2);
    else if (want_idx && want_marg) CDL_UNI(true, false, 1);
    else if (few) CDL_UNI(false, false, 2);
    else CDL_UNI(false, false, 1);
#undef CDL_UNI
    return CDL_OK;
}

template <int JH>
void launch_bwd_uniform(bool want_dtheta, bool want_scalars, int grid, hipStream_t s, const float *theta, const float *g,
                        int64_t n, const QConst &k, const UniConst &u, float *dtheta, const ScalarFinish &fin)
{
#define CDL_UNIB(D, S)                                                                                                          \
    do {                                                                                                                        \
        if (u.odd) CDL_LAUNCH("quantize_bwd_kernel", s, (quantize_bwd_uniform_kernel<JH, true, D, S>), dim3(grid), dim3(kUniThreads), 0, \
                              theta, g, n, k, u, dtheta, fin);                                                              \
        else CDL_LAUNCH("quantize_bwd_kernel", s, (quantize_bwd_uniform_kernel<JH, false, D, S>), dim3(grid), dim3(kUniThreads), 0,      \
                        theta, g, n, k, u, dtheta, fin);                                                                    \
    } while (0)
    if (want_dtheta && want_scalars) CDL_UNIB(true, true);
    else if (want_dtheta) CDL_UNIB(true, false);
    else CDL_UNIB(false, true);
#undef CDL_UNIB
}

template <int W>
void launch_bwd_w(bool want_dtheta, bool want_scalars, bool one_trip, int grid, hipStream_t s, const float *theta,
                  const float *g, int64_t n, const QConst &k, float *dtheta, const ScalarFinish &fin)
{
    constexpr int U = W > 0 ? kOneTripVectors : 1;
#define CDL_BWD(D, S) \
    do { \
        if (one_trip) CDL_LAUNCH("quantize_bwd_kernel", s, (quantize_bwd_kernel<W, D, S, U>), dim3(grid), dim3(one_trip_threads(U)), 0, \
                                 theta, g, n, k, dtheta, fin); \
        else CDL_LAUNCH("quantize_bwd_kernel", s, (quantize_bwd_kernel<W, D, S, 1>), dim3(grid), dim3(kQuantThreads), 0, \
                        theta, g, n, k, dtheta, fin); \
    } while (0)
    if (want_dtheta && want_scalars) CDL_BWD(true, true);
    else if (want_dtheta) CDL_BWD(true, false);
    else CDL_BWD(false, true);
#undef CDL_BWD
}

}  // namespace

// Level sets that reach beyond 127 (the paper's unsigned 8-bit alphabet {0, ..., 255}, eq. repo_alphabet) are
// stored as index - 128, which fits an int8 because such sets start at 0 or above.
int index_offset(const cdl_qparams &p) { return (int64_t)p.lo + p.n_levels - 1 > 127 ? 128 : 0; }

// Smallest W such that every level m > W away from the nearest one has relative weight
// m^3 exp(-kappa m (m-1)) below 3e-9, i.e. below fp32 resolution of every moment used.
int quantizer_window(double kappa, int n_levels)
{
    int W = 1;
    while (W < n_levels - 1) {
        const double m = (double)(W + 1);
        if (kappa * m * (m - 1.0) > 19.6 + 3.0 * log(m)) break;
        ++W;
    }
    return W;
}

void *quantize_scalar_area(void *ws, int64_t n, int32_t n_levels) { return reinterpret_cast<char *>(ws) + hist_bytes(n, n_levels) + kRecordBytes; }

size_t quantize_sum_bytes(int64_t n)
{
    // (one-trip grids below kStreamFrom and looping grids keep records, larger ones pairs; never less than a smaller tensor)
    const size_t records = (size_t)scalar_records(one_trip_grid(kStreamFrom)) * 4 * sizeof(unsigned long long), pairs = (size_t)one_trip_grid(n) * 2 * sizeof(double);
    const size_t small = (size_t)scalar_records(kMaxQuantBlocks) * 4 * sizeof(unsigned long long);
    return align_up(kScalarFinBytes + (n <= kOneTripEntries ? small : records > pairs ? records : pairs), 256);
}

size_t quantize_scalar_bytes(int64_t n) { return quantize_sum_bytes(n) + kSoftTableBytes; }

size_t quantize_workspace_bytes(int64_t n, int32_t n_levels)
{
    return hist_bytes(n, n_levels) + kRecordBytes + quantize_scalar_bytes(n);
}

// ---- built-in scratch for callers that cannot allocate ---------------------------------------
// One array per GPU the library runs on, held until the process ends.  In host code the array's name is only a
// stand-in: the device address comes from hipGetSymbolAddress, looked up once per device (with that device
// current) and kept; kernels and copies are always handed that address.
// kStaticScratchBytes are for the blocks' histograms and 65792 bytes that the documented limit counts with them; the records of the
// blocks that finish a marginal PMF lie behind.  The soft regime's table and rows, which take the place of the histograms, are smaller.
namespace {
constexpr size_t kStaticBesideRows = 65792;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kRecordBytes];
static_assert(kStaticScratchBytes - kStaticBesideRows >= kSoftTableBytes + 256 * (size_t)kSoftRowWords * sizeof(long long) + 256, "soft regime");

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

bool quantizer_static_fits(int64_t n, int32_t n_levels) { return hist_row_bytes(n, n_levels) + kStaticBesideRows <= kStaticScratchBytes; }

int quantizer_static_scratch(void **ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_failed(e);
    if (dev < 0 || dev >= kMaxDevices) return CDL_ERR_PARAM;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_failed(e);
        if (!p) return hip_failed(hipErrorInvalidSymbol);
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return CDL_OK;
}

int launch_quantize_fwd(const float *theta, int64_t n, const cdl_qparams &p,
                        int8_t *idx, float *soft, float *marg, float *entropy_bits,
                        void *ws, hipStream_t stream)
{
    const bool want_marg = (marg != nullptr) || (entropy_bits != nullptr);
    if (n == 0) {
        if (want_marg) {
            CDL_LAUNCH("zero_floats_kernel", stream, zero_floats_kernel, dim3(1), dim3(256), 0, marg, marg ? p.n_levels : 0,
                               entropy_bits, entropy_bits ? 1 : 0, (float *)nullptr, 0);
            return check_launch();
        }
        return CDL_OK;
    }
    QConst k = make_const(p);
    k.stream = n >= kStreamFrom;
    int64_t grid64 = want_marg ? hist_grid_for(n, hist_half(n, k, uniform_half_width(p, k))) : grid_for(n);
    if (want_marg && band_template(k) != 0 && n <= 4ll * kFinishMaxBlocks * kMargThreads * 4) grid64 = finishing_grid(grid64);
    if (grid64 > 2147483647LL) return CDL_ERR_PARAM;
    const bool one_trip = !want_marg && forward_one_trip(n, k, soft != nullptr);
    int grid = one_trip ? (int)one_trip_grid(n) : (int)grid64;
    MargFinish fin{};
    if (want_marg) {
        fin.rows = reinterpret_cast<unsigned long long *>(ws);
        fin.records = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(ws) + hist_bytes(n, p.n_levels));
        fin.tag = next_finish_tag();
        fin.inv_n = 1.0 / ((double)n * (double)(1u << kHistScaleBits));
        fin.marg = marg;
        fin.entropy_bits = entropy_bits;
    }
    const bool uniform = uniform_half_width(p, k) != 0;
    const SoftPlan plan = want_marg && (soft_fwd_from_uniform(p, n) || !uniform) ? soft_plan(p, k, n, uniform) : SoftPlan{};
    if (plan.bins) return launch_soft_fwd(theta, n, p, k, plan, idx, soft, fin, ws, stream);
    const bool want_idx = idx != nullptr, want_soft = soft != nullptr;
    const int jh = (want_soft || want_marg) ? uniform_half_width(p, k) : 0;
    if (jh && grid > kMaxQuantBlocks) grid = kMaxQuantBlocks;      // (any grid serves: the loop strides over the tensor)
    const MargForm form = want_marg ? marg_form(grid, n, p, k) : kMargRows;
    if (form == kMargSlices) {
        // (the records take the rows' place and, padded to fours, begin to take that of the others, at whose end the slices leave their entropy terms: 6 of 256 KB)
        fin.records += kRecordBytes / sizeof(unsigned long long) - 2 * kMargCollectors;
        fin.lg_per = marg_lg_per(grid, p.n_levels);
        fin.roles = MargRoles{grid, marg_slices(p.n_levels, fin.lg_per)};
        grid = fin.roles.grid();
    }
    if (jh) {
        const UniConst u = make_uniform(p, jh);
        int rcu = CDL_OK;
        if (jh == 4) rcu = launch_fwd_uniform<4>(want_idx, want_soft, want_marg, form, grid, stream, theta, n, k, u, idx, soft, fin);
        else if (jh == 8) rcu = launch_fwd_uniform<8>(want_idx, want_soft, want_marg, form, grid, stream, theta, n, k, u, idx, soft, fin);
        else rcu = launch_fwd_uniform<16>(want_idx, want_soft, want_marg, form, grid, stream, theta, n, k, u, idx, soft, fin);
        if (rcu != CDL_OK) return rcu;
    } else
    switch (band_template(k)) {
        case 1: launch_fwd<1>(want_idx, want_soft, want_marg, one_trip, form, grid, stream, theta, n, k, idx, soft, fin); break;
        case 2: launch_fwd<2>(want_idx, want_soft, want_marg, one_trip, form, grid, stream, theta, n, k, idx, soft, fin); break;
        case 3: launch_fwd<3>(want_idx, want_soft, want_marg, one_trip, form, grid, stream, theta, n, k, idx, soft, fin); break;
        case 4: launch_fwd<4>(want_idx, want_soft, want_marg, one_trip, form, grid, stream, theta, n, k, idx, soft, fin); break;
        default: launch_fwd<0>(want_idx, want_soft, want_marg, one_trip, form, grid, stream, theta, n, k, idx, soft, fin); break;
    }
    int rc = check_launch();
    if (rc == CDL_OK && want_marg && form == kMargRows) {
        const int level_blocks = (p.n_levels + 7) / 8;
        const int chunks = 64 / level_blocks < kFinChunks ? (64 / level_blocks > 1 ? 64 / level_blocks : 1) : kFinChunks;
        CDL_LAUNCH("marginal_finalize_kernel", stream, marginal_finalize_kernel, dim3(level_blocks, chunks), dim3(kFinThreads), 0,
                   fin.rows, grid, p.n_levels, fin);
        rc = check_launch();
    }
    return rc;
}

int launch_quantize_bwd(const float *theta, const float *g, int64_t n, const cdl_qparams &p,
                        float *dtheta, float *d_delta, float *d_alpha, void *scalars, hipStream_t stream)
{
    const bool want_scalars = (d_delta != nullptr) || (d_alpha != nullptr);
    if (n == 0) {
        if (want_scalars) {
            CDL_LAUNCH("zero_floats_kernel", stream, zero_floats_kernel, dim3(1), dim3(64), 0, d_delta, d_delta ? 1 : 0,
                               d_alpha, d_alpha ? 1 : 0, (float *)nullptr, 0);
            return check_launch();
        }
        return CDL_OK;
    }
    QConst k = make_const(p);
    k.stream = n >= kStreamFrom;
    const bool one_trip = gradient_one_trip(n, k);
    const int grid = one_trip ? (int)one_trip_grid(n) : want_scalars && band_template(k) != 0 ? finishing_grid(grid_for(n)) : grid_for(n);
    const double d = (double)p.delta;
    ScalarFinish fin{};
    if (want_scalars) fin = scalar_finish_args(scalars, n, grid, 1.0, d * d * d, d_delta, d_alpha);
    const SoftPlan plan = want_scalars && uniform_half_width(p, k) && soft_bwd_from_uniform(p, n) ? soft_plan(p, k, n, true) : SoftPlan{};
    if (plan.bins) {
        const int rc = launch_soft_bwd(theta, g, n, p, k, plan, dtheta, fin, reinterpret_cast<char *>(scalars) + quantize_sum_bytes(n), grid, stream);
        return rc != CDL_OK ? rc : launch_scalar_end(fin, scalars, grid, stream);
    }
    const bool want_dtheta = dtheta != nullptr;
    const int jh = uniform_half_width(p, k);
    if (jh) {
        const UniConst u = make_uniform(p, jh);
        if (jh == 4) launch_bwd_uniform<4>(want_dtheta, want_scalars, grid, stream, theta, g, n, k, u, dtheta, fin);
        else if (jh == 8) launch_bwd_uniform<8>(want_dtheta, want_scalars, grid, stream, theta, g, n, k, u, dtheta, fin);
        else launch_bwd_uniform<16>(want_dtheta, want_scalars, grid, stream, theta, g, n, k, u, dtheta, fin);
    } else
    switch (band_template(k)) {
        case 1: launch_bwd_w<1>(want_dtheta, want_scalars, one_trip, grid, stream, theta, g, n, k, dtheta, fin); break;
        case 2: launch_bwd_w<2>(want_dtheta, want_scalars, one_trip, grid, stream, theta, g, n, k, dtheta, fin); break;
        case 3: launch_bwd_w<3>(want_dtheta, want_scalars, one_trip, grid, stream, theta, g, n, k, dtheta, fin); break;
        case 4: launch_bwd_w<4>(want_dtheta, want_scalars, one_trip, grid, stream, theta, g, n, k, dtheta, fin); break;
        default: launch_bwd_w<0>(want_dtheta, want_scalars, one_trip, grid, stream, theta, g, n, k, dtheta, fin); break;
    }
    return launch_scalar_end(fin, scalars, grid, stream);
}

int launch_quantize_draw(const float *theta, const float *u, int64_t n, const cdl_qparams &p, int8_t *idx, hipStream_t stream)
{
    if (n == 0) return CDL_OK;
    QConst k = make_const(p);
    k.stream = n >= kStreamFrom;
    const bool one_trip = forward_one_trip(n, k, true);      // (two numbers read)
    const int grid = one_trip ? (int)one_trip_grid(n) : grid_for(n);
#define CDL_DRAW(WW) \
    do { \
        constexpr int U = WW > 0 ? kOneTripVectors : 1; \
        if (one_trip) CDL_LAUNCH("quantize_draw_kernel", stream, (quantize_draw_kernel<WW, U>), dim3(grid), dim3(one_trip_threads(U)), 0, theta, u, n, k, idx); \
        else CDL_LAUNCH("quantize_draw_kernel", stream, (quantize_draw_kernel<WW, 1>), dim3(grid), dim3(kQuantThreads), 0, theta, u, n, k, idx); \
    } while (0)
    switch (band_template(k)) {
        case 1: CDL_DRAW(1); break;
        case 2: CDL_DRAW(2); break;
        case 3: CDL_DRAW(3); break;
        case 4: CDL_DRAW(4); break;
        default: CDL_DRAW(0); break;
    }
#undef CDL_DRAW
    return check_launch();
}

namespace {
template <int W>
void launch_entropy_bwd_w(bool want_dtheta, bool want_scalars, bool add, bool one_trip, int grid, hipStream_t s, const float *theta,
                          const float *marg, const float *g_in, int64_t n, const QConst &k, float mul,
                          float *dtheta, const ScalarFinish &fin)
{
    constexpr int U = W > 0 ? kOneTripVectors : 1;
#define CDL_EB(D, S, A) \
    do { \
        if (one_trip) CDL_LAUNCH("entropy_bwd_kernel", s, (entropy_bwd_kernel<W, D, S, A, U>), dim3(grid), dim3(one_trip_threads(U)), 0, \
                                 theta, marg, g_in, n, k, mul, dtheta, fin); \
        else CDL_LAUNCH("entropy_bwd_kernel", s, (entropy_bwd_kernel<W, D, S, A, 1>), dim3(grid), dim3(kQuantThreads), 0, \
                        theta, marg, g_in, n, k, mul, dtheta, fin); \
    } while (0)
    if (want_dtheta && want_scalars && add) CDL_EB(true, true, true);
    else if (want_dtheta && want_scalars) CDL_EB(true, true, false);
    else if (want_dtheta && add) CDL_EB(true, false, true);
    else if (want_dtheta) CDL_EB(true, false, false);
    else CDL_EB(false, true, false);
#undef CDL_EB
}
}  // namespace

int launch_entropy_bwd(const float *theta, const float *marg, const float *g_in, int64_t n, const cdl_qparams &p,
                       float scale, float *dtheta, float *d_delta, float *d_alpha, void *ws, hipStream_t stream)
{
    const bool want_scalars = (d_delta != nullptr) || (d_alpha != nullptr);
    if (n == 0) {
        if (want_scalars) {
            CDL_LAUNCH("zero_floats_kernel", stream, zero_floats_kernel, dim3(1), dim3(64), 0, d_delta, d_delta ? 1 : 0,
                               d_alpha, d_alpha ? 1 : 0, (float *)nullptr, 0);
            return check_launch();
        }
        return CDL_OK;
    }
    QConst k = make_const(p);
    k.stream = n >= kStreamFrom;
    const bool one_trip = entropy_one_trip(n, k, want_scalars, g_in != nullptr);
    const int grid = one_trip ? (int)one_trip_grid(n) : grid_for(n);
    const bool want_dtheta = dtheta != nullptr;
    const double alpha = (double)p.alpha, delta = (double)p.delta;
    const double mul_theta = (double)scale * (-2.0 * alpha * delta / (double)n);
    ScalarFinish fin{};
    void *const scalars = want_scalars ? quantize_scalar_area(ws, n, p.n_levels) : nullptr;
    if (want_scalars) fin = scalar_finish_args(scalars, n, grid, mul_theta, (double)scale * delta * delta / (double)n, d_delta, d_alpha);
    switch (band_template(k)) {
        case 1: launch_entropy_bwd_w<1>(want_dtheta, want_scalars, g_in != nullptr, one_trip, grid, stream, theta, marg, g_in, n, k, (float)mul_theta, dtheta, fin); break;
        case 2: launch_entropy_bwd_w<2>(want_dtheta, want_scalars, g_in != nullptr, one_trip, grid, stream, theta, marg, g_in, n, k, (float)mul_theta, dtheta, fin); break;
        case 3: launch_entropy_bwd_w<3>(want_dtheta, want_scalars, g_in != nullptr, one_trip, grid, stream, theta, marg, g_in, n, k, (float)mul_theta, dtheta, fin); break;
        case 4: launch_entropy_bwd_w<4>(want_dtheta, want_scalars, g_in != nullptr, one_trip, grid, stream, theta, marg, g_in, n, k, (float)mul_theta, dtheta, fin); break;
        default: launch_entropy_bwd_w<0>(want_dtheta, want_scalars, g_in != nullptr, one_trip, grid, stream, theta, marg, g_in, n, k, (float)mul_theta, dtheta, fin); break;
    }
    return launch_scalar_end(fin, scalars, grid, stream);
}

}  // namespace cdl
