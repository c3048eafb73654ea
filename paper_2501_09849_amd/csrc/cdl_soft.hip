// Soft regime (few or many levels, most of them live: the paper starts training at alpha = 500, Sec. V-B).
//
// Once the quantizer's parameters are fixed every quantity of an entry is a function of theta alone.  With
// r = theta / delta - c0 (c0 the centre of the level set) and mu(r), var(r), c3(r) the mean, variance and third central moment of
// the level offset under the CPMF,
//     Q_d = delta (c0 + mu),   mu' = 2 kappa var,   var' = 2 kappa c3
// (kappa = alpha delta^2), because a derivative with respect to r brings down a cumulant of the CPMF and a factor 2 kappa.  All
// three are analytic with features no finer than the CPMF's own width sigma = 1 / sqrt(2 kappa), so one polynomial per interval
// of an eighth of sigma replaces the loop over the levels: a gather from LDS and 27 fused multiply-adds in double per entry where 31
// levels took 250 instructions.
//
// The polynomial is made from its highest derivative: c3 at eight Chebyshev nodes and mu, var at the middle of the interval are sums
// over the levels, and mu(t) is the second integral of the interpolated c3 (ninth degree).  Integration makes errors smaller
// where differentiation multiplies them by 1 / (kappa h) each time: from an interpolated mean the third moment had 3e-8 of its size,
// and no digit right where kappa is 1e-8.  So made, every coefficient has the relative precision of a double however small kappa
// is, and mu, var and 2 (r - mu) var - c3 come out within 1e-15, 7e-15 and 2e-13 of their largest value (6 - 33 levels, kappa 1e-12
// to 1.2, against sums in 80 bits; the loop over the levels: 3e-15, 4e-13, 2e-11).
// The table is made by a kernel of its own.
//
// Marginal PMF: the sum of P_k(r) over the entries is wanted for every level k.  An entry adds the Chebyshev polynomials
// T_0 .. T_6 of its place in its interval to seven cells of a histogram; since on an interval P_k = sum_m c_km T_m up to 6e-13 of
// its peak, the sums over the entries follow from the cells - at the end, once per interval and level.  The terms are doubles in
// fixed point (LDS integer atomics, 2^-44, cells of 64 bits: 8.4 lane updates per clock and CU against 12.4 of 32 bits), so that
// their rounding stays below the interpolation's error also where every entry is the same and nothing averages out.  (Six terms
// in fp32, rounded to 2^-18, on intervals twice as long: 7e-8 of a probability there.)
//
// That is for the sets that the kernels on a common centre serve otherwise, whose arithmetic is double too.  The forward pass of
// the sets that only the loop in fp32 would serve takes intervals twice as long and six moments (mu 5e-15, marginal PMF 3e-9).
//
// 25.6 M entries, 31 levels at the initial sharpness: forward 98 us, backward 88 (2.3 and 3.5 TB/s; LDS atomics 35 us and gathers of
// 80 bytes an entry 26 us on the LDS pipe, 61 us of memory traffic at the copy rate), both together 187 where the loop over the
// levels takes 403.
//
// Entries beyond the table's range (theta more than twice as far out as the last level) are evaluated one by one as the
// other kernels do, and add their probabilities to a histogram of levels.
#include "cdl_internal.h"
#include "cdl_soft.h"

#include <math.h>

namespace cdl {

namespace {

constexpr int kSoftBwdThreads = 256;
// An entry adds rint(T_m * 2^b) to a cell, with b as large as keeps a block's sums below 2^62 (44 up to 2^26 entries, then one less for
// every doubling).  magic = 1.5 * 2^(52 - b): T_m + magic has a spacing of 2^-b, so its bits are those of magic plus that integer;
// what the constant adds is taken off at the end, with the count T_0.
constexpr int kSoftMostBits = 44;
constexpr int kSoftFinBlocks = 64;
constexpr int kNodes = 8;                   // Chebyshev nodes of an interval, for c3
constexpr int kCoefs = kSoftCoefs;          // coefficients of t^q in mu, t in [-1, 1] along the interval
static_assert(kCoefs == kNodes + 2 && kCoefs % 2 == 0, "two integrations; pairs of coefficients are loaded");

struct SoftConst {
    int bins, copies, lg_copies, n_levels, small_set;
    int hist_copies, lg_hist_copies;
    double half_range, inv_h, c0, inv_delta, delta, kappa;
    double r_safe;
    double lo_off;         // offset of the lowest level from the centre
    double scale, magic;   // 2^b, 1.5 * 2^(52 - b) (forward)
};

// ---- the table: [bins][kCoefs] ----

// Chebyshev nodes, values there -> coefficients of the T_m, and the coefficients of t^q in T_m.  (Two steps: the product of the two
// matrices has entries of several hundred, which the roundings of the values would be multiplied by.)
struct NodeMatrix { double node[kNodes], cheb[kNodes][kNodes], power[kNodes][kNodes]; };

constexpr int kTableThreads = 128;          // eight threads to a node; node kNodes is the middle of the interval

__global__ __launch_bounds__(kTableThreads)
void soft_table_kernel(SoftConst s, NodeMatrix m, double *__restrict__ table)
{
    __shared__ double c3[kNodes], cheb[kNodes], mid[2];
    const int bin = blockIdx.x, node = threadIdx.x >> 3, part = threadIdx.x & 7;
    const double x = node < kNodes ? m.node[node] : 0.0;
    const double r = -s.half_range + (bin + 0.5 * (1.0 + x)) / s.inv_h;
    // offsets from the nearest level, so that the largest weight is about one
    const double near = fmin(fmax(rint(r - s.lo_off), 0.0), (double)(s.n_levels - 1)) + s.lo_off, d0 = r - near;
    auto weight = [&](int k, double &j) {
        j = s.lo_off + k - near;
        return exp(s.kappa * j * (2.0 * d0 - j));
    };
    auto add8 = [](double &v) {
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    };
    // (a level j away from the nearest one weighs at most exp(-kappa j^2): the others are below 3e-20 of it)
    const double band = ceil(sqrt(45.0 / s.kappa)), at = near - s.lo_off;
    const int first = (int)fmax(0.0, at - band), last = (int)fmin((double)(s.n_levels - 1), at + band);
    double Z = 0.0, S = 0.0, j;
    for (int k = first + part; k <= last; k += 8) {
        const double w = weight(k, j);
        Z += w;
        S = fma(j, w, S);
    }
    add8(Z);
    add8(S);
    const double mean = S / Z;
    double V = 0.0, T = 0.0;
    for (int k = first + part; k <= last; k += 8) {
        const double w = weight(k, j), d = j - mean, dw = d * w;
        V = fma(d, dw, V);
        T = fma(d * d, dw, T);
    }
    add8(V);
    add8(T);
    if (part == 0) {
        if (node < kNodes) c3[node] = T / Z;
        else if (node == kNodes) { mid[0] = near + mean; mid[1] = V / Z; }
    }
    __syncthreads();
    const int q = threadIdx.x;
    if (q < kNodes) {
        double a = 0.0;
#pragma unroll
        for (int i = 0; i < kNodes; ++i) a = fma(m.cheb[q][i], c3[i], a);
        cheb[q] = a;
    }
    __syncthreads();
    const double kh = s.kappa / s.inv_h;        // d var / dt = kappa h c3, d mu / dt = kappa h var
    double *out = table + (size_t)bin * kCoefs;
    if (q < kNodes) {
        double c = 0.0;
#pragma unroll
        for (int a = 0; a < kNodes; ++a) c = fma(m.power[a][q], cheb[a], c);
        out[q + 2] = kh * (kh * c) / (double)((q + 1) * (q + 2));
    } else if (q < kCoefs) {
        out[q - kNodes] = q == kNodes ? mid[0] : kh * mid[1];
    }
}

// The table in LDS as arrays of 16 bytes per interval (two coefficients each), every array in `copies` copies side by
// side: the copy is the group of banks, so that the lanes of a gather, each in its own interval, do not meet.
template <int T>
__device__ __forceinline__ void load_table(const SoftConst &s, const double *__restrict__ table, uint4 *lds)
{
    const uint4 *d = reinterpret_cast<const uint4 *>(table);
    for (int i = threadIdx.x; i < s.bins << s.lg_copies; i += T) {
        const int b = i >> s.lg_copies;
#pragma unroll
        for (int q = 0; q < kCoefs / 2; ++q) lds[q * (s.bins << s.lg_copies) + i] = d[b * (kCoefs / 2) + q];
    }
}

struct SoftPlace { int bin; double t; bool in; };
__device__ __forceinline__ SoftPlace soft_place(double r, const SoftConst &s)
{
    SoftPlace p;
    p.in = fabs(r) <= s.half_range;
    const double x = fmin(fmax((r + s.half_range) * s.inv_h, 0.0), (double)s.bins);
    p.bin = min((int)x, s.bins - 1);
    p.t = fma(2.0, x - (double)p.bin, -1.0);
    return p;
}

struct SoftCoef { double c[kCoefs]; };
__device__ __forceinline__ SoftCoef soft_coef(int bin, const SoftConst &s, const uint4 *lds)
{
    const int at = (bin << s.lg_copies) + ((int)threadIdx.x & (s.copies - 1)), plane = s.bins << s.lg_copies;
    SoftCoef q;
#pragma unroll
    for (int i = 0; i < kCoefs / 2; ++i) {
        const double2 v = *reinterpret_cast<const double2 *>(lds + i * plane + at);
        q.c[2 * i] = v.x;
        q.c[2 * i + 1] = v.y;
    }
    return q;
}

// Sums over all levels in double, for entries outside the table (at most 33 levels), with offsets from the nearest level.
// r is held at +-r_safe, where the CPMF is one level to 1e-13 (theta may be infinite).
struct SoftSums { double near, d0, Z, S1, S2, S3; };
__device__ __forceinline__ double soft_clamp(double r, const SoftConst &s) { return fmin(fmax(r, -s.r_safe), s.r_safe); }
__device__ __forceinline__ SoftSums soft_direct(double r, const SoftConst &s)
{
    const double near = fmin(fmax(rint(r - s.lo_off), 0.0), (double)(s.n_levels - 1)) + s.lo_off;
    SoftSums q{near, r - near, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int k = 0; k < s.n_levels; ++k) {
        const double j = s.lo_off + k - near, w = exp(s.kappa * j * (2.0 * q.d0 - j));
        q.Z += w;
        q.S1 = fma(j, w, q.S1);
        q.S2 = fma(j * j, w, q.S2);
        q.S3 = fma(j * j * j, w, q.S3);
    }
    return q;
}

// ---- forward ----
// One block of 1024 threads per compute unit.  LDS: [table][levels][cells: (M bins) x hist_copies].  A cell lies in the bank
// group of its copy, as in the other histogram kernels.
template <int M, bool IDX, bool SOFT>
__global__ __launch_bounds__(kSoftThreads)
void soft_fwd_kernel(const float *__restrict__ theta, int64_t n, QConst k, SoftConst s, const double *__restrict__ table,
                     int8_t *__restrict__ idx, float *__restrict__ soft, long long *__restrict__ rows /* [gridDim.x][M bins + levels] */)
{
    extern __shared__ __attribute__((aligned(16))) uint4 soft_lds[];
    unsigned long long *levels = reinterpret_cast<unsigned long long *>(soft_lds + kCoefs / 2 * (s.bins << s.lg_copies));
    unsigned long long *cells = levels + s.n_levels;
    const int n_cells = M * s.bins;
    load_table<kSoftThreads>(s, table, soft_lds);
    for (int i = threadIdx.x; i < n_cells << s.lg_hist_copies; i += kSoftThreads) cells[i] = 0ull;
    if ((int)threadIdx.x < s.n_levels) levels[threadIdx.x] = 0ull;
    __syncthreads();
    unsigned long long *mine = cells + ((int)threadIdx.x & (s.hist_copies - 1));

    // true: done; false: an entry beyond the table
    auto inside = [&](float th, float &sv) -> bool {
        const double r = fma((double)th, s.inv_delta, -s.c0);
        const SoftPlace p = soft_place(r, s);
        if (p.in) {
            if (SOFT) {
                const SoftCoef q = soft_coef(p.bin, s, soft_lds);
                double mu = q.c[kCoefs - 1];
#pragma unroll
                for (int i = kCoefs - 2; i >= 0; --i) mu = fma(mu, p.t, q.c[i]);
                sv = (float)(s.delta * (s.c0 + mu));
            }
            unsigned long long *c = mine + ((M * p.bin) << s.lg_hist_copies);
            atomicAdd(c, 1ull);
            double before = 1.0, now = p.t;
#pragma unroll
            for (int m = 1; m < M; ++m) {
                c += s.hist_copies;
                atomicAdd(c, (unsigned long long)__double_as_longlong(now + s.magic));
                const double next = fma(2.0 * p.t, now, -before);
                before = now;
                now = next;
            }
        }
        return p.in;
    };
    auto outside = [&](float th) -> float {
        if (s.small_set) {
            const double r = soft_clamp(fma((double)th, s.inv_delta, -s.c0), s);
            const SoftSums q = soft_direct(r, s);
            const double scale = s.scale / q.Z;
#pragma unroll 1
            for (int l = 0; l < s.n_levels; ++l) {
                const double j = s.lo_off + l - q.near;
                atomicAdd(levels + l, (unsigned long long)rint(exp(s.kappa * j * (2.0 * q.d0 - j)) * scale));
            }
            return (float)(s.delta * (s.c0 + q.near + q.S1 / q.Z));
        }
        GenericSums q;
        generic_sums<IDX>(th, k, q);
        const float inv = fast_rcp(q.Z), two_u = 2.0f * q.u, scale = inv * (float)s.scale;
#pragma unroll 1
        for (int j = q.jlo; j <= q.jhi; ++j)
            atomicAdd(levels + ((int)q.cf - k.lo + j), (unsigned long long)rintf(generic_weight(j, two_u, k) * scale));
        return fmaf(q.S1 * inv, k.delta, q.cf * k.delta);
    };

    const int64_t n4 = n >> 2, stride = (int64_t)gridDim.x * kSoftThreads;
    int64_t v = (int64_t)blockIdx.x * kSoftThreads + threadIdx.x;
    float4 ahead = {0.0f, 0.0f, 0.0f, 0.0f};
    if (v < n4) ahead = load_stream4(theta + 4 * v, k.stream);
    for (int64_t base = (int64_t)blockIdx.x * kSoftThreads; base < n4; base += stride, v += stride) {
        const float th[4] = {ahead.x, ahead.y, ahead.z, ahead.w};
        if (v + stride < n4) ahead = load_stream4(theta + 4 * (v + stride), k.stream);
        if (v < n4) {
            float sv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            bool in[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) in[e] = inside(th[e], sv[e]);
            if (!(in[0] && in[1] && in[2] && in[3])) {
#pragma unroll 1
                for (int e = 0; e < 4; ++e) {
                    if (e == 0 ? in[0] : (e == 1 ? in[1] : (e == 2 ? in[2] : in[3]))) continue;
                    const float sv_e = outside(e == 0 ? th[0] : (e == 1 ? th[1] : (e == 2 ? th[2] : th[3])));
                    sv[0] = e == 0 ? sv_e : sv[0]; sv[1] = e == 1 ? sv_e : sv[1];
                    sv[2] = e == 2 ? sv_e : sv[2]; sv[3] = e == 3 ? sv_e : sv[3];
                }
            }
            if (SOFT) store_stream4(soft + 4 * v, sv[0], sv[1], sv[2], sv[3], k.stream);
            if (IDX) {
                int ci[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) ci[e] = (int)anchor_level<true>(th[e], k);
                reinterpret_cast<uint32_t *>(idx)[v] = pack_indices(ci[0], ci[1], ci[2], ci[3], k.idx_off);
            }
        }
    }
    // ragged tail: the last 1..3 entries
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        for (int64_t e = n4 << 2; e < n; ++e) {
            float sv = 0.0f;
            if (!inside(theta[e], sv)) sv = outside(theta[e]);
            if (SOFT) soft[e] = sv;
            if (IDX) idx[e] = (int8_t)((int)anchor_level<true>(theta[e], k) - k.idx_off);
        }
    __syncthreads();
    long long *row = rows + (size_t)blockIdx.x * (n_cells + s.n_levels);
    auto cell_sum = [&](int i) {
        unsigned long long v = 0ull;
        for (int j = 0; j < s.hist_copies; ++j) v += cells[(i << s.lg_hist_copies) + ((j + i) & (s.hist_copies - 1))];
        return v;
    };
    for (int i = threadIdx.x; i < n_cells; i += kSoftThreads) {
        const int m = i % M;
        unsigned long long v = cell_sum(i);
        if (m) v -= cell_sum(i - m) * (unsigned long long)__double_as_longlong(s.magic);
        row[i] = (long long)v;
    }
    if ((int)threadIdx.x < s.n_levels) row[n_cells + threadIdx.x] = (long long)levels[threadIdx.x];
}

// From the moments to the marginal PMF.  Block b takes the intervals [b bins / B, (b + 1) bins / B): adds the rows' cells,
// turns the M moments S_m of an interval into weights of its M Chebyshev nodes x_q (the discrete orthogonality of the T_m:
// w_q = (S_0 + 2 sum_m S_m T_m(x_q)) / M gives sum_q w_q f(x_q) = the sum of f over the entries for every polynomial f of
// degree M - 1), and adds w_q P_k(x_q) for all levels k.  The rows' integers are added up as doubles, in a fixed order.
constexpr int kSoftFinThreads = 1024;
constexpr int kFinCells = 64;                               // at least the cells of a block
static_assert(kSoftMoments * ((kSoftMaxBins + kSoftFinBlocks - 1) / kSoftFinBlocks) <= kFinCells &&
              kSoftMoreMoments * ((kSoftMoreBins + kSoftFinBlocks - 1) / kSoftFinBlocks) <= kFinCells, "cells of a block");
struct NodePlace { double x[kSoftMoreMoments]; };

template <int M>
__global__ __launch_bounds__(kSoftFinThreads)
void soft_marginal_kernel(const long long *__restrict__ rows, int n_rows, SoftConst s, NodePlace nodes, MargFinish fin)
{
    __shared__ double part[kSoftFinThreads];
    __shared__ double red[kSoftFinThreads];
    __shared__ double sums[kFinCells];
    __shared__ double weight[kFinCells], place[kFinCells], from[kFinCells];
    const int tid = threadIdx.x, n_cells = M * s.bins, row = n_cells + s.n_levels;
    const int b0 = (int)((int64_t)blockIdx.x * s.bins / gridDim.x), b1 = (int)((int64_t)(blockIdx.x + 1) * s.bins / gridDim.x);
    const int cells = M * (b1 - b0);
    {
        constexpr int kSubs = kSoftFinThreads / kFinCells;
        const int c = tid & (kFinCells - 1), sub = tid / kFinCells;
        double v = 0.0;
        if (c < cells) {
#pragma unroll 16
            for (int r = sub; r < n_rows; r += kSubs) v += (double)rows[(size_t)r * row + M * b0 + c];
        }
        part[tid] = v;
        __syncthreads();
        if (tid < kFinCells) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < kSubs; ++q) t += part[q * kFinCells + tid];
            sums[tid] = tid % M ? t : t * s.scale;      // (T_0 is counted in ones)
        }
        __syncthreads();
    }
    // eight threads to a node for the normaliser
    {
        const int node = tid >> 3, lane8 = tid & 7;
        const int i = node / M, q = node % M;
        const double x = nodes.x[q];
        const double r = -s.half_range + (b0 + i + 0.5 * (1.0 + x)) / s.inv_h;
        const double near = fmin(fmax(rint(r - s.lo_off), 0.0), (double)(s.n_levels - 1)) + s.lo_off, d0 = r - near;
        double Z = 0.0;
        if (node < cells)
            for (int l = lane8; l < s.n_levels; l += 8) {
                const double d = r - (s.lo_off + l);
                Z += exp(s.kappa * (d0 * d0 - d * d));
            }
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) Z += __shfl_xor(Z, off, 64);
        if (node < cells && lane8 == 0) {
            double w = 0.5 * sums[M * i], before = 1.0, now = x;
#pragma unroll
            for (int m = 1; m < M; ++m) {
                w = fma(sums[M * i + m], now, w);
                const double next = fma(2.0 * x, now, -before);
                before = now;
                now = next;
            }
            weight[node] = w * (2.0 / M) / Z;
            place[node] = r;
            from[node] = d0 * d0;
        }
    }
    __syncthreads();
    // level x part of the nodes
    int lg = 3;
    while ((1 << lg) < s.n_levels) ++lg;
    const int level = tid & ((1 << lg) - 1), sub = tid >> lg, subs = kSoftFinThreads >> lg;
    double m = 0.0;
    if (level < s.n_levels) {
        const double o = s.lo_off + level;
        for (int node = sub; node < cells; node += subs) {
            const double d = place[node] - o;
            m = fma(weight[node], exp(s.kappa * (from[node] - d * d)), m);
        }
    }
    red[tid] = m;
    __syncthreads();
    unsigned long long own = 0ull;
    if (tid < s.n_levels) {
        double t = 0.0;
        for (int q = 0; q < subs; ++q) t += red[(q << lg) + tid];
#pragma unroll 4
        for (int r = blockIdx.x; r < n_rows; r += gridDim.x) t += (double)rows[(size_t)r * row + n_cells + tid];
        own = (unsigned long long)__double2ll_rn(t * ((double)(1 << kHistScaleBits) / s.scale));
    }
    if (blockIdx.x != gridDim.x - 1) {
        if (tid < s.n_levels) marginal_publish(own, (size_t)blockIdx.x * s.n_levels + tid, fin);
    } else {
        marginal_collect<kSoftFinThreads, 8>(own, (int)gridDim.x - 1, s.n_levels, fin);
    }
}

// ---- backward ----
template <bool DTHETA>
__global__ __launch_bounds__(kSoftBwdThreads, 5)
void soft_bwd_kernel(const float *__restrict__ theta, const float *g, int64_t n, QConst k, SoftConst s, const double *__restrict__ table,
                     float *dtheta /* may be g */, ScalarFinish fin)
{
    extern __shared__ __attribute__((aligned(16))) uint4 soft_lds[];
    load_table<kSoftBwdThreads>(s, table, soft_lds);
    __syncthreads();
    const double to_var = s.inv_h / s.kappa, to_c3 = 2.0 * to_var * to_var, two_inv_h = 2.0 * s.inv_h;
    double acc_d = 0.0, acc_a = 0.0;
    auto terms = [&](double r, double gd, double mu, double two_kappa_var, double var, double c3) -> float {
        acc_d = fma(gd, (s.c0 + mu) + 2.0 * s.kappa * fma(r - s.c0 - 2.0 * mu, var, -c3), acc_d);
        acc_a = fma(gd, fma(2.0 * (r - mu), var, -c3), acc_a);
        return (float)(gd * two_kappa_var);
    };
    // true: done; false: an entry beyond the table
    auto inside = [&](float th, float ge, float &dv) -> bool {
        const double r = fma((double)th, s.inv_delta, -s.c0);
        const SoftPlace pl = soft_place(r, s);
        if (pl.in) {
            const SoftCoef q = soft_coef(pl.bin, s, soft_lds);
            double p = q.c[kCoefs - 1], p1 = 0.0, p2 = 0.0;      // the polynomial, its derivative, half its second derivative
#pragma unroll
            for (int i = kCoefs - 2; i >= 0; --i) {
                p2 = fma(p2, pl.t, p1);
                p1 = fma(p1, pl.t, p);
                p = fma(p, pl.t, q.c[i]);
            }
            dv = terms(r, (double)ge, p, p1 * two_inv_h, p1 * to_var, p2 * to_c3);
        }
        return pl.in;
    };
    auto outside = [&](float th, float ge) -> float {
        if (s.small_set) {
            const double r = soft_clamp(fma((double)th, s.inv_delta, -s.c0), s);
            const SoftSums q = soft_direct(r, s);
            const double inv = 1.0 / q.Z, m1 = q.S1 * inv, m2 = q.S2 * inv, var = fma(-m1, m1, m2);
            return terms(r, (double)ge, q.near + m1, 2.0 * s.kappa * var, var, fma(-m1, fma(-2.0 * m1, m1, 3.0 * m2), q.S3 * inv));
        }
        float d_th, t_d, t_a;
        quantizer_bwd_terms<0, true>(th, k, d_th, t_d, t_a);
        acc_d += (double)(ge * t_d);
        acc_a += (double)(ge * t_a);
        return ge * d_th;
    };
    const int64_t n4 = n >> 2, stride = (int64_t)gridDim.x * kSoftBwdThreads;
    for (int64_t v = (int64_t)blockIdx.x * kSoftBwdThreads + threadIdx.x; v < n4; v += stride) {
        const float4 t = load_stream4(theta + 4 * v, k.stream), q = load_stream4(g + 4 * v, k.stream);
        const float th[4] = {t.x, t.y, t.z, t.w}, ge[4] = {q.x, q.y, q.z, q.w};
        float dv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        bool in[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) in[e] = inside(th[e], ge[e], dv[e]);
        if (!(in[0] && in[1] && in[2] && in[3])) {
#pragma unroll 1
            for (int e = 0; e < 4; ++e) {
                if (e == 0 ? in[0] : (e == 1 ? in[1] : (e == 2 ? in[2] : in[3]))) continue;
                const float dv_e = outside(e == 0 ? th[0] : (e == 1 ? th[1] : (e == 2 ? th[2] : th[3])), e == 0 ? ge[0] : (e == 1 ? ge[1] : (e == 2 ? ge[2] : ge[3])));
                dv[0] = e == 0 ? dv_e : dv[0]; dv[1] = e == 1 ? dv_e : dv[1];
                dv[2] = e == 2 ? dv_e : dv[2]; dv[3] = e == 3 ? dv_e : dv[3];
            }
        }
        if (DTHETA) store_stream4(dtheta + 4 * v, dv[0], dv[1], dv[2], dv[3], k.stream);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        for (int64_t e = n4 << 2; e < n; ++e) {
            float dv;
            if (!inside(theta[e], g[e], dv)) dv = outside(theta[e], g[e]);
            if (DTHETA) dtheta[e] = dv;
        }
    scalar_finish<kSoftBwdThreads>(acc_d, acc_a, fin);
}

SoftConst soft_const(const cdl_qparams &p, const SoftPlan &s)
{
    SoftConst c{};
    c.bins = s.bins; c.n_levels = p.n_levels; c.small_set = s.small_set;
    c.half_range = s.half_range; c.inv_h = s.inv_h; c.c0 = s.c0; c.inv_delta = s.inv_delta; c.delta = s.delta; c.kappa = s.kappa;
    c.r_safe = (double)p.n_levels + 15.0 / s.kappa;
    c.lo_off = -0.5 * (double)(p.n_levels - 1);
    return c;
}

// copies of the table and of the cells that fit `bytes` of LDS (powers of two, up to 8 and 32)
void soft_copies(SoftConst &c, size_t table_bytes, int moments, size_t hist_bytes)
{
    c.lg_copies = 0;
    while (c.lg_copies < 3 && ((size_t)c.bins * kSoftBinBytes << (c.lg_copies + 1)) <= table_bytes) ++c.lg_copies;
    c.copies = 1 << c.lg_copies;
    c.lg_hist_copies = 0;
    while (c.lg_hist_copies < 5 && ((size_t)c.bins * moments * sizeof(long long) << (c.lg_hist_copies + 1)) <= hist_bytes) ++c.lg_hist_copies;
    c.hist_copies = 1 << c.lg_hist_copies;
}

int launch_table(const SoftConst &c, void *table, hipStream_t stream)
{
    // with f = sum_m a_m T_m, a_m = (2 - [m = 0]) / kNodes sum_i f(x_i) T_m(x_i); the coefficients of T_m from its recurrence
    static const NodeMatrix m = [] {
        NodeMatrix m{};
        m.power[0][0] = 1.0;
        m.power[1][1] = 1.0;
        for (int a = 2; a < kNodes; ++a)
            for (int q = 0; q < kNodes; ++q) m.power[a][q] = (q > 0 ? 2.0 * m.power[a - 1][q - 1] : 0.0) - m.power[a - 2][q];
        for (int i = 0; i < kNodes; ++i) {
            const double angle = (2 * i + 1) * 3.14159265358979323846 / (2 * kNodes);
            m.node[i] = cos(angle);
            for (int a = 0; a < kNodes; ++a) m.cheb[a][i] = (a == 0 ? 1.0 : 2.0) / kNodes * cos(a * angle);
        }
        return m;
    }();
    CDL_LAUNCH("soft_table_kernel", stream, soft_table_kernel, dim3((unsigned)c.bins), dim3(kTableThreads), 0, c, m, reinterpret_cast<double *>(table));
    return check_launch();
}

NodePlace marginal_nodes(int moments)
{
    NodePlace p{};
    for (int q = 0; q < moments; ++q) p.x[q] = cos((2 * q + 1) * 3.14159265358979323846 / (2 * moments));
    return p;
}

template <int M>
int launch_soft_fwd_m(const float *theta, int64_t n, const QConst &k, SoftConst c, int8_t *idx, float *soft, const MargFinish &fin, void *ws,
                      hipStream_t stream)
{
    // one block per compute unit: the table up to 28 KB (one copy of the largest: 48), the levels' cells, and the cells in what is left
    soft_copies(c, 28 << 10, M, (160 << 10) - 2048 - (c.bins * kSoftBinBytes > (28 << 10) ? c.bins * kSoftBinBytes : 28 << 10));
    const int64_t grid = soft_fwd_grid(n);
    const int64_t per_block = ((n >> 2) + grid * kSoftThreads) / (grid * kSoftThreads) * (4 * kSoftThreads) + 3;
    int bits = kSoftMostBits;
    while (bits > 20 && per_block > 1ll << (62 - bits)) --bits;
    c.scale = (double)(1ll << bits);
    c.magic = 1.5 * (double)(1ll << (52 - bits));
    long long *rows = reinterpret_cast<long long *>(reinterpret_cast<char *>(ws) + kSoftTableBytes);
    const double *table = reinterpret_cast<const double *>(ws);
    const size_t lds = ((size_t)c.bins * kSoftBinBytes << c.lg_copies) + (size_t)c.n_levels * sizeof(long long) + ((size_t)c.bins * M * sizeof(long long) << c.lg_hist_copies);
    const char *name = soft || idx ? "quantize_fwd_kernel" : "quantize_fwd_kernel(marginal only)";
#define CDL_SOFT(I, S) \
    do { \
        if (lds > 65536) { \
            const hipError_t e_ = hipFuncSetAttribute((const void *)soft_fwd_kernel<M, I, S>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
            if (e_ != hipSuccess) return hip_failed(e_); \
        } \
        CDL_LAUNCH(name, stream, (soft_fwd_kernel<M, I, S>), dim3((unsigned)grid), dim3(kSoftThreads), lds, theta, n, k, c, table, idx, soft, rows); \
    } while (0)
    if (idx && soft) CDL_SOFT(true, true);
    else if (idx) CDL_SOFT(true, false);
    else if (soft) CDL_SOFT(false, true);
    else CDL_SOFT(false, false);
#undef CDL_SOFT
    const int rc = check_launch();
    if (rc != CDL_OK) return rc;
    static const NodePlace nodes = marginal_nodes(M);
    CDL_LAUNCH("marginal_finalize_kernel", stream, soft_marginal_kernel<M>, dim3(kSoftFinBlocks), dim3(kSoftFinThreads), 0, rows, (int)grid, c, nodes, fin);
    return check_launch();
}

}  // namespace

// One block per compute unit, at least two trips of the loop each
int64_t soft_fwd_grid(int64_t n)
{
    int64_t g = ((n >> 2) + 2 * kSoftThreads - 1) / (2 * kSoftThreads);
    if (g > 256) g = 256;
    return g < 1 ? 1 : g;
}

size_t soft_fwd_bytes(int64_t n, int32_t) { return kSoftTableBytes + (size_t)soft_fwd_grid(n) * kSoftRowWords * sizeof(long long); }

SoftPlan soft_plan(const cdl_qparams &p, const QConst &k, int64_t n, bool fine)
{
    SoftPlan s{};
    // (the other kernels: truncated CPMFs, sharp regimes, small tensors)
    if (k.slide || band_template(k) != 0 || p.n_levels < 6 || n < kSoftFrom) return s;
    const double delta = (double)p.delta, kappa = (double)p.alpha * delta * delta, sigma = 1.0 / sqrt(2.0 * kappa);
    s.small_set = p.n_levels <= 33;
    s.half_range = (double)(p.n_levels - 1) + 4.0;
    s.fine = fine;
    const double width = (fine ? 0.125 : 0.25) * sigma, most = 0.5 * width * (fine ? kSoftMoreBins : kSoftMaxBins);
    if (most < 0.75 * (double)(p.n_levels - 1) + 4.0) return s;      // a band much narrower than the set: the loop over the band
    if (s.half_range > most) s.half_range = most;
    // at least eight intervals: entries then spread over the banks
    s.bins = (int)ceil(2.0 * s.half_range / width);
    if (s.bins < 8) s.bins = 8;
    if (s.bins > (fine ? kSoftMoreBins : kSoftMaxBins)) s.bins = fine ? kSoftMoreBins : kSoftMaxBins;
    s.inv_h = s.bins / (2.0 * s.half_range);
    s.c0 = (double)p.lo + 0.5 * (double)(p.n_levels - 1);
    s.delta = delta;
    s.inv_delta = 1.0 / delta;
    s.kappa = kappa;
    return s;
}

int launch_soft_fwd(const float *theta, int64_t n, const cdl_qparams &p, const QConst &k, const SoftPlan &s, int8_t *idx, float *soft,
                    const MargFinish &fin, void *ws, hipStream_t stream)
{
    const SoftConst c = soft_const(p, s);
    const int rc = launch_table(c, ws, stream);
    if (rc != CDL_OK) return rc;
    return s.fine ? launch_soft_fwd_m<kSoftMoreMoments>(theta, n, k, c, idx, soft, fin, ws, stream)
                                   : launch_soft_fwd_m<kSoftMoments>(theta, n, k, c, idx, soft, fin, ws, stream);
}

int launch_soft_bwd(const float *theta, const float *g, int64_t n, const cdl_qparams &p, const QConst &k, const SoftPlan &s, float *dtheta,
                    const ScalarFinish &fin, void *table, int grid, hipStream_t stream)
{
    SoftConst c = soft_const(p, s);
    soft_copies(c, 28 << 10, 1, 0);
    int rc = launch_table(c, table, stream);
    if (rc != CDL_OK) return rc;
    const size_t lds = (size_t)c.bins * kSoftBinBytes << c.lg_copies;
    if (dtheta) CDL_LAUNCH("quantize_bwd_kernel", stream, soft_bwd_kernel<true>, dim3((unsigned)grid), dim3(kSoftBwdThreads), lds, theta, g, n, k, c,
                           reinterpret_cast<const double *>(table), dtheta, fin);
    else CDL_LAUNCH("quantize_bwd_kernel", stream, soft_bwd_kernel<false>, dim3((unsigned)grid), dim3(kSoftBwdThreads), lds, theta, g, n, k, c,
                    reinterpret_cast<const double *>(table), dtheta, fin);
    return check_launch();
}

}  // namespace cdl
