// From per-block histograms of the CPMFs to the marginal PMF and its entropy, inside the kernels (not installed).
#pragma once

#include "cdl_finish.h"
#include "cdl_marg_slices.h"

#include <math.h>

#include <type_traits>

namespace cdl {

constexpr int kHistScaleBits = 21;      // a probability p is the integer floor(p * 2^21 + 1/2)

// What becomes of the per-block histograms: the marginal PMF and its entropy.
struct MargFinish {
    unsigned long long *rows;      // [gridDim.x][n_levels], for marginal_finalize_kernel; slices: records, [workers][n_levels padded to fours]
    unsigned long long *records;   // [blocks][n_levels][2]; slices: [kMargCollectors][2]
    unsigned long long tag;
    double inv_n;                  // 1 / (n * 2^s)
    float *marg;                   // [n_levels] or null
    float *entropy_bits;           // [1] or null
    int lg_per;                    // slices of 2^lg_per levels (a multiple of four)
    MargRoles roles;               // slices
};

// How the blocks' histograms are added up: in rows for a second launch, by the last block, by blocks of their own, a slice of the levels each.
enum MargForm { kMargRows = 0, kMargLast = 1, kMargSlices = 2 };

// A record is a 64-bit sum and, as its check word, the sum combined with the tag.
__device__ __forceinline__ void marginal_publish(unsigned long long v, size_t at, const MargFinish &f)
{
    device_store(f.records + 2 * at, v);
    device_store(f.records + 2 * at + 1, v ^ f.tag);
}

// The last block's part, for all its T threads: adds the records of `rows` rows to `own` (thread i < n_levels: the
// block's own sum for level i), normalises by n * 2^s and adds up the entropy terms in a fixed order.  The sums are
// exact 64-bit integers, so their order does not matter.
template <int T, int U>
__device__ __forceinline__ void marginal_collect(unsigned long long own, int rows, int n_levels, const MargFinish &f)
{
    __shared__ unsigned long long red[T];
    if (rows > 0) {
        // threads: `lv` levels (a power of two) times T / lv rows at a time, U records in flight per thread
        int lg = 1;
        while ((1 << lg) < n_levels) ++lg;
        const int lv = 1 << lg, level = (int)threadIdx.x & (lv - 1), sub = (int)threadIdx.x >> lg, subs = T >> lg;
        unsigned long long s = 0ull;
        if (level < n_levels) {
            for (int r = sub; r < rows; r += U * subs) {
                unsigned long long v[U];
                bool waiting = true;
                while (waiting) {
                    unsigned long long c[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        // (past the end: the thread's first record once more)
                        const int row = r + u * subs < rows ? r + u * subs : r;
                        const unsigned long long *q = f.records + 2 * ((size_t)row * n_levels + level);
                        v[u] = device_load(q);
                        c[u] = device_load(q + 1);
                    }
                    waiting = false;
#pragma unroll
                    for (int u = 0; u < U; ++u) waiting = waiting || (v[u] ^ c[u]) != f.tag;
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (r + u * subs < rows) {
                        s += v[u];
                        device_store(f.records + 2 * ((size_t)(r + u * subs) * n_levels + level) + 1, v[u]);
                    }
            }
        }
        red[threadIdx.x] = s;
        __syncthreads();
        if ((int)threadIdx.x < lv)
            for (int q = 0; q < subs; ++q) own += red[q * lv + threadIdx.x];
    }
    double h = 0.0;
    if ((int)threadIdx.x < n_levels) {
        const double m = fmax((double)(long long)own * f.inv_n, 0.0);
        if (f.marg) f.marg[threadIdx.x] = (float)m;
        h = m > 0.0 ? -m * log2(m) : 0.0;
    }
    __shared__ double hs[4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) h += __shfl_down(h, off, 64);
    if ((threadIdx.x & 63) == 0 && threadIdx.x < 256) hs[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0 && f.entropy_bits) *f.entropy_bits = (float)((hs[0] + hs[1]) + (hs[2] + hs[3]));
}

// ---- slices ----
// One block takes 2.5 us for 256 KB of records; here up to sixteen blocks behind those that have entries share them, at the price of one trip more for their entropy terms.  A record
// is four levels' sums of a block, 48 bits with their sign each (a block has at most 2^15 entries of 2^21): three words with a quarter of the
// fourth sum each in their upper bits, and a check word.  Lane 4 i + j holds word j.  (Times of both sides: marg_form.)
// Four neighbouring lanes exchange values (1: lane ^ 1, 2: lane ^ 2, 3: lane 3's).
template <int HOW>
__device__ __forceinline__ int quad_other(int v)
{
    constexpr int ctrl = HOW == 1 ? 0xb1 : HOW == 2 ? 0x4e : 0xff;
    return __builtin_amdgcn_mov_dpp(v, ctrl, 0xf, 0xf, true);
}
template <int HOW>
__device__ __forceinline__ unsigned long long quad_other(unsigned long long v)
{
    return (unsigned long long)(unsigned int)quad_other<HOW>((int)(v >> 32)) << 32 | (unsigned int)quad_other<HOW>((int)v);
}
// the check word's part of word j; the sum over the four lanes is the contents' (products: two words that have changed do not make up for each other)
__device__ __forceinline__ unsigned long long quad_check(unsigned long long word, int j)
{
    const unsigned long long mul = j == 0 ? 0x9E3779B97F4A7C15ull : j == 1 ? 0xBF58476D1CE4E5B9ull : 0x94D049BB133111EBull;
    unsigned long long c = j == 3 ? 0ull : word * mul;
    c += quad_other<1>(c);
    c += quad_other<2>(c);
    return c;
}

// Thread i < n_levels padded to fours: the block's sum of level i (beyond the levels: anything)
__device__ __forceinline__ void row_publish(unsigned long long v, int n_levels, const MargFinish &f)
{
    const int n4 = (n_levels + 3) & ~3, j = (int)threadIdx.x & 3;
    if ((int)threadIdx.x >= n4) return;
    const unsigned long long v3 = quad_other<3>(v);
    const unsigned long long word = (v & 0xffffffffffffull) | (v3 >> (16 * j)) << 48;
    const unsigned long long check = quad_check(word, j) ^ f.tag;
    device_store(f.rows + (size_t)blockIdx.x * n4 + threadIdx.x, j == 3 ? check : word);
}

// The collectors' part, for all T threads of each: collector c adds slice c, of 2^lg_per levels, over the blocks that have entries,
// normalises and leaves its entropy terms to the last one, which adds those up in a fixed order.
template <int T, int U>
__device__ __forceinline__ void rows_collect(int n_levels, const MargFinish &f)
{
    __shared__ unsigned long long red[T];
    __shared__ double hs[T / 64 + kMargCollectors];
    const int lg = f.lg_per, per = 1 << lg, n4 = (n_levels + 3) & ~3, c = f.roles.collector((int)blockIdx.x), terms_from = f.roles.terms_from(c);
    const int local = (int)threadIdx.x & (per - 1), level = (c << lg) + local, sub = (int)threadIdx.x >> lg, subs = T >> lg, j = local & 3;
    const int rows = f.roles.rows_from();
    unsigned long long s = 0ull;
    unsigned long long *const column = f.rows + level;
    auto take = [&](int r, auto count) {      // records r, r + subs, ..
        constexpr int N = decltype(count)::value;
        unsigned long long w[N];
        size_t at[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            // (past the end: the thread's first record once more)
            at[u] = (size_t)(r + u * subs < rows ? r + u * subs : r) * n4;
        }
        bool waiting = true;
        while (waiting) {
#pragma unroll
            for (int u = 0; u < N; ++u) w[u] = device_load(column + at[u]);
            waiting = false;
#pragma unroll
            for (int u = 0; u < N; ++u) waiting = waiting || quad_other<3>((int)((quad_check(w[u], j) ^ f.tag) == w[u])) == 0;
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            unsigned long long top = j == 3 ? 0ull : w[u] >> 48 << (16 * j);      // (of the fourth sum)
            top += quad_other<1>(top);
            top += quad_other<2>(top);
            const unsigned long long v = j == 3 ? top : w[u];
            if (r + u * subs < rows) {
                s += (unsigned long long)((long long)(v << 16) >> 16);
                if (j == 3) device_store(column + at[u], w[u] + 1);      // (spoilt, for a replay)
            }
        }
    };
    if (level < n4) {
        if (rows <= subs) {
            if (sub < rows) take(sub, std::integral_constant<int, 1>{});
        } else {
            for (int r = sub; r < rows; r += U * subs) take(r, std::integral_constant<int, U>{});
        }
    }
    for (int off = 32; off >= per; off >>= 1) s += (unsigned long long)__shfl_xor((long long)s, off, 64);
    red[threadIdx.x] = s;
    __syncthreads();
    double h = 0.0;
    if ((int)threadIdx.x < per && level < n_levels) {
        unsigned long long sum = 0ull;
        const int step = per < 64 ? 64 : per;
        for (int q = local; q < T; q += step) sum += red[q];
        const double m = fmax((double)(long long)sum * f.inv_n, 0.0);
        if (f.marg) f.marg[level] = (float)m;
        h = m > 0.0 ? -m * log2(m) : 0.0;
    }
    if (!f.entropy_bits) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) h += __shfl_down(h, off, 64);
    if ((threadIdx.x & 63) == 0) hs[threadIdx.x >> 6] = h;
    __syncthreads();
    double terms = 0.0;
    if (threadIdx.x == 0)
        for (int q = 0; q < (per + 63) / 64; ++q) terms += hs[q];
    if (c != f.roles.slices - 1) {
        if (threadIdx.x == 0) {
            const unsigned long long bits = (unsigned long long)__double_as_longlong(terms);
            device_store(f.records + 2 * c, bits);
            device_store(f.records + 2 * c + 1, bits ^ f.tag);
        }
        return;
    }
    if ((int)threadIdx.x < terms_from) {
        unsigned long long *const q = f.records + 2 * threadIdx.x;
        unsigned long long v, check;
        do {
            v = device_load(q);
            check = device_load(q + 1);
        } while ((v ^ check) != f.tag);
        device_store(q + 1, v);
        hs[T / 64 + threadIdx.x] = __longlong_as_double((long long)v);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        for (int q = 0; q < terms_from; ++q) sum += hs[T / 64 + q];
        *f.entropy_bits = (float)(sum + terms);
    }
}

// The end of a kernel whose blocks have histograms.
// Thread i < n_levels has the block's sum for level i.
// FORM: a template parameter, since marginal_collect takes a kernel from 31 to 64 registers, the most with which eight waves of it fit a SIMD.
template <int T, int FORM>
__device__ __forceinline__ void marginal_end(unsigned long long own, int n_levels, const MargFinish &f)
{
    if constexpr (FORM == kMargSlices) {
        row_publish(own, n_levels, f);      // (the collectors: at the kernel's start)
    } else if constexpr (FORM == kMargLast) {
        if (blockIdx.x == gridDim.x - 1) marginal_collect<T, 8>(own, (int)blockIdx.x, n_levels, f);
        else if ((int)threadIdx.x < n_levels) marginal_publish(own, (size_t)blockIdx.x * n_levels + threadIdx.x, f);
    } else if ((int)threadIdx.x < n_levels) {
        f.rows[(size_t)blockIdx.x * n_levels + threadIdx.x] = own;
    }
}

}  // namespace cdl
