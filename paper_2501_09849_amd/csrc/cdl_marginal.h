// From per-block histograms of the CPMFs to the marginal PMF and its entropy, inside the kernels (not installed).
#pragma once

#include "cdl_finish.h"

#include <math.h>

namespace cdl {

constexpr int kHistScaleBits = 21;      // a probability p is the integer floor(p * 2^21 + 1/2)

// What becomes of the per-block histograms: the marginal PMF and its entropy.
struct MargFinish {
    unsigned long long *rows;      // [gridDim.x][n_levels]: left there for marginal_finalize_kernel; null: finished in the kernel
    unsigned long long *records;   // [blocks][n_levels][2]
    unsigned long long tag;
    double inv_n;                  // 1 / (n * 2^s)
    float *marg;                   // [n_levels] or null
    float *entropy_bits;           // [1] or null
};

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

// The end of a kernel whose blocks have histograms.
// Thread i < n_levels has the block's sum for level i.
// FEW: the last block finishes (a template parameter: marginal_collect takes a kernel from 31 to 64
// registers, the most with which eight waves of it fit a SIMD).
template <int T, bool FEW>
__device__ __forceinline__ void marginal_end(unsigned long long own, int n_levels, const MargFinish &f)
{
    if (FEW) {
        if (blockIdx.x == gridDim.x - 1) marginal_collect<T, 8>(own, (int)blockIdx.x, n_levels, f);
        else if ((int)threadIdx.x < n_levels) marginal_publish(own, (size_t)blockIdx.x * n_levels + threadIdx.x, f);
    } else if ((int)threadIdx.x < n_levels) {
        f.rows[(size_t)blockIdx.x * n_levels + threadIdx.x] = own;
    }
}

}  // namespace cdl
