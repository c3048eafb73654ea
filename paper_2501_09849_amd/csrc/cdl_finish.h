// Adding up per-block results inside the kernel that made them (not installed).
//
// A second, tiny launch that adds the blocks' partial results up costs as much as the pass itself for a small tensor (32 K entries: 4.4 us, and
// 7.8 us for the launch that adds up its sixteen histograms, and 3 - 4 us of host time), so where a grid has few blocks the block with
// the highest number waits for the others and finishes the job itself (6.3 us in all).  The sums of the two scalar gradients of grids of more
// blocks go in two steps: the last block of every group of consecutive blocks adds up its group's, the last of the grid those of the
// groups (backward pass of 2.4 M entries 11.9 -> 10.2 us, of 6.4 M 20.6 -> 19.4; histograms so: 2.4 M entries of 255 levels 14 -> 22).  One-trip grids
// of tensors that stream past the caches (more than 2048 blocks, 2^23 entries and more) keep the second launch: there the records of a block wait behind
// its stores of the tensor (25.6 M entries 56.0 us with a second launch, 56.6 in two steps, 18.9 M 41.2 / 43.8).  Grids of up to 2048 blocks that loop
// finish in the kernel at any size: few blocks, and the pass is bound by arithmetic (9 M entries, 7 levels on a common centre 34.5 us so, 35.5 in two
// launches; 31 levels 36.2 / 37.6; gradient of the entropy, 47 M entries of 255 levels 109.6 / 112.5).
//
// What bounds the hand-over is the number of trips to memory, one after the other, between blocks on different XCDs,
// about 0.7 us each.  A flag behind the data would cost four (data out and acknowledged, flag out, flag in, data in).
// So the data is its own flag: every record carries a check word, its contents combined with the launch's tag, and the
// reader polls the record until the check word fits - one trip out, one in, no order needed between the stores of a
// record.  Records are written and read with device-scope relaxed atomics, which bypass the caches that the XCDs do
// not share.
//
// The records live in the caller's workspace, whose contents are arbitrary: the tag is a 64-bit number that no other
// launch of the process uses, and the reader spoils the check word of every record it has taken, so that a captured
// launch can be replayed with the tag it was captured with.
//
// Every wait ends: a block waits for blocks of lower numbers of its launch alone.  Of a histogram in slices the collectors do, sixteen at most behind 256 blocks at most
// (cdl_marg_slices.h), else the last block; of the scalar sums the last block of each group of 256 waits for the others of its group, which wait for nobody, and the
// grid's last for those and for the groups' last ones; of diagnostic words and plans the last block.  An XCD starts a launch's blocks in the order of their numbers, so that the lowest
// one that has not ended has a place or is the next to get one, and it waits for nobody that has not ended: a launch by itself ends with one place on each XCD.  (Grids with records have up to
// 4097 blocks, 2^23 entries in one trip, more than are resident.)  Launches on several streams share the places: of one at most two collectors, or the 17 last blocks of groups (those with a number of 255 and so on),
// wait on an XCD, which holds a block on each of its 32 compute units at least, and the others finish beside them.
#pragma once

#include "cdl_internal.h"

namespace cdl {

// A tag no other launch of this process has (host).
unsigned long long next_finish_tag();

__device__ __forceinline__ void device_store(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long device_load(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kFinishMaxBlocks = 256;

// What becomes of the per-block sums of the two scalar gradients.
struct ScalarFinish {
    double *partial;               // [gridDim.x][2]: left there for scalar_finalize_kernel; null: finished in the kernel
    unsigned long long *records;   // [gridDim.x][4], then [groups][4]
    unsigned long long tag;
    double mul_d, mul_a;
    float *d_delta, *d_alpha;      // [1] or null
};

// Records of a grid: one per block, one per group of kFinishMaxBlocks of them.
__host__ __device__ __forceinline__ int64_t scalar_records(int64_t blocks) { return blocks + (blocks + kFinishMaxBlocks - 1) / kFinishMaxBlocks; }

// d_delta = mul_d * sum over blocks of acc_d, d_alpha = mul_a * the same of acc_a; the sums run over threads, blocks and
// groups in a fixed order.  Called by all T threads of every block.
template <int T>
__device__ __forceinline__ void scalar_finish(double acc_d, double acc_a, const ScalarFinish &f)
{
    __shared__ double red_d[T / 64], red_a[T / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto block_sum = [&](double &d, double &a) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            d += __shfl_down(d, off, 64);
            a += __shfl_down(a, off, 64);
        }
        if (lane == 0) { red_d[wave] = d; red_a[wave] = a; }
        __syncthreads();
        d = 0.0; a = 0.0;
        if (threadIdx.x == 0)
            for (int w = 0; w < T / 64; ++w) { d += red_d[w]; a += red_a[w]; }
        __syncthreads();
    };
    block_sum(acc_d, acc_a);
    if (f.partial) {
        if (threadIdx.x == 0) {
            f.partial[2 * (size_t)blockIdx.x] = acc_d;
            f.partial[2 * (size_t)blockIdx.x + 1] = acc_a;
        }
        return;
    }
    // (the products keep the check word from fitting a record of which only one word has changed)
    auto check = [&](unsigned long long x, unsigned long long y) {
        return (x * 0x9E3779B97F4A7C15ull + y * 0xBF58476D1CE4E5B9ull) ^ f.tag;
    };
    auto publish = [&](unsigned long long *r) {
        if (threadIdx.x != 0) return;
        const unsigned long long x = (unsigned long long)__double_as_longlong(acc_d), y = (unsigned long long)__double_as_longlong(acc_a);
        device_store(r, x);
        device_store(r + 1, y);
        device_store(r + 2, check(x, y));
    };
    // adds `count` records to thread 0's sums
    auto collect = [&](unsigned long long *records, int count) {
        double d = 0.0, a = 0.0;
        for (int i = threadIdx.x; i < count; i += T) {
            unsigned long long *r = records + 4 * (size_t)i;
            unsigned long long x, y, z;
            do {
                x = device_load(r);
                y = device_load(r + 1);
                z = device_load(r + 2);
            } while (z != check(x, y));
            d += __longlong_as_double((long long)x);
            a += __longlong_as_double((long long)y);
            device_store(r + 2, 0ull);
        }
        block_sum(d, a);
        acc_d += d;
        acc_a += a;
    };
    const int last = (int)gridDim.x - 1, first = (int)blockIdx.x / kFinishMaxBlocks * kFinishMaxBlocks;
    const int leader = min(first + kFinishMaxBlocks - 1, last);
    if ((int)blockIdx.x != leader) {
        publish(f.records + 4 * (size_t)blockIdx.x);
        return;
    }
    if (leader > first) collect(f.records + 4 * (size_t)first, leader - first);
    unsigned long long *const groups = f.records + 4 * (size_t)gridDim.x;
    if (leader != last) {
        publish(groups + 4 * (size_t)(first / kFinishMaxBlocks));
        return;
    }
    if (first > 0) collect(groups, first / kFinishMaxBlocks);
    if (threadIdx.x == 0) {
        if (f.d_delta) *f.d_delta = (float)(acc_d * f.mul_d);
        if (f.d_alpha) *f.d_alpha = (float)(acc_a * f.mul_a);
    }
}

}  // namespace cdl
