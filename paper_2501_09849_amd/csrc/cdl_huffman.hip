// Huffman-coded size of a tensor of level indices (Sec. V-A, eq. Nofbits: the paper measures the
// compressed size of weights and activations as the average Huffman code length per entry).
//
// A histogram of the int8 indices (16 bytes per thread and trip; per-wave LDS histograms with eight interleaved
// copies of every bin, so that lanes collide only when they share copy and bin), whose rows - one of 256 counts per
// block - are added up by its last block (few blocks: cdl_finish.h) or by a second kernel of one block.  Either then
// sorts the counts and runs the two-queue form of Huffman's algorithm: the total code length is the sum of the weights
// of all merged nodes, which no choice among equal weights can change.
#include "cdl_internal.h"
#include "cdl_finish.h"

namespace cdl {

namespace {

constexpr int kHistThreads = 256;
constexpr int kHistCopies = 8;
constexpr int kHistMaxBlocks = 1024;

struct HuffmanOut {
    int64_t n;
    int lo, n_levels;
    unsigned long long *counts;       // [n_levels] or null
    unsigned long long *total_bits;   // [1] or null
    float *bits_per_entry;            // [1] or null
};

constexpr int kQueue = 256 + 4;      // weights of a queue and the empty places that may be looked at behind them

// Sum of the weights of the merged nodes.  leaf: the sorted counts, node: empty; places that hold no weight hold kNone.
// One step takes the two smallest of the heads L0, L1 of the leaves and M0, M1 of the nodes and appends their sum to
// the nodes.  What bounds it is one chain of a few dozen instructions per step on one wave (256 levels: 255 steps), so
// nothing in it branches or waits: the places behind the heads, L2, L3 and M2, M3, are asked for at the end of a step
// and needed at the end of the next, which hides the latency of LDS (two pops per step, each with reads that the next
// compare waits for and branches: 54 us for the kernel at 255 levels, this way 28).
template <typename T>
__device__ __forceinline__ unsigned long long merge_weights(const T *leaf, T *node, int first)
{
    constexpr T kNone = ~(T)0;             // above every weight
    int zero = 0;
    asm volatile("" : "+v"(zero));         // (every lane does the same; told so, the compiler would branch on the scalar unit)
    const T *lp = leaf + first + zero;
    const T *mp = node + zero;
    T *tail = node + zero;
    T L0 = lp[0], L1 = lp[1], L2 = lp[2], L3 = lp[3], M0 = kNone, M1 = kNone, M2 = kNone, M3 = kNone;
    unsigned long long total = 0ull;
    for (int step = 255 - first; step > 0; --step) {
        const bool two_leaves = L1 <= M0, two_nodes = M1 < L0;
        const T w = (two_nodes ? M1 : L0) + (two_leaves ? L1 : M0);       // (never both)
        total += (unsigned long long)w;
        *tail = w;
        const T l0 = two_nodes ? L0 : L1, l1 = two_nodes ? L1 : L2, m0 = two_leaves ? M0 : M1, m1 = two_leaves ? M1 : M2;
        L0 = two_leaves ? L2 : l0;
        L1 = two_leaves ? L3 : l1;
        M0 = two_nodes ? M2 : m0;
        M1 = two_nodes ? M3 : m1;
        lp += two_leaves ? 2 : (two_nodes ? 0 : 1);
        mp += two_leaves ? 0 : (two_nodes ? 2 : 1);
        M0 = mp == tail ? w : M0;
        M1 = mp + 1 == tail ? w : M1;
        ++tail;
        L2 = lp[2]; L3 = lp[3];
        M2 = mp[2]; M3 = mp[3];
    }
    return total;
}

// All threads of the block (the first 256 of them work): from the count of every byte value, in `key`, to the outputs.
// Thread t has byte value t, i.e. level (int8)t.  `key` is overwritten.
__device__ __forceinline__ void huffman_finish(unsigned long long *key /* [kQueue] */, unsigned long long *sorted /* [kQueue] */, const HuffmanOut &o)
{
    const int t = threadIdx.x;
    unsigned long long c = 0ull;
    if (t < 256) {
        const int level = (int)(int8_t)(uint8_t)t;
        const bool in_set = level >= o.lo && level < o.lo + o.n_levels;
        c = in_set ? key[t] : 0ull;
        if (o.counts && in_set) o.counts[level - o.lo] = c;
    }
    __syncthreads();
    const unsigned long long mine = (c << 8) | (unsigned int)t;      // counts made different by their bins
    if (t < 256) key[t] = mine;
    __syncthreads();
    // rank of every count among the 256: two counts per 16-byte LDS read that all lanes share, no barriers
    if (t < 256) {
        int rank = 0;
        const ulonglong2 *pairs = reinterpret_cast<const ulonglong2 *>(key);
#pragma unroll 8
        for (int q = 0; q < 128; ++q) {
            const ulonglong2 v = pairs[q];
            rank += (v.x < mine ? 1 : 0) + (v.y < mine ? 1 : 0);
        }
        sorted[rank] = c;
    }
    __syncthreads();
    if (t >= 64) return;
    // the zeros sort to the front
    int first = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) first += __popcll(__ballot(sorted[64 * q + t] == 0ull));
    first = __builtin_amdgcn_readfirstlane(first);
    unsigned long long total = 0ull;
    if (first == 255) {
        total = sorted[255];          // a single level that occurs: one bit per entry
    } else if (first < 255) {
        if (o.n < (1ll << 31)) {
            unsigned int *leaf32 = reinterpret_cast<unsigned int *>(key), *node32 = leaf32 + kQueue;
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const int i = 64 * q + t;
                if (i < kQueue) { leaf32[i] = i < 256 ? (unsigned int)sorted[i] : ~0u; node32[i] = ~0u; }
            }
            total = merge_weights<unsigned int>(leaf32, node32, first);
        } else {
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const int i = 64 * q + t;
                if (i >= 256 && i < kQueue) sorted[i] = ~0ull;
                if (i < kQueue) key[i] = ~0ull;
            }
            total = merge_weights<unsigned long long>(sorted, key, first);
        }
    }
    if (t == 0) {
        if (o.total_bits) *o.total_bits = total;
        if (o.bits_per_entry) *o.bits_per_entry = o.n > 0 ? (float)((double)total / (double)o.n) : 0.0f;
    }
}

// FEW: the last block adds the rows, as records of a count and its check word (cdl_finish.h).
template <bool FEW>
__global__ __launch_bounds__(kHistThreads)
void index_hist_kernel(const int8_t *__restrict__ idx, int64_t n, unsigned int *__restrict__ rows /* [gridDim.x][256] */,
                       unsigned long long *records /* [gridDim.x][256][2] */, unsigned long long tag, HuffmanOut out)
{
    __shared__ __attribute__((aligned(16))) unsigned int hist[kHistThreads / 64][256 * kHistCopies];
    for (int i = threadIdx.x; i < (kHistThreads / 64) * 256 * kHistCopies / 4; i += kHistThreads)
        reinterpret_cast<uint4 *>(&hist[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    unsigned int *mine = &hist[threadIdx.x >> 6][threadIdx.x & (kHistCopies - 1)];
    const int64_t n16 = n >> 4;
    const int64_t stride = (int64_t)gridDim.x * kHistThreads;
    for (int64_t v = (int64_t)blockIdx.x * kHistThreads + threadIdx.x; v < n16; v += stride) {
        const uint4 w = reinterpret_cast<const uint4 *>(idx)[v];
        const unsigned int ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int b = 0; b < 4; ++b) atomicAdd(mine + ((ws[d] >> (8 * b)) & 0xffu) * kHistCopies, 1u);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        for (int64_t e = n16 << 4; e < n; ++e) atomicAdd(mine + (unsigned int)(uint8_t)idx[e] * kHistCopies, 1u);
    __syncthreads();
    // bin b = the index byte as an unsigned number
    unsigned int s = 0u;
    for (int w = 0; w < kHistThreads / 64; ++w)
#pragma unroll
        for (int c = 0; c < kHistCopies; ++c) s += hist[w][threadIdx.x * kHistCopies + ((c + threadIdx.x) & (kHistCopies - 1))];
    if (!FEW) {
        rows[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
        return;
    }
    if (blockIdx.x != gridDim.x - 1) {
        unsigned long long *r = records + 2 * ((size_t)blockIdx.x * 256 + threadIdx.x);
        device_store(r, s);
        device_store(r + 1, s ^ tag);
        return;
    }
    unsigned long long total = s;
    const int others = (int)gridDim.x - 1;
    for (int b = 0; b < others; b += 8) {
        unsigned long long v[8];
        bool waiting = true;
        while (waiting) {
            unsigned long long c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const unsigned long long *r = records + 2 * ((size_t)(b + u < others ? b + u : b) * 256 + threadIdx.x);
                v[u] = device_load(r);
                c[u] = device_load(r + 1);
            }
            waiting = false;
#pragma unroll
            for (int u = 0; u < 8; ++u) waiting = waiting || (v[u] ^ c[u]) != tag;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + u < others) {
                total += v[u];
                device_store(records + 2 * ((size_t)(b + u) * 256 + threadIdx.x) + 1, v[u]);
            }
    }
    __syncthreads();
    unsigned long long *key = reinterpret_cast<unsigned long long *>(&hist[0][0]);
    key[threadIdx.x] = total;
    __syncthreads();
    huffman_finish(key, key + kQueue, out);
}

__global__ __launch_bounds__(1024)
void huffman_kernel(const unsigned int *__restrict__ rows, int nrows, HuffmanOut out)
{
    __shared__ __attribute__((aligned(16))) unsigned long long key[kQueue];
    __shared__ unsigned long long sorted[kQueue];
    __shared__ unsigned long long part[16][256];
    // 1024 threads = 16 groups of 64: a group takes every sixteenth row, a thread four neighbouring bins
    // (one 16-byte load), four loads in flight each (one thread per bin walking all rows one after the other
    // is nothing but memory latency)
    {
        const int q = threadIdx.x & 63, grp = threadIdx.x >> 6;
        unsigned long long c[4][4] = {};
        const uint4 *rows4 = reinterpret_cast<const uint4 *>(rows);
        int r = grp;
        for (; r + 48 < nrows; r += 64) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint4 v = rows4[(size_t)(r + 16 * u) * 64 + q];
                c[u][0] += v.x; c[u][1] += v.y; c[u][2] += v.z; c[u][3] += v.w;
            }
        }
        for (; r < nrows; r += 16) {
            const uint4 v = rows4[(size_t)r * 64 + q];
            c[0][0] += v.x; c[0][1] += v.y; c[0][2] += v.z; c[0][3] += v.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) part[grp][4 * q + e] = (c[0][e] + c[1][e]) + (c[2][e] + c[3][e]);
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        unsigned long long c = 0ull;
#pragma unroll
        for (int g = 0; g < 16; ++g) c += part[g][threadIdx.x];
        key[threadIdx.x] = c;
    }
    __syncthreads();
    huffman_finish(key, sorted, out);
}

// Up to this many blocks the histogram's last block finishes the job (all of them: 2 M entries).
constexpr int kHistFewBlocks = 64;

int hist_blocks(int64_t n)
{
    int64_t b = (n / 16 + (int64_t)kHistThreads * 8 - 1) / ((int64_t)kHistThreads * 8);
    if (b < 1) b = 1;
    if (b > kHistMaxBlocks) b = kHistMaxBlocks;
    return (int)b;
}

}  // namespace

size_t huffman_workspace_bytes(int64_t n)
{
    // (never less than a smaller tensor needs)
    const size_t blocks = (size_t)hist_blocks(n), few = blocks < kHistFewBlocks ? blocks : kHistFewBlocks;
    const size_t records = few * 256 * 2 * sizeof(unsigned long long), rows = blocks * 256 * sizeof(unsigned int);
    return records > rows ? records : rows;
}

int launch_huffman_bits(const int8_t *idx, int64_t n, int lo, int n_levels, unsigned long long *counts,
                        unsigned long long *total_bits, float *bits_per_entry, void *ws, hipStream_t stream)
{
    const int blocks = hist_blocks(n);
    const HuffmanOut out{n, lo, n_levels, counts, total_bits, bits_per_entry};
    if (blocks <= kHistFewBlocks) {
        CDL_LAUNCH("index_hist_kernel", stream, index_hist_kernel<true>, dim3(blocks), dim3(kHistThreads), 0, idx, n, (unsigned int *)nullptr,
                   reinterpret_cast<unsigned long long *>(ws), next_finish_tag(), out);
        return check_launch();
    }
    unsigned int *rows = reinterpret_cast<unsigned int *>(ws);
    CDL_LAUNCH("index_hist_kernel", stream, index_hist_kernel<false>, dim3(blocks), dim3(kHistThreads), 0, idx, n, rows,
               (unsigned long long *)nullptr, 0ull, out);
    CDL_LAUNCH("huffman_kernel", stream, huffman_kernel, dim3(1), dim3(1024), 0, rows, blocks, out);
    return check_launch();
}

}  // namespace cdl
