// Huffman-coded size of a tensor of level indices (Sec. V-A, eq. Nofbits: the paper measures the
// compressed size of weights and activations as the average Huffman code length per entry).
//
// A histogram of the int8 indices (16 bytes per thread and trip; per-wave LDS histograms with eight interleaved
// copies of every bin, so that lanes collide only when they share copy and bin), whose rows - one of 256 counts per
// block - are added up by its last block (few blocks: cdl_finish.h) or by a second kernel of one block.  Either then
// sorts the counts and runs the two-queue form of Huffman's algorithm, many nodes at a time: the total code length is
// the sum of the weights of all merged nodes, which no choice among equal weights can change.
#include "cdl_internal.h"
#include "cdl_finish.h"

namespace cdl {

namespace {

constexpr int kHistThreads = 256;
constexpr int kHistCopies = 8;
constexpr int kHistMaxBlocks = 1024;
constexpr int kHuffThreads = 1024;

struct HuffmanOut {
    int64_t n;
    int lo, n_levels;
    unsigned long long *counts;       // [n_levels] or null
    unsigned long long *total_bits;   // [1] or null
    float *bits_per_entry;            // [1] or null
};

constexpr int kWave = 64;
constexpr int kQueue = 256 + kWave;      // weights of a queue and the empty places that a window of 64 may reach behind them

// The value of lane (this lane xor S).
template <int S>
__device__ __forceinline__ unsigned int lane_xor(unsigned int v)
{
    if (S == 1) return (unsigned int)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true);      // quad_perm(1, 0, 3, 2)
    if (S == 2) return (unsigned int)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true);      // quad_perm(2, 3, 0, 1)
    if (S == 4) {                                                                                  // 3 (quad_perm), then 7 (half row mirrored)
        const int q = __builtin_amdgcn_mov_dpp((int)v, 0x1B, 0xf, 0xf, true);
        return (unsigned int)__builtin_amdgcn_mov_dpp(q, 0x141, 0xf, 0xf, true);
    }
    if (S == 8) return (unsigned int)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);     // row rotated by 8 of 16
    return (unsigned int)__shfl_xor((int)v, S, kWave);
}
template <int S>
__device__ __forceinline__ unsigned long long lane_xor(unsigned long long v)
{
    return ((unsigned long long)lane_xor<S>((unsigned int)(v >> 32)) << 32) | lane_xor<S>((unsigned int)v);
}
template <int S, typename T>
__device__ __forceinline__ T compare_exchange(T v, int lane)
{
    const T o = lane_xor<S>(v);
    const T lo = v < o ? v : o, hi = v < o ? o : v;
    return (lane & S) ? hi : lo;
}
__device__ __forceinline__ unsigned int lane_value(unsigned int v, int lane) { return (unsigned int)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ unsigned long long lane_value(unsigned long long v, int lane)
{
    return ((unsigned long long)lane_value((unsigned int)(v >> 32), lane) << 32) | lane_value((unsigned int)v, lane);
}

// Sum of the weights of the merged nodes.  leaf[first .. 255]: the sorted counts, behind them and all of node: kNone.  One wave.
// With t the sum of the two smallest weights, no node that is still to be made weighs less than t, so the weights <= t are
// taken two by two in their order whatever is made meanwhile (equal weights may be exchanged): all these pairs are merged
// at once, and the new nodes, in order, go behind the old ones, none of which weighs more.  A round takes the smallest 64 of
// the leaves and nodes that are left: the minimum of the leaves' next 64 with the nodes' next 64 in reverse is that set as a
// bitonic sequence, six compare-exchange steps sort it.  The smallest weight at least doubles in two rounds, so there are few of them
// (2.4 M entries on 255 levels, normal: 14 rounds instead of 254 dependent steps; 43 for Fibonacci's numbers, the worst of 32 bits).
// What bounds it is the chain of a round, about a hundred dependent instructions and a trip through LDS.  The kernel that
// merges 255 levels: 28 us with a step per node, 8 us so.
template <typename T>
__device__ __forceinline__ unsigned long long merge_weights(const T *leaf, T *node, int first)
{
    const int lane = threadIdx.x & (kWave - 1);
    int left = 256 - first, head = first, node_head = 0, tail = 0;
    unsigned long long total = 0ull;       // this lane's share
    while (left > 1) {
        const T l = leaf[head + lane], m = node[node_head + (kWave - 1 - lane)];
        T v = l < m ? l : m;
        v = compare_exchange<32>(v, lane);
        v = compare_exchange<16>(v, lane);
        v = compare_exchange<8>(v, lane);
        v = compare_exchange<4>(v, lane);
        v = compare_exchange<2>(v, lane);
        v = compare_exchange<1>(v, lane);
        const T t = lane_value(v, 0) + lane_value(v, 1);
        const int pairs = __popcll(__ballot(v <= t)) >> 1;
        const T sum = v + lane_xor<1>(v);
        if (lane < 2 * pairs) {
            total += (unsigned long long)v;
            if (!(lane & 1)) node[tail + (lane >> 1)] = sum;
        }
        // how many of the taken weights were leaves: those below the largest taken one, and of those that equal it the first
        const T top = lane_value(v, 2 * pairs - 1);
        const int below = __popcll(__ballot(l < top)), equal = __popcll(__ballot(l == top)), nodes_below = __popcll(__ballot(m < top));
        const int rest = 2 * pairs - below - nodes_below, leaves = below + (rest < equal ? rest : equal);
        head += leaves;
        node_head += 2 * pairs - leaves;
        tail += pairs;
        left -= pairs;
        asm volatile("" ::: "memory");     // the nodes are in LDS before the next windows are read (one wave: in order)
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) total += __shfl_xor(total, off, kWave);
    return total;
}

// All T threads of the block: from the count of every byte value, in `key`, to the outputs.  `key` is overwritten.
// Thread t < 256 has level lo + t.  Only the levels of the set are ranked: with all 256 places compared, the sizes of three
// levels took 1 us longer.
template <int T>
__device__ __forceinline__ void huffman_finish(unsigned long long *key /* [kQueue] */, unsigned long long *sorted /* [kQueue] */, const HuffmanOut &o)
{
    constexpr int kParts = T / 256;      // threads that share a level, each compares it with a part of the others
    __shared__ int ranks[kParts > 1 ? 256 : 1];
    const int t = threadIdx.x, at = t & 255;
    const bool in_set = at < o.n_levels;
    const unsigned long long c = in_set ? key[(uint8_t)(o.lo + at)] : 0ull;
    if (t < 256 && o.counts && in_set) o.counts[at] = c;
    __syncthreads();
    const unsigned long long mine = (c << 8) | (unsigned int)at;         // counts made different by their levels
    if (t < 256) {
        key[t] = in_set ? mine : ~0ull;
        if (kParts > 1) ranks[t] = 0;
    }
    __syncthreads();
    // rank of every count: two counts per 16-byte LDS read that all lanes share
    int rank = 0;
    const ulonglong2 *pairs = reinterpret_cast<const ulonglong2 *>(key);
    const int n_pairs = (o.n_levels + 1) >> 1;
#pragma unroll 8
    for (int q = t >> 8; q < n_pairs; q += kParts) {
        const ulonglong2 v = pairs[q];
        rank += (v.x < mine ? 1 : 0) + (v.y < mine ? 1 : 0);
    }
    if (kParts > 1) {
        atomicAdd(&ranks[at], rank);
        __syncthreads();
        rank = ranks[at];
    }
    if (t < 256) {
        if (in_set) sorted[256 - o.n_levels + rank] = c;
        else sorted[at - o.n_levels] = 0ull;
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
        constexpr int kTrips = kQueue / kWave;
        if (o.n < (1ll << 31)) {
            unsigned int *leaf32 = reinterpret_cast<unsigned int *>(key), *node32 = leaf32 + kQueue;
#pragma unroll
            for (int q = 0; q < kTrips; ++q) {
                const int i = kWave * q + t;
                leaf32[i] = i < 256 ? (unsigned int)sorted[i] : ~0u;
                node32[i] = ~0u;
            }
            total = merge_weights<unsigned int>(leaf32, node32, first);
        } else {
#pragma unroll
            for (int q = 0; q < kTrips; ++q) {
                const int i = kWave * q + t;
                if (i >= 256) sorted[i] = ~0ull;
                key[i] = ~0ull;
            }
            total = merge_weights<unsigned long long>(sorted, key, first);
        }
    }
    if (t == 0) {
        if (o.total_bits) *o.total_bits = total;
        if (o.bits_per_entry) *o.bits_per_entry = o.n > 0 ? (float)((double)total / (double)o.n) : 0.0f;
    }
}

// FEW: the last block adds the rows.  A record is four counts of 16 bits (a block has 2^15 entries and the 15 last ones at most) and a check word (cdl_finish.h): 1 KB a block, where a check word for
// every count was 4.  us of a call,
// with that and one trip's loads under way / so: 255 levels 131 K entries 12.8 / 11.4, 1 M 16.5 / 13.4, 2 M 20.4 / 14.8, 3 levels 2 M 15.6 / 9.7.
template <bool FEW>
__global__ __launch_bounds__(kHistThreads)
void index_hist_kernel(const int8_t *__restrict__ idx, int64_t n, unsigned int *__restrict__ rows /* [gridDim.x][256] */,
                       unsigned long long *records /* [gridDim.x][64][2] */, unsigned long long tag, HuffmanOut out)
{
    __shared__ __attribute__((aligned(16))) unsigned int hist[kHistThreads / 64][256 * kHistCopies];
    for (int i = threadIdx.x; i < (kHistThreads / 64) * 256 * kHistCopies / 4; i += kHistThreads)
        reinterpret_cast<uint4 *>(&hist[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    unsigned int *mine = &hist[threadIdx.x >> 6][threadIdx.x & (kHistCopies - 1)];
    const int64_t n16 = n >> 4;
    const int64_t stride = (int64_t)gridDim.x * kHistThreads;
    constexpr int U = FEW ? 4 : 1;      // trips whose loads are under way together (grids that leave rows: 2.36 M entries 13.8 us with one, 14.1 with four)
    for (int64_t v = (int64_t)blockIdx.x * kHistThreads + threadIdx.x; v < n16; v += U * stride) {
        uint4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u == 0 || v - (int)threadIdx.x + u * stride < n16) w[u] = reinterpret_cast<const uint4 *>(idx)[v + u * stride < n16 ? v + u * stride : v];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && v + u * stride >= n16) break;
            const unsigned int ws[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int b = 0; b < 4; ++b) atomicAdd(mine + ((ws[d] >> (8 * b)) & 0xffu) * kHistCopies, 1u);
        }
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
        unsigned long long four = (unsigned long long)s << (16 * (threadIdx.x & 3));
        four |= lane_xor<1>(four);
        four |= lane_xor<2>(four);
        if ((threadIdx.x & 3) < 2) device_store(records + 2 * ((size_t)blockIdx.x * 64 + (threadIdx.x >> 2)) + (threadIdx.x & 1), (threadIdx.x & 1) ? four ^ tag : four);
        return;
    }
    // wave w: rows w, w + 4, .., a lane four counts
    const int others = (int)gridDim.x - 1, lane = threadIdx.x & 63;
    unsigned int sum[4] = {0u, 0u, 0u, 0u};
    for (int b = threadIdx.x >> 6; b < others; b += 32) {
        unsigned long long v[8];
        bool waiting = true;
        while (waiting) {
            unsigned long long c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const unsigned long long *r = records + 2 * ((size_t)(b + 4 * u < others ? b + 4 * u : b) * 64 + lane);
                v[u] = device_load(r);
                c[u] = device_load(r + 1);
            }
            waiting = false;
#pragma unroll
            for (int u = 0; u < 8; ++u) waiting = waiting || (v[u] ^ c[u]) != tag;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + 4 * u < others) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += (unsigned int)(v[u] >> (16 * e)) & 0xffffu;
                device_store(records + 2 * ((size_t)(b + 4 * u) * 64 + lane) + 1, v[u]);      // (spoilt, for a replay)
            }
    }
    unsigned long long total = s;
    if (others > 0) {
        __syncthreads();      // (the histogram has been read)
        unsigned int *const parts = &hist[0][0] + 2 * kQueue * 2;      // behind the queues
#pragma unroll
        for (int e = 0; e < 4; ++e) parts[(threadIdx.x >> 6) * 256 + 4 * lane + e] = sum[e];
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kHistThreads / 64; ++w) total += parts[w * 256 + threadIdx.x];
    }
    __syncthreads();
    unsigned long long *key = reinterpret_cast<unsigned long long *>(&hist[0][0]);
    key[threadIdx.x] = total;
    __syncthreads();
    huffman_finish<kHistThreads>(key, key + kQueue, out);
}

__global__ __launch_bounds__(kHuffThreads)
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
    huffman_finish<kHuffThreads>(key, sorted, out);
}

// Up to this many blocks the histogram's last block finishes the job (all of them: 2 M entries; 2.36 M of 255 levels in one launch 15.5 us, in two 13.8).
constexpr int kHistFewBlocks = 64;

int64_t hist_blocks_of_eight(int64_t n)      // trips
{
    const int64_t b = (n / 16 + (int64_t)kHistThreads * 8 - 1) / ((int64_t)kHistThreads * 8);
    return b < 1 ? 1 : b > kHistMaxBlocks ? kHistMaxBlocks : b;
}

// Small tensors: as few trips as up to 64 blocks leave (the workspace has room for four times the blocks of eight).  Not the smallest: 20 K entries 6.7 us in one block, 7.0 in five.
int hist_blocks(int64_t n)
{
    const int64_t eight = hist_blocks_of_eight(n), two = 4 * eight, one = (n / 16 + kHistThreads - 1) / kHistThreads;
    int64_t b = two < one ? two : one;
    if (b > kHistFewBlocks) b = kHistFewBlocks;
    if (n < 65536) return (int)eight;
    return (int)(b > eight ? b : eight);
}

}  // namespace

size_t huffman_workspace_bytes(int64_t n)
{
    // (never less than a smaller tensor needs)
    const size_t blocks = (size_t)hist_blocks_of_eight(n), few = blocks < kHistFewBlocks ? blocks : kHistFewBlocks;
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
    CDL_LAUNCH("huffman_kernel", stream, huffman_kernel, dim3(1), dim3(kHuffThreads), 0, rows, blocks, out);
    return check_launch();
}

}  // namespace cdl
