// What the kernels on limbs of the gradient share: digits, direct loads, waits (not installed).
#pragma once

#include "cdl_div.h"
#include "cdl_internal.h"

namespace cdl {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef const void __attribute__((address_space(1))) *gptr_t;
typedef void __attribute__((address_space(3))) *lptr_t;

constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }   // s_waitcnt vmcnt(n) only
constexpr int kLgkmcnt0 = 0xc07f;                                                   // s_waitcnt lgkmcnt(0) only

__device__ __forceinline__ uint32_t bperm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// out[t]: byte t of w[0..3]
__device__ __forceinline__ void transpose4(const uint32_t (&w)[4], uint32_t *out)
{
    const uint32_t t0 = bperm(w[1], w[0], 0x05010400u), t2 = bperm(w[3], w[2], 0x05010400u);
    out[0] = bperm(t2, t0, 0x05040100u);
    out[1] = bperm(t2, t0, 0x07060302u);
    const uint32_t t1 = bperm(w[1], w[0], 0x07030602u), t3 = bperm(w[3], w[2], 0x07030602u);
    out[2] = bperm(t3, t1, 0x05040100u);
    out[3] = bperm(t3, t1, 0x07060302u);
}

// (see limbs_of4; unit: a power of two, also one that is no float)
template <int L>
__device__ __forceinline__ void limbs_of4_wide(const float (&g)[4], double unit, uint32_t (&out)[L])
{
    static_assert(L == 5 || L == 6, "the digits of 40 or 48 bits");
    constexpr double kMagic = 6755399441055744.0 + (L == 5 ? 551911719040.0 : 141289400074368.0);      // 1.5 2^52 + 0x8080808080, 0x808080808080
    uint32_t lo[4], hi[4], w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const unsigned long long v = (unsigned long long)__double_as_longlong(__builtin_fma((double)g[e], unit, kMagic));
        lo[e] = (uint32_t)v;
        hi[e] = (uint32_t)(v >> 32);
    }
    transpose4(lo, w);
#pragma unroll
    for (int l = 0; l < 4; ++l) out[l] = w[l] ^ 0x80808080u;
    if constexpr (L == 5) {
        const uint32_t h0 = bperm(hi[1], hi[0], 0x0c0c0400u), h2 = bperm(hi[3], hi[2], 0x04000c0cu);      // (0x0c: a byte of zeros)
        out[4] = (h0 | h2) ^ 0x80808080u;
    } else {
        const uint32_t h0 = bperm(hi[1], hi[0], 0x05010400u), h2 = bperm(hi[3], hi[2], 0x05010400u);
        out[4] = bperm(h2, h0, 0x05040100u) ^ 0x80808080u;
        out[5] = bperm(h2, h0, 0x07060302u) ^ 0x80808080u;
    }
}

// Digits of four values: out[l] holds digit l (a signed byte, l = 0 least significant) of g[0..3] in
// its bytes 0..3.  x = g * gscale is exact (gscale is a power of two) and |x| < 0.99 * 2^(8L-1);
// q = rint(x) = sum_l d_l 256^l with d_l in [-128, 127]: the bytes of (q + 0x80..80) ^ 0x80..80.
// Five and six limbs: added to 1.5 2^52 in double, x is rounded (to even) into the last bits of the sum, in two's complement, and
// 0x80..80 is added in the same instruction (24 instructions for four values on five limbs; in fp32, the low 16 bits and the rest
// rounded apart, 60: dL/dQ(w) of 65536 x 3072 x 768, 683 -> 619 us).  Up to four the conversion from fp32 to integers, 28
// instructions, is as fast as 20 of which eight are in double.
template <int L>
__device__ __forceinline__ void limbs_of4(const float (&g)[4], float gscale, uint32_t (&out)[L])
{
    if constexpr (L <= 4) {
        constexpr uint32_t off = L == 4 ? 0x80808080u : 0x00808080u;
        uint32_t d[4], w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = (int)rintf(g[e] * gscale);
            d[e] = ((uint32_t)q + off) ^ off;
        }
        transpose4(d, w);
#pragma unroll
        for (int l = 0; l < L; ++l) out[l] = w[l];
    } else {
        limbs_of4_wide<L>(g, (double)gscale, out);
    }
}

}  // namespace cdl
