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

// Digits of four values: out[l] holds digit l (a signed byte, l = 0 least significant) of g[0..3] in
// its bytes 0..3.  x = g * gscale is exact (gscale is a power of two) and |x| < 0.99 * 2^(8L-1);
// q = rint(x) = sum_l d_l 256^l with d_l in [-128, 127]: the bytes of (q + 0x80..80) ^ 0x80..80.
template <int L>
__device__ __forceinline__ void limbs_of4(const float (&g)[4], float gscale, uint32_t (&out)[L])
{
    if (L <= 4) {
        constexpr uint32_t off = L == 4 ? 0x80808080u : 0x00808080u;
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = (int)rintf(g[e] * gscale);
            d[e] = ((uint32_t)q + off) ^ off;
        }
        const uint32_t t0 = bperm(d[1], d[0], 0x05010400u), t2 = bperm(d[3], d[2], 0x05010400u);
        out[0] = bperm(t2, t0, 0x05040100u);
        out[1] = bperm(t2, t0, 0x07060302u);
        const uint32_t t1 = bperm(d[1], d[0], 0x07030602u), t3 = bperm(d[3], d[2], 0x07030602u);
        out[2] = bperm(t3, t1, 0x05040100u);
        if (L == 4) out[L - 1] = bperm(t3, t1, 0x07060302u);
    } else {
        // q has up to 48 bits: the low 16 (digits 0, 1) and the rest are rounded separately
        constexpr uint32_t offh = L == 6 ? 0x80808080u : 0x00808080u;
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = g[e] * gscale;
            const float H = rintf(x * (1.0f / 65536.0f));
            const float r = fmaf(-H, 65536.0f, x);          // exact, |r| <= 32768
            // r + 1.5 * 2^23 has unit spacing: its mantissa bits are those of the constant plus rint(r), ties to even
            const int t = (int)(__float_as_uint(r + 12582912.0f) + (0x8080u - 0x4B400000u));   // rint(r) + 0x8080, in [0x80, 0x10080]
            lo[e] = (uint32_t)t ^ 0x8080u;                  // bytes 0, 1: digits 0, 1
            const int h = (int)H + (t >> 16);               // carry out of the low two digits
            hi[e] = ((uint32_t)h + offh) ^ offh;
        }
        const uint32_t a0 = bperm(lo[1], lo[0], 0x05010400u), a2 = bperm(lo[3], lo[2], 0x05010400u);
        out[0] = bperm(a2, a0, 0x05040100u);
        out[1] = bperm(a2, a0, 0x07060302u);
        const uint32_t t0 = bperm(hi[1], hi[0], 0x05010400u), t2 = bperm(hi[3], hi[2], 0x05010400u);
        out[2] = bperm(t2, t0, 0x05040100u);
        out[3] = bperm(t2, t0, 0x07060302u);
        const uint32_t t1 = bperm(hi[1], hi[0], 0x07030602u), t3 = bperm(hi[3], hi[2], 0x07030602u);
        out[4] = bperm(t3, t1, 0x05040100u);
        if (L == 6) out[L - 1] = bperm(t3, t1, 0x07060302u);
    }
}

}  // namespace cdl
