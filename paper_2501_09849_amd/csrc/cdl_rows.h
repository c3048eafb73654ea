// 16 bytes of a row of an index matrix whose rows need not start on 16-byte boundaries (not installed).
#pragma once

#include <stdint.h>

namespace cdl {

typedef int cdl_v4i __attribute__((ext_vector_type(4)));
typedef int cdl_v4i_any __attribute__((ext_vector_type(4), aligned(1)));

// 16 bytes from any address in one load
__device__ __forceinline__ cdl_v4i load_any16(const int8_t *p) { return *reinterpret_cast<const cdl_v4i_any *>(p); }

// Without its first `over` bytes (0 .. 16), zeros behind the rest
__device__ __forceinline__ cdl_v4i without_first(cdl_v4i v, int over)
{
    union { cdl_v4i v; unsigned long long q[2]; } u;
    u.v = v;
    unsigned long long lo = u.q[0], hi = u.q[1];
    int s = over;
    if (s >= 8) { lo = hi; hi = 0ull; s -= 8; }
    if (s >= 8) { lo = 0ull; s = 0; }
    if (s > 0) { lo = (lo >> (8 * s)) | (hi << (64 - 8 * s)); hi >>= 8 * s; }
    u.q[0] = lo; u.q[1] = hi;
    return u.v;
}

// 16 bytes of a row from entry k0 on, zeros beyond its K entries (K >= 16; k0 may lie beyond them): a chunk that the row ends in is read from
// the row's last 16 bytes and shifted into place, so that nothing outside the row is read.
__device__ __forceinline__ cdl_v4i tail_chunk(const int8_t *row, int k0, int K)
{
    const int over = min(max(k0 + 16 - K, 0), 16);            // bytes of the chunk that lie beyond the row
    return without_first(load_any16(row + (over > 0 ? K - 16 : k0)), over);
}

}  // namespace cdl
