// Sixteen consecutive bytes of a sample row (or of a row of flags) at any byte
// address, for the kernels that take rows of any base, stride and length.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace xeng {

typedef unsigned int row16 __attribute__((ext_vector_type(4)));
typedef unsigned int row16_u __attribute__((ext_vector_type(4), aligned(1)));

// Bytes i0 .. i0 + 15 of `row`, of which those below `end` exist; the others
// read as 0x88, the zero sample.  Where the end is inside, the 16 bytes that
// end there are read and shifted down, so no load passes it; `before`: bytes
// of the row that lie before `row`.  (Global loads run in unaligned-access
// mode, which the compiler assumes for align-1 loads.)
__device__ __forceinline__ row16 load_row16(const uint8_t *row, int i0, int end, int before = 0)
{
    constexpr uint32_t Z = 0x88888888u;
    if (i0 >= end) return row16{Z, Z, Z, Z};
    const int past = i0 + 16 - end;   // bytes of the 16 that do not exist
    if (past <= 0) return *reinterpret_cast<const row16_u *>(row + i0);
    if (i0 + before >= past) {
        const row16 x = *reinterpret_cast<const row16_u *>(row + i0 - past);
        const uint32_t d[8] = {x.x, x.y, x.z, x.w, Z, Z, Z, Z};
        const int q = past >> 2, sh = past & 3;
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // dwords k + q and k + q + 1 of d, without dynamic indexing
            uint32_t lo = d[k], hi = d[k + 1];
#pragma unroll
            for (int u = 1; u < 4; ++u) {
                lo = q == u ? d[k + u] : lo;
                hi = q == u ? d[k + u + 1] : hi;
            }
            o[k] = (uint32_t)((((uint64_t)hi << 32) | lo) >> (8 * sh));
        }
        return row16{o[0], o[1], o[2], o[3]};
    }
    // fewer than 16 bytes in the whole row
    uint32_t o[4] = {Z, Z, Z, Z};
#pragma unroll
    for (int k = 0; k < 16; ++k)
        if (i0 + k < end) o[k >> 2] = (o[k >> 2] & ~(0xFFu << (8 * (k & 3)))) | ((uint32_t)row[i0 + k] << (8 * (k & 3)));
    return row16{o[0], o[1], o[2], o[3]};
}

}  // namespace xeng
