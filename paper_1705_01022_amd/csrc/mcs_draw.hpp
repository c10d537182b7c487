// The MCS draw on the device (as the host's mcs_draw): tiling origin and order
// of the four domain sets, from the Philox block (0, 0xFFFFFFFF, 0xFFFFFFFF, 4 MCS).
#pragma once

#include "../../include/okpz.h"
#include "kernels.hpp"

namespace okpz {

// Element k of permutation number `pick` (lexicographic order) of {0,1,2,3}.
__device__ __forceinline__ uint32_t perm_element(uint32_t pick, uint32_t k)
{
    uint32_t avail = 0x3210u;  // remaining elements, 4 bits each, ascending
    const uint32_t digit[4] = {pick / 6u, (pick % 6u) / 2u, pick % 2u, 0u};
    uint32_t e = 0;
    for (uint32_t i = 0; i <= k; ++i) {
        const uint32_t sh = 4u * digit[i];
        e = (avail >> sh) & 0xFu;
        const uint32_t low = avail & ((1u << sh) - 1u);
        avail = low | ((avail >> (sh + 4u)) << sh);
    }
    return e;
}

// Tiling origin of MCS m and the word w whose third element picks the order of
// the domain sets.  origin_mode by reference, read where it is used: by value
// the batch kernels held it through the draw and spilled up to seven scalar
// registers more.
__device__ __forceinline__ u32x4 mcs_origin(const StepArgs &A, const uint32_t &origin_mode, uint64_t m, uint32_t &ox,
                                            uint32_t &oy)
{
    const u32x4 w = philox4x32_10(A.key0, A.key1, 0u, 0xFFFFFFFFu, 0xFFFFFFFFu, (uint32_t)(m << 2));
    ox = w.x & A.L_mask;
    oy = w.y & A.L_mask;
    if (origin_mode == OKPZ_ORIGIN_FIXED) ox = oy = 0u;
    if (origin_mode == OKPZ_ORIGIN_COARSE) {
        ox &= ~3u;
        oy &= ~3u;
    }
    return w;
}

}  // namespace okpz
