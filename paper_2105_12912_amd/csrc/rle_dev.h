// rle_dev.h -- run expansion, shared by the kernels that write the codes out and
// those that reconstruct from them.
#pragma once

#include "encode_dev.h"

namespace ebc {

// The runs of one tile in LDS, as many as it has elements at most.  (With room for
// 1024 and the rest searched in HBM, the tiles of one run per one or two elements
// took 25 us each, at the end of the launch: 112 us instead of 86 for a
// mostly constant field of 120M elements.)
struct RleStage {
    uint16_t start[kRleTile];  // from the tile's first element on
    uint16_t val[kRleTile];
};

// The kRleItems codes of this thread in tile t, which holds nr > 1 runs from run
// rlo on (elements past the field's end take the last run's value): the run that
// holds its first element by binary search, then a forward walk.  starts: the
// batch's scanned run starts.  Called by the whole workgroup.
__device__ __forceinline__ void expand_tile(const FieldDesc& fd, uint32_t t, uint32_t rlo, uint32_t nr,
                                            const uint32_t* __restrict__ starts, RleStage& sm,
                                            uint16_t c[kRleItems])
{
    const uint32_t* S = starts + fd.rle_base;
    const uint32_t lo = S[0] + (t - fd.rt_base) * kRleTile;
    const EBC_G uint16_t* val = fd.rval;
    nr = min(nr, kRleTile);  // (runs are non-empty)
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < nr; i += kBlock) {
        sm.start[i] = i ? (uint16_t)(S[rlo + i] - lo) : 0;  // the first run may start earlier
        sm.val[i] = val[rlo + i];
    }
    __syncthreads();
    const uint32_t i0 = threadIdx.x * kRleItems;
    uint32_t a = 0, b = nr - 1;
    while (a < b) {
        const uint32_t m = (a + b + 1) >> 1;
        if (sm.start[m] <= i0) a = m;
        else b = m - 1;
    }
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        if (k) a += sm.start[min(a + 1, nr - 1)] == i0 + k ? 1u : 0u;
        c[k] = sm.val[a];
    }
}

// the code of element i
__device__ __forceinline__ uint16_t run_value(const FieldDesc& fd, uint32_t i, const uint32_t* __restrict__ starts,
                                              const uint32_t* __restrict__ tmap)
{
    const uint32_t* S = starts + fd.rle_base;
    const uint32_t t = fd.rt_base + i / kRleTile, s0 = S[0];
    uint32_t a = tmap[2 * t], b = a + tmap[2 * t + 1] - 1;
    if (b == a) return (uint16_t)a;
    while (a < b) {
        const uint32_t m = a + ((b - a + 1) >> 1);
        if (S[m] - s0 <= i) a = m;
        else b = m - 1;
    }
    return fd.rval[a];
}

__device__ __forceinline__ uint4 pack8(const uint16_t c[8])
{
    return make_uint4(c[0] | ((uint32_t)c[1] << 16), c[2] | ((uint32_t)c[3] << 16), c[4] | ((uint32_t)c[5] << 16),
                      c[6] | ((uint32_t)c[7] << 16));
}

}  // namespace ebc
