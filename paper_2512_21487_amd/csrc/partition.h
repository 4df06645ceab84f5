// The partition by expert inside a workgroup (Sec. 2.1): shared by the partition kernel and by the gate
// kernel of calls whose tokens are one workgroup's.
#pragma once
#include "common.h"

namespace moe_ep {

struct PartitionOut { int32_t *count, *offset, *pos, *perm; Clear clear; };   // as launch_dispatch writes them

// One wavefront: exclusive prefix of the rows of all experts, added to base[e] (rows of this workgroup's
// tokens' predecessors); count != NULL: rows and prefix are also written out.  El <= 512: a lane owns 8
// consecutive experts.
__device__ __forceinline__ void scan_experts(int lane, int El, const int* total, int* base, int32_t* count, int32_t* offset)
{
    int c[8], rows = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = lane * 8 + i;
        c[i] = (e < El) ? total[e] : 0;
        rows += c[i];
    }
    int xr = rows;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int yr = __shfl_up(xr, d, 64);
        if (lane >= d) xr += yr;
    }
    int r = xr - rows;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = lane * 8 + i;
        if (e < El) {
            base[e] += r;
            if (count) { count[e] = c[i]; offset[e] = r; }
        }
        if (e == El && count) offset[e] = r;
        r += c[i];
    }
    if (El == 512 && lane == 63 && count) offset[El] = r;
}

// assignment ga (token tl of the workgroup, local expert e): its row, or -1 for an expert that is not here
__device__ __forceinline__ void place_assignment(size_t ga, int tl, int e, int El, const unsigned long long* mask,
                                                 const int* base, int32_t* pos, int32_t* perm)
{
    int p = -1;
    if (e >= 0 && e < El) {
        p = base[e] + __popcll(mask[e] & ((1ull << tl) - 1ull));
        perm[p] = (int32_t)ga;
    }
    pos[ga] = p;
}

}  // namespace moe_ep
