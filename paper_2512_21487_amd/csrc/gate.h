// The gate of one token (Sec. 2.1), owned by one 16-lane row of a wavefront: shared by the gate's own launch (router.hip) and by
// the gate/up projection of a few tokens (narrow_gemm.hip).
#pragma once
#include <climits>

#include "common.h"

namespace moe_ep {

// the value lane (lane ^ pattern) of the same 16-lane row holds; ctrl is a DPP control:
// 0xB1 / 0x4E swap neighbours / pairs inside a quad, 0x141 / 0x140 mirror a half row / a row
template <int CTRL>
__device__ __forceinline__ int row_exchange(int x) { return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false); }

template <int CTRL>
__device__ __forceinline__ uint32_t row_max_step(uint32_t x) { return max(x, (uint32_t)row_exchange<CTRL>((int)x)); }
template <int CTRL>
__device__ __forceinline__ int row_min_step(int x) { return min(x, row_exchange<CTRL>(x)); }

// scores as unsigned integers of the same order, equal for equal scores (-0 == +0); 0 is below every score, also below
// the NaN whose bits are all ones, which would map to it (padding rows: an expert would be selected twice)
__device__ __forceinline__ uint32_t order_key(float v)
{
    const uint32_t u = __float_as_uint(v + 0.0f);
    return max(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u), 1u);
}
__device__ __forceinline__ float key_score(uint32_t key)
{
    return __uint_as_float(key ^ ((key & 0x80000000u) ? 0x80000000u : 0xffffffffu));
}

// idx[k], ex[k] (LDS): the k best of the E <= 16 * EPL scores in `row` and the scores; sub: lane inside the row
template <int EPL>
__device__ __forceinline__ void select_experts(const float* row, int E, int k, int sub, int* idx, float* ex)
{
    uint32_t key[EPL];   // 0: out of range or already selected
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = sub + 16 * i;
        key[i] = e < E ? order_key(row[e]) : 0u;
    }
    for (int s = 0; s < k; ++s) {
        uint32_t best = key[0];
#pragma unroll
        for (int i = 1; i < EPL; ++i) best = max(best, key[i]);
        best = row_max_step<0xB1>(best);
        best = row_max_step<0x4E>(best);
        best = row_max_step<0x141>(best);
        best = row_max_step<0x140>(best);   // every lane of the row now holds the round's winner
        int bi = INT_MAX;                   // equal scores: the lowest expert
#pragma unroll
        for (int i = EPL - 1; i >= 0; --i) bi = key[i] == best ? sub + 16 * i : bi;
        bi = row_min_step<0xB1>(bi);
        bi = row_min_step<0x4E>(bi);
        bi = row_min_step<0x141>(bi);
        bi = row_min_step<0x140>(bi);
#pragma unroll
        for (int i = 0; i < EPL; ++i) key[i] = bi == sub + 16 * i ? 0u : key[i];
        if (sub == 0) {
            idx[s] = bi;
            ex[s] = key_score(best);
        }
    }
}

// Everything that need not follow round by round, a lane per slot: ex[s] becomes exp(score - best score).  Returns their sum; softmax
// restricted to the selection = full softmax renormalised over it; the sum runs in slot order in every lane.
__device__ __forceinline__ float selection_sum(int k, int sub, float* ex)
{
    wavefront_lds_order();
    const float v0 = ex[0];
    wavefront_lds_order();
    for (int s = sub; s < k; s += 16) ex[s] = expf(ex[s] - v0);
    wavefront_lds_order();
    float sum = 0.f;
    for (int s = 0; s < k; ++s) sum += ex[s];
    return sum;
}

}  // namespace moe_ep
