// Partition of the kept assignments by local expert (Sec. 2.1; Sec. 3.1 "The MoE Part"):
// a deterministic, stable counting sort.
//   permute  from the router's per-workgroup bit masks (one bit per token and expert) every
//            64-token workgroup derives the per-expert counts, their prefix sum and the rows its
//            own tokens start at; every assignment then finds its row: expert base + rows of
//            earlier workgroups + number of earlier tokens of the workgroup with the same expert
//            (a popcount)
//   gather   the token rows are copied into expert-grouped order, 16 bytes per lane (only when
//            the gate/up projection does not gather them itself)
#include "partition.h"

namespace moe_ep {

// One launch: every workgroup (64 tokens) sums the populations of all workgroups' masks itself --
// per expert the total and the part that lies before it -- instead of waiting for a scan kernel
// (nblk * El popcounts per workgroup, from L2; a launch boundary costs more).  A thread stays with one expert and
// takes every (threads / El)-th workgroup, so that a wavefront reads the masks in the order they lie in memory
// (a wavefront per expert, a line per lane: 31 us for 8192 tokens and 128 experts, 8.7 us so).  Workgroup 0 also
// writes the per-expert counts and their prefix sum for the GEMMs.
constexpr int kPermuteThreads = 1024;

__global__ __launch_bounds__(kPermuteThreads) void dispatch_permute_kernel(
    const int32_t* __restrict__ idx, const unsigned long long* __restrict__ blk_mask, int nblk, int Tn, int k,
    int e0, int El, int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ pos,
    int32_t* __restrict__ perm, Clear clear)
{
    for (int i = blockIdx.x * kPermuteThreads + threadIdx.x; i < clear.n; i += gridDim.x * kPermuteThreads) clear.p[i] = 0;
    extern __shared__ unsigned long long smem[];
    unsigned long long* smask = smem;
    int* sbase = reinterpret_cast<int*>(smem + El);   // rows of this workgroup's tokens before it, then the row base
    int* stotal = sbase + El;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, blk = blockIdx.x;
    for (int e = tid; e < El; e += kPermuteThreads) { stotal[e] = 0; sbase[e] = 0; }
    __syncthreads();
    {
        const int per_pass = kPermuteThreads / El;   // El <= 512: at least two workgroups' masks at once
        const int e = tid % El, b0 = tid / El;
        if (b0 < per_pass) {
            int total = 0, before = 0;
#pragma unroll 4
            for (int b = b0; b < nblk; b += per_pass) {
                const unsigned long long m = blk_mask[(size_t)b * El + e];
                const int c = __popcll(m);
                total += c;
                before += (b < blk) ? c : 0;
                if (b == blk) smask[e] = m;
            }
            if (total) atomicAdd(&stotal[e], total);
            if (before) atomicAdd(&sbase[e], before);
        }
    }
    __syncthreads();
    if (wave == 0) scan_experts(lane, El, stotal, sbase, blk == 0 ? count : nullptr, offset);
    __syncthreads();
    const int t_begin = blk * kTokPerBlock;
    const int n_tok = min(kTokPerBlock, Tn - t_begin);
    for (int a = tid; a < n_tok * k; a += kPermuteThreads) {
        const size_t ga = (size_t)t_begin * k + a;  // global assignment id = t*k + slot
        place_assignment(ga, a / k, idx[ga] - e0, El, smask, sbase, pos, perm);
    }
}

// no tokens: the counts and their prefix sum are zeros
__global__ void dispatch_empty_kernel(int El, int32_t* __restrict__ count, int32_t* __restrict__ offset)
{
    for (int e = threadIdx.x; e <= El; e += blockDim.x) {
        if (e < El) count[e] = 0;
        offset[e] = 0;
    }
}

__global__ __launch_bounds__(256) void gather_rows_kernel(
    const uint4* __restrict__ tokens, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ n_rows_ptr, int k, int M8, uint4* __restrict__ xp)
{
    const int A = *n_rows_ptr;
    const int lane = threadIdx.x & 63;
    const int gw = (blockIdx.x * 256 + threadIdx.x) >> 6, nw = gridDim.x * 4;
    for (int p = gw; p < A; p += nw) {
        const int t = perm[p] / k;
        const uint4* src = tokens + (size_t)t * M8;
        uint4* dst = xp + (size_t)p * M8;
        int c = lane;
        for (; c + 192 < M8; c += 256) {
            const uint4 a0 = src[c], a1 = src[c + 64], a2 = src[c + 128], a3 = src[c + 192];
            dst[c] = a0; dst[c + 64] = a1; dst[c + 128] = a2; dst[c + 192] = a3;
        }
        for (; c < M8; c += 64) dst[c] = src[c];
    }
}

hipError_t launch_dispatch(const int32_t* idx, const unsigned long long* blk_mask, int Tn, int k, int e0, int El,
                           int32_t* count, int32_t* offset, int32_t* pos, int32_t* perm, hipStream_t s, const Clear& clear)
{
    if (Tn <= 0) {
        hipLaunchKernelGGL(dispatch_empty_kernel, dim3(1), dim3(256), 0, s, El, count, offset);
        return hipGetLastError();
    }
    const int nblk = (Tn + kTokPerBlock - 1) / kTokPerBlock;
    hipLaunchKernelGGL(dispatch_permute_kernel, dim3(nblk), dim3(kPermuteThreads),
                       El * (sizeof(unsigned long long) + 2 * sizeof(int)), s, idx, blk_mask, nblk, Tn, k, e0, El,
                       count, offset, pos, perm, clear);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const void* tokens, const int32_t* perm, const int32_t* n_rows_ptr,
                              int k, int M, void* xp, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(gather_rows_kernel, dim3(grid), dim3(256), 0, s,
                       static_cast<const uint4*>(tokens), perm, n_rows_ptr, k, M / 8,
                       static_cast<uint4*>(xp));
    return hipGetLastError();
}

}  // namespace moe_ep
