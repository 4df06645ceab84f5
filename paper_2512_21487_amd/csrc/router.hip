// Gate: per token, the top-k of E routing scores and their renormalised softmax weights
// (Sec. 2.1).  A token is owned by one 16-lane row of a wavefront, so a wavefront advances four
// tokens at once: lane l of the row holds scores l, l+16, ... in registers as integers of the same order, and
// each of the k selection rounds is a lane-local maximum, a four-step maximum over the row done with DPP
// lane exchanges (quad swaps and row mirrors: register moves, no LDS traffic), and the same for the lowest expert
// that has it.  The rounds are what the kernel lasts for, and the wavefronts of a SIMD take turns at them: a
// workgroup is 16 tokens, one wavefront per SIMD (64 tokens and 16 wavefronts: 256 tokens, 128 scores, k = 8 6.7 us
// instead of 4.7, 8192 tokens 12.4 instead of 10.5, launch included).
// The workgroup also records, per local expert, 16 bits of the 64-bit mask (one per expert and 64 tokens) of the
// tokens that selected it; the partition kernels derive counts and stable ranks from it,
// so no atomically allocated slot ever decides an order.  A call of at most 64 tokens is one workgroup of 64, which
// partitions right away out of LDS (route_and_partition): one launch less; of up to four tokens the gate/up projection's launch does
// both (narrow_gemm.hip).
// Where a call's token rows have to cross the host link first, more workgroups of the same launch fetch them (RowCopy):
// scores and rows are read in place, and the call stays on one stream.  Qwen3-235B-A22B-shaped share, pinned host I/O, copies on a stream of
// their own, scores first / now: 1 / 64 / 256 / 1024 tokens 63 / 34, 146 / 130, 207 / 188, 449 / 425 us (256 KB over the
// link instead of 128: 1 - 2 % slower).
#include "gate.h"
#include "partition.h"

namespace moe_ep {

bool rows_come_with_gate(int E, int r, bool shared_first) { return E <= 256 && (r == 1 || !shared_first); }

constexpr int kRouterTokens = 16;   // of a workgroup: 16 lanes each
constexpr int kLinkBytes = 128 * 1024;   // in flight over the host link while rows come in

template <int EPL, bool PARTITION>  // scores per lane: E <= 16 * EPL; PARTITION: one workgroup holds every token
__global__ __launch_bounds__((PARTITION ? kTokPerBlock : kRouterTokens) * 16) void router_topk_kernel(
    const float* __restrict__ logits, int Tn, int E, int k, int e0, int El,
    int32_t* __restrict__ idx, float* __restrict__ w, unsigned long long* __restrict__ blk_mask, PartitionOut part, RowCopy copy)
{
    constexpr int TOKENS = PARTITION ? kTokPerBlock : kRouterTokens, THREADS = TOKENS * 16;
    if ((int)blockIdx.x >= copy.first) {   // a workgroup that brings token rows in
        const uint4* src = static_cast<const uint4*>(copy.src);
        uint4* dst = static_cast<uint4*>(copy.dst);
        const size_t n = copy.bytes / 16, step = (size_t)(gridDim.x - copy.first) * THREADS;
        for (size_t i = (size_t)(blockIdx.x - copy.first) * THREADS + threadIdx.x; i < n; i += step) dst[i] = src[i];
        return;
    }
    extern __shared__ unsigned long long smask[];                  // [El] token masks of the local experts
    int* s_idx = reinterpret_cast<int*>(smask + El);               // [TOKENS][k] selected experts
    float* s_ex = reinterpret_cast<float*>(s_idx + TOKENS * k);    // [TOKENS][k] score, then exp(score - best score)
    int* s_total = reinterpret_cast<int*>(s_ex + TOKENS * k);      // [El] rows, [El] first row (PARTITION)
    int* s_base = s_total + El;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane & 15, tl = wave * 4 + (lane >> 4);        // lane inside the row; token inside the block
    for (int i = tid; i < El; i += THREADS) smask[i] = 0ull;
    __syncthreads();

    const int t = blockIdx.x * TOKENS + tl;
    const bool live = t < Tn;
    if (wave * 4 + blockIdx.x * TOKENS < Tn) {   // the wavefront has a token
        const float* row = logits + (size_t)min(t, Tn - 1) * E;
        select_experts<EPL>(row, E, k, sub, s_idx + tl * k, s_ex + tl * k);
        const float sum = selection_sum(k, sub, s_ex + tl * k);
        if (live)
            for (int s = sub; s < k; s += 16) {
                const int el = s_idx[tl * k + s] - e0;
                if (el >= 0 && el < El) atomicOr(&smask[el], 1ull << tl);
                idx[(size_t)t * k + s] = s_idx[tl * k + s];
                w[(size_t)t * k + s] = s_ex[tl * k + s] / sum;
            }
    }
    __syncthreads();
    if (PARTITION) {
        for (int i = tid; i < part.clear.n; i += THREADS) part.clear.p[i] = 0;
        for (int e = tid; e < El; e += THREADS) { s_total[e] = __popcll(smask[e]); s_base[e] = 0; }
        __syncthreads();
        if (wave == 0) scan_experts(lane, El, s_total, s_base, part.count, part.offset);
        __syncthreads();
        for (int a = tid; a < Tn * k; a += THREADS) place_assignment(a, a / k, s_idx[a] - e0, El, smask, s_base, part.pos, part.perm);
    } else {
        // this workgroup's quarter of the 64-token masks
        constexpr int PARTS = kTokPerBlock / kRouterTokens;
        uint16_t* dst = reinterpret_cast<uint16_t*>(blk_mask) + (size_t)(blockIdx.x / PARTS) * El * PARTS + blockIdx.x % PARTS;
        for (int i = tid; i < El; i += THREADS) dst[(size_t)i * PARTS] = (uint16_t)smask[i];
    }
}

template <bool PARTITION>
static hipError_t launch(const float* logits, int Tn, int E, int k, int e0, int El, int32_t* idx, float* w,
                         unsigned long long* blk_mask, const PartitionOut& part, const RowCopy* copy, hipStream_t s)
{
    if (E < 1 || E > 512 || k < 1 || k > 64) return hipErrorInvalidValue;
    constexpr int TOKENS = PARTITION ? kTokPerBlock : kRouterTokens;
    static_assert(kTokPerBlock == 4 * kRouterTokens && kRouterTokens == 16, "a workgroup's mask is a 16-bit quarter");
    // whole masks: the last 64 tokens' workgroups without a token write zeros
    const int nblk = (Tn + kTokPerBlock - 1) / kTokPerBlock * (kTokPerBlock / TOKENS);
    RowCopy rows{nullptr, nullptr, 0, nblk};
    int grid = nblk;
    if (copy && copy->bytes > 0) {
        if ((reinterpret_cast<uintptr_t>(copy->src) | reinterpret_cast<uintptr_t>(copy->dst) | copy->bytes) & 15) return hipErrorInvalidValue;
        rows = *copy;
        rows.first = nblk;
        const size_t most = (copy->bytes / 16 + TOKENS * 16 - 1) / (TOKENS * 16);
        constexpr int wgs = kLinkBytes / (TOKENS * 16 * 16);
        grid += (int)(most < (size_t)wgs ? most : (size_t)wgs);
    }
    const size_t lds = El * sizeof(unsigned long long) + (size_t)TOKENS * k * 8 + (PARTITION ? (size_t)El * 8 : 0);
#define MOE_EP_ROUTER(EPL)                                                                          \
    hipLaunchKernelGGL((router_topk_kernel<EPL, PARTITION>), dim3(grid), dim3(TOKENS * 16), lds, s, logits, Tn, E, k, e0, \
                       El, idx, w, blk_mask, part, rows)
    if (E <= 16) MOE_EP_ROUTER(1);
    else if (E <= 32) MOE_EP_ROUTER(2);
    else if (E <= 64) MOE_EP_ROUTER(4);
    else if (E <= 128) MOE_EP_ROUTER(8);
    else if (E <= 160) MOE_EP_ROUTER(10);
    else if (E <= 256) MOE_EP_ROUTER(16);
    else MOE_EP_ROUTER(32);
#undef MOE_EP_ROUTER
    return hipGetLastError();
}

hipError_t launch_router(const float* logits, int Tn, int E, int k, int e0, int El, int32_t* idx,
                         float* w, unsigned long long* blk_mask, hipStream_t s, const RowCopy* copy)
{
    if (Tn <= 0) return hipSuccess;
    return launch<false>(logits, Tn, E, k, e0, El, idx, w, blk_mask, PartitionOut{}, copy, s);
}

hipError_t launch_route_and_partition(const float* logits, int Tn, int E, int k, int e0, int El, int32_t* idx, float* w,
                                      int32_t* count, int32_t* offset, int32_t* pos, int32_t* perm, hipStream_t s, const RowCopy* copy, const Clear& clear)
{
    if (Tn < 1 || Tn > kTokPerBlock) return hipErrorInvalidValue;
    return launch<true>(logits, Tn, E, k, e0, El, idx, w, nullptr, PartitionOut{count, offset, pos, perm, clear}, copy, s);
}

}  // namespace moe_ep
