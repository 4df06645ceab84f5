// Weighted aggregation of the selected experts' outputs (Sec. 2.1), added to the shared experts'
// output that the shared down projection has already written into the output rows.  Token-major gather-reduce: a wavefront
// owns a piece of an output row, walks the row's kept slots in slot order, and accumulates in fp32; every load and store is 16 bytes per
// lane and contiguous over the wavefront.  No atomics, so the result is deterministic.
#include "common.h"
#include "kernels.h"

namespace moe_ep {

__device__ __forceinline__ void fma8(float* acc, float ws, const uint4& v) {
    acc[0] = fmaf(ws, bf16_lo(v.x), acc[0]); acc[1] = fmaf(ws, bf16_hi(v.x), acc[1]);
    acc[2] = fmaf(ws, bf16_lo(v.y), acc[2]); acc[3] = fmaf(ws, bf16_hi(v.y), acc[3]);
    acc[4] = fmaf(ws, bf16_lo(v.z), acc[4]); acc[5] = fmaf(ws, bf16_hi(v.z), acc[5]);
    acc[6] = fmaf(ws, bf16_lo(v.w), acc[6]); acc[7] = fmaf(ws, bf16_hi(v.w), acc[7]);
}

// 8 fp32 values of an expert's output row, weighted into the accumulator
__device__ __forceinline__ void fma8f(float* acc, float ws, const f32x4_t& lo, const f32x4_t& hi) {
    acc[0] = fmaf(ws, lo[0], acc[0]); acc[1] = fmaf(ws, lo[1], acc[1]);
    acc[2] = fmaf(ws, lo[2], acc[2]); acc[3] = fmaf(ws, lo[3], acc[3]);
    acc[4] = fmaf(ws, hi[0], acc[4]); acc[5] = fmaf(ws, hi[1], acc[5]);
    acc[6] = fmaf(ws, hi[2], acc[6]); acc[7] = fmaf(ws, hi[3], acc[7]);
}

// N rows of y, added in slot order; all N rows' loads are in flight before the first is used
template <int YMODE, int N>
__device__ __forceinline__ void add_rows(const uint4* __restrict__ y, int M8, unsigned long long& kept, int my_pos, float my_w,
                                         int ca, int cb, bool in_a, bool in_b, float* acc_a, float* acc_b)
{
    uint4 va[N], vb[N], va1[N], vb1[N];   // the second pair: the other half of fp32 rows
    float ws[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int s = __builtin_ctzll(kept);
        kept &= kept - 1;
        const int p = __builtin_amdgcn_readlane(my_pos, s);
        ws[i] = YMODE == 2 ? 1.0f : __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_w), s));
        if (YMODE == 1) {
            const uint4* row = y + (size_t)p * M8 * 2;
            if (in_a) { va[i] = row[2 * ca]; va1[i] = row[2 * ca + 1]; }
            if (in_b) { vb[i] = row[2 * cb]; vb1[i] = row[2 * cb + 1]; }
        } else {
            const uint4* row = y + (size_t)p * M8;
            if (in_a) va[i] = row[ca];
            if (in_b) vb[i] = row[cb];
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (YMODE == 1) {
            if (in_a) fma8f(acc_a, ws[i], __builtin_bit_cast(f32x4_t, va[i]), __builtin_bit_cast(f32x4_t, va1[i]));
            if (in_b) fma8f(acc_b, ws[i], __builtin_bit_cast(f32x4_t, vb[i]), __builtin_bit_cast(f32x4_t, vb1[i]));
        } else {
            if (in_a) fma8(acc_a, ws[i], va[i]);
            if (in_b) fma8(acc_b, ws[i], vb[i]);
        }
    }
}

// YMODE: 0 = y holds bf16 expert outputs, 1 = fp32 expert outputs (rows of M floats), 2 = bf16
// expert outputs that already carry their routing weight (the sum then uses weight 1)
// A wavefront's piece of work is 1024 columns (two 16-byte chunks per lane) of one row: with few tokens the
// columns of a row spread over the GPU instead of following each other in one wavefront, and the rows a token
// keeps are fetched four at a time.  Large calls stream at the copy rate either way (4.7 TB/s); DeepSeek-V2-Lite-shaped
// layer, 1 token: 7.4 -> 3.9 us, Qwen3-235B-A22B-shaped share, 256 tokens 10.2 -> 4.4 us.
template <int YMODE>
__global__ __launch_bounds__(256) void combine_kernel(
    const uint4* __restrict__ y, const int32_t* __restrict__ pos, const float* __restrict__ w, int Tn,
    int k, int M8, bool accumulate, bool all_rows, const uint4* out_src, uint4* out)
{
    const int lane = threadIdx.x & 63;
    const int gw = __builtin_amdgcn_readfirstlane((blockIdx.x * 256 + threadIdx.x) >> 6), nw = gridDim.x * 4;
    const int pieces = (M8 + 127) / 128;
    int t = gw / pieces, piece = gw - t * pieces;
    const int step_t = nw / pieces, step_piece = nw - step_t * pieces;
    for (; t < Tn; t += step_t, piece += step_piece) {
        if (piece >= pieces) { piece -= pieces; if (++t >= Tn) break; }
        const int my_pos = (lane < k) ? pos[(size_t)t * k + lane] : -1;
        const float my_w = (lane < k) ? w[(size_t)t * k + lane] : 0.f;
        unsigned long long kept = __ballot(my_pos >= 0);
        // accumulate: the row already holds the shared experts' output; a token with no kept
        // slot keeps it as it is
        // (all_rows: the rows are written somewhere else than they are read from -- straight to the
        // caller's host buffer -- so a row that only carries the shared experts' output moves too)
        if (accumulate && !all_rows && kept == 0ull) continue;
        const int ca = piece * 128 + lane, cb = ca + 64;
        const bool in_a = ca < M8, in_b = cb < M8;
        uint4 sa, sb;
        if (accumulate) {
            if (in_a) sa = out_src[(size_t)t * M8 + ca];
            if (in_b) sb = out_src[(size_t)t * M8 + cb];
        }
        float acc_a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float acc_b[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        int n = __builtin_popcountll(kept);
        for (; n >= 4; n -= 4) add_rows<YMODE, 4>(y, M8, kept, my_pos, my_w, ca, cb, in_a, in_b, acc_a, acc_b);
        if (n & 2) add_rows<YMODE, 2>(y, M8, kept, my_pos, my_w, ca, cb, in_a, in_b, acc_a, acc_b);
        if (n & 1) add_rows<YMODE, 1>(y, M8, kept, my_pos, my_w, ca, cb, in_a, in_b, acc_a, acc_b);
        if (in_a) {
            if (accumulate) fma8(acc_a, 1.0f, sa);
            uint4 o;
            o.x = pack_bf16x2(acc_a[0], acc_a[1]); o.y = pack_bf16x2(acc_a[2], acc_a[3]);
            o.z = pack_bf16x2(acc_a[4], acc_a[5]); o.w = pack_bf16x2(acc_a[6], acc_a[7]);
            out[(size_t)t * M8 + ca] = o;
        }
        if (in_b) {
            if (accumulate) fma8(acc_b, 1.0f, sb);
            uint4 o;
            o.x = pack_bf16x2(acc_b[0], acc_b[1]); o.y = pack_bf16x2(acc_b[2], acc_b[3]);
            o.z = pack_bf16x2(acc_b[4], acc_b[5]); o.w = pack_bf16x2(acc_b[6], acc_b[7]);
            out[(size_t)t * M8 + cb] = o;
        }
    }
}

hipError_t launch_combine(const void* y, const int32_t* pos, const float* w, int Tn, int k, int M,
                          bool accumulate, int y_mode, const void* out_src, void* out, int grid, hipStream_t s)
{
    if (Tn <= 0) return hipSuccess;
    if (y_mode < 0 || y_mode > 2) return hipErrorInvalidValue;
    auto* yy = static_cast<const uint4*>(y);
    auto* oo = static_cast<uint4*>(out);
    auto* src = static_cast<const uint4*>(out_src ? out_src : out);
    const long long pieces = (long long)Tn * ((M / 8 + 127) / 128);
    if (grid > (pieces + 3) / 4) grid = (int)((pieces + 3) / 4);
    const bool all_rows = out_src != nullptr && out_src != out;
    if (y_mode == 0) hipLaunchKernelGGL(combine_kernel<0>, dim3(grid), dim3(256), 0, s, yy, pos, w, Tn, k, M / 8, accumulate, all_rows, src, oo);
    else if (y_mode == 1) hipLaunchKernelGGL(combine_kernel<1>, dim3(grid), dim3(256), 0, s, yy, pos, w, Tn, k, M / 8, accumulate, all_rows, src, oo);
    else hipLaunchKernelGGL(combine_kernel<2>, dim3(grid), dim3(256), 0, s, yy, pos, w, Tn, k, M / 8, accumulate, all_rows, src, oo);
    return hipGetLastError();
}

}  // namespace moe_ep
