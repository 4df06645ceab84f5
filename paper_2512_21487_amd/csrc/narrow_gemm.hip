// Expert projections for few token rows per expert (Sec. 3.1; decode): the weights are read once and
// everything else is small, so the launch lasts as long as the weight stream from HBM.  Measured on launches of
// the gate/up projection: DeepSeek-V2-Lite-shaped layer, 33 tokens (733 MB with the shared experts) 132 + 50 us in the
// tiled kernels, 118 us here = 6.2 TB/s; Qwen3-235B-A22B-shaped share, 256 tokens (403 MB) 79 and 68 us = 5.9 TB/s.
//
// A workgroup is four wavefronts.  A wavefront owns two blocks of 16 weight rows (gate/up: the gate and the up
// rows of the same 16 activation columns) and up to four blocks of 16 token rows of one expert.  Its weights go
// from global memory straight into registers, kNarrowDepth K steps ahead of the matrix instructions (16 KB in
// flight per wavefront, two workgroups per compute unit).  The token rows, which all four wavefronts need, are
// staged through LDS kNarrowDepth K steps at a time, two buffers deep with one barrier each: read fragment by
// fragment from global memory, 16 rows per load instruction, they would cost the compute unit's address path four
// times what the same bytes cost as whole lines, and that path, not HBM, would set the pace.
// Against the 128 x 256 tiles of grouped_gemm.hip a tile is 64 (gate/up) or 128 (down) output columns wide, so
// that one token's experts already cover the GPU, and no matrix work goes into rows that are not there.
//
// Every output element is accumulated over K in the order of grouped_gemm.hip by the same instruction, and the
// epilogue rounds at the same place: the results are the same bits.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "gate.h"
#include "kernels.h"

namespace moe_ep {

namespace {

constexpr int kNarrowMaxGroups = 512;

// D K steps of weights in flight, row tiles of at most ROWS rows, WAVES wavefronts per workgroup
template <int D_, int ROWS_, int WAVES_>
struct NarrowCfg {
    static constexpr int D = D_, ROWS = ROWS_, WAVES = WAVES_, THREADS = WAVES * 64;
    static constexpr int ROW_BYTES = D * kPackK * 2;             // one token row of a staged chunk (D K steps)
    static constexpr int ROW_CHUNKS = ROW_BYTES / 16;
    static constexpr int PASS_ROWS = THREADS / ROW_CHUNKS; // token rows one load per thread stages
    static constexpr int BUFFER_BYTES = ROWS * ROW_BYTES;
    static_assert(THREADS % ROW_CHUNKS == 0 && 16 % PASS_ROWS == 0, "a block of 16 rows is whole passes");
};
using NarrowStream = NarrowCfg<kNarrowDepth, kNarrowRows, kNarrowWaves>;
// A compute unit draws about 46 GB/s, whatever is in flight (twice the K steps: no change).  Where a launch of 128-column
// tiles leaves compute units without one, half as wide tiles halve what the busiest one has to draw: down projection
// of one token of the DeepSeek-V2-Lite-shaped layer, 112 workgroups, the shared experts' 720 KB each, forward 47 -> 43 us.
using NarrowFew = NarrowCfg<kNarrowDepth, kNarrowFewRows, kNarrowFewWaves>;
// Small tiles in single wavefronts or pairs of them spread a few experts' weights evenly over the compute units, whatever the
// number of tiles is: the choice is launch_narrow_gemm's.
using NarrowFine = NarrowCfg<kNarrowDepth, kNarrowFewRows, 1>;
using NarrowPair = NarrowCfg<kNarrowDepth, kNarrowPairRows, kNarrowFewWaves>;
constexpr int kTurnBytes = 16 * kPackK * 2;                       // one block of 16 weight rows of a K step

// one wavefront's share of a tile: uniform bases, the lane's byte offsets, and how the weight base moves
// from K step to K step (seg_steps steps of w_step bytes, then a jump to the next K segment)
template <class Cfg>
struct NarrowTile {
    const char* w;         // first weight row block at K step 0
    long long w_delta;     // bytes to the second block
    uint32_t w_off;        // the lane's bytes of a block's first load; its second load is w_half further on
    uint32_t w_half;
    long long w_step, seg_jump;
    int seg_steps;
    const char* x;         // token rows
    uint32_t x_off[Cfg::ROWS / Cfg::PASS_ROWS];   // the rows this thread stages
    int KT;
};

// 16 bytes at base + lane offset + wavefront offset: the buffer form keeps bases in scalar registers (the
// pointers are valid for every offset used; the record count is not what bounds them)
template <int CACHE = 0>   // 2: non-temporal
__device__ __forceinline__ uint4 load16(const char* base, uint32_t lane_off, uint32_t wave_off)
{
    auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, 0xffffffffu, 0x00027000);
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off, wave_off, CACHE));
}

// LDS accesses of every wavefront done, loads from global memory left in flight
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// From the caller's rows a load takes 8 rows of 128 bytes (read as operands, 16 rows of 64, the address path takes
// four times as long and every line is asked for twice) and the wavefront turns a block into operands
// through 2 KB of LDS of its own; chunk c of row r lies at c ^ (r / 2 mod 8), all banks in use both ways.
template <int LOADS>   // 1: the block has 8 rows, which stand in the operand twice
__device__ __forceinline__ void turn_block(const uint4 (&w)[LOADS], int lane, char* turn, bf16x8_t (&f)[2])
{
    wavefront_lds_order();   // the block before this one has been read
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int r = i * 8 + (lane >> 3);
        *reinterpret_cast<uint4*>(turn + r * 128 + ((lane & 7) ^ (r >> 1)) * 16) = w[i];
    }
    wavefront_lds_order();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = lane & (8 * LOADS - 1);
        f[h] = *reinterpret_cast<const bf16x8_t*>(turn + r * 128 + ((h * 4 + (lane >> 4)) ^ (r >> 1)) * 16);
    }
}

template <class Cfg, bool SWIGLU, bool PACKED, int MB, bool ONCE = true>
__device__ __forceinline__ void narrow_tile(const NarrowTile<Cfg>& t, int nrows, int tid, char* lds, bool stores, uint16_t* c, int ldc)
{
    constexpr int D = Cfg::D;
    constexpr int PASSES = MB * 16 / Cfg::PASS_ROWS;
    const int lane = tid & 63;
    uint4 w[D][2][2], st[PASSES];   // [ring slot][row block][half of the K step]; the next chunk's token rows
    f32x4_t acc[2][MB];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[b][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const char* wk = t.w;
    int seg = t.seg_steps;
    // ONCE, a group of one row tile: non-temporal, for a layer's weights are read once per call, and between two calls lie
    // the other layers'.  Five layers in turn, kept / non-temporal: DeepSeek-V2-Lite-shaped layer, 1 token 65 / 62 us, 33 tokens 222 / 200;
    // Qwen3-235B-A22B-shaped share, 8 tokens 71 / 65
    auto load_w = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) w[slot][b][h] = load16<ONCE ? 2 : 0>(b == 0 ? wk : wk + t.w_delta, t.w_off, h * t.w_half);
        wk += t.w_step;
        if (--seg == 0) { seg = t.seg_steps; wk += t.seg_jump; }
    };
    // token rows: thread -> row tid / ROW_CHUNKS + PASS_ROWS * i (passes of 8 rows with four wavefronts, of 4 with two, of 2 with one),
    // 16-byte chunk tid % ROW_CHUNKS of the row's staged ROW_BYTES (32 chunks, 512 bytes).  In LDS chunk c of row r
    // lies at c ^ (r mod 16), so that both the writes (one row) and the fragment reads (16 rows, one
    // chunk column) touch all banks evenly.  Chunks past the end of a row re-read its last one, unused.
    const int st_row = tid / Cfg::ROW_CHUNKS, st_chunk = tid % Cfg::ROW_CHUNKS;
    auto load_x = [&](int ch) __attribute__((always_inline)) {
        const uint32_t k_off = min((uint32_t)(ch * Cfg::ROW_BYTES + st_chunk * 16), (uint32_t)t.KT * (kPackK * 2) - 16u);
#pragma unroll
        for (int i = 0; i < PASSES; ++i) st[i] = load16(t.x, t.x_off[i] + k_off, 0);
    };
    auto stage_x = [&](int ch) __attribute__((always_inline)) {
        char* buf = lds + (ch & 1) * Cfg::BUFFER_BYTES;
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int r = st_row + Cfg::PASS_ROWS * i;
            *reinterpret_cast<uint4*>(buf + r * Cfg::ROW_BYTES + (st_chunk ^ (r & 15)) * 16) = st[i];
        }
    };
    // weights in tile order arrive as operands: load h of a block is the k half h of its 16 rows
    char* turn = lds + 2 * Cfg::BUFFER_BYTES + (tid >> 6) * kTurnBytes;
    auto operand = [&](int slot, int b, bf16x8_t (&f)[2]) __attribute__((always_inline)) {
        if (PACKED) {
#pragma unroll
            for (int h = 0; h < 2; ++h) f[h] = __builtin_bit_cast(bf16x8_t, w[slot][b][h]);
            return;
        }
        turn_block(w[slot][b], lane, turn, f);
    };
    auto multiply = [&](int ch, int slot) __attribute__((always_inline)) {
        const char* buf = lds + (ch & 1) * Cfg::BUFFER_BYTES + (lane & 15) * Cfg::ROW_BYTES;
        bf16x8_t f[2][2];
        operand(slot, 0, f[0]);
        operand(slot, 1, f[1]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int col = ((slot * 8 + h * 4 + (lane >> 4)) ^ (lane & 15)) * 16;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const bf16x8_t x = *reinterpret_cast<const bf16x8_t*>(buf + m * 16 * Cfg::ROW_BYTES + col);
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[b][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[b][h], x, acc[b][m], 0, 0, 0);
            }
        }
    };
    const int chunks = (t.KT + D - 1) / D;
    // the weights first: the token rows wait for the row map
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < t.KT) load_w(d);
    load_x(0);
    lds_barrier();   // the wavefronts that still read the tile before this one are done
    stage_x(0);
    lds_barrier();
    int ch = 0;
    for (; (ch + 2) * D <= t.KT; ++ch) {
        load_x(ch + 1);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(ch, d);
            load_w(d);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay D steps ahead of their use
        }
        stage_x(ch + 1);
        lds_barrier();
    }
    for (; ch < chunks; ++ch) {   // the last one or two chunks
        const bool more = ch + 1 < chunks;
        if (more) load_x(ch + 1);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (ch * D + d < t.KT) multiply(ch, d);
            if ((ch + 1) * D + d < t.KT) load_w(d);
        }
        if (more) { stage_x(ch + 1); lds_barrier(); }
    }
    if (!stores) return;
    // a lane holds four consecutive output columns, 4 * (lane >> 4) + {0..3} of a block, of token row lane & 15
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int r = m * 16 + (lane & 15);
        if (r >= nrows) continue;
        uint16_t* row = c + (size_t)r * ldc + (lane >> 4) * 4;
        if (SWIGLU) {
            float h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = silu_f(acc[0][m][i]) * acc[1][m][i];
            *reinterpret_cast<uint2*>(row) = make_uint2(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]));
        } else {
#pragma unroll
            for (int b = 0; b < 2; ++b)
                *reinterpret_cast<uint2*>(row + b * 16) =
                    make_uint2(pack_bf16x2(acc[b][m][0], acc[b][m][1]), pack_bf16x2(acc[b][m][2], acc[b][m][3]));
        }
    }
}

template <class Cfg, bool SWIGLU, bool PACKED>
__device__ __forceinline__ void narrow_dispatch(const GemmArgs& a, int g, int row0, int nrows, int height, int tiles, int n0, int wave, int tid, char* lds,
                                                const uint8_t* tokens = nullptr)   // LDS: the token of a row of the ragged groups
{
    constexpr int WAVE_COLS = SWIGLU ? 16 : 32;
    // N is a multiple of 64: a wavefront's columns are all there or none is; one without any works on the last
    // ones (the barriers count it) and stores nothing
    const bool stores = n0 + wave * WAVE_COLS < a.N;
    const int n = stores ? n0 + wave * WAVE_COLS : a.N - WAVE_COLS;
    const int lane = tid & 63;
    NarrowTile<Cfg> t;
    t.KT = a.K / kPackK;
    if (PACKED) {   // weights in tile order: 4 KB per K step and wavefront, each load instruction 1 KB without gaps
        constexpr int COLS = SWIGLU ? kPackRows / 2 : kPackRows;
        const int NT = (a.N + COLS - 1) / COLS, nt = n / COLS, blk = (n - nt * COLS) / 16 * (SWIGLU ? 2 : 1);
        t.w = reinterpret_cast<const char*>(a.Wp + (((size_t)g * NT + nt) * t.KT * kPackRows + blk * 16) * kPackK);
        t.w_delta = 16 * kPackK * 2;
        t.w_half = 1024;
        t.w_off = lane * 16u;
        t.w_step = (long long)kPackRows * kPackK * 2;
        t.seg_steps = t.KT;
        t.seg_jump = 0;
    } else {
        t.w = reinterpret_cast<const char*>(a.W + (size_t)g * a.w_group_stride + (size_t)n * a.ldw);
        t.w_delta = SWIGLU ? a.w_up_offset * 2 : (long long)16 * a.ldw * 2;
        t.w_off = (uint32_t)(lane >> 3) * (uint32_t)a.ldw * 2u + (lane & 7) * 16u;
        t.w_half = 8u * (uint32_t)a.ldw * 2u;
        t.w_step = kPackK * 2;
        t.seg_steps = a.kseg_len / kPackK;
        t.seg_jump = (a.w_kseg_stride - a.kseg_len) * 2;
    }
    const bool mapped = a.a_row_map != nullptr || tokens;
    t.x = reinterpret_cast<const char*>(mapped ? a.A : a.A + (size_t)row0 * a.lda);
#pragma unroll
    for (int i = 0; i < Cfg::ROWS / Cfg::PASS_ROWS; ++i) {
        // rows past the tile's end re-read its last one; they are multiplied and not stored
        const int r = min(tid / Cfg::ROW_CHUNKS + Cfg::PASS_ROWS * i, nrows - 1);
        const int src = tokens ? tokens[row0 + r] : mapped ? a.a_row_map[row0 + r] / a.a_row_div : r;
        t.x_off[i] = (uint32_t)src * (uint32_t)a.lda * 2u;
    }
    uint16_t* c = a.C + (size_t)g * a.c_group_col_stride + (size_t)row0 * a.ldc + n;
    if constexpr (Cfg::ROWS == 16) {
        narrow_tile<Cfg, SWIGLU, PACKED, 1>(t, nrows, tid, lds, stores, c, a.ldc);
    } else if constexpr (Cfg::ROWS == 32) {   // launched where no group has more rows
        if (nrows <= 16) narrow_tile<Cfg, SWIGLU, PACKED, 1>(t, nrows, tid, lds, stores, c, a.ldc);
        else narrow_tile<Cfg, SWIGLU, PACKED, 2>(t, nrows, tid, lds, stores, c, a.ldc);
    } else {
        static_assert(Cfg::ROWS == 64, "row blocks of a tile");
        // The row tiles of a group that has several, 48 or 64 rows each, read the same weights at about the same time
        // through one L2, so these stay in the caches.  All tokens on the same experts, non-temporal / cached:
        // DeepSeek-V2-shaped share, 200 / 400 tokens 246 / 188, 368 / 279 us, Qwen3-235B-A22B-shaped share, 384 tokens 263 / 237.
        if (tiles > 1) {
            if (height == 48) narrow_tile<Cfg, SWIGLU, PACKED, 3, false>(t, nrows, tid, lds, stores, c, a.ldc);
            else narrow_tile<Cfg, SWIGLU, PACKED, 4, false>(t, nrows, tid, lds, stores, c, a.ldc);
            return;
        }
        switch ((nrows + 15) >> 4) {
            case 1: narrow_tile<Cfg, SWIGLU, PACKED, 1>(t, nrows, tid, lds, stores, c, a.ldc); break;
            case 2: narrow_tile<Cfg, SWIGLU, PACKED, 2>(t, nrows, tid, lds, stores, c, a.ldc); break;
            case 3: narrow_tile<Cfg, SWIGLU, PACKED, 3>(t, nrows, tid, lds, stores, c, a.ldc); break;
            default: narrow_tile<Cfg, SWIGLU, PACKED, 4>(t, nrows, tid, lds, stores, c, a.ldc); break;
        }
    }
}

// row tiles of n rows and the rows of each but the last: equal heights in blocks of 16
__host__ __device__ __forceinline__ int narrow_tiles(int rows, int tallest) { return (rows + tallest - 1) / tallest; }
__device__ __forceinline__ int narrow_height(int rows, int tiles) { return ((rows + 15) / 16 + tiles - 1) / tiles * 16; }

template <class Cfg, bool SWIGLU>
constexpr int narrow_cols() { return Cfg::WAVES * (SWIGLU ? 16 : 32); }

}  // namespace

// The gate's LDS in a launch that routes by itself: where token rows are staged later.
struct GateLds {
    uint32_t mask[kNarrowMaxGroups];   // tokens of a local expert, a bit each
    int idx[kGateTokens * 64];         // expert of a slot
    float ex[kGateTokens * 64];
};

// One wavefront: the gate and the partition of at most kGateTokens tokens, the row tiles before every group and the groups'
// first rows; the workgroup that writes leaves them in memory for the launches behind this one.
__device__ __forceinline__ void route_here(const GateArgs& t, int G, int lane, bool writes, GateLds& l, uint8_t* s_token, int* s_pref, int* s_row0)
{
    const int sub = lane & 15, tl = lane >> 4, slots = t.Tn * t.k;
    const bool live = tl < t.Tn;
    const float* row = t.scores + (size_t)min(tl, t.Tn - 1) * t.E;
    for (int g = lane; g < G; g += 64) l.mask[g] = 0;
    if (t.E <= 64) select_experts<4>(row, t.E, t.k, sub, l.idx + tl * t.k, l.ex + tl * t.k);
    else if (t.E <= 160) select_experts<10>(row, t.E, t.k, sub, l.idx + tl * t.k, l.ex + tl * t.k);
    else select_experts<kGateExperts / 16>(row, t.E, t.k, sub, l.idx + tl * t.k, l.ex + tl * t.k);
    const float sum = selection_sum(t.k, sub, l.ex + tl * t.k);
    if (live)
        for (int s = sub; s < t.k; s += 16) {
            const int el = l.idx[tl * t.k + s] - t.e0;
            if (el >= 0 && el < G) atomicOr(&l.mask[el], 1u << tl);
            if (writes) {
                t.idx[tl * t.k + s] = l.idx[tl * t.k + s];
                t.w[tl * t.k + s] = l.ex[tl * t.k + s] / sum;
            }
        }
    wavefront_lds_order();
    int before = 0;   // tiles, rows << 16
    for (int g0 = 0; g0 < G; g0 += 64) {
        const int g = g0 + lane, rows = g < G ? __popc(l.mask[g]) : 0;
        const int n = rows << 16 | (rows > 0 ? 1 : 0);
        int incl = n;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d, 64);
            if (lane >= d) incl += up;
        }
        const int first = before + incl - n;
        if (g < G) {
            s_pref[g] = first & 0xffff; s_row0[g] = first >> 16;
            if (writes) { t.count[g] = rows; t.offset[g] = first >> 16; }
        }
        before += __shfl(incl, 63, 64);
    }
    if (lane == 0) {
        s_pref[G] = before & 0xffff; s_row0[G] = before >> 16;
        if (writes) t.offset[G] = before >> 16;
    }
    wavefront_lds_order();
    for (int a = lane; a < slots; a += 64) {
        const int el = l.idx[a] - t.e0, tok = a / t.k;
        int p = -1;
        if (el >= 0 && el < G) {
            p = s_row0[el] + __popc(l.mask[el] & ((1u << tok) - 1u));
            s_token[p] = (uint8_t)tok;
            if (writes) t.perm[p] = a;
        }
        if (writes) t.pos[a] = p;
    }
}

// Tile ids: first those of the shared experts s (s.G == 0: none), then those of the routed groups r; each XCD
// (workgroup id mod 8) takes a contiguous run of both, in which the row tiles of one column tile are neighbours,
// so that a group with several of them finds its weights in that XCD's L2 after the first.
// GATE: the launch routes by itself, every workgroup with a routed tile for its own use, about 1 us where the gate's own launch and
// the boundary behind it are 5; shared experts' tiles do not wait for it.
template <class Cfg, bool SWIGLU, bool PACKED, bool GATE = false>
__global__ __launch_bounds__(Cfg::THREADS, 2) void narrow_gemm_kernel(GemmArgs r, GemmArgs s, GateArgs t)
{
    __shared__ int s_pref[kNarrowMaxGroups + 1], s_row0[kNarrowMaxGroups + 1];
    __shared__ __align__(16) char lds[2 * Cfg::BUFFER_BYTES + (PACKED ? 0 : Cfg::WAVES * kTurnBytes)];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __shared__ uint8_t s_token[GATE ? kGateTokens * 64 : 1];   // of a grouped row
    constexpr int COLS = narrow_cols<Cfg, SWIGLU>();
    const int s_mt = s.G > 0 ? narrow_tiles(s.dense_rows, Cfg::ROWS) : 0, s_nt = s.G > 0 ? (s.N + COLS - 1) / COLS : 0;
    const int s_total = s.G * s_mt * s_nt, s_xcd = (s_total + 7) >> 3;
    const int r_nt = (r.N + COLS - 1) / COLS;
    const int xcd = blockIdx.x & 7;
    int slot = blockIdx.x >> 3;
    const auto shared_tile = [&]() __attribute__((always_inline)) {
        const int L = xcd * s_xcd + slot;
        if (L >= s_total) return;
        const int g = L / (s_mt * s_nt), l = L - g * s_mt * s_nt, ni = l / s_mt, mi = l - ni * s_mt;
        const int h = narrow_height(s.dense_rows, s_mt);
        narrow_dispatch<Cfg, SWIGLU, PACKED>(s, g, mi * h, min(h, s.dense_rows - mi * h), h, s_mt, ni * COLS, wave, tid, lds);
    };
    bool writes = false;
    if constexpr (GATE) {
        static_assert(kGateTokens <= 16, "a group is one row tile");
        writes = blockIdx.x == min((uint32_t)s_xcd * 8u, gridDim.x - 8u);
        const int most = s_xcd + ((t.Tn * t.k * r_nt + 7) >> 3);   // slots, whatever the gate says
        for (; slot < s_xcd; slot += gridDim.x >> 3) shared_tile();
        if (slot >= most && !writes) return;
        static_assert(sizeof(GateLds) <= 2 * Cfg::BUFFER_BYTES, "fits where rows are staged");
        __syncthreads();   // a shared tile's rows have been read
        if (wave == 0) route_here(t, r.G, lane, writes, *reinterpret_cast<GateLds*>(lds), s_token, s_pref, s_row0);
    } else if (wave == 0) {   // row tiles before every routed group, from the partition's row offsets
        int before = 0;
        for (int g0 = 0; g0 < r.G; g0 += 64) {
            const int g = g0 + lane;
            const int r0 = g < r.G ? r.offset[g] : 0, r1 = g < r.G ? r.offset[g + 1] : 0;
            const int n = narrow_tiles(r1 - r0, Cfg::ROWS);
            int incl = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int up = __shfl_up(incl, d, 64);
                if (lane >= d) incl += up;
            }
            if (g < r.G) { s_pref[g] = before + incl - n; s_row0[g] = r0; }
            if (g == r.G - 1) { s_pref[r.G] = before + incl; s_row0[r.G] = r1; }
            before += __shfl(incl, 63, 64);
        }
    }
    __syncthreads();
    const uint8_t* tokens = GATE ? s_token : nullptr;
    const int r_total = __builtin_amdgcn_readfirstlane(s_pref[r.G]) * r_nt, r_xcd = (r_total + 7) >> 3;
    for (; slot < s_xcd + r_xcd; slot += gridDim.x >> 3) {
        if (!GATE && slot < s_xcd) {
            shared_tile();
        } else {
            const int L = xcd * r_xcd + slot - s_xcd;
            if (L >= r_total) continue;
            int lo = 0, hi = r.G;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_pref[mid] * r_nt <= L) lo = mid; else hi = mid;
            }
            const int g = __builtin_amdgcn_readfirstlane(lo);
            const int pref = __builtin_amdgcn_readfirstlane(s_pref[g]), mt = __builtin_amdgcn_readfirstlane(s_pref[g + 1]) - pref;
            const int row_a = __builtin_amdgcn_readfirstlane(s_row0[g]), rows = __builtin_amdgcn_readfirstlane(s_row0[g + 1]) - row_a;
            const int l = L - pref * r_nt, ni = l / mt, mi = l - ni * mt;
            const int h = narrow_height(rows, mt);
            narrow_dispatch<Cfg, SWIGLU, PACKED>(r, g, row_a + mi * h, min(h, rows - mi * h), h, mt, ni * COLS, wave, tid, lds, tokens);
        }
    }
}

// The down projection and the weighted sum of a few tokens in one launch.  A workgroup owns 16 or 8 output columns: its wavefronts
// share out the experts that have a row (the shared ones, a single reduction, first), leave the results in LDS, rounded as the
// expert outputs in memory would be, and add them up in the order of combine.hip.  As two launches the second one, its gap and
// the first one's last tiles are 8 us or more of one token's forward: the weights of every column are drawn from the start here, by
// eight wavefronts per workgroup, and the expert outputs never leave the compute unit.  The token rows are read as operands,
// by every workgroup again (out of L2): at 16 rows per expert as many bytes as the weights, which is where it ends (narrow_sum_fits, narrow_sum_pays).
struct SumArgs { const int32_t* pos; const float* w; int Tn, k; bool shared_alone; uint16_t* out; };

// 16 bytes of the lane eight further on in its row of 16 lanes
__device__ __forceinline__ uint4 from_other_half(const uint4& v)
{
    const auto turn = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x128, 0xF, 0xF, false); };
    return make_uint4(turn(v.x), turn(v.y), turn(v.z), turn(v.w));
}

// COLS columns of the tokens of one expert.  An operand of which 8 of 16 rows are there comes with one load instead of two: lanes
// 0 .. 7 of a row of 16 lanes hold the first half of the K step, lanes 8 .. 15 the second; what the matrix instruction makes of the
// other 8 rows is not stored.
template <bool PACKED, int COLS, int ROWS>
__device__ __forceinline__ void sum_item(const GemmArgs& a, int g, int row0, int nrows, int n, int lane, char* turn, uint16_t* y)
{
    constexpr int WL = COLS / 8, XL = ROWS / 8, D = sum_loads(PACKED) / (WL + XL);   // loads of a K step; K steps in flight
    const int KT = a.K / kPackK, half = lane >> 3 & 1;
    const char* wk;
    uint32_t w_off, w_half;
    long long w_step, seg_jump = 0;
    int seg_steps = KT;
    if (PACKED) {
        const int NT = (a.N + kPackRows - 1) / kPackRows, nt = n / kPackRows, blk = (n - nt * kPackRows) / 16;
        wk = reinterpret_cast<const char*>(a.Wp + (((size_t)g * NT + nt) * KT * kPackRows + blk * 16) * kPackK);
        w_off = COLS == 16 ? lane * 16u : half * 1024u + (lane >> 4) * 256u + ((n & 8) + (lane & 7)) * 16u;
        w_half = 1024;
        w_step = (long long)kPackRows * kPackK * 2;
    } else {
        wk = reinterpret_cast<const char*>(a.W + (size_t)g * a.w_group_stride + (size_t)n * a.ldw);
        w_off = (uint32_t)(lane >> 3) * (uint32_t)a.ldw * 2u + (lane & 7) * 16u;
        w_half = 8u * (uint32_t)a.ldw * 2u;
        w_step = kPackK * 2;
        seg_steps = a.kseg_len / kPackK;
        seg_jump = (a.w_kseg_stride - a.kseg_len) * 2;
    }
    const char* xk = reinterpret_cast<const char*>(a.A + (size_t)row0 * a.lda);
    const uint32_t x_off = (uint32_t)min(lane & (ROWS - 1), nrows - 1) * (uint32_t)a.lda * 2u + (ROWS == 8 ? half * 64u : 0u) + (lane >> 4) * 16u;
    uint4 w[D][WL], x[D][XL];
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    int seg = seg_steps;
    auto load = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < WL; ++h) w[slot][h] = load16<2>(wk, w_off, h * w_half);
#pragma unroll
        for (int h = 0; h < XL; ++h) x[slot][h] = load16(xk, x_off, h * 64);
        wk += w_step;
        xk += kPackK * 2;
        if (--seg == 0) { seg = seg_steps; wk += seg_jump; }
    };
    auto multiply = [&](int slot) __attribute__((always_inline)) {
        bf16x8_t f[2];
        if (PACKED) {
            f[0] = __builtin_bit_cast(bf16x8_t, w[slot][0]);
            f[1] = __builtin_bit_cast(bf16x8_t, WL == 2 ? w[slot][WL - 1] : from_other_half(w[slot][0]));
        } else turn_block(w[slot], lane, turn, f);
        const uint4 x1 = XL == 2 ? x[slot][XL - 1] : from_other_half(x[slot][0]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[0], __builtin_bit_cast(bf16x8_t, x[slot][0]), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[1], __builtin_bit_cast(bf16x8_t, x1), acc, 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < KT) load(d);
    int kt = 0;
    for (; kt + 2 * D <= KT; kt += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d);
            load(d);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay D steps ahead of their use
        }
    }
    for (; kt < KT; kt += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (kt + d < KT) multiply(d);
            if (kt + D + d < KT) load(d);
        }
    }
    const int r = lane & 15, c = (lane >> 4) * 4;
    if (r < nrows && c < COLS) *reinterpret_cast<uint2*>(y + r * COLS + c) = make_uint2(pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]));
}

template <bool PACKED, int COLS>
__global__ __launch_bounds__(kSumWaves * 64, 4) void narrow_sum_kernel(GemmArgs r, GemmArgs s, SumArgs a)
{
    __shared__ uint32_t s_item[kNarrowMaxGroups];   // groups with a row: group, first row, rows
    __shared__ int s_items, s_next;
    __shared__ __align__(16) char s_turn[PACKED ? 16 : kSumWaves * kTurnBytes];
    extern __shared__ __align__(16) char dyn[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slots = a.Tn * a.k, n = blockIdx.x * COLS, first = s.G > 0 ? 1 : 0;
    uint16_t* y = reinterpret_cast<uint16_t*>(dyn);            // [slots] rows of the routed experts, [Tn] of the shared ones
    int* s_pos = reinterpret_cast<int*>(dyn + (size_t)(slots + a.Tn) * COLS * 2);
    float* s_w = reinterpret_cast<float*>(s_pos + slots);
    if (wave == 0) {
        int items = 0;
        for (int g0 = 0; g0 < r.G; g0 += 64) {
            const int g = g0 + lane, r0 = g < r.G ? r.offset[g] : 0, rows = g < r.G ? r.offset[g + 1] - r0 : 0;
            const unsigned long long has = __ballot(rows > 0);
            if (rows > 0) s_item[items + __popcll(has & ((1ull << lane) - 1ull))] = (uint32_t)g << 20 | (uint32_t)r0 << 8 | (uint32_t)rows;
            items += __popcll(has);
        }
        if (lane == 0) { s_items = items; s_next = kSumWaves; }
    } else {
        for (int i = tid - 64; i < slots; i += kSumWaves * 64 - 64) { s_pos[i] = a.pos[i]; s_w[i] = a.w[i]; }
    }
    __syncthreads();
    const int items = __builtin_amdgcn_readfirstlane(s_items) + first;
    char* turn = s_turn + (PACKED ? 0 : wave * kTurnBytes);
    for (int i = wave; i < items;) {
        const uint32_t it = i < first ? (uint32_t)slots << 8 | (uint32_t)a.Tn : __builtin_amdgcn_readfirstlane(s_item[i - first]);
        const int g = it >> 20, row = it >> 8 & 0xfff, rows = it & 0xff;
        const GemmArgs& e = i < first ? s : r;
        const int row0 = i < first ? 0 : row;
        if (rows <= 8) sum_item<PACKED, COLS, 8>(e, g, row0, rows, n, lane, turn, y + (size_t)row * COLS);
        else sum_item<PACKED, COLS, 16>(e, g, row0, rows, n, lane, turn, y + (size_t)row * COLS);
        int next = 0;
        if (lane == 0) next = atomicAdd(&s_next, 1);
        i = __builtin_amdgcn_readfirstlane(next);
    }
    __syncthreads();
    const uint32_t* y2 = reinterpret_cast<const uint32_t*>(y);
    for (int i = tid; i < a.Tn * (COLS / 2); i += kSumWaves * 64) {
        const int t = i / (COLS / 2), c = i % (COLS / 2);
        float lo = 0.f, hi = 0.f;
        bool kept = false;
        for (int j = t * a.k; j < (t + 1) * a.k; ++j) {
            const int p = s_pos[j];
            if (p < 0) continue;
            const uint32_t v = y2[p * (COLS / 2) + c];
            lo = fmaf(s_w[j], bf16_lo(v), lo);
            hi = fmaf(s_w[j], bf16_hi(v), hi);
            kept = true;
        }
        uint32_t o = 0;
        if (first) o = y2[(slots + t) * (COLS / 2) + c];
        if (kept || !first || !a.shared_alone) {
            if (first) { lo = fmaf(1.0f, bf16_lo(o), lo); hi = fmaf(1.0f, bf16_hi(o), hi); }
            o = pack_bf16x2(lo, hi);
        }
        *reinterpret_cast<uint32_t*>(a.out + (size_t)t * r.N + n + c * 2) = o;
    }
}

static bool narrow_args_fit(const GemmArgs& a)
{
    if (a.K < kPackK || a.K % kPackK || a.kseg_len < kPackK || a.kseg_len % kPackK || a.N < 64 || a.N % 64) return false;
    if (a.G < 1 || a.G > kNarrowMaxGroups || a.epi != 0) return false;
    // lanes address token rows and a block of weight rows with 32-bit byte offsets
    const long long rows = a.a_row_map ? a.a_src_rows : kNarrowRows;
    if (rows * a.lda * 2 >= (1ll << 32) || 16ll * a.ldw * 2 >= (1ll << 32) || (a.a_row_map && a.a_row_div < 1)) return false;
    if (a.lda % 8 || a.ldw % 8 || a.w_group_stride % 8 || a.w_up_offset % 8 || a.w_kseg_stride % 8) return false;
    if ((reinterpret_cast<uintptr_t>(a.A) | reinterpret_cast<uintptr_t>(a.W) | reinterpret_cast<uintptr_t>(a.Wp)) & 15) return false;
    return !(a.ldc % 4 || a.c_group_col_stride % 4 || (reinterpret_cast<uintptr_t>(a.C) & 7));
}

bool narrow_gate_pays(int Tn, int k, int El, int H, int n_cu)
{
    const double wgs = (double)(Tn * k < El ? Tn * k : El) * ((H + 63) / 64) / n_cu;   // of a compute unit
    return k * (wgs - kGateFree) <= kGateWorth;
}

hipError_t launch_narrow_gemm(const GemmArgs& routed, const GemmArgs* shared, bool swiglu, int n_cu, double expected_rows,
                              int max_tokens, long long max_rows, hipStream_t s, int* kind, const GateArgs* gate)
{
    GemmArgs none{};
    const GemmArgs& sh = shared ? *shared : none;
    if (routed.offset == nullptr || max_rows < 1 || !narrow_args_fit(routed)) return hipErrorInvalidValue;
    if (shared && (sh.dense_rows < 1 || (sh.Wp != nullptr) != (routed.Wp != nullptr) || !narrow_args_fit(sh))) return hipErrorInvalidValue;
    // Workgroups: every tile one of its own (a compute unit holds two at a time and takes the next when one
    // ends) as far as the host can foresee the routing; groups with more rows than expected are reached by the
    // kernel's loop over tile ids.
    const long long filled = max_rows < routed.G ? max_rows : routed.G;
    const auto grid_for = [&](int tallest, int cols, long long groups) {
        const auto col_tiles = [&](const GemmArgs& a) { return (long long)(a.N + cols - 1) / cols; };
        const long long s_tiles = shared ? col_tiles(sh) * narrow_tiles(sh.dense_rows, tallest) * sh.G : 0;
        const long long most = groups + max_rows / tallest;
        long long r_tiles = (long long)(groups * (1.0 + expected_rows / tallest));
        if (r_tiles > most) r_tiles = most;
        const long long grid = (s_tiles + 7) / 8 * 8 + (r_tiles * col_tiles(routed) + 7) / 8 * 8;
        return grid < 8 ? 8 : grid > (1 << 20) ? 1 << 20 : grid;
    };
    if (gate && (!swiglu || gate->Tn < 1 || gate->Tn > kGateTokens || gate->E < 1 || gate->E > kGateExperts || gate->k < 1 || gate->k > 64 || gate->k > gate->E))
        return hipErrorInvalidValue;
    // no group has more than max_tokens rows: one row tile each
    const bool one_block = max_tokens <= NarrowFew::ROWS && (!shared || sh.dense_rows <= NarrowFew::ROWS);
    const bool two_blocks = max_tokens <= NarrowPair::ROWS && (!shared || sh.dense_rows <= NarrowPair::ROWS);
    // Only the tiles a gate/up projection of one block of rows takes exist with a gate; any other launch would read the
    // rows an earlier call has partitioned.
    static_assert(kGateTokens <= NarrowFew::ROWS && kGateTokens <= NarrowFine::ROWS, "the gate's own tokens are one block");
    if (gate && (!one_block || gate->Tn > max_tokens)) return hipErrorInvalidValue;
    const GateArgs route = gate ? *gate : GateArgs{};
    const auto go = [&](auto kernel, long long grid, int threads) { hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(threads), 0, s, routed, sh, route); };
    const auto with = [&](auto cfg, auto sw) {
        using Cfg = decltype(cfg);
        constexpr bool SW = decltype(sw)::value;
        const long long grid = grid_for(Cfg::ROWS, narrow_cols<Cfg, SW>(), filled);
        if constexpr (SW && (std::is_same_v<Cfg, NarrowStream> || std::is_same_v<Cfg, NarrowFine>))   // what a gate/up projection of one block of rows takes
            if (gate) {
                if (routed.Wp) go(narrow_gemm_kernel<Cfg, true, true, true>, grid, Cfg::THREADS);
                else go(narrow_gemm_kernel<Cfg, true, false, true>, grid, Cfg::THREADS);
                return;
            }
        if (routed.Wp) go(narrow_gemm_kernel<Cfg, SW, true>, grid, Cfg::THREADS);
        else go(narrow_gemm_kernel<Cfg, SW, false>, grid, Cfg::THREADS);
    };
    // of a share, about `kept` rows stay here
    const long long kept = (long long)(expected_rows * routed.G + 0.999);
    *kind = !swiglu && one_block && grid_for(kNarrowRows, narrow_cols<NarrowStream, false>(), kept < filled ? kept : filled) <= n_cu ? 1 : 0;
    if (two_blocks && routed.K >= kNarrowFineK && (!shared || sh.K >= kNarrowFineK)) {
        // What the busiest compute unit draws (columns times K) out of tiles of w wavefronts spread evenly, the experts
        // expected to have a row each.  Smaller tiles where that is less; with a short K the launch is start-up.  Forwards, us,
        // tiles of four (down: two) wavefronts / one: DeepSeek-V2-Lite-shaped layer, 1 / 2 / 4 / 8 tokens 42.6 / 40.2, 62.1 / 57.0, 88.3 /
        // 82.1, 127 / 120; DeepSeek-V2-shaped share, 1 / 4 / 16 tokens 58.0 / 49.2, 65.5 / 60.3, 130 / 111; Qwen3-235B-A22B-shaped share, 1 / 2
        // tokens 25.2 / 21.6, 31.8 / 26.8; with 8 K steps in flight instead of 4 44.4, 61.6, 90.7, 134; 52.5, 62.2, 118; 23.2, 30.0.
        // Four / two wavefronts, 32 rows: DeepSeek-V2-shaped share, 20 / 33 tokens 135 / 120, 145 / 135, Qwen3-235B-A22B-shaped share, 24 / 32
        // tokens 103 / 95, 104 / 100; with its load skewed, 20 / 32 tokens: Zipf 1.1 52 / 42, 58 / 54, all on 16 of its experts 115 / 113, 118 /
        // 116, on 12 105 / 97, 108 / 103.  The mean alone decides, though where all tokens choose the same eight experts, 128-column
        // tiles are one per compute unit, 64-column ones stage every token row twice: 66 / 69, 70 / 75 (weights in the caller's layout
        // 78 / 75, 79 / 75; DeepSeek-V2-shaped share 103 / 103, 102 / 97).  Beyond 32 tokens an expert can have a second
        // tile: balanced loads of 33 to 64 tokens still gain 1 - 4 %, all tokens on eight experts lose 25 %.
        // Over 1599 layers of 1024 to 7168 columns, H 256 to 5120, 1 to 256 experts, 1 to 32 tokens, none shared: 4.1 % of the time in all, 1008 layers gain
        // 3 % and more, 42 lose it (10 % at most).
        const double worth = shared ? (double)sh.K / routed.K : 0.0, touched = routed.G * (1.0 - std::exp(-expected_rows));
        const auto busiest = [&](int w) {
            const int cols = w * (swiglu ? 16 : 32);
            const double tiles = (double)((routed.N + cols - 1) / cols) * touched + (shared ? worth * ((sh.N + cols - 1) / cols) * sh.G : 0.0);
            return w * std::fmax(std::ceil(tiles / n_cu), worth);
        };
        const double now = busiest(*kind ? kNarrowFewWaves : kNarrowWaves);
        if (one_block) { if (busiest(1) < now) *kind = 2; }
        else if (busiest(kNarrowFewWaves) < now) *kind = 3;
    }
    const auto pick = [&](auto sw) {
        if (*kind == 3) with(NarrowPair{}, sw);
        else if (*kind == 2) with(NarrowFine{}, sw);
        else if (*kind == 1) with(NarrowFew{}, sw);
        else with(NarrowStream{}, sw);
    };
    if (swiglu) pick(std::true_type{}); else pick(std::false_type{});
    return hipGetLastError();
}

hipError_t launch_narrow_sum(const GemmArgs& routed, const GemmArgs* shared, const int32_t* pos, const float* w, int Tn, int k,
                             bool shared_alone, void* out, int n_cu, hipStream_t s)
{
    GemmArgs none{};
    const GemmArgs& sh = shared ? *shared : none;
    if (Tn < 1 || Tn > kSumRows || k < 1 || k > 64 || routed.offset == nullptr || routed.a_row_map || !narrow_args_fit(routed)) return hipErrorInvalidValue;
    if (shared && (sh.G != 1 || sh.dense_rows != Tn || sh.N != routed.N || (sh.Wp != nullptr) != (routed.Wp != nullptr) || !narrow_args_fit(sh)))
        return hipErrorInvalidValue;
    if (reinterpret_cast<uintptr_t>(out) & 3) return hipErrorInvalidValue;
    const SumArgs sum{pos, w, Tn, k, shared_alone, static_cast<uint16_t*>(out)};
    const auto go = [&](auto kernel, int cols) {
        const size_t lds = (size_t)(Tn * k + Tn) * cols * 2 + (size_t)Tn * k * 8;
        hipLaunchKernelGGL(kernel, dim3(routed.N / cols), dim3(kSumWaves * 64), lds, s, routed, sh, sum);
    };
    if (narrow_sum_cols(routed.N, n_cu) == 8) { if (routed.Wp) go(narrow_sum_kernel<true, 8>, 8); else go(narrow_sum_kernel<false, 8>, 8); }
    else { if (routed.Wp) go(narrow_sum_kernel<true, 16>, 16); else go(narrow_sum_kernel<false, 16>, 16); }
    return hipGetLastError();
}

}  // namespace moe_ep
