// Expert projections out of workgroups whose loads and multiplications are different wavefronts (Sec. 3.1): the tiled
// form of prefill, routed experts (ragged groups) with or without the shared ones (dense groups) in the same launch.
//
// What bounds a tile is loads that a K step has to wait for: they draw 80 GB/s from L2 and 46 GB/s from HBM for a compute unit (nothing but
// loads, never waited for together, 140 GB/s from L2, 64 bytes a cycle), and a K step of a 160 x 256 tile is 52 KB.  With the multiplications taken
// out, the loads alone were three quarters of a launch (Qwen3-30B-A3B-shaped layer, 8192 tokens, gate/up 345 of 437 us); with the loads taken out,
// the multiplications alone were 87 / 82 % of a gate/up / down launch (DeepSeek-V2-Lite-shaped layer, 4096 tokens).  The results' way out is the rest: with and
// without its stores that layer's forward takes 553 / 513 us, the Qwen3-30B-A3B-shaped one's, 8192 skewed tokens, 689 / 627.  In
// grouped_gemm.hip a wavefront loads and multiplies, and a load that finds the path full holds back the MFMAs behind it.  A launch is
// also bound by how its tiles are dealt, by number: of several rounds 6 to 16 % of the units' time has no workgroup, of one row tile per
// expert up to 30 (profiles/loader_gemm_counters.txt, where the matrix pipes are busy 54 - 59 % of a gate/up launch that fills the chip).
// Here four wavefronts only load and eight only multiply, so that the two overlap whatever each waits for:
//  - Loading: global_load_lds into two rings, the weights (three slots of 32 KB, two K steps ahead) and the token rows
//    (two slots, one K step ahead).  Each wavefront counts its own loads; one barrier of the workgroup per K step hands a
//    slot over and takes one back.  The next tile's coordinates, row map and base addresses are theirs too.
//  - Multiplying: two rows of four wavefronts, each half of the tile's 16-row blocks times 64 of its 256 weight rows, two
//    wavefronts per SIMD.  Fragments are read a few blocks ahead of v_mfma_f32_16x16x32_bf16.
// Twelve wavefronts leave 168 registers each: 96 accumulators, hence 192 rows.  The K loop and the epilogue are compiled for
// every number of row blocks, so that a tile multiplies the blocks it has: 143 rows are 9 blocks instead of 10, 94 rows 6
// instead of 8, and the row tiles of a group are of equal height.  Four multiplying wavefronts with 160 rows (1 x 4, 256
// registers) were 3 to 6 % slower with 256 and more rows per expert and the same below; 224 rows (7 blocks a
// wavefront, 168 registers) gain where they save a tile per expert (615 rows: 1 - 2 %) and lose as much where the tiles then miss
// their last round.  Also tried: weights fetched into L2 ahead by a wavefront of their own, tiles sharing the lines
// (loads alone 2 - 4 % faster, launches the same); drawing tiles from counters instead of dealing them (start-up 5 us
// longer, nothing won back, with one projection in a launch); cache policy bits (nt slower, the others equal); wavefront priorities (equal).
// Forwards before / with these kernels, us: DeepSeek-V2-Lite-shaped layer, 4096 tokens 614 / 568, 1531 tokens, weights in the
// caller's layout 342 / 304; Qwen3-30B-A3B-shaped layer, 8192 tokens 723 / 650, skewed 735 / 693; DeepSeek-V2-shaped share,
// 1600 / 2502 / 5000 tokens 341 / 289, 421 / 386, 680 / 622; Qwen3-235B-A22B-shaped share, 1024 / 2048 tokens 135 / 128, 152 / 142.
//
// Both projections of a layer can be one launch.  What a launch of several rounds loses at its end then is lost once (6 to 20 % of the units' time
// of either launch had no workgroup): tiles are drawn from counters, gate/up before down, and a down tile waits until its row tile's activation is
// complete, which it nearly always is.  The activation goes through L2 to memory, a line's counter per row tile says when it is there.  What
// mattered, forwards of the Qwen3-235B-A22B-shaped share with 1024 tokens, us (launches of their own 119): counters of several row tiles in one line and four
// wavefronts asking 183, a line each and one asking 131; a count raised by every wavefront instead of the last of eight 8 us of a launch.
// Arguments in LDS instead of in scalar registers, DeepSeek-V2-Lite-shaped layer, 4096 tokens: 566 / 554; flat instead of global stores of results, whose
// addresses then come from LDS, 561 / 553 (the compiler holds up every LDS read behind them).  One projection's tiles drawn instead of dealt: 119 / 123 for the former.
//
// Every output element is accumulated over K in the order of grouped_gemm.hip by the same instruction, and the epilogue
// rounds at the same place: the results are the same bits.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace moe_ep {

namespace {

constexpr int kLdGroups = 512;
constexpr int kLdBlocks = kLoaderRows / 16;                 // 16-row blocks of the tallest tile
constexpr int kLdLowBlocks = 8;                             // of one where lower tiles take no more rounds
constexpr int kLdWSlots = 3, kLdXSlots = 2;                 // ring slots, a K step of 64 each
constexpr int kLdWBytes = kPackRows * kPackK * 2;           // weights of a slot, 128 bytes a row
constexpr int kLdXBytes = kLoaderRows * kPackK * 2;         // token rows of a slot
constexpr int kLdXRing = kLdWSlots * kLdWBytes;             // where the token rows' ring begins
constexpr int kLdRing = kLdXRing + kLdXSlots * kLdXBytes;
constexpr int kLdCache = 32;                                // tiles of a workgroup decoded ahead
constexpr int kLdMultiply = 8, kLdLoad = 4;                 // wavefronts
constexpr int kLdThreads = (kLdMultiply + kLdLoad) * 64;
constexpr int kLdWRegions = kPackRows / 8 / kLdLoad;        // 1 KB regions (8 rows) of weights a loading wavefront fetches per K step
constexpr int kLdXRegions = kLoaderRows / 8 / kLdLoad;      // and of token rows, at most
constexpr int kLdDrawAhead = 6, kLdDrawSteps = 8;           // K steps of weights left when the next tiles are drawn; K steps drawn at a time, at least
constexpr int kXcds = 8, kLdLine = 32, kLdListBytes = 88;                     // integers of a line: a counter of its own
static_assert(kLdCounters == 4 * kXcds * kLdLine, "two lists of each projection, a share per XCD");
constexpr int kLdTold = 3;                                  // tiles whose multiplying wavefronts may be counted at a time (Told)
constexpr int loader_lds(int groups) { return kLdRing + kLdCache * (16 + 4 + 4) + 4 * kLdListBytes + (2 + kLdTold + 2 * (groups + 1)) * 4; }

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4_t global_u32x4;   // an address that comes from LDS is not known to be global: a flat store would hold up LDS reads
struct Cut { int tiles, base, rem; };   // row tiles of base blocks, the first rem of them one more
__device__ __forceinline__ Cut cut_rows(int rows, int most)   // most: blocks of the tallest, kLdLowBlocks or kLdBlocks
{
    Cut c;
    const int u = (rows + 15) / 16;
    c.tiles = most == kLdLowBlocks ? (u + kLdLowBlocks - 1) / kLdLowBlocks : (u + kLdBlocks - 1) / kLdBlocks;
    c.base = c.tiles ? u / c.tiles : 0;
    c.rem = c.tiles ? u - c.base * c.tiles : 0;
    return c;
}

struct Tile { int g, row0, nrows, ni, blocks, once, dense, down, dep; };   // ni: column tile; dep: row tile, as kLdCounters counts them
constexpr int kTileDense = 1 << 15, kTileDown = 1 << 16;    // beside the group in a tile's first word

// s_waitcnt vmcnt(N): the other counters untouched
template <int N>
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70); }
// this wavefront's LDS accesses are done, then the workgroup's
__device__ __forceinline__ void hand_over()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

#define SB() __builtin_amdgcn_sched_barrier(0)

// where a wavefront's results go: its columns of the tile's first row; columns from n_left on are not there
struct Out { uint16_t* c; int ldc, nrows, n_left; };

// ring slots of a K step, as bytes
struct Slots {
    uint32_t w, x;
    __device__ __forceinline__ Slots next() const
    {
        return {w == (kLdWSlots - 1) * kLdWBytes ? 0u : w + kLdWBytes, x == kLdXRing + (kLdXSlots - 1) * kLdXBytes ? (uint32_t)kLdXRing : x + kLdXBytes};
    }
};

// What tiles read of their launch arguments, in LDS: a list is the dense or the ragged tiles of one projection.  Four lists' arguments in scalar
// registers would not fit, and every K step would fetch some of them back from where they were put.
struct List {
    const uint16_t *A, *W;
    uint16_t* C;
    long long w_group_stride, w_kseg_stride, w_up_offset;
    int lda, ldw, ldc, N, K, kseg_len, c_group_col_stride, groups, nt, pad;
};

// a value that all lanes have, in scalar registers
template <class T>
__device__ __forceinline__ T same(T x)
{
    if constexpr (sizeof(T) == 8) {
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
        return __builtin_bit_cast(T, (uint64_t)hi << 32 | lo);
    } else return __builtin_amdgcn_readfirstlane(x);
}

// a lane's offset as the 32 bits that a load adds to its scalar base; as 64 the sums would be made, and waited for, before every load
__device__ __forceinline__ uint32_t in_32_bits(uint32_t x)
{
    asm("" : "+v"(x));
    return x;
}

// another tile of the same projection follows: its first word, which is there once a tile's last K step has been handed over
template <bool SWIGLU>
__device__ __forceinline__ bool goes_on(const int4* next)
{
    const int x = __builtin_amdgcn_readfirstlane(next->x);
    return x >= 0 && !(x & kTileDown) == SWIGLU;
}

// A gate/up tile whose rows a down tile of the launch will read: its row tile's count, and in LDS how many of the multiplying wavefronts have their
// share in memory.  A tile is told of behind the next one's K loop, the last gate/up tile behind its own.  With one K step a wavefront meets
// no hand-over in that one and tells of three tiles in a row, the first of which others may still have to tell of: kLdTold such numbers in turn.
struct Told { int32_t* done; int* waves; };
__device__ __forceinline__ void tell(const Told& t)
{
    SB();
    wait_loads<0>();   // counts stores too, which go through to memory
    SB();
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    if (lane == 0 && (__hip_atomic_fetch_add(t.waves, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & (kLdMultiply - 1)) == kLdMultiply - 1)
        __hip_atomic_fetch_add(t.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// N row blocks of a tile.  xa, wa: the lane's bytes into a slot's token rows and weights; off: the ring slots of the tile's
// first K step, handed over; on return those of the next tile's first one.  next_tile: as decoded; told: the tile before this one, told of when its
// stores have had a K loop's time.  Returns whether another tile of this projection follows, its first K step handed over.
template <int N, bool SWIGLU, bool PACKED, bool THROUGH>
__device__ __forceinline__ bool run_tile(const char* lds, uint32_t xa, uint32_t wa, int KT, const int4* next_tile, const Told& told, Slots& off, const Out& out)
{
    bool more = true;
    f32x4_t acc[N][4];
    constexpr int S = 2 * N;                                  // row blocks times the two halves of a K step
    constexpr int P = S < 4 ? S : 4;                         // token fragments read before a K step starts
    constexpr int T = N >= 5 ? 3 : N >= 3 ? 2 : 1;            // the next K step's slot is handed over T blocks before the end
    constexpr int H = S - T, LB = H - 1 > 1 ? H - 1 : 1;      // the slot's last reads are issued in block LB - 1
    constexpr int LATE = S - P + 4;                           // reads of a K step behind its start: token fragments, the second half's weights
    static_assert(H >= N, "the first half's weights are free when the next ones arrive");
    bf16x8_t w0[4], w1[4], xn[P];
    const auto read_x = [&](const Slots& slot, int r) __attribute__((always_inline)) {
        const uint32_t a = r / N ? (slot.x + xa) ^ 64u : slot.x + xa;
        return *reinterpret_cast<const bf16x8_t*>(lds + a + (r % N) * 2048);
    };
    const auto read_w = [&](const Slots& slot, int j, int nb) __attribute__((always_inline)) {
        if (PACKED) return *reinterpret_cast<const bf16x8_t*>(lds + (slot.w + wa) + ((SWIGLU ? 2 * (nb & 1) + (nb >> 1) : nb) * 2048 + j * 1024));
        const uint32_t a = j ? (slot.w + wa) ^ 64u : slot.w + wa;
        return *reinterpret_cast<const bf16x8_t*>(lds + a + (SWIGLU ? (nb < 2 ? nb * 16 : 128 + (nb - 2) * 16) : nb * 16) * 128);
    };
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) w0[nb] = read_w(off, 0, nb);
#pragma unroll
    for (int r = 0; r < P; ++r) xn[r] = read_x(off, r);
#pragma unroll
    for (int mb = 0; mb < N; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // the compiler does not know the hand-written MFMAs' latencies: wait states behind the zeroing moves
    SB();
    asm volatile("s_nop 7");
    SB();
    for (int kt = 0; kt < KT; ++kt) {
        const Slots next = off.next();
        if (kt + 1 == KT) more = goes_on<SWIGLU>(next_tile);
        bf16x8_t x[S];
#pragma unroll
        for (int r = 0; r < P; ++r) x[r] = xn[r];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (s == H && more) hand_over();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int nb = (s & 1) ? 3 - q : q;
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[s % N][nb]) : "v"(s < N ? w0[nb] : w1[nb]), "v"(x[s]));
                // the slot's remaining reads, evenly behind the first LB blocks: token fragments of the first half, the
                // second half's weights, its token fragments
                if (s < LB) {
                    constexpr int XA = N > P ? N - P : 0;
                    const int q0 = 4 * s + q;
                    for (int i = q0 * LATE / (4 * LB); i < (q0 + 1) * LATE / (4 * LB); ++i) {
                        if (i < XA) x[P + i < S ? P + i : 0] = read_x(off, P + i);
                        else if (i < XA + 4) w1[i - XA < 4 ? i - XA : 0] = read_w(off, 1, i - XA);
                        else x[P + i - 4 < S ? P + i - 4 : 0] = read_x(off, P + i - 4);
                    }
                } else if (s >= H) {   // the next K step's first ones
                    const int q0 = 4 * (s - H) + q;
                    for (int i = q0 * (4 + P) / (4 * T); i < (q0 + 1) * (4 + P) / (4 * T); ++i) {
                        if (i < 4) w0[i] = read_w(next, 0, i);
                        else xn[i - 4 < P ? i - 4 : 0] = read_x(next, i - 4);
                    }
                }
                SB();
            }
        }
        off = next;
    }
    // and before the epilogue's accumulator reads
    SB();
    asm volatile("s_nop 15");
    asm volatile("s_nop 15");
    SB();
    // A lane holds token row (lane & 15) of each block and output columns 4 * (lane >> 4) + {0..3} of it.  Two neighbouring column
    // blocks exchange halves, so that it has 8 consecutive columns of one of them, and the lanes trade places: four neighbours then
    // store 64 consecutive bytes of a row, which leave a compute unit four at a time; 16 bytes of 16 rows in turn kept a down
    // launch waiting (DeepSeek-V2-Lite-shaped layer, 4096 tokens, down launch 196 / 191 us, the launch without its epilogue 160).
    int lane;   // asked for here: kept over the K loop it would cost a register
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    if (THROUGH && told.done) tell(told);
    const int row = lane >> 2, col = (lane & 3) * 8;
    const int from = (((lane & 1) * 2 + (lane >> 1 & 1)) * 16 + row) * 4;   // the lane that computed them, as ds_bpermute counts
    const uint32_t at = (uint32_t)(row * out.ldc + col) * 2u;
    const auto store = [&](auto guard) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < N; ++mb) {
            // a row of blocks is pinned in its registers right before its turn
            asm volatile("; accumulator row" : "+v"(acc[mb][0]), "+v"(acc[mb][1]), "+v"(acc[mb][2]), "+v"(acc[mb][3]));
            if (mb * 16 >= out.nrows) break;
#pragma unroll
            for (int nb = 0; nb < (SWIGLU ? 2 : 4); nb += 2) {
                uint32_t pk[2][2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    float h[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[i] = SWIGLU ? silu_f(acc[mb][nb + j][i]) * acc[mb][(nb + j + 2) & 3][i] : acc[mb][nb + j][i];
                    pk[j][0] = pack_bf16x2(h[0], h[1]);
                    pk[j][1] = pack_bf16x2(h[2], h[3]);
                }
                const auto s0 = __builtin_amdgcn_permlane16_swap(pk[0][0], pk[1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane16_swap(pk[0][1], pk[1][1], false, false);
                uint4 o;   // every lane takes part, also for rows and columns that are not there
                o.x = __builtin_amdgcn_ds_bpermute(from, s0[0]); o.y = __builtin_amdgcn_ds_bpermute(from, s1[0]);
                o.z = __builtin_amdgcn_ds_bpermute(from, s0[1]); o.w = __builtin_amdgcn_ds_bpermute(from, s1[1]);
                if (mb * 16 + row < out.nrows && !(decltype(guard)::value && nb * 16 + col >= out.n_left)) {
                    uint16_t* const c = out.c + (size_t)(mb * 16) * out.ldc + nb * 16;
                    if (THROUGH) {   // for other XCDs to read in this launch: through L2
                        const u32x4_t v = {o.x, o.y, o.z, o.w};
                        // (the wait states are those of a store of more than 64 bits before its registers are written again)
                        asm volatile("global_store_dwordx4 %0, %1, %2 sc1\n\ts_nop 1" ::"v"(at), "v"(v), "s"(c) : "memory");
                    } else {
                        const u32x4_t v = {o.x, o.y, o.z, o.w};
                        *(global_u32x4*)(reinterpret_cast<char*>(c) + at) = v;
                    }
                }
            }
        }
    };
    if (out.n_left >= (SWIGLU ? 32 : 64)) store(std::false_type{}); else store(std::true_type{});
    return more;
}

}  // namespace

// a launch argument of the tile's list, by value: a choice between the arguments themselves would keep them in scratch memory
template <bool UP, bool DOWN, class T>
__device__ __forceinline__ T pick(bool dense, bool down, T a1, T d1, T a2, T d2)
{
    const T u = dense ? d1 : a1, v = dense ? d2 : a2;
    return !UP || (DOWN && down) ? v : u;
}

// PROJ: 1 gate/up (a1, d1), 2 down (a2, d2), 3 both, the down projection reading what this launch's gate/up projection wrote.
// sync, of both: kLdCounters zeros where tiles are drawn from, and kRowTileInts zeros per row tile behind them.
template <int PROJ, bool PACKED>
__global__ __launch_bounds__(kLdThreads) void loader_gemm_kernel(GemmArgs a1, GemmArgs d1, GemmArgs a2, GemmArgs d2, int32_t* sync)
{
    constexpr bool UP = (PROJ & 1) != 0, DOWN = (PROJ & 2) != 0, BOTH = UP && DOWN;
#define ARG(dense, down, field) (pick<UP, DOWN>(dense, down, a1.field, d1.field, a2.field, d2.field))
    const int G = ARG(false, false, G), d_rows = ARG(true, false, dense_rows);
    const bool shared = ARG(true, false, G) > 0;
    extern __shared__ uint4 lds4[];
    char* const lds = reinterpret_cast<char*>(lds4);
    int4* const s_tile = reinterpret_cast<int4*>(lds + kLdRing);
    static_assert(sizeof(List) == kLdListBytes, "loader_lds");
    List* const s_list = reinterpret_cast<List*>(s_tile + kLdCache);
    int* const s_dep = reinterpret_cast<int*>(s_list + 4);
    int* const s_ready = s_dep + kLdCache;   // down tiles whose activation rows are known to be in memory
    int* const s_filled = s_ready + kLdCache;
    int* const s_most = s_filled + 1;
    int* const s_waves = s_most + 1;
    int* const s_pref = s_waves + kLdTold;
    int* const s_row = s_pref + G + 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto columns_to_tiles = [&](int n, bool down) { return !UP || (DOWN && down) ? (n + kPackRows - 1) / kPackRows : (n + kPackRows / 2 - 1) / (kPackRows / 2); };

    if (tid < kLdTold) s_waves[tid] = 0;
    if (tid < 4) {
        const bool dense = tid & 1, down = tid >> 1;
        List l;
        l.A = ARG(dense, down, A); l.W = PACKED ? ARG(dense, down, Wp) : ARG(dense, down, W); l.C = ARG(dense, down, C);
        l.w_group_stride = ARG(dense, down, w_group_stride); l.w_kseg_stride = ARG(dense, down, w_kseg_stride); l.w_up_offset = ARG(dense, down, w_up_offset);
        l.lda = ARG(dense, down, lda); l.ldw = ARG(dense, down, ldw); l.ldc = ARG(dense, down, ldc); l.N = ARG(dense, down, N); l.K = ARG(dense, down, K);
        l.kseg_len = ARG(dense, down, kseg_len); l.c_group_col_stride = ARG(dense, down, c_group_col_stride);
        l.groups = ARG(dense, down, G); l.nt = columns_to_tiles(l.N, down); l.pad = 0;
        s_list[tid] = l;
    }
    for (int i = tid; i <= G; i += kLdThreads) s_row[i] = ARG(false, false, offset)[i];
    // Row tiles before every ragged group.  Tiles of at most kLdLowBlocks blocks where they take no more rounds (a dense tile counts as the
    // ragged ones it is worth) or are one for a workgroup all the same, since a round lasts as long as its tallest tile -- unless they are only a
    // few more (a seventh), which cost more than the others gain, in a launch that keeps three quarters of the workgroups busy.  Of 9824
    // launches of 1 to 256 experts (2 to 5800 rows each, skewed and not, shared experts beside them or not) this leaves 0.3 % of the time to the
    // better one of both, tiles of up to 12 blocks always 5.7 %, of 8 always 6.5 %.  Forwards, 12 / this, us: one expert of 146 rows, 1536 x 1536,
    // 63 / 57, two of 174, 1408 x 7168, 153 / 127, 16 of about 160, 1024 x 2880, 83 / 63 (in grouped_gemm.hip, 128 rows, 55, 125, 77); 4 of the
    // DeepSeek-V2-shaped layer's experts and its shared ones, 2000 tokens 244 / 230 (231).
    // Of both projections, whose tiles are drawn, always the tall ones: DeepSeek-V2-shaped share, 2600 tokens this rule 378, tall 370, 5003 in two chunks 727 / 722,
    // DeepSeek-V2-Lite-shaped layer, 2000 / 4096 tokens 335 / 333, 543 / 543, Qwen3-30B-A3B-shaped layer, 3000 tokens 329 / 328, skewed, 5000 tokens 467 / 466.
    if (wave == 0) {
        constexpr int PER = kLdGroups / 64;
        const int32_t* const offset = ARG(false, false, offset);
        const int NT = columns_to_tiles(ARG(false, false, N), false), d_nt = columns_to_tiles(ARG(true, false, N), false), d_G = ARG(true, false, G);
        const int d_worth = shared ? max(1, (ARG(true, false, K) + ARG(false, false, K) / 2) / ARG(false, false, K)) : 1;
        // consecutive groups of a lane: one scan over the lanes, however many groups there are.  With one per 64 groups, a forward of 1000 tokens
        // on a few of 512 experts, 384 x 1536, took 84 us instead of 75 (in grouped_gemm.hip 75).
        const int per = (G + 63) >> 6, g0 = lane * per;
        int rows[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i >= per) break;
            rows[i] = g0 + i < G ? offset[g0 + i + 1] - offset[g0 + i] : 0;
        }
        int before, filled, low;   // low: how many more there would be of kLdLowBlocks, this lane's groups
        const auto count_tiles = [&](int most) {
            int mine = 0;
            filled = low = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (i >= per) break;
                const int n = cut_rows(rows[i], most).tiles;
                mine += n;
                low += cut_rows(rows[i], kLdLowBlocks).tiles - n;
                filled += __builtin_popcountll(__ballot(n > 0));
            }
            int incl = mine;
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const int up = __shfl_up(incl, s, 64);
                if (lane >= s) incl += up;
            }
            before = __shfl(incl, 63, 64);
            int at = incl - mine;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (i >= per) break;
                if (g0 + i < G) s_pref[g0 + i] = at;
                at += cut_rows(rows[i], most).tiles;
            }
            if (lane == 0) { s_pref[G] = before; *s_filled = filled; }
        };
        count_tiles(kLdBlocks);
        const auto dense_tiles = [&](int most) { return shared ? d_G * cut_rows(d_rows, most).tiles * d_nt : 0; };
        const int d_tall = dense_tiles(kLdBlocks), d_low = dense_tiles(kLdLowBlocks);
        int most = kLdBlocks;
        const bool recount = __ballot(low > 0) != 0;
        if (!BOTH && (recount || d_low != d_tall)) {   // tiles that are drawn run in no rounds
            if (recount)
#pragma unroll
                for (int s = 1; s < 64; s <<= 1) low += __shfl_xor(low, s, 64);
            const int wgs = (int)gridDim.x, tall = before * NT + d_tall * d_worth, tiles = (before + low) * NT + d_low, lower = tiles + d_low * (d_worth - 1);
            if ((tiles <= wgs || lower <= (tall + wgs - 1) / wgs * wgs) && (lower - tall > tall / 7 || tiles <= wgs - wgs / 4)) {
                most = kLdLowBlocks;
                if (recount) count_tiles(most);
            }
        }
        if (lane == 0) *s_most = most;
    }
    __syncthreads();
    const int row_tiles = __builtin_amdgcn_readfirstlane(s_pref[G]), most = __builtin_amdgcn_readfirstlane(*s_most);
    const int d_mt = shared ? cut_rows(d_rows, most).tiles : 0;
    const auto list_of = [&](bool dense, bool down) -> const List& { return s_list[(down ? 2 : 0) + (dense ? 1 : 0)]; };
    const auto col_tiles = [&](bool dense, bool down) { return list_of(dense, down).nt; };
    const auto tiles_of = [&](bool dense, bool down) { return (dense ? list_of(true, down).groups * d_mt : row_tiles) * col_tiles(dense, down); };
    const auto steps_of = [&](bool dense, bool down) { return same(list_of(dense, down).K) / kPackK; };

    const auto decode = [&](bool dense, bool down, int L, int at) {
        // inside a group the row tiles are taken in bands; inside a band the row tile runs fastest, then the column
        // tile: the tiles of one XCD share a few row panels and a few weight panels through its L2
        constexpr int kBand = 8;
        const int nt = col_tiles(dense, down);
        int g, mt, l;
        if (dense) {
            const int per_g = d_mt * nt;
            g = L / per_g;
            mt = d_mt;
            l = L - g * per_g;
        } else {
            int lo = 0, hi = G;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_pref[mid] * nt <= L) lo = mid; else hi = mid;
            }
            g = lo;
            mt = s_pref[g + 1] - s_pref[g];
            l = L - s_pref[g] * nt;
        }
        const int band = l / (kBand * nt), band_h = min(kBand, mt - band * kBand), lb = l - band * kBand * nt;
        const int ni = lb / band_h, mi = band * kBand + (lb - ni * band_h);
        const int g_row0 = dense ? 0 : s_row[g], g_end = dense ? d_rows : s_row[g + 1];
        const Cut c = cut_rows(g_end - g_row0, most);
        const int blocks = c.base + (mi < c.rem ? 1 : 0), row0 = g_row0 + (mi * c.base + min(mi, c.rem)) * 16;
        s_tile[at] = make_int4(g | (dense ? kTileDense : 0) | (down ? kTileDown : 0), row0, min(blocks * 16, g_end - row0) | blocks << 16 | (mt == 1 ? 1 << 24 : 0), ni);
        const int dep = dense ? row_tiles + mi : s_pref[g] + mi;
        if (BOTH) { s_dep[at] = dep; s_ready[at] = 0; }
        return dep;
    };
    const auto tile_at = [&](int it, Tile& t) -> bool {
        const int4 e = s_tile[it % kLdCache];
        const int x = __builtin_amdgcn_readfirstlane(e.x);
        t.g = x & (kTileDense - 1);
        t.dense = (x & kTileDense) != 0;
        t.down = !UP || (DOWN && (x & kTileDown) != 0);
        t.row0 = __builtin_amdgcn_readfirstlane(e.y);
        const int z = __builtin_amdgcn_readfirstlane(e.z);
        t.nrows = z & 0xffff;
        t.blocks = z >> 16 & 0xff;
        t.once = z >> 24;
        t.ni = __builtin_amdgcn_readfirstlane(e.w);
        t.dep = BOTH ? __builtin_amdgcn_readfirstlane(s_dep[it % kLdCache]) : 0;
        return x >= 0;
    };

    // One projection: its tiles are dealt.  The dense tiles come first, one workgroup after the other; a workgroup that has one more than the others takes
    // d_worth ragged tiles fewer.  Where nearly every ragged group is one row tile, its tiles wait for weights that nobody
    // else reads while a dense tile keeps the matrix cores busy: every second workgroup of an XCD then goes through its tiles
    // from the last to the first, and the two kinds run side by side.  One after the other / side by side, us:
    // DeepSeek-V2-shaped share, 1200 / 1600 / 2502 tokens 290 / 274, 313 / 289, 409 / 386, DeepSeek-V2-Lite-shaped layer, 1531 tokens
    // 328 / 304; with two row tiles per expert, which share their weights, 2700 / 4096 tokens 427 / 510, 561 / 639.
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const bool few_rows = shared && row_tiles * 8 <= __builtin_amdgcn_readfirstlane(*s_filled) * 9;   // nearly every ragged group is one row tile
    struct { int total, d_total, d_worth, active, w, rem, mine, count; bool backwards; } hand{};
    if (!BOTH) {
        hand.total = same(tiles_of(false, !UP));
        hand.d_total = shared ? same(tiles_of(true, !UP)) : 0;
        hand.d_worth = shared ? max(1, (ARG(true, false, K) + ARG(false, false, K) / 2) / ARG(false, false, K)) : 1;
        const int worth = hand.total + hand.d_total * hand.d_worth, wgs = (int)gridDim.x;
        const int rounds = (worth + wgs - 1) / wgs;
        hand.active = rounds > 0 ? min(wgs, (((worth + rounds - 1) / rounds) + 7) & ~7) : 0;
        const int per_xcd = hand.active / kXcds;
        if (slot >= per_xcd) return;
        hand.w = xcd * per_xcd + slot;
        const int full = hand.d_total / hand.active;
        hand.rem = hand.d_total - full * hand.active;
        hand.mine = full + (hand.w < hand.rem ? 1 : 0);
        hand.backwards = few_rows && (slot & 1);
        // ragged tiles of this workgroup, those that make up for the dense tile it does not have first
        const int extra = hand.w < hand.rem ? 0 : max(0, min(hand.d_worth, (hand.total - (hand.w - hand.rem) + hand.active - hand.rem - 1) / (hand.active - hand.rem)));
        hand.count = hand.mine + extra + max(0, (hand.total - hand.d_worth * (hand.active - hand.rem) - hand.w + hand.active - 1) / hand.active);
    }
    const auto deal = [&](int it) {   // tile number it of this workgroup
        const int at = it % kLdCache;
        if (it >= hand.count) { s_tile[at] = make_int4(-1, 0, 0, 0); return; }
        if (hand.backwards) it = hand.count - 1 - it;
        const bool dense = it < hand.mine;
        const int v = it - hand.mine + (hand.w < hand.rem ? hand.d_worth : 0);
        const int L = dense ? it * hand.active + hand.w : v < hand.d_worth ? v * (hand.active - hand.rem) + hand.w - hand.rem : hand.d_worth * (hand.active - hand.rem) + (v - hand.d_worth) * hand.active + hand.w;
        decode(dense, !UP, L, at);
    };

    // Both projections: tiles are drawn, by the last loading wavefront.  A projection's dense and ragged tiles are two lists, and a list is eight shares of
    // neighbouring tiles, one for an XCD, with a counter each.  A workgroup draws from its XCD's shares, then from whichever share has the most left, and
    // from the down projection only when the gate/up projection has nothing left to draw: what a down tile waits for is being
    // multiplied by workgroups that wait for nothing, however few of the launch's workgroups are running.
    // Here, too, some workgroups of an XCD begin with the ragged tiles where those wait for weights that nobody else reads.
    const auto begins_ragged = [&](bool down) {   // up to half of the workgroups, no more than the ragged tiles are of the work
        const float d = (float)same(tiles_of(true, down)) * steps_of(true, down), r = (float)same(tiles_of(false, down)) * steps_of(false, down);
        const int n = gridDim.x / kXcds;
        return slot >= n - (int)(n * fminf(0.5f, r / (d + r)));
    };
    const bool ragged_up = BOTH && few_rows && begins_ragged(false), ragged_down = BOTH && few_rows && begins_ragged(true);
    bool drawing_down = false, second = false, elsewhere = false, drawn_all = false, asked = false;
    int drawn = 0, ahead = 0, ticket = 0;   // ahead: K steps of weights drawn and not yet asked for
    int peeked = 0, peek_from = 0, peek_need = 0, peek = 0;   // down tiles whose rows' counts have been asked for: how many, from which, the count they need
    int32_t* const done = sync + kLdCounters;
    const auto needed = [&](int dep) { return (dep < row_tiles ? col_tiles(false, false) : list_of(true, false).groups * col_tiles(true, false)); };
    const auto count_of = [&](int dep) { return __hip_atomic_load(done + (size_t)dep * kRowTileInts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    const auto counter = [&](bool dense, bool down, int x) { return sync + (((down ? 2 : 0) + (dense ? 1 : 0)) * kXcds + x) * kLdLine; };
    const auto at_a_time = [&](bool dense, bool down) { const int k = steps_of(dense, down); return k >= kLdDrawSteps ? 1 : (kLdDrawSteps + k - 1) / k; };
    const auto share = [&](int n, int x) { return n / kXcds + (x < n % kXcds ? 1 : 0); };
    const auto from_dense = [&]() { return second == (drawing_down ? ragged_down : ragged_up); };
    const auto ask = [&](bool dense, int x) {
        int32_t* const c = counter(dense, drawing_down, x);
        const int n = at_a_time(dense, drawing_down);
        return lane == 0 ? __hip_atomic_fetch_add(c, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    };
    const auto take = [&](bool dense, int x, int t) -> bool {   // t: what lane 0 got
        t = __builtin_amdgcn_readfirstlane(t);
        const int n = same(tiles_of(dense, drawing_down)), k = min(at_a_time(dense, drawing_down), share(n, x) - t);
        if (k <= 0) return false;
        if (lane < k) {
            const int dep = decode(dense, drawing_down, n / kXcds * x + min(x, n % kXcds) + t + lane, (drawn + lane) % kLdCache);
            if (drawing_down) { peek_need = needed(dep); peek = count_of(dep); }
        }
        peeked = drawing_down ? k : 0;
        peek_from = drawn;
        drawn += k;
        ahead += k * steps_of(dense, drawing_down);
        return true;
    };
    const auto next_list = [&]() { elsewhere = second; second = true; };
    const auto draw_now = [&]() {   // at least one tile, or the mark behind the last one
        for (;;) {
            if (!elsewhere) {
                const bool dense = from_dense();
                if (same(tiles_of(dense, drawing_down)) > 0 && take(dense, xcd, ask(dense, xcd))) return;
                next_list();
                continue;
            }
            int most_left = -1;
            if (lane < 2 * kXcds) {
                const int left = share(tiles_of(lane >= kXcds, drawing_down), lane % kXcds) - __hip_atomic_load(counter(lane >= kXcds, drawing_down, lane % kXcds), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (left > 0) most_left = min(left, 1 << 24) * (2 * kXcds) + lane;
            }
#pragma unroll
            for (int s = kXcds; s > 0; s >>= 1) most_left = max(most_left, __shfl_xor(most_left, s, 64));
            most_left = __builtin_amdgcn_readfirstlane(most_left);
            if (most_left >= 0) {
                const int i = most_left % (2 * kXcds);
                if (take(i >= kXcds, i % kXcds, ask(i >= kXcds, i % kXcds))) return;
            } else if (!drawing_down) {
                drawing_down = true;
                second = elsewhere = false;
            } else {
                if (lane == 0) s_tile[drawn % kLdCache] = make_int4(-1, 0, 0, 0);
                drawn_all = true;
                return;
            }
        }
    };
    if (!BOTH) {
        if (tid < kLdCache) deal(tid);
    } else if (wave == kLdMultiply + kLdLoad - 1)
        while (!drawn_all && ahead < 4) draw_now();
    __syncthreads();
    Tile t;
    if (!tile_at(0, t)) return;
    if (wave >= kLdMultiply) {
        // ---- loading wavefronts.  Regions of 8 rows (1 KB of LDS) are dealt to them in turn.  The weights run two K steps
        // ahead of the multiplications, the token rows one.
        const int w = wave - kLdMultiply;
        const int ld_row = lane >> 3;
        const uint32_t ld_chunk = (uint32_t)((lane & 7) ^ ((4 * (w & 1) + (lane >> 4)) & 7)) * 16u;   // the 16 bytes that belong at this lane's place
        struct { int it, ki, KT; } cx{-1, 0, 0}, cw{-1, 0, 0};   // K step of the tile whose token rows, weights come next
        uint32_t xo[kLdXRegions], wo[kLdWRegions];
        const char *xk = nullptr, *wk = nullptr;
        int nx = 0, seg = 0, seg_steps = 1;
        uint32_t x_slot = kLdXRing, w_slot = 0;
        long long w_step = 0, seg_jump = 0;
        bool once = false;
        // Until the activation rows of tile `it` are in memory: the drawing wavefront asks, the others look in LDS.  No line of them was in a
        // cache of this launch before, so there is nothing to drop: a launch begins with none, lines belong to one row, and rows are not read earlier
        // (load_x, behind this wait, is the only place that may read them).
        const auto wait_for = [&](int it, int dep) {
            int* const ready = s_ready + it % kLdCache;
            const auto is_ready = [&]() { return __builtin_amdgcn_readfirstlane(__hip_atomic_load(ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)); };
            if (w != kLdLoad - 1) {
                while (!is_ready()) __builtin_amdgcn_s_sleep(1);
            } else if (!is_ready()) {
                while (__builtin_amdgcn_readfirstlane(count_of(dep)) < needed(dep)) __builtin_amdgcn_s_sleep(16);
                if (lane == 0) __hip_atomic_store(ready, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            asm volatile("" ::: "memory");
        };
        // the token rows of a K step; false behind the last tile
        const auto load_x = [&]() __attribute__((always_inline)) -> bool {
            if (cx.ki == cx.KT) {
                Tile t;
                if (!tile_at(++cx.it, t)) { cx.KT = cx.ki = 0; --cx.it; return false; }
                if (BOTH && t.down) wait_for(cx.it, t.dep);
                const bool map = UP && !t.down && !t.dense && a1.a_row_map != nullptr;
                const int lda = same(list_of(t.dense, t.down).lda);
                cx.KT = steps_of(t.dense, t.down);
                cx.ki = 0;
                nx = (2 * t.blocks - w + kLdLoad - 1) / kLdLoad;
                xk = reinterpret_cast<const char*>(same(list_of(t.dense, t.down).A));
                if (!map) xk += (size_t)t.row0 * lda * 2;
                int src[kLdXRegions];
#pragma unroll
                for (int i = 0; i < kLdXRegions; ++i) src[i] = min((w + kLdLoad * i) * 8 + ld_row, t.nrows - 1);
                if (map) {
#pragma unroll
                    for (int i = 0; i < kLdXRegions; ++i) src[i] = a1.a_row_map[t.row0 + src[i]];
#pragma unroll
                    for (int i = 0; i < kLdXRegions; ++i) src[i] /= a1.a_row_div;
                }
#pragma unroll
                for (int i = 0; i < kLdXRegions; ++i) xo[i] = (uint32_t)src[i] * (uint32_t)lda * 2u + ld_chunk;
            }
#pragma unroll
            for (int i = 0; i < kLdXRegions; ++i)
                if (i < nx) __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(xk + in_32_bits(xo[i])), reinterpret_cast<uint4*>(lds + x_slot + w * 1024 + i * (kLdLoad * 1024)), 16, 0, 0);
            xk += kPackK * 2;
            x_slot = x_slot == kLdXRing + (kLdXSlots - 1) * kLdXBytes ? (uint32_t)kLdXRing : x_slot + kLdXBytes;
            ++cx.ki;
            return true;
        };
        // the weights of a K step; false behind the last tile.  Weights that one row tile reads are not kept in the caches
        // (aux 2: non-temporal).
        const auto load_w = [&]() __attribute__((always_inline)) -> bool {
            if (cw.ki == cw.KT) {
                Tile t;
                if (!tile_at(++cw.it, t)) { cw.KT = cw.ki = 0; --cw.it; return false; }
                if (!BOTH && w == kLdLoad - 1 && lane == 0 && cw.it + 24 >= kLdCache) deal(cw.it + 24);
                const int g = t.g, ldw = same(list_of(t.dense, t.down).ldw), N = same(list_of(t.dense, t.down).N);
                cw.KT = steps_of(t.dense, t.down);
                cw.ki = 0;
                once = t.once != 0;
                if (PACKED) {
                    wk = reinterpret_cast<const char*>(same(list_of(t.dense, t.down).W) + ((size_t)g * same(col_tiles(t.dense, t.down)) + t.ni) * ((size_t)cw.KT * kPackRows * kPackK)) + w * 1024;
#pragma unroll
                    for (int i = 0; i < kLdWRegions; ++i) wo[i] = i * (kLdLoad * 1024u) + lane * 16u;
                    w_step = kLdWBytes;
                    seg = seg_steps = cw.KT;
                    seg_jump = 0;
                } else {
                    wk = reinterpret_cast<const char*>(same(list_of(t.dense, t.down).W) + (size_t)g * same(list_of(t.dense, t.down).w_group_stride));
                    const uint32_t up = (uint32_t)same(list_of(t.dense, t.down).w_up_offset);
                    const bool pair = UP && !t.down;   // 128 rows of W_gate and of W_up
                    const int n0 = t.ni * (pair ? kPackRows / 2 : kPackRows);
#pragma unroll
                    for (int i = 0; i < kLdWRegions; ++i) {
                        const int r = (w + kLdLoad * i) * 8 + ld_row;
                        const int n = min(n0 + (pair ? r & 127 : r), N - 1);
                        wo[i] = ((pair && r >= 128 ? up : 0u) + (uint32_t)n * (uint32_t)ldw) * 2u + ld_chunk;
                    }
                    const int kseg_len = same(list_of(t.dense, t.down).kseg_len);
                    w_step = kPackK * 2;
                    seg = seg_steps = kseg_len / kPackK;
                    seg_jump = (same(list_of(t.dense, t.down).w_kseg_stride) - kseg_len) * 2;
                }
            }
            char* const dst = lds + w_slot + w * 1024;
            if (once) {
#pragma unroll
                for (int i = 0; i < kLdWRegions; ++i)
                    __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(wk + in_32_bits(wo[i])), reinterpret_cast<uint4*>(dst + i * (kLdLoad * 1024)), 16, 0, 2);
            } else {
#pragma unroll
                for (int i = 0; i < kLdWRegions; ++i)
                    __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(wk + in_32_bits(wo[i])), reinterpret_cast<uint4*>(dst + i * (kLdLoad * 1024)), 16, 0, 0);
            }
            wk += w_step;
            if (--seg == 0) { seg = seg_steps; wk += seg_jump; }
            w_slot = w_slot == (kLdWSlots - 1) * kLdWBytes ? 0u : w_slot + kLdWBytes;
            ++cw.ki;
            --ahead;
            return true;
        };
        load_w();
        load_x();
        bool more = load_w();
        for (;;) {
            // everything but the weights behind the K step that is handed over now
            if (more) wait_loads<kLdWRegions>(); else wait_loads<0>();
            hand_over();
            // The next tiles: asked for before a K step's loads and looked at behind them, or waited for.  They are written a hand-over before
            // they are read.
            if (BOTH && w == kLdLoad - 1 && peeked) {
                if (lane < peeked && peek >= peek_need) s_ready[(peek_from + lane) % kLdCache] = 1;
                peeked = 0;
            }
            if (BOTH && w == kLdLoad - 1 && !drawn_all) {
                if (asked) {
                    asked = false;
                    if (!take(from_dense(), xcd, ticket)) next_list();
                }
                if (ahead <= kLdDrawAhead && !elsewhere) {
                    if (same(tiles_of(from_dense(), drawing_down)) > 0) { ticket = ask(from_dense(), xcd); asked = true; }
                    else next_list();
                }
                if (ahead <= (elsewhere ? 4 : 1)) {
                    if (asked) { asked = false; if (!take(from_dense(), xcd, ticket)) next_list(); }
                    while (!drawn_all && ahead <= (elsewhere ? 4 : 1)) draw_now();
                }
            }
            if (!load_x()) break;
            more = load_w();
        }
        return;
    }

    // ---- multiplying wavefronts: the upper or the lower half of a tile's row blocks times 64 of its 256 weight rows
    const int wn = wave & 3, wm = wave >> 2;
    const int fr = lane & 15, kh = lane >> 4;
    const uint32_t xa = fr * 128u + (uint32_t)(kh ^ (fr >> 1)) * 16u;
    const uint32_t wa = PACKED ? wn * 8192u + (kh * 16u + fr) * 16u : (UP ? (wn * 32u + fr) * 128u : (wn * 64u + fr) * 128u) + (uint32_t)(kh ^ (fr >> 1)) * 16u;
    Slots off{0, kLdXRing};
    Told told{nullptr, nullptr};   // the gate/up tile before
    hand_over();
    for (int it = 0;;) {
        const int KT = steps_of(t.dense, t.down);
        const int top = (t.blocks + 1) >> 1, mine = wm ? t.blocks - top : top, row_a = wm ? top * 16 : 0;
        const int n_wave = t.ni * (UP && !t.down ? kPackRows / 2 : kPackRows) + wn * (UP && !t.down ? 32 : 64);
        Out out;
        out.ldc = same(list_of(t.dense, t.down).ldc);
        out.nrows = t.nrows - row_a;
        out.n_left = same(list_of(t.dense, t.down).N) - n_wave;
        out.c = same(list_of(t.dense, t.down).C) + (size_t)(t.dense ? t.g : 0) * same(list_of(t.dense, t.down).c_group_col_stride) + (size_t)(t.row0 + row_a) * out.ldc + n_wave;
        const uint32_t x_mine = xa + row_a * 128u;
        const int4* const next = s_tile + (it + 1) % kLdCache;
        bool more = true;
        if (mine == 0) {   // one block in all: the other half has it
            for (int kt = 0; kt < KT; ++kt) {
                if (kt + 1 == KT) more = UP && !t.down ? goes_on<true>(next) : goes_on<false>(next);
                if (more) hand_over();
                off = off.next();
            }
            if (BOTH && told.done) tell(told);
        } else if (UP && !t.down) {
            switch (mine) {
#define X(n) case n: more = run_tile<n, true, PACKED, BOTH>(lds, x_mine, wa, KT, next, told, off, out); break;
                X(1) X(2) X(3) X(4) X(5)
#undef X
                default: more = run_tile<kLdBlocks / 2, true, PACKED, BOTH>(lds, x_mine, wa, KT, next, told, off, out); break;
            }
        } else {
            const uint32_t w_mine = PACKED || !UP ? wa : wa + wn * 4096u;
            switch (mine) {
#define X(n) case n: more = run_tile<n, false, PACKED, false>(lds, x_mine, w_mine, KT, next, Told{nullptr, nullptr}, off, out); break;
                X(1) X(2) X(3) X(4) X(5)
#undef X
                default: more = run_tile<kLdBlocks / 2, false, PACKED, false>(lds, x_mine, w_mine, KT, next, Told{nullptr, nullptr}, off, out); break;
            }
        }
        if (BOTH) {
            told = Told{t.down ? nullptr : done + (size_t)t.dep * kRowTileInts, s_waves + it % kLdTold};
            if (!more && told.done) { tell(told); told.done = nullptr; }   // the loading wavefronts may be waiting for these rows
        }
        if (!tile_at(it + 1, t)) break;
        if (!more) hand_over();
        ++it;
    }
#undef ARG
}
#undef SB

static bool loader_args_fit(const GemmArgs& a, bool swiglu, bool ragged)
{
    if (a.K < kPackK || a.K % kPackK || a.kseg_len < kPackK || a.kseg_len % kPackK || a.N < 8 || a.N % 8) return false;
    if (a.G < 1 || a.G > kLdGroups || a.epi != 0 || a.max_units != 0) return false;
    // lanes address with 32-bit byte offsets inside one group's weights and one activation panel
    const long long w_span = ((swiglu ? a.w_up_offset : 0) + (long long)a.N * a.ldw) * 2;
    const long long x_span = (long long)(a.a_row_map ? a.a_src_rows : kLoaderRows) * a.lda * 2;
    if (a.a_row_map && (!ragged || a.a_row_div < 1 || a.a_src_rows < 1)) return false;
    if (w_span >= (1ll << 32) || x_span >= (1ll << 32) || w_span < 0) return false;
    return !(a.ldc % 8 || a.c_group_col_stride % 8 || (reinterpret_cast<uintptr_t>(a.C) & 15));
}

hipError_t launch_loader_gemm(const GemmArgs* up, const GemmArgs* up_shared, const GemmArgs* down, const GemmArgs* down_shared, int n_cu, int32_t* sync, hipStream_t s)
{
    const GemmArgs none{};
    const GemmArgs* const routed[2] = {up, down};
    const GemmArgs* const dense[2] = {up_shared, down_shared};
    if ((!up && !down) || (up_shared && !up) || (down_shared && !down) || (up && down && sync == nullptr)) return hipErrorInvalidValue;
    const GemmArgs& first = up ? *up : *down;
    for (int i = 0; i < 2; ++i) {
        const GemmArgs* r = routed[i];
        const GemmArgs* d = dense[i];
        if (r && (r->offset == nullptr || (r->Wp != nullptr) != (first.Wp != nullptr) || (i == 1 && r->a_row_map) || !loader_args_fit(*r, i == 0, true))) return hipErrorInvalidValue;
        if (d && (d->offset || d->dense_rows < 1 || (d->Wp != nullptr) != (first.Wp != nullptr) || !loader_args_fit(*d, i == 0, false))) return hipErrorInvalidValue;
    }
    if (up && down) {
        // a line of the activation belongs to one row: it is read when the row's tiles are counted, and not before
        const auto whole_lines = [](const GemmArgs& a) { return !(a.ldc % 64 || a.c_group_col_stride % 64 || (reinterpret_cast<uintptr_t>(a.C) & 127)); };
        if (up->offset != down->offset || up->G != down->G || (up_shared != nullptr) != (down_shared != nullptr) || !whole_lines(*up)) return hipErrorInvalidValue;
        if (up_shared && (up_shared->dense_rows != down_shared->dense_rows || down_shared->G != 1 || !whole_lines(*up_shared))) return hipErrorInvalidValue;
    }
    const int lds = loader_lds(first.G);
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((n_cu + kXcds - 1) / kXcds * kXcds), dim3(kLdThreads), lds, s, up ? *up : none, up_shared ? *up_shared : none, down ? *down : none,
                           down_shared ? *down_shared : none, sync);
    };
    if (first.Wp) { if (!down) go(loader_gemm_kernel<1, true>); else if (!up) go(loader_gemm_kernel<2, true>); else go(loader_gemm_kernel<3, true>); }
    else { if (!down) go(loader_gemm_kernel<1, false>); else if (!up) go(loader_gemm_kernel<2, false>); else go(loader_gemm_kernel<3, false>); }
    return hipGetLastError();
}

hipError_t loader_gemm_init()
{
    static_assert(loader_lds(kLdGroups) <= 160 * 1024, "a workgroup's LDS");
    for (const void* f : {reinterpret_cast<const void*>(&loader_gemm_kernel<1, true>), reinterpret_cast<const void*>(&loader_gemm_kernel<2, true>), reinterpret_cast<const void*>(&loader_gemm_kernel<3, true>),
                          reinterpret_cast<const void*>(&loader_gemm_kernel<1, false>), reinterpret_cast<const void*>(&loader_gemm_kernel<2, false>), reinterpret_cast<const void*>(&loader_gemm_kernel<3, false>)}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, loader_lds(kLdGroups));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace moe_ep
