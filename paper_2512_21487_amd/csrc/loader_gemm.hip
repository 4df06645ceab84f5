// Expert projections out of workgroups whose loads and multiplications are different wavefronts (Sec. 3.1): the tiled
// form of prefill, routed experts (ragged groups) with or without the shared ones (dense groups) in the same launch.
//
// What bounds a tile is the compute unit's vector memory path: it keeps about 32 KB of requests in flight, so it
// draws 80 GB/s from L2 and 46 GB/s from HBM, and a K step of a 160 x 256 tile is 52 KB.  With the multiplications taken
// out, the loads alone were three quarters of a launch (Qwen3-30B-A3B-shaped layer, 8192 tokens, gate/up 345 of 437 us).  In
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
// longer, nothing won back); cache policy bits (nt slower, the others equal); wavefront priorities (equal).
// Forwards before / with these kernels, us: DeepSeek-V2-Lite-shaped layer, 4096 tokens 614 / 568, 1531 tokens, weights in the
// caller's layout 342 / 304; Qwen3-30B-A3B-shaped layer, 8192 tokens 723 / 650, skewed 735 / 693; DeepSeek-V2-shaped share,
// 1600 / 2502 / 5000 tokens 341 / 289, 421 / 386, 680 / 622; Qwen3-235B-A22B-shaped share, 1024 / 2048 tokens 135 / 128, 152 / 142.
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

struct Tile { int g, row0, nrows, n0, blocks, once; };   // g >= routed groups: a dense one

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

// N row blocks of a tile.  xa, wa: the lane's bytes into a slot's token rows and weights; off: the ring slots of the tile's
// first K step, handed over; on return those of the next tile's first one.  more: another tile follows.
template <int N, bool SWIGLU, bool PACKED>
__device__ __forceinline__ void run_tile(const char* lds, uint32_t xa, uint32_t wa, int KT, bool more, Slots& off, const Out& out)
{
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
        bf16x8_t x[S];
#pragma unroll
        for (int r = 0; r < P; ++r) x[r] = xn[r];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (s == H && (more || kt + 1 < KT)) hand_over();
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
                if (mb * 16 + row < out.nrows && !(decltype(guard)::value && nb * 16 + col >= out.n_left))
                    *reinterpret_cast<uint4*>(reinterpret_cast<char*>(out.c + (size_t)(mb * 16) * out.ldc + nb * 16) + at) = o;
            }
        }
    };
    if (out.n_left >= (SWIGLU ? 32 : 64)) store(std::false_type{}); else store(std::true_type{});
}

}  // namespace

template <bool SWIGLU, bool PACKED>
__global__ __launch_bounds__(kLdThreads) void loader_gemm_kernel(GemmArgs a, GemmArgs d)
{
    extern __shared__ uint4 lds4[];
    char* const lds = reinterpret_cast<char*>(lds4);
    int4* const s_tile = reinterpret_cast<int4*>(lds + kLdRing);
    int* const s_filled = reinterpret_cast<int*>(s_tile + kLdCache);
    int* const s_most = s_filled + 1;
    int* const s_pref = s_most + 1;
    constexpr int COLS = SWIGLU ? kPackRows / 2 : kPackRows;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int NT = (a.N + COLS - 1) / COLS;
    // the dense groups' column tiles, and how many ragged tiles one of theirs is worth (its K may be longer)
    const int d_nt = d.G > 0 ? (d.N + COLS - 1) / COLS : 0, d_worth = d.G > 0 ? max(1, (d.K + a.K / 2) / a.K) : 1;

    // Row tiles before every ragged group.  Tiles of at most kLdLowBlocks blocks where they take no more rounds (a dense tile counts as the
    // ragged ones it is worth) or are one for a workgroup all the same, since a round lasts as long as its tallest tile -- unless they are only a
    // few more (a seventh), which cost more than the others gain, in a launch that keeps three quarters of the workgroups busy.  Of 9824
    // launches of 1 to 256 experts (2 to 5800 rows each, skewed and not, shared experts beside them or not) this leaves 0.3 % of the time to the
    // better one of both, tiles of up to 12 blocks always 5.7 %, of 8 always 6.5 %.  Forwards, 12 / this, us: one expert of 146 rows, 1536 x 1536,
    // 63 / 57, two of 174, 1408 x 7168, 153 / 127, 16 of about 160, 1024 x 2880, 83 / 63 (in grouped_gemm.hip, 128 rows, 55, 125, 77); 4 of the
    // DeepSeek-V2-shaped layer's experts and its shared ones, 2000 tokens 244 / 230 (231).
    if (wave == 0) {
        constexpr int PER = kLdGroups / 64;
        // consecutive groups of a lane: one scan over the lanes, however many groups there are.  With one per 64 groups, a forward of 1000 tokens
        // on a few of 512 experts, 384 x 1536, took 84 us instead of 75 (in grouped_gemm.hip 75).
        const int per = (a.G + 63) >> 6, g0 = lane * per;
        int rows[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i >= per) break;
            rows[i] = g0 + i < a.G ? a.offset[g0 + i + 1] - a.offset[g0 + i] : 0;
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
                if (g0 + i < a.G) s_pref[g0 + i] = at;
                at += cut_rows(rows[i], most).tiles;
            }
            if (lane == 0) { s_pref[a.G] = before; *s_filled = filled; }
        };
        count_tiles(kLdBlocks);
        const auto dense_tiles = [&](int most) { return d.G > 0 ? d.G * cut_rows(d.dense_rows, most).tiles * d_nt : 0; };
        const int d_tall = dense_tiles(kLdBlocks), d_low = dense_tiles(kLdLowBlocks);
        int most = kLdBlocks;
        const bool recount = __ballot(low > 0) != 0;
        if (recount || d_low != d_tall) {
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
    const int total = __builtin_amdgcn_readfirstlane(s_pref[a.G]) * NT, most = __builtin_amdgcn_readfirstlane(*s_most);
    const int d_mt = d.G > 0 ? cut_rows(d.dense_rows, most).tiles : 0;
    const int d_total = d.G * d_mt * d_nt;
    const int worth = total + d_total * d_worth;
    const int rounds = (worth + (int)gridDim.x - 1) / (int)gridDim.x;
    const int active = rounds > 0 ? min((int)gridDim.x, (((worth + rounds - 1) / rounds) + 7) & ~7) : 0;
    const int per_xcd = active >> 3, xcd = blockIdx.x & 7, slot_in_xcd = blockIdx.x >> 3;
    if (slot_in_xcd >= per_xcd) return;

    // The dense tiles come first, one workgroup after the other; a workgroup that has one more than the others takes
    // d_worth ragged tiles fewer.  Where nearly every ragged group is one row tile, its tiles wait for weights that nobody
    // else reads while a dense tile keeps the matrix cores busy: every second workgroup of an XCD then goes through its tiles
    // from the last to the first, and the two kinds run side by side.  One after the other / side by side, us:
    // DeepSeek-V2-shaped share, 1200 / 1600 / 2502 tokens 290 / 274, 313 / 289, 409 / 386, DeepSeek-V2-Lite-shaped layer, 1531 tokens
    // 328 / 304; with two row tiles per expert, which share their weights, 2700 / 4096 tokens 427 / 510, 561 / 639.
    const int w = xcd * per_xcd + slot_in_xcd;
    const int full = d_total / active, rem = d_total - full * active, mine = full + (w < rem ? 1 : 0);
    const bool backwards = d_total > 0 && (slot_in_xcd & 1) && __builtin_amdgcn_readfirstlane(s_pref[a.G]) * 8 <= __builtin_amdgcn_readfirstlane(*s_filled) * 9;
    // ragged tiles of this workgroup, those that make up for the dense tile it does not have first
    const int extra = w < rem ? 0 : max(0, min(d_worth, (total - (w - rem) + active - rem - 1) / (active - rem)));
    const int count = mine + extra + max(0, (total - d_worth * (active - rem) - w + active - 1) / active);

    // tile number it of this workgroup: g < 0 past the last one
    const auto decode = [&](int it) -> int4 {
        if (it >= count) return make_int4(-1, 0, 0, 0);
        if (backwards) it = count - 1 - it;
        const bool dense = it < mine;
        const int v = it - mine + (w < rem ? d_worth : 0);
        const int L = dense ? it * active + w : v < d_worth ? v * (active - rem) + w - rem : d_worth * (active - rem) + (v - d_worth) * active + w;
        // inside a group the row tiles are taken in bands; inside a band the row tile runs fastest, then the column
        // tile: the tiles of one XCD share a few row panels and a few weight panels through its L2
        constexpr int kBand = 8;
        int g, mt, l, nt = NT;
        if (dense) {
            const int per_g = d_mt * d_nt;
            g = L / per_g;
            mt = d_mt;
            nt = d_nt;
            l = L - g * per_g;
        } else {
            int lo = 0, hi = a.G;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_pref[mid] * NT <= L) lo = mid; else hi = mid;
            }
            g = lo;
            mt = s_pref[g + 1] - s_pref[g];
            l = L - s_pref[g] * NT;
        }
        const int band = l / (kBand * nt), band_h = min(kBand, mt - band * kBand), lb = l - band * kBand * nt;
        const int ni = lb / band_h, mi = band * kBand + (lb - ni * band_h);
        const int g_row0 = dense ? 0 : a.offset[g], g_end = dense ? d.dense_rows : a.offset[g + 1];
        const Cut c = cut_rows(g_end - g_row0, most);
        const int blocks = c.base + (mi < c.rem ? 1 : 0), row0 = g_row0 + (mi * c.base + min(mi, c.rem)) * 16;
        return make_int4(dense ? a.G + g : g, row0, min(blocks * 16, g_end - row0) | blocks << 16 | (mt == 1 ? 1 << 24 : 0), ni * COLS);
    };
    const auto tile_at = [&](int it, Tile& t) -> bool {
        const int4 e = s_tile[it % kLdCache];
        t.g = __builtin_amdgcn_readfirstlane(e.x);
        t.row0 = __builtin_amdgcn_readfirstlane(e.y);
        const int z = __builtin_amdgcn_readfirstlane(e.z);
        t.nrows = z & 0xffff;
        t.blocks = z >> 16 & 0xff;
        t.once = z >> 24;
        t.n0 = __builtin_amdgcn_readfirstlane(e.w);
        return t.g >= 0;
    };
    if (tid < kLdCache) s_tile[tid] = decode(tid);
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
        // the token rows of a K step; false behind the last tile
        const auto load_x = [&]() __attribute__((always_inline)) -> bool {
            if (cx.ki == cx.KT) {
                Tile t;
                if (!tile_at(++cx.it, t)) { cx.KT = cx.ki = 0; --cx.it; return false; }
                const bool dense = t.g >= a.G, map = a.a_row_map != nullptr && !dense;
                const int lda = dense ? d.lda : a.lda;
                cx.KT = (dense ? d.K : a.K) / kPackK;
                cx.ki = 0;
                nx = (2 * t.blocks - w + kLdLoad - 1) / kLdLoad;
                xk = reinterpret_cast<const char*>(dense ? d.A : a.A);
                if (!map) xk += (size_t)t.row0 * lda * 2;
                int src[kLdXRegions];
#pragma unroll
                for (int i = 0; i < kLdXRegions; ++i) src[i] = min((w + kLdLoad * i) * 8 + ld_row, t.nrows - 1);
                if (map) {
#pragma unroll
                    for (int i = 0; i < kLdXRegions; ++i) src[i] = a.a_row_map[t.row0 + src[i]];
#pragma unroll
                    for (int i = 0; i < kLdXRegions; ++i) src[i] /= a.a_row_div;
                }
#pragma unroll
                for (int i = 0; i < kLdXRegions; ++i) xo[i] = (uint32_t)src[i] * (uint32_t)lda * 2u + ld_chunk;
            }
#pragma unroll
            for (int i = 0; i < kLdXRegions; ++i)
                if (i < nx) __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(xk + xo[i]), reinterpret_cast<uint4*>(lds + x_slot + w * 1024 + i * (kLdLoad * 1024)), 16, 0, 0);
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
                if (w == 3 && lane == 0 && cw.it + 24 >= kLdCache) s_tile[(cw.it + 24) % kLdCache] = decode(cw.it + 24);
                const bool dense = t.g >= a.G;
                const int g = dense ? t.g - a.G : t.g, ldw = dense ? d.ldw : a.ldw, N = dense ? d.N : a.N;
                cw.KT = (dense ? d.K : a.K) / kPackK;
                cw.ki = 0;
                once = t.once != 0;
                if (PACKED) {
                    const int nt = dense ? d_nt : NT;
                    wk = reinterpret_cast<const char*>((dense ? d.Wp : a.Wp) + ((size_t)g * nt + t.n0 / COLS) * ((size_t)cw.KT * kPackRows * kPackK)) + w * 1024;
#pragma unroll
                    for (int i = 0; i < kLdWRegions; ++i) wo[i] = i * (kLdLoad * 1024u) + lane * 16u;
                    w_step = kLdWBytes;
                    seg = seg_steps = cw.KT;
                    seg_jump = 0;
                } else {
                    wk = reinterpret_cast<const char*>((dense ? d.W : a.W) + (size_t)g * (dense ? d.w_group_stride : a.w_group_stride));
                    const uint32_t up = (uint32_t)(dense ? d.w_up_offset : a.w_up_offset);
#pragma unroll
                    for (int i = 0; i < kLdWRegions; ++i) {
                        const int r = (w + kLdLoad * i) * 8 + ld_row;
                        const int n = min(t.n0 + (SWIGLU ? r & 127 : r), N - 1);
                        wo[i] = ((SWIGLU && r >= 128 ? up : 0u) + (uint32_t)n * (uint32_t)ldw) * 2u + ld_chunk;
                    }
                    const int kseg_len = dense ? d.kseg_len : a.kseg_len;
                    w_step = kPackK * 2;
                    seg = seg_steps = kseg_len / kPackK;
                    seg_jump = ((dense ? d.w_kseg_stride : a.w_kseg_stride) - kseg_len) * 2;
                }
            }
            char* const dst = lds + w_slot + w * 1024;
            if (once) {
#pragma unroll
                for (int i = 0; i < kLdWRegions; ++i)
                    __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(wk + wo[i]), reinterpret_cast<uint4*>(dst + i * (kLdLoad * 1024)), 16, 0, 2);
            } else {
#pragma unroll
                for (int i = 0; i < kLdWRegions; ++i)
                    __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(wk + wo[i]), reinterpret_cast<uint4*>(dst + i * (kLdLoad * 1024)), 16, 0, 0);
            }
            wk += w_step;
            if (--seg == 0) { seg = seg_steps; wk += seg_jump; }
            w_slot = w_slot == (kLdWSlots - 1) * kLdWBytes ? 0u : w_slot + kLdWBytes;
            ++cw.ki;
            return true;
        };
        load_w();
        load_x();
        bool ahead = load_w();
        for (;;) {
            // everything but the weights behind the K step that is handed over now
            if (ahead) wait_loads<kLdWRegions>(); else wait_loads<0>();
            hand_over();
            if (!load_x()) break;
            ahead = load_w();
        }
        return;
    }

    // ---- multiplying wavefronts: the upper or the lower half of a tile's row blocks times 64 of its 256 weight rows
    const int wn = wave & 3, wm = wave >> 2;
    const int fr = lane & 15, kh = lane >> 4;
    const uint32_t xa = fr * 128u + (uint32_t)(kh ^ (fr >> 1)) * 16u;
    const uint32_t wa = PACKED ? wn * 8192u + (kh * 16u + fr) * 16u : (wn * (SWIGLU ? 32u : 64u) + fr) * 128u + (uint32_t)(kh ^ (fr >> 1)) * 16u;
    Slots off{0, kLdXRing};
    hand_over();
    for (int it = 0;;) {
        Tile nxt;
        const bool more = tile_at(it + 1, nxt);
        const bool dense = t.g >= a.G;
        const int KT = (dense ? d.K : a.K) / kPackK;
        const int top = (t.blocks + 1) >> 1, mine = wm ? t.blocks - top : top, row_a = wm ? top * 16 : 0;
        const int n_wave = t.n0 + wn * (SWIGLU ? 32 : 64);
        Out out;
        out.ldc = dense ? d.ldc : a.ldc;
        out.nrows = t.nrows - row_a;
        out.n_left = (dense ? d.N : a.N) - n_wave;
        out.c = (dense ? d.C : a.C) + (size_t)(dense ? t.g - a.G : t.g) * (dense ? d.c_group_col_stride : a.c_group_col_stride) + (size_t)(t.row0 + row_a) * out.ldc + n_wave;
        const uint32_t x_mine = xa + row_a * 128u;
        switch (mine) {
            case 0:   // one block in all: the other half has it
                for (int kt = 0; kt < KT; ++kt) {
                    if (more || kt + 1 < KT) hand_over();
                    off = off.next();
                }
                break;
#define X(n) case n: run_tile<n, SWIGLU, PACKED>(lds, x_mine, wa, KT, more, off, out); break;
            X(1) X(2) X(3) X(4) X(5)
#undef X
            default: run_tile<kLdBlocks / 2, SWIGLU, PACKED>(lds, x_mine, wa, KT, more, off, out); break;
        }
        if (!more) break;
        t = nxt;
        ++it;
    }
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

hipError_t launch_loader_gemm(const GemmArgs& routed, const GemmArgs* shared, bool swiglu, int n_cu, hipStream_t s)
{
    GemmArgs none{};
    const GemmArgs& sh = shared ? *shared : none;
    if (routed.offset == nullptr || !loader_args_fit(routed, swiglu, true)) return hipErrorInvalidValue;
    if (shared && (sh.offset || sh.dense_rows < 1 || (sh.Wp != nullptr) != (routed.Wp != nullptr) || !loader_args_fit(sh, swiglu, false))) return hipErrorInvalidValue;
    const int lds = kLdRing + kLdCache * 16 + (routed.G + 3) * 4;
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((n_cu + 7) / 8 * 8), dim3(kLdThreads), lds, s, routed, sh); };
    if (routed.Wp) swiglu ? go(loader_gemm_kernel<true, true>) : go(loader_gemm_kernel<false, true>);
    else swiglu ? go(loader_gemm_kernel<true, false>) : go(loader_gemm_kernel<false, false>);
    return hipGetLastError();
}

hipError_t loader_gemm_init()
{
    const int most = kLdRing + kLdCache * 16 + (kLdGroups + 3) * 4;
    static_assert(kLdRing + kLdCache * 16 + (kLdGroups + 3) * 4 <= 160 * 1024, "a workgroup's LDS");
    for (const void* f : {reinterpret_cast<const void*>(&loader_gemm_kernel<true, true>), reinterpret_cast<const void*>(&loader_gemm_kernel<false, true>),
                          reinterpret_cast<const void*>(&loader_gemm_kernel<true, false>), reinterpret_cast<const void*>(&loader_gemm_kernel<false, false>)}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace moe_ep
