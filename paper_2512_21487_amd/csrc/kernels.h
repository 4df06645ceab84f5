// Host-side launchers of the HIP kernels (internal to the library; the public boundary is moe_ep.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace moe_ep {

// tokens per router / permute workgroup: one bit each in a 64-bit mask per expert
constexpr int kTokPerBlock = 64;

// Token rows that a launch of the gate brings in beside its own work (16-byte aligned; first: set by the launcher)
struct RowCopy { void* dst; const void* src; size_t bytes; int first; };

// integers that a launch of the partition sets to zero for the launches behind it
struct Clear { int32_t* p; int n; };

// Whether the first of r chunks is brought in that way.  Not where the shared experts come first: they wait for every chunk, and the
// others start on the link one hand-over between streams later.  Nor with more scores than a lane's 16 (E > 256), which the gate
// then reads one by one over the link.  Pinned host I/O, the first chunk on the copies' stream / with the gate, us: 1024 hidden, 32 of 256
// experts and one shared, 64 tokens, interleaved in one / two / four chunks 75 / 59, 101 / 95, 153 / 146, shared first in two / four 107 / 120,
// 174 / 199, 512 tokens 158 / 168, 272 / 284 (DeepSeek-V2-Lite-shaped layer, 64 / 4096 tokens in two 406 / 404, 1387 / 1387); 384 hidden, 512
// experts, 64 / 160 tokens in two 104 / 115, 119 / 130, 4096 in one 339 / 364, but 16 / 512 in one 71 / 56, 108 / 97.
bool rows_come_with_gate(int E, int r, bool shared_first);

// ---- gate: softmax + top-k (Sec. 2.1) and per-workgroup expert bit masks for the partition
hipError_t launch_router(const float* logits, int Tn, int E, int k, int e0, int El, int32_t* idx,
                         float* w, unsigned long long* blk_mask, hipStream_t s, const RowCopy* copy = nullptr);

// gate and partition of at most kTokPerBlock tokens in one launch; outputs as launch_router and launch_dispatch
hipError_t launch_route_and_partition(const float* logits, int Tn, int E, int k, int e0, int El, int32_t* idx, float* w,
                                      int32_t* count, int32_t* offset, int32_t* pos, int32_t* perm, hipStream_t s, const RowCopy* copy = nullptr,
                                      const Clear& clear = Clear{nullptr, 0});

// ---- partition by expert (Sec. 2.1; Sec. 3.1 "The MoE Part")
// count [El], offset [El + 1], pos [Tn * k] (row of an assignment or -1), perm [rows] (row -> assignment)
hipError_t launch_dispatch(const int32_t* idx, const unsigned long long* blk_mask, int Tn, int k, int e0, int El,
                           int32_t* count, int32_t* offset, int32_t* pos, int32_t* perm, hipStream_t s, const Clear& clear = Clear{nullptr, 0});
hipError_t launch_gather_rows(const void* tokens, const int32_t* perm, const int32_t* n_rows_ptr,
                              int k, int M, void* xp, int grid, hipStream_t s);

// ---- weighted aggregation (Sec. 2.1)
// y_mode: 0 bf16 expert outputs, weighted here; 1 fp32 expert outputs, weighted here; 2 bf16 expert
// outputs that already carry their routing weight
// accumulate: the rows at out_src already hold the shared experts' output and the sum is added to
// them.  out_src == NULL or == out: in place (rows with nothing kept are then left alone); else
// every row is read at out_src and written at out (which may be the caller's pinned host buffer)
hipError_t launch_combine(const void* y, const int32_t* pos, const float* w, int Tn, int k, int M,
                          bool accumulate, int y_mode, const void* out_src, void* out, int grid, hipStream_t s);

// ---- chunk transfers over the host link (pinned-host mode); bytes must be a multiple of 4; lds: bytes of LDS every
// workgroup keeps other kernels' workgroups out with
hipError_t launch_copy(void* dst, const void* src, size_t bytes, int grid, hipStream_t s, int threads = 256, int unroll = 4, int lds = 0);
// Compute units a launch takes beside a copy of kLinkUnits workgroups: those workgroups' own units are left out, but no more than a
// sixteenth of the device (256 units: 16), which may be a small partition of the GPU
constexpr int kLinkUnits = 16;
int units_beside_link(int n_cu);
// a one-wavefront kernel that lasts about `microseconds` (at most 1 s): stand-in for a task that
// runs on other hardware
hipError_t launch_busy(double microseconds, hipStream_t s);

// ---- expert projections as one grouped GEMM launch (Sec. 3.1, Eq. moe_detail / shared_detail)
struct GemmArgs {
    const uint16_t* A;         // activations, bf16 [rows, lda]
    const uint16_t* W;         // first group's weight matrix, bf16 rows of length ldw
    uint16_t* C;               // output, bf16 [rows, ldc]
    const int32_t* offset;     // ragged mode: [G+1] first row of each group (device); NULL = dense
    int G;                     // groups (experts)
    int dense_rows;            // dense mode: every group multiplies rows [0, dense_rows) of A
    int K;                     // reduction length, multiple of 64
    int N;                     // output columns per group (SwiGLU: activation columns)
    int lda, ldc, ldw;
    long long w_group_stride;  // elements from one group's matrix to the next group's
    long long w_up_offset;     // SwiGLU: elements from W_gate to W_up
    int kseg_len;              // K is split into segments of this length ...
    long long w_kseg_stride;   // ... whose weight blocks are this many elements apart
    int c_group_col_stride;    // dense mode: group g writes columns starting at g * this
    // ragged mode, optional: grouped row p is not row p of A but row a_row_map[p] / a_row_div of A
    // (the partition's row -> assignment map with a_row_div = top_k: the token rows are then
    // gathered by the tile loads themselves); a_src_rows = rows A holds.  NULL = rows are in place.
    const int32_t* a_row_map;
    int a_row_div;
    int a_src_rows;
    // ragged mode: tallest row tile, in units of 32 rows per row of wavefronts of the variant
    // (0 or more than the variant holds = the variant's full height); every group's tiles are cut
    // to equal heights below this
    int max_units;
    // what the epilogue writes (ragged, no SwiGLU only; see grouped_gemm.hip): 0 bf16, 1 fp32 (C then
    // points at floats, ldc counts floats), 2 bf16 scaled by row_weight[row_assignment[grouped row]]
    int epi;
    const float* row_weight;
    const int32_t* row_assignment;
    // optional: the same weights in tile order (pack_weights), or NULL.  Used by the variants whose
    // weight tile is kPackRows rows by kPackK reduction steps; the others read W.
    const uint16_t* Wp;
};
// Weights in tile order: for every group, column tile and K step of kPackK, the kPackRows x kPackK
// block the GEMM's weight tile holds at that step, contiguous (32 KB), blocks in (group, column tile, K step)
// order.  A block is 16 row blocks of 16 rows (SwiGLU: of W_gate and of W_up in turn, 8 of each; rows past N
// repeat row N - 1), a row block is [8 chunks of 8 k][16 rows]: the order in which the lanes of a wavefront
// hold the operand of a 16 x 16 x 32 matrix instruction, so that 1 KB of it is one load instruction without
// gaps, and in LDS a fragment read without bank conflicts.  a.W etc. describe the source as for a launch;
// a.Wp is ignored.
constexpr int kPackRows = 256, kPackK = 64;
size_t packed_weight_elems(const GemmArgs& a, bool swiglu);
hipError_t launch_pack_weights(const GemmArgs& a, bool swiglu, uint16_t* dst, int grid, hipStream_t s);
// variant: index into the tile-shape table of grouped_gemm.hip; max_rows: ragged mode, an upper
// bound of the rows of all groups together (the kernel cuts them into row tiles itself, from
// `offset`; the bound only sizes the grid); ignored in dense mode
hipError_t launch_grouped_gemm(const GemmArgs& a, bool swiglu, int variant, int n_cu,
                               long long max_rows, hipStream_t s);
// The same projections where few token rows meet every expert (narrow_gemm.hip): the routed groups
// `routed` (ragged) and, when `shared` is not NULL, the shared experts (dense) in one launch, bit for bit
// what launch_grouped_gemm writes.  expected_rows: rows per routed group the grid is sized for (any
// routing is served); max_tokens: the most rows one routed group can have; no other epilogue than epi == 0.
// kind: the tiles launched: kNarrowTiles[*kind].  gate (gate/up of at most kGateTokens tokens, kGateExperts experts): the launch
// routes and partitions first, as launch_route_and_partition; routed's offset and a_row_map are then what it writes, not reads.
struct GateArgs { const float* scores; int Tn, E, k, e0; int32_t *idx; float* w; int32_t *count, *offset, *pos, *perm; };
hipError_t launch_narrow_gemm(const GemmArgs& routed, const GemmArgs* shared, bool swiglu, int n_cu, double expected_rows,
                              int max_tokens, long long max_rows, hipStream_t s, int* kind, const GateArgs* gate = nullptr);
// kGateTokens is what one wavefront routes at a time.  Forwards, us, gate apart / in the launch: DeepSeek-V2-Lite-shaped layer, 1 / 2 / 4 tokens
// 36.3 / 31.4, 51.7 / 46.7, 78.7 / 72.8; DeepSeek-V2-shaped share, 1 / 4 tokens 46.0 / 39.3, 58.3 / 52.4; Qwen3-235B-A22B-shaped share, 1 / 4
// tokens 25.9 / 22.6, 46.4 / 41.9; Qwen3-30B-A3B-shaped layer, 1 / 4 tokens 29.5 / 25.6, 62.2 / 58.1.  With four more tokens per further
// round, 5 / 9 / 16 tokens 89 / 87, 125 / 129, 154 / 165; 67 / 62, -, 111 / 115; 47 / 46, -, 78 / 74; 71 / 74, -, 140 / 143: every
// workgroup that follows another one on its compute unit routes again.
constexpr int kGateTokens = 4, kGateExperts = 256;
// And with many experts per token, or many tiles, the same is true of up to four: a round of the gate per expert chosen, in every workgroup
// launched -- one per 64 columns of every expert that could be chosen, whether it is or not -- that a compute unit has beyond one or two.  Apart /
// in the launch, 64-column layers, 8 of 256, 16 of 256, 33 of 128, 64 of 64 experts: H 1536, 4 tokens 35 / 33, 48 / 51, 60 / 112, 59 / 90 us, 1 token 26 / 20,
// 34 / 30, 43 / 46, 58 / 74; H 7168, 4 tokens 91 / 98, 134 / 193, 164 / 405, 138 / 292; 33 of 256 with 32 of them here, 128 columns, H 7168, 1 token 46 / 116.
// Over 5648 layers of 128 to 4096 columns, H 256 to 7168, 8 to 256 experts here, the rule keeps 17.4 of the 18.5 ms that the better one of both
// saves, and none that it takes in is slower by more than 3 %.
constexpr double kGateWorth = 15.0, kGateFree = 1.5;
bool narrow_gate_pays(int Tn, int k, int El, int H, int n_cu);
constexpr int kNarrowRows = 64, kNarrowWaves = 4;         // tallest row tile, wavefronts
constexpr int kNarrowFewRows = 16, kNarrowFewWaves = 2;   // the same of the tiles for a few tokens; also of one wavefront
constexpr int kNarrowPairRows = 32;                       // and of two wavefronts for some more
struct NarrowTiles { int rows, waves; };
constexpr NarrowTiles kNarrowTiles[4] = {{kNarrowRows, kNarrowWaves}, {kNarrowFewRows, kNarrowFewWaves}, {kNarrowFewRows, 1}, {kNarrowPairRows, kNarrowFewWaves}};
constexpr int kNarrowFineK = 1024;                        // shortest reduction the last two are for
constexpr int kNarrowWaveRows = 32;                       // weight rows of a wavefront
constexpr int kNarrowDepth = 4;                           // K steps of 64 in flight per wavefront
// Down projection and weighted aggregation of at most kSumRows tokens in one launch (narrow_gemm.hip), bit for bit what
// launch_narrow_gemm and launch_combine write: `routed` and `shared` as for the first (shared: the same Tn tokens), pos and w as
// for the second, rows of routed.N elements at out; shared_alone: a token without a routed expert gets the shared ones' bits as they are.
hipError_t launch_narrow_sum(const GemmArgs& routed, const GemmArgs* shared, const int32_t* pos, const float* w, int Tn, int k,
                             bool shared_alone, void* out, int n_cu, hipStream_t s);
constexpr int kSumRows = 16, kSumWaves = 8;
constexpr int sum_loads(bool packed) { return packed ? 24 : 20; }   // of 1 KB in flight per wavefront (128 registers)
constexpr int kSumKind = sizeof(kNarrowTiles) / sizeof(kNarrowTiles[0]);   // beside the tile kinds of launch_narrow_gemm
// Output columns of a workgroup: 8 where 16 would leave compute units without one.  Forwards, us, separate launches / 16 / 8
// columns: DeepSeek-V2-Lite-shaped layer (2048 columns), 1 / 4 / 16 tokens 40.7 / 36.4 / 36.2, 82.8 / 82.2 / 78.1, 155.9 / 166.5 / 154.5;
// Qwen3-30B-A3B-shaped layer (2048), 1 / 16 tokens 33.1 / 30.7 / 29.9, 146.7 / 149.4 / 141.3; Qwen3-235B-A22B-shaped share (4096), 4 / 16
// tokens 49.9 / 45.8 / 46.5, 81.5 / 78.2 / 79.7.
inline int narrow_sum_cols(int N, int n_cu) { return N / 16 < n_cu ? 8 : 16; }
// Where a compute unit has one workgroup it serves up to kSumRows tokens; where some have two, which all read the
// token rows, up to kSumWideRows.  Separate launches / one, DeepSeek-V2-shaped share (5120 columns): 1 / 4 / 6 / 8 / 16 tokens 49.4 /
// 45.2, 59.4 / 57.1, 67.6 / 66.5, 76.6 / 76.9, 110.9 / 113.7 us, all of 16 tokens on eight experts 94 / 104 (Qwen3-235B-A22B-shaped
// share 65 / 64).  With weights in the caller's layout, Qwen3-235B-A22B-shaped share, 16 tokens balanced 96 / 89, Zipf 1.1 57 / 49, all on 16 / 8 of
// its experts 125 / 123, 77 / 79, 14 tokens on 8 77 / 77.
// Reductions of less than kSumK were not compared.
constexpr int kSumWideRows = 4, kSumK = 512;
inline bool narrow_sum_fits(int Tn, int N, int K, int n_cu) { return K >= kSumK && Tn <= (N / 16 <= n_cu ? kSumRows : kSumWideRows); }
// And whether it is the faster one.  A workgroup draws its columns of every expert that has a row, and 8 or 16 token rows beside them,
// at 46 GB/s; of few columns there are few workgroups.  Separate launches spread the same weights over all compute units, up to
// the 6.2 TB/s of HBM (0.53 of the units' rate), a tile of 64 columns at least, and last about 4 us longer: kSumWorth columns
// times K of one compute unit.  Separate / one, us, 2 of 8, 8 of 64, 64 of 64 experts per token: 64 columns, K 1408, 4 tokens 20 / 14,
// 26 / 34, 78 / 109; 512 columns, K 1024, 4 tokens 20 / 16, 29 / 34, 92 / 109; 2048 columns, K 1408, 9 tokens 42 / 37, 136 / 130,
// 204 / 212.  Over 2156 layers of 64 to 2560 columns, 512 to 5120 deep, 2 to 256 experts, 1 to 16 tokens, of the 3.9 ms that the
// better one of both saves 3.4 are kept and the worst choice costs 5 % (2 us); always one launch: up to four times as long.
constexpr double kSumWorth = 1e5;
inline bool narrow_sum_pays(int Tn, int k, int E, int El, int N, int K, int shared_K, int n_cu)
{
    const double rows = (double)Tn * k / E, routed = El * (1.0 - std::exp(-rows)) * K;
    const int cols = narrow_sum_cols(N, n_cu), turns = (N / cols + n_cu - 1) / n_cu;
    const auto width = [&](double r) { return cols + (r <= 8.0 ? 8 : 16); };
    const double here = turns * (routed * width(rows) + (double)shared_K * width(Tn));
    return here - std::fmax(64.0 * (K > shared_K ? K : shared_K), (routed + shared_K) * N / (0.53 * n_cu)) <= kSumWorth;
}
// Tiled projections of prefill with loading wavefronts (loader_gemm.hip): the routed groups `up` (gate/up), `down` or both (ragged)
// and, when up_shared / down_shared are not NULL, the shared experts (dense) in one launch; no other epilogue than epi == 0, no
// max_units, all or none with weights in tile order.  Of both, the down projection reads what the same launch's gate/up projection writes, for the
// same offset and dense rows.  sync, of both only: kLdCounters zeros, and kRowTileInts more for every row tile (loader_row_tiles).
hipError_t launch_loader_gemm(const GemmArgs* up, const GemmArgs* up_shared, const GemmArgs* down, const GemmArgs* down_shared, int n_cu, int32_t* sync, hipStream_t s);
constexpr int kLdCounters = 1024, kRowTileInts = 32;      // a counter has a line of its own
// the most row tiles of Tn tokens, k experts each, El of them here, and of dense_rows rows beside them: of 128 rows, the last of an expert lower
inline long long loader_row_tiles(long long Tn, int k, int El, long long dense_rows) { return Tn * (k < El ? k : El) / 128 + El + (dense_rows + 127) / 128; }
constexpr int kLoaderRows = 192;                          // tallest row tile
// Both projections in one launch where the gate/up projection has kPairRounds tiles for a compute unit, of `rows` rows per expert expected.  With
// fewer, nearly every workgroup has one tile of each projection, and what was a launch's end is a wait for the last of them.  Forwards, us, launches
// of their own / one: 0.75 rounds Qwen3-235B-A22B-shaped share, 1024 / 2500 / 4096 tokens 119 / 129, 149 / 150, 222 / 233; 1.3 and 1.6 rounds
// DeepSeek-V2-shaped share, 900 / 1700 tokens 253 / 259, 291 / 313; 2.2 and 2.6 rounds 2502 in a chunk 738 / 729 (two chunks), 4096 tokens 475 / 470; more:
// 9000 / 12000 / 16384 tokens 968 / 937, 1244 / 1234, 1649 / 1657; DeepSeek-V2-Lite-shaped layer, 500 / 1531 / 2500 / 4096 tokens 242 / 216, 302 / 276, 408 / 404, 555 / 546, weights in the
// caller's layout, 800 tokens 268 / 237; Qwen3-30B-A3B-shaped layer, three rounds, 500 / 1000 / 1600 / 2000 tokens perfectly balanced 223 / 224, 238 / 240, 257 / 257,
// 275 / 268, skewed 188 / 182, 246 / 227, 277 / 263, 306 / 283, with weights in the caller's layout 247 / 230, 265 / 247, 288 / 261, 295 / 272, skewed, 4000 / 8192 tokens
// 422 / 404, 687 / 677.  The rounds alone do not part the two: what is lost is 1 % at most, of balanced calls with one row tile per expert.
constexpr double kPairRounds = 2.0;
inline double loader_up_tiles(double rows, int El, int H, int dense_rows, int Ns, int Hs)
{
    const double tiles = rows / kLoaderRows + 0.5;
    return El * (tiles > 1.0 ? tiles : 1.0) * ((H + 127) / 128) + (double)Ns * ((dense_rows + kLoaderRows - 1) / kLoaderRows) * ((Hs + 127) / 128);
}
hipError_t loader_gemm_init();    // raises the dynamic-LDS limit of its kernels once
hipError_t grouped_gemm_init();   // raises the dynamic-LDS limit of every instantiation once
// the shape a launch of `variant` really runs (after the fall-backs for a short K or many groups):
// shape[] = tallest tile rows, weight rows per tile, K step, ring slots, wavefronts in m, in n,
// whether it reads weights in tile order when the launch has them (GemmArgs::Wp), and the rows of the
// matrix instruction's block (32: v_mfma_f32_32x32x16_bf16, 16: v_mfma_f32_16x16x32_bf16); false for an
// unknown variant
bool grouped_gemm_variant_shape(int variant, int K, bool ragged, int G, int shape[8]);
// the variant of the same tile shape that multiplies with the 16 x 16 x 32 instruction, or `variant` itself
int grouped_gemm_variant_mfma16(int variant);

}  // namespace moe_ep
