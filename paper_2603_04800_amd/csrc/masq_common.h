// Internal declarations shared by the kernel and C-ABI translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace masq {

// A grid of n workgroups of `threads`, in one dimension where its threads stay
// below the 2^32 that the runtime takes in one, else in rows of a multiple of
// 8 workgroups (the XCDs are dealt in turn as before); the kernel counts them
// with linear_block() and those past n find no work.
inline dim3 grid_of(int64_t n, int threads) {
    const int64_t most = ((int64_t{1} << 32) / threads - 1) / 8 * 8;
    if (n <= most) return dim3(static_cast<unsigned>(n));
    const int64_t rows = (n + most - 1) / most, x = ((n + rows - 1) / rows + 7) / 8 * 8;
    return dim3(static_cast<unsigned>(x), static_cast<unsigned>((n + x - 1) / x));
}
__device__ __forceinline__ int64_t linear_block() {
    return static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
}

// Tile shape of the int8 GEMM: 256 x 256 output tile per workgroup of eight
// wave64s (2 x 4, each wave 128 x 64), 64-byte K stages in a ring of four LDS
// buffers.
constexpr int kTileM = 256;
constexpr int kTileN = 256;
constexpr int kRowsDown = 16;     // rows per down-projection tile
constexpr int kDownRows = kRowsDown;
constexpr int kDownStep = 512;    // k granularity of a down-projection slice (128 per wave)
constexpr int kMaxRank = 256;
constexpr int kSmallMaxT = 16;    // batches this small use the Wq-streaming GEMM
constexpr int kSmallSlices = 64;  // down-projection k slices (at most; >= 512 columns each) summed by that GEMM

// The small-batch path: the Wq-streaming GEMM, which also adds the
// down-projection's k-slice partials itself.
inline bool small_path(int64_t T, int64_t K) { return T <= kSmallMaxT && K % 64 == 0; }

// Layout of the fused layer's int8 activation codes in its workspace.  Plain:
// code (t, k) at byte t K + k.  Row-paired (paired_codes: K % 64 == 0 and a
// batch past the small path, whose GEMM takes its A operand by LDS DMA): rows
// 2i and 2i + 1 interleave in 64-byte pieces, code (t, k) at byte
// (t / 2) 2K + (k / 64) 128 + (t % 2) 64 + k % 64, so that the two rows'
// 64-column pieces of one K stage are a single 128-byte line (one L2 request
// where the plain rows take two 64-byte ones).  An odd batch's last pair has
// an unused second row (the workspace holds T rounded up to even rows).
inline bool paired_codes(int64_t T, int64_t K) { return !small_path(T, K) && K % 64 == 0; }
__host__ __device__ inline int64_t code_row(int64_t t, int64_t K, bool pair) {
    return pair ? (t >> 1) * 2 * K + (t & 1) * 64 : t * K;
}
__host__ __device__ inline int code_col(int k, bool pair) { return pair ? k + (k & ~63) : k; }

// Stage 1 of large batches with bf16 factors, rank <= 64 (fused_stage1_ok),
// in its wide form: the down-projection runs over 128-row tiles and S k
// slices of kslice columns (about 512 workgroups, slices of at least 256
// columns); the quantisation kernel then adds the slices' partials into u.
// The fused stage 1 walks each 16-row tile along its whole row, so its time
// grows with K and hardly with T until its T / 16 workgroups reach one per
// compute unit (4096 tokens); it keeps rows shorter than 2048 columns (too
// few k slices for the wide form) and, from 4096 tokens on, rows shorter
// than 8192 columns (where reading each row once, not twice, wins).
constexpr int64_t kDownWideMinK = 2048;
constexpr int64_t kFusedFullT = 4096;
constexpr int64_t kDownWideLongK = 8192;
constexpr int kDownWideRows = 128;
inline bool down_wide(int64_t T, int64_t K) {
    return K >= kDownWideMinK && (T < kFusedFullT || K >= kDownWideLongK);
}
inline void plan_down_wide(int64_t T, int64_t K, int& S, int& kslice) {
    const int64_t tiles = (T + kDownWideRows - 1) / kDownWideRows;
    int64_t want = (512 + tiles - 1) / tiles;
    const int64_t most = (K + 255) / 256;
    if (want > most) want = most;
    if (want < 1) want = 1;
    kslice = static_cast<int>(((K + want - 1) / want + 63) / 64 * 64);
    S = static_cast<int>((K + kslice - 1) / kslice);
}

// K split of the 256 x 256 tile GEMM for grids with few tiles (fused layer,
// K % 64 == 0): S slices of at least 8 64-byte stages; each slice's int32
// accumulators go to the workspace and the last slice of a tile to arrive
// adds them and finishes the tile.
constexpr int kSplitMaxTiles = 128;   // grids with at least this many tiles are not split
constexpr int kSplitMax = 4;
inline int plan_gemm_splits(int64_t T, int64_t K, int64_t N) {
    if (T <= 0 || N <= 0 || small_path(T, K) || K % 64 != 0) return 1;
    const int64_t tiles = ((T + kTileM - 1) / kTileM) * ((N + kTileN - 1) / kTileN);
    if (tiles >= kSplitMaxTiles) return 1;
    int64_t S = 256 / tiles;
    if (S > kSplitMax) S = kSplitMax;
    if (S > (K / 64) / 8) S = (K / 64) / 8;
    return S < 1 ? 1 : static_cast<int>(S);
}

// Small-tile GEMM (k_gemm_tile): output tile shapes, and the shape and number
// of k slices a product takes.  shape < 0: the 256 x 256 kernel.
struct TileShape { int bm, bn; };
constexpr TileShape kTileShapes[] = {{32, 64}, {64, 64}, {128, 128}};
struct TilePlan { int shape, S; };
// split: slices are possible (the caller has room for their accumulators);
// slow_comp: compensation with fp32 factors or a rank past 64.
TilePlan plan_tile(int64_t T, int64_t K, int64_t N, bool split, bool w4, bool slow_comp = false);
constexpr int kTileStageK = 128;      // codes per stage of the small-tile GEMM
// At most S slices of whole stages, none of them empty.
inline int tile_slices(int64_t K, int S) {
    const int n = static_cast<int>((K + kTileStageK - 1) / kTileStageK);
    if (S > n) S = n;
    if (S <= 1) return 1;
    const int per = (n + S - 1) / S;
    return (n + per - 1) / per;
}

// Decode GEMM of the fused small-batch path (k_gemm_stream): channel groups of
// kDecCh, and the k slices its workspace holds room for: ns slices of sp
// 64-byte steps, sp <= kDecSteps.
constexpr int kDecSteps = 40;
constexpr int kDecCh = 64;
constexpr int kDecMaxSlices = 8;    // at most this many are used
inline void plan_decode(int64_t K, int64_t N, int& ns, int& sp, int& ngroups) {
    const int64_t nsteps = K / 64;
    const int64_t ns0 = (nsteps + kDecSteps - 1) / kDecSteps;
    sp = static_cast<int>((nsteps + ns0 - 1) / ns0);
    ns = static_cast<int>((nsteps + sp - 1) / sp);
    ngroups = static_cast<int>((N + kDecCh - 1) / kDecCh);
}
// Slices the decode GEMM takes of the `most` that the workspace holds: none
// for 256 channel groups and more, else up to about 448 workgroups.
inline int stream_slices(int64_t K, int groups, int most) {
    int S = groups >= 256 ? 1 : 448 / groups;
    if (S > most) S = most;
    if (S > kDecMaxSlices) S = kDecMaxSlices;
    return tile_slices(K, S);
}
constexpr int64_t kRowsPerWaveMinT = 256;   // batches this large quantise one row per wave

enum class DT : int { F32 = 0, BF16 = 1 };

struct LinearArgs {
    const void* x;
    DT x_dt;
    const int32_t* modality;
    const float* inv_smooth;
    const int8_t* wq;
    const float* w_scale;
    const void* l_down;
    const void* r_up;
    DT lr_dt;
    int64_t T, K, N;
    int rank, n_mod;
    void* y;
    DT y_dt;
};

// Workspace carve-up of the fused layer.
struct Workspace {
    int8_t* q;         // codes, row-paired when `pair` (code_row / code_col)
    bool pair;         // paired_codes(T, K)
    float* x_scale;
    float* u;          // [T][rank] fp32 down-projection u = (x S^-1) L1
    uint8_t* u_hl;     // [T][256 B] u as bf16 hi | lo rows (rank <= 64, large batches)
    float* u_part;     // [n_kslices][T][rank] fp32 partial sums over k slices (n_kslices > 1)
    int* tickets;      // [ceil(T / kDownRows)] arrival counters of the slice workgroups
    int32_t* dec_part; // small-batch path: [ns][kSmallMaxT][N] int32 partial sums per k slice,
                       // then [kSmallMaxT][N] fp32 compensation terms
    int* dec_tickets;  // small-batch path: [ngroups] arrival counters (zeroed by stage 1)
    int dec_groups;    // plan_decode's channel groups (small-batch path)
    TilePlan tile;     // plan_tile: the small-tile GEMM's shape and slices (shape < 0: 256 x 256)
    int gk_splits;     // plan_gemm_splits (256 x 256 tiles)
    int32_t* gk_part;  // [tiles][slices][bm * bn] int32 slice accumulators (slices > 1)
    int* gk_tickets;   // [tiles] arrival counters (gk_splits > 1); follow `tickets` when both exist
    int n_zero;        // ints from zero_base that stage 1 clears
    int* zero_base;
    int dw_slices, dw_kslice;   // plan_down_wide (dw_part != nullptr)
    float* dw_part;    // [dw_slices][T][rank] fp32 partials of the wide down-projection
    int dl_quarters, dl_slices;   // k slices of k_down_lds (dl_part != nullptr)
    float* dl_part;    // [dl_slices][T][rank] fp32 partials of k_down_lds
    int n_kslices;
    int kslice;
    size_t bytes;
};

Workspace plan_workspace(void* base, int64_t T, int64_t K, int64_t N, int rank, int n_mod,
                         bool w4 = false, bool slow_comp = false);

// zero_ints / n_zero: optional array the kernel clears on the way (the
// down-projection's tickets, which must start at zero).
// fin (optional): add the wide down-projection's slice partials into u (and
// its bf16 hi/lo rows) while quantising.  pair: write the codes row-paired
// (code_row / code_col; K % 64 == 0).
struct UFinish {
    const float* part;   // [slices][T][r]
    int slices, r;
    float* u;
    uint8_t* u_hl;       // may be null
};
hipError_t launch_smooth_quant(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                               int64_t T, int64_t K, int n_mod, int8_t* q, float* x_scale,
                               int* zero_ints, int n_zero, hipStream_t s,
                               const UFinish* fin = nullptr, bool pair = false);

hipError_t launch_down_wide(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                            const void* l_down, int64_t T, int64_t K, int rank, int n_mod,
                            const Workspace& w, hipStream_t s);

hipError_t launch_lowrank_down(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                               const void* l_down, DT lr_dt, int64_t T, int64_t K, int rank,
                               int n_mod, const Workspace& w, hipStream_t s);

// Quantisation and the down-projection in one launch: one k slice of u a
// tile (no arrival counters, which the launch itself would have to clear).
// Batches whose tiles and rows together pass a launch's 2^32 threads (512
// for every 16 rows of u and every 8 of codes: 44.7 million tokens) take the
// two launches, each of which reaches further.
constexpr int64_t kQuantDownMaxK = 4096;
inline bool quant_down_ok(const Workspace& w, int64_t T, int64_t K) {
    return w.n_kslices == 1 && K <= kQuantDownMaxK &&
           ((T + kDownRows - 1) / kDownRows + (T + 7) / 8) * 512 < (int64_t{1} << 32);
}
hipError_t launch_quant_down(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                             const void* l_down, DT lr_dt, int64_t T, int64_t K, int rank, int n_mod,
                             const Workspace& w, hipStream_t s);

// Stage 1 in one kernel for bf16 factors and rank <= 64 (fused_stage1_ok):
// smoothing, quantisation and the down-projection, reading each row once.
inline bool fused_stage1_ok(int64_t T, int64_t K, int rank, DT lr_dt) {
    return !small_path(T, K) && lr_dt == DT::BF16 && rank > 0 && rank <= 64;
}
// The register-resident form of stage 1 (smoothing, quantisation and, for
// bf16 factors of rank <= 64, the down-projection): bf16 activations, 16 rows
// per workgroup of kFrWaves waves, rows of a multiple of 64 columns up to
// kFrWaves x kFrMaxPairs x 64 (each wave holds at most kFrMaxPairs 64-column
// pairs of its 16 rows in registers), and the smoothing factors of every
// modality within kFrInvFloats floats of LDS, each modality's row at a
// stride of fr_inv_stride(K) floats (whole 1 KB blocks plus 16 bytes, so that
// lanes reading different modalities' factors hit different banks).
constexpr int kFrWaves = 8;
constexpr int kFrMaxPairs = 8;
constexpr int kFrInvFloats = 12304;
__host__ __device__ inline int64_t fr_inv_stride(int64_t K) { return (K + 255) / 256 * 256 + 4; }
inline bool stage1_fr_ok(DT x_dt, int64_t K, int n_mod) {
    return x_dt == DT::BF16 && K % 64 == 0 && K <= int64_t{kFrWaves} * kFrMaxPairs * 64 &&
           static_cast<int64_t>(n_mod) * fr_inv_stride(K) <= kFrInvFloats;
}
// Down-projection with the L1 fragments staged in LDS (k_down_lds): bf16
// activations and factors, rank <= 64, K % 64 == 0; slice partials
// [slices][T][rank] for the quantisation kernel to add.
constexpr int64_t kDownLdsCols = 256;    // columns staged in LDS at a time (a chunk)
constexpr int64_t kDownLdsRows = 128;    // rows of a workgroup's tile
// Chunks per k slice: the workgroups (two per CU: 66 KB of LDS each) stream
// the chunks of their slice through a software pipeline, so the slices are
// made as long as a grid of about kDownLdsWgs workgroups (one round) allows:
// fewer partials to write and to add.
constexpr int64_t kDownLdsWgs = 512;
inline int down_lds_chunks(int64_t T, int64_t K) {
    const int64_t chunks = (K + kDownLdsCols - 1) / kDownLdsCols;
    const int64_t tiles = (T + kDownLdsRows - 1) / kDownLdsRows;
    const int64_t n = (tiles * chunks + kDownLdsWgs - 1) / kDownLdsWgs;
    return static_cast<int>(n < 1 ? 1 : (n > chunks ? chunks : n));
}
// Quarters (64 columns) per k slice.  Batches whose chunks are at most half
// as many workgroups as compute units take slices of two where the workspace
// of the longer slices has room for their partials (plan_workspace): a
// workgroup's time is its quarters' latency, one after the other, and the
// chip has room for twice the workgroups.  Stage 1 in slices of four / of two:
// 300 x 512 10.0 / 8.2 us, 512 x 3584 (two non-text modalities) 13.0 / 10.5,
// 1000 x 3584 12.3 / 11.4.  Layers without that room, those whose GEMM is not
// split, keep the longer slices: the size asked for is one that callers keep.
inline int down_lds_quarters(int64_t T, int64_t K) {
    const int64_t chunks = (K + kDownLdsCols - 1) / kDownLdsCols;
    const int64_t tiles = (T + kDownLdsRows - 1) / kDownLdsRows;
    return tiles * chunks <= 128 ? 2 : 4 * down_lds_chunks(T, K);
}
inline int down_lds_slices(int64_t K, int quarters) {
    return static_cast<int>(((K + 63) / 64 + quarters - 1) / quarters);
}
inline bool down_lds_ok(DT x_dt, int64_t K) { return x_dt == DT::BF16 && K % 64 == 0; }
// Stage 1 of the fused layer for rows that k_stage1_fr cannot hold: k_down_lds,
// then the quantisation adding its partials.
constexpr bool kStage1SplitDown = true;
// Rows that k_stage1_fr can hold take it only for batches of kFusedFullT
// tokens and more with at most one non-text modality; other batches take
// the split form as well.  k_stage1_fr reads the whole of L1 for every
// non-text modality present in each 16-row group, k_down_lds once per
// 128-row tile and k slice; below kFusedFullT tokens k_stage1_fr's T / 16
// workgroups leave compute units idle, and with two non-text modalities
// more of its groups read two L1s.  (Measured, rank 64, 3584 columns:
// 2048 tokens 22.2 -> 17.7 us with one non-text modality, 33.3 -> 19.4 us
// with two; 4096 tokens 24.1 -> 25.9 us with one, 35.4 -> 31.2 us with two;
// 8192 tokens 47.7 -> 51.9 us with one, 60.1 -> 57.9 us with two.)
inline bool stage1_fr_first(int64_t T, int n_mod) { return T >= kFusedFullT && n_mod <= 2; }
hipError_t launch_down_lds(const void* x, const int32_t* mod, const float* inv_s,
                           const void* l_down, int64_t T, int64_t K, int rank, int n_mod,
                           int quarters, float* part, hipStream_t s);

hipError_t launch_stage1_fused(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                               const void* l_down, int64_t T, int64_t K, int rank, int n_mod,
                               int8_t* q, float* x_scale, float* u, uint8_t* u_hl,
                               int* zero_ints, int n_zero, hipStream_t s, bool pair = false);

// Stage 1 of the small-batch path (small_path): quantisation of every row
// and the k-sliced down-projection (partials) in one launch.
hipError_t launch_stage1_small(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                               const void* l_down, DT lr_dt, int64_t T, int64_t K, int rank,
                               int n_mod, bool cmc, const Workspace& w, hipStream_t s);

// u: the down-projection; on the small-batch path (small_path) with
// n_kslices > 1 the GEMM adds the slice partials u_part itself.  u_hl
// (optional): u as bf16 hi/lo rows, written by the fused stage 1.  dec_part /
// dec_tickets (optional, small-batch path): workspace of the decode GEMM;
// without them (the standalone product, no compensation) the single-pass
// small-batch GEMM runs.  w4: wq holds packed 4-bit codes ([N][K / 2] bytes,
// K % 64 == 0).  a_pair: q is row-paired (code_row / code_col), which the
// 256 x 256 and the small-tile kernel read (K % 64 == 0, batches past the
// small path).
hipError_t launch_gemm(const int8_t* q, const float* x_scale, const int8_t* wq,
                       const float* w_scale, int64_t T, int64_t K, int64_t N,
                       const int32_t* mod, const float* u, const uint8_t* u_hl,
                       int32_t* dec_part, int* dec_tickets, int gk_splits, int32_t* gk_part,
                       int* gk_tickets, const float* u_part, int n_kslices,
                       int rank, int n_mod, const void* r_up, DT lr_dt, bool cmc, int32_t* acc,
                       void* y, DT y_dt, hipStream_t s, TilePlan tile, bool w4 = false,
                       bool a_pair = false);

// The small-tile GEMM; arguments as launch_gemm's.  part / tickets: plan.S
// slots of bm x bn int32 per tile and an arrival counter (zero on entry, left
// zero) per tile, for plan.S > 1.
struct TileGemm {
    const int8_t* q;
    const float* x_scale;
    const int8_t* wq;
    const float* w_scale;
    int64_t T, K, N;
    const int32_t* mod;
    const float* u;
    const uint8_t* u_hl;
    int rank, n_mod;
    const void* r_up;
    DT lr_dt;
    bool cmc;
    int32_t* acc;
    void* y;
    DT y_dt;
    bool w4, a_pair;
    TilePlan plan;
    int32_t* part;
    int* tickets;
    hipStream_t stream;
};
hipError_t launch_gemm_tile(const TileGemm& g);

// The decode GEMM (small_path): u (null without compensation) holds u_slices
// partials [T][rank]; part: the decode workspace's [slices + 1][kSmallMaxT][N],
// tickets: a counter per 64 channels (zero on entry, left zero).
struct StreamGemm {
    const int8_t* q;
    const float* x_scale;
    const int8_t* wq;
    const float* w_scale;
    int64_t T, K, N;
    const int32_t* mod;
    const float* u;
    int u_slices, rank, n_mod;
    const void* r_up;
    DT lr_dt;
    void* y;
    DT y_dt;
    bool w4;
    int32_t* part;
    int* tickets;
    int only_mod;
    hipStream_t stream;
};
hipError_t launch_gemm_stream(const StreamGemm& g);

// MAS-only comparator (a weight per modality, no compensation): rows grouped
// by modality on the device, then the direct-to-LDS GEMM over tiles of one
// modality each (K % 64 == 0).  The tile table holds at most
// grouped_tab_max entries {first row, rows, modality, 0}.  The codes q are
// row-paired (code_row / code_col), the quantiser's pair layout.
inline int grouped_tab_max(int64_t T, int n_mod) {
    return static_cast<int>((T + kTileM - 1) / kTileM) + n_mod - 1;
}
hipError_t launch_group_rows(const int32_t* mod, int64_t T, int n_mod, int32_t* rows,
                             int32_t* tab, int* tab_n, int* zero_ints, int n_zero, hipStream_t s);
// MAS-only at small batches (small_path, plan_decode's slices within
// kDecMaxSlices): the decode GEMM once per modality's weight (wq
// [n_mod][N][K], w_scale [n_mod][N]), each launch storing the outputs of its
// modality's tokens only; plain codes.  part / tickets: the decode GEMM's
// workspace (tickets zero before the first launch; each launch leaves them
// zero).
hipError_t launch_gemm_decode_mas(const int8_t* q, const float* x_scale, const int8_t* wq,
                                  const float* w_scale, int64_t T, int64_t K, int64_t N,
                                  const int32_t* mod, int n_mod, int32_t* part, int* tickets,
                                  void* y, DT y_dt, hipStream_t s);
hipError_t launch_gemm_grouped(const int8_t* q, const float* x_scale, const int8_t* wq,
                               const float* w_scale, int64_t T, int64_t K, int64_t N, int n_mod,
                               const int32_t* rows, const int32_t* tab, const int* tab_n, void* y,
                               DT y_dt, int S, int32_t* part, int* tickets, hipStream_t s);

hipError_t launch_lowrank_comp(const void* x, DT x_dt, const int32_t* mod, const float* inv_s,
                               const void* l_down, const void* r_up, DT lr_dt, int64_t T,
                               int64_t K, int64_t N, int rank, int n_mod, void* y, DT y_dt,
                               hipStream_t s);

}  // namespace masq
