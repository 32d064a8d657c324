// The int8 GEMM over small tiles: batches and weights whose 256 x 256 tiles
// would leave most of the chip idle or multiply mostly padding, and rows of
// any length that is a multiple of 16.
//
//   k_gemm_tile      BM x BN output tile per workgroup of WM x WN waves, K in
//                    128-byte stages DMA'd into a ring of NST LDS buffers,
//                    optionally split into S slices per tile.
//   k_gemm_stream    batches of at most 16 tokens (decoding), below.
//
// What bounds k_gemm_tile: at few tokens the weight's stream from HBM and the
// latency of each workgroup's chain of stages (64 tokens 3584 -> 18944: 71 MB
// fetched in 17.1 us, 4.2 TB/s; 13 bytes a clock and compute unit through the
// DMA path, matrix cores 8 % busy), and with several tiles a unit the DMA path
// itself (1184 tiles of 64 x 64: 23 bytes a clock; a probe of it alone reaches
// 33).  So the shapes are chosen for bytes in flight: small rings, so that two
// (128 x 128, 64 KB), three (64 x 64, 48 KB) or four (32 x 64, 36 KB)
// workgroups share a CU and hide each other's barriers and epilogues; a 64 x 64
// ring of 5 stages, one workgroup per CU, took 25.2 us where 3 stages take 17.3
// (64 tokens, 3584 -> 18944), and one of 2 stages 20.1.  Measured per GEMM
// launch against the 256 x 256 kernel: 64 tokens 3584 -> 18944 42.1 -> 17.3 us,
// 64 tokens 18944 -> 3584 60 -> 19.1 us, 333 tokens 3584 -> 3584 30.5 -> 15.0
// us, 256 tokens 512 -> 512 (fp32) 28.4 -> 5.8 us.

#include "masq_device.h"

namespace masq {
namespace {

constexpr int kTsK = kTileStageK;

// Accumulates u L2^m onto the dequantised blocks of one wave (MI token blocks
// x NJ channel blocks of 32 x 32, lane = token lane % 32 and 4-channel groups
// as in the GEMM) for one modality m: token blocks' rows with live[i] false
// count as zero rows.  u rows: fp32 [T][r] at tok[i] (or, with u_hl, their
// bf16 hi/lo rows); rm: the modality's (L2^m)^T rows at chan[j].  All loads
// of a group of k steps are issued before its MFMAs.
template <typename LT> struct CompBlocks;

template <> struct CompBlocks<bf16_t> {
    template <int MI, int NJ>
    static __device__ __forceinline__ void run(v16f (&yb)[MI][NJ], const float* u, const uint8_t* u_hl,
                                               const bf16_t* rm, int r, const int64_t (&tok)[MI],
                                               const bool (&live)[MI], const int (&chan)[NJ], int lane) {
        const int kg = lane >> 5;
        const v4i zero = {0, 0, 0, 0};
        // (in: the step lies within r; a step past it multiplies zeros, both
        // operands, by selection, so that the loads of all steps stay in flight)
        auto mac = [&](const v4i (&hi)[MI], const v4i (&lo)[MI], const v4i (&b)[NJ], bool in)
                       __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const v8bf h = __builtin_bit_cast(v8bf, live[i] && in ? hi[i] : zero);
                const v8bf l = __builtin_bit_cast(v8bf, live[i] && in ? lo[i] : zero);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const v8bf bj = __builtin_bit_cast(v8bf, in ? b[j] : zero);
                    yb[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bj, h, yb[i][j], 0, 0, 0);
                    yb[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bj, l, yb[i][j], 0, 0, 0);
                }
            }
        };
        if (u_hl != nullptr) {                              // r <= 64: at most 4 steps of 16
            const int nks = r >> 4;
            v4i hi[4][MI], lo[4][MI], b[4][NJ];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int k = 16 * min(ks, nks - 1) + 8 * kg;
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const uint8_t* p = u_hl + tok[i] * 256 + 2 * k;
                    hi[ks][i] = *reinterpret_cast<const v4i*>(p);
                    lo[ks][i] = *reinterpret_cast<const v4i*>(p + 128);
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    b[ks][j] = *reinterpret_cast<const v4i*>(rm + static_cast<int64_t>(chan[j]) * r + k);
            }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) mac(hi[ks], lo[ks], b[ks], ks < nks);
            return;
        }
        for (int k0 = 0; k0 < r; k0 += 32) {                // r % 16 == 0: two steps a round
            v4i hi[2][MI], lo[2][MI], b[2][NJ];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int k = min(k0 + 16 * ks, r - 16) + 8 * kg;
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    float uv[8];
                    load8_f32(u + tok[i] * r + k, uv);
                    split_bf16x8(uv, hi[ks][i], lo[ks][i]);
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    b[ks][j] = *reinterpret_cast<const v4i*>(rm + static_cast<int64_t>(chan[j]) * r + k);
            }
            mac(hi[0], lo[0], b[0], true);
            mac(hi[1], lo[1], b[1], k0 + 16 < r);
        }
    }
};

template <> struct CompBlocks<float> {                      // fp32 MFMA, 8 steps of 2 columns
    template <int MI, int NJ>
    static __device__ __forceinline__ void run(v16f (&yb)[MI][NJ], const float* u, const uint8_t*,
                                               const float* rm, int r, const int64_t (&tok)[MI],
                                               const bool (&live)[MI], const int (&chan)[NJ], int lane) {
        for (int k0 = 0; k0 < r; k0 += 16) {                // r % 16 == 0; lane group g: columns 8 g ..
            const int k = k0 + 8 * (lane >> 5);
            float uv[MI][8], bv[NJ][8];
#pragma unroll
            for (int i = 0; i < MI; ++i) load8_f32(u + tok[i] * r + k, uv[i]);
#pragma unroll
            for (int j = 0; j < NJ; ++j) load8_f32(rm + static_cast<int64_t>(chan[j]) * r + k, bv[j]);
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const float a = live[i] ? uv[i][e] : 0.f;
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        yb[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[j][e], a, yb[i][j], 0, 0, 0);
                }
        }
    }
};

// LDS rows of a stage: A rows of 128 bytes, then B rows of 128 bytes (W4: 64
// bytes of packed codes).  The 16-byte piece c of a 128-byte row lies at
// place c ^ ((row / 2) % 8): the fragment reads of 32 consecutive rows at one
// piece take 256-byte LDS cycles of 16 lanes, in which the 8 row pairs hit 8
// different places.  (64-byte rows: 4 rows share a 256-byte line, piece c at
// c ^ ((row / 4) % 4).)
__device__ __forceinline__ int ts_swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int ts_swz4(int row) { return (row >> 2) & 3; }

constexpr int ts_stage_bytes(int bm, int bn, bool w4) { return bm * kTsK + bn * (w4 ? kTsK / 2 : kTsK); }

template <typename YT, typename LT, bool CMC, bool ACC, bool W4, int BM, int BN, int WM, int WN,
          int NST, int WPE>
__global__ __launch_bounds__(64 * WM * WN, WPE) void k_gemm_tile(
    const int8_t* __restrict__ A, const int8_t* __restrict__ B, const float* __restrict__ x_scale,
    const float* __restrict__ w_scale, int64_t T, int K, int N, int tiles_m, int tiles_n,
    const int32_t* __restrict__ mod, const float* __restrict__ u, const uint8_t* __restrict__ u_hl,
    int r, int n_mod, const LT* __restrict__ r_up, int32_t* __restrict__ acc_out,
    YT* __restrict__ y, int S, int32_t* __restrict__ part, int* __restrict__ tickets, bool a_pair) {
    constexpr int NW = WM * WN, NT = 64 * NW;
    constexpr int MI = BM / WM / 32, NJ = BN / WN / 32;     // 32 x 32 blocks of a wave
    constexpr int kRowB = W4 ? kTsK / 2 : kTsK;             // B bytes per row and stage
    constexpr int kStage = ts_stage_bytes(BM, BN, W4);
    constexpr int kDmaA = BM * kTsK / 1024 / NW, kDmaB = BN * kRowB / 1024 / NW;
    constexpr int kPer = kDmaA + kDmaB;                     // DMA instructions per wave and stage
    static_assert(kDmaA * NW * 1024 == BM * kTsK && kDmaB * NW * 1024 == BN * kRowB, "DMA shares");
    constexpr int kTrPitch = 80;                            // output transpose: 32 channels + 16 bytes
    static_assert(NST * kStage >= NW * 32 * kTrPitch, "transpose buffers fit the ring");
    __shared__ __attribute__((aligned(16))) uint8_t ring[NST * kStage];
    __shared__ int s_last;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    int tm, tn;
    if (!tile_coords_at(static_cast<int>(linear_block()), tiles_m, tiles_n * S, tm, tn)) return;
    const int sl = tn % S;                                  // k slice
    tn /= S;
    const int64_t row0 = static_cast<int64_t>(tm) * BM;
    const int col0 = tn * BN;
    const int nst_all = (K + kTsK - 1) / kTsK;
    const int per = (nst_all + S - 1) / S;
    const int s0 = sl * per;
    const int ns = min(per, nst_all - s0);                  // >= 1 (plan_tile)

    // the wave's epilogue operands, loaded first so that they land during the
    // main loop: tokens wm BM/WM + 32 i + lane % 32, channel groups of 4
    int64_t tok[MI];
    float dx[MI];
    int md[MI], chan[NJ];
    v4f ws[NJ][4];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        tok[i] = min(row0 + wm * (BM / WM) + 32 * i + (lane & 31), T - 1);
        dx[i] = x_scale[tok[i]];
        md[i] = CMC ? sane_mod(mod[tok[i]], n_mod) : 0;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c0 = col0 + wn * (BN / WN) + 32 * j;
        chan[j] = min(c0 + (lane & 31), N - 1);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            ws[j][g] = *reinterpret_cast<const v4f*>(w_scale + min(c0 + 8 * g + 4 * (lane >> 5), N - 4));
    }

    // ---- DMA: A 8 rows of 128 bytes per instruction, B likewise (W4: 16 rows
    // of 64).  Rows past T or N repeat the last one (results discarded).  In
    // the last stage of rows that end inside it, pieces past K read the
    // row's first piece of the stage; their A fragments count as zeros.
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ring));
    const int a_step = a_pair ? 2 * kTsK : kTsK;
    const int rem = K - (nst_all - 1) * kTsK;               // bytes of the last stage, 16..128
    const int8_t* src[kPer];
    int off[kPer], koff[kPer];                              // piece's offset in memory and in k
#pragma unroll
    for (int q = 0; q < kDmaA; ++q) {
        const int row = (wave * kDmaA + q) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ts_swz(row);
        src[q] = A + code_row(min(row0 + row, T - 1), K, a_pair) + static_cast<int64_t>(s0) * a_step;
        koff[q] = 16 * c;
        off[q] = a_pair ? (c >> 2) * 128 + (c & 3) * 16 : 16 * c;
    }
#pragma unroll
    for (int q = 0; q < kDmaB; ++q) {
        const int row = (wave * kDmaB + q) * (1024 / kRowB) + lane / (kRowB / 16);
        const int c = W4 ? (lane & 3) ^ ts_swz4(row) : (lane & 7) ^ ts_swz(row);
        src[kDmaA + q] = B + static_cast<int64_t>(min(col0 + row, N - 1)) * (W4 ? K / 2 : K) +
                         static_cast<int64_t>(s0) * kRowB;
        koff[kDmaA + q] = (W4 ? 32 : 16) * c;
        off[kDmaA + q] = 16 * c;
    }
    auto issue = [&](int st, int buf) __attribute__((always_inline)) {
        const bool last = s0 + st == nst_all - 1;           // uniform
        const uint32_t base = lds0 + static_cast<uint32_t>(buf * kStage);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t dst = base + static_cast<uint32_t>(
                                            q < kDmaA ? (wave * kDmaA + q) * 1024
                                                      : BM * kTsK + (wave * kDmaB + q - kDmaA) * 1024);
            const int o = last && koff[q] >= rem ? 0 : off[q];
            lds_dma16(src[q] + static_cast<int64_t>(st) * (q < kDmaA ? a_step : kRowB) + o,
                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(dst))));
        }
    };

    v16i acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v16i{0};

    // one stage: 4 steps of 32 k.  Lane group h = lane / 32 takes 16-byte
    // piece 2 ks + h of the rows (W4: the 8 packed bytes of the same codes).
    auto compute = [&](int buf, int valid) __attribute__((always_inline)) {   // valid: pieces within K
        const uint8_t* sa = ring + buf * kStage;
        const uint8_t* sb = sa + BM * kTsK;
        const int h = lane >> 5;
        const v4i zero = {0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            v4i fa[MI], fb[NJ];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int row = wm * (BM / WM) + 32 * i + (lane & 31);
                fa[i] = *reinterpret_cast<const v4i*>(sa + row * kTsK + (((2 * ks + h) ^ ts_swz(row)) << 4));
                if (valid < 8) fa[i] = 2 * ks + h < valid ? fa[i] : zero;
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int row = wn * (BN / WN) + 32 * j + (lane & 31);
                if constexpr (W4)
                    fb[j] = w4_operand(*reinterpret_cast<const v2i*>(
                        sb + row * kRowB + ((ks ^ ts_swz4(row)) << 4) + 8 * h));
                else
                    fb[j] = *reinterpret_cast<const v4i*>(sb + row * kRowB +
                                                          (((2 * ks + h) ^ ts_swz(row)) << 4));
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
        }
    };
    // this wave's loads of a stage are complete when at most `younger` later
    // stages' are in flight; the barrier publishes every wave's, and says
    // that every wave has read the stage before it
    auto publish = [&](int younger) __attribute__((always_inline)) {
        if (younger >= 3) MASQ_WAIT_VMCNT_LGKM0(3 * kPer);
        else if (younger == 2) MASQ_WAIT_VMCNT_LGKM0(2 * kPer);
        else if (younger == 1) MASQ_WAIT_VMCNT_LGKM0(kPer);
        else MASQ_WAIT_VMCNT_LGKM0(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    static_assert(NST >= 2 && NST <= 5, "publish counts up to three younger stages");

    for (int st = 0; st < NST - 1 && st < ns; ++st) issue(st, st);
    int st = 0, cur = 0, nxt = NST - 1;                     // stage, its buffer, the one to refill
    for (; st + NST - 1 < ns; ++st) {
        publish(NST - 2);
        issue(st + NST - 1, nxt);
        compute(cur, 8);
        cur = cur + 1 == NST ? 0 : cur + 1;
        nxt = nxt + 1 == NST ? 0 : nxt + 1;
    }
    for (; st < ns; ++st) {
        publish(min(ns - 1 - st, NST - 2));
        if (s0 + st == nst_all - 1 && rem < kTsK) compute(cur, rem >> 4);
        else compute(cur, 8);
        cur = cur + 1 == NST ? 0 : cur + 1;
    }
    if constexpr (W4) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] >>= 4;     // exact: 16 x the sum
    }

    if (S > 1) {
        // Every slice writes its accumulators to its slot of the tile's
        // workspace with agent-coherent stores (sc1) and counts its arrival
        // once they have completed; the last slice to arrive reads the
        // others' slots with the same policy and adds them (exact in any
        // order).  No fence, no waiting on other workgroups.
        constexpr int kV4 = MI * NJ * 4;
        constexpr int kSlot = BM * BN * 4;                  // bytes per slice slot
        constexpr int kPolicy = 16;                         // sc1
        const int tile = tm * tiles_n + tn;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            part + static_cast<int64_t>(tile) * S * (BM * BN), 0, S * kSlot, 0x00020000);
#pragma unroll
        for (int c = 0; c < kV4; ++c) {
            const v16i& blk = acc[c / (4 * NJ)][(c / 4) % NJ];
            const v4i v = {blk[4 * (c % 4)], blk[4 * (c % 4) + 1], blk[4 * (c % 4) + 2],
                           blk[4 * (c % 4) + 3]};
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, sl * kSlot + (c * NT + tid) * 16, 0, kPolicy);
        }
        MASQ_WAIT_VMCNT_LGKM0(0);
        __syncthreads();
        if (tid == 0)
            s_last = __hip_atomic_fetch_add(&tickets[tile], 1, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT) == S - 1;
        __syncthreads();
        if (!s_last) return;
        if (tid == 0) __hip_atomic_store(&tickets[tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int s2 = 0; s2 < S; ++s2) {
            if (s2 == sl) continue;
#pragma unroll
            for (int c = 0; c < kV4; ++c) {
                const v4i v = __builtin_amdgcn_raw_buffer_load_b128(
                    rs, s2 * kSlot + (c * NT + tid) * 16, 0, kPolicy);
                v16i& blk = acc[c / (4 * NJ)][(c / 4) % NJ];
#pragma unroll
                for (int e = 0; e < 4; ++e) blk[4 * (c % 4) + e] += v[e];
            }
        }
    } else {
        __syncthreads();                                    // the ring is free for the transposes
    }

    const int64_t trow = row0 + wm * (BM / WM);
    const int tcol = col0 + wn * (BN / WN);
    if constexpr (ACC) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int ch = tcol + 32 * j + 8 * g + 4 * (lane >> 5);
                    if (trow + 32 * i + (lane & 31) < T && ch < N) {
                        const v4i w = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2],
                                       acc[i][j][4 * g + 3]};
                        *reinterpret_cast<v4i*>(acc_out + tok[i] * N + ch) = w;
                    }
                }
        if (y == nullptr) return;
    }
    v16f yb[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                yb[i][j][e] = (static_cast<float>(acc[i][j][e]) * dx[i]) * ws[j][e >> 2][e & 3];
    if constexpr (CMC) {
        for (int m = 1; m < n_mod; ++m) {
            bool live[MI], any = false;
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                live[i] = md[i] == m;
                any = any || live[i];
            }
            if (__ballot(any) == 0ull) continue;            // wave-uniform
            CompBlocks<LT>::template run<MI, NJ>(yb, u, u_hl, r_up + static_cast<int64_t>(m - 1) * N * r,
                                                 r, tok, live, chan, lane);
        }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        if constexpr (sizeof(YT) == 2) {
            // through a per-wave LDS transpose, so that a store instruction
            // writes 64-byte row pieces; LDS operations of one wave execute
            // in order, so the buffer needs no further synchronisation
            uint8_t* scr = ring + wave * 32 * kTrPitch;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    v2i w;
                    w.x = static_cast<int32_t>(pack_bf16x2(yb[i][j][4 * g], yb[i][j][4 * g + 1]));
                    w.y = static_cast<int32_t>(pack_bf16x2(yb[i][j][4 * g + 2], yb[i][j][4 * g + 3]));
                    *reinterpret_cast<v2i*>(scr + (lane & 31) * kTrPitch + (8 * g + 4 * (lane >> 5)) * 2) = w;
                }
                const int ch = tcol + 32 * j + (lane & 3) * 8;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int rr = 16 * k + (lane >> 2);
                    const v4i d = *reinterpret_cast<const v4i*>(scr + rr * kTrPitch + (lane & 3) * 16);
                    if (trow + 32 * i + rr < T && ch < N)
                        *reinterpret_cast<v4i*>(y + (trow + 32 * i + rr) * N + ch) = d;
                }
            }
        } else {
            const bool ok = trow + 32 * i + (lane & 31) < T;
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int ch = tcol + 32 * j + 8 * g + 4 * (lane >> 5);
                    if (ok && ch < N) {
                        const v4f w = {yb[i][j][4 * g], yb[i][j][4 * g + 1], yb[i][j][4 * g + 2],
                                       yb[i][j][4 * g + 3]};
                        *reinterpret_cast<v4f*>(y + tok[i] * N + ch) = w;
                    }
                }
        }
    }
}

// ================================================================ decode GEMM
// At most 16 tokens: the layer is a stream of Wq from HBM.  A workgroup of
// four waves owns 64 output channels (16 a wave, v_mfma_i32_16x16x64_i8, the
// tokens as rows) and one of S k slices; q and Wq come in 128-byte stages
// through a ring of four LDS buffers filled by DMA (10 KB a stage, three of
// them in flight), up to three workgroups a CU, so that a grid of 296 channel
// groups (18944 channels) is resident at once without a split (1 token: 68 MB
// in 14.0 us, 4.9 TB/s).  With fewer groups the slices hand their int32
// partials over through agent-scope stores and an arrival counter per group,
// as k_gemm_tile does.
//
// The compensation of the tokens t with t % S == slice is formed by the
// workgroup itself while its first stages are in flight: the u slice partials
// of those tokens are added (thread groups over the slices, then the groups
// in order), and each thread sums over the rank for its channel.  The terms
// are handed over beside the partials.
//
// only_mod >= 0 (the MAS-only comparator, one launch per modality's weight):
// only the outputs of tokens of that modality are stored.
//
// Measured against the kernel it replaces (each wave's whole slice of Wq in
// registers, two or three workgroups a CU): 1 token 3584 -> 18944 18.8 ->
// 14.5 us, 16 tokens 22.7 -> 21.2 us (16.3 without compensation, whose loads
// hold the ring up for about 4 us; a ring of seven stages, two workgroups a
// CU, 22.0), 16 tokens 18944 -> 3584 22.7 -> 19.5 us, with packed codes 20.5
// -> 15.5 us, 4 tokens 8192 -> 28672 62.2 -> 53.7 us.
constexpr int kStrCh = 64;
constexpr int kStrStages = 4;
constexpr int kStrThreads = 256;

template <typename YT, typename LT, bool W4>
__global__ __launch_bounds__(kStrThreads, 3) void k_gemm_stream(
    const int8_t* __restrict__ A, const int8_t* __restrict__ B, const float* __restrict__ x_scale,
    const float* __restrict__ w_scale, int T, int K, int N, int S, const int32_t* __restrict__ mod,
    const float* __restrict__ u, int u_slices, int r, int n_mod, const LT* __restrict__ r_up,
    int32_t* __restrict__ part, int* __restrict__ tickets, YT* __restrict__ y, int only_mod) {
    constexpr int kRowB = W4 ? kTsK / 2 : kTsK;
    constexpr int kStage = kSmallMaxT * kTsK + kStrCh * kRowB;
    constexpr int kDmaB = kStrCh * kRowB / 1024 / 4;      // per wave: 2 (W4: 1); q: one for waves 0, 1
    __shared__ __attribute__((aligned(16))) uint8_t ring[kStrStages * kStage];
    __shared__ __attribute__((aligned(16))) float terms[kSmallMaxT][kStrCh];
    __shared__ int s_last;
    extern __shared__ __attribute__((aligned(16))) float su[];       // [own tokens][r]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = static_cast<int>(blockIdx.x) / S, sl = static_cast<int>(blockIdx.x) - g * S;
    const int col0 = g * kStrCh;
    const int nst_all = (K + kTsK - 1) / kTsK;
    const int per = (nst_all + S - 1) / S;
    const int s0 = sl * per;
    const int ns = min(per, nst_all - s0);                // >= 1 (tile_slices)

    // modalities of this workgroup's tokens (scalar)
    const bool cmc = u != nullptr;
    const int own = sl < T ? (T - sl + S - 1) / S : 0;
    unsigned present = 0;
    if (cmc)
        for (int i = 0; i < own; ++i) present |= 1u << sane_mod(mod[sl + i * S], n_mod);
    present = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(present & ~1u)));

    // u partials: item = 4 columns of one own token, summed over slices
    // [grp cnt, grp cnt + cnt) by thread group grp (one group when the items
    // fill the workgroup)
    const int nit = own * (r >> 2);
    const int grps = nit > 0 && 2 * nit <= kStrThreads ? min(kStrThreads / nit, 8) : 1;
    const int cnt = (u_slices + grps - 1) / grps;
    auto item_sum = [&](int it, int q0, int q1) __attribute__((always_inline)) {
        const int i = it / (r >> 2), c = it - i * (r >> 2);
        const float* src = u + static_cast<int64_t>(sl + i * S) * r + 4 * c;
        const int64_t step = static_cast<int64_t>(T) * r;
        v4f v = {0.f, 0.f, 0.f, 0.f};
        for (int q = q0; q < q1; q += 8) {
            v4f p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = *reinterpret_cast<const v4f*>(src + min(q + e, q1 - 1) * step);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (q + e < q1) v = v + p[e];              // slice order
        }
        return v;
    };

    // ---- DMA (rows past T or N repeat the last one; pieces past K read the
    // row's first piece of the stage, their q counts as zeros)
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ring));
    const int rem = K - (nst_all - 1) * kTsK;
    const int8_t *srcq, *srcw[kDmaB];
    int offq, offw[kDmaB];
    {
        const int row = (wave & 1) * 8 + (lane >> 3), c = (lane & 7) ^ ts_swz(row);
        srcq = A + static_cast<int64_t>(min(row, T - 1)) * K + static_cast<int64_t>(s0) * kTsK;
        offq = 16 * c;
    }
#pragma unroll
    for (int q = 0; q < kDmaB; ++q) {
        const int row = (wave * kDmaB + q) * (1024 / kRowB) + lane / (kRowB / 16);
        const int c = W4 ? (lane & 3) ^ ts_swz4(row) : (lane & 7) ^ ts_swz(row);
        srcw[q] = B + static_cast<int64_t>(min(col0 + row, N - 1)) * (W4 ? K / 2 : K) +
                  static_cast<int64_t>(s0) * kRowB;
        offw[q] = 16 * c;
    }
    auto issue = [&](int st, int buf) __attribute__((always_inline)) {
        const bool last = s0 + st == nst_all - 1;
        const uint32_t base = lds0 + static_cast<uint32_t>(buf * kStage);
        if (wave < 2)
            lds_dma16(srcq + static_cast<int64_t>(st) * kTsK + (last && offq >= rem ? 0 : offq),
                      base + static_cast<uint32_t>(wave * 1024));
#pragma unroll
        for (int q = 0; q < kDmaB; ++q)
            lds_dma16(srcw[q] + static_cast<int64_t>(st) * kRowB +
                          (last && (W4 ? 2 : 1) * offw[q] >= rem ? 0 : offw[q]),
                      base + static_cast<uint32_t>(kSmallMaxT * kTsK + (wave * kDmaB + q) * 1024));
    };
    auto publish = [&](int younger) __attribute__((always_inline)) {
        auto wait = [&](auto per_stage) __attribute__((always_inline)) {
            constexpr int P = decltype(per_stage)::value;
            static_assert(kStrStages == 4, "counts up to two younger stages");
            if (younger >= 2) MASQ_WAIT_VMCNT_LGKM0(2 * P);
            else if (younger == 1) MASQ_WAIT_VMCNT_LGKM0(P);
            else MASQ_WAIT_VMCNT_LGKM0(0);
        };
        if (wave < 2) wait(std::integral_constant<int, kDmaB + 1>{});
        else wait(std::integral_constant<int, kDmaB>{});
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    for (int st = 0; st < kStrStages - 1 && st < ns; ++st) issue(st, st);

    // ---- compensation terms of the own tokens: one copy of the code for
    // every token and rank
    if (present) {
        const int ch = min(col0 + lane, N - 1);
        Raw8<LT> rv[8];                                              // 64 columns of the channel's L2 row
        int have = -1;                                               // (modality, chunk) they are
        auto load_row = [&](int m, int k0) __attribute__((always_inline)) {
            const LT* rr = r_up + (static_cast<int64_t>(m - 1) * N + ch) * r;
#pragma unroll
            for (int q = 0; q < 8; ++q) rv[q].load(rr + min(k0 + 8 * q, r - 8));
            have = m * 64 + (k0 >> 6);
        };
        load_row(__builtin_ctz(present), 0);                         // in flight beside the u partials
        auto put = [&](int it, v4f v) __attribute__((always_inline)) {
            const int row = it / (r >> 2), c = it - row * (r >> 2);
            *reinterpret_cast<v4f*>(su + row * r + 4 * c) = v;
        };
        v4f* tmp = reinterpret_cast<v4f*>(&terms[0][0]);             // grps nit <= 256 items
        for (int it0 = tid; it0 < grps * nit; it0 += kStrThreads) {
            const int grp = it0 / nit, it = it0 - grp * nit;
            const v4f v = item_sum(it, min(grp * cnt, u_slices), min((grp + 1) * cnt, u_slices));
            if (grps > 1) tmp[it0] = v;
            else put(it, v);
        }
        __syncthreads();
        if (grps > 1) {
            if (tid < nit) {
                v4f v = tmp[tid];
                for (int q = 1; q < grps; ++q)
                    if (q * cnt < u_slices) v = v + tmp[q * nit + tid];
                put(tid, v);
            }
            __syncthreads();
        }
#pragma unroll 1
        for (int i = wave; i < own; i += 4) {                        // wave-uniform
            const int m = __builtin_amdgcn_readfirstlane(sane_mod(mod[sl + i * S], n_mod));
            float term = 0.f;
            if (m > 0) {
#pragma unroll 1
                for (int k0 = 0; k0 < r; k0 += 64) {
                    if (have != m * 64 + (k0 >> 6)) load_row(m, k0);
                    const float* ur = su + i * r + k0;
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if (k0 + 8 * q >= r) break;                  // uniform; no product past r (0 x inf)
                        float f[8], uv[8];
                        rv[q].to_f32(f);
                        load8_f32(ur + 8 * q, uv);
#pragma unroll
                        for (int e = 0; e < 8; ++e) term = fmaf(uv[e], f[e], term);
                    }
                }
                if (S > 1 && col0 + lane < N)
                    __hip_atomic_store(part + static_cast<int64_t>(S) * kSmallMaxT * N +
                                           static_cast<int64_t>(sl + i * S) * N + col0 + lane,
                                       __float_as_int(term), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (S == 1) terms[i][lane] = term;
        }
        // every load of this block is complete, so that none of its registers
        // is waited for in the main loop (which would drain the DMA ring)
        MASQ_WAIT_VMCNT_LGKM0(0);
    }

    // ---- main loop
    v4i acc = {0, 0, 0, 0};
    auto compute = [&](int buf, int valid) __attribute__((always_inline)) {
        const uint8_t* sa = ring + buf * kStage;
        const uint8_t* sb = sa + kSmallMaxT * kTsK;
        const int rw = lane & 15, cg = lane >> 4, brow = 16 * wave + rw;
        const v4i zero = {0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int c = 4 * ks + cg;
            v4i fa = *reinterpret_cast<const v4i*>(sa + rw * kTsK + ((c ^ ts_swz(rw)) << 4));
            if (valid < 8) fa = c < valid ? fa : zero;
            v4i fb;
            if constexpr (W4)
                fb = w4_operand(*reinterpret_cast<const v2i*>(
                    sb + brow * kRowB + (((c >> 1) ^ ts_swz4(brow)) << 4) + 8 * (c & 1)));
            else
                fb = *reinterpret_cast<const v4i*>(sb + brow * kRowB + ((c ^ ts_swz(brow)) << 4));
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb, acc, 0, 0, 0);
        }
    };
    int st = 0, cur = 0, nxt = kStrStages - 1;
    for (; st + kStrStages - 1 < ns; ++st) {
        publish(kStrStages - 2);
        issue(st + kStrStages - 1, nxt);
        compute(cur, 8);
        cur = (cur + 1) & (kStrStages - 1);
        nxt = (nxt + 1) & (kStrStages - 1);
    }
    for (; st < ns; ++st) {
        publish(min(ns - 1 - st, kStrStages - 2));
        compute(cur, s0 + st == nst_all - 1 ? rem >> 4 : 8);
        cur = (cur + 1) & (kStrStages - 1);
    }
    if constexpr (W4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] >>= 4;                    // exact: 16 x the sum
    }
    // acc[e]: token 4 (lane / 16) + e, channel col0 + 16 wave + lane % 16
    const int ch = col0 + 16 * wave + (lane & 15);
    if (S == 1) {
        __syncthreads();                                             // terms (written before the loop)
        if (ch >= N) return;
        const float dw = w_scale[ch];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 4 * (lane >> 4) + e;
            if (t >= T) continue;
            const int m = (cmc || only_mod >= 0) ? sane_mod(mod[t], n_mod) : 0;
            if (only_mod >= 0 && m != only_mod) continue;
            float v = (static_cast<float>(acc[e]) * x_scale[t]) * dw;
            if (cmc && m > 0) v += terms[t][16 * wave + (lane & 15)];
            Elem<YT>::store1(y + static_cast<int64_t>(t) * N + ch, v);
        }
        return;
    }
    // Hand-over without cache maintenance: agent-scope accesses, every store
    // complete (vmcnt 0) before the workgroup's arrival is counted.
    if (ch < N) {
        int32_t* pp = part + static_cast<int64_t>(sl) * kSmallMaxT * N + ch;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 4 * (lane >> 4) + e;
            if (t < T)
                __hip_atomic_store(pp + static_cast<int64_t>(t) * N, acc[e], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    MASQ_WAIT_VMCNT_LGKM0(0);
    __syncthreads();
    if (tid == 0)
        s_last = __hip_atomic_fetch_add(&tickets[g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == S - 1;
    __syncthreads();
    if (!s_last) return;
    if (tid == 0)                       // ready for the next launch
        __hip_atomic_store(&tickets[g], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // each thread finishes channel tid % 64 of tokens tid / 64 + 4 j
    constexpr int kOut = kSmallMaxT / 4;
    const int o = min(col0 + lane, N - 1);
    int pv[kOut][kDecMaxSlices], mv[kOut];
    float dxv[kOut], cv[kOut];
    const float dw = w_scale[o];
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
        const int t = min(wave + 4 * j, T - 1);
        const int32_t* pa = part + static_cast<int64_t>(t) * N + o;
#pragma unroll
        for (int q = 0; q < kDecMaxSlices; ++q)
            pv[j][q] = __hip_atomic_load(pa + static_cast<int64_t>(min(q, S - 1)) * kSmallMaxT * N,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        cv[j] = cmc ? __int_as_float(__hip_atomic_load(pa + static_cast<int64_t>(S) * kSmallMaxT * N,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    : 0.f;
        dxv[j] = x_scale[t];
        mv[j] = (cmc || only_mod >= 0) ? sane_mod(mod[t], n_mod) : 0;
    }
    if (col0 + lane >= N) return;
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
        const int t = wave + 4 * j;
        if (t >= T || (only_mod >= 0 && mv[j] != only_mod)) continue;
        int a = pv[j][0];
#pragma unroll
        for (int q = 1; q < kDecMaxSlices; ++q) a += q < S ? pv[j][q] : 0;
        float v = (static_cast<float>(a) * dxv[j]) * dw;
        if (cmc && mv[j] > 0) v += cv[j];
        Elem<YT>::store1(y + static_cast<int64_t>(t) * N + col0 + lane, v);
    }
}

template <typename YT, typename LT, bool CMC, bool ACC, bool W4>
hipError_t launch_tile_t(const TileGemm& g) {
    const int bm = kTileShapes[g.plan.shape].bm, bn = kTileShapes[g.plan.shape].bn;
    const int tiles_m = static_cast<int>((g.T + bm - 1) / bm);
    const int tiles_n = static_cast<int>((g.N + bn - 1) / bn);
    const int64_t nt = static_cast<int64_t>(tiles_m) * tiles_n * g.plan.S;
#define MASQ_TILE(BM, BN, WM, WN, NST, WPE)                                                         \
    hipLaunchKernelGGL((k_gemm_tile<YT, LT, CMC, ACC, W4, BM, BN, WM, WN, NST, WPE>),               \
                       grid_of(8 * ((nt + 7) / 8), 64 * WM * WN), dim3(64 * WM * WN), 0, g.stream,  \
                       g.q, g.wq, g.x_scale, g.w_scale, g.T, static_cast<int>(g.K),                 \
                       static_cast<int>(g.N), tiles_m, tiles_n, g.mod, g.u, g.u_hl, g.rank,         \
                       g.n_mod, static_cast<const LT*>(g.r_up), g.acc, static_cast<YT*>(g.y),       \
                       g.plan.S, g.part, g.tickets, g.a_pair)
    switch (g.plan.shape) {
        case 0: MASQ_TILE(32, 64, 1, 2, 3, 2); break;
        case 1: MASQ_TILE(64, 64, 2, 2, 3, 3); break;
        case 2: MASQ_TILE(128, 128, 2, 2, 2, 2); break;
        default: return hipErrorInvalidValue;
    }
#undef MASQ_TILE
    return hipGetLastError();
}

template <typename YT, typename LT, bool CMC, bool ACC>
hipError_t launch_tile_w(const TileGemm& g) {
    return g.w4 ? launch_tile_t<YT, LT, CMC, ACC, true>(g) : launch_tile_t<YT, LT, CMC, ACC, false>(g);
}

template <typename YT, typename LT, bool W4>
hipError_t launch_stream_t(const StreamGemm& g) {
    int ns = 0, sp = 0, groups = 0;
    plan_decode(g.K, g.N, ns, sp, groups);
    const int S = stream_slices(g.K, groups, ns);
    const size_t lds = g.u != nullptr ? static_cast<size_t>((g.T + S - 1) / S) * g.rank * sizeof(float)
                                      : 0;
    hipLaunchKernelGGL((k_gemm_stream<YT, LT, W4>), dim3(static_cast<unsigned>(groups * S)),
                       dim3(kStrThreads), lds, g.stream, g.q, g.wq, g.x_scale, g.w_scale,
                       static_cast<int>(g.T), static_cast<int>(g.K), static_cast<int>(g.N), S, g.mod, g.u,
                       g.u_slices, g.rank, g.n_mod, static_cast<const LT*>(g.r_up), g.part, g.tickets,
                       static_cast<YT*>(g.y), g.only_mod);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_stream(const StreamGemm& g) {
    if (!small_path(g.T, g.K) || g.N % 16 != 0 || g.part == nullptr || g.tickets == nullptr)
        return hipErrorInvalidValue;
#define MASQ_STREAM(YT, LT) (g.w4 ? launch_stream_t<YT, LT, true>(g) : launch_stream_t<YT, LT, false>(g))
    if (g.y_dt == DT::BF16) return g.lr_dt == DT::BF16 ? MASQ_STREAM(bf16_t, bf16_t) : MASQ_STREAM(bf16_t, float);
    return g.lr_dt == DT::BF16 ? MASQ_STREAM(float, bf16_t) : MASQ_STREAM(float, float);
#undef MASQ_STREAM
}

hipError_t launch_gemm_tile(const TileGemm& g) {
    if (g.K % 16 != 0 || g.N % 16 != 0 || g.plan.S < 1 || (g.w4 && g.K % 64 != 0) ||
        (g.a_pair && g.K % 64 != 0) || (g.plan.S > 1 && (g.part == nullptr || g.tickets == nullptr)))
        return hipErrorInvalidValue;
    // the int32 accumulator output exists only for the plain product
    if (!g.cmc) {
        if (g.acc != nullptr)
            return g.y_dt == DT::BF16 ? launch_tile_w<bf16_t, bf16_t, false, true>(g)
                                      : launch_tile_w<float, bf16_t, false, true>(g);
        return g.y_dt == DT::BF16 ? launch_tile_w<bf16_t, bf16_t, false, false>(g)
                                  : launch_tile_w<float, bf16_t, false, false>(g);
    }
    if (g.y_dt == DT::BF16)
        return g.lr_dt == DT::BF16 ? launch_tile_w<bf16_t, bf16_t, true, false>(g)
                                   : launch_tile_w<bf16_t, float, true, false>(g);
    return g.lr_dt == DT::BF16 ? launch_tile_w<float, bf16_t, true, false>(g)
                               : launch_tile_w<float, float, true, false>(g);
}

}  // namespace masq
