// The int8 GEMM over small tiles: batches and weights whose 256 x 256 tiles
// would leave most of the chip idle or multiply mostly padding, and rows of
// any length that is a multiple of 16.
//
//   k_gemm_tile      BM x BN output tile per workgroup of WM x WN waves, K in
//                    128-byte stages DMA'd into a ring of NST LDS buffers,
//                    optionally split into S slices per tile.
//
// What bounds it: the bytes a compute unit can pull through its DMA path (33
// to 40 bytes a clock; a 64 x 64 tile needs 16 KB per 64 clocks of MFMA),
// and at few tokens the weight's stream from HBM.  So the shapes are chosen
// for bytes in flight: small rings, so that two (128 x 128, 64 KB), three
// (64 x 64, 48 KB) or four (32 x 64, 36 KB) workgroups share a CU and hide
// each other's barriers and epilogues; a 64 x 64 ring of 5 stages, one
// workgroup per CU, took 25.2 us where 3 stages take 17.3 (64 tokens, 3584
// -> 18944), and one of 2 stages 20.1.  Measured per GEMM launch against the
// 256 x 256 kernel: 64 tokens 3584 -> 18944 42.1 -> 17.3 us, 64 tokens 18944
// -> 3584 60 -> 19.1 us, 333 tokens 3584 -> 3584 30.5 -> 15.0 us, 256 tokens
// 512 -> 512 (fp32) 28.4 -> 5.8 us.

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
        // (in: the step lies within r; a step past it multiplies zeros, without
        // a branch between the MFMAs)
        auto mac = [&](const v4i (&hi)[MI], const v4i (&lo)[MI], const v4i (&b)[NJ], bool in)
                       __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const v8bf h = __builtin_bit_cast(v8bf, live[i] && in ? hi[i] : zero);
                const v8bf l = __builtin_bit_cast(v8bf, live[i] && in ? lo[i] : zero);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const v8bf bj = __builtin_bit_cast(v8bf, b[j]);
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
    if (!tile_coords_at(static_cast<int>(blockIdx.x), tiles_m, tiles_n * S, tm, tn)) return;
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

template <typename YT, typename LT, bool CMC, bool ACC, bool W4>
hipError_t launch_tile_t(const TileGemm& g) {
    const int bm = kTileShapes[g.plan.shape].bm, bn = kTileShapes[g.plan.shape].bn;
    const int tiles_m = static_cast<int>((g.T + bm - 1) / bm);
    const int tiles_n = static_cast<int>((g.N + bn - 1) / bn);
    const int64_t nt = static_cast<int64_t>(tiles_m) * tiles_n * g.plan.S;
    const dim3 grid(static_cast<unsigned>(8 * ((nt + 7) / 8)));
#define MASQ_TILE(BM, BN, WM, WN, NST, WPE)                                                         \
    hipLaunchKernelGGL((k_gemm_tile<YT, LT, CMC, ACC, W4, BM, BN, WM, WN, NST, WPE>), grid,         \
                       dim3(64 * WM * WN), 0, g.stream, g.q, g.wq, g.x_scale, g.w_scale, g.T,       \
                       static_cast<int>(g.K), static_cast<int>(g.N), tiles_m, tiles_n, g.mod, g.u,  \
                       g.u_hl, g.rank, g.n_mod, static_cast<const LT*>(g.r_up), g.acc,              \
                       static_cast<YT*>(g.y), g.plan.S, g.part, g.tickets, g.a_pair)
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

}  // namespace

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
