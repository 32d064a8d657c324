// Device helpers shared by the kernel translation units.
#pragma once

#include <type_traits>

#include "masq_common.h"

namespace masq {
namespace {

typedef int32_t v2i __attribute__((ext_vector_type(2)));
typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef int32_t v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

typedef uint16_t bf16_t;   // bfloat16 stored as its bit pattern

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// Two fp32 values narrowed to bf16 bits (a in the low half), round to nearest
// even: one v_cvt_pk_bf16_f32 on gfx950.
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf));
}
__device__ __forceinline__ uint32_t f32_to_bf16(float f) { return pack_bf16x2(f, 0.f) & 0xFFFFu; }

// ---------------------------------------------------------------- element IO
template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
        const v4f a = *reinterpret_cast<const v4f*>(p);
        const v4f b = *reinterpret_cast<const v4f*>(p + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
    static __device__ __forceinline__ void store1(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
    static __device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
        const v4i a = *reinterpret_cast<const v4i*>(p);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[2 * j] = __uint_as_float(static_cast<uint32_t>(a[j]) << 16);
            v[2 * j + 1] = __uint_as_float(static_cast<uint32_t>(a[j]) & 0xFFFF0000u);
        }
    }
    static __device__ __forceinline__ void store1(bf16_t* p, float v) {
        *p = static_cast<bf16_t>(f32_to_bf16(v));
    }
};

__device__ __forceinline__ void load8_f32(const float* p, float (&v)[8]) { Elem<float>::load8(p, v); }

// Eight elements as loaded (16 or 32 bytes), converted to fp32 only when
// used, so that a software pipeline can keep the load in flight meanwhile.
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
    v4i a;
    __device__ __forceinline__ void load(const bf16_t* p) { a = *reinterpret_cast<const v4i*>(p); }
    __device__ __forceinline__ void to_f32(float (&v)[8]) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[2 * j] = __uint_as_float(static_cast<uint32_t>(a[j]) << 16);
            v[2 * j + 1] = __uint_as_float(static_cast<uint32_t>(a[j]) & 0xFFFF0000u);
        }
    }
};
template <> struct Raw8<float> {
    v4f a, b;
    __device__ __forceinline__ void load(const float* p) {
        a = *reinterpret_cast<const v4f*>(p);
        b = *reinterpret_cast<const v4f*>(p + 4);
    }
    __device__ __forceinline__ void to_f32(float (&v)[8]) const {
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
};

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// Modality ids outside [0, n_mod) are treated as text, so that a bad id can
// never index past the smoothing or factor arrays.
__device__ __forceinline__ int sane_mod(int m, int n_mod) {
    return (m >= 0 && m < n_mod) ? m : 0;
}

// XOR swizzle of the 16-byte chunk index inside a 128-byte LDS row: any 8
// (or 16) consecutive rows read at one logical chunk land on distinct banks.
__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }

// 4-bit shared weight.  A row of K codes is packed two per byte, in 4-byte
// words of 8 codes: byte b of the word holding codes 8g .. 8g + 7 carries
// code 8g + b in its low nibble and code 8g + b + 4 in its high nibble
// (two's complement).  Two packed words (16 codes) become one 16-byte int8
// MFMA operand in k order, each code multiplied by 16: masking leaves every
// nibble in the high half of its byte, so the int8 byte reads 16 c.  An int32
// sum of such products is 16 times the true one and a multiple of 16, so an
// arithmetic shift right by 4 recovers it exactly.  (|16 c q| <= 112 * 127:
// any K below 2^31 / 14224 stays in range.)
__device__ __forceinline__ v4i w4_operand(v2i p) {
    constexpr int kHi = static_cast<int>(0xF0F0F0F0u);
    return v4i{(p.x << 4) & kHi, p.x & kHi, (p.y << 4) & kHi, p.y & kHi};
}

// ================================================================ LDS DMA
// One 16-byte lane of an LDS-DMA load: the wave writes 64 x 16 contiguous
// bytes at LDS address m0 (wave-uniform), lane i at m0 + 16 i.
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(src), "s"(lds_addr) : "memory", "m0");
}

// Scheduling fence: the compiler may move no instruction across it, so the
// software pipeline below keeps the order it is written in.
#define MASQ_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// s_waitcnt vmcnt(n) lgkmcnt(0) (expcnt unconstrained).
#define MASQ_WAIT_VMCNT_LGKM0(n) \
    __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (0 << 8))

// One 4-byte lane of an LDS-DMA load: lane i writes LDS address m0 + 4 i.
__device__ __forceinline__ void lds_dma4(const void* src, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(src), "s"(lds_addr) : "memory", "m0");
}

__device__ __forceinline__ void split_bf16x8(const float (&v)[8], v4i& hi, v4i& lo) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t h = pack_bf16x2(v[2 * j], v[2 * j + 1]);
        const float h0 = __uint_as_float(h << 16), h1 = __uint_as_float(h & 0xFFFF0000u);
        hi[j] = static_cast<int32_t>(h);
        lo[j] = static_cast<int32_t>(pack_bf16x2(v[2 * j] - h0, v[2 * j + 1] - h1));
    }
}

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous
// range of tiles, ordered in groups of 8 tile-rows, so that tiles running
// together on one XCD share A and B stages in its L2.  Returns false for the
// padding workgroups of the last XCD range.
__device__ __forceinline__ bool tile_coords_at(int b, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int nt = tiles_m * tiles_n;
    const int per_xcd = (nt + 7) >> 3;
    if ((b >> 3) >= per_xcd) return false;
    const int L = (b & 7) * per_xcd + (b >> 3);
    if (L >= nt) return false;
    constexpr int GM = 8;
    const int gsize = GM * tiles_n;
    const int g = L / gsize;
    const int first_m = g * GM;
    const int gm = min(GM, tiles_m - first_m);
    const int li = L - g * gsize;
    tm = first_m + li % gm;
    tn = li / gm;
    return true;
}

}  // namespace
}  // namespace masq
