// Calibration on the GPU: the exact, non-iterative part of the offline
// calibration that produces the layer's smoothing factors and shared weight.
//
//   R^m_i   = max over the tokens of modality m of |x_ti|         (Sec. 4.1)
//   s^m_i   = sqrt(max(R^m_i, 1e-5) / max(w_i, 1e-5)),            (Sec. 4.2,
//             w_i = max_j |w_ij| over the output channels           alpha = 1/2)
//   Q(S_t W): per output channel o, step d_o = max_i |s^t_i w_io| / qmax and
//             codes rint((s^t_i w_io) / d_o) clamped to [-qmax, qmax]  (eq. PTQ)
//
// and the inputs and products of the compensation factors' calibration:
// the smoothed rows Z_m = X_m S_m^-1 of one modality, the weight difference
// dW_m = S_m W - Q(S_t W), and an fp64 GEMM for the Gram matrix, the
// whitening and the randomized truncated SVD (Sec. 3.2, 4.3).
//
// Every quantity that decides a value is computed in the same precision as
// the definition's host implementation (fp64 for the factor and the weight
// step, one rounding to fp32 at the end), so the results are bit-exact.
// The C ABI of these calls is declared in masq.h.

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "masq.h"
#include "masq_common.h"

namespace {

using bf16_t = unsigned short;

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

// 16 bytes of a row as magnitudes: 4 fp32 or 8 bf16 columns.
template <typename XT> struct Abs16;
template <> struct Abs16<float> {
    static constexpr int kCols = 4;
    static __device__ __forceinline__ void get(v4i raw, float (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(static_cast<uint32_t>(raw[j]) & 0x7FFFFFFFu);
    }
};
template <> struct Abs16<bf16_t> {
    static constexpr int kCols = 8;
    static __device__ __forceinline__ void get(v4i raw, float (&v)[8]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[2 * j] = __uint_as_float((static_cast<uint32_t>(raw[j]) << 16) & 0x7FFFFFFFu);
            v[2 * j + 1] = __uint_as_float(static_cast<uint32_t>(raw[j]) & 0x7FFF0000u);
        }
    }
};

// range [n_mod][K] := 0 (the maxima below are taken with integer atomics on
// the bits of non-negative floats, which order like the values).
__global__ __launch_bounds__(256) void k_zero_f32(float* __restrict__ p, int64_t n) {
    for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < n; i += gridDim.x * 256ll) p[i] = 0.f;
}

// grid (ceil(K / (64 C)), row chunks), C columns in a lane's 16 bytes: the
// four waves of a workgroup take every fourth row of its chunk, kRangeRows
// rows' loads in flight at once (HBM bound), per-modality maxima in
// registers; the waves combine in LDS, then one atomic max per column and
// modality, consecutive lanes on consecutive columns (a lane on its own C
// columns made every atomic instruction touch C times the lines: 16384 x 512
// bf16 took 123 us where this takes 17).  Tokens whose id is outside
// [0, n_mod) belong to no modality.
constexpr int kRangeRows = 8;
template <typename XT>
__global__ __launch_bounds__(256) void k_channel_range(const XT* __restrict__ x,
                                                       const int32_t* __restrict__ mod,
                                                       int64_t T, int K, int n_mod,
                                                       int rows_per_chunk,
                                                       float* __restrict__ range) {
    constexpr int C = Abs16<XT>::kCols;
    __shared__ __attribute__((aligned(16))) float red[4][64 * C];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = blockIdx.x * 64 * C, i = i0 + lane * C;
    const int ic = min(i, K - C);                     // K % 16 == 0: lanes past K repeat the last columns
    const int64_t t0 = static_cast<int64_t>(blockIdx.y) * rows_per_chunk;
    const int64_t t1 = t0 + rows_per_chunk < T ? t0 + rows_per_chunk : T;
    float m[4][C];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < C; ++c) m[k][c] = 0.f;
    for (int64_t t = t0 + wave; t < t1; t += 4 * kRangeRows) {
        v4i raw[kRangeRows];
        int mm[kRangeRows];
#pragma unroll
        for (int r = 0; r < kRangeRows; ++r) {        // rows past the chunk repeat row t
            const int64_t tr = t + 4 * r < t1 ? t + 4 * r : t;
            raw[r] = *reinterpret_cast<const v4i*>(x + tr * K + ic);
            mm[r] = __builtin_amdgcn_readfirstlane(mod[tr]);
        }
#pragma unroll
        for (int r = 0; r < kRangeRows; ++r) {
            float a[C];
            Abs16<XT>::get(raw[r], a);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (mm[r] == k) {
#pragma unroll
                    for (int c = 0; c < C; ++c) m[k][c] = fmaxf(m[k][c], a[c]);
                }
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k >= n_mod) break;
#pragma unroll
        for (int c = 0; c < C; ++c) red[wave][lane * C + c] = m[k][c];
        __syncthreads();
        for (int c = threadIdx.x; c < 64 * C && i0 + c < K; c += 256) {
            const float v = fmaxf(fmaxf(red[0][c], red[1][c]), fmaxf(red[2][c], red[3][c]));
            if (v > 0.f)
                atomicMax(reinterpret_cast<int*>(range + static_cast<int64_t>(k) * K + i0 + c),
                          __float_as_int(v));
        }
        __syncthreads();
    }
}

// One wave per input channel i: w_i = max_j |w_ij| over its row of W
// [K][N] (16 bytes a lane, four loads in flight: HBM bound), then s^m_i =
// fl32(sqrt(max(R, 1e-5) / max(w_i, 1e-5))) in fp64 for every modality and
// inv = fl32(1 / s) (correctly rounded).
__global__ __launch_bounds__(256) void k_smoothing_factors(const float* __restrict__ range,
                                                           const float* __restrict__ w, int K,
                                                           int N, int n_mod,
                                                           float* __restrict__ s,
                                                           float* __restrict__ inv_s) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= K) return;
    const v4f* row = reinterpret_cast<const v4f*>(w + static_cast<int64_t>(i) * N);
    const int nv = N >> 2;                            // N % 16 == 0
    float a = 0.f;
    if (nv <= 64) {                 // narrow rows: one load (100000 x 16 26.9 us in the loop, 21.3 here)
        const v4f v = row[min(lane, nv - 1)];
        a = fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)));
    } else {
        for (int j = lane; j < nv; j += 4 * 64) {
            v4f v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = row[j + 64 * q < nv ? j + 64 * q : j];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                a = fmaxf(fmaxf(a, fmaxf(fabsf(v[q].x), fabsf(v[q].y))),
                          fmaxf(fabsf(v[q].z), fabsf(v[q].w)));
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) a = fmaxf(a, __shfl_xor(a, o));
    if (lane < n_mod) {
        const double r = static_cast<double>(range[static_cast<int64_t>(lane) * K + i]);
        const double v = sqrt(fmax(r, 1e-5) / fmax(static_cast<double>(a), 1e-5));
        const float s32 = static_cast<float>(v);
        s[static_cast<int64_t>(lane) * K + i] = s32;
        inv_s[static_cast<int64_t>(lane) * K + i] = 1.0f / s32;
    }
}

// Q(S_t W) (W [K][N] fp32, paper layout; codes written as wq [N][K]) in three
// launches, so that the reads of W run on the whole chip whatever N is (one
// workgroup per 64 channels left 3584 channels 56 workgroups: 0.55 ms for
// 3584 x 3584, against about 40 us in this form):
//   k_weight_absmax   step maxima of 64 channels over one of S row chunks,
//                     max_i |s_i w_io| in fp64 (the product is exact).  The
//                     chunk's fp64 maximum of channel o is kept in bytes
//                     [8 c, 8 c + 8) of the row wq[o], which no code has
//                     reached yet (S <= K / 64, so 8 S <= K bytes).
//   k_quantize_codes  the codes of the columns past the kept maxima
//                     (kQwHead); every workgroup combines the chunks' maxima
//                     of its channels: d_o = max / qmax.
//   k_quantize_codes (head) the first kQwHead columns, once every other
//                     column is written: a workgroup reads the maxima of its
//                     64 channels, then overwrites them.
// Weights of at most kQwHead rows take one launch, whose workgroups form their
// channels' maxima themselves.
constexpr int kQwChunks = 16;
constexpr int kQwHead = 128;                          // 8 kQwChunks bytes, whole 64-column blocks
static_assert(8 * kQwChunks <= kQwHead && kQwHead % 64 == 0, "maxima lie in the head columns");
constexpr int kQwBlocks = 4;                          // 64-column blocks per workgroup, at least

// The fp64 maximum of channel o0 + tid (tid < 64) over rows i0 .. i1 - 1, by
// the 256 threads of a workgroup.
__device__ __forceinline__ double weight_absmax(const float* __restrict__ w,
                                                const float* __restrict__ s_text, int N, int o0, int i0,
                                                int i1, double (*red)[64]) {
    const int tid = threadIdx.x, cl = tid & 15, rl = tid >> 4;
    const int oc = min(o0 + 4 * cl, N - 4);           // N % 16 == 0: whole groups of 4
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    constexpr int U = 4;
    for (int i = i0 + rl; i < i1; i += 16 * U) {
        v4f v[U];
        float sv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int iu = i + 16 * u < i1 ? i + 16 * u : i;
            v[u] = *reinterpret_cast<const v4f*>(w + static_cast<int64_t>(iu) * N + oc);
            sv[u] = s_text[iu];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                a[e] = fmax(a[e], fabs(static_cast<double>(sv[u]) * static_cast<double>(v[u][e])));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red[rl][4 * cl + e] = a[e];
    __syncthreads();
    double m = red[0][tid & 63];
#pragma unroll
    for (int q = 1; q < 16; ++q) m = fmax(m, red[q][tid & 63]);
    return m;
}

__global__ __launch_bounds__(256) void k_weight_absmax(const float* __restrict__ w,
                                                       const float* __restrict__ s_text, int K,
                                                       int N, int rows_per_chunk,
                                                       int8_t* __restrict__ wq) {
    __shared__ double red[16][64];
    const int o0 = blockIdx.x * 64, i0 = blockIdx.y * rows_per_chunk;
    const double m = weight_absmax(w, s_text, N, o0, i0, min(K, i0 + rows_per_chunk), red);
    const int o = o0 + static_cast<int>(threadIdx.x);
    if (threadIdx.x < 64 && o < N)
        *reinterpret_cast<double*>(wq + static_cast<int64_t>(o) * K + 8 * blockIdx.y) = m;
}

// One code: rint(v / d) clamped to [-qmax, qmax], d > 0, rd = 1 / d.  v rd
// lies within 2^-51 |v / d| of the correctly rounded quotient, so unless it
// is that close to a half-way point (or not finite) it rounds to the same
// integer; the division itself is then never done.
__device__ __forceinline__ int weight_code(double v, double d, double rd, double qmax) {
    const double q = v * rd;
    double r = rint(q);
    if (!(fabs(q - r) < 0.5 - 1e-9)) r = rint(v / d);
    return static_cast<int>(fmin(fmax(r, -qmax), qmax));
}

// Codes of 64 channels (blockIdx.x) and the `per` 64-column blocks from
// b0 + per blockIdx.y on, below b1, transposed through LDS so that
// both the reads (along o) and the writes (along i) are contiguous.  OWN: the
// workgroup forms its channels' maxima itself (K <= kQwHead: one launch).
template <bool OWN>
__global__ __launch_bounds__(256) void k_quantize_codes(const float* __restrict__ w,
                                                        const float* __restrict__ s_text, int K,
                                                        int N, int qmax, int chunks, int b0, int b1,
                                                        int per,
                                                        int8_t* __restrict__ wq,
                                                        float* __restrict__ w_scale) {
    constexpr int kPitch = 80;                        // bytes: 16-byte aligned rows
    __shared__ double sdelta[64];
    __shared__ __attribute__((aligned(16))) int8_t tile[64 * kPitch];
    const int tid = threadIdx.x, cl = tid & 15, rl = tid >> 4;
    const int o0 = blockIdx.x * 64;
    double m = 0.0;
    if constexpr (OWN) {
        __shared__ double red[16][64];
        m = weight_absmax(w, s_text, N, o0, 0, K, red);
    } else if (tid < 64) {
        const int o = min(o0 + tid, N - 1);
        const double* mp = reinterpret_cast<const double*>(wq + static_cast<int64_t>(o) * K);
        m = mp[0];
        for (int c = 1; c < chunks; ++c) m = fmax(m, mp[c]);
    }
    if (tid < 64) {
        const double d = m / qmax;
        sdelta[tid] = d;
        if (w_scale != nullptr && o0 + tid < N) w_scale[o0 + tid] = static_cast<float>(d);
    }
    __syncthreads();
    const int oc = min(o0 + 4 * cl, N - 4);
    double d[4], rd[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        d[e] = sdelta[oc - o0 + e];
        rd[e] = 1.0 / d[e];
    }
    const double qm = static_cast<double>(qmax);
    const int first = b0 + per * static_cast<int>(blockIdx.y);
    for (int blk = first; blk < min(b1, first + per); ++blk) {
        const int i0 = blk * 64;
        // thread (cl, rl): rows i0 + 4 rl + k, channels oc ..
        v4f v[4];
        float sv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = min(i0 + 4 * rl + k, K - 1);
            v[k] = *reinterpret_cast<const v4f*>(w + static_cast<int64_t>(i) * N + oc);
            sv[k] = s_text[i];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t packed = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                int c = 0;
                if (d[e] > 0.0)
                    c = weight_code(static_cast<double>(sv[k]) * static_cast<double>(v[k][e]), d[e],
                                    rd[e], qm);
                packed |= (static_cast<uint32_t>(c) & 0xFFu) << (8 * k);
            }
            *reinterpret_cast<uint32_t*>(tile + (4 * cl + e) * kPitch + 4 * rl) = packed;
        }
        __syncthreads();
        {
            const int orow = tid >> 2, seg = (tid & 3) * 16;      // K % 16 == 0: whole pieces
            if (o0 + orow < N && i0 + seg < K)
                *reinterpret_cast<v4i*>(wq + static_cast<int64_t>(o0 + orow) * K + i0 + seg) =
                    *reinterpret_cast<const v4i*>(tile + orow * kPitch + seg);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ CMC inputs
// The compensation factors (Sec. 3.2, 4.3; eq. l1l2) come from the smoothed
// calibration rows Z_m = X_m S_m^-1 of one modality, their Gram matrix, and
// the weight difference dW_m = S_m W - Q(S_t W); the products below are the
// heavy part of that calibration at full layer sizes.

__device__ __forceinline__ double load_f64(const float* p) { return static_cast<double>(*p); }
__device__ __forceinline__ double load_f64(const bf16_t* p) {
    return static_cast<double>(__uint_as_float(static_cast<uint32_t>(*p) << 16));
}

// z [n][K]: z_ic = x[rows[i]][c] / s_c in fp64 (exact operands, one
// correctly rounded division); a row index outside [0, T) gives a zero row.
// grid (ceil(K / 256), row chunks).
template <typename XT>
__global__ __launch_bounds__(256) void k_gather_smoothed(const XT* __restrict__ x, int64_t T, int K,
                                                         const int32_t* __restrict__ rows,
                                                         int64_t n, const float* __restrict__ s,
                                                         double* __restrict__ z) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= K) return;
    const double sc = static_cast<double>(s[c]);
    for (int64_t i = blockIdx.y; i < n; i += gridDim.y) {
        const int64_t r = rows[i];
        double v = 0.0;
        if (r >= 0 && r < T) v = load_f64(x + r * K + c) / sc;
        z[i * K + c] = v;
    }
}

// dw [K][N] = s_i w_io - wq_oi d_o in fp64: both products are exact (24 x 24
// and 8 x 24 significant bits), so the one subtraction is the only rounding.
// 64 x 64 blocks: the codes wq [N][K] are read along i and transposed
// through LDS, w and dw are read and written along o.
__global__ __launch_bounds__(256) void k_weight_difference(const float* __restrict__ w,
                                                           const float* __restrict__ s,
                                                           const int8_t* __restrict__ wq,
                                                           const float* __restrict__ w_scale,
                                                           int K, int N, double* __restrict__ dw) {
    __shared__ int8_t tile[64][65];                         // [o][i]
    const int tid = threadIdx.x;
    const int o0 = blockIdx.x * 64, i0 = blockIdx.y * 64;
    {
        const int orow = tid >> 2, seg = (tid & 3) * 16, o = o0 + orow;
        for (int e = 0; e < 16; ++e) {
            const int i = i0 + seg + e;
            tile[orow][seg + e] = (o < N && i < K) ? wq[static_cast<int64_t>(o) * K + i] : int8_t(0);
        }
    }
    __syncthreads();
    const int ol = tid & 63, o = o0 + ol;
    if (o >= N) return;
    const double d = static_cast<double>(w_scale[o]);
    for (int il = tid >> 6; il < 64; il += 4) {
        const int i = i0 + il;
        if (i >= K) break;
        const int64_t at = static_cast<int64_t>(i) * N + o;
        const double a = static_cast<double>(s[i]) * static_cast<double>(w[at]);
        const double b = static_cast<double>(tile[ol][il]) * d;
        dw[at] = a - b;
    }
}

// C (i, j) at c[i * crs + j * ccs] = alpha A B (+ beta C), fp64, with A (i,
// k) at a[i * ars + k * acs] and B (k, j) at b[k * brs + j * bcs], so
// transposed operands are strides, not copies.  TI x TJ tiles, WI x WJ waves
// on v_mfma_f64_16x16x4_f64, k in steps of KS staged through two LDS buffers
// with the next two steps' loads in flight.  The instruction adds its four
// products in increasing k, each with one rounding (measured: equal to a
// chain of fma, bit for bit), so every element is the increasing-k chain of
// fused multiply-adds whatever the tile size; the sum is then multiplied by
// alpha (exact for alpha = +-1) and beta C added.  With lower, tiles wholly
// above the diagonal (every j > i) are skipped.
//
// Bound by the fp64 rate (78.6 TFLOP/s, shared by the vector and the matrix
// unit); the vector form of this kernel read one 8-byte LDS operand per four
// fma and stood at 23-28 TFLOP/s.  LDS rows [i][k] lie KS + 1 doubles apart:
// 16 rows of one k are served in one 128-byte cycle only if no two of them
// share an 8-byte slot (KS + 4, two rows a slot: 200 us where this takes
// 156).  64 x 32 tiles of four waves, several workgroups per CU, hide each
// other's barriers: measured 156 us for 256 x 3584 x 3584 (64 x 64 of eight
// waves 158, 128 x 128 452), 135-142 us for 3584 x 3584 x 256 (177, 154),
// 1.14-1.19 ms for 3072 x 3072 x 3584 (1.26, 1.38), 57 TFLOP/s there; no
// shape of these favoured a larger tile.
// v_mfma_f64_16x16x4_f64 layout: lane l holds A(l % 16, l / 16), B(l / 16,
// l % 16) and C(l / 16 + 4 e, l % 16), e = 0..3.
constexpr int kDgRows = 64, kDgCols = 32, kDgStep = 16;
template <int TI, int TJ, int KS, int WI, int WJ>
__global__ __launch_bounds__(64 * WI * WJ, 2) void k_dgemm(int64_t M, int64_t N, int64_t K,
                                               const double* __restrict__ a, int64_t ars,
                                               int64_t acs, const double* __restrict__ b,
                                               int64_t brs, int64_t bcs, double alpha, double beta,
                                               double* __restrict__ c, int64_t crs, int64_t ccs,
                                               int lower) {
    constexpr int NI = TI / WI / 16, NJ = TJ / WJ / 16;      // 16-wide blocks of a wave's edges
    constexpr int NT = 64 * WI * WJ;
    constexpr int NQA = TI * KS / NT, NQB = TJ * KS / NT;    // loads per operand and thread
    constexpr int kPitch = KS + 1;
    __shared__ double as[2][TI * kPitch];
    __shared__ double bs[2][TJ * kPitch];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = (wave / WJ) * (TI / WI), wj = (wave % WJ) * (TJ / WJ);
    const int lr = lane & 15, lk = lane >> 4;
    const int64_t tiles_j = (N + TJ - 1) / TJ;
    const int64_t i0 = masq::linear_block() / tiles_j * TI;
    const int64_t j0 = masq::linear_block() % tiles_j * TJ;
    if (i0 >= M || (lower && j0 > i0 + TI - 1)) return;      // block-uniform
    // staging: element e = tid + NT q of each operand block;
    // the fastest-moving index follows the operand's unit-stride direction.
    // Rows past M (columns past N) repeat the last one: their results are
    // not stored.  k past K is zero.
    const bool a_k_fast = acs == 1, b_k_fast = bcs != 1;
    const double *pa[NQA], *pb[NQB];
    int sa[NQA], sb[NQB], ka[NQA], kb[NQB];                  // LDS places, k within the step
#pragma unroll
    for (int q = 0; q < NQA; ++q) {
        const int e = tid + NT * q, ia = a_k_fast ? e / KS : e % TI;
        ka[q] = a_k_fast ? e % KS : e / TI;
        sa[q] = ia * kPitch + ka[q];
        pa[q] = a + (i0 + ia < M ? i0 + ia : M - 1) * ars;
        if (ka[q] < K) pa[q] += ka[q] * acs;                 // (else never read)
    }
#pragma unroll
    for (int q = 0; q < NQB; ++q) {
        const int e = tid + NT * q, jb = b_k_fast ? e / KS : e % TJ;
        kb[q] = b_k_fast ? e % KS : e / TJ;
        sb[q] = jb * kPitch + kb[q];
        pb[q] = b + (j0 + jb < N ? j0 + jb : N - 1) * bcs;
        if (kb[q] < K) pb[q] += kb[q] * brs;
    }
    // step j's operands through register set j % 2: two steps ahead of use
    double ra[2][NQA], rb[2][NQB];
    auto load_whole = [&](auto set, int64_t k0) __attribute__((always_inline)) {
        constexpr int P = decltype(set)::value;
#pragma unroll
        for (int q = 0; q < NQA; ++q) ra[P][q] = pa[q][k0 * acs];
#pragma unroll
        for (int q = 0; q < NQB; ++q) rb[P][q] = pb[q][k0 * brs];
    };
    auto load = [&](auto set, int64_t k0) __attribute__((always_inline)) {   // any k0 >= 0
        constexpr int P = decltype(set)::value;
#pragma unroll
        for (int q = 0; q < NQA; ++q) ra[P][q] = k0 + ka[q] < K ? pa[q][k0 * acs] : 0.0;
#pragma unroll
        for (int q = 0; q < NQB; ++q) rb[P][q] = k0 + kb[q] < K ? pb[q][k0 * brs] : 0.0;
    };
    auto stash = [&](auto set) __attribute__((always_inline)) {
        constexpr int P = decltype(set)::value;
#pragma unroll
        for (int q = 0; q < NQA; ++q) as[P][sa[q]] = ra[P][q];
#pragma unroll
        for (int q = 0; q < NQB; ++q) bs[P][sb[q]] = rb[P][q];
    };
    v4d acc[NI][NJ];
#pragma unroll
    for (int u = 0; u < NI; ++u)
#pragma unroll
        for (int v = 0; v < NJ; ++v) acc[u][v] = v4d{0.0, 0.0, 0.0, 0.0};
    using set0 = std::integral_constant<int, 0>;
    using set1 = std::integral_constant<int, 1>;
    auto multiply = [&](auto set) __attribute__((always_inline)) {
        constexpr int P = decltype(set)::value;
#pragma unroll
        for (int s = 0; s < KS / 4; ++s) {
            double av[NI], bv[NJ];
#pragma unroll
            for (int u = 0; u < NI; ++u) av[u] = as[P][(wi + 16 * u + lr) * kPitch + 4 * s + lk];
#pragma unroll
            for (int v = 0; v < NJ; ++v) bv[v] = bs[P][(wj + 16 * v + lr) * kPitch + 4 * s + lk];
#pragma unroll
            for (int u = 0; u < NI; ++u)
#pragma unroll
                for (int v = 0; v < NJ; ++v)
                    acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[v], acc[u][v], 0, 0, 0);
        }
    };
    load(set0{}, 0);
    load(set1{}, KS);
    stash(set0{});
    __syncthreads();
    // LDS buffer P holds step k0 (k0 / KS even: P = 0); each half stashes the
    // next step into the other buffer, last read before the previous barrier.
    // Whole steps only, so that the waits count exactly one step's loads.
    int64_t k0 = 0;
    for (; k0 + 4 * KS <= K; k0 += 2 * KS) {
        load_whole(set0{}, k0 + 2 * KS);
        multiply(set0{});
        stash(set1{});
        __syncthreads();
        load_whole(set1{}, k0 + 3 * KS);
        multiply(set1{});
        stash(set0{});
        __syncthreads();
    }
    for (; k0 < K; k0 += 2 * KS) {
        load(set0{}, k0 + 2 * KS);
        multiply(set0{});
        stash(set1{});
        __syncthreads();
        if (k0 + KS >= K) break;
        load(set1{}, k0 + 3 * KS);
        multiply(set1{});
        stash(set0{});
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < NI; ++u)
#pragma unroll
        for (int v = 0; v < NJ; ++v) {
            const int64_t j = j0 + wj + 16 * v + lr;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t i = i0 + wi + 16 * u + lk + 4 * e;
                if (i < M && j < N) {
                    double r = alpha * acc[u][v][e];
                    if (beta != 0.0) r = r + beta * c[i * crs + j * ccs];
                    c[i * crs + j * ccs] = r;
                }
            }
        }
}

// ------------------------------------------------------- MAS optimisation
// The per-modality objective mean |Q(X S^-1) Q(S W) - X W| (Sec. 4.2, eq.
// mas_quant) and its straight-through gradient: the quantizers are the
// inference ones above; these kernels dequantize their codes, take the
// residual's sign and assemble dL/ds from the two products of the backward
// pass (formed with k_dgemm).

// out [R][C] fp64 = codes [R][C] * scale[r] (exact: 8 x 24 significant bits).
// P codes of a row a thread and round (2 where C is even: one 16-byte store a
// lane, a wave's side by side), over the whole matrix in order whatever its
// shape.  Bound by the writes.  (4 codes a thread in two stores, workgroups on
// rows of their own: 3584 x 3584 21.9 us, here 18.0; 100000 x 4 13.8, here
// 3.1; 18944 x 3584 171, here 125 and 138 on a grid of 8192 workgroups.)
template <int P>
__global__ __launch_bounds__(256) void k_dequantize_rows(const int8_t* __restrict__ codes,
                                                         const float* __restrict__ scale,
                                                         int64_t R, int64_t C,
                                                         double* __restrict__ out) {
    const int64_t n = R * C;
    for (int64_t e = P * (blockIdx.x * 256ll + threadIdx.x); e < n; e += P * 256ll * gridDim.x) {
        const double sc = static_cast<double>(scale[e / C]);
        if constexpr (P == 2) {
            const uint16_t w = *reinterpret_cast<const uint16_t*>(codes + e);
            *reinterpret_cast<v2d*>(out + e) = v2d{static_cast<double>(static_cast<int8_t>(w)) * sc,
                                                   static_cast<double>(static_cast<int8_t>(w >> 8)) * sc};
        } else {
            out[e] = static_cast<double>(codes[e]) * sc;
        }
    }
}

// g_e = sign(y_e - ref_e) * inv_count; partial[b] = the sum of |y_e - ref_e|
// over block b's kMaeChunk elements (a fixed tree order, so the loss the
// caller adds up is reproducible).
constexpr int kMaeChunk = 4096;
__global__ __launch_bounds__(256) void k_mae_sign(const double* __restrict__ y,
                                                  const double* __restrict__ ref, int64_t n,
                                                  double inv_count, double* __restrict__ g,
                                                  double* __restrict__ partial) {
    __shared__ double red[4];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kMaeChunk;
    double acc = 0.0;
    for (int j = threadIdx.x; j < kMaeChunk; j += 256) {
        const int64_t e = base + j;
        if (e >= n) break;
        const double r = y[e] - ref[e];
        g[e] = r > 0.0 ? inv_count : (r < 0.0 ? -inv_count : 0.0);
        acc += fabs(r);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// loss[0] = (partial[0] + partial[1] + ... + partial[nparts - 1]) / count,
// in that order: one wave loads 64 sums at a time, then its first lane adds
// them (a load per addition would cost a memory round trip each).
__global__ __launch_bounds__(64) void k_mae_loss(const double* __restrict__ partial, int64_t nparts,
                                                 double count, double* __restrict__ loss) {
    __shared__ double buf[64];
    const int lane = threadIdx.x;
    double s = 0.0;
    for (int64_t b0 = 0; b0 < nparts; b0 += 64) {
        buf[lane] = b0 + lane < nparts ? partial[b0 + lane] : 0.0;
        __syncthreads();
        if (lane == 0) {
            const int n = static_cast<int>(nparts - b0 < 64 ? nparts - b0 : 64);
            for (int q = 0; q < n; ++q) s += buf[q];
        }
        __syncthreads();
    }
    if (lane == 0) *loss = s / count;
}

// Adam on theta = ln s (Kingma and Ba 2015), one element a thread, each
// operation rounded as written (the build disables contraction):
//   g  = lam * s * grad                (d/dtheta of the objective)
//   m1 = b1 m1 + (1 - b1) g,  m2 = b2 m2 + ((1 - b2) g) g
//   theta -= (lr (m1 / c1)) / (sqrt(m2 / c2) + eps),  c_i = 1 - b_i^step
//   s := fl32(exp(theta)),  inv_s := fl32(1 / s)
__global__ __launch_bounds__(256) void k_adam_log(double* __restrict__ theta, double* __restrict__ m1,
                                                  double* __restrict__ m2,
                                                  const double* __restrict__ grad,
                                                  float* __restrict__ s, float* __restrict__ inv_s,
                                                  int64_t K, double lam, double lr, double b1,
                                                  double omb1, double b2, double omb2, double c1,
                                                  double c2, double eps) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= K) return;
    const double g = (lam * static_cast<double>(s[i])) * grad[i];
    const double a = b1 * m1[i] + omb1 * g;
    const double v = b2 * m2[i] + (omb2 * g) * g;
    const double th = theta[i] - (lr * (a / c1)) / (sqrt(v / c2) + eps);
    m1[i] = a;
    m2[i] = v;
    theta[i] = th;
    const float sn = static_cast<float>(exp(th));
    s[i] = sn;
    inv_s[i] = 1.0f / sn;
}

// theta = ln s, m1 = m2 = 0, then s := fl32(exp(theta)), inv_s := fl32(1 / s)
// (the factors the first step's forward pass uses).
__global__ __launch_bounds__(256) void k_adam_log_init(double* __restrict__ theta,
                                                       double* __restrict__ m1,
                                                       double* __restrict__ m2,
                                                       float* __restrict__ s,
                                                       float* __restrict__ inv_s, int64_t K) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= K) return;
    const double th = log(static_cast<double>(s[i]));
    theta[i] = th;
    m1[i] = 0.0;
    m2[i] = 0.0;
    const float sn = static_cast<float>(exp(th));
    s[i] = sn;
    inv_s[i] = 1.0f / sn;
}

// colpart[i] = sum_t x[t][i] a[t][i] (thread per column, t in order; 16
// rows' loads in flight, one wave a workgroup so that few columns still
// spread over the chip).
__global__ __launch_bounds__(64) void k_column_dot(const double* __restrict__ x,
                                                   const double* __restrict__ a, int64_t T,
                                                   int64_t K, double* __restrict__ out) {
    constexpr int U = 16;
    const int64_t i = blockIdx.x * 64ll + threadIdx.x;
    if (i >= K) return;
    double acc = 0.0;
    int64_t t = 0;
    for (; t + U <= T; t += U) {
        double xv[U], av[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            xv[q] = x[(t + q) * K + i];
            av[q] = a[(t + q) * K + i];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) acc = fma(xv[q], av[q], acc);
    }
    for (; t < T; ++t) acc = fma(x[t * K + i], a[t * K + i], acc);
    out[i] = acc;
}

// grad[i] = -colpart[i] / (s_i s_i) + sum_o w[i][o] b[i][o] (a wave per row
// i, lane l summing o = l, l + 64, .. in order; 8 of them in flight).
__global__ __launch_bounds__(256) void k_mas_grad(const double* __restrict__ colpart,
                                                  const double* __restrict__ w,
                                                  const double* __restrict__ b,
                                                  const float* __restrict__ s, int64_t K,
                                                  int64_t N, double* __restrict__ grad) {
    constexpr int U = 8;
    const int lane = threadIdx.x & 63;
    const int64_t i = blockIdx.x * 4ll + (threadIdx.x >> 6);
    if (i >= K) return;
    const double* wr = w + i * N;
    const double* br = b + i * N;
    double acc = 0.0;
    int64_t o = lane;
    for (; o + 64 * (U - 1) < N; o += 64 * U) {
        double wv[U], bv[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            wv[q] = wr[o + 64 * q];
            bv[q] = br[o + 64 * q];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) acc = fma(wv[q], bv[q], acc);
    }
    for (; o < N; o += 64) acc = fma(wr[o], br[o], acc);
#pragma unroll
    for (int o2 = 32; o2 >= 1; o2 >>= 1) acc += __shfl_xor(acc, o2);
    if (lane == 0) {
        const double si = static_cast<double>(s[i]);
        grad[i] = -colpart[i] / (si * si) + acc;
    }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned8(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7u) == 0; }

}  // namespace

namespace masq {

hipError_t launch_dgemm(int64_t m, int64_t n, int64_t k, const double* a, int64_t ars,
                        int64_t acs, const double* b, int64_t brs, int64_t bcs, double alpha,
                        double beta, double* c, int64_t crs, int64_t ccs, bool lower,
                        hipStream_t s) {
    if (m <= 0 || n <= 0) return hipSuccess;
    const int64_t tiles = ((n + kDgCols - 1) / kDgCols) * ((m + kDgRows - 1) / kDgRows);
    if ((n + 127) / 128 > 0xFFFFFF) return hipErrorInvalidConfiguration;   // (never accepted: C of 17 GB a row)
    hipLaunchKernelGGL((k_dgemm<kDgRows, kDgCols, kDgStep, 2, 2>), grid_of(tiles, 256),
                       dim3(256), 0, s, m, n, k, a, ars, acs, b, brs, bcs, alpha, beta, c, crs, ccs,
                       lower ? 1 : 0);
    return hipGetLastError();
}

}  // namespace masq

extern "C" {

masq_status masq_channel_range(const void* x, masq_dtype x_dt, const int32_t* modality,
                               int64_t T, int64_t c_in, int32_t n_mod, float* range,
                               void* stream) {
    if (x_dt != MASQ_F32 && x_dt != MASQ_BF16) return MASQ_ERR_DTYPE;
    if (T < 0 || c_in <= 0 || c_in % 16 != 0 || c_in > (1LL << 30) || n_mod < 1 || n_mod > 4)
        return MASQ_ERR_SHAPE;
    if (!range || (T > 0 && (!x || !modality))) return MASQ_ERR_NULL;
    if (!aligned16(range) || (T > 0 && (!aligned16(x) || !aligned16(modality))))
        return MASQ_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    (void)hipGetLastError();
    const int64_t n = static_cast<int64_t>(n_mod) * c_in;
    hipLaunchKernelGGL(k_zero_f32, dim3(static_cast<unsigned>((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024)),
                       dim3(256), 0, s, range, n);
    if (T > 0) {
        const int K = static_cast<int>(c_in);
        const int cols = 64 * (x_dt == MASQ_BF16 ? Abs16<bf16_t>::kCols : Abs16<float>::kCols);
        const int64_t col_blocks = (K + cols - 1) / cols;
        // about 1024 workgroups, and at least a round of loads for each wave
        int64_t chunks = (1024 + col_blocks - 1) / col_blocks;
        const int64_t most = (T + 4 * kRangeRows - 1) / (4 * kRangeRows);
        if (chunks > most) chunks = most;
        const int rows = static_cast<int>((T + chunks - 1) / chunks);
        chunks = (T + rows - 1) / rows;
        const dim3 grid(static_cast<unsigned>(col_blocks), static_cast<unsigned>(chunks));
        if (x_dt == MASQ_BF16)
            hipLaunchKernelGGL(k_channel_range<bf16_t>, grid, dim3(256), 0, s,
                               static_cast<const bf16_t*>(x), modality, T, K, n_mod, rows, range);
        else
            hipLaunchKernelGGL(k_channel_range<float>, grid, dim3(256), 0, s,
                               static_cast<const float*>(x), modality, T, K, n_mod, rows, range);
    }
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_smoothing_factors(const float* range, const float* w, int64_t c_in,
                                   int64_t c_out, int32_t n_mod, float* smooth,
                                   float* inv_smooth, void* stream) {
    if (c_in <= 0 || c_in % 16 != 0 || c_out <= 0 || c_out % 16 != 0 || c_in > (1LL << 30) ||
        c_out > (1LL << 30) || n_mod < 1 || n_mod > 4)
        return MASQ_ERR_SHAPE;
    if (!range || !w || !smooth || !inv_smooth) return MASQ_ERR_NULL;
    if (!aligned16(range) || !aligned16(w) || !aligned16(smooth) || !aligned16(inv_smooth))
        return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_smoothing_factors, dim3(static_cast<unsigned>((c_in + 3) / 4)), dim3(256),
                       0, static_cast<hipStream_t>(stream), range, w, static_cast<int>(c_in),
                       static_cast<int>(c_out), n_mod, smooth, inv_smooth);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_quantize_weight(const float* w, const float* smooth_text, int64_t c_in,
                                 int64_t c_out, int32_t bits, int8_t* wq, float* w_scale,
                                 void* stream) {
    if (c_in <= 0 || c_in % 16 != 0 || c_out <= 0 || c_out % 16 != 0 || c_in > (1LL << 30) ||
        c_out > (1LL << 30) || (bits != 8 && bits != 4))
        return MASQ_ERR_SHAPE;
    if (!w || !smooth_text || !wq || !w_scale) return MASQ_ERR_NULL;
    if (!aligned16(w) || !aligned16(smooth_text) || !aligned16(wq) || !aligned16(w_scale))
        return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int K = static_cast<int>(c_in), N = static_cast<int>(c_out), qmax = (1 << (bits - 1)) - 1;
    const unsigned groups = static_cast<unsigned>((N + 63) / 64);
    const int blocks = (K + 63) / 64;
    if (K <= kQwHead) {     // few rows: one launch (16 x 512 5.7 -> 3.5 us, 128 x 3584 6.7 -> 5.1 us)
        hipLaunchKernelGGL(k_quantize_codes<true>, dim3(groups, 1), dim3(256), 0, s, w, smooth_text, K, N,
                           qmax, 0, 0, blocks, blocks, wq, w_scale);
        return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
    }
    int chunks = std::min(K / 64, kQwChunks);
    const int rows = (K + chunks - 1) / chunks;
    chunks = (K + rows - 1) / rows;
    hipLaunchKernelGGL(k_weight_absmax, dim3(groups, static_cast<unsigned>(chunks)), dim3(256), 0, s,
                       w, smooth_text, K, N, rows, wq);
    constexpr int head = kQwHead / 64;
    const int rest = blocks - head;
    const int per = rest > kQwBlocks * 65535 ? (rest + 65534) / 65535 : kQwBlocks;
    hipLaunchKernelGGL(k_quantize_codes<false>, dim3(groups, static_cast<unsigned>((rest + per - 1) / per)),
                       dim3(256), 0, s, w, smooth_text, K, N, qmax, chunks, head, blocks, per, wq,
                       static_cast<float*>(nullptr));
    hipLaunchKernelGGL(k_quantize_codes<false>, dim3(groups, 1), dim3(256), 0, s, w, smooth_text, K, N, qmax,
                       chunks, 0, head, head, wq, w_scale);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_gather_smoothed(const void* x, masq_dtype x_dt, int64_t T, int64_t c_in,
                                 const int32_t* rows, int64_t n_rows, const float* smooth,
                                 double* z, void* stream) {
    if (x_dt != MASQ_F32 && x_dt != MASQ_BF16) return MASQ_ERR_DTYPE;
    if (T < 0 || n_rows < 0 || c_in <= 0 || c_in % 16 != 0 || c_in > (1LL << 30))
        return MASQ_ERR_SHAPE;
    if (n_rows == 0) return MASQ_OK;
    if (!rows || !smooth || !z || (T > 0 && !x)) return MASQ_ERR_NULL;
    if (!aligned16(rows) || !aligned16(smooth) || !aligned16(z) || (T > 0 && !aligned16(x)))
        return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    const int K = static_cast<int>(c_in);
    const int64_t col_blocks = (K + 255) / 256;
    int64_t chunks = (2048 + col_blocks - 1) / col_blocks;
    if (chunks > n_rows) chunks = n_rows;
    if (chunks > 65535) chunks = 65535;
    const dim3 grid(static_cast<unsigned>(col_blocks), static_cast<unsigned>(chunks));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (x_dt == MASQ_BF16)
        hipLaunchKernelGGL(k_gather_smoothed<bf16_t>, grid, dim3(256), 0, s,
                           static_cast<const bf16_t*>(x), T, K, rows, n_rows, smooth, z);
    else
        hipLaunchKernelGGL(k_gather_smoothed<float>, grid, dim3(256), 0, s,
                           static_cast<const float*>(x), T, K, rows, n_rows, smooth, z);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_weight_difference(const float* w, const float* smooth, const int8_t* wq,
                                   const float* w_scale, int64_t c_in, int64_t c_out,
                                   double* dw, void* stream) {
    if (c_in <= 0 || c_in % 16 != 0 || c_out <= 0 || c_out % 16 != 0 || c_in > (1LL << 30) ||
        c_out > (1LL << 30) || (c_in + 63) / 64 > 65535)
        return MASQ_ERR_SHAPE;
    if (!w || !smooth || !wq || !w_scale || !dw) return MASQ_ERR_NULL;
    if (!aligned16(w) || !aligned16(smooth) || !aligned16(wq) || !aligned16(w_scale) ||
        !aligned16(dw))
        return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    const dim3 grid(static_cast<unsigned>((c_out + 63) / 64), static_cast<unsigned>((c_in + 63) / 64));
    hipLaunchKernelGGL(k_weight_difference, grid, dim3(256), 0, static_cast<hipStream_t>(stream),
                       w, smooth, wq, w_scale, static_cast<int>(c_in), static_cast<int>(c_out), dw);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_dgemm(int64_t m, int64_t n, int64_t k, const double* a, int64_t a_row_stride,
                       int64_t a_col_stride, const double* b, int64_t b_row_stride,
                       int64_t b_col_stride, double beta, double* c, int64_t ldc, void* stream) {
    if (m < 0 || n < 0 || k < 0 || a_row_stride < 0 || a_col_stride < 0 || b_row_stride < 0 ||
        b_col_stride < 0 || (m + 127) / 128 > 65535 ||
        (n + 127) / 128 > 0x7fffffffLL || (m > 0 && n > 0 && ldc < n))
        return MASQ_ERR_SHAPE;
    if (m == 0 || n == 0) return MASQ_OK;
    if (!c || (k > 0 && (!a || !b))) return MASQ_ERR_NULL;
    if (!aligned8(c) || (k > 0 && (!aligned8(a) || !aligned8(b)))) return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    return masq::launch_dgemm(m, n, k, a, a_row_stride, a_col_stride, b, b_row_stride,
                              b_col_stride, 1.0, beta, c, ldc, 1, false,
                              static_cast<hipStream_t>(stream)) == hipSuccess
               ? MASQ_OK
               : MASQ_ERR_HIP;
}

masq_status masq_dequantize_rows(const int8_t* codes, const float* scale, int64_t rows,
                                 int64_t cols, double* out, void* stream) {
    if (rows < 0 || cols < 0 || (cols > 0 && rows > (1LL << 40) / cols)) return MASQ_ERR_SHAPE;
    if (rows == 0 || cols == 0) return MASQ_OK;
    if (!codes || !scale || !out) return MASQ_ERR_NULL;
    if (!aligned16(codes) || !aligned16(scale) || !aligned16(out)) return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int per = cols % 2 == 0 ? 2 : 1;
    const int64_t blocks = std::min<int64_t>((rows * cols + 256 * per - 1) / (256 * per), 1 << 20);
    hipLaunchKernelGGL(per == 2 ? k_dequantize_rows<2> : k_dequantize_rows<1>,
                       dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, codes, scale, rows, cols, out);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

int64_t masq_mae_partials(int64_t count) {
    return count <= 0 ? 0 : (count + kMaeChunk - 1) / kMaeChunk;
}

masq_status masq_mae_sign(const double* y, const double* ref, int64_t count, double* g,
                          double* partial, void* stream) {
    if (count < 0 || masq_mae_partials(count) > 0x7fffffffLL) return MASQ_ERR_SHAPE;
    if (count == 0) return MASQ_OK;
    if (!y || !ref || !g || !partial) return MASQ_ERR_NULL;
    if (!aligned8(y) || !aligned8(ref) || !aligned8(g) || !aligned8(partial)) return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_mae_sign, dim3(static_cast<unsigned>(masq_mae_partials(count))), dim3(256),
                       0, static_cast<hipStream_t>(stream), y, ref, count,
                       1.0 / static_cast<double>(count), g, partial);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_mae_loss(const double* partial, int64_t count, double* loss, void* stream) {
    if (count < 0 || masq_mae_partials(count) > 0x7fffffffLL) return MASQ_ERR_SHAPE;
    if (!loss || (count > 0 && !partial)) return MASQ_ERR_NULL;
    if (!aligned8(loss) || (count > 0 && !aligned8(partial))) return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_mae_loss, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), partial,
                       masq_mae_partials(count), count > 0 ? static_cast<double>(count) : 1.0, loss);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_adam_log_step(double* theta, double* m1, double* m2, const double* grad,
                               float* smooth, float* inv_smooth, int64_t c_in, double lam,
                               double lr, double b1, double b2, double eps, int64_t step,
                               void* stream) {
    if (c_in < 0 || c_in > (1LL << 30) || step < 0 || !(lr >= 0.0) || !(b1 >= 0.0 && b1 < 1.0) ||
        !(b2 >= 0.0 && b2 < 1.0) || !(eps > 0.0) || !isfinite(lam) || !isfinite(lr))
        return MASQ_ERR_SHAPE;
    if (c_in == 0) return MASQ_OK;
    if (!theta || !m1 || !m2 || !smooth || !inv_smooth || (step > 0 && !grad))
        return MASQ_ERR_NULL;
    if (!aligned8(theta) || !aligned8(m1) || !aligned8(m2) || (step > 0 && !aligned8(grad)) ||
        (reinterpret_cast<uintptr_t>(smooth) & 3u) != 0 ||
        (reinterpret_cast<uintptr_t>(inv_smooth) & 3u) != 0)
        return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid(static_cast<unsigned>((c_in + 255) / 256));
    if (step == 0) {
        hipLaunchKernelGGL(k_adam_log_init, grid, dim3(256), 0, st, theta, m1, m2, smooth,
                           inv_smooth, c_in);
    } else {
        const double sd = static_cast<double>(step);
        hipLaunchKernelGGL(k_adam_log, grid, dim3(256), 0, st, theta, m1, m2, grad, smooth,
                           inv_smooth, c_in, lam, lr, b1, 1.0 - b1, b2, 1.0 - b2,
                           1.0 - pow(b1, sd), 1.0 - pow(b2, sd), eps);
    }
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

masq_status masq_mas_gradient(const double* x, const double* a, const double* w, const double* b,
                              const float* smooth, int64_t T, int64_t c_in, int64_t c_out,
                              double* colpart, double* grad, void* stream) {
    if (T < 0 || c_in <= 0 || c_out <= 0 || c_in > (1LL << 30) || c_out > (1LL << 30))
        return MASQ_ERR_SHAPE;
    if (!w || !b || !smooth || !colpart || !grad || (T > 0 && (!x || !a))) return MASQ_ERR_NULL;
    if (!aligned8(w) || !aligned8(b) || !aligned8(smooth) || !aligned8(colpart) ||
        !aligned8(grad) || (T > 0 && (!aligned8(x) || !aligned8(a))))
        return MASQ_ERR_ALIGN;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_column_dot, dim3(static_cast<unsigned>((c_in + 63) / 64)), dim3(64), 0, st, x,
                       a, T, c_in, colpart);
    hipLaunchKernelGGL(k_mas_grad, dim3(static_cast<unsigned>((c_in + 3) / 4)), dim3(256), 0, st,
                       colpart, w, b, smooth, c_in, c_out, grad);
    return hipGetLastError() == hipSuccess ? MASQ_OK : MASQ_ERR_HIP;
}

}  // extern "C"
