/* The launches of a library call, recorded on the CPU.  Linked against
 * libmasq.so with -rdynamic, this program's own definitions of the HIP calls
 * that launch kernels take the place of the runtime's, so that nothing
 * reaches a device; as the runtime does, a launch of 2^32 threads or more in
 * one dimension is refused.  Pointers are fake and never dereferenced.
 *
 * Each line on stdin is a call; for each, one line on stdout: its status and
 * "gx,gy,gz,bx" of every launch that was accepted.
 *   fused    T K N rank n_mod x_dt lr_dt y_dt w4
 *   gemm     T K N y_dt w4
 *   quant    T K n_mod x_dt
 *   comp     T K N rank n_mod x_dt lr_dt y_dt
 *   dgemm    m n k
 *   qweight  K N
 *   dequant  rows cols
 *   bytes    T K N rank n_mod     (the workspace size instead of a status) */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "masq.h"

typedef struct { uint32_t x, y, z; } dim3;
static struct { dim3 grid, block; size_t shared; void* stream; } pushed;
static char launches[1 << 16];
static int last_error = 0;

int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
    pushed.grid = grid;
    pushed.block = block;
    pushed.shared = shared;
    pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
    *grid = pushed.grid;
    *block = pushed.block;
    *shared = pushed.shared;
    *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shared, void* stream) {
    (void)f; (void)args; (void)shared; (void)stream;
    if ((uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32 || (uint64_t)g.z * b.z >> 32 ||
        !g.x || !g.y || !g.z)
        return last_error = 9;                       /* hipErrorInvalidConfiguration */
    const size_t n = strlen(launches);
    snprintf(launches + n, sizeof launches - n, " %u,%u,%u,%u", g.x, g.y, g.z, b.x);
    return 0;
}
int hipGetLastError(void) {
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipGetDevice(int* dev) {
    *dev = 0;
    return 0;
}
int hipDeviceGetAttribute(int* value, int attribute, int dev) {
    (void)attribute; (void)dev;
    *value = 256;                                    /* compute units */
    return 0;
}

int main(void) {
    char line[256], what[16];
    void* P = (void*)(uintptr_t)(1u << 20);
    const masq_dtype dts[2] = {MASQ_F32, MASQ_BF16};
    while (fgets(line, sizeof line, stdin)) {
        long long a[9] = {0};
        if (sscanf(line, "%15s %lld %lld %lld %lld %lld %lld %lld %lld %lld", what, a, a + 1, a + 2,
                   a + 3, a + 4, a + 5, a + 6, a + 7, a + 8) < 1)
            continue;
        long long st = -1;
        launches[0] = 0;
        if (!strcmp(what, "fused")) {
            const size_t ws = masq_linear_fused_workspace_bytes(a[0], a[1], a[2], (int32_t)a[3],
                                                                (int32_t)a[4]);
            const masq_dtype x_dt = dts[a[5] & 1], lr_dt = dts[a[6] & 1], y_dt = dts[a[7] & 1];
            st = a[8] ? masq_linear_fused_w4a8(P, x_dt, P, P, P, P, P, P, lr_dt, a[0], a[1], a[2],
                                               (int32_t)a[3], (int32_t)a[4], P, y_dt, P, ws, NULL)
                      : masq_linear_fused(P, x_dt, P, P, P, P, P, P, lr_dt, a[0], a[1], a[2],
                                          (int32_t)a[3], (int32_t)a[4], P, y_dt, P, ws, NULL);
        } else if (!strcmp(what, "gemm")) {
            st = a[4] ? masq_w4a8_gemm(P, P, P, P, a[0], a[1], a[2], NULL, P, dts[a[3] & 1], NULL)
                      : masq_w8a8_gemm(P, P, P, P, a[0], a[1], a[2], NULL, P, dts[a[3] & 1], NULL);
        } else if (!strcmp(what, "quant")) {
            st = masq_smooth_quant(P, dts[a[3] & 1], P, P, a[0], a[1], (int32_t)a[2], P, P, NULL);
        } else if (!strcmp(what, "comp")) {
            st = masq_lowrank_comp(P, dts[a[5] & 1], P, P, P, P, dts[a[6] & 1], a[0], a[1], a[2],
                                   (int32_t)a[3], (int32_t)a[4], P, dts[a[7] & 1], NULL);
        } else if (!strcmp(what, "dgemm")) {
            st = masq_dgemm(a[0], a[1], a[2], P, a[2], 1, P, a[1], 1, 0.0, P, a[1], NULL);
        } else if (!strcmp(what, "qweight")) {
            st = masq_quantize_weight(P, P, a[0], a[1], 8, P, P, NULL);
        } else if (!strcmp(what, "dequant")) {
            st = masq_dequantize_rows(P, P, a[0], a[1], P, NULL);
        } else if (!strcmp(what, "bytes")) {
            st = (long long)masq_linear_fused_workspace_bytes(a[0], a[1], a[2], (int32_t)a[3],
                                                              (int32_t)a[4]);
        }
        printf("%lld%s\n", st, launches);
    }
    return 0;
}
