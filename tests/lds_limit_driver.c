/* Host-only check of the LDS limits: the HIP calls below stand in for the runtime's (an
 * executable's symbols come before a shared library's), so nothing reaches a GPU.  Every launch with more than
 * 64 KiB of dynamic LDS must have had its limit raised on the device that is current. */
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "mquant.h"

typedef struct { uint32_t x, y, z; } dim3_t;
static struct { const void *kernel; int dev, bytes; } limits[4096];
static int n_limits, dev_now, launches, large, missing;

int hipGetDevice(int *dev) { *dev = dev_now; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *kernel, int attr, int bytes)
{
    (void)attr;
    limits[n_limits].kernel = kernel, limits[n_limits].dev = dev_now, limits[n_limits++].bytes = bytes;
    return n_limits < 4096 ? 0 : 1;
}
static struct { dim3_t grid, block; size_t lds; void *stream; } config;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream)
{
    config.grid = grid, config.block = block, config.lds = lds, config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream)
{
    *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *kernel, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    (void)grid, (void)block, (void)args, (void)stream;
    ++launches;
    if (lds <= 64 * 1024) return 0;
    ++large;
    for (int i = 0; i < n_limits; ++i)
        if (limits[i].kernel == kernel && limits[i].dev == dev_now && (size_t)limits[i].bytes >= lds) return 0;
    ++missing;
    return 0;
}

#define LOAD(name) __typeof__(&name) name##_ = (__typeof__(&name))dlsym(lib, #name); if (!name##_) return 3
#define CALL(e) do { int st_ = (e); if (st_ != MQUANT_OK) { printf("%s: %d\n", #e, st_); return 1; } } while (0)

int main(int argc, char **argv)
{
    void *lib = argc > 1 ? dlopen(argv[1], RTLD_NOW | RTLD_LOCAL) : NULL;
    if (!lib) { printf("%s\n", dlerror()); return 2; }
    LOAD(mquant_tune_set); LOAD(mquant_w4a8_gemm); LOAD(mquant_w4a8_workspace_bytes); LOAD(mquant_w4g128_gemm);
    LOAD(mquant_w4a8_linear_decode); LOAD(mquant_aifs_remap_mask); LOAD(mquant_w4a8_gemv_grouped);
    void *P = (void *)0x10000, *Q = (void *)0x20000;
    for (dev_now = 0; dev_now < 3; ++dev_now)
        for (int rep = 0; rep < 2; ++rep) {
            for (int t = -1; t < 11; ++t) {
                CALL(mquant_tune_set_(MQUANT_TUNE_GEMM_SHAPE, t));
                CALL(mquant_w4a8_gemm_(P, P, P, Q, 4096, NULL, 300, 4096, 8192, 0, 1.f, 1.f, P, (int64_t)1 << 40, NULL));
            }
            CALL(mquant_tune_set_(MQUANT_TUNE_GEMM_SHAPE, -1));
            for (int t = 0; t < 5; ++t) {
                CALL(mquant_tune_set_(MQUANT_TUNE_GEMM_TILE, t));
                CALL(mquant_w4a8_gemm_(P, P, P, Q, 4096, NULL, 300, 4096, 3584, 0, 1.f, 1.f, P, (int64_t)1 << 40, NULL));
            }
            CALL(mquant_tune_set_(MQUANT_TUNE_GEMM_TILE, -1));
            for (int t = 0; t < 14; ++t) {
                CALL(mquant_tune_set_(MQUANT_TUNE_G128_SHAPE, t));
                CALL(mquant_w4g128_gemm_(P, 8192, P, Q, 4096, 300, 4096, 8192, NULL));
            }
            CALL(mquant_tune_set_(MQUANT_TUNE_G128_SHAPE, -1));
            CALL(mquant_w4g128_gemm_(P, 18944, P, Q, 3584, 3, 3584, 18944, NULL));
            mquant_linear_t lin = {P, P, Q, 3584, 3584};
            CALL(mquant_w4a8_gemv_grouped_(P, 4, 18944, 0, 1.f, 1.f, &lin, 1, NULL));
            CALL(mquant_w4a8_linear_decode_(P, 29568, P, P, Q, 8192, 4, 8192, 29568, 0, 1.f, 1.f, 128, NULL));
            CALL(mquant_w4a8_linear_decode_(P, 29568, P, P, Q, 4096, 4, 4096, 29568, 0, 1.f, 1.f, 128, NULL));
            CALL(mquant_aifs_remap_mask_(P, Q, P, 16384, NULL));
        }
    printf("%d launches, %d large, %d without a limit on their device\n", launches, large, missing);
    return launches && large && !missing ? 0 : 1;
}
