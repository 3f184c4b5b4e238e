// Internal helpers shared by the HIP translation units of libmquant (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <stdint.h>

#include "mquant.h"

namespace mquant {

constexpr int kWave = 64;                 // CDNA wavefront width
constexpr int kNumCU = 256;               // compute units of an MI355X

// A GEMM tile and what a launch of it costs in microseconds, over r rounds of its tiles on the
// compute units (per_cu work-groups of a unit at a time; in a last round that leaves a unit one
// work-group instead of two, that one runs faster):
//   fixed + start * r + begin * tiles / CUs
//         + K / 128 * (full * full rounds + single * single rounds + tile * tiles / CUs)
struct TileCost {
    int32_t bm, bn, per_cu;
    double fixed, start, full, single, tile, begin = 0.0;
    double us(int64_t tiles, int32_t K) const
    {
        static_assert(kNumCU == 256, "shift below");
        const int shift = per_cu == 2 ? 9 : 8;              // per_cu is 1 or 2; no division on the way to a launch
        int64_t n_full = tiles >> shift, n_single = 0;
        const int64_t rest = tiles - (n_full << shift);
        if (rest > 0 && (per_cu == 1 || rest > kNumCU)) ++n_full;
        else if (rest > 0) n_single = 1;
        const double load = static_cast<double>(tiles) * (1.0 / kNumCU);
        return fixed + start * static_cast<double>(n_full + n_single) + begin * load +
               static_cast<double>(K / 128) *
                   (full * static_cast<double>(n_full) + single * static_cast<double>(n_single) + this->tile * load);
    }
};

static inline bool aligned_to(const void *p, uintptr_t a)
{
    return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0;
}

static inline bool ranges_apart(const void *a, uint64_t a_bytes, const void *b, uint64_t b_bytes)
{
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 + a_bytes <= b0 || b0 + b_bytes <= a0;
}

// Bytes from the first to behind the last of T >= 1 rows of w halves, ld apart.
static inline uint64_t rows_bytes(int32_t T, int64_t ld, int64_t w) { return (static_cast<uint64_t>(T - 1) * ld + w) * 2; }

// Whether T rows of w halves, lda apart, share no byte with T rows of wb halves, ldb apart: ranges apart, or column
// slices of one buffer side by side.
static inline bool rows_apart(const void *a, int64_t lda, int64_t w, const void *b, int64_t ldb, int64_t wb, int32_t T)
{
    if (ranges_apart(a, rows_bytes(T, lda, w), b, rows_bytes(T, ldb, wb))) return true;
    if (lda != ldb) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    const uint64_t pitch = static_cast<uint64_t>(lda) * 2;
    const uint64_t d = b0 >= a0 ? (b0 - a0) % pitch : (pitch - (a0 - b0) % pitch) % pitch;    // b's first column behind a's
    return d >= static_cast<uint64_t>(w) * 2 && d + static_cast<uint64_t>(wb) * 2 <= pitch;
}

// Kernel launch that first drops whatever error an earlier, unrelated HIP call of
// this thread left behind (HIP keeps the last error per thread until it is read, so
// a failed query made by the caller's framework would otherwise be reported as ours).
#define MQ_LAUNCH(...)                      \
    do {                                    \
        (void)hipGetLastError();            \
        hipLaunchKernelGGL(__VA_ARGS__);    \
    } while (0)

// Status of the launch just made.  With MQUANT_DEBUG set in the environment the
// HIP error text goes to stderr as well (the C-ABI carries only the status code).
static inline int launch_status()
{
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return MQUANT_OK;
    if (getenv("MQUANT_DEBUG")) fprintf(stderr, "mquant: HIP error %d: %s\n", (int)e, hipGetErrorString(e));
    return MQUANT_ERR_HIP;
}

// Dynamic LDS beyond 64 KiB has to be allowed for a kernel before it is launched with it, and the
// permission belongs to the kernel on the current device: one of these per kernel remembers the devices that have it.
// Raising the limit is idempotent: threads racing here at most repeat it.
class LdsLimit {
    std::atomic<uint64_t> devices_{0};

public:
    int raise(const void *kernel, size_t bytes)
    {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0) return MQUANT_ERR_HIP;
        const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;      // later devices ask every time
        if (devices_.load(std::memory_order_acquire) & bit) return MQUANT_OK;
        if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)) != hipSuccess)
            return MQUANT_ERR_HIP;
        devices_.fetch_or(bit, std::memory_order_release);
        return MQUANT_OK;
    }
};

// Process-wide overrides of kernel choices (mquant_tune_set); -1 / 0 = cost model.
struct TuneState {
    std::atomic<int32_t> gemm_tile{-1};
    std::atomic<int32_t> gemm_nosplit{0};
    std::atomic<int32_t> g128_tile{-1};       // index into the table of w4g128_gemm.hip
    std::atomic<int32_t> gemv_variant{-1};
    std::atomic<int32_t> gemm_sliced{-1};     // index into the table of w4a8_sliced.hip
};
TuneState &tune_state();
constexpr int kGemmShapes = 16;           // tiles of the sliced W4A8 GEMM and 256 x 384
constexpr int kG128Tiles = 14;            // tiles of the weight-only GEMM

// The front end's checks of its input (hadamard_quant.hip).
int check_rotation_args(const void *x, int64_t ldx, int32_t T, int32_t K, int32_t had_block);

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// The same for sizes and tile edges in 32 bits: the cost models ask dozens of times per call.
static inline uint32_t ceil_div32(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

// Geometry of the prepacked int4 weight layout (see w4a8_gemm.hip).
constexpr int kPackN = 32;                // output channels per packed tile (one MFMA N extent)
constexpr int kPackK = 64;                // input channels per packed tile (two 32x32x32 MFMAs)
constexpr int kPackTileBytes = kPackN * kPackK / 2;   // 1024: one 16-byte load per lane
constexpr int kMaxK = 65536;              // 16 * 128 * 8 * K < 2^31 must hold for the x16 unpack

}  // namespace mquant
