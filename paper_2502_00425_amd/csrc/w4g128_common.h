// Pieces shared by the weight-only W4 kernels: the operand types and the conversion of prepacked int4
// weights to fp16.
#pragma once

#include <hip/hip_fp16.h>

#include "mquant_internal.h"

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

namespace mquant {

constexpr int kGroup = 128;               // input channels per weight scale

// (a & mask) | c in one VALU operation (the compiler emits an AND and an OR when both
// constants are literals: a VOP3 instruction of this ISA takes no literal operand).
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t c)
{
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(mask), "v"(c));
    return r;
}

// The channels 2 j, 2 j + 1 of a dword of prepacked weights as fp16(code * scale); s2 holds the scale in both
// halves.  Both ways to the code are exact, the product is rounded once.  The odd pairs stay where they
// are, four bits up: 0x6400 | code + 8 << 4 is 1024 + 16 (code + 8), a sixteenth of which is 64 + code + 8.  So
// eight weights take one shift and twelve other operations.  SHIFTED: every pair shifted into place, three shifts
// and twelve operations, for kernels that wait for their loads and not for these: the GEMV of many tiles takes 3 to 8 %
// longer with the other form (3584 -> 37888 at 8 rows 24.0 / 25.9 us), the GEMM's 32x32 tile 1 to 3 % (18944 -> 3584 at 16
// rows 25.3 / 26.0).
struct Unpack {
    uint32_t even = 0x000F000Fu, odd = 0x00F000F0u, magic = 0x64006400u;
    __device__ __forceinline__ Unpack()
    {
        asm volatile("" : "+v"(magic));       // keep it in a VGPR (third operand of v_and_or_b32)
    }
    template <bool SHIFTED>
    __device__ __forceinline__ uint32_t pair(uint32_t v, int j, v2h s2) const
    {
        const v2h bias = {static_cast<_Float16>(1032.0f), static_cast<_Float16>(1032.0f)};
        const v2h sixteenth = {static_cast<_Float16>(0.0625f), static_cast<_Float16>(0.0625f)};
        const v2h bias_odd = {static_cast<_Float16>(-72.0f), static_cast<_Float16>(-72.0f)};
        v2h code;
        if (SHIFTED) {
            code = __builtin_bit_cast(v2h, and_or(v >> (4 * j), even, magic)) - bias;
        } else {
            const uint32_t t = j >= 2 ? v >> 8 : v;
            if (j & 1) code = __builtin_elementwise_fma(__builtin_bit_cast(v2h, and_or(t, odd, magic)), sixteenth, bias_odd);
            else code = __builtin_bit_cast(v2h, and_or(t, even, magic)) - bias;
        }
        return __builtin_bit_cast(uint32_t, code * s2);
    }
    template <bool SHIFTED>
    __device__ __forceinline__ v4u eight(uint32_t v, v2h s2) const
    {
        v4u out;
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = pair<SHIFTED>(v, j, s2);
        return out;
    }
};

// ---- the GEMV of w4g128_walk.hip, one work-group per compute unit, two to sixteen rows that fit LDS
bool g128_walk_takes(int32_t T, int32_t K, int32_t N);
int g128_walk(const __half *x, int64_t ldx, const v4u *wt, const __half *sT, __half *y, int64_t ldy, int32_t T, int32_t N,
              int32_t K, int32_t n_pad, hipStream_t stream);

}  // namespace mquant
