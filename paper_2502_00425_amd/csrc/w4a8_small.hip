// The fused prefill linear in one launch, for the smallest calls (a few dozen rows, short K, few output
// channels): rotation, quantizer, W4A8 GEMM and dequantisation in every work-group.
//
// A work-group computes 16 rows x 64 output channels.  Its eight waves first rotate and quantize the 16 rows
// (MQuant Sec. 3.2; the wave-level code of the stand-alone front end) into LDS, all of K, while the weights of
// the tile are on their way to registers; then four waves per half of K multiply a 16-channel half of a
// prepacked tile each (v_mfma_i32_16x16x64_i8), the halves of K meet in LDS.  The rotation is done again by every
// work-group of a row of tiles: that is what limits the form to short K and few channels.
#include <hip/hip_fp16.h>

#include "hadamard_segment.h"
#include "w4a8_common.h"

using namespace mquant;

namespace {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int kRows = 16, kCols = 64, kWaves = 8;
constexpr int kSmallMaxK = 1024;

// NX: segments of 512 channels per wave, 16 * ceil(K / 512) / 8.
template <int NX, int HB>
__global__ __launch_bounds__(kWaves * 64) void w4a8_small_kernel(
    const __half *__restrict__ x, int64_t ldx, const int32_t *__restrict__ perm, int8_t *__restrict__ xq,
    const uint4 *__restrict__ wp, const __half *__restrict__ w_scale, __half *__restrict__ y, int64_t ldy, int32_t T,
    int32_t N, int32_t K, Epilogue ep, float c_vis, float c_txt, int32_t tiles_n)
{
    constexpr int kSteps = NX;                             // weight loads of a wave: half of K / 128 <= 2 NX
    static_assert(NX * kWaves == kRows * (NX / 2), "segments of the rows");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // 16 rows of codes, pitch K + 16; then 4 KiB of sums
    using Seg = Segment<HB>;
    const int32_t pitch = K + 16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
    const int32_t row0 = tm * kRows;
    const int32_t rows = T - row0 < kRows ? T - row0 : kRows;

    // ---- the rows' segments first (loads return in order)
    const int32_t spr = (K + Seg::SEG - 1) / Seg::SEG;
    const int32_t total = rows * spr;
    int32_t src[NX], row_of[NX], seg_of[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        int32_t sg = wave + i * kWaves;
        sg = sg < total ? sg : total - 1;
        row_of[i] = sg / spr;
        seg_of[i] = sg - row_of[i] * spr;
        src[i] = row0 + row_of[i];
        if (perm != nullptr) {
            src[i] = perm[src[i]];
            src[i] = (src[i] < 0 || src[i] >= T) ? 0 : src[i];
        }
    }
    uint4 raw[NX];
    bool in_range[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i)
        raw[i] = Seg::load_chunk(x + static_cast<int64_t>(src[i]) * ldx, seg_of[i], 0, K, lane, in_range[i]);
    __builtin_amdgcn_sched_barrier(0);

    // ---- weights: 16-channel half h of tile nt, two consecutive k-tiles per load (the decode GEMV's pieces).
    // Waves 0..3 take the first half of K, waves 4..7 the second.
    const int wc = wave & 3, kh = wave >> 2, c = lane & 15, q = lane >> 4;
    const int32_t n = tn * kCols + wc * 16 + c;
    const int32_t n_tiles = (N + kPackN - 1) / kPackN;
    int32_t nt = tn * (kCols / kPackN) + wc / 2;
    nt = nt < n_tiles ? nt : n_tiles - 1;                  // past the last tile: never stored
    const int32_t steps = K / 128, j0 = kh * ((steps + 1) / 2), n_mine = kh == 0 ? (steps + 1) / 2 : steps / 2;
    const uint4 *wsrc = wp + static_cast<int64_t>(nt) * (K / kPackK) * 64 + (q >> 1) * 64 + (q & 1) * 32 + (wc & 1) * 16 + c;
    uint4 b[kSteps];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const int32_t j = i < n_mine ? j0 + i : 0;
        const v4u t = *reinterpret_cast<const v4u *>(wsrc + static_cast<int64_t>(j) * 128);
        b[i] = make_uint4(t[0], t[1], t[2], t[3]);
    }
    const __half ws_h = w_scale[n < N ? n : N - 1];
    __builtin_amdgcn_sched_barrier(0);

    // ---- rotate, quantize (Eq. (2)/(3)) into LDS
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        if (wave + i * kWaves < total) {                   // wave-uniform
            Seg s;
            s.set_chunk(0, raw[i], in_range[i]);
            s.rotate(lane);
            const float cm = row0 + row_of[i] < ep.n_vis ? c_vis : c_txt;
            s.quant_store(cm, reinterpret_cast<int8_t *>(smem) + row_of[i] * pitch, seg_of[i], lane);
            // the codes also go where the two launches leave them
            if (tn == 0) s.quant_store(cm, xq + static_cast<int64_t>(row0 + row_of[i]) * K, seg_of[i], lane);
        }
    }
    __syncthreads();

    // ---- multiply; rows past the last are those of the last again
    const uint8_t *arow = smem + (c < rows ? c : rows - 1) * pitch + j0 * 128 + q * 32;
    v4i acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        if (i < n_mine) {                                  // wave-uniform
            const uint4 a0 = *reinterpret_cast<const uint4 *>(arow + i * 128);
            const uint4 a1 = *reinterpret_cast<const uint4 *>(arow + i * 128 + 16);
            v4i b0, b1;
            unpack_w4x16(b[i], b0, b1);
            acc0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(as_v4i(a0), b0, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(as_v4i(a1), b1, acc1, 0, 0, 0);
        }
    }
    // lane group q holds rows 4 q .. 4 q + 3 of column c
    int32_t *sums = reinterpret_cast<int32_t *>(smem + kRows * pitch) + wc * 256 + lane;
    if (kh == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[r * 64] = acc0[r] + acc1[r];
    }
    __syncthreads();
    if (kh == 0 && n < N) {
        const float ws = __half2float(ws_h);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int32_t row = q * 4 + r;
            if (row < rows)
                store_out<kEpiStatic>(acc0[r] + acc1[r] + sums[r * 64], row0 + row, n, ep, ws, y, ldy, nullptr, N);
        }
    }
}

template <int NX, int HB>
int launch_small(const __half *x, int64_t ldx, const int32_t *perm, int8_t *xq, const uint4 *wp, const __half *w_scale,
                 __half *y, int64_t ldy, int32_t T, int32_t N, int32_t K, const Epilogue &ep, float c_vis, float c_txt,
                 hipStream_t stream)
{
    const int32_t tiles_n = static_cast<int32_t>(ceil_div(N, kCols));
    const size_t lds = static_cast<size_t>(kRows) * (K + 16) + 4096;
    MQ_LAUNCH((w4a8_small_kernel<NX, HB>), dim3(static_cast<unsigned>(ceil_div(T, kRows) * tiles_n)), dim3(kWaves * 64), lds,
              stream, x, ldx, perm, xq, wp, w_scale, y, ldy, T, N, K, ep, c_vis, c_txt, tiles_n);
    return launch_status();
}

}  // namespace

namespace mquant {

// As many work-groups as the rotation may be repeated by: one round of them on the compute units, two for K <= 512, whose
// rotation is half as long.  us, front end and GEMM as two launches / one launch (block 512): K = 512: T = 64, N = 512 5.9 /
// 3.8, T = 256, N = 2048 (512 groups) 6.0 / 5.2, T = 512, N = 2048 (1024) 7.1 / 7.9; K = 1024: T = 64, N = 512 6.1 / 5.2, T =
// 256, N = 1024 (256) 6.4 / 5.5, T = 256, N = 2048 (512) 6.6 / 7.5; K = 1536: T = 64, N = 512 6.8 / 7.1.  Called one after the other
// from the host, which takes 8 us for two launches, T = 64, 512 -> 512 9.5 / 7.0.
bool small_linear_takes(int32_t T, int32_t N, int32_t K, int32_t had_block)
{
    if (K % 128 != 0 || K > kSmallMaxK || (had_block != 128 && had_block != 512)) return false;
    return ceil_div(T, kRows) * ceil_div(N, kCols) <= (K <= 512 ? 2 * kNumCU : kNumCU);
}

int small_linear(const __half *x, int64_t ldx, const int32_t *perm, int8_t *xq, const uint4 *wp, const __half *w_scale,
                 __half *y, int64_t ldy, int32_t T, int32_t N, int32_t K, const Epilogue &ep, int32_t had_block,
                 float c_vis, float c_txt, hipStream_t stream)
{
#define MQ_SMALL(NX, HB) launch_small<NX, HB>(x, ldx, perm, xq, wp, w_scale, y, ldy, T, N, K, ep, c_vis, c_txt, stream)
    if (K <= 512) return had_block == 128 ? MQ_SMALL(2, 128) : MQ_SMALL(2, 512);
    return had_block == 128 ? MQ_SMALL(4, 128) : MQ_SMALL(4, 512);
#undef MQ_SMALL
}

}  // namespace mquant
