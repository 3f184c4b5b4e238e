// Weight-only W4 GEMV for two to sixteen rows: one work-group of sixteen waves per compute unit walks a
// contiguous run of 16-channel units (halves of the prepacked tiles).  From thirteen rows on it is asked only where the
// GEMM is not expected ahead of the GEMV with a work-group per tile (3584 -> 37888: 26.7 -> 20.6 us at twelve rows, at sixteen the
// GEMM keeps its 27).
//
// The rows and the scales of the run go to LDS once; the weights of the run are one stream whose 1 KiB
// wave-loads (16 channels x one scale group) are dealt to the waves in even contiguous shares, DEPTH of
// them in flight per wave from its first to its last.  A share begins and ends inside units: what a wave has of a
// unit goes to a slot of its own in LDS, and at the end the slots of a unit are added in the order of K, so that
// a sum does not depend on which wave is first.  What bounds it is the conversion of the weights (some 80 vector
// operations per wave-load: 3584 -> 37888 takes 17.7 us at one to four rows where reading alone takes 11.5) and, from eight
// rows on, its start: 18.7 us at 8 rows, 24.0 with a work-group per tile; 8192 -> 59136 at 4 rows 68.8 -> 48.6.
#include <hip/hip_fp16.h>

#include "mquant_internal.h"
#include "w4g128_common.h"

using namespace mquant;

namespace {

constexpr int kWaves = 16;
constexpr int kMaxPieces = 8;                   // 16-byte pieces of the rows a thread copies at most
constexpr int kScalePieces = 4;                 // ... of the scales per round
constexpr int kMaxLds = 160 * 1024;

// Wave-loads of wave w: `per` each, one more for the first `left` waves.
__device__ __forceinline__ int32_t share_begin(int32_t w, int32_t per, int32_t left) { return w * per + (w < left ? w : left); }

// Every wave has DEPTH loads at least.
template <int DEPTH, int NX>
__global__ __launch_bounds__(kWaves * 64) void w4g128_walk_kernel(
    const __half *__restrict__ x, int64_t ldx, const v4u *__restrict__ wp, const __half *__restrict__ sT,
    __half *__restrict__ y, int64_t ldy, int32_t T, int32_t N, int32_t K, int32_t n_pad, int32_t units, int32_t slots,
    uint32_t row_magic)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // rows, pitch 2 K + 16; sums; scales
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kg = lane >> 4;
    const int32_t pitch = 2 * K + 16;
    const int32_t lpu = K / kGroup;                          // loads per unit

    const int32_t groups = gridDim.x, id = blockIdx.x;
    const int32_t per_group = units / groups, rest = units - per_group * groups;
    const int32_t u0 = id * per_group + (id < rest ? id : rest);
    const int32_t n_units = per_group + (id < rest ? 1 : 0);
    const int32_t loads = n_units * lpu, per = loads / kWaves, left = loads - per * kWaves;
    const int32_t f0 = share_begin(wave, per, left), n_mine = per + (wave < left ? 1 : 0);
    const int32_t first_unit = f0 / lpu;
    int32_t cu = first_unit, cj = f0 - cu * lpu;

    float *sums = reinterpret_cast<float *>(smem + static_cast<int64_t>(T) * pitch);   // [wave][slot][row][16]
    _Float16 *scales = reinterpret_cast<_Float16 *>(sums + kWaves * slots * T * 16);   // [scale group][unit][16]

    // half a pair of tiles: lane = channel n16 + 16 kg, input channels 32 kg .. 32 kg + 31 of the group
    const int32_t lane_vec = (kg >> 1) * 64 + (kg & 1) * 32 + n16;
    auto unit_src = [&](int32_t u) { return wp + static_cast<int64_t>(u >> 1) * (2 * lpu) * 64 + (u & 1) * 16; };
    int32_t lu = cu, lj = cj;
    const v4u *lsrc = unit_src(u0 + lu) + static_cast<int64_t>(lj) * 128;
    auto load_next = [&]() -> v4u {
        if (lj == lpu) {
            lj = 0;
            ++lu;
            lsrc = unit_src(u0 + lu);
        }
        const v4u t = __builtin_nontemporal_load(lsrc + lane_vec);
        ++lj;
        lsrc += 128;
        return t;
    };

    // Loads return in the order of their issue: rows and scales, then the weights.
    const int32_t row_vecs = K / 8, x_vecs = T * row_vecs;
    const int32_t unit_vecs = 2 * n_units, s_vecs = lpu * unit_vecs;
    const v4u *s_src = reinterpret_cast<const v4u *>(sT + u0 * 16);
    auto scale_at = [&](int32_t p) {                         // 16 bytes of a scale group's row, by units
        const int32_t j = p / unit_vecs;
        return s_src[static_cast<int64_t>(j) * (n_pad / 8) + (p - j * unit_vecs)];
    };
    v4u xr[NX], sr[kScalePieces];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        int32_t v = tid + i * (kWaves * 64);
        v = v < x_vecs ? v : x_vecs - 1;
        const int32_t r = static_cast<int32_t>(__umulhi(static_cast<uint32_t>(v), row_magic));       // v / row_vecs
        xr[i] = *reinterpret_cast<const v4u *>(x + static_cast<int64_t>(r) * ldx + (v - r * row_vecs) * 8);
    }
#pragma unroll
    for (int i = 0; i < kScalePieces; ++i)
        if (tid + i * (kWaves * 64) < s_vecs) sr[i] = scale_at(tid + i * (kWaves * 64));
    __builtin_amdgcn_sched_barrier(0);
    v4u b[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        b[d] = load_next();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        int32_t v = tid + i * (kWaves * 64);
        v = v < x_vecs ? v : x_vecs - 1;
        const int32_t r = static_cast<int32_t>(__umulhi(static_cast<uint32_t>(v), row_magic));
        *reinterpret_cast<v4u *>(smem + (v + r) * 16) = xr[i];                       // row pitch 2 K + 16
    }
#pragma unroll
    for (int i = 0; i < kScalePieces; ++i)
        if (tid + i * (kWaves * 64) < s_vecs) reinterpret_cast<v4u *>(scales)[tid + i * (kWaves * 64)] = sr[i];
    for (int32_t p = tid + kScalePieces * (kWaves * 64); p < s_vecs; p += kWaves * 64)
        reinterpret_cast<v4u *>(scales)[p] = scale_at(p);
    __syncthreads();

    const uint8_t *xlane = smem + (n16 < T ? n16 : T - 1) * pitch + kg * 64;    // rows >= T are never stored
    const Unpack unpack;
    v4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};                  // two chains
    auto hand_over = [&](int32_t u) {                        // result register e of lane group kg: row 4 kg + e
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t row = kg * 4 + e;
            if (row < T) sums[((wave * slots + u - first_unit) * T + row) * 16 + n16] = acc[0][e] + acc[1][e];
            acc[0][e] = acc[1][e] = 0.f;
        }
    };
    auto step = [&](int d, bool refill) {
        const uint8_t *xa = xlane + cj * (kGroup * 2);
        const _Float16 sv = scales[(cj * n_units + cu) * 16 + n16];
        const v2h s2 = {sv, sv};
        v4u bw = b[d];
        asm volatile("" : "+v"(bw));                         // the wait for this load stays here
        if (refill) b[d] = load_next();
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const v8h af = *reinterpret_cast<const v8h *>(xa + st * 16);
            const v8h bf = __builtin_bit_cast(v8h, unpack.eight<false>(bw[st], s2));
            acc[st & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af, bf, acc[st & 1], 0, 0, 0);
        }
        if (++cj == lpu) {
            hand_over(cu);
            ++cu;
            cj = 0;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int32_t i = 0;
    for (; i + 2 * DEPTH <= n_mine; i += DEPTH)
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) step(d, true);
#pragma unroll
    for (int e = 0; e < 2 * DEPTH; ++e)
        if (i + e < n_mine) step(e % DEPTH, e < DEPTH && i + e + DEPTH < n_mine);
    if (cj != 0 && n_mine > 0) hand_over(cu);                // the share ends inside a unit
    __syncthreads();

    // the wave that load f of the run belongs to
    auto wave_of = [&](int32_t f) {
        return f < left * (per + 1) ? f / (per + 1) : left + (f - left * (per + 1)) / per;
    };
    for (int32_t o = tid; o < n_units * T * 16; o += kWaves * 64) {
        const int32_t c = o & 15, ur = o >> 4, u = ur / T, row = ur - u * T;
        const int32_t n = (u0 + u) * 16 + c;
        const int32_t w0 = wave_of(u * lpu), w1 = wave_of((u + 1) * lpu - 1);
        float sum = 0.0f;
        for (int32_t w = w0; w <= w1; ++w)
            sum += sums[((w * slots + u - share_begin(w, per, left) / lpu) * T + row) * 16 + c];
        if (n < N) y[static_cast<int64_t>(row) * ldy + n] = __float2half_rn(sum);
    }
}

struct Plan {
    int32_t groups, slots;
    int64_t lds;
    bool full;
};

constexpr int kDepth = 4;                       // weight loads in flight per wave; with six 10 % slower (3584 -> 37888 at 8 rows 18.7 / 20.6 us)

Plan plan_of(int32_t T, int32_t K, int32_t units)
{
    Plan p;
    p.groups = units < kNumCU ? units : kNumCU;
    const int32_t most = static_cast<int32_t>(ceil_div(units, p.groups)), lpu = K / kGroup;
    const int32_t share = static_cast<int32_t>(ceil_div(static_cast<int64_t>(most) * lpu, kWaves));
    p.slots = (share + lpu - 2) / lpu + 1;                  // units that a share touches at most
    p.lds = static_cast<int64_t>(T) * (2 * K + 16) + static_cast<int64_t>(kWaves) * p.slots * T * 64 +
            static_cast<int64_t>(lpu) * most * 32;
    p.full = static_cast<int64_t>(units / p.groups) * lpu >= kWaves * kDepth;
    return p;
}

template <int NX>
int launch(const __half *x, int64_t ldx, const v4u *wt, const __half *sT, __half *y, int64_t ldy, int32_t T, int32_t N,
           int32_t K, int32_t n_pad, int32_t units, const Plan &p, hipStream_t stream)
{
    auto kern = w4g128_walk_kernel<kDepth, NX>;
    static LdsLimit limit;
    if (const int st = limit.raise(reinterpret_cast<const void *>(kern), kMaxLds); st != MQUANT_OK) return st;
    const uint32_t vecs = static_cast<uint32_t>(K / 8);
    MQ_LAUNCH(kern, dim3(p.groups), dim3(kWaves * 64), static_cast<size_t>(p.lds), stream, x, ldx, wt, sT, y, ldy, T, N, K,
              n_pad, units, p.slots, static_cast<uint32_t>(((uint64_t{1} << 32) + vecs - 1) / vecs));
    return launch_status();
}

}  // namespace

namespace mquant {

// Where it is ahead of a work-group per tile (or per half tile up to four rows): 54 matrices (K 1024 .. 11008, N 10240 ..
// 152064) at seven row counts, weights from HBM, both builds in turn; time of this kernel / the other.  It needs two and a half
// units per compute unit (3584 -> 4608, 1.1 units, 1.1 .. 1.2) and wins by rows, since the others read them from L2 again for
// every tile: 8192 -> 10240 at 4 / 8 rows 0.90 / 0.68, 11008 -> 28672 at 2 / 4 / 5 rows 0.81 / 0.64 / 0.67, 5120 -> 12288 at 12 0.64.
//   K < 3072: only many units (2048 -> 37888 0.98 .. 0.90, 28672 1.18 at two rows and 0.99 at eight; 1024 -> 37888 1.04 .. 1.12)
//   K < 5120: 3584 -> 12288 0.83 and 18944 0.79 at six rows, but 16384, whose 512 tiles the other form takes in even
//     rounds, 1.06; four rows 20480 1.02, 22016 0.86; two rows 22016 1.05, 28672 0.98
//   from there on: four rows 5120 -> 12288 1.09, 16384 0.84; two rows 5120 -> 20480 0.99, 8192 -> 16384 not taken
// One row stays with the half tiles (3584 -> 37888 18.1 / 17.7 us, but 8192 -> 59136 52.9 / 55.6).
bool g128_walk_takes(int32_t T, int32_t K, int32_t N)
{
    if (T < 2 || T > 16 || K < 2048 || N > (1 << 24) || static_cast<int64_t>(T) * K * 2 > kMaxPieces * kWaves * 1024)
        return false;
    const int32_t units = static_cast<int32_t>(ceil_div(N, 16));
    if (2 * units < 5 * kNumCU) return false;
    const Plan p = plan_of(T, K, units);
    if (p.lds > kMaxLds || !p.full) return false;
    if (K < 3072) return units >= 9 * kNumCU;
    if (K < 5120) {
        if (T >= 5) return units < 4 * kNumCU || 2 * units >= 9 * kNumCU || T >= 12;
        return T >= 4 ? 4 * units >= 21 * kNumCU : units >= 7 * kNumCU;
    }
    if (T >= 5) return true;
    return T >= 4 ? K >= 8192 || units >= 4 * kNumCU : units >= 5 * kNumCU;
}

int g128_walk(const __half *x, int64_t ldx, const v4u *wt, const __half *sT, __half *y, int64_t ldy, int32_t T, int32_t N,
              int32_t K, int32_t n_pad, hipStream_t stream)
{
    const int32_t units = static_cast<int32_t>(ceil_div(N, 16));
    const Plan p = plan_of(T, K, units);
    const bool few = static_cast<int64_t>(T) * K * 2 <= 3 * kWaves * 1024;
    return few ? launch<3>(x, ldx, wt, sT, y, ldy, T, N, K, n_pad, units, p, stream)
               : launch<kMaxPieces>(x, ldx, wt, sT, y, ldy, T, N, K, n_pad, units, p, stream);
}

}  // namespace mquant
