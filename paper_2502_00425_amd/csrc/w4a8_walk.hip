// W4A8 GEMV for several rows on matrices of many output channels: one work-group of sixteen waves
// per compute unit walks a contiguous run of 16-channel units (halves of the prepacked 32-channel
// tiles).
//
// With a work-group per tile every tile reads all T rows of xq again (at sixteen rows as many bytes
// as its weights) and starts and ends a pipeline of its own.  Here the rows go to LDS once per
// compute unit, and the weights of the whole run are one stream: its 1 KiB wave-loads (16 channels x
// 128 input channels) are dealt to the waves in even contiguous shares, each wave keeps DEPTH of them in
// flight from its first to its last, and no wave waits for another in between.  Where a
// wave's share leaves a unit it adds its partial sums to the unit's in LDS (integers: in any order),
// which are dequantised and stored at the end.  What is left over a kernel that only reads the weights is the
// start (rows, first weights: 1.5 us) and 3584 -> 37888 being 9.25 units per compute unit: 16.9 -> 15.2 us at 16
// rows, 22.2 -> 16.9 at 32 (read only 11.7); 8192 -> 59136 at 16 rows 45.3 -> 42.1 (5.8 TB/s).  Loads past a share are not issued at all (wave-uniform
// tests in the last steps): clamped to one address, they queue up at the cache channel that holds it.
#include <hip/hip_fp16.h>

#include "mquant_internal.h"
#include "w4a8_common.h"

using namespace mquant;

namespace {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int kWalkWaves = 16;
constexpr int kWalkPieces = 9;                  // 16-byte pieces of xq a thread copies at most
constexpr int kWalkMaxXq = kWalkPieces * kWalkWaves * 1024;
constexpr int kWalkMaxLds = 160 * 1024;

// RB: blocks of 16 rows; NX: pieces of xq per thread.  Every wave has at least DEPTH loads.
template <int DEPTH, int RB, int NX, int EPI>
__global__ __launch_bounds__(kWalkWaves * 64) void w4a8_walk_kernel(
    const int8_t *__restrict__ xq, int32_t T, int32_t K, GemvGroup grp, int32_t total_units, Epilogue ep,
    uint32_t row_magic)
{
    constexpr int WAVES = kWalkWaves;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // T rows of xq, pitch K + 16; sums; scales
    const int32_t pitch = K + 16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, c = lane & 15;

    // units of this work-group, loads of this wave
    const int32_t groups = gridDim.x, id = blockIdx.x;
    const int32_t per_group = total_units / groups, rest = total_units - per_group * groups;
    const int32_t u0 = id * per_group + (id < rest ? id : rest);
    const int32_t n_units = per_group + (id < rest ? 1 : 0);
    const int32_t k_tiles = K / kPackK, lpu = K / 128;      // loads per unit
    const int32_t loads = n_units * lpu;
    const int32_t per_wave = loads / WAVES, left = loads - per_wave * WAVES;
    const int32_t f0 = wave * per_wave + (wave < left ? wave : left);
    const int32_t n_mine = per_wave + (wave < left ? 1 : 0);
    int32_t cu = f0 / lpu;                                  // unit (of this group) and load the wave computes
    int32_t cj = f0 - cu * lpu;
    int32_t *sums = reinterpret_cast<int32_t *>(smem + T * pitch);                      // [unit][row][16]
    float *scales = reinterpret_cast<float *>(sums + (per_group + 1) * T * 16);        // [unit][16]

    // which linear of the group a unit belongs to; u becomes its index there
    auto linear_of = [&](int32_t &u) {
        int32_t pi = 0;
        while (pi + 1 < grp.n && u >= grp.p[pi].units) {
            u -= grp.p[pi].units;
            ++pi;
        }
        return pi;
    };
    auto unit_src = [&](int32_t u) -> const uint4 * {
        const int32_t pi = linear_of(u);
        return grp.p[pi].wp + static_cast<int64_t>(u >> 1) * k_tiles * 64 + (u & 1) * 16;
    };
    // half a pair of tiles: lane = channel c + 16 q, input channels 32 q .. 32 q + 31 of the 128
    const int32_t lane_vec = (q >> 1) * 64 + (q & 1) * 32 + c;
    int32_t lu = cu, lj = cj;                               // where the next load is
    const uint4 *lsrc = unit_src(u0 + lu) + static_cast<int64_t>(lj) * 128;
    auto load_next = [&]() -> uint4 {
        if (lj == lpu) {
            lj = 0;
            ++lu;
            lsrc = unit_src(u0 + lu);
        }
        const v4u t = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(lsrc + lane_vec));
        ++lj;
        lsrc += 128;
        return make_uint4(t[0], t[1], t[2], t[3]);
    };

    // Loads return in the order of their issue: first the rows, then the weights, so that the copy into
    // LDS waits for the rows only.
    const int32_t xq_vecs = T * (K / 16);
    v4u xr[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int32_t v = static_cast<int32_t>(threadIdx.x) + i * (WAVES * 64);
        if (v < xq_vecs) xr[i] = *reinterpret_cast<const v4u *>(xq + static_cast<int64_t>(v) * 16);
    }
    __builtin_amdgcn_sched_barrier(0);
    uint4 b[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) b[d] = load_next();
    __builtin_amdgcn_sched_barrier(0);
    for (int32_t i = threadIdx.x; i < n_units * T * 16; i += WAVES * 64) sums[i] = 0;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int32_t v = static_cast<int32_t>(threadIdx.x) + i * (WAVES * 64);
        const int32_t r = static_cast<int32_t>(__umulhi(static_cast<uint32_t>(v), row_magic));   // v / (K / 16)
        if (v < xq_vecs) *reinterpret_cast<v4u *>(smem + (v + r) * 16) = xr[i];
    }
    // the scales are needed last
    __half ws = __half();
    if (static_cast<int32_t>(threadIdx.x) < n_units * 16) {
        int32_t u = u0 + static_cast<int32_t>(threadIdx.x) / 16;
        const int32_t pi = linear_of(u), n = u * 16 + c;
        ws = grp.p[pi].w_scale[n < grp.p[pi].N ? n : grp.p[pi].N - 1];
    }
    __syncthreads();

    const uint8_t *arow[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) arow[r] = smem + (r * 16 + c < T ? r * 16 + c : T - 1) * pitch + q * 32;
    v4i acc0[RB], acc1[RB];                                 // two chains: no dependent back-to-back pair
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc0[r][e] = acc1[r][e] = 0;
    auto hand_over = [&](int32_t u) {                       // row 16 r + 4 q + e, channel c
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int32_t row = r * 16 + q * 4 + e;
                if (row < T) atomicAdd(&sums[(u * T + row) * 16 + c], acc0[r][e] + acc1[r][e]);
                acc0[r][e] = acc1[r][e] = 0;
            }
    };
    uint4 an[RB][2];
    auto read_a = [&](int32_t j) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            an[r][0] = *reinterpret_cast<const uint4 *>(arow[r] + j * 128);
            an[r][1] = *reinterpret_cast<const uint4 *>(arow[r] + j * 128 + 16);
        }
    };
    read_a(cj);
    auto step = [&](int d, bool refill) {
        uint4 a[RB][2];
#pragma unroll
        for (int r = 0; r < RB; ++r) a[r][0] = an[r][0], a[r][1] = an[r][1];
        cj = cj + 1 == lpu ? 0 : cj + 1;
        read_a(cj);
        uint4 bb = b[d];
        hold(bb);
        if (refill) b[d] = load_next();
        v4i b0, b1;
        unpack_w4x16(bb, b0, b1);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            acc0[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(as_v4i(a[r][0]), b0, acc0[r], 0, 0, 0);
            acc1[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(as_v4i(a[r][1]), b1, acc1[r], 0, 0, 0);
        }
        if (cj == 0) {
            hand_over(cu);
            ++cu;
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
    if (cj != 0) hand_over(cu);                             // the share ends inside a unit
    if (static_cast<int32_t>(threadIdx.x) < n_units * 16) scales[threadIdx.x] = __half2float(ws);
    __syncthreads();

    for (int32_t u = wave; u < n_units; u += WAVES) {
        int32_t in = u0 + u;
        const GemvProblem &pr = grp.p[linear_of(in)];
        const int32_t n = in * 16 + c;
        for (int32_t row = q; row < T; row += 4)
            if (n < pr.N)
                store_out<EPI>(sums[(u * T + row) * 16 + c], row, n, ep, scales[u * 16 + c], pr.y, pr.ldy, pr.acc_out,
                               pr.N);
    }
}

// Loads in flight per wave, by the rows: two row blocks leave registers for three.
constexpr int walk_depth(int32_t T) { return T > 16 ? 3 : 6; }

int64_t walk_units(GemvGroup &grp)
{
    int64_t units = 0;
    for (int32_t i = 0; i < grp.n; ++i) {
        grp.p[i].units = static_cast<int32_t>(ceil_div(grp.p[i].N, 16));
        units += grp.p[i].units;
    }
    return units;
}

// Bytes of LDS with the units dealt to `groups` work-groups.
int64_t walk_lds(int32_t T, int32_t K, int64_t units, int32_t groups)
{
    const int64_t most = units / groups + 1;
    return static_cast<int64_t>(T) * (K + 16) + most * T * 64 + most * 64;
}

// Work-groups: one per compute unit, or several rounds of that where the sums of a run do not fit LDS.  0: none that fits.  Up
// to eight units per compute unit a second round, which copies the rows again, meets one round of the sliced GEMM's 32 x 64
// tiles: 4608 -> 32437 at 32 rows 18.6 -> 21.4 us; beyond, 35 shapes took 0.74 to 0.92 of the other's time.
int32_t walk_groups(int32_t T, int32_t K, int64_t units)
{
    for (int32_t rounds = 1; rounds <= (units > 8 * kNumCU ? 4 : 1); ++rounds) {
        const int32_t groups = rounds * kNumCU;
        if (units / groups + 1 <= kWalkWaves * 64 / 16 && walk_lds(T, K, units, groups) <= kWalkMaxLds) return groups;
    }
    return 0;
}

template <int DEPTH, int RB, int NX>
int launch_walk(const int8_t *xq, int32_t T, int32_t K, const GemvGroup &grp, int32_t units, int32_t groups,
                const Epilogue &ep, hipStream_t stream)
{
    auto kern = w4a8_walk_kernel<DEPTH, RB, NX, kEpiStatic>;
    static LdsLimit limit;
    if (const int st = limit.raise(reinterpret_cast<const void *>(kern), kWalkMaxLds); st != MQUANT_OK) return st;
    const uint32_t vecs = static_cast<uint32_t>(K / 16);
    const uint32_t row_magic = static_cast<uint32_t>(((uint64_t{1} << 32) + vecs - 1) / vecs);
    MQ_LAUNCH(kern, dim3(groups), dim3(kWalkWaves * 64), static_cast<size_t>(walk_lds(T, K, units, groups)), stream, xq, T,
              K, grp, units, ep, row_magic);
    return launch_status();
}

}  // namespace

namespace mquant {

// Where it is ahead of a work-group per tile and of the sliced GEMM: 130 matrices (K 1024 .. 14336, N 8192 .. 152064) at
// eleven row counts, weights from HBM, both builds in turn.  Two things decide.
//   uneven: whole tiles fill the compute units' rounds worse than 16-channel units do (time of this kernel / the other, N =
//     17408, 2.1 rounds of tiles: K = 3584 0.95 .. 0.79 from 5 to 32 rows, K = 8192 0.81 at 3 and 4 rows; N = 10240, K =
//     8192 0.88 .. 0.84).  Short K with three units per compute unit is left out: 3072 -> 10240 0.97 .. 1.05.
//   many: the rows are read by so many tiles that the copy into LDS pays (K = 3584, N = 37888: 5 to 8 rows 1.04 and 1.01, not
//     taken; 12 0.92, 16 0.91, 17 0.89, 24 0.82, 32 0.76; N = 152064 at 9, 16 and 32 rows 0.99, 0.86, 0.86).  From K = 4096 on at nine
//     rows 1.04 .. 1.08, so from twelve on; above K = 6144 only if units also divide better (8192 -> 152064 1.02, 59136 0.96).
// Three and four rows: where T * K is beyond what the streaming kernel copies in four pieces per thread (8192 ->
// 37888 44.0 -> 40.6 us); below that it stays ahead (3584 -> 37888 at four rows 13.5 against 14.0).
bool gemv_walk_takes(int32_t T, int32_t K, GemvGroup grp)
{
    if (T < 3 || T > kGemvMaxT || K % 128 != 0 || K < 2048 || static_cast<int64_t>(T) * K > kWalkMaxXq) return false;
    if (tune_state().gemv_variant.load(std::memory_order_relaxed) >= 0) return false;
    const int64_t units = walk_units(grp);
    int64_t tiles = 0;
    for (int32_t i = 0; i < grp.n; ++i) tiles += ceil_div(grp.p[i].N, kPackN);
    const int32_t groups = walk_groups(T, K, units);
    if (groups == 0 || units / groups * (K / 128) < kWalkWaves * walk_depth(T)) return false;
    // share of the compute units' time that whole tiles and units leave filled
    const double by_tile = static_cast<double>(tiles) / static_cast<double>(ceil_div(tiles, kNumCU) * kNumCU);
    const double by_unit = static_cast<double>(units) / static_cast<double>(ceil_div(units, kNumCU) * kNumCU);
    const bool uneven = (K >= 3584 || (K >= 3072 && units >= 4 * kNumCU)) && by_tile < 0.9 * by_unit;
    const bool many = units >= 6 * kNumCU && (K <= 6144 || by_tile < 0.97 * by_unit);
    if (T >= (K < 4096 ? 9 : 12)) return many || uneven;
    if (T >= 5) return uneven;
    return static_cast<int64_t>(T) * K > 16 * 1024 && (units >= 6 * kNumCU || (uneven && K >= 8192));
}

int gemv_walk_dispatch(const int8_t *xq, int32_t T, int32_t K, GemvGroup grp, const Epilogue &ep, hipStream_t stream)
{
    const int32_t units = static_cast<int32_t>(walk_units(grp)), groups = walk_groups(T, K, units);
    if (T > 16) return launch_walk<3, 2, kWalkPieces>(xq, T, K, grp, units, groups, ep, stream);
    if (static_cast<int64_t>(T) * K <= 2 * kWalkWaves * 1024)
        return launch_walk<6, 1, 2>(xq, T, K, grp, units, groups, ep, stream);
    return launch_walk<6, 1, kWalkPieces>(xq, T, K, grp, units, groups, ep, stream);
}

}  // namespace mquant
