// Weight-only W4 linear with group-wise scales (the weight-only setting of
// Table 13: int4 weight, one fp16 scale per 128 input channels of an output
// channel, 16-bit activations; group-wise granularity as in the appendix on
// quantization granularity).
//
//   W~[n, k] = fp16(wq[n, k] * s[n, k / 128])          (one rounding)
//   y[i, n]  = fp16(sum_k x[i, k] * W~[n, k])           (fp32 accumulation)
//
// Matrix core: v_mfma_f32_32x32x16_f16.  A = fp16 activations (M = tokens), staged
// through LDS; B = weights, dequantised in registers on their way into the MFMA.
// Lane l supplies row/column l % 32 and the 8 consecutive k of slot group l / 32.
// The contraction order inside a 64-channel k-tile is free as long as A and B
// agree: MFMA step s of a tile contracts channels {s*8..s*8+7} (lanes 0..31) and
// {32+s*8..32+s*8+7} (lanes 32..63), so that the 16 bytes a lane fetches from the
// prepacked weight are its B operands of all four steps.
//
// Prepacked weights: [n_tile][k_tile][lane][16 bytes] as for the W4A8 kernels
// (tile = 32 output x 64 input channels, lane (n % 32) + 32 * g holds channels
// 64*k_tile + 32*g .. +31 of row n), but inside a dword of 8 channels nibble j
// holds channel 2j and nibble j + 4 channel 2j + 1 (j = 0..3), each stored as
// code + 8.  (v >> 4j) & 0x000F000F then is a pair of adjacent channels in the
// two halves of a dword; OR-ing 0x6400 into each half makes the fp16 number
// 1024 + code + 8, from which 1032 is subtracted exactly before the multiply by
// the scale -- two packed fp16 operations per pair and no integer->float convert (Unpack).
// The scale table follows the weight tiles, transposed to [K/128][N padded to 32]
// so that the 32 lanes of a tile read consecutive halves.
#include <hip/hip_fp16.h>

#include <atomic>
#include <type_traits>

#include "lds_dma.h"
#include "mquant_internal.h"
#include "w4g128_common.h"

using namespace mquant;

namespace {

constexpr int64_t kG128MaxLdx = int64_t(1) << 23;   // 255 rows of 2 * ldx bytes within 32 bits

__global__ __launch_bounds__(256) void g128_prepack_kernel(
    const uint8_t *__restrict__ w, const __half *__restrict__ scales, uint32_t *__restrict__ out_w,
    __half *__restrict__ out_s, int32_t N, int32_t K, int32_t n_tiles, int32_t k_tiles)
{
    const int64_t total = static_cast<int64_t>(n_tiles) * k_tiles * 64 * 4;     // dwords
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t o = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; o < total; o += stride) {
        const int d = static_cast<int>(o & 3);
        const int lane = static_cast<int>((o >> 2) & 63);
        const int64_t tile = o >> 8;
        const int32_t kt = static_cast<int32_t>(tile % k_tiles);
        const int32_t nt = static_cast<int32_t>(tile / k_tiles);
        const int32_t n = nt * kPackN + (lane & 31);
        const int32_t k0 = kt * kPackK + (lane >> 5) * 32 + d * 8;
        uint32_t v = 0x88888888u;                                   // code 0 everywhere
        if (n < N) {
            const uint32_t src =
                *reinterpret_cast<const uint32_t *>(w + static_cast<int64_t>(n) * (K / 2) + k0 / 2) ^
                0x88888888u;                                        // nibble c of src = channel k0 + c
            v = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v |= ((src >> (4 * (2 * j))) & 0xFu) << (4 * j);
                v |= ((src >> (4 * (2 * j + 1))) & 0xFu) << (4 * (j + 4));
            }
        }
        out_w[o] = v;
    }
    const int32_t n_pad = n_tiles * kPackN;
    const int64_t total_s = static_cast<int64_t>(K / kGroup) * n_pad;
    for (int64_t o = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; o < total_s; o += stride) {
        const int32_t n = static_cast<int32_t>(o % n_pad);
        const int32_t kg = static_cast<int32_t>(o / n_pad);
        out_s[o] = n < N ? scales[static_cast<int64_t>(n) * (K / kGroup) + kg] : __float2half(1.0f);
    }
}

__device__ __forceinline__ int acc_row(int r, int g) { return (r >> 2) * 8 + g * 4 + (r & 3); }

// Work-group id -> (tm, tn): the eight XCDs (work-groups are dealt to them round
// robin) each get a contiguous run of a tile order that walks bands of `band`
// tile-rows, so the tiles an XCD holds at a time share few row and column panels.
__device__ __forceinline__ void tile_of_group(int32_t id, int32_t tiles_m, int32_t tiles_n,
                                              int32_t band, int32_t &tm, int32_t &tn)
{
    const int32_t total = tiles_m * tiles_n;
    const int32_t per = total / 8, rem = total % 8;
    const int32_t xcd = id % 8, local = id / 8;
    const int32_t t = xcd * per + (xcd < rem ? xcd : rem) + local;
    const int32_t band_tiles = band * tiles_n;
    const int32_t b = t / band_tiles;
    const int32_t in_band = t - b * band_tiles;
    const int32_t rows = (tiles_m - b * band) < band ? (tiles_m - b * band) : band;
    tm = b * band + in_band % rows;
    tn = in_band / rows;
}

// Prefill shapes: one work-group of eight waves computes an MT*32 x NWN*32 tile.  The waves
// stand as NWN column waves x KS = 8 / NWN K slices: a wave owns all MT*32 rows of one
// 32-channel column and one 64-channel k-tile of every stage, so each weight is dequantised
// once per work-group (13 VALU operations per MT MFMAs), and the KS slices of a column are
// added through LDS at the end.
//
// A stage is KS k-tiles.  Everything in it arrives by LDS-DMA: the activations (KS slabs of
// MT*32 rows x 128 bytes, 16-byte chunk c of row r at c ^ ((r >> 1) & 7): 16 consecutive rows
// cover the 64 banks once on both sides), every wave's own weight tile (1 KiB) and its 32
// scales.  NB stage buffers: after the barrier that ends the reads of stage s, its buffer is
// refilled with stage s + NB.  The barrier sits kWin MFMAs before the end of a stage, whose
// last operands are in registers by then, and the first fragments and weights of the next
// stage are requested behind it, so neither the LDS latency nor the dequantisation of a
// stage's first step is exposed.
//
// What bounds it: with few work-groups the length of K each walks (hence the slices: 18944 x
// 3584 at T = 128 makes 224 groups of 64 x 32 instead of 28 of 96 x 256, 184 -> 47 us; 3584 x 4608 at
// T = 128 37.9 -> 14.5 us), with all compute units busy the clock under matrix-core power
// (256 x 256 at 1280 x 3584 x 37888: matrix pipes 61 % of the cycles at 1.80 GHz, 361 -> 305 us
// against a 128 x 256 tile that dequantised every weight twice as often: 66 % at 1.58 GHz, 313 us).

template <int MT, int NWN>
struct G128Tile {
    static constexpr int KS = 8 / NWN;
    static constexpr int WIN = MT > 1 ? 4 : 2;        // A fragments requested ahead of the MFMA that uses them
    static constexpr int A_SLAB = MT * 32 * 128, A_STAGE = KS * A_SLAB;
    static constexpr int B_OFF = A_STAGE, S_OFF = B_OFF + 8 * 1024, STAGE = S_OFF + 8 * 256;
    static constexpr int CHA = MT * KS / 2;           // 1 KiB activation blocks a wave copies per stage
    static constexpr int PER = CHA + 2;               // ... and the weight tile and the scales
    static constexpr int RED = NWN * MT * 4 * (KS - 1) * 1024;   // slice sums in transit
    static constexpr int EPI = RED + 8 * 32 * 80;                // ... and the store patches
    static_assert((MT * KS) % 2 == 0, "blocks must divide evenly over the waves");
};

template <int MT, int NWN, int NB>
constexpr int g128_lds_bytes()
{
    using G = G128Tile<MT, NWN>;
    return NB * G::STAGE > G::EPI ? NB * G::STAGE : G::EPI;
}

template <int MT, int NWN, int NB>
__global__ __launch_bounds__(512, (g128_lds_bytes<MT, NWN, NB>() <= 80 * 1024 ? 4 : 2)) void w4g128_gemm_kernel(
    const __half *__restrict__ x, int64_t ldx, const uint8_t *__restrict__ wp,
    const __half *__restrict__ sT, __half *__restrict__ y, int64_t ldy, int32_t T, int32_t N,
    int32_t K, int32_t tiles_m, int32_t tiles_n, int32_t n_tiles32, int32_t wide_store,
    int32_t band)
{
    using G = G128Tile<MT, NWN>;
    constexpr int KS = G::KS, kWin = G::WIN;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];   // g128_lds_bytes<...>()

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int wn = wave % NWN, ks = wave / NWN;
    int32_t tm, tn;
    tile_of_group(blockIdx.x, tiles_m, tiles_n, band, tm, tn);
    const int32_t row0 = tm * MT * 32;
    const int32_t k_tiles = K / kPackK;
    const int32_t stages = (k_tiles + KS - 1) / KS;
    const int32_t n_pad = n_tiles32 * kPackN;
    const int32_t n0 = (tn * NWN + wn) * kPackN;      // first column of this wave
    // column tiles past the last one repeat it (never stored)
    const int32_t ntile = tn * NWN + wn < n_tiles32 ? tn * NWN + wn : n_tiles32 - 1;

    // ---- copies.  Uniform bases and 32-bit lane offsets; rows past T repeat row T - 1 and
    // k-tiles past the last one repeat it (neither result is used).
    const uint8_t *xbase = reinterpret_cast<const uint8_t *>(x + static_cast<int64_t>(row0) * ldx);
    const uint8_t *wbase = wp + static_cast<int64_t>(ntile) * k_tiles * kPackTileBytes;
    const uint8_t *sbase = reinterpret_cast<const uint8_t *>(sT + ntile * kPackN);
    const uint32_t lds0 = lds_address(smem);
    uint32_t aoff[G::CHA];
#pragma unroll
    for (int i = 0; i < G::CHA; ++i) {
        const int r = ((wave + 8 * i) % (MT * 4)) * 8 + (lane >> 3);
        const int32_t row = row0 + r < T ? r : T - 1 - row0;
        aoff[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(ldx * 2) +
                  (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    auto copy_piece = [&](int i, int32_t s, uint32_t buf) {   // buf: byte offset of the stage buffer
        const int b = wave + 8 * i;
        int32_t kt = s * KS + (i < G::CHA ? b / (MT * 4) : ks);
        kt = kt < k_tiles ? kt : k_tiles - 1;
        if (i < G::CHA)
            lds_dma16_uniform_base(xbase + static_cast<int64_t>(kt) * (kPackK * 2), aoff[i < G::CHA ? i : 0],
                                   lds0 + buf + b * 1024);
        else if (i == G::CHA)
            lds_dma16_uniform_base(wbase + static_cast<int64_t>(kt) * kPackTileBytes, lane * 16,
                                   lds0 + buf + G::B_OFF + wave * 1024);
        else
            lds_dma4_uniform_base(sbase + static_cast<int64_t>(kt >> 1) * n_pad * 2, (lane & 15) * 4,
                                  lds0 + buf + G::S_OFF + wave * 256);
    };

    v16f acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0.0f;

    const Unpack unpack;
    constexpr bool kShifted = MT == 1 && NWN == 1;

    // fragment (st, mt): chunk g * 4 + st of row mt * 32 + l32 of this wave's slab
    const uint32_t a_lane = ks * G::A_SLAB + l32 * 128 + (((g * 4) ^ ((l32 >> 1) & 7)) << 4);
    auto afrag = [&](uint32_t buf, int st, int mt) {
        return *reinterpret_cast<const v8h *>(smem + buf + (a_lane ^ (st << 4)) + mt * 4096);
    };
    auto btile = [&](uint32_t buf) {
        return *reinterpret_cast<const v4u *>(smem + buf + G::B_OFF + wave * 1024 + lane * 16);
    };
    auto scale = [&](uint32_t buf) {
        const _Float16 v = *reinterpret_cast<const _Float16 *>(smem + buf + G::S_OFF + wave * 256 + l32 * 2);
        return v2h{v, v};
    };

    // ---- prologue: fill every buffer, wait for stage 0, first operands
#pragma unroll
    for (int s = 0; s < NB; ++s)
        if (s < stages)
#pragma unroll
            for (int i = 0; i < G::PER; ++i) copy_piece(i, s, s * G::STAGE);
    if (NB == 3 && stages >= 3) wait_vmcnt<2 * G::PER>();
    else if (stages >= 2) wait_vmcnt<G::PER>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    uint32_t cur = 0;
    v4u bw = btile(0);
    v2h s2 = scale(0);
    v8h fr[kWin];
#pragma unroll
    for (int i = 0; i < kWin; ++i) fr[i] = afrag(0, i / MT, i % MT);
    v4u bf[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) bf[0][j] = unpack.pair<kShifted>(bw[0], j, s2);

    // A wave whose slice ends a stage early (K / 64 not a multiple of KS) leaves the loop one
    // stage early; there is no barrier in the last stage.
    const int32_t my_stages = (stages - 1) * KS + ks < k_tiles ? stages : stages - 1;
    for (int32_t s = 0; s < my_stages; ++s) {
        const uint32_t nxt = cur + G::STAGE == NB * G::STAGE ? 0 : cur + G::STAGE;
        v4u bw_n = bw;
        v2h s2_n = s2;
        constexpr int NM = 4 * MT;
        constexpr int kBar = NM - kWin, kLand = kBar - (MT < 4 ? MT : 4);
        static_assert(kLand >= 0, "");
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int st = m / MT, mt = m % MT;
            if (m == kLand) {
                // this wave's copies of the next stage have landed: its own weights and scales
                if (NB == 3 && s + 2 < stages) wait_vmcnt<G::PER>();
                else wait_vmcnt<0>();
                asm volatile("" ::: "memory");
                bw_n = btile(nxt);
                s2_n = scale(nxt);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (m == kBar && s + 1 < stages) {
                // every operand of this stage is in registers, every wave's copies have landed
                wait_lgkm0();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[m % kWin], __builtin_bit_cast(v8h, bf[st & 1]),
                                                            acc[mt], 0, 0, 0);
            const int f = m + kWin;                    // the fragment requested behind this MFMA
            if (f < NM) fr[m % kWin] = afrag(cur, f / MT, f % MT);
            else fr[m % kWin] = afrag(nxt, (f - NM) / MT, (f - NM) % MT);
            if (m >= kBar && s + NB < stages) {        // refill the buffer just freed, a few pieces per MFMA
#pragma unroll
                for (int i = (m - kBar) * G::PER / kWin; i < (m - kBar + 1) * G::PER / kWin; ++i)
                    copy_piece(i, s + NB, cur);
            }
            // the next step's weights, dealt over the MFMAs of this one
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((MT >= 4 ? MT - 4 + j : j * MT / 4) == mt)
                    bf[(st + 1) & 1][j] = unpack.pair<kShifted>(st < 3 ? bw[(st + 1) & 3] : bw_n[0], j, st < 3 ? s2 : s2_n);
            __builtin_amdgcn_sched_barrier(0);
        }
        bw = bw_n;
        s2 = s2_n;
        cur = nxt;
    }
    __syncthreads();                                    // every wave is done with the stage buffers

    // ---- add the K slices of a column.  The rows of a 32x32 block held by registers 4 q .. 4 q + 3
    // (eight rows of the block) are unit mt * 4 + q; unit u belongs to slice u % KS, every other
    // slice hands its part over through LDS.
    if constexpr (KS > 1) {
        float *red = reinterpret_cast<float *>(smem) + wn * (MT * 4 * (KS - 1) * 256);
        auto slot = [&](int u, int from) {             // from: (source slice - owner) mod KS, 1 .. KS - 1
            return red + ((u * (KS - 1) + from - 1) * 4) * 64 + lane;
        };
#pragma unroll
        for (int u = 0; u < MT * 4; ++u) {
            const int from = (ks - u % KS + KS) % KS;
            if (from != 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) slot(u, from)[e * 64] = acc[u / 4][(u % 4) * 4 + e];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MT * 4; ++u)
            if (u % KS == ks)
#pragma unroll
                for (int from = 1; from < KS; ++from)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[u / 4][(u % 4) * 4 + e] += slot(u, from)[e * 64];
    }

    if (!wide_store) {
        // every lane stores its own 2-byte results
        const int32_t n = n0 + l32;
        if (n >= N) return;
#pragma unroll
        for (int u = 0; u < MT * 4; ++u)
            if (u % KS == ks)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int32_t row = row0 + (u / 4) * 32 + (u % 4) * 8 + g * 4 + e;
                    if (row < T) y[static_cast<int64_t>(row) * ldy + n] = __float2half_rn(acc[u / 4][(u % 4) * 4 + e]);
                }
        return;
    }

    // Wide stores: the MFMA result has a lane per column; each wave turns its units through its
    // own LDS patch and stores 16 bytes per lane.
    uint8_t *patch = smem + G::RED + wave * (32 * 80);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if ((mt * 4 + r / 4) % KS == ks)
                *reinterpret_cast<__half *>(patch + acc_row(r, g) * 80 + l32 * 2) = __float2half_rn(acc[mt][r]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int rl = q * 16 + lane / 4, c = lane % 4;
            const v4u v = *reinterpret_cast<const v4u *>(patch + rl * 80 + c * 16);
            const int32_t row = row0 + mt * 32 + rl, n = n0 + c * 8;
            if ((mt * 4 + rl / 8) % KS == ks && row < T && n < N)      // N % 8 == 0 on this path
                *reinterpret_cast<v4u *>(y + static_cast<int64_t>(row) * ldy + n) = v;
        }
    }
}

// Decode shape (T <= 32): the weights are streamed once and nothing is reused.  One
// work-group owns one 32-channel tile, its NWAVES waves split K, and every wave requests
// a batch of KT k-tiles (activation fragments first, they hit L2; then the weights, with
// the non-temporal hint, and their scales) before it touches the first one.  Loads are
// branch free: k-tiles past a wave's range are clamped and their weights replaced by
// code 0, lanes whose token row is >= T read row T - 1 (rows >= T of the MFMA result
// are never stored).  The fp32 partial sums of the waves meet in LDS and are added in
// wave order.
template <int NWAVES, int KT>
__global__ __launch_bounds__(NWAVES * 64) void w4g128_gemv_kernel(
    const __half *__restrict__ x, int64_t ldx, const v4u *__restrict__ wp,
    const __half *__restrict__ sT, __half *__restrict__ y, int64_t ldy, int32_t T, int32_t N,
    int32_t K, int32_t n_pad)
{
    __shared__ float red[NWAVES][16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    const int32_t ntile = blockIdx.x;
    const int32_t k_tiles = K / kPackK;
    const int32_t per_wave = (k_tiles + NWAVES - 1) / NWAVES;
    const int32_t kt_begin = wave * per_wave;
    int32_t kt_end = kt_begin + per_wave;
    kt_end = kt_end < k_tiles ? kt_end : k_tiles;
    const int32_t n = ntile * kPackN + l32;

    v16f acc0, acc1;                                      // two chains: no back-to-back dependent MFMAs
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        acc0[r] = 0.0f;
        acc1[r] = 0.0f;
    }
    const v4u *wtile = wp + static_cast<int64_t>(ntile) * k_tiles * 64 + lane;
    const __half *xrow = x + static_cast<int64_t>(l32 < T ? l32 : T - 1) * ldx + g * 32;
    const __half *scol = sT + ntile * kPackN + l32;
    const Unpack unpack;

    auto walk = [&](auto shifted) {
        for (int32_t base = kt_begin; base < kt_end; base += KT) {
            v4u a[KT][4], b[KT];
            uint16_t sc[KT];
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                int32_t kt = base + u;
                kt = kt < kt_end ? kt : kt_end - 1;
#pragma unroll
                for (int st = 0; st < 4; ++st)
                    a[u][st] = *reinterpret_cast<const v4u *>(xrow + kt * kPackK + st * 8);
            }
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                int32_t kt = base + u;
                kt = kt < kt_end ? kt : kt_end - 1;
                b[u] = __builtin_nontemporal_load(wtile + static_cast<int64_t>(kt) * 64);
                sc[u] = __builtin_bit_cast(uint16_t, scol[static_cast<int64_t>(kt / 2) * n_pad]);
            }
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                const bool live = base + u < kt_end;                     // wave-uniform
                const _Float16 sv = __builtin_bit_cast(_Float16, sc[u]);
                const v2h s2 = {sv, sv};
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const uint32_t code = live ? b[u][st] : 0x88888888u;
                    const v8h bf = __builtin_bit_cast(v8h, unpack.eight<decltype(shifted)::value>(code, s2));
                    const v8h af = __builtin_bit_cast(v8h, a[u][st]);
                    if (st & 1) acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, bf, acc1, 0, 0, 0);
                    else acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, bf, acc0, 0, 0, 0);
                }
            }
            // all memory reads of the batch first, then the arithmetic
            __builtin_amdgcn_sched_group_barrier(0x020, 6 * KT, 0);
            __builtin_amdgcn_sched_group_barrier(0x00A, 20 * 4 * KT, 0);
        }
    };
    // The form of the conversion (Unpack).  Sixteen waves over 3584 -> 3584, 18944 -> 3584 and 29568 -> 8192, one shift / three:
    // 8 rows 6.5 / 7.2 us, 24.0 / 24.7, 40.6 / 40.8; 12 rows 7.1 / 7.6, 27.6 / 27.1, 44.6 / 42.9: from eleven rows on a long K waits for
    // the activations as well.  The sides meet between K = 8192 (12 rows 13.0 / 13.4) and 11008 (18.0 / 17.7).
    if (KT == 1 || (T > 10 && K > 10240)) walk(std::true_type{});
    else walk(std::false_type{});

    const int rmax = T <= 8 ? 4 : (T <= 16 ? 8 : 16);     // accumulator registers that can hold a row < T
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (r < rmax) red[wave][r][lane] = acc0[r] + acc1[r];
    __syncthreads();
    for (int r = wave; r < rmax; r += NWAVES) {
        const int32_t row = acc_row(r, g);
        if (row < T && n < N) {
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) sum += red[w][r][lane];
            y[static_cast<int64_t>(row) * ldy + n] = __float2half_rn(sum);
        }
    }
}

// The same for a few rows whose activations fit LDS: half a tile (16 output channels) per
// work-group, so that few output tiles still reach every compute unit (18944 -> 3584: 224 groups
// instead of 112), and v_mfma_f32_16x16x32_f16.  Lane n % 16 + 16 * kg holds the 32 channels
// 64 * (kg / 2) + 32 * (kg % 2) .. + 31 of its scale group (two k-tiles) of output row n; MFMA
// step s contracts channels s * 8 .. + 7 of the four lane groups.  The activations are copied to
// LDS once (read per k-tile from L2 they are four of six vector-memory instructions); every wave
// keeps DEPTH weight loads in flight, the first of them issued before that copy.
template <int NWAVES, int DEPTH>
__global__ __launch_bounds__(NWAVES * 64) void w4g128_gemv_half_kernel(
    const __half *__restrict__ x, int64_t ldx, const v4u *__restrict__ wp,
    const __half *__restrict__ sT, __half *__restrict__ y, int64_t ldy, int32_t T, int32_t N,
    int32_t K, int32_t n_pad)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // max(T * pitch, NWAVES * 1024)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kg = lane >> 4;
    const int32_t pitch = K * 2 + 16;
    const int32_t ntile = blockIdx.x >> 1, h = blockIdx.x & 1;
    const int32_t n = ntile * kPackN + h * 16 + n16;
    const int32_t groups = K / kGroup;
    const int32_t per_wave = (groups + NWAVES - 1) / NWAVES;
    const int32_t begin = wave * per_wave;
    const int32_t end = begin + per_wave < groups ? begin + per_wave : groups;

    const v4u *wlane = wp + static_cast<int64_t>(ntile) * (2 * groups) * 64 + (kg >> 1) * 64 + (kg & 1) * 32 + h * 16 + n16;
    const __half *scol = sT + n;
    v4u b[DEPTH];
    uint16_t sc[DEPTH];
    auto request = [&](int j, int32_t u) {                 // past the end: the last group again, not used
        u = u < groups ? u : groups - 1;
        b[j] = __builtin_nontemporal_load(wlane + static_cast<int64_t>(u) * 128);
        sc[j] = __builtin_bit_cast(uint16_t, scol[static_cast<int64_t>(u) * n_pad]);
    };
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) request(j, begin + j);
    __builtin_amdgcn_sched_barrier(0);
    for (int32_t t = 0; t < T; ++t)
        for (int32_t c = tid; c < K / 8; c += NWAVES * 64)
            *reinterpret_cast<v4u *>(smem + t * pitch + c * 16) =
                *reinterpret_cast<const v4u *>(x + static_cast<int64_t>(t) * ldx + c * 8);
    __syncthreads();

    const uint8_t *xlane = smem + (n16 < T ? n16 : T - 1) * pitch + kg * 64;   // rows >= T are never stored
    const Unpack unpack;
    v4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // two chains
    for (int32_t base = begin; base < end; base += DEPTH) {
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            if (base + j >= end) break;                    // wave-uniform
            const _Float16 sv = __builtin_bit_cast(_Float16, sc[j]);
            const v2h s2 = {sv, sv};
            const v4u bw = b[j];
            request(j, base + j + DEPTH);
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const v8h af = *reinterpret_cast<const v8h *>(xlane + (base + j) * (kGroup * 2) + st * 16);
                const v8h bf = __builtin_bit_cast(v8h, unpack.eight<false>(bw[st], s2));
                acc[st & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af, bf, acc[st & 1], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();                                       // the sums reuse the activations' LDS

    // MFMA 16x16 result register r of lane group kg holds row 4 * kg + r
    float(*red)[4][64] = reinterpret_cast<float(*)[4][64]>(smem);
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[0][r] + acc[1][r];
    __syncthreads();
    for (int r = wave; r < 4; r += NWAVES) {
        const int32_t row = kg * 4 + r;
        if (row < T && n < N) {
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) sum += red[w][r][lane];
            y[static_cast<int64_t>(row) * ldy + n] = __float2half_rn(sum);
        }
    }
}

constexpr int kGemvHalfLds = 150 * 1024;

template <int NWAVES, int DEPTH>
int launch_gemv_half(const __half *x, int64_t ldx, const v4u *wt, const __half *sT, __half *y, int64_t ldy, int32_t T,
                     int32_t N, int32_t K, int32_t n_pad, hipStream_t stream)
{
    auto kern = w4g128_gemv_half_kernel<NWAVES, DEPTH>;
    const int64_t xb = static_cast<int64_t>(T) * (static_cast<int64_t>(K) * 2 + 16);
    const int lds = static_cast<int>(xb > NWAVES * 1024 ? xb : NWAVES * 1024);
    static LdsLimit limit;
    if (lds > 64 * 1024)
        if (const int st = limit.raise(reinterpret_cast<const void *>(kern), kGemvHalfLds); st != MQUANT_OK) return st;
    MQ_LAUNCH(kern, dim3(static_cast<unsigned>(n_pad / 16)), dim3(NWAVES * 64), lds, stream, x, ldx, wt, sT, y, ldy, T,
              N, K, n_pad);
    return launch_status();
}

// What a launch of the whole-tile GEMV takes in microseconds, up to 32 rows on n 32-channel
// tiles.  A wave walks `steps` batches of its k-tiles, `busy` of the waves have any; sixteen waves fill
// a compute unit, of the eight-wave form four groups fit.  Fitted to 18 tile counts x 10 lengths of K
// (128 .. 8192) at 1 to 4 rows and to 53 matrices (K 128 .. 29568, N 32 .. 59136) at 5 to 32 rows,
// weights from HBM; rms 8 %.
double gemv_us(int32_t T, int32_t n, int32_t K)
{
    const bool many = n >= 512;
    const int32_t k_tiles = K / kPackK, waves = many ? 8 : 16;
    const uint32_t per_wave = ceil_div32(k_tiles, waves);
    const double steps = many ? per_wave : ceil_div32(per_wave, 2), busy = ceil_div32(k_tiles, per_wave);
    const double rounds = ceil_div32(n, many ? 4 * kNumCU : kNumCU), tiles = n * (1.0 / kNumCU), q = T * (1.0 / 16);
    if (many)
        return 1.41 + steps * (0.208 + 0.152 * q) + busy * (0.011 + 0.034 * q) + 0.372 * rounds +
               tiles * (0.176 + 0.163 * steps + k_tiles * (0.0384 + 0.0357 * q));
    return steps * (0.532 + 0.520 * q) + busy * (0.045 + 0.051 * q) + rounds * (1.406 * steps + 0.071 * busy) +
           tiles * (0.508 + k_tiles * (0.0095 + 0.0226 * q));
}

// The forms of the half-tile GEMV and the same for them, up to four rows: every group copies
// the rows to LDS (per round and row), then its waves walk their scale groups.  rms 6 % over the
// same sweep.
struct HalfForm {
    int waves;
    int (*launch)(const __half *, int64_t, const v4u *, const __half *, __half *, int64_t, int32_t, int32_t, int32_t,
                  int32_t, hipStream_t);
    double fixed, step, half, half_row, half_group, half_busy, round_row, round_step;
};
constexpr HalfForm kHalf[] = {
    {16, launch_gemv_half<16, 2>, 1.463, 0.396, 0.460, 0.052, 0.038, 0.035, 0.169, 0.329},
    {8, launch_gemv_half<8, 2>, 1.729, 0.226, 0.257, 0.029, 0.042, 0.028, 0.179, 0.160},
    {4, launch_gemv_half<4, 2>, 1.738, 0.061, 0.099, 0.011, 0.038, 0.039, 0.177, 0.267},
};

double half_us(const HalfForm &f, int32_t T, int32_t n, int32_t K)
{
    const uint32_t groups = K / kGroup, steps = ceil_div32(groups, f.waves);
    const double busy = ceil_div32(groups, steps);
    const uint32_t xb = static_cast<uint32_t>(T) * (2 * K + 16), rb = f.waves * 1024;
    const uint32_t lds = xb > rb ? xb : rb, fit = (160 * 1024) / lds, slots = 32 / f.waves;
    const double rounds = ceil_div32(2 * n, kNumCU * (fit < slots ? fit : slots)), halves = 2 * n * (1.0 / kNumCU);
    return f.fixed + f.step * steps + halves * (f.half + f.half_row * T + f.half_group * groups + f.half_busy * busy) +
           rounds * (f.round_row * T + f.round_step * steps);
}

template <int MT, int NWN, int NB>
int launch_g128(const __half *x, int64_t ldx, const uint8_t *wp, __half *y, int64_t ldy, int32_t T,
                int32_t N, int32_t K, hipStream_t stream)
{
    const int32_t n_tiles32 = static_cast<int32_t>(ceil_div(N, kPackN));
    const int32_t tiles_m = static_cast<int32_t>(ceil_div(T, MT * 32));
    const int32_t tiles_n = static_cast<int32_t>(ceil_div(n_tiles32, NWN));
    const int64_t w_bytes = static_cast<int64_t>(n_tiles32) * (K / kPackK) * kPackTileBytes;
    const __half *sT = reinterpret_cast<const __half *>(wp + w_bytes);
    const int32_t wide = (N % 8 == 0 && ldy % 8 == 0 && aligned_to(y, 16)) ? 1 : 0;
    const int32_t band = tiles_m <= 8 ? tiles_m : 6;
    constexpr int lds = g128_lds_bytes<MT, NWN, NB>();
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    auto kern = w4g128_gemm_kernel<MT, NWN, NB>;
    static LdsLimit limit;
    if (lds > 64 * 1024)
        if (const int st = limit.raise(reinterpret_cast<const void *>(kern), lds); st != MQUANT_OK) return st;
    MQ_LAUNCH(kern, dim3(tiles_m * tiles_n), dim3(512), lds, stream, x, ldx, wp, sT, y, ldy, T, N, K,
              tiles_m, tiles_n, n_tiles32, wide, band);
    return launch_status();
}

using G128Launch = int (*)(const __half *, int64_t, const uint8_t *, __half *, int64_t, int32_t, int32_t, int32_t,
                           hipStream_t);

// The compiled tiles and what they cost.  Fitted to the time of every tile on 53 matrices (K 128 ..
// 29568, N 32 .. 59136, the 7B and 72B projections among them) at 32 row counts from 5 to 3072, weights
// from HBM (rms 4 - 7 %): the tile the model picks is within 0.4 % of the fastest one on average.  The cost of
// starting a tile keeps small tiles from short K (128 -> 37888 at T = 128: 64 x 32 tiles 31.6 us, 64 x 256
// ones 7.2).
struct G128Variant {
    TileCost cost;
    G128Launch launch;
};
constexpr G128Variant kG128[] = {
    {{256, 256, 1, 0.770, 4.517, 2.118, 0.000, 1.149, 1.963}, launch_g128<8, 8, 3>},
    {{96, 128, 2, 2.852, 0.536, 1.017, 0.757, 0.250, 1.467}, launch_g128<3, 4, 2>},
    {{256, 128, 1, 1.352, 4.936, 1.182, 0.000, 0.664, 1.375}, launch_g128<8, 4, 2>},
    {{192, 128, 1, 1.336, 3.936, 0.963, 0.000, 0.479, 1.074}, launch_g128<6, 4, 2>},
    {{160, 128, 1, 1.274, 3.627, 0.821, 0.000, 0.424, 0.929}, launch_g128<5, 4, 3>},
    {{128, 128, 1, 1.247, 3.041, 0.758, 0.000, 0.327, 0.765}, launch_g128<4, 4, 3>},
    {{64, 128, 2, 2.649, 0.586, 1.021, 0.611, 0.071, 1.110}, launch_g128<2, 4, 3>},
    {{128, 64, 1, 1.416, 2.769, 0.518, 0.000, 0.139, 0.716}, launch_g128<4, 2, 2>},
    {{64, 64, 1, 1.376, 1.828, 0.328, 0.000, 0.043, 0.631}, launch_g128<2, 2, 3>},
    {{32, 64, 1, 2.755, 0.000, 0.268, 0.000, 0.000, 0.731}, launch_g128<1, 2, 3>},
    {{64, 32, 1, 1.318, 2.004, 0.239, 0.000, 0.064, 0.331}, launch_g128<2, 1, 2>},
    {{32, 32, 1, 1.165, 1.834, 0.147, 0.000, 0.017, 0.362}, launch_g128<1, 1, 3>},
    {{128, 256, 2, 2.742, 0.427, 2.429, 1.464, 0.476, 2.571}, launch_g128<4, 8, 2>},
    {{64, 256, 2, 2.745, 0.000, 1.828, 1.177, 0.179, 1.586}, launch_g128<2, 8, 3>},
};
constexpr int kG128Variants = sizeof(kG128) / sizeof(kG128[0]);
static_assert(kG128Variants == kG128Tiles, "mquant_tune_set validates against this");

// The tile for a shape (or the forced one) and what it is expected to take.
const G128Variant &g128_choose(int32_t T, int32_t N, int32_t K, int32_t forced, double *us_out)
{
    int best = 0;
    double best_us = 0.0;
    for (int i = 0; i < kG128Variants; ++i) {
        const TileCost &c = kG128[i].cost;
        const double us = c.us(static_cast<int64_t>(ceil_div32(T, c.bm)) * ceil_div32(N, c.bn), K);
        if (i == 0 || us < best_us) {
            best = i;
            best_us = us;
        }
    }
    *us_out = best_us;
    return kG128[forced >= 0 ? forced : best];
}

}  // namespace

extern "C" int64_t mquant_w4g128_prepacked_bytes(int32_t N, int32_t K)
{
    if (N < 0 || K < 0) return MQUANT_ERR_BAD_SHAPE;
    if (K % kGroup != 0) return MQUANT_ERR_UNSUPPORTED;
    const int64_t n_tiles = ceil_div(N, kPackN);
    return n_tiles * (K / kPackK) * kPackTileBytes + static_cast<int64_t>(K / kGroup) * n_tiles * kPackN * 2;
}

extern "C" int mquant_w4g128_prepack(const uint8_t *w, const void *scales, uint8_t *out, int32_t N,
                                     int32_t K, mquant_stream_t stream)
{
    if (N < 0 || K < 0) return MQUANT_ERR_BAD_SHAPE;
    if (K % kGroup != 0) return MQUANT_ERR_UNSUPPORTED;
    if (N == 0 || K == 0) return MQUANT_OK;
    if (!w || !scales || !out) return MQUANT_ERR_NULL;
    if (!aligned_to(w, 4) || !aligned_to(out, 16) || !aligned_to(scales, 2)) return MQUANT_ERR_ALIGNMENT;
    const int32_t n_tiles = static_cast<int32_t>(ceil_div(N, kPackN));
    const int32_t k_tiles = K / kPackK;
    const int64_t w_bytes = static_cast<int64_t>(n_tiles) * k_tiles * kPackTileBytes;
    const int64_t dwords = w_bytes / 4;
    const int grid = static_cast<int>(dwords / 256 < 4096 ? (dwords / 256 > 0 ? dwords / 256 : 1) : 4096);
    MQ_LAUNCH(g128_prepack_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream), w,
              static_cast<const __half *>(scales), reinterpret_cast<uint32_t *>(out),
              reinterpret_cast<__half *>(out + w_bytes), N, K, n_tiles, k_tiles);
    return launch_status();
}

extern "C" int mquant_w4g128_gemm(const void *x, int64_t ldx, const uint8_t *wp, void *y,
                                  int64_t ldy, int32_t T, int32_t N, int32_t K,
                                  mquant_stream_t stream)
{
    if (T < 0 || N < 0 || K < 0 || ldx < K || ldy < N) return MQUANT_ERR_BAD_SHAPE;
    if (K % kGroup != 0) return MQUANT_ERR_UNSUPPORTED;
    if (T == 0 || N == 0) return MQUANT_OK;
    if (K == 0) return MQUANT_ERR_UNSUPPORTED;
    if (!x || !wp || !y) return MQUANT_ERR_NULL;
    if (!aligned_to(x, 16) || ldx % 8 != 0 || !aligned_to(wp, 16) || !aligned_to(y, 2))
        return MQUANT_ERR_ALIGNMENT;
    const __half *xh = static_cast<const __half *>(x);
    __half *yh = static_cast<__half *>(y);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Up to twelve rows a GEMV streams the weights; from 13 to 32 one does where the GEMM is not
    // expected to be 5 % ahead of the GEMV with a work-group per tile (the walking one is not weighed here): GEMV against GEMM at 13 and 32 rows: 18944 x 3584 27.7 / 25.9 us and 46.7 /
    // 27.2, 3584 x 18944 16.9 / 16.3 and 27.9 / 17.9, 512 x 16384 3.9 / 4.4 and 5.2 / 4.6.  It also takes rows so far
    // apart that the GEMM's 32-bit offsets inside a tile would not reach, 32 of them at a time.
    const int32_t n_tiles32 = static_cast<int32_t>(ceil_div(N, kPackN));
    const int32_t forced = tune_state().g128_tile.load(std::memory_order_relaxed);
    double gemm_us;
    const G128Variant &gemm = g128_choose(T, N, K, forced, &gemm_us);
    const bool gemv = forced < 0 && (T <= 12 || (T <= 32 && gemm_us > 0.95 * gemv_us(T, n_tiles32, K)));
    if (gemv || ldx >= kG128MaxLdx) {
        const int64_t w_bytes = static_cast<int64_t>(n_tiles32) * (K / kPackK) * kPackTileBytes;
        const __half *sT = reinterpret_cast<const __half *>(wp + w_bytes);
        const v4u *wt = reinterpret_cast<const v4u *>(wp);
        const int32_t n_pad = n_tiles32 * kPackN;
        if (g128_walk_takes(T, K, N)) return g128_walk(xh, ldx, wt, sT, yh, ldy, T, N, K, n_pad, st);
        // Up to four rows that fit LDS take the half-tile form with the number of waves that is expected
        // to be fastest, or the whole-tile one: half tiles against whole ones at 1 / 4 rows: 18944 x 3584
        // 11.3 / 22.5 us and 12.4 / 23.3, 3584 x 3584 4.8 / 6.6 and 5.5 / 6.9; whole ones where every
        // group would copy rows for little work: 128 x 37888 4.2 / 4.6 and 4.3 / 6.0, 2048 x 5120 4.5 / 4.6 and 4.6 / 5.8.
        // At 6 rows the copy costs more than it saves on wide matrices (3584 x 37888 27.9 / 22.2).
        if (T <= 4 && static_cast<int64_t>(T) * (static_cast<int64_t>(K) * 2 + 16) <= kGemvHalfLds) {
            const HalfForm *best = nullptr;
            double best_us = gemv_us(T, n_tiles32, K);
            for (const HalfForm &f : kHalf) {
                const double us = half_us(f, T, n_tiles32, K);
                if (us < best_us) {
                    best = &f;
                    best_us = us;
                }
            }
            if (best) return best->launch(xh, ldx, wt, sT, yh, ldy, T, N, K, n_pad, st);
        }
        for (int32_t t0 = 0; t0 < T; t0 += 32) {
            const int32_t tc = T - t0 < 32 ? T - t0 : 32;
            const __half *xc = xh + static_cast<int64_t>(t0) * ldx;
            __half *yc = yh + static_cast<int64_t>(t0) * ldy;
            // Many tiles: small work-groups with one k-tile in flight per wave keep the register
            // count low and several groups resident per CU (fastest on 1184 tiles x 56 k-tiles);
            // few tiles: sixteen waves split K.
            if (n_tiles32 >= 512)
                MQ_LAUNCH((w4g128_gemv_kernel<8, 1>), dim3(n_tiles32), dim3(512), 0, st, xc, ldx, wt,
                          sT, yc, ldy, tc, N, K, n_pad);
            else
                MQ_LAUNCH((w4g128_gemv_kernel<16, 2>), dim3(n_tiles32), dim3(1024), 0, st, xc, ldx,
                          wt, sT, yc, ldy, tc, N, K, n_pad);
            const int status = launch_status();
            if (status != MQUANT_OK) return status;
        }
        return MQUANT_OK;
    }
    return gemm.launch(xh, ldx, wp, yh, ldy, T, N, K, st);
}
