// W4A8 GEMM with 256 x 384 tiles and three smaller ones: the largest prefill linears, and shapes whose tiles of one of these
// sizes fill the compute units' rounds better than those of w4a8_gemm.hip.
//
// What bounds the largest is power (8192 -> 59136 at T = 16384: the matrix pipes hold an MFMA in 84 % of the busy cycles, 78 % with
// 256 x 256, at 1.6 to 1.7 GHz where the rotation beside it runs at 1.9), and a large part of it goes into bringing operands to the matrix
// cores.  Per multiply-add the 256 x 384 tile takes 22 % fewer bytes out of the L2 and 27 % fewer out of LDS than 256 x 256 with
// 128 x 64 wave tiles: eight waves, two rows of four, hold 128 x 96 each, 192 accumulator registers.  The 64 that
// are left do not take two sets of operands, so the fragments of the activations go through a ring of four, each requested
// nine MFMAs ahead and used for three; a weight operand is unpacked again into its own registers as soon as the last of its
// four MFMAs has been issued, from packed bytes that were read when the step before began.
//
// The waves of 192 x 256, 128 x 384 and 128 x 256 hold 96 x 64, 64 x 96 and 64 x 64 (two work-groups on a compute unit in the
// last).  The first two are there for what would else be one full round and a few tiles of the next.  256 x 256 in this form (and
// 192 x 128, 192 x 384, 256 x 128) is up to 4 % behind the tile of w4a8_gemm.hip.
//
// A stage is 128 channels: three buffers of activations (rows of 128 bytes, 16-byte chunk c of row r at
// c ^ ((r >> 1) & 7)), copied two stages ahead, and two of weights, copied one stage ahead: 144 KiB of LDS at 256 x 384.  One
// barrier a stage, three fragments before its end, where its last operands are in registers.  (Stages of 64 channels, five of
// them: rows of 64 bytes and twice the barriers cost what the tile gains.)
//
// us, 256 x 256 -> 256 x 384, two cards: 8192 -> 59136 at T = 16384 6158 -> 5770, 3584 -> 37888 at 1280 154 -> 143 and 149 -> 145, at
// 16384 1889 -> 1780; against 128 x 256 3584 -> 4608 at 4096 71.7 -> 64.6, 8192 -> 10240 at 2048 158 -> 141.
// 192 x 256 and 128 x 384, against what was taken before them: 8192 -> 10240 at 900 82.9 -> 68.2, 6912 -> 5120 at 2048 74.1 -> 62.1,
// 5120 -> 5120 at 2048 53.6 -> 46.6, 3584 -> 4608 at 2048 38.6 -> 32.7, 3584 -> 3584 at 3000 39.9 -> 35.0.
// 128 x 256 against that of w4a8_gemm.hip: 1.6 % less on average over 108 shapes, 5120 -> 27648 at 3600 412 -> 405.
#include "lds_dma.h"
#include "w4a8_common.h"

using namespace mquant;

namespace {

template <int MT, int NT>
struct WideTile {
    static constexpr int BM = MT * 64, BN = NT * 128;
    static constexpr int A_STAGE = BM * 128, B_STAGE = BN * 64, B_OFF = 3 * A_STAGE, LDS = B_OFF + 2 * B_STAGE;
    static constexpr int FR = 4 * MT;                 // fragments of a stage
    static constexpr int BAR = FR - 3;                // the barrier sits in front of this one
    // where the packed weights of k-tile 1 and of the next stage are read: three fragments before their first use (at MT = 2 two),
    // one earlier and 256 x 384 spills
    static constexpr int RAW1 = MT < 4 ? MT : 5, RAW0 = BAR > 3 * MT ? BAR : 3 * MT;
    static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
};

// Work-group id -> (tm, tn): each of the eight XCDs (ids are dealt to them round robin) gets a
// contiguous run of an order that walks bands of `band` tile-rows.
__device__ __forceinline__ void tile_of_group(int32_t id, int32_t tiles_m, int32_t tiles_n, int32_t band, int32_t &tm,
                                              int32_t &tn)
{
    const int32_t total = tiles_m * tiles_n;
    const int32_t per = total / 8, rem = total % 8;
    const int32_t xcd = id % 8, local = id / 8;
    const int32_t t = xcd * per + (xcd < rem ? xcd : rem) + local;
    const int32_t b = t / (band * tiles_n);
    const int32_t in_band = t - b * band * tiles_n;
    const int32_t rows = (tiles_m - b * band) < band ? (tiles_m - b * band) : band;
    tm = b * band + in_band % rows;
    tn = in_band / rows;
}

template <int MT, int NT, int EPI>
__global__ __launch_bounds__(512, 2) void w4a8_wide_kernel(
    const int8_t *__restrict__ xq, const uint4 *__restrict__ wp, const __half *__restrict__ w_scale,
    __half *__restrict__ y, int64_t ldy, int32_t *__restrict__ acc_out, int32_t T, int32_t N, int32_t K, Epilogue ep,
    int32_t tiles_m, int32_t tiles_n, int32_t n_tiles32, int32_t wide_store, int32_t band)
{
    using W = WideTile<MT, NT>;
    constexpr int BM = W::BM, BN = W::BN, A_STAGE = W::A_STAGE, B_STAGE = W::B_STAGE, B_OFF = W::B_OFF;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    int32_t tm, tn;
    tile_of_group(blockIdx.x, tiles_m, tiles_n, band, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, g = lane >> 5;
    const int32_t row0 = tm * BM, stages = K / 128, ntile0 = tn * (BN / 32);

    v16i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0;

    // Copies: uniform bases and 32-bit lane offsets.  Rows past T and tiles past the padded N repeat valid ones (never
    // stored).  A stage is MT copies of activations and NT of weights for every wave.
    const uint32_t lds0 = lds_address(smem);
    const uint8_t *abase = reinterpret_cast<const uint8_t *>(xq) + static_cast<int64_t>(row0) * K;
    uint32_t a_off[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int r = (wave + j * 8) * 8 + (lane >> 3);
        const int32_t row = row0 + r < T ? r : T - 1 - row0;
        a_off[j] = static_cast<uint32_t>(row) * static_cast<uint32_t>(K) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    const uint8_t *bbase[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int b = wave + j * 8;
        int32_t nt = ntile0 + (b >> 1);
        nt = nt < n_tiles32 ? nt : n_tiles32 - 1;
        bbase[j] = reinterpret_cast<const uint8_t *>(wp) + (static_cast<int64_t>(nt) * stages * 2 + (b & 1)) * kPackTileBytes;
    }
    const uint32_t b_off = lane * 16;
    auto copy_a = [&](int j, int32_t s, uint32_t buf) {        // buf: byte offset of the stage buffer
        lds_dma16_uniform_base(abase + static_cast<int64_t>(s) * 128, a_off[j], lds0 + buf + (wave + j * 8) * 1024);
    };
    auto copy_b = [&](int j, int32_t s) {
        lds_dma16_uniform_base(bbase[j] + static_cast<int64_t>(s) * (2 * kPackTileBytes), b_off,
                               lds0 + B_OFF + (s & 1) * B_STAGE + (wave + j * 8) * 1024);
    };

    typedef uint32_t v4u_lds __attribute__((ext_vector_type(4)));
    typedef const v4u_lds __attribute__((address_space(3))) *frag_ptr;
    const uint32_t a_lane = lds0 + (wm * MT * 32 + l32) * 128 + (((g * 2) ^ ((l32 >> 1) & 7)) << 4);
    const uint32_t b_lane = lds0 + B_OFF + wn * NT * 2048 + lane * 16;
    // fragment f of a stage: step f / MT (k-tile step / 2, half step % 2), rows f % MT
    auto read_a = [&](uint32_t buf, int f) -> v4i {
        const v4u_lds u = *(frag_ptr)(uintptr_t)((a_lane ^ ((f / MT / 2 * 4 + f / MT % 2) << 4)) + buf + f % MT * 4096);
        return __builtin_bit_cast(v4i, u);
    };
    auto read_b = [&](uint32_t buf, int ks, int nt) -> v4i {
        const v4u_lds u = *(frag_ptr)(uintptr_t)(b_lane + buf + nt * 2048 + ks * 1024);
        return __builtin_bit_cast(v4i, u);
    };
    auto unpack = [](const v4i &raw, int h, v4i &b) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = static_cast<uint32_t>(raw[h * 2 + (j >> 1)]);
            b[j] = static_cast<int>(((j & 1) ? v : v << 4) & 0xF0F0F0F0u);
        }
    };

    // prologue: both weight buffers, the three of the activations; waits for stage 0
#pragma unroll
    for (int s = 0; s < 3; ++s)
        if (s < stages) {
            if (s < 2)
#pragma unroll
                for (int j = 0; j < NT; ++j) copy_b(j, s);
#pragma unroll
            for (int j = 0; j < MT; ++j) copy_a(j, s, s * A_STAGE);
        }
    if (stages >= 3) wait_vmcnt<NT + 2 * MT>();
    else if (stages == 2) wait_vmcnt<NT + MT>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    constexpr int RING = 4;
    v4i a[RING], raw[NT], b[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) raw[nt] = read_b(0, 0, nt);
#pragma unroll
    for (int i = 0; i < RING - 1; ++i) a[i] = read_a(0, i);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) unpack(raw[nt], 0, b[nt]);

    uint32_t cur = 0;
    for (int32_t s = 0; s < stages; ++s) {
        const uint32_t nxt = cur + A_STAGE == 3 * A_STAGE ? 0 : cur + A_STAGE;
        const uint32_t prev = cur == 0 ? 2 * A_STAGE : cur - A_STAGE;
        const uint32_t bcur = (s & 1) * B_STAGE, bnxt = B_STAGE - bcur;
        const bool refill_a = s >= 1 && s + 2 < stages, refill_b = s + 2 < stages;
#pragma unroll
        for (int f = 0; f < W::FR; ++f) {
            const int mt = f % MT;
            if (f == W::BAR && s + 1 < stages) {
                // every operand of this stage is in registers; the next one's copies have landed
                if (s + 2 < stages) wait_vmcnt<MT>();
                else wait_vmcnt<0>();
                wait_lgkm0();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            const int q = f + RING - 1;                        // the fragment requested here
            a[q % RING] = q < W::FR ? read_a(cur, q) : read_a(nxt, q - W::FR);
            if (f == W::RAW1)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) raw[nt] = read_b(bcur, 1, nt);
            if (f == W::RAW0)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) raw[nt] = read_b(bnxt, 0, nt);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                acc[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[f % RING], b[nt], acc[mt][nt], 0, 0, 0);
                if (mt == MT - 1) unpack(raw[nt], (f / MT + 1) & 1, b[nt]);
                if (nt == NT / 2) {
                    if (refill_a && f >= 1 && f <= MT) copy_a(f - 1, s + 2, prev);
                    if (refill_b && f >= W::BAR && f < W::BAR + NT) copy_b(f - W::BAR, s + 2);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
    }

    const int32_t wave_row0 = row0 + wm * MT * 32, wave_n0 = (ntile0 + wn * NT) * 32;
    if (!wide_store || acc_out != nullptr) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int32_t n = wave_n0 + nt * 32 + l32;
            if (n >= N) continue;
            const float ws = __half2float(w_scale[n]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int32_t row = wave_row0 + mt * 32 + acc_row(r, g);
                    if (row < T) store_out<EPI>(acc[mt][nt][r], row, n, ep, ws, y, ldy, acc_out, N);
                }
        }
        return;
    }
    // Wide path: 32 rows at a time through the wave's own LDS patch, out as 16 bytes per lane.
    constexpr int ROWB = NT * 64 + 16, LPR = NT * 4;
    __syncthreads();
    uint8_t *patch = smem + wave * (32 * ROWB);
    float ws[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int32_t n = wave_n0 + nt * 32 + l32;
        ws[nt] = __half2float(w_scale[n < N ? n : N - 1]);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int rl = acc_row(r, g);
            const int32_t row = wave_row0 + mt * 32 + rl;
            const int32_t row_in = row < T ? row : T - 1;
            const float s_row = ep.scale_of<EPI>(row_in);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                int32_t n = wave_n0 + nt * 32 + l32;
                n = n < N ? n : N - 1;
                const float v = ep.dequant<EPI>(acc[mt][nt][r] >> 4, s_row, row_in, n, N, ws[nt]);
                *reinterpret_cast<__half *>(patch + rl * ROWB + (nt * 32 + l32) * 2) = half_of_rounded_f32(v);
            }
        }
#pragma unroll
        for (int q = 0; q < 32 * LPR / 64; ++q) {
            const int i = q * 64 + lane, rl = i / LPR, c = i % LPR;
            const uint4 v = *reinterpret_cast<const uint4 *>(patch + rl * ROWB + c * 16);
            const int32_t row = wave_row0 + mt * 32 + rl, n = wave_n0 + c * 8;
            if (row < T && n < N) *reinterpret_cast<uint4 *>(y + static_cast<int64_t>(row) * ldy + n) = v;
        }
    }
}

}  // namespace

namespace mquant {

namespace {

template <int MT, int NT, int EPI>
int launch_wide_tile(const int8_t *xq, int32_t T, int32_t K, const GemvProblem &pr, const Epilogue &ep, hipStream_t stream)
{
    static_assert(EPI != kEpiSplit, "the split terms do not fit the registers");
    const int32_t N = pr.N, tiles_m = static_cast<int32_t>(ceil_div(T, MT * 64)), tiles_n = static_cast<int32_t>(ceil_div(N, NT * 128));
    const int32_t wide = (N % 8 == 0 && pr.ldy % 8 == 0 && aligned_to(pr.y, 16) && !pr.acc_out) ? 1 : 0;
    const int32_t band = tiles_m <= 8 ? tiles_m : static_cast<int32_t>(ceil_div(tiles_m, ceil_div(tiles_m, 6)));
    constexpr int lds = WideTile<MT, NT>::LDS;
    auto kern = w4a8_wide_kernel<MT, NT, EPI>;
    static LdsLimit limit;
    if (const int st = limit.raise(reinterpret_cast<const void *>(kern), lds); st != MQUANT_OK) return st;
    MQ_LAUNCH(kern, dim3(tiles_m * tiles_n), dim3(512), lds, stream, xq, pr.wp, pr.w_scale, pr.y,
              pr.ldy, pr.acc_out, T, N, K, ep, tiles_m, tiles_n, static_cast<int32_t>(ceil_div(N, kPackN)), wide,
              band);
    return launch_status();
}

}  // namespace

template <int EPI>
int launch_wide(int tile, const int8_t *xq, int32_t T, int32_t K, const GemvProblem &pr, const Epilogue &ep, hipStream_t stream)
{
    switch (tile) {
    case 0: return launch_wide_tile<4, 3, EPI>(xq, T, K, pr, ep, stream);
    case 1: return launch_wide_tile<3, 2, EPI>(xq, T, K, pr, ep, stream);
    case 2: return launch_wide_tile<2, 3, EPI>(xq, T, K, pr, ep, stream);
    default: return launch_wide_tile<2, 2, EPI>(xq, T, K, pr, ep, stream);
    }
}
template int launch_wide<kEpiStatic>(int, const int8_t *, int32_t, int32_t, const GemvProblem &, const Epilogue &, hipStream_t);
template int launch_wide<kEpiRowScale>(int, const int8_t *, int32_t, int32_t, const GemvProblem &, const Epilogue &, hipStream_t);

}  // namespace mquant
