// W4A8 GEMM with the K range of a tile sliced over the waves of its work-group: the shapes
// between the decode GEMV (a few rows) and the large prefill tiles, where an output of few
// tiles leaves most compute units idle or every tile walks a long K alone.
//
// One work-group of eight waves computes an MT*32 x NWN*32 tile.  The waves stand as NWN column
// waves x KS = 8 / NWN K slices: a wave owns all MT*32 rows of one 32-channel column and one
// 128-channel block of every stage (KS blocks), so a weight is unpacked once per work-group
// and the slices of a column are added through LDS at the end (int32: in any order).  Against a
// split of K over work-groups this needs no workspace, no second launch and no partial sums in
// memory.
//
// A stage arrives by LDS-DMA: the activations (KS slabs of MT*32 rows x 128 bytes, 16-byte
// chunk c of row r at c ^ ((r >> 1) & 7): 16 consecutive rows cover the 64 banks once) and
// every wave's own two weight tiles.  After the barrier that ends the reads of stage s its buffer
// is refilled with stage s + NB; that barrier sits WIN MFMAs before the end of the stage, whose
// last operands are in registers by then, and the first fragments and weights of the next
// stage are requested behind it.
#include "lds_dma.h"
#include "w4a8_common.h"

using namespace mquant;

namespace {

template <int MT, int NWN>
struct SlicedTile {
    static constexpr int KS = 8 / NWN;
    static constexpr int WIN = MT > 1 ? 4 : 2;        // A fragments requested ahead of the MFMA that uses them
    static constexpr int A_SLAB = MT * 32 * 128;
    static constexpr int B_OFF = KS * A_SLAB, STAGE = B_OFF + 8 * 2048;
    static constexpr int CHA = (MT * KS + 1) / 2;     // 1 KiB activation blocks a wave copies per stage
    static constexpr int PER = CHA + 2;               // ... and its two weight tiles
    // Activation block i of a wave.  Where the blocks are an odd multiple of four, two waves copy each block of the
    // last round (the same bytes to the same place), so that every wave counts the same copies.
    static __device__ __forceinline__ int a_block(int wave, int i)
    {
        return ((MT * KS) % 2 != 0 && i == CHA - 1 ? wave % 4 : wave) + 8 * i;
    }
    static constexpr int RED = NWN * MT * 4 * (KS - 1) * 1024;   // slice sums in transit
    static constexpr int CODES = RED + 8 * 32 * 80;              // ... after them the store patches
    static constexpr int SPLIT_W = CODES + kMaxSplitChannels * MT * 32;   // flagged codes [j][row], weights [j][column]
    static constexpr int epilogue_bytes(int epi)
    {
        return epi == kEpiSplit ? SPLIT_W + kMaxSplitChannels * NWN * 32 : CODES;
    }
};

template <int MT, int NWN, int NB, int EPI>
constexpr int sliced_lds_bytes()
{
    using S = SlicedTile<MT, NWN>;
    return NB * S::STAGE > S::epilogue_bytes(EPI) ? NB * S::STAGE : S::epilogue_bytes(EPI);
}

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

// Waits for a stage of this wave's copies, PER of them: at most MOST of the stages behind it, and of these the `left` that there
// are, may still be on their way.
template <int MOST, int PER>
__device__ __forceinline__ void wait_left(int32_t left)
{
    if constexpr (MOST <= 0) {
        wait_vmcnt<0>();
    } else {
        if (left >= MOST) wait_vmcnt<MOST * PER>();
        else wait_left<MOST - 1, PER>(left);
    }
}

// The same for stage s of `stages`.  The two are compiled to different loops: by the count the per-row-scale kernel of 64 x 256 takes
// 1 to 2 % longer on average, 9 % at worst, the others of up to three stages 0.5 %; this way those of four stages and those
// of 256 columns with flagged channels take up to 1.5 % longer.
template <int MOST, int PER>
__device__ __forceinline__ void wait_stage(int32_t s, int32_t stages)
{
    if constexpr (MOST <= 0) {
        wait_vmcnt<0>();
    } else {
        if (s + MOST < stages) wait_vmcnt<MOST * PER>();
        else wait_stage<MOST - 1, PER>(s, stages);
    }
}

// Several linears that share xq can go into one launch: tiles_n counts the column tiles of all.
template <int MT, int NWN, int NB, int EPI>
__global__ __launch_bounds__(512, (sliced_lds_bytes<MT, NWN, NB, kEpiStatic>() <= 80 * 1024 ? 4 : 2)) void w4a8_sliced_kernel(
    const int8_t *__restrict__ xq, GemvGroup grp, int32_t T, int32_t K, Epilogue ep, int32_t tiles_m,
    int32_t tiles_n, int32_t band)
{
    using S = SlicedTile<MT, NWN>;
    constexpr int KS = S::KS, WIN = S::WIN;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];   // sliced_lds_bytes<...>()

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int wn = wave % NWN, ks = wave / NWN;
    int32_t tm, tn;
    tile_of_group(blockIdx.x, tiles_m, tiles_n, band, tm, tn);
    int32_t pi = 0;
    while (pi + 1 < grp.n && tn >= grp.p[pi].units) {
        tn -= grp.p[pi].units;
        ++pi;
    }
    const int32_t N = grp.p[pi].N;
    const __half *__restrict__ w_scale = grp.p[pi].w_scale;
    __half *__restrict__ y = grp.p[pi].y;
    int32_t *__restrict__ acc_out = grp.p[pi].acc_out;
    const int64_t ldy = grp.p[pi].ldy;

    const int32_t row0 = tm * MT * 32;
    const int32_t k_blocks = K / 128;
    const int32_t stages = (k_blocks + KS - 1) / KS;
    const int32_t n_tiles32 = (N + kPackN - 1) / kPackN;
    const int32_t n0 = (tn * NWN + wn) * kPackN;      // first column of this wave
    // column tiles past the last one repeat it (never stored)
    const int32_t ntile = tn * NWN + wn < n_tiles32 ? tn * NWN + wn : n_tiles32 - 1;
    const __half ws_h = w_scale[n0 + l32 < N ? n0 + l32 : N - 1];

    // ---- copies.  Uniform bases and 32-bit lane offsets; rows past T repeat row T - 1 and
    // blocks past the last one repeat it (neither result is used).
    const uint8_t *xbase = reinterpret_cast<const uint8_t *>(xq) + static_cast<int64_t>(row0) * K;
    const uint8_t *wbase = reinterpret_cast<const uint8_t *>(grp.p[pi].wp) +
                           static_cast<int64_t>(ntile) * k_blocks * (2 * kPackTileBytes);
    const uint32_t lds0 = lds_address(smem);
    uint32_t aoff[S::CHA];
#pragma unroll
    for (int i = 0; i < S::CHA; ++i) {
        const int r = (S::a_block(wave, i) % (MT * 4)) * 8 + (lane >> 3);
        const int32_t row = row0 + r < T ? r : T - 1 - row0;
        aoff[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(K) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    auto copy_piece = [&](int i, int32_t s, uint32_t buf) {   // buf: byte offset of the stage buffer
        const int b = S::a_block(wave, i);
        int32_t kb = s * KS + (i < S::CHA ? b / (MT * 4) : ks);
        kb = kb < k_blocks ? kb : k_blocks - 1;
        if (i < S::CHA)
            lds_dma16_uniform_base(xbase + kb * 128, aoff[i < S::CHA ? i : 0], lds0 + buf + b * 1024);
        else
            lds_dma16_uniform_base(wbase + static_cast<int64_t>(kb) * (2 * kPackTileBytes),
                                   (i - S::CHA) * 1024 + lane * 16,
                                   lds0 + buf + S::B_OFF + wave * 2048 + (i - S::CHA) * 1024);
    };

    v16i acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0;

    // step st of a stage: chunk (st / 2) * 4 + g * 2 + st % 2 of a row, half st % 2 of weight tile st / 2
    const uint32_t a_lane = ks * S::A_SLAB + l32 * 128 + (((g * 2) ^ ((l32 >> 1) & 7)) << 4);
    auto afrag = [&](uint32_t buf, int st, int mt) {
        return *reinterpret_cast<const v4i *>(smem + buf + (a_lane ^ (((st >> 1) * 4 + (st & 1)) << 4)) + mt * 4096);
    };
    auto btile = [&](uint32_t buf, int t) {
        return *reinterpret_cast<const v4i *>(smem + buf + S::B_OFF + wave * 2048 + t * 1024 + lane * 16);
    };
    auto unpack = [](const v4i (&bw)[2], int st, int j) -> int {   // dword j of the operand of step st
        const uint32_t v = static_cast<uint32_t>(bw[st >> 1][(st & 1) * 2 + (j >> 1)]);
        return static_cast<int>(((j & 1) ? v : v << 4) & 0xF0F0F0F0u);
    };

    // ---- prologue: fill every buffer, wait for stage 0, first operands
#pragma unroll
    for (int s = 0; s < NB; ++s)
        if (s < stages)
#pragma unroll
            for (int i = 0; i < S::PER; ++i) copy_piece(i, s, s * S::STAGE);
    constexpr bool COUNT_LEFT = NB > 3 || (EPI == kEpiSplit && NWN == 8);
    if constexpr (COUNT_LEFT) wait_left<NB - 1, S::PER>(stages - 1);
    else wait_stage<NB - 1, S::PER>(0, stages);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    uint32_t cur = 0;
    v4i bw[2] = {btile(0, 0), btile(0, 1)};
    v4i fr[WIN];
#pragma unroll
    for (int i = 0; i < WIN; ++i) fr[i] = afrag(0, i / MT, i % MT);
    v4i bf[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) bf[0][j] = unpack(bw, 0, j);

    // A wave whose slice ends a stage early (K / 128 not a multiple of KS) leaves the loop one
    // stage early; there is no barrier in the last stage.
    const int32_t my_stages = (stages - 1) * KS + ks < k_blocks ? stages : stages - 1;
    for (int32_t s = 0; s < my_stages; ++s) {
        const uint32_t nxt = cur + S::STAGE == NB * S::STAGE ? 0 : cur + S::STAGE;
        v4i bw_n[2] = {bw[0], bw[1]};
        constexpr int NM = 4 * MT, BAR = NM - WIN, LAND = BAR - (MT < 4 ? MT : 4);
        static_assert(LAND >= 0, "window");
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int st = m / MT, mt = m % MT;
            if (m == LAND) {
                // this wave's copies of the next stage have landed: its own weights
                if constexpr (COUNT_LEFT) wait_left<NB - 2, S::PER>(stages - 2 - s);
                else wait_stage<NB - 2, S::PER>(s + 1, stages);
                asm volatile("" ::: "memory");
                bw_n[0] = btile(nxt, 0);
                bw_n[1] = btile(nxt, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (m == BAR && s + 1 < stages) {
                // every operand of this stage is in registers, every wave's copies have landed
                wait_lgkm0();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            acc[mt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[m % WIN], bf[st & 1], acc[mt], 0, 0, 0);
            const int f = m + WIN;                     // the fragment requested behind this MFMA
            if (f < NM) fr[m % WIN] = afrag(cur, f / MT, f % MT);
            else fr[m % WIN] = afrag(nxt, (f - NM) / MT, (f - NM) % MT);
            if (m >= BAR && s + NB < stages) {         // refill the buffer just freed, a few pieces per MFMA
#pragma unroll
                for (int i = (m - BAR) * S::PER / WIN; i < (m - BAR + 1) * S::PER / WIN; ++i)
                    copy_piece(i, s + NB, cur);
            }
            // the next step's weights, dealt over the MFMAs of this one
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((MT >= 4 ? MT - 4 + j : j * MT / 4) == mt)
                    bf[(st + 1) & 1][j] = st < 3 ? unpack(bw, st + 1, j) : unpack(bw_n, 0, j);
            __builtin_amdgcn_sched_barrier(0);
        }
        bw[0] = bw_n[0];
        bw[1] = bw_n[1];
        cur = nxt;
    }
    __syncthreads();                                    // every wave is done with the stage buffers

    // ---- flagged channels: the codes of the tile's rows and the split weights of its columns go
    // to LDS once, so that the terms below read them without a round trip to memory each
    if constexpr (EPI == kEpiSplit) {
        for (int32_t e = tid; e < ep.n_split * MT * 32; e += 512) {
            const int32_t j = e / (MT * 32), row = row0 + e % (MT * 32);
            smem[S::CODES + e] = static_cast<uint8_t>(
                ep.xq[static_cast<int64_t>(row < T ? row : T - 1) * K + ep.split_idx[j]]);
        }
        for (int32_t e = tid; e < ep.n_split * NWN * 32; e += 512) {
            const int32_t j = e / (NWN * 32), n = tn * NWN * 32 + e % (NWN * 32);
            smem[S::SPLIT_W + e] =
                static_cast<uint8_t>(ep.split_w[static_cast<int64_t>(j) * N + (n < N ? n : N - 1)]);
        }
        if (KS == 1) __syncthreads();                   // else the barrier of the slice sums
    }

    // ---- add the K slices of a column.  The rows of a 32x32 block held by registers 4 q .. 4 q + 3
    // (eight rows of the block) are unit mt * 4 + q; unit u belongs to slice u % KS, every other
    // slice hands its part over through LDS.
    if constexpr (KS > 1) {
        int32_t *red = reinterpret_cast<int32_t *>(smem) + wn * (MT * 4 * (KS - 1) * 256);
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

    // ---- dequantise (Eq. (3) row scale, per-channel scale; then the split terms in the order
    // j = 0, 1, ...) and store.  Four rows at a time: registers 4 q .. 4 q + 3 of a block.
    const float ws = __half2float(ws_h);
    const bool wide = N % 8 == 0 && ldy % 8 == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0 && acc_out == nullptr;
    const int32_t n = n0 + l32;
    uint8_t *patch = smem + S::RED + wave * (32 * 80);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((mt * 4 + q) % KS != ks) continue;
            const int32_t r0 = mt * 32 + q * 8 + g * 4;            // first of the four rows, in the tile
            int32_t a[4];
            float s_row[4], v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int32_t row = row0 + r0 + e;
                a[e] = acc[mt][q * 4 + e] >> 4;                    // exact: the sum holds 16 * acc
                s_row[e] = ep.scale_of<EPI>(row < T ? row : T - 1);    // rows past T are never stored
                v[e] = (static_cast<float>(a[e]) * s_row[e]) * ws;
            }
            if constexpr (EPI == kEpiSplit) {
                for (int32_t j = 0; j < ep.n_split; ++j) {
                    const uint32_t codes = *reinterpret_cast<const uint32_t *>(smem + S::CODES + j * (MT * 32) + r0);
                    const int32_t w = static_cast<int8_t>(smem[S::SPLIT_W + (j * NWN + wn) * 32 + l32]);
                    const float sc = ep.split_scale[j];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int32_t p = static_cast<int32_t>(static_cast<int8_t>(codes >> (8 * e))) * w;
                        v[e] = v[e] + (static_cast<float>(p) * s_row[e]) * sc;
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const __half h = half_of_rounded_f32(v[e]);
                if (wide) {
                    *reinterpret_cast<__half *>(patch + (q * 8 + g * 4 + e) * 80 + l32 * 2) = h;
                } else if (row0 + r0 + e < T && n < N) {
                    const int64_t row = row0 + r0 + e;
                    y[row * ldy + n] = h;
                    if (acc_out) acc_out[row * N + n] = a[e];
                }
            }
        }
        // The MFMA result has a lane per column: the wave's rows of the block go through its own
        // LDS patch and leave as 16 bytes per lane.
        if (wide) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int rl = q * 16 + lane / 4, c = lane % 4;
                const v4i v = *reinterpret_cast<const v4i *>(patch + rl * 80 + c * 16);
                const int32_t row = row0 + mt * 32 + rl, nc = n0 + c * 8;
                if ((mt * 4 + rl / 8) % KS == ks && row < T && nc < N)     // N % 8 == 0 on this path
                    *reinterpret_cast<v4i *>(y + static_cast<int64_t>(row) * ldy + nc) = v;
            }
        }
    }
}

template <int MT, int NWN, int NB, int EPI>
int launch_sliced(const int8_t *xq, int32_t T, int32_t K, GemvGroup grp, const Epilogue &ep, hipStream_t stream)
{
    const int64_t tiles_m = ceil_div(T, MT * 32);
    int64_t tiles_n = 0;
    for (int32_t i = 0; i < grp.n; ++i) {
        grp.p[i].units = static_cast<int32_t>(ceil_div(grp.p[i].N, NWN * 32));
        tiles_n += grp.p[i].units;
    }
    if (tiles_m * tiles_n > 0x7fffffff) return MQUANT_ERR_UNSUPPORTED;
    const int32_t band = static_cast<int32_t>(tiles_m <= 8 ? tiles_m : ceil_div(tiles_m, ceil_div(tiles_m, 6)));
    constexpr int lds = sliced_lds_bytes<MT, NWN, NB, EPI>();
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    auto kern = w4a8_sliced_kernel<MT, NWN, NB, EPI>;
    static LdsLimit limit;
    if (lds > 64 * 1024)
        if (const int st = limit.raise(reinterpret_cast<const void *>(kern), lds); st != MQUANT_OK) return st;
    MQ_LAUNCH(kern, dim3(static_cast<unsigned>(tiles_m * tiles_n)), dim3(512), lds, stream, xq, grp, T, K, ep,
              static_cast<int32_t>(tiles_m), static_cast<int32_t>(tiles_n), band);
    return launch_status();
}


using Launch = int (*)(const int8_t *, int32_t, int32_t, GemvGroup, const Epilogue &, hipStream_t);

// The compiled tiles and what they cost.  Fitted to the time of every tile on 53 matrices (K 128 ..
// 29568, N 32 .. 59136, the 7B and 72B projections among them) at 24 row counts from 33 to 3072, one HIP
// graph over weights from HBM (rms 3 - 7 %): what the model picks, the tiles of w4a8_gemm.hip included, is within
// 0.2 % of the fastest on average.  The last four have a compute unit to themselves (128, 160, 84 and 96 KiB of
// stages) and three or four stages: where tiles fill about one round, a lone work-group with two stages waits for its
// copies (us before -> now: 8192 -> 10240 at T = 128 31.5 -> 24.4, 12288 -> 8192 at 192 42.0 -> 33.0, 4736 -> 27648 at 33
// 25.6 -> 19.7).  Fitted to 92 matrices (K 512 .. 29568, N 1024 .. 59136) at thirteen row counts from 33 to 1024.  Five
// stages are no better than four.
struct Variant {
    TileCost cost;
    Launch launch[3];
};
#define MQ_SLICED(MT, NWN, NB) \
    {launch_sliced<MT, NWN, NB, kEpiStatic>, launch_sliced<MT, NWN, NB, kEpiRowScale>, launch_sliced<MT, NWN, NB, kEpiSplit>}
constexpr Variant kSliced[] = {
    {{64, 128, 2, 2.920, 1.092, 0.377, 0.335, 0.087, 1.362}, MQ_SLICED(2, 4, 2)},
    {{64, 256, 2, 3.403, 0.905, 0.718, 0.450, 0.081, 1.910}, MQ_SLICED(2, 8, 3)},
    {{192, 128, 1, 1.706, 6.723, 0.510, 0.000, 0.161, 1.679}, MQ_SLICED(6, 4, 2)},
    {{160, 128, 1, 1.991, 5.559, 0.486, 0.000, 0.135, 1.566}, MQ_SLICED(5, 4, 2)},
    {{128, 128, 1, 1.346, 4.923, 0.331, 0.000, 0.139, 1.258}, MQ_SLICED(4, 4, 3)},
    {{96, 128, 2, 3.702, 1.215, 0.517, 0.402, 0.080, 1.960}, MQ_SLICED(3, 4, 2)},
    {{128, 64, 1, 1.619, 3.996, 0.257, 0.000, 0.100, 0.679}, MQ_SLICED(4, 2, 2)},
    {{64, 64, 1, 1.523, 2.534, 0.144, 0.000, 0.033, 0.705}, MQ_SLICED(2, 2, 3)},
    {{32, 64, 2, 1.976, 0.777, 0.165, 0.139, 0.043, 0.660}, MQ_SLICED(1, 2, 2)},
    {{32, 64, 1, 1.422, 1.727, 0.114, 0.000, 0.028, 0.592}, MQ_SLICED(1, 2, 3)},
    {{32, 32, 1, 1.222, 1.928, 0.064, 0.000, 0.019, 0.319}, MQ_SLICED(1, 1, 3)},
    {{64, 128, 1, 2.529, 2.208, 0.269, 0.000, 0.027, 1.510}, MQ_SLICED(2, 4, 4)},
    {{96, 128, 1, 2.426, 3.222, 0.303, 0.000, 0.062, 1.387}, MQ_SLICED(3, 4, 4)},
    {{96, 256, 1, 2.685, 4.119, 0.512, 0.000, 0.164, 1.415}, MQ_SLICED(3, 8, 3)},
    {{128, 256, 1, 2.507, 5.304, 0.602, 0.000, 0.230, 1.424}, MQ_SLICED(4, 8, 3)},
};
#undef MQ_SLICED
// What the estimates of the last four are multiplied by.  They hold within a few percent, while those of the 96 x 128 tile that
// shares a compute unit, of split-K and of the large tiles are up to 15 % above what these take by now, most of all over several
// rounds.  By the bare estimates a quarter of 5000 drawn shapes that went to the four (K 384 .. 29696, T 33 .. 8192) was 2 to 24 %
// slower (static 16640 -> 2624 at T = 3394 147 -> 165 us, 28288 -> 24456 at 213 172 -> 197, 1152 -> 16448 at 65 1.24 times),
// 0.941 of the time on average.  With these factors 0.930 and one in fifteen, mostly 128 x 256 against 64 x 256, which gain on
// one card (0.95 with each side in a run of its own) and lose on another (1.03 in turns).
//   up to 64 rows: 1.14.  There the four take up to 20 % longer than their fit, whose rows are mostly more (every weight is then
//     read by one tile, from HBM): all of the 16 shapes of the sweep that go to them gain 10 to 30 %, without it three lose 2
//     to 7 % (2048 -> 27648 at T = 64 11.3 -> 12.2).
//   against 96 x 128: 1.07 (between 0.92 and 0.95 of its estimate there is no shape; above, 1.00 to 1.19 of its time)
//   against the other sliced tiles: 1.02 (0.98 .. 1.0 of their estimates 1.01 of their time)
//   against the plan: 1.07 (at 0.88 .. 0.94 of its estimate 1.01 to 1.07 of its time); four stages of 64 x 128 1.04, with
//     flagged channels nothing (64-row tiles at 0.88 .. 0.90: 0.99 of their time, 0.94); against six pieces of K and more
//     nothing (0.95 to 0.99 there; 18944 -> 3584 at T = 577 .. 734 0.98)
constexpr int kOneRound = 11;             // the first of the tiles that have a compute unit to themselves
constexpr double kFewRows = 1.14, kAgainstSliced = 1.02, kAgainst96 = 1.07, kAgainstPlan = 1.07, kAgainstPlan64 = 1.04;
constexpr int kManyPieces = 6;
// The operands of flagged channels push two work-groups of 96 x 128 off a compute unit, and its estimate does not know: the
// four are then taken wherever their bare estimates are ahead of it (0.73 .. 0.95 of its time).
constexpr int kCrowded = 5;
static_assert(sliced_lds_bytes<3, 4, 2, kEpiStatic>() <= 80 * 1024 && sliced_lds_bytes<3, 4, 2, kEpiSplit>() > 80 * 1024, "kCrowded");
constexpr int kVariants = sizeof(kSliced) / sizeof(kSliced[0]);
static_assert(kSliced[kCrowded].cost.bm == 96 && kSliced[kCrowded].cost.per_cu == 2, "kCrowded");
static_assert(kVariants + 1 == kGemmShapes, "mquant_tune_set validates against this");

// Up to 32 rows, one row of tiles: the weights come from HBM and are what a launch waits for, so the
// 32-row tiles have costs of their own, the part along K growing by `slope` per 16 rows beyond 16.  Same
// sweep at 17 to 32 rows (rms 5 - 8 %).
struct ShortCost {
    int variant;
    TileCost cost;
    double slope;
};
constexpr ShortCost kShort[] = {
    {8, {32, 64, 2, 2.332, 0.472, 0.131, 0.156, 0.117, 1.017}, 0.052},
    {9, {32, 64, 1, 1.702, 1.376, 0.114, 0.000, 0.067, 1.172}, 0.070},
    {10, {32, 32, 1, 1.695, 1.493, 0.067, 0.000, 0.036, 0.979}, 0.128},
};
static_assert(kSliced[8].cost.bn == 64 && kSliced[9].cost.bn == 64 && kSliced[10].cost.bn == 32, "kShort names these");

struct Choice {
    int variant;
    double us;
};

// `splits`: pieces of K in the plan that the estimate will be compared with
Choice pick(int epi, int32_t T, int32_t K, const GemvGroup &grp, int32_t splits)
{
    auto tiles_n = [&](const TileCost &c) {
        int64_t tiles = 0;
        for (int32_t i = 0; i < grp.n; ++i) tiles += ceil_div32(grp.p[i].N, c.bn);
        return tiles;
    };
    Choice best = {-1, 0.0};
    auto consider = [&](int variant, double us) {
        if (best.variant < 0 || us < best.us) best = {variant, us};
    };
    if (T <= kGemvMaxT) {
        for (const ShortCost &s : kShort) {
            const int64_t tiles = tiles_n(s.cost);
            const double start = s.cost.us(tiles, 0), walk = s.cost.us(tiles, K) - start;
            consider(s.variant, start + walk * (1.0 + s.slope * (T - 16) * (1.0 / 16)));
        }
    } else {
        auto us_of = [&](int i) {
            const TileCost &c = kSliced[i].cost;
            return c.us(tiles_n(c) * ceil_div32(T, c.bm), K);
        };
        for (int i = 0; i < kOneRound; ++i) consider(i, us_of(i));
        double factor = T <= 64 ? kFewRows : best.variant == kCrowded ? kAgainst96 : kAgainstSliced;
        if (epi == kEpiSplit && best.variant == kCrowded) factor = 1.0;
        Choice alone = {-1, best.us / factor};
        for (int i = kOneRound; i < kVariants; ++i) {
            const double us = us_of(i);
            if (us < alone.us) alone = {i, us};
        }
        if (alone.variant >= 0) {
            const bool rows64 = alone.variant == kOneRound;
            const double plan = splits >= kManyPieces || (rows64 && epi == kEpiSplit) ? 1.0 : rows64 ? kAgainstPlan64 : kAgainstPlan;
            const double us = alone.us * (T <= 64 ? kFewRows : plan);
            best = {alone.variant, us < best.us ? us : best.us};
        }
    }
    return best;
}

}  // namespace

namespace mquant {

double sliced_cost_us(int epi, int32_t T, int32_t K, const GemvGroup &grp, int32_t splits) { return pick(epi, T, K, grp, splits).us; }

// From 33 rows on always.  Of 17 to 32 rows the GEMV keeps what the GEMM is not expected to do faster by
// 2 %, or at all where the weights take 10 us and more to read (GEMV against GEMM, weights from HBM, 24
// rows: 3584 -> 3584 5.6 / 6.8 us, 3584 -> 37888 20.1 / 21.6, 8192 -> 8192 9.7 / 11.1; 18944 -> 3584 18.2 / 17.4,
// 8192 -> 59136 51.4 / 49.1, 5120 -> 27648 21.7 / 18.6), and the smallest calls (128 -> 1024 3.0 / 3.3,
// 256 -> 4096 3.5 / 3.7).
bool gemm_takes(int32_t T, int32_t K, const GemvGroup &grp)
{
    if (K % 128 != 0 || T <= 16) return false;
    if (T > kGemvMaxT) return true;
    int64_t n_tiles = 0;
    for (int32_t i = 0; i < grp.n; ++i) n_tiles += ceil_div32(grp.p[i].N, kPackN);
    if (K <= 256 && n_tiles < kNumCU) return false;
    const double margin = n_tiles * K >= int64_t{1} << 22 ? 1.0 : 0.98;     // 64 MiB of weights
    return sliced_cost_us(kEpiStatic, T, K, grp, 1) < margin * gemv_tile_us(T, n_tiles, K);
}

template <int EPI>
int sliced_dispatch(const int8_t *xq, int32_t T, int32_t K, const GemvGroup &grp, const Epilogue &ep,
                    hipStream_t stream)
{
    int v = tune_state().gemm_sliced.load(std::memory_order_relaxed);
    if (v < 0) v = pick(EPI, T, K, grp, 1).variant;
    if (v == kVariants) {                    // forced: 256 x 384, or the largest tile here for what that does not take
        if constexpr (EPI != kEpiSplit)
            if (grp.n == 1) return launch_wide<EPI>(0, xq, T, K, grp.p[0], ep, stream);
        v = kVariants - 1;
    }
    return kSliced[v].launch[EPI](xq, T, K, grp, ep, stream);
}

template int sliced_dispatch<kEpiStatic>(const int8_t *, int32_t, int32_t, const GemvGroup &, const Epilogue &, hipStream_t);
template int sliced_dispatch<kEpiRowScale>(const int8_t *, int32_t, int32_t, const GemvGroup &, const Epilogue &, hipStream_t);
template int sliced_dispatch<kEpiSplit>(const int8_t *, int32_t, int32_t, const GemvGroup &, const Epilogue &, hipStream_t);

}  // namespace mquant
