// Causal attention on AIFS-ordered tokens and rotary embedding with reordered
// position ids, for gfx950 (MQuant, arXiv 2502.00425: Sec. 3.1, Eq. (5)-(6);
// appendix "Rotary Position Embedding for AIFS").
//
// After the AIFS reorder a token's row index no longer says what it may attend.
// Its original position does: token i attends token j exactly when
// pos[j] <= pos[i] (the unified mask M^u[i,j] = M[pos[i], pos[j]] of the causal
// M; for one visual segment this is the three-region rule of Eq. (6)).  The
// kernel never materialises a [T,T] mask: it compares positions per element on
// the tiles that need it, takes whole tiles unmasked or skips them by the
// min/max of their positions, flash-attention style (online softmax, fp32
// statistics, fp16 MFMA operands).
#include <hip/hip_fp16.h>

#include <climits>
#include <cmath>

#include "lds_dma.h"
#include "mquant_internal.h"

using namespace mquant;

namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int kHeadDim = 128;          // the only head size built (28 x 128, 64 x 128 in the paper's models)
constexpr int kBQ = 128;               // queries per work-group (32 per wave)
constexpr int kBK = 64;                // keys per tile
constexpr int kAhead = 4;               // LDS fragment reads in flight ahead of the MFMA that uses them
constexpr int kTileBytes = kBK * 2 * kHeadDim;   // a key or value tile in LDS: 64 rows of 256 bytes
constexpr int kGroupLds = 4 * kTileBytes;        // two key and two value buffers of one key group
constexpr int kChunkTiles = 64;                  // tiles whose visibility a wave holds as bit masks, one lane each

// Tiles arrive by LDS-DMA (1 KiB per wave instruction, lane i at offset 16 i), so rows cannot
// be padded; instead the 16-byte chunks of a row (256 bytes, the full bank space) are XOR-swizzled, on
// the global side of the copy.  A key fragment is one chunk of 16 consecutive rows at a time: chunk c of
// row r sits at r * 256 + ((c ^ (r & 15)) << 4).  A value fragment is read transposed
// (ds_read_b64_tr_b16), 32 lanes covering four rows x 64 bytes: chunk c of row r sits at
// r * 256 + ((c ^ ((r & 3) << 2)) << 4).  Both cover the 64 banks exactly once.

// V^T tiles (vt_kernel) are 128 rows of 128 bytes: chunk c of row d sits at d * 128 + ((c ^ ((d >> 1) & 7)) << 4).
// Key order inside the V^T rows: the P V product takes its key index from the score registers
// (operand slot i of lane group g is key 16 kk + 8 (i / 4) + 4 g + i % 4), so the transpose
// stores every 16 keys as 0-3, 8-11, 4-7, 12-15 and an operand is one aligned 16-byte chunk.
__device__ __forceinline__ int vt_key_of_slot(int p)
{
    const int x = p & 15;
    return (p & ~15) | (x < 4 ? x : (x < 8 ? x + 4 : (x < 12 ? x - 4 : x)));
}

// The value of the partner lane (lane ^ 32) next to this lane's own: v_permlane32_swap on two
// copies leaves {low half, low half} and {high half, high half}; no LDS traffic, so fragment
// reads that are in flight are not waited for.
__device__ __forceinline__ void halves_of(float x, float &lo, float &hi)
{
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
    lo = __int_as_float(sw[0]);
    hi = __int_as_float(sw[1]);
}

// MFMA 32x32 result register r of lane group g holds row (r/4)*8 + g*4 + r%4.
__device__ __forceinline__ int acc_row(int r, int g) { return (r >> 2) * 8 + g * 4 + (r & 3); }

// ------------------------------------------------------------------- RoPE
//
// x'[2j] = x[2j] cos - x[2j+1] sin, x'[2j+1] = x[2j] sin + x[2j+1] cos with the
// angle pos[i] * theta_j, theta_j = base^(-2j/D): the block-diagonal rotation
// printed in the appendix, with the token's ORIGINAL position as its id.  The
// angle and its sine/cosine are formed in double (a position of 16384 leaves an
// fp32 angle accurate to 1e-3 only); one thread per (token, pair) serves all heads.
struct InvFreq {
    double f[kHeadDim / 2];
};

__global__ __launch_bounds__(256) void rope_kernel(__half *__restrict__ x, int64_t ldx,
                                                   const int32_t *__restrict__ pos, int32_t T,
                                                   int32_t n_heads, InvFreq inv)
{
    constexpr int P = kHeadDim / 2;
    const int64_t total = static_cast<int64_t>(T) * P;
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; e < total;
         e += static_cast<int64_t>(gridDim.x) * 256) {
        const int32_t i = static_cast<int32_t>(e / P);
        const int32_t j = static_cast<int32_t>(e - static_cast<int64_t>(i) * P);
        double sn, cs;
        sincos(static_cast<double>(pos[i]) * inv.f[j], &sn, &cs);
        const float c = static_cast<float>(cs), s = static_cast<float>(sn);
        __half2 *row = reinterpret_cast<__half2 *>(x + static_cast<int64_t>(i) * ldx) + j;
        for (int32_t h = 0; h < n_heads; ++h) {
            const float2 v = __half22float2(row[h * P]);
            row[h * P] = __floats2half2_rn(v.x * c - v.y * s, v.x * s + v.y * c);
        }
    }
}

// The same rotation with 16-byte accesses (x and its rows 16-byte aligned).  A wave takes one
// token and up to kRopeChunks * 4 of its heads: lane l forms the angle of pair l once, a lane then
// rotates the same four pairs (l % 16) * 4 .. + 3 in every chunk it touches, so its sines and
// cosines stay in registers.  The loads are issued before the double-precision sincos, whose latency
// is what a wave waits for: T = 1280, 32 heads (10.5 MB each way) 14.2 -> 5.6 us, 16384 tokens of 72 heads at 6.2 TB/s; a thread that
// walked all heads of one pair had one 4-byte load in flight.
constexpr int kRopeChunks = 8;             // 16-byte chunks a lane holds
__global__ __launch_bounds__(256) void rope_wide_kernel(__half *__restrict__ x, int64_t ldx,
                                                        const int32_t *__restrict__ pos, int32_t T,
                                                        int32_t n_heads, InvFreq inv)
{
    constexpr int P = kHeadDim / 2;
    static_assert(P == 64, "a lane per pair");
    const int lane = threadIdx.x & 63;
    const int32_t chunks = n_heads * (kHeadDim / 8), c0 = blockIdx.y * (64 * kRopeChunks) + lane;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6); i < T;
         i += static_cast<int64_t>(gridDim.x) * 4) {
        v8h *row = reinterpret_cast<v8h *>(x + i * ldx);
        v8h v[kRopeChunks];
#pragma unroll
        for (int u = 0; u < kRopeChunks; ++u)
            if (c0 + u * 64 < chunks) v[u] = row[c0 + u * 64];
        double sn, cs;
        sincos(static_cast<double>(pos[i]) * inv.f[lane], &sn, &cs);
        float c[4], s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            c[e] = __shfl(static_cast<float>(cs), (lane & 15) * 4 + e, 64);
            s[e] = __shfl(static_cast<float>(sn), (lane & 15) * 4 + e, 64);
        }
#pragma unroll
        for (int u = 0; u < kRopeChunks; ++u)
            if (c0 + u * 64 < chunks) {
                v8h r;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a = static_cast<float>(v[u][2 * e]), b = static_cast<float>(v[u][2 * e + 1]);
                    r[2 * e] = static_cast<_Float16>(a * c[e] - b * s[e]);
                    r[2 * e + 1] = static_cast<_Float16>(a * s[e] + b * c[e]);
                }
                row[c0 + u * 64] = r;
            }
    }
}

// -------------------------------------------------------- V^T and tile bounds
//
// The P V product wants, per head channel, the eight keys of an MFMA operand in one
// 16-byte chunk, so V goes through a one-off transpose V[T][Hkv*D] -> Vt[Hkv*D][Tp]
// (Tp = T rounded up to the key tile, tail zeroed: a zero probability times an
// uninitialised value could be NaN; keys inside a row in the order of vt_key_of_slot).
// The same launch records min and max position of every key tile.
__global__ __launch_bounds__(256) void vt_kernel(const __half *__restrict__ v, int64_t ldv,
                                                 __half *__restrict__ vt, int32_t T, int32_t Tp,
                                                 int32_t channels, const int32_t *__restrict__ pos,
                                                 int32_t *__restrict__ tile_min,
                                                 int32_t *__restrict__ tile_max)
{
    // 64 tokens x 64 channels per group; 16-byte accesses on both sides (channels is a
    // multiple of 64 here: whole heads of 128).
    __shared__ __attribute__((aligned(16))) __half tile[64][72];
    const int32_t t0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
    const int r8 = threadIdx.x >> 3, c8 = (threadIdx.x & 7) * 8;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int r = half * 32 + r8;
        const int32_t t = t0 + r;
        uint4 val = make_uint4(0u, 0u, 0u, 0u);
        if (t < T) val = *reinterpret_cast<const uint4 *>(v + static_cast<int64_t>(t) * ldv + c0 + c8);
        *reinterpret_cast<uint4 *>(&tile[r][c8]) = val;
    }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int c = half * 32 + r8;                       // channel row of the transposed tile
        __half out[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = tile[vt_key_of_slot(c8 + i)][c];
        *reinterpret_cast<uint4 *>(vt + static_cast<int64_t>(c0 + c) * Tp + t0 + c8) =
            *reinterpret_cast<const uint4 *>(out);
    }
    if (blockIdx.y == 0 && threadIdx.x < 64) {
        const int32_t t = t0 + threadIdx.x;
        int32_t lo = t < T ? pos[t] : INT_MAX, hi = t < T ? pos[t] : INT_MIN;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            lo = min(lo, __shfl_xor(lo, m, 64));
            hi = max(hi, __shfl_xor(hi, m, 64));
        }
        if (threadIdx.x == 0) {
            tile_min[blockIdx.x] = lo;
            tile_max[blockIdx.x] = hi;
        }
    }
}

// -------------------------------------------------------------- attention
//
// One work-group: 128 queries of one query head, KG key groups of four waves of 32 queries; key
// group kg takes every KG-th of the key tiles the work-group needs, and the groups' partial results meet in
// LDS at the end.  V comes as it is (VT = false, at most 64 key tiles) or transposed by vt_kernel.
// Per key tile (64 keys, shared by the four waves through LDS):
//   S^T = K Q^T     A = K rows (keys) from LDS, B = Q^T held in registers for the whole
//                   kernel; in the result a LANE is a query, its registers are keys, so
//                   the softmax statistics of a query live in one lane pair
//   P^T             the same registers, as fp16, are the B operand of
//   O^T += V^T P^T  A = V^T: rows (head channels) of the transposed tile, or read out of the row-major
//                   one by the transposing LDS read (four keys of a lane's channel); the result again
//                   has a lane per query, so the running rescale needs no cross-lane traffic.
// Software pipeline, one tile deep inside a wave: while the exponentials of tile j run on
// the vector ALU, the matrix core computes the scores of tile j+1 (a second score register
// set; the two instruction streams are written interleaved and pinned), so of the three
// parts of a tile -- scores, softmax, P V -- only two are paid in sequence.  Key tiles are
// therefore fetched one step ahead of value tiles.  Tiles travel global -> LDS by LDS-DMA
// (no staging registers), two buffers each for K and V, one barrier per tile.
// Tiles whose smallest position exceeds the group's largest query position are skipped
// altogether (no loads); a wave skips the arithmetic of a tile that is masked for all of its
// 32 queries and drops the per-element compare on tiles that are visible to all of them.  Which
// tiles those are is three 64-bit masks per 64 tiles, so that walking them takes scalar arithmetic only
// (a scalar load per tile for its bounds, in flight across the step, turned the waits for single fragments
// into waits for everything).
// What bounds it: at T = 8192 (28 heads on 4, 514 -> 485 us with the masks, flags and pipeline below) matrix and
// vector pipes, each busy half of the time at a clock that power holds at 1.8 GHz; at T = 1280 (39.8 -> 27.8 us) the
// longest work-group (20 key tiles: 2.1 us for two tiles of two key groups, of which the matrix products are 1.0)
// and 8 us that launch, prologue and epilogue take at any T.  Measured without gain: the two key groups half a
// step apart, so that the P V product of one runs under the exponentials of the other (T = 1280 28.5 -> 30.5 us: a
// second barrier per step costs more); the first tile requested before the positions have arrived (28.5 ->
// 29.5); the maximum of the next tile's scores taken under the P V product (T = 8192 +0.7 %); a raised wave priority
// around either product (-1 .. +1 %).
typedef __fp16 tr4 __attribute__((vector_size(8)));
typedef tr4 __attribute__((address_space(3))) *tr4_lds_ptr;

template <int KG, bool VT>
__global__ __launch_bounds__(KG * 256, 2) void aifs_attention_kernel(
    const __half *__restrict__ q, int64_t ldq, const __half *__restrict__ k, int64_t ldk,
    const __half *__restrict__ v, int64_t ldv, __half *__restrict__ o, int64_t ldo,
    const int32_t *__restrict__ pos, const int32_t *__restrict__ tile_min,
    const int32_t *__restrict__ tile_max, int32_t T, int32_t group, int32_t n_kv_heads, int32_t n_qblocks,
    int32_t xcds_per_kv, float scale_log2e)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];       // KG * kGroupLds
    __shared__ int32_t pos_lds2[KG][2][kBK];
    __shared__ int32_t bound_lds[2][kChunkTiles];
    __shared__ int32_t wg_qmax_lds[4];
    static_assert(kHeadDim == 128 && kBK == 64, "addressing below");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3), kg = KG > 1 ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0;
    const int tid_g = tid & 255;                           // thread of its key group
    const int l32 = lane & 31, g = lane >> 5;
    // Work-group ids are dealt round-robin to the 8 XCDs, each with its own L2.  When the
    // key/value heads divide the XCDs evenly (xcds_per_kv > 0), an XCD serves ONE key/value
    // head: its resident work-groups then walk the same key tiles at about the same time and
    // the L2 fetches each tile once for all of them (with heads simply dealt in order every
    // XCD streams all key/value heads and two thirds of the tile requests hit).  Query blocks
    // go from the last to the first: in AIFS order the later blocks of each modality see the
    // most keys, so the long work-groups start first and the short ones fill the end.
    const int32_t n_heads = group * n_kv_heads;
    int32_t head, qblock;
    if (xcds_per_kv > 0) {
        const int32_t xcd = blockIdx.x % 8, n = blockIdx.x / 8;
        const int32_t m = n * xcds_per_kv + xcd % xcds_per_kv;      // item of this key/value head
        if (m >= n_qblocks * group) return;                         // uniform: whole work-group
        head = (xcd / xcds_per_kv) * group + m % group;
        qblock = n_qblocks - 1 - m / group;
    } else {
        head = blockIdx.x % n_heads;
        qblock = n_qblocks - 1 - blockIdx.x / n_heads;
    }
    const int32_t kvh = head / group;
    const int32_t q0 = qblock * kBQ + wave * 32;
    const int32_t n_tiles = (T + kBK - 1) / kBK;

    // ---- tile copies: 16 blocks of 1 KiB per tile, four per wave.  A copy instruction takes a
    // wave-uniform base (scalar registers) and a 32-bit offset per lane.
    const uint8_t *kbase = reinterpret_cast<const uint8_t *>(k + kvh * kHeadDim);
    const uint8_t *vbase = reinterpret_cast<const uint8_t *>(v + kvh * kHeadDim * (VT ? ldv : 1));
    const uint32_t lds0 = lds_address(smem) + kg * kGroupLds;
    const int32_t c_row = wave * 4 + (lane >> 4);          // row of this lane in block 0 (block i: + 16 i)
    const uint32_t k_chunk = static_cast<uint32_t>(((lane & 15) ^ (c_row & 15)) << 4);
    const uint32_t v_chunk = static_cast<uint32_t>(((lane & 15) ^ ((c_row & 3) << 2)) << 4);
    const uint32_t k_pitch = static_cast<uint32_t>(ldk) * 2u, v_pitch = static_cast<uint32_t>(ldv) * 2u;
    // rows past T repeat the last row (their probabilities are masked to zero; values: zero_tail)
    auto dma_k = [&](int32_t t, int b) {
        const uint8_t *tile = kbase + static_cast<int64_t>(t) * kBK * ldk * 2;
        const int32_t last = T - 1 - t * kBK;              // last valid row of this tile
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int32_t row = c_row + 16 * i;
            row = row < last ? row : last;
            lds_dma16_uniform_base(tile, static_cast<uint32_t>(row) * k_pitch + k_chunk,
                                   lds0 + b * kTileBytes + (i * 4 + wave) * 1024);
        }
    };
    const int32_t vt_d = wave * 8 + (lane >> 3);           // V^T: head channel of this lane in block 0 (block i: + 32 i)
    const uint32_t vt_lane = static_cast<uint32_t>(vt_d) * v_pitch + static_cast<uint32_t>(((lane & 7) ^ ((vt_d >> 1) & 7)) << 4);
    auto dma_v = [&](int32_t t, int b) {
        if constexpr (VT) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                lds_dma16_uniform_base(vbase + (static_cast<int64_t>(i) * 32 * ldv + static_cast<int64_t>(t) * kBK) * 2, vt_lane,
                                       lds0 + (2 + b) * kTileBytes + (i * 4 + wave) * 1024);
            return;
        }
        const uint8_t *tile = vbase + static_cast<int64_t>(t) * kBK * ldv * 2;
        const int32_t last = T - 1 - t * kBK;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int32_t row = c_row + 16 * i;
            row = row < last ? row : last;
            lds_dma16_uniform_base(tile, static_cast<uint32_t>(row) * v_pitch + v_chunk,
                                   lds0 + (2 + b) * kTileBytes + (i * 4 + wave) * 1024);
        }
    };

    // Value rows past T become zeros once the copies of the last tile have landed (every lane those it copied): a zero
    // probability times what the last row holds is a NaN where that is infinite.  V^T has its zeros from vt_kernel.
    typedef v4u __attribute__((address_space(3))) *v4u_lds_ptr;
    const int32_t ragged = !VT && T % kBK != 0 ? n_tiles - 1 : -1;      // the tile that holds the end of the sequence
    auto zero_tail = [&](int32_t t, int b) {
        if (t != ragged) return;
        uint32_t at = lds0 + (2 + b) * kTileBytes + wave * 1024 + lane * 16;
        int32_t row = t * kBK + c_row;
        asm volatile("" : "+v"(at), "+v"(row) : : "memory");   // behind the wait for the copies; made here, not kept
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (row + 16 * i >= T) *(v4u_lds_ptr)(uintptr_t)(at + i * 4096) = v4u{0, 0, 0, 0};
    };

    // ---- this lane's query: position and Q^T fragments
    const int32_t qi = q0 + l32;
    const int32_t qrow = qi < T ? qi : T - 1;
    const int32_t my_pos = pos[qrow];
    // Tile bounds of a short sequence: every thread folds consecutive positions, the threads of a
    // tile meet by lane exchange.
    constexpr bool own_bounds = !VT;
    constexpr int PER = kChunkTiles * kBK / (KG * 256);     // positions of a thread
    constexpr int LPT = kBK / PER;                         // lanes that share a tile
    int32_t b_lo = INT_MAX, b_hi = INT_MIN;
    if (own_bounds && tid * PER < T) {                     // tid * PER >= T: beyond the sequence
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int32_t t = tid * PER + i;
            const int32_t p = pos[t < T ? t : T - 1];
            b_lo = t < T && p < b_lo ? p : b_lo;
            b_hi = t < T && p > b_hi ? p : b_hi;
        }
    }
    v8h qf[kHeadDim / 16];
    {
        const __half *qp = q + static_cast<int64_t>(qrow) * ldq + head * kHeadDim + g * 8;
#pragma unroll
        for (int ks = 0; ks < kHeadDim / 16; ++ks)
            qf[ks] = *reinterpret_cast<const v8h *>(qp + ks * 16);
    }
    int32_t qmin = my_pos, qmax = my_pos;
#pragma unroll
    for (int m = 16; m >= 1; m >>= 1) {                    // lanes 32.. hold the same queries
        qmin = min(qmin, __shfl_xor(qmin, m, 64));
        qmax = max(qmax, __shfl_xor(qmax, m, 64));
    }
    qmin = __builtin_amdgcn_readfirstlane(qmin);
    qmax = __builtin_amdgcn_readfirstlane(qmax);
    if (kg == 0 && lane == 0) wg_qmax_lds[wave] = qmax;
    if (own_bounds) {
#pragma unroll
        for (int m = LPT / 2; m >= 1; m >>= 1) {
            b_lo = min(b_lo, __shfl_xor(b_lo, m, 64));
            b_hi = max(b_hi, __shfl_xor(b_hi, m, 64));
        }
        if (tid % LPT == 0) {
            bound_lds[0][tid / LPT] = b_lo;
            bound_lds[1][tid / LPT] = b_hi;
        }
    }
    __syncthreads();
    const int32_t wg_qmax = __builtin_amdgcn_readfirstlane(
        max(max(wg_qmax_lds[0], wg_qmax_lds[1]), max(wg_qmax_lds[2], wg_qmax_lds[3])));

    // ---- the tiles to walk.  Masks of 64 tiles: needed by the work-group and not yet taken, needed by
    // this wave, visible as a whole to this wave.
    uint64_t left, needed, whole;
    int32_t base = 0;                                      // first tile of the masks
    auto load_masks = [&]() {
        const int32_t t = base + lane;
        const bool in = t < n_tiles;
        int32_t lo = INT_MAX, hi = INT_MAX;
        if (own_bounds) {
            lo = bound_lds[0][lane];
            hi = bound_lds[1][lane];
        } else if (in) {
            lo = tile_min[t];
            hi = tile_max[t];
            wait_vmcnt<0>();                               // here, not wherever their registers are used next
        }
        left = __ballot(in && lo <= wg_qmax);
        needed = __ballot(in && lo <= qmax);
        whole = __ballot(in && hi <= qmin && (t + 1) * kBK <= T);   // a tile with keys past the end is never whole
    };
    // Takes `n` tiles off the front; the last of them (n_tiles: none), whether this wave needs it,
    // whether all its keys are visible to the wave.
    const int32_t end = n_tiles * 4;
    auto take = [&](int n) -> int32_t {
        int bit = 0;
        for (int i = 0; i < n; ++i) {
            while (left == 0) {
                if (!VT || base + kChunkTiles >= n_tiles) return end;
                base += kChunkTiles;
                load_masks();
            }
            bit = __builtin_ctzll(left);
            left &= left - 1;
        }
        return (base + bit) * 4 + (static_cast<int32_t>(whole >> bit) & 1) * 2 + (static_cast<int32_t>(needed >> bit) & 1);
    };
    load_masks();

    v16f acc_o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[dt][r] = 0.0f;

    auto key_pos = [&](int32_t t) -> int32_t {             // threads 0..63 of a key group: position of key tid_g of tile t
        const int32_t key = t * kBK + (tid_g & 63);
        return key < T ? pos[key] : INT_MAX;
    };
    // LDS fragments: MFMA i of the score product is (ks, kb) = (i / 2, i % 2), of the P V
    // product (kk, dt) = (i / 4, i % 4); consecutive MFMAs write different accumulators.
    // Operand slot s of lane group g of the P V product is the key that score register s holds there:
    // 16 kk + 8 (s / 4) + 4 g + s % 4, two transposing reads of four keys.  Such a read takes, per 16
    // lanes, the four rows' 32 bytes that lanes 4 r .. 4 r + 3 point at and gives lane i the four rows' channel i.
    const int kswz = l32 & 15;
    const int tr_row = (lane >> 2) & 3;
    const uint32_t v_lane = g * 1024 + tr_row * 256 + (tr_row << 6) + (((lane >> 4) & 1) * 2 + ((lane >> 1) & 1)) * 16 + (lane & 1) * 8;
    typedef const v8h __attribute__((address_space(3))) *v8h_lds_ptr;
    uint32_t k_at[8], v_at[4];
    for (int i = 0; i < 8; ++i) {
        k_at[i] = lds0 + l32 * 256 + (((i * 2 + g) ^ kswz) << 4);
        asm volatile("" : "+v"(k_at[i]));
    }
    auto kfrag = [&](uint32_t kb_lds, int i) {
        return *(v8h_lds_ptr)(uintptr_t)(k_at[i >> 1] + kb_lds + (i & 1) * 8192);
    };
    const int vswz = (l32 >> 1) & 7;
    for (int i = 0; i < 4; ++i) {
        v_at[i] = lds0 + (VT ? l32 * 128 + (((i * 2 + g) ^ vswz) << 4) : v_lane ^ (i << 6));
        asm volatile("" : "+v"(v_at[i]));
    }
    auto vfrag = [&](uint32_t vb_lds, int i) {
        if constexpr (VT) return *(v8h_lds_ptr)(uintptr_t)(v_at[i >> 2] + vb_lds + (i & 3) * 4096);
        const uint32_t f = v_at[i & 3] + vb_lds + (i >> 2) * 4096;
        union {
            tr4 h[2];
            v8h f8;
        } u;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4f16((tr4_lds_ptr)(uintptr_t)f);
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4f16((tr4_lds_ptr)(uintptr_t)(f + 2048));
        return u.f8;
    };
    const v16f zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // scores of one tile on their own (first tile; tiles whose predecessor this wave skips)
    auto scores = [&](uint32_t kb_lds, v16f (&s)[2]) {
        v8h fr[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) fr[i] = kfrag(kb_lds, i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * (kHeadDim / 16); ++i) {
            s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[i % kAhead], qf[i >> 1], i < 2 ? zero16 : s[i & 1], 0, 0, 0);
            if (i + kAhead < 2 * (kHeadDim / 16)) fr[i % kAhead] = kfrag(kb_lds, i + kAhead);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Running statistics in raw-logit units; the exponent is exp2((s - m_ref) * c) as one
    // fused multiply-add per element.  m_ref is the reference maximum the accumulators are
    // scaled to; it follows the true maximum lazily: only when some query's maximum has grown
    // by more than kLazy (a factor 2^kLazy in the probabilities, harmless in fp16 and fp32)
    // are the accumulators rescaled, so most tiles skip the 64 multiplies and the exponential.
    constexpr float kLazy = 8.0f;
    const float lazy_raw = kLazy / scale_log2e;
    float m_ref = -INFINITY, l_run = 0.0f;

    // Keys past the end have position INT_MAX, which hides them from all queries but those that are there themselves: from
    // these by their index, in the tile `top` (-1: not this wave's concern).
    const int32_t top = T % kBK != 0 && __any(my_pos == INT_MAX) ? n_tiles - 1 : -1;

    // One step of the pipeline: softmax and P V of tile `cur` (scores in s_cur, values in V
    // buffer par, positions in pos buffer par) while the scores of tile `nxt` (keys in K
    // buffer par ^ 1) go to s_nxt.  On entry a barrier has published those buffers and freed
    // K buffer par (its scores are done) and V buffer par ^ 1 (its P V product is done).
    int32_t cur, nxt;
    auto step = [&](v16f (&s_cur)[2], v16f (&s_nxt)[2], const int par) {
        const int32_t nn = take(KG);
        if (nn < end) dma_k(nn >> 2, par);
        if (nxt < end) dma_v(nxt >> 2, par ^ 1);
        int32_t preg = INT_MAX;
        if (tid_g < kBK && nxt < end) preg = key_pos(nxt >> 2);
        // Flags held in vector registers: as wave-uniform branches the three ways to the next tile's scores
        // were merged by copying them, 64 registers every other tile (T = 8192 538 -> 504 us without; a scalar branch
        // around the body of need_cur alone spills more than 500 registers).  The branches below therefore narrow EXEC, which
        // the matrix instructions do not look at: a wave that skips a tile is kept from accumulating into
        // acc_o by the jump over the empty body, which the compiler keeps for bodies of this size with LDS reads in them.
        // tests/test_attention_branches.py holds it to that; waves that skip what others of the work-group need run
        // in test_attention_routes and test_attention_every_key_tile_is_visible_on_the_config_layouts.
        int32_t f_cur = cur & 3, f_nxt = nxt & 1;
        asm("" : "+v"(f_cur), "+v"(f_nxt));
        const bool need_cur = (f_cur & 1) != 0, need_nxt = f_nxt != 0;
        const uint32_t kb_lds = (par ^ 1) * kTileBytes, vb_lds = (2 + par) * kTileBytes;
        const int32_t *pos_lds = pos_lds2[kg][par];
        if (need_cur) {                                    // else: masked for all 32 queries of the wave
            // ---- mask, online softmax
            if ((f_cur & 2) == 0) {                                  // wave-uniform: some (query, key) pair is hidden
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (pos_lds[kb * 32 + acc_row(r, g)] > my_pos) s_cur[kb][r] = -INFINITY;
                if ((cur >> 2) == top) {
                    int32_t keys = T % kBK - 4 * g;                      // of this lane's registers, in acc_row(r, 0)
                    asm volatile("" : "+v"(keys));                       // computed here, not kept across the loop
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (kb * 32 + acc_row(r, 0) >= keys) s_cur[kb][r] = -INFINITY;
                }
            }
            float m_new = m_ref;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) m_new = fmaxf(m_new, s_cur[kb][r]);
            {
                float lo, hi;
                halves_of(m_new, lo, hi);                        // the query's other 32 keys
                m_new = fmaxf(lo, hi);
            }
            if (__any(m_new > m_ref + lazy_raw)) {         // also the first visible tile (m_ref = -inf)
                const float m_use = m_new == -INFINITY ? 0.0f : m_new;
                const float alpha = __builtin_amdgcn_exp2f((m_ref - m_use) * scale_log2e);   // exp2(-inf) = 0
                l_run *= alpha;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc_o[dt][r] *= alpha;
                m_ref = m_new;
            }
            const float neg = m_ref == -INFINITY ? 0.0f : -m_ref * scale_log2e;
            float l_add = 0.0f;
            v8h p[4];
            // The two branches below take the offset from different registers (`neg_alone` is
            // a copy the compiler cannot see through): written alike, the compiler merges the
            // exponentials of both and hoists them in front of the branch, out from between
            // the MFMAs of the interleaved one.
            float neg_alone = neg;
            asm volatile("" : "+v"(neg_alone));
            auto exp_pair = [&](int e, float off) {        // elements 2e, 2e+1 of the 32 scores of a lane
                const int kb = e >> 3, r = (e & 7) * 2;
                const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[kb][r], scale_log2e, off));
                const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[kb][r + 1], scale_log2e, off));
                // the denominator sums the probabilities as the P V product sees them (rounded
                // to fp16): one dot-product instruction per pair instead of two additions
                v2h ph;
                ph[0] = static_cast<_Float16>(e0);
                ph[1] = static_cast<_Float16>(e1);
                l_add = __builtin_amdgcn_fdot2(ph, v2h{1, 1}, l_add, false);
                p[kb * 2 + (r >> 3)][r & 7] = ph[0];
                p[kb * 2 + (r >> 3)][(r & 7) + 1] = ph[1];
            };
            v8h fr[kAhead];
            if (need_nxt) {
                // exponentials of this tile interleaved with the score MFMAs of the next one: one MFMA, its
                // fragment read, two exponentials per group, order pinned.  The exponentials are a
                // pipeline of their own (multiply-add of pair i + 2, exponentials of pair i + 1, conversion of pair
                // i: no instruction waits for the one before it; T = 8192 500 -> 490 us).
#pragma unroll
                for (int i = 0; i < kAhead; ++i) fr[i] = kfrag(kb_lds, i);
                __builtin_amdgcn_sched_barrier(0);
                float x[2][2], y[2][2];
                float l_two[2] = {0.0f, 0.0f};
                auto arg = [&](int e) {
                    x[e & 1][0] = __builtin_fmaf(s_cur[e >> 3][(e & 7) * 2], scale_log2e, neg);
                    x[e & 1][1] = __builtin_fmaf(s_cur[e >> 3][(e & 7) * 2 + 1], scale_log2e, neg);
                };
                auto ex = [&](int e) {
                    y[e & 1][0] = __builtin_amdgcn_exp2f(x[e & 1][0]);
                    y[e & 1][1] = __builtin_amdgcn_exp2f(x[e & 1][1]);
                };
                arg(0);
                ex(0);
                arg(1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    s_nxt[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[i % kAhead], qf[i >> 1],
                                                                          i < 2 ? zero16 : s_nxt[i & 1], 0, 0, 0);
                    if (i + kAhead < 16) fr[i % kAhead] = kfrag(kb_lds, i + kAhead);
                    if (i + 1 < 16) ex(i + 1);
                    v2h ph;
                    ph[0] = static_cast<_Float16>(y[i & 1][0]);
                    ph[1] = static_cast<_Float16>(y[i & 1][1]);
                    p[(i >> 3) * 2 + ((i & 7) >> 2)][(i & 3) * 2] = ph[0];
                    p[(i >> 3) * 2 + ((i & 7) >> 2)][(i & 3) * 2 + 1] = ph[1];
                    if (i + 2 < 16) arg(i + 2);
                    l_two[i & 1] = __builtin_amdgcn_fdot2(ph, v2h{1, 1}, l_two[i & 1], false);
                    __builtin_amdgcn_sched_barrier(0);
                }
                l_add = l_two[0] + l_two[1];
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) exp_pair(i, neg_alone);
            }
            // the first V fragments travel while the sums are exchanged
#pragma unroll
            for (int i = 0; i < kAhead; ++i) fr[i] = vfrag(vb_lds, i);
            __builtin_amdgcn_sched_barrier(0);
            {
                float lo, hi;
                halves_of(l_add, lo, hi);
                l_add = lo + hi;
            }
            l_run += l_add;
            // ---- O^T += V^T P^T (the four channel blocks alternate; same rotating window)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc_o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[i % kAhead], p[i >> 2], acc_o[i & 3], 0, 0, 0);
                if (i + kAhead < 16) fr[i % kAhead] = vfrag(vb_lds, i + kAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if (need_nxt) {
            scores(kb_lds, s_nxt);
        }
        if (tid_g < kBK) pos_lds2[kg][par ^ 1][tid_g] = preg;
        wait_vmcnt<0>();                                   // K of nn and V of nxt have landed
        if constexpr (!VT) zero_tail(nxt >> 2, par ^ 1);
        __syncthreads();
        cur = nxt;
        nxt = nn;
    };

    // ---- prologue: first tile's keys, values and positions, second tile's keys.  With two key
    // groups the sequence has at most 64 tiles and the first group's share, the larger one, counts the steps.
    static_assert(KG == 1 || KG == 2, "steps");
    int32_t steps = KG == 1 ? 0 : (__builtin_popcountll(left) + KG - 1) / KG;
    cur = take(kg + 1);                                    // group 0: exists, every token sees itself
    nxt = cur < end ? take(KG) : end;
    if (cur < end) {
        dma_k(cur >> 2, 0);
        dma_v(cur >> 2, 0);
        if (nxt < end) dma_k(nxt >> 2, 1);
        if (tid_g < kBK) pos_lds2[kg][0][tid_g] = key_pos(cur >> 2);
    }
    wait_vmcnt<0>();
    if constexpr (!VT) zero_tail(cur >> 2, 0);
    __syncthreads();
    v16f s_a[2], s_b[2];
    if ((cur & 1) != 0) scores(0, s_a);
    __syncthreads();                                       // K buffer 0 is free for the third tile
    while (KG == 1 ? cur < end : steps > 0) {
        step(s_a, s_b, 0);
        if (KG == 1 ? cur >= end : --steps == 0) break;
        step(s_b, s_a, 1);
        --steps;
    }

    // ---- normalise and store: lane = query, registers = head channels (4 consecutive per group)
    __half *orow = o + static_cast<int64_t>(qi) * ldo + head * kHeadDim;
    auto store4 = [&](int dt, int r4, const float (&f)[4]) {
        __half h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = __float2half_rn(f[e]);
        *reinterpret_cast<uint2 *>(orow + dt * 32 + r4 * 8 + g * 4) = *reinterpret_cast<const uint2 *>(h);
    };
    if constexpr (KG == 1) {
        if (qi < T) {
            const float inv_l = 1.0f / l_run;              // every token sees at least itself
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    float f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = acc_o[dt][r4 * 4 + e] * inv_l;
                    store4(dt, r4, f);
                }
        }
    } else {
        // The two key groups of a query exchange halves of the channels: group kg finishes channels
        // 64 kg .. 64 kg + 63.  The last barrier of the loop has freed the tile buffers.
        float *xch = reinterpret_cast<float *>(smem);      // [8 waves][34][64]
        float *mine = xch + (kg * 4 + wave) * (34 * 64) + lane;
        const float *theirs = xch + ((kg ^ 1) * 4 + wave) * (34 * 64) + lane;
        auto give = [&](const v16f &a, const v16f &b) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                mine[r * 64] = a[r];
                mine[(16 + r) * 64] = b[r];
            }
        };
        if (kg == 0) give(acc_o[2], acc_o[3]);
        else give(acc_o[0], acc_o[1]);
        mine[32 * 64] = m_ref;
        mine[33 * 64] = l_run;
        __syncthreads();
        const float m_o = theirs[32 * 64], l_o = theirs[33 * 64];
        const float m = fmaxf(m_ref, m_o);                 // finite: one of the groups has the token itself
        const float a = m_ref == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_ref - m) * scale_log2e);
        const float b = m_o == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_o - m) * scale_log2e);
        const float inv_l = 1.0f / (l_run * a + l_o * b);
        auto finish = [&](int dt, const v16f &acc, const float *other) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = (acc[r4 * 4 + e] * a + other[(r4 * 4 + e) * 64] * b) * inv_l;
                store4(dt, r4, f);
            }
        };
        if (qi < T) {
            if (kg == 0) {
                finish(0, acc_o[0], theirs);
                finish(1, acc_o[1], theirs + 16 * 64);
            } else {
                finish(2, acc_o[2], theirs);
                finish(3, acc_o[3], theirs + 16 * 64);
            }
        }
    }
}

int check_heads(int32_t T, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim)
{
    if (T < 0 || n_q_heads < 1 || n_kv_heads < 1) return MQUANT_ERR_BAD_SHAPE;
    if (head_dim != kHeadDim) return MQUANT_ERR_UNSUPPORTED;
    if (n_q_heads % n_kv_heads != 0) return MQUANT_ERR_BAD_SHAPE;
    return MQUANT_OK;
}

int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

template <int KG, bool VT>
int launch_attention(const __half *q, int64_t ldq, const __half *k, int64_t ldk, const __half *v, int64_t ldv,
                     __half *o, int64_t ldo, const int32_t *pos, const int32_t *tile_min, const int32_t *tile_max,
                     int32_t T, int32_t group, int32_t n_kv_heads, int64_t groups, int32_t xcds_per_kv,
                     float scale_log2e, hipStream_t stream)
{
    constexpr int lds = KG * kGroupLds;
    static_assert(8 * 34 * 64 * 4 <= 2 * kGroupLds, "exchange of the key groups");
    auto kern = aifs_attention_kernel<KG, VT>;
    static LdsLimit limit;
    if (const int st = limit.raise(reinterpret_cast<const void *>(kern), lds); st != MQUANT_OK) return st;
    MQ_LAUNCH(kern, dim3(static_cast<unsigned>(groups)), dim3(KG * 256), lds, stream, q, ldq, k, ldk, v, ldv, o, ldo,
              pos, tile_min, tile_max, T, group, n_kv_heads, static_cast<int32_t>(ceil_div(T, kBQ)), xcds_per_kv, scale_log2e);
    return launch_status();
}

}  // namespace

extern "C" int mquant_rope_apply(void *x, int64_t ldx, const int32_t *pos, int32_t T, int32_t n_heads,
                                 int32_t head_dim, double base, mquant_stream_t stream)
{
    if (T < 0 || n_heads < 1) return MQUANT_ERR_BAD_SHAPE;
    if (head_dim != kHeadDim) return MQUANT_ERR_UNSUPPORTED;
    if (!(base > 1.0) || !std::isfinite(base)) return MQUANT_ERR_BAD_SHAPE;
    if (T == 0) return MQUANT_OK;
    if (!x || !pos) return MQUANT_ERR_NULL;
    if (ldx < static_cast<int64_t>(n_heads) * head_dim) return MQUANT_ERR_BAD_SHAPE;
    if (ldx % 2 != 0 || !aligned_to(x, 4) || !aligned_to(pos, 4)) return MQUANT_ERR_ALIGNMENT;
    InvFreq inv;
    for (int j = 0; j < kHeadDim / 2; ++j) inv.f[j] = pow(base, -2.0 * j / kHeadDim);
    // A wave of the 16-byte kernel forms 64 angles for its token whatever the number of heads, and with
    // few heads most of its lanes hold no data: 4-byte kernel against 16-byte one at 16384 tokens, 1 / 2
    // / 4 / 5 / 6 / 8 heads: 5.7 / 8.1, 6.5 / 8.6, 8.3 / 9.7, 8.7 / 10.2, 11.1 / 10.7, 13.2 / 11.7 us; at 4096 tokens
    // 3.4 / 3.8, 3.6 / 3.8, 4.3 / 4.2, 4.6 / 4.4, 4.9 / 4.5, 5.5 / 4.8.
    const bool wide = n_heads >= 6 || (n_heads >= 3 && T <= 4096);
    if (wide && ldx % 8 == 0 && aligned_to(x, 16) && n_heads <= 65535) {
        const dim3 grid(static_cast<unsigned>(ceil_div(T, 4) < 65536 ? ceil_div(T, 4) : 65536),
                        static_cast<unsigned>(ceil_div(n_heads * (kHeadDim / 8), 64 * kRopeChunks)));
        MQ_LAUNCH(rope_wide_kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream),
                  static_cast<__half *>(x), ldx, pos, T, n_heads, inv);
        return launch_status();
    }
    int64_t blocks = ceil_div(static_cast<int64_t>(T) * (kHeadDim / 2), 256);
    if (blocks > 65536) blocks = 65536;
    MQ_LAUNCH(rope_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
              static_cast<hipStream_t>(stream), static_cast<__half *>(x), ldx, pos, T, n_heads, inv);
    return launch_status();
}

extern "C" int64_t mquant_aifs_attention_workspace_bytes(int32_t T, int32_t n_kv_heads, int32_t head_dim)
{
    if (T < 0 || n_kv_heads < 1) return MQUANT_ERR_BAD_SHAPE;
    if (head_dim != kHeadDim) return MQUANT_ERR_UNSUPPORTED;
    const int64_t Tp = round_up(T, kBK);
    const int64_t vt = round_up(static_cast<int64_t>(n_kv_heads) * head_dim * Tp * 2, 256);
    return vt + round_up(2 * (Tp / kBK) * 4, 256);
}

extern "C" int mquant_aifs_attention(const void *q, int64_t ldq, const void *k, int64_t ldk,
                                     const void *v, int64_t ldv, void *o, int64_t ldo,
                                     const int32_t *pos, int32_t T, int32_t n_q_heads,
                                     int32_t n_kv_heads, int32_t head_dim, void *workspace,
                                     int64_t workspace_bytes, mquant_stream_t stream_)
{
    const int st = check_heads(T, n_q_heads, n_kv_heads, head_dim);
    if (st != MQUANT_OK) return st;
    if (T == 0) return MQUANT_OK;
    if (!q || !k || !v || !o || !pos) return MQUANT_ERR_NULL;
    const int64_t qw = static_cast<int64_t>(n_q_heads) * head_dim, kw = static_cast<int64_t>(n_kv_heads) * head_dim;
    if (ldq < qw || ldo < qw || ldk < kw || ldv < kw) return MQUANT_ERR_BAD_SHAPE;
    if (ldq % 8 != 0 || ldk % 8 != 0 || ldv % 8 != 0 || ldo % 4 != 0 || !aligned_to(q, 16) ||
        !aligned_to(k, 16) || !aligned_to(v, 16) || !aligned_to(o, 8) || !aligned_to(pos, 4))
        return MQUANT_ERR_ALIGNMENT;
    const int64_t need = mquant_aifs_attention_workspace_bytes(T, n_kv_heads, head_dim);
    if (!workspace || workspace_bytes < need) return MQUANT_ERR_WORKSPACE;
    if (!aligned_to(workspace, 256)) return MQUANT_ERR_ALIGNMENT;
    hipStream_t stream = static_cast<hipStream_t>(stream_);

    const int32_t n_tiles = static_cast<int32_t>(ceil_div(T, kBK));
    const int64_t n_qblocks = ceil_div(T, kBQ);
    const int32_t group = n_q_heads / n_kv_heads;
    const int32_t xcds_per_kv = 8 % n_kv_heads == 0 ? 8 / n_kv_heads : 0;
    const int64_t groups = xcds_per_kv > 0 ? 8 * ceil_div(n_qblocks * group, xcds_per_kv) : n_qblocks * n_q_heads;
    if (groups > 0x7fffffff) return MQUANT_ERR_UNSUPPORTED;
    const __half *qh = static_cast<const __half *>(q), *kh = static_cast<const __half *>(k), *vh = static_cast<const __half *>(v);
    __half *oh = static_cast<__half *>(o);
    const float scale_log2e = static_cast<float>(1.4426950408889634 / sqrt(static_cast<double>(head_dim)));
    // Values in place or transposed first (a launch of its own, 2 to 5 us, whose tiles the P V product then reads with
    // half the LDS instructions: 2 % of a long sequence's time).  The line lies where the two meet: transposed / in
    // place, 28 heads, T = 1280 35.7 / 33.6 us, 2048 55.1 / 53.0, 3500 115.2 / 114.0, 4096 138.8 / 140.2; 64 heads, T = 1280
    // 47.6 / 44.3, 2048 87.4 / 85.1, 2500 136.5 / 138.0, 3500 238.9 / 241.5.  In place also needs an output that shares no memory
    // with V, which every work-group reads until the last has finished, and rows close enough for 32-bit offsets.
    const int64_t items = n_qblocks * n_q_heads;
    if (items * n_tiles <= 48000 && n_tiles <= kChunkTiles && ldv < int64_t{1} << 24 && rows_apart(v, ldv, kw, o, ldo, qw, T)) {
        // Two key groups, one work-group per compute unit, where the work-groups are few: the longest one, which
        // walks all key tiles, is what such a launch waits for.  One / two groups, 28 heads (T, work-groups): 77, 28
        // 8.3 / 8.5 us; 256, 56 11.9 / 12.0; 512, 112 16.6 / 15.9; 1003, 224 27.5 / 24.1; 1280, 280 33.6 / 27.8; 1408, 308
        // 37.7 / 34.6; 1792, 392 46.2 / 44.1; 2048, 448 53.0 / 50.1; 2500, 560 70.8 / 79.6; 64 heads: 512, 256 17.0 / 16.3; 640,
        // 320 22.9 / 24.7; 1003, 512 33.5 / 40.1.  Beyond one round of work-groups it takes long ones to make up for the
        // second prologue, and where the line lies depends on the layout too.  Text only / one visual span / three: 28 heads, T =
        // 1281, 308 33.7 / 34.2 / 35.1 against 28.1 / 33.2 / 32.2; 32 heads, 1281, 352 33.6 / 34.2 / 35.4 against 28.8 / 34.9 / 34.7;
        // 40 heads, 960, 320 26.1 / 29.3 / 29.6 against 25.0 / 31.7 / 31.7; 1280, 400 34.9 / 35.8 / 36.7 against 32.8 / 39.0 / 38.9; 1281,
        // 440 35.4 / 36.2 / 37.2 against 37.4 / 42.4 / 41.2.
        const bool two = n_tiles > 4 && (items <= kNumCU + kNumCU / 8 || (items <= 2 * kNumCU - kNumCU / 4 && n_tiles >= 22));
        auto launch = two ? launch_attention<2, false> : launch_attention<1, false>;
        return launch(qh, ldq, kh, ldk, vh, ldv, oh, ldo, pos, nullptr, nullptr, T, group, n_kv_heads, groups, xcds_per_kv,
                      scale_log2e, stream);
    }
    const int32_t Tp = n_tiles * kBK;
    __half *vt = static_cast<__half *>(workspace);
    int32_t *tile_min = reinterpret_cast<int32_t *>(
        static_cast<uint8_t *>(workspace) + round_up(kw * Tp * 2, 256));
    int32_t *tile_max = tile_min + n_tiles;
    MQ_LAUNCH(vt_kernel, dim3(n_tiles, static_cast<unsigned>(ceil_div(kw, 64))), dim3(256), 0, stream, vh, ldv, vt, T, Tp,
              static_cast<int32_t>(kw), pos, tile_min, tile_max);
    const int ls = launch_status();
    if (ls != MQUANT_OK) return ls;
    return launch_attention<1, true>(qh, ldq, kh, ldk, vt, Tp, oh, ldo, pos, tile_min, tile_max, T, group, n_kv_heads, groups,
                                     xcds_per_kv, scale_log2e, stream);
}
