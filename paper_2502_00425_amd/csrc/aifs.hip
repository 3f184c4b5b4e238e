// AIFS (Attention-Invariant Flexible Switching, MQuant Sec. 3.1): index vector,
// row gather and causal-mask remap.  All three are pure index/byte work.
#include "mquant_internal.h"

using namespace mquant;

extern "C" int mquant_version(void) { return 200; }

#ifndef MQUANT_BUILD_ID
#define MQUANT_BUILD_ID "unknown"
#endif
extern "C" const char *mquant_build_id(void) { return MQUANT_BUILD_ID; }

namespace mquant {
TuneState &tune_state()
{
    static TuneState st;
    return st;
}
}  // namespace mquant

extern "C" int mquant_tune_set(int32_t key, int32_t value)
{
    TuneState &t = tune_state();
    switch (key) {
    case MQUANT_TUNE_GEMM_TILE:
        if (value < -1 || value > 4) return MQUANT_ERR_BAD_SHAPE;
        t.gemm_tile.store(value, std::memory_order_relaxed);
        return MQUANT_OK;
    case MQUANT_TUNE_GEMM_NOSPLIT:
        if (value < 0 || value > 1) return MQUANT_ERR_BAD_SHAPE;
        t.gemm_nosplit.store(value, std::memory_order_relaxed);
        return MQUANT_OK;
    case MQUANT_TUNE_G128_TILE:
        if (value < -1 || value > 1) return MQUANT_ERR_BAD_SHAPE;
        t.g128_tile.store(value, std::memory_order_relaxed);
        return MQUANT_OK;
    case MQUANT_TUNE_G128_SHAPE:
        if (value < -1 || value >= kG128Tiles) return MQUANT_ERR_BAD_SHAPE;
        t.g128_tile.store(value, std::memory_order_relaxed);
        return MQUANT_OK;
    case MQUANT_TUNE_GEMM_SHAPE:
        if (value < -1 || value >= kGemmShapes) return MQUANT_ERR_BAD_SHAPE;
        t.gemm_sliced.store(value, std::memory_order_relaxed);
        return MQUANT_OK;
    case MQUANT_TUNE_GEMV_VARIANT:
        if (value < -1 || value > 3) return MQUANT_ERR_BAD_SHAPE;
        t.gemv_variant.store(value, std::memory_order_relaxed);
        return MQUANT_OK;
    default: return MQUANT_ERR_BAD_SHAPE;
    }
}

extern "C" const char *mquant_status_string(int status)
{
    switch (status) {
    case MQUANT_OK: return "ok";
    case MQUANT_ERR_NULL: return "required pointer is NULL";
    case MQUANT_ERR_BAD_SHAPE: return "bad shape, leading dimension, span or scale";
    case MQUANT_ERR_UNSUPPORTED: return "shape or block size not supported by these kernels";
    case MQUANT_ERR_WORKSPACE: return "workspace missing or too small";
    case MQUANT_ERR_HIP: return "HIP runtime error";
    case MQUANT_ERR_ALIGNMENT: return "pointer or leading dimension not sufficiently aligned";
    default: return "unknown status";
    }
}

// Stable partition of 0..T-1: visual rows first (Sec. 3.1, E^u; index form in
// the appendix on rotary position embedding).  Host code, O(T).
extern "C" int mquant_aifs_build_perm(int32_t T, const mquant_span_t *vis, int32_t n_spans,
                                      int32_t *perm, int32_t *inv_perm, int32_t *n_vis)
{
    if (n_vis == nullptr) return MQUANT_ERR_NULL;
    if (T < 0 || n_spans < 0) return MQUANT_ERR_BAD_SHAPE;
    if (n_spans > 0 && vis == nullptr) return MQUANT_ERR_NULL;
    int64_t V = 0;
    int64_t prev_end = 0;
    for (int32_t s = 0; s < n_spans; ++s) {
        const int64_t b = vis[s].start, l = vis[s].len;
        if (l < 0 || b < prev_end || b + l > T) return MQUANT_ERR_BAD_SHAPE;
        prev_end = b + l;
        V += l;
    }
    *n_vis = static_cast<int32_t>(V);
    if (perm == nullptr && inv_perm == nullptr) return MQUANT_OK;
    // Walk the sequence once; a visual row goes to the next visual slot, a
    // text row to the next text slot behind all V visual ones.
    int64_t next_vis = 0, next_txt = V;
    int32_t s = 0;
    for (int32_t i = 0; i < T; ++i) {
        while (s < n_spans && i >= vis[s].start + vis[s].len) ++s;
        const bool is_vis = s < n_spans && i >= vis[s].start;
        const int64_t slot = is_vis ? next_vis++ : next_txt++;
        if (perm) perm[slot] = i;
        if (inv_perm) inv_perm[i] = static_cast<int32_t>(slot);
    }
    return MQUANT_OK;
}

namespace {

// One 16-byte chunk per thread; grid.y walks rows.
__global__ __launch_bounds__(256) void permute_rows_kernel(
    const uint4 *__restrict__ x, int64_t ldx16, uint4 *__restrict__ xu, int64_t ldxu16,
    const int32_t *__restrict__ perm, int32_t T, int32_t chunks)
{
    const int32_t c = blockIdx.x * 256 + threadIdx.x;
    if (c >= chunks) return;
    for (int32_t i = blockIdx.y; i < T; i += gridDim.y) {
        int32_t src = perm[i];
        src = (src < 0 || src >= T) ? 0 : src;
        xu[static_cast<int64_t>(i) * ldxu16 + c] = x[static_cast<int64_t>(src) * ldx16 + c];
    }
}

// Four output bytes per thread: M^u[i, j..j+3] = M[perm[i], perm[j..j+3]].
__global__ __launch_bounds__(256) void remap_mask_kernel(
    const uint8_t *__restrict__ mask, uint8_t *__restrict__ mask_u,
    const int32_t *__restrict__ perm, int32_t T)
{
    const int32_t j0 = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (j0 >= T) return;
    for (int32_t i = blockIdx.y; i < T; i += gridDim.y) {
        int32_t pi = perm[i];
        pi = (pi < 0 || pi >= T) ? 0 : pi;
        const uint8_t *row = mask + static_cast<int64_t>(pi) * T;
        uint8_t *out = mask_u + static_cast<int64_t>(i) * T + j0;
        if (j0 + 4 <= T && (T & 3) == 0) {
            const int4 pj = *reinterpret_cast<const int4 *>(perm + j0);
            const int32_t p[4] = {pj.x, pj.y, pj.z, pj.w};
            uint32_t v = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t pq = (p[q] < 0 || p[q] >= T) ? 0 : p[q];
                v |= static_cast<uint32_t>(row[pq] != 0) << (8 * q);
            }
            *reinterpret_cast<uint32_t *>(out) = v;
        } else {
            for (int q = 0; q < 4 && j0 + q < T; ++q) {
                int32_t pq = perm[j0 + q];
                pq = (pq < 0 || pq >= T) ? 0 : pq;
                out[q] = row[pq] != 0;
            }
        }
    }
}

constexpr size_t kRemapMaxLds = 145 * 1024;

// The same remap with R output rows per work-group: their R source rows M[perm[i], :] are copied into LDS
// with 16-byte loads, and every thread then gathers four output bytes of each row from there.  The
// index vector is read once per R rows instead of once per row (it is four times the size of a mask
// row), and the byte gathers hit LDS instead of the memory pipeline.
//
// The copy: the 1 KiB pieces of all R rows are dealt over the waves and a wave requests up to four before it
// stores the first, so a work-group waits for one or two trips to memory.  A source row starts anywhere; it is
// copied from the 16-byte boundary before it, chunks that reach past the mask byte by byte.
// The stores: words of the output, aligned; where T % 4 != 0 (WORDS = false) a row starts (i T) % 4 bytes into a
// word, so a thread holds the indices of eight columns and takes the four of its word.
//
// What bounds it: trips to memory on short masks, the LDS byte reads and the copy's trips on long ones (T = 8192: 4.5
// TB/s over both directions).  With one row after the other copied by the threads that its length keeps busy and
// eight rows to a work-group, only where T % 16 == 0, T = 1280 took 5.8 us (now 3.8), 4096 17.4 (11.8), 8192 35.2 (29.8),
// 16384 124 (124), and the byte gather of the other lengths 2501 16.3 (8.3), 5001 51.6 (19.1), 8191 113 (41.2).
template <int R, int NT, bool WORDS>
__global__ __launch_bounds__(NT) void remap_mask_rows_kernel(
    const uint8_t *__restrict__ mask, uint8_t *__restrict__ mask_u,
    const int32_t *__restrict__ perm, int32_t T, int32_t pitch)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t rows[];      // R rows of pitch >= 15 + T bytes
    constexpr int NW = NT / 64, AHEAD = 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint8_t *const end = mask + static_cast<int64_t>(T) * T;
    auto source = [&](int32_t i) {                                       // row of output row i (the last for those past T)
        const int32_t pi = perm[i < T ? i : T - 1];
        return mask + static_cast<int64_t>((pi < 0 || pi >= T) ? 0 : pi) * T;
    };
    const int32_t pieces = (pitch / 16 + 63) / 64;                       // of a row
    for (int32_t i0 = blockIdx.x * R; i0 < T; i0 += gridDim.x * R) {
        __syncthreads();                                                 // the previous rows are consumed
        for (int32_t u0 = wave; u0 < R * pieces; u0 += NW * AHEAD) {
            uint4 v[AHEAD];
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {
                const int32_t u = u0 + k * NW;
                if (u < R * pieces) {                                    // wave-uniform
                    const int32_t r = u / pieces, c = (u - r * pieces) * 64 + lane;
                    const uint8_t *src = source(i0 + r);
                    const int32_t off = static_cast<int32_t>(reinterpret_cast<uintptr_t>(src) & 15);
                    const uint8_t *at = src - off + c * 16;
                    v[k] = make_uint4(0u, 0u, 0u, 0u);
                    if (c * 16 < off + T) {
                        if (at >= mask && at + 16 <= end) {
                            v[k] = *reinterpret_cast<const uint4 *>(at);
                        } else {
                            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                            for (int b = 0; b < 16; ++b)
                                if (at + b >= mask && at + b < end) w[b / 4] |= static_cast<uint32_t>(at[b]) << (b % 4 * 8);
                            v[k] = make_uint4(w[0], w[1], w[2], w[3]);
                        }
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {
                const int32_t u = u0 + k * NW;
                if (u < R * pieces) {
                    const int32_t r = u / pieces, c = (u - r * pieces) * 64 + lane;
                    if (c * 16 < pitch) *reinterpret_cast<uint4 *>(rows + r * pitch + c * 16) = v[k];
                }
            }
        }
        int32_t at[R];                                                   // where the rows start in LDS
#pragma unroll
        for (int r = 0; r < R; ++r) at[r] = r * pitch + static_cast<int32_t>(reinterpret_cast<uintptr_t>(source(i0 + r)) & 15);
        __syncthreads();
        // word j0 / 4 of a row that starts m bytes into a word: columns j0 - m .. j0 - m + 3
        for (int32_t j0 = tid * 4; j0 < (WORDS ? T : T + 3); j0 += NT * 4) {
            int32_t p[8];                                                // perm[j0 - 4 .. j0 + 3]
#pragma unroll
            for (int h = WORDS ? 1 : 0; h < 2; ++h) {
                const int32_t j = j0 - 4 + h * 4;
                if (j >= 0 && j + 4 <= T) {
                    const int4 pj = *reinterpret_cast<const int4 *>(perm + j);
                    p[h * 4] = pj.x, p[h * 4 + 1] = pj.y, p[h * 4 + 2] = pj.z, p[h * 4 + 3] = pj.w;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) p[h * 4 + q] = j + q >= 0 && j + q < T ? perm[j + q] : 0;
                }
            }
#pragma unroll
            for (int q = WORDS ? 4 : 0; q < 8; ++q) p[q] = (p[q] < 0 || p[q] >= T) ? 0 : p[q];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int32_t i = i0 + r;
                if (i < T) {
                    const uint8_t *row = rows + at[r];
                    auto word = [&](const int m) {
                        const uint32_t x = static_cast<uint32_t>(row[p[4 - m]]) | (static_cast<uint32_t>(row[p[5 - m]]) << 8) |
                                           (static_cast<uint32_t>(row[p[6 - m]]) << 16) | (static_cast<uint32_t>(row[p[7 - m]]) << 24);
                        // every byte -> 1 if non-zero, else 0
                        return ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u) >> 7;
                    };
                    uint8_t *out = mask_u + static_cast<int64_t>(i) * T;
                    if constexpr (WORDS) {
                        *reinterpret_cast<uint32_t *>(out + j0) = word(0);
                    } else {
                        const int m = static_cast<int>(reinterpret_cast<uintptr_t>(out) & 3);      // uniform
                        const uint32_t nz = m == 0 ? word(0) : m == 1 ? word(1) : m == 2 ? word(2) : word(3);
                        const int32_t j = j0 - m;
                        if (j >= 0 && j + 4 <= T) {
                            *reinterpret_cast<uint32_t *>(out + j) = nz;
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (j + q >= 0 && j + q < T) out[j + q] = static_cast<uint8_t>(nz >> (8 * q));
                        }
                    }
                }
            }
        }
    }
}

// Long rows that are whole 16-byte chunks of the mask: one row after the other copied by all threads.  In the kernel above the
// conditions of chunks that reach past the mask fill the scalar registers, so that a compute unit holds one work-group of
// sixteen waves instead of two, and its rows take one chunk more; up to 16384 columns, where eight waves a work-group are enough, it is
// ahead nevertheless.  us, kernel above / this one: T = 12000 63 / 86, 16384 129 / 146, 18448 168 / 159, 20480 264 / 186, 32768
// 648 / 531, 37104 838 / 618, 65536 2570 / 1769, 80000 4392 / 2670.
template <int R>
__global__ __launch_bounds__(1024) void remap_mask_whole_rows_kernel(
    const uint8_t *__restrict__ mask, uint8_t *__restrict__ mask_u,
    const int32_t *__restrict__ perm, int32_t T)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t rows[];      // R rows of T bytes
    const int tid = threadIdx.x;
    for (int32_t i0 = blockIdx.x * R; i0 < T; i0 += gridDim.x * R) {
        __syncthreads();                                                 // the previous rows are consumed
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (i0 + r < T) {                                            // uniform
                int32_t pi = perm[i0 + r];
                pi = (pi < 0 || pi >= T) ? 0 : pi;
                const uint4 *src = reinterpret_cast<const uint4 *>(mask + static_cast<int64_t>(pi) * T);
                for (int32_t c = tid; c < T / 16; c += 1024)
                    *reinterpret_cast<uint4 *>(rows + r * T + c * 16) = src[c];
            }
        }
        __syncthreads();
        for (int32_t j0 = tid * 4; j0 < T; j0 += 4096) {
            const int4 pj = *reinterpret_cast<const int4 *>(perm + j0);
            int32_t p[4] = {pj.x, pj.y, pj.z, pj.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = (p[q] < 0 || p[q] >= T) ? 0 : p[q];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (i0 + r < T) {
                    const uint8_t *row = rows + r * T;
                    const uint32_t x = static_cast<uint32_t>(row[p[0]]) | (static_cast<uint32_t>(row[p[1]]) << 8) |
                                       (static_cast<uint32_t>(row[p[2]]) << 16) | (static_cast<uint32_t>(row[p[3]]) << 24);
                    // every byte -> 1 if non-zero, else 0
                    const uint32_t nz = ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u) >> 7;
                    *reinterpret_cast<uint32_t *>(mask_u + static_cast<int64_t>(i0 + r) * T + j0) = nz;
                }
            }
        }
    }
}

int64_t remap_blocks(int32_t T, int R) { return ceil_div(T, R) < 8 * kNumCU ? ceil_div(T, R) : 8 * kNumCU; }

template <int R>
int launch_remap_whole_rows(const uint8_t *mask, uint8_t *mask_u, const int32_t *perm, int32_t T, hipStream_t stream)
{
    auto kern = remap_mask_whole_rows_kernel<R>;
    static LdsLimit limit;
    if (const int st = limit.raise(reinterpret_cast<const void *>(kern), kRemapMaxLds); st != MQUANT_OK) return st;
    MQ_LAUNCH(kern, dim3(static_cast<unsigned>(remap_blocks(T, R))), dim3(1024), static_cast<size_t>(R) * T, stream, mask, mask_u, perm, T);
    return launch_status();
}

// A row of any alignment, in whole 16-byte chunks.
template <int R>
size_t remap_lds_bytes(int32_t T)
{
    return static_cast<size_t>(R) * static_cast<size_t>(ceil_div(static_cast<int64_t>(T) + 15, 16) * 16);
}

template <int R, int NT>
int launch_remap_rows(const uint8_t *mask, uint8_t *mask_u, const int32_t *perm, int32_t T, hipStream_t stream)
{
    const size_t lds = remap_lds_bytes<R>(T);
    const int32_t pitch = static_cast<int32_t>(lds / R);
    auto launch = [&](auto kern, LdsLimit &limit) {
        if (lds > 64 * 1024)
            if (const int st = limit.raise(reinterpret_cast<const void *>(kern), kRemapMaxLds); st != MQUANT_OK) return st;
        MQ_LAUNCH(kern, dim3(static_cast<unsigned>(remap_blocks(T, R))), dim3(NT), lds, stream, mask, mask_u, perm, T, pitch);
        return launch_status();
    };
    static LdsLimit words, bytes;
    return T % 4 == 0 ? launch(remap_mask_rows_kernel<R, NT, true>, words) : launch(remap_mask_rows_kernel<R, NT, false>, bytes);
}

}  // namespace

extern "C" int mquant_aifs_permute(const void *x, int64_t ldx, void *x_u, int64_t ldxu,
                                   const int32_t *perm, int32_t T, int32_t K,
                                   mquant_stream_t stream)
{
    if (T < 0 || K < 0) return MQUANT_ERR_BAD_SHAPE;
    if (T == 0 || K == 0) return MQUANT_OK;
    if (!x || !x_u || !perm) return MQUANT_ERR_NULL;
    if (ldx < K || ldxu < K) return MQUANT_ERR_BAD_SHAPE;
    if (x == x_u) return MQUANT_ERR_BAD_SHAPE;            // a gather cannot run in place
    if (K % 8 != 0) return MQUANT_ERR_UNSUPPORTED;
    if (ldx % 8 != 0 || ldxu % 8 != 0 || !aligned_to(x, 16) || !aligned_to(x_u, 16))
        return MQUANT_ERR_ALIGNMENT;
    const int32_t chunks = K / 8;
    dim3 grid(static_cast<unsigned>(ceil_div(chunks, 256)),
              static_cast<unsigned>(T < 65535 ? T : 65535));
    MQ_LAUNCH(permute_rows_kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint4 *>(x), ldx / 8, static_cast<uint4 *>(x_u), ldxu / 8,
                       perm, T, chunks);
    return launch_status();
}

extern "C" int mquant_aifs_remap_mask(const uint8_t *mask, uint8_t *mask_u, const int32_t *perm,
                                      int32_t T, mquant_stream_t stream)
{
    if (T < 0) return MQUANT_ERR_BAD_SHAPE;
    if (T == 0) return MQUANT_OK;
    if (!mask || !mask_u || !perm) return MQUANT_ERR_NULL;
    if (!aligned_to(mask_u, 4) || !aligned_to(perm, 16)) return MQUANT_ERR_ALIGNMENT;
    // Rows through LDS where a row is longer than what the caches answer the byte gather from at once; few rows of
    // few waves for a short mask, whose work-groups have to fill the chip.  us, byte gather / 2 rows, 256 threads / 4
    // rows, 512 threads: T = 512 2.1 / 2.4 / 2.7, 1003 3.8 / 4.2 / 4.7, 1024 3.0 / 3.0 / 3.3, 1281 6.8 / 4.9 / 5.3, 2048 6.7 / 5.1
    // / 5.2, 2501 16.2 / 8.3 / 8.6, 3072 13.0 / 7.9 / 7.9, 6001 69.8 / 27.8 / 25.3, 8192 - / 35.4 / 29.8, 16384 - / 159 / 124, 20001
    // 1562 / - / 242, 37107, one row and 1024 threads, 5900 / 1067.
    if (T > 1024 && T <= 144 * 1024) {
        hipStream_t hs = static_cast<hipStream_t>(stream);
        if (T < 2560) return launch_remap_rows<2, 256>(mask, mask_u, perm, T, hs);
        if (T > 16384 && T % 16 == 0 && aligned_to(mask, 16)) {
            if (4 * static_cast<int64_t>(T) <= 144 * 1024) return launch_remap_whole_rows<4>(mask, mask_u, perm, T, hs);
            return launch_remap_whole_rows<1>(mask, mask_u, perm, T, hs);
        }
        if (remap_lds_bytes<4>(T) <= kRemapMaxLds) return launch_remap_rows<4, 512>(mask, mask_u, perm, T, hs);
        return launch_remap_rows<1, 1024>(mask, mask_u, perm, T, hs);
    }
    dim3 grid(static_cast<unsigned>(ceil_div(ceil_div(T, 4), 256)),
              static_cast<unsigned>(T < 65535 ? T : 65535));
    MQ_LAUNCH(remap_mask_kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream),
                       mask, mask_u, perm, T);
    return launch_status();
}
