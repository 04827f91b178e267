// gfx950 (CDNA4) kernels: page scatter/gather, and the shrink / expand pair of the batched
// LoRA term (Sec. 5.3: gather matrix-vector for decode, gather matrix-matrix for prefill).
//
// Data layout: pool = n_pages rows of H 16-bit elements; an adapter's page lists sit in an
// int32 arena as [slot][A columns r][B rows r]; x is T x H (16-bit), y is T x H (fp32).
// v = x*A keeps fp32 precision: the decode kernels store it as rows of `v_stride` floats indexed
// by the token's position in the plan's sorted token list, the prefill kernels as 16-bit pieces
// in MFMA operand order (see VPieces).  All byte offsets into the pool are 64-bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "slora_internal.hpp"

namespace slora {

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

template <int DT>
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float acc)
{
    if constexpr (DT == SLORA_F16) {
        return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b), acc, false);
    } else {
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc,
                                               false);
    }
}

template <int DT>
__device__ __forceinline__ float dot8(const u32x4 &a, const u32x4 &b, float acc)
{
    acc = dot2<DT>(a.x, b.x, acc);
    acc = dot2<DT>(a.y, b.y, acc);
    acc = dot2<DT>(a.z, b.z, acc);
    acc = dot2<DT>(a.w, b.w, acc);
    return acc;
}

// the two 16-bit values packed in a dword, widened exactly to fp32
template <int DT>
__device__ __forceinline__ void widen2(uint32_t u, float &lo, float &hi)
{
    if constexpr (DT == SLORA_F16) {
        half2_t h = __builtin_bit_cast(half2_t, u);
        lo = (float)h.x;
        hi = (float)h.y;
    } else {
        lo = __uint_as_float(u << 16);
        hi = __uint_as_float(u & 0xffff0000u);
    }
}

// one fp32 value rounded to the 16-bit storage type (nearest, ties to even) and back
template <int DT>
__device__ __forceinline__ uint16_t narrow1(float f)
{
    if constexpr (DT == SLORA_F16)
        return __builtin_bit_cast(uint16_t, (_Float16)f);
    else
        return __builtin_bit_cast(uint16_t, (__bf16)f);
}
template <int DT>
__device__ __forceinline__ uint32_t narrow2(float lo, float hi)
{
    return (uint32_t)narrow1<DT>(lo) | ((uint32_t)narrow1<DT>(hi) << 16);
}
template <int DT>
__device__ __forceinline__ float widen1(uint16_t b)
{
    if constexpr (DT == SLORA_F16)
        return (float)__builtin_bit_cast(_Float16, b);
    else
        return __uint_as_float((uint32_t)b << 16);
}

// Eight consecutive elements of a row of y: fp32 (Y16 = false) or the pool's 16-bit storage
// type (Y16 = true; the sum is formed in fp32 and rounded once, to nearest even, on the way out).
// `off` is an element offset and a multiple of 8, so every access is 16-byte aligned.
template <int DT, bool Y16>
struct Y8;
template <int DT>
struct Y8<DT, false> {
    f32x4 a, b;
    __device__ __forceinline__ void load(const void *y, int64_t off)
    {
        const float *p = static_cast<const float *>(y) + off;
        a = *reinterpret_cast<const f32x4 *>(p);
        b = *reinterpret_cast<const f32x4 *>(p + 4);
    }
    __device__ __forceinline__ void add_store(void *y, int64_t off, const float (&d)[8])
    {
        float *p = static_cast<float *>(y) + off;
        a.x += d[0];
        a.y += d[1];
        a.z += d[2];
        a.w += d[3];
        b.x += d[4];
        b.y += d[5];
        b.z += d[6];
        b.w += d[7];
        *reinterpret_cast<f32x4 *>(p) = a;
        *reinterpret_cast<f32x4 *>(p + 4) = b;
    }
};
template <int DT>
struct Y8<DT, true> {
    u32x4 r;
    __device__ __forceinline__ void load(const void *y, int64_t off)
    {
        r = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(y) + off);
    }
    __device__ __forceinline__ void add_store(void *y, int64_t off, const float (&d)[8])
    {
        float f[8];
        widen2<DT>(r.x, f[0], f[1]);
        widen2<DT>(r.y, f[2], f[3]);
        widen2<DT>(r.z, f[4], f[5]);
        widen2<DT>(r.w, f[6], f[7]);
        u32x4 o;
        o.x = narrow2<DT>(f[0] + d[0], f[1] + d[1]);
        o.y = narrow2<DT>(f[2] + d[2], f[3] + d[3]);
        o.z = narrow2<DT>(f[4] + d[4], f[5] + d[5]);
        o.w = narrow2<DT>(f[6] + d[6], f[7] + d[7]);
        *reinterpret_cast<u32x4 *>(static_cast<uint16_t *>(y) + off) = o;
    }
};

// Sum over the 64 lanes, in every lane: the pairwise tree of a butterfly (lane l with l ^ 32, then ^ 16, ... ^ 1),
// whose exchanges need no trip through LDS: row swaps for 32 and 16, then rotations inside a row of 16 - after
// the steps 32 to 8 the sums repeat every 8 lanes, so a rotation by 4 brings what ^ 4 would - and quad permutes.
// Six dependent exchanges through LDS were a part of every decode kernel's chain: 32 tokens of ranks 8-64,
// H = 4096, 13.8 -> 12.9 us per call, 39 tokens of rank 32, H = 824, 18.2 -> 15.5.  The sums are the same bits.
__device__ __forceinline__ float row_sum(float v) // over 16 lanes
{
    constexpr int kRor8 = 0x128, kRor4 = 0x124, kXor2 = 0x4e, kXor1 = 0xb1; // DPP controls
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kRor8, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kRor4, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kXor2, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kXor1, 0xf, 0xf, true));
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return row_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Sums over the lanes of four values at a time: row r of 16 lanes (in every lane of it) gets the sum of a, c, b, d
__device__ __forceinline__ float wave_sum4(float a, float b, float c, float d)
{
    const auto ab = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    const auto cd = __builtin_amdgcn_permlane32_swap(__float_as_uint(c), __float_as_uint(d), false, false);
    const float x = __uint_as_float(ab[0]) + __uint_as_float(ab[1]); // lanes 0 .. 31: a, others: b
    const float y = __uint_as_float(cd[0]) + __uint_as_float(cd[1]);
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return row_sum(__uint_as_float(s[0]) + __uint_as_float(s[1]));
}

// ... of two: lanes 0 .. 31 get the sum of a, the others that of b
__device__ __forceinline__ float wave_sum2(float a, float b)
{
    const auto ab = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    const float x = __uint_as_float(ab[0]) + __uint_as_float(ab[1]);
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return row_sum(__uint_as_float(s[0]) + __uint_as_float(s[1]));
}

// 64 lanes x 16 bytes from per-lane addresses to 1 KiB of LDS at a wave-uniform address
template <int AUX>
__device__ __forceinline__ void load_to_lds(const unsigned char *src, unsigned char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, AUX);
}
constexpr int kLoadStreaming = 2; // cache policy "nt"

// ---------------------------------------------------------------------------------------
// page scatter / gather (exact copies)
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void write_pages_kernel(uint16_t *__restrict__ pool, const int32_t *__restrict__ idx,
                                                           const uint16_t *__restrict__ src, int H, int64_t n)
{
    // workgroups stride over the pages: a small grid bounds the requests in flight when the
    // source is host memory behind the host link
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const u32x4 *s = reinterpret_cast<const u32x4 *>(src + i * H);
        u32x4 *d = reinterpret_cast<u32x4 *>(pool + (int64_t)idx[i] * H);
        for (int c = threadIdx.x; c < H / 8; c += blockDim.x) d[c] = s[c];
    }
}

__global__ __launch_bounds__(256) void gather_pages_kernel(const uint16_t *__restrict__ pool,
                                                            const int32_t *__restrict__ list,
                                                            uint16_t *__restrict__ out, int H)
{
    const int64_t j = blockIdx.x;
    const u32x4 *s = reinterpret_cast<const u32x4 *>(pool + (int64_t)list[j] * H);
    u32x4 *d = reinterpret_cast<u32x4 *>(out + j * H);
    for (int c = threadIdx.x; c < H / 8; c += blockDim.x) d[c] = s[c];
}

// Work lists of a plan for one call, from pinned host memory: 16 bytes per lane and trip
__global__ __launch_bounds__(256) void copy_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) dst[i] = src[i];
}

// ---------------------------------------------------------------------------------------
// decode path, shrink: v[pos, j] = sum_h x[tok, h] * Apage_j[h]
//
// One workgroup (4 wavefronts) = one item = a few pages of one adapter (shrink_pages) and up to
// kShrinkTok tokens that use it.  The tokens' x rows are staged once in LDS.  Each wavefront
// streams whole pages from HBM (pages wave, wave+4, ... of the item) with 16-byte non-temporal
// loads per lane, U loads per block, two blocks in flight (the next block - possibly of the
// next page - is requested before the current one is consumed, and the very first block is
// requested before x is staged).  Blocks are dotted against the staged rows with packed
// 16-bit dot products accumulating in fp32; one 64-lane butterfly per page and token.
// ---------------------------------------------------------------------------------------
constexpr int kShrinkThreads = 256;
constexpr int kShrinkWaves = kShrinkThreads / kWave;

// The wavefront's share of `n_pages` consecutive entries of a page list (entries wave, wave + nw,
// ...), dotted against the `ntok` x rows staged in LDS; put(t, j, s) receives the finished sum
// of token t and list entry j (lane 0 only).  stage() copies the x rows to LDS and ends with a
// workgroup barrier; it runs after the first block of page data has been requested.
template <int DT, int U, class Stage, class Put>
__device__ __forceinline__ void shrink_vec_core(const int32_t *__restrict__ pa, int n_pages, int ntok, int wave, int nw,
                                                int lane, const uint16_t *__restrict__ pool, int H,
                                                const u32x4 *xs, Stage stage, Put put)
{
    const int nch = H >> 3; // 16-byte chunks per row
    const int nblk = (nch + kWave * U - 1) / (kWave * U);                           // blocks per page
    const int my_pages = n_pages > wave ? (n_pages - wave + nw - 1) / nw : 0;
    const int total = my_pages * nblk;
    const u32x4 zero = u32x4{0u, 0u, 0u, 0u};

    // block `blk` of this wavefront's page number `pg`
    auto load_block = [&](int pg, int blk, u32x4(&w)[U]) {
        const u32x4 *page = reinterpret_cast<const u32x4 *>(pool + (int64_t)pa[wave + pg * nw] * H);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = (blk * U + u) * kWave + lane;
            w[u] = c < nch ? __builtin_nontemporal_load(page + c) : zero;
        }
    };
    float acc[kShrinkTok];
#pragma unroll
    for (int t = 0; t < kShrinkTok; ++t) acc[t] = 0.f;
    auto consume = [&](int pg, int blk, const u32x4(&w)[U]) {
#pragma unroll
        for (int t = 0; t < kShrinkTok; ++t) {
            if (t < ntok) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int c = (blk * U + u) * kWave + lane;
                    const u32x4 xv = c < nch ? xs[t * nch + c] : zero;
                    acc[t] = dot8<DT>(w[u], xv, acc[t]);
                }
            }
        }
        if (blk == nblk - 1) {
            const int j = wave + pg * nw;
#pragma unroll
            for (int t = 0; t < kShrinkTok; ++t) {
                if (t < ntok) {
                    const float s = wave_sum(acc[t]);
                    if (lane == 0) put(t, j, s);
                }
                acc[t] = 0.f;
            }
        }
    };

    u32x4 wa[U], wb[U];
    if (total > 0) load_block(0, 0, wa);
    stage();

    int pg = 0, blk = 0;       // position of the block held in wa
    for (int b = 0; b < total; b += 2) {
        int pg1 = pg, blk1 = blk + 1;
        if (blk1 == nblk) { blk1 = 0; ++pg1; }
        if (b + 1 < total) load_block(pg1, blk1, wb);
        consume(pg, blk, wa);
        int pg2 = pg1, blk2 = blk1 + 1;
        if (blk2 == nblk) { blk2 = 0; ++pg2; }
        if (b + 2 < total) load_block(pg2, blk2, wa);
        if (b + 1 < total) consume(pg1, blk1, wb);
        pg = pg2;
        blk = blk2;
    }
}

// The x rows of `ntok` <= TOK tokens to LDS, [ntok][H/8] chunks, CH chunks of a row per thread and trip.  All rows are requested before any is
// stored: one round trip instead of one per token.  Vector shrink, us: 45 tokens of ranks 3-100, H = 3080, 3 slots 9.5 -> 8.4; 96 tokens of
// 4 adapters, H = 4096, 3 slots 9.5 -> 8.7; 100 tokens of ranks 8-64, 1 slot 7.9 -> 6.5.  CH = 1 wherever the threads cover a row: with a
// second chunk the vector shrink of H <= 2048 had 75 registers instead of 59, six wavefronts per SIMD instead of eight: 250 tokens of rank 64, H = 1024,
// 4 slots 34 / 39 us, 250 pairs of rank 32, H = 2048 26.7 / 32.5.
template <int TOK, int CH>
__device__ __forceinline__ void stage_rows(const uint16_t *__restrict__ x, const int32_t *__restrict__ tok_idx, int pos0, int ntok,
                                           int H, int n_threads, u32x4 *xs)
{
    const int nch = H >> 3;
    const u32x4 *row[TOK];
#pragma unroll
    for (int t = 0; t < TOK; ++t) row[t] = reinterpret_cast<const u32x4 *>(x + (int64_t)tok_idx[pos0 + min(t, ntok - 1)] * H);
    for (int c = threadIdx.x; c < nch; c += CH * n_threads) {
        u32x4 a[TOK][CH];
#pragma unroll
        for (int t = 0; t < TOK; ++t)
            if (t < ntok) {
#pragma unroll
                for (int i = 0; i < CH; ++i) a[t][i] = row[t][i == 0 ? c : min(c + i * n_threads, nch - 1)];
            }
#pragma unroll
        for (int t = 0; t < TOK; ++t)
            if (t < ntok) {
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (i == 0 || c + i * n_threads < nch) xs[t * nch + c + i * n_threads] = a[t][i];
            }
    }
}

// an item of the vector shrink: pa is its first entry of the A list, put(t, j, s) as above
template <int DT, int U, class Put>
__device__ __forceinline__ void shrink_vec_item(const Item &it, const int32_t *__restrict__ pa, const uint16_t *__restrict__ pool,
                                                const uint16_t *__restrict__ x, const int32_t *__restrict__ tok_idx, int H,
                                                u32x4 *xs, Put put) // xs: [ntok][H/8]
{
    const int tid = threadIdx.x;
    shrink_vec_core<DT, U>(
        pa, it.b, it.ntok, tid / kWave, kShrinkWaves, tid & (kWave - 1), pool, H, xs,
        [&]() {
            stage_rows<kShrinkTok, U <= 4 ? 1 : 2>(x, tok_idx, it.pos0, it.ntok, H, kShrinkThreads, xs);
            __syncthreads();
        },
        put);
}

template <int DT, int U>
__global__ __launch_bounds__(kShrinkThreads) void shrink_vec_kernel(const Item *__restrict__ items,
                                                                     const int32_t *__restrict__ arena,
                                                                     const uint16_t *__restrict__ pool,
                                                                     const int32_t *__restrict__ tok_idx, int H,
                                                                     int v_stride, MultiArgs args)
{
    extern __shared__ u32x4 xs[];
    // slots vary fastest, so workgroups are dispatched in the order of the work list (by rank)
    const int cs = blockIdx.x % args.n;
    const Item it = items[blockIdx.x / args.n];
    float *__restrict__ v = args.v[cs];
    shrink_vec_item<DT, U>(it, arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank + it.a, pool,
                           static_cast<const uint16_t *>(args.x[cs]), tok_idx, H, xs,
                           [&](int t, int j, float s) { v[(int64_t)(it.pos0 + t) * v_stride + it.a + j] = s; });
}

// ---------------------------------------------------------------------------------------
// decode path, expand: y[tok, d] += sum_j v[pos, j] * Bpage_j[d]
//
// One workgroup = one item = a run of columns (a multiple of 512, up to 4096) of one adapter's
// B for up to kExpandTok tokens.  Each lane owns 8 adjacent columns, adjacent wavefronts own
// adjacent 1 KiB pieces of every B row, so a workgroup reads each row as one contiguous run
// of several KiB.  Rows are streamed with 16-byte non-temporal loads, U rows per block, two
// blocks in flight, widened to fp32 and accumulated as v[pos, j] * row for every token (v is
// wave-uniform and comes in through scalar loads); then one read-modify-write of y per token,
// whose loads are issued before the row loop when there are at most two tokens.
// ---------------------------------------------------------------------------------------
template <int DT, bool Y16, int TOK, int U, bool PREFETCH_Y>
__device__ __forceinline__ void expand_vec_body(const Item &it, const int32_t *__restrict__ pb,
                                                const uint16_t *__restrict__ pool,
                                                const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                void *__restrict__ y, const float *v, int col, bool live,
                                                int v_pos0 = -1)
{
    const int lane = threadIdx.x & (kWave - 1);
    const float *vrow = v + (int64_t)(v_pos0 < 0 ? it.pos0 : v_pos0) * v_stride; // row of v of the item's first token
    float acc[TOK][8];
#pragma unroll
    for (int t = 0; t < TOK; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] = 0.f;

    Y8<DT, Y16> yv[TOK];
    int64_t yoff[TOK];
#pragma unroll
    for (int t = 0; t < TOK; ++t) {
        yoff[t] = (int64_t)tok_idx[it.pos0 + (t < it.ntok ? t : 0)] * H + col;
        if (PREFETCH_Y && t < it.ntok && live) yv[t].load(y, yoff[t]);
    }

    const int col_ld = live ? col : it.a;
    // Ranks are taken in windows of 64: lane l first fetches the page index and the v values of
    // rank w0 + l (one coalesced load each); inside the window both are broadcast with readlane,
    // so the row loads of a block issue back to back with no dependent scalar loads between them.
    for (int w0 = 0; w0 < it.rank; w0 += kWave) {
        const int wr = min(kWave, it.rank - w0);
        const int pwin = lane < wr ? pb[w0 + lane] : 0;
        float vwin[TOK];
#pragma unroll
        for (int t = 0; t < TOK; ++t) vwin[t] = (t < it.ntok && lane < wr) ? vrow[t * v_stride + w0 + lane] : 0.f;

        // Straight-line blocks: rank indices beyond the window are clamped to its last rank (the
        // row is loaded again, from cache) and meet v = 0; lanes beyond the item's columns read the
        // item's first column and are dropped at the store.  No branch separates the U loads.
        const int nb = (wr + U - 1) / U;
        auto load_block = [&](int b, u32x4(&w)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = min(b * U + u, wr - 1);
                const int64_t page = __builtin_amdgcn_readlane(pwin, j);
                w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(pool + page * H + col_ld));
            }
        };
        auto consume = [&](int b, const u32x4(&w)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = b * U + u; // < 64: nb * U <= 64
                float f[8];
                widen2<DT>(w[u].x, f[0], f[1]);
                widen2<DT>(w[u].y, f[2], f[3]);
                widen2<DT>(w[u].z, f[4], f[5]);
                widen2<DT>(w[u].w, f[6], f[7]);
#pragma unroll
                for (int t = 0; t < TOK; ++t) {
                    if (t < it.ntok) {
                        const float vv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vwin[t]), j));
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[t][e] = fmaf(vv, f[e], acc[t][e]);
                    }
                }
            }
        };

        u32x4 w[U];
        for (int b = 0; b < nb; ++b) {
            load_block(b, w);
            consume(b, w);
        }
    }

    if (!live) return;
#pragma unroll
    for (int t = 0; t < TOK; ++t) {
        if (t < it.ntok) {
            if (!PREFETCH_Y) yv[t].load(y, yoff[t]);
            yv[t].add_store(y, yoff[t], acc[t]);
        }
    }
}

template <int DT, bool Y16>
__global__ __launch_bounds__(512) void expand_vec_kernel(const Item *__restrict__ items,
                                                          const int32_t *__restrict__ arena,
                                                          const uint16_t *__restrict__ pool,
                                                          const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                          MultiArgs args)
{
    // slots vary fastest, so workgroups are dispatched in the order of the work list (by rank)
    const int cs = blockIdx.x % args.n;
    const Item it = items[blockIdx.x / args.n];
    const int col = it.a + threadIdx.x * 8;
    const int col_end = it.a + it.b; // <= H; both are multiples of 8
    // only WHOLE wavefronts beyond the item's columns may leave: the lanes of a wavefront exchange
    // page indices and v through readlane, so every lane of a live wavefront must stay active
    if (it.a + (int)(threadIdx.x & ~(kWave - 1)) * 8 >= col_end) return;
    const bool live = col < col_end;
    const int32_t *pb = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank + it.rank;
    if (it.ntok == 1)
        expand_vec_body<DT, Y16, 1, 8, true>(it, pb, pool, tok_idx, H, v_stride, args.y[cs], args.v[cs], col, live);
    else if (it.ntok == 2)
        expand_vec_body<DT, Y16, 2, 8, true>(it, pb, pool, tok_idx, H, v_stride, args.y[cs], args.v[cs], col, live);
    else
        expand_vec_body<DT, Y16, kExpandTok, 8, false>(it, pb, pool, tok_idx, H, v_stride, args.y[cs], args.v[cs], col, live);
}

// ---------------------------------------------------------------------------------------
// decode path, both stages in ONE launch: a workgroup = one adapter group of at most kExpandTok
// tokens, one wavefront per 512 columns of H.  First the wavefronts share out the adapter's A
// pages and leave v = x*A in LDS (shrink_vec_core), then every wavefront walks the B pages for
// its own columns (expand_vec_body) and updates y.  v never leaves the compute unit, x is staged
// once per group instead of once per four pages, and a decode step is one kernel instead of
// two dependent ones (each of which spends its first microseconds waiting for work items,
// page lists and the first pages).  Used when a batch has enough such groups to fill the GPU
// with whole-group workgroups (the scheduler decides); results are bit-identical to the two
// kernels' - the same sums in the same order.  Five wavefronts per SIMD instead of four fit three workgroups of
// H = 3072 on a compute unit instead of two: 800 workgroups of rank 100, bf16 200 -> 177 us (16-bit y 194 -> 173); U >= 7 needs the registers.
// ---------------------------------------------------------------------------------------
template <int DT, bool Y16, int U>
__global__ __launch_bounds__(1024, U <= 6 ? 5 : 4) void lora_vec_fused_kernel(const Item *__restrict__ items,
                                                               const int32_t *__restrict__ arena,
                                                               const uint16_t *__restrict__ pool,
                                                               const int32_t *__restrict__ tok_idx, int H,
                                                               int v_pad, MultiArgs args)
{
    extern __shared__ u32x4 smem[]; // x rows [kExpandTok][H/8], then v [kExpandTok][v_pad] floats
    const int cs = blockIdx.x % args.n;
    const Item it = items[blockIdx.x / args.n];
    const uint16_t *__restrict__ x = static_cast<const uint16_t *>(args.x[cs]);
    const int nch = H >> 3;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int nw = blockDim.x / kWave;
    float *vl = reinterpret_cast<float *>(smem + (size_t)kExpandTok * nch);
    const int32_t *pa = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank;
    shrink_vec_core<DT, U>(
        pa, it.rank, it.ntok, wave, nw, lane, pool, H, smem,
        [&]() {
            stage_rows<kExpandTok, 1>(x, tok_idx, it.pos0, it.ntok, H, (int)blockDim.x, smem);
            __syncthreads();
        },
        [&](int t, int j, float s) { vl[t * v_pad + j] = s; });
    __syncthreads();
    // expand: 512-column strips wave, wave + nw, ... (one strip per wavefront for H <= 8192)
    const int32_t *pb = pa + it.rank;
    for (int c0 = wave * 512; c0 < H; c0 += nw * 512) {
        const int col = c0 + lane * 8;
        const bool live = col < H;
        Item strip = it;
        strip.a = c0;   // lanes beyond H read the strip's first column and are dropped at the store
        if (it.ntok == 1)
            expand_vec_body<DT, Y16, 1, 8, true>(strip, pb, pool, tok_idx, H, v_pad, args.y[cs], vl, col, live, 0);
        else if (it.ntok == 2)
            expand_vec_body<DT, Y16, 2, 8, true>(strip, pb, pool, tok_idx, H, v_pad, args.y[cs], vl, col, live, 0);
        else
            expand_vec_body<DT, Y16, kExpandTok, 8, false>(strip, pb, pool, tok_idx, H, v_pad, args.y[cs], vl, col, live, 0);
    }
}

// ---------------------------------------------------------------------------------------
// decode path, both stages in one launch, for SMALL batches whose call is captured or keeps v in the static scratch (others: lora_vec_chain_kernel,
// 6.3 / 6.1 us for one token of rank 16, 4 slots, 9.2 / 6.4 at rank 32, 9.4 / 6.1 for six groups of two tokens): a workgroup = one item of the rank-split
// expand (512 columns of a group of at most kExpandTok tokens), which computes the group's v = x*A for
// itself.  Its eight wavefronts share out the A pages and leave v in LDS; the first four then do the
// rank-split expand, whose B rows and y were requested before the first A page.  A is read once per 512
// columns - from L2 but for the first.  What bounds such a batch is the chain of dependent round trips
// and the two launches: one token of rank 8 or 16, H = 4096, 4 slots 9.6 -> 6.6 us per call, rank 32 9.4 -> 7.8.
// Beyond a page or two per wavefront and token the repeated A reads cost more than the launch (ten groups
// of rank 16 and up to four tokens 11.3 / 12.6, H = 8192 9.1 / 10.1): see the plan's
// rule.  Sixteen wavefronts (128 registers each, B rows through LDS) were slower, 0.5 to 0.9 us.
// The first column range's workgroup also leaves v in memory, where a later expand expects it.
// Results are bit-identical to the two kernels'.
// ---------------------------------------------------------------------------------------
constexpr int kSmallWaves = 8;
static_assert(kSmallRanks <= kSplitWaves * 8, "a wavefront of the expand has at most one block of ranks");

template <int DT, bool Y16, int TOK>
__device__ __forceinline__ void small_body(const Item &it, const int32_t *__restrict__ pa,
                                           const uint16_t *__restrict__ pool, const uint16_t *__restrict__ x,
                                           const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                           void *__restrict__ y, float *__restrict__ v, u32x4 *xs)
{
    constexpr int UB = TOK <= 2 ? 16 : 8;             // ranks per block of the rank-split expand
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int nch = H >> 3;
    float *vl = reinterpret_cast<float *>(xs + (size_t)TOK * nch); // v [TOK][kSmallRanks]
    float *red = vl + TOK * kSmallRanks;              // partial sums of wavefronts 1 .. 3
    const int col = it.a + lane * 8;
    const bool live = col < it.a + it.b;
    const int col_ld = live ? col : it.a;             // lanes beyond the item's columns are dropped at the store

    // wavefronts 0 .. 3: block `wave` of the B rows; rank indices beyond the last are clamped and meet v = 0
    const bool expands = wave < kSplitWaves && wave * UB < it.rank;
    u32x4 w[UB];
    Y8<DT, Y16> yv[TOK];
    int64_t yoff[TOK];
    if (expands) {
        int64_t page[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) page[u] = pa[it.rank + min(wave * UB + u, it.rank - 1)];
#pragma unroll
        for (int u = 0; u < UB; ++u)
            w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(pool + page[u] * H + col_ld));
        if (wave == 0) {
#pragma unroll
            for (int t = 0; t < TOK; ++t) {
                yoff[t] = (int64_t)tok_idx[it.pos0 + min(t, it.ntok - 1)] * H + col;
                if (t < it.ntok && live) yv[t].load(y, yoff[t]);
            }
        }
    }
    // H <= 4096: a page is one block of eight loads per lane
    shrink_vec_core<DT, 8>(
        pa, it.rank, it.ntok, wave, kSmallWaves, lane, pool, H, xs,
        [&]() {
            stage_rows<TOK, 1>(x, tok_idx, it.pos0, it.ntok, H, kSmallWaves * kWave, xs);
            __syncthreads();
        },
        [&](int t, int j, float s) {
            vl[t * kSmallRanks + j] = s;
            if (it.a == 0) v[(int64_t)(it.pos0 + t) * v_stride + j] = s;
        });
    __syncthreads();
    float acc[TOK][8];
#pragma unroll
    for (int t = 0; t < TOK; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] = 0.f;
    if (expands) {
#pragma unroll
        for (int u0 = 0; u0 < UB; u0 += 8) {
            if (u0 > 0 && wave * UB + u0 >= it.rank) break; // no eight whose rows would all be the last one, times zero
#pragma unroll
            for (int u = u0; u < u0 + 8; ++u) {
                const int j = wave * UB + u;
                float f[8];
                widen2<DT>(w[u].x, f[0], f[1]);
                widen2<DT>(w[u].y, f[2], f[3]);
                widen2<DT>(w[u].z, f[4], f[5]);
                widen2<DT>(w[u].w, f[6], f[7]);
#pragma unroll
                for (int t = 0; t < TOK; ++t) {
                    const float vv = t < it.ntok && j < it.rank ? vl[t * kSmallRanks + j] : 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[t][e] = fmaf(vv, f[e], acc[t][e]);
                }
            }
        }
    }
    if (wave > 0 && wave < kSplitWaves) {
#pragma unroll
        for (int t = 0; t < TOK; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) red[(((wave - 1) * TOK + t) * 8 + e) * kWave + lane] = acc[t][e];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int k = 0; k < kSplitWaves - 1; ++k)
#pragma unroll
        for (int t = 0; t < TOK; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[t][e] += red[((k * TOK + t) * 8 + e) * kWave + lane];
    if (!live) return;
#pragma unroll
    for (int t = 0; t < TOK; ++t)
        if (t < it.ntok) yv[t].add_store(y, yoff[t], acc[t]);
}

template <int DT, bool Y16>
__global__ __launch_bounds__(kSmallWaves *kWave) void lora_vec_small_kernel(const Item *__restrict__ items,
                                                                            const int32_t *__restrict__ arena,
                                                                            const uint16_t *__restrict__ pool,
                                                                            const int32_t *__restrict__ tok_idx, int H,
                                                                            int v_stride, MultiArgs args)
{
    extern __shared__ u32x4 smem[]; // x rows [TOK][H/8], v [TOK][kSmallRanks], the expand's partial sums
    const int cs = blockIdx.x % args.n;
    const Item it = items[blockIdx.x / args.n];
    const int32_t *pa = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank;
    const uint16_t *x = static_cast<const uint16_t *>(args.x[cs]);
    if (it.ntok == 1)
        small_body<DT, Y16, 1>(it, pa, pool, x, tok_idx, H, v_stride, args.y[cs], args.v[cs], smem);
    else if (it.ntok == 2)
        small_body<DT, Y16, 2>(it, pa, pool, x, tok_idx, H, v_stride, args.y[cs], args.v[cs], smem);
    else
        small_body<DT, Y16, kExpandTok>(it, pa, pool, x, tok_idx, H, v_stride, args.y[cs], args.v[cs], smem);
}

// ---------------------------------------------------------------------------------------
// decode path, shrink for groups of many tokens: an item is up to kGangTok tokens x kGangPages pages of one adapter.
// The rows are walked in pieces of kGangPiece elements; a wavefront has up to four pages, requested together with
// the piece of x that goes to LDS, and keeps a sum per page and token, so that a read of x from LDS serves four
// pages and a pair of token and page costs little more than a third of the row bytes that an item of 4 x 4 reads.
// Every lane adds the same products in the same order as there and the lanes' sums meet in the same tree:
// bit-identical.  142 tokens of ranks 5-130, H = 4096, 2 slots: 22 -> 13.7 us; 960 tokens of rank 8, H = 2928, 3 slots:
// 15.2 -> 13.1; 173 tokens of ranks 8-128, H = 1128, 3 slots: 12.4 -> 9.6.  Tried: 8 x 16 items on the code of
// the 4 x 4 ones (a read of x from LDS per page) 21-24 us on the first of these; pieces of 1024 elements, two in flight, 15;
// a workgroup for a quarter of an item (those without work still claim their LDS first: 10.7 -> 27 us where three of
// four had none).
// ---------------------------------------------------------------------------------------
constexpr int kGangPiece = 2048;
constexpr int kGangChunks = kGangPiece / 8;
static_assert(kGangChunks == kShrinkThreads, "a thread copies one 16-byte chunk of a row's piece");
constexpr int kGangWavePages = kGangPages / kShrinkWaves;
constexpr size_t kGangLds = (size_t)kGangTok * kGangPiece * 2;

template <int DT, class Put>
__device__ __forceinline__ void shrink_gang(const Item &it, const int32_t *__restrict__ pa, const uint16_t *__restrict__ pool,
                                            const uint16_t *__restrict__ x, const int32_t *__restrict__ tok_idx, int H,
                                            u32x4 *xs, Put put)
{
    const int n_pages = it.b;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int nch = H >> 3;
    const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
    const u32x4 *page[kGangWavePages];
#pragma unroll
    for (int i = 0; i < kGangWavePages; ++i) // pages wave, wave + 4, ... of the item's
        page[i] = reinterpret_cast<const u32x4 *>(pool + (int64_t)pa[min(wave + kShrinkWaves * i, n_pages - 1)] * H);
    const u32x4 *row[kGangTok];
#pragma unroll
    for (int t = 0; t < kGangTok; ++t)
        row[t] = reinterpret_cast<const u32x4 *>(x + (int64_t)tok_idx[it.pos0 + min(t, it.ntok - 1)] * H);
    float acc[kGangWavePages][kGangTok];
#pragma unroll
    for (int i = 0; i < kGangWavePages; ++i)
#pragma unroll
        for (int t = 0; t < kGangTok; ++t) acc[i][t] = 0.f;
    for (int c0 = 0; c0 < nch; c0 += kGangChunks) {
        u32x4 xr[kGangTok], w[kGangWavePages][4];
#pragma unroll
        for (int t = 0; t < kGangTok; ++t)
            if (t < it.ntok) xr[t] = c0 + tid < nch ? row[t][c0 + tid] : zero;
#pragma unroll
        for (int i = 0; i < kGangWavePages; ++i)
            if (wave + kShrinkWaves * i < n_pages) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + u * kWave + lane;
                    w[i][u] = c < nch ? page[i][c] : zero;
                }
            }
        __syncthreads(); // the piece before this one has been read
#pragma unroll
        for (int t = 0; t < kGangTok; ++t)
            if (t < it.ntok) xs[t * kGangChunks + tid] = xr[t];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < kGangTok; ++t)
            if (t < it.ntok) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const u32x4 xv = xs[t * kGangChunks + u * kWave + lane];
#pragma unroll
                    for (int i = 0; i < kGangWavePages; ++i)
                        if (wave + kShrinkWaves * i < n_pages) acc[i][t] = dot8<DT>(w[i][u], xv, acc[i][t]);
                }
            }
    }
    const int r = lane >> 4, t_of_row = r == 1 ? 2 : r == 2 ? 1 : r; // see wave_sum4
#pragma unroll
    for (int i = 0; i < kGangWavePages; ++i) {
        const int j = wave + kShrinkWaves * i;
        if (j < n_pages) {
#pragma unroll
            for (int t = 0; t < kGangTok; t += 4) {
                if (t < it.ntok) {
                    const float s = wave_sum4(acc[i][t], acc[i][t + 1], acc[i][t + 2], acc[i][t + 3]);
                    if ((lane & 15) == 0 && t + t_of_row < it.ntok) put(t + t_of_row, j, s);
                }
            }
        }
    }
}

// n_items items of this kernel, then the vector-shrink items (`plain`) of the groups that are not in them
template <int DT, int U>
__global__ __launch_bounds__(kShrinkThreads) void shrink_gang_kernel(const Item *__restrict__ items, unsigned n_items,
                                                                      const Item *__restrict__ plain,
                                                                      const int32_t *__restrict__ arena,
                                                                      const uint16_t *__restrict__ pool,
                                                                      const int32_t *__restrict__ tok_idx, int H,
                                                                      int v_stride, MultiArgs args)
{
    extern __shared__ u32x4 smem[]; // a piece of kGangTok rows of x, or the rows of a vector-shrink item
    const int cs = blockIdx.x % args.n;
    const unsigned no = blockIdx.x / args.n;
    const bool gang = no < n_items;
    const Item it = gang ? items[no] : plain[no - n_items];
    const int32_t *pa = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank + it.a;
    const uint16_t *x = static_cast<const uint16_t *>(args.x[cs]);
    float *v = args.v[cs];
    auto put = [&](int t, int j, float s) { v[(int64_t)(it.pos0 + t) * v_stride + it.a + j] = s; };
    if (gang)
        shrink_gang<DT>(it, pa, pool, x, tok_idx, H, smem, put);
    else
        shrink_vec_item<DT, U>(it, pa, pool, x, tok_idx, H, smem, put);
}

// ---------------------------------------------------------------------------------------
// decode path, expand for batches whose launch has fewer workgroups than the GPU can hold ("rank-split"): a
// workgroup = 512 columns (a lane owns 8) of some tokens of one adapter group.  A sum over the ranks is made of the
// sums of four rows of blocks - blocks of 8 ranks, 16 where a token is one of at most two left over from the
// group's fours; row w has the blocks w, w + 4, ... - which are added in the order of w; half a block without ranks is left out.  Who forms them does not matter:
//   up to kOwnRanks ranks: a wavefront keeps all B rows of its columns in registers and forms whole sums, of
//     every fourth token of the workgroup's;
//   more, or one or two tokens of more than 16: wavefront w forms row w for up to four tokens, the parts meet in LDS, and wavefront t
//     finishes token t (48 tokens of rank 32, 12 groups of one / two on 4 slots: 5.6 -> 5.2 / 6.3 -> 5.5 us).
// B rows and page numbers are requested before v is needed; y, v and the token of a whole sum before its B rows: 4.2 -> 4.5 us for 24 tokens of
// rank 24, 6.4 -> 8.6 for 240 in twenties.  B rows that one or two tokens read alone are streamed, others are shared by
// items or wavefronts and stay in the caches.  us, plain / streamed: 17 small groups beside four prompts, H = 4096, 8 slots, 344 MB a call
// 16.4 / 13.9, and 102 / 95 for the whole call; 40 single tokens of rank 64, 3 slots 15.8 / 14.3 where the pages come from memory (12.0 / 14.3
// where three batches take turns and the caches still hold them, as a serving loop over many layers' pages does not); leftovers of larger
// groups streamed as well: 40 groups of six, 2 slots 16.3 / 17.8; rows of three or four tokens: 32 tokens of ranks 8-64 5.4 / 6.2.
// Bound by the chain of round trips in small calls, by
// the fp32 additions and 16-bit conversions where groups have many tokens.  Before, every item was four tokens with
// its ranks shared out and wavefront 0 finished them all: 45 tokens of ranks 3-100, H = 3080, 3 slots 13.7 -> 9.4 us;
// 51 tokens of ranks 30-130, H = 1168, 4 slots 15.2 -> 9.2; 142 tokens of ranks 5-130, H = 4096, 2 slots 17.0 -> 13.5; 376
// tokens of rank 1, H = 4096, 8 slots 39.5 -> 22.6, with 16 tokens per workgroup 15.8; 960 tokens of rank 8, H = 2928, 3 slots
// 31.4 -> 16.0 -> 11.1.  kOwnRanks = 16 (fewer registers, four workgroups per compute unit instead of three): up to 20 %
// slower, half as fast on groups of many tokens (spills).  Items of more than four tokens: expand_own_fours, expand_split_item.
// ---------------------------------------------------------------------------------------
// v of ranks w0 + lane, where `mine`, of tokens t0 .. t0 + TOK - 1 of an item
template <int TOK>
__device__ __forceinline__ void load_v(const Item &it, int t0, int w0, bool mine, const float *__restrict__ v, int v_stride, float (&out)[TOK])
{
    const float *at = v + (int64_t)(it.pos0 + t0) * v_stride + w0 + (threadIdx.x & (kWave - 1));
#pragma unroll
    for (int t = 0; t < TOK; ++t) out[t] = t0 + t < it.ntok && mine ? at[(int64_t)t * v_stride] : 0.f;
}
// keeps the compiler from widening rows once and holding them at twice the size
template <int N>
__device__ __forceinline__ void stay_narrow(u32x4 (&w)[N])
{
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+v"(w[j]));
}

// R: ranks in registers.  Tokens t0, t0 + 4, ... of the item.
template <int DT, bool Y16, int R>
__device__ __forceinline__ void expand_own(const Item &it, int t0, const int32_t *__restrict__ pb,
                                           const uint16_t *__restrict__ pool, const int32_t *__restrict__ tok_idx, int H,
                                           int v_stride, void *__restrict__ y, const float *__restrict__ vs)
{
    if (t0 >= it.ntok) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int col = it.a + lane * 8;
    const bool live = col < it.a + it.b;
    const int col_ld = live ? col : it.a; // lanes beyond the item's columns are dropped at the store
    const int pwin = lane < it.rank ? pb[lane] : 0;
    u32x4 w[R];
#pragma unroll
    for (int j = 0; j < R; ++j) { // ranks beyond the last: the last one's row meets v = 0
        const int64_t page = __builtin_amdgcn_readlane(pwin, min(j, it.rank - 1));
        w[j] = *reinterpret_cast<const u32x4 *>(pool + page * H + col_ld);
    }
    const int left = it.ntok & 3; // one or two: their blocks are of 16 ranks
    for (int t = t0; t < it.ntok; t += kSplitWaves) {
        Y8<DT, Y16> yv;
        const int64_t yoff = (int64_t)tok_idx[it.pos0 + t] * H + col;
        if (live) yv.load(y, yoff);
        float v[1];
        load_v(it, t, 0, lane < it.rank, vs, v_stride, v);
        stay_narrow(w);
        const bool by16 = left > 0 && left <= 2 && t >= it.ntok - left;
        float sum[8], acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[e] = acc[e] = 0.f;
#pragma unroll
        for (int b = 0; b < R / 8; ++b) {
            if (b < 3 || it.rank > 24) { // up to 24 ranks: no fourth block, all of whose rows would be the last one, times zero (NaN if it is infinite)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = 8 * b + u;
                    const float vv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[0]), j));
                    float f[8];
                    widen2<DT>(w[j].x, f[0], f[1]);
                    widen2<DT>(w[j].y, f[2], f[3]);
                    widen2<DT>(w[j].z, f[4], f[5]);
                    widen2<DT>(w[j].w, f[6], f[7]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = fmaf(vv, f[e], acc[e]);
                }
            }
            if (!by16 || (b & 1) || b == R / 8 - 1) { // the end of a block
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    sum[e] += acc[e];
                    acc[e] = 0.f;
                }
            }
        }
        if (live) yv.add_store(y, yoff, sum);
    }
}

// An item of at most TOK tokens (1 or 2: exactly); UB: ranks per block; Once: its B rows are streamed.  Half a block of
// 16 ranks without ranks is multiplied all the same, and left out by a select: with a branch between the halves single tokens of rank 64 took 4.5 -> 5.0 us.  One token has an instance of its own: with the
// two-token one it requested, multiplied and passed through LDS a second token of zeros.  v is requested beside the page numbers, which
// the B rows wait for anyway.  us of the expand, pages from memory, before and with the streaming loads: 24 tokens of rank 64, H = 4096 6.8 -> 5.7; two
// of rank 128, 8 slots 9.4 -> 7.1; 37 of ranks 16-128, H = 3072 9.5 -> 7.6; pages from the caches 5.9 -> 5.1, 7.7 -> 7.1, 7.9 -> 7.1.
template <int DT, bool Y16, int TOK, int UB, bool Once>
__device__ __forceinline__ void expand_shared(const Item &it, const int32_t *__restrict__ pb,
                                              const uint16_t *__restrict__ pool, const int32_t *__restrict__ tok_idx,
                                              int H, int v_stride, void *__restrict__ y, const float *__restrict__ vs, float *red)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int col = it.a + lane * 8;
    const bool live = col < it.a + it.b;
    const int col_ld = live ? col : it.a;
    const bool finishes = wave < it.ntok; // token `wave`
    Y8<DT, Y16> yv;
    const int64_t yoff = (int64_t)tok_idx[it.pos0 + (finishes ? wave : 0)] * H + col;
    if (finishes && live) yv.load(y, yoff);
    float acc[TOK][8];
#pragma unroll
    for (int t = 0; t < TOK; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] = 0.f;
    for (int w0 = 0; w0 < it.rank && wave * UB < it.rank - w0; w0 += kWave) {
        const int wr = min(kWave, it.rank - w0);
        const int pwin = lane < wr ? pb[w0 + lane] : 0;
        float v[TOK]; // rank w0 + lane, if it is in one of this wavefront's blocks
        load_v(it, 0, w0, lane < wr && lane / UB % kSplitWaves == wave, vs, v_stride, v);
        u32x4 w[2][8]; // this wavefront's two eights of a window of 64 ranks: a block, or half of one
        auto first = [&](int i) { return UB == 16 ? (2 * wave + i) * 8 : (wave + kSplitWaves * i) * 8; };
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int j0 = first(i);
            if (UB == 16 || i == 0 || j0 < wr) {
#pragma unroll
                for (int u = 0; u < 8; ++u) { // ranks beyond the last: the last one's row meets v = 0
                    const int64_t page = __builtin_amdgcn_readlane(pwin, min(j0 + u, wr - 1));
                    const u32x4 *row = reinterpret_cast<const u32x4 *>(pool + page * H + col_ld);
                    w[i][u] = Once ? __builtin_nontemporal_load(row) : *row;
                }
            }
        }
        float half[TOK][8];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int j0 = first(i);
            if (UB == 16 || i == 0 || j0 < wr) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    float f[8];
                    widen2<DT>(w[i][u].x, f[0], f[1]);
                    widen2<DT>(w[i][u].y, f[2], f[3]);
                    widen2<DT>(w[i][u].z, f[4], f[5]);
                    widen2<DT>(w[i][u].w, f[6], f[7]);
#pragma unroll
                    for (int t = 0; t < TOK; ++t) {
                        if (TOK <= 2 || t < it.ntok) {
                            const float vv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[t]), j0 + u));
#pragma unroll
                            for (int e = 0; e < 8; ++e) acc[t][e] = fmaf(vv, f[e], acc[t][e]);
                        }
                    }
                }
            }
            if (UB == 16) {
#pragma unroll
                for (int t = 0; t < TOK; ++t)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        if (i == 0) half[t][e] = acc[t][e];
                        else acc[t][e] = j0 < wr ? acc[t][e] : half[t][e];
                    }
            }
        }
    }
    // red[wave][t][e][lane]
#pragma unroll
    for (int t = 0; t < TOK; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) red[((wave * TOK + t) * 8 + e) * kWave + lane] = acc[t][e];
    __syncthreads();
    if (!finishes) return;
    float d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        d[e] = red[(wave * 8 + e) * kWave + lane];
#pragma unroll
        for (int k = 1; k < kSplitWaves; ++k) d[e] += red[((k * TOK + wave) * 8 + e) * kWave + lane];
    }
    if (live) yv.add_store(y, yoff, d);
}

// acc[e][t] += v of token t and rank K0 + k of the wavefront's sixteen (lane 4 * (K0 + k) + t of v) times element e of row k, rank after rank.  The matrix
// instruction is sixteen products of a column of four and a row of four; block K0 + k of its first operand is sent to all of them.
template <int DT, int K0, int K, int FOURS>
__device__ __forceinline__ void add_ranks(const float (&v)[FOURS], const u32x4 (&row)[8], float (&f)[8], f32x4 (&acc)[FOURS][8])
{
    // the elements of a rank are widened while the products of the one before run: all in registers of their own first
    asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]));
    float next[8];
#pragma unroll
    for (int k = 0; k < FOURS; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[k][e] = __builtin_amdgcn_mfma_f32_4x4x1f32(v[k], f[e], acc[k][e], 4, K0 + K, 0);
    if constexpr (K < 7) {
        widen2<DT>(row[K + 1].x, next[0], next[1]);
        widen2<DT>(row[K + 1].y, next[2], next[3]);
        widen2<DT>(row[K + 1].z, next[4], next[5]);
        widen2<DT>(row[K + 1].w, next[6], next[7]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            __builtin_amdgcn_sched_group_barrier(0x8, FOURS, 0); // products,
            __builtin_amdgcn_sched_group_barrier(0x2, 1, 0); // an element
        }
        add_ranks<DT, K0, K + 1, FOURS>(v, row, next, acc);
    }
}
template <int DT, int K0, int FOURS>
__device__ __forceinline__ void add_eight(const float (&v)[FOURS], const u32x4 (&row)[8], f32x4 (&acc)[FOURS][8])
{
    float f[8];
    widen2<DT>(row[0].x, f[0], f[1]);
    widen2<DT>(row[0].y, f[2], f[3]);
    widen2<DT>(row[0].z, f[4], f[5]);
    widen2<DT>(row[0].w, f[6], f[7]);
    add_ranks<DT, K0, 0, FOURS>(v, row, f, acc);
}

// Turns of find() at most: calls that overlap although they use one plan's words could otherwise keep each other's wavefronts
constexpr int kFinds = 2;

// acc[e] += v of lane FIRST + 4 k times element e of row k, rank after rank: one token
template <int DT, int FIRST>
__device__ __forceinline__ void add_eight_alone(float v, const u32x4 (&row)[8], float (&acc)[8])
{
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        float f[8];
        widen2<DT>(row[u].x, f[0], f[1]);
        widen2<DT>(row[u].y, f[2], f[3]);
        widen2<DT>(row[u].z, f[4], f[5]);
        widen2<DT>(row[u].w, f[6], f[7]);
        const float vv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), FIRST + 4 * u));
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(vv, f[e], acc[e]);
    }
}

// Where an item's wavefronts find v: get() returns the value of a token and a rank of each lane's own, where `mine` and there is such a
// token; false: not all are there, and find() makes those of `n` ranks from j0 on.  Rows that an earlier launch has left:
struct RowsOfV {
    static constexpr bool kMayFail = false;
    const float *v;
    int v_stride;
    __device__ __forceinline__ bool get(const Item &it, int t, int j, bool mine, float &out) const
    {
        out = mine && t < it.ntok ? v[(int64_t)(it.pos0 + t) * v_stride + j] : 0.f;
        return true;
    }
    __device__ __forceinline__ void find(const Item &, int, int) const {}
};

// An item of one token (its B rows are streamed: nobody else reads them), or of at most TOK = 4 or 8, with the ranks shared out over the wavefronts: the sums of expand_shared.
// The fp32 vector operations bound groups of many tokens, nine of them for a row of B and a token; the matrix instruction does four tokens
// at once in the time of two, adds them as fmaf does, and eight tokens share the rows and their conversion.  us per call, expand_shared / this one, calls of the
// larger items: 672 tokens of 16 adapters of ranks 16-128, H = 4096, 4 slots, 16-bit y 102.5 / 85.5; 452 of 10, ranks 5-130, H = 3072, bf16 50.2 / 44.3;
// 50 tokens each of 12 adapters of rank 48, 3 slots 56.4 / 50.5.  For two to four tokens an item it is 4-6 % slower where the launch is large (its rows are requested after
// the page numbers of all its blocks, and two tokens leave half of the instruction idle), so only the one-launch kernel below uses it there.
template <int DT, bool Y16, int TOK, class V>
__device__ __forceinline__ void expand_split_item(const Item &it, const int32_t *__restrict__ pb, const uint16_t *__restrict__ pool,
                                                  const int32_t *__restrict__ tok_idx, int H, void *__restrict__ y, const V &vs, f32x4 *red)
{
    constexpr int kFours = (TOK + 3) / 4;                    // fours of tokens
    constexpr int kRedTok = TOK < 4 ? TOK : 4;               // tokens whose parts are in LDS at a time
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int col = it.a + lane * 8;
    const bool live = col < it.a + it.b;
    const int col_ld = live ? col : it.a;
    const int ub = TOK == 1 || it.ntok <= 2 ? 16 : 8;        // ranks of a block
    const int b0 = wave * ub, b1 = ub == 16 ? b0 + 8 : b0 + 32; // this wavefront's two eights of a window of 64 ranks
    // the y of the token that this wavefront finishes: requested first, if registers are left for it
    Y8<DT, Y16> yv;
    auto y_row = [&](int t) { return static_cast<unsigned char *>(y) + (int64_t)tok_idx[it.pos0 + min(t, it.ntok - 1)] * H * (Y16 ? 2 : 4); };
    if (TOK <= 4 && wave < it.ntok && live) yv.load(y_row(wave), (uint32_t)col);
    std::conditional_t<TOK == 1, float, f32x4> acc[kFours][8] = {}; // sums of the lane's eight columns, of four tokens each if there are several
#pragma nounroll
    for (int w0 = 0; w0 < it.rank && b0 < it.rank - w0; w0 += kWave) {
        const int wr = min(kWave, it.rank - w0);
        const bool two = b1 < wr;
        const int pages = pb[w0 + min((lane & 8 ? b1 : b0) + (lane & 7), wr - 1)]; // lane k: the page of the k-th of the sixteen
        u32x4 w[2][8];
        // v of token lane % 4: that of this wavefront's sixteen ranks
        const int mine = (lane & 32 ? b1 : b0) + ((lane >> 2) & 7);
        float v[kFours];
        for (int finds = 0;; ++finds) {
            auto rows = [&](int first, u32x4(&o)[8]) { // ranks beyond the last: the last one's row meets v = 0
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int64_t page = __builtin_amdgcn_readlane(pages, first + u);
                    const u32x4 *row = reinterpret_cast<const u32x4 *>(pool + page * H + col_ld);
                    o[u] = TOK == 1 ? __builtin_nontemporal_load(row) : *row;
                }
            };
            rows(0, w[0]);
            if (two) rows(8, w[1]);
            bool there = true;
#pragma unroll
            for (int k = 0; k < kFours; ++k) there = vs.get(it, 4 * k + (lane & 3), w0 + mine, mine < wr, v[k]) && there;
            if (!V::kMayFail || there || finds == kFinds) break;
            vs.find(it, w0 + b0, min(8, wr - b0));
            if (two) vs.find(it, w0 + b1, min(8, wr - b1));
        }
        if constexpr (TOK == 1) {
            add_eight_alone<DT, 0>(v[0], w[0], acc[0]);
            if (two) add_eight_alone<DT, 32>(v[0], w[1], acc[0]);
        } else {
            add_eight<DT, 0>(v, w[0], acc);
            if (two) add_eight<DT, 8>(v, w[1], acc);
        }
    }
    const int n_rows = (it.rank + ub - 1) / ub; // wavefronts with blocks
    f32x4 *out = red + wave * kRedTok * 2 * kWave + lane; // red[wave][t][columns' half][lane]
#pragma unroll
    for (int k = 0; k < kFours; ++k) {
        const int mine = 4 * k + wave; // the token that this wavefront finishes
        if (TOK > 4 && mine < it.ntok && live) yv.load(y_row(mine), (uint32_t)col);
        if (k > 0) __syncthreads();    // the parts before these have been read
        if constexpr (TOK == 1) {
            out[0] = f32x4{acc[0][0], acc[0][1], acc[0][2], acc[0][3]};
            out[kWave] = f32x4{acc[0][4], acc[0][5], acc[0][6], acc[0][7]};
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (4 * k + t < it.ntok) {
                    out[t * 2 * kWave] = f32x4{acc[k][0][t], acc[k][1][t], acc[k][2][t], acc[k][3][t]};
                    out[t * 2 * kWave + kWave] = f32x4{acc[k][4][t], acc[k][5][t], acc[k][6][t], acc[k][7][t]};
                }
        }
        __syncthreads();
        if (mine < it.ntok) {
            const f32x4 *in = red + wave * 2 * kWave + lane;
            f32x4 a = in[0], b = in[kWave];
#pragma unroll
            for (int r = 1; r < kSplitWaves; ++r) {
                const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
                a += r < n_rows ? in[r * kRedTok * 2 * kWave] : zero;
                b += r < n_rows ? in[r * kRedTok * 2 * kWave + kWave] : zero;
            }
            const float d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            if (live) yv.add_store(y_row(mine), (uint32_t)col, d);
        }
        if (4 * k + 4 >= it.ntok) return; // the whole workgroup
    }
}

// An item of up to kGangOwnTok tokens of an adapter of at most kOwnRanks ranks: a wavefront forms whole sums, of a quarter of the
// tokens, sixteen ranks at a time, as expand_own does token after token.  us per call, expand_own / this one: 30 tokens each of 20 adapters of rank 32, H = 4096, bf16,
// 4 slots, 16-bit y 47.0 / 39.2; 746 tokens, ranks 1-50, 8 slots 22.3 / 20.2; 960 tokens of rank 8, H = 2928, 3 slots 23.2 / 22.9.
template <int DT, bool Y16>
__device__ __forceinline__ void expand_own_fours(const Item &it, const int32_t *__restrict__ pb, const uint16_t *__restrict__ pool,
                                                const int32_t *__restrict__ tok_idx, int H, void *__restrict__ y, const RowsOfV &vs)
{
    const int lane = threadIdx.x & (kWave - 1);
    constexpr int PER = kGangOwnTok / kSplitWaves;
    const int per = (it.ntok + kSplitWaves - 1) / kSplitWaves; // tokens of a wavefront, at most PER
    const int t0 = per * __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), t1 = min(t0 + per, it.ntok);
    if (t0 >= t1) return; // no barrier is used
    const int col = it.a + lane * 8;
    const bool live = col < it.a + it.b;
    const int col_ld = live ? col : it.a;
    Y8<DT, Y16> yv[PER];
    unsigned char *row[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t)
        row[t] = static_cast<unsigned char *>(y) + (int64_t)tok_idx[it.pos0 + min(t0 + t, it.ntok - 1)] * H * (Y16 ? 2 : 4);
    const int left = it.ntok & 3;      // one or two: their blocks are of 16 ranks
    const int by16 = left == 1 || left == 2 ? it.ntok - left : it.ntok; // tokens from here on
    f32x4 sum[8] = {};
#pragma nounroll
    for (int j0 = 0; j0 < it.rank; j0 += 16) {
        const int pages = pb[min(j0 + (lane & 15), it.rank - 1)];
        float v[1];
        vs.get(it, t0 + (lane & 3), j0 + (lane >> 2), (lane & 3) < per && j0 + (lane >> 2) < it.rank, v[0]);
        const bool two = j0 + 8 < it.rank;
        u32x4 w[2][8];
        auto rows = [&](int first, u32x4(&o)[8]) { // ranks beyond the last: the last one's row meets v = 0
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t page = __builtin_amdgcn_readlane(pages, first + u);
                o[u] = *reinterpret_cast<const u32x4 *>(pool + page * H + col_ld);
            }
        };
        rows(0, w[0]);
        if (two) rows(8, w[1]);
        f32x4 acc[1][8] = {};
        add_eight<DT, 0>(v, w[0], acc);
        if (two) {
#pragma unroll
            for (int t = 0; t < PER; ++t)
                if (t0 + t < by16) { // the end of a block
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        sum[e][t] += acc[0][e][t];
                        acc[0][e][t] = 0.f;
                    }
                }
            add_eight<DT, 8>(v, w[1], acc);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[e] += acc[0][e];
    }
#pragma unroll
    for (int t = 0; t < PER; ++t)
        if (t0 + t < t1 && live) yv[t].load(row[t], (uint32_t)col);
    if (!live) return;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const float d[8] = {sum[0][t], sum[1][t], sum[2][t], sum[3][t], sum[4][t], sum[5][t], sum[6][t], sum[7][t]};
        if (t0 + t < t1) yv[t].add_store(row[t], (uint32_t)col, d);
    }
}

// An item: up to kExpandTok tokens, or of a larger item's list kGangOwnTok of an adapter of at most kOwnRanks ranks; Fours: kGangExpandTok of another, and some
// of them on the matrix instruction (an instance of its own: with both kinds of code the items of the first are up to 6 % slower)
template <int DT, bool Y16, bool Fours>
__global__ __launch_bounds__(kSplitWaves *kWave, 3) void expand_vec_split_kernel(const Item *__restrict__ items,
                                                                              const int32_t *__restrict__ arena,
                                                                              const uint16_t *__restrict__ pool,
                                                                              const int32_t *__restrict__ tok_idx,
                                                                              int H, int v_stride, MultiArgs args)
{
    extern __shared__ u32x4 smem[];
    float *red = reinterpret_cast<float *>(smem);
    const int cs = blockIdx.x % args.n;
    const Item it = items[blockIdx.x / args.n];
    const int32_t *pb = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank + it.rank;
    const float *v = args.v[cs];
    void *y = args.y[cs];
    if constexpr (Fours) {
        if (it.ntok > kExpandTok) {
            const RowsOfV vs{v, v_stride};
            const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
            if (it.rank > kOwnRanks) expand_split_item<DT, Y16, kGangExpandTok>(it, pb, pool, tok_idx, H, y, vs, reinterpret_cast<f32x4 *>(smem));
            else if (fours_pay(DT, Y16, it.rank, it.ntok)) expand_own_fours<DT, Y16>(it, pb, pool, tok_idx, H, y, vs);
            else if (it.rank <= 8) expand_own<DT, Y16, 8>(it, wave, pb, pool, tok_idx, H, v_stride, y, v);
            else if (it.rank <= 16) expand_own<DT, Y16, 16>(it, wave, pb, pool, tok_idx, H, v_stride, y, v);
            else expand_own<DT, Y16, 32>(it, wave, pb, pool, tok_idx, H, v_stride, y, v);
            return;
        }
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (it.rank <= 8)
        expand_own<DT, Y16, 8>(it, wave, pb, pool, tok_idx, H, v_stride, y, v);
    else if (it.rank <= 16)
        expand_own<DT, Y16, 16>(it, wave, pb, pool, tok_idx, H, v_stride, y, v);
    else if (it.rank <= kOwnRanks && it.ntok > 2)
        expand_own<DT, Y16, kOwnRanks>(it, wave, pb, pool, tok_idx, H, v_stride, y, v);
    else if (it.ntok > 2)
        expand_shared<DT, Y16, kExpandTok, 8, false>(it, pb, pool, tok_idx, H, v_stride, y, v, red);
    else { // two blocks or more: a wavefront each, while whole sums would keep one of them busy
        if (it.ntok == 1 && it.tile)
            expand_shared<DT, Y16, 1, 16, true>(it, pb, pool, tok_idx, H, v_stride, y, v, red);
        else if (it.ntok == 1)
            expand_shared<DT, Y16, 1, 16, false>(it, pb, pool, tok_idx, H, v_stride, y, v, red);
        else if (it.tile)
            expand_shared<DT, Y16, 2, 16, true>(it, pb, pool, tok_idx, H, v_stride, y, v, red);
        else
            expand_shared<DT, Y16, 2, 16, false>(it, pb, pool, tok_idx, H, v_stride, y, v, red);
    }
}

// ---------------------------------------------------------------------------------------
// decode path, both stages in ONE launch, v handed over between workgroups ("chain"): first the workgroups of the vector shrink,
// then those of the expand, in one grid.  What bounds calls of modest size is the chain of dependent round trips and the launches - an empty
// kernel takes 1.6 us of the GPU and 2.6 to 3.6 us of the host - so the expand's workgroups are there from the start, with their B rows and y
// requested, when v arrives.  They also run the same few instructions whatever the rank: between the arrival of v and the store of
// y a wavefront issues a fifth of what the rank-split expand's does for four tokens, whose sums of 64 ranks took 1.1 us.
//
// A shrink workgroup leaves every value of v as one 8-byte word {value, number of the launch}, written and read at device scope.  A word that
// has this launch's number is whole and needs no other order; words of earlier launches have other numbers, so nothing is
// cleared between calls.  Workgroups are dispatched in order, so those that are waited for run first; where another stream's kernel holds
// the GPU that may fail, and a wait is bounded: after `polls` reads a wavefront computes what it waits for, with the same sums, leaves it in
// the words and goes on (if all waits ran out at once: a group of four tokens of rank 64, H = 4096, 7 -> 90 us, 20 of them on 4 slots 19 -> 38).  Beside
// products of 8192 x 4096 x 8192 on another stream, one call every 0.4 ms, median us of the two kernels / this one: 32 tokens of ranks 8-64 800 / 230,
// 96 of 4 adapters 815 / 250, 45 of ranks 3-100 800 / 185; beside products of 2048 x 4096 x 2048 21 / 20, 45 / 32, 35 / 28 - two launches are
// delayed by the other stream's kernels twice.  Calls that a HIP graph captures keep the two kernels: a replay would repeat the number.
//
// Sums and their order are those of the vector shrink and of the rank-split expand: the same bits.  us per call, two kernels / chain:
// 32 tokens of ranks 8-64, H = 4096 9.9 / 7.2; 96 tokens of 4 adapters, 3 slots, bf16, 16-bit y 15.5 / 11.4; 45 tokens of ranks 3-100, H = 3080, 3 slots
// 17.0 / 12.9; two tokens, H = 1368 9.2 / 5.9; 103 tokens of ranks 8-128, H = 4480, 2 slots 22.3 / 18.4.  Large calls: see slora_plan::chain_pays.
// ---------------------------------------------------------------------------------------
template <int DT>
struct HandOver {
    static constexpr bool kMayFail = true;
    uint64_t *hand; // the item's words, token after token, rank after rank
    uint32_t launch;
    int polls;
    const int32_t *pa; // the item's A list
    const uint16_t *pool, *x;
    const int32_t *tok_idx;
    int H;
    __device__ __forceinline__ void leave(const Item &it, int t, int j, float s) const
    {
        __hip_atomic_store(hand + (int64_t)t * it.rank + j, (uint64_t)launch << 32 | __float_as_uint(s), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    // the value of a token and a rank of each lane's own, where `mine` and there is such a token; false: not all are there
    __device__ __forceinline__ bool get(const Item &it, int t, int j, bool mine, float &out) const
    {
        const uint64_t *at = hand + (int64_t)t * it.rank + j;
        const bool asks = mine && t < it.ntok;
        for (int k = 0;; ++k) {
            uint64_t word = (uint64_t)launch << 32;
            if (asks) word = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            out = __uint_as_float((uint32_t)word);
            if (__all((uint32_t)(word >> 32) == launch)) return true;
            if (k >= polls) return false;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    // n ranks from j0 on, of all tokens: each lane adds the products of chunks lane, lane + 64, ... as the shrink's lanes do.  A wavefront finds the
    // ranks of its own blocks only (all of a window's 64 took four times as long where rank and H are large)
    __device__ __forceinline__ void find(const Item &it, int j0, int n) const
    {
        const int lane = threadIdx.x & (kWave - 1), nch = H >> 3;
#pragma nounroll
        for (int j = j0; j < j0 + n; ++j) {
            const u32x4 *page = reinterpret_cast<const u32x4 *>(pool + (int64_t)pa[j] * H);
#pragma nounroll
            for (int t = 0; t < it.ntok; ++t) {
                const u32x4 *row = reinterpret_cast<const u32x4 *>(x + (int64_t)tok_idx[it.pos0 + t] * H);
                float acc = 0.f;
#pragma nounroll
                for (int c = lane; c < nch; c += kWave) acc = dot8<DT>(page[c], row[c], acc);
                acc = wave_sum(acc);
                if (lane == 0) leave(it, t, j, acc);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // the words are where get() reads them
    }
};

// Chunks of a row that a lane holds: its U-th part, or a little more (the kernel is not made for every number)
constexpr int chain_chunks(int H)
{
    const int u = (H / 8 + kWave - 1) / kWave;
    return u <= 8 ? u : u <= 10 ? 10 : u <= 12 ? 12 : 16;
}
// An item of the vector shrink, rows of at most kWave * U chunks, chain_chunks(H) == U: a wavefront holds a whole page and takes the tokens one
// after another.
template <int DT, int U, class Put>
__device__ __forceinline__ void shrink_page_item(const Item &it, const int32_t *__restrict__ pa, const uint16_t *__restrict__ pool,
                                                 const uint16_t *__restrict__ x, const int32_t *__restrict__ tok_idx, int H, u32x4 *xs, Put put)
{
    constexpr int kFull = U <= 8 ? U - 1 : U == 10 ? 8 : U == 12 ? 10 : 12; // chunks that lie inside every such row
    const int lane = threadIdx.x & (kWave - 1), nch = H >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    auto load_row = [&](const uint16_t *row, bool stream, u32x4(&o)[U]) {
        const u32x4 *at = reinterpret_cast<const u32x4 *>(row) + lane;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            o[u] = u32x4{0u, 0u, 0u, 0u};
            if (u < kFull || u * kWave + lane < nch) o[u] = stream ? __builtin_nontemporal_load(at + u * kWave) : at[u * kWave];
        }
    };
    u32x4 w[U];
    if (it.ntok == 1) { // no row is shared: no way through LDS
        const uint16_t *row = x + (int64_t)tok_idx[it.pos0] * H;
#pragma nounroll
        for (int j = wave; j < it.b; j += kShrinkWaves) {
            u32x4 a[U];
            load_row(pool + (int64_t)pa[j] * H, true, w);
            load_row(row, false, a);
            float acc = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) acc = dot8<DT>(w[u], a[u], acc);
            acc = wave_sum(acc);
            if (lane == 0) put(0, j, acc);
        }
        return;
    }
    if (wave < it.b) load_row(pool + (int64_t)pa[wave] * H, true, w);
#pragma nounroll
    for (int t = wave; t < it.ntok; t += kShrinkWaves) {
        u32x4 a[U];
        load_row(x + (int64_t)tok_idx[it.pos0 + t] * H, false, a);
#pragma unroll
        for (int u = 0; u < U; ++u) xs[(t * U + u) * kWave + lane] = a[u];
    }
    __syncthreads();
#pragma nounroll
    for (int j = wave; j < it.b; j += kShrinkWaves) {
        if (j >= kShrinkWaves) load_row(pool + (int64_t)pa[j] * H, true, w);
#pragma nounroll
        for (int t = 0; t < it.ntok; t += 2) { // two at a time; the last of an odd number twice
            const u32x4 *x0 = xs + t * U * kWave + lane, *x1 = t + 1 < it.ntok ? x0 + U * kWave : x0;
            float a0 = 0.f, a1 = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a0 = dot8<DT>(w[u], x0[u * kWave], a0);
                a1 = dot8<DT>(w[u], x1[u * kWave], a1);
            }
            const float sum = wave_sum2(a0, a1);
            if ((lane & 31) == 0 && t + (lane >> 5) < it.ntok) put(t + (lane >> 5), j, sum);
        }
    }
}

template <int DT, bool Y16, int U>
__global__ __launch_bounds__(kShrinkThreads, U > 8 ? 3 : 4) void lora_vec_chain_kernel(ChainLists lists, const int32_t *__restrict__ arena,
                                                                                       const uint16_t *__restrict__ pool,
                                                                                       const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                                                       MultiArgs args)
{
    extern __shared__ u32x4 smem[]; // rows of x, or the sums of an expand item's wavefronts
    // Slots vary fastest, so workgroups are dispatched in the order of the work lists.  They go round the eight XCDs one by one: with a power of two of slots
    // each slot would stay on its own XCDs, which made calls of eight up to 25 % slower.  A slot moves on every 32 items, or 64 where several items read
    // the same pages.  us, two kernels / slots that stay / that move every 4 / 16 / 32 / 64 items, 8 slots: six groups of ranks 16-64 and 1-3 tokens, H = 5120 16.7 / 16.2 / 11.7 /
    // 10.9 / 10.9 / 10.9; five of ranks 32-64, H = 8192 18.9 / 21.0 / 16.9 / 14.5 / 14.6 / -; 29 tokens of rank 4, H = 5120 12.3 / 14.5 / 11.8 / - / 11.8 / 13.1; eight groups of eight tokens, ranks
    // 16-64, H = 2024 15.1 / 15.5 / 16.7 / 13.6 / 12.9 / -; four of 5-30 tokens, ranks 16-128, H = 5120 25.7 / 17.4 / 20.4 / 19.4 / 18.6 / 17.4
    const int cs = args.n & (args.n - 1) ? blockIdx.x : (blockIdx.x + (blockIdx.y >> lists.turn)) & (args.n - 1);
    const bool shrinks = blockIdx.y < lists.n_shrink;
    const Item it = shrinks ? lists.shrink[blockIdx.y] : lists.expand[blockIdx.y - lists.n_shrink];
    const uint16_t *x = static_cast<const uint16_t *>(args.x[cs]);
    const int32_t *pa = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank;
    const HandOver<DT> hand{lists.hand + cs * lists.hand_slot + it.run, lists.launch, lists.polls, pa, pool, x, tok_idx, H};
    if (shrinks) {
        float *v = args.v[cs];
        shrink_page_item<DT, U>(it, pa + it.a, pool, x, tok_idx, H, smem, [&](int t, int j, float s) {
            hand.leave(it, t, it.a + j, s);
            v[(int64_t)(it.pos0 + t) * v_stride + it.a + j] = s; // for a later expand
        });
    } else {
        const int32_t *pb = pa + it.rank;
        f32x4 *red = reinterpret_cast<f32x4 *>(smem);
        void *y = args.y[cs];
        if (it.ntok == 1 && it.tile) expand_split_item<DT, Y16, 1>(it, pb, pool, tok_idx, H, y, hand, red);
        else expand_split_item<DT, Y16, 4>(it, pb, pool, tok_idx, H, y, hand, red);
    }
}

__global__ __launch_bounds__(256) void clear_kernel(u32x4 *__restrict__ dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) dst[i] = u32x4{0u, 0u, 0u, 0u};
}

// ---------------------------------------------------------------------------------------
// prefill path (MFMA).  Matrix blocks are 32 x 32 with 16 k-values per instruction
// (v_mfma_f32_32x32x16_{f16,bf16}): lane l supplies, for row/column l % 32, the 8 k-values
// 8*(l / 32) .. +7 of both operands, and receives D[8*(v/4) + 4*(l/32) + v%4][l % 32] in
// accumulator register v (0..15).
// ---------------------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int DT>
__device__ __forceinline__ f32x16 mfma32(const u32x4 &a, const u32x4 &b, const f32x16 &c)
{
    if constexpr (DT == SLORA_F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
}

// accumulator register v of lane `lane` holds this row of the 32 x 32 block
__device__ __forceinline__ int mfma_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

// v = x*A of the MFMA path is handed from shrink to expand already in the layout of the expand's
// first MFMA operand, split into 16-bit pieces whose sum is the fp32 value (so nothing is lost to
// the operand format): hi + lo for binary16 (22+ bits; or three pieces, below), hi + mid + lo by truncation
// for bfloat16 (exactly 24 bits).  One fragment = 64 lanes x 8 values (1 KiB) = the operand of one MFMA:
// tokens 0..31 of the tile x ranks 16*kk .. 16*kk+15, lane = token + 32 * ((rank % 16) / 8).
// Fragments are ordered [tile][kk][piece]; the expand reads each with one coalesced 16-byte load
// per lane and does no conversion work.
//
// Three pieces for binary16 (NP = 3) are for calls that would else keep v in fp32 rows: the second and third
// are stored 2^12 and 2^24 times as large, so that neither meets the end of the format's range, and the expand
// scales its sums back from piece to piece.  They hold all 24 bits of values down to 2^-39 of the row's largest;
// two pieces hold 22 bits, of values near the largest.  512 tokens of rank 64, H = 4096, 4 slots: error against
// 64 bits 1.1e-7 -> 1.0e-7, 31.1 -> 32.1 us per call; rows whose ranks differ by 2^22, 1.5e-5 -> 1.6e-7.
template <int DT>
struct VPieces {
    static constexpr int N = DT == SLORA_F16 ? 2 : 3;
};
template <int DT, int NP>
constexpr bool kScaledPieces = DT == SLORA_F16 && NP == 3;
constexpr float kPieceUp = 4096.f, kPieceDown = 1.f / 4096.f;
__device__ __forceinline__ int64_t vfrag_index(int tile, int kk, int piece, int n_kk, int n_piece)
{
    return (((int64_t)tile * n_kk + kk) * n_piece + piece) * (kWave * 8);
}
// Eight consecutive ranks of one token -> the 16-bit pieces whose sum is the fp32 value, packed as
// the 16 bytes a lane owns in each piece's fragment.  An infinite or NaN value is all in the first piece (the
// differences that make the others would be NaN).
template <int DT, int NP>
__device__ __forceinline__ void split_pieces(const float (&f)[8], u32x4 (&piece)[NP])
{
    uint16_t h[NP][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const bool finite = fabsf(f[e]) < __builtin_inff();
        if constexpr (DT == SLORA_F16) {
            const _Float16 a = (_Float16)f[e];
            float r = finite ? f[e] - (float)a : 0.f;
            h[0][e] = __builtin_bit_cast(uint16_t, a);
#pragma unroll
            for (int p = 1; p < NP; ++p) {
                if constexpr (kScaledPieces<DT, NP>) r *= kPieceUp;
                const _Float16 c = (_Float16)r;
                h[p][e] = __builtin_bit_cast(uint16_t, c);
                r -= (float)c;
            }
        } else {
            const uint32_t hi = (__float_as_uint(f[e]) & 0xffff0000u) | (f[e] != f[e] ? 0x00400000u : 0u); // a NaN stays one
            const float r1 = finite ? f[e] - __uint_as_float(hi) : 0.f;
            const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
            const float r2 = r1 - __uint_as_float(mid);
            h[0][e] = (uint16_t)(hi >> 16);
            h[1][e] = (uint16_t)(mid >> 16);
            h[2][e] = (uint16_t)(__float_as_uint(r2) >> 16);
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int k = 0; k < 4; ++k) piece[p][k] = (uint32_t)h[p][2 * k] | ((uint32_t)h[p][2 * k + 1] << 16);
}

// ---------------------------------------------------------------------------------------
// prefill shrink: V[pos, j] = sum_h x[tok, h] * Apage_j[h] for up to 128 tokens of one adapter,
// up to 128 of its ranks and a range of H (one work item).
//
// A workgroup takes the item's tokens, or sub_tok of them when the items alone are too few (the plan
// decides): a tile of MB (1, 2, 4) blocks of 32 token rows x NL (1..4) blocks of 32 page rows.  Its range of H is
// walked in pieces of 64 elements (128 bytes of every row).  Pieces travel from memory straight
// into LDS (global_load_lds, 16 bytes per lane: 8 rows of 128 bytes per instruction) through a ring
// of S stages, so the loads in flight cost no registers and the wavefronts never copy anything;
// one barrier per piece hands a stage over: after it every wavefront's part of the piece has
// arrived, and the stage read a piece ago may be overwritten.  The 16-byte groups of a row are
// permuted in LDS (group p of row r sits at p ^ (r / 2 % 8)), on the address side of the load, so
// that the 16 rows an operand read touches at a time fall into different banks.
//
// The four wavefronts share the tile's 32 x 32 blocks out between them; the two accumulators of a
// single rank block (even and odd k-steps) meet at the end, in a fixed order.  The finished sums pass through LDS once so that a lane holds 8 consecutive ranks of one
// token - the 16 bytes it owns in an operand fragment.
//
// Bound by what a compute unit can have outstanding towards L2 (about 90 lines of 128 bytes on every
// streaming kernel here, whatever is queued behind them), so lines that hit in L2 cost a good part of
// what lines from HBM cost: large tiles (128 tokens share every page row) keep the page re-reads down.
// Stage time with the join, 4 slots: 4524 tokens of H = 4096 (16 prompts, ranks 8-128) 60 us with a
// register ring copied to LDS (48 beside the streaming expand below), 46 now; 3781 tokens of H = 5120
// 57 -> 55; 24675 tokens of H = 4096 (ranks 16-64) 167 -> 164 = 5.3 TB/s of x and pages; 2615 tokens of
// H = 2568 (ranks 5-200, sub-tiles of 32 tokens) 62 -> 35 us.  The sums
// are formed in the same order as before and are bit-identical.  Tried: rings private to a wavefront
// (no barriers, k split over the wavefronts) 50 us on the first of these, separate deep x and shallow
// page rings with a loader role per wavefront 52-57, three workgroups per compute unit with shorter
// rings 55, other cache policies than streaming x + plain pages 52-60.
//
// The scheduler may cut the range of H into n_parts shares, one workgroup each.  A share leaves its
// partial sums (fp32) in the slot's scratch; a second, small kernel (join_shares_kernel, one
// workgroup per split tile) adds them up in the order of their numbers.  The kernel boundary
// is the only synchronisation.
//
// The finished tile goes to the expand as MFMA operand fragments (see VPieces).  For binary16
// pools every token row is first scaled by a power of two, 2^e, that puts its largest |v| into
// [2^10, 2^11): the hi piece then holds 11 bits and the lo piece 11 more whatever the magnitude
// of v (row maxima in [2^-42, 2^35); the pieces overflow from 2^40 on).  e (clamped to [-24, 40]) is left
// beside the fragments; the expand scales its accumulators back.  The tiles of a dual plan, whose v would
// otherwise be fp32 rows, always pass through the join kernel, which gives binary16 three pieces (see RowScale).
// Token rows beyond the item and ranks beyond the adapter's are read from a valid row instead;
// their results are not stored, or stored as zero (ranks up to the next multiple of 32, so the
// expand can read whole blocks).
// ---------------------------------------------------------------------------------------
constexpr int kMfmaThreads = 256;
constexpr int kPiece = 64;                           // elements of H per piece
constexpr int kPieceBytes = kPiece * 2;              // bytes of a row per piece
constexpr int kPieceBlock = kMsBlockBytes;           // bytes of 32 rows of a piece in LDS
static_assert(kMsBlockBytes == 32 * kPieceBytes, "the ring is laid out in pieces");
// Row exponents of binary16 pools: where they put a row's largest |v|, and their range.  With three pieces the
// range covers every finite sum of products of binary16 values (|v| < 2^47, multiples of 2^-48).
template <int NP>
struct RowScale {
    static constexpr int kTop = NP == 3 ? 14 : 10, kMin = NP == 3 ? -34 : -24, kMax = 40;
};
static_assert(kMsGranule % kPiece == 0 && kMsTok == 128 && kMsRanks == 128, "pieces and tiles are tied");

__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }

// N 16-byte LDS reads, waited for together.  Reads and wait are one asm block because the compiler
// cannot tell which stage of a ring filled by global_load_lds a read touches: before an ordinary
// LDS read it waits for every load in flight.
template <int N>
__device__ __forceinline__ void lds_read(const uint32_t (&a)[N], u32x4 (&o)[N])
{
    static_assert(N == 2 || N == 4 || N == 6 || N == 8 || N == 10 || N == 12, "write the block for this number of reads");
    if constexpr (N == 2)
        asm volatile(
            "ds_read_b128 %0, %2\n\t"
            "ds_read_b128 %1, %3\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1])
            : "v"(a[0]), "v"(a[1])
            : "memory");
    else if constexpr (N == 4)
        asm volatile(
            "ds_read_b128 %0, %4\n\t"
            "ds_read_b128 %1, %5\n\t"
            "ds_read_b128 %2, %6\n\t"
            "ds_read_b128 %3, %7\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3])
            : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
            : "memory");
    else if constexpr (N == 6)
        asm volatile(
            "ds_read_b128 %0, %6\n\t"
            "ds_read_b128 %1, %7\n\t"
            "ds_read_b128 %2, %8\n\t"
            "ds_read_b128 %3, %9\n\t"
            "ds_read_b128 %4, %10\n\t"
            "ds_read_b128 %5, %11\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5])
            : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5])
            : "memory");
    else if constexpr (N == 8)
        asm volatile(
            "ds_read_b128 %0, %8\n\t"
            "ds_read_b128 %1, %9\n\t"
            "ds_read_b128 %2, %10\n\t"
            "ds_read_b128 %3, %11\n\t"
            "ds_read_b128 %4, %12\n\t"
            "ds_read_b128 %5, %13\n\t"
            "ds_read_b128 %6, %14\n\t"
            "ds_read_b128 %7, %15\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7])
            : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7])
            : "memory");
    else if constexpr (N == 10)
        asm volatile(
            "ds_read_b128 %0, %10\n\t"
            "ds_read_b128 %1, %11\n\t"
            "ds_read_b128 %2, %12\n\t"
            "ds_read_b128 %3, %13\n\t"
            "ds_read_b128 %4, %14\n\t"
            "ds_read_b128 %5, %15\n\t"
            "ds_read_b128 %6, %16\n\t"
            "ds_read_b128 %7, %17\n\t"
            "ds_read_b128 %8, %18\n\t"
            "ds_read_b128 %9, %19\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7]), "=&v"(o[8]), "=&v"(o[9])
            : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]), "v"(a[9])
            : "memory");
    else if constexpr (N == 12)
        asm volatile(
            "ds_read_b128 %0, %12\n\t"
            "ds_read_b128 %1, %13\n\t"
            "ds_read_b128 %2, %14\n\t"
            "ds_read_b128 %3, %15\n\t"
            "ds_read_b128 %4, %16\n\t"
            "ds_read_b128 %5, %17\n\t"
            "ds_read_b128 %6, %18\n\t"
            "ds_read_b128 %7, %19\n\t"
            "ds_read_b128 %8, %20\n\t"
            "ds_read_b128 %9, %21\n\t"
            "ds_read_b128 %10, %22\n\t"
            "ds_read_b128 %11, %23\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7]), "=&v"(o[8]), "=&v"(o[9]), "=&v"(o[10]), "=&v"(o[11])
            : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]), "v"(a[9]), "v"(a[10]), "v"(a[11])
            : "memory");
}
// The NP fragments of a k-step, kWave * 16 bytes apart, from byte OFF past `at` on; offsets in the instructions, so that
// unrolled reads hold no address registers
template <int NP, int OFF>
__device__ __forceinline__ void lds_read_pieces(uint32_t at, u32x4 (&o)[NP])
{
    static_assert((NP == 2 || NP == 3) && OFF >= 0 && OFF + 2 * kWave * 16 < 65536, "offset field");
    if constexpr (NP == 2)
        asm volatile(
            "ds_read_b128 %0, %2 offset:%3\n\t"
            "ds_read_b128 %1, %2 offset:%4\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1])
            : "v"(at), "n"(OFF), "n"(OFF + kWave * 16)
            : "memory");
    else
        asm volatile(
            "ds_read_b128 %0, %3 offset:%4\n\t"
            "ds_read_b128 %1, %3 offset:%5\n\t"
            "ds_read_b128 %2, %3 offset:%6\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2])
            : "v"(at), "n"(OFF), "n"(OFF + kWave * 16), "n"(OFF + 2 * kWave * 16)
            : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const unsigned char *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}

// Exponent e of the power of two that scales a token row of a binary16 pool: the row's largest finite
// |v| lands in [2^kTop, 2^(kTop + 1)).  Zero and subnormal maxima get e = 0.
template <int NP>
__device__ __forceinline__ int row_exponent(float vmax)
{
    typedef RowScale<NP> S;
    const int be = (int)((__float_as_uint(vmax) >> 23) & 0xffu); // biased exponent of the row maximum
    if (be == 0) return 0;
    return min(max(S::kTop - (be - 127), S::kMin), S::kMax);
}

// Ranks beyond the adapter's become zero; returns the largest finite |value| of the eight.
__device__ __forceinline__ float mask_octet(const MsItem &it, int oct, float (&val)[8])
{
    float vmax = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float f = oct * 8 + e < it.nj ? val[e] : 0.f;
        val[e] = f;
        vmax = fabsf(f) < __builtin_inff() ? fmaxf(vmax, fabsf(f)) : vmax;
    }
    return vmax;
}

// Ranks 8 * oct .. + 7 of the item, finished, of token row `row` of v tile `tile` -> the 16 bytes
// they fill in each piece's operand fragment, scaled by `sc` first.
template <int DT, int NP>
__device__ __forceinline__ void store_octet(const MsItem &it, int tile, int row, int oct, const float (&val)[8],
                                            float sc, int v_stride, uint16_t *__restrict__ vfrag)
{
    const int n_kk = v_stride >> 4;
    const int kk = (it.j0 >> 4) + (oct >> 1);
    if (kk >= n_kk) return;
    float f[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = DT == SLORA_F16 ? val[k] * sc : val[k];
    uint16_t *dst = vfrag + vfrag_index(tile, kk, 0, n_kk, NP) + (row + 32 * (oct & 1)) * 8;
    u32x4 piece[NP];
    split_pieces<DT, NP>(f, piece);
#pragma unroll
    for (int p = 0; p < NP; ++p) *reinterpret_cast<u32x4 *>(dst + p * (kWave * 8)) = piece[p];
}

// Row exponents are kept as signed bytes, 32 per (v tile, rank block), ordered so that the 16
// exponents a lane of the expand needs - accumulator register 4 g + k of lane half q holds row
// 8 g + 4 q + k - are the 16 consecutive bytes q * 16 + g * 4 + k: one 16-byte load.
__device__ __forceinline__ int8_t *vexp_row(int8_t *vexp, const MsItem &it, int tile, int v_stride, int row)
{
    const int n_rb = (v_stride + kMsRanks - 1) / kMsRanks;
    const int g = row >> 3, qq = (row >> 2) & 1, k = row & 3;
    return vexp + ((int64_t)tile * n_rb + it.j0 / kMsRanks) * 32 + qq * 16 + g * 4 + k;
}

// Partial sums of a split tile: [share][token block][rank block][octet pair i][lane][8 floats];
// lane l holds token l % 32 of the block and the rank octets l / 32 and l / 32 + 2 i.
__device__ __forceinline__ int64_t share_block(const MsItem &it) // floats of one share
{
    return (int64_t)((it.ntok + 31) >> 5) * ((it.nj + 31) >> 5) * 1024;
}

template <int DT, int MB, int NL>
__device__ __forceinline__ void shrink_mfma_tile(const MsItem &it, unsigned item_no, int sub0, const int32_t *__restrict__ pa,
                                                 const unsigned char *__restrict__ x,
                                                 const uint16_t *__restrict__ pool,
                                                 const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                 uint16_t *__restrict__ vfrag, int8_t *__restrict__ vexp,
                                                 float *__restrict__ partial, unsigned char *lds)
{
    constexpr int kBlocks = MB + NL;                // 32-row blocks = loads per wavefront and piece
    constexpr int S = ms_stages(kBlocks);
    constexpr int kStage = kBlocks * kPieceBlock;
    constexpr int NB = NL == 3 && MB < 4 ? 4 : NL;  // rank blocks computed (the fourth of three is dropped)
    constexpr int WN = NB >= 4 / MB ? 4 / MB : NB;  // wavefronts along the ranks
    constexpr int NBW = NB / WN;                    // rank blocks per wavefront
    // A single rank block has two accumulators, for the even and the odd k-steps: one would make every
    // MFMA wait for the one before it.  They sit in two wavefronts if there are that many (KG = 2).
    constexpr int KG = NL == 1 && MB * WN <= 2 ? 2 : 1;
    constexpr int KA = NL == 1 && KG == 1 ? 2 : 1;  // accumulators of a wavefront and rank block
    constexpr int KS = 4 / KG;                      // k-steps per wavefront and piece
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t row_bytes = (int64_t)H * 2;

    // ---- copy duty: rows 8 * wave .. + 7 of every block, lane -> row lane / 8, LDS group lane % 8
    const int r8 = wave * 8 + (lane >> 3);
    const int group = ((lane & 7) ^ ((r8 >> 1) & 7)) * 16; // byte offset, in the piece, of what this lane fetches
    const unsigned char *src[kBlocks];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int r = sub0 + i * 32 + r8;
        src[i] = x + (int64_t)tok_idx[it.pos0 + (r < it.ntok ? r : 0)] * row_bytes;
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int j = i * 32 + r8;
        src[MB + i] = reinterpret_cast<const unsigned char *>(pool) + (int64_t)pa[j < it.nj ? j : 0] * row_bytes;
    }
    // Every item starts its sweep over its share at another granule (two pieces) and wraps around: tiles
    // launched together would otherwise ask the same few memory channels for the same column offset
    // of their rows at the same time.  By item: every slot of a launch, every sub-tile, and a launch
    // of any number of slots add in the same order.
    constexpr int kPerGranule = kMsGranule / kPiece;
    const int n_gran = it.c1 - it.c0, n = n_gran * kPerGranule; // granules, pieces
    const int g_first = (int)((item_no * 5u) % (unsigned)n_gran);
    auto piece_of = [&](int s) { // position in H of the s-th piece of the sweep
        const int g = s / kPerGranule + g_first;
        return (it.c0 + (g < n_gran ? g : g - n_gran)) * kPerGranule + s % kPerGranule;
    };
    auto load = [&](int s) {
        // bytes past the row's end (last granule of a ragged H) are clamped into the row; they are
        // dropped when the operands are read
        const int64_t off = min((int64_t)piece_of(s) * kPieceBytes + group, row_bytes - 16);
        unsigned char *dst = lds + (s % S) * kStage + wave * 1024;
#pragma unroll
        for (int i = 0; i < kBlocks; ++i) {
            // x rows are read once: streaming; page rows come back for the adapter's other tiles
            if (i < MB)
                load_to_lds<kLoadStreaming>(src[i] + off, dst + i * kPieceBlock);
            else
                load_to_lds<0>(src[i] + off, dst + i * kPieceBlock);
        }
    };

    const int row = lane & 31, q = lane >> 5;
    const int mb = wave % MB, wn = (wave / MB) % WN, kg = wave / (MB * WN);
    const bool computes = wave < MB * WN * KG;       // a tile of one token block leaves wavefronts without work
    f32x16 acc[NBW][KA];
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int a = 0; a < KA; ++a)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[b][a][e] = 0.f;
    // LDS addresses, in stage 0, of this lane's operands: KS of x, then KS of each rank block
    uint32_t lds_at[KS * (1 + NBW)];
#pragma unroll
    for (int i = 0; i < KS * (1 + NBW); ++i) {
        const int p = 2 * ((i % KS) * KG + kg % KG) + q; // 16-byte group of the lane's 8 k-values
        const int blk = i < KS ? mb : MB + min(wn * NBW + i / KS - 1, NL - 1);
        lds_at[i] = lds_address(lds) + blk * kPieceBlock + row * kPieceBytes + ((p ^ ((row >> 1) & 7)) * 16);
    }
    const bool ragged = row_bytes % (kMsGranule * 2) != 0;
    const int full = (int)(row_bytes / kPieceBytes); // pieces that lie inside the row

#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < n) load(s);
    for (int s = 0; s < n; ++s) {
        // piece s has arrived when at most the S - 2 younger ones are outstanding
        if (s + S - 2 < n)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * kBlocks) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + S - 1 < n) load(s + S - 1);
        if (!computes) continue;
        const uint32_t stage_at = (uint32_t)((s % S) * kStage);
        // operands of KC k-steps at a time: a lane's KC groups of x, then of each rank block
        constexpr int KC = KS * (1 + NBW) > 12 ? KS / 2 : KS;
#pragma unroll
        for (int k0 = 0; k0 < KS; k0 += KC) {
            uint32_t at[KC * (1 + NBW)];
            u32x4 op[KC * (1 + NBW)];
#pragma unroll
            for (int i = 0; i < KC * (1 + NBW); ++i) at[i] = lds_at[(i / KC) * KS + k0 + i % KC] + stage_at;
            lds_read(at, op);
            if (ragged && piece_of(s) >= full) { // uniform: groups past the row's end
#pragma unroll
                for (int i = 0; i < KC * (1 + NBW); ++i) {
                    const int p = 2 * ((k0 + i % KC) * KG + kg) + q;
                    op[i] = (int64_t)piece_of(s) * kPieceBytes + p * 16 < row_bytes ? op[i] : u32x4{0u, 0u, 0u, 0u};
                }
            }
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int b = 0; b < NBW; ++b)
                    acc[b][(k0 + k) % KA] = mfma32<DT>(op[k], op[KC * (1 + b) + k], acc[b][(k0 + k) % KA]);
        }
    }
    __syncthreads(); // the ring is free: it now stages the finished blocks

    // ---- accumulator layout -> 8 consecutive ranks of one token per lane -------------------------
    // Block (kg, mb, nb) is 32 x 32 floats; group g (four ranks) of row r sits at g ^ (r / 2 % 8).
    float *stage = reinterpret_cast<float *>(lds);
    if (computes) {
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
            float *blk = stage + ((kg * MB + mb) * NB + wn * NBW + b) * 1024;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = mfma_row(v, lane);
                float sum = acc[b][0][v];
                if constexpr (KA == 2) sum += acc[b][1][v];
                blk[r * 32 + (((row >> 2) ^ ((r >> 1) & 7)) << 2) + (row & 3)] = sum;
            }
        }
    }
    __syncthreads();
    // wavefront w finishes rows R w .. R w + R - 1; a lane has one row and every OL-th octet of ranks
    constexpr int R = 8 * MB, OL = kWave / R, NI = (NB * 4 + OL - 1) / OL;
    const int tb = (wave * R + lane % R) >> 5, r = (wave * R + lane % R) & 31; // token block and row of the tile
    const int trow = sub0 + tb * 32 + r;             // token of the item
    const int nb_act = (it.nj + 31) >> 5;
    const int o0 = lane / R;
    float val[NI][8];
    float vmax = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int oct = o0 + OL * i;
#pragma unroll
        for (int e = 0; e < 8; ++e) val[i][e] = 0.f;
        if (oct < nb_act * 4) {
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                const float *blk = stage + ((k * MB + tb) * NB + (oct >> 2)) * 1024 + r * 32;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 f = *reinterpret_cast<const f32x4 *>(blk + (((2 * (oct & 3) + h) ^ ((r >> 1) & 7)) << 2));
#pragma unroll
                    for (int e = 0; e < 4; ++e) val[i][4 * h + e] += f[e];
                }
            }
        }
    }
    // ---- a share of a split tile: leave the partial sums for join_shares_kernel -------------------
    if (it.sync >= 0) {
        if (trow < ((it.ntok + 31) & ~31)) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int oct = o0 + OL * i;
                if (oct < nb_act * 4) {
                    float *dst = partial + it.part * share_block(it) + ((int64_t)(trow >> 5) * nb_act + (oct >> 2)) * 1024 +
                                 ((oct >> 1) & 1) * 512 + (r + 32 * (oct & 1)) * 8;
                    *reinterpret_cast<f32x4 *>(dst) = f32x4{val[i][0], val[i][1], val[i][2], val[i][3]};
                    *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{val[i][4], val[i][5], val[i][6], val[i][7]};
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) vmax = fmaxf(vmax, mask_octet(it, o0 + OL * i, val[i]));
    const int tile = it.tile + (trow >> 5);
    const bool token_ok = trow < it.ntok;
    float sc = 1.f;
    if constexpr (DT == SLORA_F16) {
#pragma unroll
        for (int m = R; m < kWave; m <<= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, m, kWave)); // the token's other ranks
        const int e = row_exponent<VPieces<DT>::N>(vmax);
        sc = pow2f(e);
        if (o0 == 0 && trow < ((it.ntok + 31) & ~31)) *vexp_row(vexp, it, tile, v_stride, r) = (int8_t)(token_ok ? e : 0);
    }
    if (!token_ok) return;
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if (o0 + OL * i < nb_act * 4) store_octet<DT, VPieces<DT>::N>(it, tile, r, o0 + OL * i, val[i], sc, v_stride, vfrag);
}

template <int DT>
__global__ __launch_bounds__(kMfmaThreads, 2) void shrink_mfma_kernel(const MsItem *__restrict__ items,
                                                                       const int32_t *__restrict__ arena,
                                                                       const uint16_t *__restrict__ pool,
                                                                       const int32_t *__restrict__ tok_idx, int H,
                                                                       int v_stride, int sub_tok, MultiArgs args)
{
    // the rings of the plan's largest tile, sized at launch
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // slots vary fastest: the shares of a tile, and the tiles of an adapter, follow one another
    const int cs = blockIdx.x % args.n;
    const unsigned rest = blockIdx.x / args.n, per_item = (unsigned)(kMsTok / sub_tok);
    const unsigned item_no = rest / per_item;
    const int sub = (int)(rest % per_item) * sub_tok;
    const MsItem it = items[item_no];
    if (sub >= it.ntok) return;              // the whole workgroup
    const int rows = min(it.ntok - sub, sub_tok);
    const unsigned char *x = static_cast<const unsigned char *>(args.x[cs]);
    const int32_t *pa = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank + it.j0;
    uint16_t *vfrag = reinterpret_cast<uint16_t *>(args.v[cs] + args.vfrag_off);
    int8_t *vexp = reinterpret_cast<int8_t *>(args.v[cs] + args.vexp_off);
    float *partial = args.v[cs] + args.part_off + it.part_off;
#define SLORA_MS(MBV, NLV) \
    shrink_mfma_tile<DT, MBV, NLV>(it, item_no, sub, pa, x, pool, tok_idx, H, v_stride, vfrag, vexp, partial, lds)
#define SLORA_MS_RANKS(MBV)              \
    if (it.nj <= 32) SLORA_MS(MBV, 1);      \
    else if (it.nj <= 64) SLORA_MS(MBV, 2); \
    else if (it.nj <= 96) SLORA_MS(MBV, 3); \
    else SLORA_MS(MBV, 4);
    if (rows <= 32) { SLORA_MS_RANKS(1) }
    else if (rows <= 64) { SLORA_MS_RANKS(2) }
    else { SLORA_MS_RANKS(4) }
#undef SLORA_MS_RANKS
#undef SLORA_MS
}

// One workgroup per split tile, token block and slot; its wavefronts add up the shares of a rank block, or
// of half of one (Wide), in the order of their numbers (a fixed order: the same bits on every run) and finish it as the
// shrink itself does for a tile that was not split.  Binary16: the row maximum over the rank blocks meets in LDS.
// Bound by the round trips.  The tiles of a dual plan have up to 32 shares: Wide requests 16 of them at a time (512
// tokens of rank 64, H = 4096, 4 slots: 6.8 -> 5.2 us); others have two to five, and more threads only make their many
// small workgroups dearer (5.4 -> 6.4 us for sixteen prompts, 10.6 -> 12.7 us for 2251 tokens of rank 128 among others).
constexpr int join_waves(bool wide) { return kMsRanks / 32 * (wide ? 2 : 1); }
template <int DT, int NP, bool Wide>
__global__ __launch_bounds__(join_waves(Wide) * kWave) void join_shares_kernel(const MsItem *__restrict__ tiles, int v_stride,
                                                                               MultiArgs args)
{
    constexpr int kBlocks = kMsTok / 32, kWaves = join_waves(Wide);
    constexpr int NO = Wide ? 1 : 2;                          // octets of ranks of a lane
    constexpr int kBatch = Wide ? 16 : 4;
    __shared__ float smax[kWaves][32];
    const int cs = blockIdx.x % args.n;
    const int tb = (blockIdx.x / args.n) % kBlocks;          // token block
    const MsItem it = tiles[blockIdx.x / args.n / kBlocks];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nb = Wide ? wave >> 1 : wave, half = Wide ? wave & 1 : 0; // rank block of this wavefront, its first half
    const int row = lane & 31, q = lane >> 5;
    const int oct = nb * 4 + q + 2 * half;                    // first octet of this lane; the other is two further on
    const int mb_act = (it.ntok + 31) >> 5, nb_act = (it.nj + 31) >> 5;
    if (tb >= mb_act) return;                                 // the whole workgroup
    const bool live = nb < nb_act;
    float val[NO][8];
#pragma unroll
    for (int i = 0; i < NO; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) val[i][e] = 0.f;
    if (live) {
        const int64_t blk = share_block(it);
        const float *base = args.v[cs] + args.part_off + it.part_off + (int64_t)(tb * nb_act + nb) * 1024 + half * 512 + lane * 8;
        for (int p0 = 0; p0 < it.n_parts; p0 += kBatch) {
            f32x4 w[kBatch][2 * NO];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                if (p0 + k < it.n_parts) {
                    const float *src = base + (int64_t)(p0 + k) * blk;
#pragma unroll
                    for (int i = 0; i < NO; ++i) {
                        w[k][2 * i] = *reinterpret_cast<const f32x4 *>(src + i * 512);
                        w[k][2 * i + 1] = *reinterpret_cast<const f32x4 *>(src + i * 512 + 4);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                if (p0 + k < it.n_parts) {
#pragma unroll
                    for (int i = 0; i < NO; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            val[i][e] += w[k][2 * i][e];
                            val[i][4 + e] += w[k][2 * i + 1][e];
                        }
                }
            }
        }
    }
    float sc = 1.f;
    const bool token_ok = tb * 32 + row < it.ntok;
    float vmax = 0.f;
#pragma unroll
    for (int i = 0; i < NO; ++i) vmax = fmaxf(vmax, mask_octet(it, oct + 2 * i, val[i]));
    if constexpr (DT == SLORA_F16) {
        vmax = fmaxf(vmax, __shfl_xor(vmax, 32, kWave));
        if (q == 0) smax[wave][row] = vmax;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kWaves; ++k) vmax = fmaxf(vmax, smax[k][row]);
        const int e = row_exponent<NP>(vmax);
        sc = pow2f(e);
        if (wave == 0 && q == 0)
            *vexp_row(reinterpret_cast<int8_t *>(args.v[cs] + args.vexp_off), it, it.tile + tb, v_stride, row) = (int8_t)(token_ok ? e : 0);
    }
    if (live && token_ok) {
        uint16_t *vfrag = reinterpret_cast<uint16_t *>(args.v[cs] + args.vfrag_off);
#pragma unroll
        for (int i = 0; i < NO; ++i) store_octet<DT, NP>(it, it.tile + tb, row, oct + 2 * i, val[i], sc, v_stride, vfrag);
    }
}

// ---------------------------------------------------------------------------------------
// prefill expand: y[tok, d] += sum_j V[pos, j] * Bpage_j[d] for a run of 32-token tiles of one
// adapter and up to 256 columns.  Wavefront w owns columns 64w .. 64w+63 (two 32-column MFMA blocks)
// of every tile of the run.
//
// Adapters of up to 128 ranks (RegStages 32-rank stages): the B operands of a wavefront's columns do
// not depend on the tile; it reads them once, keeps them in registers (16 per stage) and walks the
// tiles with one read-modify-write of y each.  V of a tile is the same for all four wavefronts: it is
// copied straight into LDS (global_load_lds), a quarter by each, into one of two buffers - read by
// every wavefront for itself it was a larger part of the kernel's requests than y.  V and y of the
// next tile are requested before the current one is computed; one barrier per tile hands the
// buffers over, and the stores of a tile are only waited for a tile later.
// Adapters of up to 256 ranks do the same with V in two halves (expand_mfma_halves); those of more, and most single tiles of 129 to 256 ranks
// (expand_mfma_stream), read V and B again for every tile, without barriers.
//
// The first operand is V (tokens x ranks, fp32 precision), split by the shrink into 16-bit pieces
// (see VPieces); each piece costs one more MFMA on a path that is bound by memory, not by the
// matrix cores.  The second operand needs, per lane, 8 consecutive ranks of ONE column, but a page is
// contiguous along columns; the wavefront therefore copies a 32-rank x 64-column slab of B
// through LDS, transposing on the way in (two ranks packed per dword), and reads its operand
// back with one 16-byte LDS load.  The finished 32 x 64 tile passes through the same LDS (fp32, 16 rows at a
// time) into whole row pieces, and is rounded once if y is 16-bit, added to y if y is fp32: 16-byte accesses
// towards memory.  All global loads are unconditional: token rows beyond the tile, columns beyond the item
// and ranks beyond the adapter's are redirected to a valid row / column / page; what they produce is
// multiplied by the zero padding of V or is never stored.
//
// Bound by HBM (y read and written once).  What each part measured, per step, on batches of 4524 tokens
// (4 slots, H = 4096, fp32 y, 16 prompts of ranks 8-128) / 3781 tokens (4 slots, H = 5120, bfloat16 y) /
// 24675 tokens (4 slots, H = 4096, binary16 y): a workgroup per tile, everything read per tile
// 132 / 110 / 395 us; runs of tiles with B in registers 130 / 116 / 345; V shared through LDS
// 131 / 97 / 340; y moved with streaming (non-temporal) loads AND stores 111 / 83 / 311 us = 5.6 / 4.2 /
// 5.3 TB/s of y, B and V (streaming on one side only changes nothing).  Workgroups per launch 1024-4096 measure alike, fewer than
// 1024 and runs of 32 tiles gain nothing; three wavefronts per SIMD need registers that spill (+25 %).
// ---------------------------------------------------------------------------------------
constexpr int kSlabStride = 20; // dwords per column in LDS: 16 (32 ranks) + 4 pad, keeps 16-byte alignment
constexpr int kSlabGroupPad = 8; // extra dwords before every 8 columns: the 8 column groups a transposing store
                                 // touches then fall into different banks (8 x 20 dwords alone is a multiple of 32:
                                 // rocprofv3 counted bank conflicts on 58 % of this kernel's LDS cycles)
__device__ __forceinline__ int slab_col(int c) { return c * kSlabStride + (c >> 3) * kSlabGroupPad; }
constexpr int kTileStride = 68;  // floats per row of the y tile: 16-byte aligned, rows spread over the banks
constexpr int kWaveLds = (64 * kSlabStride + 8 * kSlabGroupPad) * 4; // a wavefront's own LDS
static_assert(16 * kTileStride * 4 <= kWaveLds && kWaveLds % 16 == 0, "half a y tile shares the B slab's LDS");

__device__ __forceinline__ void wave_lds_fence() // LDS written by one lane is read by another of the same wavefront
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wavefront's view of a run: its columns, the rows of y it moves, and the ways of B and of the
// finished deltas through its LDS.
template <int DT, bool Y16, int NP>
struct ExpandWave {
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    static constexpr bool kScaled = kScaledPieces<DT, NP>;
    static constexpr bool kFromZero = !Y16 || kScaled;   // y is added to the finished sum of products
    static constexpr int kElem = Y16 ? 2 : 4;
    static constexpr int kYVec = 16 / kElem;             // elements per 16-byte access
    static constexpr int kYLanes = 64 / kYVec;           // lanes per tile row
    static constexpr int kYRows = kWave / kYLanes;       // rows per access of the wavefront
    static constexpr int kYLoads = 32 / kYRows;          // accesses per tile
    const Item &it;
    const int32_t *pbl;
    const int32_t *tok_idx;
    uint32_t *slab;
    int H, lane, n, q, cg, kp, ygrp, yrow, tiles, last;
    bool store_ok;
    unsigned char *yg;
    const uint16_t *bcol;
    f32x16 acc[2];

    __device__ __forceinline__ ExpandWave(const Item &item, int colw, const int32_t *pages, const uint16_t *pool,
                                          const int32_t *tokens, int H_, void *y, uint32_t *lds)
        : it(item), pbl(pages), tok_idx(tokens), slab(lds), H(H_)
    {
        lane = threadIdx.x & (kWave - 1);
        n = lane & 31;
        q = lane >> 5;
        cg = lane & 7;  // column group (8 columns) this lane copies of B
        kp = lane >> 3; // rank pair this lane copies of B
        ygrp = lane % kYLanes;
        yrow = lane / kYLanes;
        tiles = it.run & 0xff; // tiles of the run
        last = it.run >> 8;    // tokens of the last one
        const int col_end = it.a + it.b;      // <= H, a multiple of 8
        const int ycol = colw + kYVec * ygrp; // a group of columns is inside or outside: both ends are multiples of 8
        store_ok = ycol < col_end;
        yg = static_cast<unsigned char *>(y) + (int64_t)min(ycol, col_end - kYVec) * kElem;
        bcol = pool + min(colw + 8 * cg, col_end - 8);
    }
    __device__ __forceinline__ int tokens_of(int t) const { return t == tiles - 1 ? last : kMfmaTok; }
    __device__ __forceinline__ void load_rows(int t, int (&row)[kYLoads]) const
    {
        const int nt = tokens_of(t);
#pragma unroll
        for (int i = 0; i < kYLoads; ++i) row[i] = tok_idx[it.pos0 + t * kMfmaTok + min(yrow + kYRows * i, nt - 1)];
    }
    __device__ __forceinline__ void load_y(const int (&row)[kYLoads], u32x4 (&w)[kYLoads]) const
    {
#pragma unroll
        for (int i = 0; i < kYLoads; ++i) w[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(yg + (int64_t)row[i] * H * kElem));
    }
    // the page numbers of the four B rows this lane copies per 32-rank stage; beyond the last rank: the last one's
    __device__ __forceinline__ void load_pg(int k0, int (&pg)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) pg[i] = pbl[min(k0 + 16 * (i >> 1) + 2 * kp + (i & 1), it.rank - 1)];
    }
    __device__ __forceinline__ void load_b(const int (&pg)[4], u32x4 (&w)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const u32x4 *>(bcol + (int64_t)pg[i] * H);
    }
    // 32 ranks x 64 columns, transposed through LDS into the operands of two k-steps x two column blocks
    __device__ __forceinline__ void transpose_b(const u32x4 (&w)[4], u32x4 (&op)[2][2]) const
    {
        wave_lds_fence(); // the previous contents have been read
#pragma unroll
        for (int rd = 0; rd < 2; ++rd) {
            uint32_t *dst = slab + slab_col(8 * cg) + 8 * rd + kp; // columns 8 cg .. 8 cg + 7: one group, same pad
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dst[(2 * e) * kSlabStride] = (w[2 * rd][e] & 0xffffu) | (w[2 * rd + 1][e] << 16);
                dst[(2 * e + 1) * kSlabStride] = (w[2 * rd][e] >> 16) | (w[2 * rd + 1][e] & 0xffff0000u);
            }
        }
        wave_lds_fence();
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                op[s][nb] = *reinterpret_cast<const u32x4 *>(slab + slab_col(nb * 32 + n) + 8 * s + 4 * q);
    }
    // B of the run, `stages` <= N stages of 32 ranks: all page numbers first, then the rows of up to AHEAD stages in flight
    // (registers that the tiles need later); first() runs behind the first rows' requests.  Four stages in flight against two, expand of
    // sixteen prompts, 4 slots, us: ranks 97-128 135 / 137, with 16-bit y 124 / 129; two stages of 64 ranks 92.3 / 92.2, one slot with 16-bit y 28.2 / 27.7.
    template <int N, class First>
    __device__ __forceinline__ void load_operands(int stages, u32x4 (&op)[N][2][2], First first) const
    {
        constexpr int kAhead = N < 4 ? N : 4;
        int pg[N][4];
        u32x4 b[kAhead][4];
#pragma unroll
        for (int s = 0; s < N; ++s)
            if (s < kAhead || s < stages) load_pg(32 * s, pg[s]);
#pragma unroll
        for (int s = 0; s < kAhead; ++s) load_b(pg[s], b[s]);
        first();
#pragma unroll
        for (int s = 0; s < N; ++s) {
            if (s >= kAhead && s >= stages) break;
            transpose_b(b[s % kAhead], op[s]);
            if (s + kAhead < N && s + kAhead < stages) load_b(pg[s + kAhead], b[s % kAhead]);
        }
    }
    static __device__ __forceinline__ void multiply(f32x16 (&sum)[2], const u32x4 &piece, const u32x4 (&op)[2])
    {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) sum[nb] = mfma32<DT>(piece, op[nb], sum[nb]);
    }
    // Binary16 pools: the shrink scaled token row i of a block of kMsRanks ranks by 2^e[i].  The accumulators
    // follow: they hold (16-bit y + products so far) * 2^e of the CURRENT block - scaled up before the first
    // block, re-scaled where the block changes, scaled back at the end.  Powers of two: every step is exact.
    static __device__ __forceinline__ void scale_rows(f32x16 (&sum)[2], const i32x4 &from, const i32x4 &to)
    {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float f = pow2f((int)(int8_t)(to[g] >> (8 * k)) - (int)(int8_t)(from[g] >> (8 * k)));
                sum[0][4 * g + k] *= f;
                sum[1][4 * g + k] *= f;
            }
    }
    __device__ __forceinline__ void times(float f) // of all sums
    {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nb][v] *= f;
    }
    // Accumulators at the start of a tile: y itself if it is 16-bit (widened, through LDS), zero if fp32.
    __device__ __forceinline__ void begin(const u32x4 (&w)[kYLoads], [[maybe_unused]] const i32x4 &scale)
    {
        if constexpr (kFromZero) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[nb][v] = 0.f;
        } else {
            float *half = reinterpret_cast<float *>(slab);
#pragma unroll
            for (int h = 0; h < 2; ++h) { // accumulator registers 8 h .. 8 h + 7 hold rows 16 h .. 16 h + 15
                wave_lds_fence();
#pragma unroll
                for (int i = 0; i < kYLoads / 2; ++i) {
                    const u32x4 &v = w[h * (kYLoads / 2) + i];
                    float *dst = half + (yrow + kYRows * i) * kTileStride + kYVec * ygrp;
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) widen2<DT>(v[e], f[2 * e], f[2 * e + 1]);
                    *reinterpret_cast<f32x4 *>(dst) = f32x4{f[0], f[1], f[2], f[3]};
                    *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{f[4], f[5], f[6], f[7]};
                }
                wave_lds_fence();
#pragma unroll
                for (int v = 0; v < 8; ++v)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[nb][8 * h + v] = half[mfma_row(v, lane) * kTileStride + nb * 32 + n];
            }
            if constexpr (DT == SLORA_F16) scale_rows(acc, i32x4{0, 0, 0, 0}, scale);
        }
    }
    // Accumulators -> row pieces of the finished y tile: rounded once if y is 16-bit, added to y if fp32
    // (the sum of products then rounds at its own size and not at y's: 1.4e-7 -> 1.24e-7 against 64 bits for
    // 512 tokens of rank 64, and one way through LDS less).  16-bit results are rounded from the sums formed
    // as they always were, so that they stay the same bit for bit.
    __device__ __forceinline__ void end(u32x4 (&w)[kYLoads], [[maybe_unused]] const i32x4 &scale)
    {
        if constexpr (DT == SLORA_F16) scale_rows(acc, scale, i32x4{0, 0, 0, 0});
        float *half = reinterpret_cast<float *>(slab);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            wave_lds_fence();
#pragma unroll
            for (int v = 0; v < 8; ++v)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) half[mfma_row(v, lane) * kTileStride + nb * 32 + n] = acc[nb][8 * h + v];
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < kYLoads / 2; ++i) {
                const float *src = half + (yrow + kYRows * i) * kTileStride + kYVec * ygrp;
                u32x4 &o = w[h * (kYLoads / 2) + i];
                if constexpr (Y16) {
                    f32x4 a = *reinterpret_cast<const f32x4 *>(src), b = *reinterpret_cast<const f32x4 *>(src + 4);
                    if constexpr (kFromZero) {
                        float f[8];
#pragma unroll
                        for (int e = 0; e < 4; ++e) widen2<DT>(o[e], f[2 * e], f[2 * e + 1]);
                        a += f32x4{f[0], f[1], f[2], f[3]};
                        b += f32x4{f[4], f[5], f[6], f[7]};
                    }
                    o = u32x4{narrow2<DT>(a.x, a.y), narrow2<DT>(a.z, a.w), narrow2<DT>(b.x, b.y), narrow2<DT>(b.z, b.w)};
                } else {
                    const f32x4 a = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(__uint_as_float(o[e]) + a[e]);
                }
            }
        }
    }
    __device__ __forceinline__ void store_y(int t, const int (&row)[kYLoads], const u32x4 (&w)[kYLoads]) const
    {
        const int nt = tokens_of(t);
#pragma unroll
        for (int i = 0; i < kYLoads; ++i) {
            int r = row[i];
            asm("" : "+v"(r)); // the address is computed anew: kept since the load, it would cost registers the tile needs
            if (yrow + kYRows * i < nt && store_ok)
                __builtin_nontemporal_store(w[i], reinterpret_cast<u32x4 *>(yg + (int64_t)r * H * kElem));
        }
    }
};

template <int DT, bool Y16, int NP, int RegStages>
__device__ __forceinline__ void expand_mfma_run(const Item &it, int wave, const int32_t *__restrict__ pbl,
                                                const uint16_t *__restrict__ pool,
                                                const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                const uint16_t *__restrict__ vfrag, const int8_t *__restrict__ vexp,
                                                void *__restrict__ y, unsigned char *lds)
{
    typedef ExpandWave<DT, Y16, NP> W;
    typedef typename W::i32x4 i32x4;
    constexpr int kYLoads = W::kYLoads;
    constexpr int kFrags = 2 * RegStages * NP;    // operand fragments (1 KiB) of V per tile
    const int n_kk = v_stride >> 4, n_rb = (v_stride + kMsRanks - 1) / kMsRanks;
    const int lane = threadIdx.x & (kWave - 1);
    const int tiles = it.run & 0xff;
    auto load_v = [&](int t) { // this wavefront's part of the fragments of tile t
        const unsigned char *src = reinterpret_cast<const unsigned char *>(vfrag + vfrag_index(it.tile + t, 0, 0, n_kk, NP)) + lane * 16;
        unsigned char *dst = lds + (t & 1) * (kFrags * 1024);
        for (int f = wave; f < kFrags; f += 4) load_to_lds<0>(src + f * 1024, dst + f * 1024);
    };
    const int colw = it.a + wave * 64;            // this wavefront's first column
    load_v(0);
    if (colw >= it.a + it.b) {                    // no columns: it only does its part of the copying
        for (int t = 0; t < tiles; ++t) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (t + 1 < tiles) load_v(t + 1);
        }
        return;
    }
    W w(it, colw, pbl, pool, tok_idx, H, y, reinterpret_cast<uint32_t *>(lds + 2 * kFrags * 1024 + wave * kWaveLds));
    int row_cur[kYLoads], row_next[kYLoads];
    u32x4 yt[kYLoads], y_next[kYLoads];
    u32x4 bop[RegStages][2][2];
    // a lane's 16 row exponents of a tile are one load
    auto exponents = [&](int t) { return *reinterpret_cast<const i32x4 *>(vexp + (int64_t)(it.tile + t) * n_rb * 32 + w.q * 16); };
    [[maybe_unused]] i32x4 e_cur = i32x4{0, 0, 0, 0}, e_next = i32x4{0, 0, 0, 0};
    if constexpr (DT == SLORA_F16) e_cur = exponents(0);
    w.load_rows(0, row_cur);
    w.load_operands(RegStages, bop, [&]() { w.load_y(row_cur, yt); });
    w.load_rows(min(1, tiles - 1), row_next);
    const uint32_t frag_at = lds_address(lds) + lane * 16;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                 // V of the first tile is complete
    asm volatile("" ::: "memory");
    for (int t = 0; t < tiles; ++t) {
        if (t + 1 < tiles) {
            load_v(t + 1);
            if constexpr (DT == SLORA_F16) e_next = exponents(t + 1);
            w.load_y(row_next, y_next);
        }
        w.begin(yt, e_cur);
        const uint32_t buf_at = frag_at + (uint32_t)((t & 1) * (kFrags * 1024));
        // pieces P0 .. P1 - 1 of every k-step, two k-steps at a time
        auto products = [&](auto first, auto end) {
            constexpr int P0 = decltype(first)::value, N = decltype(end)::value - P0;
#pragma unroll
            for (int s = 0; s < RegStages; ++s) {
                uint32_t at[2 * N];
                u32x4 piece[2 * N];
#pragma unroll
                for (int f = 0; f < 2 * N; ++f) at[f] = buf_at + ((2 * s + f / N) * NP + P0 + f % N) * 1024;
                lds_read(at, piece);
#pragma unroll
                for (int f = 0; f < 2 * N; ++f) W::multiply(w.acc, piece[f], bop[s][f / N]);
            }
        };
        if constexpr (!W::kFromZero) {
            products(std::integral_constant<int, 0>{}, std::integral_constant<int, NP>{});
        } else if constexpr (W::kScaled) {
            products(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{});
            w.times(kPieceDown);
            products(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
            w.times(kPieceDown);
            products(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
        } else {
            // from zero: first the small pieces of all ranks, then the leading ones, so that only the latter's
            // additions round at the size of the sum (512 tokens of rank 64, H = 4096, error against 64 bits: 1.24e-7 -> 1.17e-7
            // in binary16, 1.15e-7 -> 1.00e-7 in bfloat16)
            products(std::integral_constant<int, 1>{}, std::integral_constant<int, NP>{});
            products(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
        }
        w.end(yt, e_cur);
        // what was requested for the next tile has arrived, and so have the stores of the previous one
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        w.store_y(t, row_cur, yt);
        if (t + 1 < tiles) {
            // every wavefront's part of V(t + 1) is in LDS, and every one has read V(t)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < kYLoads; ++i) {
                row_cur[i] = row_next[i];
                yt[i] = y_next[i];
            }
            e_cur = e_next;
            w.load_rows(min(t + 2, tiles - 1), row_next);
        }
    }
}

// Adapters of 129 to 256 ranks: B of up to eight stages in registers, V of a tile through LDS in two halves of four
// stages, one buffer each: while a half is multiplied the next is on its way.  A barrier per half.  No registers are left for the y of
// the next tile if it is fp32.  The sums are formed as in expand_mfma_stream, which read V in every wavefront and B per
// tile, stage after stage, a chain of
// dependent loads: 2615 tokens of ranks 5-200 (a third of them 200), H = 2568, 3 slots, fp32 y 57.8 -> 53.6 us; all of rank 200 109 -> 85.
template <int DT, bool Y16, int NP>
__device__ __forceinline__ void expand_mfma_halves(const Item &it, int wave, const int32_t *__restrict__ pbl,
                                                   const uint16_t *__restrict__ pool,
                                                   const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                   const uint16_t *__restrict__ vfrag, const int8_t *__restrict__ vexp,
                                                   void *__restrict__ y, unsigned char *lds)
{
    typedef ExpandWave<DT, Y16, NP> W;
    typedef typename W::i32x4 i32x4;
    static_assert(!W::kScaled, "pieces of a scale of their own need sums of their own");
    constexpr int kYLoads = W::kYLoads;
    constexpr int kHalf = kMsRanks / 32;          // stages of a half
    constexpr int kFrags = 2 * kHalf * NP;        // operand fragments (1 KiB) of a half
    constexpr bool kAheadY = !W::kFromZero;       // y starts in the accumulators: requested a tile ahead
    const int n_kk = v_stride >> 4, n_rb = (v_stride + kMsRanks - 1) / kMsRanks;
    const int lane = threadIdx.x & (kWave - 1);
    const int tiles = it.run & 0xff;
    const int stages = (it.rank + 31) >> 5;       // kHalf + 1 .. 2 * kHalf
    auto load_v = [&](int t, int h) { // this wavefront's part of a half of tile t
        const unsigned char *src = reinterpret_cast<const unsigned char *>(vfrag + vfrag_index(it.tile + t, 2 * kHalf * h, 0, n_kk, NP)) + lane * 16;
        unsigned char *dst = lds + h * (kFrags * 1024);
        const int n = h == 0 ? kFrags : 2 * (stages - kHalf) * NP;
        for (int f = wave; f < n; f += 4) load_to_lds<0>(src + f * 1024, dst + f * 1024);
    };
    auto hand_over = [&]() { // what was requested has arrived, in every wavefront
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    const int colw = it.a + wave * 64;            // this wavefront's first column
    load_v(0, 0);
    if (colw >= it.a + it.b) {                    // no columns: it only does its part of the copying
        hand_over();
        for (int t = 0; t < tiles; ++t) {
            load_v(t, 1);
            hand_over();
            if (t + 1 < tiles) {
                load_v(t + 1, 0);
                hand_over();
            }
        }
        return;
    }
    W w(it, colw, pbl, pool, tok_idx, H, y, reinterpret_cast<uint32_t *>(lds + 2 * kFrags * 1024 + wave * kWaveLds));
    int row_cur[kYLoads], row_next[kYLoads];
    u32x4 yt[kYLoads];
    [[maybe_unused]] u32x4 y_next[kYLoads];
    u32x4 bop[2 * kHalf][2][2];
    w.load_rows(0, row_cur);
    w.load_operands(stages, bop, [&]() {
        if constexpr (kAheadY) w.load_y(row_cur, yt);
    });
    const uint32_t frag_at = lds_address(lds) + lane * 16;
    hand_over();
    for (int t = 0; t < tiles; ++t) {
        load_v(t, 1);
        if constexpr (!kAheadY) w.load_y(row_cur, yt);
        [[maybe_unused]] const i32x4 *et = reinterpret_cast<const i32x4 *>(vexp + (int64_t)(it.tile + t) * n_rb * 32 + w.q * 16);
        [[maybe_unused]] i32x4 scale = i32x4{0, 0, 0, 0};
        if constexpr (DT == SLORA_F16) scale = et[0];
        w.begin(yt, scale);
        auto products = [&](auto stage) {
            constexpr int st = decltype(stage)::value;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                u32x4 piece[NP];
                if (k == 0)
                    lds_read_pieces<NP, 2 * NP * st * 1024>(frag_at, piece);
                else
                    lds_read_pieces<NP, (2 * NP * st + NP) * 1024>(frag_at, piece);
#pragma unroll
                for (int p = 0; p < NP; ++p) W::multiply(w.acc, piece[p], bop[st][k]);
            }
        };
        products(std::integral_constant<int, 0>{});
        products(std::integral_constant<int, 1>{});
        products(std::integral_constant<int, 2>{});
        products(std::integral_constant<int, 3>{});
        if constexpr (kAheadY) w.load_rows(min(t + 1, tiles - 1), row_next);
        hand_over(); // the second half is in LDS, the first has been read
        if (t + 1 < tiles) {
            load_v(t + 1, 0);
            if constexpr (kAheadY) w.load_y(row_next, y_next);
        }
        if constexpr (DT == SLORA_F16) { // the sums so far follow the next block's scale
            const i32x4 to = et[2];
            W::scale_rows(w.acc, scale, to);
            scale = to;
        }
        products(std::integral_constant<int, 4>{});
        if (stages > 5) products(std::integral_constant<int, 5>{});
        if (stages > 6) products(std::integral_constant<int, 6>{});
        if (stages > 7) products(std::integral_constant<int, 7>{});
        if constexpr (!kAheadY) w.load_rows(min(t + 1, tiles - 1), row_next);
        w.end(yt, scale);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // the stores that follow are waited for a half later
        w.store_y(t, row_cur, yt);
        if (t + 1 < tiles) {
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < kYLoads; ++i) {
                row_cur[i] = row_next[i];
                if constexpr (kAheadY) yt[i] = y_next[i];
            }
        }
    }
}

// adapters of more ranks: V and B come from memory for every tile
template <int DT, bool Y16, int NP>
__device__ __forceinline__ void expand_mfma_stream(const Item &it, int wave, const int32_t *__restrict__ pbl,
                                                   const uint16_t *__restrict__ pool,
                                                   const int32_t *__restrict__ tok_idx, int H, int v_stride,
                                                   const uint16_t *__restrict__ vfrag, const int8_t *__restrict__ vexp,
                                                   void *__restrict__ y, unsigned char *lds)
{
    typedef ExpandWave<DT, Y16, NP> W;
    typedef typename W::i32x4 i32x4;
    constexpr int kYLoads = W::kYLoads;
    const int n_kk = v_stride >> 4, n_rb = (v_stride + kMsRanks - 1) / kMsRanks;
    const int colw = it.a + wave * 64;            // this wavefront's first column
    if (colw >= it.a + it.b) return;              // whole wavefront; no barrier is used below
    W w(it, colw, pbl, pool, tok_idx, H, y, reinterpret_cast<uint32_t *>(lds + wave * kWaveLds));
    const u32x4 *frags = reinterpret_cast<const u32x4 *>(vfrag) + w.lane;
    for (int t = 0; t < w.tiles; ++t) {
        const int tile = it.tile + t;
        int row[kYLoads], pg[4];
        u32x4 yt[kYLoads];
        w.load_rows(t, row);
        w.load_pg(0, pg);
        const i32x4 *et = reinterpret_cast<const i32x4 *>(vexp + (int64_t)tile * n_rb * 32 + w.q * 16);
        [[maybe_unused]] i32x4 e_cur = i32x4{0, 0, 0, 0};
        if constexpr (DT == SLORA_F16) e_cur = et[0];
        w.load_y(row, yt);
        w.begin(yt, e_cur);
        // pieces of a scale of their own have a sum of their own
        [[maybe_unused]] f32x16 mid[2], low[2];
        if constexpr (W::kScaled) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) mid[nb][v] = low[nb][v] = 0.f;
        }
        for (int k0 = 0; k0 < it.rank; k0 += 32) {
            if constexpr (DT == SLORA_F16) {
                if (k0 > 0 && (k0 & (kMsRanks - 1)) == 0) { // the sums so far follow the next block's scale
                    const i32x4 e_next = et[(k0 / kMsRanks) * 2];
                    W::scale_rows(w.acc, e_cur, e_next);
                    if constexpr (W::kScaled) {
                        W::scale_rows(mid, e_cur, e_next);
                        W::scale_rows(low, e_cur, e_next);
                    }
                    e_cur = e_next;
                }
            }
            u32x4 b[4], piece[2][NP], op[2][2];
            w.load_b(pg, b);
            w.load_pg(k0 + 32, pg); // clamped to the last rank past the end
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int p = 0; p < NP; ++p) piece[s][p] = frags[vfrag_index(tile, (k0 >> 4) + s, p, n_kk, NP) / 8];
            w.transpose_b(b, op);
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    if constexpr (W::kScaled)
                        W::multiply(p == 0 ? w.acc : p == 1 ? mid : low, piece[s][p], op[s]);
                    else
                        W::multiply(w.acc, piece[s][p], op[s]);
                }
        }
        if constexpr (W::kScaled) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) w.acc[nb][v] += kPieceDown * (mid[nb][v] + kPieceDown * low[nb][v]);
        }
        w.end(yt, e_cur);
        w.store_y(t, row, yt);
    }
}

template <int DT, bool Y16, int NP>
__global__ __launch_bounds__(kMfmaThreads, 2) void expand_mfma_kernel(const Item *__restrict__ items,
                                                                    const int32_t *__restrict__ arena,
                                                                    const uint16_t *__restrict__ pool,
                                                                    const int32_t *__restrict__ tok_idx, int H,
                                                                    int v_stride, int parts, MultiArgs args)
{
    // two buffers of V, for the most 32-rank stages that an adapter of the plan has in one (four from 97 ranks on: 129 to 256 in halves), then each
    // wavefront's own part
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int cs = blockIdx.x % args.n;
    // a run of tiles, or this workgroup's part of it
    Item it = items[blockIdx.x / args.n / parts];
    if (parts > 1) {
        const int part = (int)(blockIdx.x / args.n % parts), tiles = it.run & 0xff;
        const int t0 = tiles * part / parts, t1 = tiles * (part + 1) / parts;
        if (t0 == t1) return; // the whole workgroup
        it.pos0 += t0 * kMfmaTok;
        it.tile += t0;
        it.run = (t1 - t0) + 256 * (t1 == tiles ? it.run >> 8 : kMfmaTok);
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t *pbl = arena + it.arena_off + (int64_t)args.slot[cs] * 2 * it.rank + it.rank;
    const uint16_t *vfrag = reinterpret_cast<const uint16_t *>(args.v[cs] + args.vfrag_off);
    const int8_t *vexp = reinterpret_cast<const int8_t *>(args.v[cs] + args.vexp_off);
#define SLORA_ME(S) expand_mfma_run<DT, Y16, NP, S>(it, wave, pbl, pool, tok_idx, H, v_stride, vfrag, vexp, args.y[cs], lds)
    if (it.rank <= 32) SLORA_ME(1);
    else if (it.rank <= 64) SLORA_ME(2);
    else if (it.rank <= 96) SLORA_ME(3);
    else if (it.rank <= 128) SLORA_ME(4);
    // One tile has nothing to keep B for, and the halves wait for all of B before the first product, which the stream does not.  us of the expand of
    // sixteen prompts, one slot, one tile per workgroup, halves / stream, fp32 y: rank 200, H = 1712 29.3 / 26.8 (bf16 35.7 / 31.5), rank 130, H = 2048
    // 36.3 / 33.5, rank 256, H = 3072 40.4 / 38.2; 16-bit y: rank 160, H = 1496 22.5 / 20.4, rank 256, H = 1536 28.1 / 25.9, rank 160, H = 2568 32.5 / 30.4, but at
    // multiples of 1024, why is not known, rank 200, H = 1024, bf16 21.7 / 23.7, rank 256, H = 2048, bf16 38.6 / 40.2, rank 130, H = 3072 33.4 / 35.5.
    else if (it.rank <= 2 * kMsRanks && !kScaledPieces<DT, NP> && ((it.run & 0xff) > 1 || (Y16 && H % 1024 == 0))) {
        if constexpr (!kScaledPieces<DT, NP>)
            expand_mfma_halves<DT, Y16, NP>(it, wave, pbl, pool, tok_idx, H, v_stride, vfrag, vexp, args.y[cs], lds);
    }
    else expand_mfma_stream<DT, Y16, NP>(it, wave, pbl, pool, tok_idx, H, v_stride, vfrag, vexp, args.y[cs], lds);
#undef SLORA_ME
}

// ---------------------------------------------------------------------------------------
// Scratch for callers that cannot allocate: v = x*A of one call goes here instead of into a
// buffer from hipMalloc.  One copy per GPU, held until the process ends; every element the
// expand reads is written by the shrink of the same call, so nothing has to start at zero.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[SLORA_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[kMaxDevices]; // device address of `scratch` on each GPU, 0 = not resolved yet

int32_t check_launch(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SLORA_EHIP, "%s: %s", what, hipGetErrorString(e));
    return SLORA_OK;
}

} // namespace

// The device address of the static scratch on `device`, which must be the current device: the
// array's name is only a host-side handle, each GPU has its own copy at its own address.
int32_t static_scratch_address(int device, void **out)
{
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return fail(SLORA_EINVAL, "device %d outside [0, %d)", device, kMaxDevices);
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(SLORA_EHIP, "hipGetSymbolAddress(static scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return SLORA_OK;
}

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
int32_t launch_write_pages(slora_pool *pool, const int32_t *d_idx, int64_t n, const void *d_src, void *stream,
                           int32_t max_groups)
{
    if (n <= 0) return SLORA_OK;
    if (n >= (int64_t(1) << 31)) return fail(SLORA_EINVAL, "too many pages in one call");
    if (reinterpret_cast<uintptr_t>(d_src) & 15) return fail(SLORA_EINVAL, "src must be 16-byte aligned");
    const int64_t groups = max_groups > 0 && n > max_groups ? max_groups : n;
    hipLaunchKernelGGL(write_pages_kernel, dim3((unsigned)groups), dim3(256), 0, (hipStream_t)stream,
                       static_cast<uint16_t *>(pool->dev_base), d_idx, static_cast<const uint16_t *>(d_src), pool->H, n);
    return check_launch("write_pages");
}

int32_t launch_copy(void *dst, const void *src, size_t bytes, void *stream)
{
    const int64_t n = (int64_t)(bytes / 16); // whole work items: a multiple of 32 bytes
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 64)), dim3(256), 0, (hipStream_t)stream,
                       static_cast<u32x4 *>(dst), static_cast<const u32x4 *>(src), n);
    return check_launch("copy_lists");
}

int32_t launch_gather(slora_pool *pool, int64_t arena_entry, int32_t rank, void *dev_out, void *stream)
{
    hipLaunchKernelGGL(gather_pages_kernel, dim3((unsigned)rank), dim3(256), 0, (hipStream_t)stream,
                       static_cast<const uint16_t *>(pool->dev_base), pool->d_arena + arena_entry,
                       static_cast<uint16_t *>(dev_out), pool->H);
    return check_launch("gather_pages");
}

// A launch with more than 64 KiB of dynamic LDS has to be allowed once per kernel instance and device;
// `done` holds a bit per device.
static hipError_t allow_lds(std::atomic<uint64_t> &done, int device, const void *kernel, size_t lds)
{
    const uint64_t bit = uint64_t(1) << (device & 63);
    if (lds <= 65536 || (done.load() & bit)) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess) done.fetch_or(bit);
    return e;
}

// loads per block of the vector shrink: as few blocks per page as 8 loads allow, then the smallest U that fits
static int shrink_loads_per_block(int H)
{
    const int per_lane = (H / 8 + kWave - 1) / kWave;
    const int nblk = (per_lane + 7) / 8;
    return std::max(4, (per_lane + nblk - 1) / nblk);
}

static int32_t launch_small(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16)
{
    slora_pool *pool = plan->pool;
    const uint16_t *base = static_cast<const uint16_t *>(pool->dev_base);
    hipStream_t st = (hipStream_t)stream;
    const int H = pool->H;
    const dim3 grid((unsigned)(plan->ve_items.size() * (size_t)n));
    const int tok = plan->max_expand_tok <= 2 ? plan->max_expand_tok : kExpandTok;
    // at most 4 x (8 KiB of x + 6.1 KiB): below the 64 KiB that every kernel may have
    const size_t lds = (size_t)tok * (H * 2 + (kSmallRanks + (kSplitWaves - 1) * 8 * kWave) * sizeof(float));
#define SLORA_SMALL(DT, Y)                                                                                      \
    hipLaunchKernelGGL((lora_vec_small_kernel<DT, Y>), grid, dim3(kSmallWaves *kWave), lds, st, plan->d_ve,     \
                       pool->d_arena, base, plan->d_tok_idx, H, plan->v_stride, args)
    if (pool->dtype == SLORA_F16) {
        if (y16) SLORA_SMALL(SLORA_F16, true);
        else SLORA_SMALL(SLORA_F16, false);
    } else {
        if (y16) SLORA_SMALL(SLORA_BF16, true);
        else SLORA_SMALL(SLORA_BF16, false);
    }
#undef SLORA_SMALL
    return check_launch("lora_vec_small");
}

int32_t launch_fused(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16, const Route &route)
{
    slora_pool *pool = plan->pool;
    if (route.small) return launch_small(plan, n, args, stream, y16);
    if (plan->vf_items.empty()) return SLORA_OK;
    const uint16_t *base = static_cast<const uint16_t *>(pool->dev_base);
    hipStream_t st = (hipStream_t)stream;
    const int H = pool->H;
    const int strips = (H + 511) / 512;
    const dim3 block((unsigned)(std::min(strips, 16) * kWave));
    const dim3 grid((unsigned)(plan->vf_items.size() * (size_t)n));
    const int v_pad = plan->v_stride;
    const size_t lds = (size_t)kExpandTok * H * 2 + (size_t)kExpandTok * v_pad * sizeof(float);
    const int U = shrink_loads_per_block(H);
    hipError_t attr = hipSuccess;
#define SLORA_FUSED(DT, Y, UU)                                                                                       \
    {                                                                                                                \
        static std::atomic<uint64_t> done{0};                                                                        \
        attr = allow_lds(done, pool->device, reinterpret_cast<const void *>(&lora_vec_fused_kernel<DT, Y, UU>), lds); \
        if (attr == hipSuccess)                                                                                      \
            hipLaunchKernelGGL((lora_vec_fused_kernel<DT, Y, UU>), grid, block, lds, st, plan->d_vf, pool->d_arena, \
                               base, plan->d_tok_idx, H, v_pad, args);                                               \
    }
#define SLORA_FUSED_U(DT, Y)                      \
    switch (U) {                                  \
    case 4: SLORA_FUSED(DT, Y, 4); break;         \
    case 5: SLORA_FUSED(DT, Y, 5); break;         \
    case 6: SLORA_FUSED(DT, Y, 6); break;         \
    case 7: SLORA_FUSED(DT, Y, 7); break;         \
    default: SLORA_FUSED(DT, Y, 8); break;        \
    }
    if (pool->dtype == SLORA_F16) {
        if (y16) { SLORA_FUSED_U(SLORA_F16, true) } else { SLORA_FUSED_U(SLORA_F16, false) }
    } else {
        if (y16) { SLORA_FUSED_U(SLORA_BF16, true) } else { SLORA_FUSED_U(SLORA_BF16, false) }
    }
#undef SLORA_FUSED_U
#undef SLORA_FUSED
    if (attr != hipSuccess) return fail(SLORA_EHIP, "hipFuncSetAttribute(LDS size): %s", hipGetErrorString(attr));
    return check_launch("lora_vec_fused");
}

// LDS of the rank-split expand: its partial sums
constexpr size_t kSplitLds = (size_t)kSplitWaves * kExpandTok * 8 * kWave * sizeof(float);

int32_t launch_clear(void *dst, size_t bytes, void *stream)
{
    const int64_t n = (int64_t)(bytes / 16);
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256), 0, (hipStream_t)stream,
                       static_cast<u32x4 *>(dst), n);
    return check_launch("clear");
}

int32_t launch_chain(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16, const Route &route)
{
    slora_pool *pool = plan->pool;
    const uint16_t *base = static_cast<const uint16_t *>(pool->dev_base);
    hipStream_t st = (hipStream_t)stream;
    const int H = pool->H;
    ChainLists c{};
    c.shrink = plan->d_vs;
    c.expand = plan->d_ve;
    c.n_shrink = (unsigned)plan->n_vs(route);
    c.turn = plan->chain_of(route).shared ? 6 : 5;
    c.hand = plan->set->hand;
    c.hand_slot = plan->chain_of(route).words;
    c.launch = plan->set->launch;
    c.polls = (int32_t)pool->hand_polls;
    const dim3 grid((unsigned)n, (unsigned)plan->chain_wgs(route));
    const size_t lds = std::max(kSplitLds, (size_t)plan->chain_of(route).tok * chain_chunks(H) * kWave * 16);
#define SLORA_CHAIN(DT, Y, UU) \
    case UU: hipLaunchKernelGGL((lora_vec_chain_kernel<DT, Y, UU>), grid, dim3(kShrinkThreads), lds, st, c, pool->d_arena, base, plan->d_tok_idx, H, plan->v_stride, args); break
#define SLORA_CHAIN_U(DT, Y)                                                                                             \
    switch (chain_chunks(H)) {                                                                                           \
        SLORA_CHAIN(DT, Y, 1); SLORA_CHAIN(DT, Y, 2); SLORA_CHAIN(DT, Y, 3); SLORA_CHAIN(DT, Y, 4); SLORA_CHAIN(DT, Y, 5); \
        SLORA_CHAIN(DT, Y, 6); SLORA_CHAIN(DT, Y, 7); SLORA_CHAIN(DT, Y, 8); SLORA_CHAIN(DT, Y, 10); SLORA_CHAIN(DT, Y, 12); \
        SLORA_CHAIN(DT, Y, 16);                                                                                          \
    }
    if (pool->dtype == SLORA_F16) {
        if (y16) { SLORA_CHAIN_U(SLORA_F16, true) } else { SLORA_CHAIN_U(SLORA_F16, false) }
    } else {
        if (y16) { SLORA_CHAIN_U(SLORA_BF16, true) } else { SLORA_CHAIN_U(SLORA_BF16, false) }
    }
#undef SLORA_CHAIN_U
#undef SLORA_CHAIN
    return check_launch("lora_vec_chain");
}

int32_t launch_shrink(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, const Route &route)
{
    slora_pool *pool = plan->pool;
    const uint16_t *base = static_cast<const uint16_t *>(pool->dev_base);
    hipStream_t st = (hipStream_t)stream;
    const size_t n_vs = route.chain ? 0 : plan->n_vs(route);
    int32_t rc = SLORA_OK;
    if (n_vs > 0 && route.gang) {
        const dim3 grid((unsigned)(plan->shrink_wgs(route) * (size_t)n));
        const size_t lds = std::max(kGangLds, (size_t)plan->max_gv_tok * pool->H * 2);
        const int U = shrink_loads_per_block(pool->H);
#define SLORA_GANG(DT, UU) \
    hipLaunchKernelGGL((shrink_gang_kernel<DT, UU>), grid, dim3(kShrinkThreads), lds, st, plan->d_gs, (unsigned)plan->n_gs(route), plan->d_gv, pool->d_arena, base, plan->d_tok_idx, pool->H, plan->v_stride, args)
#define SLORA_GANG_U(DT)                      \
    switch (U) {                              \
    case 4: SLORA_GANG(DT, 4); break;         \
    case 5: SLORA_GANG(DT, 5); break;         \
    case 6: SLORA_GANG(DT, 6); break;         \
    case 7: SLORA_GANG(DT, 7); break;         \
    default: SLORA_GANG(DT, 8); break;        \
    }
        if (pool->dtype == SLORA_F16) {
            SLORA_GANG_U(SLORA_F16)
        } else {
            SLORA_GANG_U(SLORA_BF16)
        }
#undef SLORA_GANG_U
#undef SLORA_GANG
        rc = check_launch("shrink_gang");
        if (rc != SLORA_OK) return rc;
    } else if (n_vs > 0) {
        const dim3 grid((unsigned)(n_vs * (size_t)n));
        const size_t lds = (size_t)plan->max_shrink_tok * pool->H * 2;
        const int U = shrink_loads_per_block(pool->H);
#define SLORA_LAUNCH_SHRINK(DT, UU)                                                                              \
    hipLaunchKernelGGL((shrink_vec_kernel<DT, UU>), grid, dim3(kShrinkThreads), lds, st, plan->d_vs, pool->d_arena, \
                       base, plan->d_tok_idx, pool->H, plan->v_stride, args)
#define SLORA_SHRINK_U(DT)                                \
    switch (U) {                                          \
    case 4: SLORA_LAUNCH_SHRINK(DT, 4); break;            \
    case 5: SLORA_LAUNCH_SHRINK(DT, 5); break;            \
    case 6: SLORA_LAUNCH_SHRINK(DT, 6); break;            \
    case 7: SLORA_LAUNCH_SHRINK(DT, 7); break;            \
    default: SLORA_LAUNCH_SHRINK(DT, 8); break;           \
    }
        if (pool->dtype == SLORA_F16) {
            SLORA_SHRINK_U(SLORA_F16)
        } else {
            SLORA_SHRINK_U(SLORA_BF16)
        }
#undef SLORA_SHRINK_U
#undef SLORA_LAUNCH_SHRINK
        rc = check_launch("shrink_vec");
        if (rc != SLORA_OK) return rc;
    }
    if (!plan->ms_items.empty() && plan->mfma_on(route)) {
        const dim3 grid((unsigned)((plan->ms_items.size() << route.sub) * (size_t)n));
        const size_t lds = (size_t)plan->ms_lds[route.sub];
#define SLORA_MSK(DT)                                                                                                \
    {                                                                                                                \
        static std::atomic<uint64_t> done{0};                                                                        \
        hipError_t e = allow_lds(done, pool->device, reinterpret_cast<const void *>(&shrink_mfma_kernel<DT>), lds);            \
        if (e != hipSuccess) return fail(SLORA_EHIP, "hipFuncSetAttribute(LDS size): %s", hipGetErrorString(e));     \
        hipLaunchKernelGGL(shrink_mfma_kernel<DT>, grid, dim3(kMfmaThreads), lds, st, plan->d_ms, pool->d_arena,     \
                           base, plan->d_tok_idx, pool->H, plan->v_stride, kMsTok >> route.sub, args);               \
    }
        if (pool->dtype == SLORA_F16) SLORA_MSK(SLORA_F16) else SLORA_MSK(SLORA_BF16)
#undef SLORA_MSK
        rc = check_launch("shrink_mfma");
        if (rc != SLORA_OK) return rc;
        if (plan->n_sync > 0) {
            const dim3 jgrid((unsigned)((size_t)plan->n_sync * (kMsTok / 32) * (size_t)n));
            auto *join = pool->dtype != SLORA_F16 ? (plan->dual ? &join_shares_kernel<SLORA_BF16, 3, true> : &join_shares_kernel<SLORA_BF16, 3, false>)
                         : plan->dual             ? &join_shares_kernel<SLORA_F16, 3, true>
                                                  : &join_shares_kernel<SLORA_F16, 2, false>;
            hipLaunchKernelGGL(join, jgrid, dim3((unsigned)(join_waves(plan->dual) * kWave)), 0, st, plan->d_mj, plan->v_stride, args);
            rc = check_launch("join_shares");
            if (rc != SLORA_OK) return rc;
        }
    }
    return SLORA_OK;
}

int32_t launch_expand(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16, const Route &route)
{
    slora_pool *pool = plan->pool;
    const uint16_t *base = static_cast<const uint16_t *>(pool->dev_base);
    hipStream_t st = (hipStream_t)stream;
    // (storage type, y type) -> kernel instance
#define SLORA_PICK(KERNEL)                                                                   \
    (pool->dtype == SLORA_F16 ? (y16 ? KERNEL<SLORA_F16, true> : KERNEL<SLORA_F16, false>)   \
                              : (y16 ? KERNEL<SLORA_BF16, true> : KERNEL<SLORA_BF16, false>))
    const size_t n_ve = route.chain ? 0 : plan->n_ve(route);
    if (n_ve > 0) {
        const dim3 grid((unsigned)(plan->expand_wgs(route) * (size_t)n));
        if (plan->expand_split) {
#define SLORA_SPLIT(DT, Y)                                                                                                  \
    (route.gang_expand && plan->fours[y16] ? &expand_vec_split_kernel<DT, Y, true> : &expand_vec_split_kernel<DT, Y, false>)
            auto *kernel = pool->dtype == SLORA_F16 ? (y16 ? SLORA_SPLIT(SLORA_F16, true) : SLORA_SPLIT(SLORA_F16, false))
                                                    : (y16 ? SLORA_SPLIT(SLORA_BF16, true) : SLORA_SPLIT(SLORA_BF16, false));
#undef SLORA_SPLIT
            hipLaunchKernelGGL(kernel, grid, dim3(kSplitWaves * kWave), kSplitLds, st, route.gang_expand ? plan->d_ge : plan->d_ve,
                               pool->d_arena, base, plan->d_tok_idx, pool->H, plan->v_stride, args);
        } else
            hipLaunchKernelGGL(SLORA_PICK(expand_vec_kernel), grid, dim3((unsigned)plan->expand_threads), 0, st,
                               plan->d_ve, pool->d_arena, base, plan->d_tok_idx, pool->H, plan->v_stride, args);
        int32_t rc = check_launch("expand_vec");
        if (rc != SLORA_OK) return rc;
    }
    if (!plan->me_items.empty() && plan->mfma_on(route)) {
        const dim3 grid((unsigned)(plan->me_items.size() * (size_t)route.parts * (size_t)n));
        // LDS: two buffers of V fragments (the plan's most 32-rank stages) and the wavefronts' own parts
        const size_t lds = (size_t)2 * plan->me_stages * 2 * plan->pieces(pool->dtype) * 1024 + 4 * kWaveLds;
#define SLORA_MEK(DT, Y, NP)                                                                                           \
    {                                                                                                                \
        static std::atomic<uint64_t> done{0};                                                                        \
        hipError_t e = allow_lds(done, pool->device, reinterpret_cast<const void *>(&expand_mfma_kernel<DT, Y, NP>), lds);     \
        if (e != hipSuccess) return fail(SLORA_EHIP, "hipFuncSetAttribute(LDS size): %s", hipGetErrorString(e));     \
        hipLaunchKernelGGL((expand_mfma_kernel<DT, Y, NP>), grid, dim3(kMfmaThreads), lds, st, plan->d_me,           \
                           pool->d_arena, base, plan->d_tok_idx, pool->H, plan->v_stride, route.parts, args);        \
    }
        if (pool->dtype == SLORA_BF16) {
            if (y16) SLORA_MEK(SLORA_BF16, true, 3) else SLORA_MEK(SLORA_BF16, false, 3)
        } else if (plan->pieces(SLORA_F16) == 2) {
            if (y16) SLORA_MEK(SLORA_F16, true, 2) else SLORA_MEK(SLORA_F16, false, 2)
        } else {
            if (y16) SLORA_MEK(SLORA_F16, true, 3) else SLORA_MEK(SLORA_F16, false, 3)
        }
#undef SLORA_MEK
        int32_t rc = check_launch("expand_mfma");
        if (rc != SLORA_OK) return rc;
    }
#undef SLORA_PICK
    return SLORA_OK;
}

} // namespace slora
