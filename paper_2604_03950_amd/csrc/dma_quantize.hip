// Standalone MX quantizer (paper, Alg. 2 Steps 1, 3-7; Alg. 3): one streaming pass, HBM bound.
//
// Work split: one lane converts one 16-byte chunk (8 bf16); the 4 lanes of a quad hold one MX block
// of 32 elements, so the block maximum is two DPP quad permutes.  Loads are 16 B per lane and
// contiguous across the wave; code stores are 4 B (FP4) / 8 B (FP8) per lane, contiguous; the scale
// byte is written by the first lane of each quad.
#include "dma_device.hpp"
#include "dma_internal.hpp"
#include <math.h>

namespace dma {

constexpr int QUANT_THREADS = 256;
constexpr int QUANT_UNROLL = 4;     // chunks per thread

// MODE: 1 = E4M3 only, 2 = E2M1 only, 3 = both (low copy E2M1 + high copy E4M3), 4 = E5M2 only.
// PER_TOKEN: Alg. 2 Step 2: the row (2^row_shift = D / 8 consecutive lanes, 4 .. 64) is multiplied by 2688 / rowmax before
// the shared scales are formed, and rowmax / 2688 goes to token_scales[row].  Bound by the same read and writes, and by
// vector work: the row maximum goes through DPP and lane swaps, the lanes of a quad share the divisions (lane q those of
// chunk round q), the block maximum is taken before the scaling, and rows are counted with a shift.  32 heads of
// 8192 x 128 to MXFP4 19.3 -> 13.8 us, to MXFP8 20.0 -> 16.7 (without the token scale 13.9 and 16.7).
template <int MODE, bool IS_QUERY, bool PER_TOKEN>
__global__ void __launch_bounds__(QUANT_THREADS)
mx_quantize_kernel(const v4i* __restrict__ x, int64_t n_chunks, float c,
                   int* __restrict__ codes4, uint8_t* __restrict__ scales4,
                   v2i* __restrict__ codes8, uint8_t* __restrict__ scales8,
                   float* __restrict__ token_scales, int row_shift)
{
    const int64_t base = ((int64_t)blockIdx.x * QUANT_UNROLL) * QUANT_THREADS + threadIdx.x;
    v4i w[QUANT_UNROLL];
#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        const int64_t ch = base + (int64_t)u * QUANT_THREADS;
        w[u] = (ch < n_chunks) ? __builtin_nontemporal_load(x + ch) : v4i{0, 0, 0, 0};
    }
    float bmax[QUANT_UNROLL], inv[QUANT_UNROLL];
    if constexpr (PER_TOKEN) {
        static_assert(QUANT_UNROLL == 4, "one chunk round per lane of a quad");
        float rmax[QUANT_UNROLL];
#pragma unroll
        for (int u = 0; u < QUANT_UNROLL; ++u) {
            float v[8];
            unpack8<IS_QUERY>(w[u], c, v);
            bmax[u] = rmax[u] = quad_max(amax8(v));
        }
        // row maximum: from the quad to the 8, 16, 32 or 64 lanes of the row (rows never straddle a wave)
        if (row_shift >= 3) {
#pragma unroll
            for (int u = 0; u < QUANT_UNROLL; ++u) rmax[u] = half_row_max(rmax[u]);
        }
        if (row_shift >= 4) {
#pragma unroll
            for (int u = 0; u < QUANT_UNROLL; ++u) rmax[u] = full_row_max(rmax[u]);
        }
        if (row_shift >= 5) {
#pragma unroll
            for (int u = 0; u < QUANT_UNROLL; ++u) rmax[u] = row_pair_max(rmax[u]);
        }
        if (row_shift >= 6) {
#pragma unroll
            for (int u = 0; u < QUANT_UNROLL; ++u) rmax[u] = cross_half_max(rmax[u]);
        }
        const int q = threadIdx.x & 3;
        float s_q, mine;
        token_scale(q == 0 ? rmax[0] : q == 1 ? rmax[1] : q == 2 ? rmax[2] : rmax[3], s_q, mine);
        const int m = __float_as_int(mine);
        inv[0] = __int_as_float(__builtin_amdgcn_mov_dpp(m, 0x00, 0xF, 0xF, true));
        inv[1] = __int_as_float(__builtin_amdgcn_mov_dpp(m, 0x55, 0xF, 0xF, true));
        inv[2] = __int_as_float(__builtin_amdgcn_mov_dpp(m, 0xAA, 0xF, 0xF, true));
        inv[3] = __int_as_float(__builtin_amdgcn_mov_dpp(m, 0xFF, 0xF, 0xF, true));
        const int64_t mine_ch = base + (int64_t)q * QUANT_THREADS;          // the lane's own chunk of round q
        if ((threadIdx.x & ((1 << row_shift) - 1)) < 4 && mine_ch < n_chunks) token_scales[mine_ch >> row_shift] = s_q;
    }
#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        const int64_t ch = base + (int64_t)u * QUANT_THREADS;
        float v[8];
        unpack8<IS_QUERY>(w[u], c, v);
        float amax;
        if constexpr (PER_TOKEN) {
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = __fmul_rn(v[t], inv[u]);
            // rounding is monotone: the maximum of the scaled block is the scaled maximum (a factor of 0, of a row with an
            // infinity, makes every finite element 0)
            amax = inv[u] == 0.f ? 0.f : __fmul_rn(bmax[u], inv[u]);
        } else {
            amax = quad_max(amax8(v));              // every lane of the wave executes the DPP
        }
        if (ch >= n_chunks) continue;
        const bool writes_scale = (threadIdx.x & 3) == 0;
        if (MODE & 2) {
            const int code = e8m0_code<FMT_E2M1>(amax);
            __builtin_nontemporal_store(encode8_e2m1(v, code), codes4 + ch);
            if (writes_scale) scales4[ch >> 2] = (uint8_t)code;
        }
        if (MODE & 1) {
            const int code = e8m0_code<FMT_E4M3>(amax);
            __builtin_nontemporal_store(encode8_e4m3(v, code), codes8 + ch);
            if (writes_scale) scales8[ch >> 2] = (uint8_t)code;
        }
        if (MODE & 4) {
            const int code = e8m0_code<FMT_E5M2_X>(amax);
            __builtin_nontemporal_store(encode8_e5m2(v, code), codes8 + ch);
            if (writes_scale) scales8[ch >> 2] = (uint8_t)code;
        }
    }
}

template <int MODE, bool PER_TOKEN>
static int launch_mode(const void* x, int64_t rows, int D, int is_query, void* c4, void* s4, void* c8,
                       void* s8, float* ts, hipStream_t stream)
{
    const int64_t n_chunks = rows * (int64_t)(D / 8);
    if (n_chunks == 0) return DMA_OK_;
    const int64_t per_block = (int64_t)QUANT_THREADS * QUANT_UNROLL;
    const int64_t blocks = (n_chunks + per_block - 1) / per_block;
    if (blocks > 0x7fffffffLL) return DMA_ERR_UNSUPPORTED_;
    const float c = (float)(1.4426950408889634074 / sqrt((double)D));
    const int lpr = D / 8;
    if (PER_TOKEN && (lpr > 64 || (lpr & (lpr - 1)) != 0)) return DMA_ERR_UNSUPPORTED_;
    const int row_shift = __builtin_ctz((unsigned)lpr);
    if (is_query)
        return launch(mx_quantize_kernel<MODE, true, PER_TOKEN>, dim3((unsigned)blocks), dim3(QUANT_THREADS), stream,
                      (const v4i*)x, n_chunks, c, (int*)c4, (uint8_t*)s4, (v2i*)c8, (uint8_t*)s8, ts, row_shift);
    return launch(mx_quantize_kernel<MODE, false, PER_TOKEN>, dim3((unsigned)blocks), dim3(QUANT_THREADS), stream,
                  (const v4i*)x, n_chunks, c, (int*)c4, (uint8_t*)s4, (v2i*)c8, (uint8_t*)s8, ts, row_shift);
}

// Plain copy, 16 bytes per lane: the reference kernel for calibrating HBM traffic counters.
__global__ void __launch_bounds__(QUANT_THREADS)
diag_copy_kernel(const v4i* __restrict__ src, v4i* __restrict__ dst, int64_t n_chunks)
{
    const int64_t i = (int64_t)blockIdx.x * QUANT_THREADS + threadIdx.x;
    if (i < n_chunks) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

int launch_diag_copy(const void* src, void* dst, int64_t bytes, hipStream_t stream)
{
    const int64_t n_chunks = bytes / 16;
    if (n_chunks == 0) return DMA_OK_;
    const int64_t blocks = (n_chunks + QUANT_THREADS - 1) / QUANT_THREADS;
    if (blocks > 0x7fffffffLL) return DMA_ERR_UNSUPPORTED_;
    return launch(diag_copy_kernel, dim3((unsigned)blocks), dim3(QUANT_THREADS), stream, (const v4i*)src, (v4i*)dst, n_chunks);
}

// ---------------------------------------------------------------------------------------------
// Group maxima for Alg. 2 Step 2 at a coarser granularity than the row (Sec. 5.3 names per-block and per-tensor).
// One launch where a workgroup can read a whole block, two otherwise: maxima of rows or of shares into the output, then,
// in place, the maximum over the block or over everything.  Queries: after the pre-scale; the product is monotone, so it is
// taken of the maximum.
// ---------------------------------------------------------------------------------------------
template <int LPR>                                    // lanes per row: D / 8
__global__ void __launch_bounds__(QUANT_THREADS)
row_amax_kernel(const v4i* __restrict__ x, int64_t rows, float c, int prescale, float* __restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * QUANT_THREADS + threadIdx.x;      // one 16-byte chunk per thread
    const int64_t row = t / LPR;
    float a = 0.f;
    if (row < rows) {
        float v[8];
        unpack8<false>(x[t], 1.f, v);
        a = amax8(v);
    }
    a = group_max<LPR>(a);
    if (row < rows && t % LPR == 0) out[row] = prescale ? __fmul_rn(a, c) : a;
}

DMA_DEV float wave_max(float a)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) a = fmaxf(a, __shfl_xor(a, m, 64));
    return a;
}

// One wave per (matrix, block of block_rows rows): maximum of the block, written to each of its rows.
__global__ void __launch_bounds__(64)
block_amax_kernel(float* __restrict__ amax, int64_t S, int64_t block_rows, int64_t blocks_per_matrix)
{
    const int64_t mtx = blockIdx.x / blocks_per_matrix, blk = blockIdx.x % blocks_per_matrix;
    const int64_t r0 = blk * block_rows, r1 = (r0 + block_rows < S) ? r0 + block_rows : S;
    float* p = amax + mtx * S;
    float a = 0.f;
    for (int64_t r = r0 + threadIdx.x; r < r1; r += 64) a = fmaxf(a, p[r]);
    a = wave_max(a);
    for (int64_t r = r0 + threadIdx.x; r < r1; r += 64) p[r] = a;
}

// Maximum over the THREADS threads of a workgroup, returned to all of them.
template <int THREADS>
DMA_DEV float workgroup_max(float a)
{
    a = wave_max(a);
    if constexpr (THREADS > 64) {
        __shared__ float part[THREADS / 64];
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = a;
        __syncthreads();
        a = part[0];
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) a = fmaxf(a, part[w]);
    }
    return a;
}

// Maximum magnitude that the thread sees of n contiguous 16-byte chunks when `stride` threads share them: four loads in
// flight per thread.
DMA_DEV float strided_amax(const v4i* __restrict__ x, int64_t first, int64_t n, int64_t stride)
{
    float a = 0.f;
    for (int64_t i = first; i < n; i += QUANT_UNROLL * stride) {
        v4i w[QUANT_UNROLL];
#pragma unroll
        for (int u = 0; u < QUANT_UNROLL; ++u) w[u] = (i + u * stride < n) ? x[i + u * stride] : v4i{0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < QUANT_UNROLL; ++u) {
            float v[8];
            unpack8<false>(w[u], 1.f, v);
            a = fmaxf(a, amax8(v));
        }
    }
    return a;
}

// Per-block maximum in one pass: a workgroup reads the rows of its block and writes their maximum to each of them.
// Taken for blocks of FUSED_MIN .. FUSED_MAX rows: below, most lanes of a wave would have nothing to read; above, few
// workgroups would read long runs one after the other.  Bound by launch and memory latency up to some thousand blocks,
// by the read above.  The workgroup is as wide as the block asks for (GPU time per call, replayed from a graph; the two
// launches of the general route, this kernel with 256 threads for every block, and as it is):
//   one wave: a block of one round of its loads (4 chunks per lane, 256 chunks), and below 512 chunks when there are
//     many blocks: with 256 threads most would load one chunk or none, and the short workgroups turn over slowly.
//     D = 64, 32 rows: 3.8, 2.4, 2.3 us at 64 blocks, 5.5, 6.5, 3.5 at 4096, 30.4, 40.8, 21.0 at 32768;
//     D = 64, 40 rows: 4.7, 3.3, 2.8 at 818 blocks, 30.1, 33.4, 22.4 at 26214 (50 blocks: 4.1, 2.4, 2.5 with one wave)
//   1024 threads: from 8192 chunks, where 256 would read eight rounds or more one after the other, and no more blocks than
//     the chip has CUs: beyond that a CU hides the latency with several workgroups, and a second wave of wide ones is
//     nearly empty.  D = 128, 512 rows: 5.2, 4.9, 3.9 us with one block, 9.7, 5.8, 4.7 with 256, 12.7, 7.7, 8.8 with 320;
//     1024 rows: 6.5 .. 8.1, 7.9, 5.5 with one, 12.4, 9.0, 6.4 with 128, 18.8, 12.6, 12.6 with 256, 21.2, 14.1, 16.6 with
//     320 (4096 chunks: no clear gain)
//   256 threads: between.
constexpr int64_t FUSED_MIN = 32, FUSED_MAX = 1024;                             // rows
constexpr int64_t WAVE_CHUNKS = 64 * QUANT_UNROLL, WIDE_CHUNKS = 8192;          // 16-byte chunks of a block
constexpr int64_t MANY_BLOCKS = 512, CU_BLOCKS = 256;
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
block_amax_fused_kernel(const v4i* __restrict__ x, int64_t S, int lanes_per_row, int64_t block_rows, int64_t blocks_per_matrix,
                        float c, int prescale, float* __restrict__ amax)
{
    const int64_t mtx = blockIdx.x / blocks_per_matrix, blk = blockIdx.x % blocks_per_matrix;
    const int64_t r0 = blk * block_rows, r1 = (r0 + block_rows < S) ? r0 + block_rows : S;
    const float a = workgroup_max<THREADS>(strided_amax(x + (mtx * S + r0) * lanes_per_row, threadIdx.x, (r1 - r0) * lanes_per_row, THREADS));
    float* p = amax + mtx * S;
    for (int64_t r = r0 + threadIdx.x; r < r1; r += THREADS) p[r] = prescale ? __fmul_rn(a, c) : a;
}

// Per-tensor maximum in two launches, the first bound by the read of x, the second by its launch: up to TENSOR_PARTS
// workgroups leave the maxima of their shares in amax[0 .. parts), then every workgroup of the second grid reduces
// those and writes the result to its rows.  Workgroups of the second grid overwrite the partial maxima while others
// read them, which does no harm: a cell holds its partial maximum or the maximum of all, and the maximum over any such
// mixture is the same number.  (Four launches -- row maxima, runs of 1024 rows, one workgroup over the runs, a copy to
// every row -- stood here before; the figures are at launch_group_amax.)
constexpr int64_t TENSOR_PARTS = 1024;
__global__ void __launch_bounds__(QUANT_THREADS)
tensor_parts_kernel(const v4i* __restrict__ x, int64_t chunks, float c, int prescale, float* __restrict__ amax)
{
    const int64_t first = (int64_t)blockIdx.x * QUANT_THREADS + threadIdx.x;
    const float a = workgroup_max<QUANT_THREADS>(strided_amax(x, first, chunks, (int64_t)gridDim.x * QUANT_THREADS));
    if (threadIdx.x == 0) amax[blockIdx.x] = prescale ? __fmul_rn(a, c) : a;
}
__global__ void __launch_bounds__(QUANT_THREADS)
tensor_spread_kernel(float* amax, int64_t rows, int parts)
{
    float a = 0.f;
    for (int i = threadIdx.x; i < parts; i += QUANT_THREADS)
        a = fmaxf(a, __hip_atomic_load(amax + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    a = workgroup_max<QUANT_THREADS>(a);
    const int64_t base = (int64_t)blockIdx.x * QUANT_UNROLL * QUANT_THREADS + threadIdx.x;
#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        const int64_t r = base + u * QUANT_THREADS;
        if (r < rows) __hip_atomic_store(amax + r, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// granularity: 1 = the row, 2 = blocks of block_rows rows of each [S, D] matrix, 3 = everything.  D is 64 or 128.
// Bound by launches at the sizes of one prefill: for 32 heads of 4096 x 128, per tensor 16.0 -> 11.2 us and per block of
// 128 rows 10.2 -> 7.6 us against one launch per step of the reduction (call to call, the host's part included), 16.0 ->
// 7.2 and 7.9 -> 4.8 us of GPU time.
int launch_group_amax(const void* x, int64_t n_mat, int64_t S, int D, int is_query, int granularity, int64_t block_rows,
                      float* amax, hipStream_t stream)
{
    const int64_t rows = n_mat * S;
    const int64_t chunks = rows * (D / 8);
    const int64_t blocks = (chunks + QUANT_THREADS - 1) / QUANT_THREADS;
    if (blocks > 0x7fffffffLL) return DMA_ERR_UNSUPPORTED_;
    const float c = (float)(1.4426950408889634074 / sqrt((double)D));
    // every size check comes before the first launch: on error nothing has been enqueued
    const int64_t bpm = granularity == 2 ? (S - 1) / block_rows + 1 : 0;
    if (D != 128 && D != 64) return DMA_ERR_UNSUPPORTED_;
    if (granularity == 2 && n_mat * bpm > 0x7fffffffLL) return DMA_ERR_UNSUPPORTED_;
    if (granularity == 3) {
        // a share is at least a workgroup's worth of unrolled loads, so there are never more parts than rows
        const int64_t shares = (blocks + QUANT_UNROLL - 1) / QUANT_UNROLL;
        const int parts = (int)(shares < TENSOR_PARTS ? shares : TENSOR_PARTS);
        const int64_t spread = (rows + QUANT_UNROLL * QUANT_THREADS - 1) / (QUANT_UNROLL * QUANT_THREADS);
        const int rc = launch(tensor_parts_kernel, dim3((unsigned)parts), dim3(QUANT_THREADS), stream, (const v4i*)x, chunks, c, is_query, amax);
        if (rc != DMA_OK_) return rc;
        return launch(tensor_spread_kernel, dim3((unsigned)spread), dim3(QUANT_THREADS), stream, amax, rows, parts);
    }
    if (granularity == 2 && block_rows >= FUSED_MIN && block_rows <= FUSED_MAX) {
        const int64_t per_block = (block_rows < S ? block_rows : S) * (D / 8);       // chunks of the longest block
        auto fused = [&](auto kernel, int threads) {
            return launch(kernel, dim3((unsigned)(n_mat * bpm)), dim3(threads), stream, (const v4i*)x, S, D / 8, block_rows, bpm, c, is_query, amax);
        };
        if (per_block <= WAVE_CHUNKS || (per_block < 2 * WAVE_CHUNKS && n_mat * bpm > MANY_BLOCKS)) return fused(block_amax_fused_kernel<64>, 64);
        if (per_block >= WIDE_CHUNKS && n_mat * bpm <= CU_BLOCKS) return fused(block_amax_fused_kernel<1024>, 1024);
        return fused(block_amax_fused_kernel<QUANT_THREADS>, QUANT_THREADS);
    }
    int rc = D == 128 ? launch(row_amax_kernel<16>, dim3((unsigned)blocks), dim3(QUANT_THREADS), stream, (const v4i*)x, rows, c, is_query, amax)
                      : launch(row_amax_kernel<8>, dim3((unsigned)blocks), dim3(QUANT_THREADS), stream, (const v4i*)x, rows, c, is_query, amax);
    if (rc == DMA_OK_ && granularity == 2)
        rc = launch(block_amax_kernel, dim3((unsigned)(n_mat * bpm)), dim3(64), stream, amax, S, block_rows, bpm);
    return rc;
}

int launch_mx_quantize(const void* x, int64_t rows, int D, int mode, int is_query, void* c4, void* s4,
                       void* c8, void* s8, float* token_scales, hipStream_t stream)
{
    if (token_scales) {
        switch (mode) {
            case 1: return launch_mode<1, true>(x, rows, D, is_query, c4, s4, c8, s8, token_scales, stream);
            case 2: return launch_mode<2, true>(x, rows, D, is_query, c4, s4, c8, s8, token_scales, stream);
            case 4: return launch_mode<4, true>(x, rows, D, is_query, c4, s4, c8, s8, token_scales, stream);
        }
        return DMA_ERR_INVALID_ARG_;
    }
    switch (mode) {
        case 1: return launch_mode<1, false>(x, rows, D, is_query, c4, s4, c8, s8, nullptr, stream);
        case 2: return launch_mode<2, false>(x, rows, D, is_query, c4, s4, c8, s8, nullptr, stream);
        case 3: return launch_mode<3, false>(x, rows, D, is_query, c4, s4, c8, s8, nullptr, stream);
        case 4: return launch_mode<4, false>(x, rows, D, is_query, c4, s4, c8, s8, nullptr, stream);
    }
    return DMA_ERR_INVALID_ARG_;
}

}  // namespace dma
