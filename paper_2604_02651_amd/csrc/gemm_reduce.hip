// Sum of the partial products of a split reduction, and of the column sums that ride along, in a fixed order (bit-reproducible).
//
// A stream of up to 64 MB (256 partial products of 256 x 256) that its writers have just left in the caches, so what counts is how much
// of it is on its way at a time: a workgroup has 256 elements, each of its eight wavefronts adds up every eighth partial product, 16 bytes a
// lane and eight of them in flight; the eight sums are added through LDS.  One element a thread, four bytes a load and eight in flight: 256 partial products of
// 256 x 256 15.0 us, 13.4 here (5 TB/s), of 256 x 172 14.4 and 9.2, of 256 x 47 14 and 7; 128 of 200 x 200 8.0 and 6.
#include "common.h"

namespace {

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));      // gfx950 global loads take any alignment

constexpr int RED_WAVES = 8, RED_U = 8;

// sum over z of src[z * n + i .. i + 3] for the block's 256 elements from i0 on, one element a thread of the first 256
__device__ __forceinline__ float sum_partials(const float *__restrict__ src, int splits, int64_t n, int64_t i0, float (&lds)[RED_WAVES][256])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the last lanes of the last block read the four elements that end with the array (fewer than four elements: one each)
    const bool tiny = n < 4;
    const int64_t i = tiny ? min((int64_t)lane, n - 1) : min(i0 + 4 * lane, n - 4);
    float s[2][4] = {};
    for (int z0 = wave; z0 < splits; z0 += RED_WAVES * RED_U) {
        f32x4_any x[RED_U];
#pragma unroll
        for (int u = 0; u < RED_U; ++u) {
            const float *p = src + (int64_t)min(z0 + RED_WAVES * u, splits - 1) * n + i;
            if (tiny) x[u] = f32x4_any{*p, 0.f, 0.f, 0.f};
            else x[u] = *reinterpret_cast<const f32x4_any *>(p);
        }
#pragma unroll
        for (int u = 0; u < RED_U; ++u)
            if (z0 + RED_WAVES * u < splits) {
#pragma unroll
                for (int e = 0; e < 4; ++e) s[u % 2][e] += x[u][e];
            }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t at = i + e - i0;
        if (tiny ? e == 0 && lane < n : at >= 4 * lane && at < 256) lds[wave][at] = s[0][e] + s[1][e];
    }
    __syncthreads();
    float t = 0.f;
    if (threadIdx.x < 256) {
        float v[RED_WAVES];
#pragma unroll
        for (int w = 0; w < RED_WAVES; ++w) v[w] = lds[w][threadIdx.x];
        t = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
    return t;
}

__global__ __launch_bounds__(64 * RED_WAVES) void splitk_reduce_kernel(const float *__restrict__ partial, int splits, int64_t MN, int64_t N,
                                                                       float *__restrict__ C, int64_t ldc, const float *__restrict__ cs_partial,
                                                                       float *__restrict__ cs_out, unsigned blocks)
{
    __shared__ float lds[RED_WAVES][256];
    if (blockIdx.x >= blocks) {          // the blocks behind the matrix have the column sums
        const int64_t i0 = (int64_t)(blockIdx.x - blocks) * 256;
        const float t = sum_partials(cs_partial, splits, N, i0, lds);
        if (threadIdx.x < 256 && i0 + threadIdx.x < N) cs_out[i0 + threadIdx.x] = t;
        return;
    }
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + threadIdx.x;
    const float t = sum_partials(partial, splits, MN, i0, lds);
    if (threadIdx.x < 256 && i < MN) C[(i / N) * ldc + (i % N)] = t;
}

// The same for few partial products, an element a thread and eight loads in flight: no sums to meet in LDS.
__global__ __launch_bounds__(256) void splitk_reduce_few_kernel(const float *__restrict__ partial, int splits, int64_t MN, int64_t N,
                                                                float *__restrict__ C, int64_t ldc, const float *__restrict__ cs_partial,
                                                                float *__restrict__ cs_out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= MN + (cs_partial ? N : 0)) return;
    const bool cs = i >= MN;          // the threads behind the matrix have the column sums
    const float *p = cs ? cs_partial + (i - MN) : partial + i;
    const int64_t n = cs ? N : MN;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < splits; z += RED_U) {
        float x[RED_U];
#pragma unroll
        for (int u = 0; u < RED_U; ++u) x[u] = p[(int64_t)min(z + u, splits - 1) * n];
#pragma unroll
        for (int u = 0; u < RED_U; ++u) s[u % 4] += z + u < splits ? x[u] : 0.f;
    }
    const float t = (s[0] + s[1]) + (s[2] + s[3]);
    if (cs) cs_out[i - MN] = t;
    else C[(i / N) * ldc + (i % N)] = t;
}

} // namespace

// C = sum of `splits` partial products [splits][M][N]; cs_out = the same for [splits][N] column sums (cs_partial may be null).
int sgnn_launch_splitk_reduce(sgnn_ctx *ctx, const float *partial, int splits, int64_t M, int64_t N, float *C, int64_t ldc,
                              const float *cs_partial, float *cs_out, hipStream_t st)
{
    // us of the whole A^T B with bfloat16 operands, eight wavefronts / an element a thread: 16 partial products of 608 x 256 23.3 / 22.4, of 256 x 256
    // 20.1 / 19.4, of 200 x 200 19.0 / 18.7, 24 of 300 x 300 22.5 / 22.0, of 256 x 172 19.6 / 19.9; fp32, 32 of 256 x 256 20.0 / 19.8, of 200 x 200
    // 18.8 / 19.3, 38 of 256 x 172 20.2 / 21.1, 64 of 256 x 256 27.3 / 28.1.
    if (splits <= 16 || (splits <= 32 && M * N >= 65536)) {
        SGNN_LAUNCH(ctx, st, "splitk_reduce_kernel", "few", splitk_reduce_few_kernel, dim3(cdiv(M * N + (cs_partial ? N : 0), 256)), dim3(256), 0, st,
                    partial, splits, M * N, N, C, ldc, cs_partial, cs_out);
        return SGNN_OK;
    }
    const unsigned blocks = cdiv(M * N, 256), cs_blocks = cs_partial ? cdiv(N, 256) : 0;
    SGNN_LAUNCH(ctx, st, "splitk_reduce_kernel", SGNN_TAG, splitk_reduce_kernel, dim3(blocks + cs_blocks), dim3(64 * RED_WAVES), 0, st, partial,
                splits, M * N, N, C, ldc, cs_partial, cs_out, blocks);
    return SGNN_OK;
}
