// Layer transform and feature gradient of a mini-batch (C = op(A B), A M x K with hundreds of thousands of rows, B K x N or, given
// transposed, N x K, K and N up to 256) with A, C and the optional ReLU mask stored as bfloat16.
//
// The product reads A and the mask and writes C once, at 128 flop per byte of the three with K = N = 256: it is a copy with matrix
// instructions on the way.  So:
//  - B is rounded to bfloat16 once per workgroup and stays in LDS; workgroups are persistent and walk blocks of 256 rows, 32 a wavefront;
//  - A goes straight from memory into the operand registers of v_mfma_f32_32x32x16_bf16: a lane's operand is eight consecutive
//    values of a row, 16 bytes.  The whole 32 x K block of a wavefront is in registers, and a piece of 64 columns is requested for the next
//    block as soon as it has been multiplied: while a block is written, the next one is in flight as a whole;
//  - the operands are swapped (the instruction computes C^T), so that a lane holds 4 consecutive columns of one row in 4
//    registers; after an exchange between the halves of the wavefront it holds 8 and stores, or reads of the mask, 16 bytes.  With C
//    in the usual orientation a lane holds one column of 16 rows: 64 stores of 4 bytes a lane and block, and ballots to bring the mask's
//    bits to the lanes that need them;
//  - in a wavefront with rows of its own, rows behind the last one repeat it (the same bytes to the same place by the same
//    instruction), columns behind the last are dropped by the bounds of the buffer: no branch round a load or store, so that the waits count
//    exactly.  A wavefront without rows leaves: with C in the place of the mask or of A it would read a row that another has overwritten.
// Measured, us (gemm_skinny_bf16_kernel / here, K x N), 40000 rows: 256 x 256 23 / 20, with a mask 28 / 23; 172 x 256 21 / 17, 25 / 21; 256 x 172 19 / 18,
// 22 / 18; 128 x 128 12 / 12, 13 / 13.  131072 rows: 256 x 256 38 / 35, 52 / 43; 172 x 256 32 / 29, 46 / 40; 200 x 200 36 / 31, 51 / 43; 128 x 128 17 / 16, 24 / 21.
// Not for what does not stay in the Infinity Cache, see the launcher: its loads and stores cover 32 bytes of a row at a time, the other kernel's
// 64, and memory minds (stores with the non-temporal hint, which leave the L2 as they are: 2^20 x 256 x 256 270 -> 626 us).
#include <algorithm>
#include <type_traits>

#include "gemm_stream.h"

namespace {

typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));

constexpr int ROWS_WAVES = 8;

struct rows_args {
    int64_t M;
    int N, K;
    const u16 *A; int64_t lda;
    const int32_t *row_index;      // optional: row i of A is row row_index[i] of the matrix in memory
    const float *B; int64_t ldb;
    const float *bias;
    int relu;
    u16 *C; int64_t ldc;
    const u16 *mask; int64_t ldm;
};

template <int NT8, int S> constexpr size_t rows_lds_bytes() { return (size_t)32 * NT8 * (64 * S + 8) * 2 + (size_t)32 * NT8 * 4; }

// NT8 tiles of 32 columns of C, S pieces of 64 columns of A; TB: B is given N x K
template <int NT8, int S, bool TB, bool MASK>
__global__ __launch_bounds__(64 * ROWS_WAVES, 2) void gemm_rows_kernel(rows_args a, uint32_t row_blocks)
{
    constexpr int KP = 64 * S + 8, NP = 32 * NT8, THREADS = 64 * ROWS_WAVES;
    extern __shared__ __attribute__((aligned(16))) unsigned char rows_smem[];
    u16 *LB = reinterpret_cast<u16 *>(rows_smem);                       // [n][k]
    float *Lbias = reinterpret_cast<float *>(LB + NP * KP);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 31, kh = lane >> 5;
    const int K = a.K, N = a.N;

    // the first block of A is on its way while B goes into LDS
    u32x4_any q[S][4];
    const u16 *rowp;
    auto row_of = [&](uint32_t rb) {
        rb = min(rb, row_blocks - 1);       // past the end: the last block again, never used
        return min((int64_t)rb * (32 * ROWS_WAVES) + wave * 32 + li, a.M - 1);
    };
    auto row_pointer = [&](uint32_t rb) {
        int64_t row = row_of(rb);
        if (a.row_index) row = a.row_index[row];
        rowp = a.A + row * a.lda;
    };
    auto issue = [&](int s) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = 64 * s + 16 * t + 8 * kh;      // the last piece may end with the row: then the 16 bytes that do
            q[s][t] = *reinterpret_cast<const u32x4_any *>(rowp + (s == S - 1 ? min(k, K - 8) : k));
        }
    };
    row_pointer(blockIdx.x);
#pragma unroll
    for (int s = 0; s < S; ++s) issue(s);

    // B, zero beyond N and K: chunks of four values, eight of them in flight
    constexpr int CHUNKS = NP * 16 * S;
    for (int base = threadIdx.x; base < CHUNKS; base += 8 * THREADS) {
        f32x4 x[8];
        int n[8], k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = base + u * THREADS;
            if constexpr (TB) { n[u] = idx / (16 * S); k[u] = 4 * (idx % (16 * S)); }
            else { const int r = idx >> 6; n[u] = 32 * (r % NT8) + 4 * (idx & 7); k[u] = 8 * (r / NT8) + ((idx >> 3) & 7); }
            x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (idx < CHUNKS && n[u] < N && k[u] < K) {
                typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
                x[u] = *reinterpret_cast<const f32x4_any *>(TB ? a.B + (int64_t)n[u] * a.ldb + k[u] : a.B + (int64_t)k[u] * a.ldb + n[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (base + u * THREADS >= CHUNKS) continue;
            const uint32_t w0 = pack_bf16(x[u][0], x[u][1]), w1 = pack_bf16(x[u][2], x[u][3]);
            if constexpr (TB) *reinterpret_cast<uint2 *>(LB + n[u] * KP + k[u]) = make_uint2(w0, w1);
            else {
                LB[n[u] * KP + k[u]] = (u16)w0; LB[(n[u] + 1) * KP + k[u]] = (u16)(w0 >> 16);
                LB[(n[u] + 2) * KP + k[u]] = (u16)w1; LB[(n[u] + 3) * KP + k[u]] = (u16)(w1 >> 16);
            }
        }
    }
    for (int n = threadIdx.x; n < NP; n += THREADS) Lbias[n] = a.bias && n < N ? a.bias[n] : 0.f;
    __syncthreads();

    const bool ragged = K % 64 != 0, half_chunk = N % 8 != 0;
    constexpr uint32_t BEYOND = 0x80000000u;      // an offset outside the buffer of a wavefront's rows: the store is dropped
    for (uint32_t rb = blockIdx.x; rb < row_blocks; rb += gridDim.x) {
        const int64_t wrow = (int64_t)rb * (32 * ROWS_WAVES) + wave * 32;       // the wavefront's first row
        if (wrow >= a.M) break;
        f32x16 acc[NT8];
        const int64_t row = row_of(rb);
        const u16 *mp = MASK ? a.mask + row * a.ldm : nullptr;
        u32x4_any m[2], m_next[2];
        auto mask_issue = [&](int j, u32x4_any (&d)[2]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int n = 32 * j + 16 * h + 8 * kh;
                d[h] = *reinterpret_cast<const u32x4_any *>(mp + (j >= NT8 - 2 ? min(n, N - 8) : n));
            }
        };
        if constexpr (MASK) mask_issue(0, m_next);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            asm volatile("" ::: "memory");       // B is read again for every block and piece: kept in registers it would spill
            if (s == S - 1 && ragged) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int left = K - (64 * s + 16 * t + 8 * kh);      // values of the chunk inside the row: a multiple of 4
                    u32x4_any v = q[s][t];
                    if (left == 4) { v[0] = v[2]; v[1] = v[3]; v[2] = v[3] = 0u; }
                    if (left <= 0) v[0] = v[1] = v[2] = v[3] = 0u;
                    q[s][t] = v;
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 av = __builtin_bit_cast(bf16x8, q[s][t]);
#pragma unroll
                for (int j = 0; j < NT8; ++j) {
                    const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(LB + (32 * j + li) * KP + 64 * s + 16 * t + 8 * kh);
                    if (s == 0 && t == 0) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv, av, f32x16{}, 0, 0, 0);
                    else acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv, av, acc[j], 0, 0, 0);
                }
            }
            if (s == 0) row_pointer(rb + gridDim.x);
            issue(s);                                        // of the next block
        }
        // register 4 g + i of lane (li, kh) of tile j: row li, column 32 j + 8 g + 4 kh + i
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.C + wrow * a.ldc, 0, 0x7fffffff, 0x00020000);
        const uint32_t row_off = (uint32_t)(row - wrow) * (uint32_t)(a.ldc * 2);
#pragma unroll
        for (int j = 0; j < NT8; ++j) {
            asm volatile("" ::: "memory");
            if constexpr (MASK) {
                m[0] = m_next[0]; m[1] = m_next[1];
                if (j + 1 < NT8) mask_issue(j + 1, m_next);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t w[2][2];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const f32x4 b = *reinterpret_cast<const f32x4 *>(Lbias + 32 * j + 16 * h + 8 * g + 4 * kh);
                    float z[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        z[i] = acc[j][8 * h + 4 * g + i] + b[i];
                        z[i] = a.relu ? fmaxf(z[i], 0.f) : z[i];
                    }
                    w[g][0] = pack_bf16(z[0], z[1]); w[g][1] = pack_bf16(z[2], z[3]);
                }
                // columns 32 j + 16 h + 8 kh .. + 7 of the row: the lower half of the wavefront takes g = 0, the upper g = 1
                const auto r0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                const auto r1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                u32x4 o = {(uint32_t)r0[0], (uint32_t)r1[0], (uint32_t)r0[1], (uint32_t)r1[1]};
                const int n = 32 * j + 16 * h + 8 * kh;
                if constexpr (MASK) {
                    u32x4_any mm = m[h];
                    if (j >= NT8 - 2 && n == N - 4) { mm[0] = mm[2]; mm[1] = mm[3]; }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t lo = __builtin_bit_cast(float, mm[i] << 16) > 0.f ? 0xffffu : 0u;
                        const uint32_t hi = __builtin_bit_cast(float, mm[i] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u;
                        o[i] &= lo | hi;
                    }
                }
                const uint32_t off = row_off + (uint32_t)n * 2;
                __builtin_amdgcn_raw_buffer_store_b128(o, rsrc, j >= NT8 - 2 && n + 8 > N ? BEYOND : off, 0, 0);
                if (j >= NT8 - 2 && half_chunk)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{o[0], o[1]}, rsrc, n + 4 == N ? off : BEYOND, 0, 0);
            }
        }
    }
}

template <int NT8, int S, bool TB> int launch_rows(sgnn_ctx *ctx, const rows_args &a, hipStream_t st)
{
    constexpr size_t lds = rows_lds_bytes<NT8, S>();
    static_assert(lds <= 160 * 1024, "B fits LDS");
    const uint32_t blocks = (uint32_t)cdiv(a.M, 32 * ROWS_WAVES);
    const dim3 grid(std::min<uint32_t>(blocks, 256u)), block(64 * ROWS_WAVES);
    char tag[56];
    snprintf(tag, sizeof(tag), "N%c rows %lldx%dx%d bf16 a=2 c=2%s", TB ? 'T' : 'N', (long long)a.M, a.N, a.K, a.mask ? " mask m=2" : "");
    if (a.mask) {
        SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_rows_kernel<NT8, S, TB, true>>(ctx, lds)));
        SGNN_LAUNCH(ctx, st, "gemm_rows_kernel", tag, (gemm_rows_kernel<NT8, S, TB, true>), grid, block, lds, st, a, blocks);
    } else {
        SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_rows_kernel<NT8, S, TB, false>>(ctx, lds)));
        SGNN_LAUNCH(ctx, st, "gemm_rows_kernel", tag, (gemm_rows_kernel<NT8, S, TB, false>), grid, block, lds, st, a, blocks);
    }
    return SGNN_OK;
}

template <int NT8, bool TB> int launch_rows_s(sgnn_ctx *ctx, const rows_args &a, hipStream_t st)
{
    switch ((a.K + 63) / 64) {
    case 1: return launch_rows<NT8, 1, TB>(ctx, a, st);
    case 2: return launch_rows<NT8, 2, TB>(ctx, a, st);
    case 3: return launch_rows<NT8, 3, TB>(ctx, a, st);
    default: return launch_rows<NT8, 4, TB>(ctx, a, st);
    }
}

template <bool TB> int launch_rows_n(sgnn_ctx *ctx, const rows_args &a, hipStream_t st)
{
    switch ((a.N + 63) / 64) {
    case 2: return launch_rows_s<4, TB>(ctx, a, st);
    case 3: return launch_rows_s<6, TB>(ctx, a, st);
    default: return launch_rows_s<8, TB>(ctx, a, st);
    }
}

} // namespace

// Returns SGNN_ERR_UNSUPPORTED without launching anything for what the kernel does not handle
int sgnn_launch_gemm_rows(sgnn_ctx *ctx, int tb, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const int32_t *row_index, const float *B,
                          int64_t ldb, const float *bias, int relu, void *C, int64_t ldc, const void *mask, int64_t ldm, hipStream_t st)
{
    // Wide results whose operands are well below the 256 MB of the Infinity Cache, us there / here (rows x N x K):
    // 262144 x 172 x 128 (157 MB) 39 / 36, 262144 x 256 x 48 (159) 36 / 32; 262144 x 172 x 172 (180) 55 / 58, 262144 x 100 x 256 (187) 47 / 52,
    // 262144 x 256 x 256 (268) 71 / 71, masked (403) 113 / 116, 2^20 x 256 x 256 250 / 272; 262144 x 64 x 256 35 / 42, 131072 x 48 x 256 18 / 24.
    if (N <= 64 || 2 * M * (K + N * (mask ? 2 : 1)) > (int64_t)160 << 20) return SGNN_ERR_UNSUPPORTED;
    // Nor narrow results where rows of A are a multiple of 128 bytes apart.  A load covers 32 bytes of 32 rows; then these lie at the same place of
    // their lines, and the loads take half as long again (4096 x 72 x 256: 13.4 us, 9.6 with rows 528 bytes apart; the other kernel reads
    // whole lines, 11.7 and 11.5).  Up to 128 columns there is too little else to do.  us there / here, rows of K values, plain and masked:
    //   4096 x 72 x 256   11.7 / 13.4  13.6 / 14.2     4096 x 128 x 256   12.1 / 14.0  14.5 / 15.3     16384 x 128 x 192  11.5 / 12.4  14.6 / 14.0
    //   16384 x 100 x 256 13.4 / 14.6  16.1 / 15.7     65536 x 128 x 256  18.9 / 19.8  24.7 / 26.9     65536 x 72 x 192   13.5 / 13.6  16.4 / 15.6
    //   4096 x 160 x 256  15.9 / 15.5  18.9 / 17.7     110000 x 100 x 192 25.4 / 23.7  35.4 / 31.5     4096 x 72 x 128     8.2 / 8.0   10.2 / 9.0
    //   110000 x 128 x 256 29.1 / 30.2 40.9 / 38.2     132000 x 96 x 256  33.2 / 36.9  44.6 / 44.0     110000 x 192 x 256 35.9 / 37.2  55.4 / 51.6
    //   132000 x 192 x 256 47.4 / 52.5 64.8 / 65.1     132000 x 160 x 256 44.2 / 47.4  61.7 / 63.2     132000 x 192 x 192 42.8 / 44.1  58.8 / 60.8
    //   132000 x 256 x 256 57.5 / 57.6 81.3 / 82.1     (rows of 248 values: 72 to 256 columns 3 to 20 % faster here, 65536 masked rows of 160 and more even)
    if (lda % 64 == 0) {
        const int narrow = K > 192 ? (!mask && M > 110000 ? 192 : (!mask || M <= 65536 ? 128 : 0)) : (K > 128 && !mask && M <= 65536 ? 128 : 0);
        if (N <= narrow) return SGNN_ERR_UNSUPPORTED;
    }
    // four values at a time on every side; offsets of a wavefront's 32 rows of C in 31 bits
    if (M < 4096 || N > 256 || N % 4 || K < 8 || K > 256 || K % 4 || ldc >= (1 << 20) || (reinterpret_cast<uintptr_t>(C) & 3) || ldc % 2)
        return SGNN_ERR_UNSUPPORTED;
    rows_args a = {};
    a.M = M; a.N = (int)N; a.K = (int)K;
    a.A = static_cast<const u16 *>(A); a.lda = lda; a.row_index = row_index;
    a.B = B; a.ldb = ldb; a.bias = bias; a.relu = relu;
    a.C = static_cast<u16 *>(C); a.ldc = ldc;
    a.mask = static_cast<const u16 *>(mask); a.ldm = ldm;
    return tb ? launch_rows_n<true>(ctx, a, st) : launch_rows_n<false>(ctx, a, st);
}
