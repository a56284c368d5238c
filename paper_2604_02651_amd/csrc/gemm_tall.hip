// The tall-operand product C = act(A B + bias) of a layer's transform with A [M x K] and C [M x N] stored as bfloat16, hundreds of thousands of
// rows; B [K x N] fp32, rounded to bfloat16, K and N up to 256.  (With a mask, a row gather, fp32 storage or B given N x K:
// gemm_skinny_bf16_kernel in gemm.hip.)
//
// 128 flop per byte of A and C: a copy with matrix instructions on the way.
//  - Slices of 32 rows of A go into LDS by direct loads, whole rows at a time, up to seven slices ahead, one barrier a slice;
//  - a wavefront has 32 columns of C and keeps its part of B in registers for the whole kernel, so that the loop has nothing but LDS reads
//    of A, matrix instructions and stores, and all of LDS is there for A.  B is requested first: behind the slices its loads would wait for them;
//  - C^T is computed, as in gemm_rows.hip and gemm_bwd.hip: the lane holds 4 columns of a row in 4 registers, two exchanges make that 16
//    bytes a lane and 64 bytes of 16 rows a store;
//  - stores outside the matrix are dropped by the bounds of the buffer, so that a wavefront has the same number of loads and stores a slice and the
//    waits count exactly.  Of a row's last chunk of eight columns the wavefront that has it stores four, two and one; where the columns
//    are four more than a multiple of eight the four alone (with all three, dropped or not, a product with few steps waited for that wavefront:
//    262144 x 172 x 57 41 us, 33 without; 131072 x 172 x 256 34 and 32).
// Measured, us (the kernel in gemm.hip / here, TB/s of A and C here), K x N:
//              256 x 256           256 x 172          256 x 128          128 x 256          256 x 47
//   2^20       246 / 218 (4.9)     254 / 221 (4.1)    174 / 153 (5.2)    193 / 160 (5.0)    180 / 174 (3.6)
//   2^18       74 / 59 (4.5)       71 / 63 (3.5)      53 / 44 (4.6)      58 / 46 (4.3)      47 / 41 (3.8)
// a copy reaches 5.1.  Rows of 172 and 47 columns end in the middle of a 64-byte piece.
#include <algorithm>
#include <type_traits>

#include "gemm_stream.h"

namespace {

struct tall_args {
    const u16 *A; int64_t lda;      // [M x K], lda a multiple of 8
    const float *B; int64_t ldb;
    const float *bias;
    int relu;
    int64_t M;
    int N, K;
    u16 *C; int64_t ldc;
};

// chunks of 16 bytes of a row are swizzled so that 16 rows of one chunk lie in 16 different places of the banks' 256 bytes
template <int F> __device__ __forceinline__ int tall_swizzle(int row) { return F % 128 == 0 ? row & 15 : (row >> 1) & 7; }

template <int FK, int NT> struct tall_shape {
    // one workgroup of five to eight wavefronts a compute unit, or as many smaller ones as LDS holds
    static constexpr int STAGE = 32 * FK * 2, STAGES = NT > 4 ? 8 : 3, LDS = STAGES * STAGE + NT * 128, GROUPS = NT > 4 ? 1 : 160 * 1024 / LDS;
};

// FK: frame of K; NT: tiles of 32 columns of C, one a wavefront
template <int FK, int NT>
__global__ __launch_bounds__(64 * NT, 2) void gemm_tall_kernel(tall_args a)
{
    constexpr int STAGE = tall_shape<FK, NT>::STAGE, STAGES = tall_shape<FK, NT>::STAGES;
    constexpr int CH = FK / 8, WL = STAGE / 1024, LOADS = (WL + NT - 1) / NT, STEPS = FK / 16, STORES = 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char tall_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, kh = lane >> 5;
    const int64_t total = (a.M + 31) / 32;
    const int nslices = (int)((total - blockIdx.x + gridDim.x - 1) / gridDim.x);

    uint32_t at[LOADS];          // of load j, KB wave + NT j of the stage (the last one again where there is none): row << 16 | byte in the row
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int p = min(wave + NT * j, WL - 1) * 64 + lane, row = p / CH;
        at[j] = (uint32_t)row << 16 | 16u * (uint32_t)min((p % CH) ^ tall_swizzle<FK>(row), (a.K - 1) / 8);
    }
    auto first_row = [&](int s) { return ((int64_t)s * gridDim.x + blockIdx.x) * 32; };
    auto issue = [&](int s) {
        const int64_t r0 = first_row(min(s, nslices - 1));          // past the end: the last slice again, into a stage nobody reads
        const int last = (int)min(a.M - r0, (int64_t)32) - 1;
        unsigned char *stage = tall_smem + (s % STAGES) * STAGE;
        const unsigned char *a0 = reinterpret_cast<const unsigned char *>(a.A + r0 * a.lda);
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const uint32_t off = (uint32_t)min((int)(at[j] >> 16), last) * (uint32_t)(a.lda * 2) + (at[j] & 0xffffu);
            __builtin_amdgcn_global_load_lds(STREAM_GPTR(a0 + off), STREAM_LPTR(stage + 1024 * min(wave + NT * j, WL - 1)), 16, 0, 0);
        }
    };
    constexpr uint32_t BEYOND = 0x80000000u;      // outside the buffer: the store is dropped
    // the wavefront's 32 columns of B, zero beyond N and K: lane (li, kh) has reduction steps 16 st + 8 kh .. + 7 of column 32 wave + li
    const int n = 32 * wave + li, nc = min(n, a.N - 1);
    const uint32_t ldb = (uint32_t)a.ldb, off = 4u * (8u * (uint32_t)kh * ldb + (uint32_t)nc);
    auto b_load = [&](int st, float (&x)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = 16 * st + i;
            if (st < STEPS - 4 || a.K == FK) x[i] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.B + (int64_t)k * a.ldb) + off);
            else x[i] = a.B[(uint32_t)min(k + 8 * kh, a.K - 1) * ldb + (uint32_t)nc];          // (a frame is at most 63 wider than K)
        }
    };
    bf16x8 w[STEPS];
    float x[STEPS][8];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) b_load(st, x[st]);
    const float bias_n = (a.bias ? a.bias : a.B)[nc];
    asm volatile("" ::: "memory");          // B first: its loads would wait behind those of the slices
    // the wavefront with the chunk that is not whole: one more store a row where half of it exists, else three
    const int more = a.N % 8 == 0 || wave != (a.N - 1) / 32 ? 0 : (a.N % 8 == 4 ? 1 : 3);
    auto nothing = [&](auto count) {
#pragma unroll
        for (int t = 0; t < decltype(count)::value; ++t)
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{}, __builtin_amdgcn_make_buffer_rsrc(a.C, 0, 0x7fffffff, 0x00020000), BEYOND, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) {
        issue(s);
        asm volatile("" ::: "memory");
        // the loop's pattern, so that its first waits count the same (both counts known at compile time: else the compiler waits for everything)
        if (more == 3) nothing(std::integral_constant<int, 4 * STORES>{});
        else if (more) nothing(std::integral_constant<int, 2 * STORES>{});
        else nothing(std::integral_constant<int, STORES>{});
        asm volatile("" ::: "memory");
    }

#pragma unroll
    for (int st = 0; st < STEPS; ++st)
#pragma unroll
        for (int i = 0; i < 8; ++i) w[st][i] = (__bf16)(n < a.N && 16 * st + 8 * kh + i < a.K ? x[st][i] : 0.f);
    float *const bias = reinterpret_cast<float *>(tall_smem + STAGES * STAGE) + 32 * wave;          // the wavefront's, in LDS: read at every slice's end
    if (lane < 32) bias[lane] = a.bias ? bias_n : 0.f;
    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the bias is in LDS
    const uint32_t row_a = li * FK * 2;
    uint32_t lane_a = 16 * (kh ^ tall_swizzle<FK>(li));
    // where it writes C: row 16 t + (lane & 15) of the slice, columns 32 wave + 16 half + 8 kh .. + 7
    const int c_row = lane & 15, c_chunk = 4 * wave + 2 * ((lane >> 4) & 1) + kh;
    const int c_left = a.N - 8 * c_chunk;          // columns of the chunk that exist

    for (int s = 0; s < nslices; ++s) {
        asm volatile("" : "+v"(lane_a));                           // the chunks' addresses are put together in the loop: else a register each
        // slice s has landed (this wavefront's part)
        if (more == 3) STREAM_WAIT_VMCNT((STAGES - 2) * (LOADS + 4 * STORES) < 63 ? (STAGES - 2) * (LOADS + 4 * STORES) : 63);
        else if (more) STREAM_WAIT_VMCNT((STAGES - 2) * (LOADS + 2 * STORES));
        else STREAM_WAIT_VMCNT((STAGES - 2) * (LOADS + STORES));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();                              // everybody's part has; and everybody is through slice s - 1
        asm volatile("" ::: "memory");
        issue(s + STAGES - 1);                                     // into the stage slice s - 1 was read from
        asm volatile("" ::: "memory");
        const unsigned char *stage = tall_smem + (s % STAGES) * STAGE;
        const int64_t r0 = first_row(s);
        const int rows = (int)min(a.M - r0, (int64_t)32);
        f32x16 g;
#pragma unroll
        for (int r = 0; r < 16; ++r) g[r] = 0.f;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            u32x4 d = *reinterpret_cast<const u32x4 *>(stage + ((lane_a ^ (32u * st)) + row_a));
            if (st >= STEPS - 4 && 16 * st + 16 > a.K) {     // values behind the row's last hold anything
                const int left = a.K - (16 * st + 8 * kh);
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] &= left >= 2 * i + 2 ? 0xffffffffu : (left == 2 * i + 1 ? 0xffffu : 0u);
            }
            g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[st], __builtin_bit_cast(bf16x8, d), g, 0, 0, 0);
        }
        u32x4 o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t p[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                // register 4 q' + i of the result: column 32 wave + 8 q' + 4 kh + i
                const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + 16 * h + 8 * q + 4 * kh);
                float z[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    z[i] = g[8 * h + 4 * q + i] + b[i];
                    z[i] = a.relu ? fmaxf(z[i], 0.f) : z[i];
                }
                p[q][0] = pack_bf16(z[0], z[1]);
                p[q][1] = pack_bf16(z[2], z[3]);
            }
            // columns 16 h + 8 kh .. + 7 of the row: the lower half of the wavefront takes q = 0, the upper q = 1
            const auto r0_ = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
            const auto r1_ = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
            o[h] = u32x4{(uint32_t)r0_[0], (uint32_t)r1_[0], (uint32_t)r0_[1], (uint32_t)r1_[1]};
        }
        // rows 0 to 15 of both in the first, 16 to 31 in the second: h becomes bit 4 of the lane
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const auto r = __builtin_amdgcn_permlane16_swap(o[0][i], o[1][i], false, false);
            o[0][i] = (uint32_t)r[0];
            o[1][i] = (uint32_t)r[1];
        }
#pragma unroll
        for (int t = 0; t < STORES; ++t) {
            const int row = c_row + 16 * t;
            const uint32_t off = row < rows ? (uint32_t)row * (uint32_t)(a.ldc * 2) + 16u * (uint32_t)c_chunk : BEYOND;
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.C + r0 * a.ldc, 0, 0x7fffffff, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b128(o[t], rsrc, c_left >= 8 ? off : BEYOND, 0, 0);
            const bool part = c_left > 0 && c_left < 8;
            if (more) __builtin_amdgcn_raw_buffer_store_b64(u32x2{o[t][0], o[t][1]}, rsrc, part && (c_left & 4) ? off : BEYOND, 0, 0);
            if (more == 3) {
                __builtin_amdgcn_raw_buffer_store_b32((c_left & 4) ? o[t][2] : o[t][0], rsrc, part && (c_left & 2) ? off + 2 * (c_left & 4) : BEYOND, 0, 0);
                const uint32_t w = c_left == 7 ? o[t][3] : (c_left == 5 ? o[t][2] : (c_left == 3 ? o[t][1] : o[t][0]));
                __builtin_amdgcn_raw_buffer_store_b16((u16)w, rsrc, part && (c_left & 1) ? off + 2 * (c_left & 6) : BEYOND, 0, 0);
            }
        }
    }
    STREAM_WAIT_VMCNT(0);       // the repeated loads past the end are still in flight: nothing may leave before they land
}

template <int FK, int NT> int launch_tall(sgnn_ctx *ctx, const tall_args &a, hipStream_t st)
{
    constexpr int lds = tall_shape<FK, NT>::LDS;
    SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_tall_kernel<FK, NT>>(ctx, lds)));
    const int64_t slices = cdiv(a.M, 32);
    // a workgroup reads all of B: four slices each (two where a workgroup has two wavefronts only) before there is more than one a compute unit
    const unsigned grid = (unsigned)std::min<int64_t>(slices, std::min<int64_t>(std::max<int64_t>(slices / (NT > 2 ? 4 : 2), 256), 256 * tall_shape<FK, NT>::GROUPS));
    char tag[56];
    snprintf(tag, sizeof(tag), "NN tall %lldx%dx%d bf16 a=2 c=2", (long long)a.M, a.N, a.K);
    // recorded with the other kernel of such products; the tag tells them apart
    SGNN_LAUNCH(ctx, st, "gemm_skinny_bf16_kernel", tag, (gemm_tall_kernel<FK, NT>), dim3(grid), dim3(64 * NT), lds, st, a);
    return SGNN_OK;
}

template <int FK> int launch_tall_n(sgnn_ctx *ctx, const tall_args &a, hipStream_t st)
{
    switch ((a.N + 31) / 32) {
    case 1: case 2: return launch_tall<FK, 2>(ctx, a, st);
    case 3: case 4: return launch_tall<FK, 4>(ctx, a, st);
    case 5: case 6: return launch_tall<FK, 6>(ctx, a, st);
    default: return launch_tall<FK, 8>(ctx, a, st);
    }
}

} // namespace

// Returns SGNN_ERR_UNSUPPORTED without launching anything for what the kernel does not handle
int sgnn_launch_gemm_tall(sgnn_ctx *ctx, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const float *B, int64_t ldb,
                         const float *bias, int relu, void *C, int64_t ldc, hipStream_t st)
{
    constexpr int64_t LD_MAX = 1 << 20;          // offsets within a slice in 32 bits
    // Where the kernel of gemm.hip keeps the call.  us there / here, rows x N x K; hot: A from the Infinity Cache, as behind the product that wrote it,
    // cold: from memory.
    // Up to 64 columns are two wavefronts a workgroup, three of those a compute unit, and each workgroup reads all of B: few rows, or little of A a row,
    // and B and the first slices are half of the time.  131072 x 47 x 256 18.6 / 20.0 hot, 26.0 / 23.8 cold, x 64 x 256 17.3 / 19.9, 23.5 / 22.4;
    // x 47 x 100 12.1 / 13.7, 17.9 / 17.3, 262144 x 47 x 100 20.1 / 19.5, 28.1 / 26.9; up to 32 columns 131072 x 20 x 256 15.6 / 19.2, 20.9 / 21.5,
    // 262144 26.9 / 30.4, 35.1 / 35.7, 300000 x 32 x 256 30.5 / 34.1 hot, 131072 x 20 x 150 12.7 / 15.8,
    // 18 / 18; 400000 x 20 x 172 4 % and 12 % less here, 100001 x 3 x 129 3 % more and 7 % less.
    if (N <= 64 && (K <= 64 || M < (K <= 128 ? 250000 : 100000) || (N <= 32 && (N > 4 || K >= 160) && M < 350000))) return SGNN_ERR_UNSUPPORTED;
    // Up to 90 columns and 65 to 128 steps: three tiles of which the last is nearly empty.  180000 x 70 x 96 20.8 / 24.1, 33.4 / 32.5, 262144 x 70 x 128 27.0 / 28.4, 50.4 / 48.4;
    // 32768 x 70 x 96 even, 600000 x 70 x 128 64.8 / 55.6, 102 / 100.
    if (N > 64 && N <= 90 && K > 64 && K <= 128 && M >= 40000 && M < 500000) return SGNN_ERR_UNSUPPORTED;
    // 91 to 128 columns, three to five slices a workgroup: 49152 x 128 x 256 14.0 / 14.9, 16.7 / 16.6, 65536 15.0 / 16.2, 19.0 / 18.1,
    // x 96 x 256 14.0 / 15.8, 18.3 / 17.3, 65536 x 100 x 256 16.0 / 17.3, 27.9 / 24.4; 32768 x 128 x 256 13.5 / 12.3, 15.2 / 13.8, 90000 20.9 / 19.1, 27.7 / 20.6.
    if (N > 90 && N <= 128 && K > 128 && M >= 40000 && M < 75000) return SGNN_ERR_UNSUPPORTED;
    // Up to 64 steps a slice is 4 KB and has hardly anything to multiply between two barriers: 131072 x 172 x 57 17.7 / 20.4, 23.5 / 24.7, x 192 x 57
    // 17.6 / 20.3, 18.5 / 21.1, 262144 x 96 x 57 18.5 / 21.1, 24.4 / 24.2, 400000 x 65 x 57 26.8 / 30.0, 41.5 / 40.7, 50000 x 160 x 57 11.4 / 13.1, 15.0 / 16.4,
    // 131072 x 224 x 57 20.8 / 22.3, 25.8 / 28.5.  Small ones, one tile for each wavefront (97 to 128 columns) of more rows, and more than 192 columns of many are even or better:
    // 16384 x 70 x 57 11.4 / 11.0, 11.4 / 10.0, 131072 x 100 x 57 13.6 / 13.3, 19.1 / 17.3 (65536 11.0 / 11.4, 15.1 / 15.2), 400000 x 224 x 57 even, 256 x 57 12 % and 7 % less here;
    // and 129 to 192 columns that are no multiple of four up to 60000 rows: 50000 x 130 x 57 9 % and 24 % less.
    if (K <= 64) {
        const int64_t from = N <= 96 ? 25000 : (N <= 128 || N > 192 || N % 4 == 0 ? 40000 : 60000);
        const int64_t to = N <= 96 || (N > 128 && N <= 192) ? INT64_MAX : (N <= 128 ? 80000 : (N <= 224 ? 300000 : 0));
        if (M >= from && M < to) return SGNN_ERR_UNSUPPORTED;
        // three more stores a row for the end of it: 262144 x 255 x 17 33.7 / 41.1, 400000 52 / 60, x 256 x 17 9 % less here
        if (N > 224 && N % 4 && K <= 32 && M >= 100000 && M < 500000) return SGNN_ERR_UNSUPPORTED;
    }
    if (M < 4096 || N < 1 || N > 256 || K < 1 || K > 256 || lda % 8 || ldc % 8 || lda < K || ldc < N || lda >= LD_MAX || ldc >= LD_MAX || ldb >= LD_MAX ||
        (reinterpret_cast<uintptr_t>(A) & 15) || (reinterpret_cast<uintptr_t>(C) & 15))
        return SGNN_ERR_UNSUPPORTED;
    tall_args a;
    a.A = static_cast<const u16 *>(A); a.lda = lda; a.B = B; a.ldb = ldb; a.bias = bias; a.relu = relu;
    a.M = M; a.N = (int)N; a.K = (int)K; a.C = static_cast<u16 *>(C); a.ldc = ldc;
    switch ((K + 63) / 64) {
    case 1: return launch_tall_n<64>(ctx, a, st);
    case 2: return launch_tall_n<128>(ctx, a, st);
    case 3: return launch_tall_n<192>(ctx, a, st);
    default: return launch_tall_n<256>(ctx, a, st);
    }
}
