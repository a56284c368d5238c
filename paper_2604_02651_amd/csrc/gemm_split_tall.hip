// The split fp32 product of gemm_split.hip for a tall A [M x K] and a small B (K x N, or given N x K), K from 65 to 256, N from 65 to 256: the
// transform of a mini-batch layer and its input gradient, without a mask.
//
// The tiles of gemm_split.hip are about one a compute unit there, so that reading A, splitting, multiplying and writing C come one after the other
// (32768 x 256 x 256: the matrix pipe is busy a third of 33 us), and every tile splits its part of B anew.  Here a workgroup (one a
// compute unit, eight wavefronts) walks slices of 32 or 64 rows with all of B at hand: while a slice is multiplied the next is on its way
// and the last one leaves.
//  - A wavefront has 32 columns of C; the first two parts of its B stay in registers for the whole kernel, the third, which one product in six
//    needs, in LDS in operand order.
//  - A comes in pieces of 64 reduction steps, requested a whole slice ahead, split by all threads (each value once, where the tiles split it once
//    per 128 columns) and staged one piece ahead in LDS as three planes of 128-byte rows, the 16-byte chunks swizzled by the row.
//  - C^T is computed: the lane holds 4 columns of a row in 4 registers and, after an exchange, stores 64 bytes of 16 rows at a time.
//  - Half of the wavefronts (one a SIMD) multiply first and split then, the other half the other way round, as in gemm_split.hip; the first half goes
//    first at the matrix pipe too, or both would be done with it at the same time and one would split while it is idle (200000 x 128 x 256 97 -> 91 us).
//  - The products, their order and the two chains of sums are those of gemm_split.hip, and so is what is done where the split does not hold: the
//    wavefront's 32 x 32 results of the slice once more with the fp32 instructions, where they are not all finite or the slice, or the wavefront's
//    part of B, holds a value below 2^-112.
// Measured, us (gemm_split.hip / here), rows x K x N, B given K x N / N x K:
//               256 x 256              200 x 200              128 x 256              256 x 128              128 x 128
//   200000      203 / 163  187 / 158   197 / 139  175 / 140   127 / 91  122 / 91     116 / 86  112 / 88     80 / 54  76 / 54
//   65536       62 / 55  59 / 55       62 / 51  55 / 53       41 / 35  39 / 35       34 / 35  32 / 37       22 / 22  22 / 22
//   32768       32 / 33  31 / 32       32 / 30  27 / 33       21 / 21  20 / 21       20 / 22  19 / 23       14 / 15  14 / 16
// B given N x K with K no multiple of 64: 20000 x 256 x 96 19.5 / 17.7, 40000 x 128 x 96 19.6 / 18.2, x 128 x 200 29.4 / 25.7 (22.1, 23.2 and 31.8 with the
// last steps of B's rows loaded value by value).
// A slice of 32 rows takes 6.2 us where the matrix pipe is busy 3: the reads of A and of the third part of B from LDS, the splitting, a barrier for
// every piece.  Results of a slice written one piece later by half of the wavefronts: slower (200000 x 128 x 256 91 -> 103 us).
#include <algorithm>

#include "gemm_stream.h"

namespace {

#include "split_parts.h"

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TALL_NT = 512;
constexpr int PIECE = 64;          // reduction steps staged at a time

struct split_tall_args {
    int64_t M;
    int N, K;
    const float *A; int64_t lda;
    const float *B; int64_t ldb;
    const float *bias;
    int relu;
    float *C; int64_t ldc;
};

template <int FK, int CT> struct split_tall_shape {
    static constexpr int BR = 32 * (8 / CT), PLANE = BR * PIECE * 2, BUF = 3 * PLANE;
    static constexpr int STEPS = FK / 16, W2 = FK == 256 && CT == 4 ? 8 : STEPS;          // steps of the second part in registers: as many as fit there
    static constexpr int PARTS = CT * (STEPS + STEPS - W2) * 1024, LDS = 2 * BUF + PARTS + CT * 128 + 16;
    static_assert(LDS <= 160 * 1024, "fits");
};

// FK: frame of K; CT: tiles of 32 columns, 8 / CT tiles of 32 rows a slice; TB: B is given N x K
template <int FK, int CT, bool TB>
__global__ __launch_bounds__(TALL_NT, 2) void gemm_split_tall_kernel(split_tall_args a)
{
    using SH = split_tall_shape<FK, CT>;
    constexpr int BR = SH::BR, PLANE = SH::PLANE, BUF = SH::BUF, NP = FK / PIECE, STEPS = SH::STEPS, W2 = SH::W2, U = BR / 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char tall_lds[];
    unsigned char *const third = tall_lds + 2 * BUF;
    float *const bias = reinterpret_cast<float *>(third + SH::PARTS);
    int *const small = reinterpret_cast<int *>(bias + 32 * CT);          // of the even and of the odd slices: a value below 2^-112
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 31, kh = lane >> 5;
    const int ct = wave % CT, rt = wave / CT;
    const int N = a.N, K = a.K;
    const int64_t total = (a.M + BR - 1) / BR;
    const int nslices = (int)((total - blockIdx.x + gridDim.x - 1) / gridDim.x);
    auto first_row = [&](int s) { return ((int64_t)s * gridDim.x + blockIdx.x) * BR; };

    // A: a thread has four reduction steps of row threadIdx.x / 16 (and of the row 32 further on) of every piece
    const int a_row = threadIdx.x >> 4, a_k = 4 * (threadIdx.x & 15);
    f32x4 reg[NP][U];
    const float *row[U];
    auto rows_of = [&](int s) {
        const int64_t r0 = first_row(min(s, nslices - 1));
#pragma unroll
        for (int u = 0; u < U; ++u) row[u] = a.A + min(r0 + a_row + 32 * u, a.M - 1) * a.lda;
    };
    auto fetch = [&](int kp) {
        const int k = kp == NP - 1 ? min(PIECE * kp + a_k, K - 4) : PIECE * kp + a_k;          // the four that end with the row, put right in split()
#pragma unroll
        for (int u = 0; u < U; ++u) reg[kp][u] = *reinterpret_cast<const f32x4_any *>(row[u] + k);
    };

    // the wavefront's 32 columns of B, zero beyond N and K: lane (li, kh) has reduction steps 16 st + 8 kh .. + 7 of column 32 ct + li
    const int n = 32 * ct + li, nc = min(n, N - 1);
    bf16x8 w1[STEPS], w2[W2];
    uint32_t tiny_b = 0xffffffffu;
    rows_of(0);
#pragma unroll
    for (int st0 = 0; st0 < STEPS; st0 += 4) {
        float x[4][8];
        const bool whole = st0 + 4 < STEPS || K == FK;          // (a frame is at most 63 wider than K)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k0 = 16 * (st0 + q) + 8 * kh;
            if (TB) {
                // past the row's end the four that end with it, put right
                const float *p = a.B + (int64_t)nc * a.ldb;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int k = k0 + 4 * h, kc = whole ? k : min(k, K - 4);
                    f32x4 v = *reinterpret_cast<const f32x4_any *>(p + kc);
                    if (!whole) v = shifted(v, min(k - kc, 4));
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[q][4 * h + i] = v[i];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[q][i] = a.B[(int64_t)(whole ? k0 + i : min(k0 + i, K - 1)) * a.ldb + nc];
            }
        }
        if (st0 == 0) {
#pragma unroll
            for (int kp = 0; kp < NP; ++kp) fetch(kp);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[2][4];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i / 4][i % 4] = n < N && 16 * (st0 + q) + 8 * kh + i < K ? x[q][i] : 0.f;
            const parts4 lo = split4(v[0], tiny_b), hi = split4(v[1], tiny_b);
            auto join = [](uint2 s, uint2 t) { return __builtin_bit_cast(bf16x8, make_uint4(s.x, s.y, t.x, t.y)); };
            w1[st0 + q] = join(lo.p[0], hi.p[0]);
            if (st0 < W2) w2[st0 < W2 ? st0 + q : 0] = join(lo.p[1], hi.p[1]);
            if (rt == 0) {
                *reinterpret_cast<bf16x8 *>(third + ((st0 + q) * CT + ct) * 1024 + lane * 16) = join(lo.p[2], hi.p[2]);
                if (st0 >= W2) *reinterpret_cast<bf16x8 *>(third + ((STEPS + st0 - W2 + q) * CT + ct) * 1024 + lane * 16) = join(lo.p[1], hi.p[1]);
            }
        }
        asm volatile("" ::: "memory");          // four steps at a time: all requested together they would spill
    }
    const bool redo_all = __ballot(tiny_b < TINY) != 0;
    if (rt == 0 && kh == 0) bias[n] = a.bias ? a.bias[nc] : 0.f;
    if (threadIdx.x < 2) small[threadIdx.x] = 0;
    __syncthreads();

    // where a thread puts its four values in a plane, and where a lane reads an operand: rows of 128 bytes, two of which pass over all banks
    const int put = a_row * 128 + (((a_k >> 3) ^ ((a_row >> 1) & 7)) * 16) + (a_k & 4) * 2;
    const int get = (32 * rt + li) * 128, get_x = (li >> 1) & 7;
    uint32_t tiny = 0xffffffffu;
    auto split = [&](int kp, unsigned char *buf, int s) {          // piece kp of slice s
        if (kp == 0) tiny = 0xffffffffu;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            f32x4 v = reg[kp][u];
            if (kp == NP - 1 && K < FK) v = shifted(v, min(max(PIECE * kp + a_k - (K - 4), 0), 4));
            const float f[4] = {v[0], v[1], v[2], v[3]};
            const parts4 p = split4(f, tiny);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2 *>(buf + q * PLANE + put + u * 32 * 128) = p.p[q];
        }
        if (tiny < TINY) small[s & 1] = 1;
    };
    f32x16 acc, low;
    auto clear = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = low[r] = 0.f;
    };
    // the products of a piece, the operands of a step read one step ahead
    auto multiply = [&](int kp, const unsigned char *buf) {
        bf16x8 fa[2][3], f2[2], f3[2];
        auto read = [&](int s4) {
            const unsigned char *p = buf + get + (((2 * s4 + kh) ^ get_x) * 16);
#pragma unroll
            for (int q = 0; q < 3; ++q) fa[s4 & 1][q] = *reinterpret_cast<const bf16x8 *>(p + q * PLANE);
            const int st = 4 * kp + s4;
            f3[s4 & 1] = *reinterpret_cast<const bf16x8 *>(third + (st * CT + ct) * 1024 + lane * 16);
            if (st < W2) f2[s4 & 1] = w2[st < W2 ? st : 0];
            else f2[s4 & 1] = *reinterpret_cast<const bf16x8 *>(third + ((STEPS + st - W2) * CT + ct) * 1024 + lane * 16);
        };
        read(0);
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const int st = 4 * kp + s4, b = s4 & 1;
            if (s4 < 3) read(s4 + 1);
            __builtin_amdgcn_sched_barrier(0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[st], fa[b][0], acc, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[st], fa[b][1], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[b], fa[b][0], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[b], fa[b][1], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[st], fa[b][2], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f3[b], fa[b][0], low, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // where a lane writes C, in two rows 16 apart: columns c_col + 16 p .. + 3
    const int c_row = 32 * rt + (lane & 15), c_col = 32 * ct + 8 * ((lane >> 4) & 1) + 4 * kh;
    constexpr uint32_t BEYOND = 0x80000000u;      // outside the buffer: the store is dropped
    const bool ragged = N % 4 != 0 && ct == (N - 1) / 32;
    auto finish = [&](int s) {
        float bad = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[r] += low[r];
            bad = fmaf(acc[r], 0.f, bad);          // NaN if any of them is not finite
        }
        const int64_t r0 = first_row(s);
        if (redo_all || small[s & 1] || __ballot(!(bad == 0.f))) {
            // once more with the fp32 instructions, operands straight from memory
            const float *ap = a.A + min(r0 + 32 * rt + li, a.M - 1) * a.lda;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            constexpr int KU = 4;                  // steps whose loads are in flight together
            for (int k = 0; k < K; k += 2 * KU) {
                float va[KU], vb[KU];
#pragma unroll
                for (int u = 0; u < KU; ++u) {
                    const int kc = min(k + 2 * u + kh, K - 1);
                    va[u] = ap[kc];
                    vb[u] = TB ? a.B[(int64_t)nc * a.ldb + kc] : a.B[(int64_t)kc * a.ldb + nc];
                }
#pragma unroll
                for (int u = 0; u < KU; ++u) {
                    const bool in = k + 2 * u + kh < K;
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? vb[u] : 0.f, in ? va[u] : 0.f, acc, 0, 0, 0);
                }
            }
        }
        // register 4 q + i of lane (li, kh): row li of the tile, column 8 q + 4 kh + i
        if (a.bias) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + 32 * ct + 8 * q + 4 * kh);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[4 * q + i] += b[i];
            }
        }
        if (a.relu) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = fmaxf(acc[r], 0.f);
        }
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.C + r0 * a.ldc, 0, 0x7fffffff, 0x00020000);
        const int rows = (int)min(a.M - r0, (int64_t)BR);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            u32x4 o[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float z = acc[8 * p + 4 * h + i];          // (bit_cast of a vector's element itself takes the first)
                    o[h][i] = __builtin_bit_cast(uint32_t, z);
                }
            // rows 0 to 15 of both in the first, 16 to 31 in the second: h becomes bit 4 of the lane
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const auto r = __builtin_amdgcn_permlane16_swap(o[0][i], o[1][i], false, false);
                o[0][i] = (uint32_t)r[0];
                o[1][i] = (uint32_t)r[1];
            }
            const int col = c_col + 16 * p, left = N - col;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t off = c_row + 16 * t < rows ? (uint32_t)(c_row + 16 * t) * (uint32_t)(a.ldc * 4) + 4u * (uint32_t)col : BEYOND;
                __builtin_amdgcn_raw_buffer_store_b128(o[t], rsrc, left >= 4 ? off : BEYOND, 0, 0);
                if (ragged) {
#pragma unroll
                    for (int e = 0; e < 3; ++e) __builtin_amdgcn_raw_buffer_store_b32(o[t][e], rsrc, left < 4 && e < left ? off + 4 * e : BEYOND, 0, 0);
                }
            }
        }
    };

    split(0, tall_lds, 0);
    rows_of(1);
    fetch(0);
    __syncthreads();
    const bool ahead = wave >= 4;
    int cur = 0;
    for (int s = 0; s < nslices; ++s) {
#pragma unroll
        for (int kp = 0; kp < NP; ++kp, cur ^= 1) {
            unsigned char *here = tall_lds + cur * BUF, *there = tall_lds + (cur ^ 1) * BUF;
            const int kn = (kp + 1) % NP;
            if (kp == 0 && threadIdx.x == 0) small[(s + 1) & 1] = 0;          // read behind slice s - 1, set by the pieces of slice s + 1
            if (kp == 0) clear();
            if (ahead) {
                __builtin_amdgcn_s_setprio(2);
                multiply(kp, here);
                __builtin_amdgcn_s_setprio(0);
            }
            if (kn || s + 1 < nslices) {
                split(kn, there, kn ? s : s + 1);
                if (kn == 0) rows_of(s + 2);
                fetch(kn);          // of the next slice (behind the last one: its rows again, never used)
            }
            if (!ahead) multiply(kp, here);
            if (kp == NP - 1) finish(s);
            __syncthreads();
        }
    }
}

template <int FK, int CT, bool TB> int launch_split_tall(sgnn_ctx *ctx, const split_tall_args &a, hipStream_t st)
{
    constexpr int LDS = split_tall_shape<FK, CT>::LDS;
    SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_split_tall_kernel<FK, CT, TB>>(ctx, LDS)));
    char tag[56];
    snprintf(tag, sizeof(tag), "N%c tall %lldx%dx%d f32 split", TB ? 'T' : 'N', (long long)a.M, a.N, a.K);
    const dim3 grid((unsigned)std::min<int64_t>(cdiv(a.M, split_tall_shape<FK, CT>::BR), 256)), block(TALL_NT);
    SGNN_LAUNCH(ctx, st, "gemm_split_tall_kernel", tag, (gemm_split_tall_kernel<FK, CT, TB>), grid, block, LDS, st, a);
    return SGNN_OK;
}

template <int FK> int launch_split_tall_ct(sgnn_ctx *ctx, const split_tall_args &a, int tb, hipStream_t st)
{
    if (a.N > 128) return tb ? launch_split_tall<FK, 8, true>(ctx, a, st) : launch_split_tall<FK, 8, false>(ctx, a, st);
    return tb ? launch_split_tall<FK, 4, true>(ctx, a, st) : launch_split_tall<FK, 4, false>(ctx, a, st);
}

} // namespace

// Returns SGNN_ERR_UNSUPPORTED without launching anything for what the kernel does not handle; the caller says where it pays
int sgnn_launch_gemm_split_tall(sgnn_ctx *ctx, int tb, int64_t M, int64_t N, int64_t K, const float *A, int64_t lda, const float *B, int64_t ldb,
                                const float *bias, int relu, float *C, int64_t ldc, hipStream_t st)
{
    if (N <= 64 || N > 256 || K <= 64 || K > 256 || ldc >= (1 << 22)) return SGNN_ERR_UNSUPPORTED;          // (offsets in a slice of C in 31 bits)
    split_tall_args a;
    a.M = M; a.N = (int)N; a.K = (int)K; a.A = A; a.lda = lda; a.B = B; a.ldb = ldb; a.bias = bias; a.relu = relu;
    a.C = C; a.ldc = ldc;
    switch ((K + 63) / 64) {
    case 2: return launch_split_tall_ct<128>(ctx, a, tb, st);
    case 3: return launch_split_tall_ct<192>(ctx, a, tb, st);
    default: return launch_split_tall_ct<256>(ctx, a, tb, st);
    }
}
