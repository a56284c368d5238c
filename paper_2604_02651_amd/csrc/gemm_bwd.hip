// Both products of a layer's backward pass (Sec. III-C) in one pass over their common operand, all matrices stored as bfloat16:
//   C [M x N] = X^T D     the weight gradient: X [K x M] the saved aggregate (or the layer input), D [K x N] = dZ (or dP)
//   G [K x M] = D W^T     the gradient handed down, with the ReLU mask of X on request; W [M x N] fp32, rounded to bfloat16
// M from 65 to 256, N up to 256, K = the number of sampled vertices.
//
// Both are streams over K: 256 flop per byte of X, D and G at M = N = 256, under the ridge of the bf16 pipe, so what counts is bytes.
// Apart they read D twice, and X twice where it is also the mask of G; here a slice of rows is fetched once and feeds both:
//  - a workgroup (one a compute unit, eight wavefronts) takes slices w, w + grid, ...: BK rows of X and of D go into LDS by direct
//    loads, several slices ahead, one barrier a slice, as in gemm_tn.hip;
//  - C: the whole result in registers, operands by transposing LDS reads, as in gemm_tn.hip; one partial result a workgroup,
//    added up by gemm_reduce.hip;
//  - G: a wavefront has 32 columns of it and keeps its part of W in registers for the whole kernel, as many of its 16-step pieces
//    as fit beside C (RS), the others in LDS in operand order (with all of it there the slices would have 32 KB, one in flight).  G^T like gemm_rows.hip: the lane holds 4 columns of a
//    row in 4 registers, two exchanges make that 16 bytes a lane and 64 bytes of 16 rows a store;
//  - the mask of G is read from the slice of X in LDS, the column sums of D (the bias gradient) are added up from the slice of D;
//  - rows behind the last one of a ragged K repeat it in LDS and are zeroed in registers for C; their part of G is dropped by the bounds of
//    the buffer.  So every wavefront has the same number of loads and stores a slice, and the waits count exactly.
#include <algorithm>

#include "gemm_stream.h"

namespace {

constexpr int BWD_WAVES = 8, BWD_LDS = 160 * 1024;

struct bwd_args {
    const u16 *X; int64_t ldx;      // [K x M], ldx a multiple of 8
    const u16 *D; int64_t ldd;      // [K x N], ldd a multiple of 8
    const float *W; int64_t ldw;    // [M x N]
    int M, N;
    int64_t K;
    u16 *G; int64_t ldg;
    int g_cols;                     // columns of G that may be written, a multiple of 8
    int mask;                       // G is zero where X is not positive
    float *partial;                 // [workgroups][M][N]
    float *cs_partial;              // [workgroups][N] or NULL
};

// The 16-byte chunks of a row are swizzled by the row, within groups of 16 where a row is a whole number of passes over the banks (256
// bytes), else within groups of 8.  Rows 0 to 3 of any four lie 64 bytes apart (the transposing reads take four rows together), and
// 16 rows in 16 different chunks (the reads of D for G).
template <int F> __device__ __forceinline__ int bwd_swizzle(int row)
{
    return (F % 128 == 0 ? 4 * (row & 3) : 4 * ((row >> 1) & 1)) | ((row >> 2) & 3);
}

template <int FA, int FB, int BK, int RS> struct bwd_shape {
    static constexpr int STAGE = (FA + FB) * 2 * BK, A_BYTES = FA * 2 * BK;
    static constexpr int WLDS = (FB / 16 - RS) * (FA / 32) * 1024;
    static constexpr int FIT = (BWD_LDS - WLDS) / STAGE, STAGES = FIT < 5 ? FIT : 5;
    static constexpr int LDS = STAGES * STAGE + WLDS;
    static_assert(STAGES >= 3 && A_BYTES % (1024 * BWD_WAVES) == 0 && (FA / 32) * (BK / 32) == BWD_WAVES, "every load a slice of one operand, a tile of G for every wavefront");
};

// WM x WN wavefronts share the frame's FA x FB result C.  WHOLE: N == FB, which leaves out the masks of D's last columns and the ragged ends of W's rows
// (2^20 x 256 x 256 359 us with the tests at run time, 342 without)
template <int FA, int FB, int BK, int WM, int WN, int RS, bool WHOLE>
__global__ __launch_bounds__(64 * BWD_WAVES, 2) void gemm_bwd_kernel(bwd_args a)
{
    using SH = bwd_shape<FA, FB, BK, RS>;
    constexpr int TM = FA / 32 / WM, TN = FB / 32 / WN, STAGE = SH::STAGE, STAGES = SH::STAGES;
    constexpr int CA = FA / 8, CB = FB / 8, WL = STAGE / 1024, AL = SH::A_BYTES / 1024, LOADS = (WL + BWD_WAVES - 1) / BWD_WAVES;
    constexpr int STEPS = FB / 16, STORES = 2, MT = FA / 32, CS = (STEPS + MT - 1) / MT;
    extern __shared__ __attribute__((aligned(16))) unsigned char bwd_smem[];
    unsigned char *const wlds = bwd_smem + STAGES * STAGE;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, kh = lane >> 5;
    const int mt = wave % MT, rt = wave / MT;          // the wavefront's tile of G: columns 32 mt .., rows 32 rt .. of a slice
    const int64_t total = (a.K + BK - 1) / BK;
    const int nslices = (int)((total - blockIdx.x + gridDim.x - 1) / gridDim.x);

    // load j of a slice fills KB wave + 8 j of the stage; a wavefront without a load repeats the last one (same bytes, same place).
    // A lane's row << 16 | byte in the row: where the eight KB between two loads are 16 rows or a multiple, only the row differs
    constexpr int AJ = AL / BWD_WAVES, BJ = LOADS - AJ, KEPT = CB % 16 == 0 ? 1 : BJ;
    auto lane_at = [&](int j, bool b) {
        const int p = (min(wave + BWD_WAVES * j, WL - 1) - (b ? AL : 0)) * 64 + lane, ch = b ? CB : CA, row = p / ch;
        const int c = (p % ch) ^ (b ? bwd_swizzle<FB>(row) : bwd_swizzle<FA>(row));
        return (uint32_t)row << 16 | 16u * (uint32_t)min(c, ((b ? a.N : a.M) - 1) / 8);
    };
    const uint32_t at_x = lane_at(0, false);
    uint32_t at_d[KEPT];
#pragma unroll
    for (int j = 0; j < KEPT; ++j) at_d[j] = lane_at(AJ + j, true);
    auto first_row = [&](int s) { return ((int64_t)s * gridDim.x + blockIdx.x) * BK; };
    auto issue = [&](int s) {
        const int64_t k0 = first_row(min(s, nslices - 1));          // past the end: the last slice again, into a stage nobody reads
        const int last = (int)min(a.K - k0, (int64_t)BK) - 1;
        unsigned char *stage = bwd_smem + (s % STAGES) * STAGE;
        const unsigned char *x0 = reinterpret_cast<const unsigned char *>(a.X + k0 * a.ldx), *d0 = reinterpret_cast<const unsigned char *>(a.D + k0 * a.ldd);
        const uint32_t ldx2 = (uint32_t)a.ldx * 2, ldd2 = (uint32_t)a.ldd * 2;
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int wl = min(wave + BWD_WAVES * j, WL - 1);
            const bool b = j >= AJ;
            const uint32_t at = !b ? at_x : at_d[KEPT == 1 ? 0 : j - AJ];
            const int row = (int)(at >> 16) + (!b ? j * (64 * BWD_WAVES / CA) : (KEPT == 1 ? (j - AJ) * (64 * BWD_WAVES / CB) : 0));
            const uint32_t off = (uint32_t)min(row, last) * (b ? ldd2 : ldx2) + (at & 0xffffu);
            __builtin_amdgcn_global_load_lds(STREAM_GPTR((b ? d0 : x0) + off), STREAM_LPTR(stage + 1024 * wl), 16, 0, 0);
        }
    };
    constexpr uint32_t BEYOND = 0x80000000u;      // outside the buffer: the store is dropped
    auto store = [&](int64_t k0, const u32x4 &v, uint32_t off) {
        __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(a.G + k0 * a.ldg, 0, 0x7fffffff, 0x00020000), off, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) {
        issue(s);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < STORES; ++t) store(0, u32x4{}, BEYOND);      // the loop's pattern, so that its first waits count the same
        asm volatile("" ::: "memory");
    }

    // the wavefront's 32 rows of W, zero beyond M and N: lane (li, kh) has columns 16 st + 8 kh .. + 7 of row 32 mt + li.  Four steps at a time:
    // all requested together they would spill, one by one they cost a round trip to memory each (8192 x 128 x 256 60 us instead of 34)
    const float *w_row = a.W + (int64_t)min(32 * mt + li, a.M - 1) * a.ldw;
    auto w_pieces = [&](int st0, bf16x8 (&v)[4]) {
        float x[4][8];
        if (st0 + 4 < STEPS || WHOLE) {          // (a frame is at most 63 columns wider than N)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float *p = w_row + 16 * (st0 + q) + 8 * kh;
                const f32x4_any lo = *reinterpret_cast<const f32x4_any *>(p), hi = *reinterpret_cast<const f32x4_any *>(p + 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) { x[q][i] = lo[i]; x[q][4 + i] = hi[i]; }
            }
        } else if (a.N >= 4) {
            // past the row's end the four that end with it, put right (32 loads of one value each, eight times the requests in front of everything
            // else: 10000 x 192 x 224 48 us, 9000 x 256 x 96 38)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = 16 * (st0 + q) + 8 * kh + 4 * h, cc = min(c, a.N - 4);
                    const f32x4 v = shifted(*reinterpret_cast<const f32x4_any *>(w_row + cc), min(c - cc, 4));
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[q][4 * h + i] = v[i];
                }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 8; ++i) x[q][i] = w_row[min(16 * (st0 + q) + 8 * kh + i, a.N - 1)];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 8; ++i) v[q][i] = (__bf16)(32 * mt + li < a.M && 16 * (st0 + q) + 8 * kh + i < a.N ? x[q][i] : 0.f);
    };
    static_assert(RS % 4 == 0 && STEPS % 4 == 0, "whole groups of steps");
    bf16x8 w[RS];
#pragma unroll
    for (int st = 0; st < RS; st += 4) {
        bf16x8 v[4];
        w_pieces(st, v);
#pragma unroll
        for (int q = 0; q < 4; ++q) w[st + q] = v[q];
        asm volatile("" ::: "memory");
    }
    if (rt == 0) {
#pragma unroll
        for (int st = RS; st < STEPS; st += 4) {
            bf16x8 v[4];
            w_pieces(st, v);
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<bf16x8 *>(wlds + ((st + q - RS) * MT + mt) * 1024 + lane * 16) = v[q];
            asm volatile("" ::: "memory");
        }
    }

    const int wm = wave / WN, wn = wave % WN;
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    float cs[CS][8];
#pragma unroll
    for (int q = 0; q < CS; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i) cs[q][i] = 0.f;
    const bool live = wm < WM && wm * TM * 32 < a.M && wn * TN * 32 < a.N;       // its part of the frame holds something of C

    // where a lane reads for C: of the sixteen lanes that read together, lane x takes columns 4 (x % 4) .. of row x / 4 of the four.  Chunk
    // numbers are put together in the loop (a scalar exclusive-or'ed to the lane's part): as loop invariants they would take
    // a register for every tile and step.  The rows 8 kh + 4 t + x / 4 of a 16-row block differ between t = 0 and 1 in the lowest swizzle bit.
    const int x = lane & 15, r3 = x >> 2, half = (lane >> 4) & 1;
    const uint32_t row_a = (8 * kh + r3) * FA * 2 + (x & 1) * 8, row_b = SH::A_BYTES + (8 * kh + r3) * FB * 2 + (x & 1) * 8;
    uint32_t lane_a = 16 * ((2 * half + ((x & 3) >> 1)) ^ bwd_swizzle<FA>(8 * kh + r3)), lane_b = 16 * ((2 * half + ((x & 3) >> 1)) ^ bwd_swizzle<FB>(8 * kh + r3));
    // where it reads D for G: row 32 rt + li, chunk 2 st + kh
    const uint32_t row_d = SH::A_BYTES + (32 * rt + li) * FB * 2;
    uint32_t lane_d = 16 * (kh ^ bwd_swizzle<FB>(32 * rt + li));
    auto d_piece = [&](const unsigned char *stage, int st) { return *reinterpret_cast<const u32x4 *>(stage + ((lane_d ^ (32u * st)) + row_d)); };
    // where it writes G: row 16 t + (lane & 15) of the tile, columns 32 mt + 16 half + 8 kh .. + 7
    const int g_row = 32 * rt + (lane & 15), g_chunk = 4 * mt + 2 * half + kh;
    const bool g_live = 8 * g_chunk + 8 <= a.g_cols;

    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the part of W in LDS, read behind the first barrier
    for (int s = 0; s < nslices; ++s) {
        asm volatile("" : "+v"(lane_a), "+v"(lane_b), "+v"(lane_d));
        STREAM_WAIT_VMCNT((STAGES - 2) * (LOADS + STORES));      // slice s has landed (this wavefront's part)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();                              // everybody's part has; and everybody is through slice s - 1
        asm volatile("" ::: "memory");
        issue(s + STAGES - 1);                                     // into the stage slice s - 1 was read from
        asm volatile("" ::: "memory");
        const unsigned char *stage = bwd_smem + (s % STAGES) * STAGE;
        const int64_t k0 = first_row(s);
        const int rows = (int)min(a.K - k0, (int64_t)BK);
        if (live) {
#pragma unroll
            for (int h = 0; h < BK / 16; ++h) {
                asm volatile("" ::: "memory");          // here and below: no operands of a later block beside these
                uint2 fa[TM][2], fb[TN][2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
#pragma unroll
                    for (int j = 0; j < TN; ++j) fb[j][t] = read_tr(stage + ((lane_b ^ (64u * (wn * TN + j) + 16u * t)) + row_b + (16 * h + 4 * t) * FB * 2));
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[i][t] = read_tr(stage + ((lane_a ^ (64u * (wm * TM + i) + 16u * t)) + row_a + (16 * h + 4 * t) * FA * 2));
                }
                if (rows < BK) {               // the last slice of a ragged K: steps behind the last row count as zeros
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int left = rows - (16 * h + 8 * kh + 4 * t);
                        const uint32_t m0 = left >= 2 ? 0xffffffffu : (left == 1 ? 0xffffu : 0u), m1 = left >= 4 ? 0xffffffffu : (left == 3 ? 0xffffu : 0u);
#pragma unroll
                        for (int j = 0; j < TN; ++j) { fb[j][t].x &= m0; fb[j][t].y &= m1; }
#pragma unroll
                        for (int i = 0; i < TM; ++i) { fa[i][t].x &= m0; fa[i][t].y &= m1; }
                    }
                }
                auto operand = [](const uint2 (&f)[2]) { return __builtin_bit_cast(bf16x8, make_uint4(f[0].x, f[0].y, f[1].x, f[1].y)); };
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(fa[i]), operand(fb[j]), acc[i][j], 0, 0, 0);
            }
        }
        f32x16 g;
#pragma unroll
        for (int r = 0; r < 16; ++r) g[r] = 0.f;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            if (st % 4 == 0) asm volatile("" ::: "memory");
            u32x4 d = d_piece(stage, st);
            if (!WHOLE && st >= STEPS - 4 && 16 * st + 16 > a.N) {     // columns behind the last one hold anything (a frame is at most 63 wider than N)
                const int left = a.N - (16 * st + 8 * kh);
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] &= left >= 2 * i + 2 ? 0xffffffffu : (left == 2 * i + 1 ? 0xffffu : 0u);
            }
            bf16x8 wv;
            if (st < RS) wv = w[st < RS ? st : 0];
            else wv = *reinterpret_cast<const bf16x8 *>(wlds + ((st - RS) * MT + mt) * 1024 + lane * 16);
            g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, __builtin_bit_cast(bf16x8, d), g, 0, 0, 0);
        }
        if (a.cs_partial) {                                  // each wavefront of a row tile adds up some of the columns
#pragma unroll
            for (int q = 0; q < CS; ++q) {
                const int st = min(mt + MT * q, STEPS - 1);
                const u32x4 d = d_piece(stage, st);
                const uint32_t keep = 32 * rt + li < rows ? 0xffffffffu : 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    cs[q][2 * i] += __builtin_bit_cast(float, (d[i] << 16) & keep);
                    cs[q][2 * i + 1] += __builtin_bit_cast(float, d[i] & 0xffff0000u & keep);
                }
            }
        }
        // register 4 q + i of lane (li, kh): row li of the tile, column 8 q + 4 kh + i
        u32x4 o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t p[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                p[q][0] = pack_bf16(g[8 * h + 4 * q], g[8 * h + 4 * q + 1]);
                p[q][1] = pack_bf16(g[8 * h + 4 * q + 2], g[8 * h + 4 * q + 3]);
            }
            // columns 16 h + 8 kh .. + 7 of the row: the lower half of the wavefront takes q = 0, the upper q = 1
            const auto r0 = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
            o[h] = u32x4{(uint32_t)r0[0], (uint32_t)r1[0], (uint32_t)r0[1], (uint32_t)r1[1]};
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
            const int row = g_row + 16 * t;
            if (a.mask) {
                const u32x4 m = *reinterpret_cast<const u32x4 *>(stage + row * FA * 2 + (g_chunk ^ bwd_swizzle<FA>(row)) * 16);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t lo = __builtin_bit_cast(float, m[i] << 16) > 0.f ? 0xffffu : 0u;
                    const uint32_t hi = __builtin_bit_cast(float, m[i] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u;
                    o[t][i] &= lo | hi;
                }
            }
            store(k0, o[t], g_live && row < rows ? (uint32_t)row * (uint32_t)(a.ldg * 2) + 16u * (uint32_t)g_chunk : BEYOND);
        }
    }
    STREAM_WAIT_VMCNT(0);       // the repeated loads past the end are still in flight: nothing may leave, nor use the LDS, before they land
    asm volatile("" ::: "memory");

    // register r of lane (li, kh) of tile (i, j) is row 32 i + 8 (r / 4) + 4 kh + r % 4, column 32 j + li of the wavefront's part
    if (live) {
        float *P = a.partial + (int64_t)blockIdx.x * a.M * a.N;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = (wn * TN + j) * 32 + li;
            if (n >= a.N) continue;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = (wm * TM + i) * 32 + 8 * (r / 4) + 4 * kh + r % 4;
                    if (m < a.M) P[(int64_t)m * a.N + n] = acc[i][j][r];
                }
        }
    }
    if (a.cs_partial) {
        __syncthreads();          // everybody's loads have landed and everybody is through the last slice
        float *sums = reinterpret_cast<float *>(bwd_smem);          // [row tile][column]
#pragma unroll
        for (int q = 0; q < CS; ++q)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float v = cs[q][i];
#pragma unroll
                for (int d = 16; d >= 1; d >>= 1) v += __shfl_xor(v, d);
                const int n = 16 * (mt + MT * q) + 8 * kh + i;
                if (li == 0 && n < FB) sums[rt * FB + n] = v;
            }
        __syncthreads();
        for (int n = threadIdx.x; n < a.N; n += 64 * BWD_WAVES) {
            float v = sums[n];
            for (int r = 1; r < BK / 32; ++r) v += sums[r * FB + n];
            a.cs_partial[(int64_t)blockIdx.x * a.N + n] = v;
        }
    }
}

template <int FA, int FB, int BK, int WM, int WN, int RS, bool WHOLE> int launch_bwd_n(sgnn_ctx *ctx, const bwd_args &a, unsigned grid, hipStream_t st)
{
    constexpr int lds = bwd_shape<FA, FB, BK, RS>::LDS;
    SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_bwd_kernel<FA, FB, BK, WM, WN, RS, WHOLE>>(ctx, lds)));
    char tag[56];
    snprintf(tag, sizeof(tag), "bwd %dx%dx%lld bf16%s", a.M, a.N, (long long)a.K, a.mask ? " mask" : "");
    SGNN_LAUNCH(ctx, st, "gemm_bwd_kernel", tag, (gemm_bwd_kernel<FA, FB, BK, WM, WN, RS, WHOLE>), dim3(grid), dim3(64 * BWD_WAVES), lds, st, a);
    return SGNN_OK;
}

template <int FA, int FB, int BK, int WM, int WN, int RS> int launch_bwd(sgnn_ctx *ctx, const bwd_args &a, unsigned grid, hipStream_t st)
{
    return a.N == FB ? launch_bwd_n<FA, FB, BK, WM, WN, RS, true>(ctx, a, grid, st) : launch_bwd_n<FA, FB, BK, WM, WN, RS, false>(ctx, a, grid, st);
}

inline bool overlap(const void *p, size_t n, const void *q, size_t m)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + m && b < a + n;
}

} // namespace

// Returns SGNN_ERR_UNSUPPORTED without launching anything for what the kernel does not handle: the two products then run one after the
// other.  g_pad: the columns of G between M and the leading dimension may be written.
int sgnn_launch_gemm_bwd(sgnn_ctx *ctx, int64_t M, int64_t N, int64_t K, const void *X, int64_t ldx, const void *D, int64_t ldd, const float *W,
                         int64_t ldw, void *G, int64_t ldg, bool g_pad, bool mask, float *C, float *d_colsum, ws_alloc *ws, hipStream_t st)
{
    constexpr int64_t LD_MAX = 1 << 20;          // offsets within a slice in 32 bits
    auto al16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    const int64_t g_cols = (M + 7) & ~int64_t(7);
    if (M <= 64 || M > 256 || N < 1 || N > 256 || K < 8192 || ldx % 8 || ldd % 8 || ldg % 8 || ldx < M || ldd < N || ldx >= LD_MAX || ldd >= LD_MAX ||
        ldg >= LD_MAX || ldg < g_cols || (g_cols != M && !g_pad) || !al16(X) || !al16(D) || !al16(G))
        return SGNN_ERR_UNSUPPORTED;
    // G in the place of X is fine (a row is read by the workgroup that writes it, before it does); anything else that G shares with an
    // operand would be written while others still read it
    const size_t gb = (size_t)K * ldg * 2;
    if ((overlap(G, gb, X, (size_t)K * ldx * 2) && !(G == X && ldg == ldx)) || overlap(G, gb, D, (size_t)K * ldd * 2) ||
        overlap(G, gb, W, (size_t)M * ldw * 4))
        return SGNN_ERR_UNSUPPORTED;
    const int fa = M > 128 ? 256 : 128, fb = N > 192 ? 256 : (N > 128 ? 192 : (N > 64 ? 128 : 64)), bk = fa == 256 ? 32 : 64;
    // Narrow X and wide D: 64 columns of G for eight wavefronts at a time are little work beside the D that each of them reads, and with few rows the
    // two products out of the Infinity Cache are faster: 16384 x 128 x 256 38 us there, 44 here, 50000 x 128 x 128 40 / 43, 100 x 200 54 / 62;
    // 100000 x 128 x 256 68 / 67, 131072 x 100 x 200 78 / 78, 128 x 256 76 / 73.
    if (fa == 128 && fb > 64 && K < 110000) return SGNN_ERR_UNSUPPORTED;
    // Up to 192 columns of X beside more than 192 of D, the frame half empty, and no mask to save: 10000 x 192 x 224 43 us there, 45 here, x 160 x 224 41 / 43, x 192 x 256
    // 43 / 44.5, 14000 x 192 x 224 44 / 45.6; 16384 x 192 x 224 43.5 / 43.4, 10000 x 224 x 224 45 / 45.5, with a mask 10000 x 192 x 224 45 / 42.
    if (!mask && fa == 256 && fb == 256 && M <= 192 && K < 16000) return SGNN_ERR_UNSUPPORTED;
    // A workgroup costs its partial result, written and read, and W, and with few slices its pipeline is never full: one for every 256 rows,
    // but 128 of them while that leaves each 128 rows.  us with a workgroup for 128 / 192 / 256 / 384 / 512 rows, M = N = 256: 16384 rows 47 / 49 / 50 / 59 / 64,
    // 24000 56 / 53 / 57 / 63 / 70, 40000 64 / 63 / 63 / 67 / 73, 65536 73 / 72 / 72 / 73 / 76.
    const int64_t groups = std::min<int64_t>(256, std::max(K / 256, std::min<int64_t>(128, K / 128)));
    const size_t need = (((size_t)groups * M * N * 4 + 255) & ~size_t(255)) + (((size_t)groups * N * 4 + 255) & ~size_t(255));
    if (!ws->base || ws->off + need > ws->cap) return SGNN_ERR_UNSUPPORTED;
    bwd_args a;
    a.X = static_cast<const u16 *>(X); a.ldx = ldx; a.D = static_cast<const u16 *>(D); a.ldd = ldd; a.W = W; a.ldw = ldw;
    a.M = (int)M; a.N = (int)N; a.K = K;
    a.G = static_cast<u16 *>(G); a.ldg = ldg; a.g_cols = (int)g_cols; a.mask = mask;
    a.partial = ws->get<float>((size_t)groups * M * N);
    a.cs_partial = d_colsum ? ws->get<float>((size_t)groups * N) : nullptr;
    const unsigned grid = (unsigned)groups;
    int rc;
    if (fa == 256 && fb == 256) rc = launch_bwd<256, 256, 32, 2, 4, 8>(ctx, a, grid, st);
    else if (fa == 256 && fb == 192) rc = launch_bwd<256, 192, 32, 4, 2, 12>(ctx, a, grid, st);
    else if (fa == 256 && fb == 128) rc = launch_bwd<256, 128, 32, 4, 2, 8>(ctx, a, grid, st);
    else if (fa == 256) rc = launch_bwd<256, 64, 32, 4, 2, 4>(ctx, a, grid, st);
    else if (fb == 256) rc = launch_bwd<128, 256, 64, 2, 4, 16>(ctx, a, grid, st);
    else if (fb == 192) rc = launch_bwd<128, 192, 64, 4, 2, 12>(ctx, a, grid, st);
    else if (fb == 128) rc = launch_bwd<128, 128, 64, 2, 4, 8>(ctx, a, grid, st);
    else rc = launch_bwd<128, 64, 64, 4, 2, 4>(ctx, a, grid, st);
    if (rc) return rc;
    return sgnn_launch_splitk_reduce(ctx, a.partial, (int)groups, M, N, C, N, a.cs_partial, d_colsum, st);
}
