// Weight gradient of a mini-batch (Sec. III-C: dW = H_agg^T dZ) with both operands stored as bfloat16:
//   C [M x N] = A^T B,   A given [K x M], B given [K x N], M, N <= 256, K = the number of sampled vertices (8192 .. 10^6).
//
// The product reads 2 K (M + N) bytes and computes 2 K M N flop: with M = N = 256 that is 128 flop per byte, far below
// the machine's bf16 ridge, so the kernel is built as a stream over K and nothing else:
//  - a workgroup takes slices of 32 rows and holds the WHOLE M x N result in registers (eight wavefronts), so every row of A
//    and of B is fetched from HBM once, by one workgroup;
//  - a slice goes into LDS with direct global -> LDS loads (16 bytes a lane, no registers in between), four slices deep: three
//    are in flight behind the one being multiplied, one barrier per slice;
//  - v_mfma_f32_32x32x16_bf16 wants, per lane, eight consecutive reduction steps of one column, which in this storage are eight
//    rows apart: the transposing LDS reads (ds_read_b64_tr_b16: sixteen lanes read 4 rows x 16 columns and each gets the four
//    values of one column) deliver them two registers at a time.  With ordinary reads, two thirds of the instructions
//    of the loop were reads and byte permutes, and those, not memory, set its pace;
//  - a row of a slice takes a frame of FA (FB) elements in LDS whatever the leading dimension is, and its 16-byte chunks are
//    swizzled by the row, so that the four rows which such a read takes together lie in different banks.  The direct loads write
//    LDS in lane order, so the swizzle is in the global address a lane loads from;
//  - the column sums of B (the bias gradient that rides along) come from the matrix pipe too: one more MFMA per B
//    tile with an A operand that is 1 in result row 0 and 0 elsewhere;
//  - every workgroup writes one partial product; they are added in a fixed order by gemm_reduce.hip.
// Rows behind the last one of a ragged K repeat it in LDS and are zeroed in registers.  Columns of the frame beyond M or N repeat
// the row's last chunk: they only feed result rows and columns that are never stored.
// Measured with the reduction of the partial products, us: 256 x 256 x 2^20 202 (5.3 TB/s of A and B, the rate of a copy), 256 x 172 179, 128 x 256 149, 256 x 256 x 2^18
// 69, 256 x 47 36; with three, five stages 203 and 204, 176 and 176, 147 and 149, 69 and 70, 35 and 36.  Before the slices ahead stayed in flight (gemm_stream.h) and the
// partial products were shared by more wavefronts (gemm_reduce.hip): 242, 217, 179, 78, 45.  With ordinary reads and permutes the first was 313 of then 289.
// Where the K or the width was outside the earlier form: 200 x 193 x 56399 183 -> 40, 30 x 256 x 300007 565 -> 47.
#include <algorithm>

#include "gemm_stream.h"

namespace {

constexpr int TNS_BK = 32;          // rows of a slice
constexpr int TNS_STAGES = 4;
constexpr int TNS_WAVES = 8;

struct tns_args {
    const u16 *A; int64_t lda;      // [K x M] bfloat16, lda a multiple of 8
    const u16 *B; int64_t ldb;      // [K x N] bfloat16, ldb a multiple of 8
    int M, N;
    int64_t K;
    float *partial;                 // [splits][M][N]
    float *cs_partial;              // [splits][N] or NULL
};

// frame of an operand: F elements a row, F / 8 chunks of 16 bytes.  Chunks are swizzled in groups of four (the 32 columns of a
// tile) by the row: rows 0 to 3 of any four take different 64 bytes of the 256 that the banks span.
template <int F> struct frame {
    static constexpr int CHUNKS = F / 8, BYTES = TNS_BK * F * 2;
    static __device__ __forceinline__ int swizzle(int row) { return F >= 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};

template <int FA, int FB> constexpr int tns_stage_bytes() { return frame<FA>::BYTES + frame<FB>::BYTES; }

// WM x WN wavefronts share the frame's FA x FB result
template <int FA, int FB, int WM, int WN>
__global__ __launch_bounds__(64 * TNS_WAVES) void gemm_tn_stream_kernel(tns_args a)
{
    constexpr int TM = FA / 32 / WM, TN = FB / 32 / WN;
    constexpr int STAGE = tns_stage_bytes<FA, FB>(), LOADS = (STAGE / 1024 + TNS_WAVES - 1) / TNS_WAVES;
    constexpr int CA = frame<FA>::CHUNKS, CB = frame<FB>::CHUNKS;
    extern __shared__ __attribute__((aligned(16))) unsigned char tns_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, kh = lane >> 5;
    // workgroup w takes slices w, w + grid, ...: the workgroups read one region together, as a copy kernel does
    const int64_t total = (a.K + TNS_BK - 1) / TNS_BK;
    const int nslices = (int)((total - blockIdx.x + gridDim.x - 1) / gridDim.x);

    // the wavefront's wave-loads of a slice: load j fills KB wave + 8 j of the stage.  A lane's row and byte offset from the
    // slice's first row; a wavefront without a load repeats the last one (same bytes, same place), so that every wavefront has the
    // same number in flight and the waits below count exactly
    int row[LOADS], off[LOADS];
    bool of_b[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int pos = min(wave + TNS_WAVES * j, STAGE / 1024 - 1) * 64 + lane;
        of_b[j] = pos >= TNS_BK * CA;
        const int p = of_b[j] ? pos - TNS_BK * CA : pos, ch = of_b[j] ? CB : CA;
        row[j] = p / ch;
        const int c = (p % ch) ^ (of_b[j] ? frame<FB>::swizzle(row[j]) : frame<FA>::swizzle(row[j]));
        off[j] = 16 * min(c, ((of_b[j] ? a.N : a.M) - 1) / 8);
    }
    auto issue = [&](int s) {
        const int sl = min(s, nslices - 1);          // past the end: the last slice again, into a stage nobody reads
        unsigned char *stage = tns_smem + (s % TNS_STAGES) * STAGE;
        const int64_t k0 = ((int64_t)sl * gridDim.x + blockIdx.x) * TNS_BK;
        const int last = (int)min(a.K - k0, (int64_t)TNS_BK) - 1;
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int64_t r = k0 + min(row[j], last);
            const unsigned char *g = (of_b[j] ? reinterpret_cast<const unsigned char *>(a.B + r * a.ldb) : reinterpret_cast<const unsigned char *>(a.A + r * a.lda)) + off[j];
            __builtin_amdgcn_global_load_lds(STREAM_GPTR(g), STREAM_LPTR(stage + 1024 * min(wave + TNS_WAVES * j, STAGE / 1024 - 1)), 16, 0, 0);
        }
    };

    const int wm = wave / WN, wn = wave % WN;
    f32x16 acc[TM][TN], cs[TN];
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i][j][r] = 0.f;
            cs[j][r] = 0.f;
        }
    // A operand of the column sums: 1.0 for result row 0 (lanes with li == 0), 0 elsewhere
    bf16x8 ones;
#pragma unroll
    for (int t = 0; t < 8; ++t) ones[t] = (__bf16)(li == 0 ? 1.0f : 0.0f);
    const bool live = wm < WM && wm * TM * 32 < a.M && wn * TN * 32 < a.N;       // its part of the frame holds something of the result
    const bool do_cs = a.cs_partial && wm == 0 && wn * TN * 32 < a.N;

    // where a lane reads: of the sixteen lanes that read together, lane x takes columns 4 (x % 4) .. of row x / 4
    const int x = lane & 15, r3 = x >> 2, half = (lane >> 4) & 1;
    int at_a[TM], at_b[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
        at_a[i] = (8 * kh + r3) * FA * 2 + (((wm * TM + i) * 4 + 2 * half + ((x & 3) >> 1)) ^ frame<FA>::swizzle(r3)) * 16 + (x & 1) * 8;
#pragma unroll
    for (int j = 0; j < TN; ++j)
        at_b[j] = frame<FA>::BYTES + (8 * kh + r3) * FB * 2 + (((wn * TN + j) * 4 + 2 * half + ((x & 3) >> 1)) ^ frame<FB>::swizzle(r3)) * 16 + (x & 1) * 8;

    issue(0);
    issue(1);
    issue(2);
    for (int s = 0; s < nslices; ++s) {
        STREAM_WAIT_VMCNT(2 * LOADS);               // slice s has landed (this wavefront's part); s + 1 and s + 2 may be in flight
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();            // everybody's part has; and everybody is through slice s - 1
        asm volatile("" ::: "memory");
        issue(s + 3);                            // into the stage slice s - 1 was read from
        if (live) {
            const unsigned char *stage = tns_smem + (s % TNS_STAGES) * STAGE;
            const int rows = (int)min(a.K - ((int64_t)s * gridDim.x + blockIdx.x) * TNS_BK, (int64_t)TNS_BK);
#pragma unroll
            for (int h = 0; h < 2; ++h) {          // the two 16-step blocks of the slice
                uint2 fa[TM][2], fb[TN][2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
#pragma unroll
                    for (int j = 0; j < TN; ++j) fb[j][t] = read_tr(stage + at_b[j] + (16 * h + 4 * t) * FB * 2);
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[i][t] = read_tr(stage + at_a[i] + (16 * h + 4 * t) * FA * 2);
                }
                if (rows < TNS_BK) {               // the last slice of a ragged K: steps behind the last row count as zeros
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
                if (do_cs) {
#pragma unroll
                    for (int j = 0; j < TN; ++j) cs[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, operand(fb[j]), cs[j], 0, 0, 0);
                }
            }
        }
    }
    STREAM_WAIT_VMCNT(0);       // the repeated loads past the end are still in flight: nothing may leave before they land

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
            if (do_cs && kh == 0) a.cs_partial[(int64_t)blockIdx.x * a.N + n] = cs[j][0];      // result row 0
        }
    }
}

template <int FA, int FB, int WM, int WN> int launch_tns(sgnn_ctx *ctx, const tns_args &a, unsigned grid, hipStream_t st)
{
    constexpr int lds = TNS_STAGES * tns_stage_bytes<FA, FB>();
    SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_tn_stream_kernel<FA, FB, WM, WN>>(ctx, lds)));
    char tag[56];
    snprintf(tag, sizeof(tag), "TN stream %dx%dx%lld bf16 a=2 b=2", a.M, a.N, (long long)a.K);
    SGNN_LAUNCH(ctx, st, "gemm_tn_stream_kernel", tag, (gemm_tn_stream_kernel<FA, FB, WM, WN>), dim3(grid), dim3(64 * TNS_WAVES), lds, st, a);
    return SGNN_OK;
}

} // namespace

// Returns SGNN_ERR_UNSUPPORTED without launching anything when the shape or the storage is outside what the kernel
// handles (the caller then takes the tile kernel); otherwise launches the product and the split reduction.
int sgnn_launch_gemm_tn_stream(sgnn_ctx *ctx, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
                               float *C, int64_t ldc, float *b_colsum, ws_alloc *ws, hipStream_t st)
{
    // Reductions of fewer than 8192 rows stay with the tile kernel: there the product of operands stored as bfloat16 is, bit for
    // bit, that of the same values stored as fp32 (which the tile kernel rounds), and callers may mix the two.  It costs at
    // most some 20 us a product: 256 x 256 x 999 37 us there, 14 here.
    if (M < 1 || N < 1 || M > 256 || N > 256 || K < 8192 || lda % 8 || ldb % 8 || lda < M || ldb < N ||
        (reinterpret_cast<uintptr_t>(A) & 15) || (reinterpret_cast<uintptr_t>(B) & 15))
        return SGNN_ERR_UNSUPPORTED;
    // As many workgroups as make the partial products (written and read: 8 M N bytes each) about as much traffic as the operands,
    // no fewer than one for every four slices up to 64, at most one a compute unit.
    const int64_t slices = cdiv(K, TNS_BK);
    int64_t splits = std::max<int64_t>(K * (M + N) / (4 * M * N), std::min<int64_t>(slices / 4, 64));
    splits = std::max<int64_t>(1, std::min<int64_t>(splits, std::min<int64_t>(slices, 256)));
    // not enough scratch for one partial product per workgroup: the tile kernel needs less
    const size_t need = (((size_t)splits * M * N * 4 + 255) & ~size_t(255)) + (((size_t)splits * N * 4 + 255) & ~size_t(255));
    if (!ws->base || ws->off + need > ws->cap) return SGNN_ERR_UNSUPPORTED;
    tns_args a;
    a.A = static_cast<const u16 *>(A); a.lda = lda; a.B = static_cast<const u16 *>(B); a.ldb = ldb;
    a.M = (int)M; a.N = (int)N; a.K = K;
    a.partial = ws->get<float>((size_t)splits * M * N);
    a.cs_partial = b_colsum ? ws->get<float>((size_t)splits * N) : nullptr;
    const int fa = M > 128 ? 256 : (M > 64 ? 128 : 64), fb = N > 128 ? 256 : (N > 64 ? 128 : 64);
    int rc = SGNN_ERR_UNSUPPORTED;
    if (fa == 256 && fb == 256) rc = launch_tns<256, 256, 2, 4>(ctx, a, (unsigned)splits, st);
    else if (fa == 256 && fb == 128) rc = launch_tns<256, 128, 4, 2>(ctx, a, (unsigned)splits, st);
    else if (fa == 256) rc = launch_tns<256, 64, 4, 2>(ctx, a, (unsigned)splits, st);
    else if (fa == 128 && fb == 256) rc = launch_tns<128, 256, 2, 4>(ctx, a, (unsigned)splits, st);
    else if (fa == 128 && fb == 128) rc = launch_tns<128, 128, 2, 4>(ctx, a, (unsigned)splits, st);
    else if (fa == 128) rc = launch_tns<128, 64, 4, 2>(ctx, a, (unsigned)splits, st);
    else if (fb == 256) rc = launch_tns<64, 256, 2, 4>(ctx, a, (unsigned)splits, st);
    else if (fb == 128) rc = launch_tns<64, 128, 2, 4>(ctx, a, (unsigned)splits, st);
    else rc = launch_tns<64, 64, 2, 2>(ctx, a, (unsigned)splits, st);
    if (rc) return rc;
    return sgnn_launch_splitk_reduce(ctx, a.partial, (int)splits, M, N, C, ldc, a.cs_partial, b_colsum, st);
}
