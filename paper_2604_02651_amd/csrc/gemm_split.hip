// fp32 products on the bfloat16 matrix pipe: every operand is split exactly into three bfloat16 parts and the six products
// of the parts that matter are accumulated in fp32.
//
//   x = x1 + x2 + x3,  x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2     (round to nearest even: exact, 3 x 8 bits)
//   a b = a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1) + up to 0.92 x 2^-24 |a b|  (the three products left out)
//
// The method is that of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations" (2019).  The products of two parts are exact in fp32; the leading products and the five
// small ones have accumulators of their own, and the leading chain then has one rounding step per 16 reduction steps where
// the fp32 instructions have eight.  Error against 64 bits (2-norm), fp32 instructions / here: 32768 x 256 x 256
// 2.0e-7 / 0.7e-7, 65536 x 256 x 608 3.1e-7 / 1.1e-7, 256 x 256 x 32768 2.9e-7 / 1.3e-7.  What is left out shows where an entry is a
// single product (a diagonal operand): its error is up to 1.72 x 2^-24, one rounding to fp32 up to 1.0.
//
// What bounds these products is the matrix pipe: the fp32 instructions reach 154 TFLOP/s on a large product, the bfloat16 ones
// 1140, of which a sixth is 190.  32768 x 256 x 256: 47 us with the fp32 instructions, 33 here (30 with the splitting left
// out); 65536 x 256 x 608 185 -> 133; 256 x 256 x 32768 54 -> 43; 608 x 256 x 65536 344 -> 205; 200 x 200 x 1057 88 -> 16 (its
// reduction was not split).
//
// A workgroup computes a BM x BN tile; slices of 32 along the reduction are fetched two ahead into registers, split there, and
// staged one ahead in LDS as three planes of [row][32] bfloat16; a lane reads the eight values of an MFMA operand with one
// 16-byte load.  Rows of a tile are dealt out to its T = R / 32 blocks of 32 in turn (row r is row r / T of block r % T), so
// that both ways an operand may lie in memory fill the planes without bank conflicts.
//
// Where the split does not hold, the tile is computed again with the fp32 instructions: by a wavefront whose accumulators are
// not all finite (an infinity or NaN in the operands, an overflow), by a workgroup that has staged a value below 2^-112 in
// magnitude other than zero (the parts of such a value reach below the smallest bfloat16 number: the error would be 2^-134,
// measured 1.7e-7 of the result for operands of about 2^-112, 5e-7 at 2^-114).  That costs time with such values, which are rare
// (a softmax gradient has them where logits lie more than 65 apart): 32768 x 256 x 256 34 us, 122 if one tile or every
// one holds one (fp32 instructions before: 47); 65536 x 256 x 608 134 us, 269 and 519 (189); 256 x 256 x 32768 42, 144 (48).
#include <algorithm>

#include "common.h"

namespace {

#include "split_parts.h"

struct split_args {
    int64_t M, N, K;
    const float *A; int64_t lda;
    const int32_t *ridx;          // optional: physical row of A (as stored) for every logical one
    const float *B; int64_t ldb;
    const float *bias;
    float *C; int64_t ldc;
    int relu;
    const float *mask; int64_t ldm;
    int64_t kps;                  // reduction range of a split (a multiple of 32), K when there is one
    float *partial;               // [splits][M][N], or null
    float *colsum;                // column sums of B: [splits][N] when split
    uint32_t mtiles, ntiles, splits;
};

constexpr int SBK = 32;                                     // slice of the reduction

template <int R> struct plane {
    static constexpr int BLOCK = 32 * SBK * 2 + 64;         // bytes of a block of 32 rows; 64 more, so that row l of different
    static constexpr int BYTES = (R / 32) * BLOCK;          // blocks does not fall into the same banks
};
// byte offset in a plane of the 16-byte chunk `c` (eight reduction values) of row l of block b: chunks are swizzled so that
// the rows which a wavefront reads together fall into different banks
__device__ __forceinline__ int chunk_at(int block_bytes, int b, int l, int c) { return b * block_bytes + l * (SBK * 2) + ((c ^ (l >> 1)) & 3) * 16; }

// One operand: R rows of the tile, stored [row][reduction] (KC) or [reduction][row].  A thread holds PER units of 16 bytes (KC:
// four reduction steps of a row) or of four times 16 bytes (else: four reduction steps x four rows).  Every load is issued,
// at an address moved back into the matrix where it would leave it: a load under a condition would be waited for on the spot.
// What such a load brought is put right when the slice is staged (align): the values are shifted, zeros behind the edge.  Rows
// behind the last one repeat it if KC (they only feed results that are not stored).
template <int R, int NT, bool KC, bool GATHER> struct operand {
    static constexpr int T = R / 32, BLOCK = plane<R>::BLOCK;
    static constexpr int UNITS = KC ? R * 8 : R * 2;
    static constexpr int PER = UNITS / NT ? UNITS / NT : 1;
    static constexpr int NF = KC ? PER : 4 * PER;           // 16-byte loads per thread and slice
    static_assert(KC || PER == 1, "one block of 4 x 4 a thread");
    f32x4 reg[NF];
    const float *base[KC ? PER : 1];                        // KC: the thread's rows; else its first column (addresses are 64 bits
                                                            // throughout: a leading dimension may be as long as a graph has vertices)
    int at;                                                 // where its values go in a plane
    int rows_left;                                          // !KC: rows that exist from the thread's first on
    int32_t next[(!KC && GATHER) ? 4 : 1];                  // row numbers of the next slice

    __device__ __forceinline__ static int unit() { return (int)threadIdx.x % UNITS; }
    __device__ __forceinline__ static bool active() { return UNITS >= NT || (int)threadIdx.x < UNITS; }

    __device__ __forceinline__ void init(const float *G, int64_t ld, const int32_t *ridx, int64_t row0, int64_t rows, int64_t k0, int64_t kend)
    {
        const int i = unit(), line = i / 8;
        if constexpr (KC) {
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int64_t r = min(row0 + line + u * (NT / 8), rows - 1);
                base[u] = G + (GATHER ? (int64_t)ridx[r] : r) * ld;
            }
            at = chunk_at(BLOCK, line % T, line / T, (i % 8) >> 1) + (i & 1) * 8;
        } else {
            rows_left = (int)min(rows - row0 - 4 * line, (int64_t)4);
            base[0] = G + row0 + (4 * line - (4 - rows_left));
            at = chunk_at(BLOCK, (4 * line) % T, (4 * line) / T, (i % 8) >> 1) + (i & 1) * 8;
        }
        indices(ridx, k0, kend);
    }
    // row u of a KC operand, row e of the other kind, relative to `at` (rows that differ by a multiple of 8 T are swizzled alike)
    __device__ __forceinline__ static int step(int n) { return KC ? n * (NT / 8 / T) * (SBK * 2) : (n % T) * BLOCK + (n / T) * (SBK * 2); }

    __device__ __forceinline__ void indices(const int32_t *ridx, int64_t k0, int64_t kend)
    {
        if constexpr (!KC && GATHER) {
#pragma unroll
            for (int j = 0; j < 4; ++j) next[j] = ridx[min(k0 + 4 * (unit() % 8) + j, kend - 1)];
        }
    }
    __device__ __forceinline__ void fetch(int64_t ld, int64_t k0, int64_t kend)
    {
        const int left = (int)min(kend - k0, (int64_t)SBK), kk = 4 * (unit() % 8);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const float *p;
            if constexpr (KC) p = base[f] + k0 + min(kk, left - 4);
            else if constexpr (GATHER) p = base[0] + (int64_t)next[f] * ld;
            else p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(base[0] + k0 * ld) +
                                                     (uint64_t)(uint32_t)min(kk + f, left - 1) * (uint64_t)(4 * ld));
            reg[f] = *reinterpret_cast<const f32x4_any *>(p);
        }
    }
    // v moved down by s places, zeros from above
    __device__ __forceinline__ static f32x4 shifted(f32x4 v, int s)
    {
        v = (s & 1) ? f32x4{v[1], v[2], v[3], 0.f} : v;
        v = (s & 2) ? f32x4{v[2], v[3], 0.f, 0.f} : v;
        return s >= 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : v;
    }
    // for slices that reach behind the end of the reduction range, and tiles at the edge of the matrix
    __device__ __forceinline__ void align(int64_t k0, int64_t kend)
    {
        const int left = (int)min(kend - (k0 + 4 * (unit() % 8)), (int64_t)4);        // reduction steps that exist from the unit's first on
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if constexpr (KC) reg[f] = shifted(reg[f], min(4 - left, 4));
            else reg[f] = f < left ? shifted(reg[f], min(4 - rows_left, 4)) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __device__ __forceinline__ void stage(unsigned char *lds, uint32_t &tiny)
    {
        if (!active()) return;
#pragma unroll
        for (int n = 0; n < (KC ? PER : 4); ++n) {
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = KC ? reg[KC ? n : 0][j] : reg[KC ? 0 : j][n];
            const parts4 s = split4(v, tiny);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2 *>(lds + q * plane<R>::BYTES + at + step(n)) = s.p[q];
        }
    }
};

template <int BM, int BN> constexpr int split_lds_bytes() { return 2 * 3 * (plane<BM>::BYTES + plane<BN>::BYTES); }

template <int BM, int BN, int WM, int WN, bool AKC, bool BKC, bool GATHER>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_split_kernel(split_args a)
{
    constexpr int NT = 64 * WM * WN;                         // WM x WN wavefronts
    constexpr int TM = BM / 32 / WM, TN = BN / 32 / WN;      // blocks of 32 x 32 per wavefront
    constexpr int PA = plane<BM>::BYTES, PB = plane<BN>::BYTES, BUF = 3 * (PA + PB);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];       // two buffers of the planes of A and of B
    __shared__ int small_seen;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 31, kh = lane >> 5;
    const int ta0 = (wave / WN) * TM, tb0 = (wave % WN) * TN;       // the wavefront's first row and column block
    // Tiles that read the same operand rows (the column tiles of a row block; all tiles of a reduction range) go to one XCD,
    // next to each other.
    const uint32_t members = a.splits > 1 ? a.mtiles * a.ntiles : a.ntiles, groups = a.splits > 1 ? a.splits : a.mtiles;
    const uint32_t group = (blockIdx.x / 8 / members) * 8 + blockIdx.x % 8, mem = (blockIdx.x / 8) % members;
    if (group >= groups) return;
    const uint32_t bx = a.splits > 1 ? mem % a.mtiles : group, by = a.splits > 1 ? mem / a.mtiles : mem, bz = a.splits > 1 ? group : 0;
    const int64_t m0 = (int64_t)bx * BM, n0 = (int64_t)by * BN;
    const int64_t kbeg = (int64_t)bz * a.kps, kend = min(a.K, kbeg + a.kps);

    if (threadIdx.x == 0) small_seen = 0;
    // the leading products and the others are summed apart: the roundings of the five small products are then small ones
    f32x16 acc[TM][TN], low[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;
    uint32_t tiny = 0xffffffffu;
    f32x4 cs = {0.f, 0.f, 0.f, 0.f};                         // column sums of B: the thread's four columns
    const bool do_cs = !BKC && a.colsum && bx == 0;

    operand<BM, NT, AKC, GATHER> oa;
    operand<BN, NT, BKC, false> ob;
    oa.init(a.A, a.lda, a.ridx, m0, a.M, kbeg, kend);
    ob.init(a.B, a.ldb, nullptr, n0, a.N, kbeg, kend);
    auto fetch = [&](int64_t k0) {
        oa.fetch(a.lda, k0, kend);
        ob.fetch(a.ldb, k0, kend);
        oa.indices(a.ridx, k0 + SBK, kend);
    };
    auto stage = [&](int64_t k0, unsigned char *buf) {
        if (k0 + SBK > kend || (!AKC && m0 + BM > a.M)) oa.align(k0, kend);
        if (k0 + SBK > kend || (!BKC && n0 + BN > a.N)) ob.align(k0, kend);
        oa.stage(buf, tiny);
        ob.stage(buf + 3 * PA, tiny);
        if constexpr (!BKC) {
            if (do_cs) {
#pragma unroll
                for (int f = 0; f < operand<BN, NT, BKC, false>::NF; ++f) cs += ob.reg[f];
            }
        }
    };
    // The six products of a half slice as six steps; a step's operands are read from LDS one step ahead (the barriers keep the
    // compiler from moving the reads down to their use, where each would be waited for).
    auto multiply = [&](const unsigned char *buf) {
        bf16x8 fa[3][TM], fb[3][TN];
        auto read_a = [&](int ks, int q) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[q][i] = *reinterpret_cast<const bf16x8 *>(buf + q * PA + chunk_at(plane<BM>::BLOCK, ta0 + i, li, 2 * ks + kh));
        };
        auto read_b = [&](int ks, int q) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[q][j] = *reinterpret_cast<const bf16x8 *>(buf + 3 * PA + q * PB + chunk_at(plane<BN>::BLOCK, tb0 + j, li, 2 * ks + kh));
        };
        auto step = [&](f32x16 (&c)[TM][TN], int qa, int qb) {
            __builtin_amdgcn_sched_barrier(0);
            // the blocks in turn, so that no accumulator waits for itself
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[qa][i], fb[qb][j], c[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        read_a(0, 0);
        read_b(0, 0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            read_a(ks, 1); step(acc, 0, 0);
            read_b(ks, 1); step(low, 1, 0);
            read_a(ks, 2); step(low, 0, 1);
            read_b(ks, 2); step(low, 1, 1);
            // A0 is still needed for the last step: the next half slice's is read behind it
            step(low, 2, 0);
            if (ks == 0) read_b(1, 0);
            step(low, 0, 2);
            if (ks == 0) read_a(1, 0);
        }
    };
    fetch(kbeg);
    stage(kbeg, lds);
    if (kbeg + SBK < kend) fetch(kbeg + SBK);
    __syncthreads();
    // Slice s is multiplied from one buffer while slice s + 1 is split into the other and slice s + 2 is requested.  Half of
    // the wavefronts split first and multiply then, the other half the other way round: each SIMD has one of both kinds,
    // so that its matrix pipe and its vector ALU work at the same time.
    int cur = 0;
    for (int64_t k0 = kbeg; k0 < kend; k0 += SBK, cur ^= 1) {
        unsigned char *here = lds + cur * BUF, *there = lds + (cur ^ 1) * BUF;
        const bool more = k0 + SBK < kend;
        if (wave >= WM * WN / 2) multiply(here);
        if (more) {
            stage(k0 + SBK, there);
            if (k0 + 2 * SBK < kend) fetch(k0 + 2 * SBK);
        }
        if (wave < WM * WN / 2) multiply(here);
        __syncthreads();
    }

    // does the split hold?
    if (tiny < TINY) small_seen = 1;
    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] += low[i][j][r];
                bad = fmaf(acc[i][j][r], 0.f, bad);          // NaN if any of them is not finite
            }
    __syncthreads();
    if (small_seen || __ballot(!(bad == 0.f))) {
        // once more with the fp32 instructions, operands straight from memory
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        constexpr int KU = 4;      // steps whose loads are in flight together
        for (int64_t k = kbeg; k < kend; k += 2 * KU) {
            float va[KU][TM], vb[KU][TN];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int64_t kk = k + 2 * u + kh, kc = min(kk, kend - 1);
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int64_t r = min(m0 + (BM / 32) * li + ta0 + i, a.M - 1), line = AKC ? r : kc, col = AKC ? kc : r;
                    va[u][i] = a.A[(GATHER ? (int64_t)a.ridx[line] : line) * a.lda + col];
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int64_t c = min(n0 + (BN / 32) * li + tb0 + j, a.N - 1);
                    vb[u][j] = BKC ? a.B[c * a.ldb + kc] : a.B[kc * a.ldb + c];
                }
            }
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const bool in = k + 2 * u + kh < kend;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? va[u][i] : 0.f, in ? vb[u][j] : 0.f, acc[i][j], 0, 0, 0);
            }
        }
    }

    if constexpr (!BKC) {
        if (do_cs) {          // the loop ended with a barrier and the planes are free
            // eight threads hold the same four columns
            static_assert(operand<BN, NT, BKC, false>::UNITS <= NT, "a thread keeps its columns in every slice");
            float *red = reinterpret_cast<float *>(lds);
            if ((int)threadIdx.x < BN * 2) *reinterpret_cast<f32x4 *>(red + threadIdx.x * 4) = cs;
            __syncthreads();
            if ((int)threadIdx.x < BN && n0 + threadIdx.x < a.N) {
                float t = 0.f;
                for (int q = 0; q < 8; ++q) t += red[((threadIdx.x / 4) * 8 + q) * 4 + threadIdx.x % 4];
                a.colsum[(a.partial ? (int64_t)bz * a.N : 0) + n0 + threadIdx.x] = t;
            }
        }
    }

    // The tile goes through LDS (the planes are free), so that rows leave, and the mask is read, 16 bytes a lane.
    constexpr int LDT = BN + 4, C4 = BN / 4, PASSES = BM * C4 / NT, BATCH = PASSES < 8 ? PASSES : 8;
    static_assert(BM * LDT * 4 <= 2 * BUF && NT % C4 == 0 && PASSES % BATCH == 0, "the tile fits, a thread keeps its columns");
    float *tile = reinterpret_cast<float *>(lds);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float *p = tile + ((BM / 32) * (8 * (r / 4) + 4 * kh + r % 4) + ta0 + i) * LDT + (BN / 32) * li + tb0;
#pragma unroll
            for (int j = 0; j < TN; ++j) p[j] = acc[i][j][r];
        }
    __syncthreads();
    const bool plain = a.partial != nullptr;
    float *out = plain ? a.partial + (int64_t)bz * a.M * a.N : a.C;
    const int64_t ldo = plain ? a.N : a.ldc;
    const int c0 = 4 * ((int)threadIdx.x % C4);
    const int64_t col = n0 + c0;
    if (col >= a.N) return;
    const bool whole = col + 4 <= a.N;                       // else the last one to three columns of the matrix
    float bj[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) bj[e] = (!plain && a.bias) ? a.bias[min(col + e, a.N - 1)] : 0.f;
    for (int p0 = 0; p0 < PASSES; p0 += BATCH) {
        f32x4 m[BATCH];
        if (!plain && a.mask) {
#pragma unroll
            for (int p = 0; p < BATCH; ++p) {
                const float *mp = a.mask + min(m0 + ((p0 + p) * NT + (int)threadIdx.x) / C4, a.M - 1) * a.ldm;
                if (whole) m[p] = *reinterpret_cast<const f32x4_any *>(mp + col);
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) m[p][e] = mp[min(col + e, a.N - 1)];
            }
        }
#pragma unroll
        for (int p = 0; p < BATCH; ++p) {
            const int r = ((p0 + p) * NT + (int)threadIdx.x) / C4;
            if (m0 + r >= a.M) continue;
            f32x4 z = *reinterpret_cast<const f32x4 *>(tile + r * LDT + c0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                z[e] += bj[e];
                if (!plain && a.relu) z[e] = fmaxf(z[e], 0.f);
                if (!plain && a.mask && !(m[p][e] > 0.f)) z[e] = 0.f;
            }
            float *o = out + (m0 + r) * ldo + col;
            if (whole) *reinterpret_cast<f32x4_any *>(o) = z;
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < a.N) o[e] = z[e];
        }
    }
}

template <int BM, int BN, int WM, int WN>
int launch_split(sgnn_ctx *ctx, int ta, int tb, split_args a, hipStream_t st)
{
    a.mtiles = cdiv(a.M, BM);
    a.ntiles = cdiv(a.N, BN);
    const uint64_t members = a.splits > 1 ? (uint64_t)a.mtiles * a.ntiles : a.ntiles, groups = a.splits > 1 ? a.splits : a.mtiles;
    const uint64_t nblocks = cdiv(groups, 8) * 8ull * members;
    if (nblocks > 0x7fffffffull) return sgnn_fail(ctx, SGNN_ERR_UNSUPPORTED, "sgnn_gemm: more than 2^31 tiles");
    char tag[56];
    snprintf(tag, sizeof(tag), "%c%c %dx%d %lldx%lldx%lld f32 split", ta ? 'T' : 'N', tb ? 'T' : 'N', BM, BN, (long long)a.M, (long long)a.N, (long long)a.K);
    const dim3 grid((unsigned)nblocks), block(64 * WM * WN);
    constexpr int LDS = split_lds_bytes<BM, BN>();
    const bool g = a.ridx != nullptr;
#define SGNN_SPLIT_CASE(TA_, TB_, G_)                                                                              \
    if (ta == TA_ && tb == TB_ && g == G_) {                                                                       \
        SGNN_HIP(ctx, (sgnn_allow_lds<&gemm_split_kernel<BM, BN, WM, WN, !TA_, TB_, G_>>(ctx, LDS)));                     \
        SGNN_LAUNCH(ctx, st, "gemm_split_kernel", tag, (gemm_split_kernel<BM, BN, WM, WN, !TA_, TB_, G_>), grid, block, LDS, st, a); \
        return SGNN_OK;                                                                                            \
    }
    SGNN_SPLIT_CASE(false, false, false)
    SGNN_SPLIT_CASE(false, true, false)
    SGNN_SPLIT_CASE(true, false, false)
    SGNN_SPLIT_CASE(false, false, true)
    SGNN_SPLIT_CASE(false, true, true)
    SGNN_SPLIT_CASE(true, false, true)
#undef SGNN_SPLIT_CASE
    return sgnn_fail(ctx, SGNN_ERR_UNSUPPORTED, "sgnn_gemm: trans_a and trans_b together are not implemented");
}

} // namespace

// C = act(op(A) op(B) + bias), fp32, all layouts but A^T B^T; any M, N, K with at least four elements along each contiguous
// direction (the caller has checked).
int sgnn_launch_gemm_split(sgnn_ctx *ctx, int ta, int tb, int64_t M, int64_t N, int64_t K, const float *A, int64_t lda, const int32_t *ridx,
                           const float *B, int64_t ldb, const float *bias, int relu, float *C, int64_t ldc, const float *mask, int64_t ldm,
                           float *b_colsum, ws_alloc *ws, hipStream_t st)
{
    split_args a = {};
    a.M = M; a.N = N; a.K = K; a.A = A; a.lda = lda; a.ridx = ridx; a.B = B; a.ldb = ldb; a.bias = bias; a.C = C; a.ldc = ldc;
    a.relu = relu; a.mask = mask; a.ldm = ldm; a.kps = K; a.splits = 1; a.colsum = b_colsum;
    // The widest tile of which there are enough for the 256 compute units: a 256 x 128 tile splits an element of A for 128
    // columns and one of B for 256 rows, a 64 x 64 tile each for 64.  32768 x 256 x 256, us with 256 x 128 / 128 x 128 tiles:
    // 33 / 42; 65536 x 256 x 608 133 / 168.  A^T B, whose operands both lie [reduction][rows], from 128 tiles on: 4096 x 4096 x 4096
    // 862 / 1098 (64 x 64 tiles 1805), 20000 x 200 x 300 44 / 61 (61); with 128 tiles, 2048 x 2048 x 2048, 156 / 138 (285).
    // Long reductions make up for few tiles with ranges, so A^T B takes the wide tile there as well, 256 x 256 x 32768 43 / 50, and
    // 128 x 64 from half that length on: 608 x 256 x 8000 50 us, 67 with 64 x 64, which is only better where it holds all
    // of M (40 x 256 x 50000 43 us, 52).
    const bool plain = !bias && !relu && !mask;
    const bool long_ab = !ta && plain && K >= 4096;      // A B and A B^T too, where the tiles alone do not fill the chip
    const int64_t t256 = (int64_t)cdiv(M, 256) * cdiv(N, 128), t128 = (int64_t)cdiv(M, 128) * cdiv(N, 128);
    int64_t bm = 64, bn = 64;
    if (N > 64 && (ta ? M > 128 && (K >= 8192 || t256 > 128) : t256 >= 160)) bm = 256, bn = 128;
    else if (N > 64 && (ta ? M > 64 && (K >= 8192 || t128 >= 160) : t128 >= 160)) bm = 128, bn = 128;
    else if (long_ab && M > 128) bm = N > 64 ? 256 : 128, bn = N > 64 ? 128 : 64;
    else if (!long_ab && ((int64_t)cdiv(M, 128) * cdiv(N, 64) >= 256 || (ta && M > 64 && K >= 4096))) bm = 128;
    // More tiles than compute units: the second round is a whole one however few they are, where the kernel for a tall A goes on slice by slice.  us
    // there / here, N = 256: 16384 x 256 22 / 25, 20000 x 256 37 / 28 (128 x 128 tiles up to there), 32768 x 256 32 / 33, 40000 x 256 59 / 43, 200000 x 128 127 / 91.
    if (!ta && !ridx && !mask && bn == 128 && (bm == 256 ? t256 : t128) > 256) {
        const int rc = sgnn_launch_gemm_split_tall(ctx, tb, M, N, K, A, lda, B, ldb, bias, relu, C, ldc, st);
        if (rc != SGNN_ERR_UNSUPPORTED) return rc;
    }
    // A long reduction onto few tiles is split, to at most 128 ranges of 128 steps or more (each writes its partial product, and
    // a second kernel reads them all: 256 x 256 x 32768 43 us with 128 ranges, 59 with 256; 608 x 256 x 65536 277 us with 42,
    // 205 with 128).  A B and A B^T take as many as give every compute unit a tile, a multiple of eight (the ranges are dealt to
    // the eight XCDs): 256 x 256 x 65536 67 us, 2010 unsplit; 1024 x 256 x 8416 46 with 32 ranges, 58 with 64 and 16, 263 unsplit;
    // 8192 x 256 x 8192 251 with 8, 297 with 12; 100 x 40 x 30000 24 with 128 ranges of 64 x 64 tiles, 28 with 234 of 128 x 64.
    // The number of ranges, and with it the order of the sums, depends on the shape alone wherever there is
    // scratch for them.  Where there is not, it is the number that gives each compute unit one 128-row tile, for which an A^T B of 4096
    // steps and more needs scratch, or one range otherwise: never what the scratch happens to hold.
    const int64_t tiles = (int64_t)cdiv(M, (uint64_t)bm) * cdiv(N, (uint64_t)bn);
    float *cs_partial = nullptr;
    const size_t ws_off = ws->off;
    const bool filled = ta && bn == 128 && K < 8192;     // wide tiles that were taken for their number: 20000 x 200 x 300 124 us in two ranges
    if (plain && tiles < 256 && !filled && (ta ? K >= 256 : long_ab)) {
        const int64_t tiles128 = (int64_t)cdiv(M, 128) * cdiv(N, N > 64 ? 128 : 64);
        const int64_t wanted = ta ? std::max<int64_t>(768 / tiles, 1) : (int64_t)cdiv(cdiv(256, (uint64_t)tiles), 8) * 8;
        const int64_t full = std::min<int64_t>(M * N <= 16384 ? 256 : 128, std::min<int64_t>(K / 128, wanted));
        const int64_t few = K >= 4096 ? std::min<int64_t>(full, cdiv(256, (uint64_t)tiles128)) : 1;
        const int64_t least = ta ? few : 1;
        for (int64_t want : {full, few, least}) {
            ws->off = ws_off;
            ws->ok = true;
            a.kps = (int64_t)cdiv(cdiv(K, want), SBK) * SBK;
            a.splits = cdiv(K, a.kps);
            if (a.splits <= 1) break;
            a.partial = ws->get<float>((size_t)a.splits * M * N);
            if (b_colsum) a.colsum = cs_partial = ws->get<float>((size_t)a.splits * N);
            if (ws->ok) break;
        }
        if (a.splits <= 1) {
            a.kps = K;
            a.splits = 1;
            a.partial = nullptr;
            a.colsum = b_colsum;
            cs_partial = nullptr;
        } else if (!ws->ok)
            return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_gemm: scratch too small for the split reduction: call sgnn_ctx_reserve");
    }
    int rc;
    if (bm == 256) rc = launch_split<256, 128, 4, 2>(ctx, ta, tb, a, st);
    else if (bn == 128) rc = launch_split<128, 128, 2, 4>(ctx, ta, tb, a, st);
    else if (bm == 128) rc = launch_split<128, 64, 2, 2>(ctx, ta, tb, a, st);
    else rc = launch_split<64, 64, 2, 2>(ctx, ta, tb, a, st);
    if (rc) return rc;
    if (a.splits > 1) {
        rc = sgnn_launch_splitk_reduce(ctx, a.partial, (int)a.splits, M, N, C, ldc, cs_partial, cs_partial ? b_colsum : nullptr, st);
        ws->off = ws_off;      // what the caller launches next on this stream may have the scratch
    }
    return rc;
}
