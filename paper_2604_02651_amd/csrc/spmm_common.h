// What the sparse-product kernels share: chunks of feature rows, the plan of a matrix, the epilogue of a finished row.
#pragma once
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "block_prims.h"
#include "common.h"

namespace spmm {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

template <int VEC> struct vec_t;
template <> struct vec_t<1> { typedef float type; };
template <> struct vec_t<2> { typedef f32x2 type; };
template <> struct vec_t<4> { typedef f32x4 type; };

template <int VEC> __device__ __forceinline__ void vload(float (&dst)[VEC], const float *p)
{
    if constexpr (VEC == 1) dst[0] = *p;
    else {
        typename vec_t<VEC>::type v = *reinterpret_cast<const typename vec_t<VEC>::type *>(p);
#pragma unroll
        for (int i = 0; i < VEC; ++i) dst[i] = v[i];
    }
}

// A feature row stored as bfloat16 (16-bit patterns: the upper half of an fp32): widened while it is read.
struct bf16_bits { uint16_t v; };

template <int VEC> __device__ __forceinline__ void vload(float (&dst)[VEC], const bf16_bits *p)
{
    if constexpr (VEC == 1) dst[0] = __builtin_bit_cast(float, (uint32_t)p->v << 16);
    else if constexpr (VEC == 2) {
        const uint32_t w = *reinterpret_cast<const uint32_t *>(p);
        dst[0] = __builtin_bit_cast(float, w << 16);
        dst[1] = __builtin_bit_cast(float, w & 0xffff0000u);
    } else {
        static_assert(VEC == 4, "vector width");
        const uint2 w = *reinterpret_cast<const uint2 *>(p);
        dst[0] = __builtin_bit_cast(float, w.x << 16);
        dst[1] = __builtin_bit_cast(float, w.x & 0xffff0000u);
        dst[2] = __builtin_bit_cast(float, w.y << 16);
        dst[3] = __builtin_bit_cast(float, w.y & 0xffff0000u);
    }
}

// A gathered chunk as the load instruction returns it (fp32 values, or packed bfloat16 pairs), and its i-th value.
// Widening a bfloat16 chunk right behind its load would make every gather wait for the one before it; kept raw, all
// gathers of a round are in flight together and the widening happens where the value is multiplied.
template <int VEC, typename XT> struct raw_chunk { float v[VEC]; };
template <int VEC> struct raw_chunk<VEC, bf16_bits> { uint32_t w[(VEC + 1) / 2]; };

template <int VEC> __device__ __forceinline__ void raw_load(raw_chunk<VEC, float> &r, const float *p) { vload<VEC>(r.v, p); }
template <int VEC> __device__ __forceinline__ void raw_load(raw_chunk<VEC, bf16_bits> &r, const bf16_bits *p)
{
    if constexpr (VEC == 1) r.w[0] = p->v;
    else if constexpr (VEC == 2) r.w[0] = *reinterpret_cast<const uint32_t *>(p);
    else {
        const uint2 q = *reinterpret_cast<const uint2 *>(p);
        r.w[0] = q.x; r.w[1] = q.y;
    }
}
template <int VEC> __device__ __forceinline__ float raw_get(const raw_chunk<VEC, float> &r, int i) { return r.v[i]; }
template <int VEC> __device__ __forceinline__ float raw_get(const raw_chunk<VEC, bf16_bits> &r, int i)
{
    const uint32_t w = r.w[i >> 1];
    return __builtin_bit_cast(float, (i & 1) ? (w & 0xffff0000u) : (w << 16));
}

template <int VEC> __device__ __forceinline__ void vstore(float *p, const float (&src)[VEC])
{
    if constexpr (VEC == 1) *p = src[0];
    else {
        typename vec_t<VEC>::type v;
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = src[i];
        *reinterpret_cast<typename vec_t<VEC>::type *>(p) = v;
    }
}

// A finished output row segment: fp32 as it is, or rounded to bfloat16 (nearest even) and packed.
template <int VEC> __device__ __forceinline__ void vstore_out(float *out, int64_t elem, const float (&src)[VEC], int out_bf16)
{
    if (!out_bf16) { vstore<VEC>(out + elem, src); return; }
    uint16_t *p = reinterpret_cast<uint16_t *>(out) + elem;
    uint16_t h[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) h[i] = __builtin_bit_cast(uint16_t, (__bf16)src[i]);
    if constexpr (VEC == 1) *p = h[0];
    else if constexpr (VEC == 2) *reinterpret_cast<uint32_t *>(p) = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
    else *reinterpret_cast<uint2 *>(p) = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
}

// Device-scope stores and loads (relaxed atomics, one word each): the store goes through to the
// level of the memory system that all compute dies share and the load reads from there, so data
// handed from one wavefront to another inside a kernel needs no write-back or invalidation of a
// whole cache.  p points at the lane's first word; the VEC words of a lane are 64 words apart, so
// that every store or load instruction of the wavefront covers 256 contiguous bytes.
template <int VEC> __device__ __forceinline__ void vstore_device(float *p, const float (&src)[VEC])
{
#pragma unroll
    for (int i = 0; i < VEC; ++i) __hip_atomic_store(p + i * 64, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int VEC> __device__ __forceinline__ void vload_device(float (&dst)[VEC], const float *p)
{
#pragma unroll
    for (int i = 0; i < VEC; ++i) dst[i] = __hip_atomic_load(p + i * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Row offsets are int32 (mini-batch matrices) or int64 (a full graph with 2^31 entries or more).
__device__ __forceinline__ int64_t rp_load(const void *__restrict__ rowptr, int rp64, uint64_t i)
{
    return rp64 ? static_cast<const int64_t *>(rowptr)[i] : (int64_t) static_cast<const int32_t *>(rowptr)[i];
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

constexpr int SPMM_NT = 256;       // threads of a workgroup
#ifndef SPMM_SHORT_LEN
#define SPMM_SHORT_LEN 8
#endif
constexpr int SPMM_SHORT = SPMM_SHORT_LEN;      // smallest length from which a row counts as long
constexpr int SPMM_CHUNK = 64;     // entries per piece of a long row: what one wavefront fetches at once
constexpr int SPMM_MAX_PIECES = 256;   // pieces per row: longer rows get longer pieces

// Entries per piece of a row with `len` entries: 64, doubled until the row has at most
// SPMM_MAX_PIECES pieces, so that the wavefront that adds the partial rows of a hub row up has a
// bounded number of them to read.
__host__ __device__ inline int64_t spmm_piece_len(int64_t len)
{
    int64_t c = SPMM_CHUNK;
    while (len > c * SPMM_MAX_PIECES) c *= 2;
    return c;
}
constexpr unsigned SPMM_PIECE_WAVES = 2048;
constexpr int SPMM_PLAN_NT = 1024;  // rows per workgroup of the plan kernel

// Plan of a matrix (device memory): header, first chunk number per row, chunk descriptors.
struct spmm_plan_view {
    uint32_t *n_chunks;     // header word 0
    uint32_t *part_base;    // [rows], defined for long rows only
    uint2 *desc;            // [max_chunks] (row, chunk index inside the row)
    uint32_t *ticket;       // [max_chunks], used at the first chunk number of a long row; zero between products
};

// Rows longer than this count as long: four times the mean row length of the matrix, and at least
// 1/65536 of its entries (a full graph with 10^9 entries has long rows in the hundreds that one
// wavefront walks without holding anything up; what must be cut are its hubs).  Evaluated on the
// device from the true entry count when the plan is built (header word 1 of the plan).
__host__ __device__ inline int spmm_long_len(uint32_t rows, uint64_t entries)
{
    const uint64_t mean = rows ? entries / rows : 0;
    uint64_t t = 4 * mean;
    if (t < SPMM_SHORT) t = SPMM_SHORT;
    if (t < (entries >> 16)) t = entries >> 16;      // never more than 65536 long rows, however large the matrix
    if (t > (1u << 20)) t = 1u << 20;
    return (int)t;
}

// Rows that one wavefront walks as a block: about 128 entries, at most 32 rows, and no fewer than 4096 wavefronts while
// the rows last.  Measured: 16 entries / 8 rows -> 32 / 16: 7 % faster on a 2^20-row matrix with 1.3 entries a row;
// 32 / 16 -> 128 / 32: the five products of a 2^18-row step with 6.3 entries a row 6-9 % faster each (steps/s + 3.4 %),
// those of the 2^20-row step 1-4 %, dense-degree and small mini-batches unchanged; more gathers in flight per
// wavefront, 16 instead of 8, were slower at every size.  The plan holds the figure for the true entry count (header
// word 2); the host sizes the grid with the capacity in its place, which can only give fewer rows.
#ifndef SPMM_BLOCK_ENTRIES
#define SPMM_BLOCK_ENTRIES 128
#endif
#ifndef SPMM_BLOCK_ROWS
#define SPMM_BLOCK_ROWS 32
#endif
#ifndef SPMM_U4
#define SPMM_U4 8
#endif
__host__ __device__ inline int spmm_rows_per_wave(uint32_t rows, uint64_t entries)
{
    const uint64_t mean = rows && entries >= rows ? entries / rows : 1;
    uint64_t r = SPMM_BLOCK_ENTRIES / (mean < SPMM_BLOCK_ENTRIES ? mean : SPMM_BLOCK_ENTRIES);
    if (r > SPMM_BLOCK_ROWS) r = SPMM_BLOCK_ROWS;
    if (r > rows / 4096) r = rows / 4096;
    return r < 1 ? 1 : (int)r;
}

inline uint32_t spmm_max_chunks(uint32_t rows, uint64_t capacity)
{
    // a long row has more than SPMM_SHORT entries whatever the mean is, and more than four times the
    // mean (rounded down, so at least twice the exact mean once there is an entry per row): at most
    // capacity / SPMM_SHORT of them and at most half the rows, each with at most one partly filled
    // chunk, plus the full chunks
    const uint64_t n = std::min<uint64_t>(capacity / SPMM_SHORT, (uint64_t)rows / 2 + 1) + capacity / SPMM_CHUNK + 2;
    // and no more than 65536 long rows (spmm_long_len) of at most SPMM_MAX_PIECES pieces each
    return (uint32_t)std::min<uint64_t>(n, (uint64_t)65536 * SPMM_MAX_PIECES + 2);
}

inline spmm_plan_view plan_view(void *plan, uint32_t rows, uint32_t max_chunks)
{
    uint8_t *p = static_cast<uint8_t *>(plan);
    spmm_plan_view v;
    v.n_chunks = reinterpret_cast<uint32_t *>(p);
    v.part_base = reinterpret_cast<uint32_t *>(p + 256);
    v.desc = reinterpret_cast<uint2 *>(p + 256 + (((size_t)rows * 4 + 255) & ~size_t(255)));
    v.ticket = reinterpret_cast<uint32_t *>(v.desc + max_chunks);
    return v;
}

// What happens to a finished output row: out = act(acc + bias), then (optionally) zero where the
// mask matrix is not positive - the ReLU backward of the layer below, fused into this product.
struct spmm_epi {
    const float *bias;
    int relu;
    const float *mask;
    int64_t ldm;
    const float *add;   // optional matrix added to the result last (the skip path of a residual layer)
    int64_t ldadd;
    int out_bf16;       // the result is stored as bfloat16 (rounded to nearest even; `out` then points at 16-bit elements)
    int mask_bf16;      // the mask matrix is stored as bfloat16
    // softmax cross-entropy of the finished rows (kernels instantiated with XENT; bias is the only other epilogue then)
    const int32_t *labels;      // class of every output row
    void *dO;                   // gradient rows (softmax - onehot) * inv_rows, or null
    int dO_bf16;
    int64_t lddo;
    float inv_rows;
    float *loss_partial;        // one partial sum of -log p_label per workgroup
    float *cs_partial;          // [workgroups][d] column sums of the stored gradient, or null
    int write_out;              // the logits are written to `out` as well
    // A long row is finished by whichever of its piece wavefronts comes last, so its share of the sums cannot go into
    // that wavefront's running sums (the result would depend on the race).  It is added, as 64-bit fixed-point
    // integers, to one of XENT_SLOTS rows of d + 1 counters chosen by the row number: integer addition is exact in
    // any order, and the final kernel adds the slots up and leaves zeros.  [slot][d + 1], column d holds the loss terms.
    unsigned long long *fix;
};
constexpr int XENT_SLOTS = 256;
constexpr double XENT_FIX_CS = 1152921504606846976.0;      // 2^60: a gradient entry is at most 1 in magnitude, their sum too
constexpr double XENT_FIX_LOSS = 1073741824.0;             // 2^30: loss terms are below 2^10, at most 2^20 long rows
// One term of such a sum.  What is no finite number in that range (a NaN or an infinity among the row's logits, a label whose class its
// logit takes out) has no integer: it goes into the wavefront's own sum, where a NaN or an infinity gives the same result in any order.
__device__ __forceinline__ void xent_add_fixed(unsigned long long *p, float t, double unit, float &own)
{
    if (fabsf(t) < 1048576.f) atomicAdd(p, (unsigned long long)(long long)llrint((double)t * unit));
    else own += t;
}

// per-wavefront running sums of the cross-entropy epilogue
template <int VEC, int CH> struct spmm_xent_sums {
    float loss;
    float cs[CH][VEC];
};

// Wavefront-wide sum / maximum for the row epilogue: four DPP steps make every lane of a 16-lane row hold the row's
// result (quad swaps, half mirror, mirror: register-to-register, no LDS round trips as with the shuffle built-ins, of
// which a reduction needs six in a dependent chain), four lane reads combine the rows.  The order of the additions is fixed.
template <int CTRL> __device__ __forceinline__ float dpp_f32(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
template <bool MAX> __device__ __forceinline__ float wave_reduce_rows(float x)
{
    auto op = [](float a, float b) { return MAX ? fmaxf(a, b) : a + b; };
    x = op(x, dpp_f32<0xB1>(x));      // quad_perm [1, 0, 3, 2]
    x = op(x, dpp_f32<0x4E>(x));      // quad_perm [2, 3, 0, 1]
    x = op(x, dpp_f32<0x141>(x));     // row_half_mirror
    x = op(x, dpp_f32<0x140>(x));     // row_mirror
    const int xi = __builtin_bit_cast(int, x);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 0)), r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 16)),
                r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 32)), r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 48));
    return op(op(r0, r1), op(r2, r3));
}

} // namespace spmm

// spmm_group.hip
bool sgnn_spmm_panel_wanted(const sgnn_csr *A, int64_t d, int x_bf16);
// entries a row from which on a matrix is the panel kernel's (or_short: spmm_short_kernel takes the others)
uint32_t sgnn_spmm_panel_mean(const sgnn_csr *A, int64_t d, int x_bf16, bool or_short);
int sgnn_launch_spmm_panel(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, const int32_t *row_index, int d, float *out,
                           int64_t ldo, const spmm::spmm_epi &ep, uint32_t mean_limit, ws_alloc *ws, hipStream_t st);
bool sgnn_spmm_short_wanted(const sgnn_csr *A, const int32_t *row_index, int64_t d, int x_bf16, const spmm::spmm_epi &ep);
int sgnn_spmm_short_frame(int64_t d, int x_bf16);      // columns of a partial row
int sgnn_launch_spmm_short(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, const int32_t *row_index, int d, float *out,
                           int64_t ldo, const spmm::spmm_epi &ep, uint32_t mean_limit, ws_alloc *ws, hipStream_t st);
// The product with the loss in its epilogue; ep's partial sums have a row per workgroup.  A partial row has `frame` columns, 0 for a
// width that the kernel is not built for.
int sgnn_spmm_short_xent_frame(int64_t d, int x_bf16);
unsigned sgnn_spmm_short_xent_grid(const sgnn_csr *A);
int sgnn_launch_spmm_short_xent(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, int d, float *out, int64_t ldo,
                                const spmm::spmm_epi &ep, ws_alloc *ws, hipStream_t st);
