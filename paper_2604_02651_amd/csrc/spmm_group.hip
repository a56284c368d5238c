// Sparse products by groups of lanes: the kernel for matrices with many entries a row and the one for few.
#include "spmm_common.h"

using namespace spmm;

namespace {

#include "spmm_panel.h"
#include "spmm_short.h"

} // namespace

bool sgnn_spmm_panel_wanted(const sgnn_csr *A, int64_t d, int x_bf16)
{
    return x_bf16 ? spmm_panel_wanted<bf16_bits>(A, d) : spmm_panel_wanted<float>(A, d);
}

uint32_t sgnn_spmm_panel_mean(const sgnn_csr *A, int64_t d, int x_bf16, bool or_short)
{
    return x_bf16 ? spmm_panel_mean<bf16_bits>(A, d, or_short) : spmm_panel_mean<float>(A, d, or_short);
}

int sgnn_launch_spmm_panel(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, const int32_t *row_index, int d, float *out,
                           int64_t ldo, const spmm_epi &ep, uint32_t mean_limit, ws_alloc *ws, hipStream_t st)
{
    if (x_bf16) return launch_panel(ctx, A, static_cast<const bf16_bits *>(X), ldx, row_index, d, out, ldo, ep, mean_limit, ws, st);
    return launch_panel(ctx, A, static_cast<const float *>(X), ldx, row_index, d, out, ldo, ep, mean_limit, ws, st);
}

bool sgnn_spmm_short_wanted(const sgnn_csr *A, const int32_t *row_index, int64_t d, int x_bf16, const spmm_epi &ep)
{
    return x_bf16 ? spmm_short_wanted<bf16_bits>(A, row_index, d, ep) : spmm_short_wanted<float>(A, row_index, d, ep);
}

int sgnn_spmm_short_frame(int64_t d, int x_bf16) { return x_bf16 ? spmm_short_frame<bf16_bits>(d) : spmm_short_frame<float>(d); }

int sgnn_launch_spmm_short(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, const int32_t *row_index, int d, float *out,
                           int64_t ldo, const spmm_epi &ep, uint32_t mean_limit, ws_alloc *ws, hipStream_t st)
{
    if (x_bf16) return launch_short(ctx, A, static_cast<const bf16_bits *>(X), ldx, row_index, d, out, ldo, ep, mean_limit, ws, st);
    return launch_short(ctx, A, static_cast<const float *>(X), ldx, row_index, d, out, ldo, ep, mean_limit, ws, st);
}

int sgnn_spmm_short_xent_frame(int64_t d, int x_bf16) { return x_bf16 ? xent_frame<bf16_bits>(d) : xent_frame<float>(d); }

unsigned sgnn_spmm_short_xent_grid(const sgnn_csr *A) { return spmm_short_xent_grid(A); }

int sgnn_launch_spmm_short_xent(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, int d, float *out, int64_t ldo,
                                const spmm_epi &ep, ws_alloc *ws, hipStream_t st)
{
    if (x_bf16) return launch_short_xent(ctx, A, static_cast<const bf16_bits *>(X), ldx, d, out, ldo, ep, ws, st);
    return launch_short_xent(ctx, A, static_cast<const float *>(X), ldx, d, out, ldo, ep, ws, st);
}
