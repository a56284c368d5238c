// Sparse aggregation of the GCN layer (Sec. III-B Eq. 5 and the transposed SpMM of Sec. III-C):
// out = A X with A in CSR.
//
// Row-split with a side path for long rows.  A wavefront owns a block of consecutive output rows
// and walks their entries as one stream: the CSR entries of the block are contiguous, so they are
// fetched 64 at a time with one coalesced load, and several gathered feature rows are in flight
// however short the rows are.  The 64 lanes cover the columns (VEC*CH of them per lane), so every
// feature row is read with coalesced vector loads and every output row is written once.  Rows
// much longer than the mean (power-law graphs have them) would leave one wavefront walking
// alone long after the others are done, so a plan built once per matrix cuts them into pieces of
// 64 entries (longer pieces for hub rows, so that no row has more than 256 of them):
//   spmm_plan_kernel    (once per matrix) piece descriptors of the long rows, one ticket per long row
//   spmm_main_kernel    the first wavefronts take pieces (one partial row per piece), the others take
//                       blocks of rows; both kinds run side by side.  A piece wavefront that has
//                       stored its partial row draws a ticket of its row; the one that draws the last
//                       ticket adds the partial rows of the row up, in piece order, and writes the row.
// Most products take one of two other kernels (spmm_group.hip), whose groups of lanes gather several rows of X by one instruction:
// spmm_short_kernel, or spmm_panel_kernel for matrices with many entries a row.  The main kernel has the rest: three column panels
// and more of few entries a row, fewer columns than 16 bytes, several epilogues at once, and the loss in the epilogue where
// the row is wider than one panel.
// No atomics touch floating-point data and the order of every sum is fixed: results are
// bit-reproducible.  Nothing waits on another wavefront.  Two products that use the same plan must
// not run at the same time (they would share the tickets).
#include "spmm_common.h"

using namespace spmm;

namespace {

__global__ void spmm_plan_clear_kernel(uint32_t *n_chunks) { *n_chunks = 0; }

// One thread per row: the long rows of a workgroup reserve their chunk numbers with one atomic add and
// record their first one in part_base[row].  The (row, chunk) descriptors are then written by all threads in turn, each finding the row of
// a chunk by a search over the rows' first ones in LDS: a hub row has up to 256 of them, and written by its own thread they
// were most of the kernel (2^18 rows of 6.4 entries, one row of 8000: 13 us).  The chunk numbering depends on timing; the values
// computed from it do not.
__global__ __launch_bounds__(SPMM_PLAN_NT) void spmm_plan_kernel(uint32_t rows, const void *__restrict__ rowptr, int rp64, uint64_t capacity,
                                                        uint32_t *__restrict__ n_chunks,
                                                        uint32_t max_chunks, uint32_t *__restrict__ part_base,
                                                        uint2 *__restrict__ desc, uint32_t *__restrict__ ticket)
{
    __shared__ uint32_t scan_lds[SPMM_PLAN_NT / 64 + 1];
    __shared__ uint32_t wg_base, first[SPMM_PLAN_NT];
    const uint32_t row = blockIdx.x * SPMM_PLAN_NT + threadIdx.x;
    // the row's offsets are requested together with the count of entries, which the length of a long row depends on
    const uint64_t r0 = min(row, rows - 1);
    const int64_t end = rp_load(rowptr, rp64, rows), e0 = rp_load(rowptr, rp64, r0), e1 = rp_load(rowptr, rp64, r0 + 1);
    const uint64_t entries = min((uint64_t)end, capacity);
    const int long_len = spmm_long_len(rows, entries);
    if (row == 0) {
        n_chunks[1] = (uint32_t)long_len;
        n_chunks[2] = (uint32_t)spmm_rows_per_wave(rows, entries);
        n_chunks[3] = (uint32_t)min(entries / rows, (uint64_t)0xffffffffu);
    }
    int64_t len = 0;
    if (row < rows) len = min(e1, (int64_t)capacity) - min(e0, (int64_t)capacity);
    const int64_t plen = spmm_piece_len(len);
    const uint32_t nch = len > long_len ? (uint32_t)((len + plen - 1) >> (63 - __clzll(plen))) : 0u;   // plen is a power of two
    // one atomic per workgroup of 1024 rows (atomics on one address cost about 10 ns each, whoever issues
    // them): the long rows of the workgroup take consecutive piece numbers
    uint32_t wg_total;
    const uint32_t excl = block_excl_scan<uint32_t, SPMM_PLAN_NT>(nch, &wg_total, scan_lds);
    if (wg_total == 0) return;
    if (threadIdx.x == 0) wg_base = atomicAdd(n_chunks, wg_total);
    first[threadIdx.x] = excl;
    __syncthreads();
    if (nch) part_base[row] = wg_base + excl;
    for (uint32_t p = threadIdx.x; p < wg_total && wg_base + p < max_chunks; p += SPMM_PLAN_NT) {
        uint32_t t = 0;                // the last row whose first chunk is p or one before (rows without chunks have their successor's)
#pragma unroll
        for (uint32_t step = SPMM_PLAN_NT / 2; step; step /= 2)
            if (first[t + step] <= p) t += step;
        desc[wg_base + p] = make_uint2(blockIdx.x * SPMM_PLAN_NT + t, p - first[t]);
        ticket[wg_base + p] = 0;       // the first one of a row is its ticket, the panel kernel has one per panel
    }
}

// Cross-entropy of one finished row of logits v (bias already added), held by the wavefront as chunk (m, lane) =
// columns (m * 64 + lane) * VEC ..: the row's softmax from one maximum and one sum across the wavefront, the
// gradient row written where the logits would be read back from otherwise.  Probabilities are exp(x - max) / sum,
// as in the stand-alone loss kernel.  A label outside [0, d) contributes the log-sum-exp alone.
template <int VEC, int CH, bool SHARED_ROW = false>
__device__ __forceinline__ void spmm_row_xent(const float (&v)[CH][VEC], const spmm_epi &ep, int64_t row, int32_t y, int d, int lane,
                                              spmm_xent_sums<VEC, CH> &xs)
{
    unsigned long long *fix = SHARED_ROW ? ep.fix + (uint64_t)(row % XENT_SLOTS) * (uint64_t)(d + 1) : nullptr;
    auto add_loss = [&](float t) {
        if constexpr (SHARED_ROW) xent_add_fixed(fix + d, t, XENT_FIX_LOSS, xs.loss);
        else xs.loss += t;
    };
    // d is a multiple of VEC (the launcher's condition for this instantiation): a lane's VEC columns of a chunk are
    // inside the row or outside it together
    float mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < CH; ++m)
        if ((m * 64 + lane) * VEC < d) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) mx = fmaxf(mx, v[m][i]);
        }
    mx = wave_reduce_rows<true>(mx);
    float e[CH][VEC], s = 0.f;
#pragma unroll
    for (int m = 0; m < CH; ++m) {
        const bool in = (m * 64 + lane) * VEC < d;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            e[m][i] = in ? exp_neg(v[m][i] - mx) : 0.f;
            s += e[m][i];
        }
    }
    s = wave_reduce_rows<false>(s);
    const float inv = __builtin_amdgcn_rcpf(s), lse = log_ge1(s);       // 1 ulp each
    if ((uint32_t)y >= (uint32_t)d && lane == 0) add_loss(mx + lse);
#pragma unroll
    for (int m = 0; m < CH; ++m) {
        const int col = (m * 64 + lane) * VEC;
        if (col < d) {
            // the label's column, if it is one of this lane's: one test and one loss term per chunk, not one per column
            const uint32_t rel = (uint32_t)(y - col);
            if (rel < (uint32_t)VEC) {
                float vy = v[m][0];
#pragma unroll
                for (int i = 1; i < VEC; ++i) vy = rel == (uint32_t)i ? v[m][i] : vy;
                add_loss(lse - (vy - mx));
            }
            float g[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                const bool hit = rel == (uint32_t)i;
                g[i] = (e[m][i] * inv - (hit ? 1.f : 0.f)) * ep.inv_rows;
                if (ep.dO_bf16) g[i] = (float)(__bf16)g[i];       // the column sums add what is stored
                if constexpr (SHARED_ROW) {
                    if (ep.cs_partial) xent_add_fixed(fix + col + i, g[i], XENT_FIX_CS, xs.cs[m][i]);
                } else xs.cs[m][i] += g[i];
            }
            if (ep.dO) vstore_out<VEC>(static_cast<float *>(ep.dO), row * ep.lddo + col, g, ep.dO_bf16);
        }
    }
}

// bias: the lane's VEC bias values (zeros without a bias), loaded once per wavefront: a lane's columns never change,
// and a load of them in front of every row's store cost a third of the kernel on a 2^20-row matrix
template <int VEC>
__device__ __forceinline__ void spmm_epilogue(float (&v)[VEC], const spmm_epi &ep, int64_t row, int col, const float (&bias)[VEC])
{
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        v[i] += bias[i];
        if (ep.relu) v[i] = fmaxf(v[i], 0.f);
    }
    if (ep.mask) {
        float m[VEC];
        if (ep.mask_bf16) vload<VEC>(m, reinterpret_cast<const bf16_bits *>(ep.mask) + row * ep.ldm + col);
        else vload<VEC>(m, ep.mask + row * ep.ldm + col);
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = m[i] > 0.f ? v[i] : 0.f;
    }
    if (ep.add) {
        float a[VEC];
        vload<VEC>(a, ep.add + row * ep.ldadd + col);
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] += a[i];
    }
}

// One wavefront walks `rows_per_wave` consecutive rows as one stream of entries.  The entries of
// consecutive rows are contiguous in the CSR arrays, so 64 of them are fetched with one coalesced
// load (lane l keeps entry e + l) and handed out by lane index; U gathered feature rows are in
// flight at a time whatever the lengths of the rows, the 64 lanes covering the columns.  Every
// value that steers the walk (row number, row bounds, entry number) is the same in all lanes.
// A row longer than long_len is left out: its chunks and the fix-up write it.
template <int VEC, int CH, typename XT, bool XENT>
__device__ __forceinline__ void spmm_wave_rows(uint32_t rows, const void *__restrict__ rowptr, int rp64,
                                               const int32_t *__restrict__ colidx, const float *__restrict__ val,
                                               uint64_t capacity, const XT *__restrict__ X, int64_t ldx,
                                               const int32_t *__restrict__ row_index, int d, uint64_t wave, int rows_per_wave,
                                               int long_len, float *__restrict__ out, int64_t ldo,
                                               const spmm_epi &ep, const float (&bias)[CH][VEC], spmm_xent_sums<VEC, CH> &xs)
{
    constexpr int U = CH * VEC <= 4 ? SPMM_U4 : (CH * VEC <= 8 ? 4 : 2);
    const int lane = threadIdx.x & 63;
    const uint64_t r0 = wave * (uint64_t)rows_per_wave;
    if (r0 >= rows) return;
    const int nr = (int)min((uint64_t)rows_per_wave, rows - r0);
    // lane k: start of row r0 + k, as an offset from the start of the block's first row (a block of
    // rows holds far fewer than 2^31 entries, so everything behind this line is 32-bit)
    int64_t rpl = 0;
    if (lane <= nr) rpl = min(rp_load(rowptr, rp64, r0 + lane), (int64_t)min(capacity, (uint64_t)0x7fffffffffffffffull));
    const int64_t block_base = readlane64(rpl, 0);
    const int32_t rp = lane <= nr ? (int32_t)(rpl - block_base) : 0;
    int32_t ylane = 0;      // XENT: lane k holds the label of row r0 + k
    if constexpr (XENT) ylane = lane < nr ? ep.labels[r0 + lane] : 0;
    colidx += block_base;
    val += block_base;
    const int e_end = __builtin_amdgcn_readlane(rp, nr);
    int e = __builtin_amdgcn_readlane(rp, 0);
    int row = 0, row_end = __builtin_amdgcn_readlane(rp, 1);
    bool row_long = row_end - e > long_len;
    float acc[CH][VEC];
#pragma unroll
    for (int m = 0; m < CH; ++m)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[m][i] = 0.f;

    // the current row is complete: write it (unless it is a long one) and move to the next
    auto next_row = [&]() {
        if (!row_long) {
            const int64_t o = (int64_t)(r0 + row) * ldo;
            if constexpr (XENT) {
#pragma unroll
                for (int m = 0; m < CH; ++m)
#pragma unroll
                    for (int i = 0; i < VEC; ++i) acc[m][i] += bias[m][i];
                spmm_row_xent<VEC, CH>(acc, ep, (int64_t)(r0 + row), __builtin_amdgcn_readlane(ylane, __builtin_amdgcn_readfirstlane(row)),
                                       d, lane, xs);
            }
#pragma unroll
            for (int m = 0; m < CH; ++m) {
                const int col = (m * 64 + lane) * VEC;
                if (col < d) {
                    if constexpr (XENT) {
                        if (ep.write_out) vstore_out<VEC>(out, o + col, acc[m], 0);
                    } else {
                        spmm_epilogue<VEC>(acc[m], ep, (int64_t)(r0 + row), col, bias[m]);
                        vstore_out<VEC>(out, o + col, acc[m], ep.out_bf16);
                    }
                }
            }
        }
#pragma unroll
        for (int m = 0; m < CH; ++m)
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[m][i] = 0.f;
        ++row;
        if (row < nr) {
            const int rs = row_end;
            row_end = __builtin_amdgcn_readlane(rp, __builtin_amdgcn_readfirstlane(row + 1));
            row_long = row_end - rs > long_len;
        }
    };

    for (;;) {
        while (row < nr && (e >= row_end || row_long)) {
            if (row_long) e = max(e, row_end);
            next_row();
        }
        if (row >= nr) break;
        // e is an entry of a row this wavefront sums: fetch up to 64 entries from there
        const int n = min(64, e_end - e);
        int32_t src = 0;
        float a = 0.f;
        if (lane < n) {
            const int32_t c = colidx[e + lane];
            a = val[e + lane];
            src = row_index ? row_index[c] : c;
        }
        int used = n;
        for (int j0 = 0; j0 < n && used == n; j0 += U) {
            raw_chunk<VEC, XT> v[U][CH];
            float av[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int jj = __builtin_amdgcn_readfirstlane(min(j0 + t, n - 1));
                const XT *x = X + (int64_t)__builtin_amdgcn_readlane(src, jj) * ldx;
                av[t] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), jj));
#pragma unroll
                for (int m = 0; m < CH; ++m) {
                    const int col = (m * 64 + lane) * VEC;
                    if (col < d) raw_load<VEC>(v[t][m], x + col);
                }
            }
#pragma unroll
            for (int t = 0; t < U; ++t) {
                if (j0 + t < n && used == n) {
                    const int ee = e + j0 + t;
                    while (ee >= row_end) next_row();     // ee < e_end: a later row of this block holds it
                    if (row_long) used = j0 + t;          // stop in front of the long row
                    else {
#pragma unroll
                        for (int m = 0; m < CH; ++m) {
                            const int col = (m * 64 + lane) * VEC;
                            if (col < d) {
#pragma unroll
                                for (int i = 0; i < VEC; ++i) acc[m][i] = fmaf(av[t], raw_get<VEC>(v[t][m], i), acc[m][i]);
                            }
                        }
                    }
                }
            }
        }
        e += used;
    }
}

// acc += sum over the n <= 64 entries starting at e, which lane l < n holds as (src, a): U feature
// rows in flight at a time, handed out by lane index.  keep(j) tells whether entry j still counts
// and may move the caller's row state; it is called in entry order.
template <int VEC, int CH, int U, typename XT, typename Keep>
__device__ __forceinline__ void spmm_wave_entries(float (&acc)[CH][VEC], int32_t src, float a, int n, const XT *__restrict__ X,
                                                  int64_t ldx, int d, int lane, Keep keep)
{
    bool go = true;
    for (int j0 = 0; j0 < n && go; j0 += U) {
        raw_chunk<VEC, XT> v[U][CH];
        float av[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int jj = __builtin_amdgcn_readfirstlane(min(j0 + t, n - 1));
            const XT *x = X + (int64_t)__builtin_amdgcn_readlane(src, jj) * ldx;
            av[t] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), jj));
#pragma unroll
            for (int m = 0; m < CH; ++m) {
                const int col = (m * 64 + lane) * VEC;
                if (col < d) raw_load<VEC>(v[t][m], x + col);
            }
        }
#pragma unroll
        for (int t = 0; t < U; ++t) {
            if (j0 + t < n && go) {
                go = keep(j0 + t);
                if (go) {
#pragma unroll
                    for (int m = 0; m < CH; ++m) {
                        const int col = (m * 64 + lane) * VEC;
                        if (col < d) {
#pragma unroll
                            for (int i = 0; i < VEC; ++i) acc[m][i] = fmaf(av[t], raw_get<VEC>(v[t][m], i), acc[m][i]);
                        }
                    }
                }
            }
        }
    }
}

template <int VEC, int CH> struct spmm_unroll { static constexpr int U = CH * VEC <= 1 ? 16 : (CH * VEC <= 4 ? 8 : (CH * VEC <= 8 ? 4 : 2)); };

// Wavefronts [0, n_piece_waves) take pieces of long rows (grid-stride over the pieces the plan
// lists) and write one partial row per piece; the others take blocks of rows_per_wave rows.
// A long row is finished by whichever of its piece wavefronts stores its partial row last: the
// partial row is written with device-scope stores, the wavefront waits for them to complete and
// draws a ticket of the row, and the holder of the last ticket reads all partial rows back with
// device-scope loads and adds them up in piece order - the same sum whoever does it.  That wavefront also puts the ticket counter
// back to zero for the next product with this plan.
template <int VEC, int CH, typename XT, bool XENT = false>
__global__ __launch_bounds__(SPMM_NT) void spmm_main_kernel(uint32_t rows, const void *__restrict__ rowptr, int rp64,
                                                            const int32_t *__restrict__ colidx,
                                                            const float *__restrict__ val, uint64_t capacity,
                                                            const XT *__restrict__ X, int64_t ldx,
                                                            const int32_t *__restrict__ row_index, int d,
                                                            unsigned n_piece_waves, const uint32_t *__restrict__ n_chunks,
                                                            uint32_t max_chunks, const uint2 *__restrict__ desc,
                                                            uint32_t *__restrict__ ticket, float *part, float *__restrict__ out,
                                                            int64_t ldo, spmm_epi ep, int rows_per_wave, uint32_t mean_limit)
{
    if (mean_limit && n_chunks[3] >= mean_limit) return;        // the panel kernel's matrix
    constexpr int U = spmm_unroll<VEC, CH>::U;
    const int lane = threadIdx.x & 63;
    const uint32_t wave = blockIdx.x * (uint32_t)(SPMM_NT / 64) + (threadIdx.x >> 6);
    float bias[CH][VEC];
#pragma unroll
    for (int m = 0; m < CH; ++m)
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const int col = (m * 64 + lane) * VEC + i;
            bias[m][i] = (ep.bias && col < d) ? ep.bias[col] : 0.f;
        }
    const int64_t cap = (int64_t)min(capacity, (uint64_t)0x7fffffffffffffffull);
    spmm_xent_sums<VEC, CH> xs;
    xs.loss = 0.f;
#pragma unroll
    for (int m = 0; m < CH; ++m)
#pragma unroll
        for (int i = 0; i < VEC; ++i) xs.cs[m][i] = 0.f;
    // a finished row held as sum (bias not yet added): written, or with XENT turned into its loss and gradient row
    auto finish = [&](float (&sum)[CH][VEC], int64_t row, auto shared_row) {
        const int64_t orow = row * ldo;
        if constexpr (XENT) {
#pragma unroll
            for (int m = 0; m < CH; ++m)
#pragma unroll
                for (int i = 0; i < VEC; ++i) sum[m][i] += bias[m][i];
            spmm_row_xent<VEC, CH, decltype(shared_row)::value>(sum, ep, row, ep.labels[row], d, lane, xs);
        }
#pragma unroll
        for (int m = 0; m < CH; ++m) {
            const int col = (m * 64 + lane) * VEC;
            if (col < d) {
                if constexpr (XENT) {
                    if (ep.write_out) vstore_out<VEC>(out, orow + col, sum[m], 0);
                } else {
                    spmm_epilogue<VEC>(sum[m], ep, row, col, bias[m]);
                    vstore_out<VEC>(out, orow + col, sum[m], ep.out_bf16);
                }
            }
        }
    };
    if (wave < n_piece_waves) {
        const uint32_t total = min(*n_chunks, max_chunks);
        constexpr int PSTRIDE = CH * VEC * 64;
        // The partial row of a piece goes out with device-scope stores; once they have completed it is
        // visible to every wavefront of the device, and only then may the ticket be drawn.  Neither wait
        // is taken on the spot: the stores of piece k are waited for, and its ticket drawn, after piece
        // k+1 has been summed, and the number drawn is looked at after piece k+2 (the gathers of the
        // pieces in between hide both latencies).  `owed`: stored, ticket not drawn; `drawn`: ticket
        // requested, number not looked at yet.
        uint32_t owed_first = 0, owed_nch = 0, owed_row = 0;
        uint32_t drawn_first = 0, drawn_nch = 0, drawn_row = 0, drawn_t = 0;
        bool owed = false, drawn = false;
        auto draw_ticket = [&]() {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            drawn_t = 0;
            if (lane == 0) drawn_t = atomicAdd(&ticket[owed_first], 1u);
            drawn_first = owed_first; drawn_nch = owed_nch; drawn_row = owed_row;
            drawn = true; owed = false;
        };
        auto finish_row = [&]() {
            drawn = false;
            const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)drawn_t);
            if (t + 1 != drawn_nch) return;
            // last ticket: all partial rows of the row are complete; they are read with device-scope loads
            float sum[CH][VEC];
#pragma unroll
            for (int m = 0; m < CH; ++m)
#pragma unroll
                for (int i = 0; i < VEC; ++i) sum[m][i] = 0.f;
            const float *pr = part + (int64_t)drawn_first * PSTRIDE + lane;
            uint32_t c = 0;
            for (; c + U <= drawn_nch; c += U) {
                float v[U][CH][VEC];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int m = 0; m < CH; ++m) {
                        const int col = (m * 64 + lane) * VEC;
                        if (col < d) vload_device<VEC>(v[u][m], pr + (int64_t)(c + u) * PSTRIDE + m * VEC * 64);
                    }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int m = 0; m < CH; ++m) {
                        const int col = (m * 64 + lane) * VEC;
                        if (col < d) {
#pragma unroll
                            for (int i = 0; i < VEC; ++i) sum[m][i] += v[u][m][i];
                        }
                    }
            }
            for (; c < drawn_nch; ++c) {
#pragma unroll
                for (int m = 0; m < CH; ++m) {
                    const int col = (m * 64 + lane) * VEC;
                    if (col < d) {
                        float v[VEC];
                        vload_device<VEC>(v, pr + (int64_t)c * PSTRIDE + m * VEC * 64);
#pragma unroll
                        for (int i = 0; i < VEC; ++i) sum[m][i] += v[i];
                    }
                }
            }
            finish(sum, (int64_t)drawn_row, std::true_type{});      // finished by whoever came last: sums through the slots
            if (lane == 0) ticket[drawn_first] = 0;
        };
        for (uint32_t pc = wave; pc < total; pc += n_piece_waves) {
            const uint2 rc = desc[pc];
            const int64_t re = min(rp_load(rowptr, rp64, (uint64_t)rc.x + 1), cap);
            const int64_t rs = min(rp_load(rowptr, rp64, rc.x), re);
            const int64_t plen = spmm_piece_len(re - rs);
            const int64_t c0 = rs + (int64_t)rc.y * plen;
            const int64_t c1 = min(re, c0 + plen);
            float acc[CH][VEC];
#pragma unroll
            for (int m = 0; m < CH; ++m)
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[m][i] = 0.f;
            for (int64_t cb = c0; cb < c1; cb += SPMM_CHUNK) {      // 64 entries at a time
                const int n = (int)min(c1 - cb, (int64_t)SPMM_CHUNK);
                int32_t src = 0;
                float a = 0.f;
                if (lane < n) {
                    const int32_t c = colidx[cb + lane];
                    a = val[cb + lane];
                    src = row_index ? row_index[c] : c;
                }
                spmm_wave_entries<VEC, CH, U, XT>(acc, src, a, n, X, ldx, d, lane, [](int) { return true; });
            }
            if (re - rs <= plen) {
                // the row's only piece: it is the row, written as the row-block wavefronts write theirs
                // With the loss epilogue its sums go the way of the rows shared between wavefronts (integer adds): the
                // numbering of the pieces depends on the timing of the plan kernel, so which wavefront gets this row does
                // too, and a float sum per wavefront would not come out the same bits twice.
                finish(acc, (int64_t)rc.x, std::integral_constant<bool, XENT>{});
                continue;
            }
            if (drawn) finish_row();
            if (owed) draw_ticket();
            // a partial row holds the words of the wavefront's registers in register order: word (m, i)
            // of lane l at (m * VEC + i) * 64 + l
            float *o = part + (int64_t)pc * PSTRIDE + lane;
#pragma unroll
            for (int m = 0; m < CH; ++m) {
                const int col = (m * 64 + lane) * VEC;
                if (col < d) vstore_device<VEC>(o + m * VEC * 64, acc[m]);
            }
            // pieces of this row that exist (the list may have been cut short at max_chunks)
            owed_first = pc - rc.y;
            owed_nch = min((uint32_t)((re - rs + plen - 1) / plen), total - owed_first);
            owed_row = rc.x;
            owed = true;
        }
        if (drawn) finish_row();
        if (owed) { draw_ticket(); finish_row(); }
    } else {
        // blocks of rows, grid-stride: the grid is capped (a launch holds fewer than 2^32 threads), a full graph
        // of 10^8 rows has more blocks than that
        const int rpw = n_chunks ? (int)n_chunks[2] : rows_per_wave;
        const int long_len = n_chunks ? (int)n_chunks[1] : 0x7fffffff;
        const uint64_t n_row_waves = (uint64_t)gridDim.x * (SPMM_NT / 64) - n_piece_waves;
        for (uint64_t w = wave - n_piece_waves; w * (uint64_t)rpw < rows; w += n_row_waves)
            spmm_wave_rows<VEC, CH, XT, XENT>(rows, rowptr, rp64, colidx, val, capacity, X, ldx, row_index, d, w, rpw, long_len, out,
                                              ldo, ep, bias, xs);
    }
    if constexpr (XENT) {
        // every wavefront of the workgroup arrives here (a workgroup is all pieces or all row blocks): its sums are
        // added in a fixed order and leave as the workgroup's partial loss and partial column sums
        __shared__ float xl[SPMM_NT / 64];
        __shared__ float xc[SPMM_NT / 64][CH * VEC * 64];
        const int wv = threadIdx.x >> 6;
        const float l = wave_sum(xs.loss);
        if (lane == 0) xl[wv] = l;
#pragma unroll
        for (int m = 0; m < CH; ++m)
#pragma unroll
            for (int i = 0; i < VEC; ++i) xc[wv][(m * VEC + i) * 64 + lane] = xs.cs[m][i];
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int w = 0; w < SPMM_NT / 64; ++w) t += xl[w];
            ep.loss_partial[blockIdx.x] = t;
        }
        if (ep.cs_partial) {
            for (int idx = threadIdx.x; idx < CH * VEC * 64; idx += SPMM_NT) {
                const int l2 = idx & 63, mi = idx >> 6, m = mi / VEC, i = mi % VEC;
                const int col = (m * 64 + l2) * VEC + i;
                if (col < d) {
                    float t = 0.f;
                    for (int w = 0; w < SPMM_NT / 64; ++w) t += xc[w][idx];
                    ep.cs_partial[(int64_t)blockIdx.x * d + col] = t;
                }
            }
        }
    }
}

// The slots of the loss's integer sums: in the context's persistent area, zero between calls (xent_final_kernel sees to it)
static_assert(SGNN_PERSIST_XENT_BYTES == XENT_SLOTS * 513 * sizeof(unsigned long long), "slots of up to 512 columns");
int xent_slots(sgnn_ctx *ctx, unsigned long long **fix, hipStream_t st)
{
    *fix = reinterpret_cast<unsigned long long *>(ctx->persist + SGNN_PERSIST_XENT_OFF);
    return sgnn_zero_open(ctx, SGNN_ZERO_XENT, *fix, SGNN_PERSIST_XENT_BYTES, st);
}

// rc: of the launch of the product
int xent_final(sgnn_ctx *ctx, int rc, const spmm_epi &ep, unsigned grid, int d, float *loss, float *colsum, hipStream_t st)
{
    if (rc == SGNN_OK)
        rc = sgnn_launch_xent_final(ctx, ep.loss_partial, (int)grid, ep.inv_rows, loss, ep.cs_partial, d, colsum, ep.fix, XENT_SLOTS,
                                    1.0 / XENT_FIX_CS, 1.0 / XENT_FIX_LOSS, st);
    return sgnn_zero_close(ctx, rc, SGNN_ZERO_XENT, ep.fix, SGNN_PERSIST_XENT_BYTES, st);
}

int build_plan(sgnn_ctx *ctx, const sgnn_csr *A, void *plan, bool cleared, hipStream_t st)
{
    const uint32_t max_chunks = spmm_max_chunks(A->rows, A->capacity);
    const spmm_plan_view pv = plan_view(plan, A->rows, max_chunks);
    if (!cleared)
        SGNN_LAUNCH(ctx, st, "spmm_plan_clear_kernel", SGNN_TAG, spmm_plan_clear_kernel, dim3(1), dim3(1), 0, st, pv.n_chunks);
    SGNN_LAUNCH(ctx, st, "spmm_plan_kernel", SGNN_TAG, spmm_plan_kernel, dim3(cdiv(A->rows, SPMM_PLAN_NT)), dim3(SPMM_PLAN_NT), 0, st, A->rows,
                A->rowptr, A->rowptr_is_i64, A->capacity, pv.n_chunks, max_chunks, pv.part_base, pv.desc, pv.ticket);
    return SGNN_OK;
}


// XENT: the cross-entropy epilogue; loss_out / colsum_out receive the mean loss and the column sums of the gradient
template <int VEC, int CH, typename XT, bool XENT = false>
int launch_vc(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, const int32_t *row_index, int d, float *out,
              int64_t ldo, const spmm_epi &ep_in, ws_alloc *ws, hipStream_t st, float *loss_out = nullptr, float *colsum_out = nullptr,
              uint32_t mean_limit = 0)
{
    spmm_epi ep = ep_in;
    const int rows_per_wave = spmm_rows_per_wave(A->rows, A->capacity);   // lower bound of the plan's figure
    const unsigned rows_per_block = (unsigned)(SPMM_NT / 64) * (unsigned)rows_per_wave;
    char tag[56];
    if (XENT)
        snprintf(tag, sizeof(tag), "%ux%u d=%d <%d,%d> in=%d out=%d xent dO=%d", A->rows, A->cols, d, VEC, CH, (int)sizeof(XT),
                 ep.write_out ? 4 : 0, ep.dO ? (ep.dO_bf16 ? 2 : 4) : 0);
    else
        snprintf(tag, sizeof(tag), "%ux%u d=%d <%d,%d> in=%d out=%d%s", A->rows, A->cols, d, VEC, CH, (int)sizeof(XT), ep.out_bf16 ? 2 : 4,
                 ep.mask ? (ep.mask_bf16 ? " m=2" : " m=4") : "");
    const bool may_have_long = A->capacity > (uint64_t)SPMM_SHORT;
    spmm_plan_view pv = {nullptr, nullptr, nullptr, nullptr};
    float *part = nullptr;
    uint32_t max_chunks = 0;
    unsigned n_piece_waves = 0;
    if (may_have_long) {
        max_chunks = spmm_max_chunks(A->rows, A->capacity);
        void *plan = A->plan;
        if (!plan) {   // no plan attached to the matrix: build one for this call
            plan = ws->get<uint8_t>(sgnn_csr_plan_bytes(A->rows, A->capacity));
            if (!ws->ok)
                return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm: scratch too small (%zu bytes needed): call sgnn_ctx_reserve",
                                 ws->off);
            int rc = build_plan(ctx, A, plan, false, st);
            if (rc) return rc;
        }
        pv = plan_view(plan, A->rows, max_chunks);
        part = ws->get<float>((size_t)max_chunks * (CH * VEC * 64));
        if (!ws->ok)
            return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm: scratch too small (%zu bytes needed): call sgnn_ctx_reserve",
                             ws->off);
        // wavefronts that take pieces: 2048, more for matrices with many entries (about 32 pieces of 64 entries
        // each if every entry sat in a long row); those that find no piece leave at once
        const uint64_t want = std::min<uint64_t>(std::max<uint64_t>(A->capacity / 2048, SPMM_PIECE_WAVES), 65536);
        n_piece_waves = cdiv(std::min<uint64_t>(max_chunks, want), SPMM_NT / 64) * (SPMM_NT / 64);
    }
    // The host sizes the grid from the capacity (the entry count is on the device), which for a sparse mini-batch is many
    // times the true count: most of the workgroups of such a launch would find no block of rows and leave at once, and
    // dispatching a quarter of a million of them cost a third of the kernel's time.  16384 workgroups fill the machine
    // several times over; the wavefronts stride over whatever is left.
    // (with the cross-entropy epilogue every workgroup leaves a row of partial sums for the final kernel: a quarter of that)
    const unsigned row_blocks = std::min<unsigned>(cdiv(A->rows, rows_per_block), XENT ? 4096u : 16384u);
    const unsigned grid = n_piece_waves / (SPMM_NT / 64) + row_blocks;
    if (XENT) {
        ep.loss_partial = ws->get<float>(grid);
        ep.cs_partial = colsum_out ? ws->get<float>((size_t)grid * d) : nullptr;
        if (!ws->ok)
            return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm_xent: scratch too small (%zu bytes needed): call sgnn_ctx_reserve", ws->off);
        const int rc = xent_slots(ctx, &ep.fix, st);
        if (rc) return rc;
    }
    auto product = [&]() -> int {
        SGNN_LAUNCH(ctx, st, "spmm_main_kernel", tag, (spmm_main_kernel<VEC, CH, XT, XENT>), dim3(grid),
                    dim3(SPMM_NT), 0, st, A->rows, A->rowptr, A->rowptr_is_i64, A->colidx, A->val, A->capacity, X, ldx, row_index, d,
                    n_piece_waves, pv.n_chunks, max_chunks, pv.desc, pv.ticket, part, out, ldo, ep, rows_per_wave, mean_limit);
        return SGNN_OK;
    };
    const int rc = product();
    return XENT ? xent_final(ctx, rc, ep, grid, d, loss_out, colsum_out, st) : rc;
}

template <int VEC, typename XT>
int launch_v(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, const int32_t *row_index, int d, float *out,
             int64_t ldo, const spmm_epi &ep, ws_alloc *ws, hipStream_t st, uint32_t mean_limit)
{
    const int per = (d + VEC - 1) / VEC;   // lanes needed for one pass over the row
    const int ch = (per + 63) / 64;
    switch (ch) {
    case 1: return launch_vc<VEC, 1, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    case 2: return launch_vc<VEC, 2, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    case 3: return launch_vc<VEC, 3, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    case 4: return launch_vc<VEC, 4, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    case 5: return launch_vc<VEC, 5, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    case 6: return launch_vc<VEC, 6, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    case 7: return launch_vc<VEC, 7, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);
    default: return launch_vc<VEC, 8, XT>(ctx, A, X, ldx, row_index, d, out, ldo, ep, ws, st, nullptr, nullptr, mean_limit);    // the caller has checked the width
    }
}

} // namespace

size_t sgnn_spmm_ws_bytes(uint64_t max_entries, uint32_t B, uint32_t d_max)
{
    // a plan built on the fly plus the partial rows, for the smallest long-row threshold
    const size_t max_chunks = spmm_max_chunks(B, max_entries);
    return max_chunks * (((size_t)d_max + 255) * sizeof(float) + 12) + (size_t)B * 4 + 5 * 256;
}

extern "C" uint64_t sgnn_csr_plan_bytes(uint32_t rows, uint64_t capacity)
{
    return 256 + (((uint64_t)rows * 4 + 255) & ~uint64_t(255)) + (uint64_t)spmm_max_chunks(rows, capacity) * 12 + 512;
}

// the plan's piece counter, which has to be zero when the plan is built (null without a plan)
uint32_t *sgnn_spmm_plan_counter(const sgnn_csr *A)
{
    return A->plan && A->rows ? plan_view(A->plan, A->rows, 0).n_chunks : nullptr;
}

int sgnn_launch_spmm_plan(sgnn_ctx *ctx, const sgnn_csr *A, bool cleared, hipStream_t st)
{
    if (!A->plan || A->rows == 0) return SGNN_OK;
    return build_plan(ctx, A, A->plan, cleared, st);
}

template <typename XT>
static int launch_x(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, const int32_t *row_index, int64_t d, float *out,
                    int64_t ldo, const spmm_epi &ep, ws_alloc *ws, hipStream_t st)
{
    const uintptr_t bits = reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(ep.mask) |
                           reinterpret_cast<uintptr_t>(ep.add);
    // the narrowest vector with which one wavefront still covers the row
    const int64_t lds_ = ldx | ldo | (ep.mask ? ep.ldm : 0) | (ep.add ? ep.ldadd : 0);
    const bool ok4 = d % 4 == 0 && lds_ % 4 == 0 && (bits & 15) == 0;
    const bool ok2 = d % 2 == 0 && lds_ % 2 == 0 && (bits & 7) == 0;
    const int vec = d <= 64 ? 1 : ((d <= 128 && ok2) ? 2 : (ok4 ? 4 : (ok2 ? 2 : 1)));
    if (d > 64 * 8 * vec) return sgnn_fail(ctx, SGNN_ERR_UNSUPPORTED, "sgnn_spmm: feature width %d is beyond %d columns", (int)d, 64 * 8 * vec);
    // Groups of lanes work on the rows, by one of two kernels, where they can.  Both need the plan.
    constexpr int x16 = sizeof(XT) == 2;
    sgnn_csr planned = *A;
    uint32_t mean_limit = 0;
    const bool panel = sgnn_spmm_panel_wanted(A, d, x16);
    bool by_groups = A->capacity > (uint64_t)SPMM_SHORT && sgnn_spmm_short_wanted(A, row_index, d, x16, ep);
    if ((panel || by_groups) && !A->plan) {     // no plan attached to the matrix: one for this call
        planned.plan = ws->get<uint8_t>(sgnn_csr_plan_bytes(A->rows, A->capacity));
        if (!ws->ok)
            return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm: scratch too small (%zu bytes needed): call sgnn_ctx_reserve", ws->off);
        const int rc = build_plan(ctx, A, planned.plan, false, st);
        if (rc) return rc;
        A = &planned;
    }
    // partial rows in whole panels may take more scratch than spmm_main_kernel's do
    if (by_groups) {
        ws_alloc w2 = *ws;
        w2.get<float>((size_t)spmm_max_chunks(A->rows, A->capacity) * (size_t)sgnn_spmm_short_frame(d, x16));
        by_groups = w2.ok;
    }
    // A matrix with room for many entries a row: whether it has them is known on the device only, so two kernels are
    // launched and the one whose matrix it is not leaves at once (about 3 us of the 100 or more that such a product takes).
    if (panel) {
        ws_alloc w2 = *ws;      // the two kernels share the scratch of the partial rows
        mean_limit = sgnn_spmm_panel_mean(A, d, x16, by_groups);
        const int rc = sgnn_launch_spmm_panel(ctx, A, X, x16, ldx, row_index, (int)d, out, ldo, ep, mean_limit, &w2, st);
        if (rc) return rc;
    }
    if (by_groups) return sgnn_launch_spmm_short(ctx, A, X, x16, ldx, row_index, (int)d, out, ldo, ep, mean_limit, ws, st);
    if (vec == 4) return launch_v<4, XT>(ctx, A, X, ldx, row_index, (int)d, out, ldo, ep, ws, st, mean_limit);
    if (vec == 2) return launch_v<2, XT>(ctx, A, X, ldx, row_index, (int)d, out, ldo, ep, ws, st, mean_limit);
    return launch_v<1, XT>(ctx, A, X, ldx, row_index, (int)d, out, ldo, ep, ws, st, mean_limit);
}

// The product with the loss by groups of lanes; SGNN_ERR_UNSUPPORTED, without a launch, for widths outside it and with too little scratch
template <typename XT>
static int launch_short_xent(sgnn_ctx *ctx, const sgnn_csr *A_in, const XT *X, int64_t ldx, int64_t d, float *out, int64_t ldo, const spmm_epi &ep_in,
                             float *loss, float *colsum, ws_alloc *ws, hipStream_t st)
{
    constexpr int x16 = sizeof(XT) == 2;
    const int frame = sgnn_spmm_short_xent_frame(d, x16);
    if (!frame) return SGNN_ERR_UNSUPPORTED;
    sgnn_csr A = *A_in;
    spmm_epi ep = ep_in;
    ws_alloc w2 = *ws;
    if (!A.plan) A.plan = w2.get<uint8_t>(sgnn_csr_plan_bytes(A.rows, A.capacity));
    const unsigned grid = sgnn_spmm_short_xent_grid(&A);
    ep.loss_partial = w2.get<float>(grid);
    ep.cs_partial = colsum ? w2.get<float>((size_t)grid * d) : nullptr;
    ws_alloc w3 = w2;
    w3.get<float>((size_t)spmm_max_chunks(A.rows, A.capacity) * (size_t)frame);
    if (!w3.ok) return SGNN_ERR_UNSUPPORTED;
    if (!A_in->plan) {
        const int rc = build_plan(ctx, A_in, A.plan, false, st);
        if (rc) return rc;
    }
    int rc = xent_slots(ctx, &ep.fix, st);
    if (rc) return rc;
    rc = sgnn_launch_spmm_short_xent(ctx, &A, X, x16, ldx, (int)d, out, ldo, ep, &w2, st);
    return xent_final(ctx, rc, ep, grid, (int)d, loss, colsum, st);
}

// O = A X + bias with the softmax cross-entropy of O's rows in the epilogue (see spmm_row_xent).  Returns
// SGNN_ERR_UNSUPPORTED without launching anything for widths or alignments the fused kernels are not built for
// (more than 512 columns; rows that do not allow the vector width the column count asks for, where the kernel for short rows does not take them): the caller then
// runs the product and the loss kernel one after the other.
template <typename XT>
static int launch_xent_x(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, int64_t d, float *out, int64_t ldo,
                         const spmm_epi &ep, float *loss, float *colsum, ws_alloc *ws, hipStream_t st)
{
    // a lane moves VEC consecutive elements of X, of the logits (fp32) and of the gradient at once
    auto fits = [](const void *ptr, int64_t ld, int elem_bytes, int vec) {
        return !ptr || ((reinterpret_cast<uintptr_t>(ptr) % (uintptr_t)(vec * elem_bytes)) == 0 && ld % vec == 0);
    };
    auto ok = [&](int vec) {
        return d % vec == 0 && fits(X, ldx, (int)sizeof(XT), vec) && fits(ep.write_out ? out : nullptr, ldo, 4, vec) &&
               fits(ep.dO, ep.lddo, ep.dO_bf16 ? 2 : 4, vec);
    };
    const bool ok4 = ok(4), ok2 = ok(2);
    const bool main_kernel = d <= 64 || (d <= 128 && ok2) || (d <= 512 && ok4);
    // The kernel for short rows takes any width and alignment.  Where spmm_main_kernel does not and the matrix may have many entries a row, the product by the
    // panel kernel and then the loss.  us, product and loss / here, bfloat16 95 / 130 / 190 columns: 2^20 x 1.27 370 / 163, 528 / 258, 641 / 269;
    // 2^18 x 6.4 116 / 97, 201 / 136, 231 / 137; 32768 x 2.9 38 / 27, 42 / 31, 43 / 32.
    if (A->capacity > (uint64_t)SPMM_SHORT && (main_kernel || !sgnn_spmm_panel_wanted(A, d, sizeof(XT) == 2))) {
        const int rc = launch_short_xent(ctx, A, X, ldx, d, out, ldo, ep, loss, colsum, ws, st);
        if (rc != SGNN_ERR_UNSUPPORTED) return rc;
    }
    if (!main_kernel) return SGNN_ERR_UNSUPPORTED;
    if (d <= 64) return launch_vc<1, 1, XT, true>(ctx, A, X, ldx, nullptr, (int)d, out, ldo, ep, ws, st, loss, colsum);
    if (d <= 128 && ok2) return launch_vc<2, 1, XT, true>(ctx, A, X, ldx, nullptr, (int)d, out, ldo, ep, ws, st, loss, colsum);
    if (d <= 256 && ok4) return launch_vc<4, 1, XT, true>(ctx, A, X, ldx, nullptr, (int)d, out, ldo, ep, ws, st, loss, colsum);
    if (d <= 512 && ok4) return launch_vc<4, 2, XT, true>(ctx, A, X, ldx, nullptr, (int)d, out, ldo, ep, ws, st, loss, colsum);
    return SGNN_ERR_UNSUPPORTED;
}

int sgnn_launch_spmm_xent(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, int64_t d, const float *bias,
                          const int32_t *labels, float *out, int64_t ldo, float *loss, void *dO, int dO_bf16, int64_t lddo,
                          float *dO_colsum, ws_alloc *ws, hipStream_t st)
{
    spmm_epi ep = {};
    ep.bias = bias;
    ep.labels = labels;
    ep.dO = dO; ep.dO_bf16 = dO_bf16 ? 1 : 0; ep.lddo = lddo;
    ep.inv_rows = 1.f / (float)A->rows;
    ep.write_out = out ? 1 : 0;
    if (x_bf16) return launch_xent_x(ctx, A, static_cast<const bf16_bits *>(X), ldx, d, out, ldo, ep, loss, dO_colsum, ws, st);
    return launch_xent_x(ctx, A, static_cast<const float *>(X), ldx, d, out, ldo, ep, loss, dO_colsum, ws, st);
}

// X: cols x d, fp32 or (x_bf16) bfloat16 bit patterns, leading dimension ldx in elements
int sgnn_launch_spmm(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, const int32_t *row_index, int64_t d,
                     float *out, int64_t ldo, const float *bias, int relu, const float *mask, int64_t ldm, const float *add,
                     int64_t ldadd, ws_alloc *ws, hipStream_t st)
{
    return sgnn_launch_spmm_x(ctx, A, X, x_bf16, ldx, row_index, d, out, 0, ldo, bias, relu, mask, 0, ldm, add, ldadd, ws, st);
}

// The same with the result (out_bf16) and the mask (mask_bf16) optionally stored as bfloat16; their leading
// dimensions are in elements.
int sgnn_launch_spmm_x(sgnn_ctx *ctx, const sgnn_csr *A, const void *X, int x_bf16, int64_t ldx, const int32_t *row_index, int64_t d,
                       void *out, int out_bf16, int64_t ldo, const float *bias, int relu, const void *mask, int mask_bf16,
                       int64_t ldm, const float *add, int64_t ldadd, ws_alloc *ws, hipStream_t st)
{
    const spmm_epi ep = {bias, relu, static_cast<const float *>(mask), ldm, add, ldadd, out_bf16 ? 1 : 0, (mask && mask_bf16) ? 1 : 0};
    if (A->rows == 0 || d == 0) return SGNN_OK;
    if (x_bf16) return launch_x(ctx, A, static_cast<const bf16_bits *>(X), ldx, row_index, d, static_cast<float *>(out), ldo, ep, ws, st);
    return launch_x(ctx, A, static_cast<const float *>(X), ldx, row_index, d, static_cast<float *>(out), ldo, ep, ws, st);
}
