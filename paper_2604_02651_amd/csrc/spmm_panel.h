// The sparse product for matrices with many entries a row: several entries per gather instruction, columns in panels.
// Included by spmm_group.hip, inside its anonymous namespace.
//
// What bounds the product there is the gathers: every entry reads a row of X, nnz * d elements in all, many times the
// size of X itself, out of L2 and the Infinity Cache.  Two things make them cheaper than one row per wavefront-wide
// instruction:
//  - G lanes of 16 bytes cover one entry's share of a panel and 64 / G entries are gathered by one instruction, so the
//    instruction moves up to 1 KB however narrow the row is (47 fp32 columns: 188 bytes before);
//  - rows wider than 512 bytes are cut into panels, and where their number is even the workgroups of one XCD (consecutive
//    workgroups go to the eight XCDs in turn) work on one panel, so that the part of X an XCD's 4 MB L2 is asked for is that much
//    narrower; an odd number of them (608 fp32 columns: five) is gone through one after the other by all XCDs.
// The sums of the 64 / G groups of lanes are added in registers when a row is complete, in a fixed order.
// Rows that the plan lists as long are taken in items of up to 1024 entries (16 pieces of the plan); rows of several items
// hand partial rows over as in spmm_main_kernel, with one ticket per row and panel.
// Measured, us (spmm_main_kernel / here): 65536 rows, 9.2 M entries, fp32, 256 columns 1014 / 650, 41 columns 515 / 200;
// 600 k rows, 30.6 M entries, fp32, 100 columns 2050 / 1710, 47 columns 1490 / 750; bf16 256 columns 2276 / 1630.  At 256
// columns the gathers then arrive at 14.5 TB/s; a matrix whose X fits every L2 whole reaches 15 to 17 TB/s.  Requesting the
// gathers of one batch of entries ahead of the sums of the last (128 registers more in flight) was slower, so was
// twice the occupancy at half the registers: the L2s' rate is the bound, not the latency.

struct spmm_panel_args {
    uint32_t rows;
    const void *rowptr;
    int rp64;
    const int32_t *colidx;
    const float *val;
    int64_t cap;
    int64_t ldx;
    const int32_t *row_index;
    int d;
    int panels, interleave;      // interleave: how many panels are worked on at a time (1, 2, 4 or 8, divides panels: 1 if odd)
    const uint32_t *n_chunks;    // plan header
    uint32_t mean_limit;         // entries a row from which on the matrix is this kernel's
    uint32_t max_chunks;
    const uint2 *desc;
    uint32_t *ticket;
    float *part;                 // partial rows of d floats, at the row's first piece number + the item's
    float *out;
    int64_t ldo;
    int rows_per_task;           // at most 63
    int wide_epi;                // out, mask and add allow 16-byte (fp32) / 8-element accesses at every column that is a multiple of VEC
};

// Which matrices go this way: those with as many entries a row as spmm_panel_mean says.  The count itself is on the device; the host
// launches both kernels if the capacity is 40 entries a row and 65536 more, which the capacity of a mini-batch matrix (twice the
// expected entries, sixteen more a row and 65536 more) is from a mean of 12 on, or 60 a row (a mean of 22) under 8192 rows, where
// the second launch is a fifth of the product: 1024 x 16 and 4096 x 20 17 us with both launches, whichever kernel works, 14 with one.
// So a matrix whose capacity is its entries takes the kernel from a mean of 40 (60) on.
// The limits against spmm_short_kernel stand at PANEL_BANDS.
// Against spmm_main_kernel, rows x mean and fp32 256 columns: 4096 x 80 39 / 56, 16384 x 13 40 / 43, 65536 x 24 186 / 166, 65536 x 12.5 127 / 101,
// 262144 x 16 483 / 517, 262144 x 12.5 428 / 415; fp32 47 columns: 16384 x 13 23 / 32, 65536 x 12.5 62 / 63, 262144 x 12.5 187 / 164.
constexpr uint32_t spmm_panel_room(uint32_t rows) { return rows < 8192 ? 60 : 40; }
constexpr int SPMM_PANEL_MAX = 16;

// Plan pieces that make up an item of a long row of `nch` pieces of `plen` entries: up to 1024 entries, fewer on a matrix with so few
// pieces that they would not give every wavefront of the machine one.  A row with fewer pieces than there are panels is one
// item (it has as many ticket slots as pieces).  A lone wavefront takes about a microsecond for 32 entries: with items of
// 1024 whatever the matrix, a layer on 1057 rows with 24.6 k entries took 171 us instead of 110.
__device__ __forceinline__ uint32_t spmm_item_pieces(int64_t plen, uint32_t nch, uint32_t n_pieces, int panels)
{
    if (nch <= (uint32_t)panels) return nch;
    const uint32_t want = min(n_pieces / 8192u, 16u) * SPMM_CHUNK / (uint32_t)plen;
    return want ? want : 1u;
}

// 16 bytes from an address that is a multiple of the element size only (gfx950 global loads take any alignment)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));

template <typename XT> struct panel_vec;
template <> struct panel_vec<float> {
    static constexpr int VEC = 4;
    static __device__ __forceinline__ float get(const u32x4_any &q, int i) { return __builtin_bit_cast(float, (uint32_t)q[i]); }
};
template <> struct panel_vec<bf16_bits> {
    static constexpr int VEC = 8;
    static __device__ __forceinline__ float get(const u32x4_any &q, int i)
    {
        const uint32_t w = q[i >> 1];
        return __builtin_bit_cast(float, (i & 1) ? (w & 0xffff0000u) : (w << 16));
    }
};

// x summed over the 64 / G lanes that share lane % G, in every lane
template <int G> __device__ __forceinline__ float group_sum(float x)
{
    if constexpr (G <= 8) x += dpp_f32<0x128>(x);      // row_ror:8
    // the swap exchanges halves between two registers: the second copy must not share the first one's
    if constexpr (G <= 16) {
        uint32_t u = __builtin_bit_cast(uint32_t, x), w = u;
        asm("" : "+v"(w));
        const auto r = __builtin_amdgcn_permlane16_swap(u, w, false, false);
        x = __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
    }
    if constexpr (G <= 32) {
        uint32_t u = __builtin_bit_cast(uint32_t, x), w = u;
        asm("" : "+v"(w));
        const auto r = __builtin_amdgcn_permlane32_swap(u, w, false, false);
        x = __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
    }
    return x;
}

// OFF32: every byte of X lies within 4 GB of its start, so a lane's offset is 32 bits and is computed once per entry.
template <int G, typename XT, bool OFF32>
__global__ __launch_bounds__(SPMM_NT, 4) void spmm_panel_kernel(spmm_panel_args a, const XT *__restrict__ X, spmm_epi ep)
{
    if (a.n_chunks[3] < a.mean_limit) return;          // short rows after all: another kernel's matrix
    constexpr int VEC = panel_vec<XT>::VEC, NE = 64 / G, W = G * VEC;
    constexpr int U = 8;                               // gathers in flight per wavefront, 1 KB each
    const int lane = threadIdx.x & 63, k = lane % G, g = lane / G;
    const uint32_t slot = (blockIdx.x / a.interleave) * (uint32_t)(SPMM_NT / 64) + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nslots = (gridDim.x / a.interleave) * (uint32_t)(SPMM_NT / 64);
    const int long_len = (int)a.n_chunks[1];
    const uint32_t n_pieces = min(*a.n_chunks, a.max_chunks);

    for (int p = (int)(blockIdx.x % a.interleave); p < a.panels; p += a.interleave) {
        // the lane's VEC columns: those from col0 on; at the right edge the 16 bytes that end with the row are read
        // instead, and the first col0 - colb of them belong to the lane before
        const int col0 = p * W + k * VEC, colb = min(col0, a.d - VEC), skip = col0 - colb;
        const bool wide = a.wide_epi && skip == 0;
        const char *__restrict__ xb = reinterpret_cast<const char *>(X);
        const int64_t row_bytes = a.ldx * (int64_t)sizeof(XT);          // below 2^32 if OFF32
        const uint32_t col_bytes = (uint32_t)colb * (uint32_t)sizeof(XT);

        float acc[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
        // n <= 64 entries from e on: lane l gets entry e + l
        auto fetch = [&](int64_t e, int n, int32_t &c, float &v) {
            c = 0; v = 0.f;
            if (lane < n) {
                c = __builtin_nontemporal_load(a.colidx + e + lane);
                v = __builtin_nontemporal_load(a.val + e + lane);
                if (a.row_index) c = a.row_index[c];
                if constexpr (OFF32) c = (int32_t)((uint32_t)c * (uint32_t)row_bytes);
            }
        };
        auto load = [&](int32_t c, float v, int j, u32x4_any &q, float &av) {
            const int32_t src = __builtin_amdgcn_ds_bpermute(j * 4, c);
            av = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(j * 4, __builtin_bit_cast(int, v)));
            if constexpr (OFF32) q = *reinterpret_cast<const u32x4_any *>(xb + (uint32_t)((uint32_t)src + col_bytes));
            else q = *reinterpret_cast<const u32x4_any *>(xb + ((int64_t)src * row_bytes + col_bytes));
        };
        // acc += the n <= 64 entries that the lanes hold: group g takes entries g, g + NE, ...
        auto gather = [&](int32_t c, float v, int n) {
            int j0 = 0;
            for (; j0 + U * NE <= n; j0 += U * NE) {
                u32x4_any q[U];
                float av[U];
#pragma unroll
                for (int t = 0; t < U; ++t) load(c, v, j0 + t * NE + g, q[t], av[t]);
#pragma unroll
                for (int t = 0; t < U; ++t)
#pragma unroll
                    for (int i = 0; i < VEC; ++i) acc[i] = fmaf(av[t], panel_vec<XT>::get(q[t], i), acc[i]);
            }
            if (j0 < n) {
                u32x4_any q[U];
                float av[U];
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (j0 + t * NE < n) load(c, v, min(j0 + t * NE + g, n - 1), q[t], av[t]);
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (j0 + t * NE + g < n) {      // a lane without an entry must not add 0 * x: x may be infinite
#pragma unroll
                        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(av[t], panel_vec<XT>::get(q[t], i), acc[i]);
                    }
            }
        };
        auto reduce = [&]() {
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = group_sum<G>(acc[i]);
        };
        // the finished row is in acc of every group: epilogue and store by group 0
        auto write_row = [&](int64_t row) {
            if (g == 0 && col0 < a.d) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    if (ep.bias) acc[i] += ep.bias[colb + i];
                    if (ep.relu) acc[i] = fmaxf(acc[i], 0.f);
                }
                if (wide) {
#pragma unroll
                    for (int h = 0; h < VEC; h += 4) {
                        float v[4] = {acc[h], acc[h + 1], acc[h + 2], acc[h + 3]};
                        if (ep.mask) {
                            float m[4];
                            if (ep.mask_bf16) vload<4>(m, reinterpret_cast<const bf16_bits *>(ep.mask) + row * ep.ldm + col0 + h);
                            else vload<4>(m, ep.mask + row * ep.ldm + col0 + h);
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] = m[i] > 0.f ? v[i] : 0.f;
                        }
                        if (ep.add) {
                            float m[4];
                            vload<4>(m, ep.add + row * ep.ldadd + col0 + h);
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] += m[i];
                        }
                        vstore_out<4>(a.out, row * a.ldo + col0 + h, v, ep.out_bf16);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        if (i < skip) continue;
                        float v[1] = {acc[i]};
                        const int64_t col = colb + i;
                        if (ep.mask) {
                            float m[1];
                            if (ep.mask_bf16) vload<1>(m, reinterpret_cast<const bf16_bits *>(ep.mask) + row * ep.ldm + col);
                            else vload<1>(m, ep.mask + row * ep.ldm + col);
                            v[0] = m[0] > 0.f ? v[0] : 0.f;
                        }
                        if (ep.add) v[0] += ep.add[row * ep.ldadd + col];
                        vstore_out<1>(a.out, row * a.ldo + col, v, ep.out_bf16);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
        };

        // long rows, item by item; a wavefront looks at its share of the pieces at a time, at most 16
        const uint32_t scan = min(max((n_pieces + nslots - 1) / nslots, 1u), 16u);
        for (uint64_t base = (uint64_t)slot * scan; base < n_pieces; base += (uint64_t)nslots * scan) {
            uint2 rc = make_uint2(0, 0);
            int64_t rs = 0, re = 0, plen = SPMM_CHUNK;
            bool head = false;
            if (lane < (int)scan && base + lane < n_pieces) {
                rc = a.desc[base + lane];
                re = min(rp_load(a.rowptr, a.rp64, (uint64_t)rc.x + 1), a.cap);
                rs = min(rp_load(a.rowptr, a.rp64, rc.x), re);
                plen = spmm_piece_len(re - rs);
                head = rc.y % spmm_item_pieces(plen, (uint32_t)((re - rs + plen - 1) / plen), n_pieces, a.panels) == 0;
            }
            for (uint64_t m = __ballot(head); m; m &= m - 1) {
                const int l = __builtin_ctzll(m);
                const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)rc.x, l), pc = (uint32_t)__builtin_amdgcn_readlane((int)rc.y, l);
                const int64_t s = readlane64(rs, l), e1 = readlane64(re, l), pl = spmm_piece_len(e1 - s);
                const uint32_t all = (uint32_t)((e1 - s + pl - 1) / pl), ip = spmm_item_pieces(pl, all, n_pieces, a.panels);
                const int64_t c0 = s + (int64_t)pc * pl, c1 = min(e1, c0 + (int64_t)ip * pl);
                int32_t c;
                float v;
                fetch(c0, (int)min(c1 - c0, (int64_t)64), c, v);
                for (int64_t e = c0; e < c1; e += 64) {
                    int32_t c2 = 0;
                    float v2 = 0.f;
                    if (e + 64 < c1) fetch(e + 64, (int)min(c1 - e - 64, (int64_t)64), c2, v2);
                    gather(c, v, (int)min(c1 - e, (int64_t)64));
                    c = c2; v = v2;
                }
                reduce();
                const uint32_t first = (uint32_t)base + l - pc;
                const uint32_t nch = min(all, n_pieces - first), items = (nch + ip - 1) / ip;
                if (items <= 1) {
                    write_row(row);
                    continue;
                }
                // partial row out with device-scope stores, then a ticket; the last ticket adds the partial rows up
                if (g == 0 && col0 < a.d) {
                    float *o = a.part + (int64_t)(first + pc) * a.d;
#pragma unroll
                    for (int i = 0; i < VEC; ++i)
                        if (i >= skip) __hip_atomic_store(o + colb + i, acc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                uint32_t t = 0;
                if (lane == 0) t = atomicAdd(&a.ticket[first + p], 1u);
                t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
                if (t + 1 != items) continue;
                if (col0 < a.d)
                    for (uint32_t it = g; it < items; it += NE) {
                        const float *o = a.part + (int64_t)(first + it * ip) * a.d;
#pragma unroll
                        for (int i = 0; i < VEC; ++i)
                            if (i >= skip) acc[i] += __hip_atomic_load(o + colb + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                reduce();
                write_row(row);
                if (lane == 0) a.ticket[first + p] = 0;
            }
        }

        // the other rows, in blocks; the first entries of the next row are requested before the gathers of this one
        for (uint64_t r0 = (uint64_t)slot * a.rows_per_task; r0 < a.rows; r0 += (uint64_t)nslots * a.rows_per_task) {
            const int nr = (int)min((uint64_t)a.rows_per_task, a.rows - r0);
            int64_t rpl = 0;
            if (lane <= nr) rpl = min(rp_load(a.rowptr, a.rp64, r0 + lane), a.cap);
            const int64_t bb = readlane64(rpl, 0);
            const int32_t rp = lane <= nr ? (int32_t)(rpl - bb) : 0;
            // rows are taken in order; a long one is left out
            auto row_at = [&](int r, int &s, int &t) {
                for (; r < nr; ++r) {
                    s = __builtin_amdgcn_readlane(rp, r);
                    t = __builtin_amdgcn_readlane(rp, r + 1);
                    if (t - s <= long_len) break;
                }
                return r;
            };
            int s = 0, t = 0, r = row_at(0, s, t);
            if (r >= nr) continue;
            int32_t c;
            float v;
            fetch(bb + s, min(t - s, 64), c, v);
            for (;;) {
                int r2 = r, s2 = s + 64, t2 = t;
                if (s2 >= t) r2 = row_at(r + 1, s2, t2);
                int32_t c2 = 0;
                float v2 = 0.f;
                if (r2 < nr) fetch(bb + s2, min(t2 - s2, 64), c2, v2);
                gather(c, v, min(t - s, 64));
                if (r2 != r) {
                    reduce();
                    write_row((int64_t)r0 + r);
                }
                if (r2 >= nr) break;
                r = r2; s = s2; t = t2; c = c2; v = v2;
            }
        }
    }
}

// Entries a row from which on this kernel is the faster one of the two by groups of lanes, by rows of the matrix, type of X and how spmm_short_kernel
// covers a row: groups of 8, 16 or 32 lanes, two panels.  A group of lanes walks a row alone there: with few rows it is the chains of gathers that count,
// longest with four values a lane and eight rows a wavefront (all groups of a wavefront share a row here, and there where rows are very few).  With many rows it is how
// the two take hub rows: from 1.5 million entries or so on there are so many pieces that spmm_short_kernel has a group for each, and this kernel
// has the better hold on the caches, the more so the larger X is.
// Each number is the middle of the range in which the sum of what is lost on either side is least, over some 7000 R-MAT matrices of 1000 to 500000 rows and 8 to 250
// entries a row; the rule loses 0.6 % to the faster kernel in the mean and more than 10 % in one matrix of fifty, beside a limit.  us here / there, rows x mean:
//                  bf16 47      bf16 100     bf16 256     fp32 32      fp32 47      fp32 100     fp32 256
//   2048 x 22      14 / 12      15 / 13      20 / 14      10 / 11      11 / 12      14 / 14      14 / 15
//   2048 x 48      16 / 14      18 / 17      24 / 24      10 / 12      14 / 14      18 / 19      18 / 20
//   4096 x 34      17 / 15      19 / 16      30 / 23      11 / 13      15 / 17      19 / 19      21 / 21
//   8191 x 22      18 / 20      21 / 21      32 / 27      12 / 17      16 / 18      20 / 22      27 / 32
//   8191 x 42      22 / 26      27 / 28      47 / 47      14 / 21      19 / 25      28 / 36      39 / 50
//   12000 x 18     22 / 21      23 / 25      38 / 30      14 / 16      17 / 20      23 / 25      36 / 34
//   16384 x 30     31 / 37      35 / 40      63 / 53      21 / 28      26 / 31      39 / 43      62 / 61
//   20480 x 34     42 / 47      56 / 54      90 / 69      26 / 33      38 / 42      56 / 57      86 / 82
//   32768 x 34     65 / 49      75 / 52      114 / 77     41 / 36      56 / 44      72 / 64      124 / 108
//   49152 x 34     83 / 70      93 / 80      120 / 110    55 / 54      72 / 67      88 / 94      147 / 154
//   49152 x 48     99 / 87      112 / 112    156 / 150    66 / 65      86 / 91      112 / 127    181 / 208
//   65536 x 26     90 / 66      103 / 84     138 / 111    58 / 48      78 / 69      98 / 95      159 / 166
//   65536 x 42     112 / 97     124 / 129    169 / 180    74 / 72      98 / 106     125 / 152    206 / 255
//   91000 x 30     126 / 107    141 / 118    184 / 176    82 / 77      108 / 97     136 / 150    224 / 259
//   91000 x 42     136 / 143    149 / 176    204 / 230    88 / 102     121 / 143    162 / 196    284 / 340
//   131072 x 22    137 / 88     145 / 108    177 / 163    88 / 64      117 / 91     142 / 142    255 / 260
//   131072 x 34    165 / 137    177 / 172    226 / 250    110 / 93     147 / 142    187 / 215    353 / 402
//   262144 x 22    227 / 149    245 / 193    304 / 338    145 / 102    202 / 168    267 / 294    530 / 553
//   262144 x 34    273 / 242    302 / 309    414 / 496    177 / 170    258 / 269    390 / 438    787 / 840
//   262144 x 48    324 / 320    369 / 431    561 / 676    212 / 224    323 / 362    536 / 607    1112 / 1156
struct panel_band { uint32_t rows; uint8_t limit[2][4]; };       // up to so many rows; fp32, bfloat16; none: by entries, see spmm_panel_mean
constexpr panel_band PANEL_BANDS[] = {
    {2499, {{54, 56, 34, 30}, {100, 100, 100, 100}}}, {6499, {{10, 16, 28, 20}, {36, 64, 90, 120}}},  {16999, {{12, 12, 22, 22}, {16, 12, 46, 44}}},
    {22499, {{16, 26, 32, 50}, {22, 30, 80, 90}}},    {44999, {}},                                      {61999, {{54, 38, 32, 32}, {58, 44, 48, 38}}},
    {119999, {{36, 32, 28, 28}, {38, 36, 32, 30}}},   {0xffffffffu, {{40, 30, 20, 20}, {44, 28, 24, 20}}}};

// Entries a row from which on a matrix is this kernel's.  or_short: spmm_short_kernel has the others; else spmm_main_kernel, for rows of three
// panels and more and the epilogues that spmm_short_kernel does not have.
template <typename XT> uint32_t spmm_panel_mean(const sgnn_csr *A, int64_t d, bool or_short)
{
    constexpr int VEC = panel_vec<XT>::VEC;
    const uint64_t row = (uint64_t)d * sizeof(XT);
    if (!or_short) return row >= 512 && A->rows >= 32768 && row * A->cols < (96ull << 20) ? 32u : 13u;
    const int cover = d <= 8 * VEC ? 0 : (d <= 16 * VEC ? 1 : (d <= 32 * VEC ? 2 : 3));
    const panel_band *b = PANEL_BANDS;
    while (A->rows > b->rows) ++b;
    if (!b->limit[0][0]) return (cover >= 2 && sizeof(XT) == 4 ? 1600000u : 1900000u) / A->rows;
    return b->limit[sizeof(XT) == 2][cover];
}

template <typename XT> bool spmm_panel_wanted(const sgnn_csr *A, int64_t d)
{
    return A->capacity >= (uint64_t)spmm_panel_room(A->rows) * A->rows + 65536 && d >= panel_vec<XT>::VEC && d <= (int64_t)SPMM_PANEL_MAX * 32 * panel_vec<XT>::VEC;
}

// The arguments but for the panels, the rows of a task and the limit; false if the scratch does not hold the partial rows
inline bool panel_args(spmm_panel_args &a, const sgnn_csr *A, int64_t ldx, const int32_t *row_index, int d, int part_d, float *out,
                       int64_t ldo, const spmm_epi &ep, ws_alloc *ws)
{
    a.rows = A->rows; a.rowptr = A->rowptr; a.rp64 = A->rowptr_is_i64; a.colidx = A->colidx; a.val = A->val;
    a.cap = (int64_t)std::min<uint64_t>(A->capacity, 0x7fffffffffffffffull);
    a.ldx = ldx; a.row_index = row_index; a.d = d; a.out = out; a.ldo = ldo;
    a.max_chunks = spmm_max_chunks(A->rows, A->capacity);
    const spmm_plan_view pv = plan_view(A->plan, A->rows, a.max_chunks);
    a.part = ws->get<float>((size_t)a.max_chunks * (size_t)part_d);
    a.n_chunks = pv.n_chunks; a.desc = pv.desc; a.ticket = pv.ticket;
    const int ob = ep.out_bf16 ? 2 : 4, mb = ep.mask_bf16 ? 2 : 4;
    auto fits = [](const void *p, int64_t ld, int bytes) { return !p || (reinterpret_cast<uintptr_t>(p) % (uintptr_t)(4 * bytes) == 0 && ld % 4 == 0); };
    a.wide_epi = fits(out, ldo, ob) && fits(ep.mask, ep.ldm, mb) && fits(ep.add, ep.ldadd, 4);
    return ws->ok;
}

template <int G, typename XT>
int launch_panel_g(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, spmm_panel_args a, const spmm_epi &ep, hipStream_t st)
{
    constexpr int W = G * panel_vec<XT>::VEC;
    a.panels = (a.d + W - 1) / W;
    a.interleave = a.panels % 8 == 0 ? 8 : (a.panels % 4 == 0 ? 4 : (a.panels % 2 == 0 ? 2 : 1));
    // tasks of up to 16 rows, no fewer than 16384 wavefronts while the rows last; the wavefronts stride over what is left
    a.rows_per_task = (int)std::min<uint64_t>(16, std::max<uint64_t>(1, (uint64_t)A->rows * a.interleave / 16384));
    const uint64_t tasks = std::max<uint64_t>(cdiv(A->rows, a.rows_per_task), a.max_chunks);
    const unsigned grid = (unsigned)std::min<uint64_t>((uint64_t)cdiv(tasks, SPMM_NT / 64) * a.interleave, 8192);
    char tag[56];
    snprintf(tag, sizeof(tag), "%ux%u d=%d G=%d in=%d out=%d%s", A->rows, A->cols, a.d, G, (int)sizeof(XT), ep.out_bf16 ? 2 : 4,
             ep.mask ? (ep.mask_bf16 ? " m=2" : " m=4") : "");
    const bool off32 = !a.row_index && (uint64_t)A->cols * (uint64_t)a.ldx * sizeof(XT) <= 0xffffffffull;
    if (off32)
        SGNN_LAUNCH(ctx, st, "spmm_panel_kernel", tag, (spmm_panel_kernel<G, XT, true>), dim3(grid), dim3(SPMM_NT), 0, st, a, X, ep);
    else
        SGNN_LAUNCH(ctx, st, "spmm_panel_kernel", tag, (spmm_panel_kernel<G, XT, false>), dim3(grid), dim3(SPMM_NT), 0, st, a, X, ep);
    return SGNN_OK;
}

template <typename XT>
int launch_panel(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, const int32_t *row_index, int d, float *out, int64_t ldo,
                 const spmm_epi &ep, uint32_t mean_limit, ws_alloc *ws, hipStream_t st)
{
    spmm_panel_args a = {};
    if (!panel_args(a, A, ldx, row_index, d, d, out, ldo, ep, ws))
        return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm: scratch too small (%zu bytes needed): call sgnn_ctx_reserve", ws->off);
    a.mean_limit = mean_limit;
    // The narrowest panel that holds the row, 32 lanes (512 bytes) at most.  Narrower panels keep more of X in an XCD's L2
    // (dense-degree mini-batch, 256 fp32 columns: L2 misses 45 M a call in spmm_main_kernel, 21 M with panels of 16 lanes, 15 M
    // with 8) but read the matrix and reduce the rows once more per panel: 673 / 890 us with 16 / 8 lanes against 650.
    constexpr int VEC = panel_vec<XT>::VEC;
    if (d <= 8 * VEC) return launch_panel_g<8, XT>(ctx, A, X, a, ep, st);
    if (d <= 16 * VEC) return launch_panel_g<16, XT>(ctx, A, X, a, ep, st);
    return launch_panel_g<32, XT>(ctx, A, X, a, ep, st);
}
