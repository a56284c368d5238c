// The sparse product for matrices with few entries a row: a stream of rows for every group of lanes.  Included by spmm_group.hip,
// inside its anonymous namespace.
//
// What bounds the product there is how many gathers are in flight, not their bytes: spmm_main_kernel has one row of X per
// instruction of the wavefront (512 bytes where 256 columns are stored as bfloat16, 94 where 47 are) and steers every entry with
// scalar code.  Here G lanes of 16 bytes cover an entry's share of a panel, as in the panel kernel, but each of the 64 / G groups of
// a wavefront has rows of its own, so that nothing is added up across lanes and an instruction gathers 1 KB however narrow the
// rows are:
//  - a wavefront takes up to 8 rows for every group.  Their entries are staged in LDS, (byte offset in X, value) each, the last one of a
//    row marked in the offset's free bit: a group walks its entries eight at a time and writes a row where it sees the mark;
//  - ReLU masks and added rows of the block are requested first and go straight into LDS, nothing waits for them at a row's end;
//  - rows that the plan lists as long are taken piece by piece, one piece for every group, in the same loop.  The pieces are the
//    first blocks of the grid.  Where there are fewer pieces than wavefronts the groups of a wavefront share one: then the chain of gathers
//    of a piece (eight for a group alone) is what the product waits for;
//  - partial rows of a long row are handed over as in spmm_main_kernel, word i of lane k at i * G + k, so that a store instruction covers
//    whole memory lines (columns in their order, 4 bytes in every 32: 20000 rows of 64 entries more 147 us instead of 101).
// Measured, us (spmm_main_kernel / here), R-MAT rows x mean:
//                      bf16 256       bf16 128       bf16 47        fp32 256       fp32 100
//   2^20 x 1.27        246 / 218      160 / 118      136 / 60       400 / 423      217 / 200
//   500000 x 3         170 / 144      119 / 68       109 / 50       294 / 279      140 / 122
//   2^18 x 6.4         129 / 103      106 / 57       96 / 46        218 / 204      123 / 93
//   65536 x 12         76 / 51        65 / 36        60 / 40        90 / 76        64 / 43
//   32768 x 2.9        27 / 16        21 / 13        17 / 12        28 / 20        24 / 13
// 2^18 rows of exactly six entries, 256 bfloat16 columns: 124 / 97, of which 9.7 TB/s arrive; a kernel that does nothing but such
// gathers takes the same.  What the R-MAT matrix takes beyond it is the ragged end of rows and pieces.
// With the loss in the epilogue a group holds a whole row of logits (one panel): its maximum and sum are reductions over the group's lanes,
// two to eight rows at a time, where spmm_main_kernel has one row on 64 lanes of one to four columns.
//                      bf16 172       bf16 100       bf16 47        fp32 100       fp32 47
//   2^20 x 1.27        407 / 325      274 / 211      228 / 132      309 / 270      233 / 152
//   2^18 x 6.4         204 / 156      146 / 108      129 / 83       149 / 128      128 / 80
//   32768 x 2.9        54 / 36        33 / 30        29 / 28        37 / 31        29 / 26
// What bounded it then is the instructions of a row's end (counters, 2^20 x 1.27 with 172 bfloat16 columns: 167 vector instructions a row, of which the product
// is 48; the vector units busy 89 % of the time).  With the following it has 121, of which the product is 39, and 81 %:
// six bfloat16 values a lane where they cover the row, two values rounded at once, a maximum without canonical operands, the correction of the
// exponential in two products: from one call to the next, the final sum included, before / after, us:
//                      bf16 256   bf16 172   bf16 100   bf16 70    bf16 47    fp32 100   fp32 47
//   2^20 x 1.27        338 / 299  330 / 270  211 / 194  203 / 163  134 / 110  283 / 275  158 / 151
//   2^18 x 6.4         180 / 167  165 / 136  120 / 107  119 / 95   94 / 74    142 / 138  88 / 80
//   32768 x 2.9        41 / 34    40 / 31    34 / 28    34 / 28    32 / 25    33 / 30    29 / 25
// Rejected: 16 rows a block for groups of 16 and 32 lanes (2^20 x 172: 277 instead of 289, the products without a loss 2 % slower).
// The lanes at the right edge store 16 bytes like the others, over columns of their neighbour's; column by column 2^20 x 1.27 with
// 172 columns took 400.  Three chunks a lane and eight lanes a row (fewer instructions a row, twice the registers): 474, 356 for 2^18 x 6.4.
// Rejected: rows of up to 64 entries as rows of a group (2^18 x 6.4, 256 bfloat16 columns: 136 -> 145 us, 32768 x 2.9: 18 -> 25, the groups of a
// wavefront wait for one another), four gathers in flight at five wavefronts a SIMD (156 against 149 at the time), panels of 256 bytes (132 against 120),
// two pieces and more per partial row (125 -> 130, 141, 147 with two, five, eight).
constexpr int SHORT_U = 8;                   // gathers in flight per wavefront, 1 KB each
// Partial rows of a long row: 64, more where each would be the sum of more than 256 entries and the plan has the pieces for it.  A partial
// row is one chain of gathers, reading a partial row back is one more trip to memory.  65536 rows of 6 entries and 8 rows of 1e5, 256 / 128 / 47
// bfloat16 columns, us: 186 / 110 / 78 with 64 whatever the length, 110 / 69 / 55 with this rule, 100 / 52 / 37 with all groups of the last
// wavefront adding partial rows up (spmm_main_kernel 113 / 87 / 65).  Every piece a partial row: 8 rows of 2e4 instead, 47 columns, 37 instead of 30.
constexpr uint32_t SHORT_ITEMS = 64;
constexpr uint32_t SHORT_ITEM_LEN = 256;
constexpr int SHORT_SUM = 4;                 // of which a group reads so many at a time
constexpr uint32_t SHORT_SHARED = 4096;      // fewer pieces than this (a wavefront for each, four a SIMD): the groups share them
constexpr uint64_t SHORT_GRID = 8192;        // workgroups of a panel, at most (2^20 rows of 1.27: 210 us, 218 and 222 with 4096 and 2048)
constexpr int SHORT_ROWS = 8;                // rows that a group of lanes takes at a time, at most
template <int G> struct short_window { static constexpr int LEN = G == 32 ? 256 : 512; };      // entries of a block in LDS at a time

enum { SHORT_PLAIN, SHORT_MASK, SHORT_ADD, SHORT_BIAS, SHORT_XENT };      // what happens to a finished row

// x over the G lanes of a group (lane / G), in each of them
template <int G, bool MAX> __device__ __forceinline__ float lanes_reduce(float x)
{
    auto op = [](float a, float b) { return MAX ? fmaxf(a, b) : a + b; };
    if constexpr (MAX) {
        // in assembler: fmaxf makes its operands canonical first, four instructions a step.  (Two wait states lie between
        // a register's write and its read by another lane; the lanes of a group are active together.)
#define SGNN_MAX_STEP(CTRL) asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 " CTRL " row_mask:0xf bank_mask:0xf" : "=v"(x) : "v"(x))
        SGNN_MAX_STEP("quad_perm:[1,0,3,2]");
        SGNN_MAX_STEP("quad_perm:[2,3,0,1]");
        SGNN_MAX_STEP("row_half_mirror");
        if constexpr (G >= 16) SGNN_MAX_STEP("row_mirror");
#undef SGNN_MAX_STEP
    } else {
        x += dpp_f32<0xB1>(x);                              // quad_perm [1, 0, 3, 2]
        x += dpp_f32<0x4E>(x);                              // quad_perm [2, 3, 0, 1]
        x += dpp_f32<0x141>(x);                             // row_half_mirror
        if constexpr (G >= 16) x += dpp_f32<0x140>(x);      // row_mirror
    }
    if constexpr (G >= 32) {
        uint32_t u = __builtin_bit_cast(uint32_t, x), w = u;
        asm("" : "+v"(w));
        const auto r = __builtin_amdgcn_permlane16_swap(u, w, false, false);
        x = op(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
    }
    return x;
}

// Rows per group of lanes: about 48 entries, and no fewer than 4096 wavefronts while the rows last
__device__ __forceinline__ int short_rows(uint32_t rows, uint32_t mean, int groups, int interleave)
{
    const uint64_t fill = (uint64_t)rows * (uint64_t)interleave / (4096u * (uint64_t)groups);
    const uint64_t r = min((uint64_t)(48u / max(mean, 1u)), fill);
    return (int)min(max(r, (uint64_t)1), (uint64_t)SHORT_ROWS);
}

// Whether the groups of a wavefront share every row as they share a piece: where there are too few rows for the chip and a group's chain
// of gathers through a row, longer with the mean and with the values a lane adds up per entry, is what the product waits for.  us, spmm_main_kernel /
// one row a group / shared, R-MAT rows x mean, matrices of which the host does not know that they have many entries:
//                     bf16 47            bf16 256          fp32 47           fp32 256         with the loss, bf16 47
//   1024 x 30         16 / 19 / 14       19 / 15 / 16      16 / 14 / 14      18 / 14 / 14     27 / 34 / 24
//   1024 x 110        48 / 105 / 14      54 / 74 / 23      47 / 57 / 14      52 / 54 / 20     59 / 131 / 26
//   2048 x 60         40 / 78 / 14       45 / 56 / 25      40 / 37 / 15      43 / 42 / 21     51 / 90 / 29
//   4096 x 60         36 / 42 / 17       38 / 29 / 28      36 / 22 / 17      41 / 28 / 28     47 / 58 / 32
//   8192 x 80         74 / 94 / 37       87 / 96 / 57      74 / 54 / 36      92 / 97 / 97     88 / 112 / 52
//   16384 x 50        77 / 54 / 46       95 / 84 / 87      77 / 46 / 46      109 / 97 / 97    92 / 68 / 63
// From 14000 rows on only with more entries a row (alone / shared, with the loss, 12 bfloat16 columns): 16384 x 40 45 / 52, 16384 x 60 80 / 62,
// 24000 x 60 57 / 84, 24000 x 100 95 / 108, 24000 x 150 155 / 142, 32768 x 100 120 / 131, 32768 x 150 201 / 162; 12000 x 40 48 / 43.
// A quarter and a half of the factor: the same or slower at every size (8192 x 60, 47 bfloat16 columns 61 and 31 us, 30 with this one).
__device__ __forceinline__ bool short_shares_rows(uint32_t rows, uint32_t mean, int values)
{
    return rows <= 65536u && 7ull * mean * (uint64_t)values > rows && mean >= (rows > 20000u ? 128u : (rows > 14000u ? 50u : 0u));
}

// The offsets of two rows, requested together (a branch around each of them cost a round trip to memory)
__device__ __forceinline__ void row_offsets(const spmm_panel_args &a, uint64_t i, uint64_t j, int64_t &x, int64_t &y)
{
    if (a.rp64) { const int64_t *r = static_cast<const int64_t *>(a.rowptr); x = r[i]; y = r[j]; }
    else { const int32_t *r = static_cast<const int32_t *>(a.rowptr); x = r[i]; y = r[j]; }
    y = min(y, a.cap);
    x = min(x, y);
}

// A lane's VEC values of a row of X: 16 bytes, or 12, from an address that is a multiple of the element size only
template <int DWORDS> struct __attribute__((packed, aligned(2))) short_chunk { uint32_t q[DWORDS]; };

template <typename XT> __device__ __forceinline__ float chunk_get(uint32_t w, int i)
{
    if constexpr (sizeof(XT) == 4) return __builtin_bit_cast(float, w);
    else return __builtin_bit_cast(float, (i & 1) ? (w & 0xffff0000u) : (w << 16));
}

// Two values rounded to nearest even, in one instruction
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The lane's columns, from element `elem` on, up to 16 bytes at a time at any alignment (gfx950 global stores take it).  At the right edge the
// first of them are the lane's before as well: both write the same bytes.
template <int VEC> __device__ __forceinline__ void short_store_bf16(float *out, int64_t elem, const uint32_t (&w)[VEC / 2])
{
    short_chunk<VEC / 2> c;
#pragma unroll
    for (int i = 0; i < VEC / 2; ++i) c.q[i] = w[i];
    *reinterpret_cast<short_chunk<VEC / 2> *>(reinterpret_cast<uint16_t *>(out) + elem) = c;
}
template <int VEC> __device__ __forceinline__ void short_store(float *out, int64_t elem, const float (&v)[VEC], int out_bf16)
{
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
    if (out_bf16) {
        uint32_t w[VEC / 2];
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i) w[i] = bf16_pair(v[2 * i], v[2 * i + 1]);
        short_store_bf16<VEC>(out, elem, w);
    } else {
#pragma unroll
        for (int h = 0; h + 4 <= VEC; h += 4) { const f32x4_any q = {v[h], v[h + 1], v[h + 2], v[h + 3]}; *reinterpret_cast<f32x4_any *>(out + elem + h) = q; }
        if constexpr (VEC % 4) { const f32x2_any q = {v[VEC - 2], v[VEC - 1]}; *reinterpret_cast<f32x2_any *>(out + elem + VEC - 2) = q; }
    }
}

// r * ld for r < 64 and ld < 2^56: one full product of 32 bits and one of 24, where a 64-bit product takes three of 32, each four times as long as an addition
__device__ __forceinline__ int64_t row_offset(uint32_t r, int64_t ld)
{
    return (int64_t)((uint64_t)r * (uint32_t)ld + ((uint64_t)((r & 63u) * ((uint32_t)((uint64_t)ld >> 32) & 0xffffffu)) << 32));
}

// VEC: values a lane holds, 16 bytes or (six bfloat16 values, with the loss) 12.
template <int G, typename XT, bool OFF32, int EPI, int VEC = panel_vec<XT>::VEC>
__global__ __launch_bounds__(SPMM_NT, 4) void spmm_short_kernel(spmm_panel_args a, const XT *__restrict__ X, spmm_epi ep)
{
    if (a.mean_limit && a.n_chunks[3] >= a.mean_limit) return;        // the panel kernel's matrix
    constexpr int NE = 64 / G, W = G * VEC, U = SHORT_U, CAPW = short_window<G>::LEN;
    typedef short_chunk<VEC * (int)sizeof(XT) / 4> chunk;
    constexpr bool XENT = EPI == SHORT_XENT;
    __shared__ uint2 staged[SPMM_NT / 64][CAPW];
    constexpr bool SIDE = EPI == SHORT_MASK || EPI == SHORT_ADD;         // a matrix beside X is read at the rows' ends
    __shared__ __attribute__((aligned(16))) u32x4_any side[SIDE ? SPMM_NT / 64 : 1][SIDE ? SHORT_ROWS * 64 : 1];
    const int lane = threadIdx.x & 63, k = lane % G, g = lane / G;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint2 *st = staged[wv];
    // blocks of work: a piece of a long row for every group of lanes, then R rows for every group
    const uint32_t n_pieces = min(*a.n_chunks, a.max_chunks);
    const int long_len = (int)a.n_chunks[1];
    const int rows_each = short_rows(a.rows, a.n_chunks[3], NE, a.interleave), rows_all = rows_each * NE;
    // (with few pieces all groups share one: then the length of the chain of gathers counts, not the number of wavefronts)
    const bool shared_rows = short_shares_rows(a.rows, a.n_chunks[3], NE * panel_vec<XT>::VEC), shared = shared_rows || n_pieces < SHORT_SHARED;
    const uint32_t per_block = shared ? 1 : NE, n_units = n_pieces + (shared_rows ? a.rows : 0);      // pieces, and rows that are shared like them
    // (32 bits: at most 2^24 pieces and 2^31 blocks of two rows.  Scalars are short here: held in 64 bits the loss forms spilled more)
    const uint32_t piece_blocks = (n_units + per_block - 1) / per_block;
    const uint32_t blocks = piece_blocks + (shared_rows ? 0 : (uint32_t)((a.rows + (uint64_t)rows_all - 1) / rows_all));
    const uint32_t first_block = blockIdx.x / (unsigned)a.interleave * (SPMM_NT / 64) + wv;
    const uint32_t nwaves = gridDim.x / (unsigned)a.interleave * (SPMM_NT / 64);
    const char *__restrict__ xb = reinterpret_cast<const char *>(X);
    const int64_t row_bytes = a.ldx * (int64_t)sizeof(XT);          // below 2^32 if OFF32

    const int p = (int)(blockIdx.x % (unsigned)a.interleave);       // as many panels at a time as there are
    // the lane's columns, as in the panel kernel
    const int col0 = p * W + k * VEC, colb = min(col0, a.d - VEC), skip = col0 - colb;
    const bool on = col0 < a.d;
    const uint32_t col_bytes = (uint32_t)colb * (uint32_t)sizeof(XT);
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    // The wavefront's sums of the loss and of the gradient's columns, and the labels of a block's rows.  Which wavefront has a long row
    // goes with the timing of the plan kernel: such rows are added up as integers, in any order the same, over the workgroup (word
    // i * G + k is value i of lane k) and then over the workgroups.  (Straight into memory, 22 lines a row: 2^18 x 6.4 with
    // 172 columns 213 us instead of 161.)
    __shared__ unsigned long long fixed[XENT ? W + 1 : 1];
    __shared__ int32_t labels[XENT ? SPMM_NT / 64 : 1][XENT ? 64 : 1];
    // a lane's bias values, from LDS at every row's end: held in registers they spilled
    __shared__ __attribute__((aligned(16))) float bias[EPI == SHORT_BIAS || XENT ? W : 1];
    if constexpr (EPI == SHORT_BIAS || XENT) {
        if (threadIdx.x < G) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) bias[k * VEC + i] = ep.bias ? ep.bias[colb + i] : 0.f;
        }
        if constexpr (XENT)
            for (int i = threadIdx.x; i <= W; i += SPMM_NT) fixed[i] = 0;
        __syncthreads();
    }
    float loss = 0.f, cs[XENT ? VEC : 1] = {};
    // Loss and gradient of the row of logits in acc: spmm_row_xent with a group of lanes a row.  The columns below `skip` are in
    // the lane before too: they count in the maximum, where that does not matter, and not in the sums.
    auto xent = [&](auto elem_of, int32_t y, auto shared_row) {
        constexpr bool SHARED = decltype(shared_row)::value;
        auto add_loss = [&](float t) {
            if constexpr (SHARED) xent_add_fixed(&fixed[W], t, XENT_FIX_LOSS, loss);
            else loss += t;
        };
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            acc[i] += bias[k * VEC + i];
            mx = fmaxf(mx, acc[i]);
        }
        if (ep.write_out && on) short_store<VEC>(a.out, elem_of(a.ldo), acc, 0);
        mx = lanes_reduce<G, true>(mx);
        const int rel = y - colb;
        const bool has_y = rel >= skip && rel < VEC;
        float sum = 0.f, vy = acc[0];
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            vy = rel == i ? acc[i] : vy;
            acc[i] = exp_neg(acc[i] - mx);
            sum += i >= skip ? acc[i] : 0.f;
        }
        sum = lanes_reduce<G, false>(sum);
        const float inv = __builtin_amdgcn_rcpf(sum), lse = log_ge1(sum);       // 1 ulp each
        if (has_y) add_loss(lse - (vy - mx));
        if ((uint32_t)y >= (uint32_t)a.d && k == 0) add_loss(mx + lse);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(acc[i], inv, rel == i ? -1.f : 0.f) * ep.inv_rows;
        auto add_columns = [&]() {      // the column sums add what is stored
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                if constexpr (SHARED) xent_add_fixed(&fixed[i * G + k], acc[i], XENT_FIX_CS, cs[i]);
                else cs[i] += acc[i];
            }
        };
        if (ep.dO_bf16) {
            uint32_t w[VEC / 2];
#pragma unroll
            for (int i = 0; i < VEC / 2; ++i) {
                w[i] = bf16_pair(acc[2 * i], acc[2 * i + 1]);
                acc[2 * i] = chunk_get<bf16_bits>(w[i], 0);
                acc[2 * i + 1] = chunk_get<bf16_bits>(w[i], 1);
            }
            if (ep.dO && on) short_store_bf16<VEC>(static_cast<float *>(ep.dO), elem_of(ep.lddo), w);
            add_columns();
        } else {
            if (ep.dO && on) short_store<VEC>(static_cast<float *>(ep.dO), elem_of(ep.lddo), acc, 0);
            add_columns();
        }
    };
    const char *__restrict__ side_base = reinterpret_cast<const char *>(EPI == SHORT_ADD ? ep.add : ep.mask);
    const int64_t side_row = (EPI == SHORT_ADD ? ep.ldadd : ep.ldm) * (int64_t)sizeof(XT);       // below 2^25
    auto beside = [&](const u32x4_any &m) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            if constexpr (EPI == SHORT_ADD) acc[i] += panel_vec<XT>::get(m, i);
            else acc[i] = panel_vec<XT>::get(m, i) > 0.f ? acc[i] : 0.f;
        }
    };
    // the lane's columns of a row that is complete in acc
    auto store = [&](auto elem_of) {
        if constexpr (EPI == SHORT_BIAS) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                acc[i] += bias[k * VEC + i];
                if (ep.relu) acc[i] = fmaxf(acc[i], 0.f);
            }
        }
        short_store<VEC>(a.out, elem_of(a.ldo), acc, ep.out_bf16);
    };

    for (uint32_t block = first_block; block < blocks; block += nwaves) {
        const bool pieces = block < piece_blocks;
        const int R = pieces ? 1 : rows_each, RW = R * NE, gb = g * R;
        const uint64_t u0 = pieces ? (uint64_t)block * per_block : (uint64_t)(block - piece_blocks) * rows_all;       // the first piece or row
        if constexpr (SIDE) {
            if (!pieces) {
                const char *first_row = side_base + (int64_t)u0 * side_row;
                const uint32_t last = (uint32_t)min((uint64_t)a.rows - 1 - u0, (uint64_t)63);
                for (int r = 0; r < R; ++r) {
                    const uint32_t off = min((uint32_t)(gb + r), last) * (uint32_t)side_row + col_bytes;
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(first_row + off),
                                                     (__attribute__((address_space(3))) void *)(side[wv] + r * 64), 16, 0, 0);
                }
            }
        }
        int len, so = 0, se = 0, limit;       // entries of the lane's unit; its place in the block's list (rows); entries to go through
        int64_t s;                            // where they begin
        uint64_t longs = 0;
        uint32_t left = 0, none = 0;
        uint32_t row = 0, pc = 0, nch = 0, ip = 1;       // nch: 0 where the lane's unit has nothing to add up or to write
        if (pieces) {
            len = 0; s = 0;
            if (u0 >= n_pieces) {             // a row that is shared
                int64_t re;
                row = (uint32_t)u0 - n_pieces;
                row_offsets(a, row, (uint64_t)row + 1, s, re);
                nch = re - s <= long_len;
                len = nch && lane == 0 ? (int)(re - s) : 0;
            } else if (lane < (int)per_block && u0 + lane < n_pieces) {
                const uint2 rc = a.desc[u0 + lane];
                int64_t rs, re;
                row_offsets(a, rc.x, (uint64_t)rc.x + 1, rs, re);
                const int64_t plen = spmm_piece_len(re - rs);
                const int sh = 63 - __clzll(plen);
                row = rc.x; pc = rc.y;
                nch = min((uint32_t)((re - rs + plen - 1) >> sh), n_pieces - ((uint32_t)u0 + lane - pc));
                ip = nch <= (uint32_t)a.panels ? nch : min((nch + SHORT_ITEMS - 1) / SHORT_ITEMS, max(SHORT_ITEM_LEN >> sh, 1u));
                s = rs + ((int64_t)pc << sh);
                if (pc % ip == 0) len = (int)min(re - s, (int64_t)ip << sh);
                if (len == 0) nch = 0;
            }
            limit = 0;
#pragma unroll
            for (int v = 0; v < NE; ++v) limit = max(limit, __builtin_amdgcn_readlane(len, v));
        } else {
            // lane l < RW holds row u0 + l, the lanes behind the block and behind the matrix a row without entries
            const uint64_t k0 = min(u0 + min(lane, RW), (uint64_t)a.rows), k1 = min(u0 + min(lane + 1, RW), (uint64_t)a.rows);
            int64_t rs, re;
            if constexpr (XENT) labels[wv][lane] = ep.labels[min(k0, (uint64_t)a.rows - 1)];
            row_offsets(a, k0, k1, rs, re);
            s = readlane64(rs, 0);
            len = (int)(re - rs);
            const bool is_long = len > long_len;
            // places in the block's list of entries, long rows left out: [so, se) for the lane's row
            longs = __ballot(is_long);
            so = (int)(rs - s);
            for (uint64_t m = longs; m; m &= m - 1) {
                const int l = __builtin_ctzll(m), n = __builtin_amdgcn_readlane(len, l);
                if (lane > l) so -= n;
            }
            se = so + (is_long ? 0 : len);
            limit = __builtin_amdgcn_readlane(se, 63);
            const uint32_t group_rows = (1u << R) - 1u;
            left = (uint32_t)(__ballot(len > 0 && !is_long) >> gb) & group_rows;
            none = (uint32_t)(__ballot(k1 > k0 && len == 0) >> gb) & group_rows;
        }
        const int gu = shared ? 0 : g;        // the group's piece
        const int glen = __shfl(len, gu, 64), begin = __shfl(so, gb, 64), end = __shfl(se, gb + R - 1, 64);

        // the group's row r is complete in acc
        auto emit = [&](uint32_t r) {
            if constexpr (SIDE) beside(side[wv][r * 64 + lane]);
            auto elem_of = [&](int64_t ld) { return (int64_t)u0 * ld + row_offset((uint32_t)gb + r, ld) + colb; };
            if constexpr (XENT) xent(elem_of, labels[wv][gb + r], std::false_type{});
            else store(elem_of);
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
        };

        for (int w0 = 0; w0 < limit; w0 += pieces ? SPMM_CHUNK : CAPW) {
            int at, stop;            // the group's entries in LDS
            if (pieces) {            // up to 64 entries of every group's piece
                int32_t c[NE];
                float v[NE];
                int n_j[NE];
#pragma unroll
                for (int j = 0; j < NE; ++j) {       // no branch round the loads: they are in flight together
                    n_j[j] = __builtin_amdgcn_readlane(len, j) - w0;
                    const int64_t e = readlane64(s, j) + (lane < n_j[j] ? w0 + lane : 0);
                    c[j] = a.colidx[e];
                    v[j] = a.val[e];
                }
                if (a.row_index) {
#pragma unroll
                    for (int j = 0; j < NE; ++j) c[j] = a.row_index[c[j]];
                }
#pragma unroll
                for (int j = 0; j < NE; ++j) {
                    if constexpr (OFF32) c[j] = (int32_t)((uint32_t)c[j] * (uint32_t)row_bytes);
                    if (lane < n_j[j]) st[j * SPMM_CHUNK + lane] = make_uint2((uint32_t)c[j], __builtin_bit_cast(uint32_t, v[j]));
                }
                const int n = min(glen - w0, SPMM_CHUNK), part = (n + NE - 1) / NE;
                at = shared ? min(g * part, n) : g * SPMM_CHUNK;
                stop = shared ? min(at + part, n) : at + n;
            } else {
                const int cnt = min(limit - w0, CAPW);
                for (int j0 = 0; j0 < cnt; j0 += 128) {
                    int32_t c[2];
                    float v[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int q = w0 + min(j0 + j * 64 + lane, cnt - 1);
                        int64_t e = s + q;
                        for (uint64_t m = longs; m; m &= m - 1) {
                            const int l = __builtin_ctzll(m), o = __builtin_amdgcn_readlane(so, l), n = __builtin_amdgcn_readlane(len, l);
                            if (q >= o) e += n;
                        }
                        c[j] = a.colidx[e];
                        v[j] = a.val[e];
                    }
                    if (a.row_index) {
#pragma unroll
                        for (int j = 0; j < 2; ++j) c[j] = a.row_index[c[j]];
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int q = j0 + j * 64 + lane;
                        if constexpr (OFF32) c[j] = (int32_t)((uint32_t)c[j] * (uint32_t)row_bytes);
                        if (q < cnt) st[q] = make_uint2((uint32_t)c[j], __builtin_bit_cast(uint32_t, v[j]));
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                // the last entry of a row is marked: rows are an even number of bytes, so bit 0 of an offset is free, and so
                // is the sign of a row number
                if (se > so && se - 1 >= w0 && se - 1 < w0 + cnt) st[se - 1 - w0].x |= OFF32 ? 1u : 0x80000000u;
                at = max(begin - w0, 0);
                stop = min(end - w0, cnt);
            }
            // lanes right of the last column stand still (with the loss they read the last columns once more: its sums go over all lanes)
            if (!XENT && !on) stop = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (; at < stop; at += U) {
                uint2 w[U];
                chunk q[U];
#pragma unroll
                for (int t = 0; t < U; ++t) w[t] = st[min(at + t, stop - 1)];
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (at + t < stop) {
                        if constexpr (OFF32) q[t] = *reinterpret_cast<const chunk *>(xb + (uint32_t)((w[t].x & ~1u) + col_bytes));
                        else q[t] = *reinterpret_cast<const chunk *>(xb + ((int64_t)(w[t].x & 0x7fffffffu) * row_bytes + col_bytes));
                    }
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (at + t < stop) {
#pragma unroll
                        for (int i = 0; i < VEC * (int)sizeof(XT) / 4; ++i) asm volatile("" : "+v"(q[t].q[i]));      // nothing of the widening moves up in front of the branch
#pragma unroll
                        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(__builtin_bit_cast(float, w[t].y), chunk_get<XT>(q[t].q[i * (int)sizeof(XT) / 4], i), acc[i]);
                        if (OFF32 ? (w[t].x & 1u) != 0 : (int32_t)w[t].x < 0) {
                            emit((uint32_t)__builtin_ctz(left));
                            left &= left - 1;
                        }
                    }
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (!pieces) {
            if (XENT || on)
                for (; none; none &= none - 1) emit((uint32_t)__builtin_ctz(none));
            continue;
        }

        // the group's piece is complete in acc; of a shared one every group has the sum, and the first goes on with it
        if (shared) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = group_sum<G>(acc[i]);
        }
        const uint32_t grow = __shfl(row, gu, 64), gpc = __shfl(pc, gu, 64), gnch = __shfl(nch, gu, 64), gip = __shfl(ip, gu, 64);
        const bool mine = (XENT || on) && gnch && !(shared && g > 0);
        const uint32_t first = (uint32_t)u0 + gu - gpc, items = (gnch + gip - 1) / gip;
        bool whole = items <= 1;
        if (!whole) {
            // partial row out with device-scope stores, then a ticket; the last ticket adds the partial rows up
            // (word i of lane k at i * G + k: every store covers whole memory lines)
            const int64_t stride = (int64_t)a.panels * W;
            float *o = a.part + (int64_t)first * stride + p * W + k;
            int last = 0;
            if (mine) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) __hip_atomic_store(o + (int64_t)gpc * stride + i * G, acc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                uint32_t t = 0;
                if (k == 0) t = atomicAdd(&a.ticket[first + p], 1u);
                last = __shfl(t, g * G, 64) + 1 == items;
            }
            // (of a shared piece the other groups, too, add some of them up)
            if (shared) last = __shfl(last, 0, 64);
            if (last && (XENT || on)) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
                for (uint32_t it = shared ? g * SHORT_SUM : 0; it < items; it += shared ? NE * SHORT_SUM : SHORT_SUM) {
                    float v[SHORT_SUM][VEC];
#pragma unroll
                    for (int j = 0; j < SHORT_SUM; ++j)
#pragma unroll
                        for (int i = 0; i < VEC; ++i)
                            v[j][i] = __hip_atomic_load(o + (int64_t)(min(it + j, items - 1) * gip) * stride + i * G, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int j = 0; j < SHORT_SUM; ++j)
                        if (it + j < items) {
#pragma unroll
                            for (int i = 0; i < VEC; ++i) acc[i] += v[j][i];
                        }
                }
                if (k == 0 && mine) a.ticket[first + p] = 0;
            }
            if (shared && last) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = group_sum<G>(acc[i]);
            }
            whole = last;
        }
        if (mine && whole) {
            if constexpr (SIDE) beside(*reinterpret_cast<const u32x4_any *>(side_base + (int64_t)grow * side_row + col_bytes));
            // (the numbering of the pieces goes with the timing of the plan kernel: sums of such rows through the slots)
            auto elem_of = [&](int64_t ld) { return (int64_t)grow * ld + colb; };
            if constexpr (XENT) {
                if (u0 < n_pieces) xent(elem_of, ep.labels[grow], std::true_type{});
                else xent(elem_of, ep.labels[grow], std::false_type{});
            } else store(elem_of);
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    }
    if constexpr (XENT) {
        // the wavefronts' sums, added in a fixed order, leave as the workgroup's
        __shared__ float loss_sums[SPMM_NT / 64], column_sums[SPMM_NT / 64][W];
        loss = wave_sum(loss);
        if (lane == 0) loss_sums[wv] = loss;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float t = group_sum<G>(cs[i]);
            if (g == 0 && i >= skip) column_sums[wv][colb + i] = t;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int w = 0; w < SPMM_NT / 64; ++w) t += loss_sums[w];
            ep.loss_partial[blockIdx.x] = t;
        }
        unsigned long long *slot = ep.fix + (uint64_t)(blockIdx.x % XENT_SLOTS) * (uint64_t)(a.d + 1);
        for (int w = threadIdx.x; w <= W; w += SPMM_NT) {
            const unsigned long long t = fixed[w];
            const int kc = (w % G) * VEC, b = min(kc, a.d - VEC), c = w < W ? b + w / G : a.d;
            if (t && (w == W || w / G >= kc - b)) atomicAdd(slot + c, t);
        }
        if (ep.cs_partial)
            for (int c = threadIdx.x; c < a.d; c += SPMM_NT) {
                float t = 0.f;
                for (int w = 0; w < SPMM_NT / 64; ++w) t += column_sums[w][c];
                ep.cs_partial[(int64_t)blockIdx.x * a.d + c] = t;
            }
    }
}

// Which calls go this way: one panel or two (300 fp32 columns, three panels, one after the other: 200000 rows of 3 entries 75 us in
// spmm_main_kernel, 79 here, 8192 of 4 20 and 44) with at most one of bias / ReLU, mask and added matrix, the last two of X's type
// and in whole 16 bytes (they go into LDS by direct loads).
// Not two panels of 400000 rows and more through a row index either: the panels read the two parts of a row of X, which is seldom read
// again, at different times (200 fp32 columns: 500000 x 3 285 us in spmm_main_kernel, 298 here, 2^20 x 1.27 447 and 494; 2^18 x 6.4 245 and 239).
template <typename XT> bool spmm_short_wanted(const sgnn_csr *A, const int32_t *row_index, int64_t d, const spmm_epi &ep)
{
    constexpr int VEC = panel_vec<XT>::VEC;
    auto whole = [&](const void *p, int64_t ld) {
        const int64_t row = ld * (int64_t)sizeof(XT);
        return d % VEC == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0 && row % 16 == 0 && row < (1 << 25);
    };
    if (d < VEC || d > 2 * 32 * VEC || (row_index && d > 32 * VEC && A->rows >= 400000)) return false;
    if (ep.mask) return !ep.add && !ep.bias && !ep.relu && (ep.mask_bf16 != 0) == (sizeof(XT) == 2) && whole(ep.mask, ep.ldm);
    if (ep.add) return !ep.bias && !ep.relu && sizeof(XT) == 4 && whole(ep.add, ep.ldadd);
    return true;
}

template <int G, typename XT>
int launch_short_g(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, spmm_panel_args a, const spmm_epi &ep, hipStream_t st)
{
    constexpr int W = G * panel_vec<XT>::VEC, NE = 64 / G;
    a.panels = (a.d + W - 1) / W;
    a.interleave = a.panels;                   // one or two
    // How many blocks of rows and pieces there are is known on the device only: workgroups for blocks of four rows a group and a wavefront each
    // for 2048 pieces, the wavefronts stride over what is left.  Workgroups without a block cost as well: 32768 x 2.9, 256 fp32
    // columns, with 8192 a panel 30 us, with the 1540 of this rule 21.
    const uint64_t want = cdiv(A->rows, (SPMM_NT / 64) * NE * SHORT_ROWS / 2) + std::min<uint64_t>(cdiv(a.max_chunks, SPMM_NT / 64), 512);
    const unsigned grid = (unsigned)std::min<uint64_t>(want, SHORT_GRID) * (unsigned)a.interleave;
    char tag[56];
    snprintf(tag, sizeof(tag), "%ux%u d=%d G=%d in=%d out=%d%s", A->rows, A->cols, a.d, G, (int)sizeof(XT), ep.out_bf16 ? 2 : 4,
             ep.mask ? (ep.mask_bf16 ? " m=2" : " m=4") : "");
    const bool off32 = !a.row_index && (uint64_t)A->cols * (uint64_t)a.ldx * sizeof(XT) <= 0xffffffffull;
#define SGNN_SHORT(E)                                                                                                                        \
    do {                                                                                                                                     \
        if (off32) SGNN_LAUNCH(ctx, st, "spmm_short_kernel", tag, (spmm_short_kernel<G, XT, true, E>), dim3(grid), dim3(SPMM_NT), 0, st, a, X, ep); \
        else SGNN_LAUNCH(ctx, st, "spmm_short_kernel", tag, (spmm_short_kernel<G, XT, false, E>), dim3(grid), dim3(SPMM_NT), 0, st, a, X, ep);      \
    } while (0)
    if (ep.mask) SGNN_SHORT(SHORT_MASK);
    else if (ep.bias || ep.relu) SGNN_SHORT(SHORT_BIAS);
    else if (!ep.add) SGNN_SHORT(SHORT_PLAIN);
    else if constexpr (sizeof(XT) == 4) SGNN_SHORT(SHORT_ADD);
#undef SGNN_SHORT
    return SGNN_OK;
}

// columns of a partial row: whole panels
template <typename XT> int spmm_short_frame(int64_t d)
{
    constexpr int VEC = panel_vec<XT>::VEC;
    const int w = (d <= 8 * VEC ? 8 : (d <= 16 * VEC ? 16 : 32)) * VEC;
    return (int)((d + w - 1) / w) * w;
}

template <typename XT>
int launch_short(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, const int32_t *row_index, int d, float *out, int64_t ldo,
                 const spmm_epi &ep, uint32_t mean_limit, ws_alloc *ws, hipStream_t st)
{
    constexpr int VEC = panel_vec<XT>::VEC;
    spmm_panel_args a = {};
    if (!panel_args(a, A, ldx, row_index, d, spmm_short_frame<XT>(d), out, ldo, ep, ws))
        return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm: scratch too small (%zu bytes needed): call sgnn_ctx_reserve", ws->off);
    a.mean_limit = mean_limit;
    if (d <= 8 * VEC) return launch_short_g<8, XT>(ctx, A, X, a, ep, st);
    if (d <= 16 * VEC) return launch_short_g<16, XT>(ctx, A, X, a, ep, st);
    return launch_short_g<32, XT>(ctx, A, X, a, ep, st);
}

// The loss in the epilogue: a group of lanes holds the whole row
template <typename XT> int xent_frame(int64_t d)
{
    constexpr int VEC = panel_vec<XT>::VEC;
    return d < VEC || d > 32 * VEC ? 0 : spmm_short_frame<XT>(d);
}

// Workgroups: each leaves a row of partial sums to the final kernel.  Twice what the chip holds at four a compute unit.  us with 4096 / 2048 / 1536 /
// 1024: 2^20 x 1.27, 172 columns 332 / 331 / 335 / 342, 47 columns 135 / 129 / 135 / 131; 2^18 x 6.4, 47 columns 89 / 88 / 86 / 80, fp32 91 / 83 / 95 / 82.
inline unsigned spmm_short_xent_grid(const sgnn_csr *A) { return std::min<unsigned>(cdiv(A->rows, 64) + 512u, 2048u); }

template <int G, typename XT, int VEC = panel_vec<XT>::VEC>
int launch_short_xent_g(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, const spmm_panel_args &a, const spmm_epi &ep, hipStream_t st)
{
    char tag[56];
    snprintf(tag, sizeof(tag), "%ux%u d=%d G=%d in=%d out=%d xent dO=%d", A->rows, A->cols, a.d, G, (int)sizeof(XT), ep.write_out ? 4 : 0,
             ep.dO ? (ep.dO_bf16 ? 2 : 4) : 0);
    const unsigned grid = spmm_short_xent_grid(A);
    const bool off32 = (uint64_t)A->cols * (uint64_t)a.ldx * sizeof(XT) <= 0xffffffffull;
    if (off32) SGNN_LAUNCH(ctx, st, "spmm_short_kernel", tag, (spmm_short_kernel<G, XT, true, SHORT_XENT, VEC>), dim3(grid), dim3(SPMM_NT), 0, st, a, X, ep);
    else SGNN_LAUNCH(ctx, st, "spmm_short_kernel", tag, (spmm_short_kernel<G, XT, false, SHORT_XENT, VEC>), dim3(grid), dim3(SPMM_NT), 0, st, a, X, ep);
    return SGNN_OK;
}

template <typename XT>
int launch_short_xent(sgnn_ctx *ctx, const sgnn_csr *A, const XT *X, int64_t ldx, int d, float *out, int64_t ldo, const spmm_epi &ep, ws_alloc *ws,
                      hipStream_t st)
{
    constexpr int VEC = panel_vec<XT>::VEC;
    spmm_panel_args a = {};
    if (!panel_args(a, A, ldx, nullptr, d, spmm_short_frame<XT>(d), out, ldo, ep, ws))
        return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_spmm_xent: scratch too small (%zu bytes needed): call sgnn_ctx_reserve", ws->off);
    a.panels = a.interleave = 1;
    const int g = d <= 8 * VEC ? 8 : (d <= 16 * VEC ? 16 : 32);
    // six values a lane where as many lanes cover the row with them: the epilogue's instructions are per value of a lane, used or not
    // (172 columns: 29 of 32 lanes instead of 22)
    if constexpr (sizeof(XT) == 2) {
        if (d > 4 * g && d <= 6 * g) {
            if (g == 8) return launch_short_xent_g<8, XT, 6>(ctx, A, X, a, ep, st);
            if (g == 16) return launch_short_xent_g<16, XT, 6>(ctx, A, X, a, ep, st);
            return launch_short_xent_g<32, XT, 6>(ctx, A, X, a, ep, st);
        }
    }
    if (g == 8) return launch_short_xent_g<8, XT>(ctx, A, X, a, ep, st);
    if (g == 16) return launch_short_xent_g<16, XT>(ctx, A, X, a, ep, st);
    return launch_short_xent_g<32, XT>(ctx, A, X, a, ep, st);
}
