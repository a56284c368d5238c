// Induced, normalised, rescaled mini-batch subgraph as CSR (Sec. III-D, Eqs. 21-24; the full-range
// case of Algorithm 2).
//
// The sampled rows of the full CSR are treated as one flat edge sequence of length
// F = sum_{v in S} deg(v), cut into tiles of 2048 edges, one workgroup per tile, so the work per
// workgroup does not depend on the degree distribution (a hub row of 10^5 edges is spread over
// many workgroups; thousands of short rows share one).  Membership of a column in S is one bit
// test in the sampler's bitmap; its compact id is the sampler's rank prefix plus a popcount.
// Because the output CSR is in the same order as the flat sequence, the output position of a
// surviving edge is (survivors in earlier tiles) + (survivors before it inside the tile):
//
//   1. induced_deg_kernel      row length of every sampled row and per-workgroup sums
//   2. induced_offsets_kernel  flat offsets P[B+1] (exclusive prefix of the row lengths)
//   3. induced_count_kernel    survivors per tile (wave ballots / popcounts)
//   4. prefix sum              survivors in earlier tiles, for every tile; only where many tiles are expected, otherwise
//                              each workgroup of pass 5 adds up the counts of the tiles before its own
//   5. induced_fill_kernel     survivors only (keep words of pass 3): ordered compaction, colidx, val, rowptr
//   6. induced_renorm_kernel   only for norm_mode 1: weights from the degrees of the induced graph
// A tile marks the starts of the rows it touches in a bit mask of its 2048 edges in LDS, so finding the row of an
// edge is a count of bits (tile_table).
#include <algorithm>

#include "block_prims.h"
#include "common.h"

namespace {

constexpr int IND_NT = 256;
constexpr int IND_ITEMS = 8;
constexpr int IND_TILE = IND_NT * IND_ITEMS;      // 2048 flat edges per workgroup (4096 and 8192 with 512 threads measured slower)
constexpr int IND_WORDS = IND_ITEMS * (IND_NT / 64);   // 64-bit keep words of a tile: one per slab and wavefront
// Rows a tile's LDS table holds, less one (more only when rows average under two edges).  9 KB in the count pass, 19 KB in
// the fill pass: LDS does not limit occupancy.  With 512 about half of the tiles of a graph with six edges a row, most of
// them far fewer, went to the searches in global memory: 10^6 rows of 4 10^7, count pass 91 us against 53, fill pass 44
// against 36; with 2048 the fill pass loses occupancy and nothing is gained.
constexpr int IND_ROWS = 1024;
constexpr int IND_FILL_SLOTS = 2;                 // survivors a thread of the fill pass works on at a time (4 spill: 35 -> 62 us)
constexpr unsigned IND_MAX_GRID = 8192;
// Expected tiles up to which a workgroup of the fill pass adds up the survivors of the tiles before its own, instead of
// reading a prefix sum that launches of their own have written.  271 tiles: fill pass 7.6 -> 7.7 us and a launch of 3.5 us
// less; 6570 tiles: 34 -> 46 us for 6.5 us less, so that is no gain.  Where the prefix sum takes three launches
// (room for more than 65536 tiles, which are those of the whole graph), 2930 tiles: 37 -> 40 us for 14 us less.  Between and beyond,
// all launches together: 976 tiles 43 us, 52 with the prefix sum's launch; 1952 tiles 66 and 66; 4052 tiles 86, 98 with three;
// 5859 tiles 114, 111 with three.
constexpr uint64_t IND_OWN_PREFIX = 1024, IND_OWN_PREFIX_3 = 4096;
// The number of tiles is known on the device only, and a sample of the highest degrees has many times the expected ones.  Where there
// are more than IND_MANY the count pass therefore sums them up in groups of 256 as well, so that a workgroup reads at most its own
// group's tiles and one count for each group before it: 40000 rows of 4 10^6 vertices, 966 tiles expected, 23662 there, fill pass
// 128 -> 78 us.  Below, the atomic additions of the groups cost more than they save (4052 tiles: count pass 44 -> 61 us, fill pass 26 -> 24).
constexpr unsigned IND_GROUP = IND_NT;
constexpr uint64_t IND_MANY = 8192;
constexpr int DEG_TILE = 2048;                    // sampled rows per workgroup in the offset kernels

// Row and column range of a shard (Algorithm 2: [R0, R1) x [C0, C1) in global vertex ids); the whole graph by default.
struct shard_range { int64_t r0, r1, c0, c1; };

// Coarse membership filter for sparse samples of large graphs: one byte per bitmap word, bit b set iff byte b of the
// word holds a sampled vertex (1 bit per 8 vertices).  With a sample of 1 % of 10^8 vertices the 14 MB bitmap does not
// stay in a 4 MB L2 and every edge's probe is a cache-line fetch from further away; the filter (N / 64 bytes) does stay,
// and turns away the 93 % of the edges whose eight-vertex group holds no sampled vertex at all.
// Workgroups wg of n_wg, 256 threads each.
__device__ __forceinline__ void coarse_filter(const uint64_t *__restrict__ bitmap, uint64_t W, uint8_t *__restrict__ coarse,
                                              unsigned wg, unsigned n_wg)
{
    for (uint64_t w = (uint64_t)wg * 256 + threadIdx.x; w < W; w += (uint64_t)n_wg * 256) {
        const uint64_t x = bitmap[w];
        uint32_t c = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) c |= ((x >> (8 * b)) & 0xffull) ? (1u << b) : 0u;
        coarse[w] = (uint8_t)c;
    }
}

// The first n_deg_wg workgroups take the rows; those behind them build the coarse filter meanwhile, which no row needs
// (a launch of its own was 5 us; these hide behind the gathers of the row lengths).
// plan_count: piece counter of the plan that will be attached to the result, cleared here instead of in a launch of its own (or null);
// so are the n_groups survivor counts of the tile groups.
template <class RP>
__global__ __launch_bounds__(256) void induced_deg_kernel(const RP *__restrict__ rowptr, const int32_t *__restrict__ S,
                                                          uint32_t B, shard_range rg, uint32_t *__restrict__ deg,
                                                          int64_t *__restrict__ rowstart, uint64_t *__restrict__ wg_sum,
                                                          unsigned long long *__restrict__ total64, uint32_t *__restrict__ plan_count,
                                                          uint32_t *__restrict__ group_total, unsigned n_groups, unsigned n_deg_wg, const uint64_t *__restrict__ bitmap, uint64_t W,
                                                          uint8_t *__restrict__ coarse)
{
    if (blockIdx.x >= n_deg_wg) {
        coarse_filter(bitmap, W, coarse, blockIdx.x - n_deg_wg, gridDim.x - n_deg_wg);
        return;
    }
    if (plan_count && blockIdx.x == 0 && threadIdx.x == 0) *plan_count = 0u;
    for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < n_groups; i += n_deg_wg * 256) group_total[i] = 0u;
    __shared__ uint64_t lds[256 / 64];
    if (blockIdx.x == 0 && threadIdx.x == 0) *total64 = 0ull;     // survivors of the whole mini-batch, summed by the count pass
    uint64_t s = 0;
    // every load unconditional (a thread behind the last row repeats it), so that a thread's eight pairs of gathers are in
    // flight together: 2^18 rows of 2.4 M vertices 9 -> 7 us (10^6 rows of 4 10^7 stay at 27: a memory line for every row)
    int32_t v[DEG_TILE / 256];
    int64_t rs[DEG_TILE / 256], re[DEG_TILE / 256];
#pragma unroll
    for (int k = 0; k < DEG_TILE / 256; ++k) v[k] = S[min(blockIdx.x * DEG_TILE + k * 256 + threadIdx.x, B - 1)];
#pragma unroll
    for (int k = 0; k < DEG_TILE / 256; ++k) { rs[k] = (int64_t)rowptr[v[k]]; re[k] = (int64_t)rowptr[(int64_t)v[k] + 1]; }
#pragma unroll
    for (int k = 0; k < DEG_TILE / 256; ++k) {
        const uint32_t i = blockIdx.x * DEG_TILE + k * 256 + threadIdx.x;
        // a sampled row outside the shard's row range contributes no edge: it comes out as an empty row
        const uint32_t dgr = (v[k] >= rg.r0 && v[k] < rg.r1) ? (uint32_t)(re[k] - rs[k]) : 0u;
        if (i < B) {
            deg[i] = dgr;
            rowstart[i] = rs[k];   // kept for the tile kernels: no second gather through S
            s += dgr;
        }
    }
    const uint64_t t = block_sum<uint64_t, 256>(s, lds);
    if (threadIdx.x == 0) wg_sum[blockIdx.x] = t;
}

// Also tells every tile of IND_TILE flat edges which row its first edge belongs to: the row that covers the
// flat offset c * IND_TILE writes its number to tile_row[c] (a hub row covers many tile starts, most rows
// none), so that the tile kernels need no search for their first row.
__global__ __launch_bounds__(256) void induced_offsets_kernel(const uint32_t *__restrict__ deg, uint32_t B,
                                                              const uint64_t *__restrict__ wg_sum,
                                                              uint64_t *__restrict__ P, uint32_t *__restrict__ tile_row)
{
    __shared__ uint64_t lds[256 / 64 + 1];
    uint64_t part = 0;
    for (unsigned i = threadIdx.x; i < blockIdx.x; i += 256) part += wg_sum[i];
    const uint64_t base = block_sum<uint64_t, 256>(part, lds);
    // blocked arrangement: thread t owns rows i0 .. i0+7
    const uint32_t i0 = blockIdx.x * DEG_TILE + threadIdx.x * (DEG_TILE / 256);
    uint32_t d[DEG_TILE / 256];
    uint64_t s = 0;
#pragma unroll
    for (int k = 0; k < DEG_TILE / 256; ++k) {
        d[k] = (i0 + k < B) ? deg[i0 + k] : 0u;
        s += d[k];
    }
    uint64_t total;
    uint64_t ex = block_excl_scan<uint64_t, 256>(s, &total, lds) + base;
#pragma unroll
    for (int k = 0; k < DEG_TILE / 256; ++k) {
        if (i0 + k < B) {
            P[i0 + k] = ex;
            for (uint64_t c = (ex + IND_TILE - 1) / IND_TILE; c * IND_TILE < ex + d[k]; ++c) tile_row[c] = i0 + k;
        }
        ex += d[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) P[B] = base + total;
}

// largest r in [lo, hi] with P[r] <= f   (P[lo] <= f is guaranteed by the caller)
__device__ __forceinline__ uint32_t find_row(const uint64_t *__restrict__ P, uint32_t lo, uint32_t hi, uint64_t f)
{
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        if (P[mid] <= f) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Per-tile row table in LDS.  Rows r_lo .. r_lo+nr-1 intersect the tile [f0, f1); those with entries in it are numbered
// in order, and
//   start[w]  bit b is set iff such a row starts at offset 64 w + b of the tile (one that starts in front of it: offset 0)
//   ebase[j]  = rowptr[S[r]] - P[r] for the j-th of them: the position in colidx of flat edge f of that row is ebase + f
// The row of an edge is the number of start bits at or below its offset, minus one.  A wavefront's 64 edges of a slab lie
// in one word of `start`, so that is a count under a lane mask of a word and a prefix that are the same for the whole
// wavefront: no search.  (A binary search of the row starts was ten dependent rounds of LDS reads for each of the eight
// edges of a thread.)  What bounds the count pass then is the bit test of every edge, 13 M gathers of words that
// only an L2 holds, at about 250 a nanosecond: 2^18 rows of 2.4 M vertices, 66 -> 53 us (52 MB of column ids);
// 2^15 rows of 2^18 vertices, 12 -> 8 us.
// Two copies of `start`, used in turn: one is cleared for the next tile while the other is read.
// staged == false (more rows than the table holds: rows averaging under two edges, or the run of empty
// rows behind the last tile of a shard) falls back to searching P in global memory.
struct tile_table {
    unsigned long long start[2][IND_WORDS];
    int64_t ebase[IND_ROWS + 1];
};

// Rows r_lo .. r_lo + nr - 1 of a tile: from the row of its first edge to the row of the first edge of the next
// tile (which holds the tile's last edge, or starts right behind it and is then never found by the search);
// the last tile takes every row up to the last one.
__device__ __forceinline__ void tile_rows(const uint32_t *__restrict__ tile_row, uint64_t c, uint64_t n_tiles, uint32_t B,
                                          uint32_t &r_lo, uint32_t &nr)
{
    r_lo = c ? tile_row[c] : 0;        // the first tile also takes the empty rows in front of the first edge
    const uint32_t r_hi = c + 1 < n_tiles ? tile_row[c + 1] : B - 1;
    nr = r_hi - r_lo + 1;
}

// Staging of a tile's row table.  The first IND_NT rows arrive in registers: flat offset, first entry and length of row
// r_lo + threadIdx.x, requested while the tile before this one was being worked on (tile_prefetch), so that the two
// round trips that fetch a tile's rows - tile_row, then P / row starts / lengths - are off its critical path.
struct tile_pref {
    uint64_t p;
    int64_t rs;
    uint32_t d;
};

__device__ __forceinline__ tile_pref tile_prefetch(const int64_t *__restrict__ rowstart, const uint64_t *__restrict__ P,
                                                   const uint32_t *__restrict__ deg, bool valid, uint32_t r_lo, uint32_t nr)
{
    tile_pref t = {0, 0, 0};
    if (valid && threadIdx.x < nr && nr <= (uint32_t)IND_ROWS + 1) {
        t.p = P[r_lo + threadIdx.x];
        t.rs = rowstart[r_lo + threadIdx.x];
        t.d = deg[r_lo + threadIdx.x];
    }
    return t;
}

// Row starts of the tile as seen by a wavefront: lane w < IND_WORDS holds word w of `start` and the number of bits in
// the words before it.
struct tile_starts {
    uint64_t word;
    uint32_t pre;
};

// number of the row (among those with entries in the tile) of offset 64 wd + lane; wd is the same for the whole wavefront
__device__ __forceinline__ uint32_t row_of_lane(const tile_starts &ts, unsigned wd, unsigned lane)
{
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ts.word, (int)wd);
    const uint32_t w1 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(ts.word >> 32), (int)wd);
    const uint32_t pre = (uint32_t)__builtin_amdgcn_readlane((int)ts.pre, (int)wd);
    const uint64_t w = (uint64_t)w1 << 32 | w0;
    // the tile's first bit is always set, so the count is at least one
    return pre + __builtin_amdgcn_mbcnt_hi(w1, __builtin_amdgcn_mbcnt_lo(w0, 0u)) + (uint32_t)((w >> lane) & 1ull) - 1u;
}

// Two barriers; afterwards ebase (and row_no, if given: the row's index behind r_lo) can be read.  All of start[buf] is
// zero on entry; start[buf ^ 1] is on return.
template <bool ROW_NO>
__device__ __forceinline__ bool stage_tile(tile_table &tt, uint16_t *row_no, int buf, const tile_pref &pf,
                                           const int64_t *__restrict__ rowstart, const uint64_t *__restrict__ P,
                                           const uint32_t *__restrict__ deg, uint64_t f0, uint32_t tile_len, uint32_t r_lo,
                                           uint32_t nr, tile_starts &ts)
{
    const bool staged = nr <= (uint32_t)IND_ROWS + 1;
    // offset in the tile at which row k's entries start, -1 if it has none here
    auto offset = [&](uint32_t k, uint64_t p, uint32_t d) -> int32_t {
        const int64_t rel = (int64_t)p - (int64_t)f0;      // signed on purpose: the row may start in front of the tile
        return (k < nr && d != 0 && rel < (int64_t)tile_len) ? (int32_t)max(rel, (int64_t)0) : -1;
    };
    if (staged) {
        for (uint32_t k = threadIdx.x; k < nr; k += IND_NT) {
            const int32_t x = k < IND_NT ? offset(k, pf.p, pf.d) : offset(k, P[r_lo + k], deg[r_lo + k]);
            if (x >= 0) atomicOr(&tt.start[buf][x >> 6], 1ull << (x & 63));
        }
    }
    __syncthreads();
    const unsigned lane = lane_id();
    ts.word = lane < IND_WORDS ? tt.start[buf][lane] : 0ull;
    const uint32_t pc = (uint32_t)__popcll(ts.word);
    ts.pre = wave_incl_scan(pc) - pc;
    if (threadIdx.x < IND_WORDS) tt.start[buf ^ 1][threadIdx.x] = 0ull;
    if (staged) {
        for (uint32_t k0 = 0; k0 < nr; k0 += IND_NT) {         // every lane stays in the loop: the prefix is read across lanes
            const uint32_t k = k0 + threadIdx.x;
            uint64_t p = pf.p;
            int64_t rs = pf.rs;
            uint32_t d = pf.d;
            if (k0) {
                const uint32_t r = r_lo + min(k, nr - 1);
                p = P[r]; rs = rowstart[r]; d = deg[r];
            }
            const int32_t x = offset(k, p, d);
            const uint32_t pre = (uint32_t)__shfl((int)ts.pre, max(x, 0) >> 6);
            if (x >= 0) {
                const uint32_t j = pre + (uint32_t)__popcll(tt.start[buf][x >> 6] & ((1ull << (x & 63)) - 1ull));
                tt.ebase[j] = rs - (int64_t)p;
                if constexpr (ROW_NO) row_no[j] = (uint16_t)k;
            }
        }
    }
    __syncthreads();
    return staged;
}

__global__ __launch_bounds__(IND_NT) void induced_count_kernel(const int64_t *__restrict__ rowstart,
                                                               const uint32_t *__restrict__ deg,
                                                               const int32_t *__restrict__ colidx, uint32_t B,
                                                               const uint64_t *__restrict__ bitmap,
                                                               const uint8_t *__restrict__ coarse, shard_range rg,
                                                               const uint64_t *__restrict__ P,
                                                               const uint32_t *__restrict__ tile_row,
                                                               uint32_t *__restrict__ tile_total,
                                                               uint32_t *group_total,                   // or null
                                                               uint64_t *__restrict__ keepbits,
                                                               uint64_t *__restrict__ n_tiles_out,
                                                               unsigned long long *__restrict__ total64)
{
    __shared__ tile_table tt;
    __shared__ uint32_t wave_cnt[2][IND_NT / 64];
    const unsigned lane = lane_id(), wave = (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x < 2 * IND_WORDS) tt.start[threadIdx.x / IND_WORDS][threadIdx.x % IND_WORDS] = 0ull;
    __syncthreads();
    // column range of the shard in 32 bits: column ids are below 2^31
    const uint32_t c_lo = (uint32_t)min(max(rg.c0, (int64_t)0), (int64_t)1 << 31);
    const uint32_t c_n = (uint32_t)min(max(rg.c1, (int64_t)c_lo), (int64_t)1 << 31) - c_lo;
    const uint64_t F = P[B];
    const uint64_t n_tiles = (F + IND_TILE - 1) / IND_TILE;
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_tiles_out = n_tiles;
    if (n_tiles <= IND_MANY) group_total = nullptr;
    unsigned long long wg_total = 0;      // 64 bits: the 32-bit prefix over the tile counts wraps beyond 2^32 survivors
    // software pipeline over the workgroup's tiles: the rows of the tile after next and the table of the next tile are
    // requested before the current tile's edges are gathered
    const uint64_t g = gridDim.x;
    uint32_t r_lo = 0, nr = 0, r_lo1 = 0, nr1 = 0;
    if (blockIdx.x < n_tiles) tile_rows(tile_row, blockIdx.x, n_tiles, B, r_lo, nr);
    if (blockIdx.x + g < n_tiles) tile_rows(tile_row, blockIdx.x + g, n_tiles, B, r_lo1, nr1);
    tile_pref pf = tile_prefetch(rowstart, P, deg, blockIdx.x < n_tiles, r_lo, nr);
    int buf = 0;
    for (uint64_t c = blockIdx.x; c < n_tiles; c += g, buf ^= 1) {
        const uint64_t f0 = c * IND_TILE;
        const uint32_t tile_len = (uint32_t)(min(F, f0 + IND_TILE) - f0);
        tile_starts ts;
        const bool staged = stage_tile<false>(tt, nullptr, buf, pf, rowstart, P, deg, f0, tile_len, r_lo, nr, ts);
        uint32_t r_lo2 = 0, nr2 = 0;
        if (c + 2 * g < n_tiles) tile_rows(tile_row, c + 2 * g, n_tiles, B, r_lo2, nr2);
        pf = tile_prefetch(rowstart, P, deg, c + g < n_tiles, r_lo1, nr1);
        // Branch-free, one step for all eight edges at a time, and every load unconditional (an edge that does not need
        // it reads an address that some other one reads): the gathers of a step are then in flight together.  A
        // load that only some lanes want is compiled to a branch and a wait for the load before it.
        int32_t u[IND_ITEMS];
        if (staged) {
            int64_t e[IND_ITEMS];
#pragma unroll
            for (int k = 0; k < IND_ITEMS; ++k) {
                const uint32_t x = k * IND_NT + threadIdx.x;
                const bool in = x < tile_len;                   // an offset behind the end of the last tile reads the tile's first edge
                const uint32_t j = row_of_lane(ts, k * (IND_NT / 64) + wave, lane);
                e[k] = tt.ebase[in ? j : 0u] + (int64_t)(f0 + (in ? x : 0u));
            }
#pragma unroll
            for (int k = 0; k < IND_ITEMS; ++k) u[k] = colidx[e[k]];
        } else {
#pragma unroll 1
            for (int k = 0; k < IND_ITEMS; ++k) {
                const uint32_t x = k * IND_NT + threadIdx.x;
                const uint64_t f = f0 + (x < tile_len ? x : 0u);
                const uint32_t r = find_row(P, r_lo, r_lo + nr - 1, f);
                const int32_t q = colidx[rowstart[r] + (int64_t)(f - P[r])];
#pragma unroll
                for (int kk = 0; kk < IND_ITEMS; ++kk) u[kk] = kk == k ? q : u[kk];
            }
        }
        // no edge, or a column outside the shard: its column reads as vertex 0 and its keep bit is taken back below
        bool in[IND_ITEMS];
#pragma unroll
        for (int k = 0; k < IND_ITEMS; ++k) {
            in[k] = (k * IND_NT + threadIdx.x < tile_len) & ((uint32_t)u[k] - c_lo < c_n);
            u[k] = in[k] ? u[k] : 0;
        }
        if (coarse) {
            // the filter first (all eight probes in flight), the bitmap only for the edges it lets through (the others
            // share the first word)
            uint32_t cf[IND_ITEMS];
#pragma unroll
            for (int k = 0; k < IND_ITEMS; ++k) cf[k] = coarse[(uint32_t)u[k] >> 6];
#pragma unroll
            for (int k = 0; k < IND_ITEMS; ++k) {
                in[k] = in[k] & (((cf[k] >> (((uint32_t)u[k] >> 3) & 7)) & 1u) != 0u);
                u[k] = in[k] ? u[k] : 0;
            }
        }
        uint64_t word[IND_ITEMS];
#pragma unroll
        for (int k = 0; k < IND_ITEMS; ++k) word[k] = bitmap[(uint32_t)u[k] >> 6];
        // one keep word per slab and wavefront, kept for the fill pass; the count is their popcount
        uint32_t cnt = 0;
        uint64_t mine = 0;
#pragma unroll
        for (int k = 0; k < IND_ITEMS; ++k) {
            const uint64_t bal = __ballot(in[k] & (((word[k] >> (u[k] & 63)) & 1ull) != 0ull));
            cnt += (uint32_t)__popcll(bal);
            mine = lane == (unsigned)k ? bal : mine;
        }
        if (lane < IND_ITEMS) keepbits[c * IND_WORDS + lane * (IND_NT / 64) + wave] = mine;
        if (lane == 0) wave_cnt[buf][wave] = cnt;
        __syncthreads();       // also: the row table may be reused
        if (threadIdx.x == 0) {
            uint32_t t = 0;
#pragma unroll
            for (int w = 0; w < IND_NT / 64; ++w) t += wave_cnt[buf][w];
            tile_total[c] = t;
            if (group_total && t) atomicAdd(&group_total[c / IND_GROUP], t);
            wg_total += t;
        }
        r_lo = r_lo1; nr = nr1; r_lo1 = r_lo2; nr1 = nr2;
    }
    if (threadIdx.x == 0 && wg_total) atomicAdd(total64, wg_total);     // integer: the sum does not depend on the order
}

// Fill pass.  The keep words of the count pass say which edges survive, so only survivors are looked at again:
// position = survivors in earlier tiles + survivors before the edge in the tile (prefix over the popcounts of
// the tile's keep words).  Row offsets come from the row side: every row that starts inside the tile gets the
// position of the first survivor at or behind its start, which also covers rows without any stored entry.
// OWN_PREFIX: tile_off_all holds the counts of the tiles themselves, group_total those of the groups of tiles, and the workgroup
// adds up those before its tile.
template <class RP, bool OWN_PREFIX>
__global__ __launch_bounds__(IND_NT) __attribute__((amdgpu_waves_per_eu(7, 7))) void induced_fill_kernel(
    const RP *__restrict__ rowptr, const int32_t *__restrict__ colidx, const float *__restrict__ gval,
    const int32_t *__restrict__ S, const int64_t *__restrict__ rowstart, const uint32_t *__restrict__ deg, uint32_t B,
    const uint64_t *__restrict__ bitmap, const uint32_t *__restrict__ rank, const uint64_t *__restrict__ P,
    const uint32_t *__restrict__ tile_row, const uint32_t *__restrict__ tile_off_all, const uint32_t *__restrict__ group_total, const uint64_t *__restrict__ n_tiles_p, const uint64_t *__restrict__ keepbits, float inv_p, int write_val,
    int32_t *__restrict__ rowptr_S, int32_t *__restrict__ colidx_S, float *__restrict__ val_S, uint64_t capacity,
    uint32_t *__restrict__ nnz_dev, uint32_t *__restrict__ status, const unsigned long long *__restrict__ total64,
    int sticky_capacity, int deg_by_rank)
{
    __shared__ tile_table tt;
    __shared__ uint16_t row_no[IND_ROWS + 1];
    __shared__ uint64_t balw[IND_WORDS];
    __shared__ uint32_t pre[IND_WORDS + 1];
    __shared__ uint32_t xs[IND_TILE];
    __shared__ uint32_t sum_lds[IND_NT / 64];
    const uint64_t F = P[B];
    const uint64_t n_tiles = *n_tiles_p;
    const unsigned lane = lane_id(), wave = (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x < 2 * IND_WORDS) tt.start[threadIdx.x / IND_WORDS][threadIdx.x % IND_WORDS] = 0ull;
    __syncthreads();
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            const unsigned long long t64 = *total64;
            const uint32_t total = (uint32_t)t64;
            if (t64 > 0x7fffffffull) atomicOr(status, SGNN_ST_NNZ_OVERFLOW);
            // entries beyond the capacity are dropped below: without a host read-back of the count the caller learns
            // of it through the sticky status word (sgnn_ctx_status)
            if (sticky_capacity && t64 > capacity) atomicOr(status, SGNN_ST_CAPACITY_OVERFLOW);
            rowptr_S[B] = (int32_t)total;
            if (nnz_dev) *nnz_dev = total;
        }
        if (n_tiles == 0)       // not a single edge: every row is empty
            for (uint32_t r = threadIdx.x; r < B; r += IND_NT) rowptr_S[r] = 0;
    }
    // software pipeline over the workgroup's tiles, as in the count pass: the next tile's keep words, offset and row
    // table are requested while the current tile's survivors are gathered
    const uint64_t g = gridDim.x;
    uint32_t r_lo = 0, nr = 0, r_lo1 = 0, nr1 = 0;
    if (blockIdx.x < n_tiles) tile_rows(tile_row, blockIdx.x, n_tiles, B, r_lo, nr);
    if (blockIdx.x + g < n_tiles) tile_rows(tile_row, blockIdx.x + g, n_tiles, B, r_lo1, nr1);
    tile_pref pf = tile_prefetch(rowstart, P, deg, blockIdx.x < n_tiles, r_lo, nr);
    uint64_t kw = 0;               // wavefront 0: keep word `lane` of the tile
    uint32_t tile_off = 0;         // survivors in earlier tiles (exclusive prefix of the tile counts)
    // OWN_PREFIX: survivors of the tiles before tile c, every thread; `off` are those of the tiles before tile a.  Wrapping 32-bit
    // sums, as the prefix sum's.
    auto before_tile = [&](uint64_t c, uint64_t a, uint32_t off) -> uint32_t {
        uint64_t n_groups = 0;
        if (n_tiles > IND_MANY) {
            n_groups = c / IND_GROUP;
            a = n_groups * IND_GROUP;
            off = 0;
        }
        uint32_t t = 0;
#pragma unroll 1
        for (uint64_t i = a + threadIdx.x; i < c; i += IND_NT) t += tile_off_all[i];
#pragma unroll 1
        for (uint64_t i = threadIdx.x; i < n_groups; i += IND_NT) t += group_total[i];
        return off + block_sum<uint32_t, IND_NT>(t, sum_lds);
    };
    if (blockIdx.x < n_tiles) {
        if (wave == 0 && lane < IND_WORDS) kw = keepbits[(uint64_t)blockIdx.x * IND_WORDS + lane];
        tile_off = OWN_PREFIX ? before_tile(blockIdx.x, 0, 0) : tile_off_all[blockIdx.x];
    }
    int buf = 0;
    for (uint64_t c = blockIdx.x; c < n_tiles; c += g, buf ^= 1) {
        const uint64_t f0 = c * IND_TILE;
        const uint32_t tile_len = (uint32_t)(min(F, f0 + IND_TILE) - f0);
        const bool last = c + 1 == n_tiles;
        if (wave == 0) {
            const uint64_t w = lane < IND_WORDS ? kw : 0ull;
            if (lane < IND_WORDS) balw[lane] = w;
            const uint32_t pc = (uint32_t)__popcll(w);
            const uint32_t inc = wave_incl_scan(pc);
            if (lane < IND_WORDS) pre[lane] = inc - pc;
            if (lane == IND_WORDS - 1) pre[IND_WORDS] = inc;
        }
        tile_starts ts;
        const bool staged = stage_tile<true>(tt, row_no, buf, pf, rowstart, P, deg, f0, tile_len, r_lo, nr, ts);     // ends with a barrier
        const uint32_t tile_off_cur = tile_off;
        const uint64_t p_cur = pf.p;
        uint32_t r_lo2 = 0, nr2 = 0;
        if (c + 2 * g < n_tiles) tile_rows(tile_row, c + 2 * g, n_tiles, B, r_lo2, nr2);
        pf = tile_prefetch(rowstart, P, deg, c + g < n_tiles, r_lo1, nr1);
        if (c + g < n_tiles) {
            if (wave == 0 && lane < IND_WORDS) kw = keepbits[(c + g) * IND_WORDS + lane];
            tile_off = OWN_PREFIX ? before_tile(c + g, c, tile_off_cur) : tile_off_all[c + g];
        }

        // Survivors, in their order: the flat offsets of the set bits of the keep words are written to a list in LDS, each
        // with the number of its row, and thread i takes survivor i, i + 256, ... (IND_FILL_SLOTS of them at a time).
        // A thread then holds the state of a few survivors instead of one slot for each of its eight edges, of which one
        // in eight survives on a typical mini-batch: half the registers, twice the tiles in flight on a compute unit.
#pragma unroll
        for (int k = 0; k < IND_ITEMS; ++k) {
            const uint32_t wd = k * (IND_NT / 64) + wave;
            const uint64_t w = balw[wd];
            const uint32_t at = pre[wd] + __builtin_amdgcn_mbcnt_hi((uint32_t)(w >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)w, 0u));
            const uint32_t j = row_of_lane(ts, wd, lane);       // no meaning in a tile that is not staged, and not used there
            if ((w >> lane) & 1ull) xs[at] = (k * IND_NT + threadIdx.x) | j << 16;
        }

        // row offsets.  A row that starts right at the end of the tile is empty if it is not the row the next
        // tile begins with (that tile writes that one); behind the last tile every such row is empty.
        for (uint32_t k = threadIdx.x; k < nr; k += IND_NT) {
            const int64_t x = (int64_t)(staged && k < IND_NT ? p_cur : P[r_lo + k]) - (int64_t)f0;
            if (x < 0) continue;
            if (x < (int64_t)tile_len) {
                const uint32_t wd = (uint32_t)x >> 6;
                rowptr_S[r_lo + k] = (int32_t)(tile_off_cur + pre[wd] + (uint32_t)__popcll(balw[wd] & ((1ull << (x & 63)) - 1ull)));
            } else if (x == (int64_t)tile_len && (last || k + 1 < nr)) rowptr_S[r_lo + k] = (int32_t)(tile_off_cur + pre[IND_WORDS]);
        }
        __syncthreads();
        const uint32_t n_surv = pre[IND_WORDS];
        for (uint32_t i0 = 0; i0 < n_surv; i0 += IND_FILL_SLOTS * IND_NT) {
            // Every load is unconditional: a slot behind the last survivor repeats it, and only the stores are guarded.
            uint32_t r[IND_FILL_SLOTS];
            int64_t e[IND_FILL_SLOTS];
#pragma unroll
            for (int k = 0; k < IND_FILL_SLOTS; ++k) {
                const uint32_t q = xs[min(i0 + k * IND_NT + threadIdx.x, n_surv - 1)];
                const uint64_t f = f0 + (q & 0xffffu);
                if (staged) {
                    e[k] = tt.ebase[q >> 16] + (int64_t)f;
                    r[k] = r_lo + row_no[q >> 16];
                } else {
                    r[k] = find_row(P, r_lo, r_lo + nr - 1, f);
                    e[k] = rowstart[r[k]] + (int64_t)(f - P[r[k]]);
                }
            }
            int32_t u[IND_FILL_SLOTS], v[IND_FILL_SLOTS];
            uint32_t dr[IND_FILL_SLOTS];
            float gv[IND_FILL_SLOTS];
#pragma unroll
            for (int k = 0; k < IND_FILL_SLOTS; ++k) { u[k] = colidx[e[k]]; v[k] = S[r[k]]; dr[k] = deg[r[k]]; }
            if (write_val && gval) {
#pragma unroll
                for (int k = 0; k < IND_FILL_SLOTS; ++k) gv[k] = gval[e[k]];
            }
            // compact column ids; a surviving column is itself a sampled vertex, so with every sampled row inside the row
            // range its degree is already in deg[] (B entries, cache resident) and need not be gathered from rowptr
            uint64_t word[IND_FILL_SLOTS];
            uint32_t cid[IND_FILL_SLOTS];
#pragma unroll
            for (int k = 0; k < IND_FILL_SLOTS; ++k) { word[k] = bitmap[(uint32_t)u[k] >> 6]; cid[k] = rank[(uint32_t)u[k] >> 6]; }
#pragma unroll
            for (int k = 0; k < IND_FILL_SLOTS; ++k) cid[k] += (uint32_t)__popcll(word[k] & ((1ull << (u[k] & 63)) - 1ull));
            int64_t du[IND_FILL_SLOTS];
            if (write_val && !gval) {
                if (deg_by_rank) {
#pragma unroll
                    for (int k = 0; k < IND_FILL_SLOTS; ++k) du[k] = (int64_t)deg[min(cid[k], B - 1)];
                } else {
#pragma unroll
                    for (int k = 0; k < IND_FILL_SLOTS; ++k) du[k] = (int64_t)rowptr[(int64_t)u[k] + 1] - (int64_t)rowptr[u[k]];
                }
            }
#pragma unroll
            for (int k = 0; k < IND_FILL_SLOTS; ++k) {
                const uint32_t i = i0 + k * IND_NT + threadIdx.x;
                const uint32_t pos = tile_off_cur + i;
                if (i >= n_surv || pos >= capacity) continue;
                colidx_S[pos] = (int32_t)cid[k];
                if (write_val) {
                    float a;
                    if (gval) a = gv[k];
                    else {
                        // 1 / sqrt(deg(v) deg(u)) in single precision: product, reciprocal square root, one Newton step.
                        // Against the double-precision formula rounded once: a few 1e-7 relative (two roundings of
                        // 2^-24 here, one for 1/p, the Newton step leaves under one more), inside the 1e-6 the weights are held to.
                        // A row that holds an edge lies inside the row range: deg is its full length.
                        const float xx = (float)dr[k] * (float)du[k];
                        float y = __frsqrt_rn(xx);
                        const float err = fmaf(-xx * y, y, 1.0f);
                        a = fmaf(0.5f * y, err, y);
                    }
                    if (u[k] != v[k]) a *= inv_p;
                    val_S[pos] = a;
                }
            }
        }
        __syncthreads();   // the keep words and the row table are reused by the next tile
        r_lo = r_lo1; nr = nr1; r_lo1 = r_lo2; nr1 = nr2;
    }
}

// norm_mode 1: a_ij = 1/sqrt(c_i c_j) with c = entry counts of the induced rows, off-diagonal / p.
__global__ __launch_bounds__(256) void induced_renorm_kernel(const int32_t *__restrict__ rowptr_S,
                                                             const int32_t *__restrict__ colidx_S,
                                                             float *__restrict__ val_S, uint32_t B, uint64_t capacity,
                                                             double p)
{
    // a wavefront per row
    const uint32_t row = (blockIdx.x * 256 + threadIdx.x) >> 6;
    if (row >= B) return;
    const int64_t rs = rowptr_S[row], re = min((int64_t)rowptr_S[row + 1], (int64_t)capacity);
    const double ci = (double)(rowptr_S[row + 1] - rowptr_S[row]);
    for (int64_t e = rs + lane_id(); e < re; e += 64) {
        const int32_t j = colidx_S[e];
        const double cj = (double)(rowptr_S[j + 1] - rowptr_S[j]);
        double a = 1.0 / sqrt(ci * cj);
        if ((uint32_t)j != row) a /= p;
        val_S[e] = (float)a;
    }
}

template <class RP>
int launch_typed(sgnn_ctx *ctx, const sgnn_graph *g, const int32_t *S, uint32_t B, const uint64_t *bitmap,
                 const uint32_t *rank, int norm_mode, int rescale, shard_range rg, sgnn_csr *out, int sticky_capacity,
                 hipStream_t st)
{
    const RP *rowptr = static_cast<const RP *>(g->rowptr);
    ws_alloc ws(ctx);
    const uint64_t max_tiles = g->E / IND_TILE + 2;
    const unsigned n_deg_wg = cdiv(B, DEG_TILE);
    uint32_t *deg = ws.get<uint32_t>(B);
    int64_t *rowstart = ws.get<int64_t>(B);
    uint64_t *deg_sum = ws.get<uint64_t>(n_deg_wg);
    uint64_t *P = ws.get<uint64_t>((size_t)B + 1);
    uint32_t *tile_total = ws.get<uint32_t>(max_tiles);
    uint32_t *tile_row = ws.get<uint32_t>(max_tiles + 1);
    uint64_t *keepbits = ws.get<uint64_t>(max_tiles * IND_WORDS);
    uint32_t *tile_off = ws.get<uint32_t>(max_tiles + 1);
    uint32_t *scan_tmp = ws.get<uint32_t>(sgnn_scan_tmp_elems(max_tiles));
    uint64_t *n_tiles = ws.get<uint64_t>(1);
    unsigned long long *total64 = ws.get<unsigned long long>(1);
    // the coarse filter pays when the bitmap is far larger than an L2 and the sample is sparse
    const uint64_t W = (g->N + 63) / 64;
    const bool use_coarse = g->N >= (1ull << 24) && (uint64_t)B * 32 < g->N;
    uint8_t *coarse = use_coarse ? ws.get<uint8_t>(W) : nullptr;
    if (!ws.ok)
        return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_induced_csr: scratch too small (%zu bytes needed): call sgnn_ctx_reserve",
                         ws.off);

    const uint64_t expected_tiles = (uint64_t)((double)g->E * (double)B / (double)std::max<uint64_t>(g->N, 1) / IND_TILE);
    const bool own_prefix = expected_tiles <= (max_tiles > SGNN_SCAN_SINGLE_MAX ? IND_OWN_PREFIX_3 : IND_OWN_PREFIX);
    uint32_t *group_total = own_prefix ? tile_off : nullptr;        // no prefix sum then: its place is free
    const unsigned n_groups = own_prefix ? (unsigned)(max_tiles / IND_GROUP + 1) : 0u;
    const unsigned n_coarse_wg = use_coarse ? (unsigned)std::min<uint64_t>(cdiv(W, 1024), 1024) : 0u;
    SGNN_LAUNCH(ctx, st, "induced_deg_kernel", SGNN_TAG, induced_deg_kernel<RP>, dim3(n_deg_wg + n_coarse_wg), dim3(256), 0, st, rowptr, S, B,
                rg, deg, rowstart, deg_sum, total64, sgnn_spmm_plan_counter(out), group_total, n_groups, n_deg_wg, bitmap, W, coarse);
    SGNN_LAUNCH(ctx, st, "induced_offsets_kernel", SGNN_TAG, induced_offsets_kernel, dim3(n_deg_wg), dim3(256), 0, st, deg, B,
                deg_sum, P, tile_row);
    // Workgroups walk their tiles in a software pipeline (the next tile's row table is requested while the current
    // tile's edges are gathered).  Where the expected number of tiles, E B / N / 2048, is a few times the 2048
    // workgroups of the count pass that are resident at once, exactly those are launched (large graph: 94 -> 78 us);
    // with more tiles the larger grid measured better (the chip is then full anyway), as it does for the fill pass.
    const unsigned grid_fill = (unsigned)std::min<uint64_t>(max_tiles, IND_MAX_GRID);
    const unsigned grid = (expected_tiles >= 2048 && expected_tiles < IND_MAX_GRID) ? 2048u : grid_fill;
    SGNN_LAUNCH(ctx, st, "induced_count_kernel", SGNN_TAG, induced_count_kernel, dim3(grid), dim3(IND_NT), 0, st, rowstart, deg,
                g->colidx, B, bitmap, coarse, rg, P, tile_row, tile_total, group_total, keepbits, n_tiles, total64);
    if (!own_prefix) {
        const int rc = sgnn_scan_u32_devn(ctx, tile_total, tile_off, n_tiles, max_tiles, scan_tmp, st);
        if (rc) return rc;
    }
    double p = 1.0;
    if (rescale && B > 1) p = ((double)B - 1.0) / ((double)g->N - 1.0);
    SGNN_LAUNCH(ctx, st, "induced_fill_kernel", SGNN_TAG, (own_prefix ? induced_fill_kernel<RP, true> : induced_fill_kernel<RP, false>), dim3(grid_fill), dim3(IND_NT), 0, st, rowptr,
                g->colidx, norm_mode == 0 ? g->val : nullptr, S, rowstart, deg, B, bitmap, rank, P, tile_row, own_prefix ? tile_total : tile_off,
                group_total, n_tiles, keepbits, (float)(1.0 / p), norm_mode == 0 ? 1 : 0, out->rowptr, out->colidx, out->val,
                out->capacity, out->nnz_dev, ctx->status, total64, sticky_capacity,
                (rg.r0 <= 0 && rg.r1 >= (int64_t)g->N) ? 1 : 0);
    if (norm_mode == 1)
        SGNN_LAUNCH(ctx, st, "induced_renorm_kernel", SGNN_TAG, induced_renorm_kernel, dim3(cdiv((uint64_t)B * 64, 256)),
                    dim3(256), 0, st, out->rowptr, out->colidx, out->val, B, out->capacity, p);
    return SGNN_OK;
}

// Full graph as a matrix for the evaluation forward (Sec. VI: full-graph inference): int32 row offsets and
// the weights of Eq. 3, a_vu = 1 / sqrt(deg(v) deg(u)), evaluated in double precision and rounded once
// (the same arithmetic as the mini-batch weights).  One wavefront per row, grid-stride; a set-up kernel.
template <typename RP>
__global__ __launch_bounds__(256) void graph_normalize_kernel(uint64_t N, const RP *__restrict__ rowptr,
                                                              const int32_t *__restrict__ colidx,
                                                              const float *__restrict__ val_in, int32_t *__restrict__ rowptr32,
                                                              float *__restrict__ val)
{
    const int lane = threadIdx.x & 63;
    const uint64_t wave = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (uint64_t)gridDim.x * 4;
    for (uint64_t v = wave; v < N; v += nwaves) {
        const int64_t rs = (int64_t)rowptr[v], re = (int64_t)rowptr[v + 1];
        if (lane == 0 && rowptr32) {
            rowptr32[v] = (int32_t)rs;
            if (v + 1 == N) rowptr32[N] = (int32_t)re;
        }
        const double dv = (double)(re - rs);
        for (int64_t e = rs + lane; e < re; e += 64) {
            if (val_in) val[e] = val_in[e];
            else {
                const int64_t u = colidx[e];
                const double du = (double)((int64_t)rowptr[u + 1] - (int64_t)rowptr[u]);
                val[e] = (float)(1.0 / sqrt(dv * du));
            }
        }
    }
}

} // namespace

size_t sgnn_induced_ws_bytes(uint64_t N, uint64_t E, uint32_t B)
{
    const uint64_t max_tiles = E / IND_TILE + 2;
    return (size_t)(N + 63) / 64 + 256 + (size_t)B * 12 + ((size_t)B + 1) * 8 + (size_t)cdiv(B, DEG_TILE) * 8 + max_tiles * 4 + (max_tiles + 1) * 4 +
           max_tiles * IND_WORDS * 8 + (max_tiles + 1) * 4 + sgnn_scan_tmp_elems(max_tiles) * 4 + 16 + 13 * 256;
}

int sgnn_launch_induced(sgnn_ctx *ctx, const sgnn_graph *g, const int32_t *S, uint32_t B, const uint64_t *bitmap,
                        const uint32_t *rank, int norm_mode, int rescale, int64_t R0, int64_t R1, int64_t C0, int64_t C1,
                        sgnn_csr *out, int sticky_capacity, hipStream_t st)
{
    const shard_range rg = {R0, R1, C0, C1};
    if (g->rowptr_is_i64) return launch_typed<int64_t>(ctx, g, S, B, bitmap, rank, norm_mode, rescale, rg, out, sticky_capacity, st);
    return launch_typed<int32_t>(ctx, g, S, B, bitmap, rank, norm_mode, rescale, rg, out, sticky_capacity, st);
}

int sgnn_launch_graph_normalize(sgnn_ctx *ctx, const sgnn_graph *g, int32_t *rowptr32, float *val, hipStream_t st)
{
    if (g->N == 0) return SGNN_OK;
    const unsigned nwg = (unsigned)std::min<uint64_t>((g->N + 3) / 4, 1u << 16);
    if (g->rowptr_is_i64)
        SGNN_LAUNCH(ctx, st, "graph_normalize_kernel", SGNN_TAG, graph_normalize_kernel<int64_t>, dim3(nwg), dim3(256), 0, st, g->N,
                    static_cast<const int64_t *>(g->rowptr), g->colidx, g->val, rowptr32, val);
    else
        SGNN_LAUNCH(ctx, st, "graph_normalize_kernel", SGNN_TAG, graph_normalize_kernel<int32_t>, dim3(nwg), dim3(256), 0, st, g->N,
                    static_cast<const int32_t *>(g->rowptr), g->colidx, g->val, rowptr32, val);
    return SGNN_OK;
}
