// Uniform vertex sampling without replacement (Sec. III-D "Vertex Sampling", Eq. 20).
//
// The sample is the B vertices with the smallest (key(v), v), key(v) being 64 bits of
// Philox4x32-10 (Salmon et al., SC'11) counted by (v/2, step) and keyed by the seed.  Whole keys are
// never stored.  A pass that recomputes them is bound by the 20 quarter-rate 32 x 32 -> 64 multiplies
// of a Philox call (about 19 us per 2^23 calls, measured), three passes cost three times that; with
// scratch for two bytes per vertex the first pass also stores the top 16 bits of every key, and the
// later passes read those instead: they decide all but 2^-11 (candidates) and 2^-16 (ties with the
// threshold's prefix) of the vertices, and only for these is the key computed again.
//
//   1. sampler_hist_kernel     histogram of the top 11 key bits (LDS histograms, one merge)
//   2. sampler_collect_kernel  the bin b* that holds the B-th smallest key and the rank r inside (every workgroup for
//                              itself), and (key, v) of every vertex in bin b* -> candidate list (about N/2048)
//   3. sampler_threshold_kernel exact r-th smallest (key, v) of the candidates; up to 2^22 vertices a part of the next pass
//   4. sampler_emit_kernel     bitmap word per 64 vertices from wave ballots + per-workgroup counts
//   5. sampler_rank_kernel     rank prefix per bitmap word and the ascending list S
//
// Up to SMALL_N vertices one workgroup does all of it (sampler_small_kernel).  Sparse samples of large graphs know the bin of the threshold
// beforehand and go through the keys once: sampler_hist_window_kernel, sampler_mark_kernel, sampler_count_kernel, sampler_rank_kernel.
#include "block_prims.h"
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <mutex>

#include "common.h"
#include "philox.h"

namespace {

constexpr int HIST_BITS = 11;
constexpr int HIST_BINS = 1 << HIST_BITS;
constexpr int SAMP_NT = 256;
constexpr int SCAN_NT = 1024;            // key passes: few large workgroups, so that few of them meet on one address
constexpr unsigned EMIT_MAX_WG = 1024;

struct sampler_state {
    uint32_t bin;       // histogram bin of the threshold key
    uint32_t r;         // 1-based rank of the threshold inside that bin
    uint32_t ncand;     // candidates appended by the collect pass
    uint32_t thr_v;     // threshold vertex
    uint64_t thr_key;   // threshold key
    uint32_t fallback;  // windowed call whose threshold's bin fell outside the window
    uint32_t nfew;      // windowed call: candidates in the threshold's part of its bin
};

// Keys of vertices 2j (even) and 2j+1 (odd).  There are fewer than 2^31 vertices: the upper half of the counter's j is the constant 0, which
// leaves 18 of the 20 products to the vector unit.
__device__ __forceinline__ void vertex_pair_keys(uint64_t j, uint64_t seed, uint64_t step, uint64_t &ke, uint64_t &ko)
{
    philox_out o = philox4x32_10((uint32_t)j, 0u, (uint32_t)step, (uint32_t)(step >> 32),
                                 (uint32_t)seed, (uint32_t)(seed >> 32));
    ke = ((uint64_t)o.w1 << 32) | o.w0;
    ko = ((uint64_t)o.w3 << 32) | o.w2;
}

__device__ __forceinline__ uint64_t spread_even(uint32_t x32)
{
    uint64_t x = x32;
    x = (x | (x << 16)) & 0x0000FFFF0000FFFFull;
    x = (x | (x << 8)) & 0x00FF00FF00FF00FFull;
    x = (x | (x << 4)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x << 2)) & 0x3333333333333333ull;
    x = (x | (x << 1)) & 0x5555555555555555ull;
    return x;
}

// The merge of the workgroups' histograms costs one device-wide atomic per bin and workgroup, and atomics on one
// address are taken one after the other (about 50 ns each, measured): with 2048 workgroups the merge took four
// times as long as the keys.  Hence at most a few hundred workgroups of 1024 threads.
// prefix (may be NULL): word j receives the top 16 bits of the keys of vertices 2j (low half) and 2j+1.
__global__ __launch_bounds__(SCAN_NT) void sampler_hist_kernel(uint64_t N, uint64_t seed, uint64_t step,
                                                               uint32_t *__restrict__ hist, uint32_t *__restrict__ prefix,
                                                               sampler_state *__restrict__ state)
{
    __shared__ uint32_t lh[HIST_BINS];
    if (blockIdx.x == 0 && threadIdx.x == 0) state->ncand = 0;
    for (int i = threadIdx.x; i < HIST_BINS; i += SCAN_NT) lh[i] = 0;
    __syncthreads();
    const uint64_t J = (N + 1) >> 1;
    for (uint64_t j = (uint64_t)blockIdx.x * SCAN_NT + threadIdx.x; j < J; j += (uint64_t)gridDim.x * SCAN_NT) {
        uint64_t ke, ko;
        vertex_pair_keys(j, seed, step, ke, ko);
        atomicAdd(&lh[ke >> (64 - HIST_BITS)], 1u);
        if (2 * j + 1 < N) atomicAdd(&lh[ko >> (64 - HIST_BITS)], 1u);
        if (prefix) prefix[j] = (uint32_t)(ke >> 48) | ((uint32_t)(ko >> 48) << 16);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HIST_BINS; i += SCAN_NT) {
        uint32_t c = lh[i];
        if (c) atomicAdd(&hist[i], c);
    }
}

// Workgroup-local candidate list: matches are rare, so a workgroup gathers its own in LDS and reserves room in the
// global list with ONE atomic add, instead of one add per match on a single hot address.
template <uint32_t LCAP> struct cand_lds {
    uint64_t key[LCAP];
    uint32_t v[LCAP];
    uint32_t n, base, fail;
};

template <uint32_t LCAP>
__device__ __forceinline__ void cand_append(cand_lds<LCAP> &l, bool me, bool mo, uint64_t ke, uint64_t ko, uint64_t j,
                                            uint32_t *__restrict__ ncand, uint64_t *__restrict__ cand_key,
                                            uint32_t *__restrict__ cand_v, uint32_t cap, uint32_t *__restrict__ status)
{
    if (!(me || mo)) return;
    const uint32_t cnt = (me ? 1u : 0u) + (mo ? 1u : 0u);
    uint32_t p = atomicAdd(&l.n, cnt);
    if (p + cnt <= LCAP) {
        if (me) { l.key[p] = ke; l.v[p] = (uint32_t)(2 * j); ++p; }
        if (mo) { l.key[p] = ko; l.v[p] = (uint32_t)(2 * j + 1); }
    } else {
        // the local list is full (far beyond the expected load): straight to the global list.
        // Reservations only grow, so every one before the first that failed fitted, and they
        // fill [0, first failing offset) without holes.
        atomicMin(&l.fail, p);
        uint32_t q = atomicAdd(ncand, cnt);
        if (me) { if (q < cap) { cand_key[q] = ke; cand_v[q] = (uint32_t)(2 * j); } else atomicOr(status, SGNN_ST_CAND_OVERFLOW); ++q; }
        if (mo) { if (q < cap) { cand_key[q] = ko; cand_v[q] = (uint32_t)(2 * j + 1); } else atomicOr(status, SGNN_ST_CAND_OVERFLOW); }
    }
}

// every thread of the workgroup; NT threads
template <uint32_t LCAP, int NT>
__device__ __forceinline__ void cand_flush(cand_lds<LCAP> &l, uint32_t *__restrict__ ncand, uint64_t *__restrict__ cand_key,
                                           uint32_t *__restrict__ cand_v, uint32_t cap, uint32_t *__restrict__ status)
{
    __syncthreads();
    const uint32_t n_local = min(l.n, l.fail);
    if (threadIdx.x == 0) l.base = n_local ? atomicAdd(ncand, n_local) : 0u;
    __syncthreads();
    const uint32_t base = l.base;
    for (uint32_t i = threadIdx.x; i < n_local; i += NT) {
        if (base + i < cap) { cand_key[base + i] = l.key[i]; cand_v[base + i] = l.v[i]; }
        else atomicOr(status, SGNN_ST_CAND_OVERFLOW);
    }
}

// The one pass over the keys of a windowed call.  For a sparse sample of a large graph the bin of the threshold is
// known before any key is: the B-th smallest of N uniform keys lies at B/N of the key range, give or take
// sqrt(B (1 - B/N)) / N of it, so the host names a window [b_lo, b_hi] of one or two histogram bins that holds it
// (six standard deviations either side).  This pass then does three things with every key while it has it: counts
// it if it is below the window (below[w]: those of workgroup w), appends it to the candidate list if its bin is in the window, and sets the
// vertex's bit in the output bitmap if the bin lies below the window (such a vertex is in the sample whatever the threshold turns out to be).
// Nothing per vertex is stored for later passes - no key prefixes - and no later pass touches a key again.  The histogram is one of the
// candidates: a bin of the window in 1024 parts (window_part), so that the next pass has the part of the threshold, and few candidates are in it.
// What bounds the pass is the vector unit, 18 products of 16 clocks and 18 three-way xors a Philox call: 4 10^7 vertices 58.3 -> 50.5 us with the
// xors in one instruction each; the whole sample 93 -> 69 without a launch of one workgroup that selects among all candidates.
constexpr uint32_t WIN_LCAP = 2048;
constexpr unsigned WIN_MAX_WG = 512;                      // two a compute unit: what it holds
// a candidate's place in the histogram: the window has one bin or two
__device__ __forceinline__ uint32_t window_part(uint64_t k, uint32_t b_lo)
{
    return (uint32_t)(k >> (64 - HIST_BITS - 10)) - (b_lo << 10);
}
__global__ __launch_bounds__(SCAN_NT) void sampler_hist_window_kernel(uint64_t N, uint64_t seed, uint64_t step,
                                                                      uint32_t *__restrict__ hist, uint32_t *__restrict__ below,
                                                                      uint32_t b_lo, uint32_t b_hi,
                                                                      sampler_state *__restrict__ state,
                                                                      uint64_t *__restrict__ cand_key, uint32_t *__restrict__ cand_v,
                                                                      uint32_t cap, uint32_t *__restrict__ status,
                                                                      uint64_t *__restrict__ bitmap, uint64_t W)
{
    __shared__ uint32_t lds[SCAN_NT / 64];
    __shared__ cand_lds<WIN_LCAP> cl;
    __shared__ __attribute__((aligned(8))) uint8_t strip[SCAN_NT / 64][64];
    if (threadIdx.x == 0) { cl.n = 0; cl.fail = 0xffffffffu; }
    if (blockIdx.x == 0 && threadIdx.x == 0) state->nfew = 0;
    __syncthreads();
    const unsigned wave = threadIdx.x >> 6, lane = lane_id();
    // A wavefront takes eight bitmap words (512 vertices) per round: lane l computes the keys of vertices 8l .. 8l+7 of
    // the span (four Philox blocks) and reduces them to one byte of the bitmap; the 64 bytes pass through a
    // wavefront-private strip of LDS, from which lanes 0 .. 7 read and write their eight words with one 64-byte store
    // (as the emit pass over stored prefixes does: no bit interleaving of ballots).
    volatile uint8_t *my_bytes = strip[wave];
    volatile uint64_t *my_words = reinterpret_cast<volatile uint64_t *>(strip[wave]);
    uint32_t n_below = 0;
    const uint64_t W8 = (W + 7) & ~7ull;
    for (uint64_t wb = ((uint64_t)blockIdx.x * (SCAN_NT / 64) + wave) * 8; wb < W8; wb += (uint64_t)gridDim.x * (SCAN_NT / 64) * 8) {
        const uint64_t v0 = wb * 64 + 8 * lane;                  // first of the lane's eight vertices
        uint32_t byte = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t ve = v0 + 2 * q, vo = ve + 1;
            if (ve < N) {
                uint64_t ke, ko;
                vertex_pair_keys(ve >> 1, seed, step, ke, ko);
                const uint32_t be_ = (uint32_t)(ke >> (64 - HIST_BITS)), bo_ = (uint32_t)(ko >> (64 - HIST_BITS));
                const bool me = be_ >= b_lo && be_ <= b_hi;
                bool mo = false;
                byte |= (be_ < b_lo ? 1u : 0u) << (2 * q);
                if (vo < N) {
                    mo = bo_ >= b_lo && bo_ <= b_hi;
                    byte |= (bo_ < b_lo ? 1u : 0u) << (2 * q + 1);
                }
                if (me) atomicAdd(&hist[window_part(ke, b_lo)], 1u);
                if (mo) atomicAdd(&hist[window_part(ko, b_lo)], 1u);
                cand_append(cl, me, mo, ke, ko, ve >> 1, &state->ncand, cand_key, cand_v, cap, status);
            }
        }
        n_below += __popc(byte);
        my_bytes[lane] = (uint8_t)byte;          // volatile: written and read in program order; LDS serves a wavefront in order
        if (lane < 8) {
            const uint64_t word = my_words[lane];
            if (wb + lane < W) bitmap[wb + lane] = word;
        }
    }
    cand_flush<WIN_LCAP, SCAN_NT>(cl, &state->ncand, cand_key, cand_v, cap, status);
    n_below = block_sum<uint32_t, SCAN_NT>(n_below, lds);
    if (threadIdx.x == 0) below[blockIdx.x] = n_below;
}

// Bin of the B-th smallest key and its rank in there, from the histogram: 1024 threads, two bins a thread.  Every workgroup
// of the collect pass does this for itself (8 KB from an L2 and a scan, under two microseconds side by side): a
// launch of its own for one workgroup cost 2.4 us on a small graph and 4.8 behind a long pass.
__device__ __forceinline__ void pick_bin(uint32_t B, const uint32_t *__restrict__ hist, uint32_t &bin_out, uint32_t &r_out)
{
    __shared__ uint32_t lds[SCAN_NT / 64 + 1];
    __shared__ uint32_t sel[2];
    const uint2 h = reinterpret_cast<const uint2 *>(hist)[threadIdx.x];
    uint32_t total;
    const uint32_t ex = block_excl_scan<uint32_t, SCAN_NT>(h.x + h.y, &total, lds);
    // exactly one thread owns the bin of the B-th smallest key (1 <= B <= N)
    if (ex < B && B <= ex + h.x) { sel[0] = 2 * threadIdx.x; sel[1] = B - ex; }
    else if (ex + h.x < B && B <= ex + h.x + h.y) { sel[0] = 2 * threadIdx.x + 1; sel[1] = B - ex - h.x; }
    __syncthreads();
    bin_out = sel[0];
    r_out = sel[1];
}
static_assert(HIST_BINS == 2 * SCAN_NT, "two bins a thread");

template <bool PREFIX>
__global__ __launch_bounds__(SCAN_NT) void sampler_collect_kernel(uint64_t N, uint32_t B, uint64_t seed, uint64_t step,
                                                                  const uint32_t *__restrict__ hist,
                                                                  sampler_state *__restrict__ state,
                                                                  uint64_t *__restrict__ cand_key,
                                                                  uint32_t *__restrict__ cand_v, uint32_t cap,
                                                                  uint32_t *__restrict__ status,
                                                                  const uint32_t *__restrict__ prefix)
{
    // Matches are rare (one vertex in 2048): gathered per workgroup (cand_lds).
    constexpr uint32_t LCAP = 1024;
    __shared__ cand_lds<LCAP> cl;
    uint32_t bin, r;
    pick_bin(B, hist, bin, r);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state->bin = bin;
        state->r = r;
    }
    const uint64_t J = (N + 1) >> 1;
    if (threadIdx.x == 0) { cl.n = 0; cl.fail = 0xffffffffu; }
    __syncthreads();
    auto append = [&](bool me, bool mo, uint64_t ke, uint64_t ko, uint64_t j) {
        cand_append(cl, me, mo, ke, ko, j, &state->ncand, cand_key, cand_v, cap, status);
    };
    const uint64_t J_rounds = PREFIX ? (J + 3) / 4 : J;      // loop items: quads of prefix words, or Philox blocks
    for (uint64_t j = (uint64_t)blockIdx.x * SCAN_NT + threadIdx.x; j < J_rounds; j += (uint64_t)gridDim.x * SCAN_NT) {
        if constexpr (PREFIX) {
            // a thread takes four prefix words (eight vertices) per round; the stored prefixes hold the bin, and the
            // keys themselves are computed for the matches only
            const uint4 pp4 = *reinterpret_cast<const uint4 *>(prefix + 4 * j);      // the array is padded to whole quads
            const uint32_t pw[4] = {pp4.x, pp4.y, pp4.z, pp4.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t jj = 4 * j + q;
                const bool he = 2 * jj < N && ((pw[q] & 0xffffu) >> (16 - HIST_BITS)) == bin;
                const bool ho = 2 * jj + 1 < N && (pw[q] >> (32 - HIST_BITS)) == bin;
                if (he || ho) {
                    uint64_t k0, k1;
                    vertex_pair_keys(jj, seed, step, k0, k1);
                    append(he, ho, k0, k1, jj);
                }
            }
        } else {
            uint64_t ke, ko;
            vertex_pair_keys(j, seed, step, ke, ko);
            append((uint32_t)(ke >> (64 - HIST_BITS)) == bin, (2 * j + 1 < N) && (uint32_t)(ko >> (64 - HIST_BITS)) == bin, ke, ko, j);
        }
    }
    cand_flush<LCAP, SCAN_NT>(cl, &state->ncand, cand_key, cand_v, cap, status);
}

// Exact r-th smallest (key, v) among the candidates of the threshold's bin, by one workgroup; what it costs is the
// trips to memory, the barriers in a row and, at a few hundred candidates, the fetching of its own code.  So: one radix
// pass over the 8 bits below the 11 that the bin has decided (none if there are no more than FEW: without it 1000 candidates cost 1000
// comparisons of each with all, 20 us), then the
// candidates that still agree - one in 256 of those in the bin - move to a list in LDS, and the ones below each are counted
// by as many threads as there are for it.  A thread requests THR_BATCH keys at a time.  Where more than NT remain
// (vertex counts beyond 2^29 for 1024 threads) another eight bits are decided first.
// A launch of its own (1024 threads), 4 10^7 vertices (39 thousand candidates): 33 -> 16.5 us, what is left is one compute unit's rate
// of reads and LDS atomics; 2.4 10^6 vertices and fewer: 5 to 7 us before and after.  With 32 keys a thread in registers it spilled (24 us).
constexpr int THR_BATCH = 16;

template <int NT>
__device__ __forceinline__ void select_threshold(uint32_t n, uint32_t bin, uint32_t r, const uint64_t *cand_key, const uint32_t *cand_v,
                                                 uint64_t &thr_key, uint32_t &thr_v)
{
    constexpr uint32_t FEW = 64;
    static_assert(NT >= 256, "a digit a thread, and an entry of the list a thread");
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sel_digit, sel_r;
    __shared__ uint64_t found_key;
    __shared__ uint32_t found_v;
    __shared__ uint64_t list_key[NT];
    __shared__ uint32_t list_v[NT], list_below[NT];
    __shared__ uint32_t n_list;
    uint64_t pk = (uint64_t)bin << (64 - HIST_BITS);          // decided high bits of the key
    uint32_t pv = 0;                                          // decided high bits of the vertex
    int kd = HIST_BITS;                                       // how many of them are decided
    list_below[threadIdx.x] = 0;
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
    if (threadIdx.x == 0) { sel_digit = 0; sel_r = 1; n_list = 0; found_key = 0; found_v = 0; }
    __syncthreads();

    // f(key, index) for every candidate whose key agrees with the decided bits; a thread's first batch stays in registers
    auto fetch = [&](uint32_t i0, uint64_t (&k)[THR_BATCH]) {
#pragma unroll
        for (int q = 0; q < THR_BATCH; ++q) k[q] = cand_key[min(i0 + q * NT + threadIdx.x, n - 1)];
    };
    uint64_t first[THR_BATCH];
    if (n) fetch(0, first);
    auto for_agreeing = [&](auto f) {
        for (uint32_t i0 = 0; i0 < n; i0 += THR_BATCH * NT) {
            uint64_t k[THR_BATCH];
            if (i0) fetch(i0, k);
#pragma unroll
            for (int q = 0; q < THR_BATCH; ++q) {
                k[q] = i0 ? k[q] : first[q];
                if (i0 + q * NT + threadIdx.x < n && (k[q] >> (64 - kd)) == (pk >> (64 - kd))) f(k[q], i0 + q * NT + threadIdx.x);
            }
        }
    };
    // the digit of the r-th smallest from the histogram of digits, and its rank among the candidates with that digit
    auto select = [&]() {
        if (threadIdx.x < 64) {
            // lane l owns digits 4l .. 4l+3
            const uint32_t a0 = hist[4 * threadIdx.x], a1 = hist[4 * threadIdx.x + 1], a2 = hist[4 * threadIdx.x + 2],
                           a3 = hist[4 * threadIdx.x + 3];
            const uint32_t s = a0 + a1 + a2 + a3;
            const uint32_t ex = wave_incl_scan(s) - s;
            if (ex < r && r <= ex + s) {
                uint32_t d = 4 * threadIdx.x, e = ex;
                if (r > e + a0) { e += a0; ++d; if (r > e + a1) { e += a1; ++d; if (r > e + a2) { e += a2; ++d; } } }
                sel_digit = d;
                sel_r = r - e;
            }
        }
        __syncthreads();
        r = sel_r;
    };
    bool found = false;
    for (bool radix = n > FEW; !found && !(radix && kd == 64); radix = true) {
        if (radix) {
            const int width = min(8, 64 - kd), lo = 64 - kd - width;
            for_agreeing([&](uint64_t k, uint32_t) { atomicAdd(&hist[(uint32_t)(k >> lo) & ((1u << width) - 1u)], 1u); });
            __syncthreads();
            select();
            pk |= (uint64_t)sel_digit << lo;
            kd += width;
        }
        for_agreeing([&](uint64_t k, uint32_t i) {
            const uint32_t at = atomicAdd(&n_list, 1u);
            if (at < NT) { list_key[at] = k; list_v[at] = cand_v[i]; }
        });
        __syncthreads();
        const uint32_t m = n_list;
        found = m <= NT;
        if (found) {
            // the vertices differ, so exactly one candidate has r - 1 others below it; the candidates an entry is
            // compared with are shared out among 1024 / m2 threads
            uint32_t m2 = 64;
            while (m2 < m) m2 *= 2;
            const uint32_t t = threadIdx.x & (m2 - 1), part = threadIdx.x / m2, parts = NT / m2;
            if (t < m) {
                const uint64_t k = list_key[t];
                const uint32_t v = list_v[t];
                uint32_t below = 0;
#pragma unroll 4
                for (uint32_t i = part; i < m; i += parts) below += (list_key[i] < k) | ((list_key[i] == k) & (list_v[i] < v));
                if (below) atomicAdd(&list_below[t], below);
            }
            __syncthreads();
            if (threadIdx.x < m && list_below[threadIdx.x] == r - 1) { found_key = list_key[threadIdx.x]; found_v = list_v[threadIdx.x]; }
            __syncthreads();
            pk = found_key;
            pv = found_v;
        } else {
            __syncthreads();                               // every thread has read the count
            if (threadIdx.x < 256) hist[threadIdx.x] = 0;
            if (threadIdx.x == 0) n_list = 0;
            __syncthreads();
        }
    }
    // more candidates of one key than the list holds: the vertex decides
    for (int vd = 0; !found && vd < 32; vd += 8) {
        for_agreeing([&](uint64_t, uint32_t i) {
            const uint32_t v = cand_v[i];
            if (vd == 0 || (v >> (32 - vd)) == (pv >> (32 - vd))) atomicAdd(&hist[(v >> (24 - vd)) & 255u], 1u);
        });
        __syncthreads();
        select();
        pv |= sel_digit << (24 - vd);
        __syncthreads();
        if (threadIdx.x < 256) hist[threadIdx.x] = 0;
        __syncthreads();
    }
    thr_key = pk;
    thr_v = pv;
}

// A launch of its own, where there are too many candidates for every workgroup of the emit pass to look at all of them.
// Leaves the histogram zeroed for the next call.
__global__ __launch_bounds__(SCAN_NT) void sampler_threshold_kernel(sampler_state *__restrict__ state, uint32_t *__restrict__ bin_hist,
                                                                 const uint64_t *__restrict__ cand_key,
                                                                 const uint32_t *__restrict__ cand_v, uint32_t cap)
{
    const uint32_t n = min(state->ncand, cap);
    reinterpret_cast<uint2 *>(bin_hist)[threadIdx.x] = make_uint2(0u, 0u);
    uint64_t tk;
    uint32_t tv;
    select_threshold<SCAN_NT>(n, state->bin, state->r, cand_key, cand_v, tk, tv);
    if (threadIdx.x == 0) {
        state->thr_key = tk;
        state->thr_v = tv;
        state->ncand = 0;      // every thread read it long ago (barriers above): the list is empty for the next call
    }
}

// The threshold at the head of the emit pass: every workgroup selects it for itself, and the first zeroes the histogram for the next call
// (the rank pass empties the list).  Instead of a launch for one workgroup, whose 2 to 5 us of work and gap the others waited for, every
// workgroup reads the candidates (some 2048 at the largest such N, never more than the list holds): with the grids of sampler_launches 2.6 10^5 vertices 24.1 -> 18.2 us the whole sample, 10^6 46 -> 26,
// 2.4 10^6 36.1 -> 32.3.
constexpr uint64_t FUSED_THR_MAX_N = 1ull << 22;
struct thr_src {
    const uint64_t *key;
    const uint32_t *v;
    uint32_t *bin_hist;
    uint32_t cap;
};

template <bool FUSED>
__device__ __forceinline__ void emit_threshold(const sampler_state *__restrict__ state, const thr_src &src, uint64_t &tk, uint32_t &tv)
{
    if constexpr (FUSED) {
        if (blockIdx.x == 0)
            for (int i = threadIdx.x; i < HIST_BINS; i += SAMP_NT) src.bin_hist[i] = 0;
        select_threshold<SAMP_NT>(min(state->ncand, src.cap), state->bin, state->r, src.key, src.v, tk, tv);
    } else {
        tk = state->thr_key;
        tv = state->thr_v;
    }
}

// Windowed calls, second pass: the part of the window that holds the threshold, from the counts of the first pass, by every workgroup for itself; the
// candidates of the parts below it get their bits (the vertices of the bins below the window have theirs from the key pass), the places of those
// in it go to the list `few`.
// The window misses the threshold once in 10^9 calls.  Then the first workgroup goes through the keys by itself, twice (20 ms for 4 10^7
// vertices), for the bin and for its candidates, and selects the threshold; the count pass recomputes the keys and overwrites the bitmap.
// (Passes of the whole chip for it would be launches that every call pays for: one that left at once cost 4.5 us.)
// Candidates are written and read here: no __restrict__.
__global__ __launch_bounds__(SCAN_NT) void sampler_mark_kernel(uint64_t N, uint32_t B, uint64_t seed, uint64_t step, sampler_state *state,
                                                               const uint32_t *hist, const uint32_t *below, uint32_t n_wg, uint32_t b_lo,
                                                               uint64_t *cand_key, uint32_t *cand_v, uint32_t cap, uint64_t *bitmap,
                                                               uint32_t *few, uint32_t few_cap, uint32_t *status)
{
    __shared__ uint32_t lds[SCAN_NT / 64];
    uint32_t nb = 0;
    for (uint32_t i = threadIdx.x; i < n_wg; i += SCAN_NT) nb += below[i];
    nb = block_sum<uint32_t, SCAN_NT>(nb, lds);
    uint32_t n = state->ncand, bin, r;
    const bool miss = B <= nb || B - nb > n;
    n = min(n, cap);
    if (!miss) {
        pick_bin(B - nb, hist, bin, r);
        if (blockIdx.x == 0 && threadIdx.x == 0) { state->r = r; state->fallback = 0; }
        for (uint32_t i = blockIdx.x * SCAN_NT + threadIdx.x; i < n; i += gridDim.x * SCAN_NT) {
            const uint32_t part = window_part(cand_key[i], b_lo), v = cand_v[i];
            if (part < bin) atomicOr((unsigned long long *)&bitmap[v >> 6], 1ull << (v & 63));
            if (part != bin) continue;
            const uint32_t at = atomicAdd(&state->nfew, 1u);
            if (at < few_cap) few[at] = i;
            else atomicOr(status, SGNN_ST_CAND_OVERFLOW);
        }
        return;
    }
    if (blockIdx.x) return;
    constexpr uint32_t LCAP = 1024;
    __shared__ cand_lds<LCAP> cl;
    __shared__ uint32_t lh[HIST_BINS], n_list;
    reinterpret_cast<uint2 *>(lh)[threadIdx.x] = make_uint2(0u, 0u);
    if (threadIdx.x == 0) { cl.n = 0; cl.fail = 0xffffffffu; state->nfew = 0; }         // nfew: the length of this list
    __syncthreads();
    const uint64_t J = (N + 1) >> 1;
    for (uint64_t j = threadIdx.x; j < J; j += SCAN_NT) {
        uint64_t ke, ko;
        vertex_pair_keys(j, seed, step, ke, ko);
        atomicAdd(&lh[ke >> (64 - HIST_BITS)], 1u);
        if (2 * j + 1 < N) atomicAdd(&lh[ko >> (64 - HIST_BITS)], 1u);
    }
    __syncthreads();
    pick_bin(B, lh, bin, r);
    for (uint64_t j = threadIdx.x; j < J; j += SCAN_NT) {
        uint64_t ke, ko;
        vertex_pair_keys(j, seed, step, ke, ko);
        cand_append(cl, (uint32_t)(ke >> (64 - HIST_BITS)) == bin, (2 * j + 1 < N) && (uint32_t)(ko >> (64 - HIST_BITS)) == bin, ke, ko, j,
                    &state->nfew, cand_key, cand_v, cap, status);
    }
    cand_flush<LCAP, SCAN_NT>(cl, &state->nfew, cand_key, cand_v, cap, status);
    __syncthreads();
    if (threadIdx.x == 0) n_list = atomicAdd(&state->nfew, 0u);
    __syncthreads();
    uint64_t tk;
    uint32_t tv;
    select_threshold<SCAN_NT>(min(n_list, cap), bin, r, cand_key, cand_v, tk, tv);
    if (threadIdx.x == 0) {
        state->thr_key = tk;
        state->thr_v = tv;
        state->fallback = 1;
    }
}

// Workgroup g owns bitmap words [g*wpw, (g+1)*wpw), wpw a multiple of 8.  A wavefront takes 64 words
// (a quarter of the workgroup's, if that is fewer) at a time and builds two of them per iteration: lane l evaluates vertices 2j and 2j+1 of Philox block
// j = 32*w0 + l.  Lane l keeps word l of the 64, so that the wave writes them with one 512-byte store:
// an 8-byte store by a single lane per word reached memory as a partial write of its own, a quarter of a
// million of them at a rate of about one per nanosecond.
__device__ __forceinline__ void emit_words(uint64_t N, uint64_t seed, uint64_t step, uint64_t tk, uint32_t tv, uint64_t *__restrict__ bitmap,
                                           uint64_t W, uint64_t wpw, uint32_t *__restrict__ wg_count)
{
    __shared__ uint32_t lds[SAMP_NT / 64];
    const uint64_t wbeg = (uint64_t)blockIdx.x * wpw;
    const uint64_t wend = min(W, wbeg + wpw);
    const unsigned wave = threadIdx.x >> 6, lane = lane_id();
    uint32_t cnt = 0;
    const unsigned span = (unsigned)min((uint64_t)64, wpw / (SAMP_NT / 64));     // words a wavefront takes at a time: an even number, as wpw is a multiple of 8
    for (uint64_t chunk = wbeg + span * wave; chunk < wend; chunk += span * (SAMP_NT / 64)) {
        uint64_t mine = 0;
        for (unsigned it = 0; it < span / 2; ++it) {
            const uint64_t w0 = chunk + 2 * it;
            if (w0 >= wend) break;
            const uint64_t j = w0 * 32 + lane;
            const uint64_t ve = 2 * j, vo = 2 * j + 1;
            bool ie = false, io = false;
            if (ve < N) {
                uint64_t ke, ko;
                vertex_pair_keys(j, seed, step, ke, ko);
                ie = ke < tk || (ke == tk && (uint32_t)ve <= tv);
                io = vo < N && (ko < tk || (ko == tk && (uint32_t)vo <= tv));
            }
            const uint64_t be = __ballot(ie), bo = __ballot(io);
            const uint64_t word0 = spread_even((uint32_t)be) | (spread_even((uint32_t)bo) << 1);
            const uint64_t word1 = spread_even((uint32_t)(be >> 32)) | (spread_even((uint32_t)(bo >> 32)) << 1);
            if (lane == 2 * it) mine = word0;
            if (lane == 2 * it + 1) mine = word1;
            cnt += __popcll(word0) + __popcll(word1);
        }
        if (lane < span && chunk + lane < wend) bitmap[chunk + lane] = mine;
    }
    if (lane == 0) lds[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < SAMP_NT / 64; ++i) t += lds[i];
        wg_count[blockIdx.x] = t;
    }
}

template <bool FUSED>
__global__ __launch_bounds__(SAMP_NT) void sampler_emit_kernel(uint64_t N, uint64_t seed, uint64_t step,
                                                               const sampler_state *__restrict__ state,
                                                               uint64_t *__restrict__ bitmap, uint64_t W, uint64_t wpw,
                                                               uint32_t *__restrict__ wg_count, thr_src src)
{
    uint64_t tk;
    uint32_t tv;
    emit_threshold<FUSED>(state, src, tk, tv);
    emit_words(N, seed, step, tk, tv, bitmap, W, wpw, wg_count);
}

// Windowed calls, last but one: every workgroup counts its words, finds the threshold among the few candidates of its part and sets the bits of
// those of them that are in and in its words.  Leaves the histogram zeroed for the next call (the rank pass empties the candidates' list).
__global__ __launch_bounds__(SAMP_NT) void sampler_count_kernel(uint64_t N, uint64_t seed, uint64_t step,
                                                                const sampler_state *__restrict__ state, uint32_t *__restrict__ hist,
                                                                const uint64_t *__restrict__ cand_key, const uint32_t *__restrict__ cand_v,
                                                                const uint32_t *__restrict__ few, uint32_t few_cap, uint64_t *bitmap,
                                                                uint64_t W, uint64_t wpw, uint32_t *__restrict__ wg_count)
{
    constexpr uint32_t TILE = 32;                          // 4 10^7 vertices have 20 candidates in a part, 10^8 50
    __shared__ uint32_t lds[SAMP_NT / 64];
    __shared__ uint64_t tile_key[TILE], found_key;
    __shared__ uint32_t tile_v[TILE], found_v;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < HIST_BINS; i += SAMP_NT) hist[i] = 0;
    if (state->fallback) {
        emit_words(N, seed, step, state->thr_key, state->thr_v, bitmap, W, wpw, wg_count);
        return;
    }
    const uint32_t m = min(state->nfew, few_cap), r = state->r;
    const uint64_t wbeg = (uint64_t)blockIdx.x * wpw;
    const uint64_t wend = min(W, wbeg + wpw);
    uint32_t cnt = 0;
    for (uint64_t w = wbeg + threadIdx.x; w < wend; w += SAMP_NT) cnt += (uint32_t)__popcll(bitmap[w]);
    if (threadIdx.x == 0) { found_key = 0; found_v = 0; }
    // the vertices differ, so exactly one has r - 1 others below it
    for (uint32_t i0 = 0; i0 < m; i0 += SAMP_NT) {
        const uint32_t i = i0 + threadIdx.x, c = few[min(i, m - 1)], v = cand_v[c];
        const uint64_t k = cand_key[c];
        uint32_t less = 0;
        for (uint32_t j0 = 0; j0 < m; j0 += TILE) {
            const uint32_t nj = min(TILE, m - j0);
            __syncthreads();
            if (threadIdx.x < nj) {
                const uint32_t cj = few[j0 + threadIdx.x];
                tile_key[threadIdx.x] = cand_key[cj];
                tile_v[threadIdx.x] = cand_v[cj];
            }
            __syncthreads();
            if (i < m)
                for (uint32_t j = 0; j < nj; ++j) less += (tile_key[j] < k) | ((tile_key[j] == k) & (tile_v[j] < v));
        }
        if (i < m && less == r - 1) { found_key = k; found_v = v; }
    }
    __syncthreads();
    const uint64_t tk = found_key;
    const uint32_t tv = found_v;
    for (uint32_t i = threadIdx.x; i < m; i += SAMP_NT) {
        const uint32_t c = few[i], v = cand_v[c];
        const uint64_t k = cand_key[c];
        if ((v >> 6) < wbeg || (v >> 6) >= wend || k > tk || (k == tk && v > tv)) continue;
        atomicOr((unsigned long long *)&bitmap[v >> 6], 1ull << (v & 63));
        ++cnt;
    }
    cnt = block_sum<uint32_t, SAMP_NT>(cnt, lds);
    if (threadIdx.x == 0) wg_count[blockIdx.x] = cnt;
}

// The same from the stored key prefixes.  A wavefront takes eight bitmap words (512 vertices) per round: lane l
// loads the prefixes of vertices 8l .. 8l+7 of the span with one 16-byte load and reduces them to one byte of the
// bitmap (a prefix below the threshold's is in, one above is out, an equal one - 2^-16 of the vertices - has its key
// computed again); the 64 bytes pass through a wavefront-private strip of LDS, from which lanes 0 .. 7 read and
// write their eight words with one 64-byte store.  No scalar bit interleaving, no key arithmetic.
template <bool FUSED>
__global__ __launch_bounds__(SAMP_NT) void sampler_emit_prefix_kernel(uint64_t N, uint64_t seed, uint64_t step,
                                                                      const sampler_state *__restrict__ state,
                                                                      uint64_t *__restrict__ bitmap, uint64_t W, uint64_t wpw,
                                                                      uint32_t *__restrict__ wg_count,
                                                                      const uint32_t *__restrict__ prefix, thr_src src)
{
    __shared__ uint32_t lds[SAMP_NT / 64];
    __shared__ __attribute__((aligned(8))) uint8_t strip[SAMP_NT / 64][64];
    uint64_t tk;
    uint32_t tv;
    emit_threshold<FUSED>(state, src, tk, tv);
    const uint32_t tp = (uint32_t)(tk >> 48);
    const uint64_t wbeg = (uint64_t)blockIdx.x * wpw;
    const uint64_t wend = min(W, wbeg + wpw);
    const unsigned wave = threadIdx.x >> 6, lane = lane_id();
    volatile uint8_t *my_bytes = strip[wave];
    volatile uint64_t *my_words = reinterpret_cast<volatile uint64_t *>(strip[wave]);
    uint32_t cnt = 0;
    // wbeg and wpw are multiples of 8: a round's eight words lie inside [wbeg, wend) or behind W (vertices >= N: empty)
    for (uint64_t wb = wbeg + 8 * wave; wb < wend; wb += 8 * (SAMP_NT / 64)) {
        const uint64_t v0 = wb * 64 + 8 * lane;                  // first of the lane's eight vertices
        uint32_t byte = 0;
        if (v0 < N) {
            const uint4 pp4 = *reinterpret_cast<const uint4 *>(prefix + (v0 >> 1));      // the array is padded to whole quads
            const uint32_t pw[4] = {pp4.x, pp4.y, pp4.z, pp4.w};
            bool tie = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t pe = pw[q] & 0xffffu, po = pw[q] >> 16;
                byte |= (pe < tp ? 1u : 0u) << (2 * q) | (po < tp ? 1u : 0u) << (2 * q + 1);
                tie = tie || pe == tp || po == tp;
            }
            if (tie) {
#pragma unroll 1
                for (int q = 0; q < 4; ++q) {
                    const uint32_t pe = pw[q] & 0xffffu, po = pw[q] >> 16;
                    if (pe != tp && po != tp) continue;
                    const uint64_t ve = v0 + 2 * q, vo = ve + 1;
                    uint64_t ke, ko;
                    vertex_pair_keys(ve >> 1, seed, step, ke, ko);
                    const uint32_t ie = (ke < tk || (ke == tk && (uint32_t)ve <= tv)) ? 1u : 0u;
                    const uint32_t io = (ko < tk || (ko == tk && (uint32_t)vo <= tv)) ? 1u : 0u;
                    byte = (byte & ~(3u << (2 * q))) | ie << (2 * q) | io << (2 * q + 1);
                }
            }
            // vertices at and behind N (the odd partner of the last vertex, the padding of the last quad) are out
            if (v0 + 8 > N) byte &= (1u << (N - v0)) - 1u;
        }
        my_bytes[lane] = (uint8_t)byte;          // volatile: written and read in program order; LDS serves a wavefront in order
        if (lane < 8) {
            const uint64_t word = my_words[lane];
            if (wb + lane < wend) bitmap[wb + lane] = word;
            cnt += (uint32_t)__popcll(word);
        }
    }
    cnt = wave_sum(cnt);
    if (lane == 0) lds[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < SAMP_NT / 64; ++i) t += lds[i];
        wg_count[blockIdx.x] = t;
    }
}

template <int P>
__global__ __launch_bounds__(SAMP_NT) void sampler_rank_kernel(const uint64_t *__restrict__ bitmap, uint64_t W,
                                                               uint64_t wpw, const uint32_t *__restrict__ wg_count,
                                                               uint32_t B, uint32_t *__restrict__ rank,
                                                               int32_t *__restrict__ S, uint32_t *__restrict__ status, uint32_t *__restrict__ ncand)
{
    __shared__ uint32_t lds[SAMP_NT / 64 + 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) *ncand = 0;            // the list is empty for the next call
    // sampled vertices in all earlier workgroups
    uint32_t part = 0;
    for (unsigned i = threadIdx.x; i < blockIdx.x; i += SAMP_NT) part += wg_count[i];
    uint32_t running = block_sum<uint32_t, SAMP_NT>(part, lds);
    const uint64_t wbeg = (uint64_t)blockIdx.x * wpw;
    const uint64_t wend = min(W, wbeg + wpw);
    for (uint64_t base = wbeg; base < wend; base += SAMP_NT / P) {
        const uint64_t w = base + threadIdx.x / P;
        uint64_t word = w < wend ? bitmap[w] : 0ull;
        const int at = 64 / P * (threadIdx.x % P);
        if constexpr (P > 1) word &= ((1ull << (64 / P)) - 1) << at;
        uint32_t total;
        uint32_t ex = block_excl_scan<uint32_t, SAMP_NT>(__popcll(word), &total, lds) + running;
        if (w < wend && at == 0) rank[w] = ex;
        while (word) {
            const int b = __ffsll((unsigned long long)word) - 1;
            if (ex < B) S[ex] = (int32_t)(w * 64 + b);
            ++ex;
            word &= word - 1;
        }
        running += total;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0 && running != B) atomicOr(status, SGNN_ST_CAND_OVERFLOW);
}

// All of it by one workgroup, for graphs of up to SMALL_N vertices: a thread keeps the keys of up to eight pairs of vertices in registers, and
// histogram, candidates and bitmap stay in LDS.  Bound by barriers in a row, the fetching of its own code and one compute unit's Philox (0.3 us a
// thousand vertices), where five launches cost 17 to 19 us: 4096 vertices 18.4 -> 6.9 us, 16384 19.0 -> 10.7.  With sixteen pairs a thread
// it took 17.8 us for 32768 vertices (19.2 by the five) and 2 us more than this for all smaller ones: the longer code.
constexpr uint64_t SMALL_N = 16384;
__global__ __launch_bounds__(SCAN_NT) void sampler_small_kernel(uint32_t N, uint32_t B, uint64_t seed, uint64_t step, int32_t *__restrict__ S,
                                                                uint64_t *__restrict__ bitmap, uint32_t *__restrict__ rank,
                                                                uint32_t *__restrict__ status)
{
    constexpr int Q = (int)(SMALL_N / 2 / SCAN_NT);
    constexpr uint32_t THR_LIST = SCAN_NT;
    __shared__ __attribute__((aligned(8))) uint32_t lh[HIST_BINS];
    __shared__ uint32_t bits[SMALL_N / 32];
    __shared__ uint64_t list_key[THR_LIST];
    __shared__ uint32_t list_v[THR_LIST], list_below[THR_LIST];
    __shared__ uint32_t lds[SCAN_NT / 64 + 1], sel[3], n_list, found_v;
    __shared__ uint64_t found_key;
    const uint32_t t = threadIdx.x, J = (N + 1) >> 1;
    uint64_t ke[Q], ko[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        ke[q] = ko[q] = 0;
        if (q * SCAN_NT < J) vertex_pair_keys(q * SCAN_NT + t, seed, step, ke[q], ko[q]);
    }
    // f(key, vertex) for every vertex whose key agrees with the decided bits
    uint64_t pk = 0;
    int kd = 0;
    auto agrees = [&](uint64_t k) { return kd == 0 || (k >> (64 - kd)) == (pk >> (64 - kd)); };
    auto for_agreeing = [&](auto f) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t v = 2 * (q * SCAN_NT + t);
            if (v < N && agrees(ke[q])) f(ke[q], v);
            if (v + 1 < N && agrees(ko[q])) f(ko[q], v + 1);
        }
    };
    // the bits of the B-th smallest key, eleven at a time until no more than THR_LIST keys agree with them (once for keys of a generator)
    uint32_t r = B, m;
    if (t < THR_LIST) list_below[t] = 0;
    if (t < SMALL_N / 32) bits[t] = 0;
    if (t == 0) n_list = found_v = 0, found_key = 0; // kept, and reported, if one key had more vertices than the list holds
    do {
        const int width = min(HIST_BITS, 64 - kd), lo = 64 - kd - width;
        reinterpret_cast<uint2 *>(lh)[t] = make_uint2(0u, 0u);
        __syncthreads();
        for_agreeing([&](uint64_t k, uint32_t) { atomicAdd(&lh[(uint32_t)(k >> lo) & ((1u << width) - 1u)], 1u); });
        __syncthreads();
        const uint2 h = reinterpret_cast<const uint2 *>(lh)[t];
        uint32_t total;
        const uint32_t ex = block_excl_scan<uint32_t, SCAN_NT>(h.x + h.y, &total, lds);
        if (ex < r && r <= ex + h.x) { sel[0] = 2 * t; sel[1] = r - ex; sel[2] = h.x; }
        else if (ex + h.x < r && r <= ex + h.x + h.y) { sel[0] = 2 * t + 1; sel[1] = r - ex - h.x; sel[2] = h.y; }
        __syncthreads();
        pk |= (uint64_t)sel[0] << lo;
        kd += width;
        r = sel[1];
        m = sel[2];
    } while (m > THR_LIST && kd < 64);
    if (m <= THR_LIST) {
        for_agreeing([&](uint64_t k, uint32_t v) {
            const uint32_t at = atomicAdd(&n_list, 1u);
            list_key[at] = k;
            list_v[at] = v;
        });
        __syncthreads();
        // the vertices differ, so exactly one candidate has r - 1 others below it; the candidates an entry is compared with are shared out
        // among 1024 / m2 threads
        uint32_t m2 = 64;
        while (m2 < m) m2 *= 2;
        const uint32_t c = t & (m2 - 1), parts = SCAN_NT / m2;
        if (c < m) {
            const uint64_t k = list_key[c];
            const uint32_t v = list_v[c];
            uint32_t below = 0;
            for (uint32_t i = t / m2; i < m; i += parts) below += (list_key[i] < k) | ((list_key[i] == k) & (list_v[i] < v));
            if (below) atomicAdd(&list_below[c], below);
        }
        __syncthreads();
        if (t < m && list_below[t] == r - 1) { found_key = list_key[t]; found_v = list_v[t]; }
    }
    __syncthreads();
    const uint64_t tk = found_key;
    const uint32_t tv = found_v;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t j = q * SCAN_NT + t, v = 2 * j;
        const uint32_t ie = v < N && (ke[q] < tk || (ke[q] == tk && v <= tv)), io = v + 1 < N && (ko[q] < tk || (ko[q] == tk && v + 1 <= tv));
        if (ie | io) atomicOr(&bits[j >> 4], (ie | io << 1) << (2 * (j & 15)));
    }
    __syncthreads();
    // a thread has sixteen vertices
    uint32_t x = (bits[t >> 1] >> (16 * (t & 1))) & 0xffffu, total;
    uint32_t ex = block_excl_scan<uint32_t, SCAN_NT>(__popc(x), &total, lds);
    const uint32_t w = t / 4;
    if (t % 4 == 0 && w * 64 < N) {
        rank[w] = ex;
        bitmap[w] = (uint64_t)bits[2 * w] | (uint64_t)bits[2 * w + 1] << 32;
    }
    for (; x; x &= x - 1, ++ex)
        if (ex < B) S[ex] = (int32_t)(16 * t + __ffs(x) - 1);
    if (t == 0 && total != B) atomicOr(status, SGNN_ST_CAND_OVERFLOW);
}
static_assert(SMALL_N / 16 == SCAN_NT, "sixteen vertices a thread");

} // namespace

// scratch layout of the sampler inside the context's persistent area
size_t sgnn_sampler_persist_bytes() { return HIST_BINS * sizeof(uint32_t) + 256; }

static uint32_t cand_capacity(uint64_t N) { return (uint32_t)(2 * (N >> HIST_BITS) + 8192); }

// the key prefixes pay once a pass over the keys costs more than their traffic; below that the keys are recomputed
static size_t prefix_bytes(uint64_t N) { return N >= (1ull << 20) ? (size_t)(((N + 1) >> 1) + 4) * sizeof(uint32_t) : 0; }   // padded to whole quads

size_t sgnn_sampler_ws_bytes(uint64_t N)
{
    const size_t cap = cand_capacity(N);
    return cap * 12 + EMIT_MAX_WG * 4 + 4 * 256 + prefix_bytes(N) + 256;
}

// The launches.  ctx may be NULL (no profiling, errors through sgnn_fail(NULL, ...)); every buffer
// comes from the caller of this function: hist (HIST_BINS words, zero on entry, left zero), state,
// the candidate list of `cap` entries, EMIT_MAX_WG workgroup counts and the sticky status word.
#define SAMP_LAUNCH(name, kernel, grid, block, ...)                                                        \
    do {                                                                                                  \
        if (ctx && ctx->prof_on) sgnn_prof_begin(ctx, st, name, "");                                       \
        hipLaunchKernelGGL(kernel, grid, block, 0, st, __VA_ARGS__);                                       \
        if (ctx && ctx->prof_on) sgnn_prof_end(ctx, st);                                                   \
        SGNN_LAUNCH_CHECK(ctx, name);                                                                     \
    } while (0)

// Window of histogram bins that holds the threshold of a sparse sample of a large graph (see
// sampler_hist_window_kernel): the B-th smallest of N uniform keys lies at x = B/N of the key range with a standard
// deviation of sqrt(B (1 - B/N)) / N; six of them either side must span at most two bins, or there is no window.
// shift: moves the window by whole bins (a test's way to the fallback passes; 0 in use).
struct sampler_window { int on; uint32_t b_lo, b_hi; };
static sampler_window sampler_window_for(uint64_t N, uint32_t B, int shift)
{
    sampler_window w = {0, 0, 0};
    if (N < (1ull << 20) || (uint64_t)B * 4 > N) return w;
    const double p = (double)B / (double)N, x = p * HIST_BINS;
    const double h = 6.0 * HIST_BINS * std::sqrt((double)B * (1.0 - p)) / (double)N + 1e-6;
    if (h >= 0.45) return w;
    const long lo = std::lround(std::floor(x - h)) + shift, hi = std::lround(std::floor(x + h)) + shift;
    w.on = 1;
    w.b_lo = (uint32_t)std::min<long>(std::max<long>(lo, 0), HIST_BINS - 1);
    w.b_hi = (uint32_t)std::min<long>(std::max<long>(hi, 0), HIST_BINS - 1);
    return w;
}

static int sampler_launches(sgnn_ctx *ctx, uint64_t N, uint32_t B, uint64_t seed, uint64_t step, int32_t *S,
                            uint64_t *bitmap, uint32_t *rank, uint32_t *hist, sampler_state *state, uint64_t *cand_key,
                            uint32_t *cand_v, uint32_t cap, uint32_t *wg_count, uint32_t *status, uint32_t *prefix,
                            sampler_window win, hipStream_t st)
{
    if (N <= SMALL_N) {
        SAMP_LAUNCH("sampler_small_kernel", sampler_small_kernel, dim3(1), dim3(SCAN_NT), (uint32_t)N, B, seed, step, S, bitmap, rank, status);
        return SGNN_OK;
    }
    const uint64_t J = (N + 1) >> 1;
    const unsigned grid =
        (unsigned)std::min<uint64_t>(cdiv(J, SCAN_NT), std::min<uint64_t>(std::max<uint64_t>(256, N >> 19), 2048));
    const uint64_t W = (N + 63) / 64;
    // a workgroup of the emit pass has a threshold to select before its 2048 vertices or more: 5.2 10^5 vertices by 256 workgroups 21.4 us the
    // whole sample, by 1024 23.9; 4 10^6 45.1 and 39.6
    const unsigned egrid =
        (unsigned)std::min<uint64_t>(cdiv(W, 8), std::min<uint64_t>(std::max<uint64_t>(256, N >> 11), EMIT_MAX_WG));
    const uint64_t wpw = (uint64_t)cdiv(cdiv(W, egrid), 8) * 8;
    if (win.on) {
        // one pass over the keys; the array of ranks, which the last pass writes, holds the list `few` until then
        const unsigned wgrid = (unsigned)std::min<uint64_t>(cdiv(J, SCAN_NT), WIN_MAX_WG);
        SAMP_LAUNCH("sampler_hist_window_kernel", sampler_hist_window_kernel, dim3(wgrid), dim3(SCAN_NT), N, seed, step, hist, wg_count, win.b_lo,
                    win.b_hi, state, cand_key, cand_v, cap, status, bitmap, W);
        SAMP_LAUNCH("sampler_mark_kernel", sampler_mark_kernel, dim3(64), dim3(SCAN_NT), N, B, seed, step, state, (const uint32_t *)hist,
                    (const uint32_t *)wg_count, wgrid, win.b_lo, cand_key, cand_v, cap, bitmap, rank, (uint32_t)W, status);
        SAMP_LAUNCH("sampler_count_kernel", sampler_count_kernel, dim3(egrid), dim3(SAMP_NT), N, seed, step, (const sampler_state *)state, hist,
                    (const uint64_t *)cand_key, (const uint32_t *)cand_v, (const uint32_t *)rank, (uint32_t)W, bitmap, W, wpw, wg_count);
        SAMP_LAUNCH("sampler_rank_kernel", wpw * 4 <= SAMP_NT ? sampler_rank_kernel<4> : sampler_rank_kernel<1>, dim3(egrid), dim3(SAMP_NT), bitmap, W, wpw, wg_count, B, rank, S,
                    status, &state->ncand);
        return SGNN_OK;
    }
    // a workgroup's merge costs up to 2048 atomics however few keys it had (the comment at the kernel): 64 workgroups for 5.2 10^5 vertices
    // 23.1 us the whole sample, 256 26.9; 4 10^6 45.5 and 37.3
    const unsigned hgrid = std::min(grid, (unsigned)std::max<uint64_t>(64, N >> 13));
    SAMP_LAUNCH("sampler_hist_kernel", sampler_hist_kernel, dim3(hgrid), dim3(SCAN_NT), N, seed, step, hist, prefix, state);
    if (prefix)
        SAMP_LAUNCH("sampler_collect_kernel", sampler_collect_kernel<true>, dim3(grid), dim3(SCAN_NT), N, B, seed, step,
                    (const uint32_t *)hist, state, cand_key, cand_v, cap, status, (const uint32_t *)prefix);
    else
        SAMP_LAUNCH("sampler_collect_kernel", sampler_collect_kernel<false>, dim3(grid), dim3(SCAN_NT), N, B, seed, step,
                    (const uint32_t *)hist, state, cand_key, cand_v, cap, status, (const uint32_t *)nullptr);
    const bool fused = N <= FUSED_THR_MAX_N;
    const thr_src src = {cand_key, cand_v, hist, cap};
    if (!fused)
        SAMP_LAUNCH("sampler_threshold_kernel", sampler_threshold_kernel, dim3(1), dim3(SCAN_NT), state, hist, (const uint64_t *)cand_key,
                    (const uint32_t *)cand_v, cap);
    if (prefix)
        SAMP_LAUNCH("sampler_emit_kernel", fused ? sampler_emit_prefix_kernel<true> : sampler_emit_prefix_kernel<false>, dim3(egrid),
                    dim3(SAMP_NT), N, seed, step, state, bitmap, W, wpw, wg_count, (const uint32_t *)prefix, src);
    else
        SAMP_LAUNCH("sampler_emit_kernel", fused ? sampler_emit_kernel<true> : sampler_emit_kernel<false>, dim3(egrid), dim3(SAMP_NT), N,
                    seed, step, state, bitmap, W, wpw, wg_count, src);
    SAMP_LAUNCH("sampler_rank_kernel", wpw * 4 <= SAMP_NT ? sampler_rank_kernel<4> : sampler_rank_kernel<1>, dim3(egrid), dim3(SAMP_NT), bitmap, W, wpw, wg_count, B, rank, S,
                status, &state->ncand);
    return SGNN_OK;
}

int sgnn_launch_sampler(sgnn_ctx *ctx, uint64_t N, uint32_t B, uint64_t seed, uint64_t step, int32_t *S,
                        uint64_t *bitmap, uint32_t *rank, hipStream_t st)
{
    uint32_t *hist = reinterpret_cast<uint32_t *>(ctx->persist);
    sampler_state *state = reinterpret_cast<sampler_state *>(ctx->persist + HIST_BINS * sizeof(uint32_t));
    ws_alloc ws(ctx);
    const uint32_t cap = cand_capacity(N);
    uint64_t *cand_key = ws.get<uint64_t>(cap);
    uint32_t *cand_v = ws.get<uint32_t>(cap);
    uint32_t *wg_count = ws.get<uint32_t>(EMIT_MAX_WG);
    // SGNN_SAMPLER_WINDOW_SHIFT: whole bins by which the window is moved off its place (tests of the fallback passes)
    const char *shift_env = std::getenv("SGNN_SAMPLER_WINDOW_SHIFT");
    const sampler_window win = sampler_window_for(N, B, shift_env ? std::atoi(shift_env) : 0);
    // a windowed call stores nothing per vertex; otherwise two bytes of key prefix per vertex from 2^20 vertices on
    uint32_t *prefix = (!win.on && prefix_bytes(N)) ? ws.get<uint32_t>(prefix_bytes(N) / sizeof(uint32_t)) : nullptr;
    if (!ws.ok)
        return sgnn_fail(ctx, SGNN_ERR_CAPACITY, "sgnn_sample_uniform: scratch too small (%zu bytes needed): call sgnn_ctx_reserve",
                         ws.off);
    // histogram and list are empty between calls, also behind one that failed half way
    int rc = sgnn_zero_open(ctx, SGNN_ZERO_SAMPLER, ctx->persist, sgnn_sampler_persist_bytes(), st);
    if (rc) return rc;
    rc = sampler_launches(ctx, N, B, seed, step, S, bitmap, rank, hist, state, cand_key, cand_v, cap, wg_count, ctx->status, prefix, win, st);
    return sgnn_zero_close(ctx, rc, SGNN_ZERO_SAMPLER, ctx->persist, sgnn_sampler_persist_bytes(), st);
}

// ---- the same sampler without any allocation: scratch in a file-scope device array ---------------------

namespace {

constexpr uint64_t STATIC_MAX_N = SGNN_STATIC_SAMPLER_MAX_N;
constexpr uint32_t STATIC_CAP = (uint32_t)(2 * (STATIC_MAX_N >> HIST_BITS) + 8192);     // cand_capacity(STATIC_MAX_N)
constexpr size_t ST_HIST = 0;                                        // uint32[HIST_BINS]
constexpr size_t ST_STATE = ST_HIST + HIST_BINS * sizeof(uint32_t);  // sampler_state
constexpr size_t ST_STATUS = ST_STATE + 256;                         // uint32 sticky status (when the caller passes none)
constexpr size_t ST_WG = ST_STATUS + 256;                            // uint32[EMIT_MAX_WG]
constexpr size_t ST_CKEY = ST_WG + EMIT_MAX_WG * sizeof(uint32_t);   // uint64[STATIC_CAP]
constexpr size_t ST_CV = ST_CKEY + (size_t)STATIC_CAP * sizeof(uint64_t);   // uint32[STATIC_CAP]
constexpr size_t ST_BYTES = (ST_CV + (size_t)STATIC_CAP * sizeof(uint32_t) + 255) & ~size_t(255);
constexpr int MAX_DEVICES = 64;

// zeroes the histogram and the selection state: the array keeps the last call's contents, and a call that
// was abandoned half way (a failed launch) may have left counts behind
__global__ __launch_bounds__(SAMP_NT) void sampler_static_clear_kernel(uint32_t *__restrict__ words, uint32_t n)
{
    for (uint32_t i = blockIdx.x * SAMP_NT + threadIdx.x; i < n; i += gridDim.x * SAMP_NT) words[i] = 0;
}

} // namespace

// Every GPU the library runs on holds its own copy of this array, at its own address, until the process ends.
static __device__ __align__(256) uint8_t scratch[ST_BYTES];

// device address of `scratch` on each GPU, resolved once per device with that device current
static uint8_t *g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mutex;

static int static_scratch(int device, uint8_t **out)
{
    if (device < 0 || device >= MAX_DEVICES)
        return sgnn_fail(nullptr, SGNN_ERR_UNSUPPORTED, "sgnn_sample_uniform_static: device %d outside the supported 0..%d", device,
                         MAX_DEVICES - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        uint8_t *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return sgnn_fail(nullptr, SGNN_ERR_HIP, "sgnn_sample_uniform_static: hipGetSymbolAddress failed on device %d: %s", device,
                             hipGetErrorString(e));
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return SGNN_OK;
}

// Called by sgnn_ctx_create (the library's set-up call) with the context's device current, so that a later
// sgnn_sample_uniform_static on that device finds the address resolved.
int sgnn_static_scratch_init(int device)
{
    uint8_t *p = nullptr;
    return static_scratch(device, &p);
}

extern "C" int sgnn_sample_uniform_static(uint64_t N, uint32_t B, uint64_t seed, uint64_t step, int32_t *S, uint64_t *bitmap,
                                          uint32_t *rank, uint32_t *status_dev, sgnn_stream stream)
{
    if (!S || !bitmap || !rank) return sgnn_fail(nullptr, SGNN_ERR_INVALID_ARG, "sgnn_sample_uniform_static: null output pointer");
    if (B == 0 || B > N)
        return sgnn_fail(nullptr, SGNN_ERR_INVALID_ARG, "sgnn_sample_uniform_static: need 1 <= B <= N (B=%u, N=%llu)", B,
                         (unsigned long long)N);
    if (N > STATIC_MAX_N)
        return sgnn_fail(nullptr, SGNN_ERR_CAPACITY, "sgnn_sample_uniform_static: N = %llu exceeds the %llu vertices the static "
                         "scratch is sized for; use sgnn_sample_uniform with a context", (unsigned long long)N,
                         (unsigned long long)STATIC_MAX_N);
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return sgnn_fail(nullptr, SGNN_ERR_HIP, "sgnn_sample_uniform_static: hipGetDevice failed");
    uint8_t *ptr = nullptr;
    int rc = static_scratch(device, &ptr);
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    uint32_t *hist = reinterpret_cast<uint32_t *>(ptr + ST_HIST);
    sampler_state *state = reinterpret_cast<sampler_state *>(ptr + ST_STATE);
    uint32_t *status = status_dev ? status_dev : reinterpret_cast<uint32_t *>(ptr + ST_STATUS);
    sgnn_ctx *ctx = nullptr;
    // histogram and state are contiguous: one small fill kernel (no memset node: the call may be captured)
    SAMP_LAUNCH("sampler_static_clear_kernel", sampler_static_clear_kernel, dim3(2), dim3(SAMP_NT), hist,
                (uint32_t)((ST_STATUS - ST_HIST) / sizeof(uint32_t)));
    return sampler_launches(nullptr, N, B, seed, step, S, bitmap, rank, hist, state, reinterpret_cast<uint64_t *>(ptr + ST_CKEY),
                            reinterpret_cast<uint32_t *>(ptr + ST_CV), cand_capacity(N), reinterpret_cast<uint32_t *>(ptr + ST_WG),
                            status, nullptr, sampler_window{0, 0, 0}, st);      // no room for key prefixes in the static array: every pass recomputes the keys
}
