// pc_plan.hip -- the sieve's tile list, built on the device: estimated work
// per segment, the number of column ranges each of the leaf-dense segments is
// cut into, and the cuts.
//
// A tile of columns [col_lo, col_hi) clears the earlier columns without
// counting them, so that a segment's columns spread over many workgroups at
// little extra cost, and the same list serves one query and a batch round.
// Building it here leaves the host out of the loop: no read-back of the
// estimates, no upload of the list (two synchronisations of about 40 us per
// query), and a batch round's first segments are cut too (its launch used to
// last as long as the largest query's first segment on one workgroup).
#include "pc_block.h"
#include "pc_internal.h"
#include "pc_leafrange.h"

// Threads of a row's workgroup: a column takes some 400 instructions, so a row
// of thousands of columns is a chain of turns before the sieve can start
// (pi(10^15): 1.09 ms with 256, 1.00 with 512, 0.99 with 1024, which costs a
// batch of many short rows 1%).
#define PL_T 512

// Work is estimated in vector instructions of a wavefront, from the tile times
// of pi(10^15) .. pi(10^18): a leaf item 1 (64 items share about 64
// instructions), crossing a column before p^3 passes the segment's end 240 (all
// waves), after it (64 columns at a time) 60, answering the leaves of a column
// 200 on top.  A tile starts at about 10^4 (pattern, cleared columns, counts).
#define PL_CROSS 240u
#define PL_LARGE 60u
#define PL_ANSWER 200u
#define PL_MIN 8192u     // no tile of less work than this (unless the caller says so) ...
#define PL_FEW 256u      // ... where that leaves a CU without a tile: down to
#define PL_LEAST 2048u   // this (pi(10^9) 157 -> 120 us).  A launch with a tile for every
                         // CU stays at PL_MIN: at 10^12, 366 tiles of it, tiles down to
                         // this took 265 us where those take 211
#define PL_FINE 400000u  // up to here a tile's start is more than a few percent of it

namespace {

struct plan_row {
    uint32_t q;
    uint64_t seg, lo, hi;
};

// planned row i, or (rest) row i past the planned ones
__device__ __forceinline__ plan_row pl_row(const pc_plan_args &A, uint32_t i, bool rest)
{
    plan_row r;
    r.q = 0;
    r.seg = A.seg_first + i + (rest ? A.np : 0u);
    if (A.nq > 1) { // the k-th query of the list: pfx[k] <= i < pfx[k + 1]
        const uint32_t *const pfx = rest ? A.pfx_rest : A.pfx_plan;
        uint32_t lo = 0, hi = A.nq - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (pfx[mid] <= i)
                lo = mid;
            else
                hi = mid - 1;
        }
        r.q = A.order[lo];
        r.seg = i - pfx[lo] + (rest ? A.pfx_plan[lo + 1] - A.pfx_plan[lo] : 0u);
    }
    const uint64_t span = pc_seg_span(A.seg_log2);
    r.lo = A.lo_base + (r.seg - A.seg_base) * span;
    r.hi = r.lo + span;
    return r;
}

// Estimated work of column col in [lo, hi); *past: the column and all later
// ones are past their last hard leaf.
__device__ __forceinline__ uint32_t pl_col_work(const pc_tables &TB, const pc_query &Q,
                                                uint32_t col, uint64_t lo, uint64_t hi,
                                                uint64_t rhi, uint64_t rlo, bool *past)
{
    const uint32_t b = Q.c + 1 + col;
    const ulonglong2 ub = Q.Ub[b];
    *past = ub.y < lo;
    if (*past)
        return 0;
    const uint64_t p = TB.primes[b];
    const uint32_t w = (pc_u128)p * p * p >= hi ? PL_LARGE : PL_CROSS;
    if (ub.x >= hi)
        return w;
    uint64_t m1, m2;
    pc_leaf_mrange(Q, b, p, TB.recip[b], lo, hi, rhi, rlo, &m1, &m2);
    if (m1 > m2)
        return w;
    const float n = (float)(m2 - m1 + 1);
    // candidates prime to p_1..p_c (each read and tested, the fewer the
    // leaves), or primes (each a leaf)
    const float items = p <= Q.sqrty ? n * ((float)TB.phiQ / (float)TB.Qc)
                                     : 1.5f * n / __logf((float)m2 + 2.0f);
    return w + PL_ANSWER + (uint32_t)items;
}

__global__ __launch_bounds__(PL_T) void k_plan_work(pc_plan_args A)
{
    __shared__ uint64_t scr[PL_T / 64];
    const plan_row r = pl_row(A, blockIdx.x, false);
    const pc_query &Q = A.Qs[r.q];
    const uint64_t rhi = pc_recip(r.hi), rlo = r.lo ? pc_recip(r.lo) : 0;
    uint64_t s = 0;
    for (uint32_t col = threadIdx.x; col < Q.nb; col += PL_T) {
        bool past;
        s += pl_col_work(A.T, Q, col, r.lo, r.hi, rhi, rlo, &past);
        if (past)
            break;
    }
    s = pc_block_sum<PL_T>(s, scr);
    if (threadIdx.x == 0)
        A.work[blockIdx.x] = s;
}

// Tiles per planned row and where they go: cut rows first, then the whole
// planned rows, the rest rows (k_plan_tiles) and empty tiles up to ntiles.
// The target work of a tile: with 768 workgroups at once, a launch of many
// rows is even enough at 4096 tiles' worth; a smaller one is cut to 1536 as
// long as its tiles outweigh their start.  A.extra bounds the cuts.
#define PL_PT 1024
__global__ __launch_bounds__(PL_PT) void k_plan_counts(pc_plan_args A)
{
    __shared__ uint64_t scr[PL_PT / 64];
    __shared__ uint32_t scr32[PL_PT / 64];
    const uint32_t t = threadIdx.x;
    uint64_t s = 0;
    for (uint32_t i = t; i < A.np; i += PL_PT)
        s += A.work[i];
    const uint64_t total = pc_block_sum<PL_PT>(s, scr);
    const uint64_t least = max(min(total / PL_FEW, (uint64_t)PL_MIN), (uint64_t)PL_LEAST);
    uint64_t target = max(total / 4096, max(min(total / 1536, (uint64_t)PL_FINE), least));
    if (A.tile_work) // a caller's bound: tiles of less, not of more than the rule's (2^22,
        target = min(target, A.tile_work); // taken as it is, left pi(10^12) in one tile a row: 2.51 ms)
    target = max(target, total / A.extra + 1); // sum of ceil(work / target) <= extra + rows
    auto pieces = [&](uint32_t i) -> uint32_t {
        uint64_t k = A.tile_work == ~0ull ? 1 : (A.work[i] + target - 1) / target;
        if (k > 1) {
            const uint32_t nb = A.Qs[pl_row(A, i, false).q].nb;
            k = min(k, (uint64_t)min(nb, 4096u));
        }
        return k < 2 ? 1u : (uint32_t)k;
    };
    uint32_t cuts = 0;
    for (uint32_t i = t; i < A.np; i += PL_PT) {
        const uint32_t k = pieces(i);
        cuts += k > 1 ? k : 0u;
    }
    const uint32_t ncut = pc_block_sum<PL_PT>(cuts, scr32);
    uint32_t run_cut = 0, run_one = ncut;
    for (uint32_t i0 = 0; i0 < A.np; i0 += PL_PT) {
        const uint32_t i = i0 + t;
        const uint32_t k = i < A.np ? pieces(i) : 0u;
        uint32_t tc, to;
        const uint32_t ec = pc_block_excl_scan<PL_PT>(k > 1 ? k : 0u, scr32, &tc);
        const uint32_t eo = pc_block_excl_scan<PL_PT>(k == 1 ? 1u : 0u, scr32, &to);
        if (i < A.np)
            A.cut[i] = make_uint2(k, k > 1 ? run_cut + ec : run_one + eo);
        run_cut += tc;
        run_one += to;
    }
    if (t == 0) {
        *A.nplanned = run_one;
        *A.tile_count += run_one + A.nrest;
    }
}

// The tiles: block i < np writes those of planned row i, the other blocks the
// rest rows' and the empty ones.
__global__ __launch_bounds__(PL_T) void k_plan_tiles(pc_plan_args A)
{
    __shared__ uint64_t scr[PL_T / 64];
    if (blockIdx.x >= A.np) {
        const uint32_t f = (blockIdx.x - A.np) * PL_T + threadIdx.x;
        const uint32_t at = *A.nplanned + f;
        if (at >= A.ntiles)
            return;
        pc_tile v{0, 0, 0, 0};
        if (f < A.nrest) {
            const plan_row r = pl_row(A, f, true);
            v = pc_tile{(uint32_t)r.seg, 0, A.Qs[r.q].ncol, r.q};
        }
        A.tiles[at] = v;
        return;
    }
    const plan_row r = pl_row(A, blockIdx.x, false);
    const pc_query &Q = A.Qs[r.q];
    const uint2 c = A.cut[blockIdx.x];
    const uint32_t K = c.x;
    pc_tile *const tl = A.tiles + c.y;
    for (uint32_t j = threadIdx.x; j < K; j += PL_T) {
        tl[j].seg = (uint32_t)r.seg;
        tl[j].q = r.q;
    }
    if (threadIdx.x == 0) {
        tl[0].col_lo = 0;
        tl[K - 1].col_hi = Q.ncol;
    }
    if (K < 2)
        return;
    const uint64_t rhi = pc_recip(r.hi), rlo = r.lo ? pc_recip(r.lo) : 0;
    const uint64_t tot = A.work[blockIdx.x]; // > 0: K > 1
    uint64_t run = 0;
    for (uint32_t c0 = 0; c0 < Q.nb && run < tot; c0 += PL_T) {
        const uint32_t col = c0 + threadIdx.x;
        bool past;
        const uint64_t v = col < Q.nb ? pl_col_work(A.T, Q, col, r.lo, r.hi, rhi, rlo, &past) : 0;
        uint64_t chunk;
        const uint64_t e = run + pc_block_excl_scan<PL_T>(v, scr, &chunk);
        // tile j >= 1 starts past the first column whose inclusive prefix
        // reaches j tot / K
        for (uint64_t j = (e * K) / tot + 1; j < K && j * tot <= (e + v) * K; j++) {
            tl[j].col_lo = col + 1;
            tl[j - 1].col_hi = col + 1;
        }
        run += chunk;
    }
}

} // namespace

hipError_t pc_launch_plan(const pc_plan_args &A, hipStream_t s)
{
    if (A.nq == 0 || A.extra == 0 || A.ntiles < A.np + A.nrest + A.extra)
        return hipErrorInvalidValue;
    if (A.np)
        k_plan_work<<<A.np, PL_T, 0, s>>>(A);
    k_plan_counts<<<1, PL_PT, 0, s>>>(A);
    k_plan_tiles<<<A.np + (A.ntiles + PL_T - 1) / PL_T, PL_T, 0, s>>>(A);
    return hipGetLastError();
}
