// pc_sieve.hip -- the hot path: a segmented sieve of [1, z], z = floor(x/y),
// that reads phi(u, b-1) for every hard special leaf and pi(x/p) for every P2
// term (Sections 2.3 and 3 of the paper; the counters, blocks and per-prime
// running values phi(m_min, b) that Section 3 and Section 4 describe).
//
// Layout.  A segment holds S integers prime to 30 as an LDS bitmap: 8 bits,
// one byte, for every 30 integers (pc_w30_*; 2, 3 and 5 belong to every wheel
// of c >= 3 primes), so that 2^18 bits span 983 040 integers where an odd-only
// bitmap spans 524 288: fewer segments, so fewer visits of a sieving prime to
// a segment, fewer gather rounds and a longer run of multiples per visit (one
// pi(10^18): 49.9 -> 39.7 ms per launch).  Column j < nb stands for the
// sieving prime b = c + 1 + j (p_{c+1} .. p_bmax, bmax = pi(isqrt z)); column
// nb is the state after every sieving prime is crossed.  For every
// (segment, column) the kernel records
//   cnt = the number of integers of the segment still unsieved just before
//         p_b is crossed (column nb: after the last crossing), and
//   w   = the sum of -mu(m) over the leaves of that column whose u lands in
//         the segment (column nb: the number of P2 terms landing there),
// and it sums -mu(m) * (unsieved integers of the segment that are <= u).
// phi(u, b-1) is that in-segment count plus carry = sum of cnt over the
// earlier segments in the same column, so the carry part of the hard-leaf
// sum is sum w * carry, formed by the look-back scan below (one sieve pass
// instead of a count pass and a leaf pass; PC_MODE_COUNT / PC_MODE_LEAVES run
// the two-pass form for cross-checking).
//
// Crossing p_b clears every multiple k p_b, k >= 1, including p_b itself:
// phi(u, b) counts integers coprime to p_1..p_b, so p_b must go (unlike a
// prime sieve).  Per column the workgroup first answers the leaves, then
// crosses.  Columns are processed in order; for primes with p^3 >= hi (every
// unsieved integer below the segment end then has at most two prime factors
// >= p) each wave crosses up to 64 columns of its region in one step, one
// lane per prime: an integer n = p k unsieved at the start of the step is
// first removed by p exactly when k = 1 or k >= p, which gives the
// per-column counts without ordering the lanes.
#include "pc_block.h"
#include "pc_internal.h"
#include "pc_leafrange.h"
#include <type_traits>

// PC_PHASE_TRACE=1 adds per-phase tick counters to the tile trace (a
// profiling build; the default build only records totals)
#ifndef PC_PHASE_TRACE
#define PC_PHASE_TRACE 0
#endif


// four words of the bitmap read at once
typedef uint32_t pc_quad __attribute__((ext_vector_type(4), may_alias));

// Waves per SIMD that the LDS footprint of k_sieve<LOG2_S, T, CH> allows on a
// CU (160 KiB of LDS, at most 8 waves per SIMD); the kernel asks the compiler
// to fit its registers to that many, so a code change cannot silently cost a
// resident workgroup.
template <int T> constexpr uint32_t pc_sieve_gcap() { return 2 * T > 256 ? 2 * T : 256; }
template <int LOG2_S, int T, int CH> constexpr int pc_sieve_waves_per_simd()
{
    constexpr long NW = (1l << LOG2_S) / 32, NWV = T / 64;
    constexpr long lds = 4 * (NW + 16) + 4 * (T + 1) + 4 * pc_sieve_gcap<T>() + 4 * 2 * 64 +
                         4 * (CH + 1) + (LOG2_S > 18 ? 24 : 22) * CH + 16 * (CH / 64) + 8 + 4 * NWV + 16 * NWV;
    // (the CU hands LDS out in pieces of 1280 bytes)
    constexpr long wg = 163840 / ((lds + 1279) / 1280 * 1280);
    constexpr long waves = wg * NWV < 32 ? wg * NWV : 32;
    return waves / 4 < 1 ? 1 : (int)(waves / 4);
}

template <int LOG2_S, int T, int CH, int MODE, bool BATCH>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(
    pc_sieve_waves_per_simd<LOG2_S, T, CH>()))) void k_sieve(pc_sieve_args A)
{
    static_assert(CH <= T && CH % 64 == 0, "at most one lane per column of a chunk");
    static_assert(T % 64 == 0, "wavefront multiples");
    constexpr uint32_t S = 1u << LOG2_S;   // integers prime to 30 (bits) per segment
    constexpr uint32_t SPAN = S / 8 * 30;  // integers it covers
    constexpr uint32_t NW = S / 32;        // 32-bit words
    constexpr uint32_t BL = 9;             // 512-bit counting blocks (16 words)
    constexpr uint32_t NBLK = S >> BL;
    constexpr uint32_t NWV = T / 64;
    constexpr uint32_t BPT = NBLK / T; // counting blocks per thread
    static_assert(NBLK % T == 0 && BPT >= 1 && BPT <= 2, "every thread counts one or two blocks");
    constexpr uint32_t RS = S / NWV;   // bits of the region a wavefront owns
    constexpr uint32_t RSB = RS / 8, RSI = RSB * 30; // its bytes, the integers it covers
    constexpr uint32_t RSL = LOG2_S - (NWV == 1 ? 0 : NWV == 2 ? 1 : NWV == 4 ? 2 : NWV == 8 ? 3 : 4);
    static_assert((1u << RSL) == RS && RS == 64 * BPT * 512, "a region is 64 threads' blocks");
    constexpr uint32_t GCAP = pc_sieve_gcap<T>(); // leaf items of a gather window
    constexpr uint32_t SPT = GCAP / T;            // of which each thread takes SPT
    // more leaf items: the column is answered workgroup-wide (k_sieve at 10^18:
    // 31.3 ms from 96 items on, 30.8 from 128, 30.3 from 257, 30.7 from 449)
    constexpr uint32_t LIGHT = GCAP / 4;
    constexpr uint32_t MG = 64 / NWV < CH / 64 ? 64 / NWV : CH / 64; // groups of 64 columns of a window
    static_assert(LIGHT <= GCAP, "a light column fits a window");
    // p >= XB_P: at most 112 consecutive multipliers k reach a wave's region, so
    // at most 31 of its multiples there are prime to 30
    constexpr uint32_t XB_P = RSI / 112 + 1;
    // columns that are only cleared (clear_columns): primes below 2^6 by all
    // threads together, below 2^9 by a wavefront each, below 2^11 by half of one,
    // from SPAN / 60 = 2^(LOG2_S - 4) on by one lane, between by eight (the
    // primes below these: PI_TINY, PI_WAVE, PI_HALF, PI_SEQ)
    static_assert(LOG2_S == 15 || LOG2_S == 16 || LOG2_S == 18 || LOG2_S == 19,
                  "pi(2^11), pi(2^12), pi(2^14), pi(2^15)");
    constexpr uint32_t PI_TINY = 18, PI_WAVE = 97, PI_HALF = 309, PI_SEQ = LOG2_S == 15   ? 309
                                              : LOG2_S == 16 ? 564
                                              : LOG2_S == 18 ? 1900
                                                             : 3512;
    static_assert(GCAP >= 2 * T, "a heavy column: 64 slots of gbuf per wave, then its quarter table");

    // Word w of the segment is bm[w]; no padding, so a crossing's address is
    // its byte offset with two bits masked.  Threads that count their own
    // blocks read them 16 bytes at a time, each starting at another 16 bytes of
    // its block (rot), which keeps a wavefront's reads on distinct banks.
    __shared__ __attribute__((aligned(16))) uint32_t bm[NW + 16]; // 16 spare words: a query at
                                                                  // q = S reads past the end
    __shared__ uint32_t pre[T + 1];    // prefix of the threads' counts (build_pre)
    __shared__ uint32_t gbuf[GCAP];    // gathered leaves: k << 22 | q << 2 | (mu(m) > 0) << 1 | 1
    __shared__ uint32_t g_bin[2 * 64]; // leaves per (group of columns, region) of a window (two windows)
    __shared__ uint32_t c_off[CH + 1]; // exclusive prefix of the light columns' leaf items
    __shared__ uint32_t c_p[CH];       // p_b
    __shared__ uint32_t c_rem[CH];     // (lo / 30) mod p_b
    __shared__ uint32_t c_ls[CH];      // first leaf item (m, or index of the prime m)
    __shared__ uint32_t c_lc[CH];      // leaf items; PC_CAND: items are candidates (pc_wheel_m)
    // integers first removed by p_b in this segment.  A crossing removes over the
    // whole segment, at most S / p_b of its bits, and p_b = 7 is crossed by a
    // wheel of 3 primes: two columns share a word while S / 7 < 2^16 (2^18 / 7 =
    // 37449; of 2^19 bits it removes 74898)
    constexpr bool NEW16 = S / 7 < 65536;
    __shared__ uint32_t c_new[NEW16 ? CH / 2 : CH];
    __shared__ int32_t c_w[CH];        // sum of -mu(m) over the leaves of the column
    __shared__ uint64_t c_leafy[CH / 64];
    __shared__ uint64_t c_heavy[CH / 64];
    __shared__ uint32_t s_first_large, s_first_skip;
    __shared__ uint32_t scr32[NWV];
    __shared__ pc_s128 scr128[NWV];

    const uint64_t t_start = A.trace ? __builtin_amdgcn_s_memrealtime() : 0;
    uint32_t n_cand = 0, n_leafy = 0, n_leafy_small = 0;
#if PC_PHASE_TRACE
    // 0 set-up, 1 per-column set-up, 2 gathers, 3 heavy columns, 4 wavefront
    // columns, 5 batched crossings, 7 chunk results, 8 final column; event
    // counts: 0 column crossings by a wave, 1 answered columns, 2 gather rounds
    uint32_t ph[9] = {}, ev[3] = {};
    uint64_t ph_last = t_start;
#define PC_EV(k) (ev[k]++)
#define PC_PH(k)                                                                        \
    do {                                                                                \
        if (A.trace) {                                                                  \
            const uint64_t t_ = __builtin_amdgcn_s_memrealtime();                       \
            ph[k] += (uint32_t)(t_ - ph_last);                                          \
            ph_last = t_;                                                               \
        }                                                                               \
    } while (0)
#else
#define PC_PH(k) \
    do {         \
    } while (0)
#define PC_EV(k) ((void)0)
#endif
    pc_tile tile = A.tiles[blockIdx.x];
    tile.seg = pc_uniform(tile.seg);
    tile.col_lo = pc_uniform(tile.col_lo);
    tile.col_hi = pc_uniform(tile.col_hi);
    tile.q = pc_uniform(tile.q);
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    if (tile.col_lo >= tile.col_hi) // an empty tile
        return;
    const uint64_t seg = tile.seg;
    const uint64_t lo = A.lo_base + (seg - A.seg_base) * SPAN;
    const uint64_t hi = lo + SPAN;
    const uint64_t lob = lo / 30; // the segment's first byte (lo is a multiple of 30)
    const uint64_t row = seg - A.seg0;
    const pc_query &Q = A.Qs[tile.q];
    // this row's cells of cnt / wgt: columns [0, r_len) from r_off on (a
    // bound on the columns that still have hard leaves at or above lo)
    const uint64_t r_off = Q.row_off ? pc_uniform64(Q.row_off[row]) : row * Q.nb;
    const uint32_t r_len =
        Q.row_off ? pc_uniform((uint32_t)(Q.row_off[row + 1] - Q.row_off[row])) : Q.nb;
    const uint32_t qc = pc_uniform(Q.c);
    const uint64_t *const Xb1 = pc_uniform_ptr(Q.Xb) + qc + 1; // X_b of column j of chunk cb: Xb1[cb + j]
    const double *const Xd1 = pc_uniform_ptr(Q.Xd) + qc + 1; // and its value in fp64
    const pc_tables &TB = A.T;
    const uint64_t rhi = pc_recip(hi);
    const uint64_t rlo = lo ? pc_recip(lo) : 0;
    const uint32_t ncol = Q.ncol;

    // --- pre-sieved state: the wheel pattern (p_4..p_c already crossed), and the
    // multiples of 17 .. 67 where the tile's columns start past them: six more
    // words each instead of 40% of the clears that the columns below 1000 take
    // (with the clears by half wavefronts and more, k_sieve at 10^12 131 -> 111
    // us, decompose(10^16, 4 icbrt) 4.28 -> 4.12 ms, 10^18 30.0 -> 29.5 ms) ---
    const uint32_t col_lo = tile.col_lo, col_hi = tile.col_hi;
    const bool ps = qc == PC_PS_FIRST - 1 && col_lo >= PC_PS_LAST - qc; // (uniform)
    {
        const uint32_t P = TB.pattern_bits;
        const uint32_t g0 = (uint32_t)((8 * lob) % P);
        const uint32_t step = (32u * T) % P; // from word w to word w + T
        uint32_t off = (uint32_t)(((uint64_t)g0 + 32u * tid) % P);
        for (uint32_t w = tid; w < NW; w += T) {
            const uint32_t wi = off >> 5, sh = off & 31;
            uint32_t v = TB.pattern[wi] >> sh;
            if (sh)
                v |= TB.pattern[wi + 1] << (32 - sh);
            bm[w] = v;
            off += step;
            if (off >= P)
                off -= P;
        }
    }
    if (ps) {
        uint32_t off[PC_PS_GROUPS];
#pragma unroll
        for (uint32_t g = 0; g < PC_PS_GROUPS; g++) {
            const uint32_t P = pc_presieve_period(g);
            off[g] = ((uint32_t)(lob % P) + 4u * tid) % P;
        }
#pragma unroll 4
        for (uint32_t w = tid; w < NW; w += T) {
            uint32_t v = bm[w];
#pragma unroll
            for (uint32_t g = 0; g < PC_PS_GROUPS; g++) {
                uint32_t x;
                __builtin_memcpy(&x, TB.presieve + pc_presieve_at(g) + off[g], 4);
                v &= x;
                off[g] += 4u * T % pc_presieve_period(g);
                off[g] -= off[g] >= pc_presieve_period(g) ? pc_presieve_period(g) : 0u;
            }
            bm[w] = v;
        }
    }
    for (uint32_t i = tid; i < 128; i += T)
        g_bin[i] = 0;
    __syncthreads();

    // Thread tid's 16 BPT words, in quads of four; the step-th quad it reads is
    // step ^ rot, so that 16 consecutive threads read 16 distinct quads of the
    // banks at a time.
    constexpr uint32_t QPT = 4 * BPT;
    const uint32_t rot = BPT == 1 ? (tid >> 2) & 3u : (tid >> 1) & 7u;
    const pc_quad *const bmq = reinterpret_cast<const pc_quad *>(bm) + tid * QPT;
    auto quad_count = [&](uint32_t step) -> uint32_t {
        const pc_quad v = bmq[step ^ rot];
        return (uint32_t)(__builtin_popcount(v.x) + __builtin_popcount(v.y) +
                          __builtin_popcount(v.z) + __builtin_popcount(v.w));
    };
    // unsieved integers in each quarter (of 128 BPT bits) of thread tid's words
    auto quarter_counts = [&](uint32_t (&qs)[4]) {
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) {
            qs[k] = quad_count(k * BPT);
            if (BPT > 1)
                qs[k] += quad_count(k * BPT + 1);
        }
        // what was read k-th is quarter k ^ (rot / BPT): put back in order
        const uint32_t r = rot / BPT;
        auto swap_if = [](bool s, uint32_t &a, uint32_t &b) {
            const uint32_t t = s ? b : a;
            b = s ? a : b;
            a = t;
        };
        swap_if(r & 1u, qs[0], qs[1]);
        swap_if(r & 1u, qs[2], qs[3]);
        swap_if(r & 2u, qs[0], qs[2]);
        swap_if(r & 2u, qs[1], qs[3]);
    };
    // A thread's own words with finer sums: their unsieved count, and in *pk
    // its quarters.  A byte each while a quarter's 128 bits fit one; else the
    // prefix counts of the first one, two and three quarters, 10 bits each.
    constexpr bool QB = BPT == 1;
    auto block_counts_q = [&](uint32_t *pk) -> uint32_t {
        uint32_t qs[4];
        quarter_counts(qs);
        if (QB) {
            *pk = qs[0] | qs[1] << 8 | qs[2] << 16 | qs[3] << 24;
            return qs[0] + qs[1] + qs[2] + qs[3];
        }
        const uint32_t p1 = qs[0], p2 = p1 + qs[1], p3 = p2 + qs[2];
        *pk = p1 | (p2 << 10) | (p3 << 20);
        return p3 + qs[3];
    };
    // unsieved integers below q among the words of the thread that counts q's
    // block, from their quarters pk and total tb (not read if QB): the half of
    // q's quarter on q's side is read (up from the quarter's start, or down
    // from its end)
    constexpr uint32_t QW = 4 * BPT, HW = QW / 2; // words of a quarter, of half of one
    auto quarter_count = [&](uint32_t q, uint32_t pk, uint32_t tb) -> uint32_t {
        const uint32_t w = (q >> 5) & (QW - 1), qq = (q >> 5) / QW & 3u;
        const uint32_t part = (1u << (q & 31u)) - 1u; // bits below q in its word
        const bool up = w >= HW;
        uint32_t base; // the count at the quarter's start, or (up) at its end
        if (QB) {
            base = __builtin_amdgcn_sad_u8(pk & ((1u << 8u * qq) - 1u), 0u, 0u) +
                   (up ? (pk >> 8u * qq) & 255u : 0u);
        } else {
            const uint32_t below = qq ? (pk >> (10u * (qq - 1u))) & 1023u : 0u;
            const uint32_t through = qq < 3u ? (pk >> (10u * qq)) & 1023u : tb;
            base = up ? through : below;
        }
        const uint32_t *const v = bm + ((q >> 5) & ~(QW - 1)) + (up ? HW : 0u);
        const uint32_t wh = up ? w - HW : w; // q's word in the half
        uint32_t lt = 0, all = 0;            // bits of the half below q, all of them
#pragma unroll
        for (uint32_t k = 0; k < HW; k++) {
            const uint32_t b = v[k];
            lt += (uint32_t)__builtin_popcount(b & (k < wh ? ~0u : k == wh ? part : 0u));
            all += (uint32_t)__builtin_popcount(b);
        }
        return base + lt - (up ? all : 0u);
    };

    // pre[] = exclusive prefix of the threads' counts, with the quarter
    // prefixes of every thread's words beside it in the half of gbuf that no
    // leaf occupies meanwhile; returns the segment total.  Every thread must
    // call it; a wave reads only words of its own region before the first
    // barrier.
    uint32_t *const preq = gbuf + GCAP - T;
    auto build_pre = [&]() -> uint32_t {
        uint32_t pq;
        const uint32_t n = block_counts_q(&pq), inc = pc_wave_incl_scan_u32(n);
        const uint32_t w = tid >> 6;
        if (lane == 63)
            scr32[w] = inc;
        __syncthreads(); // every wave is past what it read of pre, gbuf and scr32 before
        uint32_t ex = inc - n;
#pragma unroll
        for (uint32_t i = 0; i < NWV; i++)
            ex += i < w ? scr32[i] : 0u;
        pre[tid] = ex;
        preq[tid] = pq;
        if (tid == T - 1)
            pre[T] = ex + n;
        __syncthreads();
        return pre[T];
    };
    // unsieved integers among bits [0, q), q <= S, against build_pre
    auto count_pre = [&](uint32_t q) -> uint32_t {
        const uint32_t i = q / (512 * BPT);
        const uint32_t ex = pre[i];
        return q < S ? ex + quarter_count(q, preq[i], QB ? 0u : pre[i + 1] - ex) : ex;
    };
    const double lobd = (double)lob;
    auto rem_lob = [&](uint32_t p, double rp) -> uint32_t { return pc_rem_near(lob, lobd, p, rp); };
    // The multiples of a prime p by residue class: the multipliers 30 k + res(i)
    // fall on byte p k + floor(p res(i) / 30) of the integers, always at one bit
    // of it.  With p = 30 a + res(g) the byte's part that depends on i is
    // a res(i) + floor(res(g) res(i) / 30); the second term and the bit come
    // from byte g of two words that a lane keeps for its i = lane mod 8.
    const uint32_t l_res = pc_w30_res(lane & 7u);
    uint32_t l_tab0 = 0, l_tab1 = 0;
#pragma unroll
    for (uint32_t g = 0; g < 8; g++) {
        const uint32_t v = pc_w30_res(g) * l_res, e = v / 30u;
        const uint32_t byte = e << 3 | (v - 30u * e) * 17u >> 6;
        if (g < 4)
            l_tab0 |= byte << (8 * g);
        else
            l_tab1 |= byte << (8 * (g - 4));
    }
    // the lane's class of p: *bit, and the byte of 30 k + res(i) past p k
    const uint32_t l_res8 = 8u * l_res;
    auto class_of = [&](uint32_t p, uint32_t *bit) -> uint32_t {
        const uint32_t a = p / 30u, g = ((p - 30u * a) * 17u) >> 6; // g: the residue's number
        const uint32_t eb = __builtin_amdgcn_perm(l_tab1, l_tab0, 0x0c0c0c00u | g);
        *bit = eb & 7u;
        return l_res * a + (eb >> 3);
    };

    // Clear the multiples of the columns [k0, k1) (their primes lie in order),
    // in any order, with no counts: columns whose state no leaf of this tile
    // reads.  Ends with a barrier.  Every thread must call it.
    auto clear_columns = [&](uint32_t k0, uint32_t k1) {
        char *const sb = reinterpret_cast<char *>(bm);
        for (uint32_t kb = k0; kb < k1; kb += CH) {
            const uint32_t n = min((uint32_t)CH, k1 - kb);
            const uint32_t b0 = qc + 1 + kb;
            const uint32_t ntiny = min(n, PI_TINY + 1 - min(PI_TINY + 1, b0));
            const uint32_t nwave = min(n, PI_WAVE + 1 - min(PI_WAVE + 1, b0));
            const uint32_t nhalf = min(n, PI_HALF + 1 - min(PI_HALF + 1, b0));
            const uint32_t nseq = n - min(n, PI_SEQ + 1 - min(PI_SEQ + 1, b0));
            if (tid < n) {
                const uint32_t b = qc + 1 + kb + tid, p = TB.primes[b];
                const uint32_t rem = rem_lob(p, TB.rcpd[b]);
                c_p[tid] = p;
                c_rem[tid] = rem;
                if (tid >= n - nseq) { // few multiples: one lane takes them in order
                    const uint32_t r30 = 30u * rem;
                    const uint32_t q = pc_quot_near(r30, p, __builtin_amdgcn_rcpf((float)p));
                    const uint32_t j = pc_w30_next(q + (q * p != r30 ? 1u : 0u));
                    uint32_t gap = __builtin_amdgcn_alignbit(PC_W30_GAPS, PC_W30_GAPS,
                                                             4u * ((j * 17u >> 6) & 7u));
                    for (uint32_t d = j * p - r30; d < SPAN;) {
                        const uint32_t bit = pc_w30_bit(d);
                        __hip_atomic_fetch_and(bm + (bit >> 5), ~(1u << (bit & 31)),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        d += (gap & 15u) * p;
                        gap = __builtin_amdgcn_alignbit(gap, gap, 4);
                    }
                }
            }
            __syncthreads();
            // L lanes a column, L / 8 rounds of its eight classes side by side: a
            // lane's multiples lie L / 8 p bytes apart, at one bit of their words
            // for L >= 32 (eight lanes alone take 500 steps in turn for p = 67: 14
            // us, where the whole tile of a small query takes 60)
            auto by_lanes = [&](auto lanes, uint32_t k0, uint32_t k1) {
                constexpr uint32_t L = decltype(lanes)::value;
                for (uint32_t k = k0 + tid / L; k < k1; k += T / L) {
                    const uint32_t p = c_p[k], step = L / 8 * p;
                    uint32_t bit;
                    const uint32_t e = class_of(p, &bit);
                    int32_t at = (int32_t)(tid % L / 8 * p + e) - (int32_t)c_rem[k];
                    const uint32_t keep = ~(1u << ((((uint32_t)at << 3) | bit) & 31u));
                    if (at < 0)
                        at += (int32_t)step;
                    at &= ~3;
                    auto clear = [&](int32_t w) {
                        __hip_atomic_fetch_and(reinterpret_cast<uint32_t *>(sb + w), keep,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    };
                    for (; at < (int32_t)(SPAN / 30 - min(SPAN / 30, step)); at += 2 * (int32_t)step) {
                        clear(at);
                        clear(at + (int32_t)step);
                    }
                    if (at < (int32_t)(SPAN / 30))
                        clear(at);
                }
            };
            by_lanes(std::integral_constant<uint32_t, T>{}, 0, ntiny);
            by_lanes(std::integral_constant<uint32_t, 64>{}, ntiny, nwave);
            by_lanes(std::integral_constant<uint32_t, 32>{}, nwave, nhalf);
            // the others: one lane per class of a column
            for (uint32_t k = nhalf + (tid >> 3); k < n - nseq; k += T / 8) {
                const uint32_t p = c_p[k];
                uint32_t bit;
                int32_t at = (int32_t)class_of(p, &bit) - (int32_t)c_rem[k];
                if (at < 0)
                    at += (int32_t)p;
                for (; at < (int32_t)(SPAN / 30); at += (int32_t)p)
                    __hip_atomic_fetch_and(reinterpret_cast<uint32_t *>(sb + (at & ~3)),
                                           ~(1u << ((((uint32_t)at << 3) | bit) & 31u)),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
        }
    };

    // a tile that owns the columns from col_lo on needs the earlier ones only cleared
    if (col_lo)
        clear_columns(ps ? PC_PS_LAST - qc : 0u, col_lo);
    uint32_t total = build_pre();
    PC_PH(0);
    // Wavefront wv owns bits [R0, R1).  rc = its unsieved integers, kept exact
    // through every crossing: a leaf whose u lies in a higher region counts
    // all of them, one in this region counts a prefix of it.
    const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t R0 = wv * RS, R1 = R0 + RS;
    uint32_t rc = (uint32_t)__builtin_amdgcn_readfirstlane((int)(pre[64 * wv + 64] - pre[64 * wv]));
    // unsieved integers of this wave's region below bit q of the segment (in:
    // q lies in the region or at the segment's end), from the lanes' counts c0, their exclusive
    // prefix pe and quarters pq
    auto region_count = [&](bool in, uint32_t q, uint32_t pe, uint32_t c0, uint32_t pq) -> uint32_t {
        const uint32_t d = in ? q - R0 : 0u;
        const int32_t src = (int32_t)min(d / (512 * BPT), 63u);
        uint32_t c = (uint32_t)__shfl((int)pe, src, 64);
        const uint32_t pk = (uint32_t)__shfl((int)pq, src, 64);
        const uint32_t tb = QB ? __builtin_amdgcn_sad_u8(pk, 0u, 0u)
                               : (uint32_t)__shfl((int)c0, src, 64);
        if (in) // (q = S, past the last region's last bit, counts all of it)
            c += d < RS ? quarter_count(q, pk, tb) : tb;
        return c;
    };
    unsigned long long nleaf = 0;      // hard leaves answered by this thread
    int64_t acc_local = 0;             // sum of -mu(m) * in-segment count (hard leaves)
    int64_t acc_p2 = 0;                // sum of in-segment counts (P2 terms)
    pc_s128 acc_carry = 0;             // PC_MODE_LEAVES: carry * w
    uint32_t g_par = 0;                // g_bin half of the current window

    // Leaf item it of column j: *m and *w = -mu(m), false if the candidate m
    // is not squarefree with lpf(m) > p_b.
    auto leaf_filter = [&](uint32_t j, uint32_t it, uint32_t *m, int32_t *w) -> bool {
        const uint32_t lc = c_lc[j], ls = c_ls[j];
        if (lc & PC_CAND) {
            const int32_t v = TB.mulpfw[ls + it];
            const uint32_t av = v < 0 ? (uint32_t)(-v) : (uint32_t)v;
            n_cand++;
            *m = pc_wheel_m(TB, ls + it);
            *w = v > 0 ? -1 : 1;
            return av > c_p[j];
        }
        *m = TB.primes[ls + it];
        *w = 1;
        return true;
    };
    // q = bits of the segment up to u = floor(X_b / m), u in [lo, hi); X is X_b
    // modulo 2^32 and Xd its value in fp64 (an IEEE division with a 64-bit
    // remainder takes five times the instructions of pc_quot_off).
    const double qbase = 0.25 - (double)lo;
    // *bad collects quotients outside the segment (never, if the m range is
    // right; leaf_check flags them), which are taken as its last bit here.
    auto leaf_q = [&](uint32_t X, double Xd, uint32_t m, uint32_t *bad) -> uint32_t {
        bool in;
        const uint32_t off = pc_quot_off(X, Xd, m, (uint32_t)lo, qbase, SPAN, &in);
        *bad |= in ? 0u : 1u;
        return pc_w30_le(min(off, SPAN - 1));
    };
    auto leaf_check = [&](uint32_t bad) {
        if (bad)
            atomicOr(A.err, 2);
    };

    const uint32_t ncross = min(col_hi, Q.nb);
    bool recounted = false; // the carried count was checked against the bitmap (uniform)
    for (uint32_t cb = col_lo; cb < ncross; cb += CH) {
        const uint32_t jall = min((uint32_t)CH, ncross - cb);
        if (tid == 0) {
            s_first_large = jall;
            s_first_skip = jall;
        }
        if (tid < (NEW16 ? CH / 2 : CH))
            c_new[tid] = 0;
        __syncthreads();
        // --- one lane per column: first multiple, leaf range ---
        bool leafy = false, heavy = false, large = false, skip = false;
        uint32_t light = 0; // leaf items to gather
        if (tid < jall) {
            const uint32_t j = tid, col = cb + j, b = qc + 1 + col;
            const uint64_t p = TB.primes[b];
            const uint64_t rp = TB.recip[b];
            c_p[j] = (uint32_t)p;
            c_rem[j] = rem_lob((uint32_t)p, TB.rcpd[b]);
            large = (pc_u128)p * p * p >= hi;
            uint32_t ls = 0, lc = 0;
            // every hard leaf of b and of the later primes lies below ub.y
            const ulonglong2 ub = Q.Ub[b];
            skip = ub.y < lo;
            if (MODE != PC_MODE_COUNT && ub.x < hi && !skip)
                pc_leaf_range(TB, Q, b, p, rp, lo, hi, rhi, rlo, &ls, &lc);
            c_ls[j] = ls;
            c_lc[j] = lc;
            c_w[j] = 0;
            leafy = lc != 0;
            heavy = (lc & ~PC_CAND) > LIGHT;
            light = heavy ? 0u : lc & ~PC_CAND;
            n_leafy += leafy ? 1u : 0u;
            n_leafy_small += leafy && !large ? 1u : 0u;
        }
        {
            uint32_t tot;
            const uint32_t ex = pc_block_excl_scan<T>(light, scr32, &tot);
            if (tid < CH)
                c_off[tid] = ex;
            if (tid == T - 1)
                c_off[CH] = tot;
        }
        {
            const uint64_t bl = __ballot(leafy), bh = __ballot(heavy), bg = __ballot(large);
            const uint64_t bs = __ballot(skip);
            if (lane == 0 && tid < CH) {
                c_leafy[tid >> 6] = bl;
                c_heavy[tid >> 6] = bh;
                if (bg)
                    atomicMin(&s_first_large, (tid & ~63u) + (uint32_t)__builtin_ctzll(bg));
                if (bs)
                    atomicMin(&s_first_skip, (tid & ~63u) + (uint32_t)__builtin_ctzll(bs));
            }
        }
        __syncthreads();
        PC_PH(1);
        // columns [jend, jall) and every later chunk's are past their last hard
        // leaf (skip, a suffix): they are only cleared, after this chunk
        const uint32_t jend = s_first_skip;
        const uint32_t first_large = BATCH ? min(s_first_large, jend) : jend;

        // For 64 columns from cg0 on (one column per lane): p, the region's
        // first byte modulo p (v_r), and the first multiple of p in the region
        // prime to 30, v_j p - 30 v_r integers from its start (v_d; RSI or
        // more: none), computed together; v_rem collects each column's
        // removals in its lane and goes to c_new once per 64 columns.  With
        // k0 = floor(first byte / p), the multiple's multiplier is 30 k0 + v_j,
        // v_j <= 31.
        uint32_t cg0 = 0x80000000u, v_p = 1, v_r = 0, v_j = 0, v_d = RSI, v_rem = 0;
            // (j - cg0 >= 64: reload)
        auto flush_removed = [&]() {
            const uint32_t col = cg0 + lane;
            if (v_rem)
                atomicAdd(&c_new[NEW16 ? col >> 1 : col], NEW16 ? v_rem << ((col & 1u) * 16u) : v_rem);
            v_rem = 0;
        };
        auto load_group = [&](uint32_t j) { // the columns from j on
            {
                flush_removed();
                cg0 = j;
                v_p = 1;
                v_r = 0;
                v_j = 0;
                v_d = RSI;
                if (j + lane < jend) {
                    const uint32_t p = c_p[j + lane];
                    const uint32_t e = c_rem[j + lane] + wv * RSB;
                    const float rp = __builtin_amdgcn_rcpf((float)p);
                    const uint32_t r = e - pc_quot_near(e, p, rp) * p;
                    // the least multiplier that reaches the region: ceil(30 r / p)
                    const uint32_t r30 = 30u * r, q = pc_quot_near(r30, p, rp);
                    v_p = p;
                    v_r = r;
                    v_j = pc_w30_next(q + (q * p != r30 ? 1u : 0u));
                    v_d = v_j * p - r30;
                }
            }
        };
        // a group that holds column j
        auto ensure_group = [&](uint32_t j) {
            if (j - cg0 >= 64)
                load_group(j);
        };
        // Cross column cg0 + k, which has a multiple in this wave's region.
        // Lane (i, t) = (lane mod 8, lane / 8) takes the multipliers
        // 30 (k0 + t + 8 s) + res(i), s = 0, 1, ...: bit
        // 8 ((t + 8 s) p + a res(i)) + class byte - 8 v_r of the region (the
        // class byte is 8 floor(res(g) res(i) / 30) + its bit), so a lane's
        // multiples lie 64 p bits, 2 p words, apart at one bit of their words.
        // Most of the sparse segments' time goes here, one visit per (column,
        // region) with 15 to 60 multiples: 16 vector instructions when one
        // round does it, the rest scalar (25 with bytes and bits apart, and
        // two 32-bit multiplies among them; k_sieve at 10^18 33.4 -> 32.8 ms).
        auto cross_k = [&](int32_t k) {
            PC_EV(0);
            const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)v_p, k);
            const uint32_t r8 = 8u * (uint32_t)__builtin_amdgcn_readlane((int)v_r, k);
            const uint32_t a = p / 30u, g = ((p - 30u * a) * 17u) >> 6; // g: the residue's number
            const uint32_t eb = __builtin_amdgcn_perm(l_tab1, l_tab0, 0x0c0c0c00u | g);
            // bit of the region in round 0 (negative or RS and more: none)
            const int32_t x = (int32_t)(__umul24(lane & 56u, p) + (__umul24(l_res8, a) + eb) - r8);
            const uint32_t bit = 1u << (x & 31), keep = ~bit;
            uint32_t *w = bm + (int32_t)(wv * (RS / 32)) + (x >> 5);
            const int32_t step = (int32_t)(64u * p); // bits per round
            auto clear = [&](uint32_t *at) -> uint32_t {
                return __hip_atomic_fetch_and(at, keep, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP) & bit;
            };
            uint32_t old = 0;
            if ((uint32_t)x < RS)
                old = clear(w);
            uint32_t removed = (uint32_t)__builtin_popcountll(__ballot(old != 0));
            // Round s: -8 p < bit - s step < step.  From s = 1 on no lane lies
            // below the region, and none past its end while (s + 1) step <= RS.
            if (step < (int32_t)(RS + 8u * p)) {
                int32_t top = 2 * step; // of the next round
                const uint32_t dw = 2u * p;
                w += dw;
                if (top <= (int32_t)RS) {
                    const uint32_t sh = x & 31;
                    uint32_t hits = 0;
                    for (; top + step <= (int32_t)RS; top += 2 * step, w += 2 * dw)
                        hits += (clear(w) >> sh) + (clear(w + dw) >> sh); // two in flight
                    if (top <= (int32_t)RS) {
                        hits += clear(w) >> sh;
                        top += step;
                        w += dw;
                    }
                    removed += pc_wave_sum_u32(hits);
                }
                for (; top - step < (int32_t)(RS + 8u * p); top += step, w += dw) {
                    old = 0;
                    if ((uint32_t)(x + top - step) < RS)
                        old = clear(w);
                    removed += (uint32_t)__builtin_popcountll(__ballot(old != 0));
                }
            }
            rc -= removed;
            v_rem = pc_write_lane(v_rem, (uint32_t)k, removed);
        };
        auto cross_region = [&](uint32_t j) {
            ensure_group(j);
            const int32_t k = (int32_t)(j - cg0);
            if ((uint32_t)__builtin_amdgcn_readlane((int)v_d, k) < RSI)
                cross_k(k);
        };
        // Large columns [ja, jb) of the cached group (every one at or past
        // first_large, with p >= XB_P) crossed in this wave's region in one
        // step, one lane per column.  An integer n = p k unsieved at the start
        // is first removed by p exactly when k = 1 or k >= p (p^3 >= hi leaves
        // n at most two prime factors, none below the first column's prime),
        // so each lane first reads its multiples and credits those, then
        // clears them; the order of the columns no longer matters.  The gathered
        // leaves [es0, es1) (all of this region) of these columns are answered in
        // between: their count at the start, less the credited multiples below
        // them of the earlier columns.
        auto xbatch = [&](uint32_t ja, uint32_t jb, uint32_t es0, uint32_t es1) {
            const uint32_t col = cg0 + lane;
            const uint32_t p = v_p, d0 = col >= ja && col < jb ? v_d : RSI;
            const uint32_t *const rw = bm + wv * (RS / 32);
            // the gaps between multipliers from the first one on, a nibble each
            const uint32_t gi = (v_j * 17u >> 6) & 7u; // (v_j = 31 is residue 1 again: 0)
            const uint32_t gap0 = __builtin_amdgcn_alignbit(PC_W30_GAPS, PC_W30_GAPS, 4u * gi);
            // n = rlo + d >= p^2  <=>  d >= tb;  n = p  <=>  d = ip
            const uint64_t p2 = (uint64_t)p * p, rlo = lo + wv * RSI;
            const uint32_t tb = p2 <= rlo ? 0u : (uint32_t)min<uint64_t>(RSI, p2 - rlo);
            const uint32_t ip = rlo <= p ? (uint32_t)(p - rlo) : RSI;
            uint32_t cm = 0; // credited multiples: bit i <-> the region's i-th multiple
            {
                uint32_t d = d0, gap = gap0;
                for (uint32_t i = 1; __ballot(d < RSI); i <<= 1)
                    if (d < RSI) {
                        const uint32_t bit = pc_w30_bit(d);
                        if (((rw[bit >> 5] >> (bit & 31)) & 1u) && (d >= tb || d == ip))
                            cm |= i;
                        d += (gap & 15u) * p;
                        gap = __builtin_amdgcn_alignbit(gap, gap, 4);
                    }
            }
            if (es0 < es1) {
                bool have = false;
                uint32_t pe = 0, pc0 = 0, pq = 0; // lane prefix of the region's block counts;
                // first block (or, one block a lane, its count and quarter prefixes)
                const float rp = __builtin_amdgcn_rcpf((float)p);
                // the region's multiples of the lane's column up to n integers past
                // its start: multipliers k <= (n + 30 v_r) / p, less those before v_j
                const uint32_t k0 = v_j == 31u ? 8u : v_j * 17u >> 6;
                auto multiples_to = [&](uint32_t n) -> uint32_t {
                    return pc_w30_le(pc_quot_near(n + 30u * v_r, p, rp)) - k0;
                };
                for (uint32_t s = es0; s < es1; s += 64) {
                    const uint32_t e = s + lane < es1 ? gbuf[s + lane] : 0u;
                    const uint32_t q = (e >> 2) & 0xFFFFFu;
                    const bool in = (e & 1) && (e >> 22) >= ja - cg0;
                    uint64_t pend = __ballot(in);
                    if (!pend)
                        continue;
                    if (!have) {
                        pc0 = block_counts_q(&pq);
                        pe = pc_wave_incl_scan_u32(pc0) - pc0;
                        have = true;
                    }
                    uint32_t c = region_count(in, q, pe, pc0, pq);
                    // less the earlier columns' credited multiples below q:
                    // leaf by leaf (all lanes count for one leaf) or column
                    // by column (all leaves count one column), the shorter
                    uint64_t cols = __ballot(cm != 0);
                    if (4 * __builtin_popcountll(pend) <= __builtin_popcountll(cols)) {
                        while (pend) {
                            const int32_t l = (int32_t)__builtin_ctzll(pend);
                            pend &= pend - 1;
                            const uint32_t ql = (uint32_t)__builtin_amdgcn_readlane((int)q, l);
                            const uint32_t kl = (uint32_t)__builtin_amdgcn_readlane((int)e, l) >> 22;
                            uint32_t below = 0;
                            if (ql > R0) {
                                const uint32_t n = pc_w30_int(ql - R0 - 1); // the last integer counted
                                if (lane < kl && cm != 0 && n >= d0) {
                                    const uint32_t t = multiples_to(n); // 1 .. 31
                                    below = (uint32_t)__builtin_popcount(cm & ((1u << t) - 1u));
                                }
                            }
                            const uint32_t tot = pc_wave_sum_u32(below);
                            if (lane == (uint32_t)l)
                                c -= tot;
                        }
                    } else {
                        // n: the last integer that the leaf counts; a credited
                        // multiple d of column k lies below it if d <= n
                        const int32_t ke = (int32_t)(e >> 22);
                        const int32_t n = in && q > R0 ? (int32_t)pc_w30_int(q - R0 - 1) : -1;
                        while (cols) {
                            const int32_t k = (int32_t)__builtin_ctzll(cols);
                            cols &= cols - 1;
                            const uint32_t dk = (uint32_t)__builtin_amdgcn_readlane((int)d0, k);
                            const uint32_t pk = (uint32_t)__builtin_amdgcn_readlane((int)p, k);
                            const uint32_t gk = (uint32_t)__builtin_amdgcn_readlane((int)gi, k);
                            uint32_t ck = (uint32_t)__builtin_amdgcn_readlane((int)cm, k);
                            const int32_t nk = ke > k ? n : -1;
                            const uint32_t r0 = pc_w30_res(gk);
                            while (ck) { // (positions in scalar arithmetic)
                                const uint32_t i = gk + (uint32_t)__builtin_ctz(ck);
                                ck &= ck - 1;
                                const uint32_t d = dk + (pc_w30_int(i) - r0) * pk;
                                c -= (int32_t)d <= nk ? 1u : 0u;
                            }
                        }
                    }
                    if (in)
                        acc_local += (e & 2) ? -(int64_t)c : (int64_t)c;
                }
            }
            {
                uint32_t d = d0, gap = gap0;
                while (__ballot(d < RSI))
                    if (d < RSI) {
                        const uint32_t bit = pc_w30_bit(d);
                        __hip_atomic_fetch_and(bm + wv * (RS / 32) + (bit >> 5), ~(1u << (bit & 31)),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        d += (gap & 15u) * p;
                        gap = __builtin_amdgcn_alignbit(gap, gap, 4);
                    }
            }
            const uint32_t cr = (uint32_t)__builtin_popcount(cm);
            if (d0 < RSI)
                v_rem = cr;
            rc -= pc_wave_sum_u32(cr);
        };
        // the first column of [j, je) (within the cached group) from which on
        // xbatch applies, or je
        auto xbatch_from = [&](uint32_t j, uint32_t je) -> uint32_t {
            if (!BATCH)
                return je;
            const uint32_t col = cg0 + lane;
            const uint64_t lg = __ballot(col >= j && col < je && col >= first_large && v_p >= XB_P);
            return lg ? cg0 + (uint32_t)__builtin_ctzll(lg) : je;
        };
        // cross the leafless columns [j, je) in this wave's region, visiting
        // only those with a multiple in it
        auto cross_run = [&](uint32_t j, uint32_t je) {
            while (j < je) {
                ensure_group(j);
                const uint32_t ge = min(je, cg0 + 64);
                const uint32_t xb = xbatch_from(j, ge);
                uint64_t msk = __ballot(v_d < RSI && cg0 + lane >= j && cg0 + lane < xb);
                while (msk) {
                    const int32_t k = (int32_t)__builtin_ctzll(msk);
                    msk &= msk - 1;
                    cross_k(k);
                }
                if (xb < ge)
                    xbatch(xb, ge, 0, 0);
                j = ge;
            }
        };

        // Gather windows.  The leaves of the light columns of a window (columns
        // in order from a leafy one on, up to the next heavy one, MG groups of
        // 64 columns or GCAP leaf items) are found by the whole workgroup, one
        // item per slot, and put into gbuf in bins by (group of 64 columns,
        // region of u), so that a wave finds the leaves of its own region, and
        // those of the regions above it, side by side: all lanes of an answer
        // hold leaves (in slot order one in NWV did; one pi(10^18): 39.7 -> 34.6 ms
        // per launch), and a window needs no barrier past its gather.
        uint32_t v_bin = 0, w_used = 0; // lane i: the first leaf of bin i in gbuf; the leaves held
        auto bin_at = [&](uint32_t i) -> uint32_t {
            return i < 64 ? (uint32_t)__builtin_amdgcn_readlane((int)v_bin, (int)i) : w_used;
        };
        // the window from the leafy light column j0 on; returns its end
        auto gather = [&](uint32_t j0) -> uint32_t {
            PC_PH(4);
            PC_EV(2);
            g_par ^= 1;
            // the next heavy column at or after j0 ends the window
            uint32_t lim = jend;
            {
                uint32_t wd = j0 >> 6;
                uint64_t msk = c_heavy[wd] & (~0ull << (j0 & 63));
                while (!msk && ++wd < (jend + 63) / 64)
                    msk = c_heavy[wd];
                if (msk)
                    lim = min(jend, wd * 64 + (uint32_t)__builtin_ctzll(msk));
            }
            lim = min(lim, j0 + 64 * MG);
            const uint32_t o0 = c_off[j0];
            uint32_t we = j0;
            for (uint32_t base = j0; base < lim; base += 64) {
                const uint32_t col = base + lane;
                bool ok = false;
                if (col < lim)
                    ok = c_off[col + 1] - o0 <= GCAP;
                const uint64_t m = __ballot(ok);
                we = base + (uint32_t)__builtin_popcountll(m);
                if (~m)
                    break;
            }
            const uint32_t used = pc_uniform(c_off[we] - o0);
            const uint32_t h0 = we - j0 > 1 ? 1u << (31 - __builtin_clz(we - j0 - 1)) : 0u;
            uint32_t *const bins = g_bin + g_par * 64;
            if (tid < 64)
                g_bin[(g_par ^ 1) * 64 + tid] = 0; // the next window's
            uint32_t ee[SPT], bn[SPT], rk[SPT], bad = 0;
#pragma unroll
            for (uint32_t i = 0; i < SPT; i++) {
                ee[i] = 0;
                bn[i] = 0;
                rk[i] = 0;
                const uint32_t s = i * T + tid;
                if (i * T + wv * 64 >= used) // (uniform in the wave)
                    continue;
                // the column of slot s: the last one whose offset is <= s
                uint32_t a = j0, oa = 0;
                for (uint32_t h = h0; h; h >>= 1) {
                    const uint32_t c = a + h;
                    const uint32_t o = c < we ? c_off[c] - o0 : 0xFFFFu;
                    if (o <= s) {
                        a = c;
                        oa = o;
                    }
                }
                int32_t wl = 0; // -mu(m) of this slot's leaf, 0 if none
                if (s < used) {
                    uint32_t m;
                    int32_t w;
                    if (leaf_filter(a, s - oa, &m, &w)) {
                        const uint32_t q = leaf_q((uint32_t)Xb1[cb + a], Xd1[cb + a], m, &bad);
                        ee[i] = ((a - j0) & 63u) << 22 | (q << 2) | (w < 0 ? 2u : 0u) | 1u;
                        bn[i] = ((a - j0) >> 6) * NWV + min(q >> RSL, NWV - 1);
                        rk[i] = atomicAdd(&bins[bn[i]], 1u);
                        wl = w;
                        nleaf++;
                    }
                }
                // The wave's slots are consecutive, so its lanes hold runs of one
                // column: its weight takes one add per run, from a wave scan.
                const uint32_t key = s < used ? a : 0xFFFFu;
                const uint32_t inc = pc_wave_incl_scan_u32((uint32_t)wl);
                const uint32_t key_next = (uint32_t)__shfl_down((int)key, 1, 64);
                const bool tail = lane == 63 || key_next != key;
                const uint64_t below = __ballot(tail) & ((1ull << lane) - 1);
                const int32_t pt = below ? 63 - __builtin_clzll(below) : 0;
                const uint32_t base = (uint32_t)__shfl((int)inc, pt, 64);
                const int32_t run = (int32_t)(inc - (below ? base : 0u));
                if (tail && key != 0xFFFFu && run != 0)
                    atomicAdd(&c_w[key], run);
            }
            leaf_check(bad);
            __syncthreads(); // (and every wave is past the last window's leaves)
            const uint32_t n = bins[lane], inc = pc_wave_incl_scan_u32(n);
            v_bin = inc - n;
            w_used = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
#pragma unroll
            for (uint32_t i = 0; i < SPT; i++) {
                const uint32_t at = (uint32_t)__shfl((int)v_bin, (int)bn[i], 64) + rk[i];
                if (ee[i])
                    gbuf[at] = ee[i];
            }
            __syncthreads();
            PC_PH(2);
            return we;
        };
        // For each column of the group (one a lane) the pieces of 64 of this wave's
        // leaves [s0, s1) that hold leaves of it, a bit each, gathered in the wave's
        // words of pre (which nothing reads between build_pre and the next one).  A
        // column's leaves lie side by side but for the order of the waves that put
        // them there, so they fill one to three pieces of up to 32.  Where z is small
        // all leaves fall into the first region, and reading every piece for every
        // column took longer than the crossings (batches of 4096 queries of 10^6.1 ..
        // 10^8: 2.57 -> 2.08 ms, of 10^8 .. 10^9: 3.73 -> 3.03; one pi(10^18) 34.7 ->
        // 34.3).  Bins of a single piece go the same way: a test for them costs the
        // sparse segments more (one pi(10^18) 34.5 ms, pi(2^66) 531 ms against 525).
        uint32_t *const cpiece = pre + 64 * wv;
        static_assert(GCAP <= 64 * 32, "a bit per piece");
        auto find_pieces = [&](uint32_t s0, uint32_t s1) -> uint32_t {
            cpiece[lane] = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (uint32_t s = s0, bit = 1; s < s1; s += 64, bit <<= 1)
                if (s + lane < s1)
                    __hip_atomic_fetch_or(cpiece + (gbuf[s + lane] >> 22), bit, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            return cpiece[lane];
        };
        // The leaves of column cg0 + k among this wave's [s0, s1) (e0: the
        // first 64 of them, one a lane; pieces: find_pieces' word of the column): a
        // prefix of the region for each.
        auto answer = [&](uint32_t k, uint32_t s0, uint32_t s1, uint32_t e0, uint32_t pieces) {
            PC_EV(1);
            bool have = false;
            uint32_t pe = 0, pc0 = 0, pq = 0; // the lanes' counts, as in xbatch
            for (; pieces; pieces &= pieces - 1) {
                const uint32_t s = s0 + 64u * (uint32_t)__builtin_ctz(pieces);
                const uint32_t e = s == s0 ? e0 : s + lane < s1 ? gbuf[s + lane] : 0u;
                const uint32_t q = (e >> 2) & 0xFFFFFu;
                const bool in = (e & 1) && (e >> 22) == k;
                if (__ballot(in)) {
                    if (!have) {
                        pc0 = block_counts_q(&pq);
                        pe = pc_wave_incl_scan_u32(pc0) - pc0;
                        have = true;
                    }
                    const uint32_t c = region_count(in, q, pe, pc0, pq);
                    if (in)
                        acc_local += (e & 2) ? -(int64_t)c : (int64_t)c;
                }
            }
        };
        // Many leaves: the whole workgroup answers them against pre[].  A wave
        // takes 64 items at a time, wave wv the pieces wv, wv + NWV, ..., each
        // next piece's table reads in flight while one is worked off (the first
        // one's while the counts are built).  Prime items are all leaves; the
        // candidates that pass the table's test are packed into the wave's 64
        // slots of gbuf, so that the divisions and counts run on full
        // wavefronts.  Three barriers a column: a wave counts only words of its
        // own region, so it need not wait for the others' crossings first.
        auto heavy_col = [&](uint32_t j) {
            PC_PH(4);
            const uint32_t lc = c_lc[j], n = lc & ~PC_CAND, ls = pc_uniform(c_ls[j]);
            const bool cand = pc_uniform(lc) & PC_CAND;
            const uint32_t p = c_p[j];
            const uint32_t *const src =
                (cand ? reinterpret_cast<const uint32_t *>(TB.mulpfw) : TB.primes) + ls;
            const uint32_t X = pc_uniform((uint32_t)Xb1[cb + j]);
            const double Xd = __longlong_as_double(
                (long long)pc_uniform64((uint64_t)__double_as_longlong(Xd1[cb + j])));
            uint32_t next = tid < n ? src[tid] : 0u;
            build_pre();
            int32_t wsum = 0;
            int64_t lsum = 0;
            uint32_t bad = 0;
            uint32_t *const slot = gbuf + wv * 64; // wheel number | (mu(m) > 0) << 31
            uint32_t held = 0;                     // filled slots (uniform)
            for (uint32_t base = wv * 64;; base += T) {
                const bool more = base < n; // (uniform)
                const uint32_t it = base + lane, v = next;
                next = it + T < n ? src[it + T] : 0u;
                uint32_t m = v;
                int32_t w = 1;
                bool have = it < n;
                if (cand) {
                    // squarefree (v != 0), lpf(m) > p_b
                    const bool keep = (uint32_t)max((int32_t)v, -(int32_t)v) > p;
                    const uint64_t bal = __ballot(keep);
                    const uint32_t at = held + (uint32_t)__builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                    const uint32_t e = (ls + it) | ((int32_t)v > 0 ? 0x80000000u : 0u);
                    n_cand += have ? 1u : 0u;
                    if (keep && at < 64)
                        slot[at] = e;
                    held += (uint32_t)__builtin_popcountll(bal);
                    if (held < 64 && more)
                        continue;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    have = lane < held;
                    const uint32_t f = have ? slot[lane] : 0u;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    if (keep && at >= 64)
                        slot[at - 64] = e;
                    held = held > 64 ? held - 64 : 0u;
                    m = pc_wheel_m(TB, f & 0x7FFFFFFFu);
                    w = (f >> 31) ? -1 : 1;
                }
                if (have) {
                    const uint32_t q = leaf_q(X, Xd, m, &bad);
                    lsum += (int64_t)(w * (int32_t)count_pre(q));
                    wsum += w;
                    nleaf++;
                }
                if (!more)
                    break;
            }
            leaf_check(bad);
            acc_local += lsum;
            const uint32_t ws = pc_wave_sum_u32((uint32_t)wsum);
            if (lane == 0 && ws != 0)
                atomicAdd(&c_w[j], (int32_t)ws);
            __syncthreads(); // every read of the column's state precedes its crossing
            PC_PH(3);
        };
        // Columns [j0, we), their light leaves gathered: each wave visits, in
        // order, the columns that have leaves (those in its region are answered
        // before the crossing) or a multiple in its region; after a group of 64
        // columns it adds its region's count at their columns (the count at the
        // group's start minus the removals of its earlier columns) to the
        // leaves of the regions above.
        auto window = [&](uint32_t j0, uint32_t we) {
            for (uint32_t j = j0, b = 0; j < we; j += 64, b += NWV) {
                load_group(j);
                const uint32_t ge = min(we, j + 64);
                const uint32_t s0 = bin_at(b + wv), s1 = bin_at(b + wv + 1), s2 = bin_at(b + NWV);
                const uint32_t e0 = s0 + lane < s1 ? gbuf[s0 + lane] : 0u;
                const uint32_t rc0 = rc;
                const uint32_t col = cg0 + lane;
                const bool inw = col < ge;
                const uint32_t xb = xbatch_from(j, ge); // columns from xb on: one xbatch step
                const bool sm = col < xb;
                const uint64_t own = s0 < s1 ? __ballot(sm && c_lc[sm ? col : cg0] != 0) : 0;
                const uint64_t crs = __ballot(sm && v_d < RSI);
                uint64_t todo = own | crs;
                const uint32_t v_piece = own ? find_pieces(s0, s1) : 0u;
                while (todo) {
                    const int32_t k = (int32_t)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    if ((own >> k) & 1)
                        answer((uint32_t)k, s0, s1, e0,
                               (uint32_t)__builtin_amdgcn_readlane((int)v_piece, k));
                    if ((crs >> k) & 1)
                        cross_k(k);
                }
                if (xb < ge)
                    xbatch(xb, ge, s0, s1);
                if (s1 < s2) {
                    const uint32_t rem = inw ? v_rem : 0u;
                    const uint32_t at = rc0 - (pc_wave_incl_scan_u32(rem) - rem);
                    int32_t t = 0;
                    for (uint32_t s = s1; s < s2; s += 64) {
                        const uint32_t e = s + lane < s2 ? gbuf[s + lane] : 0u;
                        const int32_t c = __shfl((int)at, (int)(e >> 22), 64);
                        t += e & 1 ? (e & 2 ? -c : c) : 0;
                    }
                    acc_local += t;
                }
            }
        };
        // Columns in order.  Each wave crosses its own region, so between the
        // workgroup-wide steps (gather, heavy column) the waves move through
        // the columns independently.
        uint32_t j = 0, jb_next = 0; // jb_next: the next leafy column, once known
        uint32_t lw_at = ~0u;        // c_leafy word cached for columns [64 lw_at, 64 lw_at + 64)
        uint64_t lw = 0;
        while (j < jend) {
            if ((j >> 6) != lw_at) {
                lw_at = j >> 6;
                lw = c_leafy[lw_at];
            }
            if ((lw >> (j & 63)) & 1) { // leaves, then the crossing
                const bool hv = (c_heavy[j >> 6] >> (j & 63)) & 1;
                if (hv) {
                    heavy_col(j);
                    cross_region(j);
                    j++;
                } else {
                    const uint32_t we = gather(j);
                    window(j, we);
                    j = we;
                }
                continue;
            }
            if (jb_next <= j) { // the next leafy column after j
                uint32_t wd = j >> 6;
                uint64_t msk = c_leafy[wd] & (~0ull << (j & 63));
                while (!msk && ++wd < (jend + 63) / 64)
                    msk = c_leafy[wd];
                jb_next = msk ? min(jend, wd * 64 + (uint32_t)__builtin_ctzll(msk)) : jend;
            }
            // a leafless run, each wave in its own region (large primes a
            // group of 64 at a time, xbatch)
            cross_run(j, jb_next);
            j = jb_next;
        }
        flush_removed();
        PC_PH(4);
        __syncthreads(); // c_new complete; every wave is past the last window
        // --- chunk results: cnt before each crossing, and w ---
        {
            const uint32_t v = tid >= jend ? 0u
                               : NEW16     ? (c_new[tid >> 1] >> ((tid & 1u) * 16u)) & 0xFFFFu
                                           : c_new[tid];
            uint32_t tot;
            const uint32_t ex = pc_block_excl_scan<T>(v, scr32, &tot);
            const uint32_t col = cb + tid;
            // columns at or past the cut hold no leaf here or below: 0 (if stored)
            if (tid < jall && col < r_len) {
                const bool cut = tid >= jend;
                const uint64_t idx = r_off + col;
                if (MODE != PC_MODE_LEAVES)
                    Q.cnt[idx] = cut ? 0u : total - ex;
                if (MODE == PC_MODE_TALLY)
                    Q.wgt[idx] = cut ? 0 : c_w[tid];
                if (MODE == PC_MODE_LEAVES && !cut && c_w[tid] != 0)
                    acc_carry += (pc_s128)c_w[tid] * (pc_s128)Q.carry[idx];
            }
            // every column before the cut must be stored: the row's bound holds
            if (tid < jend && col >= r_len)
                atomicOr(A.err, 8);
            total -= tot;
        }
        PC_PH(7);
        if (jend < jall) {
            // Device invariant: the unsieved count carried through every
            // crossing so far (each wave's own hits, summed per column) must
            // equal a fresh count of the bitmap.
            if (build_pre() != total && tid == 0)
                atomicOr(A.err, 32);
            recounted = true;
            // Every column from cb + jend on is past its last hard leaf: its
            // count is read by no leaf and it removes nothing a later leaf of
            // this segment counts, so its multiples are only cleared.  Its
            // stored counts are 0.
            if (MODE != PC_MODE_LEAVES)
                for (uint32_t col = cb + jall + tid; col < min(ncross, r_len); col += T) {
                    Q.cnt[r_off + col] = 0;
                    if (MODE == PC_MODE_TALLY)
                        Q.wgt[r_off + col] = 0;
                }
            if (col_hi == ncol) // (else nothing reads the segment any more)
                clear_columns(cb + jend, ncross);
            PC_PH(5);
            break;
        }
    }

    // --- final column: P2 lookups pi(x/p) = phi(x/p, bmax) + bmax - 1 ---
    pc_s128 extra_p2 = 0; // PC_MODE_LEAVES: carry * (lookups), kept by thread 0
    if (col_hi == ncol) {
        __syncthreads();
        const uint32_t rec = build_pre(); // (the carried total skips the cleared-only columns)
        if (!recounted && rec != total && tid == 0)
            atomicOr(A.err, 32); // the invariant above, for a segment with no cut
        total = rec;
        uint32_t k1 = 1, k2 = 0;
        {
            // x/p < hi <=> p > x/hi;  x/p >= lo <=> p <= x/lo  (above 2^64: every
            // segment but the first has lo >= 2^16, so both quotients are < 2^52)
            const uint64_t tA = Q.x_hi ? pc_div_wide(Q.x, Q.xd, hi) : pc_div(Q.x, hi, rhi);
            const uint64_t tB =
                !lo ? ~0ull : Q.x_hi ? pc_div_wide(Q.x, Q.xd, lo) : pc_div(Q.x, lo, rlo);
            const uint64_t pl = tA > Q.y ? tA : Q.y;
            const uint64_t ph = tB < Q.sqrtx ? tB : Q.sqrtx;
            if (pl < ph) {
                k1 = pc_pi_lookup(TB.pitab, pl) + 1;
                k2 = pc_pi_lookup(TB.pitab, ph);
            }
        }
        if (MODE != PC_MODE_COUNT) {
            const uint64_t x = Q.x;     // modulo 2^64 above 2^64
            const double xd = Q.xd;
            for (uint32_t k = k1 + tid; k <= k2; k += T) {
                uint32_t off; // x/p_k - lo
                const bool in = k < TB.k32
                                    ? pc_quot_in(x, xd, TB.primes[k], lo, SPAN, &off)
                                    : pc_quot_in64(x, xd, TB.primes_hi[k - TB.k32], lo, SPAN,
                                                   &off);
                if (!in) {
                    atomicOr(A.err, 4);
                    continue;
                }
                acc_p2 += count_pre(pc_w30_le(off));
            }
        }
        if (tid == 0) {
            const uint32_t np = k2 >= k1 ? k2 - k1 + 1 : 0;
            if (MODE != PC_MODE_LEAVES)
                Q.cntP[row] = total;
            if (MODE == PC_MODE_TALLY)
                Q.wP[row] = (int32_t)np;
            if (MODE == PC_MODE_LEAVES)
                extra_p2 = (pc_s128)np * (pc_s128)Q.carryP[row];
        }
    }
    if (MODE != PC_MODE_COUNT) {
        const pc_s128 h = pc_block_sum128<T>((pc_s128)acc_local + acc_carry, scr128);
        const pc_s128 q = pc_block_sum128<T>((pc_s128)acc_p2 + extra_p2, scr128);
        nleaf = pc_wave_sum(nleaf);
        if (lane == 0 && nleaf)
            atomicAdd(&Q.sums->n_hard, nleaf);
        if (A.trace) {
            uint32_t *tr = A.trace + (size_t)blockIdx.x * PC_TRACE_W;
            const uint32_t nc = pc_wave_sum_u32(n_cand);
            const uint32_t nl = pc_wave_sum_u32(n_leafy);
            const uint32_t ns = pc_wave_sum_u32(n_leafy_small);
            if (lane == 0) {
                atomicAdd(&tr[1], (uint32_t)nleaf);
                atomicAdd(&tr[2], nc);
                atomicAdd(&tr[3], nl);
                atomicAdd(&tr[4], ns);
            }
            __syncthreads();
            PC_PH(8);
            if (tid == 0) {
                tr[0] = (uint32_t)(__builtin_amdgcn_s_memrealtime() - t_start);
#if PC_PHASE_TRACE
                for (int k = 0; k < 9; k++)
                    tr[5 + k] = ph[k];
                tr[11] = ev[0]; // phase 6 is unused
                tr[14] = ev[1];
                tr[15] = ev[2];
#endif
            }
        }
        if (tid == 0) {
            pc_atomic_add128(&Q.sums->hard_local, h);
            pc_atomic_add128(&Q.sums->p2_local, q);
        }
    }
}
#undef PC_PH
#undef PC_EV

// ---------------------------------------------------------------------------
// Queries with c < 3 (y < 5, so x < 125 and z < 32): the same sums from the
// definitions by one thread, the integers 1 .. z as the bits of one word.
// ---------------------------------------------------------------------------
__global__ void k_sieve_tiny(pc_tables T, pc_query Q)
{
    if (threadIdx.x != 0 || blockIdx.x != 0)
        return;
    uint64_t left = 0;
    for (uint32_t n = 1; n <= (uint32_t)Q.z; n++) {
        bool ok = true;
        for (uint32_t i = 1; i <= Q.c; i++)
            ok = ok && n % T.primes[i] != 0;
        left |= (uint64_t)ok << n;
    }
    auto phi = [&](uint64_t u) { return (int64_t)__builtin_popcountll(left & ((2ull << u) - 1)); };
    int64_t hard = 0, p2 = 0;
    unsigned long long nhard = 0;
    for (uint32_t b = Q.c + 1; b <= Q.c + Q.nb; b++) {
        const uint64_t p = T.primes[b], h1 = Q.x / (p * p * p), h2 = Q.x / (p * Q.y1);
        for (uint64_t m = max(Q.y / p, p) + 1; m <= min(Q.y, max(h1, h2)); m++) {
            const int32_t v = T.mulpf[m];
            if ((uint64_t)(v < 0 ? -v : v) <= p) // mu(m) = 0 or lpf(m) <= p_b
                continue;
            const int64_t f = phi(Q.x / (p * m));
            hard += v > 0 ? -f : f;
            nhard++;
        }
        for (uint32_t n = (uint32_t)p; n <= (uint32_t)Q.z; n += (uint32_t)p)
            left &= ~(1ull << n);
    }
    for (uint32_t k = Q.a + 1; k <= Q.kx; k++)
        p2 += phi(Q.x / T.primes[k]);
    Q.sums->hard_local += hard;
    Q.sums->p2_local += p2;
    Q.sums->n_hard += nhard;
}

hipError_t pc_launch_sieve_tiny(const pc_tables &T, const pc_query &Q, hipStream_t s)
{
    if (Q.z > 62)
        return hipErrorInvalidValue;
    k_sieve_tiny<<<1, 64, 0, s>>>(T, Q);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Look-back scan over the segments of a window, independently per column:
// carry[s][col] = carry_in[col] + sum_{s' < s} cnt[s'][col], over the rows
// that store the column (a prefix of the window's rows: row lengths never
// grow).  Workgroups take tickets in order; ticket t is block t - blkoff[k]
// of chunk k: 256 columns by rows_per_chunk rows, or, the last block of a
// chunk, the P2 column (cntP, wP) of its rows.  A workgroup publishes
// its column sums and looks back through earlier chunks until one has
// published an inclusive prefix (decoupled look-back); a column stored in a
// chunk's first row is stored in every earlier chunk, so every look-back
// finds its words.
//
// PC_MODE_TALLY needs only sum w * carry, which splits over a chunk as
//   sum_r w_r (P + l_r) = P * sum_r w_r + sum_r w_r l_r,
// P = the carry at the chunk's first row (from the look-back), l_r = the
// counts of the chunk's rows above r: one pass over cnt and wgt before the
// look-back, each read once, SCAN_U rows of loads in flight per thread.
// PC_MODE_COUNT writes every carry out for the leaf pass (a second pass).
// ---------------------------------------------------------------------------
#define SCAN_T 256
#define SCAN_U 8
#define SCAN_RMAX 1024
#define LB_A (1ull << 62)
#define LB_P (2ull << 62)
#define LB_V ((1ull << 62) - 1)

// The ticket's share of the look-back: publish agg (the chunk's sum), return
// the sum of the earlier chunks, whose words are at index word(jc).
template <typename F>
__device__ __forceinline__ uint64_t scan_look_back(const pc_scan_args &A, uint64_t *st,
                                                   uint32_t rc, uint64_t agg, F word)
{
    if (rc == 0) {
        __hip_atomic_store(st, LB_P | agg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return 0;
    }
    __hip_atomic_store(st, LB_A | agg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t pre = 0;
    int64_t jc = (int64_t)rc - 1;
    uint32_t spins = 0;
    while (jc >= 0) {
        const uint64_t v = __hip_atomic_load(A.status + word((uint32_t)jc), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t f = v >> 62;
        if (f == 0) {
            if (++spins > (1u << 26)) { // never expected: earlier tickets always run
                atomicOr(A.err, 1);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        pre += v & LB_V;
        if (f == 2)
            break;
        jc--;
    }
    __hip_atomic_store(st, LB_P | ((pre + agg) & LB_V), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    return pre;
}

// The P2 column of chunk rc (rows [r0, r0 + nr)): each thread a run of rows.
template <int MODE>
__device__ __forceinline__ void scan_p2(const pc_scan_args &A, uint32_t tk, uint32_t rc,
                                        uint64_t r0, uint32_t nr, uint64_t *s_pre, pc_s128 *scr)
{
    uint64_t *const scr64 = reinterpret_cast<uint64_t *>(scr);
    const uint32_t per = (nr + SCAN_T - 1) / SCAN_T;
    const uint32_t i0 = min(nr, threadIdx.x * per), i1 = min(nr, i0 + per);
    uint64_t agg = 0;
    for (uint32_t i = i0; i < i1; i++)
        agg += A.cntP[r0 + i];
    uint64_t tot;
    uint64_t run = pc_block_excl_scan<SCAN_T>(agg, scr64, &tot);
    if (threadIdx.x == 0)
        *s_pre = scan_look_back(A, A.status + (uint64_t)tk * SCAN_T, rc, tot, [&](uint32_t jc) {
            return (uint64_t)(A.blkoff[jc + 1] - 1) * SCAN_T;
        });
    __syncthreads();
    run += A.carry_in[A.nb] + *s_pre; // the carry at the thread's first row
    pc_s128 acc = 0;
    for (uint32_t i = i0; i < i1; i++) {
        if (MODE == PC_MODE_TALLY)
            acc += (pc_s128)A.wP[r0 + i] * (pc_s128)run;
        else
            A.carryP[r0 + i] = run;
        run += A.cntP[r0 + i];
    }
    if (rc == A.nchunk - 1 && threadIdx.x == 0)
        A.carry_out[A.nb] = A.carry_in[A.nb] + *s_pre + tot;
    if (MODE == PC_MODE_TALLY) {
        acc = pc_block_sum128<SCAN_T>(acc, scr);
        if (threadIdx.x == 0)
            pc_atomic_add128(&A.sums->p2_dot, acc);
    }
}

template <int MODE> __global__ __launch_bounds__(SCAN_T) void k_scan(pc_scan_args A)
{
    __shared__ uint64_t s_pre;
    __shared__ uint32_t s_ticket, s_chunk;
    __shared__ uint64_t s_off[SCAN_RMAX + 1];
    __shared__ pc_s128 scr[SCAN_T / 64];
    if (threadIdx.x == 0) {
        const uint32_t t = atomicAdd(A.ticket, 1u);
        uint32_t lo = 0, hi = A.nchunk - 1; // the chunk k with blkoff[k] <= t < blkoff[k+1]
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (A.blkoff[mid] <= t)
                lo = mid;
            else
                hi = mid - 1;
        }
        s_ticket = t;
        s_chunk = lo;
    }
    __syncthreads();
    const uint32_t tk = s_ticket, rc = s_chunk;
    const uint32_t cb = tk - A.blkoff[rc];
    const uint64_t r0 = (uint64_t)rc * A.rows_per_chunk;
    const uint32_t nr = (uint32_t)min<uint64_t>(A.rows_per_chunk, A.nrows - r0);
    if (cb + 1 == A.blkoff[rc + 1] - A.blkoff[rc]) {
        scan_p2<MODE>(A, tk, rc, r0, nr, &s_pre, scr);
        return;
    }
    for (uint32_t i = threadIdx.x; i <= nr; i += SCAN_T)
        s_off[i] = A.row_off[r0 + i];
    __syncthreads();
    const uint32_t col = cb * SCAN_T + threadIdx.x;
    // rows of the chunk that store the column: a prefix [0, na)
    uint32_t na = 0;
    {
        uint32_t lo = 0, hi = nr; // the first row whose length is <= col
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_off[mid + 1] - s_off[mid] > col)
                lo = mid + 1;
            else
                hi = mid;
        }
        na = lo;
    }
    const bool act = na > 0;
    uint64_t agg = 0, pre = 0;
    int64_t wsum = 0;   // PC_MODE_TALLY: sum of w over the chunk
    pc_s128 wl = 0;     //                sum of w * (counts of the chunk above the row)
    if (act) {
        if (MODE == PC_MODE_TALLY) {
            uint32_t i = 0;
            for (; i + SCAN_U <= na; i += SCAN_U) {
                uint32_t c[SCAN_U];
                int32_t w[SCAN_U];
#pragma unroll
                for (uint32_t u = 0; u < SCAN_U; u++) {
                    c[u] = A.cnt[s_off[i + u] + col];
                    w[u] = A.wgt[s_off[i + u] + col];
                }
#pragma unroll
                for (uint32_t u = 0; u < SCAN_U; u++) {
                    if (w[u]) {
                        wsum += w[u];
                        wl += (pc_s128)((int64_t)w[u] * (int64_t)agg);
                    }
                    agg += c[u];
                }
            }
            for (; i < na; i++) {
                const int32_t w = A.wgt[s_off[i] + col];
                if (w) {
                    wsum += w;
                    wl += (pc_s128)((int64_t)w * (int64_t)agg);
                }
                agg += A.cnt[s_off[i] + col];
            }
        } else {
            for (uint32_t i = 0; i < na; i++)
                agg += A.cnt[s_off[i] + col];
        }
        // look-back words: one per (ticket, thread); chunk rc - 1 holds this
        // column in its block cb
        pre = scan_look_back(A, A.status + (uint64_t)tk * SCAN_T + threadIdx.x, rc, agg,
                             [&](uint32_t jc) {
                                 return ((uint64_t)A.blkoff[jc] + cb) * SCAN_T + threadIdx.x;
                             });
    }
    pc_s128 dh = 0;
    if (act) {
        const uint64_t P = A.carry_in[col] + pre; // carry at the chunk's first row
        if (MODE == PC_MODE_TALLY) {
            dh = (pc_s128)wsum * (pc_s128)P + wl;
        } else {
            uint64_t carry = P;
            for (uint32_t i = 0; i < na; i++) {
                A.carry_rows[s_off[i] + col] = carry;
                carry += A.cnt[s_off[i] + col];
            }
        }
        // a column stored through the window's last row continues in the next window
        if (rc == A.nchunk - 1 && na == nr)
            A.carry_out[col] = P + agg;
    }
    if (MODE == PC_MODE_TALLY) {
        dh = pc_block_sum128<SCAN_T>(dh, scr);
        if (threadIdx.x == 0)
            pc_atomic_add128(&A.sums->hard_dot, dh);
    }
}

hipError_t pc_launch_scan(const pc_scan_args &A, int mode, hipStream_t s)
{
    if (A.nrows == 0)
        return hipSuccess;
    if (A.rows_per_chunk == 0 || A.rows_per_chunk > SCAN_RMAX ||
        (uint64_t)A.nchunk * A.rows_per_chunk < A.nrows)
        return hipErrorInvalidValue;
    if (mode == PC_MODE_TALLY)
        k_scan<PC_MODE_TALLY><<<A.nticket, SCAN_T, 0, s>>>(A);
    else
        k_scan<PC_MODE_COUNT><<<A.nticket, SCAN_T, 0, s>>>(A);
    return hipGetLastError();
}

template <int LOG2_S, int T, int CH>
static hipError_t launch_modes(const pc_sieve_args &A, int mode, bool batch, hipStream_t s)
{
    const uint32_t g = A.ntiles;
    if (batch) {
        if (mode == PC_MODE_TALLY)
            k_sieve<LOG2_S, T, CH, PC_MODE_TALLY, true><<<g, T, 0, s>>>(A);
        else if (mode == PC_MODE_COUNT)
            k_sieve<LOG2_S, T, CH, PC_MODE_COUNT, true><<<g, T, 0, s>>>(A);
        else
            k_sieve<LOG2_S, T, CH, PC_MODE_LEAVES, true><<<g, T, 0, s>>>(A);
    } else {
        if (mode == PC_MODE_TALLY)
            k_sieve<LOG2_S, T, CH, PC_MODE_TALLY, false><<<g, T, 0, s>>>(A);
        else if (mode == PC_MODE_COUNT)
            k_sieve<LOG2_S, T, CH, PC_MODE_COUNT, false><<<g, T, 0, s>>>(A);
        else
            k_sieve<LOG2_S, T, CH, PC_MODE_LEAVES, false><<<g, T, 0, s>>>(A);
    }
    return hipGetLastError();
}

hipError_t pc_launch_sieve(const pc_sieve_args &A, uint32_t seg_log2, uint32_t wg, int mode,
                           hipStream_t s)
{
    const bool batch = (mode & 0x100) == 0;
    mode &= 0xFF;
    if (A.ntiles == 0)
        return hipSuccess;
    // one-wavefront segments for the leaf-dense low end of [1, z]
    if (seg_log2 == 15 && wg == 64)
        return launch_modes<15, 64, 64>(A, mode, batch, s);
    if (seg_log2 == 16 && wg == 64)
        return launch_modes<16, 64, 64>(A, mode, batch, s);
    if (seg_log2 == 18 && wg == 256)
        return launch_modes<18, 256, 256>(A, mode, batch, s);
    if (seg_log2 == 18 && wg == 512)
        return launch_modes<18, 512, 512>(A, mode, batch, s);
    if (seg_log2 == 19 && wg == 512)
        return launch_modes<19, 512, 256>(A, mode, batch, s);
    if (seg_log2 == 19 && wg == 1024)
        return launch_modes<19, 1024, 1024>(A, mode, batch, s);
    return hipErrorInvalidValue;
}
