// pc_internal.h -- structures shared between the host planner and the kernel
// launchers of the prime-counting library.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pc_device.h"

// One sieve tile: segment `seg` (absolute index), responsible for the
// per-segment columns [col_lo, col_hi).  Column j < nb stands for the sieving
// prime b = c + 1 + j; column nb is the state after every sieving prime is
// crossed (read by the P2 lookups).
struct pc_tile {
    uint32_t seg;
    uint32_t col_lo;
    uint32_t col_hi;
    uint32_t q;             // query (index into the launch's query array)
};

// Shared device tables (read-only during a query).
struct pc_tables {
    const uint32_t *primes; // primes[k] = p_k, 1-based (primes[1] = 2), p_k < 2^32
    const uint64_t *primes_hi; // p_k for k >= k32 (the primes above 2^32): primes_hi[k - k32]
    uint64_t k32;           // index of the first prime above 2^32 (UINT64_MAX: none tabulated)
    const uint64_t *recip;  // recip[k] = floor((2^64-1)/p_k) for k <= n_recip
    const double *rcpd;     // rcpd[k] = 1/p_k correctly rounded, k <= n_recip
    const uint2 *pitab;     // pi table, see pc_pi_lookup
    const int32_t *mulpf;   // mu(n)*lpf(n) for n <= ymax; INT32_MAX at n = 1; 0 if mu = 0
    const int32_t *mulpfw;  // the same of the k-th integer prime to 2 .. 13 (pc_wheel_m), in order
    const uint32_t *pattern; // pre-sieve bits for p_4..p_c (8 bits per 30 integers), period
                            // pattern_bits (+64 bits)
    const uint8_t *presieve; // the multiples of 17 .. 67 (pc_presieve_*)
    const uint32_t *phitab; // phi(r, c) for r < Q_c
    const uint32_t *wres;   // the residues r < Q_c prime to p_1..p_c, ascending (phi(Q_c, c) of them)
    uint32_t pattern_bits;  // 8 prod_{4 <= i <= c} p_i
    uint32_t Qc;            // prod_{1 <= i <= c} p_i
    uint32_t phiQ;          // phi(Q_c, c)
};

// The bitmaps of the integers prime to the primes 17 .. 67 (p_7 .. p_19), in six
// groups: byte i of group g stands for 30 i .. 30 i + 29 (pc_w30_*) and repeats
// after the product of the group's primes; each is followed by its first four
// bytes, so that a word is read at any byte of the period.
constexpr uint32_t PC_PS_FIRST = 7, PC_PS_LAST = 19, PC_PS_GROUPS = 6;
constexpr uint32_t pc_presieve_period(uint32_t g)
{
    return g == 0 ? 17 * 19 * 23 : g == 1 ? 29 * 31 : g == 2 ? 37 * 41 : g == 3 ? 43 * 47
                                 : g == 4 ? 53 * 59 : 61 * 67;
}
constexpr uint32_t pc_presieve_at(uint32_t g) // first byte of group g (PC_PS_GROUPS: the size)
{
    return g == 0 ? 0 : pc_presieve_at(g - 1) + pc_presieve_period(g - 1) + 4;
}

struct pc_sums;

// Per-query scalars.
struct pc_query {
    uint64_t x, y, z;       // x: its low 64 bits when x_hi != 0
    uint64_t x_hi;          // x = x_hi 2^64 + x, x <= 2^72
    double xd;              // x rounded to double
    uint64_t y1, recip_y1;  // y + 1 and its reciprocal
    uint64_t sqrtx;         // isqrt(x)
    uint64_t sqrty;         // isqrt(y): p_b^2 > y  <=>  p_b > sqrty
    uint64_t Qc, recip_Qc;
    uint32_t c, a, bmax, nb, ncol;
    uint32_t kx;            // pi(isqrt(x))
    const uint64_t *Xb;     // Xb[b] = floor(x / p_b) modulo 2^64, 1-based, b <= a and the sieving primes
    uint32_t *Xbh;          // its high word (above 2^64; null: every X_b < 2^64)
    uint64_t sieve_end;     // the sieve covers [0, sieve_end): segments * pc_seg_span
    uint64_t nseg;          // segments (rows of cnt and wgt when the query has one window)
    const ulonglong2 *Ub;   // Ub[b].x <= u of every hard leaf of b <= Ub[b].y, and Ub[b].y is
                            // also >= that bound for every later sieving prime (x > y: none)
    pc_sums *sums;          // device accumulators of this query
    // Sieve counts and leaf weights of the sieving columns j < nb, stored as a
    // staircase: row r (= seg - seg0) holds columns [0, row_off[r+1] -
    // row_off[r]) from row_off[r] on, a bound on the columns that still have
    // a hard leaf at or above the row's first integer (it never grows with r);
    // row_off null: every row holds all nb columns, row r from r nb on.
    const uint64_t *row_off;
    uint32_t *cnt;          // unsieved count before p_b is crossed
    int32_t *wgt;           // sum of -mu(m) over the leaves of the column in the row
    const uint64_t *carry;  // PC_MODE_LEAVES: exclusive carries, same layout
    uint32_t *cntP;         // per row: the count after the last crossing (P2 column)
    int32_t *wP;            // per row: the P2 terms landing in the row
    const uint64_t *carryP; // PC_MODE_LEAVES: exclusive carries of cntP
    // Easy leaves per b (pc_leaf_setup_band), taken in bands of PC_EZ_BAND
    // consecutive b, band g = the b from PC_EZ_BAND g on:
    //   primes (p_b^2 > y): e_rng[b] = {lo, hi}, the prime indices k of
    //     lo <= k < hi whose pi(X_b / p_k) counts twice (pc_easy_primes);
    //   candidates (p_b^2 <= y): e_rng[b] = {PC_CAND | m1, m2}, the leaves'
    //     m1 <= m <= m2 (pc_easy_cands);
    //   {0, 0}: none.
    // Unit j of a band is PC_EZ_UNIT prime indices from e_bk[g] + PC_EZ_UNIT j
    // on, or PC_EZ_TILE wheel numbers (pc_wheel_m) from e_bk[nband + g] +
    // PC_EZ_TILE j on, against every b of the band; e_boff[g] / e_boff[nband +
    // g]: exclusive prefix of the units, e_total[0] / e_total[1] their sums.
    // e_lim[g] = {the largest lo, the smallest hi} of the band's b (empty
    // unless every b of it has primes).  Xd[b] = X_b rounded to double.
    uint2 *e_rng;
    uint32_t *e_bk;
    uint64_t *e_boff;
    uint2 *e_lim;
    double *Xd;
    uint64_t *e_total;
    ulonglong2 *Ub_w;       // writable view of Ub (set-up kernels)
    uint64_t *Xb_w;         // writable view of Xb (set-up kernels)
};

// X_b of a query: its low word, high word and value in fp64 (above 2^64 the
// high word is nonzero for the primes p_b below x / 2^64).
struct pc_xv {
    uint64_t lo;
    uint32_t hi;
    double d;
};

__device__ __forceinline__ pc_xv pc_xb(const pc_query &Q, uint32_t b)
{
    pc_xv v;
    v.lo = Q.Xb[b];
    v.hi = Q.Xbh ? Q.Xbh[b] : 0u;
    v.d = Q.x_hi ? Q.Xd[b] : (double)v.lo;
    return v;
}

// floor(X / p) for a prime p > X's high word (X / p < 2^64), rp = pc_recip(p)
__device__ __forceinline__ uint64_t pc_xv_div(pc_xv X, uint32_t p, uint64_t rp)
{
    return X.hi ? pc_div_wide32(X.hi, X.lo, p, nullptr) : pc_div(X.lo, p, rp);
}

// floor(X / d) for d < 2^46 when the quotient is below 2^64, rd = pc_recip(d)
__device__ __forceinline__ uint64_t pc_xv_div64(pc_xv X, uint64_t d, uint64_t rd)
{
    return X.hi ? pc_div_wide(X.lo, X.d, d) : pc_div(X.lo, d, rd);
}

// floor(X / m) for m < 2^32 when the quotient is below 2^50
__device__ __forceinline__ uint64_t pc_xv_small_q(pc_xv X, uint32_t m)
{
    return X.hi ? pc_div_small_qd(X.lo, X.d, m) : pc_div_small_q(X.lo, m);
}

enum { PC_MODE_TALLY = 0, PC_MODE_COUNT = 1, PC_MODE_LEAVES = 2 };

// b per band of the easy leaves (one per lane of a wavefront; bands of a query:
// a / PC_EZ_BAND + 1), prime indices and wheel numbers per unit.
#define PC_EZ_BAND 64
#define PC_EZ_UNIT 256
#define PC_EZ_TILE 2048

// per-tile trace record: 0 ticks (100 MHz), 1 hard leaves, 2 candidates read,
// 3 leafy columns, 4 of them with p^3 < segment end, 5.. phase ticks
#define PC_TRACE_W 16

struct pc_sieve_args {
    pc_tables T;
    const pc_query *Qs;     // device array; tile.q indexes it
    const pc_tile *tiles;
    uint32_t ntiles;
    uint32_t pad;
    uint64_t seg0;          // first segment of the window: row = seg - seg0
    uint64_t lo_base;       // segment seg starts at lo_base + (seg - seg_base) * pc_seg_span
    uint64_t seg_base;
    int32_t *err;
    uint32_t *trace;        // optional, PC_TRACE_W words per tile (profiling aid)
};

// Launchers (each returns hipSuccess or the first HIP error).
hipError_t pc_launch_base_primes(uint32_t *base, uint32_t *nbase, hipStream_t s);
hipError_t pc_launch_pitab(uint64_t nentries, const uint32_t *base, uint32_t nbase,
                           uint32_t *bits, uint32_t *cnts, uint2 *pitab, uint32_t *primes,
                           uint64_t *primes_hi, uint32_t *scan_tmp, hipStream_t s);
hipError_t pc_launch_recip(const uint32_t *primes, uint64_t *recip, double *rcpd, uint32_t n,
                           hipStream_t s);
hipError_t pc_launch_mulpf(const uint32_t *primes, uint32_t nsmall, uint64_t ymax,
                           int32_t *mulpf, hipStream_t s);
hipError_t pc_launch_mulpfw(const pc_tables &T, uint64_t n, int32_t *mulpfw, hipStream_t s);
hipError_t pc_launch_count_nonzero(const int32_t *a, uint64_t n, unsigned long long *out,
                                   hipStream_t s);
hipError_t pc_launch_presieve(uint8_t *out, hipStream_t s);
hipError_t pc_launch_wheel(uint32_t c, const uint32_t *primes, uint32_t *pattern,
                           uint32_t pattern_words, uint32_t *phitab, uint32_t *wres,
                           hipStream_t s);
hipError_t pc_launch_lookup(const uint2 *pitab, const uint64_t *in, uint32_t n, uint64_t *out,
                            hipStream_t s);

// Leaves outside the sieve: S1, trivial and easy special leaves, into the
// query's sums.  The set-up (X_b, Ub, the trivial leaves, the easy leaves'
// ranges and bands) and the easy kernels use the arrays named in pc_query.
hipError_t pc_launch_s1(const pc_tables &T, const pc_query &Q, uint32_t nblocks, hipStream_t s);
hipError_t pc_launch_leaf_setup(const pc_tables &T, const pc_query &Q, hipStream_t s);
// S1 and the easy leaves in one launch: 2 neasy + ns1 workgroups
hipError_t pc_launch_leaves(const pc_tables &T, const pc_query &Q, uint32_t neasy, uint32_t ns1,
                            hipStream_t s);
hipError_t pc_launch_easy_cands(const pc_tables &T, const pc_query &Q, uint32_t nblocks,
                                hipStream_t s);
hipError_t pc_launch_easy_primes(const pc_tables &T, const pc_query &Q, uint32_t nblocks,
                                 hipStream_t s);
hipError_t pc_launch_fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t s);

// Up to three word ranges copied from host memory that the device reads (pinned)
// and four cleared, in one launch.
struct pc_prep_args {
    const uint64_t *src[3];
    uint64_t *dst[3];
    uint64_t n[3];
    uint64_t *zero[4];
    uint64_t nz[4];
};
hipError_t pc_launch_prep(const pc_prep_args &A, hipStream_t s);

// The tile list of a sieve launch (pc_plan.hip), written to tiles[ntiles]:
// the planned rows of every query (its first ones, the leaf-dense low end),
// each whole or cut into column ranges, the rest rows whole, and empty tiles.
// One query (nq = 1): segments from seg_first on, np planned and nrest more;
// several: query order[k] has the planned rows pfx_plan[k] .. pfx_plan[k+1] - 1
// and the rest rows pfx_rest[k] .. pfx_rest[k+1] - 1, its segments from 0 on.
struct pc_plan_args {
    pc_tables T;
    const pc_query *Qs;
    const uint32_t *order, *pfx_plan, *pfx_rest;
    uint64_t seg_first, lo_base, seg_base; // as pc_sieve_args
    uint64_t tile_work; // at most this work a tile; 0: by the launch's work alone, ~0: no cuts
    uint64_t *work;     // np: estimated work
    uint2 *cut;         // np: tiles, the first one's index
    uint32_t *nplanned; // tiles of the planned rows
    uint32_t *tile_count; // += the tiles that are not empty
    pc_tile *tiles;
    uint32_t nq, np, nrest;
    uint32_t extra;     // the cuts add at most this many tiles
    uint32_t ntiles;    // >= np + nrest + extra
    uint32_t seg_log2;
};
hipError_t pc_launch_plan(const pc_plan_args &A, hipStream_t s);

// Sieve and carry scan.
hipError_t pc_launch_sieve(const pc_sieve_args &A, uint32_t seg_log2, uint32_t wg, int mode,
                           hipStream_t s);
// The hard leaves and P2 lookups of a query with c < 3 (y < 5, z < 32), into
// the query's sums.
hipError_t pc_launch_sieve_tiny(const pc_tables &T, const pc_query &Q, hipStream_t s);
// The carries of one window: per sieving column an exclusive scan of the
// staircase rows (decoupled look-back over chunks of rows), and the same for
// the P2 column (cntP).  Workgroup tickets run chunk by chunk; chunk k has
// blkoff[k+1] - blkoff[k] of them: a block of 256 columns each (those below the
// chunk's first row length) and one for the P2 column.
struct pc_scan_args {
    const uint32_t *cnt;
    const int32_t *wgt;
    const uint64_t *row_off;  // nrows + 1 (staircase, as pc_query)
    const uint32_t *blkoff;   // nchunk + 1: first ticket of each chunk
    uint64_t *carry_rows;     // PC_MODE_COUNT: exclusive carries, staircase layout
    const uint32_t *cntP;
    const int32_t *wP;
    uint64_t *carryP;         // PC_MODE_COUNT: exclusive carries of cntP
    const uint64_t *carry_in; // per column (nb + 1, the last one P2), from earlier windows
    uint64_t *carry_out;      // per column, for the next window
    uint64_t *status;         // [blkoff[nchunk] * 256] look-back words, zeroed
    uint32_t *ticket;         // zeroed
    pc_sums *sums;            // hard_dot, p2_dot
    int32_t *err;
    uint64_t nrows;
    uint32_t nb;
    uint32_t rows_per_chunk;  // at most 1024
    uint32_t nchunk;          // ceil(nrows / rows_per_chunk)
    uint32_t nticket;         // blkoff[nchunk]
};
hipError_t pc_launch_scan(const pc_scan_args &A, int mode, hipStream_t s);

// The seeds of a window that starts at m (Section 4): out[j] = phi(m, c + j)
// for 0 <= j <= nb, from phi(m, c) by eq. (4.1), each term closed (one left,
// Legendre from the pi table) or expanded depth first.  T's wheel is of size
// c; T's primes and reciprocals cover p_{c+nb}; the pi table covers
// m^(2/3) (pi_limit, else err |= 16); m <= 2^48.  nrec >= the columns j with
// p_{c+j}^3 <= m (one workgroup each); term: nb + 1 words of scratch.
hipError_t pc_launch_seed(const pc_tables &T, uint32_t c, uint64_t m, uint32_t nb,
                          uint32_t nrec, uint64_t pi_limit, int64_t *term, uint64_t *out,
                          int32_t *err, hipStream_t s);

// Final combination of the partial sums into pi(x) and its parts.
struct pc_sums {
    pc_s128 s1, s2t, s2e, hard_local, hard_dot, p2_local, p2_dot;
    unsigned long long n_s1, n_easy, n_hard, crossings, n_trivial;
    unsigned long long n_easy_terms; // candidates, single primes and group values of the easy leaves
};
struct pc_final {
    pc_s128 s1, s2t, s2e, s2h, p2, phi;
    uint64_t pi, pi_hi;     // pi(x) = pi_hi 2^64 + pi
    uint64_t ok;            // 1: pi in [0, 2^64); 2: pi in [2^64, 2^128); 0: negative
    uint64_t pad;
};
// Batches: the queries' set-up (X_b, S1, per-b leaf set-up, easy offsets),
// their easy leaves, and their carries and combination, each over all queries
// of the batch.  bq / bf: the query of each block, the first block of each
// query (bf[nq] = blocks).
hipError_t pc_launch_batch_setup(const pc_tables &T, const pc_query *Qs, const uint32_t *bq_xb,
                                 const uint32_t *bf_xb, uint32_t nb_xb, const uint32_t *bq_s1,
                                 const uint32_t *bf_s1, uint32_t nb_s1, uint32_t nq,
                                 hipStream_t s);
hipError_t pc_launch_batch_easy(const pc_tables &T, const pc_query *Qs, const uint32_t *bq,
                                const uint32_t *bf, uint32_t nblocks, hipStream_t s);
hipError_t pc_launch_batch_finish(const pc_query *Qs, const uint32_t *bq, const uint32_t *bf,
                                  uint32_t nblocks, uint32_t nq, pc_final *out, hipStream_t s);
// The caller-memory batch path: a round's results, and results known on the
// host ((position, value) pairs), written into the caller's output array.
hipError_t pc_launch_batch_out(const pc_final *fin, const uint64_t *pos, uint32_t nq,
                               const int32_t *err, uint64_t *out, hipStream_t s);
hipError_t pc_launch_scatter_u64(const ulonglong2 *kv, uint64_t n, uint64_t *out, hipStream_t s);

// What one query brings back to the host, written by the combination into
// pinned memory (no copy).
struct pc_back {
    pc_final fin;
    pc_sums sums;
    int32_t err[4]; // the error flag, the sieve's tiles
};
hipError_t pc_launch_combine(const pc_sums *sums, const pc_query &Q, uint64_t kp2,
                             const int32_t *err, pc_back *out, hipStream_t s);
