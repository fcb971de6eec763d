// pc_leafwork.h -- the per-item work of the parts of phi(x, a) = S1 + S2 that
// need no sieve, shared by the one-query kernels (pc_leaves.hip) and the
// batched kernels (pc_batch.hip):
//   S1  ordinary leaves  sum_{n <= y, mu(n) != 0, lpf(n) > p_c} mu(n) phi(x/n, c),
//       phi(u, c) from the wheel (Section 4: phi(m, c) in O(1));
//   S2t trivial special leaves (u = x/(m p_b) < p_b, phi = 1; m is then prime);
//   S2e easy special leaves (p_b <= u < p_b^2, u <= y), Legendre's formula
//       phi(u, b-1) = pi(u) - b + 2 (Section 4), independent of each other
//       (Section 3);
// and the final combination pi(x) = phi(x, a) + a - 1 - P2.
#pragma once

#include "pc_block.h"
#include "pc_internal.h"
#include "pc_leafrange.h"

// X_b = floor(x / p_b), 1 <= b <= a + 1 (X_0 = x): its low word, its high
// word (above 2^64, when Xbh is not null) and its value in fp64.
__device__ __forceinline__ pc_xv pc_xb_item(const pc_tables &T, const pc_query &Q, uint32_t b)
{
    uint64_t lo, hi = 0;
    if (b == 0) {
        lo = Q.x;
        hi = Q.x_hi;
    } else if (!Q.x_hi) {
        lo = pc_div(Q.x, T.primes[b], T.recip[b]);
    } else {
        lo = pc_div_u128_32(Q.x_hi, Q.x, T.primes[b], &hi, nullptr);
    }
    pc_xv X;
    X.lo = lo;
    X.hi = (uint32_t)hi;
    X.d = hi ? (double)(((pc_u128)hi << 64) | lo) : (double)lo;
    Q.Xb_w[b] = lo;
    if (Q.Xbh)
        Q.Xbh[b] = (uint32_t)hi;
    Q.Xd[b] = X.d;
    return X;
}

// The S1 term mu(n) phi(x/n, c) of a squarefree n <= y with lpf(n) > p_c; v =
// mu(n) lpf(n).
__device__ __forceinline__ pc_s128 pc_s1_term(const pc_tables &T, const pc_query &Q, uint64_t n,
                                              int32_t v)
{
    pc_s128 phi;
    if (!Q.x_hi) {
        const uint64_t u = pc_div_any(Q.x, (uint32_t)n);
        const uint64_t qq = pc_div(u, Q.Qc, Q.recip_Qc);
        phi = (pc_s128)(qq * T.phiQ + T.phitab[u - qq * Q.Qc]);
    } else { // above 2^64: u = x / n in 128 bits, u = qq Q_c + r with qq < 2^64
        uint64_t uh;
        const uint64_t ul = pc_div_u128_32(Q.x_hi, Q.x, (uint32_t)n, &uh, nullptr);
        uint32_t r;
        const uint64_t qq = pc_div_wide32(uh, ul, (uint32_t)Q.Qc, &r); // uh < Q_c: x <= 2^72
        phi = (pc_s128)qq * T.phiQ + T.phitab[r];
    }
    return v > 0 ? phi : -phi;
}

// S1 over the items i0, i0 + stride, ...: adds to *acc, returns the terms.
// With the whole wheel the n are the integers prime to p_1..p_6 (every one
// squarefree counts), a fifth of all; a smaller wheel belongs to y < 13.
__device__ __forceinline__ unsigned long long pc_s1_items(const pc_tables &T, const pc_query &Q,
                                                          uint64_t i0, uint64_t stride,
                                                          pc_s128 *acc)
{
    unsigned long long terms = 0;
    if (Q.c == 6) {
        const uint64_t n = pc_wheel_count(T, Q, Q.y);
        for (uint64_t k = i0; k < n; k += stride) {
            const int32_t v = T.mulpfw[k];
            if (v != 0) {
                *acc += pc_s1_term(T, Q, pc_wheel_m(T, (uint32_t)k), v);
                terms++;
            }
        }
    } else {
        const uint32_t pcc = T.primes[Q.c];
        for (uint64_t n = 1 + i0; n <= Q.y; n += stride) {
            const int32_t v = T.mulpf[n];
            if (v != 0 && (uint32_t)(v < 0 ? -v : v) > pcc) {
                *acc += pc_s1_term(T, Q, n, v);
                terms++;
            }
        }
    }
    return terms;
}

// pi(floor(X / p)), X in fp64 and its low word, rp = 1 / p, quotient < 2^31.
__device__ __forceinline__ uint32_t pc_pi_quot_exact(const pc_tables &T, uint64_t X, double Xd,
                                                     uint32_t p, double rp)
{
    return pc_pi_lookup32(T.pitab, pc_quot31r(X, Xd, p, rp));
}

// The same less one, without a remainder: one fma forms the quotient less one
// in fixed point with 20 fractional bits in the low bits of a double (2^-20 is
// its last place, as 1.5 2^32 < the sum < 2^33), raised by 4 units.  X rp is
// off by less than 3 units (quotient < 2^31, X and rp off by 2^-53, 1 / p from
// pc_rcp_f64 by 2^-51), so the integer part is right unless the fraction came
// out below 8 units: *amb collects the least fraction, and the caller repeats
// the exact way where some lane's is below PC_AMB (one step in a few thousand).
// The table's entry and the bits counted in it come from shifts of the same
// double.  About 10 instructions, none of them a 32-bit multiply, where the
// remainder test takes 19.  on: lanes that hold a term (the others read the
// first entry).
#define PC_AMB 8u
__device__ __forceinline__ uint32_t pc_pi_quot_less1(const uint2 *pitab, double Xd, double rp,
                                                     bool on, uint32_t *amb)
{
    constexpr double kMagic = 6442450944.0 - 1.0 + 4.0 / 1048576.0;
    const uint64_t v = (uint64_t)__double_as_longlong(__builtin_fma(Xd, rp, kMagic));
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    const uint32_t off = __builtin_amdgcn_alignbit(hi, lo, 23) & (on ? 0x0FFFFFF8u : 0u);
    const uint2 e = *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(pitab) + off);
    const uint32_t i = __builtin_amdgcn_alignbit(hi, lo, 21); // (quotient - 1) / 2, modulo 32
    *amb = min(*amb, on ? lo & 0xFFFFFu : PC_AMB);
    return e.y + (uint32_t)__builtin_popcount(e.x << (~i & 31u));
}

// Per-b set-up of the special leaves outside the sieve, c < b < a:
//   trivial leaves: primes m with max(p_b, x/p_b^2) < m <= y  (counted);
//   easy range:     e1 = max(y/p_b, H_b, p_b) + 1 <= m <= e2 = min(y, x/p_b^2),
//                   H_b = max(x/p_b^3, x/(p_b (y+1))).
// For a sieving prime it also records the u range of its hard leaves (Ub) and
// the odd multiples below the sieve end.
//
// p_b^2 <= y: the m of the range are tested one by one (pc_easy_cands).
// p_b^2 > y: they are prime.  With s = isqrt(X_b), X = X_b:
//   singles, primes m <= s: phi(u, b-1) = pi(u) - b + 2, u = X / m, so their
//     part is the sum of pi(X / p_k) over k1 <= k < k1 + ns less ns (b - 2);
//   groups, primes m > s, taken by K = pi(X / m), klo <= K < klo + nk: with
//     C(v) = min(max(v, s), e2) and V_K = pi(C(X / p_K)), the primes with
//     pi(u) = K number V_K - V_{K+1} (also when there are none), so their part
//     sum_K (V_K - V_{K+1}) (K - b + 2) telescopes to
//       sum_{klo <= K <= klo + nk} V_K + V_klo (klo - b + 1)
//         - V_{klo + nk} (klo + nk + 2 - b).
//     V_klo = pi(e2) and V_{klo + nk} = pi(s); the K between need no C.
// So both parts sum pi(X / p_k), the singles over [k1, k1 + ns), the groups
// over [klo + 1, klo + nk), and these ranges hardly differ: both end near
// pi(s), and e1 - 1 = max(p_b, X / (y + 1)) and X / e2 = max(p_b, X / y) differ
// by at most one, so each end differs by a prime or two.  The common range is
// taken once and counted twice (pc_easy_primes); the ends are added here.
//
// The calling workgroup (NT threads; every thread calls) takes the b of block
// index b0 / NT; its wavefronts are bands.  Added up over the calls: the
// trivial leaves, the crossings, and the constant parts of S2e.
struct pc_setup_sums {
    uint64_t triv = 0, cross = 0, terms = 0;
    int64_t leaves = 0;
    pc_s128 cst = 0;
};

__device__ __forceinline__ void pc_leaf_setup_band(const pc_tables &T, const pc_query &Q,
                                                   uint32_t b, pc_setup_sums *S)
{
    // y + 1 >= isqrt z: a sieving prime past p_a is p_{a+1} = y + 1 (z >= (y + 1)^2,
    // so x is just below (y + 1)^3; x = 294, y = 6).  It has no leaf, but the
    // sieve forms its range, so its X_b is set too.
    pc_xv X{};
    if (b <= Q.a || b <= Q.c + Q.nb)
        X = pc_xb_item(T, Q, b);
    if (b > Q.c && b <= Q.c + Q.nb) { // a sieving prime
        const uint64_t p = T.primes[b], rp = T.recip[b];
        // odd multiples k p_b, k odd, below the sieve end
        S->cross += (pc_div(Q.sieve_end - 1, p, rp) + 1) / 2;
        // u range of the hard leaves of b: y/p < m <= y, m > p, m <= max(x/p^3, x/(p(y+1)))
        uint64_t m1 = pc_div(Q.y, p, rp) + 1;
        if (m1 < p + 1)
            m1 = p + 1;
        const uint64_t h1 = pc_div(pc_xv_div(X, (uint32_t)p, rp), p, rp);
        const uint64_t h2 = pc_xv_div64(X, Q.y1, Q.recip_y1);
        uint64_t m2 = h1 > h2 ? h1 : h2;
        if (m2 > Q.y)
            m2 = Q.y;
        ulonglong2 ub;
        ub.x = 1;
        ub.y = 0;
        if (m1 <= m2) {
            ub.x = pc_xv_small_q(X, (uint32_t)m2);
            ub.y = pc_xv_small_q(X, (uint32_t)m1);
        }
        Q.Ub_w[b] = ub;
    }
    uint32_t lo = 0, hi = 0;                 // e_rng of a prime b
    uint32_t w0 = UINT32_MAX, w1 = 0;        // wheel numbers of a candidate b
    uint2 rng = make_uint2(0, 0);
    const bool in = b > Q.c && b < Q.a;
    if (in) {
        const uint64_t p = T.primes[b], rp = T.recip[b];
        const uint64_t tp = pc_xv_div(X, (uint32_t)p, rp); // floor(x / p^2): u >= p <=> m <= tp
        uint64_t m1 = pc_div(Q.y, p, rp) + 1;
        if (m1 < p + 1)
            m1 = p + 1;
        const uint64_t h1 = pc_div(tp, p, rp);
        const uint64_t h2 = pc_xv_div64(X, Q.y1, Q.recip_y1);
        const uint64_t H = h1 > h2 ? h1 : h2;
        const uint64_t e1 = H + 1 > m1 ? H + 1 : m1;
        const uint64_t e2 = tp < Q.y ? tp : Q.y;
        if (p > Q.sqrty) {
            if (e1 <= e2) {
                uint64_t s = X.hi ? pc_isqrt_wide(X.hi, X.lo) : pc_isqrt(X.lo);
                if (s < e1 - 1)
                    s = e1 - 1;
                if (s > e2)
                    s = e2;
                const uint32_t k1 = pc_pi_lookup(T.pitab, e1 - 1) + 1;
                const uint32_t ps = pc_pi_lookup(T.pitab, s);
                const uint32_t s1 = ps + 1; // singles [k1, s1)
                uint32_t g0 = 0, g1 = 0;    // groups between the ends [g0, g1)
                S->cst -= (pc_s128)(s1 - k1) * ((int64_t)b - 2);
                S->leaves += s1 - k1;
                S->terms += s1 - k1;
                if (s < e2) { // K = pi(u) for u in [X / e2, X / (s + 1)]
                    const uint32_t klo =
                        pc_pi_lookup(T.pitab, pc_xv_small_q(X, (uint32_t)e2));
                    const uint32_t kend =
                        pc_pi_lookup(T.pitab, pc_xv_small_q(X, (uint32_t)(s + 1))) + 1;
                    const int64_t v0 = pc_pi_lookup(T.pitab, e2), v1 = ps;
                    S->cst += v0 + v1 + (pc_s128)v0 * ((int64_t)klo - b + 1) -
                              (pc_s128)v1 * ((int64_t)kend + 2 - b);
                    S->leaves += v0 - v1;
                    S->terms += kend - klo + 1;
                    g0 = klo + 1;
                    g1 = kend;
                }
                lo = max(k1, g0);
                hi = min(s1, g1);
                if (lo >= hi)
                    lo = hi = s1; // nothing in common
                auto add = [&](uint32_t ka, uint32_t kb) {
                    for (uint32_t k = ka; k < kb; k++)
                        S->cst += pc_pi_quot_exact(T, X.lo, X.d, T.primes[k], T.rcpd[k]);
                };
                add(k1, min(lo, s1)); // the singles and the groups outside [lo, hi)
                add(max(hi, k1), s1);
                add(g0, min(lo, g1));
                add(max(hi, g0), g1);
                if (lo < hi)
                    rng = make_uint2(lo, hi);
                else
                    lo = hi = 0;
            }
            // trivial: m prime, m > max(m1 - 1, tp), m <= y
            const uint64_t t0 = tp > m1 - 1 ? tp : m1 - 1;
            if (t0 < Q.y)
                S->triv += Q.a - pc_pi_lookup(T.pitab, t0);
        } else if (e1 <= e2) {
            // every m with lpf(m) > p_b > p_c is prime to p_1..p_c: only
            // those are items, by their wheel numbers (pc_wheel_m)
            w0 = (uint32_t)pc_wheel_count(T, Q, e1 - 1);
            w1 = (uint32_t)pc_wheel_count(T, Q, e2);
            S->terms += w1 - w0;
            if (w0 < w1)
                rng = make_uint2((uint32_t)e1 | PC_CAND, (uint32_t)e2);
            else
                w0 = UINT32_MAX;
        }
    }
    if (b <= Q.a)
        Q.e_rng[b] = rng;
    // the band: this wavefront's b
    const bool some = lo < hi;
    uint32_t p_lo = some ? lo : UINT32_MAX, p_hi = some ? hi : 0;
    uint32_t l_lo = !in ? 0 : some ? lo : UINT32_MAX, l_hi = !in ? UINT32_MAX : some ? hi : 0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        p_lo = min(p_lo, (uint32_t)__shfl_xor((int)p_lo, d, 64));
        p_hi = max(p_hi, (uint32_t)__shfl_xor((int)p_hi, d, 64));
        l_lo = max(l_lo, (uint32_t)__shfl_xor((int)l_lo, d, 64));
        l_hi = min(l_hi, (uint32_t)__shfl_xor((int)l_hi, d, 64));
        w0 = min(w0, (uint32_t)__shfl_xor((int)w0, d, 64));
        w1 = max(w1, (uint32_t)__shfl_xor((int)w1, d, 64));
    }
    const uint32_t nband = Q.a / PC_EZ_BAND + 1, g = b / PC_EZ_BAND;
    if (pc_lane() == 0 && g < nband) {
        Q.e_bk[g] = p_lo;
        Q.e_boff[g] = p_hi > p_lo ? (p_hi - p_lo + PC_EZ_UNIT - 1) / PC_EZ_UNIT : 0;
        Q.e_bk[nband + g] = w0;
        Q.e_boff[nband + g] = w1 > w0 ? (w1 - w0 + PC_EZ_TILE - 1) / PC_EZ_TILE : 0;
        Q.e_lim[g] = make_uint2(l_lo, l_hi);
    }
}

// S, summed over the workgroup, into the query's sums.
template <int NT>
__device__ __forceinline__ void pc_setup_flush(const pc_query &Q, const pc_setup_sums &S,
                                               pc_s128 *scr)
{
    uint64_t *const scr64 = reinterpret_cast<uint64_t *>(scr);
    const uint64_t tr = pc_block_sum<NT>(S.triv, scr64);
    const uint64_t cr = pc_block_sum<NT>(S.cross, scr64);
    const uint64_t te = pc_block_sum<NT>(S.terms, scr64);
    const uint64_t le = pc_block_sum<NT>((uint64_t)S.leaves, scr64);
    const pc_s128 cst = pc_block_sum128<NT>(S.cst, scr);
    if (threadIdx.x == 0) {
        pc_atomic_add128(&Q.sums->s2t, (pc_s128)tr);
        pc_atomic_add128(&Q.sums->s2e, cst);
        atomicAdd(&Q.sums->n_trivial, (unsigned long long)tr);
        atomicAdd(&Q.sums->crossings, (unsigned long long)cr);
        atomicAdd(&Q.sums->n_easy, (unsigned long long)le);
        atomicAdd(&Q.sums->n_easy_terms, (unsigned long long)te);
    }
}

// After the per-b set-up: Ub[b].y becomes the largest u of a hard leaf of any
// sieving prime p_b' with b' >= b, so that in a segment [lo, hi) the columns
// whose Ub.y < lo form a suffix: no prime from there on has a hard leaf at or
// above lo, and the sieve needs neither their counts nor their order (they
// are only cleared).  The calling workgroup (NT threads) does one query.
template <int NT> __device__ __forceinline__ void pc_ub_suffix(const pc_query &Q, uint64_t *sh)
{
    const uint32_t b0 = Q.c + 1, n = Q.nb;
    const uint32_t per = (n + NT - 1) / NT;
    const uint32_t lo = min(n, threadIdx.x * per), hi = min(n, lo + per);
    uint64_t m = 0;
    for (uint32_t i = lo; i < hi; i++)
        m = max(m, Q.Ub_w[b0 + i].y);
    sh[threadIdx.x] = m;
    __syncthreads();
    for (uint32_t d = 1; d < NT; d <<= 1) { // suffix maximum over the threads' pieces
        uint64_t v = sh[threadIdx.x];
        if (threadIdx.x + d < NT)
            v = max(v, sh[threadIdx.x + d]);
        __syncthreads();
        sh[threadIdx.x] = v;
        __syncthreads();
    }
    uint64_t run = threadIdx.x + 1 < NT ? sh[threadIdx.x + 1] : 0;
    for (uint32_t i = hi; i > lo; i--) {
        run = max(run, Q.Ub_w[b0 + i - 1].y);
        Q.Ub_w[b0 + i - 1].y = run;
    }
}

// Exclusive prefix of the n units of a kind over the bands, in place, and
// their sum into *total, by the calling workgroup.
template <int NT>
__device__ __forceinline__ void pc_band_scan(uint64_t *off, uint32_t n, uint64_t *total,
                                             uint64_t *scr)
{
    uint64_t run = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += NT) {
        const uint32_t i = i0 + threadIdx.x;
        const uint64_t v = i < n ? off[i] : 0;
        uint64_t tot;
        const uint64_t ex = pc_block_excl_scan<NT>(v, scr, &tot);
        if (i < n)
            off[i] = run + ex;
        run += tot;
    }
    if (threadIdx.x == 0)
        *total = run;
}

// the last band g with off[g] <= u (uniform)
__device__ __forceinline__ uint32_t pc_band_of(const uint64_t *off, uint32_t nband, uint64_t u)
{
    uint32_t lo = 0, hi = nband - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= u)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The prime easy leaves (p_b^2 > y): *acc += 2 pi(X_b / p_k) over the band's b
// and lo_b <= k < hi_b, in units of PC_EZ_UNIT prime indices, one per thread
// (NT = PC_EZ_UNIT), against the b of a band.  The calling workgroup takes the
// contiguous units [U lb / nlb, U (lb + 1) / nlb).  A thread loads p_k and
// 1/p_k once per unit; X_b and the ranges are uniform (scalar loads).  Where
// the unit lies in every b's range (99% of them at x = 10^18) no lane tests
// its own, and four table reads are in flight.
//
// Integer issue bounds it, and the table reads (L2-resident, u <= y) close
// behind: one pi(10^18) takes 4.0 ms (4.3 beside the candidates; 12.2 with singles and groups summed
// apart and a remainder test per quotient).
template <int NT>
__device__ __forceinline__ void pc_easy_primes(const pc_tables &T, const pc_query &Q, uint64_t lb,
                                               uint64_t nlb, int64_t *acc)
{
    static_assert(NT == PC_EZ_UNIT, "one thread per prime index of a unit");
    const uint32_t nband = Q.a / PC_EZ_BAND + 1;
    const uint64_t *const boff = Q.e_boff;
    const uint64_t U = Q.e_total[0];
    const uint64_t u0 = U * lb / nlb, u1 = U * (lb + 1) / nlb;
    if (u0 >= u1)
        return;
    uint32_t g = pc_band_of(boff, nband, u0);
    uint64_t gend = g + 1 < nband ? boff[g + 1] : U;
    uint64_t a = 0;
    const uint32_t kcap = Q.a + 1; // p_k and 1/p_k exist for k <= a + 1
    for (uint64_t u = u0; u < u1; u++) {
        while (u >= gend) {
            g++;
            gend = g + 1 < nband ? boff[g + 1] : U;
        }
        const uint32_t k0 = Q.e_bk[g] + (uint32_t)(u - boff[g]) * PC_EZ_UNIT;
        const uint32_t k = k0 + threadIdx.x, kk = min(k, kcap);
        const uint32_t m = T.primes[kk];
        const double rm = T.rcpd[kk];
        const uint32_t b0 = max(g * PC_EZ_BAND, Q.c + 1), b1 = min(g * PC_EZ_BAND + PC_EZ_BAND, Q.a);
        const uint2 lim = Q.e_lim[g];
        // unsigned sums of 16 values of pi, each at most pi(2^31) < 2^27
        uint32_t b = b0;
        if (lim.x <= k0 && k0 + PC_EZ_UNIT <= lim.y) {
            for (; b + 16 <= b1; b += 16) {
                uint32_t s = 0;
                for (uint32_t h = 0; h < 16; h += 4) {
                    uint32_t v[4], amb = PC_AMB;
#pragma unroll
                    for (uint32_t i = 0; i < 4; i++)
                        v[i] = pc_pi_quot_less1(T.pitab, Q.Xd[b + h + i], rm, true, &amb);
                    if (__ballot(amb < PC_AMB)) {
                        for (uint32_t i = 0; i < 4; i++)
                            s += pc_pi_quot_exact(T, Q.Xb[b + h + i], Q.Xd[b + h + i], m, rm) - 1u;
                    } else {
                        s += v[0] + v[1] + v[2] + v[3];
                    }
                }
                a += s + 16u;
            }
        }
        for (; b < b1; b++) {
            const uint2 r = Q.e_rng[b];
            if (r.x & PC_CAND)
                continue;
            const bool in = k >= r.x && k < r.y;
            if (!__ballot(in))
                continue;
            uint32_t amb = PC_AMB;
            uint32_t v = pc_pi_quot_less1(T.pitab, Q.Xd[b], rm, in, &amb) + 1u;
            if (__ballot(amb < PC_AMB)) {
                if (in)
                    v = pc_pi_quot_exact(T, Q.Xb[b], Q.Xd[b], m, rm);
            }
            a += in ? v : 0u;
        }
    }
    *acc += (int64_t)(2 * a);
}

// The candidate easy leaves (p_b^2 <= y): *acc -= mu(m) phi(u, b-1), u = X_b / m,
// over the band's b and the squarefree m of b's range with lpf(m) > p_b.  The
// calling workgroup (NT threads; every thread calls) takes tiles lb, lb + nlb,
// ... of PC_EZ_TILE wheel numbers of a band: it keeps those m that can be a
// leaf of the band's first b (lpf(m) > p_b; a third of them where p_b^2 is
// near y), packed in LDS, and then each thread takes one m, with 1/m formed
// once, against the b of the band.  (One item per (b, m), the table tested for
// each, took 6.3 ms of one pi(10^18); this takes 0.7 ms, 3.8 beside the prime leaves.)
template <int NT> struct pc_cand_lds {
    uint32_t m[PC_EZ_TILE]; // m's wheel number | (mu(m) > 0) << 31
    uint32_t l[PC_EZ_TILE]; // lpf(m)
    uint32_t n;
};
template <int NT>
__device__ __forceinline__ void pc_easy_cands(const pc_tables &T, const pc_query &Q, uint64_t lb,
                                              uint64_t nlb, pc_cand_lds<NT> &L, int64_t *acc,
                                              unsigned long long *nleaf)
{
    const uint32_t nband = Q.a / PC_EZ_BAND + 1, lane = pc_lane();
    const uint64_t *const boff = Q.e_boff + nband;
    const uint64_t U = Q.e_total[1];
    const uint32_t kend = (uint32_t)pc_wheel_count(T, Q, Q.y); // wheel numbers of m <= y
    for (uint64_t u = lb; u < U; u += nlb) {
        const uint32_t g = pc_uniform(pc_band_of(boff, nband, u));
        const uint32_t b0 = max(g * PC_EZ_BAND, Q.c + 1), b1 = min(g * PC_EZ_BAND + PC_EZ_BAND, Q.a);
        const uint32_t k0 = Q.e_bk[nband + g] + (uint32_t)(u - boff[g]) * PC_EZ_TILE;
        const uint32_t p0 = T.primes[b0];
        __syncthreads(); // the last tile's reads
        if (threadIdx.x == 0)
            L.n = 0;
        __syncthreads();
#pragma unroll 4
        for (uint32_t i = 0; i < PC_EZ_TILE / NT; i++) {
            const uint32_t k = k0 + i * NT + threadIdx.x;
            const int32_t v = k < kend ? T.mulpfw[k] : 0;
            const uint32_t l = v < 0 ? (uint32_t)(-v) : (uint32_t)v;
            const bool keep = l > p0;
            const uint64_t bal = __ballot(keep);
            uint32_t at = 0;
            if (lane == 0 && bal)
                at = atomicAdd(&L.n, (uint32_t)__builtin_popcountll(bal));
            at = pc_uniform(at) + (uint32_t)__builtin_popcountll(bal & ((1ull << lane) - 1));
            if (keep) {
                L.m[at] = k | (v > 0 ? 0x80000000u : 0u);
                L.l[at] = l;
            }
        }
        __syncthreads();
        const uint32_t n = L.n;
        for (uint32_t i = threadIdx.x; (i & ~63u) < n; i += NT) {
            const bool have = i < n;
            const uint32_t e = have ? L.m[i] : 0u, l = have ? L.l[i] : 0u;
            const uint32_t m = pc_wheel_m(T, e & 0x7FFFFFFFu);
            const double rm = pc_rcp_f64(m);
            int64_t s = 0;
            uint32_t cnt = 0;
            for (uint32_t b = b0; b < b1; b++) {
                const uint2 r = Q.e_rng[b];
                if (!(r.x & PC_CAND))
                    continue;
                const bool in = l > T.primes[b] && m >= (r.x & ~PC_CAND) && m <= r.y;
                if (!__ballot(in))
                    continue;
                uint32_t amb = PC_AMB;
                uint32_t v = pc_pi_quot_less1(T.pitab, Q.Xd[b], rm, in, &amb);
                if (__ballot(amb < PC_AMB)) {
                    if (in)
                        v = pc_pi_lookup32(T.pitab, pc_quot31(Q.Xb[b], Q.Xd[b], m)) - 1u;
                }
                if (in) { // phi(u, b-1) = pi(u) - b + 2
                    s += (int64_t)v + 3 - (int64_t)b;
                    cnt++;
                }
            }
            *acc += (e >> 31) ? -s : s;
            *nleaf += cnt;
        }
    }
}

// pi(x) = S1 + S2t + S2e + S2h + a - 1 - P2, with
//   S2h = in-segment sums + sum w * carry, and
//   P2  = sum_{k=a+1}^{kx} (phi(x/p_k, B) + B - 1) - sum_{k=a+1}^{kx} (k - 1),
//   B = c + nb = max(c, bmax) primes crossed by the sieve.
__device__ __forceinline__ void pc_combine_one(const pc_sums &S, const pc_query &Q, uint64_t kp2,
                                               pc_final *out)
{
    const pc_s128 s2h = S.hard_local + S.hard_dot;
    const pc_s128 B = (pc_s128)(Q.c + Q.nb);
    const pc_s128 a = Q.a, K = kp2;
    pc_s128 p2 = S.p2_local + S.p2_dot;
    if (K > a)
        p2 += (K - a) * (B - 1) - ((K - 1) * K / 2 - (a - 1) * a / 2);
    const pc_s128 phi = S.s1 + S.s2t + S.s2e + s2h;
    const pc_s128 pi = phi + a - 1 - p2;
    out->s1 = S.s1;
    out->s2t = S.s2t;
    out->s2e = S.s2e;
    out->s2h = s2h;
    out->p2 = p2;
    out->phi = phi;
    out->pi = (uint64_t)pi;
    out->pi_hi = (uint64_t)(pi >> 64);
    out->ok = pi < 0 ? 0 : (pi >> 64) == 0 ? 1 : 2;
}
