// pc_device.h -- integer helpers shared by the gfx950 kernels and the host
// planner of the prime-counting library.
//
// All arithmetic of the method is exact integer arithmetic.  The GPU has no
// integer divide instruction, so every quotient on a hot path is formed by a
// multiply-high with a precomputed 64-bit reciprocal of the divisor and one
// correction step (division by invariant integers, Granlund & Montgomery,
// PLDI 1994), or -- for divisors that change per lane -- from an fp64
// estimate corrected by an exact integer remainder test.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned __int128 pc_u128;
typedef __int128 pc_s128;

#define PC_HD __host__ __device__ __forceinline__

// r = floor((2^64 - 1) / d) for d >= 1.
PC_HD uint64_t pc_recip(uint64_t d) { return ~0ull / d; }

PC_HD uint64_t pc_mulhi(uint64_t a, uint64_t b)
{
    return (uint64_t)(((pc_u128)a * b) >> 64);
}

// floor(n / d) given r = pc_recip(d).  For any n < 2^64 and d >= 1:
// n*r/2^64 = n/d - n(1+e)/(d 2^64) with e = (2^64-1) mod d < d, which lies in
// (n/d - 1, n/d]; so q0 = mulhi(n, r) is floor(n/d) or one less.
PC_HD uint64_t pc_div(uint64_t n, uint64_t d, uint64_t r)
{
    uint64_t q = pc_mulhi(n, r);
    uint64_t rem = n - q * d;
    if (rem >= d)
        q++;
    return q;
}

// floor(n / d) for d < 2^32 when the quotient is known to be < 2^50: the
// fp64 estimate has relative error below 2^-51, so it is within 1 of the
// true quotient and one signed remainder test fixes it.
PC_HD uint64_t pc_div_small_q(uint64_t n, uint32_t d)
{
    uint64_t q = (uint64_t)((double)n / (double)d);
    int64_t rem = (int64_t)(n - q * (uint64_t)d);
    if (rem < 0)
        q--;
    else if (rem >= (int64_t)d)
        q++;
    return q;
}

// Quotients on the leaf paths, where the divisor changes from lane to lane
// and the dividend is shared (the caller converts it to fp64 once).  1/d is
// the hardware fp64 reciprocal estimate refined by two Newton steps; each
// step squares the relative error, so any estimate better than 2^-20 ends
// within a few units of 2^-52.  The product with fl(n) is then within
// n/d * 2^-49 of n/d, under 1/4 for n/d < 2^47, and the truncated estimate
// is floor(n/d) or one off, which one exact remainder test corrects.
__device__ __forceinline__ double pc_rcp_f64(uint32_t d)
{
    const double dd = (double)d;
    double r = __builtin_amdgcn_rcp(dd);
    r = __builtin_fma(__builtin_fma(-dd, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-dd, r, 1.0), r, r);
    return r;
}

// floor(n / d) for 1 <= d < 2^32 when the quotient is known to be below
// 2^32 - 1; nd = (double)n.  The estimate is raised by 2^-10, more than its
// error (2^-17 here), so the truncation is floor(n/d) or one above it, and
// only the sign of the remainder needs testing.  (The general form of
// pc_quot31; the leaf kernels' divisors are below 2^31 and take that.)
__device__ __forceinline__ uint32_t pc_quot32(uint64_t n, double nd, uint32_t d)
{
    const uint32_t q = (uint32_t)__builtin_fma(nd, pc_rcp_f64(d), 0x1p-10);
    const int64_t rem = (int64_t)(n - (uint64_t)q * d);
    return q - (rem < 0 ? 1u : 0u);
}

// pc_quot32 for divisors d < 2^31, with rd = 1/d correctly rounded (a table
// entry): the estimate's error is then below 2^-19, well under the same 2^-10
// margin, and the remainder n - q d of the estimate q lies in [-d, d), so its
// low 32 bits read as a signed number are its value.
__device__ __forceinline__ uint32_t pc_quot31r(uint64_t n, double nd, uint32_t d, double rd)
{
    const uint32_t q = (uint32_t)__builtin_fma(nd, rd, 0x1p-10);
    const int32_t rem = (int32_t)((uint32_t)n - q * d);
    return q - (rem < 0 ? 1u : 0u);
}

// pc_quot31r with 1/d from pc_rcp_f64.
__device__ __forceinline__ uint32_t pc_quot31(uint64_t n, double nd, uint32_t d)
{
    const uint32_t q = (uint32_t)__builtin_fma(nd, pc_rcp_f64(d), 0x1p-10);
    const int32_t rem = (int32_t)((uint32_t)n - q * d);
    return q - (rem < 0 ? 1u : 0u);
}

// pc_quot_in for a 64-bit divisor 2^32 <= d < 2^40 (the primes above 2^32 of
// P2 when x > 2^64): n is x modulo 2^64 and nd the rounded x; the remainder of
// the estimate, formed modulo 2^64, is small and exact.
__device__ __forceinline__ bool pc_quot_in64(uint64_t n, double nd, uint64_t d, uint64_t base,
                                             uint32_t span, uint32_t *off)
{
    const double t = nd / (double)d - (double)base;
    if (!(t > -2.0 && t < (double)span + 2.0))
        return false;
    int32_t q = (int32_t)t;
    const int64_t rem = (int64_t)(n - (base + (uint64_t)(int64_t)q) * d);
    if (rem < 0)
        q--;
    else if (rem >= (int64_t)d)
        q++;
    *off = (uint32_t)q;
    return q >= 0 && (uint32_t)q < span;
}

// floor(n / d) - base for 1 <= d < 2^32, base < 2^47, n/d < 2^47:
// returns false if the quotient lies outside [base, base + span), span <
// 2^30, else true with *off = the quotient - base.  nd = (double)n.
__device__ __forceinline__ bool pc_quot_in(uint64_t n, double nd, uint32_t d, uint64_t base,
                                           uint32_t span, uint32_t *off)
{
    const double t = nd * pc_rcp_f64(d) - (double)base;
    if (!(t > -2.0 && t < (double)span + 2.0))
        return false;
    int32_t q = (int32_t)t;
    const int64_t rem = (int64_t)(n - (base + (uint64_t)(int64_t)q) * d);
    if (rem < 0)
        q--;
    else if (rem >= (int64_t)d)
        q++;
    *off = (uint32_t)q;
    return q >= 0 && (uint32_t)q < span;
}

// u - base for u = floor(n / m), given n modulo 2^32, its value nd in fp64,
// base modulo 2^32 and base4 = 1/4 - base; m < 2^31, u < 2^48, base < 2^48.
// 1/m is off by a few units of 2^-53 (pc_rcp_f64) and nd by 2^-53 of itself, so
// the estimate is off by less than u 2^-50 <= 1/4; raised by 1/4 its floor is u
// or u + 1, and the remainder n - q m, in [-m, m), is its low 32 bits read as a
// signed number: their sign decides.  *in: u lies in [base, base + span), span
// <= 2^21 (else the result says nothing).
__device__ __forceinline__ uint32_t pc_quot_off(uint32_t n, double nd, uint32_t m, uint32_t base,
                                                double base4, uint32_t span, bool *in)
{
    const double t = __builtin_fma(nd, pc_rcp_f64(m), base4); // u - base, raised
    uint32_t off = (uint32_t)(int32_t)t;
    off += (uint32_t)((int32_t)(n - (base + off) * m) >> 31);
    *in = off < span && t > -1.0;
    return off;
}

// floor(e / p) for e < 2^30, p <= 2^24 and a quotient below 2^17, rp = 1 / p in
// fp32, off by at most one unit: the estimate is off by less than 2^-22 of the
// quotient, so its floor is within one, and one step corrects it.
PC_HD uint32_t pc_quot_near(uint32_t e, uint32_t p, float rp)
{
    uint32_t q = (uint32_t)((float)e * rp);
    const int32_t r = (int32_t)(e - q * p);
    if (r < 0)
        q--;
    else if (r >= (int32_t)p)
        q++;
    return q;
}

// n mod p for n < 2^47, p < 2^31, nd = (double)n, rp = 1 / p: adding 2^52 leaves
// the nearest integer to n / p (off by less than 2^-5 before it is rounded) in
// the low bits of the double; the remainder, less than p in size, is formed
// modulo 2^32.
PC_HD uint32_t pc_rem_near(uint64_t n, double nd, uint32_t p, double rp)
{
    const uint32_t q = (uint32_t)__builtin_bit_cast(uint64_t, __builtin_fma(nd, rp, 0x1p52));
    const int32_t r = (int32_t)((uint32_t)n - q * p);
    return (uint32_t)(r + (r < 0 ? (int32_t)p : 0));
}

// Exact floor(n / d) for any n < 2^64, 1 <= d < 2^32: fp64 estimate, one
// exact refinement of the remainder, then a final one-step correction.
PC_HD uint64_t pc_div_any(uint64_t n, uint32_t d)
{
    if (d == 1)
        return n;
    double dd = (double)d;
    uint64_t q = (uint64_t)((double)n / dd);      // q <= 2^63, within 2^11 of the truth
    int64_t rem = (int64_t)(n - q * (uint64_t)d); // |rem| <= 2^11 d < 2^43
    q += (int64_t)((double)rem / dd);             // now within 1
    rem = (int64_t)(n - q * (uint64_t)d);
    while (rem < 0) {
        q--;
        rem += d;
    }
    while (rem >= (int64_t)d) {
        q++;
        rem -= d;
    }
    return q;
}

// Queries above 2^64: x = hi 2^64 + lo (x <= 2^72).
//
// floor((hi 2^64 + lo) / d) for 1 <= d < 2^32 and hi < d (so the quotient is
// below 2^64), by long division in base 2^32; *rem receives the remainder.
PC_HD uint64_t pc_div_wide32(uint64_t hi, uint64_t lo, uint32_t d, uint32_t *rem)
{
    uint64_t r = hi;
    const uint64_t n1 = (r << 32) | (lo >> 32);
    const uint64_t q1 = n1 / d;
    r = n1 - q1 * d;
    const uint64_t n0 = (r << 32) | (lo & 0xFFFFFFFFull);
    const uint64_t q0 = n0 / d;
    if (rem)
        *rem = (uint32_t)(n0 - q0 * d);
    return (q1 << 32) | q0;
}

// floor(x / d) for x = hi 2^64 + lo (xd = x rounded to double) when the
// quotient is below 2^64 and d < 2^46: the fp64 estimate q0 is within
// q 2^-51 + 1 < 2^13 of the quotient, so the remainder x - q0 d, formed
// modulo 2^64, is a signed number below 2^59 in size; one integer division of
// it brings the estimate within one, and the remainder's sign settles it.
PC_HD uint64_t pc_div_wide(uint64_t lo, double xd, uint64_t d)
{
    const double t = xd / (double)d;
    uint64_t q = t < 0x1p64 ? (uint64_t)t : ~0ull;
    int64_t rem = (int64_t)(lo - q * d);
    q += rem / (int64_t)d;
    rem = (int64_t)(lo - q * d);
    while (rem < 0) {
        q--;
        rem += (int64_t)d;
    }
    while (rem >= (int64_t)d) {
        q++;
        rem -= (int64_t)d;
    }
    return q;
}

// floor(x / d) for x = hi 2^64 + lo, 1 <= d < 2^32, any hi: the quotient's
// high word in *qhi, its low word returned (long division in base 2^32).
PC_HD uint64_t pc_div_u128_32(uint64_t hi, uint64_t lo, uint32_t d, uint64_t *qhi, uint32_t *rem)
{
    *qhi = hi / d;
    return pc_div_wide32(hi % d, lo, d, rem);
}

// floor(x / d) for 1 <= d < 2^32 when the quotient is below 2^50, x given as
// its low word lo and its value xd in fp64 (x may exceed 2^64): the estimate
// is within one of the quotient and the remainder, formed modulo 2^64, is
// exact.  For x < 2^64 this is pc_div_small_q.
PC_HD uint64_t pc_div_small_qd(uint64_t lo, double xd, uint32_t d)
{
    uint64_t q = (uint64_t)(xd / (double)d);
    const int64_t rem = (int64_t)(lo - q * (uint64_t)d);
    if (rem < 0)
        q--;
    else if (rem >= (int64_t)d)
        q++;
    return q;
}

// isqrt(hi 2^64 + lo) for values below 2^126: the fp64 root is within one of
// the integer root below 2^104, and the loops settle it.
PC_HD uint64_t pc_isqrt_wide(uint64_t hi, uint64_t lo)
{
    const pc_u128 n = ((pc_u128)hi << 64) | lo;
    uint64_t r = (uint64_t)__builtin_sqrt((double)n);
    while (r > 0 && (pc_u128)r * r > n)
        r--;
    while ((pc_u128)(r + 1) * (r + 1) <= n)
        r++;
    return r;
}

// The sieve's bitmap keeps only the integers prime to 30 (2, 3 and 5 always
// belong to the wheel): 8 bits, one byte, for every 30 integers.  With the
// offset d of an integer from a multiple of 30, bit 8 (d / 30) + i stands for
// the i-th of the residues 1, 7, 11, 13, 17, 19, 23, 29; for those residues
// that is floor(4 d / 15).
#define PC_W30_MASK 0x208A2882u            // bit r set: r < 30 is prime to 30
#define PC_W30_RES 0x1D1713110D0B0701ull   // the residues, a byte each
#define PC_W30_GAPS 0x26424246u            // residue i + 1 less residue i, a nibble each

// integers covered by a segment of 2^log2s bits
PC_HD uint64_t pc_seg_span(uint32_t log2s) { return 15ull << (log2s - 2); }

// residue i
PC_HD uint32_t pc_w30_res(uint32_t i) { return (uint32_t)(PC_W30_RES >> (8 * i)) & 255u; }

// integers prime to 30 among 0 .. d, d < 2^27
PC_HD uint32_t pc_w30_le(uint32_t d)
{
    const uint32_t q = d / 30u, r = d - 30u * q;
    return 8u * q + (uint32_t)__builtin_popcount(PC_W30_MASK & ((2u << r) - 1u));
}

// the bit of d, d prime to 30, d < 2^21: the fraction of 4 d / 15 is then
// between 1/15 and 14/15, and the fp32 product is off by less than 1/16
PC_HD uint32_t pc_w30_bit(uint32_t d) { return (uint32_t)((float)d * (4.0f / 15.0f)); }

// the integer of a bit
PC_HD uint32_t pc_w30_int(uint32_t bit) { return 30u * (bit >> 3) + pc_w30_res(bit & 7u); }

// the least j' >= j prime to 30, 0 <= j <= 30
PC_HD uint32_t pc_w30_next(uint32_t j)
{
    return j < 30u ? j + (uint32_t)__builtin_ctz(PC_W30_MASK >> j) : 31u;
}

// Integer square and cube roots, exact (used by the host planner).
PC_HD uint64_t pc_isqrt(uint64_t n)
{
    uint64_t r = (uint64_t)__builtin_sqrt((double)n);
    while (r > 0 && (pc_u128)r * r > n)
        r--;
    while ((pc_u128)(r + 1) * (r + 1) <= n)
        r++;
    return r;
}

PC_HD uint64_t pc_icbrt(uint64_t n)
{
    uint64_t r = (uint64_t)__builtin_cbrt((double)n);
    while (r > 0 && (pc_u128)r * r * r > n)
        r--;
    while ((pc_u128)(r + 1) * (r + 1) * (r + 1) <= n)
        r++;
    return r;
}

// pi table: entry e holds a 32-bit mask of the odd numbers 64e+1 .. 64e+63
// (bit j <-> 64e + 2j + 1 is prime) and the number of odd primes below 64e.
// pi(n) = [n >= 2] + (odd primes <= n).
PC_HD uint32_t pc_pi_lookup(const uint2 *tab, uint64_t n)
{
    if (n < 2)
        return 0;
    uint64_t i = (n - 1) >> 1; // odd index of the largest odd number <= n
    uint2 e = tab[i >> 5];
    uint32_t sh = 31u - (uint32_t)(i & 31);
    return 1u + e.y + (uint32_t)__builtin_popcount((e.x << sh)); // bits 0..(i&31)
}

// The same for 2 <= n < 2^32, in 32-bit arithmetic.
PC_HD uint32_t pc_pi_lookup32(const uint2 *tab, uint32_t n)
{
    const uint32_t i = (n - 1) >> 1;
    const uint2 e = tab[i >> 5];
    return 1u + e.y + (uint32_t)__builtin_popcount(e.x << (31u - (i & 31)));
}
