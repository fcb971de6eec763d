// pc_seed.hip -- the seeds of a sieve started in the middle (Section 4):
// phi(m, b) for one m and every c <= b <= c + nb, computed on their own, so
// that a window of segments starting at m needs nothing from the windows
// before it.
//
// From phi(m, c) (the wheel), eq. (4.1) gives each next column:
//     phi(m, b) = phi(m, b-1) - t_b,   t_b = phi(floor(m / p_b), b-1),
// and the seeds are one prefix sum of the terms.  Each term is taken by the
// rule that fits it (the multifaceted scheme of Section 4):
//   * u = floor(m / p_b) < p_b:      only 1 survives (0 if u = 0), t_b = [u >= 1]
//     (the tail past pi(sqrt m), where each column is the last one less 1);
//   * p_b^2 > u:                     Legendre, t_b = pi(u) - (b-1) + 1, from the
//     pi table (u < m^(2/3) here, inside the table's range);
//   * otherwise:                     eq. (4.1) again on (u, b-1): phi(u, c) less
//     the children (floor(u / p_i), i-1), c < i < b, each resolved the same way
//     depth first.  These are the b with p_b^3 <= m, a few hundred to a few
//     thousand columns; their children's children are dealt out to the
//     threads of one workgroup per column.
// Two launches: the terms (one workgroup per column p_b <= icbrt m, then one
// thread per closed column) and the prefix sum (one workgroup).
#include "pc_block.h"
#include "pc_internal.h"

namespace {

constexpr uint32_t SEED_T = 1024;   // threads per workgroup of the term kernel
constexpr uint32_t SCAN_T = 1024;   // threads of the prefix-sum workgroup
// terms each of them takes at a time: more loads in flight against more cache
// lines per load (phi_seed at 3 * 10^10, 20000 columns: 1: 103 us, 2: 90, 4: 86.5,
// 8: 91, 16: 96)
constexpr uint32_t SCAN_PER = 4;
// Children of a column that expand, and the first: p_i < p_b and p_i^3 <= m / p_b, so
// p_i <= m^(1/4) <= 2^12 for m <= 2^48: fewer than pi(2^12) = 564
constexpr uint32_t SEED_A = 568;
constexpr int SEED_MAXD = 32;       // depth bound: m <= 2^48 and p_{c+1} >= 3

struct seed_ctx {
    const uint32_t *primes;
    const uint64_t *recip;
    const uint2 *pitab;
    const uint32_t *phitab;
    uint64_t pi_limit;
    uint64_t Qc, rQc;
    uint32_t phiQ, c;
    int32_t *err;
};

// phi(v, c) from the wheel: phi(Q_c, c) per full period plus the table
__device__ __forceinline__ int64_t seed_wheel(const seed_ctx &S, uint64_t v)
{
    const uint64_t q = pc_div(v, S.Qc, S.rQc);
    return (int64_t)(q * S.phiQ + S.phitab[v - q * S.Qc]);
}

// The node (v, k), k >= c, when its value is closed: true and *val set;
// false when eq. (4.1) has to expand it (v >= q^2, q = p_{k+1}).
__device__ __forceinline__ bool seed_leaf_p(const seed_ctx &S, uint64_t v, uint32_t k, uint64_t q,
                                            int64_t *val)
{
    if (k <= S.c) {
        *val = seed_wheel(S, v);
        return true;
    }
    if (v < q) {
        *val = v ? 1 : 0;
        return true;
    }
    if (v < q * q) {
        if (v > S.pi_limit) { // the caller sized the pi table for every such v
            atomicOr(S.err, 16);
            *val = 0;
        } else {
            *val = (int64_t)pc_pi_lookup(S.pitab, v) - (int64_t)k + 1;
        }
        return true;
    }
    return false;
}

__device__ __forceinline__ bool seed_leaf(const seed_ctx &S, uint64_t v, uint32_t k, int64_t *val)
{
    return seed_leaf_p(S, v, k, S.primes[k + 1], val);
}

// phi(v, k) by eq. (4.1) depth first, with an explicit stack: a node that
// expands adds phi(v, c) with its sign and takes its children in turn.  P and R
// are the primes from p_{c+1} on and their reciprocals; the node at hand stays
// in registers, since most children are closed and only an expanding one goes
// through the stack (private memory).
__device__ int64_t seed_phi(const seed_ctx &S, uint64_t v, uint32_t k, const uint32_t *P,
                            const uint64_t *R)
{
    int64_t total;
    if (seed_leaf(S, v, k, &total))
        return total;
    uint64_t sv[SEED_MAXD];
    uint32_t sk[SEED_MAXD], si[SEED_MAXD];
    int d = 0;
    total = seed_wheel(S, v);
    uint32_t i = S.c + 1;
    for (;;) {
        if (i > k) {
            if (d == 0)
                break;
            d--;
            v = sv[d];
            k = sk[d];
            i = si[d];
            continue;
        }
        const uint64_t p = P[i - S.c - 1];
        const uint64_t w = pc_div(v, p, R[i - S.c - 1]);
        const int64_t sgn = (d & 1) ? 1 : -1; // children sit one level down
        int64_t lv;
        if (seed_leaf_p(S, w, i - 1, p, &lv)) {
            total += sgn * lv;
            i++;
        } else {
            if (d + 1 >= SEED_MAXD) {
                atomicOr(S.err, 16);
                return 0;
            }
            sv[d] = v;
            sk[d] = k;
            si[d] = i + 1;
            d++;
            v = w;
            k = i - 1;
            i = S.c + 1;
            total += sgn * seed_wheel(S, w);
        }
    }
    return total;
}

// term[0] = phi(m, c); term[j] = t_{c+j} for 1 <= j <= nb.
//
// Workgroups 0 .. nrec - 1 take the columns j = 1 .. nrec whose terms may
// expand; the rest one closed column per thread.  A term that expands is
// phi(u, c) less its children phi(floor(u / p_i), i-1), c < i < b.  The
// children with p_i^3 <= u expand in turn, a few dozen of several hundred; the
// workgroup shares out their own children, the pairs i2 < i of the first A primes, so that no thread walks a whole child's tree.  Bound by
// latency: a chain of a division and a pi-table read per node, up to 46 nodes
// a pair at m = 2 * 10^10, so every column gets 16 wavefronts and reads its
// primes from LDS (phi_seed at 2 * 10^10, 15000 columns: 300 -> 76 us; the
// triangle over all children, most of its pairs empty, took 224 us of it).
__global__ __launch_bounds__(SEED_T) void k_seed_terms(seed_ctx S, uint64_t m, uint32_t nb,
                                                       uint32_t nrec, int64_t *term)
{
    __shared__ int64_t scr[SEED_T / 64];
    __shared__ uint64_t R[SEED_A];
    __shared__ uint32_t P[SEED_A];
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x >= nrec) {
        const uint64_t e = (uint64_t)(blockIdx.x - nrec) * SEED_T + tid;
        if (e == 0)
            term[0] = seed_wheel(S, m);
        const uint64_t j = nrec + e;
        if (e == 0 || j > nb)
            return;
        const uint32_t b = S.c + (uint32_t)j;
        int64_t v = 0;
        if (!seed_leaf(S, pc_div(m, S.primes[b], S.recip[b]), b - 1, &v))
            atomicOr(S.err, 16); // the caller counted the columns that expand
        term[j] = v;
        return;
    }
    const uint32_t j = blockIdx.x + 1, b = S.c + j;
    const uint64_t u = pc_div(m, S.primes[b], S.recip[b]);
    int64_t s;
    if (seed_leaf(S, u, b - 1, &s)) { // closed (uniform over the workgroup)
        if (tid == 0)
            term[j] = s;
        return;
    }
    const uint32_t na = b - 1 - S.c;
    uint32_t A = 1; // children 1 .. A - 1 expand (child 0 is closed by the wheel)
    s = 0;
    for (uint32_t a0 = 0; a0 < na; a0 += SEED_T) {
        const uint32_t a = a0 + tid;
        bool open = false;
        if (a < na) {
            const uint64_t p = S.primes[S.c + 1 + a], r = S.recip[S.c + 1 + a];
            const uint64_t v = pc_div(u, p, r);
            int64_t lv;
            open = !seed_leaf_p(S, v, S.c + a, p, &lv);
            s += open ? seed_wheel(S, v) : lv;
            if ((open || a == 0) && a < SEED_A) {
                P[a] = (uint32_t)p;
                R[a] = r;
            }
        }
        A += (uint32_t)__syncthreads_count(open);
    }
    if (A > SEED_A) { // not for m <= 2^48
        if (tid == 0)
            atomicOr(S.err, 16);
        A = SEED_A;
    }
    const uint32_t npair = A * (A - 1) / 2; // A < 2^10
    for (uint32_t t = tid; t < npair; t += SEED_T) {
        // pair t = a (a - 1) / 2 + a2, 0 <= a2 < a
        uint32_t a = (uint32_t)((__builtin_sqrtf(8.0f * (float)t + 1.0f) + 1.0f) * 0.5f);
        while (a * (a + 1) / 2 <= t)
            a++;
        while (a * (a - 1) / 2 > t)
            a--;
        const uint32_t a2 = t - a * (a - 1) / 2;
        const uint64_t v = pc_div(u, P[a], R[a]);
        s -= seed_phi(S, pc_div(v, P[a2], R[a2]), S.c + a2, P, R);
    }
    s = pc_block_sum<SEED_T>(s, scr);
    if (tid == 0)
        term[j] = seed_wheel(S, u) - s;
}

// out[j] = term[0] - (term[1] + ... + term[j]) = phi(m, c + j), 0 <= j <= nb:
// SCAN_PER consecutive terms a thread and round, all read at once
__global__ __launch_bounds__(SCAN_T) void k_seed_scan(const int64_t *term, uint32_t nb,
                                                      uint64_t *out, int32_t *err)
{
    __shared__ int64_t scr[SCAN_T / 64];
    int64_t base = 0;
    bool neg = false;
    for (uint64_t r = 0; r <= nb; r += SCAN_T * SCAN_PER) {
        const uint64_t j0 = r + threadIdx.x * SCAN_PER;
        int64_t v[SCAN_PER], loc = 0, tot;
#pragma unroll
        for (uint32_t k = 0; k < SCAN_PER; k++)
            v[k] = term[min(j0 + k, (uint64_t)nb)];
#pragma unroll
        for (uint32_t k = 0; k < SCAN_PER; k++)
            loc += j0 + k > nb ? 0 : j0 + k ? -v[k] : v[k];
        int64_t run = base + pc_block_excl_scan<SCAN_T>(loc, scr, &tot);
        base += tot;
#pragma unroll
        for (uint32_t k = 0; k < SCAN_PER; k++) {
            run += j0 + k ? -v[k] : v[k];
            if (j0 + k <= nb) {
                neg |= run < 0;
                out[j0 + k] = (uint64_t)run;
            }
        }
    }
    if (neg)
        atomicOr(err, 16);
}

} // namespace

hipError_t pc_launch_seed(const pc_tables &T, uint32_t c, uint64_t m, uint32_t nb,
                          uint32_t nrec, uint64_t pi_limit, int64_t *term, uint64_t *out,
                          int32_t *err, hipStream_t s)
{
    seed_ctx S{};
    S.primes = T.primes;
    S.recip = T.recip;
    S.pitab = T.pitab;
    S.phitab = T.phitab;
    S.pi_limit = pi_limit;
    S.Qc = T.Qc;
    S.rQc = pc_recip(T.Qc);
    S.phiQ = T.phiQ;
    S.c = c;
    S.err = err;
    nrec = std::min(nrec, nb);
    const uint32_t nclosed = nb - nrec + 1; // with j = 0
    k_seed_terms<<<nrec + (nclosed + SEED_T - 1) / SEED_T, SEED_T, 0, s>>>(S, m, nb, nrec, term);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    k_seed_scan<<<1, SCAN_T, 0, s>>>(term, nb, out, err);
    return hipGetLastError();
}
