// pc_leaves.hip -- one-query kernels for the parts of phi(x, a) = S1 + S2 that
// need no sieve (S1, trivial and easy special leaves) and the final
// combination; the per-item work is in pc_leafwork.h.
#include "pc_leafwork.h"

#define LV_T 256

// ---------------------------------------------------------------------------
// S1: one lane per item (grid-stride).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void s1_wg(const pc_tables &T, const pc_query &Q, uint32_t wg,
                                      uint32_t nwg)
{
    __shared__ pc_s128 scr[LV_T / 64];
    __shared__ unsigned long long scr64[LV_T / 64];
    pc_s128 acc = 0;
    unsigned long long terms =
        pc_s1_items(T, Q, (uint64_t)wg * LV_T + threadIdx.x, (uint64_t)nwg * LV_T, &acc);
    acc = pc_block_sum128<LV_T>(acc, scr);
    terms = pc_block_sum<LV_T>(terms, scr64);
    if (threadIdx.x == 0) {
        pc_atomic_add128(&Q.sums->s1, acc);
        atomicAdd(&Q.sums->n_s1, terms);
    }
}

__global__ __launch_bounds__(LV_T) void k_s1(pc_tables T, pc_query Q)
{
    s1_wg(T, Q, blockIdx.x, gridDim.x);
}

hipError_t pc_launch_s1(const pc_tables &T, const pc_query &Q, uint32_t nblocks, hipStream_t s)
{
    k_s1<<<nblocks, LV_T, 0, s>>>(T, Q);
    return hipGetLastError();
}

// X_b and the per-b set-up of the special leaves (pc_leaf_setup_band); at most
// 1024 workgroups, so that few of them meet at the sums.
__global__ __launch_bounds__(LV_T) void k_leaf_setup(pc_tables T, pc_query Q)
{
    __shared__ pc_s128 scr[LV_T / 64];
    pc_setup_sums S;
    const uint32_t n = max(Q.a, Q.c + Q.nb) + 1; // b < n
    for (uint32_t b0 = blockIdx.x * LV_T; b0 < n; b0 += gridDim.x * LV_T)
        pc_leaf_setup_band(T, Q, b0 + threadIdx.x, &S);
    pc_setup_flush<LV_T>(Q, S, scr);
}

// The bands' unit offsets (workgroups 0 and 1, a kind each) and the suffix
// maxima of the hard-leaf u ranges (workgroup 2).
#define BS_T 1024
__global__ __launch_bounds__(BS_T) void k_band_scan(pc_query Q)
{
    __shared__ uint64_t sh[BS_T];
    const uint32_t nband = Q.a / PC_EZ_BAND + 1, w = blockIdx.x;
    if (w < 2)
        pc_band_scan<BS_T>(Q.e_boff + w * nband, nband, Q.e_total + w, sh);
    else
        pc_ub_suffix<BS_T>(Q, sh);
}

hipError_t pc_launch_leaf_setup(const pc_tables &T, const pc_query &Q, hipStream_t s)
{
    const uint32_t n = Q.a > Q.c + Q.nb ? Q.a + 1 : Q.c + Q.nb + 1;
    const uint32_t blocks = (n + LV_T - 1) / LV_T;
    k_leaf_setup<<<blocks < 1024 ? blocks : 1024, LV_T, 0, s>>>(T, Q);
    k_band_scan<<<3, BS_T, 0, s>>>(Q);
    return hipGetLastError();
}

// Candidate easy leaves of one query (pc_easy_cands).
#define EZ_T PC_EZ_UNIT
__device__ __forceinline__ void easy_cands_wg(const pc_tables &T, const pc_query &Q, uint32_t wg,
                                              uint32_t nwg)
{
    __shared__ pc_s128 scr[EZ_T / 64];
    __shared__ unsigned long long scr64[EZ_T / 64];
    __shared__ pc_cand_lds<EZ_T> L;
    if (wg >= Q.e_total[1])
        return;
    unsigned long long nleaf = 0;
    int64_t acc = 0;
    pc_easy_cands<EZ_T>(T, Q, wg, nwg, L, &acc, &nleaf);
    const pc_s128 s = pc_block_sum128<EZ_T>((pc_s128)acc, scr);
    nleaf = pc_block_sum<EZ_T>(nleaf, scr64);
    if (threadIdx.x == 0 && nleaf) {
        pc_atomic_add128(&Q.sums->s2e, s);
        atomicAdd(&Q.sums->n_easy, nleaf);
    }
}

__global__ __launch_bounds__(EZ_T) void k_easy_cands(pc_tables T, pc_query Q)
{
    easy_cands_wg(T, Q, blockIdx.x, gridDim.x);
}

// The prime easy leaves of one query (pc_easy_primes).
__device__ __forceinline__ void easy_primes_wg(const pc_tables &T, const pc_query &Q, uint32_t wg,
                                               uint32_t nwg)
{
    __shared__ pc_s128 scr[EZ_T / 64];
    int64_t acc = 0;
    pc_easy_primes<EZ_T>(T, Q, wg, nwg, &acc);
    const pc_s128 s = pc_block_sum128<EZ_T>((pc_s128)acc, scr);
    if (threadIdx.x == 0 && s != 0)
        pc_atomic_add128(&Q.sums->s2e, s);
}

__global__ __launch_bounds__(EZ_T) void k_easy_primes(pc_tables T, pc_query Q)
{
    easy_primes_wg(T, Q, blockIdx.x, gridDim.x);
}

// The candidates, the prime leaves and S1 of a small query side by side: each
// is a chain of a few table reads on part of the chip, and one launch takes the
// place of three in a row (pi(10^9) 128 -> 109 us, pi(10^12) 209 -> 190).  A
// large query's kernels are faster apart, each with its own registers.
__global__ __launch_bounds__(EZ_T) void k_leaves(pc_tables T, pc_query Q, uint32_t neasy,
                                               uint32_t ns1)
{
    static_assert(EZ_T == LV_T, "workgroups of one size");
    if (blockIdx.x < neasy)
        easy_cands_wg(T, Q, blockIdx.x, neasy);
    else if (blockIdx.x < 2 * neasy)
        easy_primes_wg(T, Q, blockIdx.x - neasy, neasy);
    else
        s1_wg(T, Q, blockIdx.x - 2 * neasy, ns1);
}

hipError_t pc_launch_leaves(const pc_tables &T, const pc_query &Q, uint32_t neasy, uint32_t ns1,
                            hipStream_t s)
{
    k_leaves<<<2 * neasy + ns1, EZ_T, 0, s>>>(T, Q, neasy, ns1);
    return hipGetLastError();
}

hipError_t pc_launch_easy_cands(const pc_tables &T, const pc_query &Q, uint32_t nblocks,
                                hipStream_t s)
{
    k_easy_cands<<<nblocks, EZ_T, 0, s>>>(T, Q);
    return hipGetLastError();
}

hipError_t pc_launch_easy_primes(const pc_tables &T, const pc_query &Q, uint32_t nblocks,
                                 hipStream_t s)
{
    k_easy_primes<<<nblocks, EZ_T, 0, s>>>(T, Q);
    return hipGetLastError();
}

__global__ __launch_bounds__(LV_T) void k_prep(pc_prep_args A)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * LV_T + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * LV_T;
#pragma unroll
    for (int r = 0; r < 3; r++)
        for (uint64_t i = i0; i < A.n[r]; i += stride)
            A.dst[r][i] = A.src[r][i];
#pragma unroll
    for (int r = 0; r < 4; r++)
        for (uint64_t i = i0; i < A.nz[r]; i += stride)
            A.zero[r][i] = 0;
}

hipError_t pc_launch_prep(const pc_prep_args &A, hipStream_t s)
{
    uint64_t n = 1;
    for (int r = 0; r < 4; r++) {
        n = n < A.nz[r] ? A.nz[r] : n;
        if (r < 3)
            n = n < A.n[r] ? A.n[r] : n;
    }
    const uint64_t nb = (n + LV_T - 1) / LV_T;
    k_prep<<<(uint32_t)(nb < 1024 ? nb : 1024), LV_T, 0, s>>>(A);
    return hipGetLastError();
}

__global__ void k_fill_u64(uint64_t *p, uint64_t n, uint64_t v)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        p[i] = v;
}

hipError_t pc_launch_fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    uint64_t nb = (n + 255) / 256;
    if (nb > 65536)
        nb = 65536;
    k_fill_u64<<<(uint32_t)nb, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

// pi(x) and its parts from the partial sums (pc_combine_one), with the sums
// and the flags, into the host's memory: one word a thread.
__global__ __launch_bounds__(64) void k_combine(const pc_sums *S, pc_query Q, uint64_t kp2,
                                               const int32_t *err, pc_back *out)
{
    __shared__ pc_back b;
    static_assert(sizeof(pc_back) % 8 == 0, "copied as 64-bit words");
    if (threadIdx.x == 0) {
        b.sums = *S;
        pc_combine_one(b.sums, Q, kp2, &b.fin);
        for (int i = 0; i < 4; i++)
            b.err[i] = err[i];
    }
    __syncthreads();
    const uint64_t *const w = reinterpret_cast<const uint64_t *>(&b);
    for (uint32_t i = threadIdx.x; i < sizeof(pc_back) / 8; i += 64)
        reinterpret_cast<uint64_t *>(out)[i] = w[i];
}

hipError_t pc_launch_combine(const pc_sums *sums, const pc_query &Q, uint64_t kp2,
                             const int32_t *err, pc_back *out, hipStream_t s)
{
    k_combine<<<1, 64, 0, s>>>(sums, Q, kp2, err, out);
    return hipGetLastError();
}
