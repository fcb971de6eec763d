// Device check of the two quotients of the leaf kernels that take no exact
// remainder or only its low half, where they can go wrong: dividends at, just
// above and just below a multiple of the divisor.
//   pc_pi_quot_less1 (pc_leafwork.h): against a pi table whose entries number
//     the odd integers, so that the result tells the quotient's pair {2k - 1, 2k};
//     wrong only if it differs and the caller would not repeat it the exact way
//     (amb at or above PC_AMB);
//   pc_quot_off (pc_device.h): the quotient's offset in a segment.
// Built as a shared library by the package build; the test calls
// pc_leaf_quot_check() through ctypes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pc_leafwork.h"

namespace {

__device__ __forceinline__ uint64_t splitmix(uint64_t z)
{
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

constexpr uint32_t ENTRIES = 1u << 25; // 64 integers each: quotients below 2^31

__global__ void k_table(uint2 *tab)
{
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e < ENTRIES)
        tab[e] = make_uint2(0xFFFFFFFFu, 32u * e);
}

// out: 0 wrong pc_pi_quot_less1 with the table's 1/m, 1 with pc_rcp_f64's, 2 wrong
// pc_quot_off, 3 a quotient outside the segment taken as inside, 4 terms that the
// caller repeats (of those with a random remainder), 5 all of these
__global__ void k_check(const uint2 *tab, uint64_t n, uint64_t seed, unsigned long long *out)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t r0 = splitmix(seed ^ (4 * i)), r1 = splitmix(seed ^ (4 * i + 1));
        const uint64_t r2 = splitmix(seed ^ (4 * i + 2)), r3 = splitmix(seed ^ (4 * i + 3));
        const uint32_t kind = (uint32_t)r1 & 3; // remainder 0, m - 1, 1 or random
        uint32_t m = (uint32_t)(r0 >> (33 + ((r1 >> 2) & 31) % 28));
        m = m < 17 ? 17 : m;
        const uint32_t rem = kind == 0 ? 0 : kind == 1 ? m - 1 : kind == 2 ? 1 : (uint32_t)r3 % m;
        { // quotients 2 .. 2^31 - 2, the largest among them
            uint32_t q = (uint32_t)(r2 >> (33 + ((r1 >> 7) & 31) % 30));
            q = (r1 >> 12 & 63) == 0 ? 0x7FFFFFFEu - (uint32_t)(r2 & 7) : q < 2 ? 2 : q;
            q = q > 0x7FFFFFFEu ? 0x7FFFFFFEu : q;
            const uint64_t X = (uint64_t)q * m + rem;
            const uint32_t want = (q - 1) / 2 + 1;
            const double rp[2] = {1.0 / (double)m, pc_rcp_f64(m)};
            for (int k = 0; k < 2; k++) {
                uint32_t amb = 0xFFFFFFFFu;
                const uint32_t got = pc_pi_quot_less1(tab, (double)X, rp[k], true, &amb);
                if (amb >= PC_AMB && got != want)
                    atomicAdd(&out[k], 1ull);
                if (kind == 3 && m > 1000) {
                    atomicAdd(&out[5], 1ull);
                    if (amb < PC_AMB)
                        atomicAdd(&out[4], 1ull);
                }
            }
        }
        { // u < 2^48 (X up to 2^79), in a segment of 2^21 integers or next to it
            const uint64_t u = r2 >> (16 + ((r1 >> 18) & 47));
            const pc_u128 X = (pc_u128)u * m + rem;
            const double Xd = (double)X;
            const uint32_t span = 1966080;
            const uint32_t at = (r1 >> 40 & 3) == 0 ? 0 : (r1 >> 40 & 3) == 1 ? span - 1 : (uint32_t)r3 % span;
            const uint64_t lo = u < at ? 0 : u - at;
            bool in;
            const uint32_t off = pc_quot_off((uint32_t)X, Xd, m, (uint32_t)lo, 0.25 - (double)lo, span, &in);
            if (!in || off != u - lo)
                atomicAdd(&out[2], 1ull);
            // the next integer past the segment's end, and the last before its start
            if (u >= span) {
                const uint64_t l2 = u - span;
                (void)pc_quot_off((uint32_t)X, Xd, m, (uint32_t)l2, 0.25 - (double)l2, span, &in);
                if (in)
                    atomicAdd(&out[3], 1ull);
            }
            const uint64_t l3 = u + 1;
            (void)pc_quot_off((uint32_t)X, Xd, m, (uint32_t)l3, 0.25 - (double)l3, span, &in);
            if (in)
                atomicAdd(&out[3], 1ull);
        }
    }
}

} // namespace

extern "C" int pc_leaf_quot_check(uint64_t n, uint64_t seed, uint64_t *out6)
{
    uint2 *tab = nullptr;
    unsigned long long *d = nullptr;
    hipError_t e = hipMalloc(&tab, (size_t)ENTRIES * sizeof(uint2));
    if (e == hipSuccess)
        e = hipMalloc(&d, 6 * 8);
    if (e == hipSuccess)
        e = hipMemset(d, 0, 6 * 8);
    if (e == hipSuccess) {
        k_table<<<ENTRIES / 256, 256>>>(tab);
        k_check<<<4096, 256>>>(tab, n, seed, d);
        e = hipDeviceSynchronize();
    }
    if (e == hipSuccess)
        e = hipMemcpy(out6, d, 6 * 8, hipMemcpyDeviceToHost);
    (void)hipFree(tab);
    (void)hipFree(d);
    return (int)e;
}
