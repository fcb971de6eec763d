// The host planner (pc_host.hip) on a device that is host memory: allocations
// fail on demand, the table kernels run as plain loops and the others do
// nothing.  Each case makes a call fail part way and checks what the next call
// finds.  Usage: failing_calls <case>; prints OK.
#include "pc_host.hip"

#include "pc_leafrange.h"

static int g_fails = 0;
#define CHECK(cond, ...)                                  \
    do {                                                  \
        if (!(cond) && g_fails++ < 20) {                  \
            std::printf("FAIL %s:%d ", __FILE__, __LINE__); \
            std::printf(__VA_ARGS__);                     \
            std::printf("\n");                            \
        }                                                 \
    } while (0)

// --- the runtime: the allocation with g_fail_in others before it fails ---
static long g_fail_in = -1;
static bool g_fired = false;
static hipError_t take(void **p, size_t n)
{
    if (g_fail_in >= 0 && g_fail_in-- == 0) {
        g_fired = true;
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    *p = std::malloc(n);
    std::memset(*p, 0xEE, n);
    return hipSuccess;
}
extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return take(p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return take(p, n); }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)16; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)16; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)16; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

// --- the table kernels ---
static std::vector<int32_t> mulpf_to(uint64_t Y) // mu(n) lpf(n)
{
    std::vector<int32_t> v(Y + 1, 0), mu(Y + 1, 1), lpf(Y + 1, 0);
    for (uint64_t p = 2; p <= Y; p++)
        if (!lpf[p]) {
            for (uint64_t n = p; n <= Y; n += p) {
                if (!lpf[n])
                    lpf[n] = (int32_t)p;
                mu[n] = -mu[n];
            }
            for (uint64_t n = p * p; n <= Y; n += p * p)
                mu[n] = 0;
        }
    for (uint64_t n = 2; n <= Y; n++)
        v[n] = mu[n] * lpf[n];
    v[1] = INT32_MAX;
    return v;
}
static bool prime_to_wheel(uint64_t n)
{
    return n % 2 && n % 3 && n % 5 && n % 7 && n % 11 && n % 13;
}
hipError_t pc_launch_base_primes(uint32_t *, uint32_t *nbase, hipStream_t) { *nbase = 1; return hipSuccess; }
hipError_t pc_launch_pitab(uint64_t nent, const uint32_t *, uint32_t, uint32_t *, uint32_t *, uint2 *tab,
                           uint32_t *primes, uint64_t *, uint32_t *, hipStream_t)
{
    std::vector<uint8_t> comp(64 * nent, 0);
    uint32_t k = 0, odd = 0;
    primes[0] = 0;
    for (uint64_t n = 2; n < comp.size(); n++) {
        if (comp[n])
            continue;
        primes[++k] = (uint32_t)n;
        for (uint64_t m = n * n; m < comp.size(); m += n)
            comp[m] = 1;
    }
    for (uint64_t e = 0; e < nent; e++) {
        uint32_t w = 0;
        for (uint32_t j = 0; j < 32; j++)
            w |= (64 * e + 2 * j + 1 > 1 && !comp[64 * e + 2 * j + 1] ? 1u : 0u) << j;
        tab[e] = make_uint2(w, odd);
        odd += (uint32_t)__builtin_popcount(w);
    }
    return hipSuccess;
}
hipError_t pc_launch_recip(const uint32_t *p, uint64_t *r, double *d, uint32_t n, hipStream_t)
{
    for (uint32_t k = 1; k <= n; k++) {
        r[k] = pc_recip(p[k]);
        d[k] = 1.0 / p[k];
    }
    return hipSuccess;
}
hipError_t pc_launch_mulpf(const uint32_t *, uint32_t, uint64_t Y, int32_t *out, hipStream_t)
{
    const std::vector<int32_t> v = mulpf_to(Y);
    std::copy(v.begin(), v.end(), out);
    return hipSuccess;
}
hipError_t pc_launch_mulpfw(const pc_tables &T, uint64_t n, int32_t *out, hipStream_t)
{
    uint64_t m = 0;
    for (uint64_t k = 0; k < n; k++) {
        do
            m++;
        while (!prime_to_wheel(m));
        out[k] = T.mulpf[m];
    }
    return hipSuccess;
}
hipError_t pc_launch_count_nonzero(const int32_t *a, uint64_t n, unsigned long long *out, hipStream_t)
{
    for (uint64_t i = 1; i <= n; i++)
        *out += a[i] != 0;
    return hipSuccess;
}
hipError_t pc_launch_lookup(const uint2 *tab, const uint64_t *in, uint32_t n, uint64_t *out, hipStream_t)
{
    for (uint32_t i = 0; i < n; i++)
        out[i] = pc_pi_lookup(tab, in[i]);
    return hipSuccess;
}
hipError_t pc_launch_fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t)
{
    std::fill(p, p + n, v);
    return hipSuccess;
}
hipError_t pc_launch_batch_finish(const pc_query *Q, const uint32_t *, const uint32_t *, uint32_t, uint32_t nq,
                                  pc_final *out, hipStream_t)
{
    for (uint32_t i = 0; i < nq; i++) { // any value that tells the queries apart
        out[i] = pc_final{};
        out[i].pi = Q[i].x / 3;
        out[i].ok = 1;
    }
    return hipSuccess;
}
hipError_t pc_launch_seed(const pc_tables &, uint32_t, uint64_t, uint32_t nb, uint32_t, uint64_t, int64_t *,
                          uint64_t *out, int32_t *err, hipStream_t)
{
    std::fill(out, out + nb + 1, 77);
    *err |= 16; // an inconsistency found on the device
    return hipSuccess;
}
// --- and those that no case looks at ---
#define NOP(name, ...) hipError_t name(__VA_ARGS__) { return hipSuccess; }
using PT = const pc_tables &;
using PQ = const pc_query &;
using U = uint32_t;
using UP = const uint32_t *;
NOP(pc_launch_presieve, uint8_t *, hipStream_t)
NOP(pc_launch_wheel, U, UP, U *, U, U *, U *, hipStream_t)
NOP(pc_launch_s1, PT, PQ, U, hipStream_t)
NOP(pc_launch_leaf_setup, PT, PQ, hipStream_t)
NOP(pc_launch_leaves, PT, PQ, U, U, hipStream_t)
NOP(pc_launch_easy_cands, PT, PQ, U, hipStream_t)
NOP(pc_launch_easy_primes, PT, PQ, U, hipStream_t)
NOP(pc_launch_prep, const pc_prep_args &, hipStream_t)
NOP(pc_launch_plan, const pc_plan_args &, hipStream_t)
NOP(pc_launch_sieve, const pc_sieve_args &, U, U, int, hipStream_t)
NOP(pc_launch_sieve_tiny, PT, PQ, hipStream_t)
NOP(pc_launch_scan, const pc_scan_args &, int, hipStream_t)
NOP(pc_launch_combine, const pc_sums *, PQ, uint64_t, const int32_t *, pc_back *, hipStream_t)
NOP(pc_launch_batch_setup, PT, const pc_query *, UP, UP, U, UP, UP, U, U, hipStream_t)
NOP(pc_launch_batch_easy, PT, const pc_query *, UP, UP, U, hipStream_t)
NOP(pc_launch_batch_out, const pc_final *, const uint64_t *, U, const int32_t *, uint64_t *, hipStream_t)
NOP(pc_launch_scatter_u64, const ulonglong2 *, uint64_t, uint64_t *, hipStream_t)

// --- cases ---

// A table whose growth runs out of memory is not taken for built afterwards.
static void ensure_all(uint64_t pi, uint64_t recip, uint64_t y)
{
    ensure_pi(pi);
    ensure_mulpf(y);
    ensure_recip(recip);
    ensure_wheel(kWheelC);
    ensure_mulpfw(y);
}

static void check_tables(uint64_t pi, uint64_t recip, uint64_t y)
{
    Tables &T = g_T;
    CHECK(T.pi_limit >= pi && T.recip_n >= recip && T.y_limit >= y && T.w_limit >= y, "limits");
    CHECK(T.pitab.p && T.primes.p && T.recip.p && T.rcpd.p && T.mulpf.p && T.mulpfw.p, "a table is gone");
    if (g_fails)
        return;
    CHECK(T.pitab.cap >= (T.pi_limit / 64 + 1) * 8, "pi table short of its limit");
    CHECK(T.recip.cap >= (T.recip_n + 1) * 8 && T.rcpd.cap >= (T.recip_n + 1) * 8, "reciprocals short");
    CHECK(T.mulpf.cap >= (T.y_limit + 1) * 4, "mu*lpf short of its limit");
    const uint64_t at[3][2] = {{10, 4}, {1000000, 78498}, {999983, 78498}};
    for (auto &v : at)
        CHECK(pc_pi_lookup(ptr<uint2>(T.pitab), v[0]) == v[1], "pi(%llu)", (unsigned long long)v[0]);
    for (uint64_t k : {(uint64_t)1, (uint64_t)100, recip})
        CHECK(ptr<uint64_t>(T.recip)[k] == pc_recip(ptr<uint32_t>(T.primes)[k]), "1 / p_%llu", (unsigned long long)k);
    const std::vector<int32_t> v = mulpf_to(y);
    uint64_t k = 0;
    for (uint64_t n = 1; n <= y; n++) {
        CHECK(ptr<int32_t>(T.mulpf)[n] == v[n], "mu lpf(%llu)", (unsigned long long)n);
        if (prime_to_wheel(n))
            CHECK(ptr<int32_t>(T.mulpfw)[k++] == v[n], "mu lpf by the wheel at %llu", (unsigned long long)n);
    }
}

static void case_tables()
{
    init_stream();
    for (long k = 0;; k++) {
        drop_tables(true);
        ensure_all(1 << 20, 200, 1000);
        g_fired = false;
        g_fail_in = k;
        bool threw = false;
        try {
            ensure_all(9000000, 300000, 2500000);
        } catch (const pc_error &e) {
            threw = true;
            CHECK(e.st == PC_ENOMEM, "status %d", (int)e.st);
        }
        g_fail_in = -1;
        CHECK(threw == g_fired, "allocation %ld", k);
        ensure_all(1 << 20, 200, 1000);
        check_tables(1 << 20, 200, 1000);
        if (g_fails)
            std::printf("after allocation %ld failed\n", k);
        if (!g_fired || g_fails)
            return;
    }
}

// A batch that runs out of memory leaves no queries in the round's slot and no
// size of a buffer that it no longer has.
static void case_batch()
{
    const std::vector<uint64_t> few{3000000, 5000000}, many{9000001, 8000000, 7000000, 6000000,
                                                            5500000, 4000000, 3500000};
    std::vector<uint64_t> out(16);
    const pc_config cfg{0, 0, 0, 0, PC_FLAG_NO_GRAPH, 0, 0, 0};
    for (long k = 0;; k++) {
        pc_shutdown();
        CHECK(pc_pi_count_batch_ex(many.data(), 1, &cfg, out.data()) == PC_OK, "%s", pc_last_error());
        g_fired = false;
        g_fail_in = k;
        const pc_status st = pc_pi_count_batch_ex(many.data(), many.size(), &cfg, out.data());
        g_fail_in = -1;
        CHECK((st != PC_OK) == g_fired, "allocation %ld: %s", k, pc_last_error());
        out.assign(16, 1);
        CHECK(pc_pi_count_batch_ex(few.data(), few.size(), &cfg, out.data()) == PC_OK, "%s",
              pc_last_error());
        for (size_t i = 0; i < out.size(); i++)
            CHECK(out[i] == (i < few.size() ? few[i] / 3 : 1), "allocation %ld: result %zu", k, i);
        CHECK(g_slot.R.empty(), "allocation %ld: queries left", k);
        if (!g_fired || g_fails)
            return;
    }
}

// Seeds that the device found inconsistent are not written out.
static void case_seeds()
{
    for (uint32_t b_hi : {1000u, 600000u}) { // through pinned memory, and past it (4 MiB)
        std::vector<uint64_t> out(b_hi - 5, 1);
        CHECK(pc_phi_seed(1000000, 6, b_hi, out.data()) == PC_EINTERNAL, "b_hi %u: status", b_hi);
        CHECK(std::count(out.begin(), out.end(), 1) == (long)out.size(), "b_hi %u: written", b_hi);
    }
}

int main(int argc, char **argv)
{
    const std::string c = argc > 1 ? argv[1] : "";
    if (c == "tables")
        case_tables();
    else if (c == "batch")
        case_batch();
    else if (c == "seeds")
        case_seeds();
    else
        CHECK(false, "no such case");
    if (!g_fails)
        std::printf("OK\n");
    std::fflush(stdout);
    std::_Exit(g_fails ? 1 : 0); // (no static destructors: the device is not a real one)
}
