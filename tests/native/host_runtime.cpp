// Host-only driver for libqs's handling of its pinned result buffers and launch
// sizes: this program defines every HIP entry point that the library imports
// (an executable's symbols come before those of the shared objects it loads),
// so that the library's host code runs without a device.  Launches and waits
// are recorded, launches fail on demand, and operator new throws on demand.
// Built and run by tests/test_host_runtime.py; prints "ok <case>" and exits 0.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "qs.h"

namespace {
struct Event {
    char kind;  // 'L' launch, 'S' wait for a stream, 'H' / 'F' pinned allocation / release, 'M' copy, 'A' allocation
    void *stream;
    uint64_t threads;  // launch: threads; allocation: bytes
};
std::vector<Event> events;
long fail_launch = -1;  // launches until one fails
bool fail_new = false;
int last_error = 0;

void note(char kind, void *stream, uint64_t threads = 0)
{
    const bool f = fail_new;
    fail_new = false;
    events.push_back({kind, stream, threads});
    fail_new = f;
}
// Events of a kind on a stream after position from (stream null: any).
int count(char kind, void *stream, size_t from)
{
    int c = 0;
    for (size_t i = from; i < events.size(); ++i)
        c += events[i].kind == kind && (!stream || events[i].stream == stream);
    return c;
}
size_t first(char kind, size_t from)
{
    size_t i = from;
    while (i < events.size() && events[i].kind != kind) ++i;
    return i;
}
}  // namespace

void *operator new(size_t n)
{
    if (fail_new) throw std::bad_alloc();
    void *p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new[](size_t n) { return operator new(n); }
void operator delete(void *p) noexcept { free(p); }
void operator delete[](void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
void operator delete[](void *p, size_t) noexcept { free(p); }

extern "C" {
struct Dim3 {
    uint32_t x, y, z;
};
static struct {
    Dim3 grid, block;
    size_t shared;
    void *stream;
} config;
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream)
{
    config = {grid, block, shared, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream)
{
    *grid = config.grid;
    *block = config.block;
    *shared = config.shared;
    *stream = config.stream;
    return 0;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { note('S', nullptr); return 0; }
int hipEventCreate(void **e) { *e = nullptr; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0; return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipMalloc(void **p, size_t n) { note('A', nullptr, n); *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
const char *hipGetErrorString(int) { return "error"; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int hipGetSymbolAddress(void **, const void *) { return 1; }
int hipHostMalloc(void **p, size_t n, unsigned) { note('H', nullptr); *p = calloc(1, n); return 0; }
int hipHostFree(void *p) { note('F', nullptr); free(p); return 0; }
int hipLaunchKernel(const void *, Dim3 grid, Dim3 block, void **, size_t, void *stream)
{
    const uint64_t threads = (uint64_t)grid.x * block.x;
    if (fail_launch >= 0 && fail_launch-- == 0) return last_error = 719;
    note('L', stream, threads);
    return 0;
}
int hipMemcpyAsync(void *, const void *, size_t, int, void *stream) { note('M', stream); return 0; }
int hipStreamSynchronize(void *stream) { note('S', stream); return 0; }
}

#define CHECK(cond)                                                           \
    do {                                                                      \
        if (!(cond)) {                                                        \
            printf("%s:%d: %s (%s)\n", __FILE__, __LINE__, #cond, qs_last_error()); \
            return 1;                                                         \
        }                                                                     \
    } while (0)

static void *const A = (void *)0xA000, *const B = (void *)0xB000;

static qs_state handle(int n, void *stream)
{
    qs_state s = nullptr;
    return qs_alloc(n, QS_C64, nullptr, 0, stream, &s) == QS_OK ? s : nullptr;
}
static int32_t *diagonal(int n)
{
    void *p = nullptr;
    hipMalloc(&p, sizeof(int32_t) << n);
    memset(p, 0, sizeof(int32_t) << n);
    return (int32_t *)p;
}

// A call that fails half-way leaves launches behind that may still write the
// handle's pinned buffer: their stream is waited for before the buffer serves
// anything else, also when the handle has moved to another stream since.
static int failed_call(bool switch_stream)
{
    const int n = 16, p = 3;
    const double tzz[p] = {0.1, 0.2, 0.3}, tx[p] = {-0.9, -0.6, -0.3};
    int32_t *diag = diagonal(n);
    double e = 0, nrm = 0, g[2 * p];
    qs_state s = handle(n, A);
    CHECK(s && qs_adjoint_grad(s, diag, 40, p, tzz, tx, nullptr, 0, &e, g, g + p) == QS_OK);
    fail_launch = 7;
    CHECK(qs_adjoint_grad(s, diag, 40, p, tzz, tx, nullptr, 0, &e, g, g + p) == QS_ERR_HIP);
    fail_launch = -1;
    const size_t at = events.size();
    if (switch_stream) {
        CHECK(qs_set_stream(s, B) == QS_OK);
        CHECK(qs_free(s) == QS_OK);  // the buffer goes back to the pool
        CHECK(count('S', A, at) >= 1);
        qs_state t = handle(n, B);  // and from there to another handle
        CHECK(t && qs_expect(t, diag, &e, &nrm) == QS_OK && qs_free(t) == QS_OK);
        CHECK(count('H', nullptr, at) == 0);
    } else {
        // the next call clears its flags in the buffer from the host
        uint64_t shot;
        CHECK(qs_sample(s, 1, 1, &shot, 0) == QS_OK);
        CHECK(first('S', at) < first('L', at));
        const size_t then = events.size();
        CHECK(qs_set_stream(s, B) == QS_OK);  // nothing left to wait for
        CHECK(events.size() == then);
        CHECK(qs_free(s) == QS_OK);
    }
    return 0;
}

// No exception leaves the library: without host memory for the pool of pinned
// buffers the results go through pageable memory.
static int no_memory()
{
    const int n = 14;
    int32_t *diag = diagonal(n);
    double e = 0, nrm = 0;
    uint64_t out[64];
    qs_state s = handle(n, A);
    CHECK(s);
    fail_new = true;
    int threw = 0;
    qs_status st[3] = {};
    try {
        st[0] = qs_expect(s, diag, &e, &nrm);
        st[1] = qs_sample(s, 1, 64, out, 0);
        st[2] = qs_cost_histogram(s, diag, 64, out, 0);
    } catch (...) {
        threw = 1;
    }
    fail_new = false;
    CHECK(!threw);
    CHECK(st[0] == QS_OK && st[1] == QS_OK && st[2] == QS_OK);
    CHECK(count('H', nullptr, 0) == 0);
    CHECK(qs_free(s) == QS_OK);
    return 0;
}

// Launches stay below 2^32 threads, the runtime's limit, for every number of
// shots of a small state.
static int many_shots()
{
    uint64_t *out = (uint64_t *)0x100000;  // never touched: the shots would go to device memory
    qs_state s = handle(5, A);
    CHECK(s);
    for (const int64_t shots : {(int64_t)1, (int64_t)1 << 20, ((int64_t)1 << 32) + 5, (int64_t)1 << 39}) {
        const size_t at = events.size();
        CHECK(qs_sample(s, 1, shots, out, 1) == QS_OK);
        CHECK(count('L', A, at) >= 1);
        for (size_t i = at; i < events.size(); ++i) CHECK(events[i].kind != 'L' || events[i].threads < ((uint64_t)1 << 32));
    }
    CHECK(qs_free(s) == QS_OK);
    return 0;
}

// A histogram with more bins than a workgroup's LDS holds has one row of sums:
// one thread per bin each to clear it and to write it out, not dozens.
static int many_bins()
{
    const int n = 10, nbins = 1 << 20;
    int32_t *diag = diagonal(n);
    uint64_t *out = (uint64_t *)0x100000;  // never touched: the masses would go to device memory
    qs_state s = handle(n, A);
    CHECK(s && qs_cost_histogram(s, diag, nbins, out, 1) == QS_OK);
    uint64_t threads = 0;
    for (const Event &e : events) threads += e.kind == 'L' ? e.threads : 0;
    CHECK(threads <= 2ull * nbins + (1u << 16));
    CHECK(qs_free(s) == QS_OK);
    return 0;
}

// Every size, precision and layout, angles in tangent form and beyond: each pass
// finds a kernel.
static int every_plan()
{
    void *const psi = (void *)0x10000000, *const lam = (void *)0x20000000;  // never touched
    const int32_t *diag = (const int32_t *)0x30000000;
    for (int prec : {(int)QS_C64, (int)QS_C128, QS_C64 | QS_SYM, QS_C128 | QS_SYM})
        for (int n = 1; n <= 35; ++n) {
            const size_t bytes = qs_state_bytes(n, prec);
            if (!bytes) continue;
            qs_state s = nullptr;
            CHECK(qs_alloc(n, prec, psi, bytes, A, &s) == QS_OK);
            for (int p = 1; p <= 3; ++p)
                for (double large : {0.0, 2.4}) {
                    const double tzz[3] = {0.1, 0.2, 0.3}, tx[3] = {large ? large : -0.9, large ? large : -0.6, -0.3};
                    double e = 0, nrm = 0, g[6];
                    CHECK(qs_forward(s, diag, 300, p, tzz, tx, &e, &nrm) == QS_OK);
                    CHECK(n < 2 || qs_adjoint_grad(s, diag, 300, p, tzz, tx, lam, bytes, &e, g, g + 3) == QS_OK);
                    CHECK(qs_apply_mixer(s, tx[1]) == QS_OK);
                }
            CHECK(qs_free(s) == QS_OK);
        }
    return 0;
}

// The partial sums of a deep batch are reduced in groups of rounds: its working
// memory beside states, steps and phase tables stays bounded.
static int deep_batch()
{
    const int n = 22, p = 6000, ne = n * (n - 1) / 2;
    std::vector<int32_t> w(ne, 3);
    const qs_circuit c = {n, p, w.data()};
    qs_batch b = nullptr;
    CHECK(qs_batch_create(1, &c, QS_C64, A, &b) == QS_OK);
    std::vector<double> tzz(p, 0.1), tx(p, -0.2), gz(p), gx(p);
    double e = 0;
    const size_t at = events.size();
    CHECK(qs_batch_forward_grad(b, tzz.data(), tx.data(), &e, gz.data(), gx.data()) == QS_OK);
    for (size_t i = at; i < events.size(); ++i) CHECK(events[i].kind != 'A' || events[i].threads <= (64u << 20));
    CHECK(qs_batch_free(b) == QS_OK);
    return 0;
}

int main(int argc, char **argv)
{
    const std::string which = argc > 1 ? argv[1] : "";
    int rc = 2;
    if (which == "switched_stream") rc = failed_call(true);
    else if (which == "same_stream") rc = failed_call(false);
    else if (which == "no_memory") rc = no_memory();
    else if (which == "many_shots") rc = many_shots();
    else if (which == "many_bins") rc = many_bins();
    else if (which == "deep_batch") rc = deep_batch();
    else if (which == "every_plan") rc = every_plan();
    if (rc == 0) printf("ok %s\n", which.c_str());
    return rc;
}
