// The library's host code over a HIP runtime that launches nothing: every
// runtime call the library makes is defined here and recorded, so that what
// it allocates, announces and launches can be checked for any size on a
// machine without a GPU (tests/test_host_runtime.py).  Usage: driver CHECK;
// exit status 0 = every expectation of that check held.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <set>
#include <string>
#include <utility>
#include <vector>

#include "exemcl.h"

// ---------------------------------------------------------------------------
// The runtime.
// ---------------------------------------------------------------------------
namespace fake {
struct Launch {
    std::string name;
    dim3 grid, block;
    size_t lds;
};
std::vector<Launch> launches;
std::vector<size_t> allocs;                      // sizes asked of the pool
std::map<const void *, std::string> &kernels() {  // host stub -> device name (filled before main)
    static std::map<const void *, std::string> m;
    return m;
}
hipError_t last = hipSuccess;                    // until hipGetLastError
std::set<std::pair<int, const void *>> announced;  // (device, kernel) with more than 64 KiB of LDS
int device = 0;
std::string fail_kernel;                         // launches of kernels with this in their name fail
uintptr_t next_ptr = uintptr_t(1) << 40;
size_t pool_left = SIZE_MAX;

hipError_t check(const std::string &name, const void *f, dim3 g, dim3 b, size_t lds) {
    if (!fail_kernel.empty() && name.find(fail_kernel) != std::string::npos) return hipErrorLaunchFailure;
    // a grid's extents are 32 bits of work-items; y and z 16 bits of workgroups
    if ((uint64_t)g.x * b.x > UINT32_MAX || g.x < 1 || g.y < 1 || g.y > 65535 || g.z != 1) return hipErrorInvalidConfiguration;
    if ((uint64_t)b.x * b.y * b.z > 1024 || lds > 160 * 1024) return hipErrorInvalidConfiguration;
    if (lds > 64 * 1024 && !announced.count({device, f})) return hipErrorInvalidValue;
    return hipSuccess;
}
hipError_t launch(const void *f, dim3 g, dim3 b, size_t lds) {
    const std::string name = kernels().count(f) ? kernels()[f] : "?";
    launches.push_back({name, g, b, lds});
    const hipError_t e = check(name, f, g, b, lds);
    if (e != hipSuccess) last = e;
    return e;
}
}  // namespace fake

extern "C" {
void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    fake::kernels()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
    cfg_grid = g, cfg_block = b, cfg_lds = lds, cfg_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st) {
    *g = cfg_grid, *b = cfg_block, *lds = cfg_lds, *st = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t) {
    return fake::launch(f, g, b, lds);
}
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t, hipEvent_t, hipEvent_t, int) {
    return fake::launch(f, g, b, lds);
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int) {
    fake::announced.insert({fake::device, f});
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t lds) {
    *n = lds > 80 * 1024 ? 1 : 2;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = fake::device;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;  // compute units
    return hipSuccess;
}
hipError_t hipMemPoolCreate(hipMemPool_t *p, const hipMemPoolProps *) {
    *p = (hipMemPool_t)0x10;
    return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void **p, size_t bytes, hipMemPool_t, hipStream_t) {
    if (bytes > fake::pool_left) return hipErrorOutOfMemory;
    fake::allocs.push_back(bytes);
    *p = (void *)fake::next_ptr;
    fake::next_ptr += (bytes + 4095) / 4096 * 4096;
    return hipSuccess;
}
hipError_t hipFreeAsync(void *, hipStream_t) { return hipSuccess; }
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = fake::last;
    fake::last = hipSuccess;
    return e;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    *p = malloc(bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)0x20;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = (hipEvent_t)0x30;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.0f;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    *p = (void *)(uintptr_t(1) << 45);
    return hipSuccess;
}
}

// ---------------------------------------------------------------------------
// The checks.
// ---------------------------------------------------------------------------
static int failures = 0;
static void expect(bool ok, const char *what, const std::string &at = "") {
    if (ok) return;
    if (++failures <= 20) fprintf(stderr, "FAILED: %s %s\n", what, at.c_str());
}

static void *const kV = (void *)0x1000;
static int32_t *const kI = (int32_t *)0x2000;
static float *const kF = (float *)0x3000;

// A stream of its own for every call: no block kept from another one.
static void *fresh_stream() {
    static uintptr_t s = 0x100000;
    return (void *)(s += 0x100);
}

// Launch sizes.  Calls whose staging or evaluation takes more workgroups than
// a grid's 32 bits of work-items hold in one extent.
static void check_grids() {
    struct Call { int64_t n, d, l, k; int prec; const char *what; };
    const Call calls[] = {
        {1000000, 1536, 275000, 2, EXEMCL_BF16, "2^23 workgroups of 512: long rows"},
        {1000, 20, 40000000, 32, EXEMCL_FP16, "2^25 tiles of two wavefronts, 16 bits"},
        {1000, 3, 36000000, 32, EXEMCL_FP32, "2^25 tiles of two wavefronts, fp32"},
        {1000, 3, 40, 40000000, EXEMCL_FP32, "one set group's tiles"},
    };
    for (const Call &c : calls)
        expect(exemplar_eval(kV, c.n, c.d, kI, c.l, c.k, c.prec, kF, fresh_stream()) == EXEMCL_OK, c.what);
    setenv("EXEMCL_PERSIST", "0", 1);
    expect(exemplar_eval(kV, 40000000, 300, kI, 4000, 1, EXEMCL_FP32, kF, fresh_stream()) == EXEMCL_OK, "plain grid");
    unsetenv("EXEMCL_PERSIST");
    expect(exemplar_gain((float *)kV, INT32_MAX, 3, kI, 2, kI, 2, kF, fresh_stream()) == EXEMCL_OK, "cache of 2^31 points");
}

// Every device is told of a kernel's LDS before the kernel's first launch on it.
static void check_devices() {
    for (int dev : {0, 1, 0, 5}) {
        fake::device = dev;
        for (int64_t d : {3, 40, 100, 300, 512, 600, 1000, 1536})
            for (int prec : {EXEMCL_FP32, EXEMCL_FP16, EXEMCL_BF16})
                for (int64_t n : {900, 7000, 150000})
                    for (int64_t l : {5, 3000})
                        expect(exemplar_eval(kV, n, d, kI, l, 3, prec, kF, fresh_stream()) == EXEMCL_OK, "eval on device",
                               std::to_string(dev) + " d " + std::to_string(d) + " precision " + std::to_string(prec));
        for (int64_t d : {3, 100, 512, 600}) {
            const std::string at = std::to_string(dev) + " d " + std::to_string(d);
            expect(exemplar_gain((float *)kV, 7000, d, kI, 40, kI, 50, kF, fresh_stream()) == EXEMCL_OK, "gain on device", at);
            expect(exemplar_greedy((float *)kV, 20000, d, 3, kI, kF, fresh_stream()) == EXEMCL_OK, "greedy on device", at);
        }
    }
}

// A block whose count of workgroups could not be cleared is no block for a
// later call on its stream.
static void check_counter() {
    void *st = fresh_stream();
    fake::fail_kernel = "zero_kernel";
    expect(exemplar_eval(kV, 1000, 8, kI, 16, 5, EXEMCL_FP32, kF, st) == EXEMCL_EDEVICE, "the failed launch is reported");
    fake::fail_kernel = "";
    fake::launches.clear();
    const size_t before = fake::allocs.size();
    expect(exemplar_eval(kV, 1000, 8, kI, 16, 5, EXEMCL_FP32, kF, st) == EXEMCL_OK, "the next call");
    expect(fake::allocs.size() == before + 1, "a block of its own");
    expect(fake::launches.size() == 2 && fake::launches[0].name.find("zero_kernel") != std::string::npos,
           "its count cleared, then one launch");
    fake::launches.clear();
    expect(exemplar_eval(kV, 1000, 8, kI, 16, 5, EXEMCL_FP32, kF, st) == EXEMCL_OK, "a third call");
    expect(fake::allocs.size() == before + 1 && fake::launches.size() == 1, "the kept block, one launch");
}

// EXEMCL_WORKSPACE_LIMIT.  A call that is accepted never holds more than the
// limit (the 256 bytes behind a block, where a count is kept, aside), and
// every limit under which fp32 tiles of 4 bytes per coordinate fit is
// accepted, whatever the present tiles need.
struct Call {
    enum Kind { EVAL, GAIN, GREEDY, STREAMED } kind;
    int64_t n, d, l, k;
    int prec;
    std::string text() const {
        static const char *names[] = {"eval", "gain", "greedy", "streamed"};
        return std::string(names[kind]) + " n " + std::to_string(n) + " d " + std::to_string(d) + " l " +
               std::to_string(l) + " k " + std::to_string(k) + " precision " + std::to_string(prec);
    }
};

static int run(const Call &c, int64_t limit, int64_t *held) {
    static std::vector<float> V, out;
    static std::vector<int32_t> sets;
    setenv("EXEMCL_WORKSPACE_LIMIT", std::to_string(limit).c_str(), 1);
    fake::allocs.clear();
    fake::launches.clear();
    int rc = -1;
    void *st = fresh_stream();
    if (c.kind == Call::EVAL) rc = exemplar_eval(kV, c.n, c.d, kI, c.l, c.k, c.prec, kF, st);
    if (c.kind == Call::GAIN) rc = exemplar_gain((float *)kV, c.n, c.d, kI, c.k, kI, c.l, kF, st);
    if (c.kind == Call::GREEDY) rc = exemplar_greedy((float *)kV, c.n, c.d, c.k, kI, kF, st);
    if (c.kind == Call::STREAMED) {  // reads host memory
        V.resize(std::max<size_t>(V.size(), (size_t)(c.n * c.d)));
        out.resize(std::max<size_t>(out.size(), (size_t)c.l));
        sets.assign((size_t)(c.l * c.k), 0);
        rc = exemplar_eval_streamed(V.data(), c.n, c.d, sets.data(), c.l, c.k, c.prec, 0, out.data(), st);
    }
    unsetenv("EXEMCL_WORKSPACE_LIMIT");
    *held = 0;
    for (size_t b : fake::allocs) *held += (int64_t)b - 256;
    return rc;
}

// What a call needs with fp32 tiles of 4 bytes per coordinate: blocks of 8
// coordinates and 32 sets up to d = 256, of 16 and 16 above, whole counts of
// blocks of which some are rounded up, a partial sum per wavefront.
static int64_t up(int64_t x) { return (x + 255) / 256 * 256; }
static int64_t need(const Call &c) {
    const int64_t n = c.n, d = c.d, k = c.k, tm = d <= 256 ? 32 : 16;
    int64_t blocks = tm == 32 ? (d + 7) / 8 : (d + 15) / 16;
    for (int64_t b : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 13, 14, 16, 20, 24, 28, 32})
        if (b >= blocks) {
            blocks = b;
            break;
        }
    const int64_t tile = (blocks <= 4 && tm == 32 ? 256 : 128) + blocks * 1024;
    const int64_t waves = blocks <= 8 && tm == 32 ? 4 : 8, rows = waves * (tm == 16 ? 16 : blocks <= 16 ? 64 : 32);
    const int64_t ld = d > 8 ? (d + 3) / 4 * 4 : d, copy = ld == d ? 0 : up(n * ld * 4);
    auto work = [&](int64_t points, int64_t groups, int64_t members) {
        return up(up((points + rows - 1) / rows * waves * groups * tm * 4) + groups * members * tile);
    };
    if (c.kind == Call::EVAL) return copy + work(n, 1, k);
    if (c.kind == Call::GAIN) return copy + up(up(n * 4) + (k + tm - 1) / tm * tile) + work(n, 1, 1);
    if (c.kind == Call::GREEDY) {
        const int64_t nb = std::min<int64_t>(1024, (n + 4095) / 4096);
        return copy + up(n * 4) + up(n) + 3 * up(n * 4) + up(tile) + 2 * up(nb * 4) + work(n, 1, 1);
    }
    const int64_t R = (std::min(n, (int64_t(64) << 20) / (ld * 4)) + rows - 1) / rows * rows, ne = c.l * k;
    const int64_t lds = (d + 3) / 4 * 4;
    return 2 * up(R * lds * 4) + up(ne * lds * 4) + up(ne * 4) + up(c.l * 8) + up(c.l) + up(c.l * 4) +
           work(R, (c.l + tm - 1) / tm, k);
}

static void check_limits() {
    std::vector<Call> calls;
    for (int64_t d : {3, 8, 20, 21, 52, 100, 129, 170, 197, 256, 257, 300, 353, 449, 512})
        for (int64_t n : {1, 60, 1000, 10000, 40000}) {
            for (int64_t k : {1, 40, 900}) {
                calls.push_back({Call::EVAL, n, d, 200, k, EXEMCL_FP32});
                calls.push_back({Call::GAIN, n, d, 300, k, EXEMCL_FP32});
                if (n <= 1000) calls.push_back({Call::STREAMED, n, d, 33, k, EXEMCL_FP32});
            }
            calls.push_back({Call::GREEDY, n, d, 0, std::min<int64_t>(n, 3), EXEMCL_FP32});
        }
    for (const Call &c : calls) {
        int64_t held = 0;
        const int64_t least = need(c);
        expect(run(c, least, &held) == EXEMCL_OK, "accepted under the limit it needs", c.text() + " limit " + std::to_string(least));
        for (double f : {0.5, 0.9, 1.0, 1.01, 1.1, 1.3, 1.7, 2.0, 3.0, 10.0}) {
            const int64_t limit = (int64_t)(f * (double)least);
            const int rc = run(c, limit, &held);
            expect(rc == EXEMCL_OK || rc == EXEMCL_ENOMEM, "status", c.text());
            expect(held <= limit, "held at most the limit", c.text() + " limit " + std::to_string(limit) + " held " + std::to_string(held));
            expect(rc == EXEMCL_OK || fake::launches.empty(), "nothing queued when refused", c.text());
        }
    }
    // no bytes for what is not there: a copy of fp32 rows that are read in
    // place, more partial sums than are written
    expect(exemplar_eval_noalloc(kV, 170000, 101, kI, 40, 3, EXEMCL_FP32, kF, nullptr) == EXEMCL_OK, "rows read in place");
    int64_t ws = 0;
    expect(exemplar_plan(20000, 1536, 4096, 16, EXEMCL_BF16, nullptr, &ws) == EXEMCL_OK && ws < 625 * 4096 * 4 + 2048 * (3200 * 49),
           "long rows: a partial sum per 32 points");
    // the other plans, and what is reported
    for (int prec : {EXEMCL_FP32, EXEMCL_FP16, EXEMCL_BF16})
        for (int64_t d : {1, 2, 3, 16, 17, 100, 128, 256, 512, 513, 1000, 1536})
            for (int64_t n : {1, 1000, 7000, 100000})
                for (int64_t l : {1, 40, 4096})
                    for (int64_t k : {1, 8, 32}) {
                        const Call c{Call::EVAL, n, d, l, k, prec};
                        int64_t held = 0, ws = 0;
                        expect(exemplar_plan(n, d, l, k, prec, nullptr, &ws) == EXEMCL_OK, "plan");
                        expect(run(c, INT64_MAX, &held) == EXEMCL_OK && held <= ws, "the plan's bytes hold the call", c.text());
                        expect(run(c, ws, &held) == EXEMCL_OK && held <= ws, "the plan's bytes suffice as a limit", c.text());
                    }
}

// "precision n d kernel" of exemplar_eval's contraction kernel, a line each.
static void print_kernels() {
    for (int prec : {EXEMCL_FP32, EXEMCL_FP16, EXEMCL_BF16})
        for (int64_t n : {1, 6143, 6144, 12000})
            for (int64_t d : {1, 2, 3, 16, 17, 512, 513, 1024, 1025, 1 << 20, (1 << 20) + 1}) {
                fake::launches.clear();
                expect(exemplar_eval(kV, n, d, kI, 40, 3, prec, kF, fresh_stream()) == EXEMCL_OK, "eval");
                for (const auto &x : fake::launches)
                    if (x.name.find("eval_") != std::string::npos)
                        printf("%d %lld %lld %s\n", prec, (long long)n, (long long)d, x.name.c_str());
            }
}

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "grids") check_grids();
    else if (what == "devices") check_devices();
    else if (what == "counter") check_counter();
    else if (what == "limits") check_limits();
    else if (what == "kernels") print_kernels();
    else expect(false, "no such check", what);
    if (failures) fprintf(stderr, "%d checks failed\n", failures);
    else printf("%s: checks passed\n", what.c_str());
    return failures ? 1 : 0;
}
