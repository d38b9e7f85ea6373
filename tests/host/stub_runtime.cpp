// Drives libmpr.so on a HIP runtime of its own: kernels launched here stay
// queued and do nothing but write the host records that calls wait for, one
// kernel at a time and only when the stream is asked about or drained.  The
// launch check and the allocation that fail can be chosen, so what a call
// leaves behind on its error paths can be looked at without a GPU.
//   stub_runtime <libmpr.so> errors   every launch check of every call fails once
//   stub_runtime <libmpr.so> idle     synchronous calls return with the stream drained
//   stub_runtime <libmpr.so> wait     a wait of 400 ms leaves the processor to others
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <time.h>

#include <chrono>
#include <deque>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "../../include/mpr.h"

static std::map<const void *, std::string> names;
struct Kernel { std::function<void()> run; bool writes; };  // writes: a host record
static std::deque<Kernel> queued;
static bool retiring = false;  // the last kernel has written its record and still runs
static int fail_at = -1, checks = 0, allocations_fail = 0;
static std::chrono::steady_clock::time_point hold;  // nothing runs before
static bool sticky = false;  // an error that hipGetLastError has yet to report
struct Call { dim3 grid, block; size_t shared; hipStream_t stream; };
static Call call;

static void run_one()
{
    if (queued.empty()) return;
    queued.front().run();
    queued.pop_front();
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, dim3 *,
                           dim3 *, int *)
{
    names[host] = device;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, hipStream_t s) { call = Call{g, b, n, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *n, hipStream_t *s)
{
    *g = call.grid, *b = call.block, *n = call.shared, *s = call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t)
{
    const std::string &k = names[f];
    auto record = [&](int at, int64_t first) {
        int64_t *rec = *(int64_t **)args[at], seq = *(int64_t *)args[at + 1];
        queued.push_back({[=] {
            if (!rec) return;
            rec[0] = first, rec[1] = rec[2] = rec[3] = 0;
            rec[7] = seq;
        }, rec != nullptr});
    };
    static int64_t hash = 1;
    if (k.find("14sp_scan_kernel") != k.npos) record(4, 32);
    else if (k.find("12check_kernel") != k.npos && grid.x == 1) record(8, 0);
    else if (k.find("19tiny_checked_kernel") != k.npos) record(9, 0);
    else if (k.find("16check_end_kernel") != k.npos) record(0, 0);
    else if (k.find("19period_small_kernel") != k.npos) record(8, hash++);
    else if (k.find("18period_rows_kernel") != k.npos) record(11, hash++);
    else if (k.find("19period_rows8_kernel") != k.npos) record(12, hash++);
    else queued.push_back({[] {}, false});
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const bool e = checks++ == fail_at || sticky;
    sticky = false;
    return e ? hipErrorUnknown : hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t)
{
    if (queued.empty()) return retiring = false, hipSuccess;
    if (std::chrono::steady_clock::now() < hold) return hipErrorNotReady;
    retiring = true;
    run_one();
    return hipErrorNotReady;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    while (!queued.empty()) run_one();
    retiring = false;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t)
{
    if (allocations_fail) { sticky = true; return hipErrorOutOfMemory; }
    *p = malloc(n);
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char s[256]; *p = s; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
}

static void *lib;
template <class F> static F *entry(const char *n)
{
    F *f = (F *)dlsym(lib, n);
    if (!f) fprintf(stderr, "no %s\n", n), exit(2);
    return f;
}

int main(int argc, char **argv)
{
    if (argc != 3 || !(lib = dlopen(argv[1], RTLD_NOW | RTLD_GLOBAL))) return fprintf(stderr, "%s\n", dlerror()), 2;
    auto *plan = entry<decltype(mpr_sparse_plan_bytes)>("mpr_sparse_plan_bytes");
    auto *find = entry<decltype(mpr_find_period_ex)>("mpr_find_period_ex");
    auto *gemm = entry<decltype(mpr_minplus_gemm_checked)>("mpr_minplus_gemm_checked");
    const bool errors = !strcmp(argv[2], "errors");
    std::vector<uint16_t> A(400 * 400), C(400 * 400);
    std::vector<char> ws(64 << 20);
    int64_t mu, lam, c;
    size_t bytes;
    int32_t verdict = 0;
    if (!strcmp(argv[2], "wait")) {
        hold = std::chrono::steady_clock::now() + std::chrono::milliseconds(400);
        const clock_t busy = clock();
        const mpr_status e = plan(A.data(), 300, 300, &bytes, nullptr);
        const double part = (double)(clock() - busy) / CLOCKS_PER_SEC / 0.4;
        printf(e == MPR_OK && part < 0.25 ? "ok\n" : "status %d, %.0f %% of the wait busy\n", e, 100 * part);
        return e != MPR_OK || part >= 0.25;
    }
    struct Case { std::string name; std::function<mpr_status()> call; };
    std::vector<Case> cases;
    for (int64_t n : {20, 300})
        cases.push_back({"plan n=" + std::to_string(n), [=, &A, &bytes] { return plan(A.data(), n, n, &bytes, nullptr); }});
    for (int64_t n : {20, 100, 300})
        for (int flags : {0, 1, 8, 9, 5}) {
            const int64_t ld = (n + 7) / 8 * 8;
            cases.push_back({"search n=" + std::to_string(n) + " flags=" + std::to_string(flags), [=, &A, &ws, &mu, &lam, &c] {
                return find(A.data(), n, ld, 6, flags, &mu, &lam, &c, nullptr, ws.data(), ws.size(), nullptr);
            }});
        }
    for (int64_t n : {33, 300}) {
        cases.push_back({"checked product n=" + std::to_string(n), [=, &A, &C, &verdict] {
            return gemm(-1, 0, n, n, n, A.data(), n, A.data(), n, C.data(), n, &verdict, nullptr);
        }});
    }
    int bad = 0;
    auto look = [&](const Case &k, const char *when) {
        size_t left = 0;
        for (const Kernel &q : queued) left += !errors || q.writes;
        const bool runs = !errors && retiring && k.name[0] != 'c';  // the check's record is the product's end
        if (!left && !runs && !verdict) return;
        printf("%s, %s: %zu kernels still queued, %s, verdict %d\n", k.name.c_str(), when, left,
               runs ? "one running" : "none running", verdict);
        bad++, verdict = 0;
        (void)hipStreamSynchronize(nullptr);
    };
    for (const Case &k : cases) {
        fail_at = -1, checks = 0;
        const mpr_status ok = k.call();
        if (ok != MPR_OK && ok != MPR_ENOTFOUND) printf("%s: status %d\n", k.name.c_str(), ok), bad++;
        if (!errors) look(k, "returned");
        (void)hipStreamSynchronize(nullptr);
        const int launches = checks;
        for (int f = 0; errors && f < launches; f++) {
            fail_at = f, checks = 0;
            const mpr_status e = k.call();
            if (e != MPR_EHIP && e != MPR_ENOTFOUND && e != MPR_OK) printf("%s: status %d\n", k.name.c_str(), e), bad++;
            look(k, ("launch check " + std::to_string(f) + " failed").c_str());
            (void)hipStreamSynchronize(nullptr);
        }
    }
    if (errors) {  // a failed allocation is reported once, not by the next launch check as well
        fail_at = -1, allocations_fail = 1;
        const mpr_status e = plan(A.data(), 20, 20, &bytes, nullptr);
        allocations_fail = 0;
        const mpr_status f = plan(A.data(), 20, 20, &bytes, nullptr);
        if (e != MPR_ENOMEM || f != MPR_OK) printf("failed allocation: %d, then %d\n", e, f), bad++;
    }
    if (!bad) printf("ok\n");
    return bad != 0;
}
