// A stand-in for the HIP runtime that runs the library's host code without a device: memory is
// host memory, a launch is written to the log and only does what the host reads back (counts,
// statistics, publications).  Linked into an executable, these definitions come before the
// runtime's own.  Each command runs one sequence of calls and prints what happened.
#include <cxxabi.h>
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <unordered_map>
#include <vector>

#include "common.hpp"
#include "treepm.h"

namespace {

std::mutex mu;
std::map<void *, size_t> live;
size_t live_bytes = 0;
int mallocs = 0, fail_at = -1; // fail_at: the first allocation that fails, counted from 0
// (registered before this file's own objects are constructed)
std::unordered_map<const void *, std::string> &names()
{
    static std::unordered_map<const void *, std::string> n;
    return n;
}
std::vector<std::string> trace;

// What the device would report for every box.
struct Report {
    uint32_t nodes1 = 8, groups = 2000;
    uint64_t cells = 100000, parts = 100000, pairs = 1000000, longest = 300, rows = 0, items = 0;
} rep;

void note(const std::string &s) { trace.push_back(s); }

bool has(const std::string &s, const char *what) { return s.find(what) != std::string::npos; }

void set_stats(unsigned long long *st)
{
    const unsigned long long v[6] = {rep.cells, rep.parts, rep.pairs, rep.longest, rep.rows, rep.items};
    memcpy(st, v, sizeof v);
}

template <typename T>
T arg(void **args, int i)
{
    return *static_cast<T *>(args[i]);
}

// Called with mu held.
void run_kernel(const std::string &k, void **args)
{
    note(k);
    if (has(k, "::k_publish(")) {
        uint32_t *m = arg<uint32_t *>(args, 6), at = 1;
        for (int r = 0; r < 3; ++r) {
            const uint32_t n = arg<uint32_t>(args, 2 * r + 1);
            if (n) memcpy(m + at, arg<const uint32_t *>(args, 2 * r), 4 * n);
            at += n;
        }
        __atomic_store_n(&m[0], arg<uint32_t>(args, 7), __ATOMIC_RELEASE);
        note("published");
    } else if (has(k, "k_set<unsigned int>")) {
        uint32_t *p = arg<uint32_t *>(args, 0);
        for (size_t i = 0; i < arg<size_t>(args, 1); ++i) p[i] = arg<uint32_t>(args, 2);
    } else if (has(k, "k_set<unsigned long>")) {
        uint64_t *p = arg<uint64_t *>(args, 0);
        for (size_t i = 0; i < arg<size_t>(args, 1); ++i) p[i] = arg<uint64_t>(args, 2);
    } else if (has(k, "k_build_init")) {
        memset(arg<unsigned *>(args, 0), 0, 24);
    } else if (has(k, "k_tree_scan")) {
        uint32_t *tot = arg<uint32_t *>(args, 2);
        memset(tot, 0, (tpm::kMaxLevel + 1) * 4);
        tot[0] = 1;
        tot[1] = rep.nodes1;
    } else if (has(k, "k_scan_one<") || has(k, "k_scan_tile<")) {
        void *total = arg<void *>(args, has(k, "k_scan_one<") ? 2 : 3);
        if (total && has(k, "<unsigned int>")) *static_cast<uint32_t *>(total) = rep.groups;
        if (total && has(k, "<unsigned long>"))
            *static_cast<uint64_t *>(total) = rep.cells + rep.parts;
    } else if (has(k, "k_group_compact") || has(k, "k_group_bbox")) {
        const bool bbox = has(k, "k_group_bbox");
        const uint32_t cap = arg<uint32_t>(args, 3);
        const tpm::GroupArrays gr = bbox ? arg<tpm::GroupArrays>(args, 1) : tpm::GroupArrays{};
        const void *need[] = {gr.node, gr.first, gr.count, gr.cgx, gr.cgy, gr.cgz, gr.hgx,
                              gr.hgy, gr.hgz, gr.xgx, gr.xgy, gr.xgz, gr.lox, gr.loy,
                              gr.loz, gr.hix, gr.hiy, gr.hiz};
        const size_t size[] = {4, 4, 4, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8};
        if (bbox) {
            *arg<unsigned *>(args, 5) = 6;
            *arg<unsigned *>(args, 6) = 64;
        }
        if (bbox)
            for (int a = 0; a < 18; ++a) {
                const auto it = live.find(const_cast<void *>(need[a]));
                if (it == live.end() || it->second < cap * size[a])
                    note("group array " + std::to_string(a) + " too small for " + std::to_string(cap));
            }
    } else if (has(k, "k_walk_results(") || has(k, "k_walk_publish(")) {
        const tpm::WalkBox B = arg<tpm::WalkBox>(args, 0);
        set_stats(B.stats);
        if (B.mailbox) {
            B.mailbox[1] = 0;
            memcpy(B.mailbox + 2, B.stats, 48);
            __atomic_store_n(&B.mailbox[0], B.seq, __ATOMIC_RELEASE);
            note("published");
        }
    } else if (has(k, "k_walk_stats")) {
        set_stats(arg<unsigned long long *>(args, 4));
    }
}

} // namespace

extern "C" {
static dim3 cfg_grid, cfg_block;
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *)
{
    int st;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    names()[host] = st == 0 ? d : name;
    free(d);
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t)
{
    cfg_grid = g;
    cfg_block = b;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s)
{
    *g = cfg_grid;
    *b = cfg_block;
    *sh = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t)
{
    std::lock_guard<std::mutex> lk(mu);
    run_kernel(names()[f], args);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> lk(mu);
    if (mallocs++ >= fail_at && fail_at >= 0) return hipErrorOutOfMemory;
    *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    live[*p] = n;
    live_bytes += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lk(mu);
    const auto it = live.find(p);
    if (it == live.end()) return hipErrorInvalidValue;
    munmap(p, it->second);
    live_bytes -= it->second;
    live.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)288 << 30; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipPeekAtLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidValue; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace {

treepm_params params(int precision)
{
    treepm_params p{};
    p.L = 1.0;
    p.mesh = 1.0 / 64;
    p.r_cut = 3.0 / 64;
    p.eps = p.mesh / 20;
    p.theta = 0.5;
    p.n_leaf = 10;
    p.n_crit = 64;
    p.precision = precision;
    return p;
}

struct Arrays {
    std::vector<double> v;
    explicit Arrays(int64_t n) : v((size_t)n * 4, 0.25) {}
    const double *at(int a) const { return v.data() + v.size() / 4 * a; }
};

int build(treepm_ctx *c, const Arrays &a)
{
    return treepm_build(c, (int64_t)a.v.size() / 4, a.at(0), a.at(1), a.at(2), a.at(3), TREEPM_DEVICE,
                        nullptr);
}

int number(int argc, char **argv, int i, int def) { return i < argc ? atoi(argv[i]) : def; }

// What was launched from trace[from] on.
void print(size_t from)
{
    for (size_t i = from; i < trace.size(); ++i) printf("%s\n", trace[i].c_str());
}

} // namespace

int main(int argc, char **argv)
{
    const std::string cmd = argc > 1 ? argv[1] : "";
    treepm_ctx *c = nullptr;
    if (cmd == "walk") { // groups: the launches of a walk, and its return
        rep.groups = (uint32_t)number(argc, argv, 2, 2000);
        const treepm_params p = params(TREEPM_FP32);
        const Arrays a(200000);
        if (treepm_create(&p, 0, &c) || build(c, a)) return 1;
        const size_t from = trace.size();
        treepm_stats st{};
        if (treepm_walk(c, nullptr, &st)) return 1;
        print(from);
        printf("returned %lld\n", (long long)st.interactions);
        treepm_destroy(c);
    } else if (cmd == "groups") { // k: a build whose k-th group array fails, and the next one
        treepm_params p = params(TREEPM_FP32);
        const Arrays a((1 << 20) + 1);
        rep.groups = 1000;
        if (treepm_create(&p, 0, &c) || build(c, a)) return 1;
        // more groups: the arrays grow, the other buffers do not
        rep.groups = 400000;
        treepm_release_cached(0);
        fail_at = mallocs + number(argc, argv, 2, 0);
        printf("failed %d\n", build(c, a));
        fail_at = -1;
        const size_t from = trace.size();
        if (build(c, a)) return 1;
        print(from);
        printf("built\n");
        treepm_destroy(c);
    } else if (cmd == "force") { // precision, interactions, rows, eps / r_cut: a force call after a walk
        const int prec = number(argc, argv, 2, 0);
        rep.pairs = strtoull(argv[3], nullptr, 10);
        rep.rows = strtoull(argv[4], nullptr, 10);
        rep.items = rep.rows ? 4 : 0;
        treepm_params p = params(prec ? TREEPM_FP64 : TREEPM_FP32);
        if (argc > 5) p.eps = p.r_cut * atof(argv[5]);
        const Arrays a(200000);
        treepm_stats st{};
        void *out = nullptr;
        if (treepm_create(&p, 0, &c) || build(c, a) || treepm_walk(c, nullptr, &st) ||
            hipMalloc(&out, 3 * 200000 * 8) != hipSuccess)
            return 1;
        const size_t from = trace.size();
        const int before = mallocs;
        double *o = static_cast<double *>(out);
        printf("force %d\n",
               treepm_force_short(c, o, o + 200000, o + 400000, p.precision, TREEPM_DEVICE, nullptr));
        print(from);
        printf("allocations %d\n", mallocs - before);
        treepm_destroy(c);
    } else if (cmd == "slots") { // groups, longest and mean list: the memory held after 3 walks
        rep.groups = (uint32_t)number(argc, argv, 2, 0);
        rep.longest = (uint64_t)number(argc, argv, 3, 0);
        rep.cells = (uint64_t)rep.groups * (uint64_t)number(argc, argv, 4, 0);
        rep.parts = 0;
        const treepm_params p = params(TREEPM_FP32);
        const Arrays a(1000000);
        if (treepm_create(&p, 0, &c)) return 1;
        const size_t from = trace.size();
        for (int k = 0; k < 3; ++k) {
            if (build(c, a)) return 1;
            treepm_stats st{};
            if (treepm_walk(c, nullptr, &st)) return 1;
            treepm_release_cached(0); // what the context does not hold is not counted
            printf("held %zu\n", live_bytes);
        }
        print(from);
        treepm_destroy(c);
    } else if (cmd == "server") { // n, groups, longest and mean list, requests, budget
        const int64_t n = number(argc, argv, 2, 0);
        rep.groups = (uint32_t)number(argc, argv, 3, 0);
        rep.longest = (uint64_t)number(argc, argv, 4, 0);
        rep.cells = (uint64_t)rep.groups * (uint64_t)number(argc, argv, 5, 0);
        rep.parts = 0;
        rep.nodes1 = (uint32_t)(n / 2);
        const treepm_params p = params(TREEPM_FP32);
        const Arrays a(n);
        std::vector<float> out((size_t)n * 3);
        treepm_ens *e = nullptr;
        if (treepm_ens_create(0, (size_t)atoll(argv[7]), 2, &e)) return 1;
        for (int k = 0; k < number(argc, argv, 6, 1); ++k) {
            uint64_t t = 0;
            if (treepm_ensemble_submit(e, 7, &p, n, a.at(0), a.at(1), a.at(2), a.at(3), &t)) return 1;
            int rc = TREEPM_PENDING;
            for (int w = 0; w < 5000 && rc == TREEPM_PENDING; ++w) {
                std::this_thread::sleep_for(std::chrono::milliseconds(1));
                rc = treepm_ensemble_poll(e, t, out.data(), out.data() + n, out.data() + 2 * n, nullptr);
            }
            int64_t bytes = 0;
            treepm_ens_info(e, nullptr, nullptr, &bytes, nullptr);
            printf("served %d\nresident %lld\n", rc, (long long)bytes);
        }
        treepm_ens_destroy(e);
    } else {
        return 2;
    }
    return 0;
}
