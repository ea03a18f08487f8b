// A HIP runtime that runs nothing: memory is host memory, launches are noted
// and dropped, so that the library's host code (what it allocates, frees and
// launches, and when) can be checked on a machine without a GPU.  The program
// defines the runtime's functions itself and links the library, which then
// takes them instead of the real ones.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "pstd.h"

namespace {

std::map<char*, size_t> g_live;       // allocations
std::set<hipStream_t> g_capturing;
int g_fail_in = -1;                   // allocations until one fails (-1: none does)
std::vector<size_t>* g_sizes = nullptr;  // of allocations, where noted
int g_violations = 0;                 // calls that a capture does not allow
std::function<void(const std::string&, dim3, void**)> g_on_launch;

// kernel names by their host stubs (filled by the library's constructors, which
// run before this program's)
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
hipError_t g_last = hipSuccess;

hipError_t forbidden_while_capturing(const char* what) {
    if (g_capturing.empty()) return hipSuccess;
    std::printf("%s while a stream is captured\n", what);
    ++g_violations;
    return g_last = hipErrorStreamCaptureUnsupported;
}

// bytes from p to the end of the live allocation it points into, -1 if none
int64_t room(const void* p) {
    auto it = g_live.upper_bound((char*)p);
    if (it == g_live.begin()) return -1;
    --it;
    const int64_t off = (char*)p - it->first;
    return off < (int64_t)it->second ? (int64_t)it->second - off : -1;
}

int g_failures = 0;
void check(bool ok, const char* what) {
    if (ok) return;
    std::printf("FAILED: %s\n", what);
    ++g_failures;
}
#define CHECK(x) check((x), #x)

}  // namespace

extern "C" {

hipError_t hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (hipError_t e = forbidden_while_capturing("hipMalloc")) return e;
    if (g_fail_in == 0) {
        g_fail_in = -1;
        return g_last = hipErrorOutOfMemory;
    }
    if (g_fail_in > 0) --g_fail_in;
    if (g_sizes) g_sizes->push_back(n);
    *p = std::calloc(1, n ? n : 1);
    g_live[(char*)*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    if (hipError_t e = forbidden_while_capturing("hipFree")) return e;
    if (!g_live.erase((char*)p)) {
        std::printf("hipFree of memory that is not allocated\n");
        ++g_violations;
        return hipErrorInvalidValue;
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    if (hipError_t e = forbidden_while_capturing("hipMemcpy")) return e;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
    if (hipError_t e = forbidden_while_capturing("hipMemset")) return e;
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return forbidden_while_capturing("hipDeviceSynchronize"); }
hipError_t hipStreamSynchronize(hipStream_t) { return forbidden_while_capturing("hipStreamSynchronize"); }
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) {
    return e == hipErrorStreamCaptureUnsupported ? "operation not permitted when stream is capturing" : "error";
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* s) {
    *p = const_cast<void*>(s);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    g_capturing.insert(s);
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
    g_capturing.erase(s);
    *g = (hipGraph_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = g_capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return forbidden_while_capturing("hipEventSynchronize"); }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *x = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) {
    std::free(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t g) {
    std::free(g);
    return hipSuccess;
}

// the launch interface of compiled code
struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
static std::vector<Config> g_config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
    g_config.push_back({g, b, s, st});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
    const Config c = g_config.back();
    g_config.pop_back();
    *g = c.grid;
    *b = c.block;
    *s = c.shared;
    *st = c.stream;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
    names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    if (grid.x == 0 || grid.y == 0 || grid.z == 0 || block.x * block.y * block.z == 0) return g_last = hipErrorInvalidConfiguration;
    if (g_on_launch) g_on_launch(names()[f], grid, args);
    return hipSuccess;
}

}  // extern "C"

namespace {

// the default geometry on n cells per axis, the surface DFT on every step
pstd_problem problem(int n = 48) {
    pstd_problem p;
    pstd_problem_init_defaults(&p);
    for (int a = 0; a < 3; ++a) {
        p.n[a] = n;
        p.tfsf[a][2] += n - 48;
        p.tfsf[a][3] += n - 48;
        p.surf_hi[a] += n - 48;
    }
    p.dft_begin = 0;
    p.dft_end = 100;
    return p;
}

bool has(const std::string& s, const char* t) { return s.find(t) != std::string::npos; }

// Box far fields captured by a caller: nothing is allocated, freed or waited
// for while the stream is captured, whatever the number of directions, and what
// the captured launches use stays allocated until the solver goes.
void far_field_captured() {
    hipStream_t st;
    hipStreamCreateWithFlags(&st, 0);
    const pstd_problem p = problem();
    const int64_t few = 64, many = 70000, most = (1 << 20) + 5;
    std::vector<double> in(3 * most, 0.1), out(2 * most);
    for (int warm = 0; warm < 3; ++warm) {  // by nothing, by a few directions, by points
        pstd_solver* s = nullptr;
        CHECK(pstd_create(&p, st, &s) == PSTD_OK);
        CHECK(pstd_run(s, 3) == PSTD_OK);
        if (warm == 1) CHECK(pstd_far_field(s, in.data(), few, out.data()) == PSTD_OK);
        if (warm == 2) {
            std::vector<double> far(3 * few, 1e3);
            CHECK(pstd_project(s, far.data(), few, out.data()) == PSTD_OK);
        }
        std::vector<const void*> used;
        int64_t summed = 0;
        g_on_launch = [&](const std::string& name, dim3 grid, void** a) {
            if (!has(name, "far_eval_kernel")) return;
            const int64_t nd = *(int64_t*)a[1];
            const void* coef = *(void**)a[2];
            const void* part = *(void**)a[3];
            CHECK(room(coef) > 0);
            CHECK(room(part) >= (int64_t)grid.y * nd * 16);
            used.push_back(coef);
            used.push_back(part);
            summed += nd;
        };
        g_violations = 0;
        hipStreamBeginCapture(st, hipStreamCaptureModeGlobal);
        const pstd_status got = pstd_far_field(s, in.data(), many, out.data());
        hipGraph_t graph;
        hipStreamEndCapture(st, &graph);
        CHECK(g_violations == 0);
        if (warm == 0) {  // refused, and the capture is left whole
            CHECK(got == PSTD_EHIP);
            CHECK(used.empty());
        } else {
            CHECK(got == PSTD_OK);
            CHECK(summed == many);
        }
        std::vector<const void*> held;
        held.swap(used);
        CHECK(pstd_far_field(s, in.data(), most, out.data()) == PSTD_OK);
        std::vector<double> far(3 * 40000, 1e3);
        CHECK(pstd_project(s, far.data(), 40000, out.data()) == PSTD_OK);
        for (const void* q : held) CHECK(room(q) > 0);
        g_on_launch = nullptr;
        CHECK(pstd_destroy(s) == PSTD_OK);
    }
    CHECK(g_live.empty());
}

// Batches whose launch groups cannot be rebuilt for want of memory: the run fails,
// and the next one, with memory again, launches every instance with tables that
// are allocated.
void batch_rebuild() {
    hipStream_t st;
    hipStreamCreateWithFlags(&st, 0);
    const std::vector<pstd_problem> p = {problem(48), problem(64), problem(160), problem(48)};
    const std::vector<int64_t> once(p.size(), 3), grow(p.size(), 3000);
    int failed = 0;
    for (int k = 0;; ++k) {
        pstd_batch* b = nullptr;
        CHECK(pstd_batch_create(p.data(), (int32_t)p.size(), st, &b) == PSTD_OK);
        CHECK(pstd_batch_run(b, once.data()) == PSTD_OK);
        std::map<std::string, int> instances;  // launched, by kernel
        int launches = 0;
        g_on_launch = [&](const std::string& name, dim3, void** a) {
            if (!has(name, "pass_kernel")) return;
            const void *desc = *(void**)a[1], *off = *(void**)a[2];
            const int n = *(int*)a[3];
            CHECK(n > 0 && room(desc) > 0 && room(off) >= (int64_t)(n + 1) * (int64_t)sizeof(int));
            instances[name] += n;
            ++launches;
        };
        g_fail_in = k;
        const bool grown = pstd_batch_run(b, grow.data()) == PSTD_OK;  // the step tables grow, and the groups with them
        CHECK(grown == (g_fail_in >= 0));
        g_fail_in = -1;
        if (!grown) {
            ++failed;
            CHECK(launches == 0);
        }
        (void)hipGetLastError();
        instances.clear();
        CHECK(pstd_batch_run(b, once.data()) == PSTD_OK);
        int total = 0;
        for (const auto& i : instances) total += i.second;
        CHECK(total == 3 * 3 * (int)p.size());  // steps, passes, instances
        g_on_launch = nullptr;
        CHECK(pstd_batch_destroy(b) == PSTD_OK);
        CHECK(g_live.empty());
        if (grown) break;
    }
    CHECK(failed > (int)p.size());
}

// Short runs of a batch beyond the cache go pass by pass over all instances; from
// twelve such launches on, by sets on the branches.
void batch_short_runs() {
    hipStream_t st;
    hipStreamCreateWithFlags(&st, 0);
    const std::vector<pstd_problem> p(4, problem(160));
    pstd_batch* b = nullptr;
    CHECK(pstd_batch_create(p.data(), (int32_t)p.size(), st, &b) == PSTD_OK);
    for (int steps = 1; steps <= 5; ++steps) {
        int launches = 0, instances = 0;
        g_on_launch = [&](const std::string& name, dim3, void** a) {
            if (!has(name, "pass_kernel")) return;
            ++launches;
            instances += *(int*)a[3];
        };
        const std::vector<int64_t> n(p.size(), steps);
        CHECK(pstd_batch_run(b, n.data()) == PSTD_OK);
        std::printf("%d steps: %d launches\n", steps, launches);
        CHECK(launches == (steps < 4 ? 3 * steps : 12 * steps));
        CHECK(instances == 12 * steps);
    }
    g_on_launch = nullptr;
    CHECK(pstd_batch_destroy(b) == PSTD_OK);
}

// What is timed for an axis is the launch that a step makes, with the plane values
// staged as it stages them; and a tile shape set on an axis is the one that runs.
void timed_launches() {
    hipStream_t st;
    hipStreamCreateWithFlags(&st, 0);
    std::set<std::string> seen;
    g_on_launch = [&](const std::string& name, dim3, void**) {
        for (const char* k : {"pass_xy_kernel", "pass_seg_xy_kernel", "pass_kernel"})
            if (has(name, k)) {
                seen.insert(k);
                break;
            }
    };
    using Names = std::set<std::string>;
    auto launched = [&](auto&& call) {
        seen.clear();
        CHECK(call() == PSTD_OK);
        return seen;
    };
    double us;
    {
        const pstd_problem p = problem();
        pstd_solver* s = nullptr;
        CHECK(pstd_create(&p, st, &s) == PSTD_OK);
        for (int axis = 0; axis < 2; ++axis)
            CHECK(launched([&] { return pstd_pass_time(s, axis, 3, &us); }) == Names{"pass_xy_kernel"});
        CHECK(launched([&] { return pstd_pass_time(s, 2, 3, &us); }) == Names{"pass_kernel"});
        std::vector<size_t> sizes;
        g_sizes = &sizes;
        CHECK(pstd_autotune(s, 2) == PSTD_OK);
        g_sizes = nullptr;
        int rings = 0;
        for (size_t n : sizes) rings += n == 4 * 48 * 48 * 2 * sizeof(float);
        CHECK(rings == 3);  // x and y, and z
        CHECK(launched([&] { return pstd_set_tile(s, 0, 8, 32, 0); }).empty());  // x alone
        CHECK(launched([&] { return pstd_run(s, 1); }) == Names{"pass_kernel"});
        CHECK(launched([&] { return pstd_pass_time(s, 0, 3, &us); }) == Names{"pass_kernel"});
        CHECK(pstd_set_tile(s, 1, 8, 32, 0) == PSTD_OK);
        CHECK((launched([&] { return pstd_run(s, 1); }) == Names{"pass_kernel", "pass_xy_kernel"}));
        CHECK(pstd_destroy(s) == PSTD_OK);
    }
    {
        pstd_problem p = problem(96);
        for (int a = 0; a < 3; ++a) p.sub_core[a] = 48;
        p.sub_halo = 8;
        p.sub_taper = 3;
        pstd_solver* s = nullptr;
        CHECK(pstd_create(&p, st, &s) == PSTD_OK);
        const Names fused{"pass_kernel", "pass_seg_xy_kernel"}, apart{"pass_kernel"};
        int32_t was[3][5], info[5];
        for (int axis = 0; axis < 3; ++axis) CHECK(pstd_tile_info(s, axis, was[axis]) == PSTD_OK);
        CHECK(was[0][0] == 64 && was[0][3] == 48 && was[0][4] == -1 && was[1][4] == -1 && was[2][4] == 0);
        CHECK(launched([&] { return pstd_run(s, 1); }) == fused);
        CHECK(launched([&] { return pstd_pass_time(s, 1, 3, &us); }) == Names{"pass_seg_xy_kernel"});
        CHECK(pstd_set_tile(s, 0, 8, 16, 0) == PSTD_OK);
        CHECK(pstd_tile_info(s, 0, info) == PSTD_OK && info[3] == 16 && info[4] == 0);
        CHECK(launched([&] { return pstd_run(s, 1); }) == apart);
        CHECK(pstd_set_tile(s, 1, 8, 16, 0) == PSTD_OK);  // the same on both
        CHECK(launched([&] { return pstd_run(s, 1); }) == apart);
        CHECK(launched([&] { return pstd_pass_time(s, 1, 3, &us); }) == apart);
        // the shapes noted before bring the noted form back
        for (int axis = 0; axis < 3; ++axis)
            CHECK(pstd_set_tile(s, axis, was[axis][1], was[axis][3], was[axis][4]) == PSTD_OK);
        CHECK(launched([&] { return pstd_run(s, 1); }) == fused);
        CHECK(pstd_set_tile(s, 2, 8, 48, -1) == PSTD_EUNSUPPORTED);
        CHECK(pstd_destroy(s) == PSTD_OK);
    }
    {
        // a core that fits the pencils of the fused form and leaves too many idle
        pstd_problem p = problem(96);
        for (int a = 0; a < 3; ++a) p.sub_core[a] = 32;
        p.sub_halo = 16;
        p.sub_taper = 3;
        pstd_solver* s = nullptr;
        CHECK(pstd_create(&p, st, &s) == PSTD_OK);
        CHECK(launched([&] { return pstd_run(s, 1); }) == Names{"pass_kernel"});
        CHECK(pstd_destroy(s) == PSTD_OK);
    }
    g_on_launch = nullptr;
}

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "far_field_captured") far_field_captured();
    else if (what == "batch_rebuild") batch_rebuild();
    else if (what == "batch_short_runs") batch_short_runs();
    else if (what == "timed_launches") timed_launches();
    else return 2;
    std::printf("%d failures\n", g_failures);
    return g_failures ? 1 : 0;
}
