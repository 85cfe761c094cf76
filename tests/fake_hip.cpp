// A HIP runtime for tests of the library's host side without a GPU.  Loaded
// into the global scope before libttx.so, it takes the place of the runtime:
// device memory is host memory, kernels are recorded instead of run.
//
// Recorded launches are checked: fewer than 2^32 work items, and for the
// launches over many problems that the tables they are given lie in live
// allocations and name a problem for every chunk.
#include <dlfcn.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "box.h"
#include "contract.h"
#include "ttx_internal.h"

namespace {

struct Config {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
};
struct Launch {
    std::string name;
    uint64_t grid, items;
    uint32_t first;                  // contractions: the launch's first workgroup
    std::vector<const void*> ptr;    // launches over many problems: their tables
    int shift = 0, chunk = 0;
    uint32_t chunks = 0;
};
std::map<const void*, std::string> g_names;
std::map<uintptr_t, size_t> g_live;
std::vector<Config> g_configs;
std::vector<Launch> g_launches;
std::vector<std::vector<Launch>> g_graphs;
std::vector<Launch>* g_capture = nullptr;
int g_unsound = 0;                   // launches that a GPU would refuse or that read what is not there
int g_mallocs_left = -1;             // allocations until they fail (-1: never)
int g_plans = 0;                     // calls of plan_box
float g_elapsed = 1.0f;              // what the next pair of events is apart, in ms

bool live(const void* p, size_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    auto it = g_live.upper_bound(a);
    if (it == g_live.begin()) return false;
    --it;
    return a >= it->first && a + bytes <= it->first + it->second;
}

bool sound(const Launch& l) {
    if (l.items >= uint64_t(1) << 32) return false;
    if (l.name.find("k_box_batch") == std::string::npos) {
        for (const void* p : l.ptr)
            if (!live(p, 4)) return false;
        return true;
    }
    const auto* desc = static_cast<const ttx::BoxBatchDesc*>(l.ptr[0]);
    const auto* first = static_cast<const uint32_t*>(l.ptr[1]);
    const auto* bucket = static_cast<const uint32_t*>(l.ptr[2]);
    if (l.grid < uint64_t(l.chunks) << l.chunk) return false;
    for (uint32_t c = 0; c < l.chunks; ++c) {
        if (!live(bucket + (c >> l.shift), 8)) return false;
        uint32_t lo = bucket[c >> l.shift], hi = bucket[(c >> l.shift) + 1];
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (!live(first + mid, 4)) return false;
            if (first[mid] <= c) lo = mid;
            else hi = mid - 1;
        }
        if (!live(first + lo, 4) || !live(desc + lo, sizeof(*desc))) return false;
        const uint32_t n = desc[lo].f64.ntiles;
        if (first[lo] > c || c - first[lo] >= (n + (1u << l.chunk) - 1) >> l.chunk) return false;
    }
    return true;
}

void run(const Launch& l) {
    if (!sound(l)) ++g_unsound;
    g_launches.push_back(l);
}

}  // namespace

extern "C" {

// -- what the tests read and set ---------------------------------------------------
int fake_launches() { return int(g_launches.size()); }
const char* fake_name(int i) { return g_launches[i].name.c_str(); }
uint64_t fake_grid(int i) { return g_launches[i].grid; }
uint32_t fake_first(int i) { return g_launches[i].first; }
int fake_unsound() { return g_unsound; }
int fake_plans() { return g_plans; }
void fake_fail_mallocs_after(int n) { g_mallocs_left = n; }
void fake_reset() {
    g_launches.clear();
    g_unsound = g_plans = 0;
    g_elapsed = 1.0f;
    g_mallocs_left = -1;
}
// Sets how time_candidates answers: candidate i takes us[i] microseconds, any
// further one `rest`, the last of the list `last` (which it launches once).
static std::vector<double> g_us;
static double g_rest = 0, g_last = 0;
void fake_times(int n, const double* us, double rest, double last) {
    g_us.assign(us, us + n);
    g_rest = rest;
    g_last = last;
}

// -- the runtime ---------------------------------------------------------------------
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
    g_configs.push_back(Config{grid, block, shmem, stream});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream) {
    const Config c = g_configs.back();
    g_configs.pop_back();
    *grid = c.grid;
    *block = c.block;
    *shmem = c.shmem;
    *stream = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    Launch l;
    l.name = g_names[f];
    l.grid = grid.x;
    l.items = uint64_t(grid.x) * block.x;
    l.first = 0;
    if (l.name.find("k_contract") != std::string::npos) {
        l.first = static_cast<const ttx::ContractArgs*>(args[0])->first;
    } else if (l.name.find("k_box_batch") != std::string::npos) {
        for (int i = 0; i < 3; ++i) l.ptr.push_back(*static_cast<void* const*>(args[i]));
        l.shift = *static_cast<const int*>(args[3]);
        l.chunk = *static_cast<const int*>(args[4]);
        l.chunks = *static_cast<const uint32_t*>(args[5]);
    } else if (l.name.find("k_batch") != std::string::npos) {
        for (int i : {0, 1, 4}) l.ptr.push_back(*static_cast<void* const*>(args[i]));
    }
    if (g_capture) g_capture->push_back(l);
    else run(l);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
    if (g_mallocs_left == 0) return hipErrorOutOfMemory;
    if (g_mallocs_left > 0) --g_mallocs_left;
    *p = std::calloc(1, bytes ? bytes : 1);
    g_live[reinterpret_cast<uintptr_t>(*p)] = bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (p) {
        g_live.erase(reinterpret_cast<uintptr_t>(p));
        std::free(p);
    }
    return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
    if (!live(to, n)) ++g_unsound;
    else std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) {
    *s = reinterpret_cast<hipStream_t>(uintptr_t(64));
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return hipStreamCreate(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    g_graphs.emplace_back();
    g_capture = &g_graphs.back();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    g_capture = nullptr;
    *g = reinterpret_cast<hipGraph_t>(g_graphs.size());
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    *e = reinterpret_cast<hipGraphExec_t>(g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
    for (const Launch& l : g_graphs[reinterpret_cast<uintptr_t>(e) - 1]) run(l);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(uintptr_t(64));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = g_elapsed *= 1.05f;   // what is timed first wins
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
hipError_t hipModuleLoadData(hipModule_t* m, const void*) {
    *m = reinterpret_cast<hipModule_t>(uintptr_t(64));
    return hipSuccess;
}
hipError_t hipModuleUnload(hipModule_t) { return hipSuccess; }
hipError_t hipModuleGetFunction(hipFunction_t* f, hipModule_t, const char*) {
    *f = reinterpret_cast<hipFunction_t>(uintptr_t(64));
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 4;
    return hipSuccess;
}

}  // extern "C"

// -- the library's own functions that a test counts or answers for ------------------
// Each forwards to the definition in libttx.so, which the caller has loaded.
static void* in_library(const char* symbol) {
    static void* lib = dlopen(std::getenv("FAKE_HIP_LIBRARY"), RTLD_NOW | RTLD_NOLOAD);
    return lib ? dlsym(lib, symbol) : nullptr;
}

namespace ttx {

bool plan_box(const Problem& p, bool beta0, BoxPlan* out, bool batched) {
    typedef bool (*F)(const Problem&, bool, BoxPlan*, bool);
    static const F f = reinterpret_cast<F>(in_library("_ZN3ttx8plan_boxERKNS_7ProblemEbPNS_7BoxPlanEb"));
    ++g_plans;
    return f(p, beta0, out, batched);
}

ttx_status time_candidates(const Problem&, bool, int count, int,
                           const std::function<hipError_t(int, const void*, void*, hipStream_t)>& launch, int* best_i,
                           double* best_us, double* all_us) {
    launch(count - 1, reinterpret_cast<void*>(uintptr_t(1) << 40), reinterpret_cast<void*>(uintptr_t(1) << 42), nullptr);
    *best_i = -1;
    *best_us = 1e300;
    for (int i = 0; i < count; ++i) {
        const double us = i + 1 == count ? g_last : i < int(g_us.size()) ? g_us[i] : g_rest;
        if (all_us) all_us[i] = us;
        if (us < *best_us) *best_us = us, *best_i = i;
    }
    return TTX_OK;
}

}  // namespace ttx
