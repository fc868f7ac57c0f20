// A HIP runtime without a device, for tests of the library's host code: device
// allocations are addresses out of a budget (never read or written), copies and
// kernels do nothing, and every launch is recorded with its grid, block and the
// leading arguments.  The few kernels whose results the host reads (cloud checks,
// voxel counts, extents) are stood in for by configured values.  Loaded globally
// before the library, so that the library binds to these symbols.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string name;
    uint32_t grid, block;
    std::vector<uint64_t> args;
};

std::map<const void*, std::string> g_kernels;
std::vector<Launch> g_launches;
std::map<std::string, int> g_watch;        // kernels whose leading arguments are recorded
std::map<std::string, int64_t> g_values;   // results stood in for
std::map<uintptr_t, size_t> g_live;
uintptr_t g_next = (uintptr_t)1 << 44;
size_t g_used = 0, g_peak = 0, g_budget = ~(size_t)0;
int64_t g_failed = 0, g_bad_frees = 0, g_fail_at = -1, g_mallocs = 0, g_allocations = 0;
hipError_t g_last = hipSuccess;
hipError_t fail(hipError_t e) { return g_last = e; }

struct Call {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
std::vector<Call> g_calls;

int64_t value(const char* key, int64_t otherwise) {
    const auto it = g_values.find(key);
    return it == g_values.end() ? otherwise : it->second;
}

// what the library's k_check leaves per workgroup
struct CheckPart {
    double box[6], first[3];
    int64_t bad;
    int32_t flags, pad;
};

template <typename T>
T arg(void** args, int k) {
    return *static_cast<T*>(args[k]);
}

void stand_in(const std::string& name, uint32_t grid, void** args) {
    auto is = [&](const char* s) { return name.find(s) != std::string::npos; };
    if (is("7k_checkE")) {
        auto* out = arg<CheckPart*>(args, 4);
        const double half = 0.5 * (double)value("extent", 10);
        for (uint32_t b = 0; b < grid; ++b)
            out[b] = CheckPart{{-half, -half, -half, half, half, half}, {0, 0, 0}, INT64_MAX, 0, 0};
    } else if (is("11k_ds_startsE")) {
        *arg<int32_t*>(args, 3) = (int32_t)value("downsampled", arg<int64_t>(args, 1));
    } else if (is("12k_map_voxelsE")) {
        const int64_t levels = arg<int64_t>(args, 3) / arg<int64_t>(args, 2);
        auto* info = arg<int32_t*>(args, 8);
        for (int64_t l = 0; l <= levels; ++l) {
            info[2 * l] = (int32_t)(l * value("voxels", 100));
            info[2 * l + 1] = (int32_t)(l * value("blocks", 10));
        }
    } else if (is("5k_maxE")) {
        *arg<double*>(args, 2) = (double)value("extent", 10);
    }
}

}  // namespace

extern "C" {

// ---------------------------------------------------------------- controls
void fake_reset() {
    g_launches.clear();
    g_failed = g_bad_frees = g_mallocs = g_allocations = 0;
    g_peak = g_used;
}
void fake_budget(int64_t bytes) { g_budget = bytes < 0 ? ~(size_t)0 : (size_t)bytes; }
void fake_fail_at(int64_t k) {   // the k-th device allocation from now fails, and those after it (-1: none)
    g_mallocs = 0;
    g_fail_at = k;
}
void fake_watch(const char* name, int n) { g_watch[name] = n; }
void fake_set(const char* key, int64_t v) { g_values[key] = v; }
int64_t fake_used() { return (int64_t)g_used; }
int64_t fake_peak() { return (int64_t)g_peak; }
int64_t fake_allocations() { return g_allocations; }
int64_t fake_failed() { return g_failed; }
int64_t fake_bad_frees() { return g_bad_frees; }
int64_t fake_last_error() { return (int64_t)g_last; }
int64_t fake_launches() { return (int64_t)g_launches.size(); }
const char* fake_name(int64_t k) { return g_launches[(size_t)k].name.c_str(); }
uint32_t fake_grid(int64_t k) { return g_launches[(size_t)k].grid; }
uint32_t fake_block(int64_t k) { return g_launches[(size_t)k].block; }
uint64_t fake_arg(int64_t k, int i) { return g_launches[(size_t)k].args[(size_t)i]; }
int fake_args(int64_t k) { return (int)g_launches[(size_t)k].args.size(); }

// ---------------------------------------------------------------- registration and launches
void** __hipRegisterFatBinary(const void*) {
    static void* handle[4];
    return handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
    g_kernels[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t st) {
    g_calls.push_back(Call{grid, block, shared, st});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* st) {
    const Call c = g_calls.back();
    g_calls.pop_back();
    *grid = c.grid;
    *block = c.block;
    *shared = c.shared;
    *st = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    const std::string& name = g_kernels[f];
    Launch l{name, grid.x, block.x, {}};
    for (const auto& w : g_watch)
        if (name.find(w.first) != std::string::npos)
            for (int k = 0; k < w.second; ++k) {
                uint64_t v;
                std::memcpy(&v, args[k], sizeof v);
                l.args.push_back(v);
            }
    g_launches.push_back(l);
    // the limit of a device launch: fewer than 2^32 threads
    if (grid.x == 0 || (uint64_t)grid.x * block.x >= (1ull << 32)) return fail(hipErrorInvalidConfiguration);
    stand_in(name, grid.x, args);
    return hipSuccess;
}

// ---------------------------------------------------------------- memory
hipError_t hipMalloc(void** p, size_t bytes) {
    *p = nullptr;
    ++g_allocations;
    if ((g_fail_at >= 0 && g_mallocs++ >= g_fail_at) || bytes > g_budget || g_used > g_budget - bytes) {
        ++g_failed;
        return fail(hipErrorOutOfMemory);
    }
    g_live[g_next] = bytes;
    *p = (void*)g_next;
    g_next += (bytes + 4095) & ~(size_t)4095;
    g_used += bytes;
    if (g_used > g_peak) g_peak = g_used;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (p == nullptr) return hipSuccess;
    const auto it = g_live.find((uintptr_t)p);
    if (it == g_live.end()) {
        ++g_bad_frees;
        return fail(hipErrorInvalidValue);
    }
    g_used -= it->second;
    g_live.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
    *p = std::calloc(bytes ? bytes : 1, 1);
    return *p ? hipSuccess : fail(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = (void*)((uintptr_t)1 << 43);
    return hipSuccess;
}

// ---------------------------------------------------------------- device, streams, events
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    std::strcpy(p->name, "no device");
    p->multiProcessorCount = 256;
    p->warpSize = 64;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 64;
    return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)std::malloc(16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free((void*)s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = (hipEvent_t)std::malloc(16);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    std::free((void*)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    static uint32_t x = 1;   // times of no meaning, all different
    x = x * 1664525u + 1013904223u;
    *ms = 1.0f + (float)(x >> 8) / (float)(1u << 24);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

}  // extern "C"
