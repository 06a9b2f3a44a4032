// A HIP runtime that launches nothing: loaded before the real one, it records
// what libtsgemm's host code asks for (launches with their arguments,
// allocations, attributes) and refuses what HIP refuses, so that the host code
// can be tested without a GPU.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace {
struct Record {
    const char* name;  // mangled kernel name
    uint32_t grid, block;
    uint64_t shmem, stream;
    uint64_t args[12];
};
struct Config {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
};
std::recursive_mutex mu;
std::map<const void*, std::string> names;
std::map<const void*, int> lds_limit;
std::vector<Record> records;
std::vector<std::pair<uint64_t, uint64_t>> buffers;
uint64_t next_address = 1ull << 40;
std::atomic<int> capturing{0};
std::atomic<void (*)(const char*)> hook{nullptr};  // called after a launch ("launch") or in a capture query ("query")
thread_local std::vector<Config> configs;
thread_local bool out_of_memory = false;
thread_local hipError_t last_error = hipSuccess;

void call_hook(const char* where)
{
    if (auto h = hook.load()) h(where);
}
// Parameters of the kernels whose arguments are recorded.
int count_args(const std::string& n)
{
    if (n.find("tsmttsm_packed") != std::string::npos || n.find("tsmttsm_valu") != std::string::npos) return 12;
    if (n.find("fold_partials") != std::string::npos) return 7;
    if (n.find("clear_counter") != std::string::npos) return 1;
    return 0;
}
}  // namespace

// Host allocations, which the tests can make fail.
void* operator new(size_t n)
{
    if (!out_of_memory)
        if (void* p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {

// ---- what the tests call
void rec_out_of_memory(int on) { out_of_memory = on; }
void rec_hook(void (*h)(const char*)) { hook = h; }
void rec_capturing(int on) { capturing = on; }
void rec_clear()
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    records.clear();
}
int rec_count()
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    return (int)records.size();
}
void rec_get(int i, Record* out)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    *out = records[i];
}
// size of the allocation at `p` (0: none)
uint64_t rec_buffer(uint64_t p)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    for (auto& b : buffers)
        if (b.first == p) return b.second;
    return 0;
}

// ---- the runtime
void** __hipRegisterFatBinary(const void*)
{
    static void* handle[1];
    return handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    names[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st)
{
    configs.push_back({g, b, s, st});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st)
{
    const Config c = configs.back();
    configs.pop_back();
    *g = c.grid;
    *b = c.block;
    *s = c.shmem;
    *st = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t shmem, hipStream_t st)
{
    {
        std::lock_guard<std::recursive_mutex> lk(mu);
        // fewer than 2^32 work items; more than 64 KB of LDS only as far as the attribute allows
        if ((uint64_t)g.x * b.x >= 1ull << 32 || g.x == 0) return last_error = hipErrorInvalidConfiguration;
        if (shmem > (64u << 10) && shmem > (size_t)lds_limit[fn]) return last_error = hipErrorInvalidValue;
        Record r{names[fn].c_str(), g.x, b.x, shmem, (uint64_t)st, {}};
        // 64-bit parameters and pointers only (the rest are 32-bit)
        const int n = count_args(names[fn]);
        for (int i : n == 12 ? std::vector<int>{0, 3, 4, 5, 6, 7, 8, 9, 11} : n == 7 ? std::vector<int>{0, 5, 6}
                   : n == 1 ? std::vector<int>{0} : std::vector<int>{})
            memcpy(&r.args[i], args[i], 8);
        records.push_back(r);
    }
    call_hook("launch");
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* fn, hipFuncAttribute a, int v)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (a == hipFuncAttributeMaxDynamicSharedMemorySize) {
        if (v > 160 << 10) return last_error = hipErrorInvalidValue;
        lds_limit[fn] = v;
    }
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t lds)
{
    *n = lds ? std::max(1, std::min(2048 / threads, (int)((160 << 10) / lds))) : 2048 / threads;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    *p = reinterpret_cast<void*>(next_address);
    buffers.emplace_back(next_address, bytes);
    next_address += (bytes + 0xfffff) & ~0xfffffull;
    return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "recorded error"; }
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    *p = reinterpret_cast<void*>(1ull << 44);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    call_hook("query");
    return hipSuccess;
}
}
