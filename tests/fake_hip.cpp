// A HIP runtime that computes nothing: enough of it for the library's host code to plan and to enqueue on a machine
// without a GPU, with a chosen amount of device memory.  Loaded with RTLD_GLOBAL before the library, so that the
// library's references bind here.  Addresses it hands out are never dereferenced.
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
#include <string>

#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

namespace {
std::map<const void*, std::string> g_names;
std::map<uintptr_t, size_t> g_live;
std::string g_log;
size_t g_limit = SIZE_MAX, g_live_bytes = 0;
uintptr_t g_next = (uintptr_t)1 << 40;
dim3 g_grid, g_block;
size_t g_shared = 0;
hipStream_t g_stream = nullptr;
}  // namespace

extern "C" {
void fake_device_memory(size_t bytes) { g_limit = bytes; }
size_t fake_live_bytes() { return g_live_bytes; }
// What was called since the last time, one line each: "malloc BYTES", "malloc BYTES failed", "free", "launch KERNEL GRIDX GRIDY"
// (the generic kernel: followed by A, B, C, M, N, K, lda, ldb, ldc).
const char* fake_take_log()
{
    static std::string out;
    out.swap(g_log);
    g_log.clear();
    return out.c_str();
}

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    g_grid = grid; g_block = block; g_shared = shared; g_stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream)
{
    *grid = g_grid; *block = g_block; *shared = g_shared; *stream = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t)
{
    g_log += "launch " + g_names[f] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y);
    if (g_names[f].find("generic_gemm_kernel") != std::string::npos)      // (A, B, C, M, N, K, lda, ldb, ldc, col_major): three pointers, six int64
        for (int i = 0; i < 9; ++i) g_log += " " + std::to_string(*(const int64_t*)args[i]);
    g_log += "\n";
    return hipSuccess;
}
hipError_t hipGetDevice(int* dev) { *dev = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)((uintptr_t)1 << 39); return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes)
{
    const bool ok = bytes <= g_limit && g_live_bytes <= g_limit - bytes;
    g_log += "malloc " + std::to_string(bytes) + (ok ? "\n" : " failed\n");
    if (!ok) return hipErrorOutOfMemory;
    *p = (void*)g_next;
    g_live[g_next] = bytes;
    g_live_bytes += bytes;
    g_next += (bytes + 511) / 256 * 256;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    auto it = g_live.find((uintptr_t)p);
    if (it == g_live.end()) return hipErrorInvalidValue;
    g_live_bytes -= it->second;
    g_live.erase(it);
    g_log += "free\n";
    return hipSuccess;
}
}
