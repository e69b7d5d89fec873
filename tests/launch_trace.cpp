// The HIP runtime calls liblca makes, as far as they are needed to see which kernels a call launches, without a GPU:
// tests/launches.py links the library's objects with this file instead of with the runtime.  Nothing runs; a launch is
// a line "kernel grid block lds" (names demangled, without their argument lists).
#include <cxxabi.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

struct dim3 { uint32_t x, y, z; };

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static std::string g_log;
static int32_t g_mla[28];            // the parameter block of the last attn_mla_kernel launch, its first 112 bytes
static dim3 g_grid, g_block;
static size_t g_lds;

extern "C" {

const char *trace_log() { return g_log.c_str(); }
void trace_reset() { g_log.clear(); }
const int32_t *trace_mla_params() { return g_mla; }

void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    int status = 0;
    char *d = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    std::string s = status == 0 ? d : device;
    std::free(d);
    for (const char *drop : {"void ", "lca::", "(anonymous namespace)::"})
        for (size_t at; (at = s.find(drop)) != std::string::npos;) s.erase(at, std::strlen(drop));
    names()[host] = s.substr(0, s.find('('));
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *)
{
    g_grid = grid; g_block = block; g_lds = lds;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = g_grid; *block = g_block; *lds = g_lds; *stream = nullptr;
    return 0;
}
int hipLaunchKernel(const void *host, dim3 grid, dim3 block, void **args, size_t lds, void *)
{
    if (names()[host].rfind("attn_mla_kernel", 0) == 0) std::memcpy(g_mla, args[0], sizeof g_mla);
    char numbers[96];
    std::snprintf(numbers, sizeof numbers, "\t%llu\t%llu\t%zu\n", (unsigned long long)grid.x * grid.y * grid.z,
                  (unsigned long long)block.x * block.y * block.z, lds);
    g_log += names()[host] + numbers;
    return 0;
}
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "no error"; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int *value, int, int) { *value = 256; return 0; }       // only the number of CUs is asked for
int hipGetSymbolAddress(void **p, const void *) { *p = reinterpret_cast<void *>(0x10000); return 0; }

}
