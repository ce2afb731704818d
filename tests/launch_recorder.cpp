// Stands in for the HIP runtime in host tests: the library's launches are written down and never run,
// so which kernels a call takes can be checked without a GPU (tests/routes.py loads it ahead of the
// library).  Pointers are never followed.
#include <cxxabi.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <string>

struct Dim3 {
    uint32_t x, y, z;
};

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static std::string g_log;
static Dim3 g_grid, g_block;
static size_t g_lds;
static void *g_stream;

extern "C" {

void recorder_clear(void) { g_log.clear(); }
// one line per launch: kernel (as declared, without its namespaces and arguments), grid, block, dynamic LDS
const char *recorder_text(void) { return g_log.c_str(); }

void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    int status = 0;
    std::string mangled = device;  // (_Float16 is newer than some demanglers: spelt as its older relative)
    for (size_t at; (at = mangled.find("DF16_")) != std::string::npos;) mangled.replace(at, 5, "Dh");
    char *plain = abi::__cxa_demangle(mangled.c_str(), nullptr, nullptr, &status);
    std::string name = status == 0 ? plain : device;
    free(plain);
    // "void lmkan::(anonymous namespace)::kernel<float, 16>(lmkan::Args)" -> "kernel<float, 16>"
    for (const char *space : {"(anonymous namespace)::", "lmkan::", "void "})
        for (size_t at; (at = name.find(space)) != std::string::npos;) name.erase(at, std::string(space).size());
    int depth = 0;
    for (size_t i = 0; i < name.size(); ++i) {
        depth += name[i] == '<' ? 1 : name[i] == '>' ? -1 : 0;
        if (name[i] == '(' && depth == 0) name.resize(i);
    }
    names()[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream)
{
    g_grid = grid, g_block = block, g_lds = lds, g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = g_grid, *block = g_block, *lds = g_lds, *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void *host, Dim3 grid, Dim3 block, void **, size_t lds, void *)
{
    char sizes[160];
    snprintf(sizes, sizeof(sizes), "\t%u,%u,%u\t%u\t%zu\n", grid.x, grid.y, grid.z, block.x * block.y * block.z, lds);
    g_log += names()[host] + sizes;
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *dev)
{
    *dev = 0;
    return 0;
}
int hipGetSymbolAddress(void **p, const void *)
{
    *p = reinterpret_cast<void *>(uintptr_t(1) << 40);
    return 0;
}
int hipDeviceGetAttribute(int *v, int, int)
{
    *v = 256;
    return 0;
}
int hipEventCreate(void **) { return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *)
{
    *ms = 1.0f;
    return 0;
}
}
