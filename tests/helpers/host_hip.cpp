// A stand-in for the HIP runtime calls that libu1ml.so makes, for checks of its
// host side without a GPU: nothing runs, every kernel launch is recorded and
// held to the documented launch limits.  Loaded with RTLD_GLOBAL before
// libu1ml.so, whose calls then resolve to it.
#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    const char* name;  // mangled kernel name
    uint32_t grid[3], block[3];
    uint64_t lds;
};

static std::vector<Launch> g_log;
static std::map<const void*, std::string> g_names;
static thread_local Dim3 t_grid, t_block;
static thread_local size_t t_lds;
static thread_local void* t_stream;
static uintptr_t g_handle = 0x1000;
static int g_error;

static int handle(void** out)
{
    *out = (void*)(g_handle += 16);
    return 0;
}

extern "C" {

size_t host_hip_launches() { return g_log.size(); }
const Launch* host_hip_launch(size_t i) { return &g_log[i]; }
void host_hip_clear() { g_log.clear(); }

void** __hipRegisterFatBinary(const void*)
{
    static void* module;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* st)
{
    t_grid = g, t_block = b, t_lds = lds, t_stream = st;
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** st)
{
    *g = t_grid, *b = t_block, *lds = t_lds, *st = t_stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void**, size_t lds, void*)
{
    const uint64_t limit = 1ull << 32;  // work-items along an axis
    if (!g.x || !g.y || !g.z || g.x * (uint64_t)b.x >= limit || g.y > 65535u || g.z > 65535u ||
        b.x * (uint64_t)b.y * b.z > 1024 || lds > 160 * 1024)
        return g_error = 9;  // hipErrorInvalidConfiguration
    g_log.push_back(Launch{g_names[f].c_str(), {g.x, g.y, g.z}, {b.x, b.y, b.z}, lds});
    return 0;
}
int hipExtLaunchKernel(const void* f, Dim3 g, Dim3 b, void** a, size_t lds, void* st, void*, void*, int)
{
    return hipLaunchKernel(f, g, b, a, lds, st);
}
int hipDeviceGetAttribute(int* v, int, int)
{
    *v = 160 * 1024;
    return 0;
}
int hipGetDevice(int* d)
{
    *d = 0;
    return 0;
}
int hipGetLastError()
{
    const int e = g_error;
    g_error = 0;
    return e;
}
const char* hipGetErrorString(int e) { return e == 9 ? "invalid configuration argument" : "error"; }
int hipGetSymbolAddress(void** p, const void*) { return handle(p); }
int hipMalloc(void** p, size_t) { return handle(p); }
int hipFree(void*) { return 0; }
int hipMemcpy(void* dst, const void*, size_t n, int kind)
{
    if (kind == 2) std::memset(dst, 0, n);  // device to host
    return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { return handle(s); }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { return handle(g); }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { return handle(e); }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipGraphLaunch(void*, void*) { return 0; }
int hipEventCreate(void** e) { return handle(e); }
int hipEventCreateWithFlags(void** e, unsigned) { return handle(e); }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*)
{
    *ms = 1.0f;
    return 0;
}
}
