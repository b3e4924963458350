// A stand-in for the HIP runtime, for tests of the library's host side on a machine without a GPU: every call succeeds,
// nothing runs, and the launched kernels' names and grids are kept in order.  Load it with RTLD_GLOBAL ahead of libmpcpipe.so.
#include <atomic>
#include <cstddef>
#include <cstdio>
#include <map>
#include <string>
#include <thread>
#include <vector>

struct dim { unsigned x, y, z; };

static std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> m; return m; }
static std::vector<std::string> launched;
static thread_local struct { dim grid, block; size_t shared; void* stream; } config;

extern "C" {

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim*, dim*, int*) { kernels()[host] = name; }
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim grid, dim block, size_t shared, void* stream) { config = { grid, block, shared, stream }; return 0; }
int __hipPopCallConfiguration(dim* grid, dim* block, size_t* shared, void** stream)
{
    *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void* host, dim grid, dim, void**, size_t, void*)
{
    launched.push_back(kernels()[host] + "@" + std::to_string(grid.x));
    return 0;
}

int hipGetLastError() { return 0; }
int hipSetDevice(int) { return 0; }
int hipGetDevicePropertiesR0600(void*, int) { return 1; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** at, const void*) { *at = (void*)0x100000; return 0; }

static void* handle() { static std::atomic<size_t> n{ 0x1000 }; return (void*)(n += 16); }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = handle(); return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { *e = handle(); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = handle(); return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0; return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = handle(); return 0; }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { *e = handle(); return 0; }
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }

// ---- for the tests ----
// the kernels launched since the last call of this, a line each: name@workgroups along x
size_t fake_launches(char* out, size_t cap)
{
    std::string all;
    for (const std::string& n : launched) all += n + "\n";
    launched.clear();
    return (size_t)std::snprintf(out, cap, "%s", all.c_str());
}
// a thread that calls set(a, min_tiles) and set(b, min_tiles) in turn until stopped
static std::thread toggler;
static std::atomic<bool> stop;
void fake_toggle_start(int (*set)(int, int), int a, int b, int min_tiles)
{
    stop = false;
    toggler = std::thread([=] { while (!stop) { set(a, min_tiles); set(b, min_tiles); } });
}
void fake_toggle_stop() { stop = true; toggler.join(); }

}  // extern "C"
