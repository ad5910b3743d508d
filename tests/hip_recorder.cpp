// A stand-in for the HIP runtime that runs nothing on any device: it hands out addresses, counts and names what is launched,
// refuses grids that the runtime refuses, and fails calls on request.  Loaded into the global scope before libkge.so, it lets a test on the CPU see what
// the library's host code enqueues, in which order, and what it does when a call of the runtime fails.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <string>

namespace {

struct Dim3 { uint32_t x, y, z; };
struct Module { int id; };
struct Kernel { int module; std::string name; };
struct Graph { int kernels; };

std::map<const void*, Kernel>& kernels() { static std::map<const void*, Kernel> m; return m; }
std::map<void*, size_t>& sizes() { static std::map<void*, size_t> m; return m; }
std::string& events() { static std::string s; return s; }
std::map<std::string, int>& failing() { static std::map<std::string, int> m; return m; }  // calls until the one that fails
void* capturing = nullptr;
int captured = 0, modules = 0, pending = 0, waits = 0;

int outcome(const char* call) {
    auto it = failing().find(call);
    if (it == failing().end() || --it->second != 0) return 0;
    failing().erase(it);
    return pending = 2;  // (out of memory)
}

struct Event { bool recorded; };
void record(void* e) { if (e) static_cast<Event*>(e)->recorded = true; }

int launch(const void* f, Dim3 grid, Dim3 block) {
    const Kernel& k = kernels()[f];
    if (const int e = outcome("hipLaunchKernel")) return e;
    const uint64_t most = UINT32_MAX;  // threads per dimension
    if (!grid.x || !grid.y || !grid.z || (uint64_t)grid.x * block.x > most || (uint64_t)grid.y * block.y > most || grid.y > 65535) {
        events() += "refused " + k.name + "\n";
        return pending = 9;  // (invalid configuration)
    }
    if (capturing) { ++captured; return 0; }
    char line[64];
    snprintf(line, sizeof(line), "kernel %d ", k.module);
    events() += line + k.name;
    snprintf(line, sizeof(line), " %u\n", grid.x * grid.y * grid.z);
    events() += line;
    return 0;
}

}  // namespace

extern "C" {

// ---- for the test
const char* recorder_events() { return events().c_str(); }
void recorder_clear() { events().clear(); waits = 0; }
int recorder_waits() { return waits; }  // waits of one stream for another
void recorder_fail(const char* call, int nth) { failing()[call] = nth; }

// ---- the runtime
void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(new Module{modules++}); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void** m, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels()[f] = {reinterpret_cast<Module*>(m)->id, name};
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static Dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*) { return launch(f, grid, block); }
int hipExtLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*, void* start, void* stop, int) {
    const int e = launch(f, grid, block);
    if (!e) { record(start); record(stop); }
    return e;
}
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
const char* hipGetErrorString(int) { return "asked for by the test"; }
int hipGetLastError() { const int e = pending; pending = 0; return e; }
int hipGetSymbolAddress(void** p, const void*) { static char area[1 << 23]; *p = area; return 0; }
int hipMalloc(void** p, size_t n) {
    if (const int e = outcome("hipMalloc")) return e;
    *p = mmap(nullptr, n, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);  // (addresses that nothing may touch)
    if (*p == MAP_FAILED) return pending = 2;
    sizes()[*p] = n;
    return 0;
}
int hipFree(void* p) {
    if (p) munmap(p, sizes()[p]);
    return 0;
}
int hipMemset(void*, int, size_t) { return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) {
    if (const int e = outcome("hipMemcpyAsync")) return e;
    events() += "copy\n";
    return 0;
}
int hipEventCreate(void** e) { *e = new Event{}; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = new Event{}; return 0; }
int hipEventDestroy(void* e) { delete static_cast<Event*>(e); return 0; }
int hipEventElapsedTime(float* ms, void* start, void* stop) {  // every kernel takes 1 ms
    if (!static_cast<Event*>(start)->recorded || !static_cast<Event*>(stop)->recorded) return pending = 400;  // (invalid handle)
    *ms = 1.f;
    return 0;
}
int hipEventRecord(void* e, void*) {
    record(e);
    return outcome("hipEventRecord");
}
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { ++waits; return outcome("hipStreamWaitEvent"); }
int hipStreamIsCapturing(void* s, int* status) { *status = s && s == capturing; return 0; }
int hipStreamBeginCapture(void* s, int) {
    if (const int e = outcome("hipStreamBeginCapture")) return e;
    capturing = s;
    captured = 0;
    return 0;
}
int hipStreamEndCapture(void*, void** graph) {
    capturing = nullptr;
    *graph = nullptr;
    if (const int e = outcome("hipStreamEndCapture")) return e;
    *graph = new Graph{captured};
    return 0;
}
int hipGraphInstantiate(void** exec, void* graph, void*, char*, size_t) {
    *exec = nullptr;
    if (const int e = outcome("hipGraphInstantiate")) return e;
    *exec = new Graph(*static_cast<Graph*>(graph));
    return 0;
}
int hipGraphDestroy(void* graph) { delete static_cast<Graph*>(graph); return 0; }
int hipGraphExecDestroy(void* exec) { delete static_cast<Graph*>(exec); return 0; }
int hipGraphUpload(void*, void*) { return outcome("hipGraphUpload"); }
int hipGraphLaunch(void* exec, void*) {
    if (const int e = outcome("hipGraphLaunch")) return e;
    char line[64];
    snprintf(line, sizeof(line), "graph %d\n", static_cast<Graph*>(exec)->kernels);
    events() += line;
    return 0;
}

}  // extern "C"
