// A stand-in for the HIP runtime calls that libsbh makes, for tests of its host code without a GPU.
// Loaded (RTLD_GLOBAL) before the library, its definitions are the ones the library binds to.
// Device pointers are numbers that nothing dereferences, kernels do not run, and every call is
// written to a log that the test reads.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

namespace {

struct Dim3 {
    uint32_t x, y, z;
};

struct Call {   // of a <<< >>> launch
    Dim3 grid, block;
    size_t lds;
    void* stream;
} g_call;
std::string g_log;
// of every launch (of workgroups of g_block, if that is not 0): its first g_nargs arguments' leading 8 bytes
std::vector<uint64_t> g_args;
std::vector<uint32_t> g_blocks;    // and its workgroup's size
int g_nargs = 0;
uint32_t g_block = 0;
uintptr_t g_next = (uintptr_t)1 << 40, g_event = 0x1000;
void* g_capturing = (void*)-1;     // the stream under capture
int g_done = 1, g_device = 0, g_refuse = 0, g_error = 0;
unsigned char g_info[512];         // what a copy to the host finds

constexpr int kOutOfMemory = 2, kInvalidConfiguration = 9, kNotReady = 600;

void note(const char* what, const void* a, unsigned long long b, const void* c)
{
    char line[160];
    std::snprintf(line, sizeof(line), "%s %llx %llu %llx dev%d\n", what, (unsigned long long)(uintptr_t)a, b,
                  (unsigned long long)(uintptr_t)c, g_device);
    g_log += line;
}

}  // namespace

extern "C" {

// --- for the test
const char* stand_in_log() { return g_log.c_str(); }
void stand_in_clear() { g_log.clear(); g_args.clear(); g_blocks.clear(); }
void stand_in_error(int e) { g_error = e; }   // the runtime's last error
void stand_in_events_done(int done) { g_done = done; }
void stand_in_capture(void* stream) { g_capturing = stream; }
void stand_in_refuse(int allocations) { g_refuse = allocations; }   // the next ones fail
void stand_in_info(const void* p, int bytes) { std::memcpy(g_info, p, (size_t)bytes); }
void stand_in_copy_args(int n, int block) { g_nargs = n; g_block = (uint32_t)block; }
uint64_t stand_in_arg(int i) { return g_args[(size_t)i]; }
unsigned stand_in_block(int i) { return g_blocks[(size_t)i]; }

// --- the runtime's
int hipGetDevice(int* d) { *d = g_device; return 0; }
int hipSetDevice(int d) { g_device = d; return 0; }
int hipGetLastError() { const int e = g_error; g_error = 0; return e; }
int hipDeviceSynchronize() { note("devicesync", nullptr, 0, nullptr); return 0; }
int hipStreamSynchronize(void* s) { note("streamsync", nullptr, 0, s); return 0; }
int hipStreamIsCapturing(void* s, int* st) { *st = s == g_capturing ? 1 : 0; return 0; }
int hipMallocAsync(void** p, size_t bytes, void* s)
{
    if (g_refuse > 0) {
        --g_refuse;
        note("refused", nullptr, bytes, s);
        return kOutOfMemory;
    }
    *p = (void*)g_next;
    g_next += (bytes + 0xFFF) & ~(size_t)0xFFF;
    note("malloc", *p, bytes, s);
    return 0;
}
int hipFreeAsync(void* p, void* s) { note("free", p, 0, s); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)(g_event += 16); return 0; }
int hipEventRecord(void* e, void* s) { note("record", e, 0, s); return 0; }
int hipEventQuery(void*)
{
    if (!g_done) g_error = kNotReady;
    return g_done ? 0 : kNotReady;
}
int hipEventSynchronize(void* e) { note("eventsync", e, 0, nullptr); return 0; }
int hipEventDestroy(void* e) { note("destroy", e, 0, nullptr); return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned) { note("wait", e, 0, s); return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipMemcpyAsync(void* dst, const void*, size_t bytes, int kind, void*)
{
    if (kind == 2) std::memcpy(dst, g_info, bytes);   // device to host
    return 0;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* s)
{
    g_call = {grid, block, lds, s};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** s)
{
    *grid = g_call.grid;
    *block = g_call.block;
    *lds = g_call.lds;
    *s = g_call.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t, void* s)
{
    const uint64_t threads = (uint64_t)grid.x * block.x;
    note(threads >> 32 ? "toolarge" : "launch", f, threads, s);
    const bool keep = g_nargs > 0 && (g_block == 0 || block.x == g_block);
    if (keep) g_blocks.push_back(block.x);
    for (int i = 0; i < g_nargs && keep; ++i) {
        uint64_t v = 0;
        std::memcpy(&v, args[i], 8);
        g_args.push_back(v);
    }
    if (threads >> 32) g_error = kInvalidConfiguration;   // the limit of a launch along x
    return g_error;
}

}  // extern "C"
