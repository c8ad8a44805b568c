// Stands in for the HIP runtime so that the library's host side runs without a GPU: every launch is recorded (kernel,
// grid, block, dynamic LDS) and checked against what the runtime would accept, nothing is executed.  Loaded with
// RTLD_GLOBAL in front of the library, its symbols are the ones the library binds to.
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdio>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <utility>

struct Dim3 { uint32_t x, y, z; };

namespace {
std::mutex mu;
std::condition_variable cv;
std::string records;
std::map<const void*, std::string> names;
std::map<std::pair<int, const void*>, long> lds_allowed;   // (device, kernel) -> dynamic LDS asked for
thread_local int device = 0;
struct Call { Dim3 grid, block; size_t lds; void* stream; };
thread_local Call call;
bool hold_next_grant = false;
int launches = 0;
thread_local int last_error = 0;
std::thread turner;
std::atomic<bool> turning;
}  // namespace

extern "C" {
void stub_set_device(int d) { device = d; }
// the next hipFuncSetAttribute returns only after another thread has launched a kernel (or two seconds later)
void stub_hold_next_grant() { std::lock_guard<std::mutex> g(mu); hold_next_grant = true; }
const char* stub_records() { return records.c_str(); }
void stub_clear() { std::lock_guard<std::mutex> g(mu); records.clear(); }

// another thread gives an option one value and the other in turn, as fast as it can, until stub_turn_end
void stub_turn(int (*set_option)(int, int), int option, int one, int other) {
    turning = true;
    turner = std::thread([=] {
        while (turning) { set_option(option, one); set_option(option, other); }
    });
}
void stub_turn_end() { turning = false; turner.join(); }

void** __hipRegisterFatBinary(const void*) { static void* handle[1]; return handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) { call = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = call.grid; *block = call.block; *lds = call.lds; *stream = call.stream;
    return 0;
}
int hipGetDevice(int* d) { *d = device; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int hipDeviceSynchronize() { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return 0; }
int hipMemcpy(void*, const void*, size_t, int) { return 1; }
int hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(0x7000000000); return 0; }
int hipFuncSetAttribute(const void* fn, int, int value) {
    std::unique_lock<std::mutex> g(mu);
    lds_allowed[{device, fn}] = value;
    if (hold_next_grant) {
        hold_next_grant = false;
        const int before = launches;
        cv.wait_for(g, std::chrono::seconds(2), [&] { return launches != before; });
    }
    return 0;
}
int hipLaunchKernel(const void* fn, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
    std::lock_guard<std::mutex> g(mu);
    const auto it = lds_allowed.find({device, fn});
    const long allowed = it == lds_allowed.end() ? 65536 : it->second;
    const char* wrong = "";
    if ((long)lds > allowed) wrong = " LDS-NOT-ALLOWED";
    if ((uint64_t)grid.x * block.x >> 32 || grid.y > 65535 || grid.z > 65535) wrong = " GRID-TOO-LARGE";
    char line[256];
    snprintf(line, sizeof line, " %u %u %u %u %zu %d%s\n", grid.x, grid.y, grid.z, block.x, lds, device, wrong);
    records += names[fn] + line;
    ++launches;
    cv.notify_all();
    if (*wrong) last_error = 1;
    return *wrong ? 1 : 0;
}
}
