// The HIP entry points that librmsnl.so uses, as a recorder: nothing is launched, every launch is noted with its kernel's
// name, grid and stream, memory is a range of numbers, and the state that the library asks for (a stream under capture,
// a failing allocation) is set by the test.  Loaded with RTLD_GLOBAL in front of the library, whose references then bind here.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <unistd.h>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

namespace {
struct Dim { uint32_t x, y, z; };
struct Config { Dim grid, block; size_t lds; void* stream; };
struct Watch { std::string name; int arg, bytes; };
std::recursive_mutex mu;
std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
std::set<void*> capturing;
std::vector<Watch> watched;
std::string log_text;
uintptr_t next_address = uintptr_t(1) << 40;
int fail_mallocs = 0, mallocs = 0, launch_pause_us = 0;
size_t malloc_bytes = 0;
thread_local std::vector<Config> configs;
thread_local int last_error = 0;
int error(int e) { if (e) last_error = e; return e; }
}

extern "C" {
// ---- what a test sets and reads
void rec_capture(void* stream, int on) { std::lock_guard<std::recursive_mutex> l(mu); if (on) capturing.insert(stream); else capturing.erase(stream); }
void rec_launch_pause(int us) { launch_pause_us = us; }
void rec_fail_mallocs(int n) { fail_mallocs = n; }
int rec_mallocs() { return mallocs; }
size_t rec_malloc_bytes() { return malloc_bytes; }
void rec_watch(const char* name, int arg, int bytes) { std::lock_guard<std::recursive_mutex> l(mu); watched.push_back({name, arg, bytes}); }
const char* rec_take() { static std::string out; std::lock_guard<std::recursive_mutex> l(mu); out.swap(log_text); log_text.clear(); return out.c_str(); }

// ---- HIP
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    names()[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void* stream) { configs.push_back({grid, block, lds, stream}); return 0; }
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* lds, void** stream)
{
    const Config c = configs.back();
    configs.pop_back();
    *grid = c.grid; *block = c.block; *lds = c.lds; *stream = c.stream;
    return 0;
}
int hipLaunchKernel(const void* fn, Dim grid, Dim block, void** args, size_t lds, void* stream)
{
    if (launch_pause_us) usleep(launch_pause_us);        // (outside the lock: other threads' launches may come in between)
    if (uint64_t(grid.x) * block.x >= (uint64_t(1) << 32) || block.x > 1024 || grid.x == 0) return error(9);
    std::lock_guard<std::recursive_mutex> l(mu);
    const std::string& n = names()[fn];
    char line[400];
    snprintf(line, sizeof line, "%s %u %u %zu %zu", n.c_str(), grid.x, block.x, lds, size_t(stream));
    log_text += line;
    for (const Watch& w : watched)
        if (n.find(w.name) != std::string::npos)
            for (int b = 0; b < w.bytes; b += 8) {
                uint64_t v;
                memcpy(&v, static_cast<const char*>(args[w.arg]) + b, 8);
                snprintf(line, sizeof line, " %llu", (unsigned long long)v);
                log_text += line;
            }
    log_text += '\n';
    return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "recorded"; }
int hipMalloc(void** p, size_t n)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    ++mallocs;
    if (fail_mallocs > 0) { --fail_mallocs; return error(2); }
    malloc_bytes += n;
    *p = reinterpret_cast<void*>(next_address);
    next_address += (n + 4095) / 4096 * 4096 + (1 << 20);
    return 0;
}
int hipFree(void*) { return 0; }
int hipMemset(void*, int, size_t) { return 0; }
int hipGetSymbolAddress(void** p, const void* symbol)
{
    static std::map<const void*, uintptr_t> at;
    std::lock_guard<std::recursive_mutex> l(mu);
    *p = reinterpret_cast<void*>(at.emplace(symbol, (uintptr_t(1) << 39) + at.size() * (uintptr_t(1) << 32)).first->second);
    return 0;
}
int hipStreamIsCapturing(void* s, int* status)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    if (!s && !capturing.empty()) return error(906);     // hipErrorStreamCaptureImplicit
    *status = capturing.count(s) ? 1 : 0;
    return 0;
}
int hipThreadExchangeStreamCaptureMode(int* mode) { static thread_local int now = 0; const int was = now; now = *mode; *mode = was; return 0; }
int hipEventCreate(void** e) { *e = e; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return 0; }
}
