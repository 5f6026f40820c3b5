// A HIP runtime that runs nothing: it records the calls that the library's host code makes, keeps
// the order that streams and events give them, follows stream capture, lets a chosen call fail and
// gives every launch a duration. Loaded with RTLD_GLOBAL before liblooporbit.so, its functions
// take the place of libamdhip64's (tests/test_host_calls.py).
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
using Clock = std::map<hipStream_t, long>;  // launches of each stream that are known to precede
struct Event {
    Clock seen;
    unsigned long long capture = 0;
    double at = 0.0;
};
std::map<hipStream_t, Clock> g_clock;
std::map<hipStream_t, long> g_launched, g_waited;
std::map<hipStream_t, unsigned long long> g_capture;
std::map<const void*, std::string> g_names;
std::vector<std::pair<std::string, double>> g_cost;
std::vector<std::string> g_log;
std::string g_fail;
int g_fail_nth = 0;
uintptr_t g_next = 0x1000;
double g_now = 0.0;  // microseconds; launches follow one another
hipError_t g_last = hipSuccess;
struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t s;
} g_config;

hipError_t call(const std::string& line) {
    g_log.push_back(line);
    if (!g_fail.empty() && line.find(g_fail) != std::string::npos && --g_fail_nth == 0) {
        g_fail.clear();
        return g_last = hipErrorUnknown;
    }
    return hipSuccess;
}
std::string at(const char* what, hipStream_t s) {
    char b[160];
    snprintf(b, sizeof b, "%s @%lx", what, (unsigned long)(uintptr_t)s);
    return b;
}
hipError_t launch(const void* f, dim3 grid, void** args, hipStream_t s) {
    const std::string& name = g_names[f];
    char b[64];
    snprintf(b, sizeof b, " grid %u", grid.x);
    const hipError_t e = call(at(("launch " + name).c_str(), s) + b);
    if (e != hipSuccess) return e;
    if (name.find("k_xcc_probe") != std::string::npos)
        for (int i = 0; i < 8; ++i) (*static_cast<int**>(args[0]))[i] = 1;
    double us = 1.0;
    for (const auto& c : g_cost)
        if (name.find(c.first) != std::string::npos) us = c.second;
    g_now += us;
    g_clock[s][s] = ++g_launched[s];
    return hipSuccess;
}
}  // namespace

extern "C" {
// ---- the test's side
void rec_reset() {
    g_log.clear();
    g_clock.clear();
    g_launched.clear();
    g_waited.clear();
    g_fail.clear();
    g_last = hipSuccess;
}
long rec_log(char* out, long size) {
    std::string all;
    for (const auto& l : g_log) all += l + "\n";
    if ((long)all.size() < size) memcpy(out, all.c_str(), all.size() + 1);
    return (long)all.size() + 1;
}
void rec_fail(const char* what, int nth) {
    g_fail = what;
    g_fail_nth = nth;
}
void rec_cost(const char* name, double us) { g_cost.emplace_back(name, us); }
void rec_capture(hipStream_t s, unsigned long long id) { g_capture[s] = id; }
void rec_end_capture(unsigned long long id) {
    for (auto& c : g_capture)
        if (c.second == id) c.second = 0;
}
// Launches of other streams that neither precede later work of stream s nor were waited for.
long rec_unordered(hipStream_t s) {
    long n = 0;
    for (const auto& l : g_launched)
        if (l.first != s) n += l.second - std::max(g_clock[s][l.first], g_waited[l.first]);
    return n;
}

// ---- the library's side
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_names[f] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    g_config = {grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *s = g_config.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s) {
    return launch(f, grid, args, s);
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s, hipEvent_t, hipEvent_t,
                              int) {
    return launch(f, grid, args, s);
}
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
    return call("attribute");
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return call("func attribute"); }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static char scratch[256];
    *p = scratch;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    const hipError_t e = call("malloc");
    if (e == hipSuccess) *p = calloc(1, n + 256);
    return e;
}
hipError_t hipFree(void* p) {
    free(p);
    return call("free");
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    const hipError_t e = call("memcpy");
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return call("memcpy async");
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(g_next += 16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    const hipError_t e = call(at("stream synchronize", s));
    if (e == hipSuccess) g_waited[s] = g_launched[s];
    return e;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t s, hipStreamCaptureStatus* st, unsigned long long* id) {
    *id = g_capture[s];
    *st = *id ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    unsigned long long id;
    return hipStreamGetCaptureInfo(s, st, &id);
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new Event());
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    delete reinterpret_cast<Event*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    const hipError_t err = call(at("record", s));
    if (err == hipSuccess) *reinterpret_cast<Event*>(e) = {g_clock[s], g_capture[s], g_now};
    return err;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const hipError_t err = call(at("wait", s));
    if (err != hipSuccess) return err;
    const Event& ev = *reinterpret_cast<Event*>(e);
    if (g_capture[s] && ev.capture != g_capture[s]) return g_last = hipErrorStreamCaptureIsolation;
    g_capture[s] = ev.capture;  // a stream that waits for recorded work joins its capture
    for (const auto& c : ev.seen) {
        long& k = g_clock[s][c.first];
        if (c.second > k) k = c.second;
    }
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(1e-3 * (reinterpret_cast<Event*>(b)->at - reinterpret_cast<Event*>(a)->at));
    return hipSuccess;
}
}
