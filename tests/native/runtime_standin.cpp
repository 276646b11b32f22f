// Stands in for the HIP runtime (loaded ahead of it), so that submission can be followed without a GPU: nothing is computed, but streams, events and the host link
// keep time, kernels of the library that write time stamps and completion flags write them, and every call is noted.
//   a kernel takes 5 us, a stamp 2 us, the link brings 53 bytes a ns, one transfer at a time; the host takes no time
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "kernels.hpp"
#include "small_net.hpp"

using namespace strait;

static std::mutex mu;
static std::map<const void*, std::string> kernels;
static std::map<const void*, long long> stream_ns, event_ns;
static long long link_ns, now_ns;                          // the link is free, the host is there
static std::string notes;
static thread_local struct { dim3 grid, block; size_t lds; hipStream_t stream; } call;
static std::atomic<bool> held{false};                      // results are not there yet
static std::vector<std::pair<uint32_t*, uint32_t>> to_set;
static std::atomic<int> held_stamp{-1};                    // nor is this stamp
static std::vector<std::pair<uint64_t*, uint64_t>> to_stamp;
static char streams_made[64];
static int n_streams_made;

static void note(const char* format, ...) {
    char line[512];
    va_list a;
    va_start(a, format);
    vsnprintf(line, sizeof line, format, a);
    va_end(a);
    notes += line;
    notes += '\n';
}
static long long& clock_of(hipStream_t s) {
    long long& t = stream_ns[s];
    return t = std::max(t, now_ns);
}
static void set_flag(uint32_t* flag, uint32_t seq) {
    if (held) to_set.push_back({flag, seq});
    else __atomic_store_n(flag, seq, __ATOMIC_RELEASE);
}
static void stamp(HostControl* ctl, int which, long long ns) {
    if (which == held_stamp) to_stamp.push_back({&ctl->stamp[which], (uint64_t)(ns / 10) + 1});
    else __atomic_store_n(&ctl->stamp[which], (uint64_t)(ns / 10) + 1, __ATOMIC_RELEASE);
}
static long long transfer(hipStream_t s, size_t bytes) {   // returns its start
    long long& t = clock_of(s);
    const long long start = std::max(t, link_ns);
    link_ns = t = start + (long long)(bytes / 53.0);
    return start;
}

extern "C" {

const char* standin_notes() {                              // since it was asked last
    static std::string given;
    std::lock_guard<std::mutex> lk(mu);
    given = std::move(notes);
    notes.clear();
    return given.c_str();
}
void standin_idle() {                                      // everything that was enqueued is done
    std::lock_guard<std::mutex> lk(mu);
    for (auto& s : stream_ns) now_ns = std::max(now_ns, s.second);
}
void standin_hold() { held = true; }
void standin_hold_stamp(int which) { held_stamp = which; }
void standin_release() {
    std::lock_guard<std::mutex> lk(mu);
    held = false;
    held_stamp = -1;
    for (auto& f : to_stamp) __atomic_store_n(f.first, f.second, __ATOMIC_RELEASE);
    to_stamp.clear();
    for (auto& f : to_set) __atomic_store_n(f.first, f.second, __ATOMIC_RELEASE);
    to_set.clear();
}

void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    if (strstr(name, "strait")) kernels[f] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) { call = {grid, block, lds, stream}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = call.grid; *block = call.block; *lds = call.lds; *stream = call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t s) {
    std::lock_guard<std::mutex> lk(mu);
    const std::string& name = kernels[f];
    auto is = [&](const char* part) { return name.find(part) != std::string::npos; };
    auto finished = [&](HostControl* ctl, unsigned chunks, unsigned seq, long long ns) {
        stamp(ctl, STAMP_DONE, ns);
        for (unsigned c = 0; c < chunks; ++c) set_flag(&ctl->flag[c], seq);
    };
    long long& t = clock_of(s);
    if (is("stamp_kernel")) {
        HostControl* ctl = *(HostControl**)args[0];
        const int which = *(int*)args[1];
        const unsigned n4 = *(unsigned*)args[4], seq = *(unsigned*)args[5];
        if (n4) memcpy(*(void**)args[3], *(void**)args[2], n4 * 4);
        note("stamp %d %p %lld", which, (void*)s, t);
        stamp(ctl, which, t);
        if (seq) set_flag(&ctl->k1_seq, seq);
        t += 2000;
    } else if (is("copy_in_kernel")) {
        HostControl* ctl = *(HostControl**)args[6];
        const int piece = *(int*)args[8];
        const size_t bytes = *(size_t*)args[2] * 4;
        const long long start = transfer(s, bytes);
        note("copy_in %zu %p %lld grid %u", bytes, (void*)s, start, grid.x);
        stamp(ctl, STAMP_PIECES + 2 * piece, start);
        stamp(ctl, STAMP_PIECES + 2 * piece + 1, t);
    } else if (is("copy_out_kernel")) {
        HostControl* ctl = *(HostControl**)args[6];
        const size_t bytes = *(size_t*)args[2];
        note("copy_out %zu %p %lld grid %u", bytes, (void*)s, t, grid.x);
        stamp(ctl, *(int*)args[9] ? STAMP_D2H0 : STAMP_K1, t);
        t += (long long)(bytes / 53.0);
        finished(ctl, *(unsigned*)args[5], *(unsigned*)args[8], t);
    } else if (is("classify_out_kernel") || is("small_net_kernel")) {
        const ClassifyOut& p = is("small_net") ? ((SmallNet*)args[0])->out : *(ClassifyOut*)args[0];
        note("kernel %s %p %lld grid %u", name.c_str(), (void*)s, t, grid.x);
        t += 5000;
        stamp(p.ctl, STAMP_K1, t);
        finished(p.ctl, 1, p.seq, t);
    } else {
        note("kernel %s %p %lld grid %u block %u", name.c_str(), (void*)s, t, grid.x, block.x);
        t += 5000;
    }
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t s) {
    std::lock_guard<std::mutex> lk(mu);
    memcpy(dst, src, n);
    if (kind == hipMemcpyHostToDevice) note("memcpy %zu %p %lld", n, (void*)s, transfer(s, n));
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::mutex> lk(mu);
    event_ns[e] = clock_of(s);
    note("record %p %p %lld", (void*)e, (void*)s, event_ns[e]);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    std::lock_guard<std::mutex> lk(mu);
    long long& t = clock_of(s);
    t = std::max(t, event_ns[e]);
    note("wait %p %p %lld", (void*)e, (void*)s, t);
    return hipSuccess;
}
static hipError_t memory(void** p, size_t n) {
    n = (n + 4095) / 4096 * 4096;
    return (*p = aligned_alloc(4096, n)) ? (memset(*p, 0, std::min<size_t>(n, 1u << 20)), hipSuccess) : hipErrorOutOfMemory;
}
hipError_t hipMalloc(void** p, size_t n) { return memory(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return memory(p, n); }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) { memcpy(dst, src, n); return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)&streams_made[n_streams_made++ % 64]; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void*)e); return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) { *c = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return held || held_stamp >= 0 ? hipErrorNotReady : hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}
