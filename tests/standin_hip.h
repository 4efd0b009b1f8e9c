// A HIP runtime of counters, to run the library's host code without a GPU: each stream counts
// what was enqueued on it, events carry what their recording implies, and one call can be made
// to fail.  Memory is host memory.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

namespace {

typedef std::map<int, int> Known;   // stream -> operations known to be finished with it
struct Stream { int id, n = 0; Known known; };
struct Event { Known known; };

std::vector<Stream *> g_streams;
Known g_finished;
int g_calls = 0, g_fail_at = -1, g_bad = 0;
bool g_failed = false;

Stream *as(hipStream_t s) { return reinterpret_cast<Stream *>(s); }
Event *as(hipEvent_t e) { return reinterpret_cast<Event *>(e); }

void merge(Known &a, const Known &b) {
    for (auto &kv : b) a[kv.first] = std::max(a[kv.first], kv.second);
}

bool fails() {   // whether this call of the step is the one that fails
    if (g_calls++ != g_fail_at) return false;
    g_failed = true;
    return true;
}

hipError_t put(hipStream_t s) {
    if (fails()) return hipErrorUnknown;
    Stream *st = as(s);
    st->known[st->id] = ++st->n;
    return hipSuccess;
}

bool idle() {   // whether everything enqueued has been waited for
    for (Stream *s : g_streams)
        if (g_finished[s->id] < s->n) return false;
    return true;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    return *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024, hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipFree(void *p) {
    if (!idle()) ++g_bad, std::printf("memory freed with work in flight, call %d failed\n", g_fail_at);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    const hipError_t e = put(st);
    if (e == hipSuccess) std::memcpy(d, s, n);
    return e;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
    const hipError_t e = put(st);
    if (e == hipSuccess) std::memset(d, v, n);
    return e;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    if (fails()) return hipErrorUnknown;
    Stream *st = new Stream;
    st->id = (int)g_streams.size();
    g_streams.push_back(st);
    *s = reinterpret_cast<hipStream_t>(st);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = reinterpret_cast<hipEvent_t>(new Event), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (fails()) return hipErrorUnknown;
    as(e)->known = as(s)->known;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (fails()) return hipErrorUnknown;
    merge(as(s)->known, as(e)->known);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (fails()) return hipErrorUnknown;
    merge(g_finished, as(s)->known);
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
}
