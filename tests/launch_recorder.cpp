// A HIP runtime for tests of the host side: memory is host memory, kernels do
// not run, and every launch (kernel, grid, block, dynamic LDS), every limit set
// on a kernel and every byte of device memory is recorded.  Loaded before the
// library with RTLD_GLOBAL, so that the library binds to these functions.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Rec {
    std::map<const void *, std::string> names;
    std::vector<std::string> log;
    std::map<void *, size_t> device;
    size_t device_bytes = 0;
};
Rec &rec() {
    static Rec r;
    return r;
}
std::string name_of(const void *f) {
    auto it = rec().names.find(f);
    return it == rec().names.end() ? "?" : it->second;
}
dim3 cfg_grid, cfg_block;
size_t cfg_shared;
hipStream_t cfg_stream;
char something[64];
template <typename T>
hipError_t give(T *out) {
    *out = (T)something;
    return hipSuccess;
}

}  // namespace

extern "C" {

int rec_size() { return (int)rec().log.size(); }
const char *rec_line(int k) { return rec().log[k].c_str(); }
void rec_clear() { rec().log.clear(); }
size_t rec_device_bytes() { return rec().device_bytes; }

void **__hipRegisterFatBinary(const void *) { return (void **)something; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) {
    rec().names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
    cfg_grid = grid;
    cfg_block = block;
    cfg_shared = shared;
    cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s) {
    *grid = cfg_grid;
    *block = cfg_block;
    *shared = cfg_shared;
    *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t shared, hipStream_t) {
    rec().log.push_back("launch " + name_of(f) + " " + std::to_string((uint64_t)grid.x * grid.y * grid.z) + " " +
                        std::to_string(block.x * block.y * block.z) + " " + std::to_string(shared));
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value) {
    rec().log.push_back("limit " + name_of(f) + " " + std::to_string(value));
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) {
    *p = std::calloc(n ? n : 1, 1);
    if (!*p) return hipErrorOutOfMemory;
    rec().device[*p] = n;
    rec().device_bytes += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = rec().device.find(p);
    if (it != rec().device.end()) {
        rec().device_bytes -= it->second;
        rec().device.erase(it);
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = std::calloc(n, 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { return give(p); }

hipError_t hipGetDeviceCount(int *n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return give(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return give(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return give(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.f;
    return hipSuccess;
}

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return give(g); }
hipError_t hipStreamGetCaptureInfo_v2(hipStream_t, hipStreamCaptureStatus *st, unsigned long long *, hipGraph_t *g,
                                      const hipGraphNode_t **deps, size_t *n) {
    *st = hipStreamCaptureStatusActive;
    *deps = nullptr;
    *n = 0;
    return give(g);
}
hipError_t hipStreamUpdateCaptureDependencies(hipStream_t, hipGraphNode_t *, size_t, unsigned) { return hipSuccess; }
hipError_t hipGraphAddEventRecordNode(hipGraphNode_t *node, hipGraph_t, const hipGraphNode_t *, size_t, hipEvent_t) {
    return give(node);
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) { return give(e); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

}  // extern "C"
