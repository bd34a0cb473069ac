// The HIP calls and kernel launches of the host runtime, on host memory: every call that
// enqueues something is recorded by name, and the n-th call of a name can be made to fail.
// Copies and fills are done at once; kernels do nothing.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "gsim_internal.h"

namespace {
std::string calls;                 // names, each followed by a space
std::map<std::string, int> fail_at;  // name -> calls until one fails

bool fails(const char* name) {
    calls += name;
    calls += ' ';
    auto it = fail_at.find(name);
    return it != fail_at.end() && --it->second == 0;
}
hipError_t call(const char* name) { return fails(name) ? hipErrorUnknown : hipSuccess; }
int launch(const char* name) { return fails(name) ? 1 : 0; }
template <typename H>
hipError_t make(const char* name, H* h) {
    if (fails(name)) return hipErrorOutOfMemory;
    *h = reinterpret_cast<H>(std::malloc(8));
    return hipSuccess;
}
template <typename H>
hipError_t drop(H h) {
    std::free(reinterpret_cast<void*>(h));
    return hipSuccess;
}
}  // namespace

namespace gsim {
void arm_launch_events(hipEvent_t, hipEvent_t) {}
bool disarm_launch_events() { return false; }
int launch_resident(const ModelDev<float>*, const StepDev<float>*, int, int, int, int, int, size_t, void*) { return launch("resident"); }
hipError_t resident_bodies(int block, int, size_t, int* n) {
    *n = block == 256 ? 512 : 256;
    return hipSuccess;
}
int launch_stage_copy(const StageSeg* s, int n, void*) {
    for (int i = 0; i < n; ++i) {
        if (s[i].src) std::memcpy(s[i].dst, s[i].src, s[i].n);
        else std::memset(s[i].dst, 0, s[i].n);
    }
    return launch("stage_copy");
}
template <typename T> int launch_elem_fwd(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, size_t, bool, bool, void*) { return launch("elem_fwd"); }
template <typename T> int launch_part_fwd(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, int, void*) { return launch("part_fwd"); }
template <typename T> int launch_elem_adj(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, size_t, bool, bool, void*) { return launch("elem_adj"); }
template <typename T> int launch_part_adj(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, int, bool, void*) { return launch("part_adj"); }
template <typename T> int launch_fill(T*, int64_t, T, void*) { return launch("fill"); }
template <typename T> int launch_persist(const ModelDev<T>*, const StepDev<T>*, int, const Tile*, const Tile*, const int32_t*, int, int, size_t, bool, void*) { return launch("persist"); }
template <typename T> int launch_dual(const ModelDev<T>*, const StepDev<T>*, const StepDev<T>*, const Tile*, int, const Tile*, int, int, int, size_t, bool particles, bool, bool, void*) { return launch(particles ? "part_dual" : "elem_dual"); }
template <typename T> int launch_mixed(const ModelDev<T>*, const StepDev<T>* sd, const TileSeg*, int, int, int, const TileSeg*, int, int, int, int, int, size_t, bool, void*) {
    calls += "x=" + std::to_string((unsigned long long)sd->x) + " ";  // the first query's input state
    return launch("mixed");
}
template <typename T> int launch_contact_reduce(const ModelDev<T>*, const StepDev<T>*, int, void*) { return launch("contact_reduce"); }
template <typename T> int launch_loss(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, int, int, void*) { return launch("loss"); }
template <typename T> int launch_fused_fwd(const ModelDev<T>*, const StepDev<T>*, const int32_t*, int, size_t, void*) { return launch("fused_fwd"); }
template <typename T> int launch_fused_adj(const ModelDev<T>*, const StepDev<T>*, const int32_t*, int, size_t, bool, void*) { return launch("fused_adj"); }
template <typename T> int launch_fused_params(const ModelDev<T>*, const StepDev<T>*, void*) { return launch("fused_params"); }
template <typename T> int launch_fused_grads(const ModelDev<T>*, const StepDev<T>*, void*) { return launch("fused_grads"); }
template <typename T> hipError_t fused_static_lds(bool, size_t* b) {
    *b = 1024;
    return hipSuccess;
}
#define FOR(T)                                                                                                            \
    template int launch_elem_fwd<T>(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, size_t, bool, bool, void*); \
    template int launch_part_fwd<T>(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, int, void*);               \
    template int launch_elem_adj<T>(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, size_t, bool, bool, void*); \
    template int launch_part_adj<T>(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, int, bool, void*);         \
    template int launch_fill<T>(T*, int64_t, T, void*);                                                                     \
    template int launch_persist<T>(const ModelDev<T>*, const StepDev<T>*, int, const Tile*, const Tile*, const int32_t*, int, \
                                   int, size_t, bool, void*);                                                               \
    template int launch_dual<T>(const ModelDev<T>*, const StepDev<T>*, const StepDev<T>*, const Tile*, int, const Tile*,     \
                                int, int, int, size_t, bool, bool, bool, void*);                                            \
    template int launch_mixed<T>(const ModelDev<T>*, const StepDev<T>*, const TileSeg*, int, int, int, const TileSeg*, int,  \
                                 int, int, int, int, size_t, bool, void*);                                                  \
    template int launch_contact_reduce<T>(const ModelDev<T>*, const StepDev<T>*, int, void*);                               \
    template int launch_loss<T>(const ModelDev<T>*, const StepDev<T>*, const Tile*, int, int, int, int, void*);              \
    template int launch_fused_fwd<T>(const ModelDev<T>*, const StepDev<T>*, const int32_t*, int, size_t, void*);             \
    template int launch_fused_adj<T>(const ModelDev<T>*, const StepDev<T>*, const int32_t*, int, size_t, bool, void*);       \
    template int launch_fused_params<T>(const ModelDev<T>*, const StepDev<T>*, void*);                                      \
    template int launch_fused_grads<T>(const ModelDev<T>*, const StepDev<T>*, void*);                                       \
    template hipError_t fused_static_lds<T>(bool, size_t*);
FOR(float)
FOR(double)
}  // namespace gsim

extern "C" {
const char* host_hip_calls() { return calls.c_str(); }
void host_hip_reset() {
    calls.clear();
    fail_at.clear();
}
void host_hip_fail(const char* name, int nth) { fail_at[name] = nth; }

hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "refused by the test"; }
hipError_t hipDeviceSynchronize() { return call("device_sync"); }
hipError_t hipEventCreate(hipEvent_t* e) { return make("event", e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return make("event", e); }
hipError_t hipEventDestroy(hipEvent_t e) { return drop(e); }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) {
    *t = 0;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return call("event_record"); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { return drop(g); }
hipError_t hipGraphExecDestroy(hipGraphExec_t g) { return drop(g); }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) { return make("graph", x); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return call("graph_launch"); }
hipError_t hipHostFree(void* p) { return drop(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return call("copy");
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return call("capture"); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return make("stream", s); }
hipError_t hipStreamDestroy(hipStream_t s) { return drop(s); }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return make("end_capture", g); }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return call("wait_event"); }
}
