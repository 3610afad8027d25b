// Stand-in for the HIP runtime under which the library's host code runs on the CPU: device memory is
// host memory, copies happen at once, kernels are not run.  What the host code asks of the runtime is
// kept as a log of short lines, in order:
//   launch KERNEL STREAM | sync STREAM | begin STREAM DEVICE | end STREAM | replay STREAM | exec_destroy
// STREAM is the handle's value (0: the default stream); streams created here count up from 1000.
// "exec_destroy busy" marks an executable graph destroyed while a replay may still run, and
// "bad window JOB" a sweep launched with a force-window layout outside its lattice or capacity.
#include <hip/hip_ext.h>

#include "lbib_internal.h"

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {
std::string g_log;
std::map<const void*, std::string> g_kernel;
std::map<void*, int> g_graph;                // executable graph: replays since the last wait for them
std::set<hipStream_t> g_capturing;
int g_device = 0;
long long g_handle = 1000;
struct Config { dim3 grid, block; size_t shmem; hipStream_t stream; };
std::vector<Config> g_config;

void say(const std::string& s) { g_log += s + "\n"; }
std::string name(hipStream_t s) { return std::to_string((long long)(size_t)s); }
void waited() { for (auto& g : g_graph) g.second = 0; }

void check_windows(dim3 grid, void** args) {
    using namespace lbib;
    const Pools& P = *(const Pools*)args[0];
    int last = -1;
    for (unsigned t = 0; t < grid.x; ++t) {
        const int j = P.tiles[t].x;
        if (j == last) continue;
        last = j;
        const JobDev& J = P.jobs[j];
        const int dims[3] = {J.nx, J.ny, J.nz};
        for (int b = J.body0; b < J.body0 + J.nbodies; ++b)
            if (!win_valid(P.fdesc[b], dims, P.bodies[b].win_cap, J.bc)) say("bad window " + std::to_string(j));
    }
}

hipError_t launched(const void* f, dim3 grid, void** args, hipStream_t s) {
    const std::string& k = g_kernel[f];
    if (k.find("k_sweep") != std::string::npos) check_windows(grid, args);
    say("launch " + k + " " + name(s));
    return hipSuccess;
}
}  // namespace

extern "C" {

unsigned stub_sweep_tile(unsigned T, unsigned bid, int chunk) { return lbib::sweep_tile(lbib::sweep_order(T, chunk), bid); }
const char* stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_set_device(int d) { g_device = d; }
void stub_log_device() { say("device " + std::to_string(g_device)); }
void stub_set_capturing(void* s, int on) { if (on) g_capturing.insert((hipStream_t)s); else g_capturing.erase((hipStream_t)s); }

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* n, unsigned, uint3*, uint3*, dim3*, dim3*, int*) { g_kernel[f] = n; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) { g_config.push_back({g, b, m, s}); return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
    const Config c = g_config.back();
    g_config.pop_back();
    *g = c.grid; *b = c.block; *m = c.shmem; *s = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void** a, size_t, hipStream_t s) { return launched(f, g, a, s); }
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3, void** a, size_t, hipStream_t s, hipEvent_t, hipEvent_t, int) { return launched(f, g, a, s); }

hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(n, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { waited(); free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }

hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)(size_t)++g_handle; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)(size_t)++g_handle; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    say("sync " + name(s));
    if (s || g_device == 0) waited();   // the default stream is the current device's; lattices live on device 0
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
    *c = g_capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    static hipStreamCaptureMode cur = hipStreamCaptureModeGlobal;
    const hipStreamCaptureMode old = cur;
    cur = *m;
    *m = old;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    say("begin " + name(s) + " " + std::to_string(g_device));
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) { say("end " + name(s)); *g = (hipGraph_t)(size_t)++g_handle; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *e = (hipGraphExec_t)(size_t)++g_handle;
    g_graph[*e] = 0;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) { ++g_graph[e]; say("replay " + name(s)); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    say(g_graph[e] ? "exec_destroy busy" : "exec_destroy");
    g_graph.erase(e);
    return hipSuccess;
}

}  // extern "C"
