// The host library on the CPU: stands in for the HIP runtime (memory is host
// memory, filled with NaN words; events and streams are counters) and for the
// kernel launchers, which record what they were asked to launch and run nothing.
// Linked with spiir_host.cpp by tests/hoststub.py.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <vector>

#include "spiir_internal.h"

using namespace spiir;

namespace {
enum Kind { kStage, kFilter, kFilterLocal, kFilterPipe, kFilterMfma, kChain, kUpadd };
struct Launch {
    int kind, X, mode, nblocks, lanes;
    LaunchArgs args;
};
std::vector<Launch> g_log;
int g_events = 0;

int note(Kind kind, const LaunchArgs& a, int64_t nblocks, int X = 0, int mode = 0, int lanes = 0)
{
    g_log.push_back(Launch{kind, X, mode, (int)nblocks, lanes, a});
    return 0;
}
}  // namespace

// ---------------------------------------------------------------- launchers
namespace spiir {
int launch_stage(const LaunchArgs& a, int, void*) { return note(kStage, a, a.nreq); }
int launch_filter(int, int, const LaunchArgs& a, int n, int L, int, void*) { return note(kFilter, a, n, 0, 0, L); }
int launch_filter_mfma(const LaunchArgs& a, int n, int, void*) { return note(kFilterMfma, a, n); }
int launch_upadd(const LaunchArgs& a, int n, int, void*) { return note(kUpadd, a, n); }
int launch_filter_local(int, int, const LaunchArgs& a, int n, int L, int, void*)
{
    return note(kFilterLocal, a, n, 0, 0, L);
}
int launch_filter_pipe(int X, PipeMode mode, int, const LaunchArgs& a, int n, int lanes, int, void*)
{
    return note(kFilterPipe, a, n, X, (int)mode, lanes);
}
int launch_chain(const LaunchArgs& a, int64_t n, void*) { return note(kChain, a, n); }
int launch_prep(const c64*, const c64*, int64_t, int, c32*, c32*, c32*, const int32_t*, c32*, void*) { return 0; }
int launch_fill(void* p, int64_t bytes, void*)
{
    std::memset(p, 0, (size_t)bytes);
    return 0;
}
int filter_max_lds() { return 160 * 1024; }
int allow_filter_lds() { return 0; }
int scratch_ptr(int, void** out)
{
    static std::vector<char> scratch(kScratchBytes + 256);
    *out = (void*)(((uintptr_t)scratch.data() + 255) & ~(uintptr_t)255);
    return 0;
}
}  // namespace spiir

// ---------------------------------------------------------------- HIP
extern "C" {
hipError_t hipMalloc(void** p, size_t n)
{
    *p = std::aligned_alloc(256, (n + 255) & ~(size_t)255);
    if (*p) std::memset(*p, 0xff, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = (hipEvent_t)std::malloc(1);
    ++g_events;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::free((void*)e);
    --g_events;
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

// ---------------------------------------------------------------- the record
int stub_events() { return g_events; }
void stub_clear() { g_log.clear(); }
int stub_launches() { return (int)g_log.size(); }
// kind, X, mode, workgroups, lanes, requests of launch i
void stub_launch(int i, int32_t* out)
{
    const Launch& l = g_log[i];
    const int32_t v[6] = {l.kind, l.X, l.mode, l.nblocks, l.lanes, l.args.nreq};
    std::memcpy(out, v, sizeof(v));
}
// n, nchunk, dual, direct, z_direct, T of request k of launch i; its bank
const BankDev* stub_request(int i, int k, int32_t* out)
{
    const ReqArg& q = g_log[i].args.req[k];
    const int32_t v[6] = {q.n, q.nchunk, q.dual, q.direct, q.z_direct, q.T};
    std::memcpy(out, v, sizeof(v));
    return q.bd;
}
// chunk end states of a bank split in time: P + 1 rows of n_slots complex values
float* stub_uend(const BankDev* bd, int64_t* n)
{
    *n = 2 * (int64_t)(bd->P + 1) * bd->n_slots;
    return (float*)bd->uend;
}
float* stub_euend(const BankDev* bd) { return (float*)bd->euend; }
}
