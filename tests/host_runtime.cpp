// A HIP runtime of host memory and recorded calls, and stand-ins for the kernels, under
// which the library's host layer (csrc/api.cpp) runs without a GPU: launches take place
// at once, in the order they are enqueued.  An evolution kernel moves the step counts of
// its instances by the rules it shares with the real one (internal.h); an instance
// collapses at the step that its first Phi value names.  A snapshot holds the step it is
// of, in every entry.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "../paper_1706_07413_amd/csrc/internal.h"

namespace {
std::string g_log;                  // one line per recorded call
std::map<void*, size_t> g_held;     // device allocations
size_t g_total = (size_t)288 << 30, g_limit = ~(size_t)0, g_in_use = 0, g_peak = 0;
size_t g_refused = 0;               // allocations past the limit
long long g_setup = 0;              // allocations and copies
hipError_t g_last = hipSuccess;
int g_cus = 4, g_per_cu = 1;
intptr_t g_streams = 0;

void note(const std::string& s) { g_log += s + "\n"; }
std::string str(const void* p) { return std::to_string((intptr_t)p); }
}  // namespace

extern "C" {

// ---- what a test sets and reads ----
void fake_reset(long long total, long long limit, int cus, int per_cu)
{
    g_log.clear();
    g_total = (size_t)total;
    g_limit = (size_t)limit;
    g_cus = cus;
    g_per_cu = per_cu;
    g_peak = g_in_use;
    g_refused = 0;
    g_setup = 0;
    g_last = hipSuccess;
}
const char* fake_log() { return g_log.c_str(); }
long long fake_in_use() { return (long long)g_in_use; }
long long fake_peak() { return (long long)g_peak; }
long long fake_setup() { return g_setup; }
long long fake_refused() { return (long long)g_refused; }

// ---- the runtime ----
hipError_t hipMalloc(void** p, size_t n)
{
    ++g_setup;
    if (n > g_limit - g_in_use) {
        ++g_refused;
        return g_last = hipErrorOutOfMemory;
    }
    // (no more host memory than is touched)
    *p = std::calloc(1, n ? n : 1);
    if (!*p) return g_last = hipErrorOutOfMemory;
    g_held[*p] = n;
    g_in_use += n;
    g_peak = g_in_use > g_peak ? g_in_use : g_peak;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    auto it = g_held.find(p);
    if (it == g_held.end()) return p ? hipErrorInvalidValue : hipSuccess;
    g_in_use -= it->second;
    g_held.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_b, size_t* total)
{
    *total = g_total;
    *free_b = (g_limit < g_total ? g_limit : g_total) - g_in_use;
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { ++g_setup; std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? g_cus
         : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 1;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)(++g_streams); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { note("wait " + str(s) + " " + str(e)); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)(++g_streams); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { note("record " + str(s) + " " + str(e)); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { note("capture"); return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) { *x = nullptr; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { note("replay"); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

}  // extern "C"

// ---- the kernels ----
namespace adscl {

#define OK_FN(name, ...) \
    hipError_t name(__VA_ARGS__) { return hipSuccess; }

size_t table_len(ClassCfg c) { return (size_t)3 * c.P * 64 * c.W; }
bool class_supported(ClassCfg) { return true; }
size_t evolve_lds_bytes(ClassCfg) { return 0; }
OK_FN(prepare_evolve, ClassCfg, size_t)
hipError_t evolve_per_cu(ClassCfg, bool, int* n) { *n = g_per_cu; return hipSuccess; }
bool pair_supported(ClassCfg) { return false; }
OK_FN(prepare_evolve_pair, ClassCfg, size_t)
OK_FN(launch_evolve_pair, ClassCfg, int, int, const EvolveArgs&, hipStream_t)
bool scheme_class_supported(ClassCfg) { return true; }
OK_FN(prepare_evolve_scheme, ClassCfg, int, bool, size_t)
bool big_class_supported(ClassCfg) { return false; }
size_t big_lds_bytes(ClassCfg) { return 0; }
OK_FN(prepare_evolve_big, ClassCfg, int, bool, size_t)
hipError_t big_capacity(ClassCfg, int, bool, int, int* n) { *n = 1024; return hipSuccess; }
OK_FN(launch_evolve_big, ClassCfg, int, bool, int, const EvolveArgs&, const BigArgs&, hipStream_t)

static void run_instance(const EvolveArgs& a, int b, bool again)
{
    InstStatus& st = a.status[b];
    if (st.state == ST_COLLAPSED || st.state == ST_NONFINITE) return;
    const int64_t end = segment_end(st.steps, st.target, a.ic[b].n_final, a.snap_every, a.slice, a.tail, again);
    const double stop = a.Phi[a.ic[b].off + 1];
    if (st.steps >= end) return;
    if (stop > 0.0 && stop <= (double)end && stop >= (double)st.steps) {
        st.steps = (int64_t)stop;
        st.state = ST_COLLAPSED;
    } else {
        st.steps = end;
    }
}

hipError_t launch_evolve(ClassCfg c, bool full, int n_blocks, const EvolveArgs& a, hipStream_t s)
{
    note("evolve " + str(s) + " P" + std::to_string(c.P) + " W" + std::to_string(c.W) + " full" + std::to_string(full) +
         " blocks" + std::to_string(n_blocks) + " keep" + std::to_string(a.keep != nullptr) + " ckpt" +
         std::to_string(a.ckpt ? a.ckpt_every : 0) + " slice" + std::to_string(a.slice));
    for (int i = 0; i < n_blocks; ++i) {
        bool again = a.again != 0;
        const int p = launch_place(i, a.order_first, a.order_n, again);
        run_instance(a, a.order[p], again);
    }
    return hipSuccess;
}

hipError_t launch_evolve_scheme(ClassCfg c, int, bool, bool, int n_blocks, const EvolveArgs& a, hipStream_t s)
{
    return launch_evolve(c, false, n_blocks, a, s);
}

OK_FN(launch_init_gaussian, int, const InstConst*, const double*, const double*, double*, double*, int64_t, hipStream_t)
OK_FN(launch_init_modes, int, const InstConst*, const double*, const double*, int, const double* const*, double*, double*,
      int64_t, hipStream_t)
OK_FN(launch_pins, int, const InstConst*, double*, double*, hipStream_t)
hipError_t launch_reset_status(int n, InstStatus* st, hipStream_t)
{
    for (int b = 0; b < n; ++b) {
        st[b] = InstStatus();
        st[b].t_c = -1.0;
        st[b].minA = 1.0;
    }
    return hipSuccess;
}
hipError_t launch_set_targets(int n, const InstConst* ic, InstStatus* st, int64_t max_steps, hipStream_t)
{
    for (int b = 0; b < n; ++b) {
        int64_t t = st[b].steps + max_steps;
        if (t > ic[b].n_final) t = ic[b].n_final;
        if (t < st[b].steps) t = st[b].steps;
        st[b].target = t;
    }
    return hipSuccess;
}
hipError_t launch_finalize(int n, int64_t, const InstConst* ic, InstStatus* st, const double* const*, double*,
                           int64_t total, int, int, double, bool final, int32_t every, int32_t slots, double* snaps,
                           hipStream_t, int32_t)
{
    for (int b = 0; b < n; ++b) {
        const int64_t k = st[b].steps;
        if (snaps && every > 0 && k % every == 0 && k / every < slots)
            for (int f = 0; f < 5; ++f)
                for (int i = 0; i < ic[b].N; ++i) snaps[((size_t)(k / every) * 5 + f) * total + ic[b].off + i] = (double)k;
        if (final && (st[b].state == ST_RUNNING || st[b].state == ST_DONE))
            st[b].state = k >= ic[b].n_final ? ST_DONE : ST_RUNNING;
    }
    return hipSuccess;
}
OK_FN(launch_diagnostics, int, const InstConst*, const double* const*, const double*, int64_t, int, double, double*,
      double*, hipStream_t)
OK_FN(static_scratch_init, int)
double* static_scratch(int) { return nullptr; }
OK_FN(launch_spectrum, const double*, const SpecRow*, const SpecTile*, int, int, double*, double*, double*, hipStream_t)

size_t adjoint_scratch_len(ClassCfg c) { return (size_t)16 * c.P * 64 * c.W; }
size_t stage_record_len(ClassCfg c) { return (size_t)16 * c.P * 64 * c.W; }
OK_FN(prepare_adjoint, ClassCfg, size_t)
hipError_t launch_adjoint(ClassCfg, bool, int n_blocks, const AdjointArgs& a, hipStream_t s)
{
    note("reverse " + str(s) + " blocks" + std::to_string(n_blocks) + " keep" + std::to_string(a.keep != nullptr));
    return hipSuccess;
}
OK_FN(launch_endpoint, ClassCfg, bool, int, const EndArgs&, hipStream_t)
hipError_t launch_adj_prepare(int n, const InstConst* ic, const InstStatus* st, int64_t K, int64_t r, InstStatus* rst,
                              AdjSeg* sg, hipStream_t)
{
    note("segment " + std::to_string(r) + " of " + std::to_string(K));
    for (int b = 0; b < n; ++b) {
        const int64_t n1 = ic[b].n_final - r * K;
        const bool act = st[b].state == ST_DONE && n1 > 0;
        sg[b] = AdjSeg{act && n1 > K ? n1 - K : 0, act ? n1 : 0, act ? 1 : 0, 0};
        rst[b] = InstStatus();
        rst[b].steps = sg[b].n0;
        rst[b].target = sg[b].n1;
        rst[b].state = act ? ST_RUNNING : ST_COLLAPSED;
    }
    return hipSuccess;
}
hipError_t launch_adj_finish(int n, const InstConst*, const InstStatus* st, const double*, int64_t, const double* const*,
                             const double*, int, const double*, const double*, int, double*, double*, int32_t* valid,
                             hipStream_t)
{
    for (int b = 0; b < n; ++b) valid[b] = st[b].state == ST_DONE;
    return hipSuccess;
}
OK_FN(launch_fill, double*, int64_t, double, hipStream_t)
OK_FN(launch_mask, int, InstStatus*, const int32_t*, hipStream_t)
OK_FN(launch_gd_init, int, double, const GdState&, hipStream_t)
OK_FN(launch_gd_update, int, int, double*, const double*, const double*, const int32_t*, const GdState&, double*,
      hipStream_t)

}  // namespace adscl
