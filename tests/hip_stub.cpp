// Stand-in for the HIP runtime on a host without a GPU, for tests of the host
// path: device memory is host memory, kernels do nothing but what the host
// path depends on (zero fills, an identity as the level operator, the solver
// state's iteration count), captured launches are recorded per graph, and
// every call of interest is counted.  Loaded before libtpfdm with global
// symbols, it takes the runtime's place.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct State {   // the solver state's layout (PcgState)
    double rz, pq, rr, bb, alpha, beta, tol2;
    int iter, done, maxit, norm;
};
struct Step {
    std::string name;
    State* state;   // k_pcg_reduce_beta only
};
struct Graph {
    std::vector<Step> steps;
};

std::map<const void*, std::string> kernels;
std::map<void*, size_t> sizes;
Graph* capture = nullptr;
hipError_t last = hipSuccess;
std::string fail;
int converge_at = 1 << 30, start_done = 0;
std::string watch;
int watch_arg = 0;
std::vector<char> watched;
int graph_launches = 0, iterations = 0, syncs = 0, live_execs = 0;

State* run(const Step& s) {
    if (s.name.find("k_pcg_reduce_beta") == std::string::npos) return nullptr;
    ++iterations;
    State* st = s.state;
    if (st->done) return st;
    ++st->iter;
    if (st->iter >= converge_at) st->done = 1;
    else if (st->iter >= st->maxit) st->done = 3;
    return st;
}

}  // namespace

extern "C" {

// ---- controls of the tests
void stub_set(int converge, int done_at_start, const char* fail_in_capture) {
    converge_at = converge;
    start_done = done_at_start;
    fail = fail_in_capture;
    graph_launches = iterations = syncs = 0;
}
void stub_watch(const char* kernel, int arg, int bytes) {   // keep an argument of the last launch of a kernel
    watch = kernel;
    watch_arg = arg;
    watched.assign(static_cast<size_t>(bytes), 0);
}
void stub_watched(void* out) { std::memcpy(out, watched.data(), watched.size()); }
int stub_graph_launches() { return graph_launches; }
int stub_iterations() { return iterations; }
int stub_syncs() { return syncs; }
int stub_live_graphs() { return live_execs; }

// ---- registration and launches
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    kernels[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static dim3 c_grid, c_block;
static size_t c_shared;
static hipStream_t c_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
    c_grid = g, c_block = b, c_shared = sh, c_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s) {
    *g = c_grid, *b = c_block, *sh = c_shared, *s = c_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
    const std::string& name = kernels[f];
    auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
    auto ptr = [&](int i) { return *static_cast<void**>(args[i]); };
    if (!watch.empty() && is(watch.c_str())) std::memcpy(watched.data(), args[watch_arg], watched.size());
    if (capture && !fail.empty() && is(fail.c_str())) return last = hipErrorLaunchFailure;
    Step s{name, is("k_pcg_reduce_beta") ? static_cast<State*>(ptr(3)) : nullptr};
    if (capture) {
        capture->steps.push_back(s);
    } else if (is("k_fill")) {
        std::memset(ptr(0), 0, sizes[ptr(0)]);
    } else if (is("k_mg_apply")) {
        std::memcpy(ptr(1), ptr(0), sizes[ptr(1)]);
    } else if (is("k_pcg_reduce_start")) {
        State* st = static_cast<State*>(ptr(2));
        *st = State{};
        st->maxit = *static_cast<int*>(args[4]);
        st->done = start_done ? start_done : st->maxit == 0 ? 3 : 0;
    } else {
        run(s);
    }
    return hipSuccess;
}

// ---- memory
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::calloc(1, n);
    sizes[*p] = n;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
    sizes.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t) {
    for (size_t r = 0; r < h; ++r) std::memcpy(static_cast<char*>(d) + r * dp, static_cast<const char*>(s) + r * sp, w);
    return hipSuccess;
}

// ---- streams, events, graphs
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(16); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++syncs; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { capture = new Graph; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = reinterpret_cast<hipGraph_t>(capture);
    capture = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    ++live_execs;
    *e = reinterpret_cast<hipGraphExec_t>(new Graph(*reinterpret_cast<Graph*>(g)));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete reinterpret_cast<Graph*>(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    --live_execs;
    delete reinterpret_cast<Graph*>(e);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
    ++graph_launches;
    for (const Step& s : reinterpret_cast<Graph*>(e)->steps) run(s);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(16); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 1.0f; return hipSuccess; }

// ---- device queries and errors
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 8; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}

}  // extern "C"
