// Host logic of the C-ABI with the HIP runtime and the kernels replaced by
// stand-ins that record what is launched, on which stream and how: which
// contexts take several steps a launch and which stores their steps use while
// contexts on other streams have work enqueued, and that no call names the
// stream of another context.  No GPU.  Exit status 0 when every check holds.
#include "lbm.h"
#include "lbm_kernels.hpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <vector>

namespace {
constexpr uintptr_t kOwnStreams = 0x100000;
std::set<hipStream_t> g_named;   // streams named by any call
int g_single, g_several, g_graphs, g_events;
std::vector<char> g_cached;      // stores of the single steps, captured ones too
int g_fit = 4;                   // blocks of launch_steps per compute unit
bool g_crowded;                  // the blocks of launch_steps do not meet
int g_bad = 0;

void name(hipStream_t s) {   // one that the library made to capture on aside
    if (reinterpret_cast<uintptr_t>(s) < kOwnStreams) g_named.insert(s);
}
void clear() {
    g_named.clear();
    g_single = g_several = g_graphs = 0;
    g_cached.clear();
}
void check(bool ok, const char* what) {
    if (!ok) {
        std::printf("wrong: %s\n", what);
        ++g_bad;
    }
}
}  // namespace

// ---------------------------------------------------------------- HIP runtime
extern "C" {
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    name(st);
    std::memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { name(s); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    static uintptr_t next = kOwnStreams;
    *s = reinterpret_cast<hipStream_t>(next += 16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
    name(s);
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = reinterpret_cast<hipGraph_t>(0x10);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    static uintptr_t next = 0x200000;
    *e = reinterpret_cast<hipGraphExec_t>(next += 16);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { name(s); ++g_graphs; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) { name(s); ++g_events; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    ++g_events;
    *e = reinterpret_cast<hipEvent_t>(0x30);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { name(s); ++g_events; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { ++g_events; return hipErrorNotReady; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }
}

// -------------------------------------------------------------------- kernels
namespace lbm {
hipError_t static_scratch(void**) { return hipErrorInvalidValue; }
hipError_t launch_step(const StepLaunch& a, hipStream_t s) {
    name(s);
    ++g_single;
    g_cached.push_back(a.cached);
    return hipSuccess;
}
hipError_t launch_steps(const StepLaunch& a, int, void*, int64_t, uint32_t*, uint32_t*, hipStream_t s) {
    name(s);
    ++g_several;
    if (g_crowded) ++a.ctr[1];
    return hipSuccess;
}
hipError_t steps_occupancy(const StepLaunch&, int* n) { *n = g_fit; return hipSuccess; }
hipError_t step_occupancy(int, int, int, int* n) { *n = 5; return hipSuccess; }
hipError_t launch_finalize(const double*, int, double*, uint32_t*, hipStream_t s) { name(s); return hipSuccess; }
hipError_t launch_zero(void* p, int64_t n, hipStream_t s) { name(s); std::memset(p, 0, n); return hipSuccess; }
hipError_t launch_rescale(int, void*, int64_t, float, hipStream_t s) { name(s); return hipSuccess; }
hipError_t launch_adjoint_step(const AdjLaunch& a, hipStream_t s) { name(s); g_cached.push_back(a.cached); return hipSuccess; }
hipError_t launch_fold(double*, const float*, int64_t, int64_t, hipStream_t s) { name(s); return hipSuccess; }
hipError_t launch_adjoint_seed(float*, int64_t, int, float, hipStream_t s) { name(s); return hipSuccess; }
hipError_t launch_finalize6(const double*, int, double*, hipStream_t s) { name(s); return hipSuccess; }
hipError_t launch_add_uniform(double*, int64_t, double, double, double, hipStream_t s) { name(s); return hipSuccess; }
}  // namespace lbm

namespace {
hipStream_t stream(int k) { return reinterpret_cast<hipStream_t>((uintptr_t)0x1000 * (k + 1)); }
// a context of `chunks` full chunks on a stream
struct Ctx {
    lbm_ctx* c = nullptr;
    void* ws = nullptr;
    Ctx(int chunks, hipStream_t s, int storage = LBM_F32, int nx = 256) {
        const int ny = 4096 / nx, nz = (chunks + 15) / 16;
        std::vector<uint8_t> g((size_t)nx * ny * nz, 1);
        std::fill(g.begin(), g.begin() + (size_t)chunks * 256, (uint8_t)0);
        size_t bytes = 0;
        check(lbm_workspace_query(g.data(), nx, ny, nz, storage, LBM_INDEX_BITMAP, &bytes, nullptr) == LBM_OK, "query");
        ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
        const double f[3] = {1e-6, 0, 0};
        check(lbm_setup(&c, g.data(), nx, ny, nz, 1.0, 3.0 / 16, LBM_SET_E, f, storage, LBM_INDEX_BITMAP, ws, bytes,
                        s) == LBM_OK, "setup");
    }
    ~Ctx() {
        lbm_destroy(c);
        std::free(ws);
    }
    // what a call of 8 steps launched
    bool several() {
        clear();
        lbm_step(c, 8);
        check(g_several + g_single > 0, "launches");
        return g_several > 0;
    }
    bool cached() {
        clear();
        lbm_step(c, 2);
        return g_cached.back() != 0;
    }
    void drained() {
        double u[3];
        lbm_mean_velocity(c, u);
    }
};

void several_contexts() {
    Ctx a(600, stream(0)), b(600, stream(1)), d(340, stream(2)), e(600, stream(0)), h(350, stream(3));
    check(a.several(), "one context takes several steps a launch");
    check(a.several(), "and again");
    check(!b.several(), "a second that does not fit beside it takes single steps");
    check(!h.several(), "so does a third, of more than a third of the GPU");
    check(d.several(), "one of less takes several beside the first");
    h.drained();
    check(!a.several(), "the first does not fit beside the others either");
    check(!e.several(), "nor one on its stream");
    b.drained();
    check(e.several(), "but beside the smaller one alone");
    e.drained();
    a.drained();
    check(b.several(), "the second does once the first's stream has been drained");
    b.drained();
    d.drained();
    check(a.several(), "the first again");
    lbm_step(a.c, 1);
    check(!b.several(), "a single step behind launches of several hides nothing");
    a.drained();
    b.drained();
    Ctx f(600, hipStreamPerThread), g(600, hipStreamPerThread);
    check(f.several(), "a stream per thread");
    check(!g.several(), "is another one in each thread");
}

// A context's calls name no stream but its own, nor do they touch events: the
// stream of an idle context may be gone, another thread may be capturing.
void own_stream() {
    Ctx a(600, stream(0));
    lbm_step(a.c, 8);
    a.drained();
    clear();
    g_events = 0;
    {
        Ctx b(300, stream(1)), d(1000, stream(1));
        for (lbm_ctx* c : {b.c, d.c}) lbm_step(c, 40);
        b.drained();
        d.drained();
    }
    check(g_named == std::set<hipStream_t>{stream(1)}, "a context's calls stay on its stream");
    Ctx b(300, stream(1));
    for (int k = 0; k < 3; ++k)
        for (lbm_ctx* c : {a.c, b.c}) lbm_step(c, 8);
    check(g_events == 0, "no events");
}

void stores() {
    // 4,000 chunks: 160 MB of FP32 states
    Ctx a(4000, stream(0)), b(4000, stream(1));
    check(a.cached(), "states inside the cache are stored there");
    check(!b.cached(), "two contexts' states that do not fit it together are streamed");
    check(!a.cached(), "by both");
    b.drained();
    check(a.cached(), "until the other's stream is drained");
    // a replayed graph holds the stores it was captured with
    clear();
    lbm_step(a.c, 32);
    check(g_graphs == 1 && g_cached.size() == 32 && g_cached.back(), "captured with cached stores");
    b.cached();
    clear();
    lbm_step(a.c, 32);
    check(g_graphs == 1 && g_cached.size() == 32 && !g_cached.back(), "captured again with streaming stores");
    b.drained();
    clear();
    lbm_step(a.c, 32);
    check(g_graphs == 1 && g_cached.empty(), "the first graph again");
}
// 16-bit states: streaming stores while they fit the L2s.
void small_states() {
    for (int storage : {LBM_F16, LBM_BF16, LBM_F16R}) {
        // 19.5 KB (F16R 20.5) per chunk and its coordinates
        Ctx a(1500, stream(0), storage), b(1700, stream(0), storage), d(1700, stream(0), storage, 4);
        check(!a.cached(), "states of 30 MB are streamed");
        check(b.cached(), "states of 35 MB are stored in the caches");
        check(!d.cached(), "but not with rows of four voxels");
    }
    Ctx e(1000, stream(0));
    check(e.cached(), "FP32 states of any size are");
}
// Replayed graphs of larger images: captured on first use, again after any
// change of what their launches bake in, and not by launches of several steps.
void graphs() {
    Ctx a(1000, stream(0));
    int steps = 0;
    // graph replays and single launches (captured ones too) of n steps
    auto run = [&](int n, int replays, int singles) {
        clear();
        steps += n;
        return lbm_step(a.c, n) == LBM_OK && g_several == 0 && g_graphs == replays && g_single == singles;
    };
    check(run(1, 0, 1), "a first step");
    check(run(65, 2, 33), "one capture, two replays, a single step");
    check(run(64, 2, 32), "an odd start is captured apart");
    check(run(64, 2, 0), "then replayed only");
    const auto fresh = [&](const char* what) {
        check(run(32, 1, 32), what);
        check(run(32, 1, 0), "and replayed");
    };
    static float field[3 * 256 * 1000];
    alignas(256) static char ws[256];
    lbm_set_collision(a.c, LBM_COLLIDE_TRT);
    check(run(1, 0, 1), "nothing pending after a change of collision");
    fresh("captured after a change of collision");
    lbm_set_force_field(a.c, field);
    fresh("after a force field");
    lbm_set_wall(a.c, LBM_WALL_FULLWAY, ws, 256);
    fresh("after full-way walls");
    lbm_set_symmetry(a.c, 1, 0);
    fresh("after symmetry planes");
    lbm_set_symmetry(a.c, 0, 0);
    lbm_set_wall(a.c, LBM_WALL_HALFWAY, nullptr, 0);
    fresh("after halfway walls");
    lbm_set_graphs(a.c, 0);
    check(run(64, 0, 64), "plain launches on request");
    Ctx b(1000, stream(0), LBM_F16);
    lbm_step(b.c, 33);
    lbm_set_storage_exponent(b.c, 9);
    clear();
    lbm_step(b.c, 32);
    check(g_graphs == 1 && g_single == 32, "after a change of the storage exponent");
}

// After a launch whose blocks did not meet: single steps for 8 calls, then 16,
// ..., and several a launch again once they do.
void crowded_gpu() {
    Ctx a(600, stream(0));
    double u[3];
    auto call = [&] {
        const bool s = a.several();
        lbm_history(a.c, 1, u);
        return s;
    };
    check(call() && call(), "several steps a launch");
    for (int apart : {8, 16, 32}) {
        g_crowded = true;
        check(call(), "a launch that did not meet");
        g_crowded = false;
        for (int k = 0; k < apart; ++k) check(!call(), "single steps for a while");
    }
    check(call() && call(), "several again");
    g_crowded = true;
    check(call(), "another time");
    g_crowded = false;
    for (int k = 0; k < 8; ++k) check(!call(), "the wait starts small again");
    check(call(), "and ends");
}

// Full-way walls hold no state of their own.
void wall_workspace() {
    Ctx a(1000, stream(0));
    size_t bytes = 0;
    check(lbm_wall_workspace_query(a.c, &bytes) == LBM_OK && bytes > 0 && bytes <= 4096, "a token workspace");
    alignas(256) static char ws[8192];
    check(bytes <= sizeof ws && lbm_set_wall(a.c, LBM_WALL_FULLWAY, ws, bytes) == LBM_OK, "of that size is accepted");
    check(lbm_set_wall(a.c, LBM_WALL_FULLWAY, nullptr, bytes) == LBM_EWORKSPACE, "none is refused");
    check(lbm_set_wall(a.c, LBM_WALL_FULLWAY, ws + 8, bytes) == LBM_EWORKSPACE, "a misaligned one too");
    check(lbm_set_wall(a.c, LBM_WALL_FULLWAY, ws, bytes - 1) == LBM_EWORKSPACE, "and a smaller one");
}
}  // namespace

int main() {
    own_stream();
    several_contexts();
    stores();
    small_states();
    graphs();
    crowded_gpu();
    wall_workspace();
    std::printf("bad %d\n", g_bad);
    return g_bad != 0;
}
