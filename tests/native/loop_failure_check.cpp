// The native decoding loop's host code against a device that is made of a
// queue: a step that fails while its kernels are still queued must not lend its
// results to a later step, nor have its memory freed under it.
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>

#include "decode_loop.hip"

static void require(bool ok, const char* what) {
    if (ok) return;
    printf("failed: %s\n", what);
    exit(1);
}

// The device: what is enqueued runs at once (a short step), at the next
// enqueueing (queued work that the device comes to later), or at a wait.
namespace dev {
enum When { kAtOnce, kAtNextEnqueue, kAtWait };
When when = kAtOnce;
bool wait_fails = false, collect_fails = false;
int step = 0;         // what the device's outputs are made of
int enqueued = 0, waits = 0, freed = 0;
std::vector<std::function<void()>> queue;

void drain() {
    for (auto& f : queue) f();
    queue.clear();
}
void push(std::function<void()> f) {
    ++enqueued;
    queue.push_back(std::move(f));
    if (when == kAtOnce) drain();
}
}  // namespace dev

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { ++dev::freed; free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
    ++dev::waits;
    if (dev::wait_fails) return hipErrorUnknown;
    dev::drain();
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorUnknown; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorUnknown; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }

size_t spec_verify_workspace_bytes(int32_t, int32_t, int32_t, sv_dtype_t) { return 16; }
sv_status_t spec_verify_exact(const void*, const void*, sv_dtype_t, const int32_t*, const float*, int32_t B, int32_t,
                              int32_t, float, int32_t* acc, int32_t* nxt, void*, size_t, hipStream_t) {
    if (dev::when == dev::kAtNextEnqueue) dev::drain();
    const int s = dev::step;
    dev::push([=] {
        for (int b = 0; b < B; ++b) acc[b] = 0, nxt[b] = 100 * s + b;
    });
    return SV_OK;
}
sv_status_t spec_verify_exact_early_exit(const void*, const void*, sv_dtype_t, const int32_t*, const float*, int32_t,
                                         int32_t, int32_t, float, int32_t*, int32_t*, void*, size_t, hipStream_t) {
    return SV_ERR_HIP;
}
sv_status_t spec_verify_sigmoid(const void*, const void*, sv_dtype_t, const int32_t*, const float*, int32_t, int32_t,
                                int32_t, float, float, float, int32_t*, int32_t*, void*, size_t, hipStream_t) {
    return SV_ERR_HIP;
}
}  // extern "C"

namespace sv {
sv_status_t launch_collect(const int32_t* acc, const int32_t* nxt, const void* ws, int32_t B, uint32_t* host,
                           hipStream_t) {
    dev::push([=] {
        for (int b = 0; b < B; ++b) host[2 + b] = (uint32_t)acc[b], host[2 + B + b] = (uint32_t)nxt[b];
        host[1] = static_cast<const uint32_t*>(ws)[1];
        __atomic_store_n(host, 1u, __ATOMIC_RELEASE);
    });
    // (an error that is reported although the kernel was queued)
    return dev::collect_fails ? SV_ERR_HIP : SV_OK;
}
}  // namespace sv

static const int B = 3;
static int32_t acc[B], nxt[B], host_out[2 * B];
static uint32_t ws[4];

static sv_loop* create() {
    static float dummy[4];
    static int32_t tok[4];
    sv_loop_desc_t d{};
    d.batch = B, d.gamma_max = 4, d.vocab = 10, d.temperature = 1.0f;
    d.draft = d.target = dummy, d.tokens = tok, d.uniforms = dummy;
    d.accepted_len = acc, d.next_token = nxt, d.host_out = host_out, d.workspace = ws, d.workspace_bytes = sizeof ws;
    sv_loop* loop = nullptr;
    require(spec_verify_loop_create(&d, &loop) == SV_OK, "create");
    return loop;
}

static sv_status_t step(sv_loop* loop, int number) {
    dev::step = number;
    int32_t g = 0;
    return spec_verify_loop_step(loop, 2, &g);
}

static void require_results_of(int number, const char* what) {
    for (int b = 0; b < B; ++b) require(host_out[b] == 0 && host_out[B + b] == 100 * number + b, what);
}

int main() {
    // short steps end by the done word, long ones by the wait
    sv_loop* loop = create();
    for (int i = 1; i <= 4; ++i) {
        dev::when = (i % 2) ? dev::kAtOnce : dev::kAtWait;
        const int waits = dev::waits;
        require(step(loop, i) == SV_OK, "a good step");
        require_results_of(i, "a good step's results");
        require(dev::waits - waits == (i % 2 ? 0 : 1), "waits of a good step");
    }
    // a step fails with its kernels queued (its wait, then its enqueueing); the
    // device comes to them while the next step is under way
    for (int kind = 0; kind < 2; ++kind) {
        dev::when = dev::kAtNextEnqueue;
        dev::wait_fails = kind == 0, dev::collect_fails = kind == 1;
        require(step(loop, 10 + kind) == SV_ERR_HIP, "a failed step");
        dev::wait_fails = dev::collect_fails = false;
        require(step(loop, 20 + kind) == SV_OK, "the step after a failed one");
        require_results_of(20 + kind, "the results of the step after a failed one");
    }
    // as long as the wait fails, nothing more is enqueued
    dev::when = dev::kAtWait;
    dev::wait_fails = true;
    require(step(loop, 30) == SV_ERR_HIP, "a failed step");
    const int enqueued = dev::enqueued;
    require(step(loop, 31) == SV_ERR_HIP && dev::enqueued == enqueued, "a step while the wait fails");
    dev::wait_fails = false;
    // destroyed after a failed step: its kernels have run before the memory goes
    require(spec_verify_loop_destroy(loop) == SV_OK && dev::queue.empty() && dev::freed == 1, "destroy");
    // ... and where they cannot be waited for the memory stays
    loop = create();
    dev::wait_fails = true;
    require(step(loop, 40) == SV_ERR_HIP, "a failed step");
    uint32_t* block = loop->host;
    require(spec_verify_loop_destroy(loop) == SV_ERR_HIP && dev::freed == 1, "destroy while the wait fails");
    dev::drain();
    free(block);
    printf("all checks passed\n");
}
