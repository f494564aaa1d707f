// A decoding loop around the fused verification step: one call per
// iteration replays the step for the iteration's number of drafts from a
// HIP graph captured once per gamma (the verification followed by a kernel that
// stores the accepted lengths and next tokens in pinned host memory), waits for
// them, and returns the next gamma by the draft-length rule of the paper's
// experiments (Sec. 4, hyperparameters: gamma starts at 5, grows by 2 after
// an iteration that accepts every draft, otherwise shrinks by 1; here kept
// within 1 .. gamma_max, and with several batch elements every element must
// accept every draft to grow).
//
// In the exact mode each step runs either the single pass or the early exit
// (Sec. 3.1 stops at the first rejection): as the descriptor says, or chosen
// from the previous step's acceptance (early_exit_pays).
//
// Host code only: the device work is the library's verification kernel and the
// kernel that collects its results.  All device buffers and host_out belong to
// the caller; the loop object holds the descriptor, a pinned block for the
// collected results and the instantiated graphs.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <chrono>
#include <cstring>
#include <new>
#include <vector>

#include "plan.hpp"
#include "spec_verify.h"

struct sv_loop {
    sv_loop_desc_t d;
    uint32_t* host = nullptr;          // pinned { done, error flag, outputs [2B] } (from the first step on)
    uint32_t* host_dev = nullptr;      // the device's address of it
    std::vector<hipGraphExec_t> exec;  // by 2 gamma + early exit (0, 1 unused); null until first use
    bool settled = true;               // nothing that a step enqueued can still store in the block
    bool early = false;                // the next step's choice (exact mode)
    int32_t last_early = -1;           // the last step's choice
};

namespace {

// The collected results have arrived: a poll of the done word, by time, since
// waiting for the stream costs the runtime's wake-up on top of the work (28.6 us
// an iteration against 24.2, B = 1, V = 51,865 fp32, the inputs in place).  The
// bound is a fixed 200 us from the enqueueing on, for the short steps that the
// wake-up weighs on.  What takes longer is polled for 200 us and then left to the
// stream's wait: large steps (B = 64, gamma 20, V = 128,256 bf16 takes 104 us,
// twice the batch in fp32 four times that), a producer's work still ahead on the
// stream, a device that failed.
bool arrived(const uint32_t* done) {
    constexpr auto kSpin = std::chrono::microseconds(200);
    const auto end = std::chrono::steady_clock::now() + kSpin;
    do {
        for (int i = 0; i < 32; ++i) {
            if (__atomic_load_n(done, __ATOMIC_ACQUIRE) != 0u) return true;
            __builtin_ia32_pause();
        }
    } while (std::chrono::steady_clock::now() < end);
    return false;
}

// The verification of the leading [B, gamma, V] parts of the static buffers
// and the collection of its outputs and of the workspace's error flag, enqueued
// on the loop's stream.
sv_status_t enqueue(const sv_loop* loop, int32_t gamma, bool early) {
    const sv_loop_desc_t& d = loop->d;
    sv_status_t st;
    if (d.mode == 0 && early)
        st = spec_verify_exact_early_exit(d.draft, d.target, d.dtype, d.tokens, d.uniforms, d.batch, gamma, d.vocab,
                                          d.temperature, d.accepted_len, d.next_token, d.workspace,
                                          d.workspace_bytes, d.stream);
    else if (d.mode == 0)
        st = spec_verify_exact(d.draft, d.target, d.dtype, d.tokens, d.uniforms, d.batch, gamma, d.vocab,
                               d.temperature, d.accepted_len, d.next_token, d.workspace, d.workspace_bytes,
                               d.stream);
    else
        st = spec_verify_sigmoid(d.draft, d.target, d.dtype, d.tokens, d.uniforms, d.batch, gamma, d.vocab,
                                 d.temperature, d.alpha, d.beta, d.accepted_len, d.next_token, d.workspace,
                                 d.workspace_bytes, d.stream);
    if (st != SV_OK) return st;
    return sv::launch_collect(d.accepted_len, d.next_token, d.workspace, d.batch, loop->host_dev, d.stream);
}

sv_status_t capture(sv_loop* loop, int32_t gamma, bool early) {
    const sv_loop_desc_t& d = loop->d;
    if (hipStreamBeginCapture(d.stream, hipStreamCaptureModeThreadLocal) != hipSuccess) return SV_ERR_HIP;
    const sv_status_t st = enqueue(loop, gamma, early);
    hipGraph_t graph = nullptr;
    const hipError_t end = hipStreamEndCapture(d.stream, &graph);
    if (st != SV_OK || end != hipSuccess || graph == nullptr) {
        if (graph != nullptr) (void)hipGraphDestroy(graph);
        return st != SV_OK ? st : SV_ERR_HIP;
    }
    hipGraphExec_t exec = nullptr;
    const hipError_t inst = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (inst != hipSuccess) return SV_ERR_HIP;
    loop->exec[2 * gamma + (early ? 1 : 0)] = exec;
    return SV_OK;
}

}  // namespace

extern "C" {

sv_status_t spec_verify_loop_create(const sv_loop_desc_t* desc, sv_loop** out) {
    if (desc == nullptr || out == nullptr) return SV_ERR_NULL;
    *out = nullptr;
    const sv_loop_desc_t& d = *desc;
    if (d.draft == nullptr || d.target == nullptr || d.tokens == nullptr || d.uniforms == nullptr ||
        d.accepted_len == nullptr || d.next_token == nullptr || d.host_out == nullptr || d.workspace == nullptr)
        return SV_ERR_NULL;
    if ((d.mode != 0 && d.mode != 1) || d.early_exit < 0 || d.early_exit > 2) return SV_ERR_PARAM;
    if (d.batch < 1 || d.gamma_max < 1 || d.vocab < 1) return SV_ERR_SHAPE;
    for (int32_t g = 1; g <= d.gamma_max; ++g) {
        const size_t need = spec_verify_workspace_bytes(d.batch, g, d.vocab, d.dtype);
        if (need == 0) return SV_ERR_SHAPE;
        if (d.workspace_bytes < need) return SV_ERR_WORKSPACE;
    }
    sv_loop* loop = new (std::nothrow) sv_loop;
    if (loop == nullptr) return SV_ERR_ALLOC;
    loop->d = d;
    loop->exec.assign(2 * ((size_t)d.gamma_max + 1), nullptr);
    loop->early = d.mode == 0 && d.early_exit == 1;
    *out = loop;
    return SV_OK;
}

sv_status_t spec_verify_loop_step(sv_loop* loop, int32_t gamma, int32_t* next_gamma) {
    if (loop == nullptr || next_gamma == nullptr) return SV_ERR_NULL;
    const sv_loop_desc_t& d = loop->d;
    if (gamma < 1 || gamma > d.gamma_max) return SV_ERR_PARAM;
    if (loop->host == nullptr) {
        // allocated once, here (a step needs the GPU anyway; creating the loop
        // does not); coherent, since the host reads it while the kernel runs
        void *host = nullptr, *dev = nullptr;
        if (hipHostMalloc(&host, sizeof(uint32_t) * (2 + 2 * (size_t)d.batch), hipHostMallocCoherent) != hipSuccess ||
            host == nullptr)
            return SV_ERR_HIP;
        if (hipHostGetDevicePointer(&dev, host, 0) != hipSuccess || dev == nullptr) {
            (void)hipHostFree(host);
            return SV_ERR_HIP;
        }
        loop->host = static_cast<uint32_t*>(host);
        loop->host_dev = static_cast<uint32_t*>(dev);
    }
    // An earlier step that failed (its enqueueing, or the wait) may have left its
    // kernels on the stream, whose done word would pass for this step's: they
    // are waited for first.  Every other step ended after its done word or after
    // the stream's wait.
    if (!loop->settled && hipStreamSynchronize(d.stream) != hipSuccess) return SV_ERR_HIP;
    loop->settled = false;
    loop->host[1] = 0;
    __atomic_store_n(loop->host, 0u, __ATOMIC_RELEASE);
    const bool early = loop->early;
    if (d.use_graphs) {
        hipGraphExec_t& e = loop->exec[2 * gamma + (early ? 1 : 0)];
        if (e == nullptr) {
            const sv_status_t st = capture(loop, gamma, early);
            if (st != SV_OK) return st;
        }
        if (hipGraphLaunch(e, d.stream) != hipSuccess) return SV_ERR_HIP;
    } else {
        const sv_status_t st = enqueue(loop, gamma, early);
        if (st != SV_OK) return st;
    }
    loop->last_early = (d.mode == 0 && early) ? 1 : 0;
    // (a replayed graph is waited for whole: destroying the loop frees it)
    if ((d.use_graphs || !arrived(loop->host)) && hipStreamSynchronize(d.stream) != hipSuccess) return SV_ERR_HIP;
    loop->settled = true;
    std::memcpy(d.host_out, loop->host + 2, sizeof(int32_t) * 2 * (size_t)d.batch);
    if (loop->host[1] != 0) return SV_ERR_TIMEOUT;
    bool all = true;
    long long accepted = 0;
    for (int32_t b = 0; b < d.batch; ++b) {
        all = all && d.host_out[b] == gamma;
        accepted += (d.host_out[b] > 0) ? d.host_out[b] : 0;
    }
    if (d.mode == 0 && d.early_exit == 2) loop->early = sv::early_exit_pays(accepted, d.batch, gamma);
    *next_gamma = all ? (gamma + 2 < d.gamma_max ? gamma + 2 : d.gamma_max) : (gamma > 1 ? gamma - 1 : 1);
    return SV_OK;
}

int32_t spec_verify_loop_last_early_exit(const sv_loop* loop) { return loop == nullptr ? -1 : loop->last_early; }

sv_status_t spec_verify_loop_destroy(sv_loop* loop) {
    if (loop == nullptr) return SV_OK;
    sv_status_t st = SV_OK;
    if (!loop->settled && hipStreamSynchronize(loop->d.stream) != hipSuccess) {
        // a failed step's kernels may still run: what they use is left allocated
        delete loop;
        return SV_ERR_HIP;
    }
    for (hipGraphExec_t e : loop->exec)
        if (e != nullptr && hipGraphExecDestroy(e) != hipSuccess) st = SV_ERR_HIP;
    if (loop->host != nullptr && hipHostFree(loop->host) != hipSuccess) st = SV_ERR_HIP;
    delete loop;
    return st;
}

}  // extern "C"
