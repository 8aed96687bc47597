// A CPU build of the library's host side (llma_api.hip, compiled for the host only) runs on this: the HIP calls it makes
// on one stream whose work waits in a queue until somebody synchronises, and launchers that note what they were given.
// Device memory is host memory.  The fake model accepts no draft and always answers token 7.
#include <stdlib.h>
#include <string.h>

#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <set>
#include <vector>

#include "common.h"
#include "kernels.h"

static std::deque<std::function<void()>> queue;
static long executed = 0, enqueued = 0;
static std::map<const void *, unsigned> allocations;       // and their numbers
static unsigned allocations_made = 0;
static std::set<const void *> lost;                       // to a reset
static int stale_uses = 0;
static bool not_ours(const void *p) { return lost.count(p) != 0; }
static long pinned = 0, fetched = 0;
static size_t alloc_limit = ~(size_t)0, refused = 0;       // larger allocations fail; the last one that did
static std::map<const char *, size_t> pinned_blocks;
static bool is_pinned(const void *p) {
    auto it = pinned_blocks.upper_bound((const char *)p);
    return it != pinned_blocks.begin() && (const char *)p < (--it)->first + it->second;
}
static int last_error_in = -1, event_record_in = -1;      // calls until the next injected failure (-1: none)
static std::vector<int> prompt_T, gemm_rows, gemm_split;

struct graph { std::vector<std::function<void()>> work; };
static graph *recording = nullptr;
static bool can_capture = false;                          // off: every step runs eagerly
static int graph_launches = 0, graphs_alive = 0;

static void enqueue(std::function<void()> f) {
    if (recording) { recording->work.push_back(std::move(f)); return; }
    queue.push_back(std::move(f));
    ++enqueued;
}
static void run_until(long n) {
    while (executed < n && !queue.empty()) { queue.front()(); queue.pop_front(); ++executed; }
}
static hipError_t inject(int &in) { return in >= 0 && in-- == 0 ? hipErrorUnknown : hipSuccess; }

extern "C" {
int stub_pending() { return (int)queue.size(); }
void stub_fail_last_error(int calls) { last_error_in = calls; }
void stub_fail_event_record(int calls) { event_record_in = calls; }
void stub_capture(int on) { can_capture = on != 0; }
long stub_pinned() { return pinned; }                                              // bytes of pinned memory asked for so far
int stub_graph_launches() { return graph_launches; }
int stub_graphs_alive() { return graphs_alive; }                                    // instantiated, not destroyed
static int take(std::vector<int> &v, int *out, int cap) {
    int n = 0;
    for (; n < (int)v.size() && n < cap; ++n) out[n] = v[n];
    v.clear();
    return n;
}
int stub_prompt_T(int *out, int cap) { return take(prompt_T, out, cap); }          // cache length each prompt pass started from
int stub_gemm_rows(int *out, int cap) { return take(gemm_rows, out, cap); }        // rows of every decoding GEMM launched
int stub_gemm_split(int *out, int cap) { return take(gemm_split, out, cap); }      // and whether it took the lo planes

struct ev { long at; };
void stub_alloc_limit(long bytes) { alloc_limit = bytes < 0 ? ~(size_t)0 : (size_t)bytes; }
unsigned long stub_refused() { return refused; }
long stub_fetched() { const long n = fetched; fetched = 0; return n; }              // bytes copied to the host since the last look
hipError_t hipMalloc(void **p, size_t n) {
    if (n > alloc_limit) { refused = n; *p = nullptr; return hipErrorOutOfMemory; }
    *p = calloc(n ? n : 1, 1);
    if (!*p) return hipErrorOutOfMemory;
    allocations[*p] = ++allocations_made;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    run_until(enqueued);
    stale_uses += p && not_ours(p);
    if (p && !not_ours(p)) { allocations.erase(p); free(p); }
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    pinned += (long)n;
    const hipError_t e = hipMalloc(p, n);
    pinned_blocks[(const char *)*p] = n;
    return e;
}
hipError_t hipHostFree(void *p) { pinned_blocks.erase((const char *)p); return hipFree(p); }
hipError_t hipPointerGetAttribute(void *data, hipPointer_attribute what, hipDeviceptr_t p) {
    if (what != HIP_POINTER_ATTRIBUTE_BUFFER_ID || !allocations.count(p)) return hipErrorInvalidValue;
    *(unsigned *)data = allocations[p];
    return hipSuccess;
}
// The device is reset: what was allocated is gone, or its address already belongs to somebody else (the memory itself is
// left alone).  Uses and frees of such addresses are counted.
void stub_device_reset(int reused) {
    run_until(enqueued);
    for (auto &a : allocations) lost.insert(a.first);
    if (!reused) allocations.clear();
    for (auto &a : allocations) a.second = ++allocations_made;
}
int stub_stale_uses() { return stale_uses; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (kind == hipMemcpyDeviceToHost) fetched += (long)n;
    if (kind == hipMemcpyHostToDevice && !is_pinned(s)) {                           // pageable: staged before the call returns
        auto copy = std::make_shared<std::vector<char>>((const char *)s, (const char *)s + n);
        enqueue([=] { memcpy(d, copy->data(), n); });
    } else enqueue([=] { memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { run_until(enqueued); memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { enqueue([=] { memset(d, v, n); }); return hipSuccess; }
hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { run_until(enqueued); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    if (!can_capture) return hipErrorNotSupported;
    recording = new graph;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    *g = (hipGraph_t)recording;
    recording = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    *x = (hipGraphExec_t) new graph(*(graph *)g);
    ++graphs_alive;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    ++graph_launches;
    for (auto &f : ((graph *)x)->work) enqueue(f);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (graph *)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    if (!queue.empty()) abort();                                                    // (it may still be running)
    delete (graph *)x;
    --graphs_alive;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t) new ev{0}; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (ev *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { ((ev *)e)->at = enqueued; return inject(event_record_in); }
hipError_t hipEventSynchronize(hipEvent_t e) { run_until(((ev *)e)->at); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipGetLastError(void) { return inject(last_error_in); }
const char *hipGetErrorString(hipError_t) { return "injected"; }
}

GemmPlan make_gemm_plan(int N, int K, int tiles_per_task) {
    GemmPlan p{};
    p.N = N; p.K = K; p.KSp = K / 32; p.tasks = N / 16; p.tiles_per_task = tiles_per_task; p.tk_waves = 8; p.n_split = 1;
    for (int &ft : p.tk_ft) ft = 1;
    return p;
}
bool tilek_ft_valid(const GemmPlan &, int, int ft) { return ft == 1; }
long tilek_cost(const GemmPlan &p, int) { return p.tasks; }
int panel_prompt_split(const GemmPlan &, int) { return 1; }
size_t panel_part_bytes(const GemmPlan &, int, int) { return 0; }
void launch_pack_weight(const void *, void *, int, int, int, int, int, hipStream_t) {}
void launch_kv_import_bf16(const void *, const void *, void *, void *, void *, void *, int, int, int, int, hipStream_t) {}
void launch_kv_import_f32(const void *, const void *, void *, void *, int, int, int, int, hipStream_t) {}
bool launch_gemm_bf16(const GemmArgs &a, hipStream_t) {
    gemm_rows.push_back(a.rows);
    gemm_split.push_back(a.split);
    enqueue([] {});
    return true;
}
void launch_gemm_panel_bf16(const GemmArgs &, hipStream_t) { enqueue([] {}); }
void launch_rstd_rows(const float *, int, float, float *, int, hipStream_t) {}
void launch_attn_bf16(const AttnArgs &, hipStream_t) {}
void launch_gemm_f32(const GemmArgs &, hipStream_t) { enqueue([] {}); }
void launch_attn_f32(const AttnArgs &, hipStream_t) {}
void launch_take_step(const StepState &s, int n_seqs, int max_k, hipStream_t) {
    enqueue([=] {
        for (int b = 0; b < n_seqs; ++b) {
            const int slot = s.io.slot[b];
            s.batch_slots[b] = slot;
            s.keff[b] = s.io.keff[b];
            s.T[slot] = s.io.T[b];
            s.pending[slot] = s.io.pending[b];
            s.lo_from[slot] = s.io.lo_from[b];
        }
        memcpy(s.draft, s.io.draft, sizeof(int) * n_seqs * max_k);
    });
}
void launch_setup_step_rows(const StepState &, int, int, int, const float *, int, const EmbedArgs &, const GenState *, const unsigned long long *, int,
                            hipStream_t) {
    enqueue([] {});
}
void launch_setup_prefill_rows(const StepState &s, const int *, const int *, int, int slot, const float *, int, const EmbedArgs &, hipStream_t) {
    enqueue([=] { prompt_T.push_back(s.T[slot]); });
}
void launch_advance_T(const StepState &s, int slot, int by, hipStream_t) { enqueue([=] { s.T[slot] += by; }); }
void launch_trigger_scan(const GenState *, int, int, unsigned long long *, hipStream_t) {}
// (the fake scan matches every reference, at the checksums of its inputs as they lie in device memory)
static int checksum(const int *p, long n) {
    unsigned h = 1;
    for (long i = 0; i < n; ++i) h = h * 31u + (unsigned)p[i];
    return (int)(h & 0x7fffffffu);
}
void launch_trigger_plain(const int *y, int y_len, const int *ref, const int *doc_offsets, int ref_len, int n_docs, int, unsigned long long *part, int *result, bool, hipStream_t) {
    enqueue([=] {
        for (int i = 0; i < trigger_spans(ref_len); ++i) part[i] = 0;
        result[0] = 1;
        result[1] = checksum(ref, ref_len);
        result[2] = checksum(y, y_len) ^ checksum(doc_offsets, n_docs + 1);
    });
}
void launch_trigger_host(const int *in, int *dev, int pieces, int y_len, int ref_len, int n_docs, int n, unsigned long long *part, int *result, hipStream_t st) {
    stale_uses += not_ours(result) + not_ours(dev);
    enqueue([=] { memcpy(dev, in, (size_t)pieces * 16); });
    launch_trigger_plain(dev, y_len, dev + y_len, dev + y_len + ref_len, ref_len, n_docs, n, part, result, false, st);
}
void launch_argmax_accept(const float *, const int *, int, const StepState &s, int n_seqs, int, int max_k, int, const GenState *gen, hipStream_t) {
    enqueue([=] {
        for (int b = 0; b < n_seqs; ++b) {
            const int slot = s.batch_slots[b];
            if (gen) {
                const GenState &G = gen[b];
                if (*G.n_out >= G.max_new) continue;
                const int st = (*G.n_steps)++, now = ++*G.n_out;
                G.y[now - 1] = 7;
                G.trace[4 * st] = G.trace[4 * st + 1] = 1;
                G.trace[4 * st + 2] = G.trace[4 * st + 3] = -1;
                G.host_count[(st & 1) * G.host_stride] = now;
                if (now >= G.max_new) G.host_count[((st & 1) ^ 1) * G.host_stride] = now;
            } else {
                s.io.nacc[b] = 0;
                s.io.next[b] = s.io.emit[b * (max_k + 1)] = 7;
            }
            s.T[slot] += 1;
            s.pending[slot] = 7;
        }
    });
}
