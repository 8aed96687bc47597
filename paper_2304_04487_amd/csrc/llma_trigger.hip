// llma_find_trigger: the trigger scan (paper: Method, the n-gram match step of Algorithm 1) from host lists, stateless.
#include <string.h>
#include <unistd.h>

#include <initializer_list>
#include <string>
#include <utility>

#include "../../include/llma.h"
#include "common.h"
#include "kernels.h"

void llma_set_error_text(const char *text);     // llma_api.hip: text for llma_last_error(NULL)

// What a call needs beside its arguments: pinned host memory that holds [result(4) | y | ref | doc_offsets], and device
// memory for a copy of it and the spans' keys.  A call that allocated and freed, and copied with two synchronous calls, took 41 us
// where one with buffers of its own takes 18.  So every thread keeps its buffers from one call for the next, up to
// TRIGGER_KEEP_WORDS of each, until it ends, and nothing of a call's inputs.  No buffer or lock is shared between threads; their
// launches are, they go to the default stream.  Larger calls allocate device memory of their own and free it; their inputs pass through the
// kept pinned buffer half a mebibyte at a time.  300 k / 1 M / 4 M / 20 M tokens 79 / 210 / 620 / 3150 us; with pinned memory of
// the call's size, which takes longer to get than it saves, 175 / 365 / 750 / 31000, staged in pageable memory 150 / 340 / 1150 / 20000.
#define TRIGGER_KEEP_WORDS (1 << 18)
#define RESULT_WORDS 4                          // in front: matched, doc, pos (and the inputs stay 16-byte aligned)
namespace {
// an allocation's number in this process (never given twice), 0 if p is not the start of one any more
uint64_t allocation_of(const void *p) {
    uint64_t id = 0;
    if (p && hipPointerGetAttribute(&id, HIP_POINTER_ATTRIBUTE_BUFFER_ID, (hipDeviceptr_t)p) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return id;
}
struct Buffers {
    int *host = nullptr, *host_dev = nullptr, *dev = nullptr;
    uint64_t host_id = 0, dev_id = 0;
    size_t words = 0;                           // of either
    int device = -1;
    pid_t owner = 0;
    // hipDeviceReset frees what the device holds, and its addresses may belong to others by now (0.06 us to ask)
    bool host_ours() const { return host_id != 0 && allocation_of(host) == host_id; }
    bool dev_ours() const { return dev_id != 0 && allocation_of(dev) == dev_id; }
    void release() {
        if (!host && !dev) return;
        // (a forked child has no use of its parent's device)
        if (owner == getpid()) {
            if (host_ours()) (void)hipHostFree(host);
            if (dev_ours()) (void)hipFree(dev);
        }
        host = host_dev = dev = nullptr;
        host_id = dev_id = 0;
        words = 0;
    }
    hipError_t reserve(size_t need) {
        int current = -1;
        hipError_t e = hipGetDevice(&current);
        if (e != hipSuccess) return e;
        if (need <= words && current == device && owner == getpid() && host_ours() && dev_ours()) return hipSuccess;
        release();
        size_t n = 4096;
        while (n < need) n *= 2;
        owner = getpid();
        device = current;
        if ((e = hipMalloc((void **)&dev, n * 4)) == hipSuccess && (dev_id = allocation_of(dev)) == 0) {
            (void)hipFree(dev);
            e = hipErrorNotSupported;
        }
        if (e == hipSuccess && (e = hipHostMalloc((void **)&host, n * 4, hipHostMallocMapped | hipHostMallocCoherent)) == hipSuccess && (host_id = allocation_of(host)) == 0) {
            (void)hipHostFree(host);
            e = hipErrorNotSupported;
        }
        if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&host_dev, host, 0);
        if (e != hipSuccess) { release(); return e; }
        words = n;
        return hipSuccess;
    }
    ~Buffers() { release(); }
};
struct Words { const int32_t *at; size_t n; };
// the lists back to back into device memory, through the two halves of the thread's pinned buffer behind the result: one is on
// its way while the other is filled
hipError_t copy_through(const Buffers &b, int *dev, std::initializer_list<Words> lists) {
    const size_t half = (b.words - RESULT_WORDS) / 2;
    int *piece = b.host + RESULT_WORDS, *other = piece + half;
    size_t held = 0;
    auto flush = [&]() {
        hipError_t e = hipStreamSynchronize(nullptr);                       // (the other half has left)
        if (e == hipSuccess) e = hipMemcpyAsync(dev, piece, held * 4, hipMemcpyHostToDevice, nullptr);
        dev += held;
        held = 0;
        std::swap(piece, other);
        return e;
    };
    for (Words w : lists)
        while (w.n > 0) {
            const size_t take = w.n < half - held ? w.n : half - held;
            memcpy(piece + held, w.at, take * 4);
            held += take;
            w.at += take;
            w.n -= take;
            if (held < half) continue;
            const hipError_t e = flush();
            if (e != hipSuccess) return e;
        }
    return held > 0 ? flush() : hipSuccess;
}
}

static int fail(int code, const std::string &text) {
    llma_set_error_text(text.c_str());
    return code;
}

extern "C" int llma_find_trigger(const int32_t *y, int32_t y_len, const int32_t *ref, const int32_t *doc_offsets,
                                 int32_t n_docs, int32_t n, int32_t *doc_out, int32_t *pos_out) {
    if (!doc_out || !pos_out || !doc_offsets || n_docs < 0 || y_len < 0 || (!y && y_len > 0))
        return fail(LLMA_E_INVAL, "llma_find_trigger: null pointer or negative count");
    if (n < 1) return fail(LLMA_E_INVAL, "llma_find_trigger: n must be >= 1");
    for (int j = 0; j < n_docs; ++j)
        if (doc_offsets[j + 1] < doc_offsets[j] || doc_offsets[0] != 0)
            return fail(LLMA_E_INVAL, "llma_find_trigger: doc_offsets must start at 0 and be non-decreasing");
    *doc_out = -1;
    *pos_out = -1;
    const int ref_len = n_docs > 0 ? doc_offsets[n_docs] : 0;
    if (ref_len > 0 && !ref) return fail(LLMA_E_INVAL, "llma_find_trigger: null reference");
    if (ref_len == 0 || y_len < n) return 0;

    const size_t n_in = (size_t)y_len + (size_t)ref_len + (size_t)(n_docs + 1), in_words = (n_in + 3) / 4 * 4;
    const size_t need = RESULT_WORDS + in_words + 2 * (size_t)trigger_spans(ref_len);
    static thread_local Buffers b;
    const bool large = need > TRIGGER_KEEP_WORDS;
    int *large_dev = nullptr;
    hipError_t e = b.reserve(large ? TRIGGER_KEEP_WORDS : need);
    if (e == hipSuccess && large) e = hipMalloc((void **)&large_dev, need * 4);
    if (e != hipSuccess) {
        (void)hipGetLastError();                // (reported here, not by a later call)
        return fail(LLMA_E_NOMEM, std::string("llma_find_trigger: allocation: ") + hipGetErrorString(e));
    }
    b.host[0] = -1;
    if (!large) {
        int *in = b.host + RESULT_WORDS;
        memcpy(in, y, (size_t)y_len * 4);
        memcpy(in + y_len, ref, (size_t)ref_len * 4);
        memcpy(in + y_len + ref_len, doc_offsets, (size_t)(n_docs + 1) * 4);
        launch_trigger_host(b.host_dev + RESULT_WORDS, b.dev, (int)(in_words / 4), y_len, ref_len, n_docs, n, (unsigned long long *)(b.dev + in_words), b.host_dev, nullptr);
    } else {
        e = copy_through(b, large_dev, {{y, (size_t)y_len}, {ref, (size_t)ref_len}, {doc_offsets, (size_t)(n_docs + 1)}});
        if (e == hipSuccess)
            launch_trigger_plain(large_dev, y_len, large_dev + y_len, large_dev + y_len + ref_len, ref_len, n_docs, n, (unsigned long long *)(large_dev + in_words), b.host_dev, false, nullptr);
    }
    if (e == hipSuccess) e = hipGetLastError();
    const hipError_t waited = hipStreamSynchronize(nullptr);        // (the kernels read and write the buffers: also after an error)
    if (large) (void)hipFree(large_dev);
    if (e == hipSuccess) e = waited;
    if (e != hipSuccess) return fail(LLMA_E_HIP, std::string("llma_find_trigger: ") + hipGetErrorString(e));
    const int found = __atomic_load_n(&b.host[0], __ATOMIC_ACQUIRE);
    if (found != 0 && found != 1) return fail(LLMA_E_HIP, "llma_find_trigger: the scan left no result");
    if (found) { *doc_out = b.host[1]; *pos_out = b.host[2]; }
    return found;
}
