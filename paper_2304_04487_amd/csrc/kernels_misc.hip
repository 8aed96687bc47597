// Small kernels around the GEMMs and attention: row set-up with the embedding gather, the vocabulary arg max with the prefix-accept / KV-truncate decision
// (paper: Algorithm 1, the compare loop after the verification forward), and the n-gram
// trigger scan over the reference (paper: Method, the match that starts a copy).
#include "common.h"
#include "kernels.h"

// ---------------------------------------------------------------------------------------------
// trigger: scan of the reference for the n-token tail of y
// ---------------------------------------------------------------------------------------------
// Flat position p is a candidate when it lies at least n tokens into its document and the n
// tokens before it equal the tail of y; its score is how far that agreement extends backwards
// (bounded by the document start and by the start of y).  The best candidate maximises
// (score, then smallest flat position) -- flat order is (document, position) order.
//
// What bounds it: one workgroup reads at the rate of its own loads in flight (600 011 tokens: 180 us = 13 GB/s),
// so a reference is cut into spans of TRIGGER_SPAN positions, one workgroup each, 16 loads per thread in flight;
// the spans' best keys are merged by whoever needs them (a maximum: the order does not matter).  Most positions stop at
// the one-token test.  What survives it is one position in 32000 for uniform ids, but 5 % of a text whose last token is a
// comma or a newline, so each wave gathers its survivors and handles them a lane each: the document by binary search, seven more
// tokens, all requested at once.  The few that go on are followed one at a time by their wave, 64 tokens per step, best
// prospect first -- in a repetitive text the first drops all others -- and side by side, 16 tokens per step, while there are many.
// (Every survivor followed by its wave, one after the other, took 31 us at 5 % of 4096 positions, 223 at 50 %: now 5 and 10.)
// A call over 600 011 tokens on the device: 245 us in one workgroup, now 8.1; one span (the usual reference of a few
// documents) is one launch (1472 host tokens: 44.3 -> 41.1 us, the rest is the copies).
//
// The document list may come from device memory the host cannot check: a start below 0 is taken as 0, so that no
// list makes the backward walk leave the reference.
__device__ __forceinline__ int doc_of(const int *doc_offsets, int n_docs, int p) {
    int lo = 0, hi = n_docs;              // largest j with doc_offsets[j] <= p
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (doc_offsets[mid] <= p) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ unsigned long long block_max(unsigned long long best) {
    butterfly<32>([&](auto off) {
        const unsigned long long o = lane_xor<off.value>(best);
        best = o > best ? o : best;
    });
    __shared__ unsigned long long wbest[4];                     // (256 threads)
    if ((threadIdx.x & 63) == 0) wbest[threadIdx.x >> 6] = best;
    __syncthreads();
    best = wbest[0];
    for (int w = 1; w < 4; ++w) best = wbest[w] > best ? wbest[w] : best;
    return best;
}

__device__ __forceinline__ unsigned long long trigger_key(int score, int p) {
    return ((unsigned long long)score << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)p);
}
__device__ __forceinline__ int key_position(unsigned long long key) { return (int)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull)); }

// best key (score << 32 | ~position) of the positions [p_lo, p_hi), p_hi - p_lo <= TRIGGER_SPAN; 256 threads
__device__ __forceinline__ unsigned long long scan_span(const int *y, int i, const int *ref, const int *doc_offsets, int n_docs,
                                                        int p_lo, int p_hi, int n) {
    constexpr int U = TRIGGER_SPAN / 256, PROBE = 8, STRIDE = 16;
    __shared__ unsigned short hits_of[4][TRIGGER_SPAN / 4];     // each wave's survivors of the one-token test: p - p_lo, ascending
    unsigned long long best = 0ull;
    int prev[U];
    if (p_lo < p_hi) {                                          // (uniform; y's length may still be on its way from memory)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p_lo + u * 256 + (int)threadIdx.x;
            prev[u] = ref[p < 1 ? 0 : (p < p_hi ? p - 1 : p_hi - 1)];
        }
    }
    if (i >= n && p_lo < p_hi) {                                // uniform
        const int lane = threadIdx.x & 63;
        const auto token_before = [&](int q, int t) { return ref[q - 1 - t > 0 ? q - 1 - t : 0]; };    // (compared only where it exists)
        const auto tail = [&](int t) { return y[i - 1 - t > 0 ? i - 1 - t : 0]; };
        unsigned short *const hit = hits_of[threadIdx.x >> 6];
        int total = 0;
        int want[PROBE];
#pragma unroll
        for (int t = 0; t < PROBE; ++t) want[t] = tail(t);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p_lo + u * 256 + (int)threadIdx.x;
            const bool same = p >= 1 && p < p_hi && prev[u] == want[0];
            const unsigned long long hits = __ballot(same);
            if (same) hit[total + __popcll(hits & ((1ull << lane) - 1ull))] = (unsigned short)(p - p_lo);
            total += __popcll(hits);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (what one lane wrote, another reads: within the wave, no barrier)
        for (int h0 = 0; h0 < total; h0 += 64) {                // a survivor per lane
            const bool mine = h0 + lane < total;
            const int q = p_lo + hit[mine ? h0 + lane : 0];
            int got[PROBE];
#pragma unroll
            for (int t = 1; t < PROBE; ++t) got[t] = token_before(q, t);
            int start = doc_offsets[doc_of(doc_offsets, n_docs, q)];
            start = start > 0 ? start : 0;
            const int limit = !mine ? 0 : (q - start < i ? q - start : i);
            int score = limit > 0 ? 1 : 0;                      // (limit < 0: a document list that decreases)
#pragma unroll
            for (int t = 1; t < PROBE; ++t)
                if (score == t && t < limit && got[t] == want[t]) score = t + 1;
            bool more = score == PROBE && limit > PROBE;        // the comparison goes on
            if (!more && score >= n) {
                const unsigned long long key = trigger_key(score, q);
                best = key > best ? key : best;
            }
            for (unsigned long long left; (left = __ballot(more)) != 0ull;) {
                // what cannot beat the wave's best is dropped; of the others the one with the most to gain is
                // followed to its end by the whole wave, 64 tokens at a time
                unsigned long long top = best;
                const unsigned long long bound = more ? trigger_key(limit, q) : 0ull;
                unsigned long long lead = bound;
                if ((left & (left - 1ull)) != 0ull) {           // (one alone is simply followed)
                    butterfly<32>([&](auto off) {
                        const unsigned long long a = lane_xor<off.value>(top), b = lane_xor<off.value>(lead);
                        top = a > top ? a : top;
                        lead = b > lead ? b : lead;
                    });
                    if (lead <= top) break;
                    left = __ballot(bound == lead);
                }
                const int src = __ffsll(left) - 1;
                lead = __shfl(bound, src);
                const int ql = key_position(lead), ll = (int)(lead >> 32);
                int sl = __shfl(score, src);
                for (; sl < ll; sl += 64) {
                    const int t = sl + lane;
                    const unsigned long long stop = __ballot(t >= ll || token_before(ql, t) != tail(t));
                    if (stop != 0ull) { sl += __ffsll(stop) - 1; break; }
                }
                if (sl >= n) {
                    const unsigned long long key = trigger_key(sl, ql);
                    best = key > best ? key : best;
                    top = key > top ? key : top;
                }
                more = more && lane != src && bound > top;
                if (__popcll(__ballot(more)) <= 4) continue;
                // many left: each goes on by itself for a while
                int x[STRIDE], z[STRIDE];
#pragma unroll
                for (int e = 0; e < STRIDE; ++e) { x[e] = token_before(q, score + e); z[e] = tail(score + e); }
                const int from = score;
                bool go = more;
#pragma unroll
                for (int e = 0; e < STRIDE; ++e) {
                    go = go && from + e < limit && x[e] == z[e];
                    score += go;
                }
                if (more && !go) {
                    if (score >= n) {
                        const unsigned long long key = trigger_key(score, q);
                        best = key > best ? key : best;
                    }
                    more = false;
                }
            }
        }
    }
    return block_max(best);
}

// llma_generate: grid (spans of the longest reference, sequences); part[sequence][span] = the span's best key
__global__ __launch_bounds__(256) void trigger_scan_kernel(const GenState *gp, unsigned long long *part) {
    const GenState G = gp[blockIdx.y];
    const int i = *G.n_out;
    const long first = (long)blockIdx.x * TRIGGER_SPAN;         // (the grid may be larger than this sequence's reference)
    const int p_lo = first < G.ref_len ? (int)first : G.ref_len;
    int p_hi = G.ref_len - p_lo > TRIGGER_SPAN ? p_lo + TRIGGER_SPAN : G.ref_len;
    if (G.k <= 0 || i >= G.max_new) p_hi = p_lo;
    const unsigned long long best = scan_span(G.y, i, G.ref, G.doc_offsets, G.n_docs, p_lo, p_hi, G.n);
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = best;
}
void launch_trigger_scan(const GenState *gen_dev, int n_seqs, int spans, unsigned long long *part, hipStream_t st) {
    hipLaunchKernelGGL(trigger_scan_kernel, dim3(spans, n_seqs), dim3(256), 0, st, gen_dev, part);
}

// check_offsets (callers whose document list lives in device memory, where the host cannot look):
// the list must start at 0, never decrease and end at ref_len; otherwise result = (-1, -1, -1).  Every
// workgroup checks a share of the list; a fault is the largest of all keys.
#define TRIGGER_BAD_LIST (~0ull)
__device__ __forceinline__ void trigger_write_result(unsigned long long best, const int *doc_offsets, int n_docs, int *result) {
    if (best == TRIGGER_BAD_LIST) { result[0] = -1; result[1] = -1; result[2] = -1; return; }
    if (best == 0ull) { result[0] = 0; result[1] = -1; result[2] = -1; return; }
    const int p = key_position(best), doc = doc_of(doc_offsets, n_docs, p);
    result[0] = 1; result[1] = doc; result[2] = p - doc_offsets[doc];
}
__global__ __launch_bounds__(256) void trigger_plain_kernel(const int *y, int y_len, const int *ref, const int *doc_offsets, int ref_len,
                                                            int n_docs, int n, unsigned long long *part, int *result, int check_offsets) {
    if (ref_len <= 0 || n_docs <= 0) {
        if (threadIdx.x == 0) { result[0] = 0; result[1] = -1; result[2] = -1; }
        return;
    }
    int bad = 0;
    if (check_offsets) {
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n_docs; j += gridDim.x * 256) bad |= doc_offsets[j + 1] < doc_offsets[j];
        if (blockIdx.x == 0 && threadIdx.x == 0) bad |= (doc_offsets[0] != 0) | (doc_offsets[n_docs] != ref_len);
    }
    const int p_lo = (int)blockIdx.x * TRIGGER_SPAN;
    const int p_hi = ref_len - p_lo > TRIGGER_SPAN ? p_lo + TRIGGER_SPAN : ref_len;
    unsigned long long best = scan_span(y, y_len, ref, doc_offsets, n_docs, p_lo, p_hi, n);
    if (check_offsets && __syncthreads_or(bad)) best = TRIGGER_BAD_LIST;
    if (threadIdx.x != 0) return;
    if (gridDim.x == 1) trigger_write_result(best, doc_offsets, n_docs, result);
    else part[blockIdx.x] = best;
}
__global__ __launch_bounds__(256) void trigger_plain_merge_kernel(const unsigned long long *part, int spans, const int *doc_offsets, int n_docs, int *result) {
    unsigned long long best = 0ull;
    for (int t = threadIdx.x; t < spans; t += 256) {
        const unsigned long long o = part[t];
        best = o > best ? o : best;
    }
    best = block_max(best);
    if (threadIdx.x == 0) trigger_write_result(best, doc_offsets, n_docs, result);
}
void launch_trigger_plain(const int *y, int y_len, const int *ref, const int *doc_offsets, int ref_len, int n_docs, int n,
                          unsigned long long *part, int *result, bool check_offsets, hipStream_t st) {
    const int spans = (ref_len <= 0 || n_docs <= 0) ? 1 : trigger_spans(ref_len);
    hipLaunchKernelGGL(trigger_plain_kernel, dim3(spans), dim3(256), 0, st, y, y_len, ref, doc_offsets, ref_len, n_docs, n, part, result,
                       check_offsets ? 1 : 0);
    if (spans > 1) hipLaunchKernelGGL(trigger_plain_merge_kernel, dim3(1), dim3(256), 0, st, part, spans, doc_offsets, n_docs, result);
}

// Inputs in pinned host memory cross the bus once, 16 bytes per lane and eight requests per lane in flight: each is a round trip of
// microseconds, and a scan that read them in place would make several in a row.
__device__ __forceinline__ void take_pieces(const u32x4 *in, u32x4 *out, int pieces, int first, int stride) {
    constexpr int U = 8;
    for (int i0 = first; i0 < pieces; i0 += U * stride) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = in[i0 + u * stride < pieces ? i0 + u * stride : i0];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * stride < pieces) out[i0 + u * stride] = v[u];
    }
}
__global__ __launch_bounds__(256) void take_pieces_kernel(const u32x4 *in, u32x4 *out, int pieces) {
    take_pieces(in, out, pieces, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
}
// a reference of one span: copy and scan in one workgroup, one launch
__global__ __launch_bounds__(256) void trigger_host_kernel(const u32x4 *in, int *dev, int pieces, int y_len, int ref_len, int n_docs, int n, int *result) {
    take_pieces(in, (u32x4 *)dev, pieces, threadIdx.x, 256);
    __syncthreads();
    const int *ref = dev + y_len, *doc_offsets = ref + ref_len;
    const unsigned long long best = scan_span(dev, y_len, ref, doc_offsets, n_docs, 0, ref_len, n);
    if (threadIdx.x == 0) trigger_write_result(best, doc_offsets, n_docs, result);
}
void launch_trigger_host(const int *in, int *dev, int pieces, int y_len, int ref_len, int n_docs, int n, unsigned long long *part, int *result, hipStream_t st) {
    // (one workgroup for all: as long as the copy is a few trips of it)
    if (trigger_spans(ref_len) == 1 && pieces <= 4 * 8 * 256) {
        hipLaunchKernelGGL(trigger_host_kernel, dim3(1), dim3(256), 0, st, (const u32x4 *)in, dev, pieces, y_len, ref_len, n_docs, n, result);
        return;
    }
    const int blocks = (pieces + 8 * 256 - 1) / (8 * 256);
    hipLaunchKernelGGL(take_pieces_kernel, dim3(blocks), dim3(256), 0, st, (const u32x4 *)in, (u32x4 *)dev, pieces);
    launch_trigger_plain(dev, y_len, dev + y_len, dev + y_len + ref_len, ref_len, n_docs, n, part, result, false, st);
}

// ---------------------------------------------------------------------------------------------
// row set-up
// ---------------------------------------------------------------------------------------------
// Host memory is read and written by these kernels directly, a handful of words per sequence: every copy between host and
// device was a launch of its own (3.6 us on the device, more on the host), six to nine of them per verification step.
// A four-layer 7B step of one row: 474 -> 426 us per call.  One workgroup reads, each word once: uncached words asked for by
// every thread that needs them cost 135 us at 144 rows.
__device__ __forceinline__ void host_write(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

// verification steps: brings the device's copies of what the host knows up to date
__global__ __launch_bounds__(256) void take_step_kernel(StepState s, int n_seqs, int max_k) {
    for (int i = threadIdx.x; i < n_seqs * max_k; i += 256) s.draft[i] = s.io.draft[i];
    for (int b = threadIdx.x; b < n_seqs; b += 256) {
        const int slot = s.io.slot[b], keff = s.io.keff[b], T = s.io.T[b], pending = s.io.pending[b], lo_from = s.io.lo_from[b];
        s.batch_slots[b] = slot;
        s.keff[b] = keff;
        s.T[slot] = T;
        s.pending[slot] = pending;
        s.lo_from[slot] = lo_from;
    }
}
void launch_take_step(const StepState &s, int n_seqs, int max_k, hipStream_t st) {
    hipLaunchKernelGGL(take_step_kernel, dim3(1), dim3(256), 0, st, s, n_seqs, max_k);
}

// h[r] = E[tok]; bf16: x = h * gain as hi/lo tiled planes, per (row, 16-feature tile) sum of squares, one thread per tile
template <bool BF16>
__device__ __forceinline__ void embed_row(const EmbedArgs &e, int r, int tok) {
    if (!BF16) {
        const float *src = (const float *)e.embed + (size_t)tok * e.d;
        for (int c = threadIdx.x; c < e.d; c += 256) e.h[(size_t)r * e.d + c] = src[c];
        return;
    }
    const int n_tiles = e.d / 16;
    for (int ft = threadIdx.x; ft < n_tiles; ft += 256) {
        const u32x4 *src = (const u32x4 *)((const bf16_t *)e.embed + (size_t)tok * e.d + ft * 16);
        u32x4 raw[2] = {src[0], src[1]};
        float ss = 0.f;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float v[8], x[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[2 * j] = __uint_as_float(raw[half][j] << 16);
                v[2 * j + 1] = __uint_as_float(raw[half][j] & 0xFFFF0000u);
            }
            const int c0 = ft * 16 + half * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j) { ss += v[j] * v[j]; x[j] = v[j] * e.gain[c0 + j]; }
            *(f32x4 *)(e.h + (size_t)r * e.d + c0) = (f32x4){v[0], v[1], v[2], v[3]};
            *(f32x4 *)(e.h + (size_t)r * e.d + c0 + 4) = (f32x4){v[4], v[5], v[6], v[7]};
            u32x2 h0, l0, h1, l1;
            split4(x, h0, l0);
            split4(x + 4, h1, l1);
            const size_t o = xtile_off(r, c0, e.KSp, e.quads);
            *(u32x4 *)((bf16_t *)e.nx_hi + o) = (u32x4){h0[0], h0[1], h1[0], h1[1]};
            *(u32x4 *)((bf16_t *)e.nx_lo + o) = (u32x4){l0[0], l0[1], l1[0], l1[1]};
        }
        e.ssq_out[(size_t)r * n_tiles + ft] = ss;
    }
}

// One workgroup per row: token, position, slot, the row's rotary (cos, sin) pairs out of the position table, and the
// row's embedding.  Generation steps (gp set): every row's workgroup finds the step's trigger for itself -- the maximum
// over the spans' keys, or the scan itself when the reference is one span -- and the first row's publishes keff, the
// drafts and the trigger's place.  Three launches (scan, set-up, embedding: 3.3 + 3.4 + 2.7 us at d = 512, nine rows) became one of 5.9 us.
template <bool BF16>
__global__ __launch_bounds__(256) void setup_step_rows_kernel(StepState s, int m, int max_k, const float *cs, int half, EmbedArgs e,
                                                              const GenState *gp, const unsigned long long *part, int spans) {
    const int idx = blockIdx.x;
    const int b = idx / m, j = idx % m;
    const int slot = s.batch_slots[b];
    const int T = s.T[slot];
    int keff, tok = s.pending[slot];
    // (the row's rotary pairs, at most 128 words, are requested with the first loads and stored with the last)
    const float cs_word = cs[(size_t)(T + j) * 2 * half + ((int)threadIdx.x < 2 * half ? threadIdx.x : 0)];
    if (gp == nullptr) {
        keff = s.keff[b];
        if (j > 0) tok = s.draft[b * max_k + j - 1];
    } else {
        const GenState G = gp[b];
        const int n_out = *G.n_out;
        unsigned long long best = 0ull;
        if (spans == 1) {
            best = scan_span(G.y, n_out < G.max_new ? n_out : -1, G.ref, G.doc_offsets, G.n_docs, 0, G.k > 0 ? G.ref_len : 0, G.n);   // (n >= 1)
        } else {
            for (int t = threadIdx.x; t < spans; t += 256) {
                const unsigned long long o = part[(size_t)b * spans + t];
                best = o > best ? o : best;
            }
            best = block_max(best);
        }
        keff = 0;
        if (best != 0ull) {
            const int p = key_position(best), doc = doc_of(G.doc_offsets, G.n_docs, p);
            const int left_in_doc = G.doc_offsets[doc + 1] - p;
            const int budget = G.max_new - n_out - 1;
            keff = G.k < left_in_doc ? G.k : left_in_doc;
            keff = keff < budget ? keff : budget;
            keff = keff < 0 ? 0 : keff;
            if (j > 0 && j <= keff) tok = G.ref[p + j - 1];
            if (j == 0) {
                if (threadIdx.x == 0) { G.cur[0] = doc; G.cur[1] = p - G.doc_offsets[doc]; }
                for (int t = threadIdx.x; t < keff; t += 256) s.draft[b * max_k + t] = G.ref[p + t];
            }
        }
        if (j == 0 && threadIdx.x == 0) s.keff[b] = keff;
    }
    tok = j <= keff ? tok : 0;                                    // rows past keff are padding
    const int pos = T + j;
    embed_row<BF16>(e, idx, tok);
    if ((int)threadIdx.x < 2 * half) s.row_cs[(size_t)idx * 2 * half + threadIdx.x] = cs_word;
    if (threadIdx.x == 0) {
        s.row_tok[idx] = tok;
        s.row_pos[idx] = pos;
        s.row_slot[idx] = slot;
    }
}
void launch_setup_step_rows(const StepState &s, int n_seqs, int m, int max_k, const float *cs, int half, const EmbedArgs &e,
                            const GenState *gen_dev, const unsigned long long *part, int spans, hipStream_t st) {
    if (e.gain) hipLaunchKernelGGL((setup_step_rows_kernel<true>), dim3(n_seqs * m), dim3(256), 0, st, s, m, max_k, cs, half, e, gen_dev, part, spans);
    else hipLaunchKernelGGL((setup_step_rows_kernel<false>), dim3(n_seqs * m), dim3(256), 0, st, s, m, max_k, cs, half, e, gen_dev, part, spans);
}

template <bool BF16>
__global__ __launch_bounds__(256) void setup_prefill_rows_kernel(StepState s, const int *prompt, const int *base, int slot, const float *cs, int half, EmbedArgs e) {
    const int j = blockIdx.x;
    int pos, tok;
    if (e.segs != nullptr) {
        const PromptSeg seg = e.segs[segment_of<&PromptSeg::row0>(e.segs, e.n_segs, j)];
        slot = seg.slot;
        pos = s.T[slot] + j - seg.row0;
        tok = prompt[seg.tok0 + j - seg.row0];
    } else {
        pos = s.T[slot] + j;
        tok = prompt[pos - *base];
    }
    embed_row<BF16>(e, j, tok);
    if (threadIdx.x == 0) {
        s.row_tok[j] = tok;
        s.row_pos[j] = pos;
        s.row_slot[j] = slot;
        if (j == 0) s.batch_slots[0] = slot;
    }
    for (int i = threadIdx.x; i < 2 * half; i += 256) s.row_cs[(size_t)j * 2 * half + i] = cs[(size_t)pos * 2 * half + i];
}
void launch_setup_prefill_rows(const StepState &s, const int *prompt_dev, const int *base_dev, int m, int slot,
                               const float *cs, int half, const EmbedArgs &e, hipStream_t st) {
    if (e.gain) hipLaunchKernelGGL((setup_prefill_rows_kernel<true>), dim3(m), dim3(256), 0, st, s, prompt_dev, base_dev, slot, cs, half, e);
    else hipLaunchKernelGGL((setup_prefill_rows_kernel<false>), dim3(m), dim3(256), 0, st, s, prompt_dev, base_dev, slot, cs, half, e);
}

__global__ void advance_T_kernel(StepState s, int slot, int by) { s.T[slot] += by; }
void launch_advance_T(const StepState &s, int slot, int by, hipStream_t st) {
    hipLaunchKernelGGL(advance_T_kernel, dim3(1), dim3(1), 0, st, s, slot, by);
}

// ---------------------------------------------------------------------------------------------
// vocabulary arg max (lowest id on exact ties) + prefix accept + KV truncate
// ---------------------------------------------------------------------------------------------
// One workgroup per sequence.  o_j = arg max of row j for j = 0..keff; a = longest prefix with
// o_i == draft_i; the step emits o_0..o_a, the cache keeps the rows of the pending token and
// of the a accepted drafts (T += a + 1; rows beyond are overwritten by the next step), and
// o_a becomes the pending token.
// Bound by latency: a row is 2000 partials (8 KB of values) at vocabulary 32000, and the decision is a chain of small reads.
// Sixteen waves take a row each (33 rows: three rounds), 2048 partials in flight, requested before the draft
// count is known; of the token ids, which ascend with the partials, only the winner's is read; the drafts are compared by 33 lanes
// at once; what the bookkeeping adds to is requested at the start.  Four partials
// per load, a chain of comparisons for each of the four.  Back to back at 1 / 9 / 17 / 33 rows 3.9 / 5.1 / 6.8 / 10.6 -> 2.6 / 3.4 / 4.1 / 6.1 us, a fp32
// model's 512 partials at five rows 3.2 -> 2.3 (ids and values read side by side, one chain with ties in it; one thread's walk over the drafts was 41 at 33).
#define ACCEPT_THREADS 1024
__global__ __launch_bounds__(ACCEPT_THREADS) void argmax_accept_kernel(const float *__restrict__ pval, const int *__restrict__ pidx,
                                                                       int n_part, StepState s, int m, int max_k, int vocab, const GenState *gen) {
    constexpr int WAVES = ACCEPT_THREADS / 64;
    __shared__ int o[40];
    const int b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (gen != nullptr) gen += b;                                // llma_generate: one GenState per sequence of the batch
    const int keff = s.keff[b];
    const int slot = s.batch_slots[b];
    int n_out = 0, step = 0, doc = 0, doc_pos = 0;
    if (gen != nullptr) { n_out = *gen->n_out; step = *gen->n_steps; doc = gen->cur[0]; doc_pos = gen->cur[1]; }
    const int T = s.T[slot];
    int draft = -1;
    // one row per wave at a time: wave w reduces rows w, w + 16, ... over the per-tile partials (rows past keff are
    // rows of the step too: their partials exist, what they say is dropped)
    for (int j = wave; j < m; j += WAVES) {
        const size_t r = (size_t)b * m + j;
        float bv = LLMA_NEG_INF;
        int bt = 0x7fffffff;
        const float *const row = pval + r * n_part;
        const auto look = [&](auto width, auto in_flight) {      // a lane takes `width` neighbours at a time
            constexpr int E = decltype(width)::value, U = decltype(in_flight)::value, TRIP = 64 * E;
            float best[E];                                       // per place in the group: a chain of their own, indices ascend
            int where[E];
#pragma unroll
            for (int e = 0; e < E; ++e) { best[e] = LLMA_NEG_INF; where[e] = 0x7fffffff; }
            for (int first = 0; first < n_part; first += U * TRIP) {
                float v[U][E];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int t = first + u * TRIP + lane * E;
                    __builtin_memcpy(v[u], __builtin_assume_aligned(row + (t < n_part ? t : 0), 4 * E), 4 * E);
                }
                if (j > keff) return;                            // uniform; padding (the count arrived with the first partials)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int t = first + u * TRIP + lane * E;
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        if (t < n_part && v[u][e] > best[e]) { best[e] = v[u][e]; where[e] = t + e; }
                }
            }
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (best[e] > bv || (best[e] == bv && where[e] < bt)) { bv = best[e]; bt = where[e]; }
        };
        if (n_part % 4 != 0) look(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
        else if (n_part <= 512) look(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
        else look(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
        if (j > keff) break;
        butterfly<32>([&](auto off) {
            const float ov = lane_xor<off.value>(bv);
            const int ot = lane_xor<off.value>(bt);
            if (ov > bv || (ov == bv && ot < bt)) { bv = ov; bt = ot; }
        });
        if (bt >= n_part) {                                      // (uniform) nothing above minus infinity: the first that is it
            for (int t = lane; t < n_part && bt >= n_part; t += 64)
                if (row[t] == LLMA_NEG_INF) bt = t;
            butterfly<32>([&](auto off) {
                const int ot = lane_xor<off.value>(bt);
                bt = ot < bt ? ot : bt;
            });
        }
        // a row without any comparable logit (all NaN: reachable through imported caches or weights that
        // hold non-finite values) must still yield a token id the next step's embedding gather can use
        int bi = bt >= n_part ? 0 : (n_part == vocab ? bt : pidx[r * n_part + bt]);      // (fp32 models: a partial per token)
        if ((unsigned)bi >= (unsigned)vocab) bi = 0;
        if (lane == 0) o[j] = bi;
        if (j == 0 && lane < keff) draft = s.draft[b * max_k + lane];
    }
    // the first wave decides: lane j compares draft j
    __syncthreads();
    if (wave != 0) return;
    if (gen != nullptr && n_out >= gen->max_new) return;         // a finished sequence / a step enqueued past the end: leave all state alone
    const unsigned long long same = __ballot(lane < keff && o[lane < keff ? lane : 0] == draft);
    const int a = __ffsll(~same) - 1;                            // (lane keff <= 32 never agrees)
    if (lane <= a) {
        if (gen != nullptr) gen->y[n_out + lane] = o[lane];
        else host_write(s.io.emit + b * (max_k + 1) + lane, o[lane]);
    }
    if (lane != 0) return;
    if (gen == nullptr) {
        host_write(s.io.nacc + b, a);
        host_write(s.io.next + b, o[a]);
    }
    s.T[slot] = T + a + 1;
    s.pending[slot] = o[a];
    if (gen != nullptr) {
        gen->trace[step * 4 + 0] = 1 + keff;
        gen->trace[step * 4 + 1] = a + 1;
        gen->trace[step * 4 + 2] = keff > 0 ? doc : -1;
        gen->trace[step * 4 + 3] = keff > 0 ? doc_pos : -1;
        const int now = n_out + a + 1;
        *gen->n_out = now;
        *gen->n_steps = step + 1;
        // the host reads the count of step `step` after that step's event, while the next step may be running: two places
        // in turn; the last step of a sequence fills both
        host_write(gen->host_count + (size_t)(step & 1) * gen->host_stride, now);
        if (now >= gen->max_new) host_write(gen->host_count + (size_t)((step & 1) ^ 1) * gen->host_stride, now);
    }
}
void launch_argmax_accept(const float *pval, const int *pidx, int n_part, const StepState &s, int n_seqs, int m,
                          int max_k, int vocab, const GenState *gen, hipStream_t st) {
    hipLaunchKernelGGL(argmax_accept_kernel, dim3(n_seqs), dim3(ACCEPT_THREADS), 0, st, pval, pidx, n_part, s, m, max_k, vocab, gen);
}
