// C ABI of the library (include/llma.h) and the host orchestration of a decoding step:
// which kernels run in which order for the verification forward (paper: Eq. 3), the accept /
// truncate decision and the LLMA loop (paper: Algorithm 1).  All arithmetic of the method runs
// in the kernels; this file validates arguments, owns device memory and enqueues launches.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "../../include/llma.h"
#include "common.h"
#include "kernels.h"

static thread_local std::string g_err;      // errors of calls that have no context
void llma_set_error_text(const char *text) { g_err = text ? text : ""; }   // for the library's other source files

#define PREFILL_ROWS_F32 48      // fp32 path: prompt rows per pass
#define PREFILL_ROWS_MAX 2048    // bf16 path: prompt rows per pass (whole prompt when it fits)

struct EventPair { hipEvent_t a, b; };

enum StepKind { STEP_PREFILL = 0, STEP_VERIFY = 1, STEP_GEN = 2, STEP_PROMPTS = 3 /* a prompt pass over several sequences */ };

// what a captured step graph was recorded for: (kind, sequences, rows per sequence, attention chunks, slot, trigger spans)
typedef std::array<int, 6> GraphKey;
struct GraphSlot { int seen = 0; uint64_t used = 0; hipGraphExec_t exec = nullptr; };     // used: when last, in run_step calls
#define GEN_STAGE_WORDS 16384    // words of a generation's inputs (and results) that pass through pinned memory (more: straight from the caller's)
#define GRAPH_SLOTS_MAX 256      // shapes remembered; beyond them the one not used for longest is forgotten

struct llma_ctx {
    llma_model_cfg cfg;
    hipStream_t st = nullptr;          // the caller's stream: everything is ordered on it
    hipStream_t run_st = nullptr;      // where the launchers enqueue: st, or cap_st while capturing
    hipStream_t cap_st = nullptr;      // private stream used only to capture step graphs
    std::map<GraphKey, GraphSlot> graphs;
    uint64_t graph_clock = 0;
    int *pin = nullptr;                // pinned host memory of steps: HostIo's arrays, then the decoding loop's output counts [2][max_batch]
    HostIo host{};                     // host addresses of the arrays (s.io: the device's)
    int *pin_counts = nullptr, *pin_counts_dev = nullptr;
    hipEvent_t cnt_ev[2] = {nullptr, nullptr};
    bool bf16 = false;
    std::vector<void *> allocs;
    int64_t dev_bytes = 0;
    std::string err;

    // weights (owned copies; bf16 matrices re-tiled)
    void *embed = nullptr, *lm_head = nullptr;
    float *final_norm = nullptr;
    std::vector<void *> wqkv, wo, wgu, wd;
    std::vector<float *> n1, n2;
    // KV cache per layer: [max_batch][H][seq_cap][dh]; bf16 with kv_split: a second (lo) plane.
    // seq_cap = max_seq rounded up to whole attention chunks, so a chunk's block loads never leave the allocation
    int seq_cap = 0;
    std::vector<void *> kc, vc, kc_lo, vc_lo;
    float *cs_table = nullptr;
    bool kv_split = false;

    // scratch for up to Rmax rows.  bf16: x/q/att/act are tiled hi/lo planes; fp32: row-major in *_hi
    int Rmax = 0;
    float *h = nullptr;
    void *xhi = nullptr, *xlo = nullptr, *q = nullptr, *q_lo = nullptr, *att_hi = nullptr, *att_lo = nullptr, *act_hi = nullptr, *act_lo = nullptr;
    float *po = nullptr, *pm = nullptr, *pl = nullptr;
    int *gen_segs = nullptr;           // PromptSeg[] of the pass over several sequences' prompts
    size_t cap_segs = 0;
    int n_segs = 0;                    // set while such a pass is enqueued, else 0
    const int *rows_live = nullptr;    // set per step: device count of live rows - 1 (generation, one sequence) or null
    float *part = nullptr;             // partial sums of launches that cut K over workgroups (contexts whose steps or passes can exceed 16 rows)
    int nc_max = 0;
    // bf16 GEMM work division, per-tile sums of squares of the residual rows, rstd of prompt rows
    GemmPlan plan_qkv{}, plan_o{}, plan_gu{}, plan_down{}, plan_lm{};
    float *ssq = nullptr, *rstd = nullptr;
    int Pmax = 0;                      // prompt rows processed per pass
    float *pval = nullptr;
    int *pidx = nullptr;
    int n_part = 0;

    StepState s{};
    GenState *gen_dev = nullptr;
    int *gen_prompt = nullptr;                    // prompts; in a generation the references and document lists behind them
    int *gen_part = nullptr;                      // the trigger's keys, [sequence of the batch][gen_spans] 64-bit words
    int gen_spans = 1;                            // spans the trigger scans per sequence in the current generation
    int *gen_y = nullptr, *gen_trace = nullptr;   // [sequence of the batch][max_new + 64] tokens, x 4 trace words
    int *gen_counters = nullptr;                  // n_out[max_batch], n_steps[max_batch], cur[max_batch][2], prefill base
    // s.T, s.pending, lo_from, s.batch_slots, gen_counters and gen_dev lie in one allocation, in this order, so that a generation
    // sends them in one copy; pin_block: pinned memory of the same layout.  pin_stage: a generation's inputs and results on their way
    int *block = nullptr, *pin_block = nullptr, *pin_stage = nullptr;
    size_t block_words = 0, block_states = 0;     // all of it; the words before gen_dev
    size_t cap_prompt = 0, cap_part = 0, cap_y = 0, cap_trace = 0;      // words

    // what the host knows about every slot; the device's copies (s.T, s.pending, lo_from) are brought up to date by the
    // next verification step, which carries them, or by sync_state before anything else reads them
    std::vector<int> T_host, pending_host;
    std::vector<char> stale;
    // Caches imported as bf16 values have all-zero lo planes: positions below lo_from[slot] (device
    // ints, host mirror) need no lo reads.  It is set when all layers of a slot have been imported
    // with one length and nothing was computed on the slot in between (imp_len records the lengths
    // since then, -1 = none); steps only ever write at positions >= T >= lo_from, reset clears it.
    std::vector<int> lo_from_host, imp_len;
    int *lo_from = nullptr;
    float *logits_dump = nullptr;
    int dump_rows = 0;
    int opt_split = 1, opt_timing = 0, opt_graph = 1;
    std::vector<EventPair> events;
};

static int fail(llma_ctx *c, int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    g_err = buf;
    return code;
}
#define HIP_TRY(c, expr)                                                                             \
    do {                                                                                             \
        hipError_t e_ = (expr);                                                                      \
        if (e_ != hipSuccess)                                                                        \
            return fail((c), e_ == hipErrorOutOfMemory ? LLMA_E_NOMEM : LLMA_E_HIP, "%s: %s", #expr, \
                        hipGetErrorString(e_));                                                      \
    } while (0)

static int dev_alloc(llma_ctx *c, void **p, size_t bytes) {
    if (bytes == 0) bytes = 16;
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) return fail(c, LLMA_E_NOMEM, "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
    c->allocs.push_back(*p);
    c->dev_bytes += (int64_t)bytes;
    return LLMA_OK;
}
#define ALLOC(c, ptr, bytes)                                         \
    do {                                                             \
        int rc_ = dev_alloc((c), (void **)&(ptr), (size_t)(bytes));  \
        if (rc_ != LLMA_OK) return rc_;                              \
    } while (0)

static void dev_free_one(llma_ctx *c, void *p) {
    if (!p) return;
    for (size_t i = 0; i < c->allocs.size(); ++i)
        if (c->allocs[i] == p) { c->allocs.erase(c->allocs.begin() + i); break; }
    (void)hipFree(p);
}

// ------------------------------------------------------------------------------------------------
// create / destroy
// ------------------------------------------------------------------------------------------------
static int check_cfg(const llma_model_cfg *g) {
    if (g->n_layers < 1 || g->d_model < 1 || g->n_heads < 1 || g->head_dim < 1 || g->d_ffn < 1 || g->vocab < 1)
        return fail(nullptr, LLMA_E_INVAL, "model dimensions must be positive");
    if (g->n_heads * g->head_dim != g->d_model) return fail(nullptr, LLMA_E_INVAL, "n_heads * head_dim != d_model");
    if (g->max_seq < 2 || g->max_batch < 1 || g->max_k < 0 || g->max_k > 32)
        return fail(nullptr, LLMA_E_INVAL, "need max_seq >= 2, max_batch >= 1, 0 <= max_k <= 32");
    if (g->dtype == LLMA_DTYPE_BF16) {
        if (g->d_model % 32 || g->d_ffn % 32 || g->vocab % 16)
            return fail(nullptr, LLMA_E_INVAL, "bf16 needs d_model %% 32 == 0, d_ffn %% 32 == 0, vocab %% 16 == 0");
        if (g->d_model > 1 << 23 || g->d_ffn > 1 << 23)       // 32-bit offsets inside a row block's activations (192 rows x 2^23 x 2 bytes; the block GEMM takes up to 2^21 columns)
            return fail(nullptr, LLMA_E_INVAL, "bf16 needs d_model and d_ffn <= 2^23");
        if (g->head_dim != 64 && g->head_dim != 128) return fail(nullptr, LLMA_E_INVAL, "bf16 needs head_dim 64 or 128");
    } else if (g->dtype == LLMA_DTYPE_F32) {
        if (g->head_dim != 32 && g->head_dim != 64 && g->head_dim != 128)
            return fail(nullptr, LLMA_E_INVAL, "fp32 needs head_dim 32, 64 or 128");
        if (g->d_model % 4) return fail(nullptr, LLMA_E_INVAL, "fp32 needs d_model %% 4 == 0");
    } else {
        return fail(nullptr, LLMA_E_INVAL, "unknown dtype %d", g->dtype);
    }
    if (!(g->rms_eps >= 0.f) || !(g->rope_theta > 0.f)) return fail(nullptr, LLMA_E_INVAL, "bad rms_eps / rope_theta");
    return LLMA_OK;
}

// copies one matrix into context-owned memory: fp32 as is, bf16 re-tiled (N rows, K padded to KSp k-steps)
static int take_matrix(llma_ctx *c, void **dst, const void *src, int N, int K, int KSp, int rope_dh) {
    if (c->bf16) {
        ALLOC(c, *dst, (size_t)(N / 16) * KSp * 1024);
        launch_pack_weight(src, *dst, N, K, KSp, rope_dh, c->cfg.d_model, c->st);
    } else {
        size_t bytes = (size_t)N * K * 4;
        ALLOC(c, *dst, bytes);
        HIP_TRY(c, hipMemcpyAsync(*dst, src, bytes, hipMemcpyDeviceToDevice, c->st));
    }
    return LLMA_OK;
}

static int autotune_tilek(llma_ctx *c);
static int create_impl(llma_ctx *c, const llma_weights *w) {
    const llma_model_cfg &g = c->cfg;
    const int L = g.n_layers, d = g.d_model, F = g.d_ffn, V = g.vocab, H = g.n_heads, dh = g.head_dim;
    const size_t es = c->bf16 ? 2 : 4;
    if (c->bf16) {
        c->plan_qkv = make_gemm_plan(3 * d, d, 1);
        c->plan_o = make_gemm_plan(d, d, 1);
        c->plan_gu = make_gemm_plan(F, d, 2);
        c->plan_down = make_gemm_plan(d, F, 1);
        c->plan_lm = make_gemm_plan(V, d, 1);
        if (const char *forced = getenv("LLMA_BLOCK_ROWS")) {     // tests: long prompt passes in blocks of 12 or 16 row tiles, or (0) none
            const int rt = atoi(forced);
            if (rt == 0 || rt == 12 || rt == 16)
                for (GemmPlan *p : {&c->plan_qkv, &c->plan_o, &c->plan_gu, &c->plan_down}) p->block_rt = rt;
        }
    }
    // ---- weights
    ALLOC(c, c->embed, (size_t)V * d * es);
    HIP_TRY(c, hipMemcpyAsync(c->embed, w->embed, (size_t)V * d * es, hipMemcpyDeviceToDevice, c->st));
    int rc = take_matrix(c, &c->lm_head, w->lm_head, V, d, c->plan_lm.KSp, 0);
    if (rc) return rc;
    ALLOC(c, c->final_norm, d * 4);
    HIP_TRY(c, hipMemcpyAsync(c->final_norm, w->final_norm, d * 4, hipMemcpyDeviceToDevice, c->st));
    c->wqkv.assign(L, nullptr); c->wo.assign(L, nullptr); c->wgu.assign(L, nullptr); c->wd.assign(L, nullptr);
    c->n1.assign(L, nullptr); c->n2.assign(L, nullptr);
    c->kc.assign(L, nullptr); c->vc.assign(L, nullptr); c->kc_lo.assign(L, nullptr); c->vc_lo.assign(L, nullptr);
    for (int l = 0; l < L; ++l) {
        if (!w->wqkv[l] || !w->wo[l] || !w->wgu[l] || !w->wdown[l] || !w->norm1[l] || !w->norm2[l])
            return fail(c, LLMA_E_INVAL, "null weight pointer in layer %d", l);
        if ((rc = take_matrix(c, &c->wqkv[l], w->wqkv[l], 3 * d, d, c->plan_qkv.KSp, dh))) return rc;
        if ((rc = take_matrix(c, &c->wo[l], w->wo[l], d, d, c->plan_o.KSp, 0))) return rc;
        if ((rc = take_matrix(c, &c->wgu[l], w->wgu[l], 2 * F, d, c->plan_gu.KSp, 0))) return rc;
        if ((rc = take_matrix(c, &c->wd[l], w->wdown[l], d, F, c->plan_down.KSp, 0))) return rc;
        ALLOC(c, c->n1[l], d * 4);
        ALLOC(c, c->n2[l], d * 4);
        HIP_TRY(c, hipMemcpyAsync(c->n1[l], w->norm1[l], d * 4, hipMemcpyDeviceToDevice, c->st));
        HIP_TRY(c, hipMemcpyAsync(c->n2[l], w->norm2[l], d * 4, hipMemcpyDeviceToDevice, c->st));
    }
    // ---- KV cache, zero-filled so that never-written positions hold finite values
    c->seq_cap = (g.max_seq + ATTN_CHUNK - 1) / ATTN_CHUNK * ATTN_CHUNK;
    const size_t kv_bytes = (size_t)g.max_batch * H * c->seq_cap * dh * es;
    for (int l = 0; l < L; ++l) {
        ALLOC(c, c->kc[l], kv_bytes);
        ALLOC(c, c->vc[l], kv_bytes);
        HIP_TRY(c, hipMemsetAsync(c->kc[l], 0, kv_bytes, c->st));
        HIP_TRY(c, hipMemsetAsync(c->vc[l], 0, kv_bytes, c->st));
        if (c->kv_split) {
            ALLOC(c, c->kc_lo[l], kv_bytes / 2);                  // lo planes: one byte per element
            ALLOC(c, c->vc_lo[l], kv_bytes / 2);
            HIP_TRY(c, hipMemsetAsync(c->kc_lo[l], 0, kv_bytes / 2, c->st));
            HIP_TRY(c, hipMemsetAsync(c->vc_lo[l], 0, kv_bytes / 2, c->st));
        }
    }
    // ---- rotary table: cos/sin(pos * theta^(-2i/dh)) in double, stored fp32
    {
        const int half = dh / 2;
        std::vector<float> cs((size_t)g.max_seq * half * 2);
        for (int i = 0; i < half; ++i) {
            const double inv = pow((double)g.rope_theta, -2.0 * i / (double)dh);
            for (int p = 0; p < g.max_seq; ++p) {
                const double ang = (double)p * inv;
                cs[((size_t)p * half + i) * 2] = (float)cos(ang);
                cs[((size_t)p * half + i) * 2 + 1] = (float)sin(ang);
            }
        }
        ALLOC(c, c->cs_table, cs.size() * 4);
        HIP_TRY(c, hipMemcpy(c->cs_table, cs.data(), cs.size() * 4, hipMemcpyHostToDevice));
    }
    // ---- scratch
    const int m_max = g.max_k + 1;
    c->Rmax = g.max_batch * m_max;
    // (the prompts of a batch share passes where its steps have more than 48 rows: llma_generate_batch)
    const long prompt_rows = (long)g.max_seq * (c->Rmax > 48 ? g.max_batch : 1);
    c->Pmax = c->bf16 ? (prompt_rows < PREFILL_ROWS_MAX ? (int)prompt_rows : PREFILL_ROWS_MAX) : PREFILL_ROWS_F32;
    if (c->Rmax < c->Pmax) c->Rmax = c->Pmax;
    const size_t Rp = ((size_t)c->Rmax + 127) / 128 * 128 + 48;  // slack: the GEMMs read whole row tiles / row blocks
    std::vector<std::pair<void *, size_t>> zero;
    auto zalloc = [&](void **p, size_t bytes) -> int { int r = dev_alloc(c, p, bytes); if (r == LLMA_OK) zero.push_back({*p, bytes}); return r; };
    if ((rc = zalloc((void **)&c->h, Rp * d * 4))) return rc;
    if (c->bf16) {
        const size_t Tt = Rp / 16;                                // row tiles
        const size_t x_bytes = Tt * c->plan_qkv.KSp * 1024, q_bytes = Tt * (d / 32) * 1024, act_bytes = Tt * c->plan_down.KSp * 1024;
        if ((rc = zalloc(&c->xhi, x_bytes)) || (rc = zalloc(&c->xlo, x_bytes)) || (rc = zalloc(&c->q, q_bytes)) ||
            (rc = zalloc(&c->q_lo, q_bytes)) || (rc = zalloc(&c->att_hi, x_bytes)) || (rc = zalloc(&c->att_lo, x_bytes)) ||
            (rc = zalloc(&c->act_hi, act_bytes)) || (rc = zalloc(&c->act_lo, act_bytes)))
            return rc;
        if ((rc = zalloc((void **)&c->ssq, Rp * (d / 16) * 4))) return rc;
        if ((rc = zalloc((void **)&c->rstd, Rp * 4))) return rc;
        c->nc_max = c->seq_cap / ATTN_CHUNK;
        // attention partials: [sequences][heads][chunks][rows], up to 48 rows per sequence (longer
        // prompt passes run the walking kernel, which has no partials)
        const size_t np = (size_t)g.max_batch * H * c->nc_max * 48;
        // partial sums of the split-K GEMM: batched steps of more than 48 rows, and prompt passes too short to fill
        // the chip without a split
        const int step_rows = g.max_batch * (g.max_k + 1);
        size_t part = 0;
        for (const GemmPlan *pl : {&c->plan_qkv, &c->plan_o, &c->plan_gu, &c->plan_down, &c->plan_lm}) {
            if (step_rows > 48) part = std::max(part, panel_part_bytes(*pl, step_rows, pl->n_split));
            if (pl != &c->plan_lm)
                for (int rows = 49; rows < c->Pmax + 16; rows += 16) {
                    const int r = rows < c->Pmax ? rows : c->Pmax;
                    part = std::max(part, panel_part_bytes(*pl, (r + 15) / 16 * 16, panel_prompt_split(*pl, r)));
                }
        }
        // and O and down of steps and short passes of 17 .. 48 rows, in the decoding GEMM's K slices
        const int few = std::min(48, std::max(step_rows, c->Pmax));
        if (few > 16) {
            for (const GemmPlan *pl : {&c->plan_o, &c->plan_down}) part = std::max(part, panel_part_bytes(*pl, few, pl->tk_waves));
            for (const GemmPlan *pl : {&c->plan_qkv, &c->plan_lm}) part = std::max(part, panel_part_bytes(*pl, few, tilek_groups(*pl)));
        }
        if (part > 0) ALLOC(c, c->part, part);
        ALLOC(c, c->po, np * dh * 4);
        ALLOC(c, c->pm, np * 4);
        ALLOC(c, c->pl, np * 4);
    } else {
        if ((rc = zalloc(&c->q, Rp * d * 4)) || (rc = zalloc(&c->att_hi, Rp * d * 4)) || (rc = zalloc(&c->act_hi, Rp * F * 4)))
            return rc;
    }
    for (auto &z : zero) HIP_TRY(c, hipMemsetAsync(z.first, 0, z.second, c->st));
    c->n_part = c->bf16 ? V / 16 : V;
    const size_t lm_rows = (size_t)g.max_batch * m_max;      // only decoding steps run the LM head
    ALLOC(c, c->pval, lm_rows * c->n_part * 4);
    ALLOC(c, c->pidx, lm_rows * c->n_part * 4);
    // ---- step state
    StepState &s = c->s;
    ALLOC(c, s.row_tok, Rp * 4);
    ALLOC(c, s.row_pos, Rp * 4);
    ALLOC(c, s.row_slot, Rp * 4);
    ALLOC(c, s.row_cs, Rp * dh * 4);
    HIP_TRY(c, hipMemsetAsync(s.row_cs, 0, Rp * dh * 4, c->st));
    {
        const size_t B = g.max_batch;
        c->block_states = (8 * B + 4 + 1) / 2 * 2;                // (GenState holds pointers: eight-byte aligned)
        c->block_words = c->block_states + sizeof(GenState) / 4 * B;
        static_assert(sizeof(GenState) % 8 == 0, "");
        ALLOC(c, c->block, c->block_words * 4);
        s.T = c->block; s.pending = c->block + B; c->lo_from = c->block + 2 * B; s.batch_slots = c->block + 3 * B;
        c->gen_counters = c->block + 4 * B;
        c->gen_dev = (GenState *)(c->block + c->block_states);
    }
    ALLOC(c, s.keff, g.max_batch * 4);
    ALLOC(c, s.draft, (size_t)g.max_batch * (g.max_k + 1) * 4);
    HIP_TRY(c, hipMemsetAsync(s.T, 0, g.max_batch * 4, c->st));
    HIP_TRY(c, hipMemsetAsync(s.pending, 0xFF, g.max_batch * 4, c->st));
    HIP_TRY(c, hipMemsetAsync(s.keff, 0, g.max_batch * 4, c->st));
    HIP_TRY(c, hipMemsetAsync(s.row_pos, 0, Rp * 4, c->st));
    HIP_TRY(c, hipMemsetAsync(s.row_slot, 0, Rp * 4, c->st));
    c->T_host.assign(g.max_batch, 0);
    c->pending_host.assign(g.max_batch, -1);
    c->stale.assign(g.max_batch, 0);
    c->lo_from_host.assign(g.max_batch, 0);
    c->imp_len.assign((size_t)g.max_batch * g.n_layers, -1);
    HIP_TRY(c, hipMemsetAsync(c->lo_from, 0, g.max_batch * 4, c->st));
    s.lo_from = c->lo_from;
    HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_st, hipStreamNonBlocking));
    {
        const size_t B = g.max_batch, sizes[9] = {B, B, B, B, B, B * (g.max_k + 1), B, B, B * m_max};
        size_t words = 2 * B;
        for (size_t n : sizes) words += n;
        words = (words + 3) / 4 * 4;
        const size_t block_at = words;
        words += (c->block_words + 3) / 4 * 4 + GEN_STAGE_WORDS;
        HIP_TRY(c, hipHostMalloc((void **)&c->pin, words * sizeof(int), hipHostMallocMapped | hipHostMallocCoherent));
        memset(c->pin, 0, words * sizeof(int));
        int *dev = nullptr;
        HIP_TRY(c, hipHostGetDevicePointer((void **)&dev, c->pin, 0));
        int **h[9] = {&c->host.slot, &c->host.keff, &c->host.T, &c->host.pending, &c->host.lo_from, &c->host.draft, &c->host.nacc, &c->host.next, &c->host.emit};
        int **d[9] = {&s.io.slot, &s.io.keff, &s.io.T, &s.io.pending, &s.io.lo_from, &s.io.draft, &s.io.nacc, &s.io.next, &s.io.emit};
        size_t at = 0;
        for (int i = 0; i < 9; at += sizes[i], ++i) { *h[i] = c->pin + at; *d[i] = dev + at; }
        c->pin_counts = c->pin + at;
        c->pin_counts_dev = dev + at;
        c->pin_block = c->pin + block_at;
        c->pin_stage = c->pin_block + (c->block_words + 3) / 4 * 4;
    }
    HIP_TRY(c, hipEventCreateWithFlags(&c->cnt_ev[0], hipEventDisableTiming));
    HIP_TRY(c, hipEventCreateWithFlags(&c->cnt_ev[1], hipEventDisableTiming));
    HIP_TRY(c, hipStreamSynchronize(c->st));
    HIP_TRY(c, hipGetLastError());
    return autotune_tilek(c);
}

// ------------------------------------------------------------------------------------------------
// decoding-step GEMM arguments outside a forward (tuning, timing): matrix `which` of layer `layer`
// (0 QKV, 1 O, 2 gate/up, 3 down, 4 LM head) over `rows` rows of whatever the scratch planes hold
// ------------------------------------------------------------------------------------------------
static GemmArgs step_gemm_args(llma_ctx *c, int which, int layer, int rows) {
    const llma_model_cfg &g = c->cfg;
    GemmArgs ga{};
    ga.rows = rows; ga.split = c->opt_split; ga.eps = g.rms_eps; ga.rstd_in = c->rstd;
    ga.ssq_tiles = g.d_model / 16; ga.H = g.n_heads; ga.dh = g.head_dim; ga.max_seq = c->seq_cap; ga.nx_KSp = c->plan_qkv.KSp;
    switch (which) {
        case 0:
            ga.W = c->wqkv[layer]; ga.plan = c->plan_qkv; ga.Xhi = c->xhi; ga.Xlo = c->xlo; ga.epi = EPI_QKV; ga.ssq_in = c->ssq;
            ga.row_pos = c->s.row_pos; ga.row_slot = c->s.row_slot; ga.row_cs = c->s.row_cs; ga.q_hi = c->q; ga.q_lo = c->q_lo;
            ga.k_hi = c->kc[layer]; ga.k_lo = c->kc_lo[layer]; ga.v_hi = c->vc[layer]; ga.v_lo = c->vc_lo[layer];
            break;
        case 1:
            ga.W = c->wo[layer]; ga.plan = c->plan_o; ga.Xhi = c->att_hi; ga.Xlo = c->att_lo; ga.epi = EPI_RESID; ga.out = c->h;
            ga.gain = c->n2[layer]; ga.nx_hi = c->xhi; ga.nx_lo = c->xlo; ga.ssq_out = c->ssq;
            break;
        case 2:
            ga.W = c->wgu[layer]; ga.plan = c->plan_gu; ga.Xhi = c->xhi; ga.Xlo = c->xlo; ga.epi = EPI_SWIGLU; ga.ssq_in = c->ssq;
            ga.act_hi = c->act_hi; ga.act_lo = c->act_lo; ga.act_KSp = c->plan_down.KSp;
            break;
        case 3:
            ga.W = c->wd[layer]; ga.plan = c->plan_down; ga.Xhi = c->act_hi; ga.Xlo = c->act_lo; ga.epi = EPI_RESID; ga.out = c->h;
            ga.gain = c->n1[layer]; ga.nx_hi = c->xhi; ga.nx_lo = c->xlo; ga.ssq_out = c->ssq;
            break;
        default:
            ga.W = c->lm_head; ga.plan = c->plan_lm; ga.Xhi = c->xhi; ga.Xlo = c->xlo; ga.epi = EPI_LMHEAD; ga.ssq_in = c->ssq;
            ga.out = nullptr; ga.pval = c->pval; ga.pidx = c->pidx; ga.n_part = c->n_part;
            break;
    }
    return ga;
}

// How many feature tiles a workgroup of the decoding GEMM takes is pure work division (a tile's sums are
// the same for any value), and which value streams a matrix fastest depends on how its tile count falls
// on the device's compute units (tilek_ft_default's rule) and on how well the device hides the last round.  So it is
// measured: every value that can win, at one row (for steps of up to 4) and at the middle of one, two and three row
// tiles (9, 25, 41 rows), on the context's own matrices and zeroed scratch, a few dozen launches each; a value has
// to beat the default by 5 % to replace it (2 % at one row, where they differ least).
static int autotune_tilek(llma_ctx *c) {
    if (!c->bf16 || getenv("LLMA_NO_AUTOTUNE") != nullptr) return LLMA_OK;
    const llma_model_cfg &g = c->cfg;
    GemmPlan *plans[5] = {&c->plan_qkv, &c->plan_o, &c->plan_gu, &c->plan_down, &c->plan_lm};
    if (const char *forced = getenv("LLMA_TILEK_FT")) {       // tests: this many tiles per workgroup wherever the kernel admits it
        const int ft = atoi(forced);
        for (GemmPlan *p : plans)
            for (int nt = 1; nt <= 3; ++nt)
                if (tilek_ft_valid(*p, nt, ft)) { p->tk_ft[nt - 1] = ft; if (nt == 1) p->tk_ft[3] = ft; }
        return LLMA_OK;
    }
    const int step_rows = g.max_batch * (g.max_k + 1);
    hipEvent_t e0, e1;
    HIP_TRY(c, hipEventCreate(&e0));
    HIP_TRY(c, hipEventCreate(&e1));
    const int reps = g.n_layers < 8 ? 16 : (2 * g.n_layers < 48 ? 2 * g.n_layers : 48);
    for (int which = 0; which < 5; ++which)
        for (int at = 0; at < 4; ++at) {                                  // (index into GemmPlan::tk_ft)
            const int nt = at == 3 ? 1 : at + 1;
            if (16 * (nt - 1) + 1 > step_rows) continue;                  // this context never launches that many row tiles
            int rows = at == 3 ? 1 : 16 * nt - 7;
            rows = rows < step_rows ? rows : step_rows;
            GemmPlan &p = *plans[which];
            if (tilek_bucket(rows) != at) continue;                       // a context of up to 4 rows per step
            const float win = at == 3 ? 0.98f : 0.95f;
            const int dflt = p.tk_ft[at];
            // mean launch time of this matrix at `rows` rows with FT = ft
            auto time_ft = [&](int ft, float *us) -> int {
                p.tk_ft[at] = ft;
                float ms = 0.f;
                for (int pass = 0; pass < 2; ++pass) {                    // pass 0 warms up
                    const int n = pass ? reps : 3;
                    HIP_TRY(c, hipEventRecord(e0, c->st));
                    for (int r = 0; r < n; ++r) {
                        GemmArgs ga = step_gemm_args(c, which, r % g.n_layers, rows);
                        if (!launch_gemm_bf16(ga, c->st)) return fail(c, LLMA_E_INVAL, "autotune: launch refused");
                    }
                    HIP_TRY(c, hipEventRecord(e1, c->st));
                    HIP_TRY(c, hipEventSynchronize(e1));
                    HIP_TRY(c, hipEventElapsedTime(&ms, e0, e1));
                }
                *us = ms * 1e3f / reps;
                return LLMA_OK;
            };
            // values that leave the busiest compute unit a quarter more to stream are not worth a try
            auto worth = [&](int ft) { return tilek_ft_valid(p, nt, ft) && 4 * tilek_cost(p, ft) <= 5 * tilek_cost(p, dflt); };
            int n_worth = 0;
            for (int ft = 1; ft <= 4; ++ft) n_worth += worth(ft);
            if (n_worth < 2) continue;
            float best_us = 0.f, dflt_us = 0.f;
            int best = dflt;
            for (int ft = 1; ft <= 4; ++ft) {
                if (!worth(ft)) continue;
                float us = 0.f;
                if (int rc = time_ft(ft, &us)) return rc;
                if (ft == dflt) dflt_us = us;
                if (best_us == 0.f || us < best_us) { best_us = us; best = ft; }
            }
            // A candidate replaces the default only if it wins by 5 % (one row: 2 %) twice: in the sweep and again
            // head to head (default first, candidate second), so that one disturbed measurement
            // -- clocks still ramping, another process on the card -- cannot pick a slower shape.
            bool adopt = best != dflt && dflt_us > 0.f && best_us < win * dflt_us;
            if (adopt) {
                float d2 = 0.f, b2 = 0.f;
                if (int rc = time_ft(dflt, &d2)) return rc;
                if (int rc = time_ft(best, &b2)) return rc;
                adopt = b2 < win * d2;
            }
            p.tk_ft[at] = adopt ? best : dflt;
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    HIP_TRY(c, hipGetLastError());
    return LLMA_OK;
}

extern "C" int llma_create(const llma_model_cfg *cfg, const llma_weights *w, void *hip_stream, llma_ctx **out) {
    if (!cfg || !w || !out) return fail(nullptr, LLMA_E_INVAL, "llma_create: null argument");
    *out = nullptr;
    int rc = check_cfg(cfg);
    if (rc) return rc;
    if (!w->embed || !w->lm_head || !w->final_norm || !w->wqkv || !w->wo || !w->wgu || !w->wdown || !w->norm1 || !w->norm2)
        return fail(nullptr, LLMA_E_INVAL, "llma_create: null weight pointer");
    llma_ctx *c = new (std::nothrow) llma_ctx();
    if (!c) return fail(nullptr, LLMA_E_NOMEM, "llma_create: host allocation failed");
    c->cfg = *cfg;
    c->st = (hipStream_t)hip_stream;
    c->run_st = c->st;
    c->bf16 = cfg->dtype == LLMA_DTYPE_BF16;
    c->kv_split = c->bf16 && cfg->kv_split != 0;
    rc = create_impl(c, w);
    if (rc) {
        std::string e = c->err;
        llma_destroy(c);
        g_err = e;
        return rc;
    }
    *out = c;
    return LLMA_OK;
}

extern "C" int llma_destroy(llma_ctx *c) {
    if (!c) return LLMA_OK;
    (void)hipStreamSynchronize(c->st);
    for (auto &g : c->graphs) if (g.second.exec) (void)hipGraphExecDestroy(g.second.exec);
    if (c->cap_st) (void)hipStreamDestroy(c->cap_st);
    if (c->pin) (void)hipHostFree(c->pin);
    for (int i = 0; i < 2; ++i) if (c->cnt_ev[i]) (void)hipEventDestroy(c->cnt_ev[i]);
    for (auto &e : c->events) { (void)hipEventDestroy(e.a); (void)hipEventDestroy(e.b); }
    for (void *p : c->allocs) (void)hipFree(p);
    delete c;
    return LLMA_OK;
}

extern "C" const char *llma_last_error(const llma_ctx *c) { return c ? c->err.c_str() : g_err.c_str(); }
extern "C" int64_t llma_device_bytes(const llma_ctx *c) { return c ? c->dev_bytes : 0; }

extern "C" int llma_describe(const llma_ctx *c, char *buf, int32_t cap) {
    if (!c || !buf || cap < 1) return LLMA_E_INVAL;
    if (!c->bf16) { snprintf(buf, (size_t)cap, "fp32 path (plain vector-ALU kernels, nothing tuned)"); return LLMA_OK; }
    const GemmPlan *pl[5] = {&c->plan_qkv, &c->plan_o, &c->plan_gu, &c->plan_down, &c->plan_lm};
    const char *nm[5] = {"qkv", "o", "gate_up", "down", "lm_head"};
    int n = snprintf(buf, (size_t)cap, "decoding GEMM, feature tiles per workgroup at 1/2/3 row tiles, up to 4 rows (K slices):");
    for (int i = 0; i < 5 && n > 0 && n < cap; ++i)
        n += snprintf(buf + n, (size_t)(cap - n), " %s %d/%d/%d, %d (%d)", nm[i], pl[i]->tk_ft[0], pl[i]->tk_ft[1], pl[i]->tk_ft[2], pl[i]->tk_ft[3], pl[i]->tk_waves);
    return LLMA_OK;
}

// ------------------------------------------------------------------------------------------------
// the forward over the rows described by ctx->s.row_* (paper: Eq. 3)
// ------------------------------------------------------------------------------------------------
static int forward_f32(llma_ctx *c, int n_seqs, int m, bool lm_head) {
    const llma_model_cfg &g = c->cfg;
    const int d = g.d_model, F = g.d_ffn, V = g.vocab, H = g.n_heads, dh = g.head_dim, L = g.n_layers;
    const int R = n_seqs * m;
    hipStream_t st = c->run_st;
    GemmArgs ga{};
    ga.rows = R; ga.eps = g.rms_eps; ga.H = H; ga.dh = dh; ga.max_seq = c->seq_cap;
    ga.row_pos = c->s.row_pos; ga.row_slot = c->s.row_slot; ga.row_cs = c->s.row_cs;
    AttnArgs aa{};
    aa.Qhi = c->q; aa.T = c->s.T; aa.batch_slots = c->s.batch_slots; aa.slot_const = -1; aa.n_seqs = n_seqs; aa.m = m; aa.H = H; aa.dh = dh;
    aa.max_seq = c->seq_cap; aa.scale = 1.0f / sqrtf((float)dh); aa.out_hi = c->att_hi;
    for (int l = 0; l < L; ++l) {                          // (RMSNorm, RoPE and the cache append run inside the GEMMs)
        ga.W = c->wqkv[l]; ga.Xhi = c->h; ga.N = 3 * d; ga.K = d; ga.epi = EPI_QKV; ga.gain = c->n1[l];
        ga.q_hi = c->q; ga.k_hi = c->kc[l]; ga.v_hi = c->vc[l];
        launch_gemm_f32(ga, st);
        aa.Khi = c->kc[l]; aa.Vhi = c->vc[l];
        launch_attn_f32(aa, st);
        ga.W = c->wo[l]; ga.Xhi = c->att_hi; ga.N = d; ga.K = d; ga.epi = EPI_RESID; ga.out = c->h;
        launch_gemm_f32(ga, st);
        ga.W = c->wgu[l]; ga.Xhi = c->h; ga.N = F; ga.K = d; ga.epi = EPI_SWIGLU; ga.gain = c->n2[l]; ga.act_hi = c->act_hi;
        launch_gemm_f32(ga, st);
        ga.W = c->wd[l]; ga.Xhi = c->act_hi; ga.N = d; ga.K = F; ga.epi = EPI_RESID; ga.out = c->h;
        launch_gemm_f32(ga, st);
    }
    if (lm_head) {
        ga.W = c->lm_head; ga.Xhi = c->h; ga.N = V; ga.K = d; ga.epi = EPI_LMHEAD; ga.gain = c->final_norm;
        ga.out = c->logits_dump; ga.pval = c->pval; ga.pidx = c->pidx; ga.n_part = c->n_part;
        launch_gemm_f32(ga, st);
    }
    HIP_TRY(c, hipGetLastError());
    return LLMA_OK;
}

// bf16: per layer  QKV GEMM (+RMSNorm scale, RoPE, KV append) -> attention -> O GEMM (+residual,
// next-norm input) -> gate/up GEMM (+RMSNorm scale, SwiGLU) -> down GEMM (+residual, next-norm input)
static int forward_bf16(llma_ctx *c, int n_seqs, int m, int n_chunks, bool lm_head, int slot) {
    const llma_model_cfg &g = c->cfg;
    const int d = g.d_model, H = g.n_heads, dh = g.head_dim, L = g.n_layers;
    const int R = n_seqs * m;
    hipStream_t st = c->run_st;
    const int ksp_d = c->plan_qkv.KSp;          // k-steps per row tile of every activation plane that feeds a K = d GEMM
    GemmArgs base{};
    base.rows = R; base.eps = g.rms_eps;
    base.split = c->opt_split || !lm_head;                 // (the option is about steps; the panel GEMM always feeds both planes)
    base.rows_live = c->rows_live;                         // llma_generate, one sequence: the trigger's draft count (device)
    // Steps and prompt passes of up to 48 rows use the tile-K GEMM, longer ones the panel GEMM (weights streamed once
    // for all rows): the steps in its split-K form, because a few hundred rows alone make too few workgroups to
    // fill the chip, and so do prompt passes as far as that pays for the partial sums (7B, 189 rows: 2.01 -> 1.01 ms for
    // four layers; 15 rows: 1.83 -> 0.44 ms through the tile-K GEMM).
    const bool panel = R > 48;
    bool refused = false;
    auto tilek_gemm = [&](GemmArgs &ga) { refused = !launch_gemm_bf16(ga, st) || refused; };
    auto split_of = [&](const GemmArgs &ga) { return lm_head ? ga.plan.n_split : panel_prompt_split(ga.plan, R); };
    auto panel_gemm = [&](GemmArgs &ga) {
        if (split_of(ga) > 1) { ga.ksplit = split_of(ga); ga.part = c->part; }
        launch_gemm_panel_bf16(ga, st);
    };
    // panel GEMM whose epilogue scales by the rows' rstd: in the split-K form the waves of its first kernel
    // compute it (its finishing kernel is the reader), otherwise a launch of its own
    auto panel_norm_gemm = [&](GemmArgs &ga) {
        if (split_of(ga) > 1) ga.rstd_out = c->rstd;
        else launch_rstd_rows(c->ssq, d / 16, g.rms_eps, c->rstd, R, st);
        panel_gemm(ga);
    };
    base.rstd_in = c->rstd;
    base.part = c->part;
    base.ssq_tiles = d / 16; base.H = H; base.dh = dh; base.max_seq = c->seq_cap; base.nx_KSp = ksp_d;
    AttnArgs aa{};
    aa.Qhi = c->q; aa.Qlo = c->q_lo; aa.T = c->s.T; aa.batch_slots = c->s.batch_slots; aa.slot_const = n_seqs == 1 ? slot : -1; aa.n_seqs = n_seqs; aa.m = m; aa.H = H; aa.dh = dh;
    aa.rows_live = c->rows_live;
    if (c->n_segs) { aa.segs = (const PromptSeg *)c->gen_segs; aa.n_segs = c->n_segs; }
    aa.lo_from = c->kv_split ? c->lo_from : nullptr;
    aa.max_seq = c->seq_cap; aa.n_chunks = n_chunks; aa.scale = 1.0f / sqrtf((float)dh);
    aa.po = c->po; aa.pm = c->pm; aa.pl = c->pl; aa.out_hi = c->att_hi; aa.out_lo = c->att_lo; aa.out_KSp = ksp_d; aa.quads = R > XTILE_ROWWISE;
    for (int l = 0; l < L; ++l) {
        GemmArgs ga = base;
        ga.W = c->wqkv[l]; ga.plan = c->plan_qkv; ga.Xhi = c->xhi; ga.Xlo = c->xlo; ga.epi = EPI_QKV; ga.ssq_in = c->ssq;
        ga.row_pos = c->s.row_pos; ga.row_slot = c->s.row_slot; ga.row_cs = c->s.row_cs; ga.q_hi = c->q; ga.q_lo = c->q_lo;
        ga.k_hi = c->kc[l]; ga.k_lo = c->kc_lo[l]; ga.v_hi = c->vc[l]; ga.v_lo = c->vc_lo[l];
        if (panel) { panel_norm_gemm(ga); }
        else { ga.rstd_out = c->rstd; tilek_gemm(ga); }
        aa.Khi = c->kc[l]; aa.Klo = c->kc_lo[l]; aa.Vhi = c->vc[l]; aa.Vlo = c->vc_lo[l];
        launch_attn_bf16(aa, st);
        ga = base;
        ga.W = c->wo[l]; ga.plan = c->plan_o; ga.Xhi = c->att_hi; ga.Xlo = c->att_lo; ga.epi = EPI_RESID; ga.out = c->h;
        ga.gain = c->n2[l]; ga.nx_hi = c->xhi; ga.nx_lo = c->xlo; ga.ssq_out = c->ssq;
        if (panel) panel_gemm(ga); else tilek_gemm(ga);
        ga = base;
        ga.W = c->wgu[l]; ga.plan = c->plan_gu; ga.Xhi = c->xhi; ga.Xlo = c->xlo; ga.epi = EPI_SWIGLU; ga.ssq_in = c->ssq;
        ga.act_hi = c->act_hi; ga.act_lo = c->act_lo; ga.act_KSp = c->plan_down.KSp;
        if (panel) {
            panel_norm_gemm(ga);
        } else if (c->opt_timing && lm_head) {                 // (decoding steps only)
            EventPair ep;
            HIP_TRY(c, hipEventCreate(&ep.a));
            HIP_TRY(c, hipEventCreate(&ep.b));
            HIP_TRY(c, hipEventRecord(ep.a, st));
            tilek_gemm(ga);
            HIP_TRY(c, hipEventRecord(ep.b, st));
            c->events.push_back(ep);
        } else {
            tilek_gemm(ga);
        }
        ga = base;
        ga.W = c->wd[l]; ga.plan = c->plan_down; ga.Xhi = c->act_hi; ga.Xlo = c->act_lo; ga.epi = EPI_RESID; ga.out = c->h;
        ga.gain = (l + 1 < L) ? c->n1[l + 1] : c->final_norm; ga.nx_hi = c->xhi; ga.nx_lo = c->xlo; ga.ssq_out = c->ssq;
        if (panel) panel_gemm(ga); else tilek_gemm(ga);
    }
    if (lm_head) {
        GemmArgs ga = base;
        ga.W = c->lm_head; ga.plan = c->plan_lm; ga.Xhi = c->xhi; ga.Xlo = c->xlo; ga.epi = EPI_LMHEAD; ga.ssq_in = c->ssq;
        ga.out = c->logits_dump; ga.pval = c->pval; ga.pidx = c->pidx; ga.n_part = c->n_part;
        if (panel) { panel_norm_gemm(ga); }
        else { ga.rstd_out = c->rstd; tilek_gemm(ga); }
    }
    if (refused) return fail(c, LLMA_E_INVAL, "forward: a step of %d rows reached the decoding-step GEMM (1..48 rows)", R);
    HIP_TRY(c, hipGetLastError());
    return LLMA_OK;
}

static int forward(llma_ctx *c, int n_seqs, int m, int n_chunks, bool lm_head, int slot) {
    return c->bf16 ? forward_bf16(c, n_seqs, m, n_chunks, lm_head, slot) : forward_f32(c, n_seqs, m, lm_head);
}

// One step = row set-up + forward + bookkeeping, always the same launches for a given
// (kind, rows, attention chunk count, slot): the second time a shape is seen its launches are
// captured into a HIP graph and from then on replayed.  All per-step data (tokens, positions,
// cache lengths, drafts) lives in device memory, so a replay needs no new arguments.
static int step_body(llma_ctx *c, int kind, int n_seqs, int m, int n_chunks, int slot) {
    hipStream_t st = c->run_st;
    const int mk = c->cfg.max_k;
    EmbedArgs e{};
    e.embed = c->embed; e.h = c->h; e.d = c->cfg.d_model;
    if (c->bf16) { e.gain = c->n1[0]; e.nx_hi = c->xhi; e.nx_lo = c->xlo; e.ssq_out = c->ssq; e.KSp = c->plan_qkv.KSp; e.quads = n_seqs * m > XTILE_ROWWISE; }
    c->rows_live = nullptr;
    if (kind == STEP_PREFILL || kind == STEP_PROMPTS) {
        if (kind == STEP_PROMPTS) { c->n_segs = e.n_segs = n_seqs; e.segs = (const PromptSeg *)c->gen_segs; }
        launch_setup_prefill_rows(c->s, c->gen_prompt, c->gen_counters + 4 * c->cfg.max_batch, m, slot, c->cs_table, c->cfg.head_dim / 2, e, st);
        int rc = forward(c, 1, m, n_chunks, false, slot);
        c->n_segs = 0;
        if (rc || kind == STEP_PROMPTS) return rc;              // (whose lengths differ from pass to pass of the same shape)
        launch_advance_T(c->s, slot, m, st);
        return LLMA_OK;
    }
    c->rows_live = (kind == STEP_GEN && n_seqs == 1) ? c->s.keff : nullptr;
    const GenState *gen = kind == STEP_GEN ? c->gen_dev : nullptr;
    unsigned long long *part = (unsigned long long *)c->gen_part;
    if (!gen) launch_take_step(c->s, n_seqs, mk, st);
    else if (c->gen_spans > 1) launch_trigger_scan(gen, n_seqs, c->gen_spans, part, st);
    launch_setup_step_rows(c->s, n_seqs, m, mk, c->cs_table, c->cfg.head_dim / 2, e, gen, part, c->gen_spans, st);
    int rc = forward(c, n_seqs, m, n_chunks, true, slot);
    if (rc) return rc;
    launch_argmax_accept(c->pval, c->pidx, c->n_part, c->s, n_seqs, m, mk, c->cfg.vocab, gen, st);
    return LLMA_OK;
}

static void drop_graphs(llma_ctx *c) {
    (void)hipStreamSynchronize(c->st);
    for (auto &g : c->graphs) if (g.second.exec) (void)hipGraphExecDestroy(g.second.exec);
    c->graphs.clear();
}

// The slot of a shape.  Prompt passes have a new shape nearly every time (several sequences' above all), so a full map gives up the
// shape not used for longest: the decoding steps' stay.  (When a full map took no more and ended every replay, the steps of
// a context that had seen 257 shapes ran eagerly from then on.)
static GraphSlot &graph_slot(llma_ctx *c, const GraphKey &key) {
    auto it = c->graphs.find(key);
    if (it == c->graphs.end()) {
        if (c->graphs.size() >= GRAPH_SLOTS_MAX) {
            auto oldest = c->graphs.begin();
            for (auto g = c->graphs.begin(); g != c->graphs.end(); ++g)
                if (g->second.used < oldest->second.used) oldest = g;
            if (oldest->second.exec) {
                (void)hipStreamSynchronize(c->st);          // (its last launch may be on its way)
                (void)hipGraphExecDestroy(oldest->second.exec);
            }
            c->graphs.erase(oldest);
        }
        it = c->graphs.emplace(key, GraphSlot{}).first;
    }
    it->second.used = ++c->graph_clock;
    return it->second;
}

static int run_step(llma_ctx *c, int kind, int n_seqs, int m, int t_max, int slot) {
    // attention chunks launched: enough for the longest sequence.  A launched chunk streams its K/V
    // blocks before it knows whether it lies past the sequence's end, so the count is rounded up
    // (fewer distinct launch shapes, i.e. graphs) only by a few percent: to whole buckets of 1, 4 or
    // 16 chunks for up to 32, 128 or more chunks
    int n_chunks = (t_max + m + ATTN_CHUNK - 1) / ATTN_CHUNK;
    const int bucket = n_chunks <= 32 ? 1 : (n_chunks <= 128 ? 4 : 16);
    n_chunks = (n_chunks + bucket - 1) / bucket * bucket;
    if (c->bf16 && n_chunks > c->nc_max) n_chunks = c->nc_max;
    if (kind == STEP_PROMPTS) n_chunks = t_max;                 // row blocks of the attention
    c->run_st = c->st;
    if (!c->opt_graph || c->opt_timing) return step_body(c, kind, n_seqs, m, n_chunks, slot);
    const GraphKey key = {kind, n_seqs, m, n_chunks, slot, kind == STEP_GEN ? c->gen_spans : 0};     // every field that shapes a launch or is baked into one
    GraphSlot &gs = graph_slot(c, key);
    if (gs.exec == nullptr) {
        if (gs.seen++ == 0) return step_body(c, kind, n_seqs, m, n_chunks, slot);   // first time eagerly
        hipGraph_t graph = nullptr;
        if (hipStreamBeginCapture(c->cap_st, hipStreamCaptureModeRelaxed) != hipSuccess) { c->opt_graph = 0; return step_body(c, kind, n_seqs, m, n_chunks, slot); }
        c->run_st = c->cap_st;
        int rc = step_body(c, kind, n_seqs, m, n_chunks, slot);
        c->run_st = c->st;
        hipError_t e = hipStreamEndCapture(c->cap_st, &graph);
        if (rc) { if (graph) (void)hipGraphDestroy(graph); return rc; }
        if (e != hipSuccess || graph == nullptr) return fail(c, LLMA_E_HIP, "graph capture failed: %s", hipGetErrorString(e));
        e = hipGraphInstantiate(&gs.exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) { gs.exec = nullptr; return fail(c, LLMA_E_HIP, "hipGraphInstantiate: %s", hipGetErrorString(e)); }
    }
    HIP_TRY(c, hipGraphLaunch(gs.exec, c->st));
    return LLMA_OK;
}

// ------------------------------------------------------------------------------------------------
// sequence state
// ------------------------------------------------------------------------------------------------
static int check_slot(llma_ctx *c, int seq, const char *who) {
    if (!c) return fail(nullptr, LLMA_E_INVAL, "%s: null context", who);
    if (seq < 0 || seq >= c->cfg.max_batch) return fail(c, LLMA_E_RANGE, "%s: slot %d outside [0,%d)", who, seq, c->cfg.max_batch);
    return LLMA_OK;
}
static int push_state(llma_ctx *c, int seq) {       // host mirror -> device
    HIP_TRY(c, hipMemcpyAsync(c->s.T + seq, &c->T_host[seq], 4, hipMemcpyHostToDevice, c->st));
    HIP_TRY(c, hipMemcpyAsync(c->s.pending + seq, &c->pending_host[seq], 4, hipMemcpyHostToDevice, c->st));
    HIP_TRY(c, hipMemcpyAsync(c->lo_from + seq, &c->lo_from_host[seq], 4, hipMemcpyHostToDevice, c->st));
    HIP_TRY(c, hipStreamSynchronize(c->st));
    c->stale[seq] = 0;
    return LLMA_OK;
}
static int sync_state(llma_ctx *c, int seq) { return c->stale[seq] ? push_state(c, seq) : LLMA_OK; }
// something is about to be computed on the slot: the record of imported lengths no longer describes a pure import
static void forget_imports(llma_ctx *c, int seq) {
    for (int l = 0; l < c->cfg.n_layers; ++l) c->imp_len[(size_t)seq * c->cfg.n_layers + l] = -1;
}

extern "C" int llma_reset(llma_ctx *c, int32_t seq) {
    int rc = check_slot(c, seq, "llma_reset");
    if (rc) return rc;
    c->T_host[seq] = 0;
    c->pending_host[seq] = -1;
    c->lo_from_host[seq] = 0;
    forget_imports(c, seq);
    c->stale[seq] = 1;
    return LLMA_OK;
}

extern "C" int llma_get_state(llma_ctx *c, int32_t seq, int32_t *T, int32_t *pending) {
    int rc = check_slot(c, seq, "llma_get_state");
    if (rc) return rc;
    if ((rc = sync_state(c, seq))) return rc;
    int t = 0, p = -1;
    HIP_TRY(c, hipMemcpyAsync(&t, c->s.T + seq, 4, hipMemcpyDeviceToHost, c->st));
    HIP_TRY(c, hipMemcpyAsync(&p, c->s.pending + seq, 4, hipMemcpyDeviceToHost, c->st));
    HIP_TRY(c, hipStreamSynchronize(c->st));
    if (T) *T = t;
    if (pending) *pending = p;
    return LLMA_OK;
}

extern "C" int llma_truncate(llma_ctx *c, int32_t seq, int32_t new_len) {
    int rc = check_slot(c, seq, "llma_truncate");
    if (rc) return rc;
    if (new_len < 0 || new_len > c->T_host[seq])
        return fail(c, LLMA_E_RANGE, "llma_truncate: new length %d outside [0, T = %d]", new_len, c->T_host[seq]);
    c->T_host[seq] = new_len;
    if (c->lo_from_host[seq] > new_len) c->lo_from_host[seq] = new_len;    // rows written from here on have lo planes
    c->stale[seq] = 1;
    return LLMA_OK;
}

extern "C" int llma_set_pending(llma_ctx *c, int32_t seq, int32_t token) {
    int rc = check_slot(c, seq, "llma_set_pending");
    if (rc) return rc;
    if (token < 0 || token >= c->cfg.vocab) return fail(c, LLMA_E_RANGE, "llma_set_pending: token %d outside [0,%d)", token, c->cfg.vocab);
    c->pending_host[seq] = token;
    c->stale[seq] = 1;
    return LLMA_OK;
}

extern "C" int llma_kv_import(llma_ctx *c, int32_t seq, int32_t layer, const void *k, const void *v, int32_t len) {
    int rc = check_slot(c, seq, "llma_kv_import");
    if (rc) return rc;
    if (!k || !v) return fail(c, LLMA_E_INVAL, "llma_kv_import: null pointer");
    if (layer < 0 || layer >= c->cfg.n_layers) return fail(c, LLMA_E_RANGE, "llma_kv_import: layer %d", layer);
    if (len < 0 || len > c->cfg.max_seq) return fail(c, LLMA_E_RANGE, "llma_kv_import: len %d > max_seq %d", len, c->cfg.max_seq);
    const llma_model_cfg &g = c->cfg;
    const size_t es = c->bf16 ? 2 : 4;
    const size_t slot_off = (size_t)seq * g.n_heads * c->seq_cap * g.head_dim * es;
    void *kc = (char *)c->kc[layer] + slot_off, *vc = (char *)c->vc[layer] + slot_off;
    void *kl = c->kv_split ? (char *)c->kc_lo[layer] + slot_off / 2 : nullptr, *vl = c->kv_split ? (char *)c->vc_lo[layer] + slot_off / 2 : nullptr;
    if (len > 0) {
        if (c->bf16) launch_kv_import_bf16(k, v, kc, kl, vc, vl, g.n_heads, len, g.head_dim, c->seq_cap, c->st);
        else launch_kv_import_f32(k, v, kc, vc, g.n_heads, len, g.head_dim, c->seq_cap, c->st);
    }
    HIP_TRY(c, hipGetLastError());
    c->imp_len[(size_t)seq * g.n_layers + layer] = len;
    if (layer == g.n_layers - 1) {
        c->T_host[seq] = len;
        bool all = c->kv_split != 0;
        for (int l = 0; l < g.n_layers; ++l) all = all && c->imp_len[(size_t)seq * g.n_layers + l] == len;
        c->lo_from_host[seq] = all ? len : 0;
        return push_state(c, seq);
    }
    return LLMA_OK;
}

static int check_tokens(llma_ctx *c, const int32_t *t, int n, const char *who) {
    for (int i = 0; i < n; ++i)
        if (t[i] < 0 || t[i] >= c->cfg.vocab) return fail(c, LLMA_E_RANGE, "%s: token[%d] = %d outside [0,%d)", who, i, t[i], c->cfg.vocab);
    return LLMA_OK;
}

// feeds gen_prompt[T - base .. ) in chunks on top of the slot's cache, n_feed rows in all (the device knows T and base); rows only write KV, no LM head
static int prefill_passes(llma_ctx *c, int seq, int n_feed) {
    for (int off = 0; off < n_feed; off += c->Pmax) {
        const int m = n_feed - off < c->Pmax ? n_feed - off : c->Pmax;
        int rc = run_step(c, STEP_PREFILL, 1, m, c->T_host[seq], seq);
        if (rc) return rc;
        c->T_host[seq] += m;
    }
    return LLMA_OK;
}
// the same with the prompt's first token at gen_prompt[tok0]
static int prefill_rows(llma_ctx *c, int seq, int n_feed, int tok0 = 0) {
    int rc = sync_state(c, seq);
    if (rc) return rc;
    const int base = c->T_host[seq] - tok0;
    HIP_TRY(c, hipMemcpyAsync(c->gen_counters + 4 * c->cfg.max_batch, &base, 4, hipMemcpyHostToDevice, c->st));
    HIP_TRY(c, hipStreamSynchronize(c->st));
    return prefill_passes(c, seq, n_feed);
}

static int ensure_cap(llma_ctx *c, int **buf, size_t *cap, size_t need);
// The prompts of several sequences (reset slots; gen_prompt holds all of them, sequence b's from offsets[b] on) in passes of up to
// Pmax rows, sequence after sequence: the weights go through the chip once per pass instead of once per sequence, and a
// pass fills it.  Six prompts of 166..230 tokens and the first step's
// tokens, 7B, four layers: 8.1 -> 5.5 ms, of which two steps take 1.4.
// The K ranges are those of the pass's rows, so a sequence's K / V depend on the other prompts' lengths at rounding level.  Shared
// passes that keep every sequence's own ranges (sequences of the same ranges together, short ones alone) give the bits of
// llma_prefill and were measured: the six-sequence generation of 40 tokens 24.0 -> 25.5 ms.
static int prefill_together(llma_ctx *c, int n_seqs, const int32_t *seqs, const int32_t *offsets) {
    int b = 0, done = 0;                                        // next row: token `done` of sequence b
    std::vector<PromptSeg> segs;
    while (b < n_seqs) {
        segs.clear();
        int rows = 0, blocks = 0;
        while (b < n_seqs && rows < c->Pmax) {
            const int left = offsets[b + 1] - offsets[b] - 1 - done, take = left < c->Pmax - rows ? left : c->Pmax - rows;
            if (take > 0) {
                segs.push_back(PromptSeg{rows, take, seqs[b], offsets[b] + done, blocks});
                rows += take;
                blocks += (take + PROMPT_BLOCK - 1) / PROMPT_BLOCK;
                done += take;
            }
            if (take == left) { ++b; done = 0; }
        }
        if (rows == 0) break;
        if (rows <= 48) {                                       // (a short remainder: the form of short passes, one sequence at a time)
            for (const PromptSeg &s : segs) {
                const int base = c->T_host[s.slot] - s.tok0;    // (a pass reads token T - base of gen_prompt)
                HIP_TRY(c, hipMemcpyAsync(c->gen_counters + 4 * c->cfg.max_batch, &base, 4, hipMemcpyHostToDevice, c->st));
                HIP_TRY(c, hipStreamSynchronize(c->st));
                int rc = run_step(c, STEP_PREFILL, 1, s.rows, c->T_host[s.slot], s.slot);
                if (rc) return rc;
                c->T_host[s.slot] += s.rows;
            }
            continue;
        }
        int rc = ensure_cap(c, &c->gen_segs, &c->cap_segs, segs.size() * sizeof(PromptSeg) / sizeof(int));
        if (rc) return rc;
        HIP_TRY(c, hipMemcpyAsync(c->gen_segs, segs.data(), segs.size() * sizeof(PromptSeg), hipMemcpyHostToDevice, c->st));
        HIP_TRY(c, hipStreamSynchronize(c->st));                // (the list is written anew for the next pass)
        if ((rc = run_step(c, STEP_PROMPTS, (int)segs.size(), rows, blocks, segs[0].slot))) return rc;
        for (const PromptSeg &s : segs) {
            launch_advance_T(c->s, s.slot, s.rows, c->st);
            c->T_host[s.slot] += s.rows;
        }
        HIP_TRY(c, hipGetLastError());
    }
    HIP_TRY(c, hipStreamSynchronize(c->st));
    return LLMA_OK;
}

static int ensure_cap(llma_ctx *c, int **buf, size_t *cap, size_t need) {
    if (need <= *cap) return LLMA_OK;
    drop_graphs(c);                                   // captured launches hold the old pointer
    if (*buf) { dev_free_one(c, *buf); *buf = nullptr; *cap = 0; }
    const size_t ncap = need + need / 2 + 64;
    ALLOC(c, *buf, ncap * 4);
    *cap = ncap;
    return LLMA_OK;
}

extern "C" int llma_prefill(llma_ctx *c, int32_t seq, const int32_t *prompt, int32_t len) {
    int rc = check_slot(c, seq, "llma_prefill");
    if (rc) return rc;
    if (!prompt || len < 1) return fail(c, LLMA_E_INVAL, "llma_prefill: need a prompt of at least one token");
    if (c->T_host[seq] + len > c->cfg.max_seq)
        return fail(c, LLMA_E_RANGE, "llma_prefill: T %d + len %d > max_seq %d", c->T_host[seq], len, c->cfg.max_seq);
    if ((rc = check_tokens(c, prompt, len, "llma_prefill"))) return rc;
    if ((rc = ensure_cap(c, &c->gen_prompt, &c->cap_prompt, len))) return rc;
    HIP_TRY(c, hipMemcpyAsync(c->gen_prompt, prompt, (size_t)len * 4, hipMemcpyHostToDevice, c->st));
    forget_imports(c, seq);
    if ((rc = sync_state(c, seq))) return rc;
    if ((rc = prefill_rows(c, seq, len - 1))) return rc;
    c->pending_host[seq] = prompt[len - 1];
    HIP_TRY(c, hipMemcpyAsync(c->s.pending + seq, &c->pending_host[seq], 4, hipMemcpyHostToDevice, c->st));
    HIP_TRY(c, hipStreamSynchronize(c->st));
    return LLMA_OK;
}

// ------------------------------------------------------------------------------------------------
// verify step
// ------------------------------------------------------------------------------------------------
// Error return of a call that has enqueued part of a step: the step's kernels read and write pinned host memory, which the
// next call rewrites at once, so none of them may still be on its way.
static int drained(llma_ctx *c, int rc) {
    (void)hipStreamSynchronize(c->st);
    return rc;
}

extern "C" int llma_verify_step_batch(llma_ctx *c, int32_t n_seqs, const int32_t *seqs, const int32_t *drafts, int32_t k,
                                      int32_t *n_accepted, int32_t *next_token, int32_t *emitted) {
    if (!c) return fail(nullptr, LLMA_E_INVAL, "llma_verify_step: null context");
    const llma_model_cfg &g = c->cfg;
    if (!seqs || n_seqs < 1 || n_seqs > g.max_batch) return fail(c, LLMA_E_INVAL, "llma_verify_step: bad slot list");
    if (k < 0 || k > g.max_k) return fail(c, LLMA_E_RANGE, "llma_verify_step: k %d outside [0, max_k %d]", k, g.max_k);
    if (k > 0 && !drafts) return fail(c, LLMA_E_INVAL, "llma_verify_step: null drafts with k > 0");
    int t_max = 0;
    for (int b = 0; b < n_seqs; ++b) {
        int rc = check_slot(c, seqs[b], "llma_verify_step");
        if (rc) return rc;
        for (int b2 = 0; b2 < b; ++b2)
            if (seqs[b2] == seqs[b]) return fail(c, LLMA_E_INVAL, "llma_verify_step: slot %d listed twice", seqs[b]);
        if (c->pending_host[seqs[b]] < 0) return fail(c, LLMA_E_STATE, "llma_verify_step: slot %d has no pending token", seqs[b]);
        if (c->T_host[seqs[b]] + k + 1 > g.max_seq)
            return fail(c, LLMA_E_RANGE, "llma_verify_step: T %d + k + 1 > max_seq %d", c->T_host[seqs[b]], g.max_seq);
        if (c->T_host[seqs[b]] > t_max) t_max = c->T_host[seqs[b]];
    }
    if (k > 0) {
        int rc = check_tokens(c, drafts, n_seqs * k, "llma_verify_step(draft)");
        if (rc) return rc;
    }
    if (c->logits_dump && n_seqs * (k + 1) > c->dump_rows)
        return fail(c, LLMA_E_RANGE, "llma_verify_step: logits dump holds %d rows, step has %d", c->dump_rows, n_seqs * (k + 1));
    const int m = k + 1, mk = g.max_k;
    const HostIo &io = c->host;                // (nothing on the device reads or writes it now: every step is waited for, failed ones too)
    for (int b = 0; b < n_seqs; ++b) {
        io.slot[b] = seqs[b];
        io.keff[b] = k;
        io.T[b] = c->T_host[seqs[b]];
        io.pending[b] = c->pending_host[seqs[b]];
        io.lo_from[b] = c->lo_from_host[seqs[b]];
        for (int j = 0; j < k; ++j) io.draft[(size_t)b * mk + j] = drafts[(size_t)b * k + j];
        io.nacc[b] = -1;                       // (checked below)
    }
    for (int b = 0; b < n_seqs; ++b) forget_imports(c, seqs[b]);
    int rc = run_step(c, STEP_VERIFY, n_seqs, m, t_max, n_seqs == 1 ? seqs[0] : 0);
    if (rc) return drained(c, rc);
    HIP_TRY(c, hipStreamSynchronize(c->st));
    HIP_TRY(c, hipGetLastError());
    const int *const nacc = io.nacc, *const nxt = io.next, *const em = io.emit;
    for (int b = 0; b < n_seqs; ++b) c->stale[seqs[b]] = 0;
    for (int b = 0; b < n_seqs; ++b) {
        bool ok = nacc[b] >= 0 && nacc[b] <= k && nxt[b] >= 0 && nxt[b] < g.vocab;
        for (int j = 0; ok && j <= nacc[b]; ++j) ok = em[(size_t)b * (mk + 1) + j] >= 0 && em[(size_t)b * (mk + 1) + j] < g.vocab;
        if (!ok) return fail(c, LLMA_E_HIP, "llma_verify_step: device returned accepted count %d / token %d outside their ranges for slot %d", nacc[b], nxt[b], seqs[b]);
    }
    for (int b = 0; b < n_seqs; ++b) {
        c->T_host[seqs[b]] += nacc[b] + 1;
        c->pending_host[seqs[b]] = nxt[b];
        if (n_accepted) n_accepted[b] = nacc[b];
        if (next_token) next_token[b] = nxt[b];
        if (emitted)
            for (int j = 0; j <= nacc[b]; ++j) emitted[(size_t)b * (k + 1) + j] = em[(size_t)b * (mk + 1) + j];
    }
    return LLMA_OK;
}

extern "C" int llma_verify_step(llma_ctx *c, int32_t seq, const int32_t *draft, int32_t k, int32_t *n_accepted,
                                int32_t *next_token, int32_t *emitted) {
    return llma_verify_step_batch(c, 1, &seq, draft, k, n_accepted, next_token, emitted);
}

// ------------------------------------------------------------------------------------------------
// llma_generate (paper: Algorithm 1)
// ------------------------------------------------------------------------------------------------
extern "C" int llma_generate_batch(llma_ctx *c, int32_t n_seqs, const int32_t *seqs, const int32_t *prompts,
                                   const int32_t *prompt_offsets, const int32_t *refs, const int32_t *doc_offsets,
                                   const int32_t *n_docs, int32_t n, int32_t k, int32_t max_new, int32_t *out_tokens,
                                   int32_t *n_out, llma_step_rec *trace, int32_t *n_steps) {
    if (!c) return fail(nullptr, LLMA_E_INVAL, "llma_generate: null context");
    const llma_model_cfg &g = c->cfg;
    if (!seqs || n_seqs < 1 || n_seqs > g.max_batch) return fail(c, LLMA_E_INVAL, "llma_generate: bad slot list (1..max_batch %d slots)", g.max_batch);
    if (!prompts || !prompt_offsets || !out_tokens || !n_out || max_new < 1) return fail(c, LLMA_E_INVAL, "llma_generate: null / empty argument");
    if (n < 1) return fail(c, LLMA_E_INVAL, "llma_generate: n must be >= 1");
    if (k < 0 || k > g.max_k) return fail(c, LLMA_E_RANGE, "llma_generate: k %d outside [0, max_k %d]", k, g.max_k);
    if (prompt_offsets[0] != 0) return fail(c, LLMA_E_INVAL, "llma_generate: prompt_offsets[0] != 0");
    int rc;
    // per sequence: where its reference tokens and its document list start in the concatenated inputs
    std::vector<int> ref_start(n_seqs + 1, 0), docs_start(n_seqs + 1, 0);
    for (int b = 0; b < n_seqs; ++b) {
        if ((rc = check_slot(c, seqs[b], "llma_generate"))) return rc;
        for (int b2 = 0; b2 < b; ++b2)
            if (seqs[b2] == seqs[b]) return fail(c, LLMA_E_INVAL, "llma_generate: slot %d listed twice", seqs[b]);
        const int plen = prompt_offsets[b + 1] - prompt_offsets[b];
        if (plen < 1) return fail(c, LLMA_E_INVAL, "llma_generate: sequence %d has an empty prompt", b);
        if ((long)plen + max_new + k > g.max_seq)
            return fail(c, LLMA_E_RANGE, "llma_generate: prompt %d + max_new %d + k %d > max_seq %d", plen, max_new, k, g.max_seq);
        const int nd = n_docs ? n_docs[b] : 0;
        if (nd < 0 || (nd > 0 && !doc_offsets)) return fail(c, LLMA_E_INVAL, "llma_generate: bad documents");
        int rlen = 0;
        if (nd > 0) {
            const int32_t *dof = doc_offsets + docs_start[b];
            if (dof[0] != 0) return fail(c, LLMA_E_INVAL, "llma_generate: doc_offsets[0] != 0");
            for (int j = 0; j < nd; ++j)
                if (dof[j + 1] < dof[j]) return fail(c, LLMA_E_INVAL, "llma_generate: doc_offsets decrease at %d", j);
            rlen = dof[nd];
            if (rlen > 0 && !refs) return fail(c, LLMA_E_INVAL, "llma_generate: null reference");
        }
        ref_start[b + 1] = ref_start[b] + rlen;
        docs_start[b + 1] = docs_start[b] + (doc_offsets ? nd + 1 : 0);
    }
    const int total_prompt = prompt_offsets[n_seqs], total_ref = ref_start[n_seqs];
    if ((rc = check_tokens(c, prompts, total_prompt, "llma_generate(prompt)"))) return rc;
    if (total_ref && (rc = check_tokens(c, refs, total_ref, "llma_generate(ref)"))) return rc;
    if (c->logits_dump && n_seqs * (k + 1) > c->dump_rows) return fail(c, LLMA_E_RANGE, "llma_generate: logits dump too small");

    hipStream_t st = c->st;
    const int ystride = max_new + 64;                       // per-sequence output / trace rows on the device
    const bool together = c->bf16 && n_seqs > 1 && n_seqs * (k + 1) > 48;      // (the prompts, see below)
    // device document lists: every sequence gets one (a sequence without reference: the single entry 0)
    std::vector<int> dof_host, dof_at(n_seqs);
    for (int b = 0; b < n_seqs; ++b) {
        const int nd = n_docs ? n_docs[b] : 0;
        dof_at[b] = (int)dof_host.size();
        if (nd > 0) dof_host.insert(dof_host.end(), doc_offsets + docs_start[b], doc_offsets + docs_start[b] + nd + 1);
        else dof_host.push_back(0);
    }
    // [prompts | references | document lists] on the device
    const size_t ref_at = ((size_t)total_prompt + 3) / 4 * 4, docs_at = ref_at + ((size_t)total_ref + 3) / 4 * 4, in_words = docs_at + dof_host.size();
    if ((rc = ensure_cap(c, &c->gen_prompt, &c->cap_prompt, in_words))) return rc;
    // spans the trigger scans per sequence: enough for the longest reference, a power of two (few distinct launch shapes)
    int max_ref = 0, spans = 1;
    for (int b = 0; b < n_seqs; ++b) max_ref = ref_start[b + 1] - ref_start[b] > max_ref ? ref_start[b + 1] - ref_start[b] : max_ref;
    while (spans < trigger_spans(max_ref)) spans *= 2;
    c->gen_spans = spans;
    if ((rc = ensure_cap(c, &c->gen_part, &c->cap_part, (size_t)2 * n_seqs * spans))) return rc;
    if ((rc = ensure_cap(c, &c->gen_y, &c->cap_y, (size_t)n_seqs * ystride))) return rc;
    if ((rc = ensure_cap(c, &c->gen_trace, &c->cap_trace, (size_t)4 * n_seqs * ystride))) return rc;

    // Everything the device has to know goes there in two copies out of pinned memory, which nothing on the device reads or writes now (every call
    // is waited for, failed ones too), and nobody waits for them: ten pageable copies and four waits took 60 us of a call.
    int *const cnt_out = c->gen_counters, *const cnt_steps = c->gen_counters + g.max_batch, *const cnt_cur = c->gen_counters + 2 * g.max_batch;
    for (int b = 0; b < n_seqs; ++b) {                      // x: reset each slot; prompt[len-1] becomes the pending token
        c->T_host[seqs[b]] = 0;
        c->pending_host[seqs[b]] = prompts[prompt_offsets[b + 1] - 1];
        c->lo_from_host[seqs[b]] = 0;
        forget_imports(c, seqs[b]);
    }
    {
        int *const w = c->pin_block;
        const size_t B = g.max_batch;
        std::copy(c->T_host.begin(), c->T_host.end(), w);
        std::copy(c->pending_host.begin(), c->pending_host.end(), w + B);
        std::copy(c->lo_from_host.begin(), c->lo_from_host.end(), w + 2 * B);
        std::copy(seqs, seqs + n_seqs, w + 3 * B);
        std::fill(w + 3 * B + n_seqs, w + c->block_states, 0);
        for (int b = 0; b < n_seqs; ++b) {
            GenState s{};
            s.y = c->gen_y + (size_t)b * ystride; s.trace = c->gen_trace + (size_t)4 * b * ystride;
            s.n_out = cnt_out + b; s.n_steps = cnt_steps + b; s.cur = cnt_cur + 2 * b;
            s.host_count = c->pin_counts_dev + b; s.host_stride = g.max_batch;
            s.ref = c->gen_prompt + ref_at + ref_start[b]; s.doc_offsets = c->gen_prompt + docs_at + dof_at[b];
            s.ref_len = ref_start[b + 1] - ref_start[b]; s.n_docs = n_docs ? n_docs[b] : 0; s.n = n; s.k = k; s.max_new = max_new; s.prompt = c->gen_prompt;
            memcpy(w + c->block_states + sizeof(GenState) / 4 * b, &s, sizeof s);
        }
    }
    memset(c->pin_counts, 0, (size_t)2 * g.max_batch * sizeof(int));
    std::vector<int> T0(n_seqs);
    auto prepare = [&]() -> int {
        HIP_TRY(c, hipMemcpyAsync(c->block, c->pin_block, (c->block_states + sizeof(GenState) / 4 * n_seqs) * 4, hipMemcpyHostToDevice, st));
        std::fill(c->stale.begin(), c->stale.end(), 0);
        if (in_words <= GEN_STAGE_WORDS) {
            memcpy(c->pin_stage, prompts, (size_t)total_prompt * 4);
            if (total_ref) memcpy(c->pin_stage + ref_at, refs, (size_t)total_ref * 4);
            memcpy(c->pin_stage + docs_at, dof_host.data(), dof_host.size() * 4);
            HIP_TRY(c, hipMemcpyAsync(c->gen_prompt, c->pin_stage, in_words * 4, hipMemcpyHostToDevice, st));
        } else {
            HIP_TRY(c, hipMemcpyAsync(c->gen_prompt, prompts, (size_t)total_prompt * 4, hipMemcpyHostToDevice, st));
            if (total_ref) HIP_TRY(c, hipMemcpyAsync(c->gen_prompt + ref_at, refs, (size_t)total_ref * 4, hipMemcpyHostToDevice, st));
            HIP_TRY(c, hipMemcpyAsync(c->gen_prompt + docs_at, dof_host.data(), dof_host.size() * 4, hipMemcpyHostToDevice, st));
            HIP_TRY(c, hipStreamSynchronize(st));           // (the caller's memory)
        }
        // prompt[0 .. len-2] of every sequence.  Together where the steps have more than 48 rows: those of fewer rows give every
        // sequence the same bits as a call of its own, which its prompt in a pass of another length would not.
        if (n_seqs == 1) return prefill_passes(c, seqs[0], total_prompt - 1);
        if (together) return prefill_together(c, n_seqs, seqs, prompt_offsets);
        for (int b = 0; b < n_seqs; ++b)
            if (int r = prefill_rows(c, seqs[b], prompt_offsets[b + 1] - prompt_offsets[b] - 1, prompt_offsets[b])) return r;
        return LLMA_OK;
    };
    if ((rc = prepare())) return drained(c, rc);
    for (int b = 0; b < n_seqs; ++b) T0[b] = c->T_host[seqs[b]];

    // ---- the decoding loop: trigger -> rows -> forward -> accept, all on the device, all sequences of
    //      the batch in one step (k + 1 rows each; a sequence that has its max_new tokens idles: its
    //      trigger copies nothing and the accept kernel leaves its state alone).  The host only reads
    //      the output counts back to know when to stop, and it does so one step late: step s+1 is
    //      already enqueued when the counts of step s are awaited, so the GPU never waits for the host.
    const int m = k + 1;
    if (n_seqs > 1) {                                       // (prompt passes leave a slot of their own there; one sequence's is the same)
        const hipError_t e = hipMemcpyAsync(c->s.batch_slots, c->pin_block + 3 * g.max_batch, (size_t)n_seqs * 4, hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return drained(c, fail(c, LLMA_E_HIP, "llma_generate: %s", hipGetErrorString(e)));
    }
    std::vector<int> produced(n_seqs, 0);
    int steps = 0, enq = 0;
    auto enqueue = [&]() -> int {
        // cache length bound for the attention grid: every enqueued step adds at most m positions
        int t_max = 0;
        for (int b = 0; b < n_seqs; ++b) t_max = T0[b] + produced[b] > t_max ? T0[b] + produced[b] : t_max;
        int r = run_step(c, STEP_GEN, n_seqs, m, t_max + 2 * m, n_seqs == 1 ? seqs[0] : 0);
        if (r) return r;
        HIP_TRY(c, hipEventRecord(c->cnt_ev[enq & 1], st));
        ++enq;
        return LLMA_OK;
    };
    auto decode = [&]() -> int {
        int r = enqueue();
        while (r == LLMA_OK) {
            if ((r = enqueue())) break;                         // one step ahead
            HIP_TRY(c, hipEventSynchronize(c->cnt_ev[steps & 1]));
            bool done = true;
            for (int b = 0; b < n_seqs; ++b) {
                const int now = __atomic_load_n(&c->pin_counts[(size_t)(steps & 1) * g.max_batch + b], __ATOMIC_ACQUIRE);
                if (now > max_new || now < produced[b] || (now == produced[b] && produced[b] < max_new))
                    return fail(c, LLMA_E_HIP, "llma_generate: device output count of sequence %d went %d -> %d", b, produced[b], now);
                produced[b] = now;
                done = done && now >= max_new;
            }
            ++steps;
            if (done) break;
        }
        return r;
    };
    if ((rc = decode())) return drained(c, rc);
    // results: the counters and pending tokens in one copy, tokens and traces in one each, one wait (which also drains the step that ran ahead).  Where
    // they are more than the stage holds, the counters first, and then what the steps produced straight to the caller.
    const size_t y_words = (size_t)n_seqs * ystride;
    const bool staged = (trace ? 5 : 1) * y_words <= GEN_STAGE_WORDS;
    int *const y_host = c->pin_stage, *const trace_host = y_host + y_words;
    const int *const took = c->pin_block + 5 * (size_t)g.max_batch;
    auto fetch = [&]() -> int {
        HIP_TRY(c, hipMemcpyAsync(c->pin_block, c->block, c->block_states * 4, hipMemcpyDeviceToHost, st));
        if (staged) {
            HIP_TRY(c, hipMemcpyAsync(y_host, c->gen_y, y_words * 4, hipMemcpyDeviceToHost, st));
            if (trace) HIP_TRY(c, hipMemcpyAsync(trace_host, c->gen_trace, 4 * y_words * 4, hipMemcpyDeviceToHost, st));
        }
        HIP_TRY(c, hipStreamSynchronize(st));
        for (int b = 0; b < n_seqs; ++b)
            if (took[b] < 1 || took[b] > max_new) return fail(c, LLMA_E_HIP, "llma_generate: device step count of sequence %d is %d", b, took[b]);
        if (staged) return LLMA_OK;
        for (int b = 0; b < n_seqs; ++b) {
            HIP_TRY(c, hipMemcpyAsync(out_tokens + (size_t)b * max_new, c->gen_y + (size_t)b * ystride, (size_t)max_new * 4, hipMemcpyDeviceToHost, st));
            if (trace) HIP_TRY(c, hipMemcpyAsync(trace + (size_t)b * max_new, c->gen_trace + (size_t)4 * b * ystride, (size_t)took[b] * sizeof(llma_step_rec), hipMemcpyDeviceToHost, st));
        }
        HIP_TRY(c, hipStreamSynchronize(st));
        return LLMA_OK;
    };
    if ((rc = fetch())) return drained(c, rc);
    for (int b = 0; b < n_seqs; ++b) {
        const int seq = seqs[b];
        c->T_host[seq] = T0[b] + produced[b];
        c->pending_host[seq] = c->pin_block[g.max_batch + seq];
        if (staged) {
            memcpy(out_tokens + (size_t)b * max_new, y_host + (size_t)b * ystride, (size_t)max_new * 4);
            if (trace) memcpy(trace + (size_t)b * max_new, trace_host + (size_t)4 * b * ystride, (size_t)took[b] * sizeof(llma_step_rec));
        }
        n_out[b] = produced[b];
        if (n_steps) n_steps[b] = took[b];
    }
    return LLMA_OK;
}

extern "C" int llma_generate(llma_ctx *c, int32_t seq, const int32_t *prompt, int32_t prompt_len, const int32_t *ref,
                             const int32_t *doc_offsets, int32_t n_docs, int32_t n, int32_t k, int32_t max_new,
                             int32_t *out_tokens, int32_t *n_out, llma_step_rec *trace, int32_t *n_steps) {
    if (!c) return fail(nullptr, LLMA_E_INVAL, "llma_generate: null context");
    if (prompt_len < 1) return fail(c, LLMA_E_INVAL, "llma_generate: null / empty argument");
    if (n_docs < 0 || (n_docs > 0 && !doc_offsets)) return fail(c, LLMA_E_INVAL, "llma_generate: bad documents");
    const int32_t poff[2] = {0, prompt_len};
    return llma_generate_batch(c, 1, &seq, prompt, poff, ref, doc_offsets, &n_docs, n, k, max_new, out_tokens, n_out, trace, n_steps);
}

// ------------------------------------------------------------------------------------------------
// inspection / options
// ------------------------------------------------------------------------------------------------
extern "C" int llma_set_logits_dump(llma_ctx *c, float *dev_buf, int32_t capacity_rows) {
    if (!c) return fail(nullptr, LLMA_E_INVAL, "llma_set_logits_dump: null context");
    if (dev_buf && capacity_rows < 1) return fail(c, LLMA_E_INVAL, "llma_set_logits_dump: capacity_rows < 1");
    drop_graphs(c);
    c->logits_dump = dev_buf;
    c->dump_rows = dev_buf ? capacity_rows : 0;
    return LLMA_OK;
}

extern "C" int llma_set_option(llma_ctx *c, int32_t option, int32_t value) {
    if (!c) return fail(nullptr, LLMA_E_INVAL, "llma_set_option: null context");
    switch (option) {
        case LLMA_OPT_ACT_SPLIT: drop_graphs(c); c->opt_split = value ? 1 : 0; return LLMA_OK;
        case LLMA_OPT_KERNEL_TIMING: c->opt_timing = value ? 1 : 0; return LLMA_OK;
        case LLMA_OPT_USE_GRAPH: c->opt_graph = value ? 1 : 0; return LLMA_OK;
        default: return fail(c, LLMA_E_INVAL, "llma_set_option: unknown option %d", option);
    }
}

extern "C" int llma_time_step_gemm(llma_ctx *c, int32_t which, int32_t rows, int32_t reps, double *mean_us) {
    if (!c || !mean_us) return fail(c, LLMA_E_INVAL, "llma_time_step_gemm: null argument");
    if (c->cfg.dtype != LLMA_DTYPE_BF16) return fail(c, LLMA_E_INVAL, "llma_time_step_gemm: bf16 models only");
    if (which < 0 || which > 4) return fail(c, LLMA_E_RANGE, "llma_time_step_gemm: matrix %d (0 QKV, 1 O, 2 gate/up, 3 down, 4 LM head)", which);
    if (rows < 1 || rows > c->cfg.max_batch * (c->cfg.max_k + 1) || reps < 1 || reps > 100000)
        return fail(c, LLMA_E_RANGE, "llma_time_step_gemm: rows %d (1..max_batch (max_k + 1) = %d) or reps %d (1..100000) out of range",
                    rows, c->cfg.max_batch * (c->cfg.max_k + 1), reps);
    const llma_model_cfg &g = c->cfg;
    HIP_TRY(c, hipStreamSynchronize(c->st));
    if (which == 0) {           // the QKV epilogue appends K and V at (row_slot, row_pos): slot 0, position 0 for every row
        HIP_TRY(c, hipMemsetAsync(c->s.row_pos, 0, sizeof(int32_t) * rows, c->st));
        HIP_TRY(c, hipMemsetAsync(c->s.row_slot, 0, sizeof(int32_t) * rows, c->st));
    }
    hipEvent_t e0, e1;
    HIP_TRY(c, hipEventCreate(&e0));
    HIP_TRY(c, hipEventCreate(&e1));
    for (int pass = 0; pass < 2; ++pass) {              // pass 0 warms up (first-launch set-up of the kernel)
        const int n = pass ? reps : (reps < g.n_layers ? reps : g.n_layers);
        HIP_TRY(c, hipEventRecord(e0, c->st));
        for (int r = 0; r < n; ++r) {
            GemmArgs ga = step_gemm_args(c, which, r % g.n_layers, rows);
            ga.part = c->part;
            if (rows <= 48 && ga.epi != EPI_RESID) ga.rstd_out = c->rstd;
            if (rows > 48) {                            // the step's own choice: panel kernel, split-K form
                if (ga.plan.n_split > 1) { ga.ksplit = ga.plan.n_split; ga.part = c->part; if (ga.epi != EPI_RESID) ga.rstd_out = c->rstd; }
                launch_gemm_panel_bf16(ga, c->st);
            } else if (!launch_gemm_bf16(ga, c->st)) {
                return fail(c, LLMA_E_RANGE, "llma_time_step_gemm: launch refused for %d rows", rows);
            }
        }
        HIP_TRY(c, hipEventRecord(e1, c->st));
        HIP_TRY(c, hipEventSynchronize(e1));
    }
    HIP_TRY(c, hipGetLastError());
    float ms = 0.f;
    HIP_TRY(c, hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *mean_us = (double)ms * 1e3 / reps;
    return LLMA_OK;
}

extern "C" int llma_time_ffn_gemm(llma_ctx *c, int32_t rows, int32_t reps, double *mean_us) {
    if (rows > 48) return fail(c, LLMA_E_RANGE, "llma_time_ffn_gemm: rows %d outside 1..48", rows);
    return llma_time_step_gemm(c, 2, rows, reps, mean_us);
}

extern "C" int llma_get_kernel_timing(llma_ctx *c, int64_t *launches, double *total_ms) {
    if (!c || !launches || !total_ms) return fail(c, LLMA_E_INVAL, "llma_get_kernel_timing: null argument");
    HIP_TRY(c, hipStreamSynchronize(c->st));
    double tot = 0.0;
    for (auto &e : c->events) {
        float ms = 0.f;
        HIP_TRY(c, hipEventElapsedTime(&ms, e.a, e.b));
        tot += ms;
        (void)hipEventDestroy(e.a);
        (void)hipEventDestroy(e.b);
    }
    *launches = (int64_t)c->events.size();
    *total_ms = tot;
    c->events.clear();
    return LLMA_OK;
}
