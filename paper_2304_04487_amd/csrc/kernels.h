// Host-side launchers of the HIP kernels (each enqueues on the given stream and returns).
#pragma once
#include "common.h"

// ---- bf16 path (kernels_bf16.hip)
GemmPlan make_gemm_plan(int N, int K, int tiles_per_task);
bool tilek_ft_valid(const GemmPlan &p, int nt, int ft);     // can the decoding GEMM run ft feature tiles per workgroup at nt row tiles?
long tilek_cost(const GemmPlan &p, int ft);                 // tiles the busiest compute unit streams
int tilek_ft_default(const GemmPlan &p, int nt, bool few_rows);
static inline int tilek_bucket(int rows) { return rows <= 4 ? 3 : (rows + 15) / 16 - 1; }   // index into GemmPlan::tk_ft
void launch_pack_weight(const void *src, void *dst, int N, int K, int KSp, int rope_dh, int d, hipStream_t st);
void launch_kv_import_bf16(const void *k, const void *v, void *kh, void *kl, void *vh, void *vl, int H, int len, int dh,
                           int max_seq, hipStream_t st);
bool launch_gemm_bf16(const GemmArgs &a, hipStream_t st);   // false (nothing launched) unless 1 <= rows <= 48
void launch_gemm_panel_bf16(const GemmArgs &a, hipStream_t st);
int panel_prompt_split(const GemmPlan &p, int rows);                   // K ranges that suit a prompt pass of so many rows (1: no split)
size_t panel_part_bytes(const GemmPlan &p, int rows, int ns);          // scratch for the partial sums of ns ranges
void launch_rstd_rows(const float *ssq, int ssq_tiles, float eps, float *rstd, int rows, hipStream_t st);
void launch_attn_bf16(const AttnArgs &a, hipStream_t st);

// ---- fp32 path (kernels_f32.hip)
void launch_kv_import_f32(const void *k, const void *v, void *kc, void *vc, int H, int len, int dh,
                          int max_seq, hipStream_t st);
void launch_gemm_f32(const GemmArgs &a, hipStream_t st);
void launch_attn_f32(const AttnArgs &a, hipStream_t st);

// ---- shared small kernels (kernels_misc.hip)
struct HostIo {               // pinned host memory the kernels of a step read and write directly (device addresses)
    int *slot, *keff, *T, *pending, *lo_from;   // in, [n_seqs]: what the host knows about each sequence of a verification step
    int *draft;                          // in, [n_seqs][max_k]
    int *nacc, *next, *emit;             // out: [n_seqs], [n_seqs], [n_seqs][max_k+1]
};
struct StepState {            // device pointers describing the rows of the step in flight
    int *row_tok, *row_pos, *row_slot;   // [R]
    float *row_cs;                       // [R][head_dim/2][2] (cos, sin) of each row's position
    int *T, *pending;                    // [max_batch]
    int *batch_slots;                    // [n_seqs]
    int *keff;                           // [n_seqs] drafts actually used per sequence
    int *draft;                          // [n_seqs][max_k]
    int *lo_from;                        // [max_batch] (see AttnArgs)
    HostIo io;
};
struct GenState {             // device-resident state of llma_generate, one per sequence of the batch
    int *y; int *n_out; int *n_steps; int *trace;  // y[max_new], trace[max_new][4]
    int *cur;                            // [2] (doc, pos) of the trigger of the step in flight
    int *host_count; int host_stride;    // pinned: [2][host_stride], n_out after the even / odd steps
    const int *ref; const int *doc_offsets; int ref_len, n_docs;
    int n, k, max_new;
    const int *prompt;                   // device copy of the prompt (prefill)
};

// verification step: slots, lengths, pending tokens and drafts from s.io (the host's) into the device's copies
void launch_take_step(const StepState &s, int n_seqs, int max_k, hipStream_t st);
struct EmbedArgs {            // what the row set-up does with a row's token: h[r] = embed[token], and for bf16 models the first GEMM's input
    const void *embed; float *h; int d;
    const float *gain; void *nx_hi, *nx_lo; float *ssq_out; int KSp; bool quads;   // bf16 only (gain null: fp32): x = h * gain as tiled planes, sums of squares
    const PromptSeg *segs; int n_segs;                                 // prompt pass over several sequences (else null)
};
// rows of a step: row (b, j) = pending[slot_b] (j = 0) or draft[b][j-1]; pos = T[slot_b] + j; embedded into e.h.
// Generation steps (gen_dev set): the drafts are those of the best of part[b][0 .. spans), or with one span of the
// reference's scan, which then runs here; keff / draft are filled
void launch_setup_step_rows(const StepState &s, int n_seqs, int m, int max_k, const float *cs, int half, const EmbedArgs &e,
                            const GenState *gen_dev, const unsigned long long *part, int spans, hipStream_t st);
// rows of a prefill chunk for one slot: tokens prompt[T[slot] - *base_dev + j], pos = T[slot] + j; with e.segs of several
// sequences: each segment's tokens from prompt[tok0] on, at its own slot's T
void launch_setup_prefill_rows(const StepState &s, const int *prompt_dev, const int *base_dev, int m, int slot,
                               const float *cs, int half, const EmbedArgs &e, hipStream_t st);
void launch_advance_T(const StepState &s, int slot, int by, hipStream_t st);
// final arg max over the per-row partials, then prefix accept + KV truncate + bookkeeping
void launch_argmax_accept(const float *pval, const int *pidx, int n_part, const StepState &s, int n_seqs, int m,
                          int max_k, int vocab, const GenState *gen /*device array [n_seqs] or null*/, hipStream_t st);
// trigger: a reference is scanned in spans of TRIGGER_SPAN positions, one workgroup each
#define TRIGGER_SPAN 4096
static inline int trigger_spans(int ref_len) { return ref_len < 1 ? 1 : (ref_len - 1) / TRIGGER_SPAN + 1; }
// for each sequence being generated: part[b][span] = the span's best key (0 = none).  spans: at least trigger_spans of
// the longest reference
void launch_trigger_scan(const GenState *gen_dev, int n_seqs, int spans, unsigned long long *part, hipStream_t st);
// stateless trigger on device arrays (llma_find_trigger): result[0..2] = matched, doc, pos; part: scratch
// [trigger_spans(ref_len)]; with check_offsets the kernel itself validates doc_offsets and reports (-1, -1, -1) for a bad list
void launch_trigger_plain(const int *y, int y_len, const int *ref, const int *doc_offsets, int ref_len, int n_docs, int n,
                          unsigned long long *part, int *result, bool check_offsets, hipStream_t st);
// the same from pinned host memory: in = [y | ref | doc_offsets], `pieces` groups of four words, copied to dev (device) and
// scanned there; part: device scratch; result: pinned
void launch_trigger_host(const int *in, int *dev, int pieces, int y_len, int ref_len, int n_docs, int n, unsigned long long *part, int *result, hipStream_t st);
