// bf16 kernels of the verification forward (paper: Eq. 3 -- one causal forward over the
// pending token plus k copied tokens): weight re-tiling, the skinny weight-streaming GEMM
// with its fused epilogues (RMSNorm scaling, RoPE + KV append, SwiGLU, residual + next-norm
// preparation, vocabulary arg-max partials), and causal attention of a few query rows over a
// long KV cache.
//
// Everything here is HBM-bound at the row counts of a decoding step (1 + k <= 33 rows): the
// kernels are organised around streaming each weight / KV byte exactly once with fully
// coalesced 16-byte-per-lane loads, and use the MFMA unit because it consumes those
// registers directly.  Activations enter the MFMAs as hi + lo bf16 pairs (the extra MFMAs are
// free while memory-bound), which keeps 16 significand bits of every activation.
// In decoding steps, and in everything else of up to 48 rows, reduction orders are fixed by the matrix
// shapes and by absolute key positions, never by the number of rows: row j of a k-row step is
// bit-identical to the same token processed in a one-row step, in another step or in a short prompt
// pass.  Steps of more rows share another order, fixed by the shape too (GemmPlan::n_split).  Prompt
// passes of more than 48 rows (one sequence's, or several sequences' together) cut the K axis by how many
// rows they have and how many compute units there are (panel_prompt_split), so the K/V of a prefix differ
// at rounding level between passes of different lengths (logits on top by 3e-5 where the oracle is 1.5e-4 away).
#include <stdlib.h>

#include <atomic>
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

// Kernels that use more than 64 KB of dynamic LDS need the limit raised once per device.  `done`
// (one per kernel instantiation) holds a bit per device id; concurrent first calls may both set the
// attribute, which is harmless.
static void allow_full_lds(const void *kernel, std::atomic<uint64_t> &done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    const uint64_t bit = 1ull << dev;
    if (done.load(std::memory_order_acquire) & bit) return;
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    done.fetch_or(bit, std::memory_order_release);
}

// =============================================================================================
// weight re-tiling: row-major [N][K] bf16 -> 1 KiB MFMA A-operand blocks (see common.h)
// =============================================================================================
// rope_dh > 0 (the fused q/k/v matrix, d = model width): the 16 rows of a q or k tile are the
// rotary pairs (i, i + rope_dh/2) for 8 consecutive i -- rows 0..7 hold i, rows 8..15 hold
// i + rope_dh/2 -- so that the GEMM epilogue finds both elements of a pair in one wavefront.
__device__ __forceinline__ size_t src_row_of(size_t ft, int i, int rope_dh, int d) {
    if (rope_dh == 0) return ft * 16 + i;
    const int tiles_per_sec = d / 16;
    const int sec = (int)(ft / tiles_per_sec);
    if (sec == 2) return ft * 16 + i;
    const int tin = (int)(ft % tiles_per_sec);
    const int tph = rope_dh / 16;
    const int head = tin / tph, j = tin % tph;
    const int c = (i < 8) ? (8 * j + i) : (rope_dh / 2 + 8 * j + (i - 8));
    return (size_t)sec * d + (size_t)head * rope_dh + c;
}

__global__ void pack_weight_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int N, int K, int KSp,
                                   int rope_dh, int d) {
    // one thread per 16-byte piece of the destination
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)(N / 16) * KSp * 64;
    if (idx >= total) return;
    int lane = (int)(idx & 63);
    size_t blk = idx >> 6;
    int ks = (int)(blk % KSp);
    size_t ft = blk / KSp;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (ks < K / 32) {
        size_t row = src_row_of(ft, lane & 15, rope_dh, d);
        size_t col = (size_t)ks * 32 + (size_t)(lane >> 4) * 8;
        v = src[(row * K + col) / 8];
    }
    dst[idx] = v;
}

void launch_pack_weight(const void *src, void *dst, int N, int K, int KSp, int rope_dh, int d, hipStream_t st) {
    size_t total = (size_t)(N / 16) * KSp * 64;
    unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(pack_weight_kernel, dim3(blocks), dim3(256), 0, st, (const u32x4 *)src, (u32x4 *)dst, N, K, KSp, rope_dh, d);
}

// plain [H][len][dh] bf16 -> tiled K / V cache of one (slot, layer); lo planes (if any) are zeroed
__global__ void kv_import_bf16_kernel(const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
                                      bf16_t *__restrict__ kh, uint8_t *__restrict__ kl,
                                      bf16_t *__restrict__ vh, uint8_t *__restrict__ vl,
                                      int H, int len, int dh, int max_seq) {
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)H * len * dh;
    if (idx >= total) return;
    int c = (int)(idx % dh);
    int pos = (int)((idx / dh) % len);
    int h = (int)(idx / ((size_t)dh * len));
    size_t base = (size_t)h * max_seq * dh;
    size_t ko = base + kcache_off(pos, c, dh), vo = base + vcache_off(pos, c, dh);
    kh[ko] = k[idx];
    vh[vo] = v[idx];
    if (kl) { kl[ko] = 0; vl[vo] = 0; }
}

void launch_kv_import_bf16(const void *k, const void *v, void *kh, void *kl, void *vh, void *vl, int H, int len, int dh,
                           int max_seq, hipStream_t st) {
    size_t total = (size_t)H * len * dh;
    unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(kv_import_bf16_kernel, dim3(blocks), dim3(256), 0, st, (const bf16_t *)k, (const bf16_t *)v,
                       (bf16_t *)kh, (uint8_t *)kl, (bf16_t *)vh, (uint8_t *)vl, H, len, dh, max_seq);
}

// =============================================================================================
// skinny GEMM  Y[rows][N] = X[rows][K] . W[N][K]^T,  rows <= 16*NT
// =============================================================================================
// Two kernels share the fused epilogues below: the tile-K kernel for decoding steps (few rows,
// HBM-bound weight streaming) and the panel kernel for prompt processing (hundreds of rows,
// MFMA-bound).  D[i][n] = sum_k A[i][k] B[k][n] with i = feature, n = activation row, so a lane
// ends with features 4(l/16)..+3 of row l%16 of every row tile.
// ---- fused epilogues.  Lane l holds features 16 task + 4 (l/16) .. +3 of row 16 t + l%16.
// Everything an epilogue reads from memory is fetched by epi_prefetch() before the partial sums
// are reduced, so the kernel has one memory round trip on its critical path instead of three.
template <int NT>
struct EpiIn {
    f32x4 hv[NT], gv;          // RESID: residual values, next norm's gains
    int pos[NT], slot[NT];     // QKV: position and cache slot of the row
    f32x4 cs01[NT], cs23[NT];  // QKV: (cos, sin) of the lane's four rotary pairs
};

// QKV: section (q, k, v), head and tile of the head; head_dim is 64 or 128.  (No division: one is a few hundred cycles between
// the last sum and the kernel's end.)
struct QkvPlace { int sec, head, j; };
__device__ __forceinline__ QkvPlace qkv_place(const GemmArgs &a, int task) {
    const int tps = a.H * a.dh / 16, sh = a.dh == 128 ? 3 : 2;
    const int sec = (task >= tps) + (task >= 2 * tps), tin = task - sec * tps;
    return QkvPlace{sec, tin >> sh, tin & ((1 << sh) - 1)};
}

template <int NT, int EPI>
__device__ __forceinline__ void epi_prefetch(const GemmArgs &a, const GemmPlan &p, int task, int lane, EpiIn<NT> &in) {
    const int n = lane & 15, g4 = lane >> 4;
    const int f0 = task * 16 + g4 * 4;
    if (EPI == EPI_RESID) in.gv = *(const f32x4 *)(a.gain + f0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int row = t * 16 + n < a.rows ? t * 16 + n : 0;       // (unconditional loads: one under a branch waits for everything in flight)
        if (EPI == EPI_RESID) {
            in.hv[t] = *(const f32x4 *)(a.out + (size_t)row * p.N + f0);
        } else if (EPI == EPI_QKV) {
            in.pos[t] = a.row_pos[row];
            in.slot[t] = a.row_slot[row];
            const int half = a.dh / 2, i0 = 8 * qkv_place(a, task).j + (g4 & 1) * 4;
            const f32x4 *cp = (const f32x4 *)(a.row_cs + ((size_t)row * half + i0) * 2);
            in.cs01[t] = cp[0];
            in.cs23[t] = cp[1];
        }
    }
}

// QUADS: the order of the pieces in activation tiles (xtile_piece)
template <int NT, int EPI, int TILES, bool QUADS>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &a, const GemmPlan &p, int task, int lane,
                                              f32x4 (&acc)[TILES][NT], const float *rstd_s, const EpiIn<NT> &in) {
    const int n = lane & 15, g4 = lane >> 4;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int row = t * 16 + n;
        const bool live = row < a.rows;
        const int f0 = task * 16 + g4 * 4;
        if (EPI == EPI_RESID) {
            float x[4];
            float ss = 0.f;
            const f32x4 hv = in.hv[t] + acc[0][t];
#pragma unroll
            for (int r = 0; r < 4; ++r) { ss += hv[r] * hv[r]; x[r] = hv[r] * in.gv[r]; }
            if (live) {
                *(f32x4 *)(a.out + (size_t)row * p.N + f0) = hv;
                u32x2 hi, lo;
                split4(x, hi, lo);
                const size_t o = xtile_off(row, f0, a.nx_KSp, QUADS);
                *(u32x2 *)((bf16_t *)a.nx_hi + o) = hi;
                *(u32x2 *)((bf16_t *)a.nx_lo + o) = lo;
            }
            ss += lane_xor<16>(ss);
            ss += lane_xor<32>(ss);
            if (live && g4 == 0) a.ssq_out[(size_t)row * (p.N / 16) + task] = ss;
        } else if (EPI == EPI_SWIGLU) {
            if (live) {
                const float rs = rstd_s[row];
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float gg = acc[0][t][r] * rs, uu = acc[1][t][r] * rs;
                    v[r] = gg / (1.0f + __expf(-gg)) * uu;
                }
                u32x2 hi, lo;
                split4(v, hi, lo);
                const size_t o = xtile_off(row, f0, a.act_KSp, QUADS);
                *(u32x2 *)((bf16_t *)a.act_hi + o) = hi;
                *(u32x2 *)((bf16_t *)a.act_lo + o) = lo;
            }
        } else if (EPI == EPI_LMHEAD) {
            const float rs = live ? rstd_s[row] : 0.f;
            const f32x4 lg = acc[0][t] * rs;
            if (a.out != nullptr && live) *(f32x4 *)(a.out + (size_t)row * p.N + f0) = lg;
            float bv = lg[0];
            int bi = f0;
#pragma unroll
            for (int r = 1; r < 4; ++r)
                if (lg[r] > bv) { bv = lg[r]; bi = f0 + r; }
            auto better = [&](float ov, int oi) {
                if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            };
            better(lane_xor<16>(bv), lane_xor<16>(bi));
            better(lane_xor<32>(bv), lane_xor<32>(bi));
            if (g4 == 0 && live) {
                a.pval[(size_t)row * a.n_part + task] = bv;
                a.pidx[(size_t)row * a.n_part + task] = bi;
            }
        } else if (EPI == EPI_QKV) {
            // tile rows 0..7 = rotary first halves i, rows 8..15 = their partners i + dh/2
            const int d = a.H * a.dh;
            const QkvPlace place = qkv_place(a, task);
            const int sec = place.sec, head = place.head, j = place.j;
            const float rs = live ? rstd_s[row] : 0.f;
            float v[4], o4[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = acc[0][t][r] * rs;
            const int pos = in.pos[t];
            const size_t head_base = ((size_t)in.slot[t] * a.H + head) * (size_t)a.max_seq * a.dh;
            if (sec < 2) {
                const int half = a.dh / 2;
                const int i0 = 8 * j + (g4 & 1) * 4;
                const float cs[8] = {in.cs01[t][0], in.cs01[t][1], in.cs01[t][2], in.cs01[t][3],
                                     in.cs23[t][0], in.cs23[t][1], in.cs23[t][2], in.cs23[t][3]};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float pr = lane_xor<32>(v[r]);
                    o4[r] = (g4 < 2) ? (v[r] * cs[2 * r] - pr * cs[2 * r + 1]) : (v[r] * cs[2 * r] + pr * cs[2 * r + 1]);
                }
                const int c0 = (g4 < 2) ? i0 : half + i0;
                if (live) {
                    u32x2 hi, lo;
                    split4(o4, hi, lo);
                    if (sec == 0) {
                        const size_t o = xtile_off(row, head * a.dh + c0, d / 32, QUADS);
                        *(u32x2 *)((bf16_t *)a.q_hi + o) = hi;
                        *(u32x2 *)((bf16_t *)a.q_lo + o) = lo;
                    } else {
                        const size_t o = head_base + kcache_off(pos, c0, a.dh);
                        *(u32x2 *)((bf16_t *)a.k_hi + o) = hi;
                        if (a.k_lo) {                                   // one byte per element (see lo8x2)
                            const float res[4] = {o4[0] - bf16_to_f32((bf16_t)(hi[0] & 0xffffu)), o4[1] - bf16_to_f32((bf16_t)(hi[0] >> 16)),
                                                  o4[2] - bf16_to_f32((bf16_t)(hi[1] & 0xffffu)), o4[3] - bf16_to_f32((bf16_t)(hi[1] >> 16))};
                            *(uint32_t *)((uint8_t *)a.k_lo + o) = lo8x4(res);
                        }
                    }
                }
            } else if (live) {
                const int c0 = j * 16 + g4 * 4;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    bf16_t hi, lo;
                    split_bf16(v[r], hi, lo);
                    const size_t o = head_base + vcache_off(pos, c0 + r, a.dh);
                    ((bf16_t *)a.v_hi)[o] = hi;
                    if (a.v_lo) ((uint8_t *)a.v_lo)[o] = lo8x1(v[r] - bf16_to_f32(hi));
                }
            }
        }
    }
}

// adds sp[j .. j + U) below j1 to ss, in order: U loads in flight
template <int U>
__device__ __forceinline__ void add_tiles(const float *sp, int j, int j1, float &ss) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = sp[j + u < j1 ? j + u : j1 - 1];
#pragma unroll
    for (int u = 0; u < U; ++u) ss += j + u < j1 ? v[u] : 0.f;
}
// sum of sp[j0 .. j1), in order; j1 - j0 <= chunk, which is the same for all threads; j1 >= 1.  Loads are unconditional (see epi_prefetch) and as many as there
// are, rounded up to fours, at most sixteen at a time: always sixteen, QKV of d 1024 / 2048 (4 / 8 to add) took 9.2 / 16.4 us at 48 rows instead of 7.5 / 14.1
__device__ __forceinline__ float sum_of_tiles(const float *sp, int j0, int j1, int chunk) {
    float ss = 0.f;
    if (chunk <= 2) {                                   // (rows of up to 512 features)
        if (j0 >= j1) return ss;
        const float v0 = sp[j0], v1 = sp[j1 - 1];
        return j1 - j0 == 2 ? v0 + v1 : v0;
    }
    int j = j0, left = chunk;
    for (; left > 12; j += 16, left -= 16) add_tiles<16>(sp, j, j1, ss);
    if (left > 8) add_tiles<12>(sp, j, j1, ss);
    else if (left > 4) add_tiles<8>(sp, j, j1, ss);
    else if (left > 0) add_tiles<4>(sp, j, j1, ss);
    return ss;
}

// 16 bytes per lane through a buffer descriptor: base and size are wave-uniform, an offset past the size reads zeros
typedef __amdgpu_buffer_rsrc_t rsrc_t;
#define BUFFER_NOWHERE 0x40000000u     // past the end of every buffer it is used with (48 rows of at most 2^23 columns: below 1 GiB), also with an offset inside one added
__device__ __forceinline__ rsrc_t buffer_of(const void *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00027000);
}
template <bool NON_TEMPORAL>
__device__ __forceinline__ u32x4 buffer_load16(rsrc_t r, unsigned off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, NON_TEMPORAL ? 2 : 0);
}

// the arguments as seen from row r0 (a multiple of 16) on
__device__ __forceinline__ void offset_rows(GemmArgs &a, const GemmPlan &p, int r0) {
    const int t0 = r0 / 16;
    a.rows = a.rows - r0;
    if (a.out) a.out += (size_t)r0 * p.N;
    if (a.nx_hi) { a.nx_hi = (bf16_t *)a.nx_hi + (size_t)t0 * a.nx_KSp * 512; a.nx_lo = (bf16_t *)a.nx_lo + (size_t)t0 * a.nx_KSp * 512; }
    if (a.ssq_out) a.ssq_out += (size_t)r0 * (p.N / 16);
    if (a.act_hi) { a.act_hi = (bf16_t *)a.act_hi + (size_t)t0 * a.act_KSp * 512; a.act_lo = (bf16_t *)a.act_lo + (size_t)t0 * a.act_KSp * 512; }
    if (a.pval) { a.pval += (size_t)r0 * a.n_part; a.pidx += (size_t)r0 * a.n_part; }
    if (a.row_pos) { a.row_pos += r0; a.row_slot += r0; a.row_cs += (size_t)r0 * a.dh; }
    if (a.q_hi) { a.q_hi = (bf16_t *)a.q_hi + (size_t)t0 * (a.H * a.dh / 32) * 512; a.q_lo = (bf16_t *)a.q_lo + (size_t)t0 * (a.H * a.dh / 32) * 512; }
}

// ---------------------------------------------------------------------------------------------
// tile-K kernel (decoding steps): one workgroup per FT consecutive feature tiles, its waves split
// the K axis; each wave streams its weight blocks from HBM with non-temporal 1 KiB loads, the
// next batch in flight while the current one feeds the MFMAs; B operands come straight from the
// tiled activation planes (1 KiB contiguous per k-step and plane, shared through L2 by all
// workgroups); the waves' partial sums meet in LDS and are added in slice order (the 16 slices of QKV and the LM head in
// groups where tilek_groups says so: the order of launch_gemm_slices, whose sums have to be the same); the waves share the
// (feature tile, row tile) pairs of the fused epilogue.  The number of K slices depends on the matrix shape only, so
// the order of every sum is the same for any number of rows and any FT.  With 16 slices and more than one row tile a
// wave takes two slices one after the other (half the waves, twice the registers).
// Bound by the weight stream at one row; with more rows by the activations, which every workgroup reads: see
// tilek_ft_default.  Per layer of 7B, back to back: 75 us at one row (405 MB), 80 at 9 (84 before three gate/up pairs
// shared a workgroup), 98 at 17 (108), 122 at 33 (147).  13B at 33 rows 229 -> 201 us: eight waves instead of four
// for O and down (28 -> 23, 64 -> 53 us).
// The chain from a launch's start to its first MFMA and from the last one to its end is what short launches consist of, and a
// few percent of long ones: epilogue inputs and sums of squares by unconditional loads, the first operands before the live-row
// count, no division, all slices' sums read from LDS at once.  Back to back at 9 rows: d 512 QKV / O / gate/up / down 4.76 / 3.65 / 4.29 /
// 5.22 -> 3.83 / 3.30 / 3.72 / 4.87 us, 7B 18.6 / 9.4 / 30.1 / 20.1 -> 18.1 / 9.1 / 29.5 / 19.8 (an empty launch of a replayed graph: 1.6).
// Stores past the L2 and arguments preloaded into registers changed nothing.
// A ring of single k-steps with every load unconditional (zeros past the slice) was slower: the blocks of a
// tile are best requested several in a row (O 10.4 us in ones, 9.1 in fours, 8.7 with the requests past the end left out).
// ---------------------------------------------------------------------------------------------
#ifndef TK_TRACE
#define TK_TRACE(slot)      // (timeline probe of the one-off microbenchmarks; nothing in the library build)
#endif
// threads the kernel is built for, i.e. registers per wave: 128 at one row tile (16 waves, or two workgroups of 8, per
// compute unit); 256 with more row tiles, and for three or four gate/up pairs (that matrix always has 8 K slices)
constexpr int tilek_max_threads(int nt, int tiles_per_task, int ft) { return nt == 1 && (tiles_per_task == 1 || ft < 3) ? 1024 : 512; }
constexpr int tilek_turn_group(int epi) { return epi == EPI_RESID ? 24 : (epi == EPI_LMHEAD ? 48 : 12); }
// (a remainder by a power of two, 7B's slices of K = 4096 and d 512's, without the division: it stands before the kernel's first load)
__device__ __forceinline__ int tilek_turn(int group, int len) { return len < 2 ? 0 : (len & (len - 1)) == 0 ? (group * 7) & (len - 1) : (group * 7) % len; }
// SL, K slices per wave, is a constant of the kernel: as a runtime count it cost the matrices of one slice per wave
// registers (O and down of 13B in launches of 17 rows, mostly one of them live: 123 registers and 28.5 us on average,
// 94 and 21.2 as a constant)
template <int NT, int EPI, bool SPLIT, int FT, int SL = 1>
__global__ __launch_bounds__((tilek_max_threads(NT, EPI == EPI_SWIGLU ? 2 : 1, FT))) void gemm_tilek_bf16(GemmArgs a) {
    constexpr int TILES = (EPI == EPI_SWIGLU) ? 2 : 1;
    constexpr int AT = FT * TILES;                 // weight tiles per k-step
    // k-steps per load batch (two batches in flight): one weight tile and one row tile per wave (O, down at
    // up to 16 rows: 256 workgroups, one per compute unit) need four for enough bytes in flight
    constexpr int UB = (AT * NT >= 4) ? 1 : (AT * NT == 1 ? 4 : 2);
    constexpr int PL = SPLIT ? 2 : 1;
    constexpr bool QUADS = NT * 16 > XTILE_ROWWISE;  // (a launch of NT row tiles has more than 16 (NT - 1) rows)
    static_assert(XTILE_ROWWISE % 16 == 0 && XTILE_ROWWISE <= 48, "every launch of NT row tiles must use one order; the panel kernel has more than 48 rows");
    extern __shared__ f32x4 red[];                 // [S][AT][NT][64], then rstd[16*NT] floats
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6, S = W * SL;
    TK_TRACE(0);
    // llma_generate launches k + 1 rows in every step; how many of them carry a token (1 + the
    // drafts the trigger found) is only known on the device.  The dead rows cost nothing here:
    // their lanes read past the end of a descriptor (zeros, no traffic) and the epilogue skips them.
    auto clamp_rows = [&]() {
        if (a.rows_live != nullptr) {
            const int live = *a.rows_live + 1;
            a.rows = live < a.rows ? live : a.rows;
        }
    };
    if (NT > 1) clamp_rows();
    const GemmPlan &p = a.plan;
    const int KSp = p.KSp;
    const int task0 = blockIdx.x * FT;
    // slice boundaries floor(KSp * slice / S); S is 8 or 16 (a shift; a 64-bit division here costs
    // a few hundred instructions before the kernel's first load)
    const int s_sh = 31 - __builtin_clz(S);
    int ks0 = 0, ks1 = 0, turn = 0;                // the K slice being streamed, and where in it the walk starts
    // If every workgroup walked its slices from their first k-step, the whole chip would at any moment
    // read the blocks of the same few k-steps of every tile -- addresses a fixed stride apart, which
    // fall on few memory channels.  So the walk over a slice starts `turn` k-steps in and wraps around
    // (QKV 18.9 -> 18.4 us, down 18.9 -> 17.9 us per launch at the 7B shapes), seven steps further from group to group (five: LM head
    // of 7B 42.5 us at one row, seven or one: 39.8; QKV 18.85 and 18.4 at nine; three: 42.6 and 18.65).  The start is a
    // function of the tile's group of 12 (24 for O and down, 48 for the LM head: whole workgroups of the form in slices) -- the same for 1, 2, 3 or 4 tiles per workgroup -- and of the
    // slice length, so a tile's sums are added in an order that no launch parameter changes.
    const int turn_grp = task0 / tilek_turn_group(EPI);
    auto k_turn = [&](int len) { return tilek_turn(turn_grp, len); };
    float *rstd_s = (float *)(red + (size_t)S * AT * NT * 64);

    // Every operand is fetched through a buffer descriptor of its own (one per weight tile, one per activation plane):
    // wave-uniform base and size, one 32-bit offset per lane and k-step for all tiles (a 64-bit pointer per tile took
    // twice the registers: three gate/up pairs at three row tiles spilled, 51 -> 40 us at 33 rows).  Rows without a
    // token get an offset past the end: zeros, and no traffic.  Three weight tiles and one row tile are the exception, their
    // weights go by pointer: QKV of 7B at one row 18.15 us through descriptors, 17.9 by pointer; with one, two or four
    // tiles pointers are no better or worse (13B at one row: O 11.8 and 12.0 us, QKV 25.9 and 26.0).
    constexpr bool W_BY_POINTER = NT == 1 && AT == 3;
    const unsigned w_lane = (unsigned)lane * 16u;
    rsrc_t wb[AT];
    const u32x4 *wp[AT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
            int task = task0 + f;
            task = task < p.tasks ? task : p.tasks - 1;          // ragged last workgroup: recompute the last tile
            const char *tile = (const char *)a.W + ((size_t)(task + i * p.tasks) * KSp) * 1024;
            if (W_BY_POINTER) wp[f * TILES + i] = (const u32x4 *)(tile + w_lane);
            else wb[f * TILES + i] = buffer_of(tile, (unsigned)KSp * 1024u);
        }
    auto load_w = [&](int i, int k) -> u32x4 {
        if constexpr (W_BY_POINTER) return __builtin_nontemporal_load(wp[i] + (size_t)k * 64);
        else return buffer_load16<true>(wb[i], (unsigned)k * 1024u + w_lane);
    };
    // One row tile (the usual decoding step): the wave's first operands are requested before the live-row count is
    // known, which is a round trip to memory of its own (0.5 us at d 512).
    u32x4 avA[AT][UB];
    if (NT == 1) {
        const int k_lo = (KSp * wave * SL) >> s_sh, k_hi = (KSp * (wave * SL + 1)) >> s_sh;
        if (k_lo < k_hi) {
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                int k = (k_lo + u < k_hi ? k_lo + u : k_hi - 1) + k_turn(k_hi - k_lo);
                k = k >= k_hi ? k - (k_hi - k_lo) : k;
#pragma unroll
                for (int i = 0; i < AT; ++i) avA[i][u] = load_w(i, k);
            }
        }
    }
    const unsigned x_bytes = (unsigned)(NT * KSp) * 1024u;
    const rsrc_t xh = buffer_of(a.Xhi, x_bytes), xl = buffer_of(a.Xlo, x_bytes);
    int nt_live = NT;                              // row tiles with at least one live row (uniform)
    unsigned x_lane[NT];
    auto place_rows = [&]() {
        nt_live = (a.rows + 15) >> 4;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            x_lane[t] = t * 16 + (lane & 15) < a.rows ? (unsigned)(t * KSp) * 1024u + (unsigned)xtile_piece(lane, QUADS) * 16u : BUFFER_NOWHERE;
    };
    place_rows();

    auto issue = [&](int ks, u32x4 (&av)[AT][UB], u32x4 (&bv)[PL][NT][UB], bool weights = true) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            int k = ks + u;
            k = (k < ks1 ? k : ks1 - 1) + turn;
            k = k >= ks1 ? k - (ks1 - ks0) : k;
            const unsigned off = (unsigned)k * 1024u;
            if (weights)
#pragma unroll
            for (int i = 0; i < AT; ++i) av[i][u] = load_w(i, k);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (t == 0 || t < nt_live) {           // a row tile without a live row is skipped altogether
                    bv[0][t][u] = buffer_load16<false>(xh, off + x_lane[t]);
                    if (SPLIT) bv[PL - 1][t][u] = buffer_load16<false>(xl, off + x_lane[t]);
                }
        }
    };
    f32x4 acc[AT][NT];
    auto compute = [&](int ks, u32x4 (&av)[AT][UB], u32x4 (&bv)[PL][NT][UB]) {
#pragma unroll
        for (int u = 0; u < UB; ++u)
            if (ks + u < ks1) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (t == 0 || t < nt_live)
#pragma unroll
                    for (int i = 0; i < AT; ++i) {
                        acc[i][t] = mfma16x16x32(av[i][u], bv[0][t][u], acc[i][t]);
                        if (SPLIT) acc[i][t] = mfma16x16x32(av[i][u], bv[PL - 1][t][u], acc[i][t]);
                    }
            }
    };

    u32x4 bvA[PL][NT][UB], avB[AT][UB], bvB[PL][NT][UB];
    int slice = wave * SL;
    int ks = (KSp * slice) >> s_sh;
    ks1 = (KSp * (slice + 1)) >> s_sh;
    ks0 = ks; turn = k_turn(ks1 - ks0);
    if (ks < ks1) issue(ks, avA, bvA, NT > 1);      // (one row tile: the weights are already on their way)
    if (NT == 1) { clamp_rows(); place_rows(); }
    // epilogue inputs and rstd while the first batch is in flight
    // (after the sums, wave w finishes the (feature tile, row tile) pairs w, w + W, ...)
    constexpr int UNITS = FT * NT;
    EpiIn<1> in;
    if (wave < UNITS && task0 + wave / NT < p.tasks) {
        GemmArgs at = a;
        offset_rows(at, p, (wave % NT) * 16);
        epi_prefetch<1, EPI>(at, p, task0 + wave / NT, lane, in);
    }
    if (EPI != EPI_RESID && threadIdx.x < 256) {
        const int row = threadIdx.x >> 4, i = threadIdx.x & 15;
        const int chunk = (a.ssq_tiles + 15) / 16;
        const int j0 = i * chunk, j1 = (j0 + chunk < a.ssq_tiles) ? j0 + chunk : a.ssq_tiles;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int r = t * 16 + row;
            float ss = 0.f;
            if (r < a.rows) {
                ss = sum_of_tiles(a.ssq_in + (size_t)r * a.ssq_tiles, j0, j1, chunk);
            }
            ss += lane_xor<1>(ss);
            ss += lane_xor<2>(ss);
            ss += lane_xor<4>(ss);
            ss += lane_xor<8>(ss);
            if (i == 0) rstd_s[r] = 1.0f / sqrtf(ss / (float)(a.ssq_tiles * 16) + a.eps);
        }
    }
#pragma unroll
    for (int sl = 0; sl < SL; ++sl) {
        if (sl > 0) {
            slice = wave * SL + sl;
            ks = (KSp * slice) >> s_sh;
            ks1 = (KSp * (slice + 1)) >> s_sh;
            ks0 = ks; turn = k_turn(ks1 - ks0);
            if (ks < ks1) issue(ks, avA, bvA);
        }
#pragma unroll
        for (int i = 0; i < AT; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[i][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
        while (ks < ks1) {
            if (ks + UB < ks1) issue(ks + UB, avB, bvB);
            compute(ks, avA, bvA);
            TK_TRACE(1);
            ks += UB;
            if (ks >= ks1) break;
            if (ks + UB < ks1) issue(ks + UB, avA, bvA);
            compute(ks, avB, bvB);
            ks += UB;
        }
        // ---- the slices' partial sums meet in LDS and are added below, in slice order or in groups of slices
#pragma unroll
        for (int i = 0; i < AT; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) red[((slice * AT + i) * NT + t) * 64 + lane] = acc[i][t];
    }
    TK_TRACE(2);
    __syncthreads();
    for (int u = wave; u < UNITS; u += W) {
        const int f = u / NT, t = u % NT, task = task0 + f;
        if (task >= p.tasks || t >= nt_live) continue;
        GemmArgs at = a;
        offset_rows(at, p, t * 16);
        if (u != wave) epi_prefetch<1, EPI>(at, p, task, lane, in);
        f32x4 sum[TILES][1];
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
            const f32x4 *const slices = red + ((f * TILES + i) * NT + t) * 64 + lane;
            constexpr int STRIDE = AT * NT * 64;
            // (8 or 16 slices, all requested before the first is added: in a loop that adds one after the other each waits for its own)
            f32x4 r[16];
#pragma unroll
            for (int w = 0; w < 8; ++w) r[w] = slices[w * STRIDE];
            if (S == 16) {
#pragma unroll
                for (int w = 8; w < 16; ++w) r[w] = slices[w * STRIDE];
                // in groups (tilek_groups): what one workgroup of the form in slices sums
                const int groups = EPI == EPI_QKV || EPI == EPI_LMHEAD ? tilek_groups(p) : 1;
                if (groups == 4) {
#pragma unroll
                    for (int g = 0; g < 16; g += 4) r[g] = ((r[g] + r[g + 1]) + r[g + 2]) + r[g + 3];
                    r[0] = ((r[0] + r[4]) + r[8]) + r[12];
                } else {
#pragma unroll
                    for (int w = 1; w < 8; ++w) r[0] += r[w];
                    if (groups == 2) {
#pragma unroll
                        for (int w = 9; w < 16; ++w) r[8] += r[w];
                        r[0] += r[8];
                    } else {
#pragma unroll
                        for (int w = 8; w < 16; ++w) r[0] += r[w];
                    }
                }
            } else {
#pragma unroll
                for (int w = 1; w < 8; ++w) r[0] += r[w];
            }
            sum[i][0] = r[0];
        }
        gemm_epilogue<1, EPI, TILES, QUADS>(at, p, task, lane, sum, rstd_s + 16 * t, in);
    }
    TK_TRACE(3);
}

// Which (feature tiles per workgroup) values the tile-K kernel can run for a matrix at nt row tiles: the
// K slices' partial sums (slices x tiles x row tiles KiB) must fit LDS.
bool tilek_ft_valid(const GemmPlan &p, int nt, int ft) {
    if (ft < 1 || ft > 4 || nt < 1 || nt > 3) return false;
    return (size_t)p.tk_waves * p.tiles_per_task * ft * nt * 1024 + 256 <= 160 * 1024 - 1024;
}
static int cu_count() {
    static std::atomic<int> n_cu{0};                  // (the same for every device of this kind; concurrent first calls find the same)
    int n = n_cu.load(std::memory_order_relaxed);
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) n = prop.multiProcessorCount;
        if (n <= 0) n = 256;
        n_cu.store(n, std::memory_order_relaxed);
    }
    return n;
}
// A workgroup streams from its compute unit alone, so a launch takes as long as the unit with the most tiles: rounds of
// workgroups x tiles per workgroup.  The value with the least of that wins, of equal ones the largest: every workgroup
// reads all rows' activations, which is half of the traffic at 16 rows and one tile (pair) each.  7B gate/up, 688 pairs:
// three per workgroup (230 workgroups, one round) instead of one takes 30.6 instead of 34.9 us at nine rows, 33.4
// instead of 43.9 at 17, 39.3 instead of 63.6 at 33; two (344 workgroups) 37.  Steps of up to four rows have next to
// no activation traffic: there the smallest of equal values wins for the matrices with 8 slices (gate/up at one row
// 29.6 against 30.1 us: two workgroups per compute unit overlap each other's start and end).
long tilek_cost(const GemmPlan &p, int ft) {
    const long n_cu = cu_count();
    return ((p.tasks + ft - 1) / ft + n_cu - 1) / n_cu * ft;
}
int tilek_ft_default(const GemmPlan &p, int nt, bool few_rows) {
    int best = 1;
    long best_cost = 0;
    for (int ft = 1; ft <= 4; ++ft) {
        if (!tilek_ft_valid(p, nt, ft)) continue;
        const long cost = tilek_cost(p, ft);
        if (best_cost == 0 || cost < best_cost || (cost == best_cost && !(few_rows && p.tk_waves == 8))) { best = ft; best_cost = cost; }
    }
    return best;
}

template <int NT, int EPI, int FT, int SL>
static void launch_tilek_slices(const GemmArgs &a, hipStream_t st) {
    constexpr int TILES = (EPI == EPI_SWIGLU) ? 2 : 1;
    const GemmPlan &p = a.plan;
    const int S = p.tk_waves, W = S / SL;                            // K slices (8 or 16) and waves
    size_t lds = (size_t)S * FT * TILES * NT * 1024 + 256;
    // One gate/up pair per workgroup: at most two workgroups per compute unit, by asking for more than a third of its LDS.
    // The kernel's 77 registers would let three in; with two, the workgroups of the last round go to whichever units are
    // done first: 7B at one row (688 workgroups) 30.1 -> 29.35 us, a k = 0 step of 32 layers 2.96 -> 2.93 ms; 13B 44.6 -> 44.4
    if (NT == 1 && EPI == EPI_SWIGLU && FT == 1 && lds < 56 * 1024) lds = 56 * 1024;
    dim3 grid((p.tasks + FT - 1) / FT), block(W * 64);
    if (a.split) {
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void *)gemm_tilek_bf16<NT, EPI, true, FT, SL>, done);
        hipLaunchKernelGGL((gemm_tilek_bf16<NT, EPI, true, FT, SL>), grid, block, lds, st, a);
    } else {
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void *)gemm_tilek_bf16<NT, EPI, false, FT, SL>, done);
        hipLaunchKernelGGL((gemm_tilek_bf16<NT, EPI, false, FT, SL>), grid, block, lds, st, a);
    }
}

template <int NT, int EPI, int FT>
static void launch_tilek(const GemmArgs &a, hipStream_t st) {
    // 16 slices and more than one row tile: eight waves of two slices (gate/up always has eight slices)
    constexpr int MAX_WAVES = tilek_max_threads(NT, EPI == EPI_SWIGLU ? 2 : 1, FT) / 64;
    if constexpr (NT > 1 && EPI != EPI_SWIGLU) {
        if (a.plan.tk_waves > MAX_WAVES) return launch_tilek_slices<NT, EPI, FT, 2>(a, st);
    }
    launch_tilek_slices<NT, EPI, FT, 1>(a, st);
}

template <int NT, int EPI>
static void launch_gemm_nt_epi(const GemmArgs &a, hipStream_t st) {
    const int ft = a.plan.tk_ft[tilek_bucket(a.rows)];
    switch (tilek_ft_valid(a.plan, NT, ft) ? ft : tilek_ft_default(a.plan, NT, a.rows <= 4)) {
        case 1: launch_tilek<NT, EPI, 1>(a, st); break;
        case 2: launch_tilek<NT, EPI, 2>(a, st); break;
        case 3: launch_tilek<NT, EPI, 3>(a, st); break;
        default:
            if constexpr (!(EPI == EPI_SWIGLU && NT == 3)) launch_tilek<NT, EPI, 4>(a, st);     // (its partial sums exceed LDS)
            break;
    }
}

template <int NT>
static void launch_gemm_nt(const GemmArgs &a, hipStream_t st) {
    switch (a.epi) {
        case EPI_RESID: launch_gemm_nt_epi<NT, EPI_RESID>(a, st); break;
        case EPI_SWIGLU: launch_gemm_nt_epi<NT, EPI_SWIGLU>(a, st); break;
        case EPI_QKV: launch_gemm_nt_epi<NT, EPI_QKV>(a, st); break;
        default: launch_gemm_nt_epi<NT, EPI_LMHEAD>(a, st); break;
    }
}

// ---------------------------------------------------------------------------------------------
// Panel GEMM (prompt passes and steps of more than 48 rows): a workgroup computes a block of weight tiles x
// RT row tiles over a range of the K axis.  Its 8 waves take two (or one) weight tiles each and all RT row tiles; where the K
// axis is split, 5 to 7 waves of two tiles are another way to give every compute unit one workgroup (panel_cut).  The
// block's activations pass through LDS in chunks of KC k-steps, three chunks deep, loaded straight into LDS (buffer
// loads; no registers, no LDS stores); every wave streams its own weight blocks from memory / L2, where the workgroups
// of the other row blocks find them again, into a ring of WD register sets.  One barrier per chunk.
// Bound by MFMA issue on long prompts (1535 rows, four layers: 4.97 TFLOP of bf16 products in 4.1 ms = 1.2 PFLOP/s; a
// large library product runs at 1.37 here), by the weight stream and the start and end of each launch at few rows.
// What made the difference (7B, four layers' prompt pass of 1535 rows / a layer's GEMMs at 144 rows: 5.44 ms / 194 us
// before): the order of requests is the source's (the compiler moved every one next to its use), the activations
// take no registers on the way to LDS, no mask on the weights and no early exit inside a turn of the ring (either
// made every turn end with a wait for all loads in flight), and the buffer form of the loads into LDS (the global
// form counts as a flat access: behind one the compiler waits for everything).  4.85 ms / 177 us.  Then the requests
// spread over the chunk's MFMAs (all made at its start they kept the wave from its first MFMA for a third of the chunk)
// and the barrier moved before its last group: 4.63 -> 4.51 ms / 170.5 -> 167.0 us, 288 rows 272 -> 258, 528 rows 441 -> 410.  A chunk
// of 9 row tiles went from 3420 to 3070 cycles, 2304 of them MFMA, but the clock from 1.62 to 1.51 GHz: long prompts
// are bound by the card's power.  Waves that take four weight tiles and half of the rows (half the LDS reads, each weight
// block loaded by two waves): 5.18 ms / 208 us; four waves of four tiles and all rows, 512 registers: 4.6 % slower than eight.
// ---------------------------------------------------------------------------------------------
// rstd[row] = rsqrt(sum of the row's per-tile sums of squares / d + eps), same summation order as
// the decoding kernels' in-kernel version (16 threads per row, contiguous chunks, butterfly); r = the
// calling thread's row (whole waves call this: the butterfly runs over 16-lane groups)
__device__ __forceinline__ void rstd_of_row(const float *__restrict__ ssq, int ssq_tiles, float eps, float *__restrict__ rstd, int rows, int r, int i) {
    const int chunk = (ssq_tiles + 15) / 16;
    const int j0 = i * chunk, j1 = (j0 + chunk < ssq_tiles) ? j0 + chunk : ssq_tiles;
    float ss = 0.f;
    if (r < rows) {
        ss = sum_of_tiles(ssq + (size_t)r * ssq_tiles, j0, j1, chunk);
    }
    ss += lane_xor<1>(ss);
    ss += lane_xor<2>(ss);
    ss += lane_xor<4>(ss);
    ss += lane_xor<8>(ss);
    if (i == 0 && r < rows) rstd[r] = 1.0f / sqrtf(ss / (float)(ssq_tiles * 16) + eps);
}

// Split-K form of the panel GEMM: the rows whose rstd a wave computes are first .. first + 3 and every step-th group of four after
// them.  A launch of few waves and many rows (a narrow matrix: one feature block) goes round several times.
struct RstdShare { int first, step; };
__host__ __device__ __forceinline__ RstdShare rstd_share(int tasks, int nw, int ft, int row_blocks, int fb, int rb, int range, int ranges, int wave) {
    const int blocks = (tasks + nw * ft - 1) / (nw * ft) * row_blocks, workgroups = blocks * ranges;       // (those of padding feature blocks have left)
    return RstdShare{4 * (range * blocks + fb * row_blocks + rb + workgroups * wave), 4 * workgroups * nw};
}

#define PANEL_KC 2          // k-steps per LDS chunk
#define PANEL_TURN 8        // k-steps of weights in registers; the K axis is cut into ranges of whole turns of this ring
#define PANEL_RT_MAX 10     // row tiles per workgroup: 4 .. 10,
#define PANEL_RT_SPLIT 12   // and up to 12 where the K axis is split, six waves take 12 weight tiles, and one row block then holds all rows
#define PANEL_STAGES 3      // chunks of activations in LDS: one in use, the others on their way
#ifndef PN_TRACE
#define PN_TRACE(slot, chunk)   // (timeline probe of the one-off microbenchmarks; nothing in the library build)
#endif
// 16 bytes per lane from a buffer straight into LDS (lane l's land at lds + 16 l); counted like any load.  (The buffer
// form: behind a global_load_lds the compiler waits for every load in flight before it uses any other load's value.)
__device__ __forceinline__ void load_to_lds(rsrc_t r, unsigned lane_off, unsigned off, u32x4 *lds) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16, (int)lane_off, (int)off, 0, 0);
}
// waits until at most N of the wave's loads are outstanding and its LDS reads are done, then for the workgroup;
// no memory access moves across it in either direction
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory"); }

// the counted wait above relies on the order in which a wave's loads were issued
__device__ __forceinline__ void requests_stay_in_order() { asm volatile("" ::: "memory"); __builtin_amdgcn_sched_barrier(0); }

// RT row tiles, NW waves of AT weight tiles each
template <int RT, int AT, int NW>
struct PanelShape {
    static_assert(PANEL_KC % 2 == 0, "an even number of groups per chunk: the first group's registers are the same in every chunk");
    static constexpr int TG = (RT + 3) / 4, TB = (RT + TG - 1) / TG;     // row tiles whose operands are read from LDS together
    static constexpr int WD = PANEL_TURN;                                // k-steps of weights in registers
    static constexpr int XB = (2 * RT * PANEL_KC + NW - 1) / NW;         // activation blocks a wave fetches per chunk
    // loads a wave has certainly requested after a chunk's activations when it comes to wait for them: the next
    // chunk's, and the weights of two chunks (before the first chunk: of the ring's first turn)
    static constexpr int LATER = XB + (WD - PANEL_KC < 2 * PANEL_KC ? WD - PANEL_KC : 2 * PANEL_KC) * AT;
    static_assert(LATER <= 63, "the wait counter has six bits");
};
template <int RT, int EPI, int AT, int NW>
__global__ __launch_bounds__(NW * 64, 2) void gemm_panel_bf16(GemmArgs a0) {
    using Shape = PanelShape<RT, AT, NW>;
    constexpr int WD = Shape::WD, XB = Shape::XB;
    constexpr int TILES = (EPI == EPI_SWIGLU) ? 2 : 1, FT = AT / TILES;
    constexpr int KC = PANEL_KC;
    constexpr int CH = 2 * RT * KC * 64;           // 16-byte pieces per stage (both planes)
    constexpr bool SLICED = EPI == EPI_SLICES, PARTIAL = SLICED || EPI == EPI_RAW;
    extern __shared__ u32x4 xs[];                  // [stages][2 planes][RT][KC][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const GemmPlan &p = a0.plan;
    const int KSp = p.KSp;
    // Workgroup order: the row blocks of one feature block get ids that differ by multiples of 8, i.e.
    // they are dispatched close together and onto the same XCD, so the feature block's weights are
    // fetched from HBM once and found in that XCD's L2 by the other row blocks.
    const int RB = a0.panel_rb;
    const int grp = blockIdx.x / (8 * RB), within = blockIdx.x % (8 * RB);
    const int fb = grp * 8 + (within & 7), rb = within >> 3;
    if (fb * NW * FT >= p.tasks) return;           // (feature blocks are padded to whole groups of 8)
    const int r0 = rb * (16 * RT);
    const int rt0 = r0 / 16;
    GemmArgs a = a0;
    offset_rows(a, p, r0);
    const int task0 = (fb * NW + wave) * FT;         // may lie past the last tile (padding feature blocks): clamped loads, no epilogue

    rsrc_t wb[AT];                                 // a descriptor per weight tile (wave-uniform)
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
            int task = task0 + f;
            task = task < p.tasks ? task : p.tasks - 1;
            wb[f * TILES + i] = buffer_of((const char *)a.W + ((size_t)(task + i * p.tasks) * KSp) * 1024, (unsigned)KSp * 1024u);
        }
    // the row block's part of the activation planes (a plane may be larger than the 4 GiB of a 32-bit offset)
    const int n_rt_total = (a0.rows + 15) / 16;                              // row tiles that exist
    const int n_rt = n_rt_total - rt0 < RT ? n_rt_total - rt0 : RT;          // and those of this block
    const unsigned x_bytes = (unsigned)n_rt * (unsigned)KSp * 1024u;
    const size_t x_start = (size_t)rt0 * KSp * 1024;
    const rsrc_t xh = buffer_of((const char *)a.Xhi + x_start, x_bytes), xl = buffer_of((const char *)a.Xlo + x_start, x_bytes);

    // SLICED: the workgroup's range is a group of n_slices K slices of the tile-K kernel, each walked from the same k-step on and
    // summed by itself, so that the sums are the same; k-steps past a range read zeros.  (Several slices: of equal, even length,
    // so that a chunk lies in one of them.)
    static_assert(!SLICED || KC == 2, "");
    const int n_slices = SLICED ? p.tk_waves / (int)gridDim.y : 1, S = n_slices * (int)gridDim.y;
    const int slice_lo = SLICED ? (int)((long)KSp * ((int)blockIdx.y * n_slices) / S) : 0;
    const int slice_len = SLICED ? (int)((long)KSp * ((int)blockIdx.y * n_slices + 1) / S) - slice_lo : 0;
    const int slice_turn = SLICED ? tilek_turn(fb * (NW * AT) / (AT == 1 ? tilek_turn_group(EPI_RESID) : (NW == 8 ? tilek_turn_group(EPI_LMHEAD) : tilek_turn_group(EPI_QKV))), slice_len) : 0;
    // where a chunk lies: its slice's first k-step and its own place in the slice
    struct Place { int lo, at; };
    auto next_chunk = [&](Place &c) {
        c.at += KC;
        if (c.at >= slice_len && c.lo + slice_len < slice_lo + n_slices * slice_len) { c.at = 0; c.lo += slice_len; }
    };
    auto place_of = [&](int chunk) {
        Place c = {slice_lo, 0};
        for (int i = 0; i < chunk; ++i) next_chunk(c);
        return c;
    };
    Place x_at = place_of(2), w_at = place_of((WD - KC) / KC);       // (the chunks requested while the first one is multiplied)
    int in_slice = 0;                                               // k-steps of the present slice multiplied
    auto slice_step = [&](const Place &c, int u) { const int t = c.at + u + slice_turn; return c.lo + (c.at + u >= slice_len ? 0 : (t >= slice_len ? t - slice_len : t)); };
    auto past_slice = [&](const Place &c, int u) { return c.at + u >= slice_len; };

    // Operand fetches.  Every address below is a wave-uniform base (scalar registers, scalar
    // arithmetic) plus one per-lane byte offset that never changes (the lane's 16 bytes of a 1 KiB
    // block); every load is unconditional (indices are clamped instead): a load under a branch makes the
    // compiler's count of loads in flight inexact, and it then waits for all of them.
    // Activation chunk kc -> LDS stage: wave w fetches the 1 KiB blocks q = j NW + w, j < XB, of the chunk's
    // [2 planes][RT][KC] blocks (the last ones twice if they do not divide); row tiles past the end read the block's first.
    const unsigned x_lane = (unsigned)xtile_piece(lane, !SLICED || a0.rows > XTILE_ROWWISE) * 16u;     // LDS holds the block in lane order
    const unsigned w_lane = (unsigned)lane * 16u;
    auto fetch_x = [&](int kc, const Place &place, int stage, int j) {
        int q = j * NW + wave;
        q = q < 2 * RT * KC ? q : 2 * RT * KC - 1;
        const int pl = q / (RT * KC), t = (q % (RT * KC)) / KC, kk = q % KC;
        int k = kc * KC + kk;
        const unsigned nowhere = SLICED && past_slice(place, kk) ? BUFFER_NOWHERE : 0u;
        k = SLICED ? slice_step(place, kk) : (k < KSp ? k : KSp - 1);
        const int tt = t < n_rt ? t : 0;
        load_to_lds(pl ? xl : xh, x_lane + nowhere, (unsigned)(tt * KSp + k) * 1024u, xs + stage * CH + q * 64);
    };
    // weights of tile i, k-step k0 (u-th of its chunk): a 1 KiB block; a k-step past the end of K lies outside the descriptor: zeros
    auto fetch_w = [&](int k0, const Place &place, int u, int i) -> u32x4 {
        const unsigned off = SLICED ? (past_slice(place, u) ? BUFFER_NOWHERE : (unsigned)slice_step(place, u) * 1024u) : (unsigned)k0 * 1024u;
        return buffer_load16<SLICED>(wb[i], off + w_lane);
    };

    f32x4 acc[AT][RT];
#pragma unroll
    for (int i = 0; i < AT; ++i)
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[i][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    constexpr bool TOTAL = SLICED && AT > 1;            // several slices: their sums
    f32x4 total[AT][RT];
    bool first_slice = true;

    // split-K form (too few rows to fill the chip otherwise): blockIdx.y picks
    // one of a0.ksplit contiguous ranges of whole turns; the raw sums go to a0.part and a second kernel
    // adds the ranges in order and runs the epilogue
    const int n_split = a0.ksplit > 1 ? a0.ksplit : 1;
    const int turns = (KSp + PANEL_TURN - 1) / PANEL_TURN;
    const int kc_lo = SLICED ? 0 : (int)((long)turns * blockIdx.y / n_split) * (PANEL_TURN / KC);
    const int kc_hi = SLICED ? (n_slices * slice_len + PANEL_TURN - 1) / PANEL_TURN * (PANEL_TURN / KC) : (int)((long)turns * (blockIdx.y + 1) / n_split) * (PANEL_TURN / KC);
    u32x4 wreg[WD][AT];
    PN_TRACE(0, 63);
#pragma unroll
    for (int l = 0; l < 2 * XB; ++l) fetch_x(kc_lo + l / XB, place_of(l / XB), l / XB, l % XB);
    requests_stay_in_order();
#pragma unroll
    for (int j = 0; j < WD - KC; ++j)
#pragma unroll
        for (int i = 0; i < AT; ++i) wreg[j][i] = fetch_w(kc_lo * KC + j, place_of(j / KC), j % KC, i);
    PN_TRACE(1, 63);
    if (PARTIAL && a0.rstd_out != nullptr) {
        // the rows' sums of squares become rstd for the finishing kernel here, four rows at a time by the launch's waves
        // in turn, while the first operands are on their way
        const RstdShare s = rstd_share(p.tasks, NW, FT, RB, fb, rb, blockIdx.y, gridDim.y, wave);
        for (int r = s.first; r < a0.rows; r += s.step) rstd_of_row(a0.ssq_in, a0.ssq_tiles, a0.eps, a0.rstd_out, a0.rows, r + (lane >> 4), lane & 15);
    }
    // The MFMAs of a chunk run in groups of TB row tiles of one k-step; a group's operands come from LDS while the
    // group before it multiplies.
    constexpr int TG = Shape::TG, TB = Shape::TB, NG = KC * TG;
    u32x4 b[2][TB][2];
    auto read_group = [&](const u32x4 *xb, int g, u32x4 (&to)[TB][2]) {
#pragma unroll
        for (int t = 0; t < TB; ++t)
            if ((g % TG) * TB + t < RT) {
                const int at = (((g % TG) * TB + t) * KC + g / TG) * 64;
                to[t][0] = xb[at];
                to[t][1] = xb[CH / 2 + at];
            }
    };
    wait_loads_and_barrier<Shape::LATER>();
    read_group(xs + lane, 0, b[0]);
    int stage = 0;
    // One chunk.  Its first group's operands are in registers already.  During its groups the wave requests, one or two
    // at a time, the activations of the chunk after the next (into the stage of the previous chunk, which all waves
    // have read) and the weights WD - KC k-steps ahead (into the ring sets of the previous chunk).  Before the last group it waits for the
    // next chunk's activations -- requested during the previous chunk; behind them it has requested the weights of two chunks and one
    // chunk's activations --, meets the other waves, and reads the next chunk's first group.  (Requests past the end
    // of the range or of K are unused.)  The order is the source's: left alone, the compiler moves every request next to its use.
    auto chunk = [&](int kc, auto slot) {
        constexpr int c = decltype(slot)::value;        // chunk within the turn of the weight ring
        constexpr int REQ = XB + KC * AT;               // requests, all made before the last group
        const u32x4 *xb = xs + stage * CH + lane;
        const int prev = stage == 0 ? PANEL_STAGES - 1 : stage - 1, next = stage == PANEL_STAGES - 1 ? 0 : stage + 1;
        auto request = [&](int l) {
            const int u = (l - XB) / AT, i = (l - XB) % AT;
            if (l < XB) fetch_x(kc + 2, x_at, prev, l);
            else wreg[(c * KC + u + WD - KC) % WD][i] = fetch_w(kc * KC + u + WD - KC, w_at, u, i);
        };
        PN_TRACE(0, kc - kc_lo);
        requests_stay_in_order();
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) {
                read_group(xb, g + 1, b[(g + 1) & 1]);
            } else {
                PN_TRACE(1, kc - kc_lo);
                wait_loads_and_barrier<Shape::LATER>();
                PN_TRACE(2, kc - kc_lo);
                read_group(xs + next * CH + lane, 0, b[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int l = 0; l < REQ; ++l)
                if (l * (NG - 1) / REQ == g) { request(l); requests_stay_in_order(); }
            const int j = c * KC + g / TG;              // ring set of this k-step (a constant after unrolling)
#pragma unroll
            for (int t = 0; t < TB; ++t)
                if ((g % TG) * TB + t < RT)
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                        for (int i = 0; i < AT; ++i) {
                            f32x4 &ac = acc[i][(g % TG) * TB + t < RT ? (g % TG) * TB + t : 0];
                            ac = mfma16x16x32(wreg[j][i], b[g & 1][t][pl], ac);
                        }
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = next;
        if constexpr (SLICED) {
            next_chunk(x_at);
            next_chunk(w_at);
            in_slice += KC;
            if (AT > 1 && in_slice == slice_len) {      // (uniform; one tile per wave: one slice per workgroup)
                in_slice = 0;
#pragma unroll
                for (int i = 0; i < AT; ++i)
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
                        total[i][t] = first_slice ? acc[i][t] : total[i][t] + acc[i][t];
                        acc[i][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
                    }
                first_slice = false;
            }
        }
    };
    // (no way out of a turn: an early exit made the compiler copy the ring's registers at the end of every turn, behind
    // a wait for all loads in flight)
    for (int kc = kc_lo; kc < kc_hi; kc += WD / KC) {
        chunk(kc, std::integral_constant<int, 0>{});
        chunk(kc + 1, std::integral_constant<int, 1>{});
        chunk(kc + 2, std::integral_constant<int, 2>{});
        chunk(kc + 3, std::integral_constant<int, 3>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // nothing may still be on its way into LDS when the workgroup ends

    if constexpr (PARTIAL) {
        // partial sums as register images: [range][tile (gate/up: gate tiles, then up tiles)][row tile][lane]
        f32x4 *part = (f32x4 *)a0.part;
#pragma unroll
        for (int f = 0; f < AT; ++f)
#pragma unroll
            for (int t = 0; t < RT; ++t)
                if (task0 + f < p.tasks && rt0 + t < n_rt_total)
                    part[(((size_t)blockIdx.y * p.tasks + task0 + f) * n_rt_total + rt0 + t) * 64 + lane] = TOTAL ? total[f][t] : acc[f][t];
        PN_TRACE(2, 63);
        return;
    }
    // ---- epilogues, one feature tile (pair) at a time
    if constexpr (!PARTIAL)
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        const int task = task0 + f;
        if (task < p.tasks) {
            EpiIn<RT> in;
            epi_prefetch<RT, EPI>(a, p, task, lane, in);
            f32x4 sum[TILES][RT];
#pragma unroll
            for (int i = 0; i < TILES; ++i)
#pragma unroll
                for (int t = 0; t < RT; ++t) sum[i][t] = acc[f * TILES + i][t];
            gemm_epilogue<RT, EPI, TILES, true>(a, p, task, lane, sum, a0.rstd_in + r0, in);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Block GEMM (long prompt passes): like the panel GEMM without a split, but both operands pass through LDS and a wave owns 8 weight tiles x
// RT / 4 row tiles (2 x 4 waves per workgroup of 16 x RT tiles).  In the panel GEMM a read from LDS feeds two products, which keeps the LDS
// as busy as the matrix cores (per k-step of nine row tiles 1266 cycles of reads and fills beside 1152 of MFMA) and costs power, the bound of
// long prompts; here 16 reads feed 64 products (RT 16).  Gate/up of 7B at 2047 rows, inside a pass, 544 -> 507 us = 1.36 -> 1.46 PFLOP/s, of which the
// last round of workgroups leaves a tenth idle.  Which passes take it: block_height.
// A k-step's (16 + 2 RT) KB come straight into one of three LDS stages.  The groups of a k-step are its row tiles, 16 MFMAs each; the next group's
// activations are read during the present one, and the next k-step's weights replace the present ones during the last group, tile by
// tile behind the tile's last product.  The sums are added in the same order as the panel GEMM's: k-step after k-step, hi then lo.
// ---------------------------------------------------------------------------------------------
#define BLOCK_STAGES 3
// The blocks of a k-step: its 16 weight tiles (gate/up: four gates, four ups per wave group), then the row tiles of the activations' hi plane and of the
// lo plane.  Which of the workgroup's n_tasks tiles (pairs) or n_rt row tiles a block holds: places past the last one take the last weight tile's and the
// first row tile's operands, whose sums are not stored.  The tile goes into the load's scalar offset, which a descriptor's size need not
// bound: only tiles that exist may be asked for.
__host__ __device__ __forceinline__ int block_weight_tile(int q, int tiles_per_task, int n_tasks) {
    const int tile = tiles_per_task == 2 ? (q >> 3) * 4 + (q & 3) : q;
    return tile < n_tasks ? tile : n_tasks - 1;
}
__host__ __device__ __forceinline__ int block_row_tile(int x, int rt, int n_rt) {
    const int t = x < rt ? x : x - rt;
    return t < n_rt ? t : 0;
}
template <int RT, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_block_bf16(GemmArgs a0) {
    constexpr int TILES = (EPI == EPI_SWIGLU) ? 2 : 1, NW = 8, FT = 8, RW = RT / 4, PAIRS = 16 / TILES;
    constexpr int BLOCKS = 16 + 2 * RT, REQ = BLOCKS / NW;         // 1 KiB blocks per k-step, and how many of them a wave fetches
    static_assert(RT % 4 == 0 && BLOCKS % NW == 0, "");
    extern __shared__ u32x4 xs[];                  // [stages][16 weight tiles, then 2 planes x RT][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wf = wave & 1, wr = wave >> 1;       // the wave's eight weight tiles and its row tiles
    const GemmPlan &p = a0.plan;
    const int KSp = p.KSp;
    const int RB = a0.panel_rb;                    // (workgroup order: see the panel GEMM)
    const int grp = blockIdx.x / (8 * RB), within = blockIdx.x % (8 * RB);
    const int fb = grp * 8 + (within & 7), rb = within >> 3;
    if (fb * PAIRS >= p.tasks) return;
    const int rt0 = rb * RT;
    const int n_rt_total = (a0.rows + 15) / 16, n_rt = n_rt_total - rt0 < RT ? n_rt_total - rt0 : RT;

    // Descriptors: the block's weight tiles (gate/up: its gate tiles and its up tiles), its part of the two activation planes.
    const int n_tasks = p.tasks - fb * PAIRS < PAIRS ? p.tasks - fb * PAIRS : PAIRS;
    const unsigned w_bytes = (unsigned)n_tasks * (unsigned)KSp * 1024u, x_bytes = (unsigned)n_rt * (unsigned)KSp * 1024u;
    const char *const w0 = (const char *)a0.W + (size_t)fb * PAIRS * KSp * 1024;
    const rsrc_t wg = buffer_of(w0, w_bytes), wu = buffer_of(w0 + (TILES == 2 ? (size_t)p.tasks * KSp * 1024 : 0), w_bytes);
    const rsrc_t xh = buffer_of((const char *)a0.Xhi + (size_t)rt0 * KSp * 1024, x_bytes), xl = buffer_of((const char *)a0.Xlo + (size_t)rt0 * KSp * 1024, x_bytes);
    const unsigned w_lane = (unsigned)lane * 16u, x_lane = (unsigned)xtile_piece(lane, true) * 16u;
    auto fetch = [&](int k, int stage, int j) {                              // block q of a k-step
        const int q = j * NW + wave;
        u32x4 *const to = xs + (stage * BLOCKS + q) * 64;
        const unsigned at = (unsigned)(k < KSp ? k : KSp - 1) * 1024u;       // (requests past the end of K are unused)
        if (j < 16 / NW) {                                                   // (constant after unrolling)
            load_to_lds(TILES == 2 && (q & 4) ? wu : wg, w_lane, (unsigned)(block_weight_tile(q, TILES, n_tasks) * KSp) * 1024u + at, to);
        } else {
            const int x = q - 16;
            load_to_lds(x < RT ? xh : xl, x_lane, (unsigned)(block_row_tile(x, RT, n_rt) * KSp) * 1024u + at, to);
        }
    };
    f32x4 acc[FT][RW];
#pragma unroll
    for (int i = 0; i < FT; ++i)
#pragma unroll
        for (int t = 0; t < RW; ++t) acc[i][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int l = 0; l < 2 * REQ; ++l) fetch(l / REQ, l / REQ, l % REQ);
    u32x4 w[FT], b[2][2];
    auto read_w = [&](int stage, int i) { w[i] = xs[(stage * BLOCKS + wf * 8 + i) * 64 + lane]; };
    auto read_x = [&](int stage, int t, u32x4 (&to)[2]) {
        const u32x4 *const x = xs + (stage * BLOCKS + 16 + wr * RW + t) * 64 + lane;
        to[0] = x[0];
        to[1] = x[RT * 64];
    };
    wait_loads_and_barrier<REQ>();
#pragma unroll
    for (int i = 0; i < FT; ++i) read_w(0, i);
    read_x(0, 0, b[0]);
    int stage = 0;
    auto step = [&](int k, auto parity) {                // b[par]: the first group's operands of this k-step
        constexpr int par = decltype(parity)::value;
        const int prev = stage == 0 ? BLOCK_STAGES - 1 : stage - 1, next = stage == BLOCK_STAGES - 1 ? 0 : stage + 1;
        requests_stay_in_order();
#pragma unroll
        for (int t = 0; t < RW; ++t) {
            const bool last = t == RW - 1;
            if (!last) {
                read_x(stage, t + 1, b[(par + t + 1) & 1]);
            } else {
                wait_loads_and_barrier<REQ>();           // the next k-step's operands are there; the one after it is on its way
                read_x(next, 0, b[(par + t + 1) & 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            constexpr int GROUPS = RW > 1 ? RW - 1 : 1;
#pragma unroll
            for (int l = 0; l < REQ; ++l)
                if (l * GROUPS / REQ == t) { fetch(k + 2, prev, l); requests_stay_in_order(); }
#pragma unroll
            for (int i = 0; i < FT; ++i) {
                acc[i][t] = mfma16x16x32(w[i], b[(par + t) & 1][0], acc[i][t]);
                if (i % 2 == 1) {
                    acc[i - 1][t] = mfma16x16x32(w[i - 1], b[(par + t) & 1][1], acc[i - 1][t]);
                    acc[i][t] = mfma16x16x32(w[i], b[(par + t) & 1][1], acc[i][t]);
                    if (last) { read_w(next, i - 1); read_w(next, i); __builtin_amdgcn_sched_barrier(0); }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = next;
    };
    for (int k = 0; k < KSp; k += 2) {                   // (K / 32 is even: launch_panel_epi)
        step(k, std::integral_constant<int, 0>{});
        step(k + 1, std::integral_constant<int, RW & 1>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // nothing may still be on its way into LDS when the workgroup ends

    GemmArgs a = a0;
    const int r0 = (rt0 + wr * RW) * 16;
    offset_rows(a, p, r0);
    if (a.rows <= 0) return;
#pragma unroll
    for (int f = 0; f < FT / TILES; ++f) {
        const int task = fb * PAIRS + wf * (FT / TILES) + f;
        if (task < p.tasks) {
            EpiIn<RW> in;
            epi_prefetch<RW, EPI>(a, p, task, lane, in);
            f32x4 sum[TILES][RW];
#pragma unroll
            for (int i = 0; i < TILES; ++i)
#pragma unroll
                for (int t = 0; t < RW; ++t) sum[i][t] = acc[i * 4 + f][t];
            gemm_epilogue<RW, EPI, TILES, true>(a, p, task, lane, sum, a0.rstd_in + r0, in);
        }
    }
}

__global__ __launch_bounds__(256) void rstd_rows_kernel(const float *__restrict__ ssq, int ssq_tiles, float eps, float *__restrict__ rstd, int rows) {
    rstd_of_row(ssq, ssq_tiles, eps, rstd, rows, blockIdx.x * 16 + (threadIdx.x >> 4), threadIdx.x & 15);
}
void launch_rstd_rows(const float *ssq, int ssq_tiles, float eps, float *rstd, int rows, hipStream_t st) {
    hipLaunchKernelGGL(rstd_rows_kernel, dim3((rows + 15) / 16), dim3(256), 0, st, ssq, ssq_tiles, eps, rstd, rows);
}

// second half of the split-K form: one wave per (feature tile (pair), row tile) adds the ranges'
// partial sums in range order and runs the fused epilogue on the result
template <int EPI, bool QUADS>
__global__ __launch_bounds__(256) void gemm_splitk_finish_bf16(GemmArgs a0) {
    constexpr int TILES = (EPI == EPI_SWIGLU) ? 2 : 1;
    __shared__ float rstd_sh[4][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const GemmPlan &p = a0.plan;
    const int n_rt = (a0.rows + 15) / 16;
    const int unit = blockIdx.x * 4 + wave;
    if (unit >= p.tasks * n_rt) return;                         // (no workgroup barrier below)
    const int task = unit / n_rt, t = unit % n_rt;
    GemmArgs a = a0;
    offset_rows(a, p, t * 16);
    EpiIn<1> in;
    epi_prefetch<1, EPI>(a, p, task, lane, in);
    if (EPI != EPI_RESID && lane < 16) rstd_sh[wave][lane] = (lane < a.rows) ? a0.rstd_in[t * 16 + lane] : 0.f;
    const f32x4 *part = (const f32x4 *)a0.part;
    f32x4 sum[TILES][1];
#pragma unroll
    for (int i = 0; i < TILES; ++i) {
        const size_t tile = (size_t)(task + i * p.tasks) * n_rt + t, stride = (size_t)p.tasks * TILES * n_rt;
        f32x4 v[8];                                             // (at most 8 ranges; all requested before the first is added)
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = part[((s < a0.ksplit ? s : 0) * stride + tile) * 64 + lane];
        requests_stay_in_order();                               // (left alone, the compiler waits for two after two of them, and requests the epilogue's inputs last)
#pragma unroll
        for (int s = 1; s < 8; ++s)
            if (s < a0.ksplit) v[0] += v[s];
        sum[i][0] = v[0];
    }
    gemm_epilogue<1, EPI, TILES, QUADS>(a, p, task, lane, sum, rstd_sh[wave], in);
}
template <int EPI, bool QUADS = true>
static void launch_splitk_finish(const GemmArgs &a, hipStream_t st) {
    const int units = a.plan.tasks * ((a.rows + 15) / 16);
    hipLaunchKernelGGL((gemm_splitk_finish_bf16<EPI, QUADS>), dim3((units + 3) / 4), dim3(256), 0, st, a);
}

// feature blocks of PT weight tiles, padded to whole groups of 8 (see the kernel's workgroup order)
static int panel_feature_blocks(const GemmPlan &p, int pt) {
    const int per = pt / p.tiles_per_task;
    return ((p.tasks + per - 1) / per + 7) / 8 * 8;
}
// the split-K form sums every weight tile for itself (gate and up tiles meet in the finishing kernel)
static GemmPlan raw_plan(const GemmPlan &p) {
    GemmPlan q = p;
    q.tasks = p.tasks * p.tiles_per_task;
    q.tiles_per_task = 1;
    return q;
}
// How a launch over `rows` rows is cut: row tiles per workgroup, its waves and their weight tiles.  The times are a model of measured
// launches (7B and 13B shapes): a round of workgroups, one per compute unit (the padding of
// feature blocks counts: it keeps the work of a ragged group of 8 on some of the XCDs), costs 5 us to start and end, and a k-step what
// its operands take to come in -- 44 KB/us per compute unit, weights and activations alike, whatever the shape -- or the
// matrix cores under the card's power limit, 0.0056 us per pair of weight and row tile.  A split costs the finishing
// kernel, 5 us, and its partial sums once written and once read at 4 TB/s.
// So many workgroups as there are compute units is what counts: 12 weight tiles instead of 16 for gate/up of 7B (1376 tiles in two ranges)
// 48.5 -> 43.8 us at 54 rows, 61.3 -> 57.6 at 144, for QKV (768 in four) 32.5 -> 30.3 and 41.8 -> 40.2; 10 for down of 13B (320 in eight)
// 39.4 -> 34.2 at 54; 8 for O and down of 7B: 17.0 -> 15.9, 33.6 -> 27.4.  11 and 12 row tiles where one row block then holds all rows and
// the weights are read once: gate/up of 7B at 176 / 189 rows 76.5 / 78.3 (unsplit, two row blocks) -> 65.3 / 69.5, the one matrix of 7B, 13B and d 512 whose prompt passes
// take them; steps of 161 .. 192 rows, whose ranges are the matrix's own, do in most: at 161 / 177 rows QKV of 7B 50.4 / 51.4 -> 43.6 / 45.7, of 13B 64.4 / 65.5 ->
// 58.2 / 61.5, of d 2048 26.8 / 27.0 -> 25.2 / 26.3, down of 13B 60.0 / 61.2 -> 56.6 / 60.4, of d 6144 81 / 84 -> 69 / 72 (O of 13B 34.9 / 35.6 -> 33.4 / 35.7).  Not
// two blocks of 11 or 12 (340 .. 376 rows: 108 -> 119 .. 127), nor five or seven waves of that height, nor prompts' QKV of 13B in three ranges: 1 .. 5 % slower, hence the
// surcharge.  189 prompt rows: splits of 2 .. 8, 2.01 -> 0.98 ms for four layers; from 1535 rows on nothing is split.
struct PanelCut { int rt, nw, at; double us; };
static PanelCut panel_cut(const GemmPlan &p, int rows, int ns) {
    const int row_tiles = (rows + 15) / 16, turns = (p.KSp + PANEL_TURN - 1) / PANEL_TURN;
    const GemmPlan q = ns > 1 ? raw_plan(p) : p;
    PanelCut best{0, 0, 0, 0.0};
    auto consider = [&](int nw, int at) {
        const int pt = nw * at;
        for (int rt = 4; rt <= (at == 1 ? 5 : (ns > 1 && nw == 6 && row_tiles <= PANEL_RT_SPLIT ? PANEL_RT_SPLIT : PANEL_RT_MAX)); ++rt) {
            const bool tall = rt > PANEL_RT_MAX;
            if (tall && rt < row_tiles) continue;
            const long groups = (long)panel_feature_blocks(q, pt) * ((row_tiles + rt - 1) / rt) * ns, rounds = (groups + cu_count() - 1) / cu_count();
            const double in = (pt + 2 * rt) / 44.0, multiply = 0.0056 * pt * rt;
            const double us = (tall ? 1.06 : 1.0) * (double)rounds * (5.0 + (double)((turns + ns - 1) / ns) * PANEL_TURN * (in > multiply ? in : multiply));
            if (best.rt == 0 || us <= best.us) best = PanelCut{rt, nw, at, us};        // (ties: fewer, taller row blocks stream the weights less often)
        }
    };
    consider(8, 2);
    if (ns > 1) { consider(7, 2); consider(6, 2); consider(5, 2); }
    if (q.tiles_per_task == 1) consider(8, 1);
    return best;
}
size_t panel_part_bytes(const GemmPlan &p, int rows, int ns) { return ns > 1 ? (size_t)ns * p.tasks * p.tiles_per_task * ((rows + 15) / 16) * 1024 : 0; }
int panel_prompt_split(const GemmPlan &p, int rows) {
    int best = 1;
    double best_us = 0.0;
    for (int ns = 1; ns <= 8 && ns <= (p.KSp + PANEL_TURN - 1) / PANEL_TURN; ++ns) {
        const double us = panel_cut(p, rows, ns).us + (ns > 1 ? 5.0 + 2e-6 * (double)panel_part_bytes(p, rows, ns) / 4.0 : 0.0);
        if (best_us == 0.0 || us < 0.97 * best_us) { best = ns; best_us = us; }      // (a split has to promise 3 %: one more that promised 1 lost 6 in a prompt of 900 tokens at d 512)
    }
    return best;
}

template <int RT, int EPI, int AT, int NW>
static void launch_panel_cfg(const GemmArgs &a, hipStream_t st) {
    const size_t lds = (size_t)PANEL_STAGES * 2 * RT * PANEL_KC * 1024;
    GemmArgs a2 = a;
    if (EPI == EPI_RAW || EPI == EPI_SLICES) a2.plan = raw_plan(a.plan);
    else a2.rstd_out = nullptr;
    const int FB = panel_feature_blocks(a2.plan, NW * AT);
    a2.panel_rb = (a.rows + 16 * RT - 1) / (16 * RT);
    dim3 grid(FB * a2.panel_rb, a.ksplit > 1 ? a.ksplit : 1), block(NW * 64);
    static std::atomic<uint64_t> done{0};
    allow_full_lds((const void *)gemm_panel_bf16<RT, EPI, AT, NW>, done);
    hipLaunchKernelGGL((gemm_panel_bf16<RT, EPI, AT, NW>), grid, block, lds, st, a2);
}
// (any height is carried out: beyond the tallest form of these waves in that one)
template <int EPI, int AT, int NW>
static void launch_panel_rt(int rt, const GemmArgs &a, hipStream_t st) {
    if (rt <= 4) { launch_panel_cfg<4, EPI, AT, NW>(a, st); return; }
    if constexpr (AT == 1) {
        launch_panel_cfg<5, EPI, AT, NW>(a, st);
    } else {
        if constexpr (NW == 6 && EPI == EPI_RAW)
            if (rt > PANEL_RT_MAX) {
                if (rt == 11) launch_panel_cfg<11, EPI, AT, NW>(a, st);
                else launch_panel_cfg<12, EPI, AT, NW>(a, st);
                return;
            }
        switch (rt) {
            case 5: launch_panel_cfg<5, EPI, AT, NW>(a, st); break;
            case 6: launch_panel_cfg<6, EPI, AT, NW>(a, st); break;
            case 7: launch_panel_cfg<7, EPI, AT, NW>(a, st); break;
            case 8: launch_panel_cfg<8, EPI, AT, NW>(a, st); break;
            case 9: launch_panel_cfg<9, EPI, AT, NW>(a, st); break;
            default: launch_panel_cfg<10, EPI, AT, NW>(a, st); break;
        }
    }
}
// Rounds of workgroups, one per compute unit, on the busiest XCD -- feature blocks of 16 weight tiles go round the eight of them, a block's row
// blocks stay on one -- and the share of all compute units that the last of them keeps busy.
struct Rounds { int n; double last; };
static Rounds panel_rounds(const GemmPlan &p, int row_blocks) {
    const int per = 16 / p.tiles_per_task, blocks = (p.tasks + per - 1) / per, units = cu_count() / 8 > 0 ? cu_count() / 8 : 1;
    auto on = [&](int xcd) { return (blocks + 7 - xcd) / 8 * row_blocks; };
    Rounds r{(on(0) + units - 1) / units, 0.0};
    for (int x = 0; x < 8; ++x) r.last += on(x) > units * (r.n - 1) ? (double)(on(x) - units * (r.n - 1)) / (8 * units) : 0.0;
    return r;
}
// Which passes without a split take the block GEMM, and in which height (0: the panel GEMM).  Both are priced alike, in us per pair of weight and row tile:
// a k-step takes what the matrix cores do under the card's power limit (0.0056 with seven row tiles in the panel GEMM, where fewer
// wait for operands; 0.0052 / 0.00505 in blocks of 12 / 16), in the last round down to two thirds of it, as compute units idle and the
// clock rises; every round ends with its epilogue, which nothing overlaps (gate/up writes half the outputs); 5 us to start and end.
// Fitted to 978 launches in each form inside prompt passes of 320 .. 2048 rows (every 16 or 32, the forms in turn; d 512, 2048, 3072, 7B and 13B): error
// 2.4 % rms, largely the same for both forms of a case.  With 3 % to be gained none of them is slower than in the panel GEMM, nor are
// those of four shapes that were not fitted (d 1600, 2560, 6144, 8192); the model before (launches back to back, the chip as a whole) took 84 of them to blocks that were
// 1 .. 15 % slower.  us panel / 12 / 16: gate/up of 7B 431 rows 143 / 236 / 164, 847 247 / 261 / 322, 1327 375 / 383 / 482 (stay), 1536 425 / 401 / 487,
// 2048 564 / 536 / 513; of 13B 512 219 / 295 / 202, 1103 453 / 463 / 591, 1792 709 / 781 / 795 (stay), 1711 705 / 642 / 787; QKV of 7B 911 166 / 156 / 192, 1679
// 281 / 298 / 357 (stays), 1920 320 / 304 / 368; of 13B 847 229 / 321 / 239 (stays), 1024 258 / 332 / 240, 2048 512 / 538 / 474; O of 13B 1664 174 / 177 / 216 (stays),
// 1792 190 / 182 / 214, 2016 201 / 317 / 229 (stays).  O and down of 7B (16 feature blocks) stay: 98 .. 114 / 120 .. 138 / 152 .. 170 and 230 .. 263 / 292 .. 305 / 373 .. 379.
static int block_height(const GemmPlan &p, int rows, const PanelCut &cut) {
    if (p.KSp % 2 != 0 || p.KSp > 65536) return 0;               // (two k-steps per turn; 32-bit offsets inside a block's operands)
    if (p.block_rt >= 0) return p.block_rt;
    if (cut.nw * cut.at != 16) return 0;                         // (8 tiles per workgroup: few workgroups as it is)
    const int row_tiles = (rows + 15) / 16;
    auto price = [&](int rt, double step_us) {
        const Rounds r = panel_rounds(p, (row_tiles + rt - 1) / rt);
        return 5.0 + 16.0 * rt * (p.KSp * step_us * (r.n - 1 + 0.66 + 0.34 * r.last) + (p.tiles_per_task == 2 ? 0.03 : 0.13) * r.n);
    };
    static const double panel_us[] = {0.0067, 0.0061, 0.0057, 0.0056, 0.0055, 0.0055, 0.0055};      // 4 .. 10 row tiles
    static_assert(sizeof panel_us / sizeof *panel_us == PANEL_RT_MAX - 3, "");
    double best_us = 0.97 * price(cut.rt, panel_us[cut.rt - 4]);
    int best = 0;
    const double b12 = price(12, 0.0052), b16 = price(16, 0.00505);
    if (b12 < best_us) { best = 12; best_us = b12; }
    if (b16 < best_us) best = 16;
    return best;
}
template <int RT, int EPI>
static void launch_block_cfg(const GemmArgs &a, hipStream_t st) {
    GemmArgs a2 = a;
    a2.panel_rb = (a.rows + 16 * RT - 1) / (16 * RT);
    const dim3 grid(panel_feature_blocks(a.plan, 16) * a2.panel_rb);
    static std::atomic<uint64_t> done{0};
    allow_full_lds((const void *)gemm_block_bf16<RT, EPI>, done);
    hipLaunchKernelGGL((gemm_block_bf16<RT, EPI>), grid, dim3(512), (size_t)BLOCK_STAGES * (16 + 2 * RT) * 1024, st, a2);
}
template <int EPI>
static void launch_panel_epi(const GemmArgs &a, hipStream_t st) {
    const PanelCut cut = panel_cut(a.plan, a.rows, a.ksplit > 1 ? a.ksplit : 1);
    if (a.ksplit > 1) {
        if (cut.at == 1) launch_panel_rt<EPI_RAW, 1, 8>(cut.rt, a, st);
        else if (cut.nw == 8) launch_panel_rt<EPI_RAW, 2, 8>(cut.rt, a, st);
        else if (cut.nw == 7) launch_panel_rt<EPI_RAW, 2, 7>(cut.rt, a, st);
        else if (cut.nw == 6) launch_panel_rt<EPI_RAW, 2, 6>(cut.rt, a, st);
        else launch_panel_rt<EPI_RAW, 2, 5>(cut.rt, a, st);
        launch_splitk_finish<EPI>(a, st);
        return;
    }
    if constexpr (EPI != EPI_LMHEAD) {                           // (the LM head runs in steps only)
        const int rt = block_height(a.plan, a.rows, cut);
        if (rt == 16) { launch_block_cfg<16, EPI>(a, st); return; }
        if (rt == 12) { launch_block_cfg<12, EPI>(a, st); return; }
    }
    if constexpr (EPI != EPI_SWIGLU)
        if (cut.at == 1) { launch_panel_rt<EPI, 1, 8>(cut.rt, a, st); return; }
    launch_panel_rt<EPI, 2, 8>(cut.rt, a, st);
}
void launch_gemm_panel_bf16(const GemmArgs &a, hipStream_t st) {
    switch (a.epi) {
        case EPI_RESID: launch_panel_epi<EPI_RESID>(a, st); break;
        case EPI_SWIGLU: launch_panel_epi<EPI_SWIGLU>(a, st); break;
        case EPI_QKV: launch_panel_epi<EPI_QKV>(a, st); break;
        default: launch_panel_epi<EPI_LMHEAD>(a, st); break;
    }
}

// O and down projection of steps of 17 .. 48 rows, in slices: workgroups of 8 tiles take one of the tile-K kernel's K slices
// each, their activations through LDS, and the finishing kernel adds the slices in the same order: the same sums, bit for bit.
// The tile-K kernel has one or two tiles per workgroup there, and every workgroup reads all activations: what comes in
// per compute unit -- 37 .. 59 KB/us, weights and activations alike -- is mostly activations (down of 7B at 33 rows: 372 MB beside
// 90 of weights; in slices 45).  7B down 17 / 33 / 48 rows 25.9 / 35.2 / 40.8 -> 22.3 / 24.4 / 24.4 us, 13B 39.6 / 52.8 / 59.0 ->
// 36.9 / 41.3 / 41.4.  It costs a second launch, 4 us: O of 7B 11.6 -> 13.7 at 17 rows, 14.7 -> 15.3 at 33, 16.6 -> 15.4 at 48, of 13B 22.3 ->
// 23.3 at 33, down at d 512 (K 2048) 9.7 -> 9.1 at 48: from 700 KB of activations per workgroup on it pays.
// Generation launches (rows_live) stay: mostly one of their rows is live, and then the launch counts.
//
// QKV and the LM head have 16 slices: a workgroup takes a group of them (tilek_groups) and 12 or 16 tiles, two per wave.  They pay
// where the tile-K kernel cannot take the matrix in one round of workgroups (more than four tiles each, or more partial sums
// than LDS holds): LM head of 7B at 17 / 32 / 33 / 48 rows 55 / 61 / 85 / 97 -> 50 / 50 / 54 / 53 us, of 13B 59 / 69 / 105 / 117 -> 58 / 58 / 60 / 60;
// QKV of 13B at 33 / 48 rows 53 / 59 -> 45; where one round does (QKV of 7B, three tiles) it is 29.7 against 28.4 at 33 rows.
template <int EPI, int AT, int NW>
static void launch_slices_rt(const GemmArgs &a, hipStream_t st) {
    static_assert(tilek_turn_group(EPI) % (AT * NW) == 0, "one start of the walk for a workgroup's tiles");
    if (a.rows <= 32) launch_panel_cfg<2, EPI_SLICES, AT, NW>(a, st);
    else launch_panel_cfg<3, EPI_SLICES, AT, NW>(a, st);
    if (a.rows <= XTILE_ROWWISE) launch_splitk_finish<EPI, false>(a, st);
    else launch_splitk_finish<EPI, true>(a, st);
}
static void launch_gemm_slices(const GemmArgs &a, hipStream_t st) {
    GemmArgs a2 = a;
    const bool grouped = a.epi != EPI_RESID;
    a2.ksplit = grouped ? tilek_groups(a.plan) : a.plan.tk_waves;
    if (!grouped) a2.rstd_out = nullptr;
    if (a.epi == EPI_RESID) launch_slices_rt<EPI_RESID, 1, 8>(a2, st);
    else if (a.epi == EPI_QKV) launch_slices_rt<EPI_QKV, 2, 6>(a2, st);
    else launch_slices_rt<EPI_LMHEAD, 2, 8>(a2, st);
}
static bool slices_pay(const GemmArgs &a) {
    if (a.part == nullptr || a.rows_live != nullptr || !a.split) return false;
    const GemmPlan &p = a.plan;
    if (a.epi == EPI_RESID) return p.tk_waves == 8 && (long)a.rows * p.K * 4 >= 700000;
    if (a.epi == EPI_SWIGLU || tilek_groups(p) == 1) return false;
    const int one_round = (p.tasks + cu_count() - 1) / cu_count(), nt = (a.rows + 15) / 16;
    return !tilek_ft_valid(p, nt, one_round);
}

// decoding-step GEMM: one launch for up to 48 rows (three row tiles).  More rows are refused (false,
// nothing launched): every workgroup re-reads all rows' operands, so larger steps belong to the panel
// kernel, and processing them here in blocks would stream the weights once per block.
bool launch_gemm_bf16(const GemmArgs &a, hipStream_t st) {
    if (a.rows < 1 || a.rows > 48) return false;
    if (a.rows <= 16) launch_gemm_nt<1>(a, st);
    else if (slices_pay(a)) launch_gemm_slices(a, st);
    else if (a.rows <= 32) launch_gemm_nt<2>(a, st);
    else launch_gemm_nt<3>(a, st);
    return true;
}

// how a [N][K] weight matrix is cut into work
GemmPlan make_gemm_plan(int N, int K, int tiles_per_task) {
    GemmPlan p;
    p.N = N; p.K = K;
    p.KSp = K / 32;
    p.tasks = N / 16;
    // tile-K kernel, K slices: 16 for matrices of 640+ tiles (QKV, LM head), else 8; feature tiles per workgroup by
    // tilek_ft_default, re-tuned per context by timing (llma_create), which cannot change any result
    p.tiles_per_task = tiles_per_task;
    p.tk_waves = (tiles_per_task != 2 && p.tasks >= 640) ? 16 : 8;
    for (int nt = 1; nt <= 3; ++nt) p.tk_ft[nt - 1] = tilek_ft_default(p, nt, false);
    p.tk_ft[3] = tilek_ft_default(p, 1, true);
    // split-K form of the panel kernel: enough ranges that feature blocks x ranges is about 200
    // workgroups per row block (2..8, a function of the matrix only, so a row's sums do not depend on
    // how many rows share the step)
    const int fb = (p.tasks + (tiles_per_task == 2 ? 8 : 16) - 1) / (tiles_per_task == 2 ? 8 : 16);
    int ns = (192 + fb / 2) / fb;
    ns = ns < 2 ? 2 : (ns > 8 ? 8 : ns);
    const int turns = (p.KSp + PANEL_TURN - 1) / PANEL_TURN;
    p.n_split = ns < turns ? ns : (turns > 0 ? turns : 1);
    p.block_rt = -1;
    return p;
}

// Keeps the loads written above this point above it: the compiler may not sink a load into the
// branch that uses its value past something that could write memory.  No value is consumed here,
// so nothing waits.  Used where many loads must be in flight before a dependent value (the
// sequence length) arrives.
__device__ __forceinline__ void loads_stay_above() { asm volatile("" ::: "memory"); }

// ---- softmax arithmetic of the attention kernels.  Scores stay as they come out of the products; row maxima (and everything that is
// exchanged about them) are powers of two, so a probability is one fused multiply-add and one exp2.
#define LOG2E 1.44269504088896341f
// e^(scale s) / 2^m; m = -inf (nothing visible so far): the score is -inf too, and the result zero
__device__ __forceinline__ float attn_exp(float s, float to_log2, float m) {
    return __builtin_amdgcn_exp2f(fmaf(s, to_log2, m == LLMA_NEG_INF ? 0.f : -m));
}
// a lane's scores of eight positions, first .. first + 3 and first + 16 .. first + 19, and of its row: the largest over the lanes of the row
// (32 positions).  masked (uniform): positions past the row's own are taken out first
__device__ __forceinline__ float attn_mask_max(float (&sv)[8], bool masked, int first, int row_pos) {
    if (masked)
#pragma unroll
        for (int i = 0; i < 8; ++i) sv[i] = first + (i >> 2) * 16 + (i & 3) > row_pos ? LLMA_NEG_INF : sv[i];
    float mx = sv[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sv[i]);
    mx = fmaxf(mx, lane_xor<16>(mx));
    return fmaxf(mx, lane_xor<32>(mx));
}
// Running (reference, sum, O) of a row: the reference moves only when a maximum passes it by 2^ATTN_REBASE (sums of terms up to that lose
// nothing in fp32), so after the first positions the accumulators are hardly ever rescaled.  A row's decision is its own: rows beside it
// that move make it multiply by one.
#define ATTN_REBASE 8.f
template <int DT>
__device__ __forceinline__ void attn_rebase(float mx, float &m, float &l, f32x4 (&o)[DT]) {
    if (__ballot(mx > m + ATTN_REBASE) == 0ull) return;             // uniform
    const float m_new = mx > m + ATTN_REBASE ? mx : m;
    const float alpha = m_new == LLMA_NEG_INF ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
    l *= alpha;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
    m = m_new;
}

// =============================================================================================
// causal attention of m <= 16*NTQ query rows of one sequence over its KV cache
// =============================================================================================
// grid = (chunks of ATTN_CHUNK key positions, heads, sequences); 4 waves per workgroup, wave w
// owns the 32 positions [32 w, 32 w + 32) of the chunk and issues all of their K and V loads
// (whole 1 KiB blocks) before any arithmetic.  S^T = K_tile . Q^T (MFMA, keys on the A side;
// with hi/lo planes S = Khi.qhi + Khi.qlo + Klo.qhi), scale, causal mask by absolute position,
// softmax statistics per query row, O^T = V^T . P^T (again hi/lo).  The four waves' (max, sum, O)
// are merged in wave order, and the chunk's partial is written for the combine kernel.  Which
// keys a row sees, and in which order they are reduced, is a function of absolute positions only.
// COMPACT (three row tiles, at most ATTN_COMPACT_ROWS rows: the 33 rows per sequence of k = 32): the
// merge buffer holds only that many rows, every row tile is published as soon as it is done (one
// tile of accumulators in registers at a time) and the registers are capped, so that two workgroups
// fit a compute unit like they do with one or two row tiles (7B, 33 rows over 3500 positions: 38.1 -> 30.8 us).
#define ATTN_COMPACT_ROWS 36
// (Several chunks per workgroup, the next one requested while one is computed, where there are more than fit the chip at once:
// no gain at 1 .. 33 rows over 2700 and 3500 positions.)
template <int DH, int NTQ, bool KVS, bool LIVE, bool COMPACT>
__device__ __forceinline__ void attn_chunk_body(const AttnArgs &a, float (&sm)[4][NTQ * 16], float (&sl)[4][NTQ * 16],
                                                 float (&so)[4][COMPACT ? ATTN_COMPACT_ROWS : NTQ * 16][DH + 4]) {
    constexpr int KSTEPS = DH / 32;   // MFMA k-steps of a q.k dot product
    constexpr int DT = DH / 16;       // 16-feature tiles of the head dimension
    constexpr int RQ = NTQ * 16;
    constexpr int OQ = COMPACT ? 1 : NTQ;                      // row tiles of accumulators held at once

    const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z / a.n_rblocks, rb = blockIdx.z % a.n_rblocks;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int slot = a.slot_const >= 0 ? a.slot_const : a.batch_slots[b];
    const int m = a.m;
    const int j0 = rb * RQ;                             // first row of this row block
    const int d_model = a.H * DH;
    const size_t head_base = ((size_t)slot * a.H + h) * (size_t)a.max_seq * DH;
    // The sequence length and the live-row count are requested first and used last: both requests
    // are in flight together with the K/V blocks instead of one after the other behind them.
    const int T = a.T[slot];
    const int live_rows = LIVE ? *a.rows_live + 1 : m;
    loads_stay_above();
    // K and V blocks of the wave's 32 positions: requested before the sequence length is known (any
    // position below max_seq lies inside the cache allocation; unused blocks are simply dropped)
    u32x4 ka[2][KSTEPS], va[DT];
    u32x2 kb[2][KSTEPS], vb[DT];                     // lo planes: one byte per element
    // query operands of a row tile: they do not depend on the sequence length either.  With more row tiles the
    // next one's take the registers behind the present one's scores (requested where they are used, each tile waited for its own: 33 rows
    // over 2700 / 3500 positions 32.2 / 36.0 -> 26.1 / 31.2 us with the combine kernel)
    u32x4 qh[KSTEPS], ql[KSTEPS];
    const unsigned q_bytes = (unsigned)((a.n_seqs * m + 15) / 16) * (unsigned)d_model * 32;      // (at most 48 rows of a sequence, or 48 in all: launch_attn_dh)
    const rsrc_t qhr = buffer_of(a.Qhi, q_bytes), qlr = buffer_of(a.Qlo, q_bytes);
    auto fetch_q = [&](int q) {
        const int j = j0 + q * 16 + n;
        const unsigned at = (unsigned)xtile_off(b * m + (j < m ? j : 0), h * DH + g * 8, d_model / 32, a.quads) * 2;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {                  // (a k-step further: the next 1 KiB block)
            qh[s] = buffer_load16<false>(qhr, at + s * 1024);
            ql[s] = buffer_load16<false>(qlr, at + s * 1024);
        }
    };
    {
        const size_t first = head_base + (size_t)(c * ATTN_CHUNK + wave * 32) * DH + lane * 8;
        const bf16_t *kh = (const bf16_t *)a.Khi + first, *vh = (const bf16_t *)a.Vhi + first;
        const uint8_t *kl = (const uint8_t *)a.Klo + first, *vl = (const uint8_t *)a.Vlo + first;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                ka[t][s] = *(const u32x4 *)(kh + t * (16 * DH) + s * 512);
                if (KVS) kb[t][s] = *(const u32x2 *)(kl + t * (16 * DH) + s * 512);
            }
        fetch_q(0);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            va[dt] = *(const u32x4 *)(vh + dt * 512);
            if (KVS) vb[dt] = *(const u32x2 *)(vl + dt * 512);
        }
    }
    loads_stay_above();
    // generation steps: rows past the trigger's draft count are padding (see the GEMM); they are
    // masked like rows past m and a row tile made of them only is skipped
    const int m_live = live_rows < m ? live_rows : m;     // LIVE: rows_live is set
    if (j0 >= m_live) return;
    const int m_blk = (m_live - j0 < RQ) ? m_live - j0 : RQ;   // live rows of this block
    const int kv_len = T + j0 + m_blk;                  // positions the block's last row can see

    const float to_log2 = a.scale * LOG2E;              // scores stay as the products leave them, maxima are powers of two (see attn_exp)
    float mrow[NTQ], lrow[NTQ];
    f32x4 o[OQ][DT];
    // every wave publishes (max, sum, O) of a row tile for the merge below
    auto publish = [&](int q, const f32x4 (&oq)[DT]) {
        float l = lrow[q];
        l += lane_xor<16>(l);
        l += lane_xor<32>(l);
        if (g == 0) { sm[wave][q * 16 + n] = mrow[q]; sl[wave][q * 16 + n] = l; }
        if (!COMPACT || q * 16 + n < ATTN_COMPACT_ROWS)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) *(f32x4 *)&so[wave][q * 16 + n][dt * 16 + 4 * g] = oq[dt];
    };
    const int chunk0 = c * ATTN_CHUNK, key0 = chunk0 + wave * 32;
    if (chunk0 >= kv_len) return;                   // uniform for the workgroup
    const bool active = key0 < kv_len;              // uniform for the wave
    const bool masked = key0 + 31 > T + j0;         // uniform: some row may not see all of these positions
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        mrow[q] = LLMA_NEG_INF;
        lrow[q] = 0.f;
    }
#pragma unroll
    for (int q = 0; q < OQ; ++q)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[q][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (COMPACT && !active) {
#pragma unroll
        for (int q = 0; q < NTQ; ++q) publish(q, o[0]);     // (zeros)
    }
    if (active) {
#pragma unroll
        for (int q = 0; q < NTQ; ++q) {
            const int oi = COMPACT ? 0 : q;
            const bool dead = LIVE && q > 0 && j0 + q * 16 >= m_live;       // uniform: no live row in this tile
            const int j = j0 + q * 16 + n;
            const int rpos = j < m_live ? T + j : -1;
            float sv[8];
            float mx = LLMA_NEG_INF;
            if (!dead) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < KSTEPS; ++s) {
                        acc = mfma16x16x32(ka[t][s], qh[s], acc);
                        acc = mfma16x16x32(ka[t][s], ql[s], acc);
                        if (KVS) acc = mfma16x16x32(lo8_operand(kb[t][s]), qh[s], acc);
                    }
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) sv[t * 4 + r4] = acc[r4];
                }
            }
            if (q < NTQ - 1) fetch_q(q + 1);
            if (!dead) {
                mx = attn_mask_max(sv, masked, key0 + 4 * g, rpos) * to_log2;
                float psum = 0.f;
                float p[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    p[i] = attn_exp(sv[i], to_log2, mx);
                    psum += p[i];
                }
                lrow[q] = psum;
                mrow[q] = mx;
                u32x2 h0, l0, h1, l1;
                split4(p, h0, l0);
                split4(p + 4, h1, l1);
                const u32x4 ph = (u32x4){h0[0], h0[1], h1[0], h1[1]};
                const u32x4 pl = (u32x4){l0[0], l0[1], l1[0], l1[1]};
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    o[oi][dt] = mfma16x16x32(va[dt], ph, o[oi][dt]);
                    o[oi][dt] = mfma16x16x32(va[dt], pl, o[oi][dt]);
                    if (KVS) o[oi][dt] = mfma16x16x32(lo8_operand(vb[dt]), ph, o[oi][dt]);
                }
            }
            if (COMPACT) {
                publish(q, o[0]);                           // (a dead tile: zeros)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) o[0][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
    }

    // ---- merge the four waves in wave order: every wave publishes (max, sum, O), then all
    //      threads add the four contributions e^{m_w - M} O_w of an output element in wave order
    if (!COMPACT) {
#pragma unroll
        for (int q = 0; q < NTQ; ++q) publish(q, o[COMPACT ? 0 : q]);
    }
    __syncthreads();
    const size_t pbase = (((size_t)b * a.H + h) * a.n_chunks + c) * ((size_t)a.n_rblocks * RQ) + j0;
    for (int idx = threadIdx.x; idx < m_blk * (DH / 4); idx += 256) {
        const int j = idx / (DH / 4), d4 = idx % (DH / 4);
        float M = LLMA_NEG_INF;
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, sm[w][j]);
        f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = sm[w][j];
            const float sc = (mw == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(mw - M);
            acc += *(const f32x4 *)&so[w][j][d4 * 4] * sc;
        }
        *(f32x4 *)(a.po + (pbase + j) * DH + d4 * 4) = acc;
    }
    if (threadIdx.x < m_blk) {
        int j = threadIdx.x;
        float M = LLMA_NEG_INF;
        for (int w = 0; w < 4; ++w) M = fmaxf(M, sm[w][j]);
        float L = 0.f;
        for (int w = 0; w < 4; ++w) {
            float mw = sm[w][j];
            L += (mw == LLMA_NEG_INF) ? 0.f : sl[w][j] * __builtin_amdgcn_exp2f(mw - M);
        }
        a.pm[pbase + j] = M;
        a.pl[pbase + j] = L;
    }
}

// LOSKIP (batched steps on caches with hi + lo planes): positions below lo_from[slot] were imported
// as bf16 values -- their lo planes hold zeros -- so a chunk that lies entirely below it runs the
// single-plane form of the body: half the K/V bytes, the same sums (the skipped terms are zeros).
template <int DH, int NTQ, bool KVS, bool LIVE, bool LOSKIP, bool COMPACT>
__global__ __launch_bounds__(256, 2) void attn_bf16_kernel(AttnArgs a) {
    constexpr int RQ = NTQ * 16;
    __shared__ float sm[4][RQ], sl[4][RQ];
    __shared__ float so[4][COMPACT ? ATTN_COMPACT_ROWS : RQ][DH + 4];
    if (KVS && LOSKIP) {
        const int slot = a.slot_const >= 0 ? a.slot_const : a.batch_slots[blockIdx.z / a.n_rblocks];
        if ((int)(blockIdx.x + 1) * ATTN_CHUNK <= a.lo_from[slot]) {     // uniform for the workgroup
            attn_chunk_body<DH, NTQ, false, LIVE, COMPACT>(a, sm, sl, so);
            return;
        }
    }
    attn_chunk_body<DH, NTQ, KVS, LIVE, COMPACT>(a, sm, sl, so);
}

// ---------------------------------------------------------------------------------------------
// Wide batched steps (several sequences, more than 48 rows in all; their GEMMs already add in an
// order of their own): a workgroup walks ATTN_WALK_CHUNKS consecutive chunks of one (sequence, head)
// instead of one.  Every chunk is computed like above -- four waves x 32 positions, all K/V blocks of
// the chunk requested at once, (max, sum, O) per wave merged through LDS in wave order -- and the merged
// chunk is folded into a running (max, sum, O) held in registers, in chunk order; one partial per
// walk goes to the combine kernel.  Four times fewer workgroups, partials and combine work than one
// chunk per workgroup (16 sequences x 4096 positions: 16384 -> 4096 workgroups per layer).  Chunks
// that lie entirely below lo_from[slot] (imported bf16 caches: all-zero lo planes) skip the lo planes.
// ---------------------------------------------------------------------------------------------
#define ATTN_WALK_CHUNKS 4
template <int DH, int NTQ, bool KVS>
__global__ __launch_bounds__(256, 2) void attn_walk_bf16_kernel(AttnArgs a) {
    constexpr int KSTEPS = DH / 32, DT = DH / 16;
    constexpr int RQ = NTQ * 16;
    constexpr int RS = (NTQ == 3) ? ATTN_COMPACT_ROWS : RQ;          // rows the merge buffer holds (a step has at most 33 per sequence)
    constexpr int OWN = (RS * (DH / 4) + 255) / 256;                  // merged output elements (float4) per thread
    __shared__ float sm[4][RQ], sl[4][RQ];
    __shared__ float so[4][RS][DH + 4];
    const int h = blockIdx.y, b = blockIdx.z / a.n_rblocks, rb = blockIdx.z % a.n_rblocks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int slot = a.batch_slots[b];
    const int T = a.T[slot];
    const int lo_from = (KVS && a.lo_from != nullptr) ? a.lo_from[slot] : 0;
    const int m = a.m, j0 = rb * RQ;
    if (j0 >= m) return;
    const int m_blk = (m - j0 < RQ) ? m - j0 : RQ;
    const int kv_len = T + j0 + m_blk;                               // positions the block's last row can see
    const int c0 = blockIdx.x * ATTN_WALK_CHUNKS;
    if (c0 * ATTN_CHUNK >= kv_len) return;                           // uniform for the workgroup
    const int c_need = (kv_len + ATTN_CHUNK - 1) / ATTN_CHUNK;
    const int c1 = c0 + ATTN_WALK_CHUNKS < c_need ? c0 + ATTN_WALK_CHUNKS : c_need;
    // chunks below c_lo lie entirely inside an imported bf16 cache: single plane
    int c_lo = KVS ? lo_from / ATTN_CHUNK : c1;
    c_lo = c_lo < c0 ? c0 : (c_lo > c1 ? c1 : c_lo);
    const int d_model = a.H * DH;
    const size_t head_base = ((size_t)slot * a.H + h) * (size_t)a.max_seq * DH;
    const bf16_t *kh = (const bf16_t *)a.Khi + head_base; const uint8_t *kl = (const uint8_t *)a.Klo + head_base;
    const bf16_t *vh = (const bf16_t *)a.Vhi + head_base; const uint8_t *vl = (const uint8_t *)a.Vlo + head_base;

    const float to_log2 = a.scale * LOG2E;
    f32x4 acc_run[OWN];
    float M_run[OWN];
#pragma unroll
    for (int i = 0; i < OWN; ++i) { acc_run[i] = (f32x4){0.f, 0.f, 0.f, 0.f}; M_run[i] = LLMA_NEG_INF; }
    float M_row = LLMA_NEG_INF, L_row = 0.f;                         // thread j < m_blk: row j's running max / sum
    for (int c = c0; c < c1; ++c) {
        const int key0 = c * ATTN_CHUNK + wave * 32;
        const bool active = key0 < kv_len;                           // uniform for the wave
        const bool use_lo = KVS && c >= c_lo;                        // uniform for the workgroup
        const bool masked = key0 + 31 > T + j0;                      // uniform: some row may not see all of these positions
        u32x4 ka[2][KSTEPS], va[DT];
        u32x2 kb[2][KSTEPS], vb[DT];                     // lo planes: one byte per element
        if (active) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) {
                    const size_t off = (size_t)(key0 / 16 + t) * (16 * DH) + s * 512 + lane * 8;
                    ka[t][s] = *(const u32x4 *)(kh + off);
                    if (KVS && use_lo) kb[t][s] = *(const u32x2 *)(kl + off);
                }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const size_t off = (size_t)(key0 / 32) * (32 * DH) + dt * 512 + lane * 8;
                va[dt] = *(const u32x4 *)(vh + off);
                if (KVS && use_lo) vb[dt] = *(const u32x2 *)(vl + off);
            }
        }
#pragma unroll
        for (int q = 0; q < NTQ; ++q) {
            const int j = j0 + q * 16 + n;
            const bool valid = j < m;
            float mrow = LLMA_NEG_INF, lsum = 0.f;
            f32x4 o[DT];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (active && j0 + q * 16 < m) {                         // (a row tile past the block's rows: nothing to do, uniform)
                const int rpos = valid ? T + j : -1;
                const int r = b * m + (valid ? j : j0);
                u32x4 qh[KSTEPS], ql[KSTEPS];
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) {
                    const size_t off = xtile_off(r, h * DH + s * 32 + g * 8, d_model / 32, true);
                    qh[s] = *(const u32x4 *)((const bf16_t *)a.Qhi + off);
                    ql[s] = *(const u32x4 *)((const bf16_t *)a.Qlo + off);
                }
                float sv[8];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < KSTEPS; ++s) {
                        acc = mfma16x16x32(ka[t][s], qh[s], acc);
                        acc = mfma16x16x32(ka[t][s], ql[s], acc);
                        if (KVS && use_lo) acc = mfma16x16x32(lo8_operand(kb[t][s]), qh[s], acc);
                    }
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) sv[t * 4 + r4] = acc[r4];
                }
                const float mx = attn_mask_max(sv, masked, key0 + 4 * g, rpos) * to_log2;
                float p[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    p[i] = attn_exp(sv[i], to_log2, mx);
                    lsum += p[i];
                }
                mrow = mx;
                u32x2 h0, l0, h1, l1;
                split4(p, h0, l0);
                split4(p + 4, h1, l1);
                const u32x4 ph = (u32x4){h0[0], h0[1], h1[0], h1[1]};
                const u32x4 pl = (u32x4){l0[0], l0[1], l1[0], l1[1]};
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    o[dt] = mfma16x16x32(va[dt], ph, o[dt]);
                    o[dt] = mfma16x16x32(va[dt], pl, o[dt]);
                    if (KVS && use_lo) o[dt] = mfma16x16x32(lo8_operand(vb[dt]), ph, o[dt]);
                }
            }
            // publish this wave's (max, sum, O) of the row tile
            lsum += lane_xor<16>(lsum);
            lsum += lane_xor<32>(lsum);
            if (g == 0) { sm[wave][q * 16 + n] = mrow; sl[wave][q * 16 + n] = lsum; }
            if (q * 16 + n < RS)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) *(f32x4 *)&so[wave][q * 16 + n][dt * 16 + 4 * g] = o[dt];
        }
        __syncthreads();
        // merge the four waves in wave order, then fold the chunk into the running state (chunk order)
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int idx = threadIdx.x + 256 * i;
            if (idx < m_blk * (DH / 4)) {
                const int j = idx / (DH / 4), d4 = idx % (DH / 4);
                float Mc = LLMA_NEG_INF;
#pragma unroll
                for (int w = 0; w < 4; ++w) Mc = fmaxf(Mc, sm[w][j]);
                if (Mc != LLMA_NEG_INF) {
                    f32x4 accc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const float mw = sm[w][j];
                        const float sc = (mw == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(mw - Mc);
                        accc += *(const f32x4 *)&so[w][j][d4 * 4] * sc;
                    }
                    const float Mn = fmaxf(M_run[i], Mc);
                    const float s_run = (M_run[i] == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(M_run[i] - Mn);
                    acc_run[i] = acc_run[i] * s_run + accc * __builtin_amdgcn_exp2f(Mc - Mn);
                    M_run[i] = Mn;
                }
            }
        }
        if (threadIdx.x < m_blk) {
            const int j = threadIdx.x;
            float Mc = LLMA_NEG_INF;
            for (int w = 0; w < 4; ++w) Mc = fmaxf(Mc, sm[w][j]);
            if (Mc != LLMA_NEG_INF) {
                float Lc = 0.f;
                for (int w = 0; w < 4; ++w) {
                    const float mw = sm[w][j];
                    Lc += (mw == LLMA_NEG_INF) ? 0.f : sl[w][j] * __builtin_amdgcn_exp2f(mw - Mc);
                }
                const float Mn = fmaxf(M_row, Mc);
                const float s_run = (M_row == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(M_row - Mn);
                L_row = L_row * s_run + Lc * __builtin_amdgcn_exp2f(Mc - Mn);
                M_row = Mn;
            }
        }
        __syncthreads();                                             // the merge buffers are written again by the next chunk
    }
    const size_t pbase = (((size_t)b * a.H + h) * a.n_chunks + blockIdx.x) * ((size_t)a.n_rblocks * RQ) + j0;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        const int idx = threadIdx.x + 256 * i;
        if (idx < m_blk * (DH / 4)) {
            const int j = idx / (DH / 4), d4 = idx % (DH / 4);
            *(f32x4 *)(a.po + (pbase + j) * DH + d4 * 4) = acc_run[i];
        }
    }
    if (threadIdx.x < m_blk) {
        a.pm[pbase + threadIdx.x] = M_row;
        a.pl[pbase + threadIdx.x] = L_row;
    }
}

// The same walk for one or two row tiles with the running state per WAVE: a wave folds its 32 positions
// of every chunk into its own (max, sum, O) in registers -- no LDS and no barrier inside the walk, so
// the eight waves of a compute unit drift apart and one wave's arithmetic hides the other's loads --
// and the four waves are merged once, in wave order, at the end of the walk.  A row's result is
// again a function of absolute positions only (wave w: positions 32 w .. 32 w + 31 of each chunk of
// the walk in chunk order; then the waves in order; then the walks in order in the combine kernel).
template <int DH, int NTQ, bool KVS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_walk_wave_bf16_kernel(AttnArgs a) {
    constexpr int KSTEPS = DH / 32, DT = DH / 16;
    constexpr int RQ = NTQ * 16;
    constexpr int OWN = (RQ * (DH / 4) + 255) / 256;                  // merged output elements (float4) per thread
    __shared__ float sm[4][RQ], sl[4][RQ];
    __shared__ float so[4][RQ][DH + 4];
    const int h = blockIdx.y, b = blockIdx.z / a.n_rblocks, rb = blockIdx.z % a.n_rblocks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int slot = a.batch_slots[b];
    const int T = a.T[slot];
    const int lo_from = (KVS && a.lo_from != nullptr) ? a.lo_from[slot] : 0;
    const int m = a.m, j0 = rb * RQ;
    if (j0 >= m) return;
    const int m_blk = (m - j0 < RQ) ? m - j0 : RQ;
    const int kv_len = T + j0 + m_blk;                               // positions the block's last row can see
    const int c0 = blockIdx.x * ATTN_WALK_CHUNKS;
    if (c0 * ATTN_CHUNK >= kv_len) return;                           // uniform for the workgroup
    const int c_need = (kv_len + ATTN_CHUNK - 1) / ATTN_CHUNK;
    const int c1 = c0 + ATTN_WALK_CHUNKS < c_need ? c0 + ATTN_WALK_CHUNKS : c_need;
    int c_lo = KVS ? lo_from / ATTN_CHUNK : c1;                      // chunks below c_lo: imported bf16 cache, single plane
    c_lo = c_lo < c0 ? c0 : (c_lo > c1 ? c1 : c_lo);
    const int d_model = a.H * DH;
    const size_t head_base = ((size_t)slot * a.H + h) * (size_t)a.max_seq * DH;
    const bf16_t *kh = (const bf16_t *)a.Khi + head_base; const uint8_t *kl = (const uint8_t *)a.Klo + head_base;
    const bf16_t *vh = (const bf16_t *)a.Vhi + head_base; const uint8_t *vl = (const uint8_t *)a.Vlo + head_base;

    // the block's query rows (both planes) stay on chip for the whole walk: in registers for one row
    // tile; for two, as MFMA operands in LDS (in the merge buffer, which is not needed before the end)
    constexpr bool QLDS = NTQ > 1;
    u32x4 qh[QLDS ? 1 : NTQ][KSTEPS], ql[QLDS ? 1 : NTQ][KSTEPS];
    u32x4 *qs = (u32x4 *)&so[0][0][0];                               // [NTQ][2 planes][KSTEPS][64 lanes]
    int rpos[NTQ];
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        const int j = j0 + q * 16 + n;
        const bool valid = j < m;
        rpos[q] = valid ? T + j : -1;
        const int r = b * m + (valid ? j : j0);
        if (!QLDS) {
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const size_t off = xtile_off(r, h * DH + s * 32 + g * 8, d_model / 32, true);
                qh[q][s] = *(const u32x4 *)((const bf16_t *)a.Qhi + off);
                ql[q][s] = *(const u32x4 *)((const bf16_t *)a.Qlo + off);
            }
        } else {
            for (int s = wave; s < KSTEPS; s += 4) {                 // (the four waves share the staging)
                const size_t off = xtile_off(r, h * DH + s * 32 + g * 8, d_model / 32, true);
                qs[((q * 2 + 0) * KSTEPS + s) * 64 + lane] = *(const u32x4 *)((const bf16_t *)a.Qhi + off);
                qs[((q * 2 + 1) * KSTEPS + s) * 64 + lane] = *(const u32x4 *)((const bf16_t *)a.Qlo + off);
            }
        }
    }
    if (QLDS) __syncthreads();
    const float to_log2 = a.scale * LOG2E;
    f32x4 o[NTQ][DT];
    float Mw[NTQ], Lw[NTQ];                                          // row n's reference (see ATTN_REBASE); the lane's share of its running sum
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        Mw[q] = LLMA_NEG_INF; Lw[q] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[q][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    // one chunk of the wave; LO: the chunk has lo planes (a constant per call site, so that every load
    // of the chunk is unconditional)
    auto chunk = [&](int c, auto lo_tag) {
        constexpr bool LO = decltype(lo_tag)::value;
        const int key0 = c * ATTN_CHUNK + wave * 32;
        if (key0 >= kv_len) return;                                  // uniform for the wave: no row sees these positions
        const bool masked = key0 + 31 > T + j0;                      // uniform: some row may not see all of them
        u32x4 ka[2][KSTEPS], va[DT];
        u32x2 kb[2][KSTEPS], vb[DT];                     // lo planes: one byte per element
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const size_t off = (size_t)(key0 / 16 + t) * (16 * DH) + s * 512 + lane * 8;
                ka[t][s] = *(const u32x4 *)(kh + off);
                if (LO) kb[t][s] = *(const u32x2 *)(kl + off);
            }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const size_t off = (size_t)(key0 / 32) * (32 * DH) + dt * 512 + lane * 8;
            va[dt] = *(const u32x4 *)(vh + off);
            if (LO) vb[dt] = *(const u32x2 *)(vl + off);
        }
        __builtin_amdgcn_sched_barrier(0);                           // all of the chunk's blocks are in flight before the first is used
#pragma unroll
        for (int q = 0; q < NTQ; ++q) {
            if (j0 + q * 16 >= m) continue;                          // a row tile past the block's rows (uniform)
            float sv[8];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) {
                    const u32x4 q_hi = QLDS ? qs[((q * 2 + 0) * KSTEPS + s) * 64 + lane] : qh[QLDS ? 0 : q][s];
                    const u32x4 q_lo = QLDS ? qs[((q * 2 + 1) * KSTEPS + s) * 64 + lane] : ql[QLDS ? 0 : q][s];
                    acc = mfma16x16x32(ka[t][s], q_hi, acc);
                    acc = mfma16x16x32(ka[t][s], q_lo, acc);
                    if (LO) acc = mfma16x16x32(lo8_operand(kb[t][s]), q_hi, acc);
                }
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) sv[t * 4 + r4] = acc[r4];
            }
            attn_rebase(attn_mask_max(sv, masked, key0 + 4 * g, rpos[q]) * to_log2, Mw[q], Lw[q], o[q]);
            float p[8], lsum = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                p[i] = attn_exp(sv[i], to_log2, Mw[q]);
                lsum += p[i];
            }
            Lw[q] += lsum;
            u32x2 h0, l0, h1, l1;
            split4(p, h0, l0);
            split4(p + 4, h1, l1);
            const u32x4 ph = (u32x4){h0[0], h0[1], h1[0], h1[1]};
            const u32x4 pl = (u32x4){l0[0], l0[1], l1[0], l1[1]};
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                f32x4 od = o[q][dt];
                od = mfma16x16x32(va[dt], ph, od);
                od = mfma16x16x32(va[dt], pl, od);
                if (LO) od = mfma16x16x32(lo8_operand(vb[dt]), ph, od);
                o[q][dt] = od;
            }
        }
    };
    for (int c = c0; c < c_lo; ++c) chunk(c, std::false_type{});
    if (KVS)
        for (int c = c_lo; c < c1; ++c) chunk(c, std::true_type{});

    // publish the waves' states, merge them in wave order, write the walk's partial
    if (QLDS) __syncthreads();                                       // every wave is done with the staged query rows
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        float lsum = Lw[q];
        lsum += lane_xor<16>(lsum);
        lsum += lane_xor<32>(lsum);
        if (g == 0) { sm[wave][q * 16 + n] = Mw[q]; sl[wave][q * 16 + n] = lsum; }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *(f32x4 *)&so[wave][q * 16 + n][dt * 16 + 4 * g] = o[q][dt];
    }
    __syncthreads();
    const size_t pbase = (((size_t)b * a.H + h) * a.n_chunks + blockIdx.x) * ((size_t)a.n_rblocks * RQ) + j0;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        const int idx = threadIdx.x + 256 * i;
        if (idx < m_blk * (DH / 4)) {
            const int j = idx / (DH / 4), d4 = idx % (DH / 4);
            float Mc = LLMA_NEG_INF;
#pragma unroll
            for (int w = 0; w < 4; ++w) Mc = fmaxf(Mc, sm[w][j]);
            f32x4 accc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float mw = sm[w][j];
                const float sc = (mw == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(mw - Mc);
                accc += *(const f32x4 *)&so[w][j][d4 * 4] * sc;
            }
            *(f32x4 *)(a.po + (pbase + j) * DH + d4 * 4) = accc;
        }
    }
    if (threadIdx.x < m_blk) {
        const int j = threadIdx.x;
        float Mc = LLMA_NEG_INF, Lc = 0.f;
        for (int w = 0; w < 4; ++w) Mc = fmaxf(Mc, sm[w][j]);
        for (int w = 0; w < 4; ++w) {
            const float mw = sm[w][j];
            Lc += (mw == LLMA_NEG_INF) ? 0.f : sl[w][j] * __builtin_amdgcn_exp2f(mw - Mc);
        }
        a.pm[pbase + j] = Mc;
        a.pl[pbase + j] = Lc;
    }
}

// merges the chunk partials of one (row, head): out = sum_c 2^{m_c - M} O_c / sum_c 2^{m_c - M} l_c,
// over the chunks that contain positions <= the row's own; writes hi/lo tiled planes.  A wave per (row, head): groups of DH / 4
// lanes, four output features per lane; group i takes chunks i, i + PARTS, .. in order, up to sixteen of them in flight, and the groups
// meet at the end.  Which chunk goes where is a function of its position only.  Bound by the round trips to the partials: with one group per
// row half of the wave was idle, and every row asked for sixteen partials however few there are.  One row over 200 / 1000 / 2000 / 3500
// positions of 7B, with the chunk kernel, 7.1 / 10.2 / 13.9 / 25.7 -> 6.3 / 8.7 / 12.7 / 20.6 us, 33 rows 12.2 / 17.8 / 20.8 / 36.0 -> 9.7 / 15.6 / 18.4 / 30.4
// (of which requesting a row tile's queries early 1.3 .. 5), d 512 6.0 -> 5.2.
// CB, chunks of a group in flight: 16, less where all launched chunks are fewer (one trip either way: the same sums).
template <int DH, bool QUADS, int CB>
__device__ __forceinline__ void attn_combine_row(const AttnArgs &a, int rq, int r, int h) {
    constexpr int LANES = DH / 4, PARTS = 64 / LANES;
    const int lane = threadIdx.x & 63, d4 = lane % LANES, part = lane / LANES;
    const int b = r / a.m, j = r % a.m;
    const int slot = a.slot_const >= 0 ? a.slot_const : a.batch_slots[b];
    // live-row count and sequence length: requested before the partials, used after them (one
    // round trip to memory for all three instead of three in a row)
    const int live_last = a.rows_live != nullptr ? *a.rows_live : a.m;
    const int T = a.T[slot];
    loads_stay_above();
    const size_t base = ((size_t)b * a.H + h) * a.n_chunks;
    // the first batch of partials is requested before the row's position is known: every launched
    // chunk has storage, and what a chunk past the row's last one holds is dropped below
    float mv[CB], lv[CB];
    f32x4 ov[CB];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            const int c = c0 + u * PARTS + part < a.n_chunks ? c0 + u * PARTS + part : a.n_chunks - 1;
            mv[u] = a.pm[(base + c) * rq + j];
            lv[u] = a.pl[(base + c) * rq + j];
            ov[u] = (*(const f32x4 *)(a.po + ((base + c) * rq + j) * DH + d4 * 4));
        }
    };
    fetch(0);
    loads_stay_above();
    if (j > live_last) return;                         // padding row of a generation step (its partials are stale: dropped)
    const int pos = T + j;
    const int nc = pos / a.part_span + 1;
    // running (max, sum, O) over the group's chunks
    float M = LLMA_NEG_INF, L = 0.f;
    f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nc; c0 += CB * PARTS) {
        if (c0 > 0) fetch(c0);
        float Mb = M;
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            mv[u] = c0 + u * PARTS + part < nc ? mv[u] : LLMA_NEG_INF;
            Mb = fmaxf(Mb, mv[u]);
        }
        const float rs = (M == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(M - Mb);
        L *= rs;
        acc *= rs;
        M = Mb;
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            if (c0 + u * PARTS >= nc) break;           // uniform
            const bool mine = mv[u] != LLMA_NEG_INF;   // (what a chunk past the end holds may be anything)
            const float w = __builtin_amdgcn_exp2f(mv[u] - M);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = mine ? fmaf(ov[u][e], w, acc[e]) : acc[e];
            L = mine ? fmaf(w, lv[u], L) : L;
        }
    }
    // the groups meet (every lane adds its partner's part to its own; the first group's lanes write)
    const auto meet = [&](float m1, float l1, const f32x4 &a1) {
        const float Mn = fmaxf(M, m1);
        const float s0 = M == LLMA_NEG_INF ? 0.f : __builtin_amdgcn_exp2f(M - Mn), s1 = m1 == LLMA_NEG_INF ? 0.f : __builtin_amdgcn_exp2f(m1 - Mn);
        L = L * s0 + l1 * s1;
        acc = acc * s0 + a1 * s1;
        M = Mn;
    };
    if constexpr (PARTS == 4) meet(lane_xor<16>(M), lane_xor<16>(L), (f32x4){lane_xor<16>(acc[0]), lane_xor<16>(acc[1]), lane_xor<16>(acc[2]), lane_xor<16>(acc[3])});
    meet(lane_xor<32>(M), lane_xor<32>(L), (f32x4){lane_xor<32>(acc[0]), lane_xor<32>(acc[1]), lane_xor<32>(acc[2]), lane_xor<32>(acc[3])});
    if (part != 0) return;
    float v[4] = {acc[0] / L, acc[1] / L, acc[2] / L, acc[3] / L};
    u32x2 hi, lo;
    split4(v, hi, lo);
    const size_t o = xtile_off(r, h * DH + d4 * 4, a.out_KSp, QUADS);
    *(u32x2 *)((bf16_t *)a.out_hi + o) = hi;
    *(u32x2 *)((bf16_t *)a.out_lo + o) = lo;
}

template <int DH, int CB>
__global__ __launch_bounds__(64) void attn_combine_bf16_kernel(AttnArgs a, int rq) { attn_combine_row<DH, false, CB>(a, rq, blockIdx.x, blockIdx.y); }

// The same where the planes' pieces go by four rows (more than XTILE_ROWWISE rows): a workgroup takes four rows, one per
// wave, and writes whole 256-byte pieces of a tile, of which one workgroup per row writes 16 bytes each at a time from four
// XCDs (a 144-row step wrote 4.5 MB where 2.4 are the result).  7B, 16 sequences of 4096, 144 rows: 10.3 -> 8.6 us.
template <int DH, int CB>
__global__ __launch_bounds__(256) void attn_combine_quads_bf16_kernel(AttnArgs a, int rq) {
    const int r = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= a.n_seqs * a.m) return;
    attn_combine_row<DH, true, CB>(a, rq, r, blockIdx.y);
}

// ---------------------------------------------------------------------------------------------
// Prompt-pass attention (more than 48 rows of one sequence): a workgroup owns 32 query rows of one
// head and walks over all 128-position chunks its rows can see; wave w takes positions
// 32 w .. 32 w + 31 of every chunk and keeps its own running (max, sum, O) over them (online
// softmax, no synchronisation inside the walk); at the end the four waves merge through LDS in wave order and the
// normalised rows go straight to the hi/lo planes -- no partials, no combine kernel.  Row blocks
// are numbered from the end of the prompt (longest walks start first).  A pass over the prompts of several sequences
// numbers their blocks one sequence after the other.
// Bound by the wave's own chain of MFMAs and softmax arithmetic -- per 32 positions 96 MFMAs and, counted in issue slots, about as much
// vector arithmetic -- and by what a compute unit takes in (192 KB per chunk of its two workgroups), so two waves per SIMD matter more than anything: the
// query rows sit in LDS, and one set of K / V registers is refilled in place (K while the softmax runs, V while the
// next scores are computed) where two sets took 474 registers and left one wave per SIMD.  A position's lo bytes are
// widened once for both row tiles.  Workgroups are numbered heads first, so that the row blocks of a head run on one XCD (ids 8
// apart, where the heads are a multiple of 8) and find its K and V in that XCD's L2: 7B, 2047 / 1535 / 1023 rows 177 / 104 / 60 -> 136 / 75 / 41 us, 852 rows
// on top of 2047 141 -> 123, d 512 2047 rows 35 -> 23; then masks only where a row's end lies inside the positions, one fused multiply-add and exp2
// per probability, and a reference that hardly ever moves: 2047 rows 120, 852 on 2047 121.5.  Half of an XCD's heads at a time (their K and V fit the L2):
// slower, 79 at 1535.  128 query rows per workgroup and K / V through LDS: 144 at 2047, 96 at 1535, 165 at 852 on 2047 (before the arithmetic changed).
// ---------------------------------------------------------------------------------------------
template <int DH, bool KVS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_prompt_bf16_kernel(AttnArgs a) {
    constexpr int KSTEPS = DH / 32, DT = DH / 16, NTQ = 2, RQ = NTQ * 16;
    __shared__ float sm[4][RQ], sl[4][RQ];
    __shared__ float so[4][RQ][DH + 4];
    static_assert(RQ == PROMPT_BLOCK, "the host counts the row blocks");
    int rb = gridDim.y - 1 - blockIdx.y;
    const int h = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4;
    int slot = a.slot_const, m = a.m, row0 = 0;         // the sequence, its rows, where they start in the pass
    if (a.segs != nullptr) {
        const PromptSeg seg = a.segs[__builtin_amdgcn_readfirstlane(segment_of<&PromptSeg::blk0>(a.segs, a.n_segs, rb))];
        slot = seg.slot; m = seg.rows; row0 = seg.row0; rb -= seg.blk0;
    }
    const int j0 = rb * RQ;
    const int m_blk = (m - j0 < RQ) ? m - j0 : RQ;
    const int d_model = a.H * DH;
    const size_t head_base = ((size_t)slot * a.H + h) * (size_t)a.max_seq * DH;
    const bf16_t *kh = (const bf16_t *)a.Khi + head_base; const uint8_t *kl = (const uint8_t *)a.Klo + head_base;
    const bf16_t *vh = (const bf16_t *)a.Vhi + head_base; const uint8_t *vl = (const uint8_t *)a.Vlo + head_base;
    const int T = a.T[slot];
    const int kv_len = T + j0 + m_blk;                  // positions the block's last row can see
    const int n_ch = (kv_len + ATTN_CHUNK - 1) / ATTN_CHUNK;

    // the block's query rows, as MFMA operands, in LDS (in the merge buffer, which is not needed before the end)
    u32x4 *qs = (u32x4 *)&so[0][0][0];                  // [NTQ][2 planes][KSTEPS][64 lanes]
    int rpos[NTQ];
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        const int j = j0 + q * 16 + n;
        rpos[q] = j < m ? T + j : -1;
        for (int s = wave; s < KSTEPS; s += 4) {
            const size_t off = xtile_off(row0 + (j < m ? j : 0), h * DH + s * 32 + g * 8, d_model / 32, true);
            qs[((q * 2 + 0) * KSTEPS + s) * 64 + lane] = *(const u32x4 *)((const bf16_t *)a.Qhi + off);
            qs[((q * 2 + 1) * KSTEPS + s) * 64 + lane] = *(const u32x4 *)((const bf16_t *)a.Qlo + off);
        }
    }
    u32x4 ka[2][KSTEPS], va[DT];
    u32x2 kb[2][KSTEPS], vb[DT];
    auto fetch_k = [&](int c) {
        const int key0 = c * ATTN_CHUNK + wave * 32;    // below the rounded capacity for every chunk
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const size_t off = (size_t)(key0 / 16 + t) * (16 * DH) + s * 512 + lane * 8;
                ka[t][s] = *(const u32x4 *)(kh + off);
                if (KVS) kb[t][s] = *(const u32x2 *)(kl + off);
            }
    };
    auto fetch_v = [&](int c) {
        const int key0 = c * ATTN_CHUNK + wave * 32;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const size_t off = (size_t)(key0 / 32) * (32 * DH) + dt * 512 + lane * 8;
            va[dt] = *(const u32x4 *)(vh + off);
            if (KVS) vb[dt] = *(const u32x2 *)(vl + off);
        }
    };
    const float to_log2 = a.scale * LOG2E;
    float mrow[NTQ], lrow[NTQ];
    f32x4 o[NTQ][DT];
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        mrow[q] = LLMA_NEG_INF;
        lrow[q] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[q][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    fetch_k(0);
    fetch_v(0);
    __syncthreads();                                    // the query rows are staged
    for (int c = 0; c < n_ch; ++c) {
        const int key0 = c * ATTN_CHUNK + wave * 32;
        if (key0 >= kv_len) break;                      // uniform for the wave, last chunk only: no row sees these positions
        const int c1 = c + 1 < n_ch ? c + 1 : c;        // (the last chunk requests itself once more)
        // scores of both row tiles, then the K registers take the next chunk while this one's softmax and V run
        float sv[NTQ][8];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 acc[NTQ];
#pragma unroll
            for (int q = 0; q < NTQ; ++q) acc[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const u32x4 klo = KVS ? lo8_operand(kb[t][s]) : (u32x4){0u, 0u, 0u, 0u};
#pragma unroll
                for (int q = 0; q < NTQ; ++q) {
                    const u32x4 q_hi = qs[((q * 2 + 0) * KSTEPS + s) * 64 + lane], q_lo = qs[((q * 2 + 1) * KSTEPS + s) * 64 + lane];
                    acc[q] = mfma16x16x32(ka[t][s], q_hi, acc[q]);
                    acc[q] = mfma16x16x32(ka[t][s], q_lo, acc[q]);
                    if (KVS) acc[q] = mfma16x16x32(klo, q_hi, acc[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < NTQ; ++q)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) sv[q][t * 4 + r4] = acc[q][r4];
        }
        __builtin_amdgcn_sched_barrier(0);
        fetch_k(c1);
        __builtin_amdgcn_sched_barrier(0);
        u32x4 ph[NTQ], pl[NTQ];
        const bool masked = key0 + 31 > T + j0;         // uniform: a row may not see all of these positions
#pragma unroll
        for (int q = 0; q < NTQ; ++q) {
            attn_rebase(attn_mask_max(sv[q], masked, key0 + 4 * g, rpos[q]) * to_log2, mrow[q], lrow[q], o[q]);
            float psum = 0.f;
            float p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                p[i] = attn_exp(sv[q][i], to_log2, mrow[q]);
                psum += p[i];
            }
            lrow[q] += psum;                            // this lane's 8 keys; lanes are added at the end
            u32x2 h0, l0, h1, l1;
            split4(p, h0, l0);
            split4(p + 4, h1, l1);
            ph[q] = (u32x4){h0[0], h0[1], h1[0], h1[1]};
            pl[q] = (u32x4){l0[0], l0[1], l1[0], l1[1]};
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const u32x4 vlo = KVS ? lo8_operand(vb[dt]) : (u32x4){0u, 0u, 0u, 0u};
#pragma unroll
            for (int q = 0; q < NTQ; ++q) {
                o[q][dt] = mfma16x16x32(va[dt], ph[q], o[q][dt]);
                o[q][dt] = mfma16x16x32(va[dt], pl[q], o[q][dt]);
                if (KVS) o[q][dt] = mfma16x16x32(vlo, ph[q], o[q][dt]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        fetch_v(c1);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();                                    // every wave is done with the staged query rows
    // ---- merge the four waves in wave order, normalise, write the hi/lo planes
#pragma unroll
    for (int q = 0; q < NTQ; ++q) {
        float l = lrow[q];
        l += lane_xor<16>(l);
        l += lane_xor<32>(l);
        if (g == 0) { sm[wave][q * 16 + n] = mrow[q]; sl[wave][q * 16 + n] = l; }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *(f32x4 *)&so[wave][q * 16 + n][dt * 16 + 4 * g] = o[q][dt];
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < m_blk * (DH / 4); idx += 256) {
        const int j = idx / (DH / 4), d4 = idx % (DH / 4);
        float M = LLMA_NEG_INF;
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, sm[w][j]);
        f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = sm[w][j];
            const float sc = (mw == LLMA_NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(mw - M);
            acc += *(const f32x4 *)&so[w][j][d4 * 4] * sc;
            L += sl[w][j] * sc;
        }
        float v[4] = {acc[0] / L, acc[1] / L, acc[2] / L, acc[3] / L};
        u32x2 hi, lo;
        split4(v, hi, lo);
        const size_t off = xtile_off(row0 + j0 + j, h * DH + d4 * 4, a.out_KSp, true);
        *(u32x2 *)((bf16_t *)a.out_hi + off) = hi;
        *(u32x2 *)((bf16_t *)a.out_lo + off) = lo;
    }
}

template <int DH, int CB>
static void launch_combine_cb(const AttnArgs &a, int rq, hipStream_t st) {
    const int rows = a.n_seqs * a.m;
    if (a.quads) hipLaunchKernelGGL((attn_combine_quads_bf16_kernel<DH, CB>), dim3((rows + 3) / 4, a.H), dim3(256), 0, st, a, rq);
    else hipLaunchKernelGGL((attn_combine_bf16_kernel<DH, CB>), dim3(rows, a.H), dim3(64), 0, st, a, rq);
}
template <int DH>
static void launch_combine(const AttnArgs &a, int rq, hipStream_t st) {
    constexpr int PARTS = 256 / DH;
    if (a.n_chunks <= 4 * PARTS) launch_combine_cb<DH, 4>(a, rq, st);
    else if (a.n_chunks <= 8 * PARTS) launch_combine_cb<DH, 8>(a, rq, st);
    else launch_combine_cb<DH, 16>(a, rq, st);
}

template <int DH, int NTQ, bool KVS>
static void launch_attn_tiles(const AttnArgs &a, hipStream_t st) {
    const dim3 grid(a.n_chunks, a.H, a.n_seqs * a.n_rblocks), block(256);
    constexpr bool FEW = NTQ == 3;                                   // COMPACT where the rows fit it
    if (a.rows_live != nullptr) {                                    // generation step of one sequence: padding rows known on the device (at most max_k + 1 = 33)
        hipLaunchKernelGGL((attn_bf16_kernel<DH, NTQ, KVS, true, false, FEW>), grid, block, 0, st, a);
    } else if (KVS && a.slot_const < 0 && a.lo_from != nullptr) {    // several sequences: their caches may have been imported
        if (FEW && a.m <= ATTN_COMPACT_ROWS) hipLaunchKernelGGL((attn_bf16_kernel<DH, NTQ, KVS, false, KVS, FEW>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((attn_bf16_kernel<DH, NTQ, KVS, false, KVS, false>), grid, block, 0, st, a);
    } else {
        if (FEW && a.m <= ATTN_COMPACT_ROWS) hipLaunchKernelGGL((attn_bf16_kernel<DH, NTQ, KVS, false, false, FEW>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((attn_bf16_kernel<DH, NTQ, KVS, false, false, false>), grid, block, 0, st, a);
    }
}
template <int DH, bool KVS>
static void launch_attn_dh(const AttnArgs &a0, hipStream_t st) {
    // up to 48 rows per workgroup; longer row lists (prompt processing) are cut into row blocks
    AttnArgs a = a0;
    if (a.n_seqs == 1 && a.m > 48 && a.slot_const >= 0) {           // prompt pass
        const int blocks = a.segs ? a.n_chunks : (a.m + PROMPT_BLOCK - 1) / PROMPT_BLOCK;
        hipLaunchKernelGGL((attn_prompt_bf16_kernel<DH, KVS>), dim3(a.H, blocks), dim3(256), 0, st, a);
        return;
    }
    const int ntq = a.m > 32 ? 3 : (a.m + 15) / 16;
    a.n_rblocks = (a.m + ntq * 16 - 1) / (ntq * 16);
    a.part_span = ATTN_CHUNK;
    if (a.rows_live == nullptr && a.slot_const < 0 && a.n_seqs * a.m > 48 && a.m <= ATTN_COMPACT_ROWS) {     // wide batched step
        a.n_chunks = (a.n_chunks + ATTN_WALK_CHUNKS - 1) / ATTN_WALK_CHUNKS;
        a.part_span = ATTN_CHUNK * ATTN_WALK_CHUNKS;
        dim3 wgrid(a.n_chunks, a.H, a.n_seqs * a.n_rblocks);
        if (ntq == 1) hipLaunchKernelGGL((attn_walk_wave_bf16_kernel<DH, 1, KVS>), wgrid, dim3(256), 0, st, a);
        else if (ntq == 2) hipLaunchKernelGGL((attn_walk_wave_bf16_kernel<DH, 2, KVS>), wgrid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((attn_walk_bf16_kernel<DH, 3, KVS>), wgrid, dim3(256), 0, st, a);
        launch_combine<DH>(a, a.n_rblocks * ntq * 16, st);
        return;
    }
    if (ntq == 1) launch_attn_tiles<DH, 1, KVS>(a, st);
    else if (ntq == 2) launch_attn_tiles<DH, 2, KVS>(a, st);
    else launch_attn_tiles<DH, 3, KVS>(a, st);
    launch_combine<DH>(a, a.n_rblocks * ntq * 16, st);
}

void launch_attn_bf16(const AttnArgs &a, hipStream_t st) {
    const bool kvs = a.Klo != nullptr;
    if (a.dh == 128) { if (kvs) launch_attn_dh<128, true>(a, st); else launch_attn_dh<128, false>(a, st); }
    else { if (kvs) launch_attn_dh<64, true>(a, st); else launch_attn_dh<64, false>(a, st); }
}
