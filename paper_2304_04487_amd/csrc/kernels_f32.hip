// fp32 path of the verification forward (paper: Eq. 3): plain vector-ALU kernels for models
// whose weights are fp32 (the tiny parity configuration).  Launch-bound by nature; written for
// exactness and for the same row-count invariance as the bf16 path: every output element is
// reduced in an order that depends on the matrix shape / absolute key positions only.
#include "common.h"
#include "kernels.h"

__global__ void kv_import_f32_kernel(const float *__restrict__ k, const float *__restrict__ v,
                                     float *__restrict__ kc, float *__restrict__ vc, int H, int len, int dh, int max_seq) {
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)H * len * dh;
    if (idx >= total) return;
    int c = (int)(idx % dh);
    int pos = (int)((idx / dh) % len);
    int h = (int)(idx / ((size_t)dh * len));
    size_t o = ((size_t)h * max_seq + pos) * dh + c;
    kc[o] = k[idx];
    vc[o] = v[idx];
}
void launch_kv_import_f32(const void *k, const void *v, void *kc, void *vc, int H, int len, int dh,
                          int max_seq, hipStream_t st) {
    size_t total = (size_t)H * len * dh;
    hipLaunchKernelGGL(kv_import_f32_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const float *)k, (const float *)v, (float *)kc, (float *)vc, H, len, dh, max_seq);
}

// One wavefront per output feature (SwiGLU: the gate and the up row; QKV: the two features of a rotary pair) and eight
// rows; lanes take four consecutive elements of the reduction axis each, butterfly reduction across the wavefront.
// RMSNorm runs inside: the wave sees every element of its rows anyway, so it adds their squares and scales the sums
// (W (x g)) rstd at the end; RoPE and the cache append run in the epilogue.  Latency-bound at the shapes it
// is used for (d 128, five rows): all loads of a pass over 512 elements are in flight together, where one element per
// lane and trip left a round trip to memory per 64 elements.  Per step of the tiny model: 22 launches -> 13 (with the row set-up that scans and embeds), O and down
// 13.7 -> 3.9 us on average, SwiGLU 8.9 -> 5.1, QKV 6.7 (+ 3.0 + 3.6 for RoPE and RMSNorm) -> 5.1.
template <int EPI, bool VEC>
__global__ __launch_bounds__(64) void gemm_f32_kernel(GemmArgs a) {
    constexpr int NR = 8, E = VEC ? 4 : 1;
    constexpr bool PAIR = EPI == EPI_SWIGLU || EPI == EPI_QKV, NORM = EPI != EPI_RESID;
    const int n = blockIdx.x, r0 = blockIdx.y * NR, lane = threadIdx.x;
    const int K = a.K, nr = a.rows - r0 < NR ? a.rows - r0 : NR;
    const int half = a.dh / 2, d = a.H * a.dh;
    // QKV: wave n = (section, head, i); its features are i and i + dh/2 of the head
    const int sec = EPI == EPI_QKV ? n / (d / 2) : 0, head = EPI == EPI_QKV ? n % (d / 2) / half : 0, i = EPI == EPI_QKV ? n % half : 0;
    const size_t f0 = EPI == EPI_QKV ? (size_t)sec * d + head * a.dh + i : n, f1 = EPI == EPI_QKV ? f0 + half : (size_t)n + a.N;
    const float *W0 = (const float *)a.W + f0 * K, *W1 = (const float *)a.W + (PAIR ? f1 : f0) * K;
    const float *X = (const float *)a.Xhi + (size_t)r0 * K;
    float acc[NR], acc1[NR], ss[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) { acc[r] = 0.f; acc1[r] = 0.f; ss[r] = 0.f; }
    for (int k0 = lane * E; k0 < K; k0 += 128 * E) {           // two groups of 64 E elements per trip
        float w0[2][E], w1[2][E], g[2][E], x[2][NR][E];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = k0 + 64 * E * h < K ? k0 + 64 * E * h : k0;
            __builtin_memcpy(w0[h], __builtin_assume_aligned(W0 + k, 4 * E), 4 * E);
            if (PAIR) __builtin_memcpy(w1[h], __builtin_assume_aligned(W1 + k, 4 * E), 4 * E);
            if (NORM) __builtin_memcpy(g[h], __builtin_assume_aligned(a.gain + k, 4 * E), 4 * E);
#pragma unroll
            for (int r = 0; r < NR; ++r) __builtin_memcpy(x[h][r], __builtin_assume_aligned(X + (size_t)(r < nr ? r : 0) * K + k, 4 * E), 4 * E);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1 && k0 + 64 * E >= K) break;
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (r < nr)                                     // uniform
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const float xv = x[h][r][e], xg = NORM ? xv * g[h][e] : xv;
                        if (NORM) ss[r] = fmaf(xv, xv, ss[r]);
                        acc[r] = fmaf(w0[h][e], xg, acc[r]);
                        if (PAIR) acc1[r] = fmaf(w1[h][e], xg, acc1[r]);
                    }
        }
    }
    // every lane ends with all sums; lane r finishes row r
    float v0 = 0.f, v1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (r < nr) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                acc[r] += __shfl_xor(acc[r], off);
                if (PAIR) acc1[r] += __shfl_xor(acc1[r], off);
                if (NORM) ss[r] += __shfl_xor(ss[r], off);
            }
            if (lane == r) { v0 = acc[r]; v1 = acc1[r]; s2 = ss[r]; }
        }
    if (lane >= nr) return;
    const int row = r0 + lane;
    if (NORM) {
        const float rstd = 1.0f / sqrtf(s2 / (float)K + a.eps);
        v0 *= rstd;
        v1 *= rstd;
    }
    if (EPI == EPI_RESID) {
        a.out[(size_t)row * a.N + n] += v0;
    } else if (EPI == EPI_SWIGLU) {
        ((float *)a.act_hi)[(size_t)row * a.N + n] = v0 / (1.0f + expf(-v0)) * v1;
    } else if (EPI == EPI_LMHEAD) {
        if (a.out) a.out[(size_t)row * a.N + n] = v0;
        a.pval[(size_t)row * a.n_part + n] = v0;
        a.pidx[(size_t)row * a.n_part + n] = n;
    } else {
        // rotate the pair by the row's position (sections q and k), write q, append k and v to the cache
        const float c = a.row_cs[((size_t)row * half + i) * 2], sn = a.row_cs[((size_t)row * half + i) * 2 + 1];
        const float o0 = sec < 2 ? v0 * c - v1 * sn : v0, o1 = sec < 2 ? v1 * c + v0 * sn : v1;
        float *dst = sec == 0 ? (float *)a.q_hi + (size_t)row * d + head * a.dh
                              : (float *)(sec == 1 ? a.k_hi : a.v_hi) + (((size_t)a.row_slot[row] * a.H + head) * a.max_seq + a.row_pos[row]) * a.dh;
        dst[i] = o0;
        dst[i + half] = o1;
    }
}
template <int EPI>
static void launch_gemm_f32_epi(const GemmArgs &a, hipStream_t st) {
    const dim3 grid(EPI == EPI_QKV ? a.N / 2 : a.N, (a.rows + 7) / 8), block(64);
    if (a.K % 4 == 0) hipLaunchKernelGGL((gemm_f32_kernel<EPI, true>), grid, block, 0, st, a);       // (rows and gains start at multiples of 16 bytes)
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, false>), grid, block, 0, st, a);
}
void launch_gemm_f32(const GemmArgs &a, hipStream_t st) {
    switch (a.epi) {
        case EPI_QKV: launch_gemm_f32_epi<EPI_QKV>(a, st); break;
        case EPI_RESID: launch_gemm_f32_epi<EPI_RESID>(a, st); break;
        case EPI_SWIGLU: launch_gemm_f32_epi<EPI_SWIGLU>(a, st); break;
        default: launch_gemm_f32_epi<EPI_LMHEAD>(a, st); break;
    }
}

// One wavefront per (row, head): lane l owns keys l, l+64, ... <= the row's position with its own
// online softmax; the 64 lane states are merged through LDS, lane order.  Which lane owns which key is a
// function of the absolute key position only.  (Merging by butterfly took six shuffles per feature: 10.8 -> 4.9 us.)
template <int DH>
__global__ __launch_bounds__(64) void attn_f32_kernel(AttnArgs a) {
    __shared__ float qs[DH];
    __shared__ float os[64][DH + 1];
    const int r = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const int b = r / a.m, j = r % a.m;
    const int slot = a.batch_slots[b];
    const int pos = a.T[slot] + j;
    const int d_model = a.H * DH;
    const float *q = (const float *)a.Qhi + (size_t)r * d_model + h * DH;
    for (int c = lane; c < DH; c += 64) qs[c] = q[c];
    __syncthreads();
    const size_t head_base = ((size_t)slot * a.H + h) * (size_t)a.max_seq * DH;
    const float *kc = (const float *)a.Khi + head_base, *vc = (const float *)a.Vhi + head_base;
    float mx = LLMA_NEG_INF, l = 0.f, acc[DH];
#pragma unroll
    for (int c = 0; c < DH; ++c) acc[c] = 0.f;
    for (int key = lane; key <= pos; key += 64) {
        const f32x4 *kr = (const f32x4 *)(kc + (size_t)key * DH), *vr = (const f32x4 *)(vc + (size_t)key * DH);
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < DH / 4; ++c) {
            const f32x4 kv = kr[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) s = fmaf(qs[4 * c + e], kv[e], s);
        }
        s *= a.scale;
        const float mnew = fmaxf(mx, s);
        const float alpha = expf(mx - mnew);          // 0 on the first key
        const float p = expf(s - mnew);
        l = l * alpha + p;
#pragma unroll
        for (int c = 0; c < DH / 4; ++c) {
            const f32x4 vv = vr[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * c + e] = acc[4 * c + e] * alpha + p * vv[e];
        }
        mx = mnew;
    }
    float M = mx;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float sc = (mx == LLMA_NEG_INF) ? 0.f : expf(mx - M);
    float L = l * sc;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) L += __shfl_xor(L, off);
#pragma unroll
    for (int c = 0; c < DH; ++c) os[lane][c] = acc[c] * sc;
    __syncthreads();
    float *out = (float *)a.out_hi + (size_t)r * d_model + h * DH;
    for (int c = lane; c < DH; c += 64) {
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 64; w += 4)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += os[w + e][c];
        out[c] = ((v[0] + v[1]) + (v[2] + v[3])) / L;
    }
}
void launch_attn_f32(const AttnArgs &a, hipStream_t st) {
    dim3 grid(a.n_seqs * a.m, a.H), block(64);
    if (a.dh == 32) hipLaunchKernelGGL((attn_f32_kernel<32>), grid, block, 0, st, a);
    else if (a.dh == 64) hipLaunchKernelGGL((attn_f32_kernel<64>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((attn_f32_kernel<128>), grid, block, 0, st, a);
}
