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

// A wave takes one output feature (SwiGLU: the gate and the up row; QKV: the two features of a rotary pair) and NR rows; lanes take four
// consecutive elements of the reduction axis each, butterfly reduction across the
// wavefront.  RMSNorm runs inside: the wave sees every element of its rows anyway, so it adds their squares and scales the sums
// (W (x g)) rstd at the end; RoPE and the cache append run in the epilogue.
// Small launches (d 128, five rows; an empty launch of a replayed graph takes 1.6 us) are bound by latency: the chain from the arguments to the last store is kept
// short.  All loads of a pass over 512 elements and everything the epilogue reads are in flight together; lanes exchange by
// register moves; and with all eight rows in one wave the butterflies were the longest part, so a wave takes two, four waves of a workgroup the
// same feature.  Back to back at 1 / 5 / 9 rows, us:
// QKV 3.1 / 4.5 / 5.6 -> 2.4 / 2.8 / 2.8, O 2.6 / 3.5 / 4.1 -> 2.0 / 2.1 / 2.2, gate/up 3.1 / 4.5 / 5.6 -> 2.4 / 2.8 / 3.0.
// Large ones are bound by what the waves load, of which the weights come again for every NR rows: four or eight rows in a wave, one wave per
// workgroup (f32_rows_per_wave).
#define F32_WAVES(NR) ((NR) == 2 ? 4 : 1)
template <int EPI, bool VEC, int NR>
__global__ __launch_bounds__(64 * F32_WAVES(NR)) void gemm_f32_kernel(GemmArgs a) {
    constexpr int E = VEC ? 4 : 1;
    constexpr bool PAIR = EPI == EPI_SWIGLU || EPI == EPI_QKV, NORM = EPI != EPI_RESID;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // QKV: grid (i, head, 3 sections x row groups); the workgroup's features are i and i + dh/2 of the head
    const int n = blockIdx.x, half = a.dh / 2, d = a.H * a.dh;
    const int sec = EPI == EPI_QKV ? blockIdx.z % 3 : 0, head = EPI == EPI_QKV ? blockIdx.y : 0, i = n;
    const int r0 = (int)(EPI == EPI_QKV ? blockIdx.z / 3 : blockIdx.y) * (F32_WAVES(NR) * NR) + wave * NR;
    const int K = a.K, nr = a.rows - r0 < NR ? a.rows - r0 : NR;
    if (nr <= 0) return;
    const size_t f0 = EPI == EPI_QKV ? (size_t)sec * d + head * a.dh + i : n, f1 = EPI == EPI_QKV ? f0 + half : (size_t)n + a.N;
    const float *W0 = (const float *)a.W + f0 * K, *W1 = (const float *)a.W + (PAIR ? f1 : f0) * K;
    const float *X = (const float *)a.Xhi + (size_t)r0 * K;
    // what the epilogue reads, for the lane's row (lane r finishes row r0 + r)
    const int row = r0 + (lane < nr ? lane : 0);
    float h_in = 0.f, c = 0.f, sn = 0.f;
    int slot = 0, pos = 0;
    auto epilogue_inputs = [&]() {
        if (EPI == EPI_RESID) h_in = a.out[(size_t)row * a.N + n];
        if (EPI == EPI_QKV) {
            c = a.row_cs[((size_t)row * half + i) * 2];
            sn = a.row_cs[((size_t)row * half + i) * 2 + 1];
            slot = a.row_slot[row];
            pos = a.row_pos[row];
        }
    };
    float acc[NR], acc1[NR], ss[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) { acc[r] = 0.f; acc1[r] = 0.f; ss[r] = 0.f; }
    bool first = true;
    for (int k0 = lane * E; k0 < K || first; k0 += 128 * E) {  // two groups of 64 E elements per trip
        float w0[2][E], w1[2][E], g[2][E], x[2][NR][E];
        const bool in0 = k0 < K, in1 = k0 + 64 * E < K;        // (lanes past the end load the row's first elements and add nothing)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = (h ? in1 : in0) ? k0 + 64 * E * h : 0;
            __builtin_memcpy(w0[h], __builtin_assume_aligned(W0 + k, 4 * E), 4 * E);
            if (PAIR) __builtin_memcpy(w1[h], __builtin_assume_aligned(W1 + k, 4 * E), 4 * E);
            if (NORM) __builtin_memcpy(g[h], __builtin_assume_aligned(a.gain + k, 4 * E), 4 * E);
#pragma unroll
            for (int r = 0; r < NR; ++r) __builtin_memcpy(x[h][r], __builtin_assume_aligned(X + (size_t)(r < nr ? r : 0) * K + k, 4 * E), 4 * E);
        }
        if (first) { epilogue_inputs(); first = false; }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!(h ? in1 : in0)) break;
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (NR <= 2 || r < nr)                          // (uniform)
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
    butterfly<32>([&](auto off) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
            if (NR <= 2 || r < nr) {                            // (uniform)
                acc[r] += lane_xor<off.value>(acc[r]);
                if (PAIR) acc1[r] += lane_xor<off.value>(acc1[r]);
                if (NORM) ss[r] += lane_xor<off.value>(ss[r]);
            }
    });
    if (lane >= nr) return;
    float v0 = acc[0], v1 = acc1[0], s2 = ss[0];
#pragma unroll
    for (int r = 1; r < NR; ++r)
        if (lane == r) { v0 = acc[r]; v1 = acc1[r]; s2 = ss[r]; }
    if (NORM) {
        const float rstd = 1.0f / sqrtf(s2 / (float)K + a.eps);
        v0 *= rstd;
        v1 *= rstd;
    }
    if (EPI == EPI_RESID) {
        a.out[(size_t)row * a.N + n] = h_in + v0;
    } else if (EPI == EPI_SWIGLU) {
        ((float *)a.act_hi)[(size_t)row * a.N + n] = v0 / (1.0f + expf(-v0)) * v1;
    } else if (EPI == EPI_LMHEAD) {
        if (a.out) a.out[(size_t)row * a.N + n] = v0;
        a.pval[(size_t)row * a.n_part + n] = v0;
        a.pidx[(size_t)row * a.n_part + n] = n;
    } else {
        // rotate the pair by the row's position (sections q and k), write q, append k and v to the cache
        const float o0 = sec < 2 ? v0 * c - v1 * sn : v0, o1 = sec < 2 ? v1 * c + v0 * sn : v1;
        float *dst = sec == 0 ? (float *)a.q_hi + (size_t)row * d + head * a.dh
                              : (float *)(sec == 1 ? a.k_hi : a.v_hi) + (((size_t)slot * a.H + head) * a.max_seq + pos) * a.dh;
        dst[i] = o0;
        dst[i + half] = o1;
    }
}
template <int EPI, int NR>
static void launch_gemm_f32_rows(const GemmArgs &a, hipStream_t st) {
    constexpr int WAVES = F32_WAVES(NR);
    const int waves = (a.rows + NR - 1) / NR, groups = (waves + WAVES - 1) / WAVES;
    const dim3 grid = EPI == EPI_QKV ? dim3(a.dh / 2, a.H, 3 * groups) : dim3(a.N, groups);
    const dim3 block(64 * (groups > 1 ? WAVES : waves));
    if (a.K % 4 == 0) hipLaunchKernelGGL((gemm_f32_kernel<EPI, true, NR>), grid, block, 0, st, a);       // (rows and gains start at multiples of 16 bytes)
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, false, NR>), grid, block, 0, st, a);
}
// Rows per wave: work division only, every sum is the same.  Two up to 48 M products; from there on as many as there are, up to eight.  us with 2 / 4 / 8 rows (8
// are the kernel of before the split): d 512 gate/up, 16 rows (34 M products) 10.2 / 8.7 / 9.5; d 1024 QKV 9 rows (28 M) 8.4 / 7.9 / 9.5, 16 (50 M) 11.1 / 10.4 / 10.9,
// 48 26.5 / 21.2 / 21.3; down 9 rows (38 M) 9.6 / 9.9 / 13.2, 48 36.0 / 30.4 / 29.6; d 2048 QKV 4 / 8 / 48 rows 17.4 / 15.4 / 19.1, 26.9 / 21.9 / 21.0,
// 107 / 89 / 69, gate/up 48 rows 271 / 237 / 175; d 4096 QKV 4 / 5 / 48 rows 61 / 49 / 58, 78 / 75 / 60, 431 / 357 / 270, O 4 / 48 23 / 18 / 28, 169 / 147 / 130.
static int f32_rows_per_wave(const GemmArgs &a) {
    const double products = (double)a.rows * a.N * a.K * (a.epi == EPI_SWIGLU ? 2 : 1);
    return a.rows <= 2 || products < 48e6 ? 2 : (a.rows <= 4 ? 4 : 8);
}
template <int EPI>
static void launch_gemm_f32_epi(const GemmArgs &a, hipStream_t st) {
    const int nr = f32_rows_per_wave(a);
    if (nr == 2) launch_gemm_f32_rows<EPI, 2>(a, st);
    else if (nr == 4) launch_gemm_f32_rows<EPI, 4>(a, st);
    else launch_gemm_f32_rows<EPI, 8>(a, st);
}
void launch_gemm_f32(const GemmArgs &a, hipStream_t st) {
    switch (a.epi) {
        case EPI_QKV: launch_gemm_f32_epi<EPI_QKV>(a, st); break;
        case EPI_RESID: launch_gemm_f32_epi<EPI_RESID>(a, st); break;
        case EPI_SWIGLU: launch_gemm_f32_epi<EPI_SWIGLU>(a, st); break;
        default: launch_gemm_f32_epi<EPI_LMHEAD>(a, st); break;
    }
}

// A workgroup per (row, head): groups of DH / 4 lanes take a key each, four dimensions per lane, group g the keys g, g + G,
// .. <= the row's position, U of them requested at once, each group with its own online softmax; the groups of a wave meet by
// butterfly, the waves through LDS, in order.  Which group owns which key is a function of the absolute key position only.
// Bound by latency: one wave with a whole key per lane had a trip of 2 x DH / 4 loads per 64 keys and a merge of 64 states
// through LDS.  dh 32, 95 keys: 3.9 -> 3.1 us back to back.
#define F32_ATTN_WAVES 4
template <int DH>
__global__ __launch_bounds__(64 * F32_ATTN_WAVES) void attn_f32_kernel(AttnArgs a) {
    constexpr int LANES = DH / 4, G = 64 * F32_ATTN_WAVES / LANES, U = 4;
    __shared__ f32x4 os[F32_ATTN_WAVES][LANES];
    __shared__ float ms[F32_ATTN_WAVES], ls[F32_ATTN_WAVES];
    const int r = blockIdx.x, h = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int group = threadIdx.x / LANES, c = threadIdx.x % LANES;
    const int b = r / a.m, j = r % a.m;
    const int slot = a.batch_slots[b];
    const int pos = a.T[slot] + j;
    const int d_model = a.H * DH;
    const f32x4 q = *(const f32x4 *)((const float *)a.Qhi + (size_t)r * d_model + h * DH + 4 * c);
    const size_t head_base = ((size_t)slot * a.H + h) * (size_t)a.max_seq * DH;
    const float *kc = (const float *)a.Khi + head_base + 4 * c, *vc = (const float *)a.Vhi + head_base + 4 * c;
    float mx = LLMA_NEG_INF, l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int key0 = 0; key0 <= pos; key0 += G * U) {            // (uniform: all lanes take part in the sums over a group)
        f32x4 kv[U], vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int key = key0 + u * G + group;
            const size_t at = (size_t)(key <= pos ? key : 0) * DH;
            kv[u] = *(const f32x4 *)(kc + at);
            vv[u] = *(const f32x4 *)(vc + at);
        }
        float s[U], mnew = mx;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s[u] = fmaf(q[3], kv[u][3], fmaf(q[2], kv[u][2], fmaf(q[1], kv[u][1], q[0] * kv[u][0])));
            butterfly<LANES / 2>([&](auto off) { s[u] += lane_xor<off.value>(s[u]); });
            s[u] = key0 + u * G + group <= pos ? s[u] * a.scale : LLMA_NEG_INF;
            mnew = fmaxf(mnew, s[u]);
        }
        const float alpha = mx == LLMA_NEG_INF ? 0.f : expf(mx - mnew);
        l *= alpha;
        acc *= alpha;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float p = s[u] == LLMA_NEG_INF ? 0.f : expf(s[u] - mnew);
            l += p;
            acc += vv[u] * p;
        }
        mx = mnew;
    }
    // the wave's groups, then the waves
    const auto meet = [&](float m1, float l1, const f32x4 &a1) {
        const float M = fmaxf(mx, m1);
        const float s0 = mx == LLMA_NEG_INF ? 0.f : expf(mx - M), s1 = m1 == LLMA_NEG_INF ? 0.f : expf(m1 - M);
        l = l * s0 + l1 * s1;
        acc = acc * s0 + a1 * s1;
        mx = M;
    };
    // (each lane adds its partner's part to its own; the lower lanes' results are the ones used)
    if constexpr (LANES <= 8) meet(lane_xor<8>(mx), lane_xor<8>(l), (f32x4){lane_xor<8>(acc[0]), lane_xor<8>(acc[1]), lane_xor<8>(acc[2]), lane_xor<8>(acc[3])});
    if constexpr (LANES <= 16) meet(lane_xor<16>(mx), lane_xor<16>(l), (f32x4){lane_xor<16>(acc[0]), lane_xor<16>(acc[1]), lane_xor<16>(acc[2]), lane_xor<16>(acc[3])});
    meet(lane_xor<32>(mx), lane_xor<32>(l), (f32x4){lane_xor<32>(acc[0]), lane_xor<32>(acc[1]), lane_xor<32>(acc[2]), lane_xor<32>(acc[3])});
    if (lane < LANES) os[wave][lane] = acc;
    if (lane == 0) { ms[wave] = mx; ls[wave] = l; }
    __syncthreads();
    if (threadIdx.x >= LANES) return;
#pragma unroll
    for (int w = 1; w < F32_ATTN_WAVES; ++w) meet(ms[w], ls[w], os[w][c]);
    *(f32x4 *)((float *)a.out_hi + (size_t)r * d_model + h * DH + 4 * c) = acc / l;
}
void launch_attn_f32(const AttnArgs &a, hipStream_t st) {
    dim3 grid(a.n_seqs * a.m, a.H), block(64 * F32_ATTN_WAVES);
    if (a.dh == 32) hipLaunchKernelGGL((attn_f32_kernel<32>), grid, block, 0, st, a);
    else if (a.dh == 64) hipLaunchKernelGGL((attn_f32_kernel<64>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((attn_f32_kernel<128>), grid, block, 0, st, a);
}
