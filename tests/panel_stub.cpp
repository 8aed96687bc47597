// The GEMMs' host side on the CPU: kernels_bf16.hip and kernels_f32.hip compiled for the host alone, on a device whose number of
// compute units the caller sets.
#include <hip/hip_runtime.h>

static int compute_units = 256;
extern "C" void stub_compute_units(int n) { compute_units = n; }
extern "C" hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
extern "C" hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { p->multiProcessorCount = compute_units; return hipSuccess; }

extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
static int launches = 0;
static dim3 launch_grid, launch_block;
static size_t launch_lds;
extern "C" hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { ++launches; return hipSuccess; }
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t) {
    launch_grid = grid; launch_block = block; launch_lds = lds;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st) {
    *grid = launch_grid; *block = launch_block; *lds = launch_lds; *st = nullptr;
    return hipSuccess;
}
extern "C" void **__hipRegisterFatBinary(const void *) { return nullptr; }
extern "C" void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
extern "C" void __hipUnregisterFatBinary(void **) {}

#include "kernels_bf16.hip"
#include "kernels_f32.hip"

#include <vector>

// rows whose rstd no wave computes when a pass (prompt) or step of `rows` rows runs the matrix in ranges of K; -1: it runs whole
extern "C" int stub_rows_without_rstd(int N, int K, int tiles_per_task, int rows, int prompt) {
    const GemmPlan p = make_gemm_plan(N, K, tiles_per_task);
    const int ns = prompt ? panel_prompt_split(p, rows) : p.n_split;
    if (ns <= 1) return -1;
    const PanelCut cut = panel_cut(p, rows, ns);
    const GemmPlan q = raw_plan(p);
    const int per = cut.nw * cut.at, blocks = (q.tasks + per - 1) / per, row_blocks = (rows + 16 * cut.rt - 1) / (16 * cut.rt);
    std::vector<char> done(rows, 0);
    for (int fb = 0; fb < blocks; ++fb)
        for (int rb = 0; rb < row_blocks; ++rb)
            for (int range = 0; range < ns; ++range)
                for (int wave = 0; wave < cut.nw; ++wave) {
                    const RstdShare s = rstd_share(q.tasks, cut.nw, cut.at, row_blocks, fb, rb, range, ns, wave);
                    for (int r = s.first; r < rows; r += s.step)
                        for (int i = r; i < r + 4 && i < rows; ++i) done[i] = 1;
                }
    int missing = 0;
    for (char d : done) missing += !d;
    return missing;
}

// a prompt pass of `rows` rows: height of the block GEMM's row blocks for this matrix (0: it runs in the panel GEMM), and into *outside the tiles that its
// workgroups ask for and that the matrix or the pass does not have
extern "C" int stub_block_tiles_outside(int N, int K, int tiles_per_task, int rows, int *outside) {
    const GemmPlan p = make_gemm_plan(N, K, tiles_per_task);
    *outside = 0;
    if (panel_prompt_split(p, rows) > 1) return 0;
    const int rt = block_height(p, rows, panel_cut(p, rows, 1));
    if (rt == 0) return 0;
    const int pairs = 16 / tiles_per_task, row_tiles = (rows + 15) / 16;
    for (int task0 = 0; task0 < p.tasks; task0 += pairs)
        for (int rt0 = 0; rt0 < row_tiles; rt0 += rt)
            for (int q = 0; q < 16 + 2 * rt; ++q) {
                const int n_tasks = p.tasks - task0 < pairs ? p.tasks - task0 : pairs, n_rt = row_tiles - rt0 < rt ? row_tiles - rt0 : rt;
                *outside += q < 16 ? task0 + block_weight_tile(q, tiles_per_task, n_tasks) >= p.tasks : rt0 + block_row_tile(q - 16, rt, n_rt) >= row_tiles;
            }
    return rt;
}

// a split launch of the panel GEMM over `rows` rows in row blocks of rt tiles: how many row tiles its grid covers (0: nothing was launched)
template <int AT, int NW>
static int panel_covers(int N, int K, int rows, int rt) {
    GemmArgs a{};
    a.plan = make_gemm_plan(N, K, 1);
    a.rows = rows;
    a.ksplit = 2;
    launches = 0;
    launch_panel_rt<EPI_RAW, AT, NW>(rt, a, nullptr);
    if (launches == 0) return 0;
    const int height = (int)(launch_lds / ((size_t)PANEL_STAGES * 2 * PANEL_KC * 1024));
    return (int)launch_grid.x / panel_feature_blocks(a.plan, AT * NW) * height;
}
extern "C" int stub_panel_covers(int at, int nw, int N, int K, int rows, int rt) {
    if (at == 1) return panel_covers<1, 8>(N, K, rows, rt);
    return nw == 8 ? panel_covers<2, 8>(N, K, rows, rt) : (nw == 7 ? panel_covers<2, 7>(N, K, rows, rt) : (nw == 6 ? panel_covers<2, 6>(N, K, rows, rt) : panel_covers<2, 5>(N, K, rows, rt)));
}

// row tiles per workgroup of a split launch: a step's (ranges by the matrix alone) or a prompt pass's (by its rows); 0: it runs whole
extern "C" int stub_split_height(int N, int K, int tiles_per_task, int rows, int prompt) {
    const GemmPlan p = make_gemm_plan(N, K, tiles_per_task);
    const int ns = prompt ? panel_prompt_split(p, rows) : p.n_split;
    return ns > 1 ? panel_cut(p, rows, ns).rt : 0;
}

extern "C" int stub_f32_rows_per_wave(int N, int K, int epi, int rows) {
    GemmArgs a{};
    a.N = N; a.K = K; a.epi = epi; a.rows = rows;
    return f32_rows_per_wave(a);
}
