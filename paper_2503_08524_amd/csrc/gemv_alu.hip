// Weight-streaming GEMV for one (or a few) activation columns on the vector ALUs.
//
// This is the batch-1 decode projection: every weight byte is read from HBM
// exactly once, 16 bytes per lane per load, a whole wave reading 1 KiB of one
// weight row per instruction.  Activations sit in LDS as fp32 (laid out so that a
// wave's reads are conflict-free), accumulation is fp32, a row's dot product is
// finished with a wave reduction.  The RMSNorm of the input (fused QKV, gate/up
// and lm_head projections) is recomputed by every workgroup in its prologue: the
// input is a few KiB that stay in L2, which is cheaper than a separate launch.
// Each wave issues its share of the activation loads first and the loads of its first
// weight rows right behind them, so the two latencies overlap and the activations, being
// first in the queue, arrive first.
//
// Epilogues: plain store; residual add; SiLU(gate)*up; and, for the fused QKV
// projection, the rotary embedding plus the append of the new K/V row to the
// cache (a wave owns the two rows (j, j + hd/2) of a head that one rotation pairs).
#include "gemv_alu.h"

namespace d3 {

namespace {

// MANY: more columns than a workgroup takes.  blockIdx.x numbers groups of NC of them, the last one may hold fewer, and blockIdx.y the workgroups of a group: those that
// read the same rows are neighbours, so that the rows come from memory once and from the L2s for the other groups.  A launch for each group before, us, a launch each /
// groups one after the other in one launch / so, and with ordinary loads: 7B widths, 32 prompts' last tokens on these projections (8 groups of 4 columns or 16 of 2),
// 2 blocks 3362 / 2875 / 1359; fp32, 4096 wide, 2 blocks, 100 tokens 15600 / 14200 / 4630, 32 sequences 6201 / 5840 / 2700, 5 sequences 1131 / 1071 / 1005; 2048
// wide, 3 blocks, 100 tokens 4510 / 2410 / 1450, 8 sequences 449 / 326 / 349; the tiny model, 4 blocks, a launch a group being all that it costs: 8 sequences
// 192 / 114 / 98, 32 sequences 651 / 149 / 118, 100 tokens 2225 / 241 / 212.
template <typename W, int NC, int MODE, bool NORM, bool MANY>
__global__ __launch_bounds__(kGemvThreads) void gemv_alu_kernel(GemvArgs a) {
    gemv_take_args(a);
    if (MANY) {
        const int first = NC * blockIdx.x;
        a.x += (size_t)first * a.x_stride;
        a.out += (size_t)first * a.out_stride;
        a.col0 += first;
        a.ncols = min(a.ncols - first, NC);
    }
    extern __shared__ float4 xs[];                     // [NC][f4_per_col]
    __shared__ float red[NC][kGemvWaves];
    __shared__ GemvEpBuf<NC> ep[kGemvWaves];
    constexpr int R = (kGemvStageR + NC - 1) / NC;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // the units' addresses are the wave's: scalar
    // Units go round-robin over the waves of the whole grid, so that at any moment the chip streams one contiguous
    // band of the matrix (spread over every memory channel); numbering the waves workgroup-fastest hands the units
    // that do not divide evenly to different workgroups, one each.
    const int wg = MANY ? blockIdx.y : blockIdx.x, n_wg = MANY ? gridDim.y : gridDim.x;
    const int gw = wave * n_wg + wg, nw = n_wg * kGemvWaves;
    GemvStageRegs<NC, R> regs;
    GemvPipe<W, kGemvDepth> pipe;
    gemv_stage_issue<NC, NORM, kGemvThreads, R>(a, tid, regs);          // activations first ...
    gemv_preload<W, MODE, kGemvDepth, MANY>(a, wg, wave, gw, nw, pipe);           // ... the weight stream right behind them
    gemv_stage_commit<W, NC, NORM, kGemvThreads, R>(a, tid, xs, regs, red);
    __syncthreads();
    float rinv[NC];
    gemv_inv_rms<NC, NORM, kGemvWaves>(a, red, rinv);
    gemv_run<W, NC, MODE, kGemvDepth, MANY>(a, xs, gw, nw, pipe, ep[wave], rinv);
}

// A workgroup's LDS is up to 60 KB of activations and, for four columns, 18 KB of finished units: past 64 KB together.
template <typename W, int NC, int MODE, bool NORM, bool MANY>
int launch_kernel(const GemvArgs& a, int grid, size_t lds, hipStream_t s) {
    auto* k = gemv_alu_kernel<W, NC, MODE, NORM, MANY>;
    if (lds + sizeof(GemvEpBuf<NC>) * kGemvWaves > 48 * 1024) {
        static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kGemvLdsBudget);
        if (once != hipSuccess) return (int)once;
    }
    hipLaunchKernelGGL(k, MANY ? dim3((a.ncols + NC - 1) / NC, grid) : dim3(grid), dim3(kGemvThreads), lds, s, a);
    return (int)hipGetLastError();
}

template <typename W, int NC, bool MANY>
int launch_nc(GemvArgs a, int mode, bool norm, int n_wg, hipStream_t s) {
    const size_t lds = (size_t)NC * gemv_f4_per_col<W>(a.K) * sizeof(float4);
    const int n_units = gemv_n_units(a, mode);
    // n_wg workgroups, a multiple of the CU count (a compute unit is the unit of bandwidth: the same number of
    // workgroups on each makes them finish together); fewer when there is not a unit for each wave, up to half as many again where a wave would have
    // to park more than kGemvEpCap (= 64 lanes) units.  One workgroup of eight waves per compute unit against three of four: the activations are
    // staged once instead of three times, and 2048 waves divide the 7B shape's units evenly (2048 of O and down, 6144 of QKV): a step of 17 blocks at
    // batch 1 1385 -> 1348 us (12 waves 1372; five or six steps in flight instead of four 1369, 1374).  Where they do not divide, it is ahead all the same:
    // 13B shape (2560 units of O and down, 7680 of QKV), 8 blocks 1019 -> 940 with the rest of the kernel's changes, O 14.8 -> 13.6 and down 31.5 -> 27.4;
    // bf16 from 1024 to 12288 wide 0.78 to 0.98 of the step, fp32 from 256 to 8192 wide and 1 to 4 columns 0.80 to 0.99.
    const int most = n_wg + (n_wg + 1) / 2, per_wg = kGemvWaves * kGemvEpCap;
    if ((long long)most * per_wg < n_units) return (int)hipErrorInvalidValue;
    int grid = (n_units + kGemvWaves - 1) / kGemvWaves;
    if (grid > n_wg) grid = (n_units + per_wg - 1) / per_wg > n_wg ? (n_units + per_wg - 1) / per_wg : n_wg;
    const int n_waves = grid * kGemvWaves;
    a.wave_units = n_units / n_waves;
    a.wave_units_over = n_units % n_waves;
    a.by_strides = Divisor((a.K / GemvChunk<W>::N + 63) / 64);
    if (mode == MODE_STORE) return norm ? launch_kernel<W, NC, MODE_STORE, true, MANY>(a, grid, lds, s) : launch_kernel<W, NC, MODE_STORE, false, MANY>(a, grid, lds, s);
    if (mode == MODE_RESID) return launch_kernel<W, NC, MODE_RESID, false, MANY>(a, grid, lds, s);
    if (mode == MODE_SWIGLU) return launch_kernel<W, NC, MODE_SWIGLU, true, MANY>(a, grid, lds, s);
    return launch_kernel<W, NC, MODE_QKV_ROPE, true, MANY>(a, grid, lds, s);
}

template <typename W>
int launch_w(const GemvArgs& a, int mode, bool norm, int n_wg, hipStream_t s) {
    const int most = (int)gemv_alu_max_cols(a.K, sizeof(W) == 4 ? 0 : 1);
    if (a.ncols < 1 || most < 1) return (int)hipErrorInvalidValue;
    if (a.ncols > most) {
        if (most == 4) return launch_nc<W, 4, true>(a, mode, norm, n_wg, s);
        if (most == 2) return launch_nc<W, 2, true>(a, mode, norm, n_wg, s);
        return launch_nc<W, 1, true>(a, mode, norm, n_wg, s);
    }
    if (a.ncols == 1) return launch_nc<W, 1, false>(a, mode, norm, n_wg, s);
    if (a.ncols == 2) return launch_nc<W, 2, false>(a, mode, norm, n_wg, s);
    return launch_nc<W, 4, false>(a, mode, norm, n_wg, s);
}

}  // namespace

size_t gemv_alu_max_cols(int K, int weight_dtype) {
    const size_t per_col = (size_t)(weight_dtype == 0 ? gemv_f4_per_col<float>(K) : gemv_f4_per_col<bf16_t>(K)) * sizeof(float4);
    size_t n = kGemvLdsBudget / per_col;
    return n >= 4 ? 4 : (n >= 2 ? 2 : (n >= 1 ? 1 : 0));
}

// Requirements (checked by the caller): K % 8 == 0, total_rows even, ncols >= 1, gemv_alu_max_cols >= 1,
// MODE_RESID without norm and of one matrix, MODE_SWIGLU / MODE_QKV_ROPE with norm, x/out/weights 16-byte aligned.
int launch_gemv_alu(const GemvArgs& a, int weight_dtype, int mode, bool norm, int n_wg, hipStream_t s) {
    return weight_dtype == 0 ? launch_w<float>(a, mode, norm, n_wg, s) : launch_w<bf16_t>(a, mode, norm, n_wg, s);
}

}  // namespace d3
