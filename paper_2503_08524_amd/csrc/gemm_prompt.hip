// Tiled GEMM on the matrix cores for the prompt pass, up to kPassCols activation columns per launch:
// out[col][row] = sum_k W[row][k] * x[col][k], bf16 weights, activations x = hi + lo (two bf16 halves).
//
// With hundreds of columns the contraction is compute-bound (the prompt pass is the one part of the path that is), so
// the design is the opposite of the skinny kernels': operands are staged in LDS and re-used from there.  A workgroup of
// eight waves owns a tile of 256 weight rows x 128 columns and walks K in stages of 64: the stage's weight slab (256 rows x
// 128 bytes) and activation slab (128 columns, hi plane and lo plane, or a plane of 32 k, hi and lo halves, per k-step: see SplitForm) go from global memory straight into LDS
// (buffer_load_dwordx4 ... lds: 16 bytes per lane, lane l of the wave lands at base + 16 l, one instruction fills eight
// 128-byte slab rows).  LDS holds three weight slabs and two activation slabs, 160 KB; one workgroup per compute unit.
//
// What bounds it, and what set the design (measured on a 8192 x 4096 x 2048 product, 256 tiles = one per compute unit):
//  * Whole cache lines.  A stage of 32 k reads 64-byte pieces of rows, every one of them pulling a 128-byte line through the
//    compute unit's L1: the loads alone then held a stage at 0.82 us (40 GB/s per compute unit) whatever their spacing and
//    however many buffers were in flight.  With 64 k per stage a row's piece is one line: 207 -> 196 us.
//  * The two wave groups (waves 0-3, 4-7) share the slabs and split the stage's k: group g multiplies k-step g of every
//    stage (32 k each), each wave a 128 x 64 piece of the tile (8 x 4 MFMA tiles, 16 fragment reads for 64 MFMAs), so there
//    are two waves per SIMD without a second set of slabs or smaller pieces.  At the end the groups exchange halves of their
//    accumulators through LDS (64 KB each way, once per tile) and each finishes two of the four column tiles.
//  * Weights come from HBM, activations mostly from a cache.  A slab requested one stage ahead has 1 us to arrive, which the loaded
//    memory's latency exceeds: a stage then took 1.42 us even with three compute units in four idle.  So the weight slabs have a third
//    buffer and are requested two stages ahead (behind the activations of the stage before, so that a wait for all but a wave's
//    last four loads covers both): 1.15 us.  7B shape, between events, 203 / 512 / 812 / 2048 columns: gate/up 110 / 173 / 260 / 571 -> 94 /
//    158 / 246 / 555 us, down 77 / 97 / 150 / 305 -> 71 / 87 / 131 / 263, O 46 / 48 / 68 / 121 -> 44 / 46 / 64 / 115.
//  * Nothing is issued in bursts.  A stage is 4 slots of 16 MFMAs (one per column tile).  The barrier sits at the start of
//    slot 2, when every wave has read all of the stage's fragments: behind it the slots' MFMAs are interleaved with the loads
//    into the buffers just freed and with the reads of the next stage's first fragments, and slot 0
//    consumes the weight fragments as they arrive.  Reads and loads issued ahead of the MFMAs instead cost 15-20 %.
// The bound is the matrix cores at the clock that their power leaves them: on operands drawn from a normal distribution they
// alone sustain 2.2 PFLOP/s in this kernel's order (both planes of an accumulator back to back; 2.0 with the planes apart; the clock drops with the toggling of the
// operands), and the launches at 2048 columns, 7B shape, 1.2 (O) to 1.4 (QKV 293 us, gate/up 536, down 262) as issued.  Launches of
// the kernel with stages of 32 k (128 x 64 per wave with two workgroups per
// compute unit, or eight waves of 64 x 64) -> the first one with stages of 64 k: QKV 350 -> 308 us (rotation and cache append now included), gate/up
// 657 -> 555, O 165 -> 115, down 362 -> 263.
//
// The LDS reads are inline assembly: the compiler orders every LDS read it knows of behind ALL outstanding direct-to-LDS
// loads, which would drain the prefetch at every stage.  Here the vmcnt / lgkmcnt waits are written out (a wave's loads
// complete in issue order, kLoads per stage), and empty asm statements that name the fragments as operands keep the MFMAs
// behind the waits.  A fragment in flight must not be moved or spilled: it is only across the stage loop's back edge, where the
// loop fits its registers exactly; at every other change of control flow the reads are waited for.  That depends on the compiler, so
// tests/test_prompt_kernel_registers.py follows every such read through the compiled code.
//
// LDS layout: a slab row is eight 16-byte segments, segment s at position s ^ ((row / 2) % 8): sixteen consecutive rows x one
// segment then touch each of the sixteen 16-byte bank groups once.  The direct load fixes where a lane's bytes land, so the
// swizzle is applied on the global side.
//
// Workgroup order: ids go to the XCDs round-robin; XCD x owns the row blocks x, x + 8, ... and walks them in groups of 4 row
// blocks x 8 column blocks, so the 32 tiles it works on at a time share 12 slabs in its L2 (16 column blocks of 2 row
// blocks: 18 slabs; gate/up at 2048 columns 640 -> 600 us, the smaller launches unchanged).  Tiles that do not fill a round of
// all compute units are cut into K parts (prompt_split).
//
// SwiGLU: a workgroup's 256 slab rows are 128 gate rows and the 128 up rows of the same outputs, four tiles of each per
// wave, so a wave finishes silu(gate) * up from its own accumulators.  Operand layouts, RMSNorm folding (1/rms from the
// producer's partial sums of squares, x * gain and the sum of squares of the new residual handed to the consumer) and
// epilogues are those of the skinny matrix-core kernels.
#include <algorithm>
#include <cmath>

#include "gemm_prompt.h"

namespace d3 {

namespace {

constexpr int kTileM = 256, kTileN = 128;      // weight rows and columns of a workgroup tile
constexpr int kABytes = kTileM * kPitch;       // weight slab of a stage
constexpr int kPlane = kTileN * kPitch;        // one plane of its activation slab: 64 hi or lo halves, or 32 k of both
constexpr int kXBytes = 2 * kPlane;
constexpr int kLdsX = 3 * kABytes;             // LDS: three weight slabs, two activation slabs
constexpr int kPromptLds = kLdsX + 2 * kXBytes;        // 160 KB, all there is
[[maybe_unused]] constexpr int kLoadsW = kABytes / 1024 / kWaves, kLoadsX = kXBytes / 1024 / kWaves, kLoads = kLoadsW + kLoadsX;   // direct loads per wave and stage
constexpr int CW = 2;                          // column tiles a wave finishes (it multiplies 2 CW)
[[maybe_unused]] constexpr int kSsqCols = kTileN * 16 / kThreads;   // columns a group of 16 threads takes the sums of squares of
constexpr int kAccWords = RW * CW * 4;         // accumulator words per lane of a finished (half) wave tile

// ---- residual projections.  The finished sums go through LDS, [128 columns][256 rows] of fp32, so that a wave then takes whole columns and
// its loads and stores are 512 bytes to 1 KB in a row.  From the accumulators' own layout an instruction touches 16 columns' rows of 32
// or 64 bytes each, which stores only (above) leave behind but the reading of the old residual waits for: 7B shape, O 137 -> 124 us at
// 2048 columns, 63 -> 59 at 512, down 110 -> 102 at 512; 13B down 489 -> 474 at 2048.  (QKV through LDS as well: 310 -> 320.)
// Rows 4 u .. + 3 of column c are float4 u ^ (c % 16) of the column: the writes of 16 columns' rows u and the reads of one column both
// spread over all banks. ----
__device__ __forceinline__ f32x4* staged(char* lds, int c, int u) { return reinterpret_cast<f32x4*>(lds) + c * 64 + (u ^ (c & 15)); }
// The columns [lo, hi) of the tile, at most 8 N of them: N per wave, lane l takes rows 4 l .. + 3 of each.  sums(i, c) is the finished
// sum of the wave's i-th column; it is called when the loads of the old residual are on their way.
[[maybe_unused]] constexpr int kPartBytes = kTileM * kTileN * 4;
static_assert(kPartBytes == (int)kPromptPartTile && kAccWords * kThreads * 4 == kPartBytes, "the workspace is laid out for these");
#ifdef __HIP_DEVICE_COMPILE__
struct PartRef { __amdgpu_buffer_rsrc_t buf; int parts, slice; };      // a tile's parts [part][128 columns][256 rows], and which one this is
template <int N>
__device__ __forceinline__ void add_residual(const GemvArgs& a, char* lds, int rb, int cb, int lo, int hi, const PartRef& pr, int wave8, int lane) {
    const int row_raw = rb * kTileM + 4 * lane;
    const bool live_row = row_raw < a.total_rows;
    const int row = live_row ? row_raw : a.total_rows - 4;         // rows past the matrix compute on clamped addresses and store nothing
    auto column = [&](int i) { const int c = lo + wave8 + kWaves * i; return c < hi ? c : hi - 1; };
    float4 old[N], gain = make_float4(1.f, 1.f, 1.f, 1.f);
    if (a.ssq_out) gain = *reinterpret_cast<const float4*>(a.gain_next + row);
#pragma unroll
    for (int i = 0; i < N; ++i) old[i] = *reinterpret_cast<const float4*>(a.out + (size_t)(cb * kTileN + column(i)) * a.out_stride + row);   // all requested before the first store, which they might alias
    f32x4 sum[N];
    if constexpr (N == kTileN / kWaves) {              // a whole tile
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] = *staged(lds, column(i), lane);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int part = 0; part < pr.parts; ++part) {
            if (part == pr.slice) {                    // its own part is in LDS
#pragma unroll
                for (int i = 0; i < N; ++i) sum[i] += *staged(lds, column(i), lane);
            } else {
                u32x4 v[N];
#pragma unroll
                for (int i = 0; i < N; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(pr.buf, 16 * lane, part * kPartBytes + column(i) * (4 * kTileM), kAgent);
#pragma unroll
                for (int i = 0; i < N; ++i) sum[i] += __builtin_bit_cast(f32x4, v[i]);
            }
        }
    }
    float sq[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const bool live = live_row && lo + wave8 + kWaves * i < hi;
        const float v[4] = {old[i].x + sum[i][0], old[i].y + sum[i][1], old[i].z + sum[i][2], old[i].w + sum[i][3]};
        sq[i] = live ? (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]) : 0.f;
        if (live) {
            const size_t oi = (size_t)(cb * kTileN + column(i)) * a.out_stride + row;
            store_row4(a.out + oi, v);
            if (a.out_split) {                         // a normalised projection reads it next: hand it x * gain (and sum(x^2) below)
                const float w[4] = {v[0] * gain.x, v[1] * gain.y, v[2] * gain.z, v[3] * gain.w};
                store_split4(a.out_split + (cb * kTileN + column(i)) * a.out_form.pitch(a.out_stride), row, w, a.out_form.lo);
            }
        }
    }
    if (a.ssq_out) {                                   // N sums over 64 lanes: halve the columns a lane carries at every step
        constexpr int kStep = 64 / N;                  // then kStep lanes hold the same column
#pragma unroll
        for (int o = 32, n = N / 2; n >= 1; o >>= 1, n >>= 1) {
            const bool up = lane & o;
#pragma unroll
            for (int i = 0; i < n; ++i) {
                const float mine = up ? sq[i + n] : sq[i], theirs = up ? sq[i] : sq[i + n];
                sq[i] = mine + __shfl_xor(theirs, o, 64);
            }
        }
#pragma unroll
        for (int o = kStep / 2; o >= 1; o >>= 1) sq[0] += __shfl_xor(sq[0], o, 64);
        const int c = lo + wave8 + kWaves * (lane / kStep);        // the lane's upper bits name the column that is left
        if (lane % kStep == 0 && c < hi) a.ssq_out[(size_t)(cb * kTileN + c) * kSsqStride + rb] = sq[0];
    }
}

// A tile in K parts: the columns are dealt out to the parts in runs, one run each with an arrival counter of its own.  A part publishes
// the other parts' runs and counts itself in, then looks at its own run: where all others have been, it adds up and finishes that; else
// it publishes it too.  Whoever arrives last at a run finishes it, so nobody waits; and parts that end together, as those of one round
// do, finish a run each.  (With one part finishing the whole tile, three 128 KB parts came in through one compute unit: 7B shape, between
// events, O 57 -> 48 us at 512 columns, 61 -> 56 at 616, 74 -> 68 at 812, down 100 -> 97, 117 -> 114, 152 -> 147.)  Columns past the last
// are neither published nor read, and sums are taken in the order of the parts, whoever takes them.
__device__ __forceinline__ void add_residual_parts(const GemvArgs& a, char* lds, int rb, int cb, int n_cols, const PartRef& pr, int* tickets, int* last_at, int tid) {
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    auto run = [&](int j) { return n_cols * j / pr.parts; };
    auto publish = [&](int lo, int hi) {
        for (int c = lo + wave8; c < hi; c += kWaves)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, *staged(lds, c, lane)), pr.buf, 16 * lane, pr.slice * kPartBytes + c * (4 * kTileM), kAgent);
    };
    const int own_lo = run(pr.slice), own_hi = run(pr.slice + 1);
    publish(0, own_lo);
    publish(own_hi, n_cols);
    wait_stores();                                     // they have reached the coherence point
    __syncthreads();
    if (tid < pr.parts) {
        const int before = tid == pr.slice ? __hip_atomic_load(&tickets[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : atomicAdd(&tickets[tid], 1);
        last_at[tid] = before == pr.parts - 1;
    }
    __syncthreads();
    if (!last_at[pr.slice]) {
        publish(own_lo, own_hi);
        wait_stores();
        __syncthreads();
        if (tid == 0) last_at[pr.slice] = atomicAdd(&tickets[pr.slice], 1) == pr.parts - 1;
        __syncthreads();
    }
    for (int j = 0; j < pr.parts; ++j) {
        if (!last_at[j]) continue;
        if (tid == 0) __hip_atomic_store(&tickets[j], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // all have been here: leave it clean
        const int lo = run(j), hi = run(j + 1);
        if (lo == hi) continue;
        if (hi - lo > 4 * kWaves) add_residual<8>(a, lds, rb, cb, lo, hi, pr, wave8, lane);
        else add_residual<4>(a, lds, rb, cb, lo, hi, pr, wave8, lane);
    }
}
#endif

// Launch order of the tiles.  Tiles [0, n_whole) have a workgroup each, the others ks of them, one per part of K.  n_rb row blocks: each
// XCD owns n_rb / 8 of them and walks them in groups of kGroupR, the last group may hold fewer; n_rb % 8 are left over.
constexpr int kGroupR = 4, kGroupC = 8;
struct TileOrder {
    int n_rb, n_cb, n_whole;
    Divisor ks, rest, group_tiles, last_group, last_chunk, left;
    TileOrder(int rb, int cb, int whole, int parts)
        : n_rb(rb), n_cb(cb), n_whole(whole), ks(parts), rest(rb * cb - whole > 0 ? rb * cb - whole : 1), group_tiles(kGroupR * cb),
          last_group(rb / 8 % kGroupR ? rb / 8 % kGroupR : kGroupR), last_chunk(last_group.d * kGroupC), left(rb % 8 ? rb % 8 : 1) {}
};

// (The buffer resource type exists in device code only.)
template <int MODE>
__global__ __launch_bounds__(kThreads, 2) void gemm_prompt_kernel(GemvArgs a, TileOrder order) {
#ifdef __HIP_DEVICE_COMPILE__
    constexpr int SW = (MODE == MODE_SWIGLU) ? 2 : 1;
    constexpr int OT = 2 * RW / SW;                    // output row tiles per workgroup (half as many gate/up pairs)
    // behind the 128 KB that the epilogues exchange sums in, once the slabs are done with:
    float* inv_rms = reinterpret_cast<float*>(prompt_lds + kPartBytes);                            // [kTileN]
    int* last_at = reinterpret_cast<int*>(prompt_lds + kPartBytes + kTileN * sizeof(float));       // [0]: of the tile; residual projections: of each run of columns
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave8 >> 2, wave = wave8 & 3, wy = wave >> 1, wx = wave & 1;
    const int li = lane & 15, lg = lane >> 4;

    // What the first loads need of the arguments, requested together: taken as they come up they are a chain of round trips to memory.  Clocks from
    // a workgroup's start to its first load / to its first MFMA, 7B shape, 512 columns, gate/up: 4300 / 13300 with divisions and arguments as they
    // came up, 3350 / 11500 with the divisors' reciprocals from the host and each load sent as soon as its address is known, 1700 / 9300 with this.
    const bf16_t* const arg_x = a.x_split;
    const size_t arg_lo = a.x_form.lo;
    const void *const arg_w0 = a.w[0], *const arg_w1 = MODE == MODE_RESID ? nullptr : a.w[1], *const arg_w2 = MODE == MODE_RESID || MODE == MODE_SWIGLU ? nullptr : a.w[2];
    const int K = a.K, total_rows = a.total_rows, rows0 = a.rows[0], rows1 = a.rows[1];
    asm volatile("" :: "s"(arg_x), "s"(arg_lo), "s"(arg_w0), "s"(arg_w1), "s"(arg_w2), "s"(K), "s"(total_rows), "s"(rows0), "s"(rows1),
                 "s"(order.n_rb), "s"(order.n_cb), "s"(order.n_whole), "s"(order.group_tiles.m));

    // ---- launch order -> tile, K part; tile -> (row block, column block) ----
    const int n_whole = order.n_whole;
    int tile_id = blockIdx.x, slice = 0, parts = 1;
    if (tile_id >= n_whole) {                          // part by part: neighbours in the order share the part's columns of K
        slice = order.rest.of(tile_id - n_whole);
        tile_id -= slice * order.rest.d;
        parts = order.ks.d;
    }
    int rb, cb;
    {
        const int own = order.n_rb / 8, even = own * 8 * order.n_cb;   // row blocks per XCD; what is left of them comes last, in plain order
        if (tile_id < even) {
            const int xcd = tile_id & 7, idx = tile_id >> 3;
            const int group = order.group_tiles.of(idx), rem = idx - group * order.group_tiles.d;
            int chunk, row;
            if (kGroupR * group + kGroupR <= own) {
                chunk = rem / (kGroupR * kGroupC);
                cb = rem % (kGroupR * kGroupC) / kGroupR;
                row = rem % kGroupR;
            } else {
                chunk = order.last_chunk.of(rem);
                const int r2 = rem - chunk * order.last_chunk.d;
                cb = order.last_group.of(r2);
                row = r2 - cb * order.last_group.d;
            }
            rb = (kGroupR * group + row) * 8 + xcd;
            cb += chunk * kGroupC;
        } else {
            cb = order.left.of(tile_id - even);
            rb = own * 8 + (tile_id - even) - cb * order.left.d;
        }
    }
    const int tiles = total_rows / 16;                 // output row tiles of the whole matrix
    // whole stages go to the parts in pairs; the last part takes what is over: an odd stage, and the half stage of K % 64 == 32
    const int pairs = K / (2 * kBK), pair0 = parts == 1 ? 0 : order.ks.of(pairs * slice);
    const int s0 = 2 * pair0, n_stages = 2 * ((parts == 1 ? pairs : order.ks.of(pairs * (slice + 1))) - pair0);
    const int s_end = (K + kBK - 1) / kBK, n_single = slice == parts - 1 ? s_end - 2 * pairs : 0;      // 0, 1 or 2
    // (the launcher sees to at least two whole stages per part)

    // ---- this wave's eight-row blocks of a stage (wave8, wave8 + 8, ...): the first 32 are weight rows, then the activations' first plane, then the second ----
    // Slab tile st = 8 wy + t is wave row wy's tile t.  Plain modes: output tile OT rb + st.  SwiGLU: tiles t < 4 are gate rows,
    // the others the up rows of the same outputs OT rb + 4 wy + t % 4.  Tiles past the matrix re-read the last one (result dropped).
    // Each block's first load goes out before the next block's address is worked out: the code up to here comes from memory too, a line at a time.
    // lane l of a load: row l / 8 of the block, LDS position l % 8, i.e. segment (l % 8) ^ ((slab row / 2) % 8) of that row
    const int prow = lane >> 3, pseg = (lane & 7) ^ ((lane >> 4) | (4 * (wave8 & 1)));
    const bool lines = arg_lo == kSplitLo;             // see SplitForm
    const int pitch_x = lines ? 4 * K : 2 * K, step_x = lines ? 2 * kPitch : kPitch, voff_w = 2 * (prow * K + pseg * 8), voff_x = prow * pitch_x + pseg * 16, voff_x64 = voff_x + 64 * pitch_x;
    __amdgpu_buffer_rsrc_t src[kLoadsW + 2];           // a block of eight weight rows each; the wave's columns c and c + 64 of a plane each
    static_assert(kLoadsX == 4, "two loads of eight columns per plane");
    auto load1 = [&](int j, int t, int lds) {         // t: stage of the whole K; lds: where its slab (weights j < kLoadsW, or activations) lies
        const int jx = j - kLoadsW;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src[j < kLoadsW ? j : kLoadsW + jx / 2], (__attribute__((address_space(3))) void*)((lds_char*)prompt_lds + lds + (wave8 + kWaves * (j < kLoadsW ? j : jx)) * 1024),
                                                 16, j < kLoadsW ? voff_w : jx % 2 ? voff_x64 : voff_x, j < kLoadsW ? t * kPitch : t * step_x, 0, 0);
    };
    int w0 = 0, w1 = kABytes, w2 = 2 * kABytes;        // the weight slabs of this stage and the next two
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        if (j < kLoadsW) {
            const int blk = wave8 + kWaves * j, st = blk >> 1, t = st % RW;
            int otile = MODE == MODE_SWIGLU ? rb * OT + (st / RW) * (RW / 2) + t % (RW / 2) : rb * OT + st;
            otile = otile < tiles ? otile : tiles - 1;
            int local = otile * 16;
            const void* w = MODE == MODE_SWIGLU && t >= RW / 2 ? arg_w1 : arg_w0;
            if (MODE != MODE_SWIGLU && MODE != MODE_RESID && local >= rows0) {
                local -= rows0;
                w = arg_w1;
                if (local >= rows1) { local -= rows1; w = arg_w2; }
            }
            const bf16_t* p = static_cast<const bf16_t*>(w) + (size_t)(local + 8 * (blk & 1)) * K;
            src[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, 2 * 8 * K, 0x00027000);
        } else if ((j - kLoadsW) % 2 == 0) {
            const int half = (j - kLoadsW) / 2;
            const bf16_t* p = arg_x + (size_t)(cb * kTileN + 8 * wave8) * (pitch_x / 2) + (half ? lines ? kPitch / 2 : arg_lo : 0);
            src[kLoadsW + half] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, 72 * pitch_x - (lines ? half * kPitch : 0), 0x00027000);
        }
        load1(j, s0, j < kLoadsW ? w0 : kLdsX);
        fixed_here();
    }
    auto load_w = [&](int t, int lds) {
#pragma unroll
        for (int j = 0; j < kLoadsW; ++j) load1(j, t, lds);
    };
    auto load_x = [&](int t, int buf) {
#pragma unroll
        for (int j = kLoadsW; j < kLoads; ++j) load1(j, t, kLdsX + buf * kXBytes);
    };
    // fragment reads: lane (i, g) takes segment 4 grp + g of row i of a weight tile and of column i of both planes, or segments g and 4 + g of column i of plane grp
    // (tile bases are multiples of 16 rows, so the swizzle depends on i alone)
    const uint32_t slot = (uint32_t)(((grp * 4 + lg) ^ ((li >> 1) & 7)) << 4), slot_b = (uint32_t)((lg ^ ((li >> 1) & 7)) << 4);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)prompt_lds;
    const uint32_t a_off = lds0 + (wy * 16 * RW + li) * kPitch + slot, b_off = lds0 + kLdsX + (wx * 64 + li) * kPitch + (lines ? grp * kPlane + slot_b : slot),
                   b_lo = lines ? b_off ^ kLoBit : b_off + kPlane;

    f32x4 acc[RW][2 * CW];                             // [row tile of the wave][column tile of the wave]
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int tt = 0; tt < 2 * CW; ++tt) acc[r][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 A0[RW], A1[RW];                             // weight fragments of this stage and the next
    PromptB f0, f1, f2;                                // activation fragments of three column tiles
    // Stage t, activations in buffer BUF, on the weight fragments A; X holds column tile 0 when it starts (requested, like A, by the stage
    // before) and column tile 3 in the end, Y the next stage's column tile 0.  MORE: a stage follows; loads: so do two; loads_w: three.
    // The two waves of a SIMD compete for its matrix cores, and the issue favours the older one, which then waited 1070 of a stage's 2420 clocks at the
    // barrier while the younger one, by itself, could not keep the matrix cores busy.  Each slot lowers the wave's priority, so that the one that is
    // behind goes first: 2340 clocks a stage (7B, 32 x 2048 columns, 2 blocks 82.3 -> 81.8 ms; the clock falls with the better use of it).
    // A wave's LDS reads return in order, so "at most n outstanding" names the oldest ones that have arrived.
    auto stage = [&](int t, auto buf_c, auto more_c, auto loads_c, auto loads_w_c, u32x4 (&A)[RW], u32x4 (&An)[RW], PromptB& X, PromptB& Y, PromptB& Z) {
        constexpr int BUF = decltype(buf_c)::value;
        constexpr bool MORE = decltype(more_c)::value;
        const uint32_t Wn = a_off + w1;
        constexpr bool loads = decltype(loads_c)::value, loads_w = decltype(loads_w_c)::value;
        const int k2 = s0 + t + 2, k3 = k2 + 1, xb = kLdsX + BUF * kXBytes;
        // slot 0: the weight fragments are used in the order of their arrival
        __builtin_amdgcn_s_setprio(1);
        read_b_frags<1, BUF * kXBytes>(Y, b_off, b_lo);
        lds_reads_left<8>(); pin_frag(A[0]); pin_frag(A[1]); pin_frag(X.h); pin_frag(X.l);
        mma_hl<0, 2>(acc, 0, A, X); fixed_here();
        lds_reads_left<6>(); pin_frag(A[2]); pin_frag(A[3]);
        mma_hl<2, 2>(acc, 0, A, X); fixed_here();
        lds_reads_left<4>(); pin_frag(A[4]); pin_frag(A[5]);
        mma_hl<4, 2>(acc, 0, A, X); fixed_here();
        lds_reads_left<2>(); pin_frag(A[6]); pin_frag(A[7]);
        mma_hl<6, 2>(acc, 0, A, X); fixed_here();
        // slot 1
        __builtin_amdgcn_s_setprio(0);
        read_b_frags<2, BUF * kXBytes>(Z, b_off, b_lo);
        lds_reads_left<2>(); pin_frag(Y.h); pin_frag(Y.l);
        mma_hl<0, 2>(acc, 1, A, Y); fixed_here();
        read_b_frags<3, BUF * kXBytes>(X, b_off, b_lo); fixed_here();
        mma_hl<2, 6>(acc, 1, A, Y); fixed_here();
        // slots 2 and 3: this wave has read all of stage t
        lds_reads_left<0>(); pin_frag(Z.h); pin_frag(Z.l); pin_frag(X.h); pin_frag(X.l);
        if constexpr (MORE) {
            vm_loads_left<loads ? kLoadsW : 0>();      // this wave's part of stage t + 1 has landed (stage t + 2's weights may be on their way) ...
            __builtin_amdgcn_s_barrier();              // ... and everybody's; nobody still reads stage t
            __builtin_amdgcn_s_setprio(3);
            mma_hl<0, 1>(acc, 2, A, Z); fixed_here(); if (loads) load1(4, k2, xb); fixed_here();
            mma_hl<1, 1>(acc, 2, A, Z); fixed_here(); if (loads) load1(5, k2, xb); fixed_here();
            mma_hl<2, 1>(acc, 2, A, Z); fixed_here(); if (loads) load1(6, k2, xb); fixed_here();
            mma_hl<3, 1>(acc, 2, A, Z); fixed_here(); if (loads) load1(7, k2, xb); fixed_here();
            mma_hl<4, 1>(acc, 2, A, Z); fixed_here(); if (loads_w) load1(0, k3, w0); fixed_here();
            mma_hl<5, 1>(acc, 2, A, Z); fixed_here(); if (loads_w) load1(1, k3, w0); fixed_here();
            mma_hl<6, 1>(acc, 2, A, Z); fixed_here(); if (loads_w) load1(2, k3, w0); read_b_frags<0, (BUF ^ 1) * kXBytes>(Y, b_off, b_lo); fixed_here();
            mma_hl<7, 1>(acc, 2, A, Z); fixed_here(); if (loads_w) load1(3, k3, w0); An[0] = lds_read_frag<0>(Wn); fixed_here();
            __builtin_amdgcn_s_setprio(2);
            mma_hl<0, 1>(acc, 3, A, X); fixed_here(); An[1] = lds_read_frag<1 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<1, 1>(acc, 3, A, X); fixed_here(); An[2] = lds_read_frag<2 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<2, 1>(acc, 3, A, X); fixed_here(); An[3] = lds_read_frag<3 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<3, 1>(acc, 3, A, X); fixed_here(); An[4] = lds_read_frag<4 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<4, 1>(acc, 3, A, X); fixed_here(); An[5] = lds_read_frag<5 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<5, 1>(acc, 3, A, X); fixed_here(); An[6] = lds_read_frag<6 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<6, 1>(acc, 3, A, X); fixed_here(); An[7] = lds_read_frag<7 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<7, 1>(acc, 3, A, X); fixed_here();
        } else {
            mma_hl<0, 8>(acc, 2, A, Z); mma_hl<0, 8>(acc, 3, A, X); fixed_here();
        }
        const int done = w0;
        w0 = w1; w1 = w2; w2 = done;
    };
    static_assert(kLoads == 8 && RW == 8 && CW == 2, "the stage is written out for these");
    constexpr std::integral_constant<int, 0> b0{};
    constexpr std::integral_constant<int, 1> b1{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    // 16 threads take one column's partial sums of squares (thread tid: columns tid / 16 + 32 u), requested between the first stage's loads and
    // the second's: they arrive with the first stage
    const bool norm = MODE != MODE_RESID && a.ssq_in;
    float sq[kSsqCols][2];
    if (norm) {
#pragma unroll
        for (int u = 0; u < kSsqCols; ++u) {
            const float* p = a.ssq_in + (size_t)min(cb * kTileN + (tid >> 4) + kThreads / 16 * u, a.ncols - 1) * kSsqStride;
            sq[u][0] = p[min(tid & 15, a.ssq_parts - 1)];
            sq[u][1] = p[min(16 + (tid & 15), a.ssq_parts - 1)];
        }
    }
    fixed_here();
    load_w(s0 + 1, w1); load_x(s0 + 1, 1);
    if (n_stages > 2) { load_w(s0 + 2, w2); vm_loads_left<kLoads + kLoadsW>(); }
    else vm_loads_left<kLoads>();
    float inv = 0.f;                                   // of column tid / 16 + 32 (tid % 16), for tid % 16 < 4
    if (norm) {
#pragma unroll
        for (int u = 0; u < kSsqCols; ++u) {           // in a fixed order
            float ss = 0.f;
            if ((tid & 15) < a.ssq_parts) ss += sq[u][0];
            if (16 + (tid & 15) < a.ssq_parts) ss += sq[u][1];
            if (a.ssq_parts > 32) {                    // a producer of few rows per workgroup
                const float* p = a.ssq_in + (size_t)min(cb * kTileN + (tid >> 4) + kThreads / 16 * u, a.ncols - 1) * kSsqStride;
                for (int i0 = 32 + (tid & 15); i0 < a.ssq_parts; i0 += 16) ss += p[i0];
            }
            ss = reduce_row(ss, AddOp());
            if ((tid & 15) == u) inv = 1.0f / sqrtf(ss / (float)K + a.eps);
        }
    }
    __syncthreads();                                   // stage 0 is in LDS
    read_b_frags<0>(f0, b_off, b_lo);
    read_a_frags(A0, a_off, std::make_integer_sequence<int, RW>{});
    all_arrived(A0); all_arrived(f0);
    int t = 0;
    for (; t + 4 < n_stages; t += 2) {
        stage(t, b0, yes, yes, yes, A0, A1, f0, f1, f2);
        stage(t + 1, b1, yes, yes, yes, A1, A0, f1, f0, f2);
    }
    all_arrived(A0); all_arrived(f0);                  // nothing in flight where the compiler may move registers
    if (n_stages > 2) {
        stage(t, b0, yes, yes, yes, A0, A1, f0, f1, f2);
        stage(t + 1, b1, yes, yes, no, A1, A0, f1, f0, f2);
        all_arrived(A0); all_arrived(f0);
        t += 2;
    }
    stage(t, b0, yes, no, no, A0, A1, f0, f1, f2);
    stage(t + 1, b1, no, no, no, A1, A0, f1, f0, f2);
    __syncthreads();
    // the stages over, one at a time (K % 64 == 32: the last holds one k-step, which is group 0's; what group 1 finds there belongs to the next row)
    for (int u = s_end - n_single; u < s_end; ++u) {
        load_w(u, 0); load_x(u, 0);
        vm_loads_left<0>();
        __syncthreads();
        if (grp == 0 || (u + 1) * kBK <= K) {
            read_a_frags(A0, a_off, std::make_integer_sequence<int, RW>{});
            read_b_frags<0>(f0, b_off, b_lo); read_b_frags<1>(f1, b_off, b_lo); read_b_frags<2>(f2, b_off, b_lo);
            all_arrived(A0); all_arrived(f0); all_arrived(f1); all_arrived(f2);
            mma_hl<0, 8>(acc, 0, A0, f0); mma_hl<0, 8>(acc, 1, A0, f1);
            mma_hl<0, 8>(acc, 2, A0, f2); fixed_here();
            read_b_frags<3>(f0, b_off, b_lo);
            all_arrived(f0);
            mma_hl<0, 8>(acc, 3, A0, f0); fixed_here();
        }
        __syncthreads();
    }

    // ---- the groups exchange halves: group g finishes the column tiles 2g, 2g + 1 ----
    f32x4 fin[RW][CW];
    {
        f32x4* mine = reinterpret_cast<f32x4*>(prompt_lds) + (size_t)wave8 * (RW * CW * 64) + lane;
        if (MODE != MODE_RESID && (tid & 15) < 4) inv_rms[(tid >> 4) + 32 * (tid & 15)] = inv;
        const f32x4* theirs = reinterpret_cast<const f32x4*>(prompt_lds) + (size_t)(wave8 ^ 4) * (RW * CW * 64) + lane;
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int tt = 0; tt < CW; ++tt) mine[(r * CW + tt) * 64] = grp ? acc[r][tt] : acc[r][CW + tt];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int tt = 0; tt < CW; ++tt) {
                const f32x4 o = theirs[(r * CW + tt) * 64];
                fin[r][tt] = grp ? o + acc[r][CW + tt] : acc[r][tt] + o;      // k-step 0's sum first
            }
    }

    PartRef pr;
    pr.parts = parts; pr.slice = slice;
    const int part_id = tile_id - n_whole;
    pr.buf = __builtin_amdgcn_make_buffer_rsrc(a.part + (size_t)max(part_id, 0) * parts * (kPartBytes / 4), 0, parts * kPartBytes, 0x00027000);
    if constexpr (MODE == MODE_RESID) {
        __syncthreads();                               // the exchanged halves have been read
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int tt = 0; tt < CW; ++tt) *staged(prompt_lds, wx * 64 + grp * 32 + tt * 16 + li, wy * 32 + 4 * r + lg) = fin[r][tt];
        __syncthreads();
        const int n_cols = min(kTileN, a.ncols - cb * kTileN);
        if (parts == 1) add_residual<kTileN / kWaves>(a, prompt_lds, rb, cb, 0, n_cols, pr, wave8, lane);
        else add_residual_parts(a, prompt_lds, rb, cb, n_cols, pr, a.part_tickets + part_id * parts, last_at, tid);
        return;
    }
    // ---- K parts of the other projections: as in add_residual_parts, with the units of the tile dealt out to the parts in runs.  (With the part that
    // arrives last adding up and finishing the whole tile: 7B shape, 512 columns, kernel trace, gate/up 157.8 -> 155.2 us, 88 of 344 tiles in two parts each.)
    // The part that comes last finds most runs waiting for it, so it takes all of them together: each part's sums are a round trip, and run by
    // run they were one more for every run (QKV at 77 columns, 7B and 70B shapes: 54.2 and 72.1 us run by run, 49.1 and 61.4
    // together, 50.5 and 64.0 where the last part finishes the whole tile). ----
    int* tickets = a.part_tickets + part_id * parts;
    constexpr unsigned all_units = (1u << CW * kUnits) - 1;        // bit tt kUnits + r
    auto run = [&](int j) { return parts == 1 ? all_units : (1u << order.ks.of(CW * kUnits * (j + 1))) - (1u << order.ks.of(CW * kUnits * j)); };
    if (parts > 1) {
        auto publish = [&](unsigned units) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int tt = 0; tt < CW; ++tt)
                    if (units >> (tt * kUnits + r % kUnits) & 1)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, fin[r][tt]), pr.buf, 16 * tid, slice * kPartBytes + (r * CW + tt) * 16 * kThreads, kAgent);
            wait_stores();                             // they have reached the coherence point
            __syncthreads();
        };
        const unsigned own = run(slice);
        publish(all_units & ~own);
        if (tid < parts) {
            const int before = tid == slice ? __hip_atomic_load(&tickets[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : atomicAdd(&tickets[tid], 1);
            last_at[tid] = before == parts - 1;
        }
        __syncthreads();
        if (!last_at[slice]) {
            publish(own);
            if (tid == 0) last_at[slice] = atomicAdd(&tickets[slice], 1) == parts - 1;
            __syncthreads();
        }
    }
    unsigned mine = all_units;                         // a whole tile is one run
    if (parts > 1) {
        mine = 0;
        for (int j = 0; j < parts; ++j) {
            if (!last_at[j]) continue;
            mine |= run(j);
            if (tid == 0) __hip_atomic_store(&tickets[j], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // all have been here: leave it clean
        }
        mine = __builtin_amdgcn_readfirstlane(mine);
        if (mine == 0) return;
    }
    const int cl0 = wx * 64 + grp * 32 + li;           // this lane's columns of the tile: cl0, cl0 + 16
    QkvColumn q_cols[CW];                              // all requested before the first store, which they might alias
    if constexpr (MODE == MODE_QKV_ROPE) {
#pragma unroll
        for (int tt = 0; tt < CW; ++tt) q_cols[tt].load(a, cb * kTileN + cl0 + 16 * tt);
        fixed_here();
    }
#pragma unroll
    for (int tt = 0; tt < CW; ++tt) {
        const unsigned units = mine >> (tt * kUnits) & ((1u << kUnits) - 1);
        if (units == 0) continue;
        f32x4 sum[RW];
        if (parts == 1) {
#pragma unroll
            for (int r = 0; r < RW; ++r) sum[r] = fin[r][tt];
        } else {
#pragma unroll
            for (int r = 0; r < RW; ++r) sum[r] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int part = 0; part < parts; ++part) {                 // in the order of the parts, whoever adds them up
                if (part == slice) {                                   // (its own it still has in registers)
#pragma unroll
                    for (int r = 0; r < RW; ++r) sum[r] += fin[r][tt];
                    continue;
                }
                u32x4 v[RW];
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    v[r] = u32x4{0, 0, 0, 0};
                    if (units >> (r % kUnits) & 1) v[r] = __builtin_amdgcn_raw_buffer_load_b128(pr.buf, 16 * tid, part * kPartBytes + (r * CW + tt) * 16 * kThreads, kAgent);
                }
#pragma unroll
                for (int r = 0; r < RW; ++r) sum[r] += __builtin_bit_cast(f32x4, v[r]);
            }
        }
        if constexpr (MODE == MODE_QKV_ROPE) {
            if (a.kv_dtype == 0) store_qkv<float>(a, sum, q_cols[tt], units, 2 * rb + wy, cb * kTileN + cl0 + 16 * tt, inv_rms[cl0 + 16 * tt]);
            else store_qkv<f16_t>(a, sum, q_cols[tt], units, 2 * rb + wy, cb * kTileN + cl0 + 16 * tt, inv_rms[cl0 + 16 * tt]);
        } else store_tiles<MODE>(a, sum, units, rb * OT + wy * (RW / SW), tiles, cb * kTileN + cl0 + 16 * tt, a.ssq_in ? inv_rms[cl0 + 16 * tt] : 1.0f);
    }
#endif
}

// ---------------- yardstick: what the matrix cores sustain ----------------
// A loop of eight waves, 64 x 64 per wave (32 MFMAs per wave and stage), on fragments that (mode >= 1) are re-read from a fixed LDS
// buffer every stage, (mode 2) with a workgroup barrier per stage: plainer than the kernel's loop above, with 12 reads for 32 MFMAs
// where that has 16 for 64.  One workgroup per launched block, no global
// memory traffic but one word per wave at the end.
constexpr int kYardRows = 4, kYardPitch = 64, kYardPlane = 128 * kYardPitch, kYardA = 256 * kYardPitch, kYardStage = kYardA + 2 * kYardPlane;
struct YardFrags { u32x4 a[kYardRows], bh[4], bl[4]; };
__device__ __forceinline__ void yard_read(YardFrags& f, uint32_t A, uint32_t B) {
    f.a[0] = lds_read_frag<0>(A); f.a[1] = lds_read_frag<1024>(A); f.a[2] = lds_read_frag<2048>(A); f.a[3] = lds_read_frag<3072>(A);
    f.bh[0] = lds_read_frag<0>(B);      f.bl[0] = lds_read_frag<kYardPlane>(B);
    f.bh[1] = lds_read_frag<1024>(B);   f.bl[1] = lds_read_frag<kYardPlane + 1024>(B);
    f.bh[2] = lds_read_frag<2048>(B);   f.bl[2] = lds_read_frag<kYardPlane + 2048>(B);
    f.bh[3] = lds_read_frag<3072>(B);   f.bl[3] = lds_read_frag<kYardPlane + 3072>(B);
}
__device__ __forceinline__ void yard_pin(YardFrags& f) {
#pragma unroll
    for (int r = 0; r < 4; ++r) { pin_frag(f.a[r]); pin_frag(f.bh[r]); pin_frag(f.bl[r]); }
}
template <int V>
__global__ __launch_bounds__(512, 2) void mfma_yardstick_kernel(float* __restrict__ sink, int stages) {
    constexpr int RWY = kYardRows;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
    unsigned* words = reinterpret_cast<unsigned*>(prompt_lds);
    for (int i = tid; i < kYardStage / 4; i += 512) words[i] = 0x3c003c00u ^ ((unsigned)i * 2654435761u & 0x00ff00ffu);   // bf16 values near 1
    __syncthreads();
    const uint32_t slot = (uint32_t)((lg ^ ((li >> 2) & 3)) << 4);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)prompt_lds;
    const uint32_t A = lds0 + ((wave >> 1) * 16 * RWY + li) * kYardPitch + slot, B = lds0 + kYardA + ((wave & 1) * 64 + li) * kYardPitch + slot;
    f32x4 acc[RWY][4];
#pragma unroll
    for (int r = 0; r < RWY; ++r)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) acc[r][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
    YardFrags f0, f1;
    yard_read(f0, A, B);
    lds_reads_left<0>();
    yard_pin(f0);
    f1 = f0;
    auto half = [&](YardFrags& cur, YardFrags& nxt) {
        if (V >= 1) lds_reads_left<0>();
        if (V >= 2) __syncthreads();
        if (V >= 1) yard_read(nxt, A, B);
        yard_pin(cur);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
            for (int r = 0; r < RWY; ++r) {            // both planes of an accumulator back to back, as the kernel above does (mma_hl)
                acc[r][tt] = mfma(cur.a[r], cur.bh[tt], acc[r][tt]);
                acc[r][tt] = mfma(cur.a[r], cur.bl[tt], acc[r][tt]);
                fixed_here();
            }
        }
    };
    for (int t = 0; t < stages; t += 2) { half(f0, f1); half(f1, f0); }
    lds_reads_left<0>();
    yard_pin(f0);
    float sum = __uint_as_float(f0.a[0][0]);
#pragma unroll
    for (int r = 0; r < RWY; ++r)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) sum += acc[r][tt][0] + acc[r][tt][3];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) sink[blockIdx.x * 8 + wave] = sum;
}

// Which tiles of a launch are cut into K parts, and how many.  A workgroup occupies a compute unit, so whole tiles take rounds of
// one tile per compute unit; the tiles of the last, partly filled round are cut so that their parts fill it.  What a part costs
// beside its stages (1.15 us each, 1.4 with all compute units busy): its start, the exchange of the accumulators (128 KB per workgroup each
// way) and a share of the finishing, counted as 10 + 2 ks stages.  Measured (us between events), whole / the last round in parts: 7B
// shape, 812 columns, QKV 336 tiles 172 / 153, gate/up 602 tiles 269 / 246; 512 columns, gate/up 344 tiles 183 / 158; fewer tiles than compute
// units, whole / 2 / 3 / 4 / 5 / 6 / 8 parts: 7B O at 203 columns (32 tiles) 88 / 55 / 48 / 39 / 44 / 47 / 45, down 203 / 116 / 88 / 77 /
// 74 / 71 / 70, at 700 (96 tiles) O 91 / 60 / 88 / 82 / 80 / 91 / 92, 70B O at 203 (64 tiles) 170 / 99 / 85 / 74 / 110 / 106 / 106: the rule's
// choice is within 4 us of the best of each.
struct PromptSplit { int n_whole, ks, cut_rounds = 0, cut_cost = 0; };
PromptSplit prompt_split(int tiles_wg, int n_stages, int n_cu, int forced, bool can_split) {
    auto fits = [&](int n, int ks) { return can_split && 2 * ks <= n_stages && n * ks <= kGemmPartTickets && n * ks * kPromptPartTile <= kPromptPartBytes; };
    if (forced >= 1) return forced > 1 && fits(tiles_wg, forced) ? PromptSplit{0, forced} : PromptSplit{tiles_wg, 1};
    const int rest = tiles_wg % n_cu;
    PromptSplit best{tiles_wg, 1};
    int best_cost = n_stages;                          // of the last round, in stages
    for (int ks = 2; ks <= kPromptMaxParts && rest > 0; ++ks) {
        if (!fits(rest, ks) || n_stages / ks < 8) break;
        const int rounds = (rest * ks + n_cu - 1) / n_cu, cost = rounds * ((n_stages + ks - 1) / ks + 10 + 2 * ks);
        if (cost < best_cost) { best = PromptSplit{tiles_wg - rest, ks, rounds, cost}; best_cost = cost; }
    }
    return best;
}

// What a launch of this kernel costs, in stages with few compute units busy, to compare with gemm_prompt_256_cost.  Both were fitted to kernel traces of the four
// projections at the 7B, 13B and 70B widths, and checked on nine widths of 1024 to 8192, 200 to 4096 columns, 700 launches timed with either kernel: the choice, which wants
// kPromptLargeGain, is nowhere the larger tiles where they are slower by more than 0.7 %, stays with the smaller where the others are up to 15 % faster (down projections of
// 2048 and 3072 wide models at 2500 columns and more, of the 70B widths at 812), and costs 0.3 % on average.  Beside its stages a whole tile costs its start and its epilogue, most of all where it reads
// and writes the residual.  A stage of the other kernel
// is 64 k of 256 columns: 1.9 of this one's, which is where that kernel gains; its tiles are twice as large, so it loses where they leave compute units
// idle or K parts have to be exchanged.  Measured, this kernel / the other, us: 7B gate/up 183 / 295 (616 columns), 274 / 267 (1024), 526 / 492 (2048), 1031 / 947
// (4096), down 100 / 143, 138 / 165, 257 / 274, 523 / 480; 70B gate/up 649 / 644 (512), 2482 / 2341 (2048), 5154 / 4697 (4096), down 358 / 355, 1334 / 1210, 2691 / 2432; 2048 wide
// QKV 87 / 99 (1800, 192 of the larger tiles), 169 / 174 (4096), gate/up 87 / 91 (700), 102 / 94 (1024), 397 / 357 (4096).
double prompt_cost(int mode, int n_stages, int n_cu, const PromptSplit& sp) {
    const double tile = mode == MODE_SWIGLU ? 9 : mode == MODE_RESID ? 14 : 11, stage = mode == MODE_RESID ? 1.08 : 1.04;
    return (sp.n_whole + n_cu - 1) / n_cu * (stage * n_stages + tile) + stage * sp.cut_cost;
}

constexpr double kPromptLargeGain = 0.985;     // of the smaller tiles' cost: the estimate is no better than that
// Both kernels' costs of a launch; the measurements' overrides make one of them infinite.
struct PromptCosts { double small, large; };
PromptCosts prompt_costs(int mode, int total_rows, int K, int ncols, size_t part_bytes, int n_cu, const Tuning& tn) {
    const int tiles = total_rows / 16, ot = mode == MODE_SWIGLU ? 8 : 16, n_rb = (tiles + ot - 1) / ot, n_cb = (ncols + kTileN - 1) / kTileN, n_stages = K / (2 * kBK) * 2;
    PromptCosts c{prompt_cost(mode, n_stages, n_cu, prompt_split(n_rb * n_cb, n_stages, n_cu, tn.prompt_ks, part_bytes > 0)), HUGE_VAL};
    if (tn.prompt_tile == 256 || (tn.prompt_tile == 0 && tn.prompt_ks == 0 && tn.prompt_cus == 0)) c.large = gemm_prompt_256_cost(mode, total_rows, K, ncols, part_bytes, n_cu);
    if (tn.prompt_tile == 256 && c.large < HUGE_VAL) c.small = HUGE_VAL;
    return c;
}

template <int MODE>
int launch_prompt(const GemvArgs& a, int n_rb, int n_cb, PromptSplit sp, hipStream_t s) {
    constexpr int lds = kPromptLds;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_prompt_kernel<MODE>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return (int)attr;
    const int grid = sp.n_whole + (n_rb * n_cb - sp.n_whole) * sp.ks;
    hipLaunchKernelGGL(gemm_prompt_kernel<MODE>, dim3(grid), dim3(kThreads), lds, s, a, TileOrder(n_rb, n_cb, sp.n_whole, sp.ks));
    return (int)hipGetLastError();
}

}  // namespace

// Requirements: those of launch_gemm_mfma (bf16 weights, K % 32 == 0, row counts multiples of 16), K >= 128, 1 <= ncols <=
// kPassCols (x_split holds ncols columns rounded up to 128, in either form); one matrix in MODE_RESID; with ssq_out at most kSsqStride row blocks.  MODE_QKV_ROPE: head_dim
// 128, ssq_in, col_at and rope_cs set, only q is written to out.
// Up to 128 columns the panel kernel is the other choice.  It slows down past 64 (its LDS pipe, or two launches of 64), the LDS-tiled
// kernel takes one column block whatever its width and wants row blocks.  Measured at 65 / 77 / 128 columns (us between events, panel -> LDS-tiled): 48 or
// more row blocks: 7B QKV 64 / 66 / 69 -> 47 / 48 / 54, gate/up 105 / 105 / 109 -> 71 / 72 / 73, 13B QKV 79 / 79 / 85 -> 59 / 61 / 65, 70B gate/up 316 /
// 316 / 326 -> 232 / 235 / 241; 32: 70B O 84 / 86 / 90 -> 71 / 74 / 79, down 216 / 218 / 225 -> 158 / 159 / 166; 20: 13B O 44 / 45 / 48 -> 42 /
// 41 / 45, down 90 / 91 / 93 -> 82 / 84 / 90; 16: 7B O 32 / 33 / 36 -> 42 / 42 / 43, down 61 / 61 / 64 -> 68 / 66 / 70.  At 64 columns the
// panel kernel needs half its time at 65 (one launch) and is ahead everywhere.
bool gemm_prompt_takes(const GemvArgs& a, int mode, const Tuning& tn) {
    const int row_blocks = a.total_rows / (mode == MODE_SWIGLU ? kTileM / 2 : kTileM);
    return a.K >= 2 * kBK && a.part && tn.mfma_wide && (a.ncols > 128 || (a.ncols > 64 && row_blocks >= tn.prompt_row_blocks));
}

bool prompt_takes_large_tiles(int mode, int total_rows, int K, int ncols, size_t part_bytes, int n_cu, const Tuning& tn) {
    const PromptCosts c = prompt_costs(mode, total_rows, K, ncols, part_bytes, n_cu, tn);
    return c.large < kPromptLargeGain * c.small;
}

bool prompt_pass_in_lines(const PromptDims& d, int ncols, size_t part_bytes, int n_cu, const Tuning& tn) {
    if (!tn.mfma_wide || ncols <= 128 || std::min(std::min(d.d_model, d.q_dim), d.d_ffn) < 2 * kBK) return false;      // all of its projections have to read this form
    const struct { int mode, rows, K; } launches[] = {{d.rope_in_qkv ? MODE_QKV_ROPE : MODE_STORE, d.qkv_rows, d.d_model}, {MODE_RESID, d.d_model, d.q_dim},
                                                      {MODE_SWIGLU, d.d_ffn, d.d_model}, {MODE_RESID, d.d_model, d.d_ffn}};
    double small = 0, best = 0;
    for (const auto& l : launches) {
        const PromptCosts c = prompt_costs(l.mode, l.rows, l.K, ncols, part_bytes, tn.prompt_cus ? tn.prompt_cus : n_cu, tn);
        small += c.small;
        best += c.large < kPromptLargeGain * c.small ? c.large : c.small;
    }
    return best < kPromptLargeGain * small;
}

int launch_gemm_prompt(const GemvArgs& a, int mode, int n_cu, const Tuning& tn, hipStream_t s, int* n_groups) {
    const int tiles = a.total_rows / 16;
    const int n_cb = (a.ncols + kTileN - 1) / kTileN;
    if (a.ncols < 1 || a.ncols > kPassCols || a.K % 32 != 0 || a.K < 2 * kBK) return (int)hipErrorInvalidValue;
    const int ot = mode == MODE_SWIGLU ? 8 : 16;       // output row tiles per workgroup: 256 slab rows
    const int n_rb = (tiles + ot - 1) / ot;
    if (a.ssq_out && n_rb > kSsqStride) return (int)hipErrorInvalidValue;
    if (n_groups) *n_groups = n_rb;
    const int n_stages = a.K / (2 * kBK) * 2, tiles_wg = n_rb * n_cb;
    const int cus = tn.prompt_cus ? tn.prompt_cus : n_cu;
    const bool parts = a.part && a.part_tickets;
    if (mode == MODE_QKV_ROPE && (a.hd != 128 || !a.ssq_in || !a.col_at || !a.rope_cs || (a.kv_dtype != 0 && a.kv_dtype != 2))) return (int)hipErrorInvalidValue;
    if (a.x_form.lines()) {
        if ((mode == MODE_RESID || a.ssq_in) && prompt_takes_large_tiles(mode, a.total_rows, a.K, a.ncols, parts ? a.part_bytes : 0, cus, tn))
            return launch_gemm_prompt_256(a, mode, cus, s, n_groups);
    }
    const PromptSplit sp = prompt_split(tiles_wg, n_stages, cus, tn.prompt_ks, parts);
    if (mode == MODE_STORE) return launch_prompt<MODE_STORE>(a, n_rb, n_cb, sp, s);
    if (mode == MODE_QKV_ROPE) return launch_prompt<MODE_QKV_ROPE>(a, n_rb, n_cb, sp, s);
    if (mode == MODE_SWIGLU) return launch_prompt<MODE_SWIGLU>(a, n_rb, n_cb, sp, s);
    return launch_prompt<MODE_RESID>(a, n_rb, n_cb, sp, s);
}

// mode 0: MFMAs alone; 1: with LDS fragment reads, 12 for 32 MFMAs; 2: with a workgroup barrier per stage as well.  n_wg workgroups of
// eight waves; sink holds 8 floats per workgroup.  Flops issued: n_wg * 8 waves * stages * 32 MFMAs * 16384.
int launch_mfma_yardstick(int mode, int stages, int n_wg, float* sink, hipStream_t s) {
    constexpr int lds = kYardStage;
    if (mode < 0 || mode > 2 || stages < 2 || stages % 2 != 0) return (int)hipErrorInvalidValue;
    if (mode == 0) hipLaunchKernelGGL(mfma_yardstick_kernel<0>, dim3(n_wg), dim3(512), lds, s, sink, stages);
    else if (mode == 1) hipLaunchKernelGGL(mfma_yardstick_kernel<1>, dim3(n_wg), dim3(512), lds, s, sink, stages);
    else hipLaunchKernelGGL(mfma_yardstick_kernel<2>, dim3(n_wg), dim3(512), lds, s, sink, stages);
    return (int)hipGetLastError();
}

}  // namespace d3
