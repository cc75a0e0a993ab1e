// Tiled GEMM of the prompt pass for launches of many tiles: out[col][row] = sum_k W[row][k] * x[col][k] as in gemm_prompt.hip, with tiles of 256 weight
// rows x 256 columns, one workgroup of eight waves per compute unit that stays for all of its tiles.
//
// What bounds it and set the design.  In the smaller tiles' kernel (256 x 128) the matrix cores are busy for 2048 of a stage's 2280 clocks, but at 1.79 GHz:
// the clock is what the power leaves.  Taken out one at a time there (7B gate/up, 2048 columns, 1.29 us a stage): all direct loads 1.02 us (2079
// clocks, 2.03 GHz), the loads of weights 1.12, the memory behind the L2 (the same two stages over and over) 1.19, the reads of weight fragments another 0.04.  So moving
// operands into the LDS costs a fifth of the time, most of it as power.  A tile twice as wide moves 48 KB where that moves 64: 64 k of 128 columns' worth
// takes 1.23 us (2235 clocks, 1.81 GHz).
//  * A step is 32 k: 64 MFMAs per wave, each wave 128 rows x 64 columns, all of them all of K (there the two halves of the workgroup split K and exchanged 64 KB
//    through LDS in the end).  Weights come 64 k at a time, whole cache lines of their rows, into one of three slabs of 32 KB, activations 32 k at a time, which
//    with their two halves side by side are a line of each column as well, into one of two slabs of 32 KB.
//  * Between two tiles the matrix cores would idle for the first loads of the second, 4 us: the loads run ahead into the workgroup's next tile, while the epilogue works from
//    registers and, for residual projections, in the one slab that is free then.
//  * Tiles do not fill whole rounds of compute units; see Order256.
// 2048 (4096) columns, kernel trace, from gemm_prompt.hip's kernel to this, us: 7B gate/up 526 -> 492 (1031 -> 947), QKV 291 -> 295 (586 -> 546), O 110 -> 129 (216 ->
// 202), down 257 -> 274 (523 -> 480); 70B 2482 -> 2341 (5154 -> 4697), 474 -> 473 (972 -> 897), 382 -> 363 (761 -> 724), 1334 -> 1210 (2691 -> 2432): launch_gemm_prompt
// estimates both.  Not kept: helpers' stages cut evenly over K (see Order256); the XCDs' tiles left over first on every other XCD, so that epilogues meet less often (75.9 ->
// 76.6 ms, 32 x 2048 columns, 2 blocks); passes of 8192 columns (74.7 -> 74.9 ms; 2048: 79).
//
// The LDS reads are inline assembly with waits written out, for the reasons given there; tests/test_prompt_kernel_registers.py follows them through this
// kernel's compiled code as well.
#include <algorithm>
#include <cmath>

#include "gemm_prompt.h"

namespace d3 {

namespace {

constexpr int kTileM = 256, kTileN = 256;
constexpr int kWSlab = kTileM * kPitch;        // 64 k of 256 weight rows
constexpr int kXSlab = kTileN * kPitch;        // 32 k of 256 columns, hi and lo halves
constexpr int kLdsX = 3 * kWSlab;              // LDS: three weight slabs, two activation slabs
constexpr int kLds = kLdsX + 2 * kXSlab;       // 160 KB, all there is
[[maybe_unused]] constexpr int kLoads = 4;                      // direct loads per wave and slab
[[maybe_unused]] constexpr size_t kPartBytes = (size_t)kTileM * kTileN * 4;
constexpr int kMinPart = 4;                    // fewest stages of a part (the pipeline's depth is three)

// Tiles in launch order, and who does what.  Workgroup w takes tile `round * n_wg + w` of every full round.  The tiles that are left, `rest` of them, are
// fewer than the workgroups: each has a main workgroup, which takes its last `main` stages, and the other workgroups share the stages before those, laid
// end to end.  So all mains walk K in step, and nearly all helpers: cut anywhere, as even shares of the stages laid end to end would be, the tiles of an
// XCD are at as many places of K as it has workgroups and share nothing in its L2 (7B gate/up, 2048 columns: 2.95 us a stage against 2.45).
// An XCD's workgroups are neighbours in w, and groups of kGroupR row blocks are walked column block by column block, so that the tiles an XCD works on at
// a time share their slabs.
constexpr int kGroupR = 8;
struct Order256 {
    int n_rb, n_cb, stages, n_wg, rounds, rest, main, helpers;
    Divisor by_helped, by_helpers, group, last_group;
    Order256() = default;
    // A main's stages.  Each part a helper has costs it some 4 stages beside its own (9 us: publishing 256 KB and counting itself in), and the main
    // that finds them some 6 (reading them, finishing the tile).
    static int main_share(int rest, int st, int wg) {
        const double tiles = (double)rest / (wg - rest);               // of a helper
        return std::min(st, (int)std::ceil((tiles * st + 4 * (tiles + 1) - 6) / (1 + tiles)));
    }
    Order256(int rb, int cb, int st, int wg, bool split)
        : n_rb(rb), n_cb(cb), stages(st), n_wg(wg), rounds(split ? rb * cb / wg : (rb * cb + wg - 1) / wg), rest(split ? rb * cb % wg : 0),
          main(main_share(rest, st, wg)), helpers(wg - rest), by_helped(st - main > 0 ? st - main : 1), by_helpers(helpers), group(kGroupR * cb),
          last_group(rb % kGroupR ? rb % kGroupR : kGroupR) {}
    // first stage of helper h in the line of the stages that helpers take: even shares, but no part of a tile below kMinPart stages
    __host__ __device__ __forceinline__ int begin(int h) const {
        const int helped = by_helped.d, at = by_helpers.of(rest * helped * h), in = at - by_helped.of(at) * helped;
        return in < kMinPart ? at - in : helped - in < kMinPart ? at + helped - in : at;
    }
};
// a barrier that waits for this wave's LDS accesses but not for its stores
__device__ __forceinline__ void lds_barrier() { lds_reads_left<0>(); __builtin_amdgcn_s_barrier(); asm volatile("" ::: "memory"); }

struct Unit { int tile, s0, n; };              // stages [s0, s0 + n) of a tile

struct Args256 { GemvArgs a; Order256 order; };
#ifdef __HIP_DEVICE_COMPILE__
// The kernel's arguments, read again: kept in registers across the loop over units they would be spilled (they are needed between the units only).
__device__ __forceinline__ Args256 args_again() {
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    typedef const __attribute__((address_space(4))) uint64_t* Words;
    constexpr int n = sizeof(Args256) / 8;
    static_assert(sizeof(Args256) % 8 == 0, "");
    struct Raw { uint64_t word[n]; } raw;
#pragma unroll
    for (int i = 0; i < n; ++i) raw.word[i] = ((Words)p)[i];
    return __builtin_bit_cast(Args256, raw);
}
#endif

template <int MODE>
__global__ __launch_bounds__(kThreads, 2) void gemm_prompt_256_kernel(Args256) {
#ifdef __HIP_DEVICE_COMPILE__
    constexpr int SW = (MODE == MODE_SWIGLU) ? 2 : 1;
    constexpr int OT = 2 * RW / SW;                    // output row tiles per workgroup (half as many gate/up pairs)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wy = wave8 >> 2, wx = wave8 & 3;         // the wave's 128 rows and 64 columns of the tile
    const int li = lane & 15, lg = lane >> 4;
    // ---- this workgroup's units ----
    int wg, round = 0, main_tile = -1, helper = 0, pos = 0, end = 0;
    const Args256 args0 = args_again();
    const int K = args0.a.K;
    {
        const Order256& order = args0.order;
        const int per_xcd = order.n_wg >> 3, xcd = blockIdx.x & 7, in_xcd = blockIdx.x >> 3;      // workgroups go to the XCDs round-robin
        wg = xcd * per_xcd + in_xcd;
        const int t0 = order.rest * xcd >> 3, t1 = order.rest * (xcd + 1) >> 3;                // the XCD's mains come first
        if (in_xcd < t1 - t0) main_tile = t0 + in_xcd;
        else if (order.rest) { helper = wg - t1; pos = order.begin(helper); end = order.begin(helper + 1); }
    }
    auto take = [&](const Order256& order, Unit& u) -> bool {
        if (round < order.rounds) {
            u.tile = round++ * order.n_wg + wg; u.s0 = 0; u.n = order.stages;
            return u.tile < order.n_rb * order.n_cb;
        }
        if (main_tile >= 0) {
            u.tile = order.rounds * order.n_wg + main_tile; u.s0 = order.by_helped.d; u.n = order.main;
            main_tile = -1;
            return true;
        }
        if (pos >= end) return false;
        const int helped = order.by_helped.d, t = order.by_helped.of(pos);
        u.tile = order.rounds * order.n_wg + t;
        u.s0 = pos - t * helped;
        u.n = min(helped - u.s0, end - pos);
        pos += u.n;
        return true;
    };
    auto place = [&](const Order256& order, int tile, int& rb, int& cb) {
        const int g = order.group.of(tile), rem = tile - g * order.group.d;
        int row;
        if (kGroupR * (g + 1) <= order.n_rb) { cb = rem / kGroupR; row = rem % kGroupR; }
        else { cb = order.last_group.of(rem); row = rem - cb * order.last_group.d; }
        rb = kGroupR * g + row;
    };
    Unit cur{}, nxt{};
    if (!take(args0.order, cur)) return;

    // ---- loads: a wave's eight-row blocks of a slab are wave8, wave8 + 8, ...; lane l of a load: row l / 8 of the block, LDS position l % 8, i.e. segment
    // (l % 8) ^ ((slab row / 2) % 8) of that row.  They run ahead of the arithmetic and into the next unit: activations (32 k at a time) two k-steps,
    // weights (64 k) three slabs.  Past the last unit nothing is fetched (a range of zero bytes). ----
    const int prow = lane >> 3, pseg = (lane & 7) ^ ((lane >> 4) | (4 * (wave8 & 1)));
    const int pitch_x = 4 * K, voff_w = 2 * (prow * K + pseg * 8), voff_x = (8 * wave8 + prow) * pitch_x + pseg * 16;
    __amdgpu_buffer_rsrc_t src_w[kLoads], src_x;
    int at_w, at_x, step_w, step_x, rows_x;            // byte offsets into the rows, what they advance by; 64 columns
    auto point_w = [&](const Args256& args, const Unit& u, bool live) {
        const GemvArgs& a = args.a;
        const int tiles = a.total_rows / 16;           // output row tiles of the whole matrix
        int rb, cb;
        place(args.order, u.tile, rb, cb);
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            // Slab tile st = 8 wy + t is wave row wy's tile t.  Plain modes: output tile OT rb + st.  SwiGLU: tiles t < 4 are gate rows, the others the up
            // rows of the same outputs OT rb + 4 wy + t % 4.  Tiles past the matrix re-read the last one (result dropped).
            const int blk = wave8 + kWaves * j, st = blk >> 1, t = st % RW;
            int otile = MODE == MODE_SWIGLU ? rb * OT + (st / RW) * (RW / 2) + t % (RW / 2) : rb * OT + st;
            otile = otile < tiles ? otile : tiles - 1;
            int local = otile * 16;
            const void* w = MODE == MODE_SWIGLU && t >= RW / 2 ? a.w[1] : a.w[0];
            if (MODE != MODE_SWIGLU && MODE != MODE_RESID && local >= a.rows[0]) {
                local -= a.rows[0];
                w = a.w[1];
                if (local >= a.rows[1]) { local -= a.rows[1]; w = a.w[2]; }
            }
            const bf16_t* p = static_cast<const bf16_t*>(w) + (size_t)(local + 8 * (blk & 1)) * K;
            src_w[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, live ? 2 * 8 * K : 0, 0x00027000);
        }
        at_w = live ? u.s0 * kPitch : 0;
        step_w = live ? kPitch : 0;
    };
    auto point_x = [&](const Args256& args, const Unit& u, bool live) {
        int rb, cb;
        place(args.order, u.tile, rb, cb);
        src_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(args.a.x_split) + (size_t)(cb * kTileN) * 2 * K, 0, live ? kTileN * pitch_x : 0, 0x00027000);
        at_x = live ? u.s0 * 2 * kPitch : 0;
        step_x = live ? kPitch : 0;
        rows_x = live ? 64 * pitch_x : 0;
    };
    auto lds_at = [&](int at) { return (__attribute__((address_space(3))) void*)((lds_char*)prompt_lds + at + wave8 * 1024); };
    auto load_w = [&](int j, int slab) { __builtin_amdgcn_raw_ptr_buffer_load_lds(src_w[j], lds_at(slab + j * kWaves * 1024), 16, voff_w, at_w, 0, 0); };
    auto load_x = [&](int j, int buf) { __builtin_amdgcn_raw_ptr_buffer_load_lds(src_x, lds_at(kLdsX + buf * kXSlab + j * kWaves * 1024), 16, voff_x, at_x + j * rows_x, 0, 0); };

    int w0 = 0, w1 = kWSlab, w2 = 2 * kWSlab;          // the weight slabs of this stage and the next two
    point_w(args0, cur, true);
#pragma unroll
    for (int j = 0; j < kLoads; ++j) load_w(j, w0);
    fixed_here();
    point_x(args0, cur, true);
#pragma unroll
    for (int j = 0; j < kLoads; ++j) load_x(j, 0);
    at_x += step_x;
    fixed_here();
#pragma unroll
    for (int j = 0; j < kLoads; ++j) load_x(j, 1);
    at_w += step_w;
#pragma unroll
    for (int j = 0; j < kLoads; ++j) load_w(j, w1);
    at_w += step_w;
    load_w(0, w2); load_w(1, w2);
    fixed_here();
    bool more = take(args0.order, nxt);

    // ---- fragment reads: lane (i, g) takes segment 4 k-step + g of row i of a weight tile, segments g and 4 + g of column i (tile bases are multiples of
    // 16 rows, so the swizzle depends on i alone) ----
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)prompt_lds, slot = (uint32_t)((lg ^ ((li >> 1) & 7)) << 4);
    const uint32_t a_step0 = lds0 + (wy * 16 * RW + li) * kPitch + slot, a_step1 = a_step0 ^ kLoBit;
    const uint32_t b_hi = lds0 + kLdsX + (wx * 64 + li) * kPitch + slot, b_lo = b_hi ^ kLoBit;

    f32x4 acc[RW][4];                                  // [row tile of the wave][column tile of the wave]
    u32x4 A0[RW], A1[RW];                              // weight fragments of this k-step and the next
    PromptB f0, f1, f2;                                // activation fragments of three column tiles
    // One k-step (32 k), the first (STEP 0) or the second of a weight slab; its activations are in buffer STEP.  As in the smaller tiles' kernel: four slots
    // of 16 MFMAs, the barrier ahead of the third, when every wave has read all of the step's fragments; behind it the loads into what is free
    // now (the activation buffer; after the slab's second step the slab too, half of whose loads wait for the next step) and the first reads of the next
    // step.  LAST: the unit's last step, whose successor's fragments are read after the epilogue, and whose slab the epilogue uses.
    auto step = [&](auto step_c, auto last_c, int arrived, u32x4 (&A)[RW], u32x4 (&An)[RW], PromptB& X, PromptB& Y, PromptB& Z) {
        constexpr int STEP = decltype(step_c)::value;
        constexpr bool LAST = decltype(last_c)::value;
        constexpr int CUR = STEP * kXSlab, NEXT = (STEP ^ 1) * kXSlab;
        const uint32_t Wn = STEP == 0 ? a_step1 + w0 : a_step0 + w1;
        // slot 0: the weight fragments are used in the order of their arrival
        __builtin_amdgcn_s_setprio(1);
        read_b_frags<1, CUR>(Y, b_hi, b_lo);
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
        read_b_frags<2, CUR>(Z, b_hi, b_lo);
        lds_reads_left<2>(); pin_frag(Y.h); pin_frag(Y.l);
        mma_hl<0, 2>(acc, 1, A, Y); fixed_here();
        read_b_frags<3, CUR>(X, b_hi, b_lo); fixed_here();
        mma_hl<2, 6>(acc, 1, A, Y); fixed_here();
        // slots 2 and 3: this wave has read all of the step
        lds_reads_left<0>(); pin_frag(Z.h); pin_frag(Z.l); pin_frag(X.h); pin_frag(X.l);
        // the next step's activations have landed, and its slab if it begins one: only the last two loads of weights may be on their way
        asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 .Larrived%=\n\ts_waitcnt vmcnt(2)\n.Larrived%=:" :: "s"(__builtin_amdgcn_readfirstlane(arrived)) : "memory", "scc");
        __builtin_amdgcn_s_barrier();
        at_x += step_x;
        if (STEP == 1 && !LAST) at_w += step_w;
        const int slab = STEP == 0 ? w2 : w0, j0 = STEP == 0 ? 2 : 0;
        __builtin_amdgcn_s_setprio(3);
        mma_hl<0, 1>(acc, 2, A, Z); fixed_here(); load_x(0, STEP); fixed_here();
        mma_hl<1, 1>(acc, 2, A, Z); fixed_here(); load_x(1, STEP); fixed_here();
        mma_hl<2, 1>(acc, 2, A, Z); fixed_here(); load_x(2, STEP); fixed_here();
        mma_hl<3, 1>(acc, 2, A, Z); fixed_here(); load_x(3, STEP); fixed_here();
        mma_hl<4, 1>(acc, 2, A, Z); fixed_here(); if (!LAST) load_w(j0, slab); fixed_here();
        mma_hl<5, 1>(acc, 2, A, Z); fixed_here(); if (!LAST) load_w(j0 + 1, slab); fixed_here();
        mma_hl<6, 1>(acc, 2, A, Z); fixed_here();
        if constexpr (LAST) {
            mma_hl<7, 1>(acc, 2, A, Z); mma_hl<0, 8>(acc, 3, A, X); fixed_here();
        } else {
            read_b_frags<0, NEXT>(Y, b_hi, b_lo); fixed_here();
            mma_hl<7, 1>(acc, 2, A, Z); fixed_here(); An[0] = lds_read_frag<0>(Wn); fixed_here();
            __builtin_amdgcn_s_setprio(2);
            mma_hl<0, 1>(acc, 3, A, X); fixed_here(); An[1] = lds_read_frag<1 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<1, 1>(acc, 3, A, X); fixed_here(); An[2] = lds_read_frag<2 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<2, 1>(acc, 3, A, X); fixed_here(); An[3] = lds_read_frag<3 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<3, 1>(acc, 3, A, X); fixed_here(); An[4] = lds_read_frag<4 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<4, 1>(acc, 3, A, X); fixed_here(); An[5] = lds_read_frag<5 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<5, 1>(acc, 3, A, X); fixed_here(); An[6] = lds_read_frag<6 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<6, 1>(acc, 3, A, X); fixed_here(); An[7] = lds_read_frag<7 * 16 * kPitch>(Wn); fixed_here();
            mma_hl<7, 1>(acc, 3, A, X); fixed_here();
        }
        if (STEP == 1) {
            const int done = w0;
            w0 = w1; w1 = w2; w2 = done;
        }
    };
    static_assert(kLoads == 4 && RW == 8, "the step is written out for these");
    constexpr std::integral_constant<int, 0> first_step{};
    constexpr std::integral_constant<int, 1> second_step{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    vm_loads_left<2 * kLoads + 2>();                   // slab 0 and k-step 0 have landed: two sets of loads and a half are younger
    __builtin_amdgcn_s_barrier();
    bool fresh = true;                                 // nothing has waited for the second k-step of the first unit yet
    for (;;) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) acc[r][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
        read_b_frags<0>(f0, b_hi, b_lo);
        read_a_frags(A0, a_step0 + w0, std::make_integer_sequence<int, RW>{});
        all_arrived(A0); all_arrived(f0);
        const int n = cur.n;
#pragma unroll 1
        for (int s = 0; s + 1 < n; ++s) {
            step(first_step, no, s == 0 && !fresh, A0, A1, f0, f1, f2);
            if (s + 3 == n) { point_w(args_again(), nxt, more); at_w -= step_w; }                    // the next slab to request is the next unit's first
            step(second_step, no, 0, A1, A0, f1, f0, f2);
        }
        all_arrived(A0); all_arrived(f0);              // nothing in flight where the compiler may move registers
        point_x(args_again(), nxt, more);
        at_x -= step_x;
        step(first_step, no, 0, A0, A1, f0, f1, f2);
        step(second_step, yes, 1, A1, A0, f1, f0, f2);
        __builtin_amdgcn_s_setprio(0);

        fresh = false;
        // ---- the unit is multiplied; the slab w2 is free ----
        unsigned all_lanes = ~0u;                      // (the lane's number and what follows from it are worked out here, not kept in registers through the steps)
        asm volatile("" : "+s"(all_lanes));
        const int lane = __builtin_amdgcn_mbcnt_hi(all_lanes, __builtin_amdgcn_mbcnt_lo(all_lanes, 0));
        const int tid = wave8 * 64 + lane, li = lane & 15, lg = lane >> 4;
        int rb, cb;
        bool cut;
        {
            const Args256 args = args_again();
            place(args.order, cur.tile, rb, cb);
            cut = cur.n < args.order.stages;
        }
        const int col0 = cb * kTileN + wx * 64;        // the wave's first column
        float inv = 1.0f;                              // RMSNorm scale of column col0 + lane: its partial sums of squares in their order
        if (MODE != MODE_RESID) {
            const GemvArgs a = args_again().a;
            const float* p = a.ssq_in + (size_t)min(col0 + lane, a.ncols - 1) * kSsqStride;
            float ss = 0.f;
            for (int i0 = 0; i0 < a.ssq_parts; i0 += 32) {
                float4 q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) q[i] = *reinterpret_cast<const float4*>(p + min(i0 + 4 * i, (a.ssq_parts - 1) & ~3));
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int at = i0 + 4 * i;
                    if (at < a.ssq_parts) ss += q[i].x;
                    if (at + 1 < a.ssq_parts) ss += q[i].y;
                    if (at + 2 < a.ssq_parts) ss += q[i].z;
                    if (at + 3 < a.ssq_parts) ss += q[i].w;
                }
            }
            inv = 1.0f / sqrtf(ss / (float)a.K + a.eps);
        }
        vm_loads_left<0>();                            // what the next unit begins with has landed: its first steps need not wait for the stores below
        char* scratch = prompt_lds + w2;
        // K parts of a tile: its column tiles are dealt out to the parts in runs with an arrival counter each.  A part publishes the other parts' runs and counts
        // itself in, then looks at its own run: where all others have been, it adds that up and finishes it; else it publishes it too.  Whoever
        // arrives last at a run finishes it, so nobody waits; parts that end together finish a run each, and one that finds all others there (most
        // mains) finishes the tile without publishing anything.
        unsigned mine = 15;                            // column tiles to finish
        if (cut) {
            const Args256 args = args_again();
            const GemvArgs& a = args.a;
            const Order256& order = args.order;
            const int t = cur.tile - order.rounds * order.n_wg, helped = order.by_helped.d;
            const bool is_main = cur.s0 == helped;
            int last = helper;                         // of the helpers that have parts of the tile: to begin with, one of them
            if (is_main) {
                last = min(order.helpers - 1, t * order.helpers / order.rest);
                while (order.begin(last) > t * helped) --last;
                while (order.begin(last + 1) <= t * helped) ++last;
            }
            int first = last;
            while (order.begin(first) > t * helped) --first;
            while (order.begin(last + 1) < (t + 1) * helped) ++last;
            const int parts = last - first + 2, me = is_main ? parts - 1 : helper - first;     // in the order of K
            int* tickets = a.part_tickets + t * kPromptMaxParts;
            int* note = reinterpret_cast<int*>(scratch);
            auto part = [&](int p) {
                const size_t slot = p == parts - 1 ? order.rest + order.helpers + t : t + first + p;
                return __builtin_amdgcn_make_buffer_rsrc(a.part + slot * (kPartBytes / 4), 0, (int)kPartBytes, 0x00027000);
            };
            auto run = [&](int p) { return (1u << 4 * (p + 1) / parts) - (1u << 4 * p / parts); };
            auto publish = [&](unsigned tts) {
                const __amdgpu_buffer_rsrc_t own = part(me);
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    if (!(tts >> tt & 1)) continue;
#pragma unroll
                    for (int r = 0; r < RW; ++r)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[r][tt]), own, 16 * tid, (r * 4 + tt) * 16 * kThreads, kAgent);
                }
                wait_stores();                         // they have reached the coherence point
                __syncthreads();
            };
            if (tid < parts) note[tid] = __hip_atomic_load(&tickets[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            bool all_here = true;
            for (int p = 0; p < parts; ++p) all_here = all_here && note[p] == parts - 1;
            if (!is_main) {
                publish(15u);
                if (tid < parts) note[tid] = atomicAdd(&tickets[tid], 1);
                __syncthreads();
            } else if (!__builtin_amdgcn_readfirstlane(all_here)) {
                const unsigned own = run(me);
                publish(15u & ~own);
                if (tid < parts)
                    note[tid] = (tid == me ? __hip_atomic_load(&tickets[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : atomicAdd(&tickets[tid], 1));
                __syncthreads();
                if (__builtin_amdgcn_readfirstlane(note[me]) != parts - 1) {
                    publish(own);
                    if (tid == 0) note[me] = atomicAdd(&tickets[me], 1);
                    __syncthreads();
                }
            }
            mine = 0;
            for (int p = 0; p < parts; ++p) {
                if (__builtin_amdgcn_readfirstlane(note[p]) != parts - 1) continue;
                mine |= run(p);
                if (tid == 0) __hip_atomic_store(&tickets[p], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // all have been here: leave it clean
            }
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                if (!(mine >> tt & 1)) continue;
                f32x4 sum[RW];
#pragma unroll
                for (int r = 0; r < RW; ++r) sum[r] = f32x4{0.f, 0.f, 0.f, 0.f};
                for (int p = 0; p < parts; ++p) {      // in the order of the parts, whoever adds them up
                    if (p == me) {
#pragma unroll
                        for (int r = 0; r < RW; ++r) sum[r] += acc[r][tt];
                        continue;
                    }
                    const __amdgpu_buffer_rsrc_t other = part(p);
                    u32x4 v[RW];
#pragma unroll
                    for (int r = 0; r < RW; ++r) v[r] = __builtin_amdgcn_raw_buffer_load_b128(other, 16 * tid, (r * 4 + tt) * 16 * kThreads, kAgent);
#pragma unroll
                    for (int r = 0; r < RW; ++r) sum[r] += __builtin_bit_cast(f32x4, v[r]);
                }
#pragma unroll
                for (int r = 0; r < RW; ++r) acc[r][tt] = sum[r];
            }
            __syncthreads();                           // the notes have been read
        }
        if (mine) {
            const GemvArgs a = args_again().a;
            const int tiles = a.total_rows / 16, total_rows = a.total_rows;
            if constexpr (MODE == MODE_RESID) {
                // The wave's sums go through its own 4 KB of the free slab, 16 columns x 64 rows at a time, so that its loads and stores are 256 bytes in a row: rows
                // 4 u .. + 3 of column c are float4 u ^ c of the column.  Lane l then takes rows 4 (l % 16) .. + 3 of the columns 4 i + l / 16.
                f32x4* own = reinterpret_cast<f32x4*>(scratch + wave8 * 4096);
                const int u = lane & 15, c4 = lane >> 4;
                constexpr int kAhead = 1;              // groups whose old residual is on its way (two: spills, and no faster)
                float4 old[kAhead + 1][4];
                const int row_w = rb * kTileM + wy * 128 + 4 * u;
                auto clamped = [&](int hf) { return min(row_w + 64 * hf, total_rows - 4); };       // rows past the matrix compute on clamped addresses and store nothing
                auto column = [&](int tt, int i) { return col0 + 16 * tt + 4 * i + c4; };
                auto request = [&](int g) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        old[g % (kAhead + 1)][i] = *reinterpret_cast<const float4*>(a.out + (size_t)min(column(g >> 1, i), a.ncols - 1) * a.out_stride + clamped(g & 1));
                };
                float4 gain[2] = {make_float4(1.f, 1.f, 1.f, 1.f), make_float4(1.f, 1.f, 1.f, 1.f)};
                if (a.ssq_out) {
                    gain[0] = *reinterpret_cast<const float4*>(a.gain_next + clamped(0));
                    gain[1] = *reinterpret_cast<const float4*>(a.gain_next + clamped(1));
                }
#pragma unroll
                for (int g = 0; g < kAhead; ++g) request(g);
                float sq[4], total[4] = {};            // of a group's four columns, this lane's part; of a column tile's column 4 u + c4 (lanes u < 4), the 128 rows
#pragma unroll
                for (int g = 0; g < 8; ++g) {
                    const int tt = g >> 1, hf = g & 1;
                    if (g + kAhead < 8) request(g + kAhead);
                    fixed_here();
                    if (!(mine >> tt & 1)) continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r) own[li * 16 + ((4 * r + lg) ^ li)] = acc[4 * hf + r][tt];
                    __builtin_amdgcn_wave_barrier();
                    f32x4 sum[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[i] = own[(4 * i + c4) * 16 + (u ^ (4 * i + c4))];
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float4 o = old[g % (kAhead + 1)][i];
                        const float v[4] = {o.x + sum[i][0], o.y + sum[i][1], o.z + sum[i][2], o.w + sum[i][3]};
                        const bool live = row_w + 64 * hf < total_rows && column(tt, i) < a.ncols;
                        const float part = live ? (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]) : 0.f;
                        sq[i] = hf ? sq[i] + part : part;
                        if (live) {
                            store_row4(a.out + (size_t)column(tt, i) * a.out_stride + row_w + 64 * hf, v);
                            if (a.out_split) {         // a normalised projection reads it next: hand it x * gain (and sum(x^2) below)
                                const float4 gn = gain[hf];
                                const float w[4] = {v[0] * gn.x, v[1] * gn.y, v[2] * gn.z, v[3] * gn.w};
                                store_split4<SPLIT_LINES>(a.out_split + (size_t)column(tt, i) * 2 * a.out_stride, row_w + 64 * hf, w, kSplitLo);
                            }
                        }
                    }
                    if (hf && a.ssq_out) {             // 16 lanes hold a column
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float sum16 = reduce_row(sq[i], AddOp());
                            if (u == i) total[tt] = sum16;
                        }
                    }
                }
                if (a.ssq_out) {                       // the two waves of a column have its two halves
                    float* sums = reinterpret_cast<float*>(own);
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt)
                        if (u < 4) sums[16 * tt + 4 * u + c4] = total[tt];
                    lds_barrier();
                    const int col = cb * kTileN + tid;
                    if (tid < kTileN && col < a.ncols && mine >> (tid >> 4 & 3) & 1)
                        a.ssq_out[(size_t)col * kSsqStride + rb] = reinterpret_cast<const float*>(scratch + (tid >> 6) * 4096)[lane] +
                                                                   reinterpret_cast<const float*>(scratch + (4 + (tid >> 6)) * 4096)[lane];
                }
            } else if constexpr (MODE == MODE_QKV_ROPE) {
                QkvColumn cc[2];                       // requested one column tile ahead of the stores, which they might alias
                cc[0].load(a, col0 + li);
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    if (tt < 3) cc[(tt + 1) & 1].load(a, col0 + 16 * (tt + 1) + li);
                    fixed_here();
                    if (!(mine >> tt & 1)) continue;
                    f32x4 sum[RW];
#pragma unroll
                    for (int r = 0; r < RW; ++r) sum[r] = acc[r][tt];
                    const float sc = __shfl(inv, 16 * tt + li, 64);
                    if (a.kv_dtype == 0) store_qkv<float>(a, sum, cc[tt & 1], 15u, 2 * rb + wy, col0 + 16 * tt + li, sc);
                    else store_qkv<f16_t>(a, sum, cc[tt & 1], 15u, 2 * rb + wy, col0 + 16 * tt + li, sc);
                }
            } else {
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    if (!(mine >> tt & 1)) continue;
                    f32x4 sum[RW];
#pragma unroll
                    for (int r = 0; r < RW; ++r) sum[r] = acc[r][tt];
                    store_tiles<MODE, SPLIT_LINES>(a, sum, 15u, rb * OT + wy * (RW / SW), tiles, col0 + 16 * tt + li, __shfl(inv, 16 * tt + li, 64));
                }
            }
        }
        if (!more) break;
        cur = nxt;
        more = take(args_again().order, nxt);
        lds_barrier();                                 // nobody uses the slab w2 any more, and all of the next unit's first loads have landed
        at_w += step_w;
        load_w(0, w2); load_w(1, w2);
        fixed_here();
    }
    vm_loads_left<0>();
#endif
}

template <int MODE>
int launch_256(const GemvArgs& a, const Order256& o, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_prompt_256_kernel<MODE>), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (attr != hipSuccess) return (int)attr;
    hipLaunchKernelGGL(gemm_prompt_256_kernel<MODE>, dim3(o.n_wg), dim3(kThreads), kLds, s, Args256{a, o});
    return (int)hipGetLastError();
}

}  // namespace

namespace {

// The launch's order; false: not for this kernel.
bool plan_256(int mode, int total_rows, int K, int ncols, size_t part_bytes, int n_cu, Order256* o) {
    if (mode == MODE_STORE || K % kBK != 0 || K < kMinPart * kBK) return false;
    const int tiles = total_rows / 16, ot = mode == MODE_SWIGLU ? 8 : 16;
    const int n_rb = (tiles + ot - 1) / ot, n_cb = (ncols + kTileN - 1) / kTileN, stages = K / kBK, n_wg = n_cu < 8 ? 8 : n_cu & ~7;
    // What is left after the full rounds is cut where each main has more than a seventh of its tile (a tile has at most kPromptMaxParts parts) and both
    // sides more than the exchange of a part costs.
    const int rest = n_rb * n_cb % n_wg, main = Order256::main_share(rest, stages, n_wg);
    const bool split = rest > 0 && 7 * main >= stages + 7 * kMinPart && main >= kPromptCutK / 2 / kBK && stages - main >= kPromptCutK / 2 / kBK && rest * kPromptMaxParts <= kGemmPartTickets &&
                       (long long)rest * stages * n_wg < (1ll << 31) && (size_t)(rest + n_wg) * kPartBytes <= part_bytes;
    *o = Order256(n_rb, n_cb, stages, n_wg, split);
    return true;
}

}  // namespace

double gemm_prompt_256_cost(int mode, int total_rows, int K, int ncols, size_t part_bytes, int n_cu) {
    Order256 o;
    if (!plan_256(mode, total_rows, K, ncols, part_bytes, n_cu, &o)) return HUGE_VAL;
    const double tile = mode == MODE_RESID ? 32 : 10, cut = mode == MODE_SWIGLU ? 34 : 64, idle = 8, stage = 1.9;       // idle: the last round leaves compute units without a tile
    return o.rounds * (stage * o.stages + tile) + (o.rest ? stage * o.main + cut : o.n_rb * o.n_cb % o.n_wg ? idle : 0);
}

// Requirements: those of launch_gemm_prompt and a finite cost; x_split in lines, of ncols columns rounded up to 256, out_split in lines; ssq_in, unless MODE_RESID.
int launch_gemm_prompt_256(const GemvArgs& a, int mode, int n_cu, hipStream_t s, int* n_groups) {
    Order256 o;
    if (!a.x_form.lines() || (a.out_split && !a.out_form.lines()) || (mode != MODE_RESID && !a.ssq_in) || !plan_256(mode, a.total_rows, a.K, a.ncols, a.part && a.part_tickets ? a.part_bytes : 0, n_cu, &o)) return (int)hipErrorInvalidValue;
    if (n_groups) *n_groups = o.n_rb;
    if (mode == MODE_QKV_ROPE) return launch_256<MODE_QKV_ROPE>(a, o, s);
    if (mode == MODE_SWIGLU) return launch_256<MODE_SWIGLU>(a, o, s);
    return launch_256<MODE_RESID>(a, o, s);
}

}  // namespace d3
