// What the two tiled GEMMs of the prompt pass (gemm_prompt.hip, gemm_prompt_256.hip) share: the fragments that their waves multiply, 128 weight rows x 64
// columns at a time, and how a wave's sums leave its registers.
#pragma once
#include <type_traits>
#include <utility>

#include "d3_common.h"

namespace d3 {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kBK = 64;                        // k per weight slab
constexpr int kPitch = 2 * kBK;                // bytes per staged row: eight 16-byte segments = one cache line (64 k of a weight row; 32 k of a column, hi and lo halves)
constexpr int kThreads = 512, kWaves = 8;
constexpr int RW = 8;                          // 16-row tiles per wave
constexpr int kUnits = RW / 2;                 // per column tile: row tiles r and r + 4 (a gate tile and its up tile, the two dims of a rotation)

// Instructions stay on their side of this point: what interleaves the MFMAs with loads and reads as written.
__device__ __forceinline__ void fixed_here() { __builtin_amdgcn_sched_barrier(0); }

template <int OFF>
__device__ __forceinline__ u32x4 lds_read_frag(uint32_t addr) {
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}
// Fragments are kept as four words and become bf16 vectors at the MFMA: a vector of bf16 that lives across the loop's back
// edge is taken apart and put together again there, while it may still be in flight.
__device__ __forceinline__ f32x4 mfma(const u32x4& fa, const u32x4& fb, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa), __builtin_bit_cast(bf16x8, fb), c, 0, 0, 0);
}
template <int N> __device__ __forceinline__ void vm_loads_left() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
template <int N> __device__ __forceinline__ void lds_reads_left() { asm volatile("s_waitcnt lgkmcnt(%0)" :: "n"(N) : "memory"); }
// Nothing that uses the fragment moves above this statement, and volatile statements keep their order: after a wait it
// keeps the MFMAs behind the wait.
__device__ __forceinline__ void pin_frag(u32x4& v) { asm volatile("" : "+v"(v)); }
// all LDS reads have arrived, these among them
__device__ __forceinline__ void all_arrived(u32x4 (&f)[RW]) {
    lds_reads_left<0>();
#pragma unroll
    for (int r = 0; r < RW; ++r) pin_frag(f[r]);
}
struct PromptB { u32x4 h, l; };                       // one column tile's activation fragments: hi and lo halves
__device__ __forceinline__ void all_arrived(PromptB& f) { lds_reads_left<0>(); pin_frag(f.h); pin_frag(f.l); }
template <int... R>
__device__ __forceinline__ void read_a_frags(u32x4 (&f)[RW], uint32_t A, std::integer_sequence<int, R...>) {
    ((f[R] = lds_read_frag<R * 16 * kPitch>(A)), ...);
}
// Column tile TT of a k-step whose activation fragments start OFF bytes behind h (hi halves) and l (lo halves; where a line holds both, their segments are four from
// those of the hi halves, and the swizzle leaves that a single bit of the address).
constexpr uint32_t kLoBit = 4 * 16;
template <int TT, int OFF = 0>
__device__ __forceinline__ void read_b_frags(PromptB& f, uint32_t h, uint32_t l) {
    f.h = lds_read_frag<OFF + TT * 16 * kPitch>(h);
    f.l = lds_read_frag<OFF + TT * 16 * kPitch>(l);
}
// 2 N MFMAs: row tiles R0 .. R0 + N - 1 of one column tile, both planes.  The two products of an accumulator stand one after the other: that
// toggles less than eight row tiles of the hi plane and then eight of the lo plane, and the clock is what the power leaves (the MFMAs
// alone on random operands 2.03 -> 2.20 PFLOP/s at 2.05 -> 2.22 GHz; 13B shape, 4 x 1024 columns, 4 blocks 16.26 -> 16.05 ms).
template <int R0, int N>
__device__ __forceinline__ void mma_hl(f32x4 (&acc)[RW][4], int tt, const u32x4 (&fa)[RW], const PromptB& fb) {
#pragma unroll
    for (int r = R0; r < R0 + N; ++r) {
        acc[r][tt] = mfma(fa[r], fb.h, acc[r][tt]);
        acc[r][tt] = mfma(fa[r], fb.l, acc[r][tt]);
    }
}

// the cache's element type from four fp32 values
__device__ __forceinline__ void store_row4(float* p, const float (&v)[4]) { *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void store_row4(f16_t* p, const float (&v)[4]) {
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    half4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (f16_t)fminf(fmaxf(v[e], -65504.f), 65504.f);
    *reinterpret_cast<half4*>(p) = h;
}

// ---- epilogues of the projections that only store, from the summed accumulators of one column tile: lane (i, g) holds column i, rows 4g..4g+3 of each
// row tile.  units: which units to store, bit r for row tiles r and r + 4; sc: the column's RMSNorm scale. ----
// otile0: the wave's first output row tile of `tiles`; FORM: of the split output (its column pitch is out_form's, or known)
template <int MODE, int FORM = SPLIT_ANY>
__device__ __forceinline__ void store_tiles(const GemvArgs& a, const f32x4 (&acc)[RW], unsigned units, int otile0, int tiles, int col, float sc) {
    constexpr int SW = (MODE == MODE_SWIGLU) ? 2 : 1;
    const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int r = 0; r < RW / SW; ++r) {
        if (!(units >> (r % kUnits) & 1)) continue;
        const int otile = otile0 + r, row = otile * 16 + 4 * lg;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = acc[r][e] * sc;
            if (MODE == MODE_SWIGLU) v[e] = v[e] / (1.0f + expf(-v[e])) * (acc[r + RW / 2][e] * sc);
        }
        if (otile < tiles && col < a.ncols) {
            if (a.out) *reinterpret_cast<float4*>(a.out + (size_t)col * a.out_stride + row) = make_float4(v[0], v[1], v[2], v[3]);
            if (a.out_split) store_split4<FORM>(a.out_split + col * (FORM == SPLIT_LINES ? 2 * (size_t)a.out_stride : a.out_form.pitch(a.out_stride)), row, v, a.out_form.lo);
        }
    }
}

// ---- QKV of a prompt pass at head_dim 128: a wave's 128 rows are one head, and row tiles r and r + 4 hold the dims j and j + 64 that one
// rotation pairs, so q and k are rotated and k and v appended to the cache straight from the accumulators (as a launch of its own
// over fp32 q, k, v that took 24 us of a 2048-column block at the 7B shape). ----
struct QkvColumn {
    int2 at;                                           // (sequence, cache row) of this lane's column
    float4 c0[RW / 2], c1[RW / 2];                     // (cos, sin) of dims j, j + 1 and j + 2, j + 3
    __device__ __forceinline__ void load(const GemvArgs& a, int col_raw) {
        const int lg = (threadIdx.x & 63) >> 4, col = col_raw < a.ncols ? col_raw : a.ncols - 1;
        at = a.col_at[col];
#pragma unroll
        for (int r = 0; r < RW / 2; ++r) {
            const float2* cs = a.rope_cs + (size_t)col * 64 + 16 * r + 4 * lg;
            c0[r] = *reinterpret_cast<const float4*>(cs);
            c1[r] = *reinterpret_cast<const float4*>(cs + 2);
        }
    }
};
template <typename T>
__device__ __forceinline__ void store_qkv(const GemvArgs& a, const f32x4 (&acc)[RW], const QkvColumn& cc, unsigned units, int head, int col, float sc) {
    const int lg = (threadIdx.x & 63) >> 4;
    if (head >= a.H + 2 * a.H_kv) return;
    const bool is_q = head < a.H, is_v = head >= a.H + a.H_kv;
    const int kvh = is_v ? head - a.H - a.H_kv : head - a.H;
    void *const kc = a.k_cache, *const vc = a.v_cache;
    asm volatile("" :: "s"(kc), "s"(vc));              // two values: the compiler would choose between their places, in a copy on the stack
    if (col >= a.ncols) return;
    float* q = a.out + (size_t)col * a.out_stride + head * 128;
    T* row = nullptr;
    if (!is_q) row = static_cast<T*>(is_v ? vc : kc) + (((size_t)cc.at.x * a.H_kv + kvh) * a.max_seq + cc.at.y) * 128;
#pragma unroll
    for (int r = 0; r < RW / 2; ++r) {
        if (!(units >> r & 1)) continue;
        const int j = 16 * r + 4 * lg;
        float lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo[e] = acc[r][e] * sc; hi[e] = acc[r + RW / 2][e] * sc; }
        if (!is_v) {
            const float4 c0 = cc.c0[r], c1 = cc.c1[r];
            const float cs[4] = {c0.x, c0.z, c1.x, c1.z}, sn[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // the two roundings of each are stated: left to the compiler, which product joins the addition unrounded changed with the code around it
                const float y0 = fmaf(lo[e], cs[e], -(hi[e] * sn[e])), y1 = fmaf(lo[e], sn[e], hi[e] * cs[e]);
                lo[e] = y0; hi[e] = y1;
            }
        }
        if (is_q) { store_row4(q + j, lo); store_row4(q + j + 64, hi); }
        else { store_row4(row + j, lo); store_row4(row + j + 64, hi); }
    }
}

// 16 bytes per lane and access, at agent scope (past the XCD's own L2, like st_agent / ld_agent)
[[maybe_unused]] constexpr int kAgent = 16;

extern __shared__ __attribute__((aligned(16))) char prompt_lds[];

}  // namespace

}  // namespace d3
