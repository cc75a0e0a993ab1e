// Small kernels around the projections: embedding gather, gain + bf16 split for
// the MFMA path, rotary embedding + KV append, greedy argmax, missing-state KV fill.
#include "d3_common.h"

namespace d3 {

namespace {

// ---------------- embedding gather: x[c][:] = E[token(c)][:] ----------------
// A workgroup per column: the column's row of the rotary table (the rotation angles depend on the position only, not on the
// block) and its row of the residual stream; on the matrix-core path (split.gain set) also what gain_split_kernel hands to the first
// projection, from the registers that hold the row anyway (as a launch of its own 5 us of a decode step, less than the step's
// noise, and 13 us of 2048 columns).
template <typename W>
__device__ __forceinline__ void embed_column(const W* __restrict__ emb, int tok, int angle_pos, int c, int d, int vocab, float* __restrict__ x,
                                             const double* __restrict__ inv_freq, int half_hd, float2* __restrict__ rope_cs, const EmbedSplit& split) {
    if ((int)threadIdx.x < half_hd) {
        double sn, cs;
        sincos((double)angle_pos * inv_freq[threadIdx.x], &sn, &cs);
        rope_cs[(size_t)c * half_hd + threadIdx.x] = make_float2((float)cs, (float)sn);
    }
    tok = tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok);   // stay inside the table whatever the caller fed
    const W* row = emb + (size_t)tok * d;
    float* xo = x + (size_t)c * d;
    float ss = 0.f;
    if (sizeof(W) == 4) {
        for (int j = threadIdx.x * 4; j < d; j += blockDim.x * 4)
            *reinterpret_cast<float4*>(xo + j) = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(row) + j);
    } else {
        // d % 8 == 0: eight bf16 per load; up to R pieces per thread and their gains are requested together, wider rows go round again
        constexpr int R = 4;
        for (int base = threadIdx.x * 8; base < d; base += R * 2048) {
            uint4 v[R];
            float4 g0[R], g1[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int at = base + r * 2048, j = at < d ? at : base;
                v[r] = *reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(row) + j);
                if (split.gain) {
                    g0[r] = *reinterpret_cast<const float4*>(split.gain + j);
                    g1[r] = *reinterpret_cast<const float4*>(split.gain + j + 4);
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int j = base + r * 2048;
                if (j >= d) break;
                const float f[8] = {bf16_lo(v[r].x), bf16_hi(v[r].x), bf16_lo(v[r].y), bf16_hi(v[r].y), bf16_lo(v[r].z), bf16_hi(v[r].z), bf16_lo(v[r].w), bf16_hi(v[r].w)};
                *reinterpret_cast<float4*>(xo + j) = make_float4(f[0], f[1], f[2], f[3]);
                *reinterpret_cast<float4*>(xo + j + 4) = make_float4(f[4], f[5], f[6], f[7]);
                if (split.gain) {
                    const float g[8] = {g0[r].x, g0[r].y, g0[r].z, g0[r].w, g1[r].x, g1[r].y, g1[r].z, g1[r].w};
                    float w[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        ss += f[e] * f[e];
                        w[e] = f[e] * g[e];
                    }
                    store_split8(split.split + c * split.form.pitch(d), j, w, split.form.lo);
                }
            }
        }
    }
    if (split.gain) {                                  // the same for the whole workgroup
        __shared__ float red[4];
        ss = wave_sum(ss);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
        __syncthreads();
        if (threadIdx.x == 0) split.ssq[(size_t)c * kSsqStride] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}
template <typename W>
__global__ __launch_bounds__(256) void embed_kernel(const W* __restrict__ emb, const int32_t* __restrict__ tokens,
                                                    ColMap cm, int d, int vocab, float* __restrict__ x,
                                                    const double* __restrict__ inv_freq, int half_hd,
                                                    float2* __restrict__ rope_cs, const int* __restrict__ row0, EmbedSplit split) {
    const int c = blockIdx.x;
    embed_column<W>(emb, tokens[cm.tok_index(c)], cm.pos(c) - (row0 ? row0[cm.seq(c)] : 0),      // a left-padded sequence counts from its first token
                    c, d, vocab, x, inv_freq, half_hd, rope_cs, split);
}
__global__ __launch_bounds__(256) void embed_runs_kernel(const bf16_t* __restrict__ emb, const int32_t* __restrict__ tokens, SeqRuns runs, int P,
                                                         int pos_begin, int d, int vocab, float* __restrict__ x,
                                                         const double* __restrict__ inv_freq, int half_hd, float2* __restrict__ rope_cs,
                                                         const int* __restrict__ row0, int2* __restrict__ col_at, EmbedSplit split) {
    const int c = blockIdx.x, r = runs.of(c), seq = runs.seq[r], pos = runs.pos[r] + (c - runs.col[r]);
    if (threadIdx.x == 0) col_at[c] = make_int2(seq, pos);
    embed_column<bf16_t>(emb, tokens[(size_t)seq * P + (pos - pos_begin)], pos - (row0 ? row0[seq] : 0), c, d, vocab, x, inv_freq, half_hd, rope_cs, split);
}

// ---------------- the last positions of a prompt pass ----------------
// dst may be the caller's hidden_dump, which is aligned to its floats and no more.
__global__ __launch_bounds__(256) void pick_rows_kernel(const float* __restrict__ x, int d, RowPick pick, float* __restrict__ dst) {
    const float* src = x + (size_t)pick.col[blockIdx.x] * d;
    float* out = dst + (size_t)pick.row[blockIdx.x] * d;
    for (int j = threadIdx.x * 4; j < d; j += blockDim.x * 4) {
        const float4 v = *reinterpret_cast<const float4*>(src + j);
        out[j] = v.x; out[j + 1] = v.y; out[j + 2] = v.z; out[j + 3] = v.w;
    }
}

// ---------------- gain + split into bf16 hi/lo, sum of squares ----------------
// The matrix-core projections fold the RMSNorm scale 1/rms into their epilogue; what they need from the
// residual is the split of x * gain and sum(x^2).  Inside a pass the residual projections produce both; this
// kernel does it for the residual that a head or a fill starts from (the embedding kernel does it itself).  One workgroup per column; a thread keeps up to 8 float4 of the
// column in registers (all loads issued together); wider columns fall back to a second read.
__global__ __launch_bounds__(256) void gain_split_kernel(const float* __restrict__ x, int x_stride,
                                                         const float* __restrict__ gain, int K,
                                                         bf16_t* __restrict__ split,
                                                         float* __restrict__ ssq, SplitForm form) {
    constexpr int R = 8;
    __shared__ float red[4];
    const int c = blockIdx.x, tid = threadIdx.x;
    const float* xc = x + (size_t)c * x_stride;
    const int n4 = K / 4;
    float ss = 0.f;
    auto emit = [&](int i4, const float4& t, const float4& gg) {
        const float f[4] = {t.x * gg.x, t.y * gg.y, t.z * gg.z, t.w * gg.w};
        ss += t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
        store_split4(split + c * form.pitch(K), i4 * 4, f, form.lo);
    };
    float4 v[R], g[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i4 = tid + r * 256;
        if (i4 < n4) {
            v[r] = *reinterpret_cast<const float4*>(xc + i4 * 4);
            g[r] = *reinterpret_cast<const float4*>(gain + i4 * 4);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i4 = tid + r * 256;
        if (i4 < n4) emit(i4, v[r], g[r]);
    }
    for (int i4 = tid + R * 256; i4 < n4; i4 += 256)
        emit(i4, *reinterpret_cast<const float4*>(xc + i4 * 4), *reinterpret_cast<const float4*>(gain + i4 * 4));
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) ssq[(size_t)c * kSsqStride] = (red[0] + red[1]) + (red[2] + red[3]);
}

// ---------------- rotary embedding + KV append ----------------
// Half-split pairing: dims (j, j + hd/2) of a head turn by pos * inv_freq[j].
template <typename T>
__device__ __forceinline__ void store_kv(T* p, float v);
template <> __device__ __forceinline__ void store_kv<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_kv<f16_t>(f16_t* p, float v) { *p = (f16_t)fminf(fmaxf(v, -65504.f), 65504.f); }

template <typename T>
__global__ __launch_bounds__(64) void rope_append_kernel(RopeArgs a) {
    const int head = blockIdx.x, c = blockIdx.y, j = threadIdx.x;
    const int half = a.hd / 2;
    if (j >= half) return;
    const int2 at = a.col_at ? a.col_at[c] : make_int2(a.cm.seq(c), a.cm.pos(c));
    const int seq = at.x, pos = at.y;
    float* row = a.qkv + (size_t)c * (a.H + 2 * a.H_kv) * a.hd + (size_t)head * a.hd;
    if (head < a.H + a.H_kv) {
        const float2 cs = a.rope_cs[(size_t)c * half + j];
        const float x0 = row[j], x1 = row[j + half];
        const float y0 = x0 * cs.x - x1 * cs.y;
        const float y1 = x0 * cs.y + x1 * cs.x;
        if (head < a.H) {
            row[j] = y0;
            row[j + half] = y1;
        } else {
            T* dst = static_cast<T*>(a.k_cache) + (((size_t)seq * a.H_kv + (head - a.H)) * a.max_seq + pos) * a.hd;
            store_kv<T>(dst + j, y0);
            store_kv<T>(dst + j + half, y1);
        }
    } else {
        T* dst = static_cast<T*>(a.v_cache) + (((size_t)seq * a.H_kv + (head - a.H - a.H_kv)) * a.max_seq + pos) * a.hd;
        store_kv<T>(dst + j, row[j]);
        store_kv<T>(dst + j + half, row[j + half]);
    }
}

// ---------------- greedy argmax, lowest index on ties ----------------
// A chain of round trips bounds it: the loads of up to 32768 logits go out in one round without a branch per thread (a round ends where the row does),
// and lanes are compared by swaps and rotations instead of LDS shuffles, the sixteen waves' winners by a row of lanes instead of one thread.
// 1024 / 32000 logits 3.5 / 6.8 -> 2.1 / 4.8 us, 32 rows of 32000 7.5 -> 5.5 (kernel trace).
struct Best { float v; int i; };
__device__ __forceinline__ Best better(const Best& a, const Best& b) { return b.v > a.v || (b.v == a.v && b.i < a.i) ? b : a; }
template <int N> __device__ __forceinline__ Best best_rotated(const Best& b) {
    return Best{row_rotated<N>(b.v), __builtin_amdgcn_update_dpp(0, b.i, 0x120 + N, 0xf, 0xf, false)};
}
__device__ __forceinline__ Best best_of_row(Best b) {          // of the 16 lanes of a row
    b = better(b, best_rotated<8>(b));
    b = better(b, best_rotated<4>(b));
    b = better(b, best_rotated<2>(b));
    return better(b, best_rotated<1>(b));
}
__device__ __forceinline__ Best best_of_wave(Best b) {
    auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(b.v), __float_as_uint(b.v), false, false);
    auto i = __builtin_amdgcn_permlane32_swap((unsigned)b.i, (unsigned)b.i, false, false);
    b = better(Best{__uint_as_float(v[0]), (int)i[0]}, Best{__uint_as_float(v[1]), (int)i[1]});
    v = __builtin_amdgcn_permlane16_swap(__float_as_uint(b.v), __float_as_uint(b.v), false, false);
    i = __builtin_amdgcn_permlane16_swap((unsigned)b.i, (unsigned)b.i, false, false);
    return best_of_row(better(Best{__uint_as_float(v[0]), (int)i[0]}, Best{__uint_as_float(v[1]), (int)i[1]}));
}
__global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ logits, int vocab, int32_t* __restrict__ out) {
    constexpr int R = 16;                              // pairs of logits in flight per thread
    __shared__ float bv[16];
    __shared__ int bi[16];
    const int c = blockIdx.x, tid = threadIdx.x;
    const float* lg = logits + (size_t)c * vocab;
    Best best{-INFINITY, 0x7fffffff};
    const int n2 = vocab / 2;                          // vocab % 2 == 0
    for (int base = 0; base < n2; base += 1024 * R) {
        float2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (base + r * 1024 >= n2) break;
            v[r] = *reinterpret_cast<const float2*>(lg + 2 * min(base + r * 1024 + tid, n2 - 1));
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (base + r * 1024 >= n2) break;
            const int p = min(base + r * 1024 + tid, n2 - 1);          // threads past the end look at the last pair once more
            best = better(better(best, Best{v[r].x, 2 * p}), Best{v[r].y, 2 * p + 1});
        }
    }
    // NaN logits never win (comparisons false); an all-NaN row yields index clamp below
    best = best_of_wave(best);
    if ((tid & 63) == 0) { bv[tid >> 6] = best.v; bi[tid >> 6] = best.i; }
    __syncthreads();
    if (tid < 16) {
        best = best_of_row(Best{bv[tid], bi[tid]});
        if (tid == 0) out[c] = best.i >= vocab ? 0 : best.i;
    }
}

// ---------------- missing-state fill (COPY) ----------------
// One workgroup per (row, sequence, KV head): read the source block's head vector once,
// write it into every dropped block.  16 bytes per lane.
__global__ __launch_bounds__(64) void fill_kernel(FillArgs a, int bytes_per_vec) {
    const int pos = a.pos_begin + blockIdx.x;
    const int seq = blockIdx.y / a.H_kv, h = blockIdx.y % a.H_kv;
    const int piece = threadIdx.x;
    if (piece * 16 >= bytes_per_vec) return;
    const size_t layer_stride = (size_t)a.max_batch * a.H_kv * a.max_seq * bytes_per_vec;
    const size_t off = (((size_t)seq * a.H_kv + h) * a.max_seq + pos) * bytes_per_vec + (size_t)piece * 16;
    char* kc = static_cast<char*>(a.k_cache);
    char* vc = static_cast<char*>(a.v_cache);
    uint4 kv = make_uint4(0, 0, 0, 0), vv = make_uint4(0, 0, 0, 0);
    if (a.src >= 0) {
        kv = *reinterpret_cast<const uint4*>(kc + (size_t)a.src * layer_stride + off);
        vv = *reinterpret_cast<const uint4*>(vc + (size_t)a.src * layer_stride + off);
    }
    for (int l = a.drop_begin; l < a.drop_begin + a.n_drop; ++l) {
        *reinterpret_cast<uint4*>(kc + (size_t)l * layer_stride + off) = kv;
        *reinterpret_cast<uint4*>(vc + (size_t)l * layer_stride + off) = vv;
    }
}

// ---------------- read-only streaming yardstick ----------------
// What the memory system gives a pure read stream issued the way the projections issue theirs (16 bytes per lane,
// streaming loads, eight in flight per lane, one contiguous band at a time): every workgroup XORs its share and
// one lane per wave stores the result so that the loads cannot be dropped.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ src, size_t n16, unsigned* __restrict__ sink) {
    const size_t stride = (size_t)gridDim.x * 256;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i + 7 * stride < n16; i += 8 * stride) {
        u32x4 v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = load_stream16(src + i + r * stride);
#pragma unroll
        for (int r = 0; r < 8; ++r) acc ^= v[r];
    }
    for (; i < n16; i += stride) acc ^= load_stream16(src + i);
    unsigned x = acc.x ^ acc.y ^ acc.z ^ acc.w;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x ^= __shfl_xor(x, o, 64);
    if ((threadIdx.x & 63) == 0) sink[blockIdx.x * 4 + (threadIdx.x >> 6)] = x;
}

// ---------------- state words of a decode step that runs in the static scratch array ----------------
__global__ __launch_bounds__(256) void static_seed_kernel(StaticSeed seed, double* __restrict__ inv_freq, int half_hd, int* __restrict__ row0,
                                                          int* __restrict__ tickets, int n_tickets, int* __restrict__ gemm_tickets,
                                                          int n_gemm_tickets) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x, n = gridDim.x * blockDim.x;
    if (tid < half_hd) inv_freq[tid] = seed.inv_freq[tid];
    if (tid < kMaxCols) row0[tid] = seed.row0[tid];
    for (int i = tid; i < n_tickets; i += n) tickets[i] = 0;
    for (int i = tid; i < n_gemm_tickets; i += n) gemm_tickets[i] = 0;
}

}  // namespace

int launch_static_seed(const StaticSeed& seed, double* inv_freq, int half_hd, int* row0, int* tickets, int n_tickets,
                       int* gemm_tickets, int n_gemm_tickets, hipStream_t s) {
    hipLaunchKernelGGL(static_seed_kernel, dim3(8), dim3(256), 0, s, seed, inv_freq, half_hd, row0, tickets, n_tickets, gemm_tickets,
                       n_gemm_tickets);
    return (int)hipGetLastError();
}

int launch_stream_read(const void* src, size_t bytes, unsigned* sink, int n_wg, hipStream_t s) {
    hipLaunchKernelGGL(stream_read_kernel, dim3(n_wg), dim3(256), 0, s, static_cast<const u32x4*>(src), bytes / 16, sink);
    return (int)hipGetLastError();
}

int launch_embed(const void* tok_emb, int weight_dtype, const int32_t* tokens, ColMap cm, int ncols, int d,
                 int vocab, float* x, const double* inv_freq, int half_hd, float2* rope_cs, const int* row0, const EmbedSplit& split, hipStream_t s) {
    if (weight_dtype == 0)
        hipLaunchKernelGGL(embed_kernel<float>, dim3(ncols), dim3(256), 0, s, static_cast<const float*>(tok_emb), tokens, cm, d, vocab, x,
                           inv_freq, half_hd, rope_cs, row0, split);
    else
        hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3(ncols), dim3(256), 0, s, static_cast<const bf16_t*>(tok_emb), tokens, cm, d, vocab, x,
                           inv_freq, half_hd, rope_cs, row0, split);
    return (int)hipGetLastError();
}

int launch_embed_runs(const void* tok_emb, const int32_t* tokens, const SeqRuns& runs, int P, int pos_begin, int ncols, int d, int vocab,
                      float* x, const double* inv_freq, int half_hd, float2* rope_cs, const int* row0, int2* col_at, const EmbedSplit& split, hipStream_t s) {
    hipLaunchKernelGGL(embed_runs_kernel, dim3(ncols), dim3(256), 0, s, static_cast<const bf16_t*>(tok_emb), tokens, runs, P, pos_begin, d, vocab, x,
                       inv_freq, half_hd, rope_cs, row0, col_at, split);
    return (int)hipGetLastError();
}

int launch_pick_rows(const float* x, int d, const RowPick& pick, float* dst, hipStream_t s) {
    hipLaunchKernelGGL(pick_rows_kernel, dim3(pick.n), dim3(256), 0, s, x, d, pick, dst);
    return (int)hipGetLastError();
}

int launch_gain_split(const float* x, int x_stride, const float* gain, int K, int ncols,
                      bf16_t* split, float* ssq, SplitForm form, hipStream_t s) {
    hipLaunchKernelGGL(gain_split_kernel, dim3(ncols), dim3(256), 0, s, x, x_stride, gain, K, split, ssq, form);
    return (int)hipGetLastError();
}

int launch_rope_append(const RopeArgs& a, int kv_dtype, hipStream_t s) {
    dim3 grid(a.H + 2 * a.H_kv, a.ncols);
    if (kv_dtype == 0) hipLaunchKernelGGL(rope_append_kernel<float>, grid, dim3(64), 0, s, a);
    else if (kv_dtype == 2) hipLaunchKernelGGL(rope_append_kernel<f16_t>, grid, dim3(64), 0, s, a);
    else return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

int launch_argmax(const float* logits, int vocab, int ncols, int32_t* out, hipStream_t s) {
    hipLaunchKernelGGL(argmax_kernel, dim3(ncols), dim3(1024), 0, s, logits, vocab, out);
    return (int)hipGetLastError();
}

int launch_fill(const FillArgs& a, int kv_dtype, hipStream_t s) {
    if (a.pos_end <= a.pos_begin || a.n_drop <= 0) return 0;
    const int bytes_per_vec = a.hd * kv_elem_bytes(kv_dtype);
    dim3 grid(a.pos_end - a.pos_begin, a.B * a.H_kv);
    hipLaunchKernelGGL(fill_kernel, grid, dim3(64), 0, s, a, bytes_per_vec);
    return (int)hipGetLastError();
}

}  // namespace d3
