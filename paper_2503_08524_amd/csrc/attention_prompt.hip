// Attention of a prompt chunk on the matrix cores: softmax(q . K^T / sqrt(hd)) . V for many consecutive queries of a sequence,
// head_dim 128, fp16 or fp32 cache.
//
// A workgroup of eight waves takes 128 entries of one KV head, an entry being a (query, query head of that KV head) pair:
// 128 / GH consecutive queries x GH heads.  It walks the cache rows from the first one to its last query's own position in tiles (64 rows of an
// fp16 cache, 32 of an fp32 cache).  The two groups of four waves take the tiles in turn (group g the tiles g, g + 2, ...) and merge their
// states through LDS in the end: the longest context, which is what a causal launch waits for, takes half as many steps, and a
// wave's chain of LDS reads, MFMAs and exponentials has another wave on its SIMD to overlap with.  The waves of a group share a tile in
// LDS: a row is read from memory once per 128 entries and from LDS once per 32.
//
// Each wave owns 32 entries and keeps everything about an entry in the two lanes (e, e + 32) that hold it, so the softmax
// needs one lane exchange per tile and no LDS:
//   scores^T [row][entry] = K [row][hd] . q^T: v_mfma_f32_32x32x16_f16, A = K rows from LDS, B = q (scaled to log2 units, hi + lo
//     fp16) from registers; lane (e, h) receives rows 8 j + 4 h .. + 3 (j = 0..3) of its entry;
//   out^T [dim][entry] += V^T [dim][row] . P^T [row][entry]: B = P (hi + lo fp16), whose eight values per lane and 16 rows are exactly
//     a B fragment under the row numbering slot 8 h + i <-> row 4 h + i (i < 4), 8 + 4 h + i - 4 (i >= 4); A = V from LDS by transpose
//     reads in the same numbering; lane (e, h) accumulates its entry's dims, so the rescaling factor is its own.
// fp32 cache rows are split into fp16 hi + lo planes on their way into LDS and both contractions take three MFMAs instead of
// two (K.q = Khi.q + Klo.qhi, P.V = P.Vhi + Phi.Vlo), which keeps the cache's precision.
//
// LDS rows are 256 bytes (sixteen 16-byte segments) without padding; K's segment s sits at s ^ (row % 16), V's at s ^ 4 (row % 4), which
// spreads the fragment reads of both over all banks.  Two buffers per group: the next tile's rows are requested before this tile is
// worked on and written to the other buffer afterwards, one barrier per step.
//
// What bounds it: the chain within a wave (K fragments -> MFMAs -> maximum -> exponentials -> V fragments -> MFMAs), about 2.8 us a
// step with the MFMAs (64 of 32 cycles per wave and step) a good third of it; the two waves of a SIMD are in the same phase most of
// the time.  7B shape, 2048 queries: 199 us (tiles of 16 queries per workgroup, context split) -> 88; 13B 1024 queries 80 -> 37; 70B
// 1024 queries, fp32 cache 365 -> 79.  One group of four waves per workgroup and two workgroups per compute unit: 89, 44, 98.
// Requesting the fragments of a step before the MFMAs of the one before spilled (113 us).
#include "attention.h"

namespace d3 {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float pa_f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 pa_half2 __attribute__((ext_vector_type(2)));
constexpr int kPaEntries = 128;                // entries of a workgroup
constexpr int kPaBuf = 32 * 1024;              // a tile of K and V
constexpr float kPaFloor = -3.0e38f;           // running maximum before the first row: below every score, and finite
constexpr float kPaSlack = 8.0f;               // a running maximum may lag behind by this much (log2): weights up to 256, no rescaling (the conditional rescaling published with FlashAttention-4)

template <typename T> struct PaTile;
template <> struct PaTile<f16_t> {
    static constexpr int KT = 64, PL = 1;      // rows of a tile, planes
    // piece p of a tile matrix (p < 4): this thread's 16 bytes
    static __device__ __forceinline__ int row(int p, int tid) { return 16 * p + (tid >> 4); }
    static __device__ __forceinline__ const f16_t* at(const f16_t* base, int r, int tid) { return base + (size_t)r * 128 + 8 * (tid & 15); }
    static __device__ __forceinline__ void put(char* buf, int r, int tid, int swz, const u32x4& v) {
        *reinterpret_cast<u32x4*>(buf + r * 256 + (((tid & 15) ^ swz) << 4)) = v;
    }
};
template <> struct PaTile<float> {
    static constexpr int KT = 32, PL = 2;
    static __device__ __forceinline__ int row(int p, int tid) { return 8 * p + (tid >> 5); }
    static __device__ __forceinline__ const float* at(const float* base, int r, int tid) { return base + (size_t)r * 128 + 4 * (tid & 31); }
    static __device__ __forceinline__ void put(char* buf, int r, int tid, int swz, const u32x4& v) {
        uint2 hi, lo;
        AttnStage<float>::split(v, hi, lo);
        char* p = buf + r * 256 + ((((tid & 31) >> 1) ^ swz) << 4) + 8 * (tid & 1);
        *reinterpret_cast<uint2*>(p) = hi;
        *reinterpret_cast<uint2*>(p + KT * 256) = lo;
    }
};

// A fragment of P.V: dims 32 cb .. + 31 (lane % 32) of sixteen rows from r16 on, in the row numbering above
__device__ __forceinline__ attn_half8 pa_v_fragment(const char* v, int r16, int cb, int lane) {
    const int s = lane & 15, h = lane >> 5;
    const int row = r16 + 4 * h + (s >> 2), seg = 4 * cb + 2 * ((lane >> 4) & 1) + ((s & 3) >> 1);
    const char* p = v + row * 256 + ((seg ^ ((s >> 2) << 2)) << 4) + 8 * (s & 1);      // row % 4 == s / 4
    typedef __attribute__((address_space(3))) attn_short4 lds_short4;
    const attn_short4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p));
    const attn_short4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p + 8 * 256));
    typedef short attn_short8 __attribute__((ext_vector_type(8)));
    const attn_short8 both = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(attn_half8, both);
}

template <typename T, int GH>
__global__ __launch_bounds__(512, 2) void attn_prompt_kernel(AttnArgs a, SeqRuns runs, int n_tiles) {
    constexpr int HD = 128, QT = kPaEntries / GH;      // queries of a workgroup
    constexpr int KT = PaTile<T>::KT, PL = PaTile<T>::PL, SUB = KT / 32;
    extern __shared__ __align__(16) char lds[];        // [2 groups][2 buffers][K planes, V planes]; in the end the merge area and the output tile
    const int tid = threadIdx.x & 255, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave8 & 3, grp = wave8 >> 2;
    const int e = lane & 31, h = lane >> 5;

    // what the first loads need of the arguments, requested together: read as they come up, each is a round trip that the next one waits behind
    asm volatile("" :: "s"(a.q), "s"(a.row0), "s"(a.q_stride), "s"(a.k_cache), "s"(a.v_cache), "s"(a.H_kv), "s"(a.max_seq), "s"(runs.n), "s"(runs.col[0]), "s"(runs.col[1]),
                       "s"(runs.seq[0]), "s"(runs.pos[0]), "s"(n_tiles));
    // ---- launch order -> (KV head, tile of queries): a run's tiles with the longest contexts first, all heads' of them, the last run's
    // ahead of the first's (whatever their contexts); a head's tiles stay on one XCD when the heads divide over them (its L2 then serves the rows to all of them) ----
    int kvh, tile;
    if (a.H_kv % 8 == 0) {
        const int per_xcd = a.H_kv / 8, i = blockIdx.x >> 3;
        kvh = (i % per_xcd) * 8 + (blockIdx.x & 7);
        tile = n_tiles - 1 - i / per_xcd;
    } else {
        kvh = blockIdx.x % a.H_kv;
        tile = n_tiles - 1 - blockIdx.x / a.H_kv;
    }
    int run = 0, left = tile;
    for (;;) {                                         // (n_tiles is the sum over the runs: ends at the last run at the latest)
        const int t = (runs.col[run + 1] - runs.col[run] + QT - 1) / QT;
        if (left < t || run + 1 >= runs.n) break;
        left -= t;
        ++run;
    }
    const int c_begin = runs.col[run] + left * QT, c_end = min(c_begin + QT, runs.col[run + 1]);   // this workgroup's columns
    const int seq = runs.seq[run];
    const int row0 = a.row0 ? a.row0[seq] : 0;         // left-padded batch: rows are counted from the sequence's first row
    const int pos_begin = runs.pos[run] + left * QT - row0;      // local row of column c_begin
    const int ctx_max = pos_begin + (c_end - c_begin);           // rows visible to the last query

    const int h0 = kvh * GH;
    const size_t head_off = (((size_t)seq * a.H_kv + kvh) * a.max_seq + row0) * HD;
    const T* Kb = static_cast<const T*>(a.k_cache) + head_off;
    const T* Vb = static_cast<const T*>(a.v_cache) + head_off;
    const float scale = 1.4426950408889634f / sqrtf((float)HD);

    // ---- this lane's entry; entries past the last column repeat its query (computed, not stored) ----
    const int qi = (32 * wave + e) / GH, head = h0 + (32 * wave + e) % GH;
    const int ci = min(c_begin + qi, c_end - 1);
    const int last_row = pos_begin + (ci - c_begin);   // the last row this entry sees
    const int wave_first = pos_begin + min((32 * wave) / GH, c_end - 1 - c_begin);            // last row of the wave's first entry ...
    const int wave_last = pos_begin + min((32 * wave + 31) / GH, c_end - 1 - c_begin);        // ... and of its last one
    const bool wave_live = c_begin + (32 * wave) / GH < c_end;

    u32x4 kreg[4], vreg[4];
    auto request = [&](int r0) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = min(r0 + PaTile<T>::row(p, tid), ctx_max - 1);         // rows past the context repeat the last one (masked)
            kreg[p] = *reinterpret_cast<const u32x4*>(PaTile<T>::at(Kb, r, tid));
            vreg[p] = *reinterpret_cast<const u32x4*>(PaTile<T>::at(Vb, r, tid));
        }
    };
    auto put = [&](char* buf) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = PaTile<T>::row(p, tid);
            PaTile<T>::put(buf, r, tid, r & 15, kreg[p]);
            PaTile<T>::put(buf + PL * KT * 256, r, tid, (r & 3) << 2, vreg[p]);
        }
    };
    request(grp * KT);

    attn_half8 qhi[8], qlo[8];                         // B fragments: dims 16 kk + 8 h .. + 7 of the entry
    {
        const float* qp = a.q + (size_t)ci * a.q_stride + (size_t)head * HD + 8 * h;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const float4 t0 = *reinterpret_cast<const float4*>(qp + 16 * kk), t1 = *reinterpret_cast<const float4*>(qp + 16 * kk + 4);
            const float qf[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float v = qf[i] * scale;
                asm("" : "+v"(v));                     // one rounded product for both halves: fused into the conversion of one of them
                                                       // only, the halves belong to different values where the two roundings differ
                const f16_t q = (f16_t)v;
                qhi[kk][i] = q;
                qlo[kk][i] = (f16_t)(v - (float)q);
            }
        }
    }
    float m = kPaFloor, lsum = 0.f;
    f32x16 acc[4];                                     // [dims 32 cb ..]: dim 32 cb + 8 (i / 4) + 4 h + i % 4
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb][i] = 0.f;

    char* own = lds + grp * 2 * kPaBuf;
    put(own);
    __syncthreads();
    const int n_steps = (ctx_max + 2 * KT - 1) / (2 * KT);
    for (int st = 0; st < n_steps; ++st) {
        const int r0 = (2 * st + grp) * KT;
        const char* kbuf = own + (st & 1) * kPaBuf;
        const char* vbuf = kbuf + PL * KT * 256;
        if (st + 1 < n_steps) request(r0 + 2 * KT);
        if (wave_live && r0 <= wave_last) {            // the same for all lanes of the wave
            f32x16 S[SUB];
#pragma unroll
            for (int t = 0; t < SUB; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) S[t][i] = 0.f;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {           // independent accumulators next to each other
                const char* kr = kbuf + e * 256 + (((2 * kk + h) ^ (e & 15)) << 4);
                attn_half8 kf[SUB], kl[SUB];
#pragma unroll
                for (int t = 0; t < SUB; ++t) {
                    kf[t] = *reinterpret_cast<const attn_half8*>(kr + t * 32 * 256);
                    if (PL == 2) kl[t] = *reinterpret_cast<const attn_half8*>(kr + (KT + t * 32) * 256);
                }
#pragma unroll
                for (int t = 0; t < SUB; ++t) S[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], qhi[kk], S[t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < SUB; ++t) S[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], qlo[kk], S[t], 0, 0, 0);
                if (PL == 2) {
#pragma unroll
                    for (int t = 0; t < SUB; ++t) S[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kl[t], qhi[kk], S[t], 0, 0, 0);
                }
            }
            if (r0 + KT - 1 > wave_first) {            // the tile reaches past some entry's own position
#pragma unroll
                for (int t = 0; t < SUB; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (r0 + 32 * t + 8 * (i >> 2) + 4 * h + (i & 3) > last_row) S[t][i] = -INFINITY;
            }
            float mx = S[0][0];
#pragma unroll
            for (int t = 0; t < SUB; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[t][i]);
            mx = reduce_halves(mx, MaxOp());
            if (__any(mx > m + kPaSlack)) {            // rare after the first tiles
                const float m_new = fmaxf(m, mx), keep = __builtin_amdgcn_exp2f(m - m_new);
                lsum *= keep;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[cb][i] *= keep;
                m = m_new;
            }
            // sixteen rows at a time: weights, V fragments, MFMAs
#pragma unroll
            for (int u = 0; u < 2 * SUB; ++u) {
                attn_half8 phi, plo;
#pragma unroll
                for (int i = 0; i < 8; i += 2) {       // (an exponential below 2^-126 counts as zero)
                    const pa_f32x2 p = {__builtin_amdgcn_exp2f(S[u >> 1][8 * (u & 1) + i] - m), __builtin_amdgcn_exp2f(S[u >> 1][8 * (u & 1) + i + 1] - m)};
                    lsum += p[0] + p[1];
                    const pa_half2 ph = __builtin_convertvector(p, pa_half2);
                    const pa_f32x2 rest = {p[0] - (float)ph[0], p[1] - (float)ph[1]};
                    const pa_half2 pl = __builtin_convertvector(rest, pa_half2);
                    phi[i] = ph[0]; phi[i + 1] = ph[1];
                    plo[i] = pl[0]; plo[i + 1] = pl[1];
                }
                attn_half8 vf[4], vl[4];
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    vf[cb] = pa_v_fragment(vbuf, 16 * u, cb, lane);
                    if (PL == 2) vl[cb] = pa_v_fragment(vbuf + KT * 256, 16 * u, cb, lane);
                }
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[cb], phi, acc[cb], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[cb], plo, acc[cb], 0, 0, 0);
                if (PL == 2) {
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl[cb], phi, acc[cb], 0, 0, 0);
                }
            }
        }
        if (st + 1 < n_steps) put(own + ((st + 1) & 1) * kPaBuf);  // its last readers passed the barrier before this step
        __syncthreads();
    }

    // ---- group 1 hands its state over (an entry that saw none of its rows: maximum at the floor, zero sums), group 0 merges ----
    lsum = reduce_halves(lsum, AddOp());
    attn_f32x4* xa = reinterpret_cast<attn_f32x4*>(lds) + tid;   // [16][256]
    float2* xm = reinterpret_cast<float2*>(lds + 64 * 1024) + tid;
    if (grp == 1) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) xa[(4 * cb + j) * 256] = attn_f32x4{acc[cb][4 * j], acc[cb][4 * j + 1], acc[cb][4 * j + 2], acc[cb][4 * j + 3]};
        *xm = make_float2(m, lsum);
    }
    __syncthreads();
    if (grp == 1) return;
    const float2 other = *xm;
    const float m_all = fmaxf(m, other.x), w0 = __builtin_amdgcn_exp2f(m - m_all), w1 = __builtin_amdgcn_exp2f(other.x - m_all);
    const float sum = lsum * w0 + other.y * w1;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const attn_f32x4 t = xa[(4 * cb + j) * 256];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[cb][4 * j + i] = acc[cb][4 * j + i] * w0 + t[i] * w1;
        }

    // ---- out = acc / sum, through LDS so that a row leaves as whole lines: the wave's 32 entries x 128 floats, float4 f of entry
    // e at f ^ e ----
    const float inv = 1.0f / sum;
    float4* o = reinterpret_cast<float4*>(lds + 68 * 1024) + wave * 32 * 32;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            o[e * 32 + ((8 * cb + 2 * j + h) ^ e)] = make_float4(acc[cb][4 * j] * inv, acc[cb][4 * j + 1] * inv, acc[cb][4 * j + 2] * inv, acc[cb][4 * j + 3] * inv);
    __builtin_amdgcn_wave_barrier();
    const int part = lane & 15;                        // sixteen lanes write one entry's 128 dims, 8 each
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int en = 4 * j + (lane >> 4), c = c_begin + (32 * wave + en) / GH;
        if (c >= c_end) continue;
        const float4 u = o[en * 32 + ((2 * part) ^ en)], w = o[en * 32 + ((2 * part + 1) ^ en)];
        const float f[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
        store_split8(a.out_split + c * a.out_form.pitch(a.H * HD), (size_t)(h0 + (32 * wave + en) % GH) * HD + 8 * part, f, a.out_form.lo);
    }
}

template <typename T, int GH>
int launch_gh(const AttnArgs& a, const SeqRuns& runs, hipStream_t s) {
    constexpr int lds = 68 * 1024 + 64 * 1024, QT = kPaEntries / GH;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_prompt_kernel<T, GH>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return (int)attr;
    int n_tiles = 0;
    for (int r = 0; r < runs.n; ++r) n_tiles += (runs.col[r + 1] - runs.col[r] + QT - 1) / QT;
    hipLaunchKernelGGL((attn_prompt_kernel<T, GH>), dim3(n_tiles * a.H_kv), dim3(512), lds, s, a, runs, n_tiles);
    return (int)hipGetLastError();
}

template <typename T>
int launch_t(const AttnArgs& a, const SeqRuns& runs, hipStream_t s) {
    switch (a.H / a.H_kv) {
        case 1: return launch_gh<T, 1>(a, runs, s);
        case 2: return launch_gh<T, 2>(a, runs, s);
        case 4: return launch_gh<T, 4>(a, runs, s);
        case 8: return launch_gh<T, 8>(a, runs, s);
        default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace

// Requirements (checked by the caller): hd 128, group size 1, 2, 4 or 8, q rotated and the runs' K/V rows in the cache; every run
// holds at least one column; out_split set (a.out is not written).
int launch_attention_prompt(const AttnArgs& a, const SeqRuns& runs, int kv_dtype, hipStream_t s) {
    if (a.hd != 128 || runs.n < 1 || runs.n > kMaxCols || !a.out_split) return (int)hipErrorInvalidValue;
    if (kv_dtype == 0) return launch_t<float>(a, runs, s);
    if (kv_dtype == 2) return launch_t<f16_t>(a, runs, s);
    return (int)hipErrorInvalidValue;
}

}  // namespace d3
