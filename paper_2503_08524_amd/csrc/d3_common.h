// Shared declarations of the D^3 HIP library (gfx950 only): kernel argument
// structs, launch wrappers, small device helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace d3 {

constexpr int kWave = 64;          // CDNA wavefront
constexpr int kMaxCols = 32;       // largest batch; columns of a decode pass
// Most columns of a prompt pass (a context holds min(this, n rounded up to 128), half of this with an fp32 cache or on the vector ALUs, n = the cache rows of one sequence, or of all where they share
// passes).  The 7B widths' O and down projections are 128 of the large tiles at 2048 columns, a full round of compute units at 4096: 32 x 2048 tokens, 2 blocks, 79.0 ms in
// passes of 2048, 74.7 of 4096, 74.9 of 8192.
constexpr int kPassCols = 4096;
constexpr int kMaxSplits = 32;     // context splits of one attention head
constexpr size_t kGemmPartBytes = 16u << 20;   // partial accumulators of a K-sliced wide MFMA projection
constexpr size_t kPromptPartTile = 128u << 10;  // ... of one K part of a tile (256 rows x 128 columns) of a prompt pass's projection
constexpr int kPromptMaxParts = 8;             // most K parts of such a tile
constexpr size_t kPromptPartBytes = 64u << 20; // most of them that a launch may publish (512 parts)
constexpr size_t kPromptPartBytes256 = 128u << 20;   // the same of a launch of the larger tiles (256 columns), which cuts contractions of kPromptCutK and more
constexpr int kPromptCutK = 24 * 64;
constexpr int kGemmPartTickets = 2048;         // row groups such a projection may have
constexpr int kSsqStride = 512;    // partial sums of squares kept per column (one per workgroup of the producing projection)

typedef uint16_t bf16_t;           // bf16 bit pattern
typedef _Float16 f16_t;            // IEEE half (KV cache only)

// bytes per KV-cache element for a d3_dtype value (0 f32, 2 f16)
inline int kv_elem_bytes(int kv_dtype) { return kv_dtype == 0 ? 4 : 2; }

// Division by a number that the host knows: a multiplication and a correction instead of the 25 dependent instructions of a division.  With
// m = floor(2^32 / d) (one less for d = 1) the product's upper word is the quotient or one less, for every x in [0, 2^31).
struct Divisor {
    int d = 1;
    uint32_t m = 0xffffffffu;
    Divisor() = default;
    explicit Divisor(int v) : d(v), m(v > 1 ? (uint32_t)((1ull << 32) / v) : 0xffffffffu) {}
    __host__ __device__ __forceinline__ int of(int x) const {
        const int q = (int)(((unsigned long long)(uint32_t)x * m) >> 32);
        return x - q * d >= d ? q + 1 : q;
    }
};

// Which (sequence, position, token) a column of the current pass stands for.
// Column c has global index g = base + c; sequence g % B, row pos_begin + g / B.
// Decode: base 0, P 1 (column b = sequence b).  Prompt pass: position-major
// enumeration of the [B][P] prompt, so the last B columns are the last positions.
struct ColMap {
    int base, B, P, pos_begin;
    int seq0 = 0;          // first sequence of the pass (a prompt chunk of one sequence: B = 1, seq0 = that sequence)
    __host__ __device__ int seq(int c) const { return seq0 + (base + c) % B; }
    __host__ __device__ int pos(int c) const { return pos_begin + (base + c) / B; }
    __host__ __device__ int tok_index(int c) const { return seq(c) * P + (base + c) / B; }
};

// The columns of a prompt pass on the matrix-core path as runs of consecutive positions, one run per sequence: run r is sequence
// seq[r], columns [col[r], col[r + 1]), the first of them at cache row pos[r].
struct SeqRuns {
    int n;
    int col[kMaxCols + 1], seq[kMaxCols], pos[kMaxCols];
    __host__ __device__ int of(int c) const {          // the run that column c belongs to
        int lo = 0, hi = n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (col[mid] <= c) lo = mid; else hi = mid - 1;
        }
        return lo;
    }
};

// 16-byte streaming load of weights that are read exactly once (non-temporal: do not
// displace the activations that live in L2)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4 load_stream16(const void* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }
// Two values rounded to nearest even: one instruction for both (with integer additions, five for each).
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

// Activations of the matrix-core projections are split x = hi + lo into two bf16 halves, in one of two forms, which a pass keeps from the embedding to the head:
//  * planes: the hi halves of a column are a row of K, and the lo halves one of another array.  What moves 16 columns or more reads 256 bytes of a row at a time.
//  * lines: 32 hi halves and then their 32 lo halves, so that one 128-byte line holds everything of 32 k, which is what a k-step of the MFMAs reads; a row is 2 K halves.  For
//    up to 8 columns, which are one MFMA operand together (64 bytes of every line twice cost a step at the 70B widths 0.5 %), and for passes that take tiles of 256 columns, whose
//    slab of activations is 32 k.  Elsewhere it loses: columns are twice as far apart, and those a large power of two apart meet on memory channels, and 16 columns' rows are read
//    by shorter pieces.  Lines / planes, us: a block's four projections at 14 columns of the 7B shape 98.5 / 96.5; prompts: 2048 wide, head_dim 64, 256 columns 554 / 541 (its down
//    projection 52 / 41), 70B widths, 128 columns, 1179 / 1154, 13B widths, 129 columns, 708 / 693, 7B shape, 128 columns, 492 / 488; decode steps of 17 to 32 columns equal to 0.5 %.
//    Rows of lines padded by 128 to 1152 bytes mend the first and the third and cost the second 2 to 7 %.
// lo: halves from a value's hi half to its lo half, which in planes is far more than in lines; pitch: halves from column to column.  (Kept in the arguments of every launch, so no larger
// than a pointer: with the pitch beside it small launches took 0.1 us more, 1024 wide, 5 prompts of 2 tokens, 2 blocks, 339.5 -> 336 us.)
constexpr int kSplitLo = 32;
struct SplitForm {
    size_t lo;
    __host__ __device__ __forceinline__ bool lines() const { return lo == kSplitLo; }
    __host__ __device__ __forceinline__ size_t pitch(size_t K) const { return lines() ? 2 * K : K; }
};
inline SplitForm split_lines() { return SplitForm{kSplitLo}; }
inline SplitForm split_planes(int K, size_t columns) { return SplitForm{columns * K}; }     // columns: of the whole plane, 32 or more
// where in its row value k's hi half is (k, k + 1, ... of one run of 32 are adjacent); a kernel that knows the form says so
enum { SPLIT_ANY, SPLIT_LINES, SPLIT_PLANES };
template <int FORM = SPLIT_ANY>
__device__ __forceinline__ size_t split_at(size_t k, size_t lo) { return FORM == SPLIT_LINES || (FORM == SPLIT_ANY && lo == kSplitLo) ? 2 * k - (k & 31) : k; }
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& hi, uint32_t& lo) {
    hi = bf16_pair(a, b);
    lo = bf16_pair(a - bf16_lo(hi), b - bf16_hi(hi));
}
// four adjacent values, k % 4 == 0; row: their row of the split
template <int FORM = SPLIT_ANY>
__device__ __forceinline__ void store_split4(bf16_t* row, size_t k, const float (&v)[4], size_t lo) {
    uint2 h, l;
    split_pair(v[0], v[1], h.x, l.x);
    split_pair(v[2], v[3], h.y, l.y);
    bf16_t* p = row + split_at<FORM>(k, lo);
    *reinterpret_cast<uint2*>(p) = h;
    *reinterpret_cast<uint2*>(p + lo) = l;
}
// eight, k % 8 == 0
__device__ __forceinline__ void store_split8(bf16_t* row, size_t k, const float (&v)[8], size_t lo) {
    uint4 h, l;
    split_pair(v[0], v[1], h.x, l.x);
    split_pair(v[2], v[3], h.y, l.y);
    split_pair(v[4], v[5], h.z, l.z);
    split_pair(v[6], v[7], h.w, l.w);
    bf16_t* p = row + split_at(k, lo);
    *reinterpret_cast<uint4*>(p) = h;
    *reinterpret_cast<uint4*>(p + lo) = l;
}
template <int FORM = SPLIT_ANY>
__device__ __forceinline__ void store_split1(bf16_t* row, size_t k, float v, size_t lo) {
    uint32_t h, l;
    split_pair(v, 0.f, h, l);
    bf16_t* p = row + split_at<FORM>(k, lo);
    p[0] = (bf16_t)h;
    p[lo] = (bf16_t)l;
}

// Data handed from one workgroup to another inside a kernel is written and read with agent-scope
// accesses (coherent across the chip's eight L2s) instead of cache-wide fences, which cost tens of
// microseconds here.  Protocol: producer st_agent(...), wait_stores(), workgroup barrier, then one
// thread bumps an arrival counter; the consumer sees the counter and reads with ld_agent(...).
__device__ __forceinline__ void st_agent(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float ld_agent(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Reductions over lanes on the vector ALU: halves of a wave and pairs of its rows of 16 lanes by lane swaps, a row by rotations.  Every lane gets the
// result, and lanes are paired as in a butterfly of shuffles by the same distances, but a shuffle is a round trip to the LDS and
// the six of a wave's sum wait for each other.
struct AddOp { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct MaxOp { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
template <int N> __device__ __forceinline__ float row_rotated(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
}
template <typename F> __device__ __forceinline__ float reduce_halves(float v, F op) {         // lanes l and l ^ 32
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
template <typename F> __device__ __forceinline__ float reduce_row_pairs(float v, F op) {      // lanes l and l ^ 16
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
template <typename F> __device__ __forceinline__ float reduce_row(float v, F op) {            // the 16 lanes of a row (after a step by n the values have period n)
    v = op(v, row_rotated<8>(v));
    v = op(v, row_rotated<4>(v));
    v = op(v, row_rotated<2>(v));
    return op(v, row_rotated<1>(v));
}
// lanes that agree modulo FROM = 8, 16 or 32
template <int FROM, typename F> __device__ __forceinline__ float reduce_across(float v, F op) {
    static_assert(FROM == 8 || FROM == 16 || FROM == 32, "");
    if (FROM == 8) v = op(v, row_rotated<8>(v));
    if (FROM <= 16) v = reduce_row_pairs(v, op);
    return reduce_halves(v, op);
}
__device__ __forceinline__ float wave_sum(float v) { return reduce_row(reduce_row_pairs(reduce_halves(v, AddOp()), AddOp()), AddOp()); }

// ---------------- projections ----------------
enum GemvMode { MODE_STORE = 0, MODE_RESID = 1, MODE_SWIGLU = 2, MODE_QKV_ROPE = 3 };

struct GemvArgs {
    // activations: fp32 [ncols][x_stride] (ALU path) or their split into bf16 halves in x_form (MFMA path)
    const float* x;
    const bf16_t* x_split;
    SplitForm x_form;
    int x_stride;        // ALU path
    unsigned part_bytes; // what part holds (kPromptPartBytes256 at most)
    const float* gain;   // RMSNorm gain [K] when the norm is fused (ALU path), else nullptr
    float eps;
    int K;
    // up to three row-stacked matrices [rows[m]][K] (STORE/RESID), or {gate, up} (SWIGLU)
    const void* w[3];
    int rows[3];
    int total_rows;      // output rows
    float* out;          // fp32 [ncols][out_stride]
    bf16_t* out_split;   // optional split copy of the output for an MFMA consumer
    SplitForm out_form;
    const float* gain_next;   // [total_rows], see ssq_out
    int out_stride;
    int ncols;
    // MODE_QKV_ROPE only: rotate q and k, append k and v to this block's cache
    const float2* rope_cs;   // [columns of the pass][hd/2] (cos, sin) of pos * base^(-2j/hd)
    void* k_cache;           // this block's [max_batch][H_kv][max_seq][hd]
    void* v_cache;
    ColMap cm;
    int col0;                // pass column of this launch's column 0
    const int2* col_at;      // prompt pass on the matrix cores, instead of cm: (sequence, cache row) of every column
    int H, H_kv, hd, max_seq, kv_dtype;
    // MFMA path, RMSNorm folded into the projections around it.  A projection whose input is a normalised
    // residual (STORE, SWIGLU) gets x * gain pre-split in x_split and scales its sums by
    // 1/sqrt(sum(ssq_in[col][0..ssq_parts)) / K + eps); a residual projection (RESID) with ssq_out set also
    // writes the split of (new x) * gain_next to out_split and its workgroup's sum of squares of the new x
    // to ssq_out[col][workgroup].
    const float* ssq_in;     // [ncols][kSsqStride]
    int ssq_parts;
    float* ssq_out;          // [ncols][kSsqStride]
    // wide MFMA kernel (17..32 columns), K cut into slices: partial accumulators and one arrival counter per row
    // group (zero between launches)
    float* part;
    int* part_tickets;
    // vector-ALU GEMV, set by its launcher: units per wave, and how many waves have one more; 64-lane strides of a row
    int wave_units, wave_units_over;
    Divisor by_strides;
};

// What the first loads of a matrix-core projection need of the arguments, requested together: read as they come up, each is a round trip to memory
// that the next one waits behind.
__device__ __forceinline__ void gemm_take_args(const GemvArgs& a) {
    asm volatile("" :: "s"(a.x_split), "s"(a.x_form.lo), "s"(a.w[0]), "s"(a.w[1]), "s"(a.w[2]), "s"(a.rows[0]), "s"(a.rows[1]),
                       "s"(a.K), "s"(a.total_rows), "s"(a.ncols), "s"(a.ssq_in), "s"(a.ssq_parts));
}
// The matrix that output row `row` of a row-stacked projection belongs to, and the row's number in it (a choice among three scalars: by index, the
// argument is read a second time, from an address that depends on the first).
__device__ __forceinline__ const bf16_t* gemm_row(const GemvArgs& a, int row) {
    const void* w = a.w[0];
    if (row >= a.rows[0]) {
        row -= a.rows[0];
        w = a.w[1];
        if (row >= a.rows[1]) { row -= a.rows[1]; w = a.w[2]; }
    }
    return static_cast<const bf16_t*>(w) + (size_t)row * a.K;
}

// Whether the workgroups of a batched projection begin their rows at different places.  Rows a multiple of 8 KB apart start on the same few memory
// channels, and workgroups that walk them in step meet there; measured, from the first k / from different ones, narrow kernel, 2 columns (8 and 16 alike):
//   rows of 16 KB  70B shape, gate/up 156.4 / 141.6 us (8 columns 6.6 TB/s), QKV 35.7 / 33.0, lm_head 90.1 / 81.4; QKV of 64 KV heads 81.0 / 70.8
//           24 KB  QKV 60.4 / 59.4, O 57.2 / 55.8, gate/up 121.9 / 119.8 (12288 wide); down 38.0 / 35.7
//           32 KB  gate/up 276 / 209, O 97.6 / 84.7, QKV 137.4 / 127.0 (16384 wide); down 81.0 / 66.2
//           40 KB  QKV 173.5 / 171.6, O 167.6 / 165.3 (20480 wide); down 107.2 / 104.2
//      48, 56 KB  down 41.1 / 39.7, 77.0 / 75.2
// Not where rows are 8 KB or no multiple of it: 7B and 13B shapes, 2 blocks and the head, 2 columns 231 / 233 and 310 / 312, 12 columns 261 / 265 and
// 350 / 351.
inline bool gemm_rounds(int K) { return K % 4096 == 0 && K >= 8192; }

// Launch-shape overrides for measurements, read from the environment ONCE by d3_create (0 / default = the library's
// own choice).  D3_MFMA_RT, D3_MFMA_WAVES: row tiles per workgroup and waves of the narrow matrix-core projection;
// D3_MFMA_WIDE=0: no panel kernel (passes are limited to kMaxCols columns); D3_WIDE_RT, D3_WIDE_KS: row tiles per wave
// and K slices of the panel kernel; D3_WIDE_SPLIT_MB: matrix size above which a pass of more than 64 columns runs as
// two 64-column launches; D3_ATTN_MFMA=0: grouped-query and query-tile attention on the vector ALUs;
// D3_ATTN_MIN_SPLIT: shortest context split; D3_PREFILL_COLS: columns per prompt chunk (a multiple of 64, at most kPassCols); D3_PROMPT_KS: K parts of the projections of the prompt pass (1..8; a contraction without two stages for every part stays whole);
// D3_PROMPT_TILE: 128 or 256, columns of a tile of the prompt pass's projections (default: the launcher's estimate with an fp16 cache, 128 with an fp32 one; D3_PROMPT_KS and D3_PROMPT_CUS mean tiles of 128 unless it says 256);
// D3_PROMPT_ROW_BLOCKS: fewest blocks of 256 rows for which 65..128 columns take the LDS-tiled kernel;
// D3_PROMPT_CUS: compute units a round of its tiles is taken to have;
// D3_PROMPT_ATTN_WGS: fewest workgroups (128 (query, head) pairs each) for which a prompt pass, shared or not, takes the whole-context attention kernel; D3_GEMV_WGS_PER_CU: workgroups
// of eight waves per compute unit of the vector-ALU GEMV (default 1).
struct Tuning {
    int gemv_wgs_per_cu = 1;
    int mfma_rt = 0, mfma_waves = 0;
    bool mfma_wide = true;
    int wide_rt = 0, wide_ks = 0;
    size_t wide_split_mb = 300;
    bool attn_mfma = true;
    int attn_min_split = 128;
    int prefill_cols = 0;
    int prompt_ks = 0, prompt_cus = 0, prompt_row_blocks = 20, prompt_tile = 0;
    int prompt_attn_wgs = 0;
};
Tuning tuning_from_env();

// returns hipError_t as int
int launch_gemv_alu(const GemvArgs& a, int weight_dtype, int mode, bool norm, int n_wg, hipStream_t s);
// n_groups: workgroups launched (= parts written to ssq_out)
int launch_gemm_mfma(const GemvArgs& a, int mode, int n_cu, const Tuning& tn, hipStream_t s, int* n_groups = nullptr);
int launch_gemm_mfma_wide(const GemvArgs& a, int mode, int n_cu, const Tuning& tn, hipStream_t s, int* n_groups);   // 17..128 columns
bool gemm_prompt_takes(const GemvArgs& a, int mode, const Tuning& tn);   // launch_gemm_mfma sends the launch to launch_gemm_prompt
// gemm_prompt_256.hip, which launch_gemm_prompt chooses by this estimate (in its own unit; infinite: not for that kernel); part_bytes: 0 without part buffer
double gemm_prompt_256_cost(int mode, int total_rows, int K, int ncols, size_t part_bytes, int n_cu);
int launch_gemm_prompt_256(const GemvArgs& a, int mode, int n_cu, hipStream_t s, int* n_groups);
// The choice of a launch whose activations are in lines: tiles of 256 columns.
bool prompt_takes_large_tiles(int mode, int total_rows, int K, int ncols, size_t part_bytes, int n_cu, const Tuning& tn);
// Whether a prompt pass keeps its split activations in lines, because its projections then take less (launch_gemm_prompt).
struct PromptDims { int d_model, q_dim, qkv_rows, d_ffn; bool rope_in_qkv; };
bool prompt_pass_in_lines(const PromptDims& d, int ncols, size_t part_bytes, int n_cu, const Tuning& tn);
int launch_gemm_prompt(const GemvArgs& a, int mode, int n_cu, const Tuning& tn, hipStream_t s, int* n_groups);   // up to kPassCols columns: LDS-tiled, compute-bound
size_t gemv_alu_max_cols(int K, int weight_dtype);   // columns one ALU launch can take (LDS bound)

// split = x * gain (bf16 halves), ssq[col * kSsqStride] = sum(x^2)
int launch_gain_split(const float* x, int x_stride, const float* gain, int K, int ncols,
                      bf16_t* split, float* ssq, SplitForm form, hipStream_t s);

// ---------------- the rest of a block ----------------
// x[c][:] = E[token(c)][:], and the pass's rotary table rope_cs[c][j] = (cos, sin)((pos(c) - row0[seq(c)]) * inv_freq[j])
// (row0 optional: the first cache row of each sequence of a left-padded batch)
// What a pass on the matrix-core path starts from, beside x (gain NULL: not wanted; bf16 tables only): launch_gain_split's outputs.
struct EmbedSplit { const float* gain; bf16_t* split; float* ssq; SplitForm form; };
// The columns of `runs`: tokens [B][P] of the cache rows from pos_begin on; also col_at[c] = (sequence, cache row) of every column.
int launch_embed_runs(const void* tok_emb, const int32_t* tokens, const SeqRuns& runs, int P, int pos_begin, int ncols, int d, int vocab,
                      float* x, const double* inv_freq, int half_hd, float2* rope_cs, const int* row0, int2* col_at, const EmbedSplit& split, hipStream_t s);   // bf16 table
// dst[row[r]][:] = x[col[r]][:], r < n: the last position of every sequence that a prompt pass finishes
struct RowPick { int n, col[kMaxCols], row[kMaxCols]; };
int launch_pick_rows(const float* x, int d, const RowPick& pick, float* dst, hipStream_t s);
int launch_embed(const void* tok_emb, int weight_dtype, const int32_t* tokens, ColMap cm, int ncols, int d,
                 int vocab, float* x, const double* inv_freq, int half_hd, float2* rope_cs, const int* row0, const EmbedSplit& split, hipStream_t s);

struct RopeArgs {
    float* qkv;            // [ncols][(H + 2 H_kv) * hd] fp32: q rotated in place
    void* k_cache;         // this block's [max_batch][H_kv][max_seq][hd]
    void* v_cache;
    const float2* rope_cs;   // [ncols][hd/2] (cos, sin) of this pass
    ColMap cm;
    const int2* col_at;      // instead of cm: (sequence, cache row) of every column
    int ncols, H, H_kv, hd, max_seq;
};
int launch_rope_append(const RopeArgs& a, int kv_dtype, hipStream_t s);

struct AttnArgs {
    const float* q;        // [ncols][q_stride]: q heads, then (rope_cs set) the newest k and v rows; rotated unless rope_cs is set
    const float2* rope_cs; // optional [ncols][hd/2] (cos, sin): rotate q and k here and append the newest K/V row
    const int* row0;       // optional [B]: first cache row of each sequence (a left-padded batch); rows below it are never read
    int qtile;             // the columns are consecutive positions of one sequence (a prompt chunk): tiles of queries share the cache rows
    int q_stride;
    const void* k_cache;   // this block's cache
    const void* v_cache;
    ColMap cm;
    int ncols, H, H_kv, hd, max_seq;
    int split_len, n_splits;
    float* part_o;         // [ncols][H][n_splits][hd]
    float* part_ml;        // [ncols][H][n_splits][2]  (max, sum)
    int* tickets;          // [ncols][H] arrival counters, zero between launches
    float* out;            // [ncols][H*hd]
    bf16_t* out_split;     // optional split copy
    SplitForm out_form;
    // set by launch_attention: what the kernel divides by: columns per position, query heads per KV head, split length
    Divisor by_b, by_group, by_split;
};
int launch_attention(const AttnArgs& a, int kv_dtype, bool use_mfma, hipStream_t s);

int launch_attention_prompt(const AttnArgs& a, const SeqRuns& runs, int kv_dtype, hipStream_t s);   // attention_prompt.hip

int launch_argmax(const float* logits, int vocab, int ncols, int32_t* out, hipStream_t s);

struct FillArgs {
    void* k_cache;         // whole cache [L][max_batch][H_kv][max_seq][hd]
    void* v_cache;
    int max_batch, H_kv, max_seq, hd;
    int B, pos_begin, pos_end;
    int drop_begin, n_drop, src;   // src < 0: zero fill
};
int launch_fill(const FillArgs& a, int kv_dtype, hipStream_t s);

// read-only streaming yardstick: reads `bytes` (a multiple of 16) once; sink: n_wg * 4 words
int launch_stream_read(const void* src, size_t bytes, unsigned* sink, int n_wg, hipStream_t s);
int launch_mfma_yardstick(int mode, int stages, int n_wg, float* sink, hipStream_t s);   // gemm_prompt.hip

// The words of state a decode step expects in its scratch area, passed by value (no host buffer to copy from) and
// written by one small kernel, which also zeroes the arrival counters.
struct StaticSeed {
    double inv_freq[64];   // head_dim / 2 <= 64 rotary frequencies
    int row0[kMaxCols];    // first cache row of each sequence (all zero unless the batch is left-padded)
};
int launch_static_seed(const StaticSeed& seed, double* inv_freq, int half_hd, int* row0, int* tickets, int n_tickets,
                       int* gemm_tickets, int n_gemm_tickets, hipStream_t s);

}  // namespace d3
