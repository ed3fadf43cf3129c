// Matrix instructions of gfx950 per operand type, shared by the GEMM kernels.
#pragma once
#include "ss_common.h"
#include "packed_layout.h"
#include "device_info.h"

namespace ss {

// Sparse: one instruction is 32 channels x 32 tokens x 64 lifted bytes (sparse) or 16 x 16 x 128 (sparse16), A = 16 bytes of
// stored values + an index word per lane, B = 32 bytes per lane in both.  Dense: DENSE_SUB k-bytes per instruction, A and B
// DENSE_SUB / 2 bytes per lane; lane (row, q) holds the bytes [q DENSE_SUB / 2, (q + 1) DENSE_SUB / 2) of
// its row within the instruction's k range, for both operands (measured: element e of A lane (i, q)
// meets element e of B lane (n, q)).
template <int DT> struct Mma;
template <> struct Mma<SS_I8> {
    typedef v16i acc_t;
    typedef v4i acc16_t;
    typedef v4i dfrag_t;
    static constexpr int ES = 1;                       // bytes per element
    static constexpr int DENSE_SUB = 32;
    static constexpr bool SCALED = true;
    __device__ static acc_t sparse(v4i a, v8i b, acc_t c, int idx) { return __builtin_amdgcn_smfmac_i32_32x32x64_i8(a, b, c, idx, 0, 0); }
    __device__ static acc16_t sparse16(v4i a, v8i b, acc16_t c, int idx) { return __builtin_amdgcn_smfmac_i32_16x16x128_i8(a, b, c, idx, 0, 0); }
    __device__ static acc_t dense(dfrag_t a, dfrag_t b, acc_t c) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0); }
};
template <> struct Mma<SS_FP8_E4M3> {
    typedef v16f acc_t;
    typedef v4f acc16_t;
    typedef v8i dfrag_t;
    static constexpr int ES = 1;
    static constexpr int DENSE_SUB = 64;
    static constexpr bool SCALED = true;
    __device__ static acc_t sparse(v4i a, v8i b, acc_t c, int idx) { return __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(a, b, c, idx, 0, 0); }
    __device__ static acc16_t sparse16(v4i a, v8i b, acc16_t c, int idx) { return __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(a, b, c, idx, 0, 0); }
    // format selectors 0 = e4m3 for both operands; block scales 0 = the unscaled form of the instruction
    __device__ static acc_t dense(dfrag_t a, dfrag_t b, acc_t c) { return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0); }
};
template <> struct Mma<SS_BF16> {
    typedef v16f acc_t;
    typedef v4f acc16_t;
    typedef v4i dfrag_t;
    static constexpr int ES = 2;
    static constexpr int DENSE_SUB = 32;
    static constexpr bool SCALED = false;
    __device__ static acc_t sparse(v4i a, v8i b, acc_t c, int idx)
    {
        return __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v16bf, b), c, idx, 0, 0);
    }
    __device__ static acc16_t sparse16(v4i a, v8i b, acc16_t c, int idx) { return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v16bf, b), c, idx, 0, 0); }
    __device__ static acc_t dense(dfrag_t a, dfrag_t b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    }
};

template <> struct Mma<SS_FP16> {
    typedef v16f acc_t;
    typedef v4f acc16_t;
    typedef v4i dfrag_t;
    static constexpr int ES = 2;
    static constexpr int DENSE_SUB = 32;
    static constexpr bool SCALED = false;
    // same operand geometry as bf16 (checked by the parity tests against the oracle)
    __device__ static acc_t sparse(v4i a, v8i b, acc_t c, int idx)
    {
        return __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v16h, b), c, idx, 0, 0);
    }
    __device__ static acc16_t sparse16(v4i a, v8i b, acc16_t c, int idx) { return __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v16h, b), c, idx, 0, 0); }
    __device__ static acc_t dense(dfrag_t a, dfrag_t b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
    }
};

// two fp32 -> packed bf16 (round to nearest even) in one v_cvt_pk_bf16_f32
__device__ inline uint32_t pack_bf16x2(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Several elements of Y in one store, also where its rows lie off a 16-byte line: a global store needs no alignment beyond that of an
// element.  By single elements every token of a wavefront is another line that gets 16 stores of two bytes.  Fused rows, single elements and now: 128 -> 727 INT8
// at M = 64 6.8 -> 3.5 us, 1216 -> 6382 bf16 at M = 639 32.0 -> 16.2, 384 -> 7291 INT8 at M = 128 8.4 -> 4.8.  Rows on such a line: 0.97 .. 1.03 (two runs of one side
// differ as much).
typedef uint32_t piece16_t __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t piece8_t __attribute__((ext_vector_type(2), aligned(2)));

// Epilogue of one accumulator block held by one lane: a[r] is channel o_lane + r (16 consecutive channels) of token
// tok; Y = bf16((float(a) * sx) * sw_lds[r]) (SCALED; the channels' scales lie in LDS) or bf16(a).  Out-of-range tokens and channels are skipped.
template <bool SCALED, typename ACC>
__device__ inline void store_block16(const ACC& a, float sx, const float* sw_lds, uint16_t* __restrict__ Y, int64_t ldy, int64_t M, int64_t O, int64_t o_lane,
                                     int64_t tok)
{
    if (tok >= M || o_lane >= O) return;
    uint32_t w[8];
    if constexpr (SCALED) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 sw = reinterpret_cast<const float4*>(sw_lds)[q];
            w[2 * q] = pack_bf16x2(((float)a[4 * q] * sx) * sw.x, ((float)a[4 * q + 1] * sx) * sw.y);
            w[2 * q + 1] = pack_bf16x2(((float)a[4 * q + 2] * sx) * sw.z, ((float)a[4 * q + 3] * sx) * sw.w);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = pack_bf16x2((float)a[2 * q], (float)a[2 * q + 1]);
    }
    uint16_t* dst = Y + tok * ldy + o_lane;
    if (o_lane + 16 <= O) {
        reinterpret_cast<piece16_t*>(dst)[0] = piece16_t{w[0], w[1], w[2], w[3]};
        reinterpret_cast<piece16_t*>(dst)[1] = piece16_t{w[4], w[5], w[6], w[7]};
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (o_lane + e < O) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
    }
}

// Epilogue of four consecutive channels o .. o + 3 (o < O) of an existing token tok held by one thread (the split-k reduce kernels):
// Y = bf16((float(a) * sx) * sw[e]) (SCALED) or bf16(a).  Out-of-range channels are skipped.
template <bool SCALED, typename QUAD>
__device__ inline void store_quad4(const QUAD& a, float sx, const float (&sw)[4], uint16_t* __restrict__ Y, int64_t ldy, int64_t O, int64_t o, int64_t tok)
{
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = (float)a[e];
        if constexpr (SCALED) v[e] = (v[e] * sx) * sw[e];
    }
    const uint32_t w[2] = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    uint16_t* dst = Y + tok * ldy + o;
    if (o + 4 <= O && (((uintptr_t)dst) & 7) == 0) *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
    else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (o + e < O) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
    }
}

// Split k, tiles of 128 channels: the raw accumulators of k-range s of tile `tile` go to the workspace as
// ws[s][tile][wave][f][tb][register quad][lane] 16-byte groups (512 TM bytes per tile and range, coalesced).  `tokens` of
// this wavefront's exist (may be <= 0); nothing is written for the others.
template <typename ACC, int FW, int TB>
__device__ inline void mid_store_partial(const ACC (&acc)[FW][TB], void* ws, int64_t item, int wave, int lane, int tokens)
{
    v4i* dst = static_cast<v4i*>(ws) + ((item * 4 + wave) * (4 * FW * TB)) * 64 + lane;
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
            if (tb * 32 + (lane & 31) < tokens)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                typedef decltype(acc[0][0][0] + acc[0][0][0]) elem_t;
                const elem_t q[4] = {acc[f][tb][4 * r4], acc[f][tb][4 * r4 + 1], acc[f][tb][4 * r4 + 2], acc[f][tb][4 * r4 + 3]};
                dst[((f * TB + tb) * 4 + r4) * 64] = __builtin_bit_cast(v4i, q);
            }
}

// The k ranges of a split row: U = S q + rest units, one more in the first `rest` ranges.
struct KRanges { int q, rest; };
inline KRanges k_ranges(int64_t U, int64_t S) { return {(int)(U / S), (int)(U % S)}; }
__device__ inline int range_first(KRanges k, int range) { return range * k.q + min(range, k.rest); }
__device__ inline int range_units(KRanges k, int range) { return k.q + (range < k.rest); }

// Kernels for few tokens (gemm_skinny.hip): one workgroup per 32 or 64 output channels streams their weights once.
// The dense kernel splits its k range over S workgroups per fragment where there are fewer 32-channel fragments than
// compute units; partial sums go through `ws` (skinny_workspace_bytes(M, O, S) bytes) and a second kernel adds them in a
// fixed order.  (Sparse shapes that gain from a split run on the tiles of gemm_mid.hip.)
constexpr int64_t SS_SKINNY_MAX_M = 64;
int skinny_splits(int64_t M, int64_t O, int64_t units, size_t ws_bytes);
size_t skinny_workspace_bytes(int64_t M, int64_t O, int S);
ss_status launch_sparse_skinny(const void* XL, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                               int64_t Kpb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream);
// the same for unlifted activations and weights packed by slide_decompose_fused (6:8): U super-units of 128 bytes per row,
// ldxb bytes between token rows
ss_status launch_sparse_fused_skinny(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                                     int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream);
ss_status launch_dense_skinny(const void* Xq, const float* s_x, const void* Wq, const float* s_w, int64_t M, int64_t O, int64_t Kb, ss_dtype dtype,
                              void* Y, int64_t ldy, void* ws, int S, hipStream_t stream);

// Tiles of 128 channels x 256 tokens for unlifted activations (gemm_fused_narrow.hip), operands as for the fused kernels below.
ss_status launch_sparse_fused_narrow(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                                     int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream);

// The 256 x 256 tile kernels: lifted rows (gemm_lifted.hip), dense (gemm.hip).
ss_status launch_sparse_tile(const void* XL, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int64_t Kpb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream);
ss_status launch_dense_tile(const void* Xq, const float* s_x, const void* Wq, const float* s_w, int64_t M, int64_t O, int64_t Kb, ss_dtype dtype,
                            void* Y, int64_t ldy, hipStream_t stream);

// Kernels that read every weight once load them non-temporally where the packed weights (rows of `lifted` bytes) are `limit` and more: a
// third of the memory-side cache, which then keeps the smaller layers and the activations, or all of it.  128 MB streamed into LDS: 20.3 us non-temporal, 23.2 otherwise.
// Time over that of ordinary loads, packed weights of 80 to 256 MB, from HBM / hot in that cache (where a model of many layers never finds them):
//   up to 32 tokens                                                   0.84 .. 0.98 (mean 0.89) / 0.86 .. 1.23 (1.04; the most at 32 tokens)
//   33 to 64 tokens, 257 to 512 panels (gemm_wide.hip)                0.86 .. 0.98 (0.90) / 0.94 .. 1.23 (1.05)
//   33 to 64 tokens, tiles of 64, a compute unit each, 8-bit types    0.91 .. 0.96 (0.94) / 1.01 .. 1.26 (1.13)
//   the same, 16-bit types                                            0.95 .. 1.00 (0.98) / 1.06 .. 1.46 (1.17)
//   the same on shared compute units (more than 512 panels)           0.92 .. 1.06 (0.97) / 1.11 .. 1.35 (1.19)
//   97 to 128 tokens, 257 to 384 panels (gemm_wide.hip)               0.83 .. 1.03 (0.96) / 1.01 .. 1.33 (1.10)
// The limit is a third of the cache in the first three, all of it in the others, whose gain is not worth that loss.  Weights of 256 MB and more: 0.81 .. 0.98
// / 0.80 .. 1.08 in all of them.  Smaller layers gain less from HBM (0.95 .. 1.04) and lose hot (1.0 .. 1.27); the 128 x 128 tiles 0.98 .. 1.02.
inline bool weights_stream(int64_t O, int64_t lifted, int64_t limit) { return O * (lifted / 8 * 5) >= limit; }

enum ss_kind { SS_KIND_LIFTED, SS_KIND_FUSED, SS_KIND_DENSE };      // sparse from lifted rows, sparse that lifts itself, dense

// Few tokens as a stream of weights (gemm_wide.hip): up to 32 tokens on as many panels as compute units or fewer, up to 64 on up to twice, unlifted rows of
// 97 to 128 on up to one and a half times as many.
// X: lifted rows, or unlifted ones and weights of slide_decompose_fused; U units of 128 bytes per row, ldxb bytes between rows.
// S > 1 (NF = 4): partial sums as of the 32-token tiles of gemm_mid.hip go through `ws`.
ss_status launch_sparse_wide(bool fused, const void* X, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream);
// fragments of 32 channels that a workgroup of theirs takes, 0 where they are not used
inline int wide_fragments(ss_kind kind, int64_t M, int64_t O, int64_t cus)
{
    const int64_t frags = (O + 127) / 128 * 4, f = (frags + cus - 1) / cus;
    if (M > 64 ? kind != SS_KIND_FUSED || M <= 96 || M > 128 || f > 6 : f > 8) return 0;
    if (f <= 4) return M <= 32 && f >= 3 ? 4 : 0;
    return f == 7 ? 8 : (int)f;
}

// Small unsplit tiles (gemm_small.hip): fw fragments x tb blocks of 32 tokens, kg groups of wavefronts.  Operands as above.
struct small_tile { int fw, tb, kg; };
ss_status launch_sparse_small(bool fused, const void* X, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                              int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, small_tile tile, hipStream_t stream);
inline int64_t small_workgroups(int64_t M, int64_t O, small_tile t) { return (O + 127) / 128 * (FRAGS_PER_PANEL / t.fw) * ((M + 32 * t.tb - 1) / (32 * t.tb)); }
// the smallest that gives no compute unit two workgroups; fw = 0: none does
inline small_tile small_shape(int64_t M, int64_t O, int64_t units, int64_t cus)
{
    for (small_tile t : {small_tile{1, 1, 4}, {2, 1, 4}, {2, 2, 3}, {2, 3, 2}, {2, 4, 2}})
        if (units >= t.kg && M > 32 * (t.tb - 1) && small_workgroups(M, O, t) <= cus) return t;
    return {0, 0, 0};
}
// Where they are used, by the lines a workgroup loads for its row.  `split`: the call would otherwise be split into k ranges.  Time over the kernels
// before these, 5700 calls on 80 to 100 % of the compute units or just within a line, all types, weights from HBM / hot, means in parentheses:
//   not split  M <= 16 (where gemm_slim.hip does not serve the call) on 33 to 64 panels 0.87 .. 1.03 (0.94) / 0.68 .. 0.99 (0.84), on 65 to 128 with 12 units
//              and more 0.80 .. 1.04 (0.93; of 600 others at most 1.07) / 0.66 .. 1.06 (0.87); 4 to 9 units, which stay on gemm_skinny.hip, 0.90 .. 1.11 /
//              0.86 .. 1.10;  M <= 32 0.68 .. 1.04 (0.89) / 0.48 .. 0.97 (0.74), M <= 64 0.48 .. 1.04 (0.71) / 0.35 .. 1.01 (0.59)
//              M > 64, tiles of 32 tokens 0.27 .. 0.72 (0.48) / 0.24 .. 0.68 (0.46), 64 0.34 .. 0.81 (0.60) / 0.32 .. 0.81 (0.62), 96 0.30 .. 0.94 (0.69) /
//              0.28 .. 0.91 (0.71), 128 0.33 .. 0.91 (0.73) / 0.32 .. 1.06 (0.79)
//   split      M <= 64 0.71 .. 1.01 (0.88) / 0.64 .. 0.75 (0.69)
//              M > 64, tiles of 32 tokens 0.49 .. 0.92 (0.69) / 0.41 .. 0.71 (0.56), 64 0.53 .. 1.01 (0.78) / 0.48 .. 0.94 (0.69), 96 0.51 .. 1.03 (0.80) /
//              0.46 .. 0.98 (0.77), 128 0.67 .. 0.98 / 0.57 .. 1.04 (5200 lines and more to 1.09)
//   three units, 33 to 48 tokens, on the tiles of three groups 0.97 .. 1.08 of the few-token kernel of before, on the 64-token tiles of gemm_mid.hip
//              0.71 .. 0.96 / 0.71 .. 1.03, which take them; with 64 tokens level (0.82 .. 1.00 and 0.78 .. 0.94), and off a 16-byte line of Y the small tiles
//              are the faster (0.54 .. 0.79 and 0.55 .. 0.87)
// Beyond the lines, these tiles over the ranges that run there, 2100 calls, means by how far beyond:
//   M <= 16    40 to 59 units 1.00 (0.88 .. 1.17); 60 to 79 on 8 to 15 panels 1.17, 16 to 23 1.10, 24 to 35 1.02, 36 to 64 0.94 (0.85 .. 1.01) / 0.85; 80 to 99
//              on 36 to 64 0.97 (0.89 .. 1.14) / 0.86, on fewer 1.06 .. 1.33; 100 and more 1.01 .. 1.66.  No line is drawn around those that gain
//   M <= 32    up to 1.2 times the line 1.01 (0.96 .. 1.18) / 0.99, 1.4 1.10 / 0.94, 1.6 1.18 / 0.91;  M <= 64 1.00 (0.85 .. 1.13) / 0.93, 1.04 / 0.89, 1.08 / 0.91
//   M > 64     32 tokens 0.84 (0.63 .. 1.05) / 0.71, 0.91 (0.63 .. 1.18) / 0.75, 0.97 / 0.77; 64 0.95 (0.82 .. 1.08) / 0.86, 0.99 / 0.90, 1.06 / 0.96;
//              96 0.98 (0.86 .. 1.19) / 0.96, 0.96 / 0.99, 1.06 / 1.11; 128 0.94 / 0.93, 0.97 / 0.97
inline bool small_pays(int64_t M, int64_t units, small_tile t, int64_t workgroups, bool fused, bool split)
{
    if (t.fw == 0 || (M <= 48 && units < 4)) return false;
    const int64_t lines = units * (32 * t.tb + t.fw * (fused ? 30 : 20));
    if (M <= 16) return !split && (t.fw == 1 || units >= 12);
    if (!split) return true;
    if (M <= 64) return lines <= (M > 32 && workgroups >= 128 ? 3200 : 2400);
    return lines <= (t.tb == 1 ? 3100 : t.tb == 2 ? 5900 : t.tb == 3 ? 7400 : 5000);
}
// Up to 16 tokens with a workgroup for every 16 channels (gemm_slim.hip), unsplit; operands as above.
ss_status launch_sparse_slim(bool fused, const void* X, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream);
// Every one of its workgroups reads all token rows, so the lines go by units and tokens.  `split`: the call would otherwise be split into k ranges.  Time
// over the kernels of before, all types, weights from HBM / hot, M = 1 .. 16:
//   at most one workgroup per compute unit, not split: 1 to 56 units 0.57 .. 0.90 / 0.55 .. 0.82, without a workspace 72 to 256 units 0.48 .. 0.93 / 0.44 .. 0.92
//   the same, split, 8 panels and more, by units (M + 8): up to 1000 0.74 .. 1.04 (mean 0.88) / 0.54 .. 0.89 (0.68), 1000 .. 1400 0.93 .. 1.33 / 0.66 .. 1.03, more
//     1.1 .. 2.0.  The worst are unlifted rows of one to four tokens on 8 to 10 panels, 9.5 units a panel and more: 1.00 .. 1.08 from HBM, but 0.70 .. 0.77 hot, so they
//     stay here (in ranges they were 0.97 of the time from HBM and 1.35 hot).  Fewer panels would leave most compute units idle, which their ranges do not
//   some compute units with two of them, by units (M + 2): up to 120 0.76 .. 0.99 / 0.76 .. 1.00 (3584 -> 4608 INT8 at M = 1 7.2 -> 6.9 us, hot 5.7 -> 4.4), 120 ..
//     170 0.88 .. 1.10 / 0.79 .. 0.98
inline bool slim_pays(int64_t M, int64_t O, int64_t units, int64_t cus, bool split)
{
    const int64_t panels = (O + 127) / 128, wgs = 8 * panels;
    if (M > 16 || wgs > 2 * cus) return false;
    if (wgs > cus) return units * (M + 2) <= 120;
    return !split || (panels >= 8 && units * (M + 8) <= 1000);
}

// Up to 32 tokens of lifted rows on half to two thirds as many panels as compute units: tiles of 32 tokens in two groups of wavefronts (gemm_mid.hip),
// not the weight stream.  A unit of lifted rows is two steps, and a wavefront for each SIMD waits for its operand reads longer than it
// multiplies; with half of the compute units idle the loads do not cover that.  Time over the stream, M = 1 .. 32, 12 to 100 units, weights
// from HBM / hot: 129 panels 0.88 .. 1.04 / 0.82 .. 1.02 (mean 0.99 / 0.90; fp8 3584 -> 16512 at M = 16 15.2 against 15.1 us, hot 11.3 against 13.8), 148 panels 0.88 .. 1.05 /
// 0.83 .. 1.03 (1.00 / 0.93), 170 panels 0.96 .. 1.06 / 0.88 .. 1.01 (1.01 / 0.95), 191 panels 0.97 .. 1.09 / 0.88 .. 1.08 (1.02 / 1.00), 256 panels 0.95 .. 1.05 /
// 0.95 .. 1.15 (1.00 / 1.01); ten units and fewer lose.  Unlifted rows gain from HBM by the stream (129 panels, M = 16 and 32: 0.98, hot 1.07).  M < 16 over the
// few-token kernels, 16 to 64 units: 0.70 .. 1.00 / 0.77 .. 1.08.
inline bool two_groups(int64_t M, int64_t O, int64_t units, int64_t cus)
{
    const int64_t panels = (O + 127) / 128;
    return M <= 32 && units >= (M < 16 ? 16 : 12) && 2 * panels >= cus + (M < 16) && 3 * panels <= 2 * cus;
}

// Kernels with tiles of 128 channels x 128 tokens, sparse ones also x 64 and x 32 where the tokens fit (gemm_mid.hip),
// for shapes that give the 256 x 256 tile kernels too few tiles to occupy the compute units.
// S > 1 splits the k range over S workgroups per tile; their partial sums go through `ws`
// (mid_workspace_bytes(kind, M, O, S) bytes) and a second kernel adds them in a fixed order.
ss_status launch_sparse_mid(const void* XL, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                            int64_t Kpb, ss_dtype dtype, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream);
// the same for unlifted activations and weights packed by slide_decompose_fused (6:8): U super-units of 128 bytes per row,
// ldxb bytes between token rows
ss_status launch_sparse_fused_mid(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                                  int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream);
ss_status launch_dense_mid(const void* Xq, const float* s_x, const void* Wq, const float* s_w, int64_t M, int64_t O, int64_t Kb, ss_dtype dtype,
                           void* Y, int64_t ldy, void* ws, int S, hipStream_t stream);
// the second kernel alone, for the partial sums of 32-token tiles
ss_status launch_mid_reduce32(const void* ws, int S, const float* s_x, const float* s_w, int64_t M, int64_t O, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream);
int mid_splits(ss_kind kind, int64_t M, int64_t O, int64_t units, size_t ws_bytes);
size_t mid_workspace_bytes(ss_kind kind, int64_t M, int64_t O, int S);
inline int64_t mid_tiles(int64_t M, int64_t O) { return ((O + 127) / 128) * ((M + 127) / 128); }
inline int64_t narrow_tiles(int64_t M, int64_t O) { return ((O + 127) / 128) * ((M + 255) / 256); }

// Which kernel family a GEMM of M tokens x O channels over `units` 128-byte k units runs on, and in how many k
// ranges (S > 1 only with a workspace).  Measured, INT8 6:8 unless said, weights from HBM, us:
//   M > 64    up to 1.25 tiles of 128 x 128 per compute unit those tiles, beyond two of them the 256 x 256 tiles (592, 3584 -> 37888 at
//             M = 256: 76 against 51).  Between, 128 x 128 tiles (two workgroups share a compute unit) where the rows are long
//             enough: their stores go out in shorter pieces, and they read more of their operands from L2.  Time over that of
//             256 x 256 tiles, weights from HBM / hot, by units per row, means over one to fourteen shapes: 321 .. 448 tiles, fused 8-bit 4
//             units 1.07 / 1.01, 8 0.99 / 1.00, 12 0.88 / 0.99, 32 0.82 / 0.93, 16-bit 8 1.02 / 1.02, 12 0.93 / 0.98; lifted 8-bit 12 1.01 / 1.07, 24
//             0.89 / 1.07, 32 0.90 / 1.03, 16-bit 12 1.00 / 1.09, 24 0.94 / 1.03, 32 0.80 / 1.03.  449 .. 512 tiles, fused 8-bit 16 0.96 / 1.07, 24 0.92 /
//             1.08, 32 0.88 / 1.05, 16-bit 24 0.97 / 1.05; lifted 8-bit 32 0.97 / 1.13, 48 0.95 / 1.09, 16-bit 48 0.92 / 1.07.  The lines go by
//             the first figure, a layer's weights coming from HBM in a model of many.
//   on at most half as many 128 x 128 tiles as compute units small unsplit tiles, unless the rows are long and can be split (small_pays) or 16 channels a
//             workgroup serve them (slim_pays).
//   M 33..64  tiles of 64 tokens otherwise (3584 -> 37888: 37 against the few-token kernel's 50; split: bf16 3584 -> 4608 13.9 against 23.6, fp8 lifted
//             4096 -> 6144 13.9 against 19.9).
//   M <= 32   a workgroup per panel (and k range; gemm_wide.hip) where there are more panels than half of the compute units (rows of 16 units and more: 3584 -> 18944
//             at M = 1, 148 panels: INT8 14.4 against 17.3, bf16 21.2 against 29.6; shorter ones by `wide` below) or the rows are long
//             and can be split (18944 -> 3584, M = 1: 19 against 23; 64 units, 4096 channels bf16, M = 1: 13 against 18;
//             56 units: M = 1 11.8 against 11.5, M = 16 12.4 against 13.9; 48 units: M = 16 11.0 against 10.7, M = 32 11.3
//             against 12.8); lifted rows by two_groups.  The few-token kernels otherwise (28 units, 3584 -> 4608, M = 1: 7.8 against 10.4), up to 16 tokens
//             mostly those of 16 channels a workgroup (slim_pays).  Half as many panels as compute units, 16 to 32 tokens: the stream has one workgroup for a panel,
//             small tiles two, and unlifted rows are streamed the faster from HBM once they are long.  Small tiles over the stream, 900 calls, all types, from HBM / hot,
//             means by units: 4 to 39 0.86 .. 0.90 / 0.62 .. 0.85, 40 to 42 0.89 .. 0.97, 43 and 44 1.05, 48 to 63 1.00 .. 1.03 / 0.76, 84 to 130 1.08 .. 1.14 / 0.76
//             (at most 1.20); lifted rows run on two groups of wavefronts there.
// M <= 64 and 257 .. 512 panels, fused 97 .. 128 tokens and 257 .. 384 panels: workgroups of five, six or eight fragments (gemm_wide.hip), one for each
//             compute unit.  Time over that of a panel for each workgroup, 16 units and more, weights from HBM / hot: M <= 64, INT8, bf16 and fp8 lifted, 120 calls
//             0.64 .. 0.98 / 0.72 .. 1.11 (3584 -> 37888 at M = 1: INT8 29.3 -> 22.1, bf16 53.5 -> 37.9).  Fused, 257 .. 384 panels, two cards, means by tokens: 65 0.94 and
//             0.97 / 1.15 and 1.18, 80 0.91 and 0.94 / 1.13 and 1.16, 96 0.89 and 0.91 / 1.11 and 1.14, 97 0.88 and 0.90 / 1.10 and 1.14, 112 0.87 and 0.89 / 1.09 and 1.10, 128 0.84 and 0.86 / 1.05
//             and 1.06 (3584 -> 37888 at M = 128 INT8 44.4 -> 36.0, hot 28.8 -> 30.5): where three blocks of 32 tokens will do, the loss hot is the larger one.
//             385 .. 512 panels at 65 .. 128 tokens 0.95 .. 1.11 / 0.75 .. 1.05.  Those, lifted rows of more than 64 tokens, and 4 to 12 units (0.91 .. 1.07) keep the tiles.
// Fused, more 128 x 128 tiles than compute units and at most one tile of 128 channels x 256 tokens for each: those
//             (gemm_fused_narrow.hip).  Time over that of the paths above, INT8 and bf16, 4 to 64 units, M = 200 .. 4096,
//             267 shapes: 0.69 .. 0.99 with weights from HBM (mean 0.79), 0.71 .. 1.01 hot.  At the fewest, a middle and the most panels for M = 129 .. 8192, 4
//             to 112 units, all types, 118 shapes: 0.69 .. 0.94 (mean 0.79) and 0.70 .. 1.04; the worst, M = 257 on 128 panels, where half of the tiles
//             hold one token: 0.83 and 1.04.  M = 11000 .. 65536 on four panels to one, 140 shapes, two cards: 0.68 .. 1.06, but on one panel with 50000 tokens and more, rows
//             of 8 and 12 KB (whose lines meet in the same memory channels) 1.00 .. 1.23.  With as many 128 x 128 tiles as compute units or
//             fewer, those (4096 -> 4096 at M = 1024: 23.2 against 26.2); with more than one 128 x 256 tile per compute unit 256 x 256 tiles
//             (fp8 4096 -> 6144 at M = 2048, 192 tiles against 384: 41 against 54).
// The dense kernels keep tiles of 128 tokens and their own lines: M <= 32, and M <= 64 unless the rows are at least 96
// units long and can be split, few-token; up to 320 tiles 128 x 128.
enum ss_path { SS_PATH_SKINNY, SS_PATH_MID, SS_PATH_NARROW, SS_PATH_TILE, SS_PATH_WIDE, SS_PATH_SLIM, SS_PATH_SMALL };
// tile_o: channels the 256 x 256 tiles take, the rest goes to 128 x 128 or 128 x 256 tiles
struct ss_plan { ss_path path; int S; int64_t tile_o = 0; small_tile small = {0, 0, 0}; };
// The 256 x 256 tile kernels run one tile per compute unit and round; a last round that is nearly empty costs as much as a
// full one.  If whole rounds can be cut off along the channels so that the rest is at most one 128 x 128 tile per compute
// unit, the rest goes to those (M = 8192, 3584 -> 4608, 2.25 rounds: bf16 210 -> 194 us, INT8 120 -> 116).  With two of them per
// compute unit (half a round) the two sides are level or worse: half a round runs at a higher clock (lifted INT8 4096 -> 6144 at M =
// 4096: 97 against 102).  Unlifted rows have tiles of 128 x 256 for that: one per compute unit, 16 units
// and more (time over 256 x 256 tiles throughout, INT8, fp8 and bf16, M = 513 .. 8192, weights from HBM, 240 shapes: 4 to 6 units 1.01 .. 1.09 (mean 1.04),
// 8 to 13 0.96 .. 1.09 (1.00), 14 and 15 0.96 .. 1.02 (0.99), 16 to 20 0.93 .. 1.01 (0.985), 24 to 48 0.91 .. 1.01 (0.96): in short rows the second
// launch costs what the rest saves).
inline int64_t tile_channels(ss_kind kind, int64_t M, int64_t O, int64_t units, int64_t cus)
{
    const int64_t tiles_o = (O + 255) / 256, tiles_t = (M + 255) / 256, rounds = tiles_o * tiles_t / cus, c = rounds * cus / tiles_t;
    const int64_t rest = O - c * 256;
    return c > 0 && c < tiles_o && (mid_tiles(M, rest) <= cus || (kind == SS_KIND_FUSED && units >= 16 && narrow_tiles(M, rest) <= cus)) ? c * 256 : O;
}
inline bool narrow_pays(int64_t M, int64_t O, int64_t cus) { return mid_tiles(M, O) > cus && narrow_tiles(M, O) <= cus; }
inline ss_plan plan_gemm(ss_kind kind, int64_t M, int64_t O, int64_t units, size_t ws_bytes)
{
    if (kind == SS_KIND_DENSE) {
        if (M <= 32) return {SS_PATH_SKINNY, skinny_splits(M, O, units, ws_bytes)};
        if (M > 64 && mid_tiles(M, O) > 320) return {SS_PATH_TILE, 1, O};
        const int S = mid_splits(kind, M, O, units, ws_bytes);
        if (M <= 64 && !(S > 1 && units >= 96)) return {SS_PATH_SKINNY, skinny_splits(M, O, units, ws_bytes)};
        return {SS_PATH_MID, S};
    }
    const int64_t tiles = mid_tiles(M, O), cus = cu_count();
    const small_tile small = small_shape(M, O, units, cus);
    if (kind == SS_KIND_LIFTED && two_groups(M, O, units, cus)) return {SS_PATH_MID, 1};
    if (units >= 16 && wide_fragments(kind, M, O, cus)) return {SS_PATH_WIDE, 1};
    if (M > 64) {
        if (kind == SS_KIND_FUSED && narrow_pays(M, O, cus)) return {SS_PATH_NARROW, 1};
        const bool many = 4 * tiles > 7 * cus;                          // more than 448
        const int64_t long_row = kind == SS_KIND_FUSED ? (many ? 24 : 12) : (many ? 48 : 24);
        if (tiles > 2 * cus || (4 * tiles > 5 * cus && units < long_row)) return {SS_PATH_TILE, 1, tile_channels(kind, M, O, units, cus)};
        const int S = mid_splits(kind, M, O, units, ws_bytes);
        if (small_pays(M, units, small, small.fw ? small_workgroups(M, O, small) : 0, kind == SS_KIND_FUSED, S > 1)) return {SS_PATH_SMALL, 1, 0, small};
        return {SS_PATH_MID, S};
    }
    const int S = mid_splits(kind, M, O, units, ws_bytes);
    const bool wide = 4 * tiles >= (M < 16 ? 3 : 2) * cus;
    const bool mid = wide || M > 32 || (S > 1 && 2 * units + M >= 128);
    if (kind == SS_KIND_FUSED && wide && M <= 32 && units > 42) return {SS_PATH_MID, S};
    if (!wide && slim_pays(M, O, units, cus, mid)) return {SS_PATH_SLIM, 1};
    if (small_pays(M, units, small, small.fw ? small_workgroups(M, O, small) : 0, kind == SS_KIND_FUSED, mid && S > 1)) return {SS_PATH_SMALL, 1, 0, small};
    return mid ? ss_plan{SS_PATH_MID, S} : ss_plan{SS_PATH_SKINNY, 1};
}

}  // namespace ss
