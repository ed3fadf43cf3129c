// slide_sparse_gemm_fused on tiles of 128 channels x 256 tokens: shapes whose 256 x 256 tiles are too few to occupy the
// compute units, while 128 x 128 tiles (gemm_mid.hip) read every operand twice as often.
//
// The operand order, the token tile in LDS and the three steps of a pair of super-units are those of gemm_fused.hip; what
// differs follows from the tile.  A wavefront accumulates 64 channels (two fragments of the panel) x 64 tokens: with half
// the accumulators there is room for the operands of two steps, so a step's reads all go out while the one before it runs.
// A step is half as long, so two steps no longer cover the latency of a load: LDS holds three token tiles and the packed
// weights of two pairs (156 KB), and whatever is read was requested three steps (one pair) before.  A workgroup does one
// tile; there is nothing to overlap its epilogue with, and all its rows go out as whole 256-byte segments.
//
// What bounds it: as in the large tiles the power limit (4096 tokens, 8192 -> 2048 INT8 56 us = 1.8 of the 2.5 POP/s that a
// large product reaches), and in short rows the launch, the first loads and the epilogue, about 7 us together.  A pair is 94 KB of
// direct loads (1570 cycles at 60 bytes a clock) beside 1536 cycles of matrix instructions; starting each XCD
// elsewhere in the k range, or bands of four token tiles instead of eight, changed nothing (10 shapes, 0.95 .. 1.06).
// Against the 128 x 128 tiles, time with weights from HBM: fp8 4096 -> 4096 at M = 2048 41.3 -> 31.7 us, 14336 -> 4096 110 ->
// 91.5, INT8 4096 -> 8192 at M = 1024 41.0 -> 31.6, bf16 3584 -> 3584 at M = 2048 54.1 -> 44.7.  Rows of an odd number of super-units
// (70 shapes of 1 to 57): 0.88 .. 0.99 of the time with a whole last pair (mean 0.95).
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "lds_pipe.h"
#include "tile_common.h"
#include "device_info.h"
#include <type_traits>

namespace ss {

constexpr int FN_VALS = 24 * 1024, FN_IDX = 6 * 1024;         // packed weights of a pair: [packed step 6][fragment 4][lane 64][16 B] and [step 6][lane 64][fragment 4][4 B], as in memory
constexpr int FN_BSLOT = BT * ROWB;
constexpr int FN_IDX_OFF = 2 * FN_VALS;
constexpr int FN_B_OFF = FN_IDX_OFF + 2 * FN_IDX;             // 60 KB
constexpr int FN_SW_OFF = FN_B_OFF + 3 * FN_BSLOT;            // 156 KB: channel scales, then token scales
constexpr int FN_SX_OFF = FN_SW_OFF + PANEL * 4;
constexpr int FN_LDS = FN_SX_OFF + BT * 4;
static_assert(FN_LDS <= 160 * 1024, "LDS budget");

// ODD: an odd number of super-units; the last pair has no u1, so no step 1, and zeros in u1's place in step 2
template <int DT, bool ODD>
__global__ __launch_bounds__(512) void k_sparse_fused_narrow(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                             const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int U,
                                                             int64_t ldxb, uint16_t* __restrict__ Y, int64_t ldy, int panels, int tiles_t)
{
    typedef Mma<DT> MM;
    constexpr int ES = MM::ES;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wo = wave & 1, wt = wave >> 1;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t lds0 = lds_address(smem), lane16 = lane * 16;
    const int P = (U + 1) >> 1;                       // pairs
    int to, tt;
    if (!tile_of_round(0, panels, tiles_t, to, tt)) return;
    const int64_t o_blk = (int64_t)to * PANEL, t_blk = (int64_t)tt * BT;

    // Direct loads of this wavefront.  Of a pair: one 1 KB piece of values of packed steps 0, 1 of u0 (group 0) and u1 (group
    // 1), one of packed step 2 of u0 (wavefronts 0 .. 3) or u1 (4 .. 7) (group 2), 768 bytes of index words; of every token tile four times eight rows.
    const uint8_t* const av_src = w_vals + (int64_t)to * U * 12288 + wave * 1024;
    const uint8_t* const am_src = w_meta + (int64_t)to * U * 3072 + wave * 768;
    const uint8_t* const b_src = Xq + t_blk * ldxb;
    uint32_t boff[4];
    {
        const int64_t left = M - t_blk;               // >= 1
        const int last = left > 255 ? 255 : (int)left - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * (i * 8 + wave) + (lane >> 3);
            boff[i] = (uint32_t)(row < last ? row : last) * (uint32_t)ldxb + place((lane & 7) ^ swz(row)) * 16;
        }
    }
    const uint32_t v_wave = lds0 + wave * 1024, m_wave = lds0 + FN_IDX_OFF + wave * 768, b_wave = lds0 + FN_B_OFF + wave * 1024;
    auto load_tokens = [&](auto i_c, int u, uint32_t slot) __attribute__((always_inline)) {
        constexpr int I = decltype(i_c)::value;
        lds_dma16_from<I * 8192>(b_src, (uint32_t)min(u, U - 1) * ROWB, boff[I], b_wave + slot);
    };
    auto load_values = [&](auto group_c, int p, uint32_t area) __attribute__((always_inline)) {
        constexpr int G = decltype(group_c)::value;
        const uint32_t at = G == 0 ? 0u : G == 1 ? 12288u : 8192u + (wave >> 2) * 8192u;
        const bool none = ODD && p + 1 == P && (G == 1 || (G == 2 && wave >= 4));
        lds_dma16_from<0>(none ? reinterpret_cast<const uint8_t*>(no_values) : av_src, none ? 0u : (uint32_t)p * 24576u + at, lane16, v_wave + area * FN_VALS + at);
    };
    // the index words of a u1 that does not exist stay as they are: they choose among tokens that are zero
    auto load_index = [&](int p, uint32_t area) __attribute__((always_inline)) {
        const uint64_t lanes = ODD && p + 1 == P && wave >= 4 ? 0 : (1ull << 48) - 1;
        lds_dma16_lanes_from<0>(am_src, (uint32_t)p * 6144u, lane16, m_wave + area * FN_IDX, lanes);
    };

    if constexpr (MM::SCALED) {                       // the tile's scales: wavefronts 0, 1 those of the channels, 4 .. 7 those of the tokens; beyond the last one it is repeated
        if (wave < 2 || wave >= 4) {
            const int64_t first = wave < 2 ? o_blk + wave * 64 : t_blk + (wave - 4) * 64, end = wave < 2 ? O : M, left = end - 1 - first;
            const int left32 = left > 63 ? 63 : (int)left;
            const uint32_t e = left < 0 ? 0u : (uint32_t)(lane < left32 ? lane : left32);
            lds_dma4_at(reinterpret_cast<const uint8_t*>((wave < 2 ? s_w : s_x) + (left < 0 ? end - 1 : first)), e * 4,
                        lds0 + (wave < 2 ? FN_SW_OFF + wave * 256 : FN_SX_OFF + (wave - 4) * 256));
        }
    }
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    auto tokens4 = [&](int u, uint32_t slot) __attribute__((always_inline)) { load_tokens(c0, u, slot); load_tokens(c1, u, slot); load_tokens(c2, u, slot); load_tokens(c3, u, slot); };
    uint32_t t0 = 0, t1 = FN_BSLOT, tz = 2 * FN_BSLOT;         // token slots of u0 and u1, and that of the next pair's u0
    load_values(c0, 0, 0); load_values(c1, 0, 0); load_values(c2, 0, 0); load_index(0, 0);
    tokens4(0, t0);
    tokens4(1, t1);
    if (P > 1) {
        load_values(c0, 1, 1); load_values(c1, 1, 1); tokens4(2, tz); load_values(c2, 1, 1); load_index(1, 1);
        wait_vmcnt<12>();
    } else wait_vmcnt<0>();
    wg_barrier();

    // LDS byte offsets of this lane's operand reads (area, fragment, rows 16 hh, slot and token block are added as they come)
    const uint32_t l_raw = (n + 32 * (g >> 1)) * 16, l_mid = (n + 32 * (g & 1)) * 16;
    const uint32_t va_raw = (g & 1) * 4096 + wo * 2048 + l_raw, va_mid = (2 + 3 * (g >> 1)) * 4096 + wo * 2048 + l_mid;
    const uint32_t vi_raw = FN_IDX_OFF + (g & 1) * 1024 + wo * 8 + l_raw, vi_mid = FN_IDX_OFF + (2 + 3 * (g >> 1)) * 1024 + wo * 8 + l_mid;
    const uint32_t vb = FN_B_OFF + (wt * 64 + n) * ROWB + 16 * (place(4 * (g & 1) + 2 * (g >> 1)) ^ swz(n));

    typedef int v2i __attribute__((ext_vector_type(2)));
    struct Ops { v4i a[4]; v2i ix[2]; v8i raw[4]; };           // a[2 f + hh]: rows 16 hh of fragment 2 wo + f; ix[hh]: the words of both fragments
    Ops R[3];                                                  // by step; the compiler shares out the registers
    v8i mid[4];
    typename MM::acc16_t acc[4][4];                            // [2 f + hh][token block]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0;

    // LDS read r of the operands of step S, in the order of their first use; area: of the pair's weights, tok: its token slot
    auto read = [&](auto step_c, auto r_c, uint32_t area, uint32_t tok) __attribute__((always_inline)) {
        constexpr int S = decltype(step_c)::value, r = decltype(r_c)::value;
        if constexpr (r < 2) R[S].ix[r] = *reinterpret_cast<const v2i*>(smem + area * FN_IDX + (S == 2 ? vi_mid : vi_raw + S * 3072) + r * 256);
        else {
            constexpr int a = r == 2 ? 0 : r < 7 ? -1 : r < 10 ? r - 6 : -1;
            if constexpr (a >= 0) R[S].a[a] = *reinterpret_cast<const v4i*>(smem + area * FN_VALS + (S == 2 ? va_mid : va_raw + S * 12288) + (a >> 1) * 1024 + (a & 1) * 256);
            else if constexpr (S < 2) {
                constexpr int k = r < 7 ? r - 3 : r - 6, b = k >> 1, h = k & 1;
                const v4i v = *reinterpret_cast<const v4i*>(smem + ((vb + tok) ^ (h * 16)) + b * 2048);
#pragma unroll
                for (int e = 0; e < 4; ++e) R[S].raw[b][4 * h + e] = v[e];
            }
        }
    };

    // Step S of pair p, whose weights lie in `area`, by the pairs that follow: of the next but one the weights and u0's tokens are
    // requested, of the next u1's tokens; the last step reads no operands (the token slots are the epilogue's by then).
    enum { MIDDLE, LAST2, LAST1 };
    auto step = [&](auto step_c, auto pos_c, int p, uint32_t area) __attribute__((always_inline)) {
        constexpr int S = decltype(step_c)::value, MEET = 3, POS = decltype(pos_c)::value;
        constexpr bool SHORT = ODD && POS == LAST1;
        constexpr int NS = S == 2 ? 0 : SHORT ? 2 : S + 1;
        __builtin_amdgcn_sched_barrier(0);
        unroll<16>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            constexpr int a = (i >> 1) & 3, b = 2 * (i >> 3) + (i & 1);
            if constexpr (SHORT && S == 0 && i < 4) {
#pragma unroll
                for (int j = 4; j < 8; ++j) asm("v_mov_b32 %0, 0" : "=v"(mid[i][j]));      // opaque: see gemm_fused.hip
            }
            if constexpr (S == 2) acc[a][b] = MM::sparse16(R[2].a[a], mid[b], acc[a][b], R[2].ix[a & 1][a >> 1]);
            else acc[a][b] = MM::sparse16(R[S].a[a], R[S].raw[b], acc[a][b], R[S].ix[a & 1][a >> 1]);
            __builtin_amdgcn_sched_barrier(0);
            // middle windows of the lane's four blocks: 8-bit types: bytes 2..5 of a block, 16-bit: elements 2..5
            if constexpr (S < 2) {
                constexpr int mb = i >> 2, j = i & 3;
                if constexpr (ES == 1) mid[mb][4 * S + j] = (int)__builtin_amdgcn_alignbyte((uint32_t)R[S].raw[mb][2 * j + 1], (uint32_t)R[S].raw[mb][2 * j], 2);
                else asm("v_mov_b32 %0, %1" : "=v"(mid[mb][4 * S + j]) : "v"(R[S].raw[mb][4 * (j >> 1) + 1 + (j & 1)]));      // opaque: see gemm_fused.hip
            }
            if constexpr (i == MEET) {
                if constexpr (POS == LAST1 ? S == 0 : POS == LAST2 && S == 2) wait_vmcnt<0>();
                else if constexpr (POS != LAST1 && S != 1) wait_vmcnt<8>();
                wait_lgkm0();
                wg_barrier();
            }
            // the half of a step that carries most of the reads has priority over the other wavefront's half (1 % at 14336 -> 4096 fp8, M = 2048)
            if constexpr (i == 0) __builtin_amdgcn_s_setprio(0);
            if constexpr (i == 8) __builtin_amdgcn_s_setprio(1);
            // requests, four a step: u1 tokens of the next pair; values and the next but one's u0 tokens; rest of those
            if constexpr (i == 5 || i == 8 || i == 11 || i == 14) {
                constexpr int d = (i - 5) / 3;
                if constexpr (S == 0 && POS != LAST1) load_tokens(std::integral_constant<int, d>{}, 2 * p + 3, t0);
                else if constexpr (POS == MIDDLE) {
                    if constexpr (S == 1 && d < 2) load_values(std::integral_constant<int, d>{}, p + 2, area);
                    else if constexpr (S == 1) load_tokens(std::integral_constant<int, d - 2>{}, 2 * p + 4, t1);
                    else if constexpr (d < 2) load_tokens(std::integral_constant<int, d + 2>{}, 2 * p + 4, t1);
                    else if constexpr (d == 2) load_values(c2, p + 2, area);
                    else load_index(p + 2, area);
                }
            }
            if constexpr (i > MEET && !(POS == LAST1 && S == 2)) {       // fourteen reads behind twelve instructions
                constexpr std::integral_constant<int, NS> ns{};
                const uint32_t next_area = S == 2 ? area ^ 1 : area, next_tok = S == 0 ? t1 : tz;
                constexpr int k = i - MEET - 1;
                if constexpr (NS == 2) {
                    if constexpr (k < 3) read(ns, std::integral_constant<int, k>{}, next_area, next_tok);
                    else if constexpr (k < 6) read(ns, std::integral_constant<int, k + 4>{}, next_area, next_tok);
                } else {
                    constexpr int first = k + (k < 2 ? k : 2);
                    read(ns, std::integral_constant<int, first>{}, next_area, next_tok);
                    if constexpr (k < 2) read(ns, std::integral_constant<int, first + 1>{}, next_area, next_tok);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    unroll<14>([&](auto r_c) __attribute__((always_inline)) { read(c0, r_c, 0, t0); });
    auto pair = [&](auto pos_c, int p) __attribute__((always_inline)) {
        const uint32_t area = p & 1;
        step(c0, pos_c, p, area);
        if constexpr (!(ODD && decltype(pos_c)::value == LAST1)) step(c1, pos_c, p, area);
        step(c2, pos_c, p, area);
        const uint32_t was0 = t0, was1 = t1;
        t0 = tz; t1 = was0; tz = was1;
    };
    for (int p = 0; p + 2 < P; ++p) pair(std::integral_constant<int, MIDDLE>{}, p);
    if (P > 1) pair(std::integral_constant<int, LAST2>{}, P - 2);
    pair(std::integral_constant<int, LAST1>{}, P - 1);

    // Epilogue: Y = bf16((float(acc) * s_x) * s_w), the whole tile staged in the token slots (the last operand reads, of step 2's
    // weights, returned before the last meeting; all requests had landed at the first meeting of the last pair): rows of 256 bytes, chunk c of row r at c ^ (r & 15).
    uint8_t* const stage = smem + FN_B_OFF;
    const int q = g;
    float4 sw[4];
    if constexpr (MM::SCALED) {
#pragma unroll
        for (int a = 0; a < 4; ++a) sw[a] = *reinterpret_cast<const float4*>(smem + FN_SW_OFF + 4 * (64 * (q & 1) + 32 * wo + 8 * a + 4 * (q >> 1)));
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int r = wt * 64 + 16 * b + n;
        const float sx = MM::SCALED ? reinterpret_cast<const float*>(smem + FN_SX_OFF)[r] : 1.0f;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const auto& v = acc[a][b];
            uint2 w;
            if constexpr (MM::SCALED)
                w = make_uint2(pack_bf16x2(((float)v[0] * sx) * sw[a].x, ((float)v[1] * sx) * sw[a].y), pack_bf16x2(((float)v[2] * sx) * sw[a].z, ((float)v[3] * sx) * sw[a].w));
            else w = make_uint2(pack_bf16x2((float)v[0], (float)v[1]), pack_bf16x2((float)v[2], (float)v[3]));
            *reinterpret_cast<uint2*>(stage + r * EP_ROWB + (((8 * (q & 1) + 4 * wo + a) ^ n) << 4) + 8 * (q >> 1)) = w;
        }
    }
    wait_lgkm0();
    wg_barrier();
    const int oc = 8 * n;
    const int64_t cols = O - o_blk;
    const bool vec = (ldy & 7) == 0 && ((uintptr_t)Y & 15) == 0 && oc + 8 <= cols;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = wave * 32 + 4 * i + q;
        const uint4 v = *reinterpret_cast<const uint4*>(stage + r * EP_ROWB + ((n ^ (r & 15)) << 4));
        if (t_blk + r < M) {
            uint16_t* dst = Y + (t_blk + r) * ldy + o_blk + oc;
            if (vec) {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(dst));
            } else {
                const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (oc + e < cols) dst[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

template <int DT, bool ODD>
static ss_status launch_narrow(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U,
                               int64_t ldxb, void* Y, int64_t ldy, hipStream_t stream)
{
    const int panels = (int)((O + PANEL - 1) / PANEL), tiles_t = (int)((M + BT - 1) / BT);
    if (allow_dynamic_lds<k_sparse_fused_narrow<DT, ODD>>(FN_LDS) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_sparse_fused_narrow<DT, ODD>), dim3(panels * tiles_t), dim3(512), FN_LDS, stream, static_cast<const uint8_t*>(Xq), s_x,
                       static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U, ldxb, static_cast<uint16_t*>(Y), ldy,
                       panels, tiles_t);
    return launch_status();
}

ss_status launch_sparse_fused_narrow(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                                     int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream)
{
#define SS_N(DT) (U & 1 ? launch_narrow<DT, true> : launch_narrow<DT, false>)(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream)
    switch (dtype) {
    case SS_I8: return SS_N(SS_I8);
    case SS_FP8_E4M3: return SS_N(SS_FP8_E4M3);
    case SS_BF16: return SS_N(SS_BF16);
    case SS_FP16: return SS_N(SS_FP16);
    }
#undef SS_N
    return SS_ERR_DTYPE;
}

}  // namespace ss
