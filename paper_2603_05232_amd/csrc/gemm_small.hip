// Sparse GEMMs on small unsplit tiles: 32 or 64 channels (one or two fragments of a panel) x 32 to 128 tokens, for layers that have too few tiles of
// 128 channels to occupy the compute units and would split their rows.
//
// A split row costs its partial sums twice (6 MB at M = 64 leave the L2s in about 2.4 us between the two kernels, 14 MB at M = 256 in 3.2) and a second
// launch, 4 to 8 us of a call together.  Small tiles read more: what a compute unit loads grows from 8 to 28 super-units of fewer lines each (3584 ->
// 3584 INT8 at M = 256 2300 -> 3500 lines), at 200 to 270 lines a microsecond and compute unit with weights from HBM (counted, with the launch), 340 to 390
// hot.  So they win until rows are long, the more the more tokens there are to sum up (small_pays, mma_types.h).
// Within a workgroup the row is still split: KG groups of wavefronts, each with a KG-th of the row and a ring of its own, whose sums meet in LDS in the
// order of the groups.  The loop is plain: wait for a unit, request a later one, read the operands, multiply.  Wavefronts that meet at every unit do all of
// that in step and nothing overlaps, so where the ring allows it a group is one wavefront, which needs no meeting (32 and 64 tokens; against groups of a
// wavefront for each 32 tokens 0.97 .. 1.03 from HBM, 0.85 .. 0.95 hot); with 96 and 128 tokens two wavefronts or three.
// us, weights from HBM / hot, split and now: INT8 3584 -> 4608 at M = 256 19.4 / 17.2 -> 13.0 / 12.0, 3584 -> 3584 at M = 256 16.8 / 15.4 -> 11.4 / 9.0, at
// M = 64 13.5 / 11.9 -> 7.7 / 5.2, at M = 32 9.4 / 7.9 -> 7.8 / 5.1; fp8 lifted 4096 -> 4096 at M = 64 11.7 / 10.5 -> 9.4 / 6.3.
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "lds_pipe.h"
#include "mid_order.h"
#include "device_info.h"

namespace ss {

// A workgroup has FW matrix-instruction fragments of 32 channels and TB blocks of 32 tokens, in KG groups of TB / TW wavefronts (TW blocks each).
// Fragment j of a panel is rows 8 j .. 8 j + 7 of its four packed fragments: lines of values are whole, and so are those of index words, of which a
// packed fragment by itself would use a quarter (62 lines a super-unit instead of 80 with 32 channels and tokens: 0.97 .. 1.02 of the time from HBM,
// 0.93 .. 0.99 hot).
// A unit of 128 bytes of a token row in LDS: token rows (swizzled), values [step][fragment][lane][16 B], index words
// [fragment][step][half 2][row 8][packed fragment 4][4 B] in 1 KB
template <int FW, int TB, int TW, int KG, bool FUSED> struct SmallUnit {
    static constexpr int GW = TB / TW;                                    // wavefronts of a group
    static constexpr int NS = FUSED ? 3 : 2;
    static constexpr int TOK = TB * 32 * ROWB, AV = NS * FW * 1024, BYTES = TOK + AV + FW * 1024;
    static constexpr int PIECES = FW * (NS + 1);                          // of values, 1 KB, and of index words, NS * 256 bytes
    static constexpr int E = (PIECES + GW - 1) / GW, LPU = 4 * TW + E;    // direct loads per wavefront: its token rows, its share of those
    static constexpr int SCALES = (PANEL + (TB * 32 + 63) / 64 * 64) * 4;
    static constexpr int FIT = (160 * 1024 - SCALES) / (KG * BYTES), RING = FIT < 4 ? FIT : 4, LDS = KG * RING * BYTES + SCALES;
};

template <int DT, int FW, int TB, int TW, int KG, bool FUSED>
__global__ __launch_bounds__(64 * (TB / TW) * KG) void k_sparse_small(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                             const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int U_all,
                                                             int64_t ldxb, uint16_t* __restrict__ Y, int64_t ldy, MidOrder order)
{
    typedef Mma<DT> MM;
    typedef SmallUnit<FW, TB, TW, KG, FUSED> SU;
    constexpr int GW = SU::GW, NS = SU::NS, RING = SU::RING, E = SU::E, PARTS = FRAGS_PER_PANEL / FW;
    static_assert(KG > 1 && RING >= 2 && (RING - 2) * SU::LPU < 64, "loads in flight");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];      // RING units for each of the groups, the scales
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kg = wave_all / GW, t = wave_all % GW, lane = threadIdx.x & 63;
    const int n = lane & 31, qb = lane >> 5;
    asm volatile("" ::"s"(Xq), "s"(w_vals), "s"(w_meta), "s"(M), "s"(U_all), "s"(ldxb));      // with the order all that the first loads wait for, in one go
    const MidItem it = mid_item(order);                                  // its "panels" are parts of FW fragments
    const int64_t panel = it.panel / PARTS, t0 = (int64_t)it.tt * (TB * 32);
    const int j0 = FW * (it.panel % PARTS);
    const uint32_t lane16 = lane * 16, lds0 = lds_address(lds), ring0 = lds0 + kg * (RING * SU::BYTES);
    constexpr int SCALES = KG * RING * SU::BYTES;
    if (MM::SCALED) {                                                    // scales of the panel's channels and of the tokens
        if (wave_all < 2) lds_dma_scales(s_w, panel * PANEL + wave_all * 64, O, lane, lds0 + SCALES + wave_all * 256);
        if (wave_all < (TB + 1) / 2) lds_dma_scales(s_x, t0 + wave_all * 64, M, lane, lds0 + SCALES + 512 + wave_all * 256);
    }
    // this group's share of the units, not empty (KG <= U_all)
    const int both = U_all / KG, more = U_all % KG, u_first = kg * both + min(kg, more), U = both + (kg < more);
    const int rot = (int)(blockIdx.x & 7) * U >> 3;                      // as in gemm_mid.hip
    const uint8_t* const x_src = Xq + t0 * ldxb + (int64_t)u_first * ROWB;
    uint32_t off[4 * TW];
    {
        const int64_t left = M - t0;                                     // >= 1
        const int last = left > TB * 32 - 1 ? TB * 32 - 1 : (int)left - 1;
#pragma unroll
        for (int i = 0; i < 4 * TW; ++i) {
            const int row = (t * 4 * TW + i) * 8 + (lane >> 3);
            off[i] = (uint32_t)(row < last ? row : last) * (uint32_t)ldxb + (((lane & 7) ^ swz(row)) << 4);
        }
    }
    uint64_t e_lanes[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int a = t + e * GW;
        const uint64_t lanes = a < NS * FW ? ~0ull : a < SU::PIECES ? (1ull << (16 * NS)) - 1 : 0ull;
        e_lanes[e] = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(lanes >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)lanes);
    }
    // lane l brings row 8 j + (l & 7) of values: packed fragment (l >> 3) & 3, half l >> 5, which is where lane l of the matrix instruction reads them;
    // of index words: step l >> 4, half (l >> 3) & 1
    const uint32_t row16 = (8 * j0 + (lane & 7)) * 16, v_off = ((lane >> 3) & 3) * 1024 + (lane >> 5) * 512 + row16;
    const uint32_t i_off = (lane >> 4) * 1024 + ((lane >> 3) & 1) * 512 + row16;
    const uint8_t* const av_src = w_vals + (panel * U_all + u_first) * (NS * 4096);
    const uint8_t* const am_src = w_meta + (panel * U_all + u_first) * (NS * 1024);
    // piece a of a unit: fragment a % FW of step a / FW of the values, then the index words of fragment a % FW; beyond the last: nothing
    auto issue = [&](int v, uint32_t slot) __attribute__((always_inline)) {
        const int u = v + rot < U ? v + rot : v + rot - U;
#pragma unroll
        for (int i = 0; i < 4 * TW; ++i) lds_dma16_at(x_src + (int64_t)u * ROWB, off[i], ring0 + slot + (t * 4 * TW + i) * 1024);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int a = t + e * GW;
            const bool values = a < NS * FW;
            const uint8_t* const src = (values ? av_src + (int64_t)u * (NS * 4096) + (a / FW) * 4096 : am_src + (int64_t)u * (NS * 1024)) + (a % FW) * 128;
            if ((e + 1) * GW <= NS * FW) lds_dma16_at(src, v_off, ring0 + slot + SU::TOK + a * 1024);
            else lds_dma16_lanes_at(src, values ? v_off : i_off, ring0 + slot + SU::TOK + a * 1024, e_lanes[e]);
        }
    };
    uint32_t vb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int row = t * 32 * TW + n;                                 // the wavefront's next block lies 4096 bytes on, same swizzle
        vb[c] = row * ROWB + (((FUSED ? 4 * qb + c : 4 * (c >> 1) + 2 * qb + (c & 1)) ^ swz(row)) << 4);
    }
    const uint32_t vi = qb * 128 + (n & 7) * 16 + (n >> 3) * 4;
    const uint8_t* const smem = lds + kg * (RING * SU::BYTES);
    typename MM::acc_t acc[FW][TW];
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int b = 0; b < TW; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][b][r] = 0;
    uint32_t slot = 0, lslot = (RING - 1) * SU::BYTES;
    auto multiply = [&]() __attribute__((always_inline)) {
        const uint8_t* st = smem + slot;
        v4i a[NS][FW];
        int ix[NS][FW];
#pragma unroll
        for (int h = 0; h < NS; ++h)
#pragma unroll
            for (int f = 0; f < FW; ++f) {
                a[h][f] = *reinterpret_cast<const v4i*>(st + SU::TOK + (FW * h + f) * 1024 + lane16);
                ix[h][f] = *reinterpret_cast<const int*>(st + SU::TOK + SU::AV + f * 1024 + h * 256 + vi);
            }
#pragma unroll
        for (int b = 0; b < TW; ++b) {
            v4i x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = *reinterpret_cast<const v4i*>(st + vb[c] + b * (32 * ROWB));
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int f = 0; f < FW; ++f) {
                    const v4i lo = x[2 * h], hi = x[2 * h + 1];
                    acc[f][b] = MM::sparse(a[h][f], v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}, acc[f][b], ix[h][f]);
                }
            if constexpr (FUSED) {                                       // middle windows: see gemm_mid.hip
                v8i m;
#pragma unroll
                for (int jd = 0; jd < 8; ++jd) {
                    auto w = [&](int k) { return (uint32_t)x[k >> 2][k & 3]; };
                    if constexpr (MM::ES == 1) m[jd] = (int)__builtin_amdgcn_alignbyte(w(2 * jd + 1), w(2 * jd), 2);
                    else m[jd] = (int)w(4 * (jd >> 1) + 1 + (jd & 1));
                }
#pragma unroll
                for (int f = 0; f < FW; ++f) acc[f][b] = MM::sparse(a[2][f], m, acc[f][b], ix[2][f]);
            }
        }
        slot = slot == (RING - 1) * SU::BYTES ? 0u : slot + SU::BYTES;
    };
#pragma unroll
    for (int i = 0; i < RING - 1; ++i)
        if (i < U) issue(i, i * SU::BYTES);
    for (int u = 0; u < both; ++u) {
        if (u + RING - 1 <= U) wait_vmcnt<(RING - 2) * SU::LPU>(); else wait_vmcnt<0>();
        if constexpr (GW > 1) wg_barrier();                              // unit u has landed, unit u - 1 is read; a wavefront by itself needs no meeting
        if (u + RING - 1 < U) issue(u + RING - 1, lslot);
        multiply();
        lslot = lslot == (RING - 1) * SU::BYTES ? 0u : lslot + SU::BYTES;
    }
    if (more) {                                                          // the first groups have one more
        wait_vmcnt<0>();
        if constexpr (GW > 1) wg_barrier();
        if (kg < more) multiply();
    }
    wait_lgkm0();
    wg_barrier();                                                        // nobody reads operands any more
    typedef decltype(acc[0][0][0] + acc[0][0][0]) elem_t;
    typedef elem_t quad_t __attribute__((ext_vector_type(4)));
    // the groups' sums, added in their order by the first
    v4i* const x = reinterpret_cast<v4i*>(lds) + t * (FW * TW * 256) + lane;
    constexpr int GROUP = TB * FW * 256;
    if (kg > 0) {
#pragma unroll
        for (int f = 0; f < FW; ++f)
#pragma unroll
            for (int b = 0; b < TW; ++b)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const quad_t q = {acc[f][b][4 * r4], acc[f][b][4 * r4 + 1], acc[f][b][4 * r4 + 2], acc[f][b][4 * r4 + 3]};
                    x[(kg - 1) * GROUP + ((f * TW + b) * 4 + r4) * 64] = __builtin_bit_cast(v4i, q);
                }
        wait_lgkm0();
    }
    wg_barrier();
    if (kg > 0) return;
#pragma unroll
    for (int k = 0; k < KG - 1; ++k)
#pragma unroll
        for (int f = 0; f < FW; ++f)
#pragma unroll
            for (int b = 0; b < TW; ++b)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const quad_t q = __builtin_bit_cast(quad_t, x[k * GROUP + ((f * TW + b) * 4 + r4) * 64]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[f][b][4 * r4 + e] += q[e];
                }
    // accumulator register 4 q + e of fragment j: channel 64 qb + 16 q + 4 j + e of the panel
    const float* const sw = reinterpret_cast<const float*>(lds + SCALES);
#pragma unroll
    for (int b = 0; b < TW; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int in_tile = (t * TW + b) * 32 + n;
        const int64_t tok = t0 + in_tile;
        if (tok >= M) continue;
        const float sx = MM::SCALED ? sw[PANEL + in_tile] : 1.0f;
        const int c = 64 * qb + 16 * q + 4 * j0;
        const int64_t o = panel * PANEL + c;
        uint32_t w[FW][2];
#pragma unroll
        for (int f = 0; f < FW; ++f) {
            float v[4];
            const float4 s = MM::SCALED ? *reinterpret_cast<const float4*>(sw + c + 4 * f) : make_float4(1.0f, 1.0f, 1.0f, 1.0f);
            const float se[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = (float)acc[f][b][4 * q + e];
                if constexpr (MM::SCALED) v[e] = (v[e] * sx) * se[e];
            }
            w[f][0] = pack_bf16x2(v[0], v[1]);
            w[f][1] = pack_bf16x2(v[2], v[3]);
        }
        uint16_t* const dst = Y + tok * ldy + o;
        if (o + 4 * FW <= O) {
            if constexpr (FW == 2) *reinterpret_cast<piece16_t*>(dst) = piece16_t{w[0][0], w[0][1], w[FW - 1][0], w[FW - 1][1]};
            else *reinterpret_cast<piece8_t*>(dst) = piece8_t{w[0][0], w[0][1]};
        } else if (o < O) {                                             // (not for channels behind the last: 15000 channels, 3 units, M = 48, bf16, 6.2 -> 5.0 us)
#pragma unroll
            for (int e = 0; e < 4 * FW; ++e)
                if (o + e < O) dst[e] = (uint16_t)(w[e >> 2][(e >> 1) & 1] >> (16 * (e & 1)));
        }
    }
}

}  // namespace ss

using namespace ss;

template <int DT, int FW, int TB, int TW, int KG, bool FUSED>
static ss_status launch_small_one(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U, int64_t ldxb,
                                 void* Y, int64_t ldy, hipStream_t stream)
{
    typedef SmallUnit<FW, TB, TW, KG, FUSED> SU;
    const int tiles_t = (int)((M + TB * 32 - 1) / (TB * 32));
    const int64_t ntiles = (O + PANEL - 1) / PANEL * (FRAGS_PER_PANEL / FW) * tiles_t;
    static_assert(SU::LDS <= 160 * 1024 && (KG - 1) * TB * FW * 4096 <= KG * SU::RING * SU::BYTES, "the rings, then the sums that are handed over");
    if (allow_dynamic_lds<k_sparse_small<DT, FW, TB, TW, KG, FUSED>>(SU::LDS) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_sparse_small<DT, FW, TB, TW, KG, FUSED>), dim3((unsigned)ntiles), dim3(64 * SU::GW * KG), SU::LDS, stream, static_cast<const uint8_t*>(Xq), s_x,
                       static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U, ldxb, static_cast<uint16_t*>(Y), ldy,
                       mid_order(ntiles, tiles_t, 1, false, U));
    return launch_status();
}

namespace ss {

ss_status launch_sparse_small(bool fused, const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, small_tile tile, hipStream_t stream)
{
#define SS_SM(DT, FW, TB, TW, KG) \
    if (tile.fw == FW && tile.tb == TB && tile.kg == KG) \
        return fused ? launch_small_one<DT, FW, TB, TW, KG, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream) \
                     : launch_small_one<DT, FW, TB, TW, KG, false>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream)
#define SS_S(DT) SS_SM(DT, 1, 1, 1, 4); SS_SM(DT, 2, 1, 1, 4); SS_SM(DT, 2, 2, 2, 3); SS_SM(DT, 2, 3, 1, 2); SS_SM(DT, 2, 4, 2, 2); break
    switch (dtype) {
    case SS_I8: SS_S(SS_I8);
    case SS_FP8_E4M3: SS_S(SS_FP8_E4M3);
    case SS_BF16: SS_S(SS_BF16);
    case SS_FP16: SS_S(SS_FP16);
    }
#undef SS_S
#undef SS_SM
    return SS_ERR_DTYPE;
}

}  // namespace ss
