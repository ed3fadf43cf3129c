// slide_sparse_gemm over lifted rows on tiles of 256 channels x 256 tokens: Y = X' . W'^T, W' packed 2:4.
//
// Tile engine, instructions, staggered operand reads and loads that run on across tiles as in gemm_fused.hip (what bounds
// it and why are told there); without the lifting a unit of 128 lifted bytes of a token row is one matrix-instruction
// step.  Token lane (n, g) of 16 x 4 takes bytes [32 g, 32 g + 32) of the unit; weight lane (r, g) takes, for rows 16 hh + r of
// a fragment, the 16 bytes of lane 16 hh + r + 32 (g >> 1) of packed step g & 1 of the unit (the packed order of the 32x32
// instruction serves the 16x16 one as it is, packed_layout.h).
//
// Ring of three units (32 KB of tokens, 20 KB of packed weights each).  In step u the workgroup meets behind the fifteenth
// matrix instruction: the operands of unit u are in registers then, its slot goes to the requests of unit u + 3, and unit u +
// 1 has landed.  The last three steps of a tile request the next tile's first three units, all but the tokens of the
// third: the epilogue stages in that unit's token slot, each wavefront where its own direct loads go, so that no meeting is
// needed, and the next tile's first step requests them.
//
// Against the 32x32 instructions with the ring drained and refilled between tiles: M = 8192, 6144 -> 4096 INT8 4:6 (two rounds) 139 ->
// 134 us, fp8 6:8 4096 -> 28672 at M = 2048 203 -> 193, 14336 -> 4096 INT8 at M = 4096 170 -> 164, short rows 0.84 .. 0.95 of the
// time (512 -> 8192 8:10 INT8 63 -> 53), rows of one unit level (34.5 us both at 128 -> 16384, M = 4096).
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "lds_pipe.h"
#include "tile_common.h"
#include "device_info.h"
#include <type_traits>

namespace ss {

constexpr int L_APANEL = 5 * 1024;                    // one packed step of a panel: values [fragment 4][lane 64][16 B], then index words [lane 64][fragment 4][4 B]
constexpr int L_AIDX = 4 * 1024;
constexpr int L_ASTEP = 2 * L_APANEL;
constexpr int L_ASLOT = 2 * L_ASTEP;
constexpr int L_BSLOT = BT * ROWB;
constexpr int L_B_OFF = 3 * L_ASLOT;                  // 60 KB
constexpr int L_SW_OFF = L_B_OFF + 3 * L_BSLOT;       // 156 KB: the tile's channel scales, then its token scales
constexpr int L_SX_OFF = L_SW_OFF + BO * 4;
constexpr int L_LDS = L_SX_OFF + BT * 4;              // 158 KB
static_assert(L_LDS <= 160 * 1024, "LDS budget");

// Chunk c of row r of the token tile is stored at chunk turn(c) ^ swz(r): keeps the chunks of two neighbouring lane groups, 2
// apart, on different banks in an LDS read (its own inverse)
__device__ inline int turn(int chunk) { return chunk ^ ((chunk & 2) << 1); }

// SHORT: rows of fewer units than the four that the steps of a tile need at least; the missing ones are zeros in all operands.
template <int DT, bool SHORT>
__global__ __launch_bounds__(512) void k_sparse(const uint8_t* __restrict__ XL, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int units,
                                                uint16_t* __restrict__ Y, int64_t ldy, int tiles_o, int tiles_t)
{
    typedef Mma<DT> MM;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wo = wave & 1, wt = wave >> 1;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t lds0 = lds_address(smem), lane16 = lane * 16;
    const int64_t npanels = (O + PANEL - 1) / PANEL;
    const int U = SHORT ? 4 : units;

    // Direct loads of this wavefront and unit: four times eight token rows, a 1 KB piece of values of each packed step
    // (panel wave >> 2, fragment wave & 3), 512 bytes of index words (step wave >> 2, panel (wave >> 1) & 1, half wave & 1)
    const int mj = wave >> 2;
    const uint32_t a_wave = lds0 + (wave >> 2) * L_APANEL + (wave & 3) * 1024;
    const uint32_t m_wave = lds0 + mj * L_ASTEP + ((wave >> 1) & 1) * L_APANEL + L_AIDX + (wave & 1) * 512, b_wave = lds0 + L_B_OFF + wave * 1024;
    const uint32_t va = (g & 1) * L_ASTEP + wo * L_APANEL + (n + 32 * (g >> 1)) * 16;
    const uint32_t vb = L_B_OFF + (wt * 64 + n) * ROWB + 16 * (turn(2 * g) ^ swz(n));      // token blocks lie 2048 bytes apart, same swizzle; the lane's second chunk at ^ 16

    const uint8_t *b_src = nullptr, *av_src = nullptr, *am_src = nullptr;
    uint32_t boff[4];
    const int64_t row_bytes = (int64_t)units * ROWB;
    auto setup_tile = [&](int to, int tt) {
        const int64_t t_blk = (int64_t)tt * BT, left = M - t_blk;        // >= 1
        const int ln = fresh_lane(), last = left > 255 ? 255 : (int)left - 1;
        b_src = XL + t_blk * row_bytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * (i * 8 + wave) + (ln >> 3);
            boff[i] = (uint32_t)(row < last ? row : last) * (uint32_t)row_bytes + turn((ln & 7) ^ swz(row)) * 16;
        }
        int64_t pv = (int64_t)to * 2 + (wave >> 2), pm = (int64_t)to * 2 + ((wave >> 1) & 1);
        pv = pv < npanels ? pv : npanels - 1;         // a panel beyond the last only feeds channels that are never stored
        pm = pm < npanels ? pm : npanels - 1;
        av_src = w_vals + pv * units * 8192 + (wave & 3) * 1024;
        am_src = w_meta + pm * units * 2048 + mj * 1024 + (wave & 1) * 512;
    };
    // Load number d of unit u into slot (at, bt): 0 .. 3 tokens, 4, 5 values, 6 index words
    auto load = [&](auto d_c, int u, uint32_t at, uint32_t bt, uint64_t lanes, auto masked_c) __attribute__((always_inline)) {
        constexpr int D = decltype(d_c)::value;
        constexpr bool MASKED = decltype(masked_c)::value;
        const bool none = SHORT && u >= units;
        const uint8_t* const src = none ? reinterpret_cast<const uint8_t*>(no_values) : D < 4 ? b_src : D < 6 ? av_src : am_src;
        const uint32_t off = none ? 0u : D < 4 ? (uint32_t)u * ROWB : D < 6 ? (uint32_t)u * 8192u + (D - 4) * 4096 : (uint32_t)u * 2048u;
        if constexpr (D < 4) {
            const uint32_t lane_off = none ? lane16 : boff[D];
            if constexpr (MASKED) lds_dma16_lanes_from<D * 8192>(src, off, lane_off, __builtin_amdgcn_readfirstlane(b_wave + bt), lanes);
            else lds_dma16_from<D * 8192>(src, off, lane_off, b_wave + bt);
        } else if constexpr (D < 6) {
            if constexpr (MASKED) lds_dma16_lanes_from<(D - 4) * L_ASTEP>(src, off, lane16, __builtin_amdgcn_readfirstlane(a_wave + at), lanes);
            else lds_dma16_from<(D - 4) * L_ASTEP>(src, off, lane16, a_wave + at);
        } else lds_dma16_lanes_from<0>(src, off, lane16, __builtin_amdgcn_readfirstlane(m_wave + at), lanes & 0xffffffffull);
    };
    constexpr std::false_type all_lanes{};
    uint32_t a0 = 0, a1 = L_ASLOT, a2 = 2 * L_ASLOT, b0 = 0, b1 = L_BSLOT, b2 = 2 * L_BSLOT;      // slots of units u, u + 1, u + 2
    auto rotate = [&]() {
        const uint32_t a = a0, b = b0;
        a0 = a1; a1 = a2; a2 = a;
        b0 = b1; b1 = b2; b2 = b;
    };
    int to, tt;
    bool have = tile_of_round(0, tiles_o, tiles_t, to, tt);
    if (!have) return;
    setup_tile(to, tt);
    unroll<7>([&](auto d_c) __attribute__((always_inline)) { load(d_c, 0, a0, b0, ~0ull, all_lanes); });
    unroll<7>([&](auto d_c) __attribute__((always_inline)) { load(d_c, 1, a1, b1, ~0ull, all_lanes); });
    unroll<3>([&](auto d_c) __attribute__((always_inline)) { load(std::integral_constant<int, decltype(d_c)::value + 4>{}, 2, a2, b2, ~0ull, all_lanes); });
    wait_vmcnt<10>();                                 // unit 0
    wg_barrier();

    struct Regs { v4i a[8], ix[2]; v8i raw[4]; };
    enum { FIRST, MIDDLE, LAST3, LAST2, LAST1 };      // position of a step in its tile
    for (int round = 0; have; ++round) {
        const int64_t o_blk = (int64_t)to * BO, t_blk = (int64_t)tt * BT;
        have = tile_of_round(round + 1, tiles_o, tiles_t, to, tt);       // the next tile
        typename MM::acc16_t acc[4][2][4];            // [fragment][rows 16 hh][token block]
        Regs R;
        auto rd = [&](uint32_t off) __attribute__((always_inline)) -> v4i { return *reinterpret_cast<const v4i*>(smem + off); };
        auto read_raw = [&](int b, int h, uint32_t at) __attribute__((always_inline)) {
            const v4i v = rd((h ? at ^ 16 : at) + b * 2048);
#pragma unroll
            for (int e = 0; e < 4; ++e) R.raw[b][4 * h + e] = v[e];
        };
        auto read_a = [&](uint32_t at, int a) __attribute__((always_inline)) { R.a[a] = rd(at + (a & 3) * 1024 + (a >> 2) * 256); };
        auto read_ix = [&](uint32_t at, int hh) __attribute__((always_inline)) { R.ix[hh] = rd(at + L_AIDX + hh * 256); };
        const uint32_t more = __builtin_amdgcn_readfirstlane(have ? ~0u : 0u);      // the last steps request for the next tile, if there is one

        // Step of unit u.  Instruction i: token blocks in two halves of 16 instructions, weight fragments 0 .. 7 within each, so
        // that everything has fourteen or more instructions between its last use and its next.  Requests, spread evenly: the
        // tokens and the first values of unit u + 3 behind the meeting, the rest of unit u + 2 ahead of it.
        auto step = [&](auto pos_c, int u) __attribute__((always_inline)) {
            constexpr int POS = decltype(pos_c)::value;
            constexpr bool LAST = POS >= LAST3;
            uint64_t lanes = 0;
            if constexpr (LAST) {                        // opaque, so that the mask is made in scalar registers here and not carried in vector registers
                uint32_t half = more;
                asm volatile("" : "+v"(half));
                half = __builtin_amdgcn_readfirstlane(half);
                lanes = ((uint64_t)half << 32) | half;
            }
            const uint32_t va0 = va + a0, va1 = va + a1, vb0 = vb + b0, vb1 = vb + b1;
            __builtin_amdgcn_sched_barrier(0);
            unroll<32>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int i = decltype(i_c)::value;
                constexpr int a = (i >> 1) & 7, b = 2 * (i >> 4) + (i & 1);
                acc[a & 3][a >> 2][b] = MM::sparse16(R.a[a], R.raw[b], acc[a & 3][a >> 2][b], R.ix[a >> 2][a & 3]);
                __builtin_amdgcn_sched_barrier(0);
                if (i == 0) read_ix(va0, 1);                                // the words of the second four fragments were in use until now
                if (i < 4) read_raw(2 + (i >> 1), i & 1, vb0);              // and so were blocks 2 and 3
                if (i == 1) __builtin_amdgcn_s_setprio(0);
                if (i == 16) __builtin_amdgcn_s_setprio(1);
                // ahead of the meeting
                if constexpr (POS == FIRST) {
                    if constexpr (i == 4 || i == 6 || i == 9 || i == 11) load(std::integral_constant<int, (i == 4 ? 0 : i == 6 ? 1 : i == 9 ? 2 : 3)>{}, 2, a2, b2, ~0ull, all_lanes);
                } else if constexpr (i == 4 || i == 9) {
                    constexpr std::integral_constant<int, (i == 4 ? 5 : 6)> d{};
                    if constexpr (POS == LAST2 || POS == LAST1) load(d, POS == LAST2 ? 0 : 1, a2, b2, lanes, std::true_type{});
                    else load(d, u + 2, a2, b2, ~0ull, all_lanes);
                }
                if (POS == LAST3 && i == 11) setup_tile(to, tt);            // the next tile's, or this one's again
                if (i == 14) {
                    if constexpr (POS == FIRST) wait_vm_mode<7>(__builtin_amdgcn_readfirstlane(1 - min(round, 1)));              // unit 1: a later tile's has landed before the epilogue's stores
                    else if constexpr (POS == LAST2) wait_vm_mode<(MM::SCALED ? 8 : 7)>(__builtin_amdgcn_readfirstlane(2 - (int)(more & 1)));
                    else if constexpr (POS == LAST1) wait_vm_mode<7>(__builtin_amdgcn_readfirstlane((int)(more & 1)));
                    else wait_vm_mode<7>(1);
                    wait_lgkm0();
                    wg_barrier();
                    if constexpr (POS == LAST3 && MM::SCALED) load_tile_scales(s_w, s_x, O, M, o_blk, t_blk, wave, lds0 + L_SW_OFF);
                }
                if constexpr (POS == LAST1) {
                    if constexpr (i == 15 || i == 21 || i == 27) load(std::integral_constant<int, 4 + (i - 15) / 6>{}, 2, a0, b0, lanes, std::true_type{});
                } else if constexpr (i >= 15 && (i - 15) % 4 == 0) {
                    constexpr std::integral_constant<int, (i - 15) / 4> d{};
                    if constexpr (LAST) load(d, POS == LAST3 ? 0 : 1, a0, b0, lanes, std::true_type{});
                    else load(d, u + 3, a0, b0, ~0ull, all_lanes);
                }
                if constexpr (POS != LAST1) {
                    if (i >= 17 && (i & 1)) read_a(va1, (i - 17) >> 1);
                    if (i == 24) read_ix(va1, 0);
                    if (i >= 16 && !(i & 1) && i < 24) read_raw((i - 16) >> 2, (i >> 1) & 1, vb1);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            rotate();
        };

        // operands of unit 0: published by the last meeting of the previous tile (or the prologue)
        read_ix(va + a0, 0);
#pragma unroll
        for (int a = 0; a < 8; ++a) read_a(va + a0, a);
#pragma unroll
        for (int r = 0; r < 4; ++r) read_raw(r >> 1, r & 1, vb + b0);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[f][hh][b][r] = 0;
        step(std::integral_constant<int, FIRST>{}, 0);
        for (int u = 1; u + 3 < U; ++u) step(std::integral_constant<int, MIDDLE>{}, u);
        step(std::integral_constant<int, LAST3>{}, U - 3);
        step(std::integral_constant<int, LAST2>{}, U - 2);
        step(std::integral_constant<int, LAST1>{}, U - 1);
        const int64_t o_sub = o_blk + wo * 128, t_sub = t_blk + wt * 64;
        const int64_t rows = M - t_sub, cols = O - o_sub;          // <= 0: nothing of this sub-tile exists
        const bool any = rows > 0 && cols > 0;
        const int rows_left = any ? (int)(rows > 64 ? 64 : rows) : 0, cols_left = any ? (int)(cols > 128 ? 128 : cols) : 0;
        store_tile16<MM::SCALED, true>(acc, reinterpret_cast<const float*>(smem + L_SX_OFF) + wt * 64, reinterpret_cast<const float*>(smem + L_SW_OFF) + wo * 128,
                                       any ? Y + t_sub * ldy + o_sub : Y, (uint32_t)ldy, rows_left, cols_left, smem + L_B_OFF + b2 + wave * 1024);
    }
}

template <int DT, bool SHORT>
static ss_status launch_sparse(const void* XL, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                               int units, void* Y, int64_t ldy, hipStream_t stream)
{
    const int tiles_o = (int)((O + BO - 1) / BO), tiles_t = (int)((M + BT - 1) / BT);
    const int cus = cu_count(), ntiles = tiles_o * tiles_t, grid = ntiles < cus ? ntiles : cus;
    if (grid <= 0) return SS_ERR_HIP;
    if (allow_dynamic_lds<k_sparse<DT, SHORT>>(L_LDS) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_sparse<DT, SHORT>), dim3(grid), dim3(512), L_LDS, stream, static_cast<const uint8_t*>(XL), s_x, static_cast<const uint8_t*>(w_vals),
                       static_cast<const uint8_t*>(w_meta), s_w, M, O, units, static_cast<uint16_t*>(Y), ldy, tiles_o, tiles_t);
    return launch_status();
}

ss_status launch_sparse_tile(const void* XL, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int64_t Kpb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t hs)
{
    const int units = (int)(Kpb / ROWB);
#define SS_L(DT) (units < 4 ? launch_sparse<DT, true>(XL, s_x, w_vals, w_meta, s_w, M, O, units, Y, ldy, hs) : launch_sparse<DT, false>(XL, s_x, w_vals, w_meta, s_w, M, O, units, Y, ldy, hs))
    switch (dtype) {
    case SS_I8: return SS_L(SS_I8);
    case SS_FP8_E4M3: return SS_L(SS_FP8_E4M3);
    case SS_BF16: return SS_L(SS_BF16);
    case SS_FP16: return SS_L(SS_FP16);
    }
#undef SS_L
    return SS_ERR_DTYPE;
}

}  // namespace ss
