// slide_sparse_gemm_fused: the 2:4 sparse GEMM of the 6:8 pattern (N = 4) on UNLIFTED quantised activations.
// The lifting operator (Sec. 3.3; window j = g(N-1)+l of a row starts at b = 2N g + 2l, Alg. 1) is applied on the way
// from LDS to the operand registers, so the lifted matrix X' (1.5 K bytes per token) is never written, read or staged:
// token tiles move K bytes per token from L2 to LDS and from LDS to registers.
//
// What bounds it.  The power limit: matrix instructions alone, operands in registers, run at 64 % of the nominal sparse
// rate, LDS operand reads cost 7 % on top and the direct loads 13 %; a loop of exactly this traffic takes the same time
// with eight wavefronts as with four that read a third less (unrecorded probe).  So what counts is energy per operation
// and, between tiles, idle cycles.  The 16x16 sparse instructions (128 lifted bytes deep) do 6 to 7 % more operations a
// second under that limit than the 32x32 ones (64 deep) on the same data in all four types, for the same operand bytes.
//
// K loop.  A super-unit is 128 unlifted bytes of a token row (one cache line) = 16 blocks of 8 bytes = 48 windows.  Two
// of them, u0 and u1, make a pair = three matrix-instruction steps of 128 lifted bytes:
//   step 0, step 1: windows l = 0 and l = 2 of u0's, u1's blocks, which are the blocks' two halves: token lane (n, g)
//     of 16 x 4 takes the 32 raw bytes of four blocks, chunks 4 (g & 1) + 2 (g >> 1) and the next of the line;
//   step 2: the middle windows (l = 1) of the lane's four blocks of u0 and four of u1, each built with one v_alignbyte
//     (8-bit types) or two register copies (16-bit types) while steps 0 and 1 run.
// The packed weights (slide_decompose_fused: three 64-byte steps per super-unit in operand order of the 32x32
// instruction) serve the 16x16 one as they are: weight lane (r, g) takes, for rows 16 hh + r of a fragment, the 16 bytes
// of lane 16 hh + r + 32 (g >> 1) of packed step g & 1 of the super-unit in steps 0 and 1, and those of lane
// 16 hh + r + 32 (g & 1) of packed step 2 of super-unit u(g >> 1) in step 2 (measured: value half h of weight lane group g
// meets 16-byte half g >> 1 of token lane group 2 (g & 1) + h).  With an odd number of super-units the last pair has no step
// 1, and zeros in u1's place in step 2 (time over that with a whole pair, u1 all zeros: 1 to 5 super-units 0.95 .. 0.97, 7 to 13 0.96 .. 0.98, 21
// to 57 0.98 .. 0.99; against the 32x32 kernel before it 3 and 5 super-units in a single round of tiles are 1.00 .. 1.05, more of either 0.90 .. 1.02).
//
// Tile engine.  Persistent workgroups, 256 channels x 256 tokens per tile, eight wavefronts (two per SIMD) of 128
// channels x 64 tokens = 8 x 4 accumulator blocks.  Operands go L2 -> LDS with direct loads into two rings: token tiles
// (32 KB per super-unit, three slots) and packed weights (10 KB per packed step: 8 KB of stored values + 2 KB of index
// words; six slots, so that the six packed steps of a pair always lie in the same ones).
//
// Pipeline.  Registers hold one step's operands; a weight fragment is refilled for the next step behind its last use,
// token fragments in two halves.  The workgroup meets once per step, behind its fifteenth matrix instruction: by then the
// reads of this step's operands have returned, so their ring slots go back to the loaders; what the reads after the
// meeting need was requested two steps before.  The requests run on across tiles: the last pair of a tile requests the
// next tile's first pair, and between two tiles there is only the epilogue, without a meeting (wavefronts may be in
// different tiles until the next one).  The epilogue stages in the token slot that is free then; it waits for the wavefront's
// own requests before its first store, because the wait counter counts stores too, and the first two meetings of a tile
// behind another then wait for no load at all.  A workgroup's first tile starts when the operands of step 0 have landed (time over waiting for
// the whole pair: rows of 2 to 8 super-units 0.93 .. 0.99, 28 and 32 0.95 .. 1.00).
//
// Token tile in LDS: 256 rows x 128 bytes, the 16-byte chunk c of row r stored at chunk place(c) ^ ((r >> 1) & 7) (the
// permutation is applied on the global-address side: a direct load writes 64 lanes x 16 bytes contiguously, i.e. eight
// whole rows, and the eight lanes of a row fetch its cache line in permuted order).  A 16-byte LDS read is served in
// phases of sixteen lanes that take eight of one lane group and eight of its neighbour (rows 0 .. 3, 12 .. 15 of the one with 4
// .. 11 of the other); place() keeps the two groups' chunks, 4 apart, on different banks.
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "lds_pipe.h"
#include "tile_common.h"
#include "device_info.h"
#include <type_traits>

namespace ss {

constexpr int F_APANEL = 5 * 1024;                    // one packed step of a panel: values [fragment 4][lane 64][16 B], then index words [lane 64][fragment 4][4 B]
constexpr int F_AIDX = 4 * 1024;
constexpr int F_ASTEP = 2 * F_APANEL;
constexpr int F_ARING = 6;
constexpr int F_BSLOT = 32 * 1024;
constexpr int F_BRING = 3;
constexpr int F_B_OFF = F_ARING * F_ASTEP;            // 60 KB
constexpr int F_SW_OFF = F_B_OFF + F_BRING * F_BSLOT; // 156 KB: the tile's channel scales, then its token scales
constexpr int F_SX_OFF = F_SW_OFF + BO * 4;
constexpr int F_LDS = F_SX_OFF + BT * 4;              // 158 KB
static_assert(F_LDS <= 160 * 1024, "LDS budget");

// ODD: an odd number of super-units
template <int DT, bool ODD>
__global__ __launch_bounds__(512) void k_sparse_fused(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                      const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int U,
                                                      int64_t ldxb, uint16_t* __restrict__ Y, int64_t ldy, int tiles_o, int tiles_t)
{
    typedef Mma<DT> MM;
    constexpr int ES = MM::ES;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wo = wave & 1, wt = wave >> 1;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t lds0 = lds_address(smem);
    const int nsteps = 3 * U, pairs = (U + 1) >> 1;
    const int64_t npanels = (O + PANEL - 1) / PANEL;
    const uint32_t lane16 = lane * 16;

    // Direct loads of this wavefront: of every packed step one 1 KB piece of values (panel wave >> 2, fragment wave & 3);
    // of every two packed steps 512 bytes of index words (step wave >> 2 of the two, panel (wave >> 1) & 1, half wave & 1;
    // lanes 0 .. 31); of every token tile four times eight rows.
    const uint32_t a_wave = lds0 + (wave >> 2) * F_APANEL + (wave & 3) * 1024, m_wave = lds0 + ((wave >> 1) & 1) * F_APANEL + F_AIDX + (wave & 1) * 512;
    const int mj = wave >> 2;
    const uint32_t b_wave = lds0 + F_B_OFF + wave * 1024;

    // LDS byte offsets of this lane's operand reads (ring slot, fragment, rows 16 hh and token block are added as they come)
    const uint32_t va_raw = (g & 1) * F_ASTEP + wo * F_APANEL + (n + 32 * (g >> 1)) * 16;
    const uint32_t va_mid = (2 + 3 * (g >> 1)) * F_ASTEP + wo * F_APANEL + (n + 32 * (g & 1)) * 16;
    const uint32_t vb = F_B_OFF + (wt * 64 + n) * ROWB + 16 * (place(4 * (g & 1) + 2 * (g >> 1)) ^ swz(n));      // token blocks lie 16 rows = 2048 bytes apart, same swizzle; the lane's second chunk at ^ 16

    // Sources of a tile's loads.  The loaders run one pair ahead of the matrix instructions.
    const uint8_t *b_src = nullptr, *av_src = nullptr, *am_src = nullptr;
    uint32_t boff[4];
    auto setup_tile = [&](int to, int tt) {
        const int64_t t_blk = (int64_t)tt * BT;
        const int ln = fresh_lane();
        b_src = Xq + t_blk * ldxb;
        const int64_t left = M - t_blk;               // >= 1
        const int last = left > 255 ? 255 : (int)left - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * (i * 8 + wave) + (ln >> 3);
            boff[i] = (uint32_t)(row < last ? row : last) * (uint32_t)ldxb + place((ln & 7) ^ swz(row)) * 16;
        }
        int64_t pv = (int64_t)to * 2 + (wave >> 2), pm = (int64_t)to * 2 + ((wave >> 1) & 1);
        pv = pv < npanels ? pv : npanels - 1;         // a panel beyond the last only feeds channels that are never stored
        pm = pm < npanels ? pm : npanels - 1;
        av_src = w_vals + (pv * nsteps * 4 + (wave & 3)) * 1024;
        am_src = w_meta + pm * nsteps * 1024 + (wave & 1) * 512;
    };
    // Load number d of group g of the pair whose first super-unit is u0.  Group 0: packed steps 0, 1 of u0 and u0's token tile;
    // 1: those of u1; 2: packed step 2 of both.  d: 0, 1 values, 2 index words, 3 .. 6 tokens (to ring slot tslot).
    // Where the row ends with u0, the values of u1 are zeros and its tokens (u0's again) are not read.
    auto load = [&](auto group_c, auto d_c, int u0, uint32_t tslot, uint64_t lanes, auto masked_c) __attribute__((always_inline)) {
        constexpr int G = decltype(group_c)::value, D = decltype(d_c)::value;
        constexpr bool MASKED = decltype(masked_c)::value;
        const int u1 = !ODD || u0 + 1 < U ? u0 + 1 : u0;
        if constexpr (D == 2) {
            const int u = G == 0 ? u0 : G == 1 ? u1 : mj ? u1 : u0;
            lds_dma16_lanes_from<(G == 0 ? 0 : G == 1 ? 3 : 2) * F_ASTEP>(am_src, __builtin_amdgcn_readfirstlane(u * 3072 + (G == 2 ? 2048 : mj * 1024)), lane16, m_wave + (G == 2 ? 3 : 1) * mj * F_ASTEP, lanes & 0xffffffffull);
        } else if constexpr (D < 2) {
            constexpr bool OF_U1 = G == 1 || (G == 2 && D == 1);
            constexpr int SLOT = G == 2 ? 2 + 3 * D : 3 * G + D;         // ring slot; packed step SLOT % 3 of its super-unit
            const bool none = ODD && OF_U1 && u1 == u0;
            const uint8_t* src = none ? reinterpret_cast<const uint8_t*>(no_values) : av_src;
            const uint32_t off = none ? 0 : (OF_U1 ? u1 : u0) * 12288 + (SLOT % 3) * 4096;
            if constexpr (MASKED) lds_dma16_lanes_from<SLOT * F_ASTEP>(src, off, lane16, a_wave, lanes);
            else lds_dma16_from<SLOT * F_ASTEP>(src, off, lane16, a_wave);
        } else {
            constexpr int P = D - 3;
            const uint32_t off = (G == 1 ? u1 : u0) * ROWB;
            if constexpr (MASKED) lds_dma16_lanes_from<P * 8192>(b_src, off, boff[P], __builtin_amdgcn_readfirstlane(b_wave + tslot), lanes);
            else lds_dma16_from<P * 8192>(b_src, off, boff[P], b_wave + tslot);
        }
    };
    constexpr std::false_type all_lanes{};
    uint32_t t0 = 0, t1 = F_BSLOT, tz = 2 * F_BSLOT;   // token slots of u0 and u1, and the one that is free for the next pair's u0
    int to, tt;
    bool have = tile_of_round(0, tiles_o, tiles_t, to, tt);
    if (!have) return;
    setup_tile(to, tt);
    unroll<17>([&](auto d_c) __attribute__((always_inline)) {
        constexpr int d = decltype(d_c)::value, G = d / 7;
        load(std::integral_constant<int, G>{}, std::integral_constant<int, d - 7 * G>{}, 0, G ? t1 : t0, ~0ull, all_lanes);
    });
    wait_vmcnt<10>();                                 // group 0
    wg_barrier();

    struct Regs { v4i a[8], ix[2]; v8i raw[4], mid[4]; };
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
        // operand reads of step s: weight fragment a = 4 hh + f, index words of rows 16 hh
        auto read_a = [&](int s, int a) __attribute__((always_inline)) { R.a[a] = rd((s == 2 ? va_mid : va_raw + s * 3 * F_ASTEP) + (a & 3) * 1024 + (a >> 2) * 256); };
        auto read_ix = [&](int s, int hh) __attribute__((always_inline)) { R.ix[hh] = rd((s == 2 ? va_mid : va_raw + s * 3 * F_ASTEP) + F_AIDX + hh * 256); };
        // middle windows of the lane's four blocks (two by two) of super-unit x of the pair; 8-bit types: bytes 2..5 of a block,
        // 16-bit: elements 2..5
        auto make_mid = [&](int x, int b, int half) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 2 * half; j < 2 * half + 2; ++j) {
                if constexpr (ES == 1) R.mid[b][4 * x + j] = (int)__builtin_amdgcn_alignbyte((uint32_t)R.raw[b][2 * j + 1], (uint32_t)R.raw[b][2 * j], 2);
                else asm("v_mov_b32 %0, %1" : "=v"(R.mid[b][4 * x + j]) : "v"(R.raw[b][4 * (j >> 1) + 1 + (j & 1)]));      // opaque: the compiler would rather keep the raw registers alive, and spill
            }
        };

        const uint32_t more = __builtin_amdgcn_readfirstlane(have ? ~0u : 0u);       // the last pair requests the next tile's first one, if there is one

        // The direct loads behind instruction i of step S, as group * 8 + number, -1 none.  They are spread evenly: the compute
        // unit takes 17 cycles for each, and a wavefront that has to wait for room in the queue issues no matrix instruction.
        // Order: the seven of group 0 (tokens first: more of them come from beyond the L2) from step 0 to step 1, the seven of
        // group 1 from step 1 to step 2, the three of group 2.  Cycles of a pair, INT8 / bf16, 3584 -> 37888 (matrix
        // instructions 3072): 3750 / 3850 like this, 3937 / 4040 with the meeting four instructions earlier, weights first and
        // even priorities (below), 4020 / 4500 with the loads in bunches.
        // SHORT: the last pair has no u1, so no step 1; its requests go to steps 0 and 2.
        constexpr auto load_at = [](bool SHORT, int S, int i) constexpr {
            constexpr int at[3][6] = {{15, 19, 23, 27, 31, -1}, {4, 9, 15, 20, 25, 30}, {4, 9, 15, 20, 25, 30}};
            constexpr int what[3][6] = {{3, 4, 5, 6, 0, -1}, {1, 2, 8, 9, 10, 11}, {12, 13, 14, 16, 17, 18}};
            constexpr int at_short[2][10] = {{15, 17, 19, 22, 25, 28, 31, -1, -1, -1}, {1, 4, 7, 10, 13, 17, 20, 23, 26, 29}};
            constexpr int what_short[2][10] = {{3, 4, 5, 6, 0, 1, 2, -1, -1, -1}, {8, 9, 10, 11, 12, 13, 14, 16, 17, 18}};
            for (int d = 0; d < (SHORT ? 10 : 6); ++d)
                if ((SHORT ? at_short[S / 2][d] : at[S][d]) == i) return SHORT ? what_short[S / 2][d] : what[S][d];
            return -1;
        };

        // Step S of pair p.  Instruction i: token blocks in two halves of 16 instructions, weight fragments 0 .. 7 within each,
        // so that everything has fourteen or more instructions between its last use and its next.
        auto step = [&](auto step_c, auto last_c, int p) __attribute__((always_inline)) {
            constexpr int S = decltype(step_c)::value;
            constexpr bool LAST = decltype(last_c)::value, SHORT = ODD && LAST, NEXT = S < 2 || !LAST;       // NEXT: the next step's operands are read
            constexpr int NS = S == 2 ? 0 : SHORT ? 2 : S + 1;
            constexpr int MEET = 14;
            const int u_ld = LAST ? 0 : 2 * p + 2;                       // first super-unit of the pair being requested
            const uint64_t lanes = LAST ? ((uint64_t)more << 32) | more : ~0ull;
            const uint32_t vb_now = vb + t1, vb_next = vb + (S == 0 ? t1 : tz);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (SHORT && S == 0) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int j = 4; j < 8; ++j) asm("v_mov_b32 %0, 0" : "=v"(R.mid[b][j]));      // opaque, as in make_mid
            }
            unroll<32>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int i = decltype(i_c)::value;
                constexpr int a = (i >> 1) & 7, b = 2 * (i >> 4) + (i & 1);
                acc[a & 3][a >> 2][b] = MM::sparse16(R.a[a], S == 2 ? R.mid[b] : R.raw[b], acc[a & 3][a >> 2][b], R.ix[a >> 2][a & 3]);
                __builtin_amdgcn_sched_barrier(0);
                if (i == 0) read_ix(S, 1);                                  // the words of the second four fragments were in use until now
                if (S == 1 && i < 4) read_raw(2 + (i >> 1), i & 1, vb_now);          // blocks 2 and 3 were in use until now
                if (S == 0 && i >= 1 && i < 9) make_mid(0, (i - 1) >> 1, (i - 1) & 1);
                if (S == 1 && i >= 4 && i < 8) make_mid(1, (i - 4) >> 1, i & 1);
                // the half of a step that carries the operand reads has priority over the other wavefront's half without
                if (i == 1) __builtin_amdgcn_s_setprio(0);
                if (i == 16) __builtin_amdgcn_s_setprio(1);
                if (S == 0 && LAST && i == 4) setup_tile(to, tt);          // the next tile's, or this one's again
                if (i == MEET) {
                    // 0 for the first pair of a tile that follows another: it landed before the epilogue's stores.  rest: nothing is requested by the last pair
                    const int later = min(p + 1 - min(round, 1), 1), rest = LAST ? (2 & ~(int)more) : 0;
                    if constexpr (SHORT && S == 0) wait_vm_mode<0>(later);
                    else if constexpr (S == 0) wait_vm_mode<3>(later);
                    else if constexpr (S == 1) wait_vm_mode<(LAST && MM::SCALED ? 8 : 7)>(LAST ? (later & (int)more) | rest : later);
                    else wait_vm_mode<(SHORT ? 5 : 6)>(LAST ? (1 & (int)more) | rest : 1);
                    wait_lgkm0();
                    wg_barrier();
                    if constexpr (S == 0 && LAST && MM::SCALED) load_tile_scales(s_w, s_x, O, M, o_blk, t_blk, wave, lds0 + F_SW_OFF);
                }
                if (S == 1 && i >= 9 && i < 13) make_mid(1, 2 + ((i - 9) >> 1), (i - 9) & 1);
                if constexpr (constexpr int l = load_at(SHORT, S, i); l >= 0)
                    load(std::integral_constant<int, (l >> 3)>{}, std::integral_constant<int, (l & 7)>{}, u_ld, l < 8 ? tz : t0, lanes, std::integral_constant<bool, LAST>{});
                if constexpr (NEXT) {
                    if (i >= 17 && (i & 1)) read_a(NS, (i - 17) >> 1);
                    if (i == 24) read_ix(NS, 0);
                    if (S == 0 && !SHORT && i >= 16 && !(i & 1) && i < 24) read_raw((i - 16) >> 2, (i >> 1) & 1, vb_next);
                    if (S == 2 && i >= 16 && !(i & 1)) read_raw((i - 16) >> 2, (i >> 1) & 1, vb_next);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        constexpr std::integral_constant<int, 0> s0{};
        constexpr std::integral_constant<int, 1> s1{};
        constexpr std::integral_constant<int, 2> s2{};

        // operands of step 0: published by the last meeting of the previous tile (or the prologue)
        read_ix(0, 0);
#pragma unroll
        for (int a = 0; a < 8; ++a) read_a(0, a);
#pragma unroll
        for (int r = 0; r < 8; ++r) read_raw(r >> 1, r & 1, vb + t0);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[f][hh][b][r] = 0;
        int p = 0;
        for (; p + 1 < pairs; ++p) {
            step(s0, std::false_type{}, p);
            step(s1, std::false_type{}, p);
            step(s2, std::false_type{}, p);
            const uint32_t was0 = t0, was1 = t1;
            t0 = tz; t1 = was0; tz = was1;
        }
        step(s0, std::true_type{}, p);
        if constexpr (!ODD) step(s1, std::true_type{}, p);
        step(s2, std::true_type{}, p);
        const uint32_t was0 = t0, was1 = t1;
        t0 = tz; t1 = was0; tz = was1;                 // tz: nobody reads it any more, nothing is requested into it before the next meeting
        const int64_t o_sub = o_blk + wo * 128, t_sub = t_blk + wt * 64;
        const int64_t rows = M - t_sub, cols = O - o_sub;          // <= 0: nothing of this sub-tile exists
        const bool any = rows > 0 && cols > 0;
        const int rows_left = any ? (int)(rows > 64 ? 64 : rows) : 0, cols_left = any ? (int)(cols > 128 ? 128 : cols) : 0;
        store_tile16<MM::SCALED>(acc, reinterpret_cast<const float*>(smem + F_SX_OFF) + wt * 64, reinterpret_cast<const float*>(smem + F_SW_OFF) + wo * 128,
                                 any ? Y + t_sub * ldy + o_sub : Y, (uint32_t)ldy, rows_left, cols_left, smem + F_B_OFF + tz + wave * (16 * EP_ROWB));
    }
}

}  // namespace ss

using namespace ss;

template <int DT, bool ODD>
static ss_status launch_fused(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U,
                              int64_t ldxb, void* Y, int64_t ldy, hipStream_t stream)
{
    const int tiles_o = (int)((O + BO - 1) / BO), tiles_t = (int)((M + BT - 1) / BT);
    const int cus = cu_count(), ntiles = tiles_o * tiles_t;
    const int grid = ntiles < cus ? ntiles : cus;
    if (grid <= 0) return SS_ERR_HIP;
    if (allow_dynamic_lds<k_sparse_fused<DT, ODD>>(F_LDS) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_sparse_fused<DT, ODD>), dim3(grid), dim3(512), F_LDS, stream, static_cast<const uint8_t*>(Xq), s_x,
                       static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U, ldxb, static_cast<uint16_t*>(Y), ldy,
                       tiles_o, tiles_t);
    return launch_status();
}

static ss_status fused_gemm(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                            int64_t K, int64_t ldx, int N, ss_dtype dtype, void* Y, int64_t ldy, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!valid_N(N) || N != 4) return SS_ERR_BAD_PATTERN_N;
    if (!valid_dtype(dtype)) return SS_ERR_DTYPE;
    const int es = elem_size(dtype);
    if (M < 0 || O < 0 || K <= 0 || (K * es) % KSTEP != 0 || ldx < K || (ldx * es) % 16 != 0 || ldy < O || M > (1 << 24) || ldy >= (1 << 22) ||
        ldx * es > (1 << 23))
        return SS_ERR_SHAPE;
    if (workspace_bytes > 0 && !workspace) return SS_ERR_NULL;
    if ((uintptr_t)workspace & 15) return SS_ERR_WORKSPACE;
    if (M == 0 || O == 0) return SS_OK;
    if (!Xq || !w_vals || !w_meta || !Y) return SS_ERR_NULL;
    if (!unscaled(dtype) && (!s_x || !s_w)) return SS_ERR_NULL;
    if (((uintptr_t)Xq & 15) || ((uintptr_t)w_vals & 15) || ((uintptr_t)w_meta & 15)) return SS_ERR_SHAPE;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const int U = (int)(K * es / KSTEP);
    const int64_t ldxb = ldx * es;
    // kernel family by shape, as for the other two GEMMs; the k loop counts super-units of 128 unlifted bytes
    const ss_plan p = plan_gemm(SS_KIND_FUSED, M, O, U, workspace_bytes);
    if (p.path == SS_PATH_SKINNY) return launch_sparse_fused_skinny(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, dtype, Y, ldy, hs);
    if (p.path == SS_PATH_SMALL) return launch_sparse_small(true, Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, dtype, Y, ldy, p.small, hs);
    if (p.path == SS_PATH_SLIM) return launch_sparse_slim(true, Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, dtype, Y, ldy, hs);
    if (p.path == SS_PATH_MID) return launch_sparse_fused_mid(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, dtype, Y, ldy, workspace, p.S, hs);
    if (p.path == SS_PATH_WIDE) return launch_sparse_wide(true, Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, dtype, Y, ldy, nullptr, 1, hs);
    if (p.path == SS_PATH_NARROW) return launch_sparse_fused_narrow(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, dtype, Y, ldy, hs);
    // channels [0, p.tile_o) on 256 x 256 tiles, the others on 128 x 128 or 128 x 256 tiles
    ss_status st = SS_ERR_DTYPE;
#define SS_F(DT) (U & 1 ? launch_fused<DT, true> : launch_fused<DT, false>)(Xq, s_x, w_vals, w_meta, s_w, M, p.tile_o, U, ldxb, Y, ldy, hs)
    switch (dtype) {
    case SS_I8: st = SS_F(SS_I8); break;
    case SS_FP8_E4M3: st = SS_F(SS_FP8_E4M3); break;
    case SS_BF16: st = SS_F(SS_BF16); break;
    case SS_FP16: st = SS_F(SS_FP16); break;
    }
#undef SS_F
    if (st != SS_OK || p.tile_o == O) return st;
    const int64_t row = (int64_t)U * 3 * FRAG_KB;        // lifted bytes of a weight row
    const uint8_t *const rest_vals = static_cast<const uint8_t*>(w_vals) + p.tile_o * (row / 2), *const rest_meta = static_cast<const uint8_t*>(w_meta) + p.tile_o * (row / 8);
    const float* const rest_s_w = s_w ? s_w + p.tile_o : s_w;
    uint16_t* const rest_Y = static_cast<uint16_t*>(Y) + p.tile_o;
    const int64_t rest = O - p.tile_o;
    if (narrow_pays(M, rest, cu_count())) return launch_sparse_fused_narrow(Xq, s_x, rest_vals, rest_meta, rest_s_w, M, rest, U, ldxb, dtype, rest_Y, ldy, hs);
    return launch_sparse_fused_mid(Xq, s_x, rest_vals, rest_meta, rest_s_w, M, rest, U, ldxb, dtype, rest_Y, ldy, nullptr, 1, hs);
}

extern "C" ss_status slide_sparse_gemm_fused(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M,
                                             int64_t O, int64_t K, int64_t ldx, int N, ss_dtype dtype, void* Y, int64_t ldy, void* stream)
{
    return fused_gemm(Xq, s_x, w_vals, w_meta, s_w, M, O, K, ldx, N, dtype, Y, ldy, nullptr, 0, stream);
}

extern "C" ss_status slide_sparse_gemm_fused_ws(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M,
                                                int64_t O, int64_t K, int64_t ldx, int N, ss_dtype dtype, void* Y, int64_t ldy, void* workspace,
                                                size_t workspace_bytes, void* stream)
{
    return fused_gemm(Xq, s_x, w_vals, w_meta, s_w, M, O, K, ldx, N, dtype, Y, ldy, workspace, workspace_bytes, stream);
}
