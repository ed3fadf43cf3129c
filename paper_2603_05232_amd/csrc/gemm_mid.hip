// slide_sparse_gemm and dense_gemm for token counts between the decode regime and the point where
// 256 x 256 tiles fill the chip (roughly 64 < M <= 1024 on layers with a few thousand output channels).
//
// There the large-tile kernels leave most compute units idle (M = 256 on a 3584-channel layer is 14
// tiles for 256 units), so these kernels use 128 (one weight panel) x 128 (tokens) tiles, one tile per
// workgroup of four wavefronts, each wavefront accumulating 64 channels x 64 tokens (2 x 2 blocks of a
// 32x32 matrix instruction).  The sparse kernel also comes with tiles of 64 tokens and, where workgroups share compute units
// or for some lifted rows (gemm_wide.hip has the other calls of up to 32 tokens), 32 tokens for calls that have no more: a call of few tokens
// is a stream of weights, and every token row that does not exist would be loaded and read all the same.  Operands go HBM/L2 -> LDS
// with direct-to-LDS loads into a ring of units of 128 k-bytes, one barrier per unit.
//   sparse: a unit is the token tile plus the panel's stored values and index words, which are already in
//           operand-register order (packed_layout.h); software pipeline, see k_sparse_mid;
//   dense:  a unit is a 16 KB token tile plus a 16 KB tile of weight rows, both XOR-swizzled; the inner loop
//           is left to the compiler's scheduler.
// The epilogue writes each lane's 16 consecutive channels of a token straight to Y.
// Sparse calls with at most half as many of these tiles as compute units, unless their rows are long, are on smaller tiles (gemm_small.hip).
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "lds_pipe.h"
#include "mid_order.h"
#include "device_info.h"
#include <type_traits>

namespace ss {

constexpr int MD_WAVES = 4;
constexpr int MD_THREADS = 64 * MD_WAVES;
constexpr int MD_TILE = 128;                        // output channels and tokens per workgroup
constexpr int MD_D_RING = 3;                        // units of the dense kernel's operand ring where a workgroup has a compute unit to itself
constexpr int MD_ROWS_LOADS = MD_TILE / (8 * MD_WAVES);   // 8 rows per wavefront-wide load: 4 loads per wavefront and tile
constexpr int MD_TOK = MD_TILE * ROWB;              // 16 KB
// Tiles of TM = 128, 64 or 32 tokens (the last two for the sparse kernels only): a wavefront accumulates FW fragments of
// 32 channels x TB blocks of 32 tokens, WT groups of wavefronts share out the tokens, the others the fragments.
template <int TM> struct MidShape {
    static constexpr int FW = TM == 32 ? 1 : 2, TB = TM == 128 ? 2 : 1, WT = TM == 32 ? 1 : 2;
    static constexpr int ACC = FW * TB;
    __device__ static int wo(int wave) { return WT == 2 ? wave & 1 : wave; }
    __device__ static int wt(int wave) { return WT == 2 ? wave >> 1 : 0; }
};
constexpr int MD_D_UNIT = 2 * MD_TOK;               // 32 KB
constexpr int MD_D_LPU = 2 * MD_ROWS_LOADS;         // direct loads per wavefront and unit

// per-lane source offsets of the direct loads that fill a [ROWS x 128 B] swizzled tile; rows beyond the
// matrix are clamped to its last row (their products are never stored)
template <int ROWS> struct MidRowLoader {
    static constexpr int LOADS = ROWS / (8 * MD_WAVES);
    const uint8_t* base;                            // first row of the tile (wave-uniform)
    uint32_t off[LOADS];
    __device__ void init(const uint8_t* mat, int64_t ld, int64_t row0, int64_t nrows, int wave, int lane)
    {
        base = mat + row0 * ld;
        const int64_t left = nrows - row0;             // >= 1
        const int last = left > ROWS - 1 ? ROWS - 1 : (int)left - 1;
        const uint32_t ld32 = (uint32_t)ld;             // 128 rows x ld fits 32 bits (row bytes <= 2^23)
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int row = (i * MD_WAVES + wave) * 8 + (lane >> 3);
            const int lc = (lane & 7) ^ swz(row);
            off[i] = (uint32_t)(row < last ? row : last) * ld32 + lc * 16;
        }
    }
    __device__ void issue(int64_t k0, uint8_t* lds_tile, int wave) const
    {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) lds_dma16(base + k0, off[i], lds_tile + (i * MD_WAVES + wave) * 8 * ROWB);
    }
};

// acc[f][tb][r] of lane (n = lane & 31, h = lane >> 5) is channel o_wave + 64 h + 16 f + r of token t_wave + 32 tb + n
// sw: the scales of the panel's channels from the wavefront's first, sx: those of the wavefront's tokens, both in LDS
template <bool SCALED, typename ACC, int FW, int TB>
__device__ inline void mid_store(const ACC (&acc)[FW][TB], const float* sx, const float* sw, uint16_t* __restrict__ Y, int64_t ldy, int64_t M, int64_t O,
                                 int64_t o_wave, int64_t t_wave, int lane)
{
    const int n = lane & 31, h = lane >> 5;
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
            store_block16<SCALED>(acc[f][tb], SCALED ? sx[tb * 32 + n] : 1.0f, sw + 64 * h + 16 * f, Y, ldy, M, O, o_wave + 64 * h + 16 * f, t_wave + tb * 32 + n);
}

// The scales of a tile's 128 channels and TM tokens, behind its operand rings in LDS: asked for ahead of the first unit, so that the epilogue of an unsplit call does not
// start with a trip to memory (0.4 us: 512 -> 4608 INT8 at M = 256 6.9 -> 6.4 us, 2048 -> 8192 fp8 at M = 300 13.5 -> 13.0, lifted 4096 -> 4096 INT8 at M = 1152
// 30.1 -> 29.0).
template <int TM> constexpr int MD_SCALES = (PANEL + TM + (TM & 32)) * 4;
template <int TM> __device__ inline void mid_scales(const float* s_x, const float* s_w, int64_t t0, int64_t M, int64_t o0, int64_t O, int wave, int lane, uint32_t lds)
{
    constexpr int T = (TM + 63) / 64;
    if (wave < 2) lds_dma_scales(s_w, o0 + wave * 64, O, lane, lds + wave * 256);
    else if (wave - 2 < T) lds_dma_scales(s_x, t0 + (wave - 2) * 64, M, lane, lds + wave * 256);
}

// Sum of the S partial accumulators of every tile in range order (bit-reproducible also for fp32) and the
// scale epilogue.  A workgroup has one (PER = 1) or all (PER = ACC) of the ACC blocks of 32 channels x 32 tokens of a wavefront of the GEMM kernel in a
// token tile of a panel (gridDim.y); thread (block, register quad, lane) owns four consecutive channels of one token.  The kernel is a memory round trip
// between two launches, so much is asked for at once: all arguments (not some behind the first branch: 2 % of a call), the scales, and eight ranges at a
// time, a rest of five to seven eight, of three or four four, of one or two two (loads beyond the last range repeat it and are not added).
// Against addresses by products of 64 bits, and eight loads for any rest: calls of 1 to 8 panels, M = 1 .. 32, 10, 18 and 25 ranges
// 0.89 .. 0.99 of the time (mean 0.94; 512 channels x 18944 bytes, bf16, M = 1: 10.2 -> 9.5 us), 8 to 14 ranges 0.93 .. 1.01 (0.97).
template <int DT, int TM, int PER>
__global__ __launch_bounds__((256 * PER)) void k_mid_reduce(const v4i* __restrict__ ws, int S, int64_t ntiles, const float* __restrict__ s_x,
                                                               const float* __restrict__ s_w, int64_t M, int64_t O, uint16_t* __restrict__ Y,
                                                               int64_t ldy, int tiles_t)
{
    typedef Mma<DT> MM;
    typedef MidShape<TM> MS;
    constexpr int TB = MS::TB, ACC = MS::ACC;
    typedef typename MM::acc_t acc_t;
    typedef decltype(acc_t{}[0] + acc_t{}[0]) elem_t;
    typedef elem_t quad_t __attribute__((ext_vector_type(4)));
    asm volatile("" ::"s"(ws), "s"(S), "s"(ntiles), "s"(s_x), "s"(s_w), "s"(M), "s"(O), "s"(Y), "s"(ldy), "s"(tiles_t));
    const int panel = blockIdx.y, tw = blockIdx.x / (ACC / PER), tt = tw / MD_WAVES, tile = panel * tiles_t + tt;
    const int ft = blockIdx.x % (ACC / PER) + (PER > 1 ? threadIdx.x >> 8 : 0), f = ft / TB, tb = ft % TB;
    const int wave = tw % MD_WAVES, wo = MS::wo(wave), wt = MS::wt(wave);
    const int lane = threadIdx.x & 63, r4 = (threadIdx.x >> 6) & 3;
    const int64_t tok = (int64_t)tt * TM + wt * (32 * TB) + tb * 32 + (lane & 31);
    const int64_t o = (int64_t)panel * PANEL + 16 * MS::FW * wo + 64 * (lane >> 5) + 16 * f + 4 * r4;
    if (tok >= M || o >= O) return;
    float sx = 1.0f, sw[4];
    if constexpr (MM::SCALED) {
        sx = s_x[tok];
#pragma unroll
        for (int e = 0; e < 4; ++e) sw[e] = s_w[o + e < O ? o + e : O - 1];
    }
    quad_t a = {0, 0, 0, 0};
    const v4i* src = ws + (((int64_t)tile * MD_WAVES + wave) * (4 * ACC) + ft * 4 + r4) * 64 + lane;
    const int64_t range_stride = ntiles * MD_WAVES * (4 * ACC) * 64;             // 16-byte groups between consecutive k ranges
    int s = 0;
    auto batch = [&](auto b_c, auto full_c) __attribute__((always_inline)) {
        constexpr int B = decltype(b_c)::value;
        constexpr bool FULL = decltype(full_c)::value;
        quad_t q[B];
#pragma unroll
        for (int d = 0; d < B; ++d) {
            q[d] = __builtin_bit_cast(quad_t, *src);
            src += FULL || s + d + 1 < S ? range_stride : 0;
        }
#pragma unroll
        for (int d = 0; d < B; ++d) a = FULL || s + d < S ? a + q[d] : a;
        s += B;
    };
    while (S - s >= 8) batch(std::integral_constant<int, 8>{}, std::true_type{});
    if (S - s > 4) batch(std::integral_constant<int, 8>{}, std::false_type{});
    else if (S - s > 2) batch(std::integral_constant<int, 4>{}, std::false_type{});
    else if (S - s > 0) batch(std::integral_constant<int, 2>{}, std::false_type{});
    store_quad4<MM::SCALED>(a, sx, sw, Y, ldy, O, o, tok);
}

// Work item of this workgroup: a tile of a k range.  Workgroup ids go round-robin over the 8 XCDs, and what the workgroups
// of an XCD share (weight panels, token tiles) is read into its L2 once, so tiles are dealt out in one contiguous run per
// XCD, panel by panel in bands of token tiles.  Bands are of equal width, at most `widest`: a narrow last band gives one XCD few
// token tiles of many panels, and the launch waits for it (bf16 lifted 4096 -> 4096 at M = 1280, bands of 8 and 2: 76 us, 5
// and 5: 69; M = 1152, INT8: 42 and 38).
// Split k: by_range false deals out a run of tiles in every range, so that the workgroups of an XCD stand in all ranges of
// their tiles; true one run over all (range, tile) pairs, which keeps an XCD in one range or two.  The second loses where the
// rows of those few columns meet in the same memory channels (4096 -> 4096 INT8 lifted at M = 256 in 4 ranges: 20.8 against
// 17.3 us; the dense kernel, 8192 -> 2048 at M = 192 in 8: 21.3 against 17.5) and gains where the loop is long and a run of
// tiles reads more token bytes than an XCD's L2 holds (18944 -> 3584 fused INT8 at M = 256 in 4 ranges: 29 against 35).
// By units of k per compute unit (tiles x units / 256), time of the second over the first, means over five operand forms, 12
// layers, M = 192 .. 640, three cards: up to 6 0.989, 8 to 12 1.07, 17 1.015, 19 and more 0.98.  So the first is taken from 7 to 19, with one
// token tile to 10 (calls more than 3 % slower than before the pipeline, of 464: 15, with the second throughout 27), and not beyond
// 4.5 MB of tokens (12288 -> 1536 bf16 at M = 256, hot: 19.7 against 23.9).
// Tiles of 64 and 32 tokens, where the weights are nearly all that is read, take the second throughout.  The dense kernel
// takes the first: by the same lines 60 of 504 calls were more than 3 % slower than with the first, 21 so.
static bool mid_by_range(int tile_tokens, int64_t ntiles, int64_t M, int tiles_t, int64_t units)
{
    const int64_t work = ntiles * units;
    return tile_tokens < MD_TILE || work < 7 * 256 || work > (tiles_t == 1 ? 10 : 19) * 256 || M * units > (36 << 10);
}
template <typename ACC, int FW, int TB> __device__ inline void mid_zero(ACC (&acc)[FW][TB])
{
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][tb][r] = 0;
}

// ---- sparse ---------------------------------------------------------------------------------------------
// One unit of k is 128 bytes of a token row in LDS.  Lifted input: a piece of a row of X', two matrix-instruction steps
// deep; B lane (n, qb) takes the 32 bytes [32 qb, 32 qb + 32) of each 64-byte step.  FUSED (6:8, weights packed by
// slide_decompose_fused): a piece of an unlifted row, a super-unit of three steps; B lane (n, qb) takes the 64 bytes
// [64 qb, 64 qb + 64), uses the first half in step 0, the second in step 1 and builds the eight middle windows of step 2
// in registers (packed_layout.h, fused order): the k loop is as long as the dense kernel's, with three sparse
// instructions where that one issues four dense ones.
//
// A workgroup is one wavefront per SIMD, and a wavefront issues in order, so nothing overlaps by itself: requesting a
// unit (26 or 31 KB at the 60 bytes a clock that a compute unit's direct loads reach), reading its operands from LDS and
// the matrix instructions would add up.  The loop is therefore a software pipeline: while the matrix instructions of
// unit u run on registers, the operands of unit u + 1 are read from LDS into a second set, and the direct loads of unit
// u + RING go into the ring slot that unit u has left, one by one between the matrix instructions.  What is left is the
// load path (a build with the loads alone takes 61 of the 73 us of 5003 -> 4099 fp16 8:10 at M = 777, one with everything
// else 48).  Loop by loop against one that left the overlap to the compiler: that shape 81 -> 73 us, 14336 -> 4096 fp8 at
// M = 1024 87 -> 73.
// Without PIPE the overlap is left to a second workgroup on the compute unit and to the compiler, every XCD starts at unit 0
// and bands are wider.  With lifted rows and up to a quarter more tiles than compute units, where most compute units hold one
// workgroup and the launch waits for those with two, that is the faster loop (lifted INT8 / bf16 against the pipeline, weights
// from HBM: 4096 -> 4096 at M = 1152, 288 tiles, 35 against 38 us / 59 against 68; 4096 -> 6144 at M = 768 35 against 37 / 58 against 64);
// with more tiles than that, or unlifted rows, the pipeline is (384 tiles, 4096 -> 4096 at M = 1536, same order: 39.5 against 41.1 us; fused, 288 tiles: 33 against 35).
// KG = 2: two groups of four wavefronts, each with half of the workgroup's k range and a ring of its own, meet at the same
// barriers; the second hands its sums to the first in LDS.  Two wavefronts per SIMD then cover each other's waits, which a
// deeper ring for one does less well, and no partial sums more are written.
template <int TM, bool FUSED> struct MidUnit {
    typedef MidShape<TM> MS;
    static constexpr int NS = FUSED ? 3 : 2;                              // steps
    static constexpr int AV = NS * 4096, AM = NS * 1024;                  // values, index words of a panel
    static constexpr int TOK = TM * ROWB;                                 // token rows
    static constexpr int BYTES = TOK + AV + AM;                           // 26 or 31 KB (TM = 128), 18 or 23 (64), 14 or 19 (32)
    static constexpr int RL = TM / 32;                                    // direct loads of token rows per wavefront (8 rows each)
    static constexpr int LPU = RL + NS + 1;                               // direct loads per wavefront
    static constexpr int NM = MS::ACC * NS;                               // matrix instructions per wavefront
    static constexpr int NB = 4 * MS::TB;                                 // LDS reads of token chunks per wavefront
    static constexpr int NR = NB + (MS::FW + 1) * NS;                     // LDS reads per wavefront
};
template <int NS, int FW, int TB> struct MidOps { v4i a[NS][FW]; int idx[NS][FW]; v8i b[TB][2]; };      // b[token block][half of the lane's 64 bytes]

template <int DT, int TM, int RING, bool FUSED, bool PIPE, bool ONCE, int KG>
__global__ __launch_bounds__(MD_THREADS * KG, (KG == 1 && RING * MidUnit<TM, FUSED>::BYTES + MD_SCALES<TM> <= 80 * 1024 ? 2 : 1)) void k_sparse_mid(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x,
                                                              const uint8_t* __restrict__ w_vals, const uint8_t* __restrict__ w_meta,
                                                              const float* __restrict__ s_w, int64_t M, int64_t O, int U_all, int64_t ldxb,
                                                              uint16_t* __restrict__ Y, int64_t ldy, MidOrder order, void* __restrict__ ws)
{
    static_assert(RING >= 2 && RING <= 8, "meet() covers up to seven units behind");
    typedef Mma<DT> MM;
    typedef MidUnit<TM, FUSED> MU;
    constexpr int NS = MU::NS, LPU = MU::LPU, NM = MU::NM, NR = MU::NR, NB = MU::NB, RL = MU::RL, TOK = MU::TOK;
    constexpr int FW = MU::MS::FW, TB = MU::MS::TB;
    typedef MidOps<NS, FW, TB> Ops;
    typedef int idx_t __attribute__((ext_vector_type(FW)));
    static_assert(KG == 1 || PIPE, "groups of wavefronts run the pipeline");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];      // RING units for each of the KG groups, the scales
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave_all % MD_WAVES, kg = wave_all / MD_WAVES, lane = threadIdx.x & 63;
    uint8_t* const smem = lds + kg * (RING * MU::BYTES);
    const int wo = MU::MS::wo(wave), wt = MU::MS::wt(wave);
    const int n = lane & 31, qb = lane >> 5;
    asm volatile("" ::"s"(Xq), "s"(w_vals), "s"(w_meta), "s"(M), "s"(U_all), "s"(ldxb));      // with the order all arguments that the first loads wait for, in one go
    const MidItem it = mid_item(order);
    const int64_t panel = it.panel, t0 = (int64_t)it.tt * TM;
    // k range of this workgroup, not empty (S <= U_all)
    const int first = range_first(order.k, it.range), count = range_units(order.k, it.range);
    // units [u0, u0 + U) of it are this group's; the host takes KG groups only for ranges of at least KG units
    const int u0 = first + kg * (count / KG), U = kg + 1 < KG ? count / KG : count - kg * (count / KG);

    // Direct loads of a unit, by wavefront: TM / 32 of token rows, NS of values ([step][fragment 4][lane 64][16 B]) and one of
    // NS * 256 bytes of index words ([step][lane 64][fragment 4][4 B]; lanes 0 .. 16 NS - 1)
    MidRowLoader<TM> lb;
    lb.init(Xq + (int64_t)u0 * ROWB, ldxb, t0, M, wave, lane);
    const uint8_t* av_src = w_vals + (panel * U_all + u0) * MU::AV + wave * (NS * 1024);
    const uint8_t* am_src = w_meta + (panel * U_all + u0) * MU::AM + wave * (NS * 256);
    const uint32_t lane16 = lane * 16, lds0 = lds_address(smem);
    // The k loop of XCD x starts x / 8 of the way into the range and wraps around: otherwise all XCDs ask the memory side
    // for the same token lines, and for few channels' worth of weights, at the same time (the loads alone, weights from
    // HBM: 75 -> 61 us on 5003 -> 4099 fp16 8:10 at M = 777; the kernel 78 -> 73).  In a split range of one token tile, where an
    // XCD's workgroups share nothing but the token rows of a range, so do the workgroups of an XCD: in step they all ask
    // for the same rows' lines (14336 -> 4096 at M = 65 and 128, ten forms: 4 % less time; unsplit or with several token
    // tiles, where they share weights or more rows than the L2 holds, up to 60 % more; tiles of 64 and 32 tokens, level).
    const int wg = (int)(blockIdx.y * order.nt + blockIdx.x);
    const int rot = PIPE ? (TM == 128 && order.tiles_t == 1 && order.S > 1 ? (wg + (wg >> 3)) & 7 : wg & 7) * U >> 3 : 0;
    auto direct_load = [&](int v, uint32_t slot, int d) __attribute__((always_inline)) {
        const uint32_t st = lds0 + slot;
        const int u = v + rot < U ? v + rot : v + rot - U;
        if (d < RL) lds_dma16_at(lb.base + (int64_t)u * ROWB, lb.off[d % RL], st + (d * MD_WAVES + wave) * 8 * ROWB);
        else if (d < RL + NS) {
            const int i = d - RL;
            lds_dma16_at<ONCE>(av_src + (int64_t)u * MU::AV + i * 1024, lane16, st + TOK + wave * (NS * 1024) + i * 1024);
        } else lds_dma16_lanes_at<ONCE>(am_src + (int64_t)u * MU::AM, lane16, st + TOK + MU::AV + wave * (NS * 256), (1ull << (16 * NS)) - 1);
    };
    // LDS reads of a unit's operands, in the order of their first use
    const uint32_t va = lane16 + wo * (FW * 1024) + TOK, vi = lane16 + wo * (FW * 4) + TOK + MU::AV;
    uint32_t vb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int row = wt * (32 * TB) + n, chunk = FUSED ? 4 * qb + c : 4 * (c >> 1) + 2 * qb + (c & 1);
        vb[c] = row * ROWB + ((chunk ^ swz(row)) << 4);                  // the second token block lies 32 rows = 4096 bytes on, same swizzle
    }
    auto operand_read = [&](Ops& R, uint32_t slot, int r) __attribute__((always_inline)) {
        const uint8_t* st = smem + slot;
        auto rd_a = [&](int h, int f) { R.a[h][f] = *reinterpret_cast<const v4i*>(st + va + h * 4096 + f * 1024); };
        auto rd_i = [&](int h) {
            const idx_t w = *reinterpret_cast<const idx_t*>(st + vi + h * 1024);
#pragma unroll
            for (int f = 0; f < FW; ++f) R.idx[h][f] = w[f];
        };
        auto rd_b = [&](int c, int tb) {
            const v4i v = *reinterpret_cast<const v4i*>(st + vb[c] + tb * 4096);
#pragma unroll
            for (int e = 0; e < 4; ++e) R.b[tb][c >> 1][4 * (c & 1) + e] = v[e];
        };
        if (r < FW) rd_a(0, r);                                          // step 0: weights, index words, first halves of the token chunks
        else if (r == FW) rd_i(0);
        else if (r < FW + 1 + NB) { const int k = r - FW - 1; rd_b(2 * (k / (2 * TB)) + (k & 1), (k >> 1) % TB); }      // second halves: step 1
        else { const int k = r - FW - 1 - NB, h = 1 + k / (FW + 1); if (k % (FW + 1) < FW) rd_a(h, k % (FW + 1)); else rd_i(h); }
    };

    constexpr int SCALES = KG * RING * MU::BYTES;
    if (MM::SCALED && order.S == 1 && kg == 0) mid_scales<TM>(s_x, s_w, t0, M, panel * PANEL, O, wave, lane, lds_address(lds) + SCALES);
    typename MM::acc_t acc[FW][TB];
    mid_zero(acc);
    auto mma = [&](const Ops& R, const v8i (&al)[TB], int i) __attribute__((always_inline)) {
        const int h = i / (FW * TB), f = (i / TB) % FW, tb = i % TB;
        acc[f][tb] = MM::sparse(R.a[h][f], FUSED && h == 2 ? al[tb] : R.b[tb][h & 1], acc[f][tb], R.idx[h][f]);
    };
    // middle windows of token block tb: 8-bit types: bytes 2..5 of block jd; 16-bit: elements 2..5 of block jd >> 1
    auto middle = [&](const Ops& R, v8i& al, int tb) __attribute__((always_inline)) {
#pragma unroll
        for (int jd = 0; jd < 8; ++jd) {
            auto x = [&](int k) { return (uint32_t)R.b[tb][k >> 3][k & 7]; };
            if constexpr (MM::ES == 1) al[jd] = (int)__builtin_amdgcn_alignbyte(x(2 * jd + 1), x(2 * jd), 2);
            else al[jd] = (int)x(4 * (jd >> 1) + 1 + (jd & 1));
        }
    };
    uint32_t slot = 0;                                                   // ring offset of the unit being computed
    // Unit u from the registers C.  NEXT: the operands of unit u + 1 go to N; LOAD: unit u + RING is requested.
    auto unit = [&](auto next_c, auto load_c, const Ops& C, Ops& N, int u) __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(next_c)::value, LOAD = decltype(load_c)::value;
        const uint32_t nslot = slot == (RING - 1) * MU::BYTES ? 0u : slot + MU::BYTES;
        v8i al[TB];
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            mma(C, al, i);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NEXT) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if ((r * (NM > 4 ? NM - 2 : NM - 1)) / NR == i) operand_read(N, nslot, r);
            }
            if constexpr (LOAD) {
#pragma unroll
                for (int d = 0; d < LPU; ++d)
                    if ((d * (RING == 2 ? NM / 2 : NM)) / LPU == i) direct_load(u + RING, slot, d);      // a ring of two: early (3584 -> 37888 fused INT8 at M = 128: 46.9 us, spread out 47.8)
            }
            if (FUSED && (i == 1 || (TB == 2 && i == 4))) middle(C, al[i / 4], i / 4);       // before step 2 starts at instruction 2 ACC
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = nslot;
    };
    // Own loads have landed but for `behind` units requested later, and own LDS reads have returned; then the same for
    // every wavefront.
    auto meet = [&](int behind) __attribute__((always_inline)) {
        bool done = false;
        auto upto = [&](auto n_c) __attribute__((always_inline)) {
            constexpr int N = decltype(n_c)::value;
            if (N < RING && !done && behind >= N) { wait_vmcnt<(N < RING ? N : 0) * LPU>(); done = true; }
        };
        upto(std::integral_constant<int, 7>{}); upto(std::integral_constant<int, 6>{}); upto(std::integral_constant<int, 5>{});
        upto(std::integral_constant<int, 4>{}); upto(std::integral_constant<int, 3>{}); upto(std::integral_constant<int, 2>{});
        upto(std::integral_constant<int, 1>{}); upto(std::integral_constant<int, 0>{});
        wg_barrier();
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    if constexpr (!PIPE) {                                               // RING - 1 units in flight, the rest is the compiler's
        uint32_t lslot = (RING - 1) * MU::BYTES;
#pragma unroll
        for (int i = 0; i < RING - 1; ++i)
            if (i < U) {
#pragma unroll
                for (int d = 0; d < LPU; ++d) direct_load(i, i * MU::BYTES, d);
            }
        for (int u = 0; u < U; ++u) {
            if (u + RING - 1 <= U) wait_vmcnt<(RING - 2) * LPU>(); else wait_vmcnt<0>();
            wg_barrier();                                                // unit u has landed, unit u - 1 is read
            if (u + RING - 1 < U) {
#pragma unroll
                for (int d = 0; d < LPU; ++d) direct_load(u + RING - 1, lslot, d);
            }
            Ops R;
#pragma unroll
            for (int r = 0; r < NR; ++r) operand_read(R, slot, r);
            v8i al[TB];
            if constexpr (FUSED) {
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) middle(R, al[tb], tb);
            }
#pragma unroll
            for (int i = 0; i < NM; ++i) mma(R, al, i);
            slot = slot == (RING - 1) * MU::BYTES ? 0u : slot + MU::BYTES;
            lslot = lslot == (RING - 1) * MU::BYTES ? 0u : lslot + MU::BYTES;
        }
    } else {
#pragma unroll
        for (int i = 0; i < RING; ++i)
            if (i < U) {
#pragma unroll
                for (int d = 0; d < LPU; ++d) direct_load(i, i * MU::BYTES, d);
            }
        Ops A, B;
        meet(U < RING ? U - 1 : RING - 1);                                   // unit 0
#pragma unroll
        for (int r = 0; r < NR; ++r) operand_read(A, 0, r);
        // Ahead of unit u: unit u + 1 has landed, and every wavefront holds unit u in registers (its slot is free).  The
        // loops are unrolled by two, so that the two operand sets trade places, and hold no branch between matrix
        // instructions: where paths meet, the compiler copies the accumulators (each copy waits for the instruction before).
        int u = 0;
        for (; u + RING + 1 < U; u += 2) {
            meet(RING - 2);
            unit(yes, yes, A, B, u);
            meet(RING - 2);
            unit(yes, yes, B, A, u + 1);
        }
        auto late = [&](int v) __attribute__((always_inline)) {
            meet(v + RING <= U ? RING - 2 : U - 2 - v);
            if (v + RING < U) {                                              // the odd unit the loop above left
#pragma unroll
                for (int d = 0; d < LPU; ++d) direct_load(v + RING, slot, d);
            }
        };
        for (; u + 2 < U; u += 2) {
            late(u);
            unit(yes, no, A, B, u);
            late(u + 1);
            unit(yes, no, B, A, u + 1);
        }
        if (u + 1 < U) {
            late(u);
            unit(yes, no, A, B, u);
            unit(no, no, B, A, u + 1);
        } else unit(no, no, A, B, u);
    }
    const int64_t o_wave = panel * PANEL + 16 * FW * wo, t_wave = t0 + wt * (32 * TB), item = (int64_t)it.range * order.nt + it.tile;
    if constexpr (KG == 2) {                                             // the second group hands its sums to the first in LDS
        static_assert(FW * TB == 1, "one accumulator block per wavefront");
        if (kg == 0 && count & 1) wg_barrier();                          // it has one unit, and one meeting, more
        wait_lgkm0();
        wg_barrier();                                                    // nobody reads operands any more
        v4i* const x = reinterpret_cast<v4i*>(lds) + wave * 256 + lane;
        typedef decltype(acc[0][0][0] + acc[0][0][0]) elem_t;
        typedef elem_t quad_t __attribute__((ext_vector_type(4)));
        auto& v = acc[0][0];
        if (kg == 1) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) x[r4 * 64] = __builtin_bit_cast(v4i, (quad_t){v[4 * r4], v[4 * r4 + 1], v[4 * r4 + 2], v[4 * r4 + 3]});
            wait_lgkm0();
        }
        wg_barrier();
        if (kg == 1) return;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const quad_t q = __builtin_bit_cast(quad_t, x[r4 * 64]);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * r4 + e] += q[e];
        }
    }
    if (order.S > 1) mid_store_partial(acc, ws, item, wave, lane, (int)(M - t_wave));
    else {
        const float* const sw = reinterpret_cast<const float*>(lds + SCALES);
        mid_store<MM::SCALED>(acc, sw + PANEL + wt * (32 * TB), sw + 16 * FW * wo, Y, ldy, M, O, o_wave, t_wave, lane);
    }
}

// ---- dense ----------------------------------------------------------------------------------------------
template <int DT, int RING>
__global__ __launch_bounds__(MD_THREADS) void k_dense_mid(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ Wq,
                                                          const float* __restrict__ s_w, int64_t M, int64_t O, int64_t Kb, uint16_t* __restrict__ Y,
                                                          int64_t ldy, MidOrder order, void* __restrict__ ws)
{
    typedef Mma<DT> MM;
    typedef typename MM::dfrag_t frag_t;
    constexpr int SUB = MM::DENSE_SUB, NSUB = ROWB / SUB, RPF = SUB / 32;    // k-bytes per instruction, instructions per unit, 16-byte reads per fragment
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wo = wave & 1, wt = wave >> 1;
    const int row = lane & 31, q = lane >> 5;
    const MidItem it = mid_item(order);
    const int64_t panel = it.panel, t0 = (int64_t)it.tt * MD_TILE;
    // k range of this workgroup: units [u0, u0 + U), not empty
    const int u0 = range_first(order.k, it.range), U = range_units(order.k, it.range);

    MidRowLoader<MD_TILE> la, lb;
    la.init(Wq + (int64_t)u0 * ROWB, Kb, panel * PANEL, O, wave, lane);
    lb.init(Xq + (int64_t)u0 * ROWB, Kb, t0, M, wave, lane);
    auto issue = [&](int u, int slot) {
        la.issue((int64_t)u * ROWB, smem + slot * MD_D_UNIT, wave);
        lb.issue((int64_t)u * ROWB, smem + slot * MD_D_UNIT + MD_TOK, wave);
    };
    // rows of the weight fragments in panel order, so that a lane's accumulators are consecutive channels
    int arow[2], brow[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) arow[f] = panel_row(2 * wo + f, row);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) brow[tb] = wt * 64 + tb * 32 + row;

    if (MM::SCALED && order.S == 1) mid_scales<MD_TILE>(s_x, s_w, t0, M, panel * PANEL, O, wave, lane, lds_address(smem) + RING * MD_D_UNIT);
    typename MM::acc_t acc[2][2];
    mid_zero(acc);
    constexpr int AHEAD = RING - 1;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (i < U) issue(i, i);
    int slot = 0, lslot = AHEAD;
    for (int u = 0; u < U; ++u) {
        if (u + AHEAD <= U) wait_vmcnt<(AHEAD - 1) * MD_D_LPU>(); else wait_vmcnt<0>();
        wg_barrier();
        if (u + AHEAD < U) issue(u + AHEAD, lslot);
        const uint8_t* sa = smem + slot * MD_D_UNIT;
        const uint8_t* sb = sa + MD_TOK;
#pragma unroll
        for (int t = 0; t < NSUB; ++t) {
            frag_t a[2], b[2];
#pragma unroll
            for (int piece = 0; piece < RPF; ++piece) {
                const int lc = t * (SUB / 16) + q * RPF + piece;
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const v4i v = *tile_chunk(sa, arow[f], lc);
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[f][4 * piece + e] = v[e];
                }
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
                    const v4i v = *tile_chunk(sb, brow[tb], lc);
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[tb][4 * piece + e] = v[e];
                }
            }
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) acc[f][tb] = MM::dense(a[f], b[tb], acc[f][tb]);
        }
        slot = slot == RING - 1 ? 0 : slot + 1;
        lslot = lslot == RING - 1 ? 0 : lslot + 1;
    }
    if (order.S > 1) mid_store_partial(acc, ws, (int64_t)it.range * order.nt + it.tile, wave, lane, (int)(M - t0) - wt * 64);
    else {
        const float* const sw = reinterpret_cast<const float*>(smem + RING * MD_D_UNIT);
        mid_store<MM::SCALED>(acc, sw + PANEL + wt * 64, sw + 32 * wo, Y, ldy, M, O, panel * PANEL + 32 * wo, t0 + wt * 64, lane);
    }
}

}  // namespace ss

using namespace ss;

template <int DT, int TM>
static ss_status launch_mid_reduce(const void* ws, int S, int64_t ntiles, const float* s_x, const float* s_w, int64_t M, int64_t O, void* Y,
                                   int64_t ldy, int tiles_t, hipStream_t stream)
{
    // Workgroups of all blocks of a wavefront where half of the compute units get one, of one block otherwise: S ranges of few tiles are a matter of latency.
    // Time of a whole call (sparse and dense) with one block over all of them, M = 40 .. 400, weights from HBM: 4 tiles 0.83 .. 0.95, 16 tiles 0.93 .. 0.99, 28 and 32 tiles 0.94 ..
    // 1.00; 48 and 56 tiles 1.00 .. 1.05.
    constexpr int ACC = MidShape<TM>::ACC;
#define SS_RD(PER) hipLaunchKernelGGL((k_mid_reduce<DT, TM, PER>), dim3((unsigned)(tiles_t * MD_WAVES * (ACC / PER)), (unsigned)(ntiles / tiles_t)), dim3(256 * PER), 0, stream, \
                       static_cast<const v4i*>(ws), S, ntiles, s_x, s_w, M, O, static_cast<uint16_t*>(Y), ldy, tiles_t)
    if (2 * ntiles * MD_WAVES > cu_count()) SS_RD(ACC);
    else SS_RD(1);
#undef SS_RD
    return launch_status();
}

template <int DT, int TM, int RING, bool FUSED, bool PIPE = true, bool ONCE = false, int KG = 1>
static ss_status launch_sparse_mid_ring(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M,
                                        int64_t O, int U, int64_t ldxb, void* Y, int64_t ldy, void* ws, int S, int tiles_t, int64_t ntiles,
                                        hipStream_t stream)
{
    constexpr int lds = KG * RING * MidUnit<TM, FUSED>::BYTES + MD_SCALES<TM>;
    static_assert(lds <= 160 * 1024 && (KG == 1 || lds >= TM * 512), "the rings, then the sums that are handed over");
    if (allow_dynamic_lds<k_sparse_mid<DT, TM, RING, FUSED, PIPE, ONCE, KG>>(lds) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_sparse_mid<DT, TM, RING, FUSED, PIPE, ONCE, KG>), dim3((unsigned)ntiles, (unsigned)S), dim3(MD_THREADS * KG), lds, stream,
                       static_cast<const uint8_t*>(Xq), s_x, static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U,
                       ldxb, static_cast<uint16_t*>(Y), ldy, mid_order(ntiles, tiles_t, S, mid_by_range(TM, ntiles, M, tiles_t, U), U, PIPE ? 8 : 16), ws);
    if (launch_status() != SS_OK) return SS_ERR_HIP;
    return S > 1 ? launch_mid_reduce<DT, TM>(ws, S, ntiles, s_x, s_w, M, O, Y, ldy, tiles_t, stream) : SS_OK;
}

// U units per token row (lifted rows, or unlifted ones when FUSED), ldxb bytes between rows
template <int DT, bool FUSED>
static ss_status launch_sparse_mid_dt(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M,
                                      int64_t O, int U, int64_t ldxb, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    const int64_t npanels = (O + PANEL - 1) / PANEL;
    const int tiles_t = (int)((M + MD_TILE - 1) / MD_TILE);              // one tile where the tokens fit a smaller one
    const int64_t ntiles = npanels * tiles_t;
    // Ring depth: with more workgroups than compute units, as deep as lets two of them share a compute unit's LDS and cover
    // each other's waits.  A workgroup alone: the whole ring is requested at once, so that a deeper one delays the first
    // unit (3584 -> 4608 at M = 256, which small tiles serve now, in 3 ranges: 20.6 us with five units, 20.4 with four, 20.0 with three), but covers longer
    // waits (5003 -> 4099 fp16 8:10 at M = 777: 65.7, 63.7, 70.9).  32 tokens at most and no more workgroups than compute units:
    // the weight stream of gemm_wide.hip (both sides there), or two groups of wavefronts with a ring of four each (two_groups).
    const bool shared = ntiles * S > cu_count();
#define SS_MID(TM, ...) launch_sparse_mid_ring<DT, TM, __VA_ARGS__>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, tiles_t, ntiles, stream)
    const bool once = weights_stream(O, (int64_t)U * MidUnit<32, FUSED>::NS * FRAG_KB, M <= 32 || (Mma<DT>::ES == 1 && !shared) ? CACHED_BYTES : CACHE_BYTES);
    if (M <= 32) {
        if constexpr (!FUSED)
            if (two_groups(M, O, U, cu_count())) return once ? SS_MID(32, 4, FUSED, true, true, 2) : SS_MID(32, 4, FUSED, true, false, 2);
        if (!shared) return launch_sparse_wide(FUSED, Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, (ss_dtype)DT, Y, ldy, ws, S, stream);
        return once ? SS_MID(32, 4, FUSED, true, true) : SS_MID(32, 4, FUSED);
    }
    if (M <= 64) {
        if (shared) return once ? SS_MID(64, 3, FUSED, true, true) : SS_MID(64, 3, FUSED);
        return once ? SS_MID(64, 4, FUSED, true, true) : SS_MID(64, 4, FUSED);
    }
    if constexpr (!FUSED)
        if (shared && 4 * ntiles <= 5 * cu_count()) return SS_MID(128, 3, FUSED, false);
    return shared ? SS_MID(128, (FUSED ? 2 : 3), FUSED) : SS_MID(128, (FUSED ? 3 : 4), FUSED);
#undef SS_MID
}

template <int DT, int RING>
static ss_status launch_dense_mid_ring(const void* Xq, const float* s_x, const void* Wq, const float* s_w, int64_t M, int64_t O, int64_t Kb, void* Y,
                                       int64_t ldy, void* ws, int S, int tiles_t, int64_t ntiles, hipStream_t stream)
{
    constexpr int lds = RING * MD_D_UNIT + MD_SCALES<MD_TILE>;
    if (allow_dynamic_lds<k_dense_mid<DT, RING>>(lds) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_dense_mid<DT, RING>), dim3((unsigned)ntiles, (unsigned)S), dim3(MD_THREADS), lds, stream, static_cast<const uint8_t*>(Xq),
                       s_x, static_cast<const uint8_t*>(Wq), s_w, M, O, Kb, static_cast<uint16_t*>(Y), ldy, mid_order(ntiles, tiles_t, S, false, Kb / ROWB), ws);
    return launch_status();
}

template <int DT>
static ss_status launch_dense_mid_dt(const void* Xq, const float* s_x, const void* Wq, const float* s_w, int64_t M, int64_t O, int64_t Kb, void* Y,
                                     int64_t ldy, void* ws, int S, hipStream_t stream)
{
    const int tiles_t = (int)((M + MD_TILE - 1) / MD_TILE);
    const int64_t ntiles = (O + PANEL - 1) / PANEL * tiles_t;
    // ring depth as for the fused sparse kernel: two units (64 KB) where two workgroups can share a compute unit
    const ss_status st = ntiles * S > cu_count()
        ? launch_dense_mid_ring<DT, 2>(Xq, s_x, Wq, s_w, M, O, Kb, Y, ldy, ws, S, tiles_t, ntiles, stream)
        : launch_dense_mid_ring<DT, MD_D_RING>(Xq, s_x, Wq, s_w, M, O, Kb, Y, ldy, ws, S, tiles_t, ntiles, stream);
    if (st != SS_OK) return st;
    return S > 1 ? launch_mid_reduce<DT, 128>(ws, S, ntiles, s_x, s_w, M, O, Y, ldy, tiles_t, stream) : SS_OK;
}

// Host side, called by the C entry points.  Arguments are already validated.
namespace ss {

ss_status launch_mid_reduce32(const void* ws, int S, const float* s_x, const float* s_w, int64_t M, int64_t O, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream)
{
    const int64_t ntiles = (O + PANEL - 1) / PANEL;
    switch (dtype) {
    case SS_I8: return launch_mid_reduce<SS_I8, 32>(ws, S, ntiles, s_x, s_w, M, O, Y, ldy, 1, stream);
    case SS_FP8_E4M3: return launch_mid_reduce<SS_FP8_E4M3, 32>(ws, S, ntiles, s_x, s_w, M, O, Y, ldy, 1, stream);
    case SS_BF16: return launch_mid_reduce<SS_BF16, 32>(ws, S, ntiles, s_x, s_w, M, O, Y, ldy, 1, stream);
    case SS_FP16: return launch_mid_reduce<SS_FP16, 32>(ws, S, ntiles, s_x, s_w, M, O, Y, ldy, 1, stream);
    }
    return SS_ERR_DTYPE;
}

// bytes of a tile's partial sums: the tile the launchers take for M tokens
static size_t mid_tile_bytes(ss_kind kind, int64_t M) { return (size_t)MD_TILE * 4 * (kind == SS_KIND_DENSE || M > 64 ? 128 : M > 32 ? 64 : 32); }

// Number of k ranges for the tiles of this shape over `units` 128-byte k units with a workspace of ws_bytes: at most one
// workgroup per compute unit, at least eight units per range, no more than the workspace holds.
// Dense kernel: as many as that allows.  Sparse, M <= 64: the same (three quarters of a workgroup per compute unit for tiles
// of up to 32 tokens, where as many as compute units are 0.94 to 1.04 of the time of that, mean 1.00; bf16 3584 -> 4608 at M = 64, 56
// units: 17.3 us in 3 ranges, 14.4 in 5, 13.8 in 7), but short rows are not split at 33..64 tokens.
// Sparse, M > 64: the S of the least S-th part of the units + cost of the partial sums, which is, counted in units, 4 + a
// 16th of the tiles x ranges written and read back, and 2 more where the ranges take over 7/8 of the compute units: on two of
// three cards a split launch of that many workgroups ends 3 to 4 us late (8192 -> 2048 lifted INT8 at M = 192: 16.4 us in 6 ranges of
// 32 tiles, 16.4 in 8 on one card, 21.3 on others).  The unsplit kernel is fast enough that a few ranges more than
// that cost more than they save (fused INT8 on these tiles, weights from HBM; the first three calls are on small tiles now, gemm_small.hip): 2048 -> 8192
// at M = 256 (16 units, 128 tiles) 15.1 us unsplit, 21.0 in 2 ranges; 2048 -> 2048 at M = 640 (16 units, 80 tiles) 11.3 unsplit, 16.1 in 2; 4096 -> 4096 at M = 512
// (32 units, 128 tiles) 22.4 unsplit, 22.0 in 2 (hot 17.4 and 20.4); 18944 -> 3584 at M = 256 (148 units, 56 tiles) 83 unsplit, 33.0 in 4.
// Over 2520 calls (five operand forms, 12 layers, M = 65 .. 512, three cards) 0.960 of the time before the pipeline with weights from
// HBM (77 more than 3 % slower) and 0.865 hot (none); a 20th and nothing for the last workgroups 0.974 (188) and 0.891 (49).
int mid_splits(ss_kind kind, int64_t M, int64_t O, int64_t units, size_t ws_bytes)
{
    const int64_t ntiles = mid_tiles(M, O);
    const bool sparse = kind != SS_KIND_DENSE;
    if (sparse && M > 32 && M <= 64 && units < 48) return 1;
    int64_t S = (sparse && M <= 32 ? 3 * cu_count() / 4 : cu_count()) / ntiles;
    if (S > units / 8) S = units / 8;
    const int64_t fit = (int64_t)(ws_bytes / ((size_t)ntiles * mid_tile_bytes(kind, M)));
    if (S > fit) S = fit;
    if (S < 2) return 1;
    if (!sparse || M <= 64) return (int)S;
    int64_t best = 1, least = 16 * units;                               // 16ths of a unit
    for (int64_t s = 2; s <= S; ++s) {
        const int64_t t = 16 * ((units + s - 1) / s + (8 * s * ntiles > 7 * cu_count() ? 6 : 4)) + s * ntiles;
        if (t < least) { least = t; best = s; }
    }
    return (int)best;
}

size_t mid_workspace_bytes(ss_kind kind, int64_t M, int64_t O, int S)
{
    return S > 1 ? (size_t)S * mid_tiles(M, O) * mid_tile_bytes(kind, M) : 0;
}

ss_status launch_sparse_mid(const void* XL, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                            int64_t Kpb, ss_dtype dtype, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    switch (dtype) {
    case SS_I8: return launch_sparse_mid_dt<SS_I8, false>(XL, s_x, w_vals, w_meta, s_w, M, O, (int)(Kpb / KSTEP), Kpb, Y, ldy, ws, S, stream);
    case SS_FP8_E4M3: return launch_sparse_mid_dt<SS_FP8_E4M3, false>(XL, s_x, w_vals, w_meta, s_w, M, O, (int)(Kpb / KSTEP), Kpb, Y, ldy, ws, S, stream);
    case SS_BF16: return launch_sparse_mid_dt<SS_BF16, false>(XL, s_x, w_vals, w_meta, s_w, M, O, (int)(Kpb / KSTEP), Kpb, Y, ldy, ws, S, stream);
    case SS_FP16: return launch_sparse_mid_dt<SS_FP16, false>(XL, s_x, w_vals, w_meta, s_w, M, O, (int)(Kpb / KSTEP), Kpb, Y, ldy, ws, S, stream);
    }
    return SS_ERR_DTYPE;
}

ss_status launch_sparse_fused_mid(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                                  int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    switch (dtype) {
    case SS_I8: return launch_sparse_mid_dt<SS_I8, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream);
    case SS_FP8_E4M3: return launch_sparse_mid_dt<SS_FP8_E4M3, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream);
    case SS_BF16: return launch_sparse_mid_dt<SS_BF16, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream);
    case SS_FP16: return launch_sparse_mid_dt<SS_FP16, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream);
    }
    return SS_ERR_DTYPE;
}

ss_status launch_dense_mid(const void* Xq, const float* s_x, const void* Wq, const float* s_w, int64_t M, int64_t O, int64_t Kb, ss_dtype dtype,
                           void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    switch (dtype) {
    case SS_I8: return launch_dense_mid_dt<SS_I8>(Xq, s_x, Wq, s_w, M, O, Kb, Y, ldy, ws, S, stream);
    case SS_FP8_E4M3: return launch_dense_mid_dt<SS_FP8_E4M3>(Xq, s_x, Wq, s_w, M, O, Kb, Y, ldy, ws, S, stream);
    case SS_BF16: return launch_dense_mid_dt<SS_BF16>(Xq, s_x, Wq, s_w, M, O, Kb, Y, ldy, ws, S, stream);
    case SS_FP16: return launch_dense_mid_dt<SS_FP16>(Xq, s_x, Wq, s_w, M, O, Kb, Y, ldy, ws, S, stream);
    }
    return SS_ERR_DTYPE;
}

}  // namespace ss
