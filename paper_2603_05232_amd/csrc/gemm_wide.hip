// Sparse GEMMs of one tile of tokens as a stream of weights, bound by HBM: up to 32 tokens with a workgroup for each panel (NF = 4
// fragments of 32 channels) and k range, and up to 64 tokens, unlifted rows of 97 to 128, on layers of
// more panels than compute units (NF = 5, 6 or 8).
//
// A wavefront owns one fragment and all tokens.  The loop is plain: wait for a unit, meet, request a later one, read the operands,
// multiply; the order is left to the compiler.  A unit takes a compute unit 1500 cycles to stream and its operand reads and
// matrix instructions a third of that, so a software pipeline in two groups of wavefronts, each with half of the k range (KG = 2 in gemm_mid.hip),
// does not pay but for the lifted rows it has kept.  NF = 4 over it with the same kind of loads, INT8 and bf16 fused, fp8 and bf16 lifted, M = 1 .. 32,
// weights from HBM / hot:
// rows of 64 to 200 units in ranges, 300 calls 0.91 .. 1.02 (mean 0.96) / 0.91 .. 1.12 (0.97), 129 to 256 panels in 12 to 100 units, fused, 168 calls 0.91 .. 1.02
// (0.96) / 0.87 .. 1.15 (0.97), and in 1 to 15 units, 216 calls 0.86 .. 1.02 (0.95) / 0.81 .. 1.10 (0.95).  There is no line by the length of a row: two to ten units gain
// most, and the calls that lose 5 % hot and more, 12 to 16 units whose weights the L2 holds (129 panels, lifted rows 192) and single longer ones, gain 1 to 5 % from HBM.
//
// More panels than compute units: a workgroup per panel gives some compute units two streams where the others have one, and a
// compute unit has about a hundred cache lines in flight whatever its workgroups ask for, so the launch waits for those with two:
// 128 MB streamed into LDS by 256 workgroups take 20.3 us, by 296 26.1.  There a workgroup owns as many fragments as leave at most one
// workgroup for each compute unit, without a k split.  3584 -> 37888 at M = 1, weights from HBM: INT8 29.3 -> 22.1 us (5.8 TB/s),
// bf16 53.5 -> 37.9 (6.7 TB/s).
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "lds_pipe.h"
#include "device_info.h"

namespace ss {

// A unit of 128 bytes of a token row in LDS: token rows (swizzled), values [fragment][step][lane][16 B], index words of the panel or
// the two panels the fragments lie in [panel][step][lane][fragment of the panel][4 B].  NF = 4: a ring of four (fused) or five units; one more, for
// which a compute unit has room where it holds one workgroup, 1.01 to 1.02 of the time.
template <int NF, int TB, bool FUSED> struct WideUnit {
    static constexpr int NS = FUSED ? 3 : 2;
    static constexpr int PANELS = NF == 4 ? 1 : 2;
    static constexpr int TOK = TB * 32 * ROWB, AV = NF * NS * 1024, AM = PANELS * NS * 1024, BYTES = TOK + AV + AM;
    static constexpr int SHARED = TB * 4 + PANELS * NS;                        // 1 KB pieces of tokens and index words
    static constexpr int E = (SHARED + NF - 1) / NF, LPU = NS + E;        // direct loads per wavefront: its values, its share of those
    static constexpr int SCALES = (PANELS * PANEL + (TB == 1 ? 64 : TB * 32)) * 4;          // of the channels and tokens, behind the ring
    static constexpr int FIT = (NF == 4 ? 80 : 160) * 1024 / BYTES, RING = FIT < 5 ? FIT : 5;
    static constexpr bool SCALES_FIT = RING * BYTES + SCALES <= (NF == 4 ? 80 : 160) * 1024;
    static constexpr int LDS = RING * BYTES + (SCALES_FIT ? SCALES : 0);
};

template <int DT, int NF, int TB, bool FUSED, bool ONCE>
__global__ __launch_bounds__(64 * NF) void k_sparse_wide(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                         const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int U_all,
                                                         int64_t ldxb, uint16_t* __restrict__ Y, int64_t ldy, void* __restrict__ ws, int cols, int S, Div by_cols,
                                                         KRanges ranges)
{
    typedef Mma<DT> MM;
    typedef WideUnit<NF, TB, FUSED> WU;
    constexpr int NS = WU::NS, RING = WU::RING;
    static_assert(RING >= 3 && (RING - 2) * WU::LPU < 64, "loads in flight");
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 31, qb = lane >> 5;
    asm volatile("" ::"s"(Xq), "s"(w_vals), "s"(w_meta), "s"(M), "s"(O), "s"(U_all), "s"(ldxb), "s"(cols), "s"(S), "s"(by_cols.mul), "s"(ranges.q));      // in one go
    const int npanels = (int)((O + PANEL - 1) / PANEL), nfrags = npanels * FRAGS_PER_PANEL;
    // work item: fragments of a k range, one run over all (range, fragments) pairs for each XCD
    const int wg = blockIdx.y * cols + blockIdx.x, item = xcd_run(wg, cols * S), range = quot(item, by_cols), col = item - range * cols;
    const int u_first = range_first(ranges, range), U = range_units(ranges, range);
    const int f_first = col * NF, p_first = f_first / FRAGS_PER_PANEL;
    const int frag = min(f_first + wave, nfrags - 1), panel = frag / FRAGS_PER_PANEL, f = frag % FRAGS_PER_PANEL;     // beyond the last: that one again, not stored
    const uint32_t lane16 = lane * 16, lds0 = lds_address(smem);

    // The scales, asked for ahead of the first unit (else the epilogue starts with a trip to memory: 3584 -> 37888 INT8 at M = 1 22.1 -> 21.6 us, at
    // M = 100 33.8 -> 33.2).  NF = 6 with 128 tokens has no room for them but in the ring, when all units are read.
    constexpr int SCALES = WU::SCALES_FIT ? RING * WU::BYTES : 0, PIECES = WU::SCALES / 256;
    auto scales = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < (PIECES + NF - 1) / NF; ++e) {
            const int piece = wave + e * NF;
            if (piece < 2 * WU::PANELS) lds_dma_scales(s_w, (int64_t)p_first * PANEL + piece * 64, O, lane, lds0 + SCALES + piece * 256);
            else if (piece < PIECES) lds_dma_scales(s_x, (piece - 2 * WU::PANELS) * 64, M, lane, lds0 + SCALES + piece * 256);
        }
    };
    if (MM::SCALED && WU::SCALES_FIT && S == 1) scales();

    // Sources of this wavefront's loads.  Lanes of tokens that do not exist load nothing (their products are never stored).
    const uint8_t* const av_src = w_vals + (((int64_t)panel * U_all + u_first) * NS * FRAGS_PER_PANEL + f) * 1024;
    const uint8_t* e_src[WU::E];
    uint32_t e_off[WU::E], e_step[WU::E], e_dst[WU::E];
    uint64_t e_lanes[WU::E];
    auto uniform = [](uint64_t v) { return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v); };
#pragma unroll
    for (int e = 0; e < WU::E; ++e) {
        const int piece = wave + e * NF;
        const bool tokens = piece < TB * 4;
        const int rows = max(0, min(8, (int)M - piece * 8)), row = piece * 8 + (lane >> 3);
        const int k = max(0, piece - TB * 4), p = min(p_first + k / NS, npanels - 1);
        const uint64_t some = rows == 8 ? ~0ull : (1ull << (8 * rows)) - 1;
        e_src[e] = reinterpret_cast<const uint8_t*>(uniform((uint64_t)(uintptr_t)(tokens ? Xq + (int64_t)u_first * ROWB : w_meta + (((int64_t)p * U_all + u_first) * NS + k % NS) * 1024)));
        e_off[e] = tokens ? (uint32_t)row * (uint32_t)ldxb + (((lane & 7) ^ swz(row)) << 4) : lane16;
        e_step[e] = __builtin_amdgcn_readfirstlane(tokens ? ROWB : NS * 1024);
        e_dst[e] = __builtin_amdgcn_readfirstlane(tokens ? piece * 1024 : WU::TOK + WU::AV + k * 1024);
        e_lanes[e] = uniform(tokens ? some : piece < WU::SHARED ? ~0ull : 0ull);
    }
    // As in gemm_mid.hip the XCDs start at different places of the row, NF = 4 in twice as many: with eight places, panels of
    // certain sizes (504 KB, 512 KB) meet in the same memory channels (time with 16 over 8, M = 4 and 24, 129 to 256 panels, weights from HBM: fused rows of 42 units
    // 0.90 .. 1.00, 96 units 0.88 .. 1.00, lifted rows of 64 units 0.95 .. 1.00, 128 units 0.93 .. 1.01; all other lengths of 21 to 148 units 0.96 .. 1.04, mean 1.00;
    // 32 and 64 places up to 1.16 and 1.22 at single lengths; NF = 5, 6 and 8 with 16 places 0.97 .. 1.15).
    constexpr int PLACES = NF == 4 ? 16 : 8;
    const int rot = (wg & (PLACES - 1)) * U / PLACES;
    auto issue = [&](int v, uint32_t slot) __attribute__((always_inline)) {
        const int u = v + rot < U ? v + rot : v + rot - U;
#pragma unroll
        for (int h = 0; h < NS; ++h)
            lds_dma16_at<ONCE>(av_src + ((int64_t)u * NS + h) * (FRAGS_PER_PANEL * 1024), lane16, lds0 + slot + WU::TOK + (wave * NS + h) * 1024);
#pragma unroll
        for (int e = 0; e < WU::E; ++e) lds_dma16_lanes_at(e_src[e] + (int64_t)u * e_step[e], e_off[e], lds0 + slot + e_dst[e], e_lanes[e]);
    };
    uint32_t vb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) vb[c] = n * ROWB + (((FUSED ? 4 * qb + c : 4 * (c >> 1) + 2 * qb + (c & 1)) ^ swz(n)) << 4);
    const uint32_t va = WU::TOK + wave * (NS * 1024) + lane16, vi = WU::TOK + WU::AV + (panel - p_first) * (NS * 1024) + lane16 + 4 * f;

    typename MM::acc_t acc[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[tb][r] = 0;
#pragma unroll
    for (int i = 0; i < RING - 1; ++i)
        if (i < U) issue(i, i * WU::BYTES);
    uint32_t slot = 0, lslot = (RING - 1) * WU::BYTES;
    for (int u = 0; u < U; ++u) {
        if (u + RING - 1 <= U) wait_vmcnt<(RING - 2) * WU::LPU>(); else wait_vmcnt<0>();
        wg_barrier();                                                    // unit u has landed, unit u - 1 is read
        if (u + RING - 1 < U) issue(u + RING - 1, lslot);
        const uint8_t* st = smem + slot;
        v4i a[NS];
        int idx[NS];
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            a[h] = *reinterpret_cast<const v4i*>(st + va + h * 1024);
            idx[h] = *reinterpret_cast<const int*>(st + vi + h * 1024);
        }
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            v4i x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = *reinterpret_cast<const v4i*>(st + vb[c] + tb * (32 * ROWB));
#pragma unroll
            for (int h = 0; h < 2; ++h)
                acc[tb] = MM::sparse(a[h], v8i{x[2 * h][0], x[2 * h][1], x[2 * h][2], x[2 * h][3], x[2 * h + 1][0], x[2 * h + 1][1], x[2 * h + 1][2], x[2 * h + 1][3]}, acc[tb], idx[h]);
            if constexpr (FUSED) {                                       // middle windows: see gemm_mid.hip
                v8i m;
#pragma unroll
                for (int jd = 0; jd < 8; ++jd) {
                    auto w = [&](int k) { return (uint32_t)x[k >> 2][k & 3]; };
                    if constexpr (MM::ES == 1) m[jd] = (int)__builtin_amdgcn_alignbyte(w(2 * jd + 1), w(2 * jd), 2);
                    else m[jd] = (int)w(4 * (jd >> 1) + 1 + (jd & 1));
                }
                acc[tb] = MM::sparse(a[2], m, acc[tb], idx[2]);
            }
        }
        slot = slot == (RING - 1) * WU::BYTES ? 0u : slot + WU::BYTES;
        lslot = lslot == (RING - 1) * WU::BYTES ? 0u : lslot + WU::BYTES;
    }
    if constexpr (MM::SCALED && !WU::SCALES_FIT) {
        wait_lgkm0();
        wg_barrier();
        scales();
        wait_vmcnt<0>();
        wg_barrier();
    }
    if (f_first + wave >= nfrags) return;
    if (NF == 4 && TB == 1 && S > 1) {
        const typename MM::acc_t part[1][1] = {{acc[0]}};
        mid_store_partial(part, ws, item, wave, lane, (int)M);
        return;
    }
    const float* const sw = reinterpret_cast<const float*>(smem + SCALES), *const sx = sw + WU::PANELS * PANEL;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
        store_block16<MM::SCALED>(acc[tb], MM::SCALED ? sx[tb * 32 + n] : 1.0f, sw + (panel - p_first) * PANEL + 64 * qb + 16 * f, Y, ldy, M, O,
                                  (int64_t)panel * PANEL + 64 * qb + 16 * f, tb * 32 + n);
}

}  // namespace ss

using namespace ss;

template <int DT, int NF, int TB, bool FUSED, bool ONCE>
static ss_status launch_wide_one(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U,
                                 int64_t ldxb, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    typedef WideUnit<NF, TB, FUSED> WU;
    constexpr int lds = WU::LDS;
    static_assert(lds <= 160 * 1024, "LDS budget");
    const int64_t nfrags = (O + PANEL - 1) / PANEL * FRAGS_PER_PANEL;
    const int cols = (int)((nfrags + NF - 1) / NF);
    if (allow_dynamic_lds<k_sparse_wide<DT, NF, TB, FUSED, ONCE>>(lds) != SS_OK) return SS_ERR_HIP;
    hipLaunchKernelGGL((k_sparse_wide<DT, NF, TB, FUSED, ONCE>), dim3((unsigned)cols, (unsigned)S), dim3(64 * NF), lds, stream,
                       static_cast<const uint8_t*>(Xq), s_x, static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U, ldxb,
                       static_cast<uint16_t*>(Y), ldy, ws, cols, S, make_div(cols), k_ranges(U, S));
    return launch_status();
}

template <int DT, bool FUSED>
static ss_status launch_wide_dt(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U,
                                int64_t ldxb, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    const int nf = (O + PANEL - 1) / PANEL <= cu_count() ? 4 : wide_fragments(FUSED ? SS_KIND_FUSED : SS_KIND_LIFTED, M, O, cu_count());
    const bool once = weights_stream(O, (int64_t)U * (FUSED ? 3 : 2) * FRAG_KB, M <= 64 ? CACHED_BYTES : CACHE_BYTES);
#define SS_W(NF, TB) return once ? launch_wide_one<DT, NF, TB, FUSED, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream) \
                                 : launch_wide_one<DT, NF, TB, FUSED, false>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream)
#define SS_WN(NF) { if (M <= 32) SS_W(NF, 1); if (M <= 64) SS_W(NF, 2); }
    if (nf == 4) SS_W(4, 1);
    if (nf == 5) SS_WN(5)
    if (nf == 6) SS_WN(6)
    if (nf == 8) SS_WN(8)
    if constexpr (FUSED) {
        if (nf == 5) SS_W(5, 4);
        if (nf == 6) SS_W(6, 4);
    }
    return SS_ERR_SHAPE;                                                 // not a call that plan_gemm sends here
#undef SS_WN
#undef SS_W
}

namespace ss {

ss_status launch_sparse_wide(bool fused, const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, void* ws, int S, hipStream_t stream)
{
    ss_status st = SS_ERR_DTYPE;
#define SS_WD(DT) st = fused ? launch_wide_dt<DT, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream) \
                             : launch_wide_dt<DT, false>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, ws, S, stream); break
    switch (dtype) {
    case SS_I8: SS_WD(SS_I8);
    case SS_FP8_E4M3: SS_WD(SS_FP8_E4M3);
    case SS_BF16: SS_WD(SS_BF16);
    case SS_FP16: SS_WD(SS_FP16);
    }
#undef SS_WD
    return st == SS_OK && S > 1 ? launch_mid_reduce32(ws, S, s_x, s_w, M, O, dtype, Y, ldy, stream) : st;
}

}  // namespace ss
