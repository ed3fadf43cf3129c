// Sparse GEMMs of up to 16 tokens with a workgroup for every 16 output channels: layers whose 32-channel workgroups (gemm_skinny.hip) leave
// most compute units idle, and whose k ranges need not be split then.
//
// What bounds it.  A compute unit gets 80 (one token, three quarters of them from beyond its L2) to 160 (16, a third) cache lines a microsecond (counted, with
// the launch), so a layer of 4096 channels on half of the compute units waits for loads while the other half has none.  Eight workgroups for a panel put it
// on all of them.  A workgroup takes rows 8 j .. 8 j + 7 of two fragments of the panel: eight rows are one whole line of stored values (rows of all four
// fragments in runs of four, half lines: 1.05 .. 1.8 of the time), and two workgroups share the lines of index words.  Eight wavefronts take stages of the row in
// turn, two stages in flight each (three or four, or sixteen wavefronts: 0.99 .. 1.15); operands go from memory to registers, and the sums meet in
// LDS in the order of the wavefronts.  The price is the token rows, which every workgroup reads whole: the kernel loses its lead with M times the
// length of the row (slim_pays, mma_types.h).  Reading them as whole lines, two lanes trading halves, changed nothing (1.00 .. 1.07).
//
// Against the kernels of before, weights from HBM / hot: INT8 3584 -> 3584 at M = 1 7.0 -> 5.3 us / 5.6 -> 3.7, 4096 -> 4096 at M = 16 lifted 9.8
// -> 7.3 / 8.3 -> 5.8, bf16 4096 -> 4096 at M = 8 10.8 -> 9.4 / 8.9 -> 6.6; 2048 -> 2048 at M = 16 5.6 -> 4.2 / 5.1 -> 3.7.
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "device_info.h"

namespace ss {

constexpr int SLIM_PARTS = 8;                         // workgroups per panel
constexpr int SLIM_WAVES = 8;

// One stage of the k range: NS matrix-instruction steps of 128 lifted bytes.  Three of them: a pair of super-units u0, u1 of unlifted rows, in the operand order
// told in gemm_fused.hip; one: a unit of lifted rows (gemm_lifted.hip).  Lane (n, g): weight row n, token n.
template <int NS> struct SlimStage { v4i a[NS]; int ix[NS]; v8i raw[NS == 3 ? 2 : 1]; };

template <bool ONCE> __device__ inline v4i slim_load(const uint8_t* p)
{
    if constexpr (ONCE) return __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
    else return *reinterpret_cast<const v4i*>(p);
}

template <int DT, bool FUSED, bool ONCE>
__global__ __launch_bounds__(64 * SLIM_WAVES) void k_sparse_slim(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                            const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int U,
                                                            int64_t ldxb, uint16_t* __restrict__ Y, int64_t ldy)
{
    typedef Mma<DT> MM;
    constexpr int NS = FUSED ? 3 : 1, NU = FUSED ? 2 : 1, WAVES = SLIM_WAVES, D = FUSED ? 2 : 4;      // D stages in flight
    constexpr uint32_t V_STEP = FUSED ? 24576 : 8192, I_STEP = V_STEP / 4, X_STEP = NU * KSTEP;
    __shared__ __attribute__((aligned(16))) v4i red[(WAVES - 1) * 64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 15, g = lane >> 4;
    // the workgroups of a panel share its index words and run on one XCD
    const int item = xcd_run(blockIdx.x, gridDim.x), panel = item / SLIM_PARTS, q = item & 1, j = (item >> 1) & 3;
    const int row = 8 * j + (n & 7), frag = 2 * q + (n >> 3);
    const uint8_t* const vals = w_vals + (int64_t)panel * U * (FUSED ? 12288 : 8192);
    const uint8_t* const meta = w_meta + (int64_t)panel * U * (FUSED ? 3072 : 2048);
    const uint32_t at = frag * 64 + row + 32 * (g >> 1), at_mid = frag * 64 + row + 32 * (g & 1);
    const uint32_t v_raw = (g & 1) * 4096 + at * 16, v_mid = (2 + 3 * (g >> 1)) * 4096 + at_mid * 16;
    const uint32_t i_raw = (g & 1) * 1024 + (row + 32 * (g >> 1)) * 16 + frag * 4, i_mid = (2 + 3 * (g >> 1)) * 1024 + (row + 32 * (g & 1)) * 16 + frag * 4;
    const bool live = n < M;                          // lanes without a token load nothing
    const uint8_t* const x = Xq + (live ? n : 0) * ldxb + (FUSED ? 64 * (g & 1) + 32 * (g >> 1) : 32 * g);
    // the scales of the epilogue, asked for ahead of everything
    const int64_t o = (int64_t)panel * PANEL + 64 * (g & 1) + 16 * (2 * q + (g >> 1)) + 4 * j;
    float sx = 1.0f, sw[4];
    if (MM::SCALED && wave == 0) {
        sx = s_x[live ? n : 0];
#pragma unroll
        for (int e = 0; e < 4; ++e) sw[e] = s_w[o + e < O ? o + e : O - 1];
    }

    // stages of the row; workgroups start in 16 places of it (k_sparse_wide)
    const int P = (U + NU - 1) / NU, rot = (int)(blockIdx.x & 15) * P / 16, count = P > wave ? (P - wave + WAVES - 1) / WAVES : 0;
    typedef SlimStage<NS> Stage;
    auto load = [&](Stage& R, int i) __attribute__((always_inline)) {
        int p = wave + i * WAVES + rot;
        p = p < P ? p : p - P;
        const uint8_t *const v = vals + (uint32_t)p * V_STEP, *const m = meta + (uint32_t)p * I_STEP;
        const bool whole = !FUSED || 2 * p + 1 < U;    // a last super-unit by itself: no step 1, and zeros in u1's place in step 2
        R.a[0] = slim_load<ONCE>(v + v_raw);
        R.ix[0] = *reinterpret_cast<const int*>(m + i_raw);
        if constexpr (FUSED) {
            if (whole) {
                R.a[1] = slim_load<ONCE>(v + 12288 + v_raw);
                R.ix[1] = *reinterpret_cast<const int*>(m + 3072 + i_raw);
                R.a[2] = slim_load<ONCE>(v + v_mid);
                R.ix[2] = *reinterpret_cast<const int*>(m + i_mid);
            } else {
                R.a[1] = R.a[2] = v4i{0, 0, 0, 0};
                R.ix[1] = R.ix[2] = 0;
                if (g < 2) {
                    R.a[2] = slim_load<ONCE>(v + v_mid);
                    R.ix[2] = *reinterpret_cast<const int*>(m + i_mid);
                }
            }
        }
        if (FUSED && !whole) R.raw[NU - 1] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
        if (live) {
            const v4i* s = reinterpret_cast<const v4i*>(x + (int64_t)p * X_STEP);
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (u == 0 || whole) {
                    const v4i lo = s[8 * u], hi = s[8 * u + 1];
                    R.raw[u] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                }
        }
    };
    typename MM::acc16_t acc = {0, 0, 0, 0};
    auto multiply = [&](const Stage& R) __attribute__((always_inline)) {
        acc = MM::sparse16(R.a[0], R.raw[0], acc, R.ix[0]);
        if constexpr (FUSED) {
            acc = MM::sparse16(R.a[1], R.raw[1], acc, R.ix[1]);
            v8i mid;                                   // middle windows of four blocks of each super-unit: see gemm_fused.hip
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if constexpr (MM::ES == 1) mid[4 * s + k] = (int)__builtin_amdgcn_alignbyte((uint32_t)R.raw[s][2 * k + 1], (uint32_t)R.raw[s][2 * k], 2);
                    else mid[4 * s + k] = R.raw[s][4 * (k >> 1) + 1 + (k & 1)];
                }
            acc = MM::sparse16(R.a[2], mid, acc, R.ix[2]);
        }
    };
    Stage st[D];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int s = 0; s < NU; ++s) st[d].raw[s] = v8i{0, 0, 0, 0, 0, 0, 0, 0};        // lanes without a token keep zeros
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < count) load(st[d], d);
    int i = 0;
    for (; i + 2 * D <= count; i += D)
#pragma unroll
        for (int d = 0; d < D; ++d) { multiply(st[d]); load(st[d], i + d + D); }
    for (; i < count; i += D)
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (i + d < count) {
                multiply(st[d]);
                if (i + d + D < count) load(st[d], i + d + D);
            }

    // the wavefronts' sums, added in their order by the first
    if (wave > 0) red[(wave - 1) * 64 + lane] = __builtin_bit_cast(v4i, acc);
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 1; w < WAVES; ++w) acc += __builtin_bit_cast(typename MM::acc16_t, red[(w - 1) * 64 + lane]);
    if (live && o < O) store_quad4<MM::SCALED>(acc, sx, sw, Y, ldy, O, o, n);
}

}  // namespace ss

using namespace ss;

template <int DT, bool FUSED>
static ss_status launch_slim(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U,
                             int64_t ldxb, void* Y, int64_t ldy, hipStream_t stream)
{
    const unsigned grid = (unsigned)((O + PANEL - 1) / PANEL * SLIM_PARTS);
    const bool once = weights_stream(O, (int64_t)U * (FUSED ? 3 : 2) * FRAG_KB, CACHED_BYTES);
    hipLaunchKernelGGL((once ? k_sparse_slim<DT, FUSED, true> : k_sparse_slim<DT, FUSED, false>), dim3(grid), dim3(64 * SLIM_WAVES), 0, stream,
                       static_cast<const uint8_t*>(Xq), s_x, static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U, ldxb,
                       static_cast<uint16_t*>(Y), ldy);
    return launch_status();
}

namespace ss {

ss_status launch_sparse_slim(bool fused, const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream)
{
#define SS_SL(DT) return fused ? launch_slim<DT, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream) \
                               : launch_slim<DT, false>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream)
    switch (dtype) {
    case SS_I8: SS_SL(SS_I8);
    case SS_FP8_E4M3: SS_SL(SS_FP8_E4M3);
    case SS_BF16: SS_SL(SS_BF16);
    case SS_FP16: SS_SL(SS_FP16);
    }
#undef SS_SL
    return SS_ERR_DTYPE;
}

}  // namespace ss
