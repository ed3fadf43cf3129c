// Sparse GEMMs of up to 16 tokens with a workgroup for every 16 output channels.
#include "ss_common.h"
#include "packed_layout.h"
#include "mma_types.h"
#include "device_info.h"

namespace ss {

#ifndef SLIM_W
#define SLIM_W 8
#endif
#ifndef SLIM_D
#define SLIM_D 3
#endif

constexpr int SLIM_PARTS = 8;                         // workgroups per panel

// What a wavefront holds of one stage of its k range, NS matrix-instruction steps of 128 lifted bytes: FUSED a pair of super-units (three steps),
// otherwise one unit (one step)
template <int NS, int TG> struct SlimStage { v4i a[NS]; int ix[NS]; v8i raw[TG][NS == 3 ? 2 : 1]; };

template <bool ONCE> __device__ inline v4i slim_load(const uint8_t* p)
{
    if constexpr (ONCE) return __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
    else return *reinterpret_cast<const v4i*>(p);
}

template <int DT, int TG, bool FUSED, bool ONCE, int WAVES, int D>
__global__ __launch_bounds__(64 * WAVES) void k_sparse_slim(const uint8_t* __restrict__ Xq, const float* __restrict__ s_x, const uint8_t* __restrict__ w_vals,
                                                            const uint8_t* __restrict__ w_meta, const float* __restrict__ s_w, int64_t M, int64_t O, int U,
                                                            int64_t ldxb, uint16_t* __restrict__ Y, int64_t ldy)
{
    typedef Mma<DT> MM;
    constexpr int NS = FUSED ? 3 : 1, NU = FUSED ? 2 : 1;
    constexpr uint32_t V_STEP = FUSED ? 24576 : 8192, I_STEP = V_STEP / 4, X_STEP = NU * KSTEP;
    __shared__ __attribute__((aligned(16))) v4i red[(WAVES - 1) * TG * 64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 15, g = lane >> 4;
    const int item = xcd_run(blockIdx.x, gridDim.x), panel = item / SLIM_PARTS, j = item & 7;
    const int row = 4 * j + (n & 3), frag = n >> 2;
    const uint8_t* const vals = w_vals + (int64_t)panel * U * (FUSED ? 12288 : 8192);
    const uint8_t* const meta = w_meta + (int64_t)panel * U * (FUSED ? 3072 : 2048);
    const uint32_t at = frag * 64 + row + 32 * (g >> 1), at_mid = frag * 64 + row + 32 * (g & 1);
    const uint32_t v_raw = (g & 1) * 4096 + at * 16, v_mid = (2 + 3 * (g >> 1)) * 4096 + at_mid * 16;
    const uint32_t i_raw = (g & 1) * 1024 + (row + 32 * (g >> 1)) * 16 + frag * 4, i_mid = (2 + 3 * (g >> 1)) * 1024 + (row + 32 * (g & 1)) * 16 + frag * 4;
    const uint8_t* x[TG];
    bool live[TG];
#pragma unroll
    for (int t = 0; t < TG; ++t) {
        const int64_t tok = 16 * t + n;
        live[t] = tok < M;
        x[t] = Xq + (live[t] ? tok : 0) * ldxb + (FUSED ? 64 * (g & 1) + 32 * (g >> 1) : 32 * g);
    }
    // the scales of the epilogue, asked for ahead of everything
    const int64_t o = (int64_t)panel * PANEL + 64 * (j & 1) + 16 * g + 4 * (j >> 1);
    float sx[TG], sw[4];
    if (MM::SCALED && wave == 0) {
#pragma unroll
        for (int t = 0; t < TG; ++t) sx[t] = s_x[live[t] ? 16 * t + n : 0];
#pragma unroll
        for (int e = 0; e < 4; ++e) sw[e] = s_w[o + e < O ? o + e : O - 1];
    }

    const int P = (U + NU - 1) / NU, rot = (int)(blockIdx.x & 15) * P / 16, count = P > wave ? (P - wave + WAVES - 1) / WAVES : 0;
    typedef SlimStage<NS, TG> Stage;
    auto load = [&](Stage& R, int i) __attribute__((always_inline)) {
        int p = wave + i * WAVES + rot;
        p = p < P ? p : p - P;
        const uint8_t *const v = vals + (uint32_t)p * V_STEP, *const m = meta + (uint32_t)p * I_STEP;
        const bool whole = !FUSED || 2 * p + 1 < U;
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
#pragma unroll
        for (int t = 0; t < TG; ++t) {
            if (live[t]) {
                const v4i* s = reinterpret_cast<const v4i*>(x[t] + (int64_t)p * X_STEP);
                const v4i lo = s[0], hi = s[1];
                R.raw[t][0] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                if (FUSED && whole) {
                    const v4i lo1 = s[8], hi1 = s[9];
                    R.raw[t][NU - 1] = v8i{lo1[0], lo1[1], lo1[2], lo1[3], hi1[0], hi1[1], hi1[2], hi1[3]};
                }
            }
            if (FUSED && !whole) R.raw[t][NU - 1] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
        }
    };
    typename MM::acc16_t acc[TG];
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] = 0;
    auto multiply = [&](const Stage& R) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < TG; ++t) {
            acc[t] = MM::sparse16(R.a[0], R.raw[t][0], acc[t], R.ix[0]);
            if constexpr (FUSED) {
                acc[t] = MM::sparse16(R.a[1], R.raw[t][1], acc[t], R.ix[1]);
                v8i mid;                               // middle windows of four blocks of each super-unit: see gemm_fused.hip
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if constexpr (MM::ES == 1) mid[4 * s + k] = (int)__builtin_amdgcn_alignbyte((uint32_t)R.raw[t][s][2 * k + 1], (uint32_t)R.raw[t][s][2 * k], 2);
                        else mid[4 * s + k] = R.raw[t][s][4 * (k >> 1) + 1 + (k & 1)];
                    }
                acc[t] = MM::sparse16(R.a[2], mid, acc[t], R.ix[2]);
            }
        }
    };
    Stage st[D];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
            for (int s = 0; s < NU; ++s) st[d].raw[t][s] = v8i{0, 0, 0, 0, 0, 0, 0, 0};     // lanes without a token keep zeros
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
    if (wave > 0) {
#pragma unroll
        for (int t = 0; t < TG; ++t) red[((wave - 1) * TG + t) * 64 + lane] = __builtin_bit_cast(v4i, acc[t]);
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 1; w < WAVES; ++w)
#pragma unroll
        for (int t = 0; t < TG; ++t) acc[t] += __builtin_bit_cast(typename MM::acc16_t, red[((w - 1) * TG + t) * 64 + lane]);
    if (o < O)
#pragma unroll
        for (int t = 0; t < TG; ++t)
            if (live[t]) store_quad4<MM::SCALED>(acc[t], sx[t], sw, Y, ldy, O, o, 16 * t + n);
}

}  // namespace ss

using namespace ss;

template <int DT, int TG, bool FUSED>
static ss_status launch_slim_tg(const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O, int U,
                                int64_t ldxb, void* Y, int64_t ldy, hipStream_t stream)
{
    const unsigned grid = (unsigned)((O + PANEL - 1) / PANEL * SLIM_PARTS);
    const bool once = weights_stream(O, (int64_t)U * (FUSED ? 3 : 2) * FRAG_KB, CACHED_BYTES);
#define SS_SLIM(ONCE) hipLaunchKernelGGL((k_sparse_slim<DT, TG, FUSED, ONCE, SLIM_W, SLIM_D * (FUSED ? 1 : 2)>), dim3(grid), dim3(64 * SLIM_W), 0, stream, static_cast<const uint8_t*>(Xq), s_x, \
                       static_cast<const uint8_t*>(w_vals), static_cast<const uint8_t*>(w_meta), s_w, M, O, U, ldxb, static_cast<uint16_t*>(Y), ldy)
    if (once) SS_SLIM(true);
    else SS_SLIM(false);
#undef SS_SLIM
    return launch_status();
}

namespace ss {

ss_status launch_sparse_slim(bool fused, const void* Xq, const float* s_x, const void* w_vals, const void* w_meta, const float* s_w, int64_t M, int64_t O,
                             int U, int64_t ldxb, ss_dtype dtype, void* Y, int64_t ldy, hipStream_t stream)
{
#define SS_SL(DT) if (M > 16) return fused ? launch_slim_tg<DT, 2, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream) \
                                           : launch_slim_tg<DT, 2, false>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream); \
                  return fused ? launch_slim_tg<DT, 1, true>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream) \
                               : launch_slim_tg<DT, 1, false>(Xq, s_x, w_vals, w_meta, s_w, M, O, U, ldxb, Y, ldy, stream)
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
