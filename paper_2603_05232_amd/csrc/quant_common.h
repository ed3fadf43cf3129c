// Pieces shared by the two quantisation kernels (lift_quant.hip, prune_quant.hip).
#pragma once
#include "ss_common.h"

namespace ss {

template <typename T> struct InVec;
template <> struct InVec<float> {
    static constexpr int N = 4; typedef float4 V;
    __device__ static void unpack(const V& v, float* f) { f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w; }
};
template <> struct InVec<uint16_t> {          // bf16 bits
    static constexpr int N = 8; typedef uint4 V;
    __device__ static void unpack(const V& v, float* f)
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) { f[2 * i] = __uint_as_float(w[i] << 16); f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u); }
    }
};
__device__ inline float load_scalar(const float* p) { return *p; }
__device__ inline float load_scalar(const uint16_t* p) { return bf16_bits_to_f32(*p); }

// Whether act_lift_quant stores its M rows of row_bytes (elements of es bytes, from input vectors of `vec` elements) through the L2
// (store_through).  A GEMM of few channels behind it is short and waits for its tokens, which plain stores leave nearer; rows of 2 to 5 KB are the worst.
// Time over plain stores, quantiser and a GEMM of 128 to 12000 channels, 9900 calls, by rows and MB of them:
//   up to 1792 bytes     lifted 4 .. 16 0.86 .. 1.05 (mean 0.94), unlifted 0.89 .. 1.03 (0.95); more 0.96 .. 1.05
//   1793 .. 5631 bytes   lifted 4 .. 8 0.88 .. 1.10 (0.95); unlifted of 3072 bytes and more 0.93 .. 1.04 (0.97), shorter 0.90 .. 1.27 (INT8 2399 x 2048, 1024
//                        channels 22.4 -> 25.9 us); 8 .. 32 with up to 1024 channels lifted 0.90 .. 1.16 (1.01), unlifted 0.94 .. 1.19 (1.03), with more
//                        0.92 .. 1.07 (0.99)
//   5632 bytes and more  lifted 4 .. 8 0.92 .. 1.02 (0.96), 8 .. 16 0.90 .. 1.04 (0.97), 16 .. 32 0.93 .. 1.06 (0.99); unlifted 0.93 .. 1.03 (0.98),
//                        0.95 .. 1.05 (0.99), 0.95 .. 1.04 (0.99)
//   fp32 to 8 bits unlifted, stores of four bytes, 0.98 .. 1.05; 16-bit codes 0.95 .. 1.18 without a line to draw; the kernel alone below 1 MB 1.03 .. 1.06,
//   1 to 4 MB 0.86 .. 1.05
inline bool lift_through(int es, int vec, int64_t M, int64_t row_bytes, int N)
{
    const bool is_short = row_bytes <= 1792, is_long = row_bytes >= 5632;
    if (es != 1 || (N == 2 && (vec != 8 || (!is_short && row_bytes < 3072)))) return false;
    return M * row_bytes >= (4 << 20) && M * row_bytes <= (is_short ? 16 << 20 : is_long ? 32 << 20 : 8 << 20);
}

template <int THREADS> __device__ inline float block_absmax(float v, float* red)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    float m = red[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) m = fmaxf(m, red[w]);
    return m;
}

// quantise one element: OUT 0 = int8, 1 = fp8 e4m3, 2 = bf16 (no scale), 3 = half (no scale)
template <int OUT> __device__ inline uint32_t quant1(float x, float r)
{
    if constexpr (OUT == 0) {
        float q = rintf(x * r);
        q = fminf(fmaxf(q, -127.0f), 127.0f);
        return (uint32_t)(int)q & 0xFFu;
    } else if constexpr (OUT == 1) {
        float q = x * r;
        q = fminf(fmaxf(q, -448.0f), 448.0f);
        return f32_to_e4m3(q);
    } else if constexpr (OUT == 2) {
        return f32_to_bf16_bits(x);
    } else {
        return f32_to_f16_bits(x);
    }
}

// The same codes with fewer instructions, for kernels where the conversion counts: only the low byte (OUT < 2) or half
// of the result is meaningful.  INT8: adding 1.5 * 2^23 to the clamped product rounds it to nearest even and leaves its
// two's complement in the low mantissa bits (clamping before or after the rounding is the same, 127 being an integer).
// FP8: the conversion instruction (e4m3fn, nearest even) agrees with f32_to_e4m3 on every float of [-448, 448].
template <int OUT> __device__ inline uint32_t quant_bits(float x, float r)
{
    if constexpr (OUT == 0) return __float_as_uint(fminf(fmaxf(x * r, -127.0f), 127.0f) + 12582912.0f);
    else if constexpr (OUT == 1) return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(fminf(fmaxf(x * r, -448.0f), 448.0f), 0.0f, 0, false);
    else return quant1<OUT>(x, r);
}
// the low bytes of four words
__device__ inline uint32_t pack_bytes(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3)
{
    return __builtin_amdgcn_perm(b1, b0, 0x0C0C0400u) | __builtin_amdgcn_perm(b3, b2, 0x04000C0Cu);
}

// four codes in a word (8-bit types)
// (rates: bf16 in, fp8 out, 2048 x 4096 without lifting 10.9 -> 7.6 us, 2048 x 14336 28.2 -> 19.5)
template <int OUT> __device__ inline uint32_t quant4(float x0, float x1, float x2, float x3, float r)
{
    if constexpr (OUT == 1) {
        auto c = [r](float x) { return fminf(fmaxf(x * r, -448.0f), 448.0f); };
        const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(c(x0), c(x1), 0, false);
        return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c(x2), c(x3), lo, true);
    } else return pack_bytes(quant_bits<OUT>(x0, r), quant_bits<OUT>(x1, r), quant_bits<OUT>(x2, r), quant_bits<OUT>(x3, r));
}

}  // namespace ss
