// act_lift_quant: fused per-token quantisation + activation lifting (Alg. 1).
//
// The kernel streams a row through one workgroup: the row is read from HBM once, kept in
// registers while the wavefronts reduce the absmax, quantised element-wise into LDS, and the
// lifted windows are then gathered from LDS so that every source element is quantised once
// and every output store is a coalesced 16-byte vector.  HBM traffic per token is therefore
// the algorithmic minimum: K input elements in, K' output elements + one scale out.
#include "ss_common.h"
#include "quant_common.h"
#include "device_info.h"
#include <type_traits>

namespace ss {

// MAXV > 0: vector loads, row kept in registers.  MAXV == 0: scalar loads, second pass re-reads the
// row (rows too long for the registers of a workgroup, short ones off a line: launch_lift).  Long rows take more
// threads per token rather than more registers per thread: the loads of a token are all in
// flight at once either way, but fewer registers leave room for more tokens per compute unit.
// RAGGED: the rows start off a 16-byte line or end within one.  The 16-byte lines that are the row's alone are
// loaded as they lie, the up to 2 (IV::N - 1) elements ahead of and behind them by one thread each, the last of the
// workgroup; element k has its code in LDS at off + k, off being the row's offset from its first line, and the gather shifts
// accordingly.  (One thread for all that a line has of the row, element by element: bf16 to fp16, 8192 x 2051 17.7 us, like this 12.8; 2048 x 8195 14.4 and 10.6.)
template <typename TIN, int OUT, int MAXV, int THREADS, bool RAGGED, bool THROUGH>
__global__ __launch_bounds__(THREADS) void k_act_lift_quant(const TIN* __restrict__ X, int64_t ldx, int K, int N,
                                                                uint8_t* __restrict__ XL, float* __restrict__ s_x, int Kp, int Kz, uint32_t inv_nw1)
{
    // Kp: stored width of a lifted row (whole 128-byte units); Kz >= n_g * 2N + 8 / ES: elements
    // of the quantised row held in LDS, those at and beyond K being zero (zero-completed last block)
    constexpr int ES = OUT >= 2 ? 2 : 1;                 // output element bytes
    extern __shared__ uint32_t lds[];                     // Kz * ES bytes
    __shared__ float red[THREADS / 64];
    const int64_t m = blockIdx.x;
    const TIN* x = X + m * ldx;
    const int t = threadIdx.x;
    auto put = [&](auto* p, auto x) __attribute__((always_inline)) { if constexpr (THROUGH) store_through(p, x); else *p = x; };
    typedef InVec<TIN> IV;
    typename IV::V v[MAXV > 0 ? MAXV : 1];
    const int off = RAGGED ? (int)(((uintptr_t)x / sizeof(TIN)) % IV::N) : 0;
    const int head = RAGGED ? (IV::N - off) % IV::N : 0;      // elements ahead of the first whole line (the rows are longer)
    const int nvec = (K - head) / IV::N, body = head + nvec * IV::N;  // whole lines, and the first element behind them
    // the element at one of the row's two ends that this thread takes, if any
    const int e = THREADS - 1 - t, edge = !RAGGED ? K : e < head ? e : body + e - head;
    float at_edge = 0.0f;

    // ---- pass 1: absmax (Alg. 1, dynamic quantisation scale)
    float amax = 0.0f;
    if constexpr (MAXV > 0) {
        if (edge < K) at_edge = load_scalar(x + edge);
        const typename IV::V* xv = reinterpret_cast<const typename IV::V*>(x + head);
#pragma unroll
        for (int i = 0; i < MAXV; ++i) {
            const int idx = t + i * THREADS;
            if (idx < nvec) {
                v[i] = xv[idx];
                if constexpr (OUT < 2) {
                    float f[IV::N]; IV::unpack(v[i], f);
#pragma unroll
                    for (int k = 0; k < IV::N; ++k) amax = fmaxf(amax, fabsf(f[k]));
                }
            }
        }
        if constexpr (RAGGED) amax = fmaxf(amax, fabsf(at_edge));
    } else if constexpr (OUT < 2) {
        for (int k = t; k < K; k += THREADS) amax = fmaxf(amax, fabsf(load_scalar(x + k)));
    }
    float r = 0.0f;
    if constexpr (OUT < 2) {
        amax = block_absmax<THREADS>(amax, red);
        constexpr float QMAX = OUT == 0 ? 127.0f : 448.0f;
        float s = 1.0f;
        if (amax > 0.0f) { r = QMAX / amax; s = amax / QMAX; }
        if (t == 0) s_x[m] = s;
    }

    // ---- N = 2 from registers: plain quantisation has no windows to gather, so the quantised vectors go straight to
    // global memory (4 or 8 bytes per lane, contiguous across the wavefront) without the round trip through LDS
    if constexpr (MAXV > 0 && !RAGGED) {
        if (N == 2) {
            constexpr int OW = IV::N * ES / 4;           // output dwords per input vector: 1 (fp32 -> 8 bit), 2, 2 or 4
            uint32_t* out32 = reinterpret_cast<uint32_t*>(XL + m * (int64_t)Kp * ES);
#pragma unroll
            for (int i = 0; i < MAXV; ++i) {
                const int idx = t + i * THREADS;
                if (idx < nvec) {
                    float f[IV::N]; IV::unpack(v[i], f);
                    uint32_t w[OW];
#pragma unroll
                    for (int k = 0; k < OW; ++k) {
                        if constexpr (ES == 1)
                            w[k] = quant4<OUT>(f[4 * k], f[4 * k + 1], f[4 * k + 2], f[4 * k + 3], r);
                        else
                            w[k] = quant1<OUT>(f[2 * k], r) | (quant1<OUT>(f[2 * k + 1], r) << 16);
                    }
                    if constexpr (OW == 1) out32[idx] = w[0];
                    else if constexpr (OW == 2) put(reinterpret_cast<uint2*>(out32) + idx, make_uint2(w[0], w[1]));
                    else put(reinterpret_cast<uint4*>(out32) + idx, make_uint4(w[0], w[1], w[2], w[3]));
                }
            }
            // zero padding of the stored width (K is a whole number of vectors here, so of dwords too)
            for (int k = K * ES / 4 + t; k < Kp * ES / 4; k += THREADS) out32[k] = 0u;
            return;
        }
    }

    // ---- pass 2a: quantise every source element once, into LDS
    typedef std::conditional_t<ES == 1, uint8_t, uint16_t> code_t;
    code_t* const codes = reinterpret_cast<code_t*>(lds);
    if constexpr (MAXV > 0) {
        if (edge < K) codes[off + edge] = (code_t)quant1<OUT>(at_edge, r);
#pragma unroll
        for (int i = 0; i < MAXV; ++i) {
            const int idx = t + i * THREADS, line = idx + (head > 0);
            if (idx < nvec) {
                float f[IV::N]; IV::unpack(v[i], f);
                if constexpr (ES == 1) {
#pragma unroll
                    for (int w = 0; w < IV::N / 4; ++w) lds[line * (IV::N / 4) + w] = quant4<OUT>(f[4 * w], f[4 * w + 1], f[4 * w + 2], f[4 * w + 3], r);
                } else {
#pragma unroll
                    for (int w = 0; w < IV::N / 2; ++w)
                        lds[line * (IV::N / 2) + w] = quant1<OUT>(f[2 * w], r) | (quant1<OUT>(f[2 * w + 1], r) << 16);
                }
            }
        }
    } else {
        for (int k = t; k < K; k += THREADS) codes[k] = (code_t)quant1<OUT>(load_scalar(x + k), r);
    }
    for (int k = K + t; k < Kz; k += THREADS) codes[off + k] = 0;
    __syncthreads();

    // ---- pass 2b: output-oriented gather of the lifted windows (window j reads b = 2N g + 2 l);
    // windows at and beyond n_w = n_g (N-1) are the zero padding of the last 128-byte unit
    const int nw1 = N - 1;
    // j / nw1 by its reciprocal ceil(2^32 / nw1): exact for j < 2^32 / nw1 (j < 2^16 here)
    auto block_of = [&](int j) { return nw1 == 1 ? j : (int)__umulhi((uint32_t)j, inv_nw1); };
    const int nwin = Kp / 4;
    const int ng = (K + 2 * N - 1) / (2 * N);
    uint4* out = reinterpret_cast<uint4*>(XL + m * (int64_t)Kp * ES);
    if constexpr (ES == 1) {
        for (int c = t; c < nwin / 4; c += THREADS) {
            int j = 4 * c, g = block_of(j), l = j - g * nw1;
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w[i] = 0;
                if (g < ng) {
                    const int b = 2 * N * g + 2 * l + off;
                    const uint32_t lo = lds[b >> 2], hi = lds[(b >> 2) + 1];
                    if constexpr (RAGGED) w[i] = __builtin_amdgcn_alignbyte(hi, lo, (uint32_t)b & 3);
                    else w[i] = (b & 2) ? ((lo >> 16) | (hi << 16)) : lo;
                }
                if (++l == nw1) { l = 0; ++g; }
            }
            put(out + c, make_uint4(w[0], w[1], w[2], w[3]));
        }
    } else {
        // 16-bit elements: a window is 8 bytes = elements b..b+3: two aligned dwords, or, b odd (RAGGED only), parts of three
        for (int c = t; c < nwin / 2; c += THREADS) {
            int j = 2 * c, g = block_of(j), l = j - g * nw1;
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                w[2 * i] = 0; w[2 * i + 1] = 0;
                if (g < ng) {
                    const int b = 2 * N * g + 2 * l + off;
                    w[2 * i] = lds[b >> 1]; w[2 * i + 1] = lds[(b >> 1) + 1];
                    if constexpr (RAGGED) {
                        const uint32_t sh = 2 * ((uint32_t)b & 1), w2 = lds[(b >> 1) + 2];
                        w[2 * i] = __builtin_amdgcn_alignbyte(w[2 * i + 1], w[2 * i], sh);
                        w[2 * i + 1] = __builtin_amdgcn_alignbyte(w2, w[2 * i + 1], sh);
                    }
                }
                if (++l == nw1) { l = 0; ++g; }
            }
            put(out + c, make_uint4(w[0], w[1], w[2], w[3]));
        }
    }
}

// elements of the quantised row kept in LDS: whole blocks plus 8 bytes that the gather may read
// past the last window, rounded to whole dwords
static inline int64_t lift_lds_elems(int64_t K, int N, int es) { return (n_groups(K, N) * 2 * N * es + 8 + 3) / 4 * 4 / es; }

template <typename TIN, int OUT>
static ss_status launch_lift(const void* X, int64_t M, int64_t K, int64_t ldx, int N, void* XL, float* s_x, hipStream_t st)
{
    typedef InVec<TIN> IV;
    const int ES = OUT >= 2 ? 2 : 1;
    const int Kp = (int)lifted_ld(K, N, ES);
    const int Kz = (int)lift_lds_elems(K, N, ES);
    const bool line_ok = (K % IV::N == 0) && (ldx % IV::N == 0) && (((uintptr_t)X & 15) == 0);
    const bool through = lift_through(ES, IV::N, M, Kp, N);
    const bool element_ok = (uintptr_t)X % sizeof(TIN) == 0;
    // a ragged row: up to IV::N - 1 codes more in LDS, ahead of it in its first line
    const int64_t nvec = K / IV::N;                           // whole 16-byte vectors per row, at most
    const size_t lds_bytes = (size_t)Kz * ES, ragged_bytes = lds_bytes + IV::N * ES;
    dim3 grid((unsigned)M);
    const uint32_t inv = N > 2 ? (uint32_t)(((1ull << 32) + N - 2) / (N - 1)) : 0u;
    const TIN* x = static_cast<const TIN*>(X);
    uint8_t* xl = static_cast<uint8_t*>(XL);
#define SS_LQ(MAXV, T, RAGGED) \
    hipLaunchKernelGGL((through ? k_act_lift_quant<TIN, OUT, MAXV, T, RAGGED, (OUT < 2)> : k_act_lift_quant<TIN, OUT, MAXV, T, RAGGED, false>), grid, dim3(T), \
                       RAGGED ? ragged_bytes : lds_bytes, st, x, ldx, (int)K, N, xl, s_x, Kp, Kz, inv)
#define SS_LQ_ROWS(RAGGED)                             \
    if (spread && nvec <= 2 * 512) SS_LQ(2, 512, RAGGED);        \
    else if (spread && nvec <= 2 * 1024) SS_LQ(2, 1024, RAGGED); \
    else if (nvec <= 4 * 256) SS_LQ(4, 256, RAGGED);   \
    else if (nvec <= 4 * 512) SS_LQ(4, 512, RAGGED);   \
    else if (nvec <= 5 * 1024) SS_LQ(5, 1024, RAGGED); \
    else if (nvec <= 10 * 1024) SS_LQ(10, 1024, RAGGED); \
    else SS_LQ(20, 1024, RAGGED);
    // Rows off a line: whole lines against scalar loads, time, M = 1 .. 30000, N = 2 .. 8: 8-bit codes (two passes over the row) of 37 to 195
    // elements 0.91 .. 1.22, 257 to 771 0.55 .. 1.07, 1003 and more 0.18 .. 1.06 (8192 x 4099 fp32 to fp8 0.46); 16-bit codes (one pass) of 37 to
    // 385 elements 0.92 .. 1.76, 515 to 771 0.73 .. 1.13, 1003 and more 0.37 .. 1.10.  Where the rows are short, a thread has an element or two.
    // Where every token has a compute unit to itself, a row is a chain of latencies: twice the threads, half the work of each (rows of more
    // than 256 vectors, two for a thread; time over four for a thread, M = 1 .. 256, five type and pattern forms: K = 3584 and 4096 0.81 .. 1.00, 8192 0.81 .. 0.99,
    // 14336 0.88 .. 1.01; four layers of a block: fp8 lifted M = 64 85.1 -> 81.2 us, INT8 M = 1 65.9 -> 64.6, M = 256 127.4 -> 125.7).
    // With more tokens than compute units rows of more than 512 threads lose (M = 300: up to 1.06).
    const bool spread = M <= cu_count() && nvec > 256;
    const bool few = !line_ok && K <= (OUT < 2 ? 256 : 512);
    // 64: the kernel's small reduction buffer
    if (!element_ok || few || nvec > 20 * 1024 || (!line_ok && ragged_bytes + 64 > 64 * 1024)) SS_LQ(0, 256, false);
    else if (line_ok) { SS_LQ_ROWS(false) }
    else { SS_LQ_ROWS(true) }
#undef SS_LQ_ROWS
#undef SS_LQ
    return launch_status();
}

}  // namespace ss

using namespace ss;

extern "C" int64_t slide_lifted_k(int64_t K, int N)
{
    if (!valid_N(N) || K <= 0 || K > (1 << 24)) return -1;
    return lifted_k(K, N);
}

extern "C" int64_t slide_lifted_ld(int64_t K, int N, ss_dtype dtype)
{
    if (!valid_N(N) || K <= 0 || K > (1 << 24) || !valid_dtype(dtype)) return -1;
    return lifted_ld(K, N, elem_size(dtype));
}

extern "C" ss_status act_lift_quant(const void* X, ss_act_dtype in_dtype, int64_t M, int64_t K, int64_t ldx, int N,
                                    ss_dtype out, void* X_lifted, float* s_x, void* stream)
{
    if (!valid_N(N)) return SS_ERR_BAD_PATTERN_N;
    if (M < 0 || K <= 0 || ldx < K || K > (1 << 24) || M > 0x7FFFFFFF) return SS_ERR_SHAPE;
    if (in_dtype != SS_IN_F32 && in_dtype != SS_IN_BF16) return SS_ERR_DTYPE;
    if (!valid_dtype(out)) return SS_ERR_DTYPE;
    // the quantised row and the kernel's small reduction buffer (at most 64 bytes) must fit in 64 KiB of LDS
    if ((size_t)lift_lds_elems(K, N, elem_size(out)) * elem_size(out) + 64 > 64 * 1024) return SS_ERR_SHAPE;
    if (M == 0) return SS_OK;
    if (!X || !X_lifted || (!unscaled(out) && !s_x)) return SS_ERR_NULL;
    if ((uintptr_t)X_lifted & 15) return SS_ERR_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (in_dtype == SS_IN_F32) {
        if (out == SS_I8) return launch_lift<float, 0>(X, M, K, ldx, N, X_lifted, s_x, st);
        if (out == SS_FP8_E4M3) return launch_lift<float, 1>(X, M, K, ldx, N, X_lifted, s_x, st);
        if (out == SS_BF16) return launch_lift<float, 2>(X, M, K, ldx, N, X_lifted, s_x, st);
        return launch_lift<float, 3>(X, M, K, ldx, N, X_lifted, s_x, st);
    }
    if (out == SS_I8) return launch_lift<uint16_t, 0>(X, M, K, ldx, N, X_lifted, s_x, st);
    if (out == SS_FP8_E4M3) return launch_lift<uint16_t, 1>(X, M, K, ldx, N, X_lifted, s_x, st);
    if (out == SS_BF16) return launch_lift<uint16_t, 2>(X, M, K, ldx, N, X_lifted, s_x, st);
    return launch_lift<uint16_t, 3>(X, M, K, ldx, N, X_lifted, s_x, st);
}
