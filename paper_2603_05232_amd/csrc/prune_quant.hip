// slide_prune_quant: offline (2N-2):2N magnitude pruning + per-channel quantisation (Sec. 4.1, App. E; Alg. 1 pass 1).
#include "ss_common.h"
#include "quant_common.h"
#include <type_traits>

namespace ss {

// One block g of a row, element by element.  The two entries dropped are the last two in the order (|w| descending,
// index ascending); this form defines the result, also for blocks that hold a NaN.
template <typename TIN, int OUT>
__device__ inline void prune_block(const TIN* __restrict__ w, int K, int L, int g, float r, uint8_t* __restrict__ wq)
{
    constexpr int ES = OUT >= 2 ? 2 : 1;
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = (k < L && g * L + k < K) ? load_scalar(w + g * L + k) : 0.0f;
    int d1 = 0, d2 = -1;
    float m1 = fabsf(v[0]);
#pragma unroll
    for (int k = 1; k < 16; ++k) if (k < L && fabsf(v[k]) <= m1) { m1 = fabsf(v[k]); d1 = k; }
    float m2 = 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) if (k < L && k != d1 && (d2 < 0 || fabsf(v[k]) <= m2)) { m2 = fabsf(v[k]); d2 = k; }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (k < L && g * L + k < K) {
            const uint32_t q = (k == d1 || k == d2) ? 0u : quant1<OUT>(v[k], r);
            if constexpr (ES == 1) wq[g * L + k] = (uint8_t)q;
            else reinterpret_cast<uint16_t*>(wq)[g * L + k] = (uint16_t)q;
        }
    }
}

// ---- rows of whole 16-byte vectors ----------------------------------------------------------------------
// Bound by HBM (the row once in, its codes once out); what has to be kept small beside that is the vector arithmetic
// per weight.  One workgroup per row.  A thread's unit is the fewest whole 2N blocks that fill whole 16-byte vectors
// (6:8 from bf16: one block = one vector), so a block is never shared between threads, every load is a vector and a
// wavefront reads contiguous memory; the row stays in registers between the absmax and the pruning.  A unit per
// thread and load instead of a block per thread with one load per element (the kernel below): 37888 x 3584 bf16 -> INT8
// 398 -> 82 us.  Matrices that the memory-side cache does not hold are loaded non-temporally, since nobody reads
// them again: the codes, which the decomposition reads next, then find room there (82 -> 63 us, 6.5 TB/s; a matrix that it may hold 1.05 of
// the time).  Not where units are several vectors: they take several loads for a cache line, which would not be there any more for
// the second (fp32 14:16 of 8539 x 2048 with its decomposition 54 -> 78 us); nor for 2:4 (8192 x 4096 fp32 -> bf16 59.1 -> 60.9).
template <typename TIN, int N> struct PruneUnit {
    static constexpr int ESI = (int)sizeof(TIN);
    static constexpr int BLOCK = 2 * N * ESI;                                  // bytes of a block
    static constexpr int UB = BLOCK % 16 == 0 ? 1 : (2 * BLOCK) % 16 == 0 ? 2 : 4;   // blocks per unit
    static constexpr int CH = UB * BLOCK / 16;                                 // 16-byte vectors per unit
    static constexpr int E = UB * 2 * N;                                       // elements per unit
    static constexpr int MAXU = CH <= 2 ? 4 : 2;                               // units a thread holds in registers (16 .. 56 of them)
    static constexpr int MAX_THREADS = CH >= 5 ? 512 : 1024;                   // register-heavy units leave room for fewer
    template <int ES> static constexpr int OW = CH * (4 / ESI) * ES;           // output dwords per unit, of codes of ES bytes
    template <int ES> static constexpr int VW = OW<ES> % 4 == 0 ? 4 : OW<ES> % 2 == 0 ? 2 : 1;      // of one output store
    template <int ES> static constexpr bool MAY_THROUGH = ES == 1 && VW<ES> >= 2 && OW<ES> == VW<ES>;      // see launch_prune_rows
};

__device__ inline void unpack_word(uint32_t w, float* f, float) { f[0] = __uint_as_float(w); }
__device__ inline void unpack_word(uint32_t w, float* f, uint16_t) { f[0] = __uint_as_float(w << 16); f[1] = __uint_as_float(w & 0xFFFF0000u); }

template <typename TIN, int OUT, int N>
__global__ __launch_bounds__((PruneUnit<TIN, N>::MAX_THREADS)) void k_prune_rows(const TIN* __restrict__ W, int K, int nunits, uint8_t* __restrict__ Wq, float* __restrict__ s_w,
                                                     int vec_out, bool once, bool through)
{
    typedef PruneUnit<TIN, N> PU;
    constexpr int ES = OUT >= 2 ? 2 : 1, ESI = PU::ESI, CH = PU::CH, EPW = 4 / ESI, L = 2 * N;
    constexpr int CW = 4 * EPW * ES / 4;                  // output dwords per input vector
    constexpr int OW = PU::template OW<ES>, VW = PU::template VW<ES>;
    static_assert(OW == CH * CW, "output dwords per unit");
    __shared__ float red[PU::MAX_THREADS / 64];
    const int64_t o = blockIdx.x;
    const int t = threadIdx.x, T = blockDim.x;
    const uint4* w = reinterpret_cast<const uint4*>(W + o * (int64_t)K);
    const int nvec = K / (16 / ESI);
    uint32_t v[PU::MAXU][CH * 4];
    auto load_row = [&](auto once_c) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PU::MAXU; ++i) {
            const int u = t + i * T;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                uint4 x = make_uint4(0, 0, 0, 0);         // beyond the row: zeros complete the last block
                if (u < nunits && u * CH + c < nvec) x = decltype(once_c)::value ? load_once(w + u * CH + c) : w[u * CH + c];
                v[i][4 * c] = x.x; v[i][4 * c + 1] = x.y; v[i][4 * c + 2] = x.z; v[i][4 * c + 3] = x.w;
            }
        }
    };
    if (CH == 1 && N > 2 && once) load_row(std::true_type{});
    else load_row(std::false_type{});
    float r = 0.0f;
    if constexpr (OUT < 2) {
        float amax = 0.0f;
#pragma unroll
        for (int i = 0; i < PU::MAXU; ++i)
#pragma unroll
            for (int j = 0; j < CH * 4; ++j) {
                float f[EPW];
                unpack_word(v[i][j], f, TIN());
#pragma unroll
                for (int e = 0; e < EPW; ++e) amax = fmaxf(amax, fabsf(f[e]));
            }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        if (T > 64) {
            if ((t & 63) == 0) red[t >> 6] = amax;
            __syncthreads();
            for (int k = 0; k < T / 64; ++k) amax = fmaxf(amax, red[k]);
        }
        constexpr float QMAX = OUT == 0 ? 127.0f : 448.0f;   // the row maximum always survives pruning
        float s = 1.0f;
        if (amax > 0.0f) { r = QMAX / amax; s = amax / QMAX; }
        if (t == 0) s_w[o] = s;
    }
    uint32_t* const out = reinterpret_cast<uint32_t*>(Wq + o * (int64_t)K * ES);
    bool odd = false;
#pragma unroll
    for (int i = 0; i < PU::MAXU; ++i) {
        const int u = t + i * T;
        if (u >= nunits) continue;
        uint32_t code[PU::E];                             // low ES bytes count
#pragma unroll
        for (int b = 0; b < PU::UB; ++b) {
            float f[L];
            uint32_t key[L];
            uint32_t top = 0;
#pragma unroll
            for (int k = 0; k < L / EPW; ++k) unpack_word(v[i][(b * L) / EPW + k], f + k * EPW, TIN());
            // Two smallest keys.  bf16: |w| and, below it, the index counted down, so that keys are distinct and ties
            // drop the higher index first.  fp32: |w| alone.
            uint32_t m1 = 0xFFFFFFFFu, m2 = 0xFFFFFFFFu;
#pragma unroll
            for (int k = 0; k < L; ++k) {
                const uint32_t a = __float_as_uint(f[k]) & 0x7FFFFFFFu;
                key[k] = ESI == 2 ? a | (uint32_t)(L - 1 - k) : a;
                top = key[k] > top ? key[k] : top;
                const uint32_t hi = key[k] > m1 ? key[k] : m1;
                m2 = hi < m2 ? hi : m2;
                m1 = key[k] < m1 ? key[k] : m1;
            }
            bool drop[L];
            int below = 0;
#pragma unroll
            for (int k = 0; k < L; ++k) { drop[k] = key[k] <= m2; below += drop[k]; }
            // fp32, equal magnitudes at the border of the two: of those equal to the second smallest only the last ones go
            if (ESI == 4 && below != 2) {
                int room = 2;
#pragma unroll
                for (int k = 0; k < L; ++k) room -= key[k] < m2;
#pragma unroll
                for (int k = L - 1; k >= 0; --k) {
                    const bool last = key[k] == m2 && room > 0;
                    drop[k] = key[k] < m2 || last;
                    room -= last;
                }
            }
            odd = odd || top > (ESI == 2 ? 0x7F80000Fu : 0x7F800000u);       // a NaN
#pragma unroll
            for (int k = 0; k < L; ++k) {
                const uint32_t q = quant_bits<OUT>(f[k], r);
                code[b * L + k] = drop[k] ? 0u : q;
            }
        }
        uint32_t ow[OW];
#pragma unroll
        for (int k = 0; k < OW; ++k) {
            if constexpr (ES == 1) ow[k] = pack_bytes(code[4 * k], code[4 * k + 1], code[4 * k + 2], code[4 * k + 3]);
            else ow[k] = code[2 * k] | (code[2 * k + 1] << 16);
        }
        uint32_t* dst = out + (int64_t)u * OW;
        if (vec_out && (u + 1) * CH <= nvec) {
            auto put = [&](auto* p, auto x) __attribute__((always_inline)) {
                if constexpr (PU::template MAY_THROUGH<ES>) {
                    if (through) store_through(p, x);
                    else *p = x;
                } else *p = x;
            };
#pragma unroll
            for (int k = 0; k < OW / VW; ++k) {
                if constexpr (VW == 4) put(reinterpret_cast<uint4*>(dst) + k, make_uint4(ow[4 * k], ow[4 * k + 1], ow[4 * k + 2], ow[4 * k + 3]));
                else if constexpr (VW == 2) put(reinterpret_cast<uint2*>(dst) + k, make_uint2(ow[2 * k], ow[2 * k + 1]));
                else dst[k] = ow[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < OW; ++k)
                if (u * CH + k / CW < nvec) dst[k] = ow[k];
        }
    }
    if (odd)                                              // magnitude order by bits does not cover NaNs: those units again, literally
        for (int u = t; u < nunits; u += T)
            for (int g = u * PU::UB; g < (u + 1) * PU::UB && g * L < K; ++g)
                prune_block<TIN, OUT>(W + o * (int64_t)K, K, L, g, r, Wq + o * (int64_t)K * ES);
}

// ---- any row length and alignment -----------------------------------------------------------------------
// One workgroup per weight row, two passes over it; thread per 2N block in the second pass.
constexpr int PQ_THREADS = 256;
template <typename TIN, int OUT>
__global__ __launch_bounds__(PQ_THREADS) void k_prune_quant(const TIN* __restrict__ W, int K, int N, uint8_t* __restrict__ Wq,
                                                             float* __restrict__ s_w)
{
    constexpr int ES = OUT >= 2 ? 2 : 1;
    __shared__ float red[PQ_THREADS / 64];
    const int64_t o = blockIdx.x;
    const TIN* w = W + o * (int64_t)K;
    const int t = threadIdx.x;
    float r = 0.0f;
    if constexpr (OUT < 2) {
        float amax = 0.0f;
        for (int k = t; k < K; k += PQ_THREADS) amax = fmaxf(amax, fabsf(load_scalar(w + k)));
        amax = block_absmax<PQ_THREADS>(amax, red);   // the row maximum always survives pruning
        constexpr float QMAX = OUT == 0 ? 127.0f : 448.0f;
        float s = 1.0f;
        if (amax > 0.0f) { r = QMAX / amax; s = amax / QMAX; }
        if (t == 0) s_w[o] = s;
    }
    const int L = 2 * N, ng = (K + L - 1) / L;            // a partial last block is completed with zeros
    for (int g = t; g < ng; g += PQ_THREADS) prune_block<TIN, OUT>(w, K, L, g, r, Wq + o * (int64_t)K * ES);
}

}  // namespace ss

using namespace ss;

template <typename TIN, int OUT, int N>
static bool launch_prune_rows(const TIN* W, int64_t O, int64_t K, uint8_t* Wq, float* s_w, hipStream_t st)
{
    typedef PruneUnit<TIN, N> PU;
    constexpr int ES = OUT >= 2 ? 2 : 1;
    // Rows of whole 16-byte vectors that fit the registers of a workgroup (up to 16384 .. 65536 elements by pattern
    // and type).  Threads: the fewest wavefronts that hold a row in MAXU units a
    // thread, so that as many rows as possible share a compute unit (3584 x 18944 bf16 -> INT8: 208 us with the
    // kernel below, 61 with a power of two of threads, 52 so).
    const int64_t nunits = (K + PU::E - 1) / PU::E;
    if ((K * PU::ESI) % 16 != 0 || ((uintptr_t)W & 15) || ((uintptr_t)Wq & 3) || nunits > (int64_t)PU::MAXU * PU::MAX_THREADS) return false;
    const int T = (int)((nunits + PU::MAXU - 1) / PU::MAXU + 63) / 64 * 64;
    constexpr int VB = 4 * PU::template VW<ES>;                          // bytes of one output store
    const int vec_out = (K * ES) % VB == 0 && ((uintptr_t)Wq % VB) == 0;
    // Stores through the L2 (store_through): 8-bit codes of 4 MB and more, a unit in one store of 8 or 16 bytes (time over plain
    // stores 0.90 .. 0.99, 1 MB 1.03; 16-bit codes 1.03, units in several stores 1.34).
    const bool through = PU::template MAY_THROUGH<ES> && O * K >= (4 << 20);
    hipLaunchKernelGGL((k_prune_rows<TIN, OUT, N>), dim3((unsigned)O), dim3(T), 0, st, W, (int)K, (int)nunits, Wq, s_w, vec_out,
                       O * K * PU::ESI >= CACHED_BYTES, through);
    return true;
}

template <typename TIN, int OUT>
static ss_status launch_prune(const void* W, int64_t O, int64_t K, int N, void* Wq, float* s_w, hipStream_t st)
{
    const TIN* w = static_cast<const TIN*>(W);
    uint8_t* wq = static_cast<uint8_t*>(Wq);
    bool done = false;
    switch (N) {
    case 2: done = launch_prune_rows<TIN, OUT, 2>(w, O, K, wq, s_w, st); break;
    case 3: done = launch_prune_rows<TIN, OUT, 3>(w, O, K, wq, s_w, st); break;
    case 4: done = launch_prune_rows<TIN, OUT, 4>(w, O, K, wq, s_w, st); break;
    case 5: done = launch_prune_rows<TIN, OUT, 5>(w, O, K, wq, s_w, st); break;
    case 6: done = launch_prune_rows<TIN, OUT, 6>(w, O, K, wq, s_w, st); break;
    case 7: done = launch_prune_rows<TIN, OUT, 7>(w, O, K, wq, s_w, st); break;
    case 8: done = launch_prune_rows<TIN, OUT, 8>(w, O, K, wq, s_w, st); break;
    }
    if (!done)
        hipLaunchKernelGGL((k_prune_quant<TIN, OUT>), dim3((unsigned)O), dim3(PQ_THREADS), 0, st, w, (int)K, N, wq, s_w);
    return launch_status();
}

extern "C" ss_status slide_prune_quant(const void* W, ss_act_dtype in_dtype, int64_t O, int64_t K, int N, ss_dtype dtype,
                                       void* Wq, float* s_w, void* stream)
{
    if (!valid_N(N)) return SS_ERR_BAD_PATTERN_N;
    if (O < 0 || K <= 0 || K > (1 << 24) || O > 0x7FFFFFFF) return SS_ERR_SHAPE;
    if (in_dtype != SS_IN_F32 && in_dtype != SS_IN_BF16) return SS_ERR_DTYPE;
    if (!valid_dtype(dtype)) return SS_ERR_DTYPE;
    if (O == 0) return SS_OK;
    if (!W || !Wq || (!unscaled(dtype) && !s_w)) return SS_ERR_NULL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (in_dtype == SS_IN_F32) {
        if (dtype == SS_I8) return launch_prune<float, 0>(W, O, K, N, Wq, s_w, st);
        if (dtype == SS_FP8_E4M3) return launch_prune<float, 1>(W, O, K, N, Wq, s_w, st);
        if (dtype == SS_BF16) return launch_prune<float, 2>(W, O, K, N, Wq, s_w, st);
        return launch_prune<float, 3>(W, O, K, N, Wq, s_w, st);
    }
    if (dtype == SS_I8) return launch_prune<uint16_t, 0>(W, O, K, N, Wq, s_w, st);
    if (dtype == SS_FP8_E4M3) return launch_prune<uint16_t, 1>(W, O, K, N, Wq, s_w, st);
    if (dtype == SS_BF16) return launch_prune<uint16_t, 2>(W, O, K, N, Wq, s_w, st);
    return launch_prune<uint16_t, 3>(W, O, K, N, Wq, s_w, st);
}
