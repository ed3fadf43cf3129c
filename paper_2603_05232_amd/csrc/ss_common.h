// Shared host/device helpers of the SlideSparse gfx950 library (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <utility>
#include "slidesparse.h"

#define SS_FORMAT_VERSION 2

namespace ss {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v16bf __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v16h __attribute__((ext_vector_type(16)));

// Rows of the packed weight buffers are padded to this many output channels; one such
// panel is the O-extent a wave accumulates, and the row order inside a panel is permuted
// so that every lane ends up holding runs of consecutive output channels.
constexpr int PANEL = 128;
// K' granularity of the packed format and of both GEMMs.
constexpr int KSTEP = 128;

// Alg. 1: n_g = ceil(K / 2N) blocks (the last one completed with zeros), K' = 4 n_g (N-1).
__host__ __device__ inline int64_t n_groups(int64_t K, int N) { return (K + 2 * N - 1) / (2 * N); }
__host__ __device__ inline int64_t lifted_k(int64_t K, int N) { return n_groups(K, N) * 4 * (N - 1); }
// Stored width (elements of es bytes) of a lifted row: K' rounded up to whole 128-byte k units;
// the columns beyond K' hold zeros (activations) / all-zero windows (weights).
inline int64_t lifted_ld(int64_t K, int N, int es) { const int64_t per = KSTEP / es; return (lifted_k(K, N) + per - 1) / per * per; }
inline bool valid_N(int N) { return N >= 2 && N <= 8; }
inline int elem_size(ss_dtype d) { return (d == SS_BF16 || d == SS_FP16) ? 2 : 1; }
inline bool valid_dtype(ss_dtype d) { return d == SS_I8 || d == SS_FP8_E4M3 || d == SS_BF16 || d == SS_FP16; }
inline bool unscaled(ss_dtype d) { return d == SS_BF16 || d == SS_FP16; }
inline ss_status launch_status()
{
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <typename F, int... I> __device__ __forceinline__ void unroll_list(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F> __device__ __forceinline__ void unroll(F&& f) { unroll_list(static_cast<F&&>(f), std::make_integer_sequence<int, N>{}); }

// Workgroup ids go round-robin over the 8 XCDs (id mod 8).  Renumbers `total` workgroups so that each XCD's share is one
// contiguous run of items: a bijection of [0, total) for any total.
__device__ inline int xcd_run(int id, int total)
{
    const int x = id & 7, rest = total & 7;
    return x * (total >> 3) + (x < rest ? x : rest) + (id >> 3);
}

// n / d for n < 2^31 by a multiplication, prepared on the host: a kernel that divides ahead of its first load makes all its loads wait for it (an integer division
// is some 25 dependent instructions, one of 64 bits 100; the tile kernels of few tokens had 570 instructions there, 1.2 us of a 10 us launch).
struct Div { uint32_t mul, shift; };
inline Div make_div(int64_t d)                       // 1 <= d < 2^31
{
    uint32_t s = 0;
    while ((1ll << s) < d) ++s;
    return {(uint32_t)(((1ull << (31 + s)) + d - 1) / d), 31 + s};      // mul d - 2^(31 + s) < 2^s, so the quotient is exact
}
__host__ __device__ inline int quot(int n, Div d) { return (int)((uint64_t)(uint32_t)n * d.mul >> d.shift); }

// What a program passes over in turn and comes to more than this is hardly found in the memory-side cache again: a third of its 256 MB.
constexpr int64_t CACHED_BYTES = 80ll << 20;
// What that cache does not hold at all.
constexpr int64_t CACHE_BYTES = 256ll << 20;
// non-temporal load and store, for data that is read once or written and not read soon
__device__ inline uint4 load_once(const uint4* p)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ inline void store_once(uint4* p, uint4 v)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(p));
}

// Stores that go through the L2 at once.  What a kernel leaves in the eight L2s is written back when it ends, at about 2.6 TB/s, before the next kernel
// starts; written through, it leaves while the kernel still reads (1300 lifted rows of 6144 bytes in a trace 7.9 -> 6.9 us: the same bytes, their 62000 requests counted as
// L2 misses instead of hits).  Where a wavefront writes whole lines and megabytes of them: part of a line goes to memory as such (fp32 4:6 pruning 1.34
// of the time), and a kernel of little output waits for the acknowledgement (1.03 .. 1.06).  Partial sums of split rows gain nothing (four layers at
// M = 64 1.009, M = 256 0.997): their kernels write at their end.
__device__ inline void store_through(uint2* p, uint2 v)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1" ::"v"(p), "v"((u32x2){v.x, v.y}) : "memory");
}
__device__ inline void store_through(uint4* p, uint4 v)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    // A vector instruction may overwrite the data of a store of more than 8 bytes after two wait states, not sooner.  The compiler, which gives its own
    // stores these, does not see this one, so they are part of the statement.
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"((u32x4){v.x, v.y, v.z, v.w}) : "memory");
}

// ---- scalar format conversions (device) --------------------------------------------------
__device__ inline float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ inline uint16_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// fp32 -> IEEE half bits, round to nearest even (v_cvt_f16_f32)
__device__ inline uint16_t f32_to_f16_bits(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

// fp32 (already clamped to [-448, 448]) -> OCP e4m3fn byte, round to nearest even.
__device__ inline uint32_t f32_to_e4m3(float f)
{
    uint32_t u = __float_as_uint(f);
    uint32_t sign = (u >> 24) & 0x80u;
    float a = __uint_as_float(u & 0x7FFFFFFFu);
    uint32_t code;
    if (a < 0.015625f) {                       // below 2^-6: multiples of 2^-9
        code = (uint32_t)rintf(a * 512.0f);    // 0..8; 8 is the smallest normal
    } else {
        uint32_t m = __float_as_uint(a);
        m += 0x7FFFFu + ((m >> 20) & 1u);      // rne to 3 mantissa bits, may carry into the exponent
        code = (m >> 20) - ((127u - 7u) << 3);
        code = code > 0x7Eu ? 0x7Eu : code;
    }
    return sign | code;
}

}  // namespace ss
