// slide_decompose: Sliding Window Decomposition (Alg. 2, greedy residual allocation) fused
// with 2:4 compression, in the packed form the GEMM kernels read (k_decompose_packed) and in a
// plain one for inspection (k_decompose_canonical: a thread per window re-runs the greedy over
// the few earlier windows of its 2N block to recover what they took).
#include "ss_common.h"
#include "packed_layout.h"
#include <type_traits>

namespace ss {

template <int ES> struct Elem;
template <> struct Elem<1> { typedef uint8_t T; __device__ static bool nz(T v, bool fp) { return fp ? (v & 0x7F) != 0 : v != 0; } };
template <> struct Elem<2> { typedef uint16_t T; __device__ static bool nz(T v, bool) { return (v & 0x7FFF) != 0; } };

// One window of the decomposition: values and positions (i0 < i1) of window l of block g of a
// row, plus the block's non-zero count.  `row` points at the row's first element, K is its
// length: elements at and beyond K read as zero (last block completed with zeros, Alg. 1's
// n_g = ceil(K / 2N)), and a block at or beyond n_g is all zero (padding of the stored width).
template <int ES>
__device__ inline void slide_window(const typename Elem<ES>::T* row, int K, int N, int g, int l, bool fp,
                                    typename Elem<ES>::T& v0, typename Elem<ES>::T& v1, uint32_t& i0, uint32_t& i1, int& nnz)
{
    typedef typename Elem<ES>::T T;
    const T* blk = row + (int64_t)g * 2 * N;
    const int left = K - g * 2 * N;                      // elements of this block inside the row (may be <= 0)
    uint32_t nzmask = 0;
    for (int p = 0; p < 2 * l + 4; ++p) nzmask |= (uint32_t)(p < left && Elem<ES>::nz(blk[p], fp)) << p;
    uint32_t used = 0, taken = 0;
    for (int w = 0; w <= l; ++w) {                       // greedy, windows in ascending order
        int cnt = 0;
        taken = 0;
        for (int d = 0; d < 4; ++d) {
            const int p = 2 * w + d;
            if (((nzmask >> p) & 1u) && !((used >> p) & 1u) && cnt < 2) { used |= 1u << p; taken |= 1u << d; ++cnt; }
        }
    }
    if (l == 0) {                                        // pattern check, once per block
        uint32_t all = nzmask;
        for (int p = 4; p < 2 * N; ++p) all |= (uint32_t)(p < left && Elem<ES>::nz(blk[p], fp)) << p;
        nnz = __popc(all);
    } else nnz = 0;
    // pad to two positions with the lowest offsets that hold no stored non-zero
    uint32_t chosen = taken;
    for (int d = 0; d < 4 && __popc(chosen) < 2; ++d) chosen |= 1u << d;
    i0 = __ffs(chosen) - 1;
    i1 = 31 - __clz(chosen);
    v0 = ((taken >> i0) & 1u) ? blk[2 * l + i0] : (T)0;
    v1 = ((taken >> i1) & 1u) ? blk[2 * l + i1] : (T)0;
}

// canonical form: one thread per (row, window)
template <int ES>
__global__ __launch_bounds__(256) void k_decompose_canonical(const typename Elem<ES>::T* __restrict__ Wq, int64_t O, int K, int N, bool fp,
                                                              typename Elem<ES>::T* __restrict__ vals, uint8_t* __restrict__ idx,
                                                              int32_t* __restrict__ violations)
{
    const int nwin = (int)n_groups(K, N) * (N - 1);
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= O * nwin) return;
    const int64_t o = id / nwin;
    const int j = (int)(id - o * nwin);
    const int g = j / (N - 1), l = j - g * (N - 1);
    typename Elem<ES>::T v0, v1; uint32_t i0, i1; int nnz;
    slide_window<ES>(Wq + o * (int64_t)K, K, N, g, l, fp, v0, v1, i0, i1, nnz);
    vals[o * (int64_t)nwin * 2 + 2 * j] = v0;
    vals[o * (int64_t)nwin * 2 + 2 * j + 1] = v1;
    idx[o * (int64_t)nwin + j] = (uint8_t)(i0 | (i1 << 2));
    if (violations && nnz > 2 * N - 2) atomicAdd(violations, 1);
}

// ---- packed form ------------------------------------------------------------------------------------------
// Bound by HBM (the quantised matrix in, 15/16 of it out for 6:8 in 8 bits), so the kernel is built around whole cache
// lines on both sides.  A group is 16 / ES blocks of a row = 32 N bytes = N - 1 steps of the packed form: the smallest
// run of blocks that fills whole steps in either window order.  A workgroup owns one group of the 128 rows of a panel:
// it copies 128 x 32N bytes to LDS with 16-byte loads (consecutive lanes along a row), thread t decomposes the group of
// packed row t (fragment t / 32, row t % 32), which yields the operand registers of lanes i and i + 32 of its fragment
// for N - 1 steps; the values go out as runs of 32 x 16 bytes, the index words meet in LDS and go out lane-major.
//
// Alg. 2's greedy as a state machine: a window sees the two elements it shares with its predecessor (those not taken
// yet) and two new ones, takes the first two non-zeros of the four and hands on what is left of the last two.  Everything
// that depends on the four availability bits (positions, byte selectors that fetch the values and write zeros where
// nothing is stored, the hand-over) is one entry of a 16-entry LDS table, so a window costs one table read, one byte
// permute and a few bit operations.
// Measured, 37888 x 3584 INT8 6:8, window order of the fused GEMM: 221 -> 58 us (a thread per lane of
// the packed form, which loads its two to four blocks straight from rows K bytes apart and runs the greedy bit by bit,
// before), with non-temporal loads (of lines that one workgroup reads) and stores 44 us (5.9 TB/s).
template <int ES, int N> struct PackGroup {
    static constexpr int BLOCKS = 16 / ES;
    static constexpr int BYTES = 32 * N;
    static constexpr int STEPS = N - 1;
    static constexpr int ROW = BYTES + 16;               // LDS bytes per row: an odd number of 16-byte chunks, so the chunk reads of 16 lanes spread over all banks
    static constexpr int WORDS = BYTES / 4;
    static constexpr int MASKS = WORDS * (4 / ES) / 32 + 1;     // words of one non-zero bit per element
};

// entry of the table for availability bits av: 8-bit types: bits 15..0 two byte selectors into the window's four
// bytes; 16-bit types: the upper word of the entry, four byte selectors into its eight.  0x0C selects a zero byte.
// Bits 27..24 the two positions (ascending, padded with the lowest offsets that hold no stored non-zero), bits 31..30
// the availability of the last two elements for the next window.
template <int ES> __device__ inline uint2 pack_entry(uint32_t av)
{
    uint32_t taken = av & (0u - av);                     // first non-zero ...
    const uint32_t rest = av & ~taken;
    taken |= rest & (0u - rest);                         // ... and the second
    uint32_t chosen = taken;
    for (int d = 0; d < 4; ++d) if (__popc(chosen) < 2) chosen |= 1u << d;
    const uint32_t i0 = __ffs(chosen) - 1, i1 = 31 - __clz(chosen);
    const bool s0 = (taken >> i0) & 1u, s1 = (taken >> i1) & 1u;
    uint32_t lo = ((i0 | (i1 << 2)) << 24) | ((av & ~taken) >> 2) << 30, hi = 0;
    if (ES == 1) lo |= (s0 ? i0 : 0x0Cu) | (s1 ? i1 : 0x0Cu) << 8;
    else hi = (s0 ? (2 * i0) | (2 * i0 + 1) << 8 : 0x0C0Cu) | (s1 ? (2 * i1) | (2 * i1 + 1) << 8 : 0x0C0Cu) << 16;
    return make_uint2(lo, hi);
}

// where window l of block b of a group goes: step of the group, lane half qa, window slot w (the two orders of
// packed_layout.h)
struct PackSlot { int step, qa, w; };
template <int ES, int N, bool FUSED> __device__ constexpr PackSlot pack_slot(int b, int l)
{
    constexpr int HW = 4 / ES, BL = 8 / ES;
    if (FUSED) {
        const int qb = b / BL, bb = b % BL, J = l == 1 ? 2 : bb / (BL / 2), wsl = l == 1 ? bb : 2 * (bb % (BL / 2)) + (l >> 1);
        return {J, wsl / HW, qb * HW + wsl % HW};
    }
    const int j = b * (N - 1) + l, wi = j % (4 * HW), rem = wi % (2 * HW);
    return {j / (4 * HW), rem / HW, (wi / (2 * HW)) * HW + rem % HW};
}

// Bytes [k0, k0 + 4) of a row of `row_bytes` bytes, zero beyond its end.  The row may start at any byte: the two aligned
// words around them are read and shifted into place; a word that sticks out of the matrix [mat, mat_end) is read byte by byte.
__device__ inline uint32_t row_word(const uint8_t* mat, const uint8_t* mat_end, const uint8_t* row, int row_bytes, int k0)
{
    const int left = row_bytes - k0;
    if (left <= 0) return 0;
    const uint8_t* p = row + k0;
    const int sh = (int)((uintptr_t)p & 3);
    auto word = [&](const uint8_t* q) -> uint32_t {
        if (q >= mat && q + 4 <= mat_end) return *reinterpret_cast<const uint32_t*>(q);
        uint32_t w = 0;
#pragma unroll 1
        for (int e = 0; e < 4; ++e) if (q + e >= mat && q + e < mat_end) w |= (uint32_t)q[e] << (8 * e);
        return w;
    };
    const uint32_t lo = word(p - sh), hi = sh && left > 4 - sh ? word(p - sh + 4) : 0u;
    const uint32_t v = __builtin_amdgcn_alignbyte(hi, lo, sh);
    return left < 4 ? v & ((1u << (8 * left)) - 1u) : v;
}

template <int ES, int N, bool FUSED>
__global__ __launch_bounds__(PANEL) void k_decompose_packed(const uint8_t* __restrict__ Wq, int64_t O, int K, bool fp, uint4* __restrict__ vals,
                                                             uint32_t* __restrict__ meta, int nsteps, int ngroups, bool aligned,
                                                             int32_t* __restrict__ violations)
{
    typedef PackGroup<ES, N> PG;
    constexpr int NW = 8 / ES, CHUNKS = PG::BYTES / 16;
    __shared__ __attribute__((aligned(16))) uint8_t rows[PANEL * PG::ROW];
    __shared__ __attribute__((aligned(16))) uint32_t words[PG::STEPS * 64 * FRAGS_PER_PANEL];
    __shared__ uint2 table[16];
    const int t = threadIdx.x;
    const int panel = blockIdx.x / ngroups, group = blockIdx.x - panel * ngroups;
    const int row_bytes = K * ES;
    // ---- the rows of the panel, in packed order
    if (t < 16) table[t] = pack_entry<ES>(t);
    if (aligned) {
        uint4 in[CHUNKS];
        auto load_rows = [&](auto once_c) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) {
                const int id = c * PANEL + t, slot = id / CHUNKS, part = id - slot * CHUNKS;
                const int64_t o = (int64_t)panel * PANEL + panel_row(slot >> 5, slot & 31);
                const int k0 = group * PG::BYTES + part * 16;
                in[c] = make_uint4(0, 0, 0, 0);
                if (o < O && k0 < row_bytes) {
                    const uint4* p = reinterpret_cast<const uint4*>(Wq + o * row_bytes + k0);
                    in[c] = decltype(once_c)::value ? load_once(p) : *p;
                }
            }
        };
        // lines that no other workgroup reads are loaded non-temporally
        if (PG::BYTES % 128 == 0 && ((row_bytes | (uintptr_t)Wq) & 127) == 0) load_rows(std::true_type{});
        else load_rows(std::false_type{});
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int id = c * PANEL + t, slot = id / CHUNKS, part = id - slot * CHUNKS;
            *reinterpret_cast<uint4*>(rows + slot * PG::ROW + part * 16) = in[c];
        }
    } else {
#pragma unroll 4
        for (int c = 0; c < 4 * CHUNKS; ++c) {
            const int id = c * PANEL + t, slot = id / (4 * CHUNKS), part = id - slot * (4 * CHUNKS);
            const int64_t o = (int64_t)panel * PANEL + panel_row(slot >> 5, slot & 31);
            *reinterpret_cast<uint32_t*>(rows + slot * PG::ROW + part * 4) =
                o < O ? row_word(Wq, Wq + O * row_bytes, Wq + o * row_bytes, row_bytes, group * PG::BYTES + part * 4) : 0u;
        }
    }
    __syncthreads();
    // ---- one group of one row per thread
    uint32_t x[PG::WORDS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const uint4 q = *reinterpret_cast<const uint4*>(rows + t * PG::ROW + c * 16);
        x[4 * c] = q.x; x[4 * c + 1] = q.y; x[4 * c + 2] = q.z; x[4 * c + 3] = q.w;
    }
    // non-zero bits, one per element: the top bit of every element of a word, gathered by a byte dot product with
    // powers of two (8 elements per round, which leaves them 7 bits up)
    uint32_t nz[PG::MASKS] = {};
    const uint32_t any = ES == 1 ? 0x7F7F7F7Fu : 0x7FFF7FFFu, top = ES == 1 ? 0x80808080u : 0x80008000u;
    const uint32_t sign = fp ? 0u : 0xFFFFFFFFu;          // the sign bit counts as a value bit for integers only
#pragma unroll
    for (int j = 0; j < PG::WORDS * (4 / ES) / 8; ++j) {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 2 * ES; ++i) {
            const uint32_t w = x[j * 2 * ES + i], f = (((w & any) + any) | (w & sign)) & top;
            const uint32_t weights = ES == 1 ? (i ? 0x80402010u : 0x08040201u) : (0x02000100u << (2 * i));
            m = __builtin_amdgcn_udot4(f, weights, m, false);
        }
        m >>= 7;
        nz[j / 4] |= m << (8 * (j % 4));
    }
    const int f = t >> 5, i = t & 31;
    uint32_t v[PG::STEPS][2][4], meta_w[PG::STEPS][2];
#pragma unroll
    for (int s = 0; s < PG::STEPS; ++s)
#pragma unroll
        for (int qa = 0; qa < 2; ++qa) {
            meta_w[s][qa] = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[s][qa][k] = 0;
        }
#pragma unroll
    for (int b = 0; b < PG::BLOCKS; ++b) {
        const int e0 = b * 2 * N;                         // first element of the block
        auto pair = [&](int e) { return (nz[e >> 5] >> (e & 31)) & 3u; };       // e is even: a pair never straddles words
        uint32_t carry = pair(e0);
#pragma unroll
        for (int l = 0; l < N - 1; ++l) {
            const int e = e0 + 2 * l;
            const uint32_t av = carry | pair(e + 2) << 2;
            const uint2 q = table[av];
            carry = q.x >> 30;
            const PackSlot s = pack_slot<ES, N, FUSED>(b, l);
            if constexpr (ES == 1) {
                const uint32_t win = (e & 2) ? __builtin_amdgcn_alignbyte(x[(e >> 2) + 1 < PG::WORDS ? (e >> 2) + 1 : 0], x[e >> 2], 2) : x[e >> 2];
                const uint32_t two = __builtin_amdgcn_perm(0, win, q.x);        // the two values in bytes 0, 1; the rest is the entry's other bits
                uint32_t& d = v[s.step][s.qa][s.w >> 1];
                d = (s.w & 1) ? __builtin_amdgcn_perm(two, d, 0x05040100u) : __builtin_amdgcn_perm(d, two, 0x07060100u);
            } else
                v[s.step][s.qa][s.w] = __builtin_amdgcn_perm(x[(e >> 1) + 1], x[e >> 1], q.y);
            meta_w[s.step][s.qa] |= ((q.x >> 24) & 15u) << (4 * s.w);
        }
    }
    if (violations) {                                     // blocks with more than 2N - 2 non-zeros
        int bad = 0;
#pragma unroll
        for (int b = 0; b < PG::BLOCKS; ++b) {
            const int e0 = b * 2 * N, w0 = e0 >> 5;
            const uint64_t two = nz[w0] | (uint64_t)(w0 + 1 < PG::MASKS ? nz[w0 + 1] : 0u) << 32;
            bad += __popc((uint32_t)(two >> (e0 & 31)) & ((1u << (2 * N)) - 1u)) > 2 * N - 2;
        }
        if (bad) atomicAdd(violations, bad);
    }
    // ---- out: values straight, index words through LDS
    const int64_t ps0 = (int64_t)panel * nsteps + group * PG::STEPS;
    // non-temporal, but for a single step of the pattern's shortest group (2:4: 1.02 to 1.06 of the time with them)
    auto put = [](uint4* p, uint4 x) { if constexpr (N > 2) store_once(p, x); else *p = x; };
    const int left = nsteps - group * PG::STEPS;          // steps of this group that exist (the last group may stick out)
#pragma unroll
    for (int s = 0; s < PG::STEPS; ++s)
#pragma unroll
        for (int qa = 0; qa < 2; ++qa) {
            if (s < left) put(vals + ((ps0 + s) * FRAGS_PER_PANEL + f) * 64 + qa * 32 + i, make_uint4(v[s][qa][0], v[s][qa][1], v[s][qa][2], v[s][qa][3]));
            words[(s * 64 + qa * 32 + i) * FRAGS_PER_PANEL + f] = meta_w[s][qa];
        }
    __syncthreads();
    for (int k = t; k < (PG::STEPS < left ? PG::STEPS : left) * 64; k += PANEL)
        put(reinterpret_cast<uint4*>(meta) + ps0 * 64 + k, reinterpret_cast<const uint4*>(words)[k]);
}

}  // namespace ss

using namespace ss;

static ss_status check_decompose(int64_t O, int64_t K, int N, ss_dtype dtype)
{
    if (!valid_N(N)) return SS_ERR_BAD_PATTERN_N;
    if (!valid_dtype(dtype)) return SS_ERR_DTYPE;
    if (O < 0 || K <= 0 || K > (1 << 24) || O > (1 << 24)) return SS_ERR_SHAPE;
    return SS_OK;
}

extern "C" ss_status slide_packed_sizes(int64_t O, int64_t K, int N, ss_dtype dtype, size_t* vals_bytes, size_t* meta_bytes)
{
    ss_status st = check_decompose(O, K, N, dtype);
    if (st != SS_OK) return st;
    if (!vals_bytes || !meta_bytes) return SS_ERR_NULL;
    const int64_t Kpb = lifted_ld(K, N, elem_size(dtype)) * elem_size(dtype);    // stored bytes of a lifted row
    const int64_t Opad = (O + PANEL - 1) / PANEL * PANEL;
    *vals_bytes = (size_t)(Opad * (Kpb / 2));
    *meta_bytes = (size_t)(Opad * (Kpb / 8));            // one 4-byte index word per 16 bytes of values
    return SS_OK;
}

template <int ES, int N, bool FUSED>
static ss_status launch_packed_n(const void* Wq, int64_t O, int64_t K, ss_dtype dtype, int nsteps, void* w_vals, void* w_meta, int32_t* violations,
                                 hipStream_t stream)
{
    const int64_t npanels = (O + PANEL - 1) / PANEL;
    const int ngroups = (nsteps + N - 2) / (N - 1);
    if (npanels * ngroups > 0x7FFFFFFF) return SS_ERR_SHAPE;
    const bool aligned = (K * ES) % 16 == 0 && ((uintptr_t)Wq & 15) == 0;
    hipLaunchKernelGGL((k_decompose_packed<ES, N, FUSED>), dim3((unsigned)(npanels * ngroups)), dim3(PANEL), 0, stream, static_cast<const uint8_t*>(Wq), O,
                       (int)K, dtype != SS_I8, static_cast<uint4*>(w_vals), static_cast<uint32_t*>(w_meta), nsteps, ngroups, aligned, violations);
    return launch_status();
}

template <int ES>
static ss_status launch_packed(const void* Wq, int64_t O, int64_t K, int N, ss_dtype dtype, bool fused, int64_t Kpb, void* w_vals, void* w_meta,
                               int32_t* violations, void* stream)
{
    const int nsteps = (int)(Kpb / FRAG_KB);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (fused) return launch_packed_n<ES, 4, true>(Wq, O, K, dtype, nsteps, w_vals, w_meta, violations, s);
#define SS_PK(N) case N: return launch_packed_n<ES, N, false>(Wq, O, K, dtype, nsteps, w_vals, w_meta, violations, s)
    switch (N) { SS_PK(2); SS_PK(3); SS_PK(4); SS_PK(5); SS_PK(6); SS_PK(7); SS_PK(8); }
#undef SS_PK
    return SS_ERR_BAD_PATTERN_N;
}

extern "C" ss_status slide_decompose(const void* Wq, int64_t O, int64_t K, int N, ss_dtype dtype, void* w_vals, void* w_meta,
                                     int32_t* violations, void* stream)
{
    ss_status st = check_decompose(O, K, N, dtype);
    if (st != SS_OK) return st;
    const int64_t Kpb = lifted_ld(K, N, elem_size(dtype)) * elem_size(dtype);
    if (O == 0) return SS_OK;
    if (!Wq || !w_vals || !w_meta) return SS_ERR_NULL;
    return elem_size(dtype) == 1 ? launch_packed<1>(Wq, O, K, N, dtype, false, Kpb, w_vals, w_meta, violations, stream)
                                 : launch_packed<2>(Wq, O, K, N, dtype, false, Kpb, w_vals, w_meta, violations, stream);
}

// Fused order: lifted bytes per row = 192 per 128 unlifted bytes (whole super-units; columns at and beyond K are zero).
static int64_t fused_lifted_row_bytes(int64_t K, ss_dtype dtype) { return (K * elem_size(dtype) + KSTEP - 1) / KSTEP * (3 * FRAG_KB); }

extern "C" ss_status slide_packed_sizes_fused(int64_t O, int64_t K, int N, ss_dtype dtype, size_t* vals_bytes, size_t* meta_bytes)
{
    ss_status st = check_decompose(O, K, N, dtype);
    if (st != SS_OK) return st;
    if (N != 4) return SS_ERR_BAD_PATTERN_N;
    if (!vals_bytes || !meta_bytes) return SS_ERR_NULL;
    const int64_t Kpb = fused_lifted_row_bytes(K, dtype);
    const int64_t Opad = (O + PANEL - 1) / PANEL * PANEL;
    *vals_bytes = (size_t)(Opad * (Kpb / 2));
    *meta_bytes = (size_t)(Opad * (Kpb / 8));
    return SS_OK;
}

extern "C" ss_status slide_decompose_fused(const void* Wq, int64_t O, int64_t K, int N, ss_dtype dtype, void* w_vals, void* w_meta,
                                           int32_t* violations, void* stream)
{
    ss_status st = check_decompose(O, K, N, dtype);
    if (st != SS_OK) return st;
    if (N != 4) return SS_ERR_BAD_PATTERN_N;
    if (O == 0) return SS_OK;
    if (!Wq || !w_vals || !w_meta) return SS_ERR_NULL;
    const int64_t Kpb = fused_lifted_row_bytes(K, dtype);
    return elem_size(dtype) == 1 ? launch_packed<1>(Wq, O, K, N, dtype, true, Kpb, w_vals, w_meta, violations, stream)
                                 : launch_packed<2>(Wq, O, K, N, dtype, true, Kpb, w_vals, w_meta, violations, stream);
}

extern "C" ss_status slide_decompose_canonical(const void* Wq, int64_t O, int64_t K, int N, ss_dtype dtype, void* vals, uint8_t* idx,
                                               int32_t* violations, void* stream)
{
    ss_status st = check_decompose(O, K, N, dtype);
    if (st != SS_OK) return st;
    if (O == 0) return SS_OK;
    if (!Wq || !vals || !idx) return SS_ERR_NULL;
    const int64_t nwin = n_groups(K, N) * (N - 1);
    const int64_t total = O * nwin;
    dim3 grid((unsigned)((total + 255) / 256)), block(256);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (elem_size(dtype) == 2)
        hipLaunchKernelGGL(k_decompose_canonical<2>, grid, block, 0, s, static_cast<const uint16_t*>(Wq), O, (int)K, N, true,
                           static_cast<uint16_t*>(vals), idx, violations);
    else
        hipLaunchKernelGGL(k_decompose_canonical<1>, grid, block, 0, s, static_cast<const uint8_t*>(Wq), O, (int)K, N,
                           dtype == SS_FP8_E4M3, static_cast<uint8_t*>(vals), idx, violations);
    return launch_status();
}
