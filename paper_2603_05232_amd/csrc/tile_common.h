// Pieces shared by the tile kernels of 256 tokens (gemm.hip, gemm_lifted.hip, gemm_fused.hip, gemm_fused_narrow.hip): the order in which persistent
// workgroups walk the output tiles, and the epilogue that stages a wavefront's accumulators through LDS so
// that every global store writes whole 256-byte row segments of Y.
#pragma once
#include "ss_common.h"
#include "mma_types.h"
#include "lds_pipe.h"

namespace ss {

constexpr int BO = 256;   // output channels per workgroup tile
constexpr int BT = 256;   // tokens per workgroup tile

// Persistent workgroups: the grid holds one workgroup per compute unit and workgroup b processes
// tiles b, b + grid, b + 2 grid, ...  Workgroup ids go round-robin to the 8 XCDs, so within a full
// round each XCD is given one contiguous run of tiles, and tiles are ordered in bands of 8 token
// tiles so that the 32 workgroups resident on an XCD share weight panels and token tiles in its L2.
// A partial last round is dealt out in runs as well where the layer has few tiles of channels and keeps the plain order where
// it has many (time of runs over plain, fused INT8 / fp8 / bf16, weights from HBM / hot, M = 640 .. 8192: 14 .. 32 tiles of channels, 33
// calls, 0.989 / 0.998; 54 .. 148 tiles, 93 calls, 1.015 / 0.997, at worst 1.066; lifted rows 1.000 / 0.996 and 1.003 / 0.995).
// Runs in a single partial round (fewer tiles than compute units) are 1 to 4 % faster.
constexpr int RUNS_MAX_TILES_O = 40;
__device__ inline bool tile_of_round(int round, int tiles_o, int tiles_t, int& to, int& tt)
{
    const int nb = gridDim.x, bid = blockIdx.x, total = tiles_o * tiles_t;
    const int base = round * nb;
    if (base + bid >= total) return false;
    const int tile = base + (base + nb <= total || tiles_o <= RUNS_MAX_TILES_O ? xcd_run(bid, min(nb, total - base)) : bid);
    constexpr int BAND = 8;
    const int per_band = BAND * tiles_o;
    const int band = tile / per_band, within = tile - band * per_band;
    const int bw = min(BAND, tiles_t - band * BAND);
    to = within / bw;
    tt = band * BAND + (within - to * bw);
    return true;
}

// The fused-lifting kernels (gemm_fused.hip, gemm_fused_narrow.hip) store chunk c of a token row at place(c) ^ swz(row), see there.
__device__ inline int place(int chunk) { return chunk ^ ((chunk >> 2) << 1); }      // its own inverse
__device__ const uint4 no_values[64] = {};            // 1 KB of stored values for the super-unit that an odd row lacks

// Direct loads of a tile's 256 channel scales and 256 token scales into LDS, by eight wavefronts: 0 .. 3 the channels', 4 .. 7 the
// tokens', 64 each; those beyond the last repeat it.
__device__ inline void load_tile_scales(const float* s_w, const float* s_x, int64_t O, int64_t M, int64_t o_blk, int64_t t_blk, int wave, uint32_t lds)
{
    const int64_t first = (wave < 4 ? o_blk : t_blk) + (wave & 3) * 64, end = wave < 4 ? O : M, left = end - 1 - first;
    const int left32 = left > 63 ? 63 : (int)left, ln = fresh_lane();
    const uint32_t e = left32 < 0 ? 0u : (uint32_t)(ln < left32 ? ln : left32);
    lds_dma4_at(reinterpret_cast<const uint8_t*>((wave < 4 ? s_w : s_x) + (left < 0 ? end - 1 : first)), e * 4, lds + wave * 256);
}

// ---- epilogue: Y = bf16((float(acc) * s_x) * s_w), staged through LDS for coalesced stores ------

// Staging holds 32 tokens x 128 channels of bf16 per wavefront at a time: rows of 256 bytes, 8 KB per wavefront.  No row
// padding: the 16-byte chunk c of row r is stored at chunk c ^ (r & 15), which spreads both the column-wise writes and the
// row-wise reads over all banks.
constexpr int EP_ROWB = 256;
constexpr int EP_WAVE_BYTES = 32 * EP_ROWB;

// token scales of this wavefront's sub-tile for the epilogue: sx[b] of lane (n, h) belongs to token 32 b + n.  Loaded
// ahead of the epilogue (callers issue this before the last k iterations) so that the latency is not exposed.
template <bool SCALED, int NB>
__device__ inline void load_token_scales(float (&sx)[NB], const float* __restrict__ s_x_sub, int rows_left)
{
    const int n = fresh_lane() & 31;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        sx[b] = 1.0f;
        if constexpr (SCALED) {
            uint32_t tk = (uint32_t)(b * 32 + n);
            tk = (int)tk < rows_left ? tk : (uint32_t)(rows_left - 1);
            if (rows_left > 0) sx[b] = s_x_sub[tk];
        }
    }
}

// Makes the compiler place its wait for the loads of sx here.  The kernels call it before they request the next tile's
// first operands with direct loads the compiler does not see: a wait placed behind those would count them in.
template <int NB> __device__ inline void settle(float (&sx)[NB])
{
#pragma unroll
    for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(sx[b]));
}

// acc[f][b][r] of lane (n = lane & 31, h = lane >> 5) is channel 64 h + 16 f + r, token 32 b + n of this
// wavefront's 128-channel x (32 NB)-token sub-tile, whose first element is Y_sub (wave-uniform) and of which
// rows_left tokens x cols_left channels exist.  `stage` is this wavefront's private 8 KB of LDS;
// `sw_lds` holds the sub-tile's 128 channel scales in LDS (fetched with the tile's first unit), sx the token scales
// (load_token_scales).  All lane-dependent offsets are 32-bit (ldy < 2^22).
// SCALED = false (bf16 operands): Y = bf16(acc), the scales are not touched.
template <bool SCALED, typename ACC, int NB>
__device__ inline void store_tile(const ACC (&acc)[4][NB], const float (&sx)[NB], const float* sw_lds, uint16_t* __restrict__ Y_sub,
                                  uint32_t ldy, int rows_left, int cols_left, uint8_t* stage)
{
    const int lane = fresh_lane(), n = lane & 31, h = lane >> 5;
    const bool vec_ok = ((ldy & 7) == 0) && (((uintptr_t)Y_sub & 15) == 0);
    const int seg = lane & 15;                      // 16-byte segment (8 channels) of the 256-byte row
    const int oc = 8 * seg;
    const uint32_t lane_elem = (uint32_t)(lane >> 4) * ldy + (uint32_t)oc;   // this lane's element offset in its first row
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        uint32_t w[4][8];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            if constexpr (SCALED) {
                float sw[16];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 v = reinterpret_cast<const float4*>(sw_lds + 64 * h + 16 * f)[i];
                    sw[4 * i] = v.x; sw[4 * i + 1] = v.y; sw[4 * i + 2] = v.z; sw[4 * i + 3] = v.w;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    w[f][q] = pack_bf16x2(((float)acc[f][b][2 * q] * sx[b]) * sw[2 * q], ((float)acc[f][b][2 * q + 1] * sx[b]) * sw[2 * q + 1]);
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q) w[f][q] = pack_bf16x2((float)acc[f][b][2 * q], (float)acc[f][b][2 * q + 1]);
            }
        }
        uint8_t* row = stage + n * EP_ROWB;
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int c = h * 8 + 2 * f;            // first of the two 16-byte chunks of this lane's 16 channels
            *reinterpret_cast<uint4*>(row + (((c) ^ (n & 15)) << 4)) = make_uint4(w[f][0], w[f][1], w[f][2], w[f][3]);
            *reinterpret_cast<uint4*>(row + (((c + 1) ^ (n & 15)) << 4)) = make_uint4(w[f][4], w[f][5], w[f][6], w[f][7]);
        }
        // wavefront-private staging: its own LDS writes only need to have completed
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 4 * i + (lane >> 4);
            const uint4 v = *reinterpret_cast<const uint4*>(stage + r * EP_ROWB + ((seg ^ (r & 15)) << 4));
            if (b * 32 + r < rows_left) {
                uint16_t* dst = Y_sub + (lane_elem + (uint32_t)(b * 32 + 4 * i) * ldy);
                if (vec_ok && oc + 8 <= cols_left) {
                    // Y is written once and not read again by this kernel: stream it past the caches
                    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                    __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(dst));
                } else {
                    const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (oc + e < cols_left) dst[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
        // the reads of this block have returned (their data went out with the stores) before the next one is staged
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// The same for the 16x16 instructions: acc[f][hh][b][r] of lane (n = lane & 15, q = lane >> 4) is channel
// 64 (q & 1) + 16 f + 8 hh + 4 (q >> 1) + r, token 16 b + n of a 128 x 64 sub-tile; the scales of its 128 channels and 64
// tokens lie in LDS.  A token block of 16 rows is staged at a time (4 KB at `stage`) by all lanes; chunk c of row r at
// c ^ r spreads the 8-byte writes and the 16-byte reads over all banks.
// All loads this wavefront has in flight (the next tile's first operands) are waited for right before the first store.  The
// wait counter counts loads and stores alike, so a later wait for those loads would also wait for the stores to be
// acknowledged; here the loads have had the first block's conversion to arrive and the stores are never waited for.
// SPLIT: the block's four groups of four rows lie 8 KB apart, which is where a wavefront's own direct loads of a token tile go.
template <bool SCALED, bool SPLIT = false, typename ACC>
__device__ inline void store_tile16(const ACC (&acc)[4][2][4], const float* sx_lds, const float* sw_lds, uint16_t* __restrict__ Y_sub, uint32_t ldy,
                                    int rows_left, int cols_left, uint8_t* stage)
{
    const int lane = fresh_lane(), n = lane & 15, q = lane >> 4;
    const bool vec_ok = ((ldy & 7) == 0) && (((uintptr_t)Y_sub & 15) == 0);
    const int oc = 8 * n;                           // reading side: 16-byte segment n (8 channels) of row 4 i + q
    const uint32_t lane_elem = (uint32_t)q * ldy + (uint32_t)oc;
    float4 sw[8];
    if constexpr (SCALED) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sw[e] = *reinterpret_cast<const float4*>(sw_lds + 64 * (q & 1) + 8 * e + 4 * (q >> 1));      // e = 2 f + hh
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const float sx = SCALED ? sx_lds[16 * b + n] : 1.0f;
        uint8_t* const row = stage + (SPLIT ? (n >> 2) * 8192 + (n & 3) * EP_ROWB : n * EP_ROWB) + 8 * (q >> 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const ACC& v = acc[e >> 1][e & 1][b];
            uint2 w;
            if constexpr (SCALED)
                w = make_uint2(pack_bf16x2(((float)v[0] * sx) * sw[e].x, ((float)v[1] * sx) * sw[e].y), pack_bf16x2(((float)v[2] * sx) * sw[e].z, ((float)v[3] * sx) * sw[e].w));
            else w = make_uint2(pack_bf16x2((float)v[0], (float)v[1]), pack_bf16x2((float)v[2], (float)v[3]));
            *reinterpret_cast<uint2*>(row + (((8 * (q & 1) + e) ^ n) << 4)) = w;
        }
        // wavefront-private staging: its own LDS writes only need to have completed
        if (b == 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * i + q;
            const uint4 v = *reinterpret_cast<const uint4*>(stage + (SPLIT ? i * 8192 + q * EP_ROWB : r * EP_ROWB) + ((n ^ r) << 4));
            if (16 * b + r < rows_left) {
                uint16_t* dst = Y_sub + (lane_elem + (uint32_t)(16 * b + 4 * i) * ldy);
                if (vec_ok && oc + 8 <= cols_left) {
                    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                    __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(dst));
                } else {
                    const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (oc + e < cols_left) dst[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
        // the reads of this block have returned (their data went out with the stores) before the next one is staged
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

template <typename ACC, int NB> __device__ inline void zero_acc(ACC (&acc)[4][NB])
{
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][b][r] = 0;
}

}  // namespace ss
