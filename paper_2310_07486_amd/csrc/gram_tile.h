// One 64 x 64 tile of G^r = S^r S^rT from the bit rows along tau, for the pair
// records and the three-replica records.
//
// Sites stand in blocks of 32 rows: block (a, b) holds x1 = 4a .. 4a + 3 and
// x2 = 8b .. 8b + 7 (row 4 (x2 - 8b) + x1 - 4a), so that the 16 elements q of
// a lane in the 32 x 32 MFMA layout take four values of x1 - y1 (by q mod 4)
// and four of x2 - y2 (by q div 4), for every even L.  A tile is 2 x 2 blocks.
#pragma once

#include <type_traits>

#include "tfim_internal.h"

namespace tfim {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Block (blk / nb8, blk mod nb8); nblk blocks cover the plane.
__host__ __device__ inline int gram_nb8(int L) { return (L + 7) >> 3; }
__host__ __device__ inline int gram_nblk(int L) { return ((L + 3) >> 2) * gram_nb8(L); }

// The fp4 K loop (operands of +-1, 0 on padding sites; 7 VALU per operand, one
// operand per MFMA).  Lane (i, h) takes the whole word of chunk 2c + h, whose
// halves feed two MFMAs: one 8-byte load per row and 128 values of tau, 256
// consecutive bytes per half-wave.
struct GramTile {
    __amdgpu_buffer_rsrc_t rows;  // one configuration's rows
    int nc, nxp, back_last;
    uint32_t flip[2], in_last;
    int voff[4];      // byte offset of this lane's row (chunk h of a pair) in the row blocks, then the columns
    uint32_t mag[4];  // 0 on a padding site

    __device__ __forceinline__ GramTile(const ShapeDev& sh) {
        const int h = (threadIdx.x >> 5) & 1;
        nc = sh.nc;
        nxp = sh.nxp;
        // In the last pair of chunks: the last chunk's bits past Ltau cancel
        // (half of them turned over; their number is a multiple of 8), and
        // with an odd number of chunks the half-wave h = 1 counts for nothing
        // and reads the last chunk again.
        const int padn = (64 * nc - sh.Lt) >> 1;
        const uint64_t flip64 = padn && h == ((nc - 1) & 1) ? ~0ull << (64 - padn) : 0ull;
        flip[0] = (uint32_t)flip64;
        flip[1] = (uint32_t)(flip64 >> 32);
        const bool beyond = (nc & 1) && h == 1;
        in_last = beyond ? 0u : ~0u;
        back_last = beyond ? 8 * nxp : 0;
    }
    // The rows of configuration cfg (R replicas).
    __device__ __forceinline__ void configuration(const ShapeDev& sh, int cfg) {
        const uint64_t pt = (uint64_t)(sh.Pt + (size_t)cfg * sh.R * nc * nxp);
        // uniform descriptor (readfirstlane is a signed int: cast before widening)
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)pt);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(pt >> 32));
        rows = __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0, sh.R * nc * nxp * 8,
                                                 0x00020000);
    }
    // Row blocks 2X, 2X + 1 and column blocks 2Y, 2Y + 1.
    __device__ __forceinline__ void tile(int L, int X, int Y) {
        const int i = threadIdx.x & 31, h = (threadIdx.x >> 5) & 1, nb8 = gram_nb8(L), nblk = gram_nblk(L);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int blk = 2 * (k < 2 ? X : Y) + (k & 1);
            const int x1 = 4 * (blk / nb8) + (i & 3), x2 = 8 * (blk % nb8) + (i >> 2);
            const bool ok = blk < nblk && x1 < L && x2 < L;
            voff[k] = 8 * ((ok ? site_slot(L, x1, x2) : 0) + h * nxp);
            mag[k] = ok ? 0x22222222u : 0u;
        }
    }
    // acc[u][v] = start + G^r of row block u, column block v.
    __device__ __forceinline__ void product(int r, const f32x16& start, f32x16 (&acc)[2][2]) const {
        auto fetch = [&](int c, u32x2 (&w)[4]) {
            const int so = (r * nc + 2 * c) * nxp * 8;
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = __builtin_amdgcn_raw_buffer_load_b64(rows, voff[k], so, 0);
        };
        auto chunk = [&](const u32x2 (&w)[4], auto firstC) {
            constexpr bool kFirst = decltype(firstC)::value;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                i32x4 o[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    o[k] = fp4_signs_operand(kFirst && k < 2 ? w[k][ks] ^ flip[ks] : w[k][ks],
                                             kFirst && k < 2 ? mag[k] & in_last : mag[k]);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 2; ++v)
                        acc[u][v] = mfma_fp4(fp4_wide(o[u]), fp4_wide(o[2 + v]),
                                             kFirst && ks == 0 ? start : acc[u][v]);
            }
        };
        // the last pair of chunks first (it starts the accumulators), then
        // pairs 0 .. n - 1, two word sets in turn, each loaded two pairs
        // ahead (past the end: the last one again, not used)
        const int n = (nc + 1) / 2 - 1;
        u32x2 w0[4], w1[4];
        {
            const int so = (r * nc + 2 * n) * nxp * 8;
#pragma unroll
            for (int k = 0; k < 4; ++k) w1[k] = __builtin_amdgcn_raw_buffer_load_b64(rows, voff[k] - back_last, so, 0);
        }
        fetch(0, w0);
        chunk(w1, std::true_type{});
        fetch(min(1, n), w1);
        int c = 0;
        for (; c + 1 < n; c += 2) {
            chunk(w0, std::false_type{});
            fetch(min(c + 2, n), w0);
            chunk(w1, std::false_type{});
            fetch(min(c + 3, n), w1);
        }
        if (c < n) chunk(w0, std::false_type{});
    }
};

// Elements 2t, 2t + 1 of a block whose accumulators started from 1.5 2^23 (+
// a small integer): the low 16 bits of each, packed.
__device__ __forceinline__ int gram_pack(const f32x16& acc, int t) {
    return (int)__builtin_amdgcn_perm(__float_as_uint(acc[2 * t + 1]), __float_as_uint(acc[2 * t]), 0x05040100u);
}
// Displacement d mod L of two sites of the plane; with a padding site, whose
// terms are 0, some bucket in range.
__device__ __forceinline__ int bucket_of(int d, int L) {
    const uint32_t u = min((uint32_t)d, (uint32_t)(d + L));  // d + L where d is negative
    return (int)min(min(u, u - (uint32_t)L), (uint32_t)(L - 1));
}
constexpr float kGramStart = 12582912.0f;  // 1.5 2^23

}  // namespace tfim
