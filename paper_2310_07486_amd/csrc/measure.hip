// Measurement: replica Gram / overlap integers on int8 MFMA, fused int64
// reductions.
//
// Paper: arXiv:2310.07486, Methods, "One-time observables" (M_xy, M-hat, the
// susceptibilities chi^(2), F^(2) and the second-moment length) with the
// tau average of "The Trotter-Suzuki formula" and the replica estimators of
// "Simulation details".
//
// For configuration (k-index i, sample s) and replica r, S^r is the
// L^2 x Ltau matrix of +-1 spins of walker kidx^-1[i] (lane s).  With
// B = (1 - S)/2 in {0,1}:
//   G^r = S S^T = Ltau - 2 (n_x + n_y) + 4 (B B^T)_xy,  n_x = sum_tau B_x,tau
//   Q^ab = S^aT S^b = L^2 - 2 (m^a_tau + m^b_tau') + 4 (B^aT B^b)_tau,tau'
// so G runs on {0,1} operands (cheap to unpack from bits) and Q on +-1 ones,
// both exact on the matrix cores.  Per pair a < b the epilogues reduce, in
// int64,
//   D_x[d] = sum_{(x1-y1) mod L = d} G^a_xy G^b_xy (and D_y in x2 - y2),
//   trQ = sum_tau Q_tau,tau,  sum Q^2,  sum Q^4,
// without storing G or Q.
//
// 1. k_transpose turns the multispin words (64 samples per word) into one
//    bit row per sample, in two layouts: bits along tau (Pt, the K axis of G)
//    and bits along xy (Px, the K axis of Q), by 64x64 bit transposes across
//    a wavefront (six xor-shuffle butterfly stages).
// 2. k_gram_mfma: one workgroup per configuration at a time, 64x64 tiles of
//    G (upper triangle of tile pairs), all replicas at once, bucket sums in
//    LDS, flushed once per configuration; for Ltau <= 8192 on fp4 MFMAs
//    (v_mfma_scale_f32_32x32x64_f8f6f4: {0, 0.5} operands, exact in fp32).
// 3. k_overlap_mfma: panels of rows tau of one configuration, every pair in
//    turn, on fp4 MFMAs with +-1 operands (Q itself in the accumulators), the
//    row operands expanded once per panel into LDS, the column operands built
//    in registers, Q^4 summed in 64-bit integers.
// The plain per-sample form (k_*_plain) computes one matrix element per
// thread with an int32 multiply-accumulate loop over unpacked spins, one
// launch per configuration: the reference point for the batched form.
#include <algorithm>
#include <type_traits>

#include "tfim_internal.h"

namespace tfim {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));


constexpr int kMaxR = 6;       // replicas handled by the MFMA kernels
constexpr int kMaxP = kMaxR * (kMaxR - 1) / 2;

constexpr int kTP = 65;  // padded row pitch (words) of the transpose tiles
constexpr size_t kTransposeLds = (size_t)64 * kTP * 8 + 64 * 4;

__global__ void __launch_bounds__(256) k_transpose(ShapeDev sh, long long items) {
    extern __shared__ uint64_t tlds[];
    uint64_t(*tile)[kTP] = (uint64_t(*)[kTP])tlds;
    int* mrow = (int*)(tlds + 64 * kTP);
    const int L2 = sh.L2, Lt = sh.Lt, nk = sh.nk, W = sh.W, R = sh.R;
    const int S = 64 * W;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (long long item = blockIdx.x; item < items; item += gridDim.x) {
        const int g = (int)(item % sh.nx);
        const long long rest = item / sh.nx;
        const int c = (int)(rest % sh.nc);
        const int cfg = (int)(rest / sh.nc);  // (r*nk + w)*W + j
        const int j = cfg % W, rw = cfg / W, w = rw % nk, r = rw / nk;
        __syncthreads();
        if (tid < 64) {
            const int s = 64 * j + tid;
            const int i = sh.kidx[((size_t)r * S + s) * nk + w];
            mrow[tid] = (i * S + s) * R + r;
        }
        // the 64 x 64 words of the tile: all 16 loads of a thread in flight
        // at once (the loops are unrolled so that they can be)
        uint64_t v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int e = tid + 256 * k;
            const int t = e >> 6, u = e & 63, tau = 64 * c + t, xy = 64 * g + u;
            v[k] = (tau < Lt && xy < L2) ? sh.S[((size_t)cfg * Lt + tau) * L2 + xy] : 0ull;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int e = tid + 256 * k;
            tile[e >> 6][e & 63] = v[k];
        }
        __syncthreads();
        // both transposes from the tile into registers, the sixteen of each
        // wave independent chains of lane exchanges; then the tile's LDS
        // serves as the staging buffer of each output in turn (one 33 KB
        // buffer per workgroup)
        uint64_t vt[16], vx[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            vt[k] = tile[lane][wv * 16 + k];  // column u: lanes = tau
            vx[k] = tile[wv * 16 + k][lane];  // row t: lanes = xy
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            vt[k] = wave_transpose64(vt[k]);  // lane = sample bit b, bits along tau
            vx[k] = wave_transpose64(vx[k]);  // lane = sample bit b, bits along xy
        }
        __syncthreads();  // every wave has read the tile
#pragma unroll
        for (int k = 0; k < 16; ++k) tile[lane][wv * 16 + k] = vt[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int e = tid + 256 * k;
            const int b = e >> 6, u = e & 63;
            sh.Pt[((size_t)mrow[b] * sh.nc + c) * sh.nxp + 64 * g + u] = tile[b][u];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) tile[lane][wv * 16 + k] = vx[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int e = tid + 256 * k;
            const int b = e >> 6, t = e & 63, tau = 64 * c + t;
            if (tau < Lt) sh.Px[((size_t)mrow[b] * sh.nx + g) * Lt + tau] = tile[b][t];
        }
    }
}

// ---------------------------------------------------------------------------
// G tiles and the D buckets.
//
// One workgroup takes one configuration at a time.  It first counts the
// down spins n^r_x of every site row (popcount along tau) into LDS; then its
// four waves share the tile pairs (X, Y), X <= Y, of the upper triangle,
// each wave alone (no barrier inside a configuration), one wave per SIMD:
// the 2 x 2 blocks of 32 x 32 of every replica's G^r = S S^T, accumulators
// in the AGPRs, K = tau in chunks of 64, the {0,1} operands built in
// registers from each lane's bit row.  With the int32 epilogue (NARROW), up
// to 4 replicas and more configurations than CUs, two workgroups share a
// CU, two waves a SIMD (one's MFMAs run while the other builds operands),
// each wave on half a tile pair (the 2 x 1 blocks of a column half) above 2
// replicas.  The epilogue forms
// G = Ltau - 2 (n_x + n_y) + 4 (B B^T)_xy and the products G^a G^b.
//
// An element (x, y) of an off-diagonal pair stands for (y, x) too, with the
// displacements negated; its products go to U, those of the diagonal
// blocks of diagonal pairs to F, and the flush folds D[d] = F[d] + U[d] +
// U[-d mod L].  In a diagonal pair the block (rows 32.., columns 0..31) is
// the mirror of (rows 0.., columns 32..): only the latter is computed, into
// U.
//
// BLK (L a multiple of 8): tile X holds the 8 x 8 block of sites
// (bx, by) = (X mod L/8, X div L/8), row r the site (8bx + r mod 8,
// 8by + r div 8).  The 16 elements of a lane then take 4 values of x1 - y1
// (one per q mod 4) and 4 of x2 - y2 (one per q div 4), so each lane sums
// them in registers and adds 8 bucket values per pair and block, not 32.
// Otherwise tile X holds the sites 64X .. 64X + 63 and every element adds
// its own two.
//
// NARROW (BLK and Ltau <= 8192): the products and the lane sums are int32
// (24-bit multiplies), and a lane's x1 - y1 sums, the same in every block
// of a tile pair, are flushed once per pair; otherwise they are int64.
// ---------------------------------------------------------------------------
constexpr int kGramWaves = 4;
// The overlap kernel squares kSqBias + Q^2 instead of Q^2 (below), which adds
// kSqBias^2 and 2 kSqBias Q^2 per element, in 64-bit integers modulo 2^64; it
// takes the first off itself, the second is taken off here, where sum Q^2 is
// formed: the record's sum Q^4 starts from -2 kSqBias sum Q^2.
constexpr unsigned long long kSqBias = 0x4B000000ull;  // the bits of 2^23
constexpr int kNarrowLt = 8192;  // the int32 epilogue: |G| <= 2^13
// waves per SIMD: two where a wave's accumulators (RR x 2 x NV blocks of
// 16 per lane) fit in half the register file, with the int32 epilogue
constexpr int gram_wpe(int RR, int NV, bool narrow) { return narrow && RR * NV <= 4 ? 2 : 1; }

template <int RR, int NV, bool BLK, bool NARROW>
__global__ void __launch_bounds__(64 * kGramWaves)
    __attribute__((amdgpu_waves_per_eu(gram_wpe(RR, NV, NARROW), gram_wpe(RR, NV, NARROW))))
k_gram_mfma(ShapeDev sh, int cfg0, int ncfg) {
    static_assert(BLK || !NARROW, "the int32 epilogue takes the 8 x 8 site blocks");
    constexpr int PP = RR * (RR - 1) / 2;
    extern __shared__ __align__(16) uint8_t smem[];
    const int L = sh.L, L2 = sh.L2, Lt = sh.Lt, nc = sh.nc, nxp = sh.nxp;
    unsigned long long* Fb = (unsigned long long*)smem;  // [PP][2][L]
    unsigned long long* Ub = Fb + PP * 2 * L;             // [PP][2][L]
    int* nS = (int*)(Ub + PP * 2 * L);                    // [RR][nxp]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = lane & 31, h = lane >> 5, sh4 = 4 * h;
    const int ntile = sh.nx;
    const int ntp = ntile * (ntile + 1) / 2;
    const int nbl = L >> 3;
    auto site = [&](int X, int r) {
        if constexpr (BLK) return (8 * (X / nbl) + (r >> 3)) * L + 8 * (X % nbl) + (r & 7);
        return 64 * X + r;
    };
    for (int e = tid; e < 2 * PP * 2 * L; e += 64 * kGramWaves) Fb[e] = 0;  // F and U
    for (int cfg = cfg0 + blockIdx.x; cfg < cfg0 + ncfg; cfg += gridDim.x) {
        const uint64_t* const pt = sh.Pt + (size_t)cfg * RR * nc * nxp;
        for (int e = tid; e < RR * nxp; e += 64 * kGramWaves) {
            const int r = e / nxp, xy = e - r * nxp;
            int n = 0;
            for (int c = 0; c < nc; ++c) n += __popcll(pt[((size_t)r * nc + c) * nxp + xy]);
            nS[e] = n;
        }
        __syncthreads();
        // work units: tile pairs, or (NV = 1) their two column halves
        for (int unit = wv; unit < ntp * (2 / NV); unit += kGramWaves) {
            const int tp = NV == 2 ? unit : unit >> 1;
            const int v0 = NV == 2 ? 0 : (unit & 1);  // first column block
            int X = 0, rem = tp;
            while (rem >= ntile - X) { rem -= ntile - X; ++X; }
            const int Y = X + rem;
            const int sa[2] = {site(X, i), site(X, 32 + i)};
            int sb[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) sb[v] = site(Y, 32 * (v0 + v) + i);
            // NARROW: fp32 accumulators of the fp4 form (below), else int32
            using Acc = std::conditional_t<NARROW, v16f, v16i>;
            Acc acc[RR][2][NV];
#pragma unroll
            for (int r = 0; r < RR; ++r)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int q = 0; q < 16; ++q) acc[r][u][v][q] = 0;
            // The fp4 K loop: 64 values of tau per MFMA.  Lane (i, h) feeds
            // row i with the 32 bits of half h of its chunk word, element
            // 8m + j (register m, nibble j) being bit 4j + m, as the e2m1
            // values 0 and 0.5 (nibble 0 or 1: one mask per register).  The
            // row side's block scale 2^4 makes each coincidence add 4, so the
            // accumulator holds 4 (B B^T), exact in fp32 (at most 4 Ltau).
            auto kloop4 = [&](auto diagC) {
                constexpr bool kDiag = decltype(diagC)::value;
                constexpr int NB = kDiag ? 0 : NV;
                const uint32_t* const pt32 = (const uint32_t*)pt;
                auto fetch = [&](int c, uint32_t (&wa)[2][RR], uint32_t (&wb)[NV][RR]) {
#pragma unroll
                    for (int r = 0; r < RR; ++r) {
                        const size_t o = ((size_t)r * nc + c) * nxp;
#pragma unroll
                        for (int u = 0; u < 2; ++u) wa[u][r] = pt32[2 * (o + sa[u]) + h];
#pragma unroll
                        for (int v = 0; v < NB; ++v) wb[v][r] = pt32[2 * (o + sb[v]) + h];
                    }
                };
                auto chunk = [&](const uint32_t (&wa)[2][RR], const uint32_t (&wb)[NV][RR]) {
                    i32x8 A[2][RR], B[NV][RR];
#pragma unroll
                    for (int r = 0; r < RR; ++r) {
#pragma unroll
                        for (int u = 0; u < 2; ++u) A[u][r] = fp4_bits_operand(wa[u][r]);
#pragma unroll
                        for (int v = 0; v < NB; ++v) B[v][r] = fp4_bits_operand(wb[v][r]);
                    }
#pragma unroll
                    for (int r = 0; r < RR; ++r)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int v = 0; v < NV; ++v) {
                                if (kDiag && NV == 2 && u == 1 && v == 0) continue;
                                const i32x8 b = kDiag ? A[NV == 2 ? v : v0][r] : B[v][r];
                                acc[r][u][v] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                    A[u][r], b, acc[r][u][v], kFp4, kFp4, 0, kScaleRow, 0, kScaleOne);
                            }
                };
                uint32_t w0a[2][RR], w0b[NV][RR], w1a[2][RR], w1b[NV][RR];
                fetch(0, w0a, w0b);
                for (int c = 0; c + 1 < nc; c += 2) {
                    fetch(c + 1, w1a, w1b);
                    chunk(w0a, w0b);
                    fetch(min(c + 2, nc - 1), w0a, w0b);
                    chunk(w1a, w1b);
                }
                if (nc & 1) chunk(w0a, w0b);
            };
            // the K loop; kDiag: Y = X, the column rows are row rows (no
            // loads of their own) and, with both column blocks, the block
            // (1, 0) is skipped
            auto kloop = [&](auto diagC) {
                constexpr bool kDiag = decltype(diagC)::value;
                constexpr int NB = kDiag ? 0 : NV;  // column-side words loaded
                auto fetch = [&](int c, uint64_t (&wa)[2][RR], uint64_t (&wb)[NV][RR]) {
#pragma unroll
                    for (int r = 0; r < RR; ++r) {
                        const size_t o = ((size_t)r * nc + c) * nxp;
#pragma unroll
                        for (int u = 0; u < 2; ++u) wa[u][r] = pt[o + sa[u]];
#pragma unroll
                        for (int v = 0; v < NB; ++v) wb[v][r] = pt[o + sb[v]];
                    }
                };
                auto chunk = [&](const uint64_t (&wa)[2][RR], const uint64_t (&wb)[NV][RR]) {
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        i32x4 A[2][RR], B[NV][RR];
#pragma unroll
                        for (int r = 0; r < RR; ++r) {
#pragma unroll
                            for (int u = 0; u < 2; ++u)
                                A[u][r] = mfma_bits_operand<false>((uint32_t)(wa[u][r] >> (32 * ks)) >> sh4);
#pragma unroll
                            for (int v = 0; v < NB; ++v)
                                B[v][r] = mfma_bits_operand<false>((uint32_t)(wb[v][r] >> (32 * ks)) >> sh4);
                        }
#pragma unroll
                        for (int r = 0; r < RR; ++r)
#pragma unroll
                            for (int u = 0; u < 2; ++u)
#pragma unroll
                                for (int v = 0; v < NV; ++v) {
                                    if (kDiag && NV == 2 && u == 1 && v == 0) continue;
                                    const i32x4 b = kDiag ? A[NV == 2 ? v : v0][r] : B[v][r];
                                    acc[r][u][v] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[u][r], b, acc[r][u][v],
                                                                                         0, 0, 0);
                                }
                    }
                };
                // two word sets in turn, the next chunk in flight during this
                // one; one straight loop block (a fetch past the last chunk
                // reloads it) keeps the loads ahead and the waits exact
                uint64_t w0a[2][RR], w0b[NV][RR], w1a[2][RR], w1b[NV][RR];
                fetch(0, w0a, w0b);
                for (int c = 0; c + 1 < nc; c += 2) {
                    fetch(c + 1, w1a, w1b);
                    chunk(w0a, w0b);
                    fetch(min(c + 2, nc - 1), w0a, w0b);
                    chunk(w1a, w1b);
                }
                if (nc & 1) chunk(w0a, w0b);
            };
            // the K loop and the epilogue of a diagonal or an off-diagonal
            // pair, each its own straight code (the accumulators never meet
            // at a branch join)
            auto finish = [&](auto diagC) {
            constexpr bool diag = decltype(diagC)::value;
            if constexpr (NARROW)
                kloop4(diagC);
            else
                kloop(diagC);
            // epilogue, block by block
            if constexpr (NARROW) {
                // |G| <= Ltau <= 8192: a product is below 2^26 and a sum of
                // 16 of them below 2^30, so both are formed in int32 with
                // 24-bit multiplies.  The x1 - y1 buckets of a lane are the
                // same in every block of the tile, so an off-diagonal pair
                // sums them over its blocks and flushes them once.
                const int x1 = 8 * (X % nbl) + 4 * h, y1 = 8 * (Y % nbl) + (i & 7);
                int sxa[PP][4];
#pragma unroll
                for (int p = 0; p < PP; ++p)
#pragma unroll
                    for (int j = 0; j < 4; ++j) sxa[p][j] = 0;
                auto flush_x = [&](unsigned long long* Db) {
#pragma unroll
                    for (int p = 0; p < PP; ++p)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            atomicAdd(&Db[(p * 2 + 0) * L + (x1 + j - y1 + L) % L],
                                      (unsigned long long)(long long)sxa[p][j]);
                            sxa[p][j] = 0;
                        }
                };
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    int rn[RR][16];  // 2 n^r of the rows of this lane's elements
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const int xs = site(X, 32 * u + 8 * (q >> 2) + 4 * h + (q & 3));
#pragma unroll
                        for (int r = 0; r < RR; ++r) rn[r][q] = 2 * nS[r * nxp + xs];
                    }
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const int V = v0 + v;
                        if (diag && NV == 2 && u == 1 && V == 0) continue;
                        unsigned long long* Db = (diag && (NV == 1 || u == V)) ? Fb : Ub;
                        const int x2 = 8 * (X / nbl) + 4 * u, y2 = 8 * (Y / nbl) + ((32 * V + i) >> 3);
                        int G[RR][16];
#pragma unroll
                        for (int r = 0; r < RR; ++r) {
                            const int nb = Lt - 2 * nS[r * nxp + sb[v]];
#pragma unroll
                            for (int q = 0; q < 16; ++q) G[r][q] = nb - rn[r][q] + (int)acc[r][u][v][q];
                        }
                        int p = 0;
#pragma unroll
                        for (int a = 0; a < RR; ++a)
#pragma unroll
                            for (int b = a + 1; b < RR; ++b, ++p) {
                                int sy[4] = {0, 0, 0, 0};
#pragma unroll
                                for (int q = 0; q < 16; ++q) {
                                    const int hv = __mul24(G[a][q], G[b][q]);
                                    sxa[p][q & 3] += hv;
                                    sy[q >> 2] += hv;
                                }
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    atomicAdd(&Db[(p * 2 + 1) * L + (x2 + j - y2 + L) % L],
                                              (unsigned long long)(long long)sy[j]);
                            }
                        if (diag) flush_x(Db);
                    }
                }
                if (!diag) flush_x(Ub);
            } else
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int V = v0 + v;  // column block in the tile
                    if (diag && NV == 2 && u == 1 && V == 0) continue;
                    unsigned long long* Db = (diag && (NV == 1 || u == V)) ? Fb : Ub;
                    const int ys = sb[v];  // this lane's column site
                    int nb[RR];
#pragma unroll
                    for (int r = 0; r < RR; ++r) nb[r] = Lt - 2 * nS[r * nxp + ys];
                    // G^r of element q (|G| <= Ltau <= 2^16)
                    auto gram = [&](int q, int (&G)[RR]) {
                        const int xs = site(X, 32 * u + 8 * (q >> 2) + 4 * h + (q & 3));
#pragma unroll
                        for (int r = 0; r < RR; ++r) G[r] = nb[r] - 2 * nS[r * nxp + xs] + 4 * acc[r][u][v][q];
                    };
                    if constexpr (BLK) {
                        // x1 - y1 by q mod 4 and x2 - y2 by q div 4, all sites valid
                        const int col = 32 * V + i;
                        const int y1 = 8 * (Y % nbl) + (col & 7), y2 = 8 * (Y / nbl) + (col >> 3);
                        const int x1 = 8 * (X % nbl) + 4 * h, x2 = 8 * (X / nbl) + 4 * u;
                        int Gq[RR][16];
#pragma unroll
                        for (int q = 0; q < 16; ++q) {
                            int G[RR];
                            gram(q, G);
#pragma unroll
                            for (int r = 0; r < RR; ++r) Gq[r][q] = G[r];
                        }
                        int p = 0;
#pragma unroll
                        for (int a = 0; a < RR; ++a)
#pragma unroll
                            for (int b = a + 1; b < RR; ++b, ++p) {
                                long long sx[4] = {0, 0, 0, 0}, sy[4] = {0, 0, 0, 0};
#pragma unroll
                                for (int q = 0; q < 16; ++q) {
                                    const long long hv = (long long)Gq[a][q] * Gq[b][q];
                                    sx[q & 3] += hv;
                                    sy[q >> 2] += hv;
                                }
#pragma unroll
                                for (int j = 0; j < 4; ++j) {
                                    atomicAdd(&Db[(p * 2 + 0) * L + (x1 + j - y1 + L) % L], (unsigned long long)sx[j]);
                                    atomicAdd(&Db[(p * 2 + 1) * L + (x2 + j - y2 + L) % L], (unsigned long long)sy[j]);
                                }
                            }
                    } else {
                        const int y = ys;
#pragma unroll
                        for (int q = 0; q < 16; ++q) {
                            const int x = site(X, 32 * u + 8 * (q >> 2) + 4 * h + (q & 3));
                            if (x >= L2 || y >= L2) continue;
                            int G[RR];
                            gram(q, G);
                            const int dx = (x % L - y % L + L) % L, dy = (x / L - y / L + L) % L;
                            int p = 0;
#pragma unroll
                            for (int a = 0; a < RR; ++a)
#pragma unroll
                                for (int b = a + 1; b < RR; ++b, ++p) {
                                    const unsigned long long hv = (unsigned long long)((long long)G[a] * G[b]);
                                    atomicAdd(&Db[(p * 2 + 0) * L + dx], hv);
                                    atomicAdd(&Db[(p * 2 + 1) * L + dy], hv);
                                }
                        }
                    }
                }
            };
            if (X == Y)
                finish(std::true_type{});
            else
                finish(std::false_type{});
        }
        __syncthreads();
        // D[d] = F[d] + U[d] + U[-d]; sum Q^2 = sum_xy G^a_xy G^b_xy =
        // sum_d D_x[d] (one workgroup holds all of this configuration's
        // buckets)
        const int rl = 2 * L + 3;
        for (int e = tid; e < PP * 2 * L; e += 64 * kGramWaves) {
            const int d = e % L;
            Fb[e] += Ub[e] + Ub[e - d + (L - d) % L];
        }
        __syncthreads();
        if (tid < PP) {
            unsigned long long q2 = 0;
            for (int d = 0; d < L; ++d) q2 += Fb[(tid * 2 + 0) * L + d];
            int64_t* const rp = sh.rec + ((size_t)cfg * PP + tid) * rl + 2 * L;
            rp[1] = (int64_t)q2;
            rp[2] = (int64_t)(0ull - 2 * kSqBias * q2);  // what the overlap kernel's squares add too much
        }
        for (int e = tid; e < PP * 2 * L; e += 64 * kGramWaves) {
            const int p = e / (2 * L), d = e % (2 * L);
            sh.rec[((size_t)cfg * PP + p) * rl + d] = (int64_t)Fb[e];
        }
        __syncthreads();
        for (int e = tid; e < 2 * PP * 2 * L; e += 64 * kGramWaves) Fb[e] = 0;
    }
}

// ---------------------------------------------------------------------------
// Q tiles: trQ and sum Q^4 of every replica pair a < b (sum Q^2 comes from
// the Gram buckets).
//
// A work item is a panel of 32 NU rows tau of one configuration, for every
// pair (a, b) in turn.  For each a the workgroup expands the panel's rows of
// replica a once into LDS, as fp4 operands of +-1 (16 bytes per lane, block
// and chunk: the order in which the lanes read them back, without bank
// conflicts); then each wave takes 64-column tiles tau' of each b > a alone,
// with no barrier: NU x 2 blocks of 32 x 32, the column operands built in
// registers from the bit rows (7 VALU per operand).  In chunk g lane (i, h)
// of a block feeds row i with the 32 bits of half h of its word, in the same
// order on both sides.  The fp32 accumulator is Q itself (|Q| <= L^2 <= 2^10,
// exact): spins past L^2 and rows past Ltau are 0 on the row side, columns
// past Ltau are +-0, so every element may enter the sum and no tile needs a
// form of its own.  trQ = sum_tau (L^2 - 2 popcount(a ^ b)) needs no product.
//
// Two workgroups per CU, two waves per SIMD: one wave's MFMAs run while the
// other forms Q^4, two instructions per element: 2^23 + Q^2 in fp32 (exact),
// whose bits are kSqBias + Q^2, and a 32 x 32 + 64 bit multiply-add.
//
// At L = 24, Ltau = 2048, 4 replicas and 1024 configurations: 5.6 ms (3.7 of
// them at the rate of the fp4 MFMAs at the 1.9 GHz that the power limit
// leaves), against 12.8 ms with int8 MFMAs, every wave building both sides'
// operands for two pairs, rank-one corrections in a K step of their own and
// three instructions per Q^4.  One workgroup per item instead of a
// persistent grid: 6.4 -> 6.0 ms (the dispatcher evens out the XCDs).
// ---------------------------------------------------------------------------
constexpr int kOverlapWaves = 4;

// NX: 0 for one chunk (L <= 8), 1 for an even number of them, 2 for an odd one.
template <int NU, int NX>
__global__ void __launch_bounds__(64 * kOverlapWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_overlap_mfma(ShapeDev sh, int cfg0, int ncfg, int npanel, int nsplit, int grouped) {
    extern __shared__ __align__(16) uint8_t smem[];
    i32x4* const Aop = (i32x4*)smem;  // [nx][NU][64]
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L2 = sh.L2, Lt = sh.Lt, nx = sh.nx, R = sh.R, P = sh.P;
    const int ntt = (Lt + 63) / 64;
    const int rl = 2 * sh.L + 3;
    const int ipc = npanel * nsplit;
    // grouped: workgroup b (on XCD b mod 8) takes the items of the
    // configurations b mod 8, b mod 8 + 8, ..., so that a configuration's
    // rows are read through one L2; otherwise the items in plain order
    const int ng = grouped ? 8 : 1, grp = grouped ? (int)blockIdx.x & 7 : 0;
    const int k = (int)blockIdx.x / ng;
    {
        if (grp + ng * (k / ipc) >= ncfg) return;
        const int cfg = cfg0 + grp + ng * (k / ipc);
        const int part = k % ipc / npanel, row0 = 32 * NU * (k % ipc % npanel);
        const uint64_t* const px = sh.Px + (size_t)cfg * R * nx * Lt;
        // uniform descriptor (readfirstlane is a signed int: cast before widening)
        const uint32_t base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)px);
        const uint32_t base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)px >> 32));
        const __amdgpu_buffer_rsrc_t words = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(((uint64_t)base_hi << 32) | base_lo), (short)0, R * nx * Lt * 8, 0x00020000);
        const int voff = 8 * i + 4 * h;
        int p = 0;
        for (int a = 0; a + 1 < R; ++a) {
            __syncthreads();  // the waves have read the previous panel
            for (int e = tid; e < nx * NU * 64; e += 64 * kOverlapWaves) {
                const int g = e / (NU * 64), row = row0 + 32 * ((e >> 6) % NU) + (e & 31), hh = (e >> 5) & 1;
                const bool ok = row < Lt;
                const uint32_t x = ok ? ((const uint32_t*)px)[2 * (((size_t)a * nx + g) * Lt + row) + hh] : 0u;
                const int nv = ok ? L2 - 64 * g - 32 * hh : 0;  // spins of this half
                const uint32_t vm = nv >= 32 ? ~0u : (nv > 0 ? (1u << nv) - 1u : 0u);
                i32x4 o;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    o[m] = (int)(((x << (3 - m)) & 0x88888888u) | (((vm >> m) & 0x11111111u) << 1));
                Aop[e] = o;
            }
            __syncthreads();
            for (int b = a + 1; b < R; ++b, ++p) {
                unsigned long long s4 = 0;
                int tr = 0;
                if (part == 0) {
                    for (int e = tid; e < nx * NU * 32; e += 64 * kOverlapWaves) {
                        const int g = e / (NU * 32), row = row0 + e % (NU * 32);
                        if (row < Lt)
                            tr += (g == 0 ? L2 : 0) - 2 * (int)__popcll(px[((size_t)a * nx + g) * Lt + row] ^
                                                                         px[((size_t)b * nx + g) * Lt + row]);
                    }
                }
                const int step = kOverlapWaves * nsplit;
                // the words of chunk g of tile t (kept below the last tile, so
                // that the scalar offset stays inside the descriptor and rows
                // past its end read 0)
                auto fetch = [&](int t, int g, uint32_t (&w)[2]) {
                    const int so = ((b * nx + g) * Lt + 64 * min(t, ntt - 1)) * 8;
                    w[0] = __builtin_amdgcn_raw_buffer_load_b32(words, voff, so, 0);
                    w[1] = __builtin_amdgcn_raw_buffer_load_b32(words, voff + 256, so, 0);
                };
                // Two operand sets and two word sets in turn, by the parity of
                // the chunk: while a chunk's MFMAs run, the next one's row
                // operands come from LDS, its column operands are built, and
                // the words of the chunk after the next but one are loaded
                // (those of the next tile's chunks 0 and 1 at the end).
                f32x16 acc[NU][2];
                i32x4 A0[NU], A1[NU], B0[2], B1[2];
                uint32_t w0[2], w1[2];
                int T = part * kOverlapWaves + wv;
                auto load = [&](int t, int g, uint32_t (&w)[2], int slot, i32x4 (&A)[NU], i32x4 (&B)[2]) {
#pragma unroll
                    for (int u = 0; u < NU; ++u) A[u] = Aop[(g * NU + u) * 64 + lane];
#pragma unroll
                    for (int v = 0; v < 2; ++v)
                        B[v] = fp4_signs_operand(w[v], 64 * t + 32 * v + i < Lt ? 0x22222222u : 0u);
                    const bool here = g + 2 < nx;
                    fetch(here ? t : t + step, here ? g + 2 : min(slot, nx - 1), w);
                };
                auto mul = [&](const i32x4 (&A)[NU], const i32x4 (&B)[2], auto firstC) {
                    constexpr bool kFirst = decltype(firstC)::value;
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int v = 0; v < 2; ++v)
                            acc[u][v] = mfma_fp4(fp4_wide(A[u]), fp4_wide(B[v]), kFirst ? f32x16{} : acc[u][v]);
                };
                fetch(T, 0, w0);
                fetch(T, min(1, nx - 1), w1);
                load(T, 0, w0, 0, A0, B0);
                for (; T < ntt; T += step) {
                    if constexpr (NX > 0) load(T, 1, w1, 1, A1, B1);
                    mul(A0, B0, std::true_type{});
                    if constexpr (NX > 0) {
                        int g = 1;
                        for (; g + 2 < nx; g += 2) {
                            load(T, g + 1, w0, 0, A0, B0);
                            mul(A1, B1, std::false_type{});
                            load(T, g + 2, w1, 1, A1, B1);
                            mul(A0, B0, std::false_type{});
                        }
                        if constexpr (NX == 2) load(T, g + 1, w0, 0, A0, B0);
                        mul(A1, B1, std::false_type{});
                        if constexpr (NX == 2) mul(A0, B0, std::false_type{});
                    }
                    load(T + step, 0, w0, 0, A0, B0);
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int v = 0; v < 2; ++v)
#pragma unroll
                            for (int q = 0; q < 16; ++q) {
                                // 2^23 + Q^2 is exact; its bits are kSqBias + Q^2
                                const uint32_t q2 =
                                    __float_as_uint(__builtin_fmaf(acc[u][v][q], acc[u][v][q], 8388608.0f));
                                s4 += (unsigned long long)q2 * q2;
                            }
                    s4 -= (unsigned long long)(NU * 32) * kSqBias * kSqBias;
                }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    s4 += (unsigned long long)__shfl_xor((long long)s4, off, 64);
                    tr += __shfl_xor(tr, off, 64);
                }
                if (lane == 0) {
                    unsigned long long* rp = (unsigned long long*)(sh.rec + ((size_t)cfg * P + p) * rl);
                    if (part == 0) atomicAdd(rp + 2 * sh.L, (unsigned long long)(long long)tr);
                    atomicAdd(rp + 2 * sh.L + 2, s4);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Plain per-sample form: one configuration per launch, one matrix element
// per thread, int32 multiply-accumulate over unpacked +-1 spins.
// ---------------------------------------------------------------------------
// +-1 spins t = 0..63 of a 64-bit row word: 1 - 2 bit_t, 0 past n valid bits.
__device__ __forceinline__ int dot64(uint64_t a, uint64_t b, int n) {
    int acc = 0;
    for (int t = 0; t < n; ++t)
        acc += (1 - 2 * (int)((a >> t) & 1ull)) * (1 - 2 * (int)((b >> t) & 1ull));
    return acc;
}

__global__ void __launch_bounds__(256) k_gram_plain(ShapeDev sh, int cfg) {
    __shared__ unsigned long long Dblk[kMaxP * 2 * 32];
    const int L = sh.L, L2 = sh.L2, R = sh.R, P = sh.P;
    for (int e = threadIdx.x; e < P * 2 * L; e += blockDim.x) Dblk[e] = 0;
    __syncthreads();
    const long long el = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (el < (long long)L2 * L2) {
        const int x = (int)(el / L2), y = (int)(el % L2);
        int G[kMaxR];
        for (int r = 0; r < R; ++r) {
            const size_t m = (size_t)cfg * R + r;
            int acc = 0;
            for (int c = 0; c < sh.nc; ++c)
                acc += dot64(sh.Pt[(m * sh.nc + c) * sh.nxp + x], sh.Pt[(m * sh.nc + c) * sh.nxp + y],
                             min(64, sh.Lt - 64 * c));
            G[r] = acc;
        }
        const int dx = ((x % L) - (y % L) + L) % L, dy = ((x / L) - (y / L) + L) % L;
        int p = 0;
        for (int a = 0; a < R; ++a)
            for (int b = a + 1; b < R; ++b, ++p) {
                const unsigned long long h = (unsigned long long)((long long)G[a] * G[b]);
                atomicAdd(&Dblk[(p * 2 + 0) * L + dx], h);
                atomicAdd(&Dblk[(p * 2 + 1) * L + dy], h);
            }
    }
    __syncthreads();
    const int rl = 2 * L + 3;
    for (int e = threadIdx.x; e < P * 2 * L; e += blockDim.x)
        atomicAdd((unsigned long long*)&sh.rec[((size_t)cfg * P + e / (2 * L)) * rl + e % (2 * L)], Dblk[e]);
}

__global__ void __launch_bounds__(256) k_overlap_plain(ShapeDev sh, int cfg) {
    __shared__ unsigned long long red[kMaxP * 3];
    const int Lt = sh.Lt, L2 = sh.L2, R = sh.R, P = sh.P;
    for (int e = threadIdx.x; e < P * 3; e += blockDim.x) red[e] = 0;
    __syncthreads();
    const long long el = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (el < (long long)Lt * Lt) {
        const int tau = (int)(el / Lt), tau2 = (int)(el % Lt);
        int p = 0;
        for (int a = 0; a < R; ++a)
            for (int b = a + 1; b < R; ++b, ++p) {
                const size_t ma = (size_t)cfg * R + a, mb = (size_t)cfg * R + b;
                int q = 0;
                for (int g = 0; g < sh.nx; ++g)
                    q += dot64(sh.Px[(ma * sh.nx + g) * Lt + tau], sh.Px[(mb * sh.nx + g) * Lt + tau2],
                               min(64, L2 - 64 * g));
                const long long q2 = (long long)q * q;
                atomicAdd(&red[p * 3 + 1], (unsigned long long)q2);
                atomicAdd(&red[p * 3 + 2], (unsigned long long)(q2 * q2));
                if (tau == tau2) atomicAdd(&red[p * 3 + 0], (unsigned long long)(long long)q);
            }
    }
    __syncthreads();
    const int rl = 2 * sh.L + 3;
    for (int e = threadIdx.x; e < P * 3; e += blockDim.x)
        atomicAdd((unsigned long long*)&sh.rec[((size_t)cfg * P + e / 3) * rl + 2 * sh.L + e % 3], red[e]);
}

// Debug dump of G^a, G^b (L2 x L2) and Q^ab (Ltau x Ltau) of one configuration.
__global__ void k_dump(ShapeDev sh, int cfg, int a, int b) {
    const int L2 = sh.L2, Lt = sh.Lt, R = sh.R;
    const long long n1 = (long long)L2 * L2, n = 2 * n1 + (long long)Lt * Lt;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (long long)gridDim.x * blockDim.x) {
        int acc = 0;
        if (e < 2 * n1) {
            const int r = e < n1 ? a : b;
            const long long f = e % n1;
            const int x = (int)(f / L2), y = (int)(f % L2);
            const size_t m = (size_t)cfg * R + r;
            for (int c = 0; c < sh.nc; ++c)
                acc += dot64(sh.Pt[(m * sh.nc + c) * sh.nxp + x], sh.Pt[(m * sh.nc + c) * sh.nxp + y],
                             min(64, Lt - 64 * c));
        } else {
            const long long f = e - 2 * n1;
            const int tau = (int)(f / Lt), tau2 = (int)(f % Lt);
            const size_t ma = (size_t)cfg * R + a, mb = (size_t)cfg * R + b;
            for (int g = 0; g < sh.nx; ++g)
                acc += dot64(sh.Px[(ma * sh.nx + g) * Lt + tau], sh.Px[(mb * sh.nx + g) * Lt + tau2],
                             min(64, L2 - 64 * g));
        }
        sh.dump[e] = acc;
    }
}

// A[i][h][d] = sum over samples and pairs of the records' D_x (h=0), D_y (h=1).
__global__ void k_buckets(ShapeDev sh) {
    const int L = sh.L, S = 64 * sh.W, P = sh.P, rl = 2 * L + 3;
    const int n = sh.nk * 2 * L;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const int i = e / (2 * L), hd = e % (2 * L);
        long long acc = 0;
        for (int s = 0; s < S; ++s)
            for (int p = 0; p < P; ++p) acc += sh.rec[((size_t)(i * S + s) * P + p) * rl + hd];
        sh.buckets[e] = acc;
    }
}

size_t gram_lds(int RR, int L) {
    const int PP = RR * (RR - 1) / 2;
    const int nxp = 64 * ((L * L + 63) / 64);
    return (size_t)2 * PP * 2 * L * 8 + (size_t)RR * nxp * 4;
}
// Panels of 128 rows where Ltau fills them, else of 64.  The items of a short
// range are split along the columns until they fill two workgroups per CU.
template <int NU, int NX>
hipError_t launch_overlap_nx(const ShapeDev& sh, int cfg0, int ncfg, int ncu, hipStream_t st) {
    static bool lds_set = false;
    if (!lds_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_overlap_mfma<NU, NX>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 16 * NU * 64 * 16);
        if (e != hipSuccess) return e;
        lds_set = true;
    }
    const int npanel = (sh.Lt + 32 * NU - 1) / (32 * NU), ntt = (sh.Lt + 63) / 64;
    int nsplit = 1;
    while ((long long)ncfg * npanel * nsplit < 2 * ncu && kOverlapWaves * nsplit < ntt) nsplit *= 2;
    const bool grouped = ncu % 8 == 0 && ncfg >= 128;
    const long long items = (long long)ncfg * npanel * nsplit;
    const long long grid = grouped ? (long long)((ncfg + 7) / 8) * 8 * npanel * nsplit : items;
    hipLaunchKernelGGL((k_overlap_mfma<NU, NX>), dim3((unsigned)grid), dim3(64 * kOverlapWaves), (size_t)sh.nx * NU * 64 * 16, st, sh,
                       cfg0, ncfg, npanel, nsplit, (int)grouped);
    return hipGetLastError();
}

template <int NU>
hipError_t launch_overlap_nu(const ShapeDev& sh, int cfg0, int ncfg, int ncu, hipStream_t st) {
    if (sh.nx == 1) return launch_overlap_nx<NU, 0>(sh, cfg0, ncfg, ncu, st);
    return sh.nx % 2 == 0 ? launch_overlap_nx<NU, 1>(sh, cfg0, ncfg, ncu, st)
                          : launch_overlap_nx<NU, 2>(sh, cfg0, ncfg, ncu, st);
}

hipError_t launch_overlap(const ShapeDev& sh, int cfg0, int ncfg, int ncu, hipStream_t st) {
    const int n64 = (sh.Lt + 63) / 64;
    return n64 == 1 || n64 == 3 ? launch_overlap_nu<2>(sh, cfg0, ncfg, ncu, st)
                                : launch_overlap_nu<4>(sh, cfg0, ncfg, ncu, st);
}

template <int RR>
hipError_t launch_mfma(const ShapeDev& sh, int cfg0, int ncfg, hipStream_t st) {
    int dev = 0, ncu = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    // a wave holds every replica's G of its unit: 64 x 64 up to 4 replicas,
    // 64 x 32 above; with the int32 epilogue and more configurations than
    // CUs two waves share a SIMD, each with at most 128 accumulators (64 x 64
    // for 2 replicas, else 64 x 32)
    constexpr int NV = RR <= 4 ? 2 : 1;
    constexpr int NVn = RR <= 2 ? 2 : 1;
    static bool lds_set = false;
    if (!lds_set) {
        for (const void* f : {(const void*)k_gram_mfma<RR, NVn, true, true>, (const void*)k_gram_mfma<RR, NV, true, true>,
                              (const void*)k_gram_mfma<RR, NV, true, false>, (const void*)k_gram_mfma<RR, NV, false, false>}) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)gram_lds(RR, 32));
            if (e != hipSuccess) return e;
        }
        lds_set = true;
    }
    const int ggrid = std::min(ncfg, ncu);
    auto narrow = [&](auto nvC) {
        constexpr int nv = decltype(nvC)::value;
        hipLaunchKernelGGL((k_gram_mfma<RR, nv, true, true>), dim3(std::min(ncfg, gram_wpe(RR, nv, true) * ncu)),
                           dim3(64 * kGramWaves), gram_lds(RR, sh.L), st, sh, cfg0, ncfg);
    };
    if (sh.L % 8 == 0 && sh.Lt <= kNarrowLt && ncfg > ncu)
        narrow(std::integral_constant<int, NVn>{});
    else if (sh.L % 8 == 0 && sh.Lt <= kNarrowLt)
        narrow(std::integral_constant<int, NV>{});
    else if (sh.L % 8 == 0)
        hipLaunchKernelGGL((k_gram_mfma<RR, NV, true, false>), dim3(ggrid), dim3(64 * kGramWaves), gram_lds(RR, sh.L),
                           st, sh, cfg0, ncfg);
    else
        hipLaunchKernelGGL((k_gram_mfma<RR, NV, false, false>), dim3(ggrid), dim3(64 * kGramWaves),
                           gram_lds(RR, sh.L), st, sh, cfg0, ncfg);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_overlap(sh, cfg0, ncfg, ncu, st);
}

}  // namespace

bool measure_ok(const ShapeDev& sh) { return sh.R >= 2 && sh.R <= kMaxR && sh.L <= 32; }


hipError_t launch_transpose(const ShapeDev& sh, hipStream_t st) {
    const long long items = (long long)sh.R * sh.nk * sh.W * sh.nc * sh.nx;
    const int grid = (int)std::min<long long>(items, 8192);
    static bool lds_set = false;  // above 64 KiB of LDS per workgroup
    if (!lds_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_transpose,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)kTransposeLds);
        if (e != hipSuccess) return e;
        lds_set = true;
    }
    hipLaunchKernelGGL(k_transpose, dim3(grid), dim3(256), kTransposeLds, st, sh, items);
    return hipGetLastError();
}

hipError_t launch_measure(const ShapeDev& sh, int mode, int cfg0, int ncfg, hipStream_t st) {
    if (ncfg <= 0) return hipSuccess;
    if (mode == 0) {
        switch (sh.R) {
            case 2: return launch_mfma<2>(sh, cfg0, ncfg, st);
            case 3: return launch_mfma<3>(sh, cfg0, ncfg, st);
            case 4: return launch_mfma<4>(sh, cfg0, ncfg, st);
            case 5: return launch_mfma<5>(sh, cfg0, ncfg, st);
            case 6: return launch_mfma<6>(sh, cfg0, ncfg, st);
            default: return hipErrorInvalidValue;
        }
    }
    for (int cfg = cfg0; cfg < cfg0 + ncfg; ++cfg) {
        const long long ng = (long long)sh.L2 * sh.L2, nq = (long long)sh.Lt * sh.Lt;
        hipLaunchKernelGGL(k_gram_plain, dim3((unsigned)((ng + 255) / 256)), dim3(256), 0, st, sh, cfg);
        hipLaunchKernelGGL(k_overlap_plain, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, st, sh, cfg);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_buckets(const ShapeDev& sh, hipStream_t st) {
    hipLaunchKernelGGL(k_buckets, dim3(16), dim3(256), 0, st, sh);
    return hipGetLastError();
}

hipError_t launch_dump(const ShapeDev& sh, int cfg, int a, int b, hipStream_t st) {
    hipLaunchKernelGGL(k_dump, dim3(1024), dim3(256), 0, st, sh, cfg, a, b);
    return hipGetLastError();
}

}  // namespace tfim
