// Measurement: replica Gram / overlap integers on MFMA, fused int64 reductions.
//
// Paper: arXiv:2310.07486, Methods, "One-time observables" (M_xy, M-hat, the
// susceptibilities chi^(2), F^(2) and the second-moment length) with the
// tau average of "The Trotter-Suzuki formula" and the replica estimators of
// "Simulation details".
//
// For configuration (k-index i, sample s) and replica r, S^r is the
// L^2 x Ltau matrix of +-1 spins of walker kidx^-1[i] (lane s), and
//   G^r = S S^T (L^2 x L^2, sums over tau),  Q^ab = S^aT S^b (Ltau x Ltau, over sites),
// both exact on the matrix cores, on fp4 operands of +-1 built from the bits with
// fp32 accumulators (G of Ltau > 8192 on int8 operands {0,1}).  Per pair a < b the
// epilogues reduce, in int64,
//   D_x[d] = sum_{(x1-y1) mod L = d} G^a_xy G^b_xy (and D_y in x2 - y2),
//   trQ = sum_tau Q_tau,tau,  sum Q^2,  sum Q^4,
// without storing G or Q.
//
// 1. k_transpose turns the multispin words (64 samples per word) into one
//    bit row per sample, in two layouts: bits along tau (Pt, the K axis of G)
//    and bits along the sites (Px, the K axis of Q), by 64x64 bit transposes in the
//    registers of a lane.
// 2. k_gram_mfma: 64x64 tiles of G (upper triangle of tile pairs), the
//    replicas one after the other on fp4 MFMAs and kept as int16, bucket sums
//    in LDS; k_gram_wide (int8 MFMAs, int64 products) for Ltau > 8192.
// 3. k_overlap_mfma: panels of rows tau of one configuration, every pair in
//    turn, on fp4 MFMAs with +-1 operands (Q itself in the accumulators), the
//    row operands expanded once per panel into LDS, the column operands built
//    in registers, Q^4 summed in 64-bit integers.
// The plain per-sample form (k_*_plain) computes one matrix element per
// thread with an int32 multiply-accumulate loop over unpacked spins, one
// launch per configuration: the reference point for the batched form.
#include <algorithm>
#include <type_traits>

#include "gram_tile.h"
#include "tfim_internal.h"

namespace tfim {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kMaxR = 6;       // replicas handled by the MFMA kernels
constexpr int kMaxP = kMaxR * (kMaxR - 1) / 2;

// 64 x 64 bits in the registers of a lane, row t in lo[t], hi[t]: row b becomes
// bit b of every row.  Halves by renaming, 16 and 8 by byte permutes, then two
// operations per dword and stage.
__device__ __forceinline__ void lane_transpose64(uint32_t (&lo)[64], uint32_t (&hi)[64]) {
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        const uint32_t x = hi[t];
        hi[t] = lo[t + 32];
        lo[t + 32] = x;
    }
    auto stage = [](uint32_t (&x)[64], int j) {
#pragma unroll
        for (int t = 0; t < 64; ++t)
            if (!(t & j)) {
                const uint32_t a = x[t], b = x[t + j];
                if (j == 16) {
                    x[t] = __builtin_amdgcn_perm(b, a, 0x05040100);
                    x[t + j] = __builtin_amdgcn_perm(b, a, 0x07060302);
                } else if (j == 8) {
                    x[t] = __builtin_amdgcn_perm(b, a, 0x06020400);
                    x[t + j] = __builtin_amdgcn_perm(b, a, 0x07030501);
                } else {
                    const uint32_t m = j == 4 ? 0x0f0f0f0fu : j == 2 ? 0x33333333u : 0x55555555u;
                    x[t] = (a & m) | ((b << j) & ~m);
                    x[t + j] = ((a >> j) & m) | (b & ~m);
                }
            }
    };
    stage(lo, 16), stage(hi, 16);
    stage(lo, 8), stage(hi, 8);
    stage(lo, 4), stage(hi, 4);
    stage(lo, 2), stage(hi, 2);
    stage(lo, 1), stage(hi, 1);
}

// Both layouts of the rows (Pt, Px) from the multispin words, one wave per tile
// of 64 site slots x 64 tau.  A lane reads the 64 words of its site and
// transposes them in registers: row b is sample b's, bits along tau, and the
// wave's 64 lanes write it as 512 bytes of Pt.  For Px a lane needs the 64 words
// of a tau: they change places through LDS, the low and the high dwords one
// after the other (17 KB, eight waves per CU).  Bound by memory, of which it
// reads the words once and writes them twice: L = 24, Ltau = 2048, 128
// configurations of 64 lanes 1026 us (exchanges between lanes) -> 777; copy rate 750.
constexpr int kTP = 68;  // dwords from site to site in LDS: quads of lanes on all banks
__global__ void __launch_bounds__(64, 2) k_transpose(ShapeDev sh, long long items) {
    __shared__ __align__(16) uint32_t swap[64 * kTP];
    const int L2 = sh.L2, Lt = sh.Lt, nk = sh.nk, W = sh.W, R = sh.R;
    const int S = 64 * W;
    const int lane = threadIdx.x;
    // Workgroup b runs on XCD b mod 8: an XCD takes all nx tiles of one
    // (configuration, chunk) in turn, since they share cache lines of S (a
    // tile reads 32-byte pieces of every tau plane).
    const int xcd = blockIdx.x & 7;
    for (long long n = blockIdx.x >> 3;; n += gridDim.x >> 3) {
        const int g = (int)(n % sh.nx);
        const long long rest = n / sh.nx * 8 + xcd;
        if (rest * sh.nx >= items) break;
        const int c = (int)(rest % sh.nc);
        const int cfg = (int)(rest / sh.nc);  // (r*nk + w)*W + j
        const int j = cfg % W, rw = cfg / W, w = rw % nk, r = rw / nk;
        const int smp = 64 * j + lane;
        const int mrow = (sh.kidx[((size_t)r * S + smp) * nk + w] * S + smp) * R + r;
        int x1, x2;
        slot_site(sh.L, 64 * g + lane, x1, x2);
        const bool site_ok = 64 * g + lane < L2;
        const int site = site_ok ? x1 + sh.L * x2 : 0;
        const uint64_t* const words = sh.S + ((size_t)cfg * Lt + 64 * (size_t)c) * L2;
        const int nt = min(64, Lt - 64 * c);
        uint32_t lo[64], hi[64];
#pragma unroll
        for (int t = 0; t < 64; ++t) {
            const uint64_t v = (words + (size_t)min(t, nt - 1) * L2)[site];
            lo[t] = (uint32_t)v;
            hi[t] = (uint32_t)(v >> 32);
        }
        // padding: zero
        if (nt < 64)
#pragma unroll
            for (int t = 1; t < 64; ++t)
                if (t >= nt) lo[t] = hi[t] = 0;
        if (64 * (g + 1) > L2)
#pragma unroll
            for (int t = 0; t < 64; ++t) {
                lo[t] = site_ok ? lo[t] : 0;
                hi[t] = site_ok ? hi[t] : 0;
            }
        uint32_t xlo[64], xhi[64];
        auto put = [&](const uint32_t (&v)[64]) {
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 64; t += 4)
                *(uint4*)(swap + kTP * lane + t) = uint4{v[t], v[t + 1], v[t + 2], v[t + 3]};
            __syncthreads();
        };
        auto get = [&](uint32_t (&x)[64]) {
#pragma unroll
            for (int u = 0; u < 64; ++u) x[u] = swap[kTP * u + lane];
        };
        put(lo);
        get(xlo);
        put(hi);
        lane_transpose64(lo, hi);
#pragma unroll
        for (int b = 0; b < 64; ++b) {
            uint64_t* const row =
                sh.Pt + ((size_t)__builtin_amdgcn_readlane(mrow, b) * sh.nc + c) * sh.nxp + 64 * g;
            row[lane] = (uint64_t)hi[b] << 32 | lo[b];
        }
        get(xhi);
        lane_transpose64(xlo, xhi);
        if (lane < nt)
#pragma unroll
            for (int b = 0; b < 64; ++b) {
                uint64_t* const row =
                    sh.Px + ((size_t)__builtin_amdgcn_readlane(mrow, b) * sh.nx + g) * Lt + 64 * c;
                row[lane] = (uint64_t)xhi[b] << 32 | xlo[b];
            }
    }
}

// ---------------------------------------------------------------------------
// G tiles and the D buckets (Ltau <= 8192).
//
// Tiles X <= Y of the upper triangle, 2 x 2 blocks of 4 x 8 sites each, in
// which the 16 elements q of a lane take four values of x1 - y1 (by q mod 4)
// and four of x2 - y2 (by q div 4).
//
// Each wave works alone on one tile (no barrier inside it), the replicas in
// turn: the K loop of one replica runs on 64 fp32 accumulators (fp4 operands
// of +-1 built in registers from the bit rows along tau, 7 VALU per operand
// and one operand per MFMA), and its G is kept as packed int16 in 32
// registers, so that all replicas of the tile fit at two waves per SIMD.  The
// accumulators start from 1.5 2^23: the low 16 bits of each are then G itself
// (|G| <= Ltau <= 2^13, exact) and two of them pack in one instruction.
// Rows and columns of sites past L are 0, the bits past Ltau of the last
// chunk cancel (half of them turned over on the row side).
//
// The epilogue forms, per block and replica pair, the sums of G^a G^b over
// the elements of equal x1 - y1 (v_mad_i32_i16) and of equal x2 - y2
// (v_dot2_i32_i16), in int32 (at most 4 products, < 2^28), and adds these 8
// values to int64 buckets in LDS.  Each bucket has ncopy copies, so that the
// lanes of a wave that share a bucket do not meet at one address; pair p is
// the fastest index (an immediate offset).
//
// An element (x, y) of an off-diagonal block stands for (y, x) too, with the
// displacements negated; its products go to U, those of the diagonal blocks
// to F, and the flush folds D[d] = F[d] + U[d] + U[-d mod L].  In a diagonal
// tile the block (1, 0) is the mirror of (0, 1) and is dropped.
//
// A workgroup takes ncw configurations at a time (as many as keep its four
// waves busy) or every nsplit-th part of the tiles of one; records are added
// to.
//
// Bound by the words' way from L2 (the loads wait 0.4 of the wave cycles; the
// matrix cores are busy 0.4).  L = 24, Ltau = 2048, 4 replicas, 1024
// configurations: 1.85 ms with every replica's accumulators at once (64 x 32
// tiles, {0, 0.5} operands, a popcount pass) -> 1.70 as above on rows in
// site order -> 1.19 with the blocks' rows consecutive -> 1.02 with loads
// four chunks ahead -> 0.90 with whole words per lane.  L = 12, Ltau = 512,
// 6 replicas, 1536 configurations, where every element went to its own LDS
// bucket before: 1.13 ms -> 0.19.
// ---------------------------------------------------------------------------
constexpr int kGramWaves = 4;
// The overlap kernel squares kSqBias + Q^2 instead of Q^2 (below), which adds
// kSqBias^2 and 2 kSqBias Q^2 per element, in 64-bit integers modulo 2^64; it
// takes the first off itself, the second is taken off here, where sum Q^2 is
// formed: the record's sum Q^4 starts from -2 kSqBias sum Q^2.
constexpr unsigned long long kSqBias = 0x4B000000ull;  // the bits of 2^23
constexpr int kNarrowLt = 8192;  // |G| <= 2^13: int16 digits, int32 lane sums
__host__ __device__ constexpr int gram_pitch(int P) { return P | 1; }  // pairs, padded to an odd count

typedef short i16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int mad_lo16(int a, int b, int c) {
    int d;
    asm("v_mad_i32_i16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ int mad_hi16(int a, int b, int c) {
    int d;
    asm("v_mad_i32_i16 %0, %1, %2, %3 op_sel:[1,1,0,0]" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ int dot16(int a, int b, int c) {
    return __builtin_amdgcn_sdot2(__builtin_bit_cast(i16x2, a), __builtin_bit_cast(i16x2, b), c, false);
}

template <int RR>
__global__ void __launch_bounds__(64 * kGramWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_gram_mfma(ShapeDev sh, int cfg0, int ncfg, int ncw, int nsplit, int ncopy, int grouped) {
    constexpr int PP = RR * (RR - 1) / 2, PT = gram_pitch(PP);
    extern __shared__ __align__(16) uint8_t smem[];
    unsigned long long* const Bk = (unsigned long long*)smem;  // [ncw][F, U][x, y][L][ncopy][PT]
    const int L = sh.L;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb8 = gram_nb8(L), nblk = gram_nblk(L);
    const int ntile = (nblk + 1) >> 1, ntp = ntile * (ntile + 1) / 2;
    // grouped: workgroup b runs on XCD b mod 8, which takes the configurations
    // b mod 8, b mod 8 + 8, ... (times ncw), so that the nsplit workgroups of one
    // read its rows through one L2
    const int ng = grouped ? 8 : 1, item = (int)blockIdx.x / ng;
    const int part = item % nsplit, c0 = (item / nsplit * ng + (grouped ? (int)blockIdx.x & 7 : 0)) * ncw;
    if (c0 >= ncfg) return;
    const int ncl = min(ncw, ncfg - c0);
    const int half = 2 * L * ncopy * PT;  // words of F or of U of one configuration
    for (int e = tid; e < ncl * 2 * half; e += 64 * kGramWaves) Bk[e] = 0;
    __syncthreads();
    GramTile tile(sh);
    f32x16 start;
#pragma unroll
    for (int q = 0; q < 16; ++q) start[q] = kGramStart;
    for (int unit = part * kGramWaves + wv; unit < ncl * ntp; unit += kGramWaves * nsplit) {
        const int cl = unit / ntp;
        int X = 0, rem = unit - cl * ntp;
        while (rem >= ntile - X) { rem -= ntile - X; ++X; }
        const int Y = X + rem;
        tile.configuration(sh, cfg0 + c0 + cl);
        tile.tile(L, X, Y);
        int pk[RR][2][2][8];  // G of elements 2t, 2t + 1
#pragma unroll
        for (int r = 0; r < RR; ++r) {
            f32x16 acc[2][2];
            tile.product(r, start, acc);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        pk[r][u][v][t] = gram_pack(acc[u][v], t);
                        asm volatile("" : "+v"(pk[r][u][v][t]));  // packed here, not where it is used
                    }
            __builtin_amdgcn_sched_barrier(0);  // the next replica's loads wait until the accumulators are free
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                if (X == Y && u == 1 && v == 0) continue;
                const int br = 2 * X + u, bc = 2 * Y + v;
                unsigned long long* const B0 = Bk + cl * 2 * half + (X == Y && u == v ? 0 : half);
                unsigned long long *bx[4], *by[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int dx = bucket_of(4 * (br / nb8 - bc / nb8) + j - (i & 3), L);
                    const int dy = bucket_of(8 * (br % nb8 - bc % nb8) + 2 * j + h - (i >> 2), L);
                    bx[j] = B0 + (dx * ncopy + ((i >> 2) & (ncopy - 1))) * PT;
                    by[j] = B0 + ((L + dy) * ncopy + (((i & 3) + 4 * h) & (ncopy - 1))) * PT;
                }
                int p = 0;
#pragma unroll
                for (int a = 0; a < RR; ++a)
#pragma unroll
                    for (int b = a + 1; b < RR; ++b, ++p) {
                        const int(&A)[8] = pk[a][u][v];
                        const int(&B)[8] = pk[b][u][v];
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            atomicAdd(by[g] + p, (unsigned long long)(long long)dot16(
                                                     A[2 * g], B[2 * g], dot16(A[2 * g + 1], B[2 * g + 1], 0)));
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            int x = 0;
#pragma unroll
                            for (int g = 0; g < 4; ++g) {
                                const int t = 2 * g + (j >> 1);
                                x = j & 1 ? mad_hi16(A[t], B[t], x) : mad_lo16(A[t], B[t], x);
                            }
                            atomicAdd(bx[j] + p, (unsigned long long)(long long)x);
                        }
                    }
            }
    }
    __syncthreads();
    // D[d] = F[d] + U[d] + U[-d]; sum Q^2 = sum_xy G^a_xy G^b_xy = sum_d D_x[d]
    const int rl = 2 * L + 3;
    for (int e = tid; e < ncl * PP * 2 * L; e += 64 * kGramWaves) {
        const int cl = e / (PP * 2 * L), f = e % (PP * 2 * L), p = f / (2 * L), xd = f % (2 * L), d = xd % L;
        const unsigned long long* const Fb = Bk + cl * 2 * half + p;
        unsigned long long v = 0;
        for (int k = 0; k < ncopy; ++k)
            v += Fb[(xd * ncopy + k) * PT] + Fb[half + (xd * ncopy + k) * PT] +
                 Fb[half + ((xd - d + (L - d) % L) * ncopy + k) * PT];
        unsigned long long* const rp = (unsigned long long*)(sh.rec + ((size_t)(cfg0 + c0 + cl) * PP + p) * rl);
        atomicAdd(rp + xd, v);
        if (xd < L) {
            atomicAdd(rp + 2 * L + 1, v);
            atomicAdd(rp + 2 * L + 2, 0ull - 2 * kSqBias * v);  // what the overlap kernel's squares add too much
        }
    }
}

// ---------------------------------------------------------------------------
// The same for Ltau > 8192, int64 products, with B = (1 - S)/2 in {0,1} and
//   G = Ltau - 2 (n_x + n_y) + 4 (B B^T)_xy,  n_x = sum_tau B_x,tau.
//
// One workgroup takes one configuration at a time.  It first counts the
// down spins n^r_x of every site row (popcount along tau) into LDS; then its
// four waves share the tile pairs (X, Y), X <= Y, of the upper triangle,
// each wave alone (no barrier inside a configuration), one wave per SIMD:
// the 2 x 2 blocks of 32 x 32 of every replica's G^r = S S^T (2 x 1 above 4
// replicas), accumulators in the AGPRs, K = tau in chunks of 64, the {0,1}
// int8 operands built in registers from each lane's bit row.  The epilogue
// forms G = Ltau - 2 (n_x + n_y) + 4 (B B^T)_xy and the products G^a G^b.
//
// BLK (L a multiple of 8): tile X holds the 8 x 8 block of sites
// (bx, by) = (X mod L/8, X div L/8), row r the site (8bx + r mod 8,
// 8by + r div 8).  The 16 elements of a lane then take 4 values of x1 - y1
// (one per q mod 4) and 4 of x2 - y2 (one per q div 4), so each lane sums
// them in registers and adds 8 bucket values per pair and block, not 32.
// Otherwise tile X holds the slots 64X .. 64X + 63 and every element adds
// its own two.
// ---------------------------------------------------------------------------
template <int RR, int NV, bool BLK>
__global__ void __launch_bounds__(64 * kGramWaves)
    __attribute__((amdgpu_waves_per_eu(1, 1)))
k_gram_wide(ShapeDev sh, int cfg0, int ncfg) {
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
        if constexpr (BLK) return site_slot(L, 8 * (X % nbl) + (r & 7), 8 * (X / nbl) + (r >> 3));
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
            v16i acc[RR][2][NV];
#pragma unroll
            for (int r = 0; r < RR; ++r)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int q = 0; q < 16; ++q) acc[r][u][v][q] = 0;
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
                                A[u][r] = mfma_bits_operand((uint32_t)(wa[u][r] >> (32 * ks)) >> sh4);
#pragma unroll
                            for (int v = 0; v < NB; ++v)
                                B[v][r] = mfma_bits_operand((uint32_t)(wb[v][r] >> (32 * ks)) >> sh4);
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
            kloop(diagC);
            // epilogue, block by block
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
                            int x1, x2, y1, y2;
                            slot_site(L, x, x1, x2);
                            slot_site(L, y, y1, y2);
                            const int dx = (x1 - y1 + L) % L, dy = (x2 - y2 + L) % L;
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
    i32x4* const Aop = (i32x4*)smem;                                        // [nx][NU][64]
    unsigned long long* const S4 = (unsigned long long*)(Aop + sh.nx * NU * 64);  // [P][64], a slot per lane
    int* const Tr = (int*)(S4 + 64 * sh.P);                                 // [P][64]
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
        for (int e = tid; e < 64 * P; e += 64 * kOverlapWaves) {
            S4[e] = 0;
            Tr[e] = 0;
        }
        __syncthreads();
        if (part == 0) {
            // trQ = sum over the panel's rows of L^2 - 2 popcount(a ^ b)
            int tr[kMaxP] = {};
            for (int e = tid; e < nx * NU * 32; e += 64 * kOverlapWaves) {
                const int g = e / (NU * 32), row = row0 + e % (NU * 32);
                if (row >= Lt) continue;
                uint64_t w[kMaxR];
#pragma unroll
                for (int r = 0; r < kMaxR; ++r) w[r] = r < R ? px[((size_t)r * nx + g) * Lt + row] : 0ull;
                int q = 0;
#pragma unroll
                for (int a = 0; a < kMaxR; ++a)
#pragma unroll
                    for (int b = a + 1; b < kMaxR; ++b, ++q)
                        if (b < R) tr[q] += (g == 0 ? L2 : 0) - 2 * (int)__popcll(w[a] ^ w[b]);
            }
            int q = 0, k6 = 0;
#pragma unroll
            for (int a = 0; a < kMaxR; ++a)
#pragma unroll
                for (int b = a + 1; b < kMaxR; ++b, ++k6)
                    if (b < R) atomicAdd(&Tr[64 * q++ + lane], tr[k6]);
        }
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
                atomicAdd(&S4[64 * p + lane], s4);
            }
        }
        __syncthreads();
        for (int q = wv; q < P; q += kOverlapWaves) {
            unsigned long long v = S4[64 * q + lane];
            int tr = Tr[64 * q + lane];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                v += (unsigned long long)__shfl_xor((long long)v, off, 64);
                tr += __shfl_xor(tr, off, 64);
            }
            if (lane == 0) {
                unsigned long long* rp = (unsigned long long*)(sh.rec + ((size_t)cfg * P + q) * rl);
                if (part == 0) atomicAdd(rp + 2 * sh.L, (unsigned long long)(long long)tr);
                atomicAdd(rp + 2 * sh.L + 2, v);
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
        const int sx = site_slot(L, x % L, x / L), sy = site_slot(L, y % L, y / L);
        int G[kMaxR];
        for (int r = 0; r < R; ++r) {
            const size_t m = (size_t)cfg * R + r;
            int acc = 0;
            for (int c = 0; c < sh.nc; ++c)
                acc += dot64(sh.Pt[(m * sh.nc + c) * sh.nxp + sx], sh.Pt[(m * sh.nc + c) * sh.nxp + sy],
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
            const int sx = site_slot(sh.L, x % sh.L, x / sh.L), sy = site_slot(sh.L, y % sh.L, y / sh.L);
            const size_t m = (size_t)cfg * R + r;
            for (int c = 0; c < sh.nc; ++c)
                acc += dot64(sh.Pt[(m * sh.nc + c) * sh.nxp + sx], sh.Pt[(m * sh.nc + c) * sh.nxp + sy],
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

size_t gram_wide_lds(int RR, int L) {
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
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
        if (e != hipSuccess) return e;
        lds_set = true;
    }
    const int npanel = (sh.Lt + 32 * NU - 1) / (32 * NU), ntt = (sh.Lt + 63) / 64;
    int nsplit = 1;
    while ((long long)ncfg * npanel * nsplit < 2 * ncu && kOverlapWaves * nsplit < ntt) nsplit *= 2;
    const long long per = (long long)npanel * nsplit;
    return over_ranges(ncfg, per, 64 * kOverlapWaves, [&](int c, int n) {
        const bool grouped = ncu % 8 == 0 && n >= 128;
        hipLaunchKernelGGL((k_overlap_mfma<NU, NX>), dim3((unsigned)((grouped ? (n + 7) / 8 * 8 : n) * per)),
                           dim3(64 * kOverlapWaves), (size_t)sh.nx * NU * 64 * 16 + (size_t)64 * sh.P * 12, st, sh,
                           cfg0 + c, n, npanel, nsplit, (int)grouped);
        return hipGetLastError();
    });
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
hipError_t launch_gram(const ShapeDev& sh, int cfg0, int ncfg, int ncu, hipStream_t st) {
    constexpr int PP = RR * (RR - 1) / 2;
    // tiles per configuration: four, two or one configuration at a time give
    // each of the four waves a tile (L <= 8: one tile, L <= 16: 6 or 10)
    const int nblk = gram_nblk(sh.L), ntile = (nblk + 1) / 2, ntp = ntile * (ntile + 1) / 2;
    int ncw = ntp == 1 ? 4 : (ntp <= 10 ? 2 : 1);
    while (ncw > 1 && (ncfg + ncw - 1) / ncw < 2 * ncu) ncw /= 2;
    // from 36 tiles (L >= 18) three workgroups share a configuration: the
    // rows are read by as many fewer configurations at a time through an
    // L2 (L = 24: 907 -> 876 us; L = 12 with its 6 tiles 172 -> 198)
    int nsplit = ntp >= 36 ? 3 : 1;
    while ((ncfg + ncw - 1) / ncw * (long long)nsplit < 2 * ncu && kGramWaves * nsplit < ncw * ntp) nsplit *= 2;
    // copies of the buckets: 8, or 4 where 8 would not leave room for two
    // workgroups on a CU
    const size_t one = (size_t)ncw * 4 * sh.L * gram_pitch(PP) * 8;
    const int ncopy = 8 * one <= 72 * 1024 ? 8 : 4;
    static bool lds_set = false;
    if (!lds_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_gram_mfma<RR>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
        if (e != hipSuccess) return e;
        lds_set = true;
    }
    return over_ranges(ncfg, nsplit, 64 * kGramWaves, [&](int c, int n) {
        const int nitem = (n + ncw - 1) / ncw;
        const bool grouped = ncu % 8 == 0 && nitem >= 128;
        hipLaunchKernelGGL(k_gram_mfma<RR>, dim3((unsigned)(grouped ? (nitem + 7) / 8 * 8 : nitem) * nsplit),
                           dim3(64 * kGramWaves), ncopy * one, st, sh, cfg0 + c, n, ncw, nsplit, ncopy, (int)grouped);
        return hipGetLastError();
    });
}

template <int RR>
hipError_t launch_gram_wide(const ShapeDev& sh, int cfg0, int ncfg, int ncu, hipStream_t st) {
    // a wave holds every replica's G of its unit: 64 x 64 up to 4 replicas,
    // 64 x 32 above
    constexpr int NV = RR <= 4 ? 2 : 1;
    static bool lds_set = false;
    if (!lds_set) {
        for (const void* f : {(const void*)k_gram_wide<RR, NV, true>, (const void*)k_gram_wide<RR, NV, false>}) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)gram_wide_lds(RR, 32));
            if (e != hipSuccess) return e;
        }
        lds_set = true;
    }
    const int grid = std::min(ncfg, ncu);
    if (sh.L % 8 == 0)
        hipLaunchKernelGGL((k_gram_wide<RR, NV, true>), dim3(grid), dim3(64 * kGramWaves), gram_wide_lds(RR, sh.L), st,
                           sh, cfg0, ncfg);
    else
        hipLaunchKernelGGL((k_gram_wide<RR, NV, false>), dim3(grid), dim3(64 * kGramWaves), gram_wide_lds(RR, sh.L), st,
                           sh, cfg0, ncfg);
    return hipGetLastError();
}

template <int RR>
hipError_t launch_mfma(const ShapeDev& sh, int cfg0, int ncfg, hipStream_t st) {
    int dev = 0, ncu = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    const hipError_t e = sh.Lt <= kNarrowLt ? launch_gram<RR>(sh, cfg0, ncfg, ncu, st)
                                            : launch_gram_wide<RR>(sh, cfg0, ncfg, ncu, st);
    if (e != hipSuccess) return e;
    return launch_overlap(sh, cfg0, ncfg, ncu, st);
}

}  // namespace

bool measure_ok(const ShapeDev& sh) { return sh.R >= 2 && sh.R <= kMaxR && sh.L <= 32; }


hipError_t launch_transpose(const ShapeDev& sh, hipStream_t st) {
    const long long items = (long long)sh.R * sh.nk * sh.W * sh.nc * sh.nx;
    // a multiple of 8; blocks past the last tile leave at once
    const long long blocks = ((long long)sh.R * sh.nk * sh.W * sh.nc + 7) / 8 * 8 * sh.nx;
    const int grid = (int)std::min<long long>(blocks, 1 << 20);
    hipLaunchKernelGGL(k_transpose, dim3(grid), dim3(64), 0, st, sh, items);
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
