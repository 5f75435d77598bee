// Three-replica records for chi^(3) and F^(3) on int8 MFMA.
//
// Paper: arXiv:2310.07486, Methods, "One-time observables" (chi^(r), F^(r)
// and the second-moment length xi^(r), here r = 3) with the independent
// replicas of "Simulation details".
//
// For configuration (k-index i, sample s) and replicas r = 0..R-1 with
// G^r = S^r S^rT (L^2 x L^2), the record of a replica triple a < b < c is
//   T_x[d] = sum_{carrier e in {a,b,c}, f < g the other two}
//            sum_{(x1 - y1) mod L = d} G^e_xy (G^f G^g)_yx     (T_y: x2 - y2)
// so that Tr[M^3] ~ sum_d T_x[d] and Tr[M-hat M^2] ~ sum_d T_x[d] cos(2 pi d/L)
// (the phase on the carrier's factor, averaged over the three choices).
//
// 1. k_gram_store computes G of every replica from the bit rows along tau
//    (the K loop of the pair records' Gram) and writes G' = G/2 (exact: every
//    entry has the parity of Ltau, which is even), |G'| <= Ltau/2, as two int8
//    digits G' = 64 h + l, l in [-32, 31] (h in [-16, 16] at Ltau = 2048), to
//    the caller's workspace, block by block of 32 x 32 sites in the order of
//    the lanes: lane (i, h) of block (rb, kb) holds row i and the 16 columns
//    8g + 4h + j (byte 4g + j).  That is at once the 16 outputs of a lane in
//    the 32 x 32 MFMA layout (G is symmetric), an int8 MFMA operand whose K
//    axis runs over the sites of block kb, and the 16 carrier elements that a
//    lane of the product needs: every access is 16 consecutive bytes per lane
//    and 1 KB per wave.  (Ltau above 16312, L = 2 and 4 only: k_triple_long.)
// 2. k_triple_mfma forms P = G'^f G'^g = 4096 h^f h^g + 64 (h^f l^g + l^f h^g)
//    + l^f l^g with three exact int8 products on v_mfma_i32_32x32x32_i8 (the
//    middle one with K doubled), |P| <= L^2 (Ltau/2)^2 < 2^31.  Its epilogue
//    multiplies P_yx by G'^e_xy of each carrier e outside {f, g} and sums
//    each lane's 16 products into four x-buckets and four y-buckets of the
//    triple {e, f, g}, in int64.  Records are scaled by 8 (G = 2 G').
#include <algorithm>

#include "gram_tile.h"
#include "tfim_internal.h"

namespace tfim {
namespace {

typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int kMaxL = 32;
constexpr int kWaves = 4;
constexpr int kBlock = 1024;             // bytes of one stored block and digit
constexpr int kStage = 16 * kBlock;      // one K step of a workgroup: 4 + 4 blocks, two digits each

// ---------------------------------------------------------------------------
// G' of every replica into the workspace: digit d of block (rb, kb) of replica
// r of configuration cl at ((((cl R + r) 2 + d) nblk + rb) nblk + kb) kBlock.
// Each wave alone takes a 64 x 64 tile of one replica (every ordered pair of
// tiles: a tile writes its mirror, so that both stores are 16 bytes per lane;
// forming the mirror again costs less than storing a tile by bytes).  The
// accumulators start from 1.5 2^23 + 64: their low 16 bits are t = G + 64,
// h = t >> 7 and l = ((t & 127) >> 1) - 32, two elements per instruction.
// L = 20, Ltau = 2048, 6 replicas, 256 configurations: 1.41 ms -> 0.40 ms.
// ---------------------------------------------------------------------------
typedef short i16x2 __attribute__((ext_vector_type(2)));

__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2)))
k_gram_store(ShapeDev sh, int cfg0, int ncfg, int nsplit, int grouped, int8_t* __restrict__ ws) {
    const int L = sh.L, R = sh.R;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nblk = gram_nblk(L), ntile = (nblk + 1) >> 1, nunit = R * ntile * ntile;
    // grouped: an XCD takes whole configurations (workgroup b runs on XCD b mod 8)
    const int ng = grouped ? 8 : 1, item = (int)blockIdx.x / ng;
    const int cl = item / nsplit * ng + (grouped ? (int)blockIdx.x & 7 : 0), part = item % nsplit;
    if (cl >= ncfg) return;
    GramTile tile(sh);
    tile.configuration(sh, cfg0 + cl);
    f32x16 start;
#pragma unroll
    for (int q = 0; q < 16; ++q) start[q] = kGramStart + 64.0f;
    for (int unit = part * kWaves + wv; unit < nunit; unit += kWaves * nsplit) {
        const int r = unit / (ntile * ntile), XY = unit - r * ntile * ntile, X = XY / ntile, Y = XY - X * ntile;
        tile.tile(L, X, Y);
        f32x16 acc[2][2];
        tile.product(r, start, acc);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int kb = 2 * X + u, rb = 2 * Y + v;
                if (kb >= nblk || rb >= nblk) continue;
                i32x4 hw, lw;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    int h2[2], l2[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int t = gram_pack(acc[u][v], 2 * g + k);
                        h2[k] = __builtin_bit_cast(int, __builtin_bit_cast(i16x2, t) >> (short)7);
                        // bit 0 of t is 0 in both halves (G is even)
                        l2[k] = __builtin_bit_cast(
                            int, __builtin_bit_cast(i16x2, (t & 0x007F007F) >> 1) - (i16x2){32, 32});
                    }
                    hw[g] = (int)__builtin_amdgcn_perm((uint32_t)h2[1], (uint32_t)h2[0], 0x06040200u);
                    lw[g] = (int)__builtin_amdgcn_perm((uint32_t)l2[1], (uint32_t)l2[0], 0x06040200u);
                }
                int8_t* const o = ws + ((((size_t)cl * R + r) * 2 * nblk + rb) * nblk + kb) * kBlock + 16 * lane;
                *(i32x4*)o = hw;
                *(i32x4*)(o + (size_t)nblk * nblk * kBlock) = lw;
            }
    }
}

// ---------------------------------------------------------------------------
// Pair products and the carrier epilogue; records [cl][NT][2][L].
//
// A workgroup takes 4 x 4 blocks (128 x 128 sites) of the output of one
// configuration, for every replica pair f < g in turn; each of its four waves
// 2 x 2 blocks, three accumulators each (192 registers, two waves per SIMD).
// The K steps (32 sites) of all pairs form one pipeline: the step's 16 KB go
// through one of two LDS buffers, loaded into registers two steps ahead, one
// barrier per step, and every LDS access is lane-linear.  A wave reads 8 KB
// of LDS for 16 MFMAs, half of what one 32 x 32 block per wave took.  The
// buckets of all triples stay in LDS (ncopy copies, so that lanes that share
// a bucket do not meet at one address) and reach the record once.
// L = 20, Ltau = 2048, 6 replicas, 256 configurations: 11.3 ms with one launch
// per pair and 8 x 8 site blocks (576 padded sites instead of 480) -> 2.3 ms.
// Matrix cores 0.40 busy, VALU 0.38: what is left is the K steps of a workgroup
// whose partner on the CU is not in its epilogue just then.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_triple_mfma(int L, int R, int ncfg, int ncopy, int psplit, int grouped, const int8_t* __restrict__ ws,
              int64_t* __restrict__ rec) {
    extern __shared__ __align__(16) uint8_t smem[];
    uint8_t* const stg = smem;                                                // [2][kStage]
    unsigned long long* const Tb = (unsigned long long*)(smem + 2 * kStage);  // [NT][x, y][L][ncopy]
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wy = wv & 1, wx = wv >> 1;
    const int nb8 = gram_nb8(L), nblk = gram_nblk(L), nwt = (nblk + 3) >> 2, ipc = nwt * nwt * psplit;
    const int NT = R * (R - 1) * (R - 2) / 6, PP = R * (R - 1) / 2;
    const int ng = grouped ? 8 : 1, item = (int)blockIdx.x / ng;
    const int cl = item / ipc * ng + (grouped ? (int)blockIdx.x & 7 : 0);
    if (cl >= ncfg) return;
    const int part = item % ipc / (nwt * nwt), Yt = item % (nwt * nwt) / nwt, Xt = item % nwt;
    // this workgroup's pairs p0 .. p1 - 1, the first (f, g)
    const int p0 = part * PP / psplit, p1 = (part + 1) * PP / psplit;
    int f = 0, g = 1 + p0;
    while (g >= R) {
        ++f;
        g += f + 1 - R;
    }
    for (int e = tid; e < NT * 2 * L * ncopy; e += 64 * kWaves) Tb[e] = 0;
    const uint64_t base = (uint64_t)(ws + (size_t)cl * R * 2 * nblk * nblk * kBlock);
    const uint32_t base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint32_t base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    const __amdgpu_buffer_rsrc_t G = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(((uint64_t)base_hi << 32) | base_lo), (short)0, R * 2 * nblk * nblk * kBlock, 0x00020000);
    // byte offset of digit d of block (rb, kb) of replica r
    auto block_at = [&](int r, int d, int rb, int kb) {
        return (((r * 2 + d) * nblk + min(rb, nblk - 1)) * nblk + min(kb, nblk - 1)) * kBlock;
    };
    auto load16 = [&](int off) { return (i32x4)__builtin_amdgcn_raw_buffer_load_b128(G, 16 * lane, off, 0); };
    // this wave's share of the staging: two blocks of one side, both digits
    const int side = wv >> 1, sb = 2 * (wv & 1);
    const int digit = nblk * nblk * kBlock;  // bytes from a block's h to its l
    int at[2];  // offsets of the two blocks (digit h) at the pair and K step two ahead
    auto fetch = [&](i32x4 (&w)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = load16(at[k >> 1] + (k & 1) * digit);
    };
    auto put = [&](int buf, const i32x4 (&w)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *(i32x4*)(stg + buf * kStage + ((side * 4 + sb + (k >> 1)) * 2 + (k & 1)) * kBlock + 16 * lane) = w[k];
    };
    int nf = f, ngp = g, nk = 0;
    auto start_pair = [&]() {
#pragma unroll
        for (int k = 0; k < 2; ++k) at[k] = block_at(side ? ngp : nf, 0, (side ? 4 * Xt : 4 * Yt) + sb + k, 0);
    };
    auto advance = [&]() {
        at[0] += kBlock;
        at[1] += kBlock;
        if (++nk == nblk) {
            nk = 0;
            if (++ngp == R) {
                ++nf;
                ngp = nf + 1;
            }
            if (ngp >= R) {  // past the last pair: any step again, not used
                nf = 0;
                ngp = 1;
            }
            start_pair();
        }
    };
    i32x4 w[4];
    start_pair();
    fetch(w);
    advance();
    put(0, w);
    fetch(w);
    advance();
    __syncthreads();
    int buf = 0;
    i32x16 hh[2][2], xx[2][2], ll[2][2];
    auto step = [&](auto firstC) {
        constexpr bool kFirst = decltype(firstC)::value;
        put(buf ^ 1, w);  // read two steps before, a barrier ago
        fetch(w);
        advance();
        const uint8_t* const sA = stg + buf * kStage + 4 * wy * kBlock + 16 * lane;
        const uint8_t* const sB = stg + buf * kStage + (8 + 4 * wx) * kBlock + 16 * lane;
        i32x4 B[2][2];
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int d = 0; d < 2; ++d) B[v][d] = *(const i32x4*)(sB + (2 * v + d) * kBlock);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const i32x4 ah = *(const i32x4*)(sA + 2 * u * kBlock), al = *(const i32x4*)(sA + (2 * u + 1) * kBlock);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                hh[u][v] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, B[v][0], kFirst ? i32x16{} : hh[u][v], 0, 0, 0);
                ll[u][v] = __builtin_amdgcn_mfma_i32_32x32x32_i8(al, B[v][1], kFirst ? i32x16{} : ll[u][v], 0, 0, 0);
                xx[u][v] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, B[v][1], kFirst ? i32x16{} : xx[u][v], 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 2; ++v)
                xx[u][v] = __builtin_amdgcn_mfma_i32_32x32x32_i8(al, B[v][0], xx[u][v], 0, 0, 0);
        }
        buf ^= 1;
    };
    const int rb0 = 4 * Yt + 2 * wy, cb0 = 4 * Xt + 2 * wx;  // the wave's first row and column block
    for (int p = p0; p < p1; ++p) {
        step(std::true_type{});
        __syncthreads();
        for (int kb = 1; kb < nblk; ++kb) {
            step(std::false_type{});
            __syncthreads();
        }
        int P[2][2][16];
        // the carriers in turn, the next one's elements in flight meanwhile
        auto carrier = [&](int c) {
            int e = min(c, R - 3);
            e += e >= f;
            return e + (e >= g);
        };
        i32x4 ch[2][2], cw[2][2];
        auto load = [&](int c, int u, int v) {
            const int o = block_at(carrier(c), 0, cb0 + v, rb0 + u);
            ch[u][v] = load16(o);
            cw[u][v] = load16(o + digit);
        };
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) load(0, u, v);
        // P = 4096 hh + 64 xx + ll
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int q = 0; q < 16; ++q) P[u][v][q] = (((hh[u][v][q] << 6) + xx[u][v][q]) << 6) + ll[u][v][q];
#pragma unroll 1
        for (int c = 0; c < R - 2; ++c) {
            const int e = carrier(c);
            // index of the sorted triple {e, f, g}
            const int ta = min(e, f), tc = max(e, g), tb = e + f + g - ta - tc;
            int t = tc - tb - 1;
            for (int k = 0; k < ta; ++k) t += (R - 1 - k) * (R - 2 - k) / 2;
            for (int k = ta + 1; k < tb; ++k) t += R - 1 - k;
            unsigned long long* const Tt = Tb + t * 2 * L * ncopy;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    long long tx[4] = {0, 0, 0, 0}, ty[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const int hb = (int)(int8_t)(ch[u][v][q >> 2] >> (8 * (q & 3)));
                        const int lb = (int)(int8_t)(cw[u][v][q >> 2] >> (8 * (q & 3)));
                        const int x = (hb << 6) + lb;
                        tx[q & 3] += (long long)x * P[u][v][q];
                        ty[q >> 2] += (long long)x * P[u][v][q];
                    }
                    load(c + 1, u, v);  // in flight during the next three blocks
                    if (rb0 + u >= nblk || cb0 + v >= nblk) continue;
                    const int rb = rb0 + u, cb = cb0 + v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int dx = bucket_of(4 * (cb / nb8 - rb / nb8) + (i & 3) - j, L);
                        const int dy = bucket_of(8 * (cb % nb8 - rb % nb8) + (i >> 2) - 2 * j - h, L);
                        atomicAdd(Tt + dx * ncopy + ((i >> 2) & (ncopy - 1)), (unsigned long long)tx[j]);
                        atomicAdd(Tt + (L + dy) * ncopy + ((i & 3) & (ncopy - 1)), (unsigned long long)ty[j]);
                    }
                }
        }
        if (++g == R) {
            ++f;
            g = f + 1;
        }
    }
    __syncthreads();
    for (int e = tid; e < NT * 2 * L; e += 64 * kWaves) {
        unsigned long long v = 0;
        for (int k = 0; k < ncopy; ++k) v += Tb[e * ncopy + k];
        atomicAdd((unsigned long long*)rec + (size_t)cl * NT * 2 * L + e, v * 8ull);
    }
}

// ---------------------------------------------------------------------------
// Ltau above kDigitLt, where G' no longer fits two digits (G = Ltau on the
// diagonal): planes of L = 2 and 4 only, since L^2 (Ltau/2)^2 < 2^31.  A workgroup
// per configuration, an element of the plane per thread: G^r in 32 bits in LDS,
// every product in 64.  Bound by the latency of the rows' words.
// ---------------------------------------------------------------------------
constexpr int kDigitLt = 16312;  // (Ltau + 64) >> 7 <= 127, Ltau a multiple of 8
constexpr int kLongSites = 16;

__global__ void __launch_bounds__(kLongSites* kLongSites) k_triple_long(ShapeDev sh, int cfg0,
                                                                        int64_t* __restrict__ rec) {
    __shared__ int G[6][kLongSites * kLongSites];
    __shared__ unsigned long long T[20 * 2 * 4];  // [NT][x, y][L]
    const int L = sh.L, L2 = sh.L2, R = sh.R, nc = sh.nc, nxp = sh.nxp, tid = threadIdx.x;
    const int NT = R * (R - 1) * (R - 2) / 6;
    const bool on = tid < L2 * L2;
    const int x = on ? tid / L2 : 0, y = on ? tid % L2 : 0;
    const int sx = site_slot(L, x % L, x / L), sy = site_slot(L, y % L, y / L);
    for (int r = 0; r < R; ++r) {
        const uint64_t* const pt = sh.Pt + ((size_t)(cfg0 + (int)blockIdx.x) * R + r) * nc * nxp;
        int n = 0;  // of opposite spins (padding bits are 0)
#pragma unroll 8
        for (int c = 0; c < nc; ++c) n += __popcll(pt[(size_t)c * nxp + sx] ^ pt[(size_t)c * nxp + sy]);
        G[r][tid] = sh.Lt - 2 * n;
    }
    for (int e = tid; e < NT * 2 * L; e += kLongSites * kLongSites) T[e] = 0;
    __syncthreads();
    const int dx = bucket_of(x % L - y % L, L), dy = bucket_of(x / L - y / L, L);
    int t = 0;
    for (int a = 0; a < R; ++a)
        for (int b = a + 1; b < R; ++b)
            for (int c = b + 1; c < R; ++c, ++t) {
                // G^e_xy (G^f G^g)_yx for the three carriers e
                auto term = [&](int e, int f, int g) {
                    long long p = 0;
                    for (int z = 0; z < L2; ++z) p += (long long)G[f][y * L2 + z] * G[g][z * L2 + x];
                    return G[e][x * L2 + y] * p;
                };
                const unsigned long long v = (unsigned long long)(term(a, b, c) + term(b, a, c) + term(c, a, b));
                if (on) {
                    atomicAdd(&T[t * 2 * L + dx], v);
                    atomicAdd(&T[t * 2 * L + L + dy], v);
                }
            }
    __syncthreads();
    for (int e = tid; e < NT * 2 * L; e += kLongSites * kLongSites)
        rec[(size_t)blockIdx.x * NT * 2 * L + e] = (int64_t)T[e];
}

// The records are sums of atomic adds: cleared first by a kernel (no memset
// node, so the launch sequence may be captured in a graph).
__global__ void k_zero_records(int64_t* __restrict__ rec, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        rec[i] = 0;
}

hipError_t launch_triples_on(const ShapeDev& sh, int cfg0, int ncfg, int64_t* rec, int8_t* gw, hipStream_t st) {
    int dev = 0, ncu = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    hipError_t e;
    if (sh.Lt > kDigitLt) {
        hipLaunchKernelGGL(k_triple_long, dim3((unsigned)ncfg), dim3(kLongSites * kLongSites), 0, st, sh, cfg0, rec);
        return hipGetLastError();
    }
    const int NT = sh.R * (sh.R - 1) * (sh.R - 2) / 6;
    const size_t nrec = (size_t)ncfg * NT * 2 * sh.L;
    hipLaunchKernelGGL(k_zero_records, dim3((unsigned)std::min<size_t>((nrec + 255) / 256, 1024)), dim3(256), 0,
                       st, rec, nrec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // an XCD takes whole configurations where there are many
    const bool grouped = ncu % 8 == 0 && ncfg >= 64;
    const int nitem = grouped ? (ncfg + 7) / 8 * 8 : ncfg;
    const int nblk = gram_nblk(sh.L), ntile = (nblk + 1) / 2, nunit = sh.R * ntile * ntile;
    // about 16 tiles to a workgroup, fewer where that leaves CUs idle
    int nsplit = std::max(1, nunit / (4 * kWaves));
    while (ncfg * nsplit < 2 * ncu && kWaves * nsplit < nunit) nsplit *= 2;
    hipLaunchKernelGGL(k_gram_store, dim3((unsigned)(nitem * nsplit)), dim3(64 * kWaves), 0, st, sh, cfg0, ncfg, nsplit,
                       (int)grouped, gw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int nwt = (nblk + 3) / 4;
    // bucket copies within 64 KB of LDS (four at 20 triples and L = 24)
    const size_t one = (size_t)NT * 2 * sh.L * 8;
    int ncopy = 8;
    while (ncopy > 1 && 2 * kStage + ncopy * one > 64 * 1024) ncopy /= 2;
    // few configurations: the pairs of one tile over several workgroups (with
    // a full chip it gains nothing: 2314 us with one, 2347 with two, 2406 with
    // five, L = 20, 256 configurations)
    const int PP = sh.R * (sh.R - 1) / 2;
    int psplit = 1;
    while (ncfg * nwt * nwt * psplit < 2 * ncu && psplit < PP) psplit = std::min(2 * psplit, PP);
    hipLaunchKernelGGL(k_triple_mfma, dim3((unsigned)(nitem * nwt * nwt * psplit)), dim3(64 * kWaves),
                       2 * kStage + ncopy * one, st, sh.L, sh.R, ncfg, ncopy, psplit, (int)grouped, (const int8_t*)gw,
                       rec);
    return hipGetLastError();
}

}  // namespace

// A plane has room for 8 x 8 sites where a block holds 4 x 8, the space that
// callers have been told to bring; blocks of 4 x 8 fill part of it (480^2 of 576^2
// bytes at L = 20).
TripleLayout triple_layout(const ShapeDev& sh, int ncfg) {
    TripleLayout t;
    t.nb = (sh.L + 7) / 8;
    t.nt = t.nb * t.nb;
    t.Np = 64 * t.nt;
    const int NT = sh.R * (sh.R - 1) * (sh.R - 2) / 6;
    t.rec_bytes = ((size_t)ncfg * NT * 2 * sh.L * 8 + 255) & ~(size_t)255;
    t.g_bytes = (size_t)ncfg * sh.R * 2 * (size_t)t.Np * t.Np;
    return t;
}

const char* triples_unsupported(const ShapeDev& sh) {
    if (sh.R < 3 || sh.R > 6) return "three-replica records need 3 to 6 replicas";
    if (sh.L > kMaxL) return "three-replica records need L <= 32";
    // |G'^f G'^g| <= L^2 (Ltau/2)^2 must fit the int32 accumulators
    const unsigned long long half = (unsigned long long)sh.Lt / 2;
    if ((unsigned long long)sh.L2 * half * half >= (1ull << 31))
        return "L^2 (Ltau/2)^2 exceeds the int32 range of the pair products";
    // a record of three carriers, 3 L^6 Ltau^3, must fit int64
    const unsigned __int128 n = (unsigned)sh.L2, t = (unsigned)sh.Lt;
    if (3 * n * n * n * t * t * t >= ((unsigned __int128)1 << 63))
        return "3 L^6 Ltau^3 exceeds the int64 range of a record";
    return nullptr;
}

hipError_t launch_triples(const ShapeDev& sh, int cfg0, int ncfg, int64_t* rec, int8_t* gw, hipStream_t st) {
    if (ncfg <= 0) return hipSuccess;
    if (sh.R < 3 || sh.R > 6) return hipErrorInvalidValue;
    return launch_triples_on(sh, cfg0, ncfg, rec, gw, st);
}

}  // namespace tfim
