// Two-time correlations on fp4 MFMA.
//
// Paper: arXiv:2310.07486, Methods, "Two-times observables": C_A(tau) is the
// average over tau1 of A(S_tau1) A(S_tau1+tau) along the periodic time
// direction, for A = sigma^Z_x summed over sites (C(tau)) and for
// A = sigma^Z_x sigma^Z_y summed over site pairs (Q2(tau)).
//
// Both come from the time Gram of one replica, H = S^T S (Ltau x Ltau,
// H_t1t2 = sum_x S_x,t1 S_x,t2, |H| <= L^2):
//   c[d]  = sum_t1 H_t1,(t1+d) mod Ltau,   q2[d] = sum_t1 H_t1,(t1+d) mod Ltau ^ 2,
// summed over the replicas of the configuration.  The contraction over sites
// runs on fp4 MFMAs with +-1 operands built in registers from the bit rows
// along the sites (7 VALU per operand, one operand per MFMA); the fp32
// accumulator is H itself, exactly.
//
// The waves of a workgroup share the upper triangle of 64 x 64 tiles of one
// configuration, each wave alone, the replicas in turn: sum_r H^r and
// sum_r (H^r)^2 of the tile's elements stay in registers (exact in fp32: below
// 2^23), two instructions per element and replica.  Then every element adds
// its two sums to the LDS buckets of its diagonal d = t2 - t1: in the MFMA
// layout the lanes of a half-wave hold 32 consecutive diagonals for each
// element q, at a fixed offset from q to q, so an addition is one LDS
// instruction without conflicts (a copy of the buckets per half-wave) and no
// address arithmetic.  Elements below the diagonal fall into 64 slots that
// nobody reads.  c fits 32 bits; q2 too while R L^4 Ltau < 2^32, else kWide
// keeps it in 64.  H is symmetric, so the record is c[d] = U[d] + U[Ltau - d]
// (c[0] = U[0]).
//
// Bound by the operand VALU (the matrix cores would allow two thirds of the
// time).  L = 24, Ltau = 2048, 4 replicas, 512 configurations: 3.60 ms with int8
// MFMAs, a correction step, two replicas at a time and the diagonals gathered
// by ds_bpermute -> 1.51 ms.
#include <algorithm>
#include <type_traits>

#include "tfim_internal.h"

namespace tfim {
namespace {

constexpr int kMaxLtTime = 4096;
constexpr int kTcWaves = 4;  // waves per workgroup
constexpr int kDrop = 64;    // slots of the elements below the diagonal

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Buckets of one half-wave's copy, slot d + kDrop.
__host__ __device__ constexpr int tc_slots(int Lt) { return 64 * ((Lt + 63) / 64) + kDrop; }

template <bool kOdd, bool kWide>
__global__ void __launch_bounds__(64 * kTcWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_timecorr_mfma(ShapeDev sh, int cfg0, int ncfg, int nsplit, int grouped, int64_t* __restrict__ rec) {
    using Q = std::conditional_t<kWide, unsigned long long, uint32_t>;
    extern __shared__ __align__(16) uint8_t smem[];
    const int L2 = sh.L2, Lt = sh.Lt, nx = sh.nx, R = sh.R, ns = tc_slots(Lt);
    Q* const q2b = (Q*)smem;                      // [2][ns]
    uint32_t* const cb = (uint32_t*)(q2b + 2 * ns);  // [2][ns]
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntt = (Lt + 63) / 64, ntp = ntt * (ntt + 1) / 2;
    // grouped: workgroup b runs on XCD b mod 8, which takes the configurations
    // b mod 8, b mod 8 + 8, ..., so that the nsplit workgroups of one read its
    // rows through one L2
    const int ng = grouped ? 8 : 1, item = (int)blockIdx.x / ng;
    const int cl = item / nsplit * ng + (grouped ? (int)blockIdx.x & 7 : 0), part = item % nsplit;
    if (cl >= ncfg) return;
    for (int e = tid; e < 2 * ns; e += 64 * kTcWaves) {
        q2b[e] = 0;
        cb[e] = 0;
    }
    __syncthreads();
    const uint64_t* const px = sh.Px + (size_t)(cfg0 + cl) * R * nx * Lt;
    const uint32_t base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)px);
    const uint32_t base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)px >> 32));
    const __amdgpu_buffer_rsrc_t words = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(((uint64_t)base_hi << 32) | base_lo), (short)0, R * nx * Lt * 8, 0x00020000);
    // the last chunk's bits past L^2 cancel: half of them are turned over on
    // the row side (their number is a multiple of 4)
    const int padn = (64 * nx - L2) >> 1;
    const uint64_t pad64 = padn ? ~0ull << (64 - padn) : 0ull;
    for (int tp = part * kTcWaves + wv; tp < ntp; tp += kTcWaves * nsplit) {
        int T = 0, rem = tp;
        while (rem >= ntt - T) { rem -= ntt - T; ++T; }
        const int T2 = T + rem;
        int row[4];       // byte offsets of this lane's rows (t1), then columns (t2)
        uint32_t mag[4];  // 0 past Ltau
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = 64 * (k < 2 ? T : T2) + 32 * (k & 1) + i;
            row[k] = 8 * min(t, Lt - 1);
            mag[k] = t < Lt ? 0x22222222u : 0u;
        }
        // Chunks in pairs: lane (i, h) loads the whole word of chunk 2g + h,
        // whose halves feed two MFMAs.  First comes an odd last chunk, by
        // halves of its word, else the last pair (either holds the padding).
        const int n = nx / 2, m = kOdd ? n : n - 1;  // pairs, and those after the first step
        const uint32_t flip = (uint32_t)(pad64 >> (32 * h));
        const uint64_t flip_pair = h ? pad64 : 0ull;
        u32x2 w0[4], w1[4];
        uint32_t wl[4];  // kOdd: the last chunk
        auto fetch = [&](int r, int g, u32x2 (&w)[4]) {
            const int so = (r * nx + 2 * g) * Lt * 8;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                w[k] = __builtin_amdgcn_raw_buffer_load_b64(words, row[k] + h * Lt * 8, so, 0);
        };
        // the first loads of replica r
        auto begin = [&](int r) {
            if constexpr (kOdd) {
                const int so = (r * nx + nx - 1) * Lt * 8;
#pragma unroll
                for (int k = 0; k < 4; ++k) wl[k] = __builtin_amdgcn_raw_buffer_load_b32(words, row[k] + 4 * h, so, 0);
                if (n > 0) {
                    fetch(r, 0, w0);
                    fetch(r, min(1, n - 1), w1);
                }
            } else {
                fetch(r, n - 1, w1);
                fetch(r, 0, w0);
            }
        };
        begin(0);
        f32x16 hs[2][2] = {}, hq[2][2] = {};
#pragma unroll 1
        for (int r = 0; r < R; ++r) {
            f32x16 acc[2][2];
            auto step = [&](const uint32_t (&w)[4], auto firstC) {
                constexpr bool kFirst = decltype(firstC)::value;
                i32x4 o[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = fp4_signs_operand(w[k], mag[k]);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 2; ++v)
                        acc[u][v] = mfma_fp4(fp4_wide(o[u]), fp4_wide(o[2 + v]), kFirst ? f32x16{} : acc[u][v]);
            };
            auto pair = [&](const u32x2 (&w)[4], auto firstC) {
                constexpr bool kFirst = decltype(firstC)::value;
                const uint64_t f = kFirst ? flip_pair : 0ull;
                const uint32_t a[4] = {w[0][0] ^ (uint32_t)f, w[1][0] ^ (uint32_t)f, w[2][0], w[3][0]};
                step(a, firstC);
                const uint32_t b[4] = {w[0][1] ^ (uint32_t)(f >> 32), w[1][1] ^ (uint32_t)(f >> 32), w[2][1], w[3][1]};
                step(b, std::false_type{});
            };
            if constexpr (kOdd) {
                const uint32_t a[4] = {wl[0] ^ flip, wl[1] ^ flip, wl[2], wl[3]};
                step(a, std::true_type{});
            } else {
                pair(w1, std::true_type{});
                fetch(r, min(1, n - 1), w1);
            }
            int g = 0;
            for (; g + 1 < m; g += 2) {
                pair(w0, std::false_type{});
                fetch(r, min(g + 2, n - 1), w0);
                pair(w1, std::false_type{});
                fetch(r, min(g + 3, n - 1), w1);
            }
            if (g < m) pair(w0, std::false_type{});
            begin(min(r + 1, R - 1));  // in flight during the sums below
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const float H = acc[u][v][q];
                        hs[u][v][q] += H;
                        hq[u][v][q] = __builtin_fmaf(H, H, hq[u][v][q]);
                    }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                if (T == T2 && u == 1 && v == 0) continue;  // below the diagonal
                // element q: slot + 27 - (8 (q div 4) + q mod 4)
                const int slot = kDrop + 64 * (T2 - T) + 32 * (v - u) + i - 4 * h - 27 + h * ns;
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int off = 27 - 8 * (q >> 2) - (q & 3);
                    atomicAdd(cb + slot + off, (uint32_t)(int)hs[u][v][q]);
                    atomicAdd(q2b + slot + off, (Q)(uint32_t)hq[u][v][q]);
                }
            }
    }
    __syncthreads();
    // c[d] = U[d] + U[Ltau - d] for d > 0, c[0] = U[0] (likewise q2).  The
    // terms of U[Ltau - d] cross the tau wrap: with an antiperiodic boundary
    // they enter c with the sign -1 (q2 squares the sign away).
    const bool anti = sh.apm != 0ull;
    int64_t* const out = rec + (size_t)cl * 2 * Lt;
    for (int e = tid; e < 2 * Lt; e += 64 * kTcWaves) {
        const int hh = e >= Lt, d = hh ? e - Lt : e;
        auto U = [&](int k) -> int64_t {
            const int s = kDrop + k;
            return hh ? (int64_t)(q2b[s] + q2b[ns + s]) : (int64_t)(int32_t)(cb[s] + cb[ns + s]);
        };
        const int64_t w = d ? U(Lt - d) : 0;
        const int64_t v = U(d) + (anti && !hh ? -w : w);
        if (nsplit == 1)
            out[e] = v;
        else
            atomicAdd((unsigned long long*)out + e, (unsigned long long)v);
    }
}

__global__ void k_zero_time(int64_t* __restrict__ rec, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        rec[i] = 0;
}

template <bool kOdd, bool kWide>
hipError_t launch_timecorr_as(const ShapeDev& sh, int cfg0, int ncfg, int64_t* rec, hipStream_t st) {
    int dev = 0, ncu = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    auto lds = [](int Lt) { return (size_t)2 * tc_slots(Lt) * (kWide ? 12 : 8); };
    static bool lds_set = false;  // above 64 KiB of LDS per workgroup
    if (!lds_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_timecorr_mfma<kOdd, kWide>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds(kMaxLtTime));
        if (e != hipSuccess) return e;
        lds_set = true;
    }
    // Up to four workgroups share a configuration's tiles and add up, 32 or
    // more tiles to a wave (Ltau = 2048: 1647 -> 1508 us with four: fewer
    // configurations at a time through an L2, and the dispatcher evens out
    // the workgroups); more where there are few configurations.
    const int ntt = (sh.Lt + 63) / 64, ntp = ntt * (ntt + 1) / 2;
    int nsplit = std::max(1, std::min(4, ntp / (32 * kTcWaves)));
    while ((long long)ncfg * nsplit < 2 * ncu && kTcWaves * nsplit < ntp) nsplit *= 2;
    if (nsplit > 1) {
        const size_t n = (size_t)ncfg * 2 * sh.Lt;
        hipLaunchKernelGGL(k_zero_time, dim3((unsigned)std::min<size_t>((n + 255) / 256, 1024)), dim3(256), 0, st, rec,
                           n);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return over_ranges(ncfg, nsplit, 64 * kTcWaves, [&](int c, int n) {
        const bool grouped = ncu % 8 == 0 && n >= 128;
        hipLaunchKernelGGL((k_timecorr_mfma<kOdd, kWide>), dim3((unsigned)(grouped ? (n + 7) / 8 * 8 : n) * nsplit),
                           dim3(64 * kTcWaves), lds(sh.Lt), st, sh, cfg0 + c, n, nsplit, (int)grouped,
                           rec + (size_t)c * 2 * sh.Lt);
        return hipGetLastError();
    });
}

}  // namespace

const char* timecorr_unsupported(const ShapeDev& sh) {
    if (sh.R < 1 || sh.R > 6) return "two-time records need 1 to 6 replicas";
    if (sh.L > 32) return "two-time records need L <= 32";
    if (sh.Lt > kMaxLtTime) return "two-time records need Ltau <= 4096";
    return nullptr;
}

size_t timecorr_record_bytes(const ShapeDev& sh, int ncfg) { return (size_t)ncfg * 2 * sh.Lt * 8; }

hipError_t launch_timecorr(const ShapeDev& sh, int cfg0, int ncfg, int64_t* rec, hipStream_t st) {
    if (ncfg <= 0) return hipSuccess;
    const bool wide = (unsigned long long)sh.R * sh.L2 * sh.L2 * sh.Lt >= 1ull << 32;
    if (sh.nx & 1)
        return wide ? launch_timecorr_as<true, true>(sh, cfg0, ncfg, rec, st)
                    : launch_timecorr_as<true, false>(sh, cfg0, ncfg, rec, st);
    return wide ? launch_timecorr_as<false, true>(sh, cfg0, ncfg, rec, st)
                : launch_timecorr_as<false, false>(sh, cfg0, ncfg, rec, st);
}

}  // namespace tfim
