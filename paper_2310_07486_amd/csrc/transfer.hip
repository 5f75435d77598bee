// Transfer matrix of one plane: matrix-free product and the largest
// eigenvalue of each parity sector.
//
// Paper: arXiv:2310.07486, Methods, "The Trotter-Suzuki formula" (the weight
// exp(-k E) of the L x L x Ltau lattice, Z = Tr T^Ltau with the transfer
// matrix T between consecutive planes, and the parity operator for the
// antiperiodic boundary) and "Simulation details" (exact diagonalisation of
// the transfer matrix, in parity sectors of half the size).
//
// With E0(s) = sum over spatial bonds (each once) of J_b s_x s_y,
//   T = D^1/2 K D^1/2,  D = diag(exp(k E0)),  K = (x)_x [[e^k, e^-k], [e^-k, e^k]],
// on 2^N states (N = L^2; bit x of the index is set when s_x = -1).  K is
// applied as N two-term butterflies, one per bit: w[s] <- e^k w[s] +
// e^-k w[s ^ 2^x].  L = 5: two passes over the vector, on tiles of 2^14 states
// in registers (k_tm_half).  L = 4: tiles of 4096 states (32 KB of LDS), first
// on bits 0..11 of contiguous chunks (and the D^1/2 scale on the way in), then
// in place on the other 4 bits with columns of 256 consecutive lower indices,
// scaling by D^1/2 on the way out.  N <= 12 (L = 2, 3) takes one block per 2^N
// states.  E0(s) comes from popcounts of s xor its neighbour-permuted copies
// against the masks of the +1 and -1 couplings; exp(k E0 / 2) is a table of
// 4N + 1 entries.
#include <algorithm>
#include <cmath>
#include <vector>

#include "tfim_internal.h"

namespace tfim {
namespace {

constexpr int kLowBits = 12;   // bits of the first pass (4096 states per block)
constexpr int kMaxN = 25;      // L <= 5

struct TmParams {
    int N, L, S0;              // sites, edge, sum of all couplings
    uint32_t jxp, jxm, jyp, jym, lastcol, full;
    double a, b;               // e^k, e^-k
    double dtab[4 * kMaxN + 1];  // exp(k E0 / 2) at E0 + 2N
};

// E0(s) + 2N, the index of exp(k E0 / 2) in a table
__device__ __forceinline__ int diag_code(const TmParams& P, uint32_t s) {
    // neighbour-permuted copies: bit i of rx is the bit of the +x neighbour of i
    const uint32_t rx = ((s >> 1) & ~P.lastcol) | ((s << (P.L - 1)) & P.lastcol);
    const uint32_t ry = ((s >> P.L) | (s << (P.N - P.L))) & P.full;
    const uint32_t dx = s ^ rx, dy = s ^ ry;
    const int e0 = P.S0 - 2 * (__popc(dx & P.jxp) - __popc(dx & P.jxm) + __popc(dy & P.jyp) -
                               __popc(dy & P.jym));
    return e0 + 2 * P.N;
}

__device__ __forceinline__ double half_diag(const TmParams& P, uint32_t s, const double* dt) {
    return dt[diag_code(P, s)];
}

// in -> out: D^1/2 scale, butterflies of bits 0 .. nlow-1 on chunks of 2^nlow
// contiguous states, and the final D^1/2 scale when no pass follows.
__global__ void __launch_bounds__(256) k_tm_low(TmParams P, const double* __restrict__ in,
                                                double* __restrict__ out, int nlow, int last) {
    __shared__ double sh[1 << kLowBits];
    __shared__ double dt[4 * kMaxN + 1];
    const int tid = threadIdx.x;
    const int chunk = 1 << nlow;
    const uint32_t base = (uint32_t)blockIdx.x << nlow;
    for (int e = tid; e < 4 * P.N + 1; e += 256) dt[e] = P.dtab[e];
    __syncthreads();
    for (int e = tid; e < chunk; e += 256) sh[e] = in[base + e] * half_diag(P, base + e, dt);
    __syncthreads();
    for (int j = 0; j < nlow; ++j) {
        for (int p = tid; p < chunk / 2; p += 256) {
            const int i0 = ((p >> j) << (j + 1)) | (p & ((1 << j) - 1));
            const int i1 = i0 | (1 << j);
            const double x0 = sh[i0], x1 = sh[i1];
            sh[i0] = P.a * x0 + P.b * x1;
            sh[i1] = P.b * x0 + P.a * x1;
        }
        __syncthreads();
    }
    for (int e = tid; e < chunk; e += 256) out[base + e] = last ? sh[e] * half_diag(P, base + e, dt) : sh[e];
}

// One pass over tiles of 4096 states: rows g = the nb bits bit0 .. bit0+nb-1
// of the index, columns c = C = 4096 / 2^nb consecutive indices below bit0
// (C = 1 in the first pass), one tile per value of the bits above.  Each
// thread holds 16 states whose row indices differ in four bits and applies
// those four butterflies in registers; LDS exchanges the states between
// groups of four bits (nb is a multiple of 4).  Optional D^1/2 scale on the way in and on the way
// out; in and out may be the same vector (each tile is read whole first).
__global__ void __launch_bounds__(256) k_tm_tile(TmParams P, const double* in, double* out, int bit0, int nb,
                                                 int first, int last) {
    __shared__ double sh[4096 + 4096 / 32];
    __shared__ double dt[4 * kMaxN + 1];
    const int tid = threadIdx.x;
    const int C = 4096 >> nb;
    const int nlo = 1 << bit0;                 // indices below bit0
    const uint32_t tiles_lo = (uint32_t)(nlo / C);
    const uint32_t lo0 = (blockIdx.x % tiles_lo) * (uint32_t)C;
    const uint32_t hi = blockIdx.x / tiles_lo;
    const uint32_t base = lo0 + (hi << (bit0 + nb));
    auto pad = [](int e) { return e + (e >> 5); };  // one spare slot per 32 doubles
    auto gidx = [&](int e) -> uint32_t { return base + (uint32_t)(e % C) + ((uint32_t)(e / C) << bit0); };
    for (int e = tid; e < 4 * P.N + 1; e += 256) dt[e] = P.dtab[e];
    if (first) __syncthreads();
    double r[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int e = tid + 256 * i;
        const uint32_t s = gidx(e);
        r[i] = first ? in[s] * half_diag(P, s, dt) : in[s];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) sh[pad(tid + 256 * i)] = r[i];
    __syncthreads();
    for (int b0 = nb - 4; b0 >= 0; b0 -= 4) {  // groups of four row bits, from the top
        const int o = tid / C, c = tid % C;
        const int g0 = ((o >> b0) << (b0 + 4)) | (o & ((1 << b0) - 1));
#pragma unroll
        for (int i = 0; i < 16; ++i) r[i] = sh[pad((g0 | (i << b0)) * C + c)];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (!(i & (1 << j))) {
                    const double x0 = r[i], x1 = r[i | (1 << j)];
                    r[i] = P.a * x0 + P.b * x1;
                    r[i | (1 << j)] = P.b * x0 + P.a * x1;
                }
#pragma unroll
        for (int i = 0; i < 16; ++i) sh[pad((g0 | (i << b0)) * C + c)] = r[i];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int e = tid + 256 * i;
        const uint32_t s = gidx(e);
        const double x = sh[pad(e)];
        out[s] = last ? x * half_diag(P, s, dt) : x;
    }
}

// Projection on a parity sector: w[s], w[~s] <- (w[s] + sign w[~s]) / 2, sign w[s].
__global__ void k_tm_project(double* __restrict__ w, uint32_t n, double sign) {
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n / 2; s += gridDim.x * blockDim.x) {
        const uint32_t t = n - 1 - s;
        const double m = 0.5 * (w[s] + sign * w[t]);
        w[s] = m;
        w[t] = sign * m;
    }
}

// Per-block partial sums of <x, y>, <y, y> and, when z is given, <z, y>
// (summed on the host in block order).
constexpr int kDotBlocks = 1024;
__global__ void __launch_bounds__(256) k_tm_dots(const double* __restrict__ x, const double* __restrict__ y,
                                                 const double* __restrict__ z, uint32_t n,
                                                 double* __restrict__ part) {
    __shared__ double r0[256], r1[256], r2[256];
    double a = 0.0, c = 0.0, d = 0.0;
    for (uint32_t s = blockIdx.x * 256 + threadIdx.x; s < n; s += kDotBlocks * 256) {
        const double ys = y[s];
        a += x[s] * ys;
        c += ys * ys;
        if (z) d += z[s] * ys;
    }
    r0[threadIdx.x] = a;
    r1[threadIdx.x] = c;
    r2[threadIdx.x] = d;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            r0[threadIdx.x] += r0[threadIdx.x + o];
            r1[threadIdx.x] += r1[threadIdx.x + o];
            r2[threadIdx.x] += r2[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x] = r0[0];
        part[kDotBlocks + blockIdx.x] = r1[0];
        part[2 * kDotBlocks + blockIdx.x] = r2[0];
    }
}

// v = (w - c z) f  (z may be null: v = w f); v may be w
__global__ void k_tm_next(const double* w, const double* __restrict__ z, double c, double f, uint32_t n,
                          double* v) {
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n; s += gridDim.x * blockDim.x)
        v[s] = (z ? w[s] - c * z[s] : w[s]) * f;
}

// ---------------------------------------------------------------------------
// Power iteration of L <= 4 in one workgroup
//
// A sector's vector is given by its first half h = 2^(N-1): v[~s] = sign v[s].
// The butterfly of bit N-1 then joins s and its complement among the other
// N-1 bits.  All K products have the factor e^k taken out of them (w[s] <-
// v[s] + e^-2k v[s ^ bit], one fused multiply-add per state; D takes its N-th
// power).  The eigenvalues are as accurate as with both factors (mean error against
// 80-bit arithmetic 1.4e-16 and 3.6e-16 at L = 2 and 3, with both factors 2.8e-16 and
// 5.2e-16; 40 and 24 samples, k = 0.1 .. 0.35, both sectors), since the Rayleigh
// quotient takes an error of the vector squared; a product by itself would lose
// (k_tm_half).  The iteration runs on y = D^1/2 v: with x = K y, <v, T v> = sum y x,
// |T v|^2 = sum D x^2, and the next y is (D x - c D^1/2 z) f, one factor per
// state where v takes two.  The sums, the normalisation and the stopping rule
// stay on the device: at L = 4 a product with separate kernels and a read-back
// of its sums took 38 us, nearly all of it launches and the wait; here 13
// (25 where the second eigenvector keeps clear of the first).
// ---------------------------------------------------------------------------
struct TmState {  // between launches of one iteration
    double lam, prev;
    int it, done;
};

struct TmPower {
    TmParams P;                  // dtab: D^1/2 with the e^kN/2 of K
    double dfull[4 * kMaxN + 1]; // D
    double t;             // e^-2k
    double sign;          // of the sector
    double tol;
    int max_iter, slice;  // products in all and in this launch
    double* v;            // out: the eigenvector, 2^N; meanwhile y and D^1/2 z
    const double* defl;   // z, a unit vector kept out of the iteration, or null
    double* ws;           // 2^N doubles of scratch
    TmState* state;
};

__device__ __forceinline__ double tm_start_value(uint32_t s, uint32_t n, double sign, bool second) {
    // the top: all ones (even sector) or +1 / -1 halves (odd sector); the
    // second: a fixed pseudo-random vector, projected on the sector below
    if (!second) return (sign > 0.0 || s < n / 2) ? 1.0 : -1.0;
    uint32_t h = s * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    h ^= h >> 13;
    return (double)(h & 0xFFFFu) / 32768.0 - 1.0;
}

__global__ void k_tm_start(double* __restrict__ v, uint32_t n, double sign, int second) {
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n; s += gridDim.x * blockDim.x)
        v[s] = tm_start_value(s, n, sign, second != 0);
}

// sums over the workgroup of three doubles, the same in every thread
__device__ __forceinline__ void tm_block_sums(double (&d)[3], double* red) {
    for (int o = 32; o; o >>= 1)
#pragma unroll
        for (int q = 0; q < 3; ++q) d[q] += __shfl_xor(d[q], o);
    const int nw = blockDim.x / 64;
    __syncthreads();  // earlier readers of red
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int q = 0; q < 3; ++q) red[3 * (threadIdx.x >> 6) + q] = d[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        d[q] = 0.0;
        for (int w = 0; w < nw; ++w) d[q] += red[3 * w + q];
    }
}

// What a layout of the half vector's states over threads and registers says
// (constants in i): state() of register i is the thread's plus at(i); a vector
// in the layout's order holds it at i * blockDim + tid; put() + put_at(i) is its
// place in the order of the layout that the next product ends on.

// L = 2, 3: a state per thread
struct TmOne {
    static constexpr __device__ uint32_t state(int tid) { return (uint32_t)tid; }
    static constexpr __device__ uint32_t put(int tid) { return (uint32_t)tid; }
    static constexpr __device__ uint32_t at(int) { return 0; }
    static constexpr __device__ uint32_t put_at(int) { return 0; }
};

// L = 4: 2^15 states in the registers of 512 threads, 64 each.  Layout 0 has
// index bits 0..5 on the lanes, 6..8 on the waves, 9..14 on the registers
// (slots 0..5); layout 1 has 0,1,10,3,11,9 on the lanes, 12..14 on the waves
// and 5,2,4,6,7,8 on the registers.
template <int kLay>
struct Tm16 {
    static constexpr __device__ uint32_t bits(int v, const int (&to)[6]) {
        uint32_t s = 0;
        for (int j = 0; j < 6; ++j) s |= (uint32_t)((v >> j) & 1) << to[j];
        return s;
    }
    static constexpr __device__ uint32_t at(int i) {
        const int slot0[6] = {9, 10, 11, 12, 13, 14}, slot1[6] = {5, 2, 4, 6, 7, 8};
        return kLay ? bits(i, slot1) : bits(i, slot0);
    }
    static constexpr __device__ uint32_t state(int tid) {
        const int lane0[6] = {0, 1, 2, 3, 4, 5}, lane1[6] = {0, 1, 10, 3, 11, 9};
        return (uint32_t)(tid >> 6) << (kLay ? 12 : 6) | (kLay ? bits(tid, lane1) : bits(tid, lane0));
    }
    // layout 0's order is the states' own; of layout 1, bits 0,1,10,3,11,9,12..14
    // are the thread and 5,2,4,6,7,8 the register
    static constexpr __device__ uint32_t put_at(int i) {
        const int slot[6] = {5, 2, 4, 6, 7, 8};
        return bits(i, slot);
    }
    static constexpr __device__ uint32_t put(int tid) {
        const int lane0[6] = {0, 1, 10, 3, 11, 9};
        return kLay ? state(tid) : (uint32_t)(tid >> 6) << 12 | bits(tid, lane0);
    }
};

// doubles at p: one offset register for all of a thread's, the constant part beside it
struct TmBuf {
    __amdgpu_buffer_rsrc_t d;
    __device__ TmBuf(const double* p, uint32_t n) {
        d = __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)(n * 8), 0x00020000);
    }
    __device__ __forceinline__ double get(int voff, int soff) const {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(d, voff, soff, 0));
    }
    __device__ __forceinline__ uint64_t word(int voff, int soff) const {
        return __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(d, voff, soff, 0));
    }
    __device__ __forceinline__ void put(double x, int voff, int soff) const {
        typedef unsigned v2u __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, x), d, voff, soff, 0);
    }
};

// last() finishes x = K y in r, R values of threads with on: then the Rayleigh
// quotient, removal of z, normalisation into r and y.  table(i, ..) is D at
// registers i, i + 1, ..; zb + zy is D^1/2 z in this layout's order.  Reads run a batch
// ahead of their use.  True when the iteration has ended.
template <int R, bool kDefl, class Lay, class Last, class Codes, class Table>
__device__ __forceinline__ bool tm_finish(const TmPower& A, double (&r)[R], const TmBuf& yb, const TmBuf& zb, int zy,
                                          Last last, Codes codes, Table table, bool on, TmState& st, double* red) {
    constexpr int kB = R < 8 ? R : 8;  // values of a batch, summed as a tree
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // no table of addresses kept over the loop
    const int nthr = R == 1 ? (int)blockDim.x : 512;
    double y[2][kB], z[2][kB];
    uint64_t u[2];
    auto fetch = [&](int i0, bool with_y) {
        const int k = (i0 / kB) & 1;
        if (with_y) {
            u[k] = codes(8 * tid, i0);
#pragma unroll
            for (int i = 0; i < kB; ++i) y[k][i] = on ? yb.get(8 * tid, (i0 + i) * nthr * 8) : 0.0;
        }
        if (kDefl)
#pragma unroll
            for (int i = 0; i < kB; ++i) z[k][i] = on ? zb.get(8 * tid, zy + (i0 + i) * nthr * 8) : 0.0;
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, true);
    last();
    double d[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i0 = 0; i0 < R; i0 += kB) {
        const int k = (i0 / kB) & 1;
        if (i0 + kB < R) fetch(i0 + kB, true);
        double g[kB];
        table(u[k], g);
#pragma unroll
        for (int i = 0; i < kB; ++i) {
            const double x = r[i0 + i];
            y[k][i] *= x;
            if (kDefl) z[k][i] *= x;
            r[i0 + i] = g[i] * x;
            g[i] = r[i0 + i] * x;
        }
#pragma unroll
        for (int o = kB / 2; o; o >>= 1)
#pragma unroll
            for (int i = 0; i < o; ++i) {
                y[k][i] += y[k][i + o];
                g[i] += g[i + o];
                if (kDefl) z[k][i] += z[k][i + o];
            }
        d[0] += y[k][0];
        d[1] += g[0];
        if (kDefl) d[2] += z[k][0];
        __builtin_amdgcn_sched_barrier(0);
    }
    fetch(0, false);
    if (R > kB) fetch(kB, false);
    tm_block_sums(d, red);  // and every y has been read
    // each state of the half stands for two
    const double c = kDefl ? 2.0 * d[2] : 0.0, f = 1.0 / sqrt(2.0 * d[1] - c * c);
    const int out = 8 * (int)Lay::put(tid);
#pragma unroll
    for (int i0 = 0; i0 < R; i0 += kB) {
        const int k = (i0 / kB) & 1;
#pragma unroll
        for (int i = 0; i < kB; ++i) {
            r[i0 + i] = (kDefl ? r[i0 + i] - c * z[k][i] : r[i0 + i]) * f;
            if (on) yb.put(r[i0 + i], out + 8 * (int)Lay::put_at(i0 + i), 0);
        }
        if (i0 + 2 * kB < R) fetch(i0 + 2 * kB, false);
    }
    st.prev = st.lam;
    st.lam = 2.0 * d[0];
    const bool end = st.it >= 2 && fabs(st.lam - st.prev) <= A.tol * fabs(st.lam);
    ++st.it;
    st.done = end || st.it >= A.max_iter;
    return st.done;
}

// y = D^1/2 v of the unit start vector, or (later launches) y so far
template <int R, bool kDefl, class Lay>
__device__ __forceinline__ void tm_begin(const TmPower& A, double (&r)[R], const double* half, bool on, TmState& st,
                                         double* red) {
    const uint32_t n = 1u << A.P.N, base = Lay::state(threadIdx.x);
    double* const out = A.v + Lay::put(threadIdx.x);
    st = *A.state;
    if (st.it > 0) {
#pragma unroll
        for (int i = 0; i < R; ++i) r[i] = on ? out[Lay::put_at(i)] : 0.0;
        __syncthreads();
        return;
    }
    double d[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t s = base + Lay::at(i);
        r[i] = on ? 0.5 * (tm_start_value(s, n, A.sign, kDefl) +
                           A.sign * tm_start_value(n - 1 - s, n, A.sign, kDefl))
                  : 0.0;
        d[1] += r[i] * r[i];
        if (kDefl && on) d[2] += A.defl[s] * r[i];
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    tm_block_sums(d, red);
    const double c = kDefl ? 2.0 * d[2] : 0.0, f = 1.0 / sqrt(2.0 * d[1] - c * c);
    if (on)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint32_t s = base + Lay::at(i);
            if (kDefl) r[i] -= c * A.defl[s];
            r[i] = r[i] * f * half_diag(A.P, s, half);
            out[Lay::put_at(i)] = r[i];
            if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    __syncthreads();
}

// the eigenvector, both halves, from y as this layout's tm_finish left it
template <int R, class Lay>
__device__ __forceinline__ void tm_vector(const TmPower& A, const double* half, bool on) {
    const int tid = threadIdx.x;
    const uint32_t n = 1u << A.P.N, base = Lay::state(tid);
    const double* const in = A.v + Lay::put(tid);
    double r[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        r[i] = on ? in[Lay::put_at(i)] / half_diag(A.P, base + Lay::at(i), half) : 0.0;
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();  // y has been read
    if (!on) return;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        A.v[base + Lay::at(i)] = r[i];
        A.v[n - 1 - (base + Lay::at(i))] = A.sign * r[i];
    }
}

// an LDS exchange per bit
template <bool kDefl>
__global__ void __launch_bounds__(256) k_tm_power_small(TmPower A) {
    __shared__ double x[2][256];
    __shared__ double red[12], half[37], full[37];  // D^1/2 and D by E0 + 2N
    const int h = 1 << (A.P.N - 1), tid = threadIdx.x;
    const bool on = tid < h;
    const TmBuf yb(A.v, 2 * h), zb(A.ws, 2 * h);
    double r[1];
    TmState st;
    if (tid < 4 * 9 + 1) half[tid] = A.P.dtab[tid], full[tid] = A.dfull[tid];
    __syncthreads();
    const int code = on ? diag_code(A.P, tid) : 0;
    const double dg = full[code];
    if (kDefl && on) A.ws[tid] = A.defl[tid] * half[code];
    tm_begin<1, kDefl, TmOne>(A, r, half, on, st, red);
    for (int k = 0; k < A.slice && !st.done; ++k) {
        for (int b = 0; b < A.P.N; ++b) {
            x[b & 1][tid] = r[0];
            __syncthreads();
            const int o = b < A.P.N - 1 ? tid ^ (1 << b) : tid ^ (h - 1);
            const double y = x[b & 1][o & 255];
            if (on) r[0] = fma(b < A.P.N - 1 ? A.t : A.t * A.sign, y, r[0]);
        }
        tm_finish<1, kDefl, TmOne>(
            A, r, yb, zb, 0, [] {}, [](int, int) { return 0ull; }, [&](uint64_t, double (&g)[1]) { g[0] = dg; }, on,
            st, red);
    }
    if (st.done) tm_vector<1, TmOne>(A, half, on);
    if (tid == 0) *A.state = st;
}

template <int kCtrl>
__device__ __forceinline__ double dpp_mov(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), kCtrl, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// swap slot 0 with lane bit 5: x of the upper lanes against y of the lower
__device__ __forceinline__ void swap_lane5(double& x, double& y) {
    const uint64_t a = __builtin_bit_cast(uint64_t, x), b = __builtin_bit_cast(uint64_t, y);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    x = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]);
    y = __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

__device__ __forceinline__ void tm16_slots(double (&r)[64], double t) {
#pragma unroll
    for (int j = 0; j < 6; ++j)
#pragma unroll
        for (int i = 0; i < 64; ++i)
            if (!(i & (1 << j))) {
                const double x0 = r[i], x1 = r[i | (1 << j)];
                r[i] = fma(t, x1, x0);
                r[i | (1 << j)] = fma(t, x0, x1);
                if ((i & 6) == 6) __builtin_amdgcn_sched_barrier(0);
            }
}

// LDS place of bits 0..4, 9, 6..8, 10..14 (bit 5 is the round), with bits 10
// and 11 added to the bank bits 2 and 4, which both layouts' lanes then spread:
// element (tid, slots 1..5 = e) of layout kLay, or its complement
template <int kLay, bool kFlip>
__device__ __forceinline__ int tm16_place(int tid, int e) {
    const int l = tid & 63, w = tid >> 6, f = kFlip ? 31 : 0;
    constexpr int kMask = 0x3fff & ~0x14;
    if (kLay == 0) {  // slot 1 = bit 10, slot 2 = bit 11; lane 5 = bit 9
        const int b = ((l & 31) | (l >> 5) << 5 | w << 6) ^ (kFlip ? kMask & 0x1ff : 0);
        const int k = e & 3, kf = (e ^ f) & 3;
        return (b ^ ((k & 1) << 2 | (k >> 1) << 4)) + (kf << 9) + (((e ^ f) >> 2) << 11);
    }
    // lanes 2, 4, 5 = bits 10, 11, 9; slots 1..5 = bits 2, 4, 6..8
    const int l2 = (l >> 2) & 1, l4 = (l >> 4) & 1;
    const int b = ((l & 0x0b) | l2 << 2 | l4 << 4 | (l >> 5) << 5 | l2 << 9 | l4 << 10 | w << 11) ^
                  (kFlip ? kMask & ~0x1c0 : 0);
    const int k = e & 3;
    return (b ^ ((k & 1) << 2 | (k >> 1) << 4)) + (((e ^ f) >> 2) << 6);
}

// A product works on its layout's register bits, on lanes 0, 1 and 3 by
// data-parallel moves, swaps lane 5 with slot 0, exchanges the rest through LDS
// in two rounds (bit 5 = 0, 1; the complement of a state is in the other
// round's registers), and ends on the other layout's register bits; the next
// goes back.  Bound by the vector ALU of one CU, 16 multiply-adds and 9 moves
// per state, and by 3 LDS accesses and 2 to 4 of L2 per state.
template <int kLay>
__device__ __forceinline__ void tm16_product(double (&r)[64], double t, double ts, double* sh) {
    constexpr int kOut = 1 - kLay;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // no addresses kept over the loop
    tm16_slots(r, t);
#pragma unroll
    for (int i = 0; i < 64; ++i) {
        r[i] = fma(t, dpp_mov<0xB1>(r[i]), r[i]);   // quad_perm 1,0,3,2
        r[i] = fma(t, dpp_mov<0x4E>(r[i]), r[i]);   // quad_perm 2,3,0,1
        r[i] = fma(t, dpp_mov<0x128>(r[i]), r[i]);  // row_ror 8
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (kLay == 0)
#pragma unroll
        for (int i = 0; i < 64; i += 2) swap_lane5(r[i], r[i + 1]);
    double y[32];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 32; ++e) sh[tm16_place<kLay, false>(tid, e)] = r[2 * e + h];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 32; ++e) r[2 * e + h] = sh[tm16_place<kOut, false>(tid, e)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const double z = sh[tm16_place<kOut, true>(tid, e)];
            if (h == 0)
                y[e] = z;
            else
                r[2 * e] = fma(ts, z, r[2 * e]);
            if (e % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int e = 0; e < 32; ++e) r[2 * e + 1] = fma(ts, y[e], r[2 * e + 1]);
}

template <int kLay>
__device__ __forceinline__ void tm16_last(double (&r)[64], double t) {
    if (kLay == 1)
#pragma unroll
        for (int i = 0; i < 64; i += 2) swap_lane5(r[i], r[i + 1]);
    tm16_slots(r, t);
}

template <bool kDefl>
__global__ void __launch_bounds__(512) k_tm_power16(TmPower A) {
    __shared__ double sh[1 << 14];
    __shared__ double dt[17];  // D at E0 = E0 of s = 0 modulo 4, the values there are
    __shared__ double red[24], half[65];
    const int tid = threadIdx.x, rem = diag_code(A.P, 0) & 3;
    double r[64];
    TmState st;
    if (tid < 65) {
        half[tid] = A.P.dtab[tid];
        if ((tid & 3) == rem) dt[tid >> 2] = A.dfull[tid];
    }
    __syncthreads();
    // per layout: a byte per state in [8 registers][tid][8], and D^1/2 z in
    // the layout's order; each thread writes and reads its own
    uint8_t* const codes = (uint8_t*)A.ws;
    double* const zy0 = A.v + (1 << 15);
    double* const zy1 = A.ws + (1 << 15);
#pragma unroll 4
    for (int i = 0; i < 64; ++i) {
        const uint32_t s0 = Tm16<0>::state(tid) + Tm16<0>::at(i), s1 = Tm16<1>::state(tid) + Tm16<1>::at(i);
        const int c0 = diag_code(A.P, s0), c1 = diag_code(A.P, s1), p = (i / 8 * 512 + tid) * 8 + i % 8;
        codes[p] = (uint8_t)(c0 >> 2);
        codes[(1 << 15) + p] = (uint8_t)(c1 >> 2);
        if (kDefl) {
            zy0[i * 512 + tid] = A.defl[s0] * half[c0];
            zy1[i * 512 + tid] = A.defl[s1] * half[c1];
        }
    }
    const TmBuf yb(A.v, 1 << 16), ws(A.ws, 1 << 16);
    auto table = [&](uint64_t u, double (&g)[8]) {
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = dt[(uint32_t)(u >> (8 * k)) & 255];
    };
    auto codes0 = [&](int voff, int i0) { return ws.word(voff, i0 * 512); };
    auto codes1 = [&](int voff, int i0) { return ws.word(voff, (1 << 15) + i0 * 512); };
    const double t = A.t, ts = A.t * A.sign;
    tm_begin<64, kDefl, Tm16<0>>(A, r, half, true, st, red);
#pragma unroll 1
    for (int k = 0; k < A.slice && !st.done; k += 2) {
        tm16_product<0>(r, t, ts, sh);
        if (tm_finish<64, kDefl, Tm16<1>>(A, r, yb, ws, 8 << 15, [&] { tm16_last<0>(r, t); }, codes1, table, true,
                                          st, red))
            break;
        tm16_product<1>(r, t, ts, sh);
        tm_finish<64, kDefl, Tm16<0>>(A, r, yb, yb, 8 << 15, [&] { tm16_last<1>(r, t); }, codes0, table, true, st,
                                      red);
    }
    if (st.done) {  // in layout 1 after an odd number of products
        if (st.it & 1)
            tm_vector<64, Tm16<1>>(A, half, true);
        else
            tm_vector<64, Tm16<0>>(A, half, true);
    }
    if (tid == 0) *A.state = st;
}

// ---------------------------------------------------------------------------
// The product of L = 5 in two passes, 14 bits and 11
//
// Tiles of 2^14 states in the registers of 512 threads, 32 each: the first
// pass on bits 0..13 of contiguous states, with D^1/2 on the way in, the second
// in place on bits 14..24 of 8 columns (64-byte rows), with D^1/2 on the way
// out.  By positions p (p0 = slot 0, p1..p9 = the thread,
// p10..p13 = slots 1..4; the second pass's p0..p2 are its columns): slots first,
// an exchange through 64 KB of LDS in two rounds (by p0) of lane 2 and the
// waves against slots 1..4, lanes 5 and 4 swapped with slots 1 and 2, the other
// lanes by data-parallel moves.  Two workgroups per CU, one's loads under the
// other's arithmetic.  Bound by memory, a read and a write of the vector per
// pass: three passes of 12 + 8 + 5 bits took 326 us at L = 5, these 103 + 128
// (copy rate: 107 each).  The butterflies keep both factors: with e^k taken out
// the error of a product against 64 bits grew from 1.3e-16 to 7.6e-16, for 5 us.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void swap_lane4(double& x, double& y) {
    const uint64_t a = __builtin_bit_cast(uint64_t, x), b = __builtin_bit_cast(uint64_t, y);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    x = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]);
    y = __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

typedef double Pair8 __attribute__((ext_vector_type(2), aligned(8)));  // vectors come 8-byte aligned

template <bool kHigh>
__global__ void __launch_bounds__(512, 4) k_tm_half(TmParams P, const double* in, double* out) {
    __shared__ double sh[1 << 13];
    __shared__ double dt[4 * kMaxN + 1];
    const int tid = threadIdx.x;
    // 32 neighbouring tiles (2 KB of a row) on an XCD at a time, the XCDs side by
    // side: the tiles in flight cover the channels and share lines.  Second pass
    // 20 us longer with 16 KB to an XCD, 8 with 512 bytes.
    const uint32_t xcd = blockIdx.x & 7, j0 = blockIdx.x >> 3;
    const uint32_t tile = kHigh ? (j0 & ~31u) << 3 | xcd << 5 | (j0 & 31) : blockIdx.x;
    const double a = P.a, b = P.b;
    // positions to index bits
    auto spread = [](uint32_t p) { return kHigh ? (p & 7) | (p & ~7u) << 11 : p; };
    const uint32_t base = tile << (kHigh ? 3 : 14);
    auto bit = [&](int j) { return (uint32_t)(tid >> j) & 1; };
    for (int e = tid; e < 4 * P.N + 1; e += 512) dt[e] = P.dtab[e];
    double r[32];
    const uint32_t s0 = base + spread((uint32_t)tid << 1);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const Pair8 v = *(const Pair8*)(in + s0 + spread((uint32_t)e << 10));
        r[2 * e] = v.x;
        r[2 * e + 1] = v.y;
    }
    if (!kHigh) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 32; ++i) r[i] *= half_diag(P, s0 + ((uint32_t)(i >> 1) << 10) + (i & 1), dt);
    }
    auto slot = [&](int j) {
#pragma unroll
        for (int i = 0; i < 32; ++i)
            if (!(i & (1 << j))) {
                const double x0 = r[i], x1 = r[i | (1 << j)];
                r[i] = a * x0 + b * x1;
                r[i | (1 << j)] = b * x0 + a * x1;
            }
    };
#pragma unroll
    for (int j = kHigh ? 1 : 0; j < 5; ++j) slot(j);
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        if (!kHigh) {
            r[i] = a * r[i] + b * dpp_mov<0xB1>(r[i]);  // quad_perm 1,0,3,2
            r[i] = a * r[i] + b * dpp_mov<0x4E>(r[i]);  // quad_perm 2,3,0,1
        }
        r[i] = a * r[i] + b * dpp_mov<0x128>(r[i]);     // row_ror 8
    }
    // LDS place of p1..p13, with p10 added to p3 for the banks
    const int put0 = tid, put1 = (tid ^ 4) + (1 << 9);
    const int get = (tid & 0x3b) | (int)(bit(2) << 2 | bit(2) << 9) | (tid >> 6) << 10;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) sh[((e & 1) ? put1 : put0) + ((e >> 1) << 10)] = r[2 * e + h];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) r[2 * e + h] = sh[((e & 1) ? get ^ 4 : get) + ((e >> 1) << 6)];
    }
#pragma unroll
    for (int j = 1; j < 5; ++j) slot(j);  // p3, p7, p8, p9
#pragma unroll
    for (int i = 0; i < 32; ++i)
        if (!(i & 2)) swap_lane5(r[i], r[i | 2]);
    slot(1);  // p6
#pragma unroll
    for (int i = 0; i < 32; ++i)
        if (!(i & 4)) swap_lane4(r[i], r[i | 4]);
    slot(2);  // p5
    // now p1,p2,p10,p4,p7,p3 on the lanes, p11..p13 on the waves, p0,p6,p5,p8,p9 on the slots
    const uint32_t s1 = base + spread(bit(0) << 1 | bit(1) << 2 | bit(2) << 10 | bit(3) << 4 | bit(4) << 7 |
                                      bit(5) << 3 | (uint32_t)(tid >> 6) << 11);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const uint32_t s = s1 + spread((e & 1) << 6 | ((e >> 1) & 1) << 5 | (uint32_t)(e >> 2) << 8);
        Pair8 v = {r[2 * e], r[2 * e + 1]};
        if (kHigh) {
            v.x *= half_diag(P, s, dt);
            v.y *= half_diag(P, s + 1, dt);
        }
        *(Pair8*)(out + s) = v;
    }
}

}  // namespace

const char* tm_unsupported(int L) {
    if (L < 2 || L * L > kMaxN) return "transfer matrix needs 2 <= L <= 5";
    return nullptr;
}

size_t tm_workspace_bytes(int L) {
    const size_t n = (size_t)1 << (L * L);
    return 3 * n * 8 + 3 * kDotBlocks * 8 + 256;
}

static TmParams tm_params(int L, double k, const int8_t* Jx, const int8_t* Jy) {
    TmParams P{};
    P.L = L;
    P.N = L * L;
    P.full = P.N == 32 ? 0xFFFFFFFFu : ((1u << P.N) - 1u);
    int S0 = 0;
    for (int i = 0; i < P.N; ++i) {
        if (Jx[i] > 0) P.jxp |= 1u << i; else P.jxm |= 1u << i;
        if (Jy[i] > 0) P.jyp |= 1u << i; else P.jym |= 1u << i;
        S0 += Jx[i] + Jy[i];
        if (i % L == L - 1) P.lastcol |= 1u << i;
    }
    P.S0 = S0;
    P.a = std::exp(k);
    P.b = std::exp(-k);
    for (int e = -2 * P.N; e <= 2 * P.N; ++e) P.dtab[e + 2 * P.N] = std::exp(0.5 * k * (double)e);
    return P;
}

static hipError_t tm_apply_params(const TmParams& P, const double* v, double* w, hipStream_t st) {
    const uint32_t n = 1u << P.N;
    if (P.N == kMaxN) {
        hipLaunchKernelGGL(k_tm_half<false>, dim3(n >> 14), dim3(512), 0, st, P, v, w);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_tm_half<true>, dim3(n >> 14), dim3(512), 0, st, P, (const double*)w, w);
        return hipGetLastError();
    }
    if (P.N == kLowBits + 4) {
        hipLaunchKernelGGL(k_tm_tile, dim3(n / 4096), dim3(256), 0, st, P, v, w, 0, kLowBits, 1, 0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_tm_tile, dim3(n / 4096), dim3(256), 0, st, P, (const double*)w, w, kLowBits, 4, 0, 1);
        return hipGetLastError();
    }
    if (P.N > kLowBits) return hipErrorInvalidValue;  // N = L^2 is 4, 9, 16 or 25
    hipLaunchKernelGGL(k_tm_low, dim3(n >> P.N), dim3(256), 0, st, P, v, w, P.N, 1);
    return hipGetLastError();
}

hipError_t tm_apply(int L, double k, const int8_t* Jx, const int8_t* Jy, const double* v, double* w,
                    hipStream_t st) {
    return tm_apply_params(tm_params(L, k, Jx, Jy), v, w, st);
}

// Power iteration in one parity sector; with defl, every product has the
// component along the unit vector defl removed (the second eigenvalue).
static hipError_t tm_power(const TmParams& P, double sign, double tol, int max_iter, double* v, double* w,
                           const double* defl, double* part, std::vector<double>& hp, double* lambda,
                           int* iters, hipStream_t st) {
    const uint32_t n = 1u << P.N;
    const int grid = (int)std::min<uint32_t>(8192, (n + 255) / 256);
    auto sums = [&](const double* x, const double* y, const double* z, double out[3]) -> hipError_t {
        hipLaunchKernelGGL(k_tm_dots, dim3(kDotBlocks), dim3(256), 0, st, x, y, z, n, part);
        hipError_t e = hipMemcpyAsync(hp.data(), part, hp.size() * 8, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        out[0] = out[1] = out[2] = 0.0;
        for (int q = 0; q < 3; ++q)
            for (int i = 0; i < kDotBlocks; ++i) out[q] += hp[q * kDotBlocks + i];
        return e;
    };
    hipLaunchKernelGGL(k_tm_start, dim3(grid), dim3(256), 0, st, v, n, sign, defl ? 1 : 0);
    hipLaunchKernelGGL(k_tm_project, dim3(grid), dim3(256), 0, st, v, n, sign);
    double d[3];
    hipError_t e = sums(v, v, defl, d);  // |v|^2 and <defl, v>
    if (e != hipSuccess) return e;
    {
        const double c = defl ? d[2] : 0.0;
        const double nn = d[1] - c * c;
        hipLaunchKernelGGL(k_tm_next, dim3(grid), dim3(256), 0, st, v, defl, c, 1.0 / std::sqrt(nn), n, v);
    }
    double lam = 0.0, prev = 0.0;
    int it = 0;
    for (; it < max_iter; ++it) {
        e = tm_apply_params(P, v, w, st);
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_tm_project, dim3(grid), dim3(256), 0, st, w, n, sign);
        if ((e = sums(v, w, defl, d)) != hipSuccess) break;
        prev = lam;
        lam = d[0];  // Rayleigh quotient: v is a unit vector orthogonal to defl
        const double c = defl ? d[2] : 0.0;
        hipLaunchKernelGGL(k_tm_next, dim3(grid), dim3(256), 0, st, w, defl, c,
                           1.0 / std::sqrt(d[1] - c * c), n, v);
        if (it >= 2 && std::fabs(lam - prev) <= tol * std::fabs(lam)) {
            ++it;
            break;
        }
    }
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    *lambda = lam;
    *iters = it;
    return e;
}

// The same in one workgroup (L <= 4), in launches of some tens of ms at most
static hipError_t tm_power_block(const TmParams& P, double k, double sign, double tol, int max_iter, double* v,
                                 double* w, const double* defl, double* part, double* lambda, int* iters,
                                 hipStream_t st) {
    TmPower A{};
    A.P = P;
    for (int e = -2 * P.N; e <= 2 * P.N; ++e) {
        A.P.dtab[e + 2 * P.N] = std::exp(0.5 * k * (double)(e + P.N));
        A.dfull[e + 2 * P.N] = std::exp(k * (double)(e + P.N));
    }
    A.t = std::exp(-2.0 * k);
    A.sign = sign;
    A.tol = tol;
    A.max_iter = max_iter;
    A.slice = 2048;
    A.v = v;
    A.defl = defl;
    A.ws = w;
    A.state = (TmState*)part;
    TmState s{};
    hipError_t e = hipMemcpyAsync(part, &s, sizeof s, hipMemcpyHostToDevice, st);
    while (e == hipSuccess && !s.done) {
        if (P.N == 16)
            hipLaunchKernelGGL(defl ? k_tm_power16<true> : k_tm_power16<false>, dim3(1), dim3(512), 0, st, A);
        else
            hipLaunchKernelGGL(defl ? k_tm_power_small<true> : k_tm_power_small<false>, dim3(1), dim3(256), 0, st, A);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(&s, part, sizeof s, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
    }
    *lambda = s.lam;
    *iters = s.it;
    return e;
}

hipError_t tm_top(int L, double k, const int8_t* Jx, const int8_t* Jy, int odd, int nev, double tol,
                  int max_iter, void* ws, double* lambda, int* iters, hipStream_t st) {
    const TmParams P = tm_params(L, k, Jx, Jy);
    const uint32_t n = 1u << P.N;
    double* v0 = (double*)ws;   // the sector's top eigenvector
    double* v1 = v0 + n;        // the second
    double* w = v1 + n;
    double* part = w + n;
    const double sign = odd ? -1.0 : 1.0;
    hipError_t e = hipSuccess;
    if (P.N <= 16) {
        e = tm_power_block(P, k, sign, tol, max_iter, v0, w, nullptr, part, &lambda[0], &iters[0], st);
        if (e == hipSuccess && nev > 1)
            e = tm_power_block(P, k, sign, tol, max_iter, v1, w, v0, part, &lambda[1], &iters[1], st);
        return e;
    }
    std::vector<double> hp(3 * kDotBlocks);
    e = tm_power(P, sign, tol, max_iter, v0, w, nullptr, part, hp, &lambda[0], &iters[0], st);
    if (e == hipSuccess && nev > 1)
        e = tm_power(P, sign, tol, max_iter, v1, w, v0, part, hp, &lambda[1], &iters[1], st);
    return e;
}

}  // namespace tfim
