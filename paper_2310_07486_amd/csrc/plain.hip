// Plain form of the sampler: one signed byte per spin, one sample per
// configuration, no multispin coding.  It is the reference point for the
// multispin path and the form in which a single disorder sample is run.
//
// Paper: arXiv:2310.07486, Methods, "The Trotter-Suzuki formula" (classical
// spins S = +-1 on the L x L x Ltau lattice, p(S) ~ exp(-k E(S)), the action
// with J on spatial and +1 on temporal bonds, periodic or antiperiodic along
// tau) and "Simulation details" (Metropolis sweeps, parallel tempering over
// k, real replicas); "Model and simulations" for J = +-1 with probability 1/2.
//
// Layouts (canonical, also on the device; ns = number of samples):
//   spins      int8 [R][nk][ns][Ltau][L*L]   +1 / -1
//   couplings  int8 [ns][2][L*L]             +1 / -1 (d = 0: +x bond, 1: +y bond)
//   k labels, walker maps, energies as in the multispin form, [R][ns][nk].
// Sample s draws every random number from word j = word_offset + s/64 and
// lane s%64 of the multispin counter layout, so it follows exactly the
// trajectory of lane s%64 of that word in a multispin run.
//
// Kernels reuse ShapeDev: W holds the number of samples ns, S and J point at
// the int8 arrays.
#include <algorithm>

#include "tfim_internal.h"

namespace tfim {
namespace {

__device__ __forceinline__ uint32_t plain_word(const ShapeDev& sh, int s) {
    return sh.word_offset + (uint32_t)s / 64u;
}

// J = -1 where bit s%64 of the coupling word (xy, d) of word j is set.
__global__ void k_plain_init_couplings(ShapeDev sh, uint32_t key0, uint32_t key1) {
    int8_t* J = (int8_t*)sh.J;
    const size_t total = (size_t)sh.W * 2 * sh.L2;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const uint32_t xy = (uint32_t)(i % sh.L2);
        const uint32_t d = (uint32_t)((i / sh.L2) % 2);
        const int s = (int)(i / (2 * (size_t)sh.L2));
        const U4 o = philox10(xy, d, 0u, ctr_word3(plain_word(sh, s), sh.sid, kTagCoupling), key0, key1);
        const uint64_t word = (uint64_t)o.v[0] | ((uint64_t)o.v[1] << 32);
        J[i] = ((word >> (s & 63)) & 1ull) ? (int8_t)-1 : (int8_t)1;
    }
}

// Hot start: spin (r, w, s, lin) = -1 where bit s%64 of the spin word is set.
__global__ void k_plain_init_spins(ShapeDev sh, uint32_t key0, uint32_t key1) {
    int8_t* S8 = (int8_t*)sh.S;
    const size_t N = (size_t)sh.L2 * sh.Lt;
    const size_t total = (size_t)sh.R * sh.nk * sh.W * N;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const uint32_t lin = (uint32_t)(i % N);
        const size_t cfg = i / N;  // (r*nk + w)*ns + s
        const int s = (int)(cfg % sh.W);
        const uint32_t rw = (uint32_t)(cfg / sh.W);
        const U4 o = philox10(lin, rw, 0u, ctr_word3(plain_word(sh, s), sh.sid, kTagSpin), key0, key1);
        const uint64_t word = (uint64_t)o.v[0] | ((uint64_t)o.v[1] << 32);
        S8[i] = ((word >> (s & 63)) & 1ull) ? (int8_t)-1 : (int8_t)1;
    }
}

// Metropolis half-sweep of colour c.  One thread takes the four sites of
// colour c at tau = 8q + 2hh + p (hh = 0..3, p = (c + x + y) mod 2) of one
// column: they share one Philox call, output hh.  A site's energy change is
// dE = 2 S h with h its local field (the wrap neighbour along tau with the
// sign -1 when antiperiodic); the move is taken iff dE <= 0 or
// R < Tu[k-index][u] with u = (12 - dE)/4 unsatisfied bonds.  Sites of one
// colour only neighbour the other colour, so threads never race.
__global__ void __launch_bounds__(256) k_plain_half(ShapeDev sh, uint32_t key0, uint32_t key1,
                                                    When when, uint32_t ahead, int c) {
    const uint32_t t = when.get() + ahead;
    int8_t* S8 = (int8_t*)sh.S;
    const int8_t* J = (const int8_t*)sh.J;
    const int L = sh.L, L2 = sh.L2, Lt = sh.Lt, nk = sh.nk, ns = sh.W;
    const int nq = (Lt + 7) / 8;
    const int sgn = sh.apm ? -1 : 1;
    const size_t total = (size_t)sh.R * nk * ns * L2 * nq;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const int q = (int)(i % nq);
        const size_t rest = i / nq;
        const int xy = (int)(rest % L2);
        const size_t cfg = rest / L2;  // (r*nk + w)*ns + s
        const int s = (int)(cfg % ns);
        const int rw = (int)(cfg / ns);
        const int r = rw / nk, w = rw % nk;
        const int x = xy % L, y = xy / L;
        const int xm = (x + L - 1) % L + L * y, xp = (x + 1) % L + L * y;
        const int ym = x + L * ((y + L - 1) % L), yp = x + L * ((y + 1) % L);
        const int8_t* jb = J + (size_t)s * 2 * L2;
        const int jxp = jb[xy], jxm = jb[xm], jyp = jb[L2 + xy], jym = jb[L2 + ym];
        const U4 o = philox10((uint32_t)(xy + L2 * q), t, ((uint32_t)rw << 1) | (uint32_t)c,
                              ctr_word3(plain_word(sh, s), sh.sid, kTagMetro), key0, key1);
        const int kix = sh.kidx[((size_t)r * ns + s) * nk + w];
        int8_t* cf = S8 + cfg * (size_t)L2 * Lt;
        const int p = (c + x + y) & 1;
#pragma unroll
        for (int hh = 0; hh < 4; ++hh) {
            const int tau = 8 * q + 2 * hh + p;
            if (tau >= Lt) break;
            const int8_t* P = cf + (size_t)tau * L2;
            const int tm = tau == 0 ? Lt - 1 : tau - 1, tp = tau == Lt - 1 ? 0 : tau + 1;
            const int cm = tau == 0 ? sgn : 1, cp = tau == Lt - 1 ? sgn : 1;
            const int h = jxp * P[xp] + jxm * P[xm] + jyp * P[yp] + jym * P[ym] +
                          cm * cf[(size_t)tm * L2 + xy] + cp * cf[(size_t)tp * L2 + xy];
            const int sv = P[xy];
            const int dE = 2 * sv * h;
            bool flip = dE <= 0;
            if (!flip) flip = o.v[hh] < sh.Tu[kix * 3 + (12 - dE) / 4];
            if (flip) cf[(size_t)tau * L2 + xy] = (int8_t)(-sv);
        }
    }
}

// n sweeps of a configuration that fits in LDS, one workgroup each: the spins
// stay in LDS from the first sweep to the last (tempering, which needs U and
// other configurations, ends a run), U is counted once at the end.  The same
// numbers and the same order of colours as k_plain_half.  Bound by the latency
// of a half-sweep, a Philox call between two barriers.  A unit (a column's
// eight planes) reads all its neighbours before the call and decides its four
// sites after it: sites of one colour are no neighbours.  kOne: a unit per
// thread, whose place and couplings then stay in registers.
// L = 8, Ltau = 32, two configurations: 14 us per sweep in three launches
// (two half-sweeps and a recount) -> 2.1; 2048 configurations of L = 16,
// Ltau = 216 with tempering at every sweep 2.2 ms per sweep -> 0.9.
constexpr size_t kPlainLds = 63 * 1024;  // spins and columns of a configuration
constexpr int kPlainRunThreads = 1024;

// a column's neighbours (offsets in a plane) and couplings
struct PlainCol {
    uint16_t xm, xp, ym, yp;
    int8_t jxm, jxp, jym, jyp;
    int odd;  // (x + y) & 1
};

__host__ __device__ inline size_t plain_run_lds(const ShapeDev& sh) {
    return (size_t)sh.L2 * (sh.Lt + sizeof(PlainCol));
}

template <bool kOne>
__global__ void __launch_bounds__(kPlainRunThreads)
k_plain_run(ShapeDev sh, int cfg0, uint32_t key0, uint32_t key1, When when, uint32_t n, Counters* ctr) {
    extern __shared__ __align__(16) char lds[];  // [L2] columns, [Ltau][L2] spins
    __shared__ uint32_t tot;
    const int L = sh.L, L2 = sh.L2, Lt = sh.Lt, nk = sh.nk, ns = sh.W;
    const int cfg = cfg0 + (int)blockIdx.x;  // (r*nk + w)*ns + s
    const int s = cfg % ns, rw = cfg / ns, r = rw / nk, w = rw % nk;
    const int tid = threadIdx.x, nthr = blockDim.x;
    PlainCol* const col = (PlainCol*)lds;
    int8_t* const sp = (int8_t*)(col + L2);
    int* const cf = (int*)((int8_t*)sh.S + (size_t)cfg * L2 * Lt);  // L2 is a multiple of 4
    for (int e = tid; e < L2 * Lt / 4; e += nthr) ((int*)sp)[e] = cf[e];
    const int8_t* const J = (const int8_t*)sh.J + (size_t)s * 2 * L2;
    for (int e = tid; e < L2; e += nthr) {
        const int x = e % L, y = e / L;
        const int xm = (x ? x - 1 : L - 1) + L * y, xp = (x + 1 < L ? x + 1 : 0) + L * y;
        const int ym = x + L * (y ? y - 1 : L - 1), yp = x + L * (y + 1 < L ? y + 1 : 0);
        col[e] = PlainCol{(uint16_t)xm, (uint16_t)xp, (uint16_t)ym, (uint16_t)yp,
                          J[xm],        J[e],         J[L2 + ym],   J[L2 + e], (x + y) & 1};
    }
    if (tid == 0) tot = 0;
    const uint32_t t0 = when.get();
    const uint32_t* const Tu = sh.Tu + 3 * sh.kidx[((size_t)r * ns + s) * nk + w];
    const uint32_t T0 = Tu[0], T1 = Tu[1], T2 = Tu[2];
    const uint32_t c3 = ctr_word3(plain_word(sh, s), sh.sid, kTagMetro);
    const int sgn = sh.apm ? -1 : 1, units = L2 * ((Lt + 7) / 8);
    __syncthreads();
    auto update = [&](const PlainCol& cl, int xy, int e, uint32_t t, int c) {
        const int tau0 = 8 * (e / L2) + ((c + cl.odd) & 1);
        int h[4], sv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int tau = min(tau0 + 2 * i, Lt - 1);  // past the end: read, not used
            const int8_t* const P = sp + tau * L2;
            const int dn = tau == 0 ? sgn * sp[(Lt - 1) * L2 + xy] : P[xy - L2];
            const int up = tau == Lt - 1 ? sgn * sp[xy] : P[xy + L2];
            h[i] = cl.jxp * P[cl.xp] + cl.jxm * P[cl.xm] + cl.jyp * P[cl.yp] + cl.jym * P[cl.ym] + dn + up;
            sv[i] = P[xy];
        }
        const U4 o = philox10((uint32_t)e, t, ((uint32_t)rw << 1) | (uint32_t)c, c3, key0, key1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int dE = 2 * sv[i] * h[i];
            const bool acc = dE <= 0 || o.v[i] < (dE == 12 ? T0 : (dE == 8 ? T1 : T2));
            if (tau0 + 2 * i < Lt && acc) sp[(tau0 + 2 * i) * L2 + xy] = (int8_t)-sv[i];
        }
    };
    const int xy0 = tid % L2;
    const PlainCol one = col[xy0];
    for (uint32_t k = 0; k < n; ++k)
        for (int c = 0; c < 2; ++c) {
            if constexpr (kOne) {
                if (tid < units) update(one, xy0, tid, t0 + k, c);
            } else {
                for (int e = tid; e < units; e += nthr) update(col[e % L2], e % L2, e, t0 + k, c);
            }
            __syncthreads();
        }
    uint32_t u = 0;
    for (int e = tid; e < L2 * Lt; e += nthr) {
        const int tau = e / L2, xy = e - tau * L2;
        const PlainCol cl = col[xy];
        const int8_t* const P = sp + tau * L2;
        const int sv = P[xy], up = tau == Lt - 1 ? sgn * sp[xy] : P[xy + L2];
        u += (cl.jxp * sv * P[cl.xp] < 0) + (cl.jyp * sv * P[cl.yp] < 0) + (sv * up < 0);
    }
    atomicAdd(&tot, u);
    for (int e = tid; e < L2 * Lt / 4; e += nthr) cf[e] = ((const int*)sp)[e];
    __syncthreads();
    if (tid == 0) sh.U[((size_t)r * ns + s) * nk + w] = tot;
    if (ctr && cfg == 0 && tid == 0) ctr->t = t0 + n;
}

// Unsatisfied bonds U of every configuration from the action: each site
// counts its +x, +y and +tau bonds (E = 2U - 3N).  One workgroup per
// configuration.  After half-sweeps that took t by value it leaves the sweep
// counter they reached on the device.
__global__ void __launch_bounds__(1024) k_plain_energy(ShapeDev sh, int cfg0, Counters* ctr, uint32_t t) {
    __shared__ uint32_t tot;
    const int8_t* S8 = (const int8_t*)sh.S;
    const int8_t* J = (const int8_t*)sh.J;
    const int L = sh.L, L2 = sh.L2, Lt = sh.Lt, nk = sh.nk, ns = sh.W;
    const int cfg = cfg0 + (int)blockIdx.x;  // (r*nk + w)*ns + s
    const int s = cfg % ns, rw = cfg / ns, r = rw / nk, w = rw % nk;
    const int8_t* cf = S8 + (size_t)cfg * L2 * Lt;
    const int8_t* jb = J + (size_t)s * 2 * L2;
    const int sgn = sh.apm ? -1 : 1;
    if (threadIdx.x == 0) tot = 0;
    __syncthreads();
    uint32_t u = 0;
#pragma unroll 4
    for (int lin = threadIdx.x; lin < L2 * Lt; lin += blockDim.x) {
        const int xy = lin % L2, tau = lin / L2;
        const int x = xy % L, y = xy / L;
        const int xp = (x + 1) % L + L * y, yp = x + L * ((y + 1) % L);
        const int8_t* P = cf + (size_t)tau * L2;
        const int tn = tau == Lt - 1 ? 0 : tau + 1;
        const int ct = tau == Lt - 1 ? sgn : 1;
        const int sv = P[xy];
        u += (jb[xy] * sv * P[xp] < 0) + (jb[L2 + xy] * sv * P[yp] < 0) +
             (ct * sv * cf[(size_t)tn * L2 + xy] < 0);
    }
    atomicAdd(&tot, u);
    __syncthreads();
    if (threadIdx.x == 0) sh.U[((size_t)r * ns + s) * nk + w] = tot;
    if (ctr && cfg == 0 && threadIdx.x == 0) ctr->t = t;
}

// One tempering step for every (r, s): pairs (i, i+1), i = m mod 2, m mod 2 + 2,
// ...; d = U_a - U_b of the walkers at k_i, k_{i+1}; accept iff d <= 0 or
// R < Tpt[i][d] (the exchange ratio with E = 2U - 3N); R = output s%4 of the
// Philox call ((s%64)/4 | i << 4, m, r, word j), one uniform per sample.
__global__ void k_plain_temper(ShapeDev sh, uint32_t key0, uint32_t key1, uint32_t m_value, const Counters* read,
                               Counters* ctr) {
    const uint32_t m = read ? read->m : m_value;
    const int nk = sh.nk, ns = sh.W;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (ctr && g == 0) ctr->m = m + 1;
    if (g >= sh.R * ns) return;
    const int r = g / ns, s = g % ns;
    const uint32_t b = (uint32_t)(s & 63);
    uint8_t* ki = sh.kidx + (size_t)g * nk;
    uint8_t* wi = sh.winv + (size_t)g * nk;
    const uint32_t* U = sh.U + (size_t)g * nk;
    const uint32_t c3 = ctr_word3(plain_word(sh, s), sh.sid, kTagTemper);
    for (int i = (int)(m & 1u); i + 1 < nk; i += 2) {
        const int wa = wi[i], wb = wi[i + 1];
        const int64_t d = (int64_t)U[wa] - (int64_t)U[wb];
        const U4 o = philox10((b >> 2) | ((uint32_t)i << 4), m, (uint32_t)r, c3, key0, key1);
        const uint32_t R = o.v[b & 3];
        bool acc = d <= 0;
        if (!acc && d <= (int64_t)sh.dmax[i]) acc = R < sh.Tpt[sh.tpt_off[i] + (uint32_t)(d - 1)];
        if (acc) {
            ki[wa] = (uint8_t)(i + 1);
            ki[wb] = (uint8_t)i;
            wi[i] = (uint8_t)wb;
            wi[i + 1] = (uint8_t)wa;
        }
    }
}

// Identity k labels: walker w of every (r, s) at k-index w.  The plain
// label arrays hold R * ns * nk entries (ns samples, not 64 per word).
__global__ void k_plain_labels(ShapeDev sh) {
    const size_t total = (size_t)sh.R * sh.W * sh.nk;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const uint8_t v = (uint8_t)(i % sh.nk);
        sh.kidx[i] = v;
        sh.winv[i] = v;
    }
}

__global__ void k_plain_zero(int64_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

constexpr int kPlainMaxP = 15;  // six replicas

// Pair records of configuration cfg = cfg0 + blockIdx.y (k-index i, sample s),
// blocks [0, gx) of x:
// G^r_xy = sum_tau S^r_x,tau S^r_y,tau of the walker at k-index i of every
// replica, one element (x, y) per thread, int32; D_x[d] += G^a_xy G^b_xy at
// d = (x1 - y1) mod L (D_y in x2 - y2), in int64.
__device__ __forceinline__ void plain_gram_block(const ShapeDev& sh, int cfg, int bx, int nbx,
                                                 unsigned long long* D) {
    const int8_t* S8 = (const int8_t*)sh.S;
    const int L = sh.L, L2 = sh.L2, Lt = sh.Lt, nk = sh.nk, ns = sh.W, R = sh.R, P = sh.P;
    const int i = cfg / ns, s = cfg % ns;
    for (int e = threadIdx.x; e < P * 2 * L; e += blockDim.x) D[e] = 0;
    __syncthreads();
    const int nel = L2 * L2;
    for (int el = bx * (int)blockDim.x + threadIdx.x; el < nel; el += nbx * (int)blockDim.x) {
        const int x = el / L2, y = el % L2;
        int G[6];
        for (int r = 0; r < R; ++r) {
            const int w = sh.winv[((size_t)r * ns + s) * nk + i];
            const int8_t* cf = S8 + ((size_t)(r * nk + w) * ns + s) * L2 * Lt;
            int acc = 0;
#pragma unroll 4
            for (int tau = 0; tau < Lt; ++tau) acc += cf[(size_t)tau * L2 + x] * cf[(size_t)tau * L2 + y];
            G[r] = acc;
        }
        const int dx = ((x % L) - (y % L) + L) % L, dy = ((x / L) - (y / L) + L) % L;
        int p = 0;
        for (int a = 0; a < R; ++a)
            for (int b = a + 1; b < R; ++b, ++p) {
                const unsigned long long h = (unsigned long long)((long long)G[a] * G[b]);
                atomicAdd(&D[(p * 2 + 0) * L + dx], h);
                atomicAdd(&D[(p * 2 + 1) * L + dy], h);
            }
    }
    __syncthreads();
    const int rl = 2 * L + 3;
    for (int e = threadIdx.x; e < P * 2 * L; e += blockDim.x)
        if (D[e]) atomicAdd((unsigned long long*)&sh.rec[((size_t)cfg * P + e / (2 * L)) * rl + e % (2 * L)], D[e]);
}

// Overlap part of the pair records, the other blocks of x:
// Q^ab_t1,t2 = sum_x S^a_x,t1 S^b_x,t2, four sites in a dword (L^2 is a
// multiple of 4), one element per thread; trQ, sum Q^2, sum Q^4 in int64
// (|Q| <= L^2).
__device__ __forceinline__ void plain_overlap_block(const ShapeDev& sh, int cfg, int bx, int nbx,
                                                    unsigned long long* red) {
    const int n4 = sh.L2 / 4, Lt = sh.Lt, nk = sh.nk, ns = sh.W, R = sh.R, P = sh.P;
    const int* S4 = (const int*)sh.S;
    const int i = cfg / ns, s = cfg % ns;
    for (int e = threadIdx.x; e < P * 3; e += blockDim.x) red[e] = 0;
    __syncthreads();
    const unsigned step = (unsigned)nbx * blockDim.x, first = (unsigned)bx * blockDim.x + threadIdx.x;
    const unsigned d1 = step / (unsigned)Lt, d2 = step % (unsigned)Lt;
    int p = 0;
    for (int a = 0; a < R; ++a)
        for (int b = a + 1; b < R; ++b, ++p) {
            const int wa = sh.winv[((size_t)a * ns + s) * nk + i];
            const int wb = sh.winv[((size_t)b * ns + s) * nk + i];
            const int* const ca = S4 + ((size_t)(a * nk + wa) * ns + s) * Lt * n4;
            const int* const cb = S4 + ((size_t)(b * nk + wb) * ns + s) * Lt * n4;
            long long m0 = 0, m1 = 0, m2 = 0;
            unsigned t1 = first / (unsigned)Lt, t2 = first % (unsigned)Lt;
            while (t1 < (unsigned)Lt) {
                const int* const pa = ca + (size_t)t1 * n4;
                const int* const pb = cb + (size_t)t2 * n4;
                int q = 0;
#pragma unroll 4
                for (int x = 0; x < n4; ++x) q = __builtin_amdgcn_sdot4(pa[x], pb[x], q, false);
                const long long q2 = (long long)q * q;
                m1 += q2;
                m2 += q2 * q2;
                if (t1 == t2) m0 += q;
                t1 += d1;
                t2 += d2;
                if (t2 >= (unsigned)Lt) {
                    t2 -= Lt;
                    ++t1;
                }
            }
            for (int o = 32; o; o >>= 1) {
                m0 += __shfl_xor(m0, o);
                m1 += __shfl_xor(m1, o);
                m2 += __shfl_xor(m2, o);
            }
            if ((threadIdx.x & 63) == 0) {
                atomicAdd(&red[p * 3], (unsigned long long)m0);
                atomicAdd(&red[p * 3 + 1], (unsigned long long)m1);
                atomicAdd(&red[p * 3 + 2], (unsigned long long)m2);
            }
        }
    __syncthreads();
    const int rl = 2 * sh.L + 3;
    for (int e = threadIdx.x; e < P * 3; e += blockDim.x)
        if (red[e]) atomicAdd((unsigned long long*)&sh.rec[((size_t)cfg * P + e / 3) * rl + 2 * sh.L + e % 3], red[e]);
}

// Both parts in one launch, with eight loads in flight per thread: bound by
// the latency of the loads (L = 8, Ltau = 32, one configuration: two launches
// of 16 and 15 us with a load at a time -> one of 8; 2048 configurations of
// L = 16, Ltau = 216 49 ms -> 3).
__global__ void __launch_bounds__(256) k_plain_records(ShapeDev sh, int cfg0, int gx) {
    __shared__ unsigned long long sums[kPlainMaxP * 2 * 24];
    const int cfg = cfg0 + blockIdx.y;
    if ((int)blockIdx.x < gx)
        plain_gram_block(sh, cfg, blockIdx.x, gx, sums);
    else
        plain_overlap_block(sh, cfg, blockIdx.x - gx, gridDim.x - gx, sums);
}

// A[i][h][d] = sum over samples and pairs of the records' D_x (h = 0), D_y (h = 1).
__global__ void k_plain_buckets(ShapeDev sh) {
    const int L = sh.L, ns = sh.W, P = sh.P, rl = 2 * L + 3;
    const int n = sh.nk * 2 * L;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const int i = e / (2 * L), hd = e % (2 * L);
        long long acc = 0;
        for (int s = 0; s < ns; ++s)
            for (int p = 0; p < P; ++p) acc += sh.rec[((size_t)(i * ns + s) * P + p) * rl + hd];
        sh.buckets[e] = acc;
    }
}

unsigned grid_of(size_t total, size_t cap = 65536) {
    size_t b = (total + 255) / 256;
    if (b > cap) b = cap;
    if (b == 0) b = 1;
    return (unsigned)b;
}

}  // namespace

hipError_t plain_init_couplings(const ShapeDev& sh, uint64_t seed, hipStream_t st) {
    const size_t total = (size_t)sh.W * 2 * sh.L2;
    hipLaunchKernelGGL(k_plain_init_couplings, dim3(grid_of(total)), dim3(256), 0, st, sh, (uint32_t)seed,
                       (uint32_t)(seed >> 32));
    return hipGetLastError();
}

hipError_t plain_init_spins(const ShapeDev& sh, uint64_t seed, hipStream_t st) {
    const size_t total = (size_t)sh.R * sh.nk * sh.W * sh.L2 * sh.Lt;
    hipLaunchKernelGGL(k_plain_init_spins, dim3(grid_of(total)), dim3(256), 0, st, sh, (uint32_t)seed,
                       (uint32_t)(seed >> 32));
    return hipGetLastError();
}

hipError_t plain_labels_identity(const ShapeDev& sh, hipStream_t st) {
    const size_t total = (size_t)sh.R * sh.W * sh.nk;
    hipLaunchKernelGGL(k_plain_labels, dim3(grid_of(total)), dim3(256), 0, st, sh);
    return hipGetLastError();
}

static hipError_t energy_and_counter(const ShapeDev& sh, Counters* ctr, uint32_t t, hipStream_t st) {
    // Wide workgroups where there are few, or where each has much to read; else
    // their start and their additions to one counter cost more than they hide.
    // us with 256 / 512 / 1024 threads: 64 configurations of 115200 sites 250 /
    // 156 / 132; 1024 of 32768 231 / 217 / 212, of 4096 53 / 52 / 55, of 1024
    // 32 / 34 / 39; 4096 of 57600 1191 / 1171 / 1176; 32768 of 1024 252 / 327 / 535.
    const int ncfg = sh.R * sh.nk * sh.W, sites = sh.L2 * sh.Lt;
    const int most = ncfg <= 256 || (ncfg <= 1024 && sites >= 1 << 14) ? 1024
                     : ncfg <= 4096 && sites >= 1 << 12                ? 512
                                                                       : 256;
    const int threads = std::min(most, (sites + 63) / 64 * 64);
    return over_ranges(ncfg, 1, threads, [&](int c, int n) {
        hipLaunchKernelGGL(k_plain_energy, dim3(n), dim3(threads), 0, st, sh, c, ctr, t);
        return hipGetLastError();
    });
}

// A workgroup per configuration, unless a run of several sweeps goes over
// few large ones.  20 sweeps and a read-back at L = 16, Ltau = 216 (6912
// units): two configurations 710 us against 505 over the whole chip, but 64
// of them 949 against 1694, and two with tempering at every sweep 1222
// against 1339; two of Ltau = 64 (2048 units) 279 against 427.
static bool plain_in_lds(const ShapeDev& sh, uint32_t n) {
    return plain_run_lds(sh) <= kPlainLds &&
           (sh.L2 * ((sh.Lt + 7) / 8) <= 4 * kPlainRunThreads || sh.R * sh.nk * sh.W > 8 || n == 1);
}

// About 50 ms, by what a sweep in LDS takes: 5 us per unit of a thread (2 with one),
// over the full chip 1.6e-5 us per unit (220 for 2048 configurations of 6912).  Runs of
// 20 ms lost 1% to their ends there, of 5 ms 4%.
uint32_t plain_run_limit(const ShapeDev& sh) {
    constexpr uint32_t kMost = 1u << 12;
    if (!plain_in_lds(sh, 2)) return kMost;  // launches of half a sweep each
    const int units = sh.L2 * ((sh.Lt + 7) / 8), per = (units + kPlainRunThreads - 1) / kPlainRunThreads;
    const double us = std::max(5.0 * per, 1.6e-5 * units * ((double)sh.R * sh.nk * sh.W));
    return (uint32_t)std::min<double>(kMost, std::max(1.0, 5e4 / us));
}

hipError_t plain_sweeps(const ShapeDev& sh, uint64_t seed, uint32_t t, uint32_t n, Counters* ctr, bool from_device,
                        hipStream_t st) {
    const When when{t, from_device ? ctr : nullptr};
    Counters* const store = from_device ? nullptr : ctr;
    const size_t total = (size_t)sh.R * sh.nk * sh.W * sh.L2 * ((sh.Lt + 7) / 8);
    const int units = sh.L2 * ((sh.Lt + 7) / 8), ncfg = sh.R * sh.nk * sh.W;
    if (plain_in_lds(sh, n)) {
        const int threads = std::min(kPlainRunThreads, (units + 63) / 64 * 64);
        const hipError_t e = over_ranges(ncfg, 1, threads, [&](int c, int m) {
            hipLaunchKernelGGL(units <= threads ? k_plain_run<true> : k_plain_run<false>, dim3(m), dim3(threads),
                               plain_run_lds(sh), st, sh, c, (uint32_t)seed, (uint32_t)(seed >> 32), when, n, store);
            return hipGetLastError();
        });
        return e == hipSuccess && from_device ? launch_advance(ctr, n, 0, st) : e;
    }
    for (uint32_t k = 0; k < n; ++k)
        for (int c = 0; c < 2; ++c) {
            hipLaunchKernelGGL(k_plain_half, dim3(grid_of(total)), dim3(256), 0, st, sh, (uint32_t)seed,
                               (uint32_t)(seed >> 32), when, k, c);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    const hipError_t e = energy_and_counter(sh, store, t + n, st);
    return e == hipSuccess && from_device ? launch_advance(ctr, n, 0, st) : e;
}

hipError_t plain_energy(const ShapeDev& sh, hipStream_t st) { return energy_and_counter(sh, nullptr, 0, st); }

hipError_t plain_temper(const ShapeDev& sh, uint64_t seed, uint32_t m, Counters* ctr, bool from_device,
                        hipStream_t st) {
    const int n = sh.R * sh.W;
    hipLaunchKernelGGL(k_plain_temper, dim3((n + 63) / 64), dim3(64), 0, st, sh, (uint32_t)seed,
                       (uint32_t)(seed >> 32), m, from_device ? ctr : nullptr, from_device ? nullptr : ctr);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && from_device ? launch_advance(ctr, 0, 1, st) : e;
}

bool plain_measure_ok(const ShapeDev& sh) { return sh.R >= 2 && sh.R <= 6 && sh.L <= 24; }

hipError_t plain_measure(const ShapeDev& sh, int cfg0, int ncfg, hipStream_t st) {
    if (ncfg <= 0) return hipSuccess;
    const size_t rl = (size_t)(2 * sh.L + 3) * sh.P;
    hipLaunchKernelGGL(k_plain_zero, dim3(grid_of((size_t)ncfg * rl, 4096)), dim3(256), 0, st,
                       sh.rec + (size_t)cfg0 * rl, (size_t)ncfg * rl);
    hipError_t e = hipGetLastError();
    // at most 65535 configurations per launch along y
    for (int c = 0; c < ncfg && e == hipSuccess; c += 65535) {
        const int n = ncfg - c < 65535 ? ncfg - c : 65535;
        const unsigned gx = grid_of((size_t)sh.L2 * sh.L2, 64);
        const unsigned gq = grid_of((size_t)sh.Lt * sh.Lt, 256);
        hipLaunchKernelGGL(k_plain_records, dim3(gx + gq, n), dim3(256), 0, st, sh, cfg0 + c, (int)gx);
        e = hipGetLastError();
    }
    return e;
}

hipError_t plain_buckets(const ShapeDev& sh, hipStream_t st) {
    hipLaunchKernelGGL(k_plain_buckets, dim3(16), dim3(256), 0, st, sh);
    return hipGetLastError();
}

}  // namespace tfim
