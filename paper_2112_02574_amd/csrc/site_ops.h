// site_ops.h -- per-site operators of the two-component Shan-Chen step, shared
// by every kernel design (paper Sec. 2):
//   pull:     f_i^J(x, t) = f*_i^J(x - xi_i, t - 1)        (eq. lbm, streaming)
//   density:  n_J = sum_i f_i^J
//   force:    F_J = -g_JK n_J sum_a W_a n_K(x + e_a) e_a
//                   -g_JJ psi_J sum_a W_a psi_J(x + e_a) e_a   (eq. sc_force)
//   velocity: (n_A + n_B) u = sum_J [sum_i f_i^J xi_i + F_J / 2]
//   collide:  f* = f - omega_J (f - f^eq(n_J, u)) + (1 - omega_J/2) S_i(u, F_J)
//             f^eq = n w_i [1 + 3 xi.u + 9/2 (xi.u)^2 - 3/2 u.u]
//             S_i  = w_i [3 xi.F + 9 (xi.u)(xi.F) - 3 u.F]     (c_s^2 = 1/3)
#pragma once

#include <type_traits>

#include "lattice.h"
#include "scmc_internal.h"

namespace scmc {

__device__ __forceinline__ int wrap1(int v, int n) {
    // periodic wrap of v in [-n, 2n)
    return v < 0 ? v + n : (v >= n ? v - n : v);
}

// 32-bit integer hash (xor-shift-multiply finaliser, constants from
// C. Wellons' "lowbias32") used to seed the stochastic-rounding stream.
__host__ __device__ __forceinline__ unsigned hash32(unsigned x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// Random stream of one site and step: a hashed key, then a linear
// congruential step per stored value (its top 16 bits are used).
struct SiteRng {
    unsigned s;
    __device__ __forceinline__ SiteRng(unsigned seed, unsigned step, unsigned site)
        : s(hash32(seed ^ hash32(step * 0x9E3779B9u ^ hash32(site)))) {}
    __device__ __forceinline__ unsigned next() {
        s = s * 1664525u + 1013904223u;
        return s >> 16;
    }
};

// Value of the other component's lane, where two neighbouring lanes share a
// node, one per component.
__device__ __forceinline__ int swap_bits(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);  // quad_perm [1, 0, 3, 2]
}
__device__ __forceinline__ float swap_pair(float v) {
    return __builtin_bit_cast(float, swap_bits(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double swap_pair(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)swap_bits((int)(unsigned)b);
    const int hi = swap_bits((int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | lo);
}

template <class R, int PSI> __device__ __forceinline__ R psi_of(R n) {
    if constexpr (PSI == 0) {
        return n;
    } else {
        return exp(R(-1) / n);
    }
}

// Pull the 2Q populations of site (x, y, z) from the post-collision buffer.
// NT: populations with xi_x = 0 (whole cache lines per wavefront) are loaded
// non-temporally; the shifted ones keep their lines in L2 for the wavefront
// that shares them.
template <int D, class ST, bool NT = false>
__device__ __forceinline__ void pull_site(
    const Member &m, const typename ST::T *__restrict__ src, int x, int y,
    int z, typename ST::R (&f)[2][Lattice<D>::Q]) {
    using L = Lattice<D>;
    using R = typename ST::R;
    const typename ST::T *base = src + m.pop_off;
    const R n0A = (R)m.n0[0], n0B = (R)m.n0[1];
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const int xs = wrap1(x - L::CX[i], m.nx);
        const int ys = wrap1(y - L::CY[i], m.ny);
        const int zs = D == 3 ? wrap1(z - L::CZ[i], m.nz) : 0;
        const long s = ((long)zs * m.ny + ys) * m.nx + xs;
        const R w = (R)L::W[i];
        if (NT && L::CX[i] == 0) {
            f[0][i] = ST::decode(__builtin_nontemporal_load(base + (long)i * m.N + s), w, n0A);
            f[1][i] = ST::decode(__builtin_nontemporal_load(base + (long)(L::Q + i) * m.N + s), w,
                                 n0B);
        } else {
            f[0][i] = ST::decode(base[(long)i * m.N + s], w, n0A);
            f[1][i] = ST::decode(base[(long)(L::Q + i) * m.N + s], w, n0B);
        }
    }
}

// Order-free sums.  Every sum over populations or stencil neighbours is
// accumulated in FP64: a handful of FP32 values, or products of two FP32
// values, add up exactly there, so the result does not depend on the order of
// the terms.  A mirror reflection of the lattice only permutes those terms
// (and flips signs, which round symmetrically), so with FP32 storage the step
// commutes bit for bit with the reflections: a droplet centred on a node
// keeps its centre, which the convergence gate of Sec. 4 checks to 1e-3,
// instead of being pushed by the same rounding bias every step.
//
// Raw moments of one component's populations, FP64: n = sum_i f_i and
// j = sum_i xi_i f_i.  In 3D the populations that arrive from one neighbouring
// column are added first, those from plane z - 1, z and z + 1 in this order
// (S; their difference D enters j_z), then the columns: the sums of a march
// through the z-planes that receives one S and D per column (moment_impl.h).
struct ColumnSums {
    double S[4], D[4];      // from x - 1, x + 1, y - 1, y + 1
    double own, ownD;       // the node's own column
    double nd, xd, yd;      // the four diagonal columns: their n, j_x, j_y
    __device__ __forceinline__ void diag(double q7, double q8, double q9, double q10) {
        const double s = q7 - q8, t = q9 - q10;
        nd = (q7 + q8) + (q9 + q10);
        xd = s + t;
        yd = s - t;
    }
    __device__ __forceinline__ void total(double &n, double &jx, double &jy, double &jz) const {
        n = (own + ((S[0] + S[1]) + (S[2] + S[3]))) + nd;
        jx = (S[0] - S[1]) + xd;
        jy = (S[2] - S[3]) + yd;
        jz = ownD + ((D[0] + D[1]) + (D[2] + D[3]));
    }
};
// directions of column sum a: from below (xi_z = 1), in the plane, from above
__device__ constexpr int COL_UP[4] = {11, 14, 15, 18};
__device__ constexpr int COL_MID[4] = {1, 2, 3, 4};
__device__ constexpr int COL_DOWN[4] = {13, 12, 17, 16};

template <int D, class R>
__device__ __forceinline__ void raw_moments(const R (&f)[Lattice<D>::Q], double &n, double &jx,
                                            double &jy, double &jz) {
    using L = Lattice<D>;
    if constexpr (D == 3) {
        ColumnSums c;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const double up = f[COL_UP[a]], down = f[COL_DOWN[a]];
            c.S[a] = (up + (double)f[COL_MID[a]]) + down;
            c.D[a] = up - down;
        }
        c.own = ((double)f[5] + (double)f[0]) + (double)f[6];
        c.ownD = (double)f[5] - (double)f[6];
        c.diag(f[7], f[8], f[9], f[10]);
        c.total(n, jx, jy, jz);
    } else {
        n = jx = jy = jz = 0;
#pragma unroll
        for (int i = 0; i < L::Q; ++i) {
            n += (double)f[i];
            if (L::CX[i]) jx += (double)L::CX[i] * (double)f[i];
            if (L::CY[i]) jy += (double)L::CY[i] * (double)f[i];
        }
    }
}

template <int D, class R>
__device__ __forceinline__ void site_density(const R (&f)[2][Lattice<D>::Q],
                                             R &nA, R &nB) {
    double a = 0, b = 0;  // in the order of the velocities, as the oracle sums
#pragma unroll
    for (int i = 0; i < Lattice<D>::Q; ++i) {
        a += (double)f[0][i];
        b += (double)f[1][i];
    }
    nA = (R)a;
    nB = (R)b;
}

// One component of the force: -g n_J c_K - g_JJ psi_J s_J (c, s: stencil sums)
template <class R> __device__ __forceinline__ R sc_force(R g, R n, R c, R gs, R psi, R s) {
#pragma clang fp contract(off)
    const R self = gs * psi * s, gn = -g * n;
    if constexpr (std::is_same<R, float>::value) return __builtin_fmaf(gn, c, -self);
    else return __builtin_fma(gn, c, -self);
}

// Stencil sums of eq. sc_force around site (x, y, z), with the stencil
// concentrations returned by fetch(t, n_A, n_B) (t = linear site index times
// UNIT, e.g. a byte offset into an array of (n_A, n_B) pairs), then the force
// on both components.  The stencil is point-symmetric, so the sum runs over
// pairs (e, -e): W e (Phi(x + e) - Phi(x - e)).  The difference is exactly
// odd under e -> -e and the pair sums are accumulated in FP64 (the order-free
// sums above).  FIELD: fetch(t, n_A, n_B, psi[2]) returns psi as well, from a
// field that holds it.
template <int D, int ORDER, int PSI, class R, int UNIT = 1, bool FIELD = false, class Fetch>
__device__ __forceinline__ void site_force_fn(const Member &m, int x, int y, int z,
                                              R nA, R nB, R (&FA)[3], R (&FB)[3],
                                              Fetch &&fetch) {
    using S = Stencil<D, ORDER>;
    static_assert(S::point_symmetric(), "stencil table must list e and -e mirrored");
    double cA[3] = {0, 0, 0}, cB[3] = {0, 0, 0};
    double sA[3] = {0, 0, 0}, sB[3] = {0, 0, 0};
    const bool selfA = m.self_on & 1, selfB = m.self_on & 2;
    // periodic column, row and plane offsets of x + d, y + d, z + d for
    // d = -2..2, formed once: a stencil neighbour is then two additions
    int xo[5], yo[5], zo[5];
#pragma unroll
    for (int d = -2; d <= 2; ++d) {
        xo[d + 2] = wrap1(x + d, m.nx) * UNIT;
        yo[d + 2] = wrap1(y + d, m.ny) * (m.nx * UNIT);
        zo[d + 2] = D == 3 ? wrap1(z + d, m.nz) * (m.nx * m.ny * UNIT) : 0;
    }
#pragma unroll
    for (int a = S::NE / 2; a < S::NE; ++a) {
        constexpr auto T = S::T;
        const int ex = T.e[a][0], ey = T.e[a][1], ez = T.e[a][2];
        const int tp = zo[2 + ez] + yo[2 + ey] + xo[2 + ex];
        const int tm = zo[2 - ez] + yo[2 - ey] + xo[2 - ex];
        R pAt, pBt, mAt, mBt;  // N * UNIT < 2^31 (the callers' forms)
        R pq[2] = {0, 0}, mq[2] = {0, 0};  // psi of both components
        if constexpr (FIELD) {
            fetch(tp, pAt, pBt, pq);
            fetch(tm, mAt, mBt, mq);
        } else {
            fetch(tp, pAt, pBt);
            fetch(tm, mAt, mBt);
        }
        const R dA = pAt - mAt, dB = pBt - mBt;
        const R W = (R)T.W[a];
        const int e3[3] = {ex, ey, ez};
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (e3[k] == 0) continue;
            const double We = (double)(W * (R)e3[k]);
            cA[k] += We * (double)dB;
            cB[k] += We * (double)dA;
        }
        // with psi = n the self sums equal the cross sums (sA = cB, sB = cA)
        if (PSI != 0 && (selfA || selfB)) {
            const R qA = FIELD ? pq[0] - mq[0] : psi_of<R, PSI>(pAt) - psi_of<R, PSI>(mAt);
            const R qB = FIELD ? pq[1] - mq[1] : psi_of<R, PSI>(pBt) - psi_of<R, PSI>(mBt);
#pragma unroll
            for (int k = 0; k < D; ++k) {
                if (e3[k] == 0) continue;
                const double We = (double)(W * (R)e3[k]);
                sA[k] += We * (double)qA;
                sB[k] += We * (double)qB;
            }
        }
    }
    const R gAB = (R)m.g[0][1], gBA = (R)m.g[1][0];
    const R gAA = (R)m.g[0][0], gBB = (R)m.g[1][1];
    const R pA = selfA ? psi_of<R, PSI>(nA) : R(0);
    const R pB = selfB ? psi_of<R, PSI>(nB) : R(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const R tA = (R)(PSI == 0 ? cB[k] : sA[k]), tB = (R)(PSI == 0 ? cA[k] : sB[k]);
        FA[k] = sc_force(gAB, nA, (R)cA[k], gAA, pA, tA);
        FB[k] = sc_force(gBA, nB, (R)cB[k], gBB, pB, tB);
    }
}

// The same from a density field laid out [J][z][y][x] (dA, dB).
template <int D, int ORDER, int PSI, class R>
__device__ __forceinline__ void site_force(const Member &m,
                                           const R *__restrict__ dA,
                                           const R *__restrict__ dB, int x,
                                           int y, int z, R nA, R nB, R (&FA)[3],
                                           R (&FB)[3]) {
    site_force_fn<D, ORDER, PSI, R>(m, x, y, z, nA, nB, FA, FB,
                                    [&](int t, R &a, R &b) {
                                        a = dA[t];
                                        b = dB[t];
                                    });
}

// The collisions spell their roundings out (fused multiply-adds where they are
// meant, no contraction elsewhere), so that every kernel that collides a node,
// and each of its components, forms the same bits.
__device__ __forceinline__ float fma_r(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) {
    return __builtin_fma(a, b, c);
}

// BGK collision with Guo forcing of one component: p is the numerator of the
// common velocity and inv its denominator's inverse, nx the exact n_J; every
// f*_i goes to emit(i, value).
//
// Velocities xi and -xi are collided together: with t = omega n_J xi.u,
//   E = w [a_J + 9/2 (xi.u) (t + 2 c_f xi.F_J)],  O = w [3 t + 3 c_f xi.F_J],
//   a_J = omega n_J (1 - 3/2 u.u) - 3 c_f u.F_J,  c_f = 1 - omega / 2,
// f*_xi = (1 - omega) f_xi + (E + O) and f*_-xi = (1 - omega) f_-xi + (E - O)
// (eq. lbm with the Guo source).  Every velocity pair then runs the same
// operations on sign-flipped operands, which keeps the step exactly
// covariant under mirror reflections (see site_density).
template <int D, class R, class Emit>
__device__ __forceinline__ void collide_component(const R (&f)[Lattice<D>::Q], double nx, R nJ,
                                                  const R (&F)[3], const R (&p)[3], R inv, R omega,
                                                  Emit &&emit) {
#pragma clang fp contract(off)
    using L = Lattice<D>;
    constexpr Opposite<D> OP = Opposite<D>::make();
    const R keep = R(1) - omega, cf = R(1) - R(0.5) * omega, on = omega * nJ;
    const R u[3] = {p[0] * inv, p[1] * inv, D == 3 ? p[2] * inv : R(0)};
    R uu = fma_r(u[0], u[0], u[1] * u[1]), uF = fma_r(u[0], F[0], u[1] * F[1]);
    if (D == 3) {
        uu = fma_r(u[2], u[2], uu);
        uF = fma_r(u[2], F[2], uF);
    }
    const R a = fma_r(on, fma_r(R(-1.5), uu, R(1)), R(-3) * cf * uF);
    double moving = 0;
#pragma unroll
    for (int i = 1; i < L::Q; ++i) {
        const int ib = OP.opp[i];
        if (ib < i) continue;
        const int c[3] = {L::CX[i], L::CY[i], L::CZ[i]};
        const int k0 = c[0] ? 0 : c[1] ? 1 : 2;  // the one or two axes of xi
        const int k1 = k0 == 0 && c[1] ? 1 : k0 < 2 && c[2] ? 2 : k0;
        R xu = c[k0] > 0 ? u[k0] : -u[k0], xF = c[k0] > 0 ? F[k0] : -F[k0];
        if (k1 != k0) {
            xu = fma_r(c[k1] > 0 ? inv : -inv, p[k1], xu);
            xF = c[k1] > 0 ? xF + F[k1] : xF - F[k1];
        }
        const R w = (R)L::W[i], cF = cf * xF, t = on * xu;
        const R X = fma_r(R(4.5) * xu, fma_r(R(2), cF, t), a);
        const R O = w * (R(3) * (t + cF));
        const R fp = fma_r(keep, f[i], fma_r(w, X, O));
        const R fm = fma_r(keep, f[ib], fma_r(w, X, -O));
        emit(i, fp);
        emit(ib, fm);
        moving += (double)fp + (double)fm;
    }
    // rest population from the mass balance sum_i f*_i = sum_i f_i (BGK
    // and the Guo source conserve mass), both sums exact in FP64: rounded
    // weights and re-rounded sums would otherwise bias the mass by the
    // same relative amount every step
    emit(0, (R)(nx - moving));
}

// Common velocity and collision of both components; every f*_i^J is handed to
// sink(J, i, value) as soon as it is formed.
template <int D, class R, class Sink>
__device__ __forceinline__ void site_collide(const Member &m,
                                             const R (&f)[2][Lattice<D>::Q],
                                             R nA, R nB, const R (&FA)[3],
                                             const R (&FB)[3], Sink &&sink) {
    using L = Lattice<D>;
    double nx[2], j[2][3];  // order-free sums (see site_density)
#pragma unroll
    for (int J = 0; J < 2; ++J) raw_moments<D, R>(f[J], nx[J], j[J][0], j[J][1], j[J][2]);
    const R oA = (R)m.omega[0], oB = (R)m.omega[1];
    R p[3], inv;
    {
#pragma clang fp contract(off)
        if (m.omega[0] == m.omega[1]) {
            // common velocity of Sec. 2
            inv = R(1) / (nA + nB);
#pragma unroll
            for (int k = 0; k < 3; ++k) p[k] = fma_r(R(0.5), FA[k] + FB[k], (R)(j[0][k] + j[1][k]));
        } else {
            // tau_A != tau_B: each component's momentum and density weighted by
            // omega_J = 1 / tau_J, the form under which the collisions change the
            // total momentum by exactly sum_J F_J
            inv = R(1) / (oA * nA + oB * nB);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                p[k] = oA * fma_r(R(0.5), FA[k], (R)j[0][k]) + oB * fma_r(R(0.5), FB[k], (R)j[1][k]);
        }
    }
#pragma unroll
    for (int J = 0; J < 2; ++J)
        collide_component<D, R>(f[J], nx[J], J == 0 ? nA : nB, J == 0 ? FA : FB, p, inv,
                                J == 0 ? oA : oB,
                                [&](int i, R v) { sink(J, i, v); });
}

// Moments that the collision needs at omega = 1: n_J and the total momentum
// j = sum_J sum_i f_i^J xi_i.  n_J is summed in FP64 (exact for the 2Q
// storage values) and kept as a pair: mom[J] = its nearest compute-precision
// value, mom[5 + J] = the remainder.  The collision's rest population uses
// the exact n_J to close the mass balance, so a steady site conserves mass
// exactly instead of re-rounding the same sum the same way every step.
constexpr int NMOM = 7;  // n_A, n_B, j_x, j_y, j_z, rem(n_A), rem(n_B)

template <int D, class R>
__device__ __forceinline__ void site_moments(const R (&f)[2][Lattice<D>::Q],
                                             R (&mom)[NMOM]) {
    double n[2], jx[2], jy[2], jz[2];  // order-free sums (see site_density)
#pragma unroll
    for (int J = 0; J < 2; ++J) raw_moments<D, R>(f[J], n[J], jx[J], jy[J], jz[J]);
    mom[0] = (R)n[0];
    mom[1] = (R)n[1];
    mom[2] = (R)(jx[0] + jx[1]);
    mom[3] = (R)(jy[0] + jy[1]);
    mom[4] = (R)(jz[0] + jz[1]);
    mom[5] = (R)(n[0] - (double)mom[0]);
    mom[6] = (R)(n[1] - (double)mom[1]);
}

// The FP64 remainders of n_A, n_B (at most half an ulp of the stored value)
// travel as two halves of one 32-bit word, in units of that ulp: 11 bits of
// the remainder keep the rest population's mass closure exact to 2^-12 ulp,
// far inside its own rounding.  FP64 compute has no remainder.
__device__ __forceinline__ unsigned pack_rem1(float n, float rem) {
    int e;
    frexpf(n, &e);
    const float q = ldexpf(rem, 24 - e);  // remainder / ulp(n_J)
    return (unsigned)__half_as_ushort(__float2half_rn(q));
}

__device__ __forceinline__ float unpack_rem1(unsigned h, float n) {
    int e;
    frexpf(n, &e);
    const float q = __half2float(__ushort_as_half((unsigned short)h));
    return ldexpf(q, e - 24);
}

template <class R>
__device__ __forceinline__ unsigned pack_rem(const R (&mm)[NMOM]) {
    if constexpr (std::is_same<R, double>::value)
        return 0u;
    else
        return pack_rem1(mm[0], mm[5]) | pack_rem1(mm[1], mm[6]) << 16;
}

template <class R>
__device__ __forceinline__ void unpack_rem(unsigned w, R (&mm)[NMOM]) {
    if constexpr (std::is_same<R, double>::value) {
        mm[5] = mm[6] = 0;
    } else {
        mm[5] = unpack_rem1(w, mm[0]);
        mm[6] = unpack_rem1(w >> 16, mm[1]);
    }
}

// The collision at omega = 1 (tau = 1), where f* = f^eq(n_J, u) + S_i / 2
// no longer depends on the individual pre-collision populations.  With
// a_J = n_J (1 - 3/2 u.u) - 3/2 u.F_J, a velocity xi and its opposite share
//   E = w [a_J + 9/2 (xi.u) (n_J xi.u + xi.F_J)]
// and differ in the sign of
//   O = w [3 n_J xi.u + 3/2 xi.F_J],   f*_xi = E + O, f*_-xi = E - O.
// Every f*_i^J goes to emit(J, i, value), which stores it and returns the
// value the next step's pull will see (the stored value as decoded).  The
// rest population closes the mass balance sum_i f*_i = n_J against those
// values with the exact n_J: rounded weights (their binary sum is not exactly
// 1) and re-rounded sums would otherwise bias the mass by the same relative
// amount every step.
// p is the momentum (n_A + n_B) u, inv = 1 / (n_A + n_B).
template <int D, class R, class Emit>
__device__ __forceinline__ void collide_tau1_component(R nJ, R remJ, const R (&F)[3],
                                                       const R (&p)[3], R inv, Emit &&emit) {
#pragma clang fp contract(off)
    using L = Lattice<D>;
    constexpr Opposite<D> OP = Opposite<D>::make();
    const R u[3] = {p[0] * inv, p[1] * inv, D == 3 ? p[2] * inv : R(0)};
    R uu = fma_r(u[0], u[0], u[1] * u[1]), uF = fma_r(u[0], F[0], u[1] * F[1]);
    if (D == 3) {
        uu = fma_r(u[2], u[2], uu);
        uF = fma_r(u[2], F[2], uF);
    }
    const R a = fma_r(nJ, fma_r(R(-1.5), uu, R(1)), R(-1.5) * uF);
    double moving = 0;
#pragma unroll
    for (int i = 1; i < L::Q; ++i) {
        const int ib = OP.opp[i];
        if (ib < i) continue;
        const int c[3] = {L::CX[i], L::CY[i], L::CZ[i]};
        const int k0 = c[0] ? 0 : c[1] ? 1 : 2;  // the one or two axes of xi
        const int k1 = k0 == 0 && c[1] ? 1 : k0 < 2 && c[2] ? 2 : k0;
        R xu = c[k0] > 0 ? u[k0] : -u[k0], xF = c[k0] > 0 ? F[k0] : -F[k0];
        if (k1 != k0) {
            xu = fma_r(c[k1] > 0 ? inv : -inv, p[k1], xu);
            xF = c[k1] > 0 ? xF + F[k1] : xF - F[k1];
        }
        const R w = (R)L::W[i];
        const R X = fma_r(R(4.5) * xu, fma_r(nJ, xu, xF), a);
        const R O = w * fma_r(R(1.5), xF, R(3) * (nJ * xu));
        const R fp = emit(i, fma_r(w, X, O)), fm = emit(ib, fma_r(w, X, -O));
        moving += (double)fp + (double)fm;
    }
    const double nJx = (double)nJ + (double)remJ;
    emit(0, (R)(nJx - moving));
}

template <int D, class R, class Emit>
__device__ __forceinline__ void collide_tau1_emit(const R (&mom)[NMOM], const R (&FA)[3],
                                                  const R (&FB)[3], Emit &&emit) {
    const R inv = R(1) / (mom[0] + mom[1]);
    R p[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k] = fma_r(R(0.5), FA[k] + FB[k], mom[2 + k]);
#pragma unroll
    for (int J = 0; J < 2; ++J)
        collide_tau1_component<D, R>(mom[J], mom[5 + J], J == 0 ? FA : FB, p, inv,
                                     [&](int i, R v) { return emit(J, i, v); });
}

// The same with every f*_i^J handed to sink(J, i, value), the
// closure taken on the values as formed.
template <int D, class R, class Sink>
__device__ __forceinline__ void collide_tau1(const R (&mom)[NMOM], const R (&FA)[3],
                                             const R (&FB)[3], Sink &&sink) {
    collide_tau1_emit<D, R>(mom, FA, FB, [&](int J, int i, R v) {
        sink(J, i, v);
        return v;
    });
}

// ---- per-node-reference offsets (FP16 / BF16 node storage): a population
// collided at node x, which streams to x + e_i, is stored as
// h = f*_i - w_i n_J(x + e_i), with n_J the FP32 densities of the step (the
// moments of its first pass), which a reference field keeps beside the
// buffer.  The node that pulls it decodes it against its own densities, so
// a pull reads one reference pair per node.  The product and the sum are
// rounded on their own (no contraction into a fused multiply-add), so that
// encoding, decoding and the mass closure agree bit for bit wherever they
// are formed.
__device__ __forceinline__ float node_ref(float w, float n) {
#pragma clang fp contract(off)
    return w * n;
}

// The collision of a node-storage site: encodes each moving population
// against the densities nb[i] = (n_A, n_B)(x + e_i) of the node it streams
// to and closes the mass balance on their decoded values, so the rest
// populations, kept in FP32 (restA, restB: they do not stream), absorb the
// rounding of the 2Q - 2 moving offsets and the node's mass is kept as with
// FP32 storage.
template <int D, class ST, class Sink>
__device__ __forceinline__ void collide_tau1_node(const typename ST::R (&mom)[NMOM],
                                                  const typename ST::R (&FA)[3],
                                                  const typename ST::R (&FB)[3],
                                                  const float2 (&nb)[Lattice<D>::Q], Sink &&sink,
                                                  float &restA, float &restB) {
    using L = Lattice<D>;
    using R = typename ST::R;
    collide_tau1_emit<D, R>(mom, FA, FB, [&](int J, int i, R v) {
        if (i == 0) {
            (J == 0 ? restA : restB) = v;
            return v;
        }
        const R ref = node_ref((R)L::W[i], J == 0 ? nb[i].x : nb[i].y);
        const typename ST::T h = ST::to_node(v, ref);
        sink(J, i, h);
        return ST::from_node(h, ref);
    });
}

// Collide and store f* at site s of the member's block of dst.
template <int D, class ST>
__device__ __forceinline__ void site_collide_store(
    const Member &m, const typename ST::R (&f)[2][Lattice<D>::Q],
    typename ST::R nA, typename ST::R nB, const typename ST::R (&FA)[3],
    const typename ST::R (&FB)[3], typename ST::T *__restrict__ dst, long s) {
    using R = typename ST::R;
    typename ST::T *base = dst + m.pop_off;
    if (m.sr) {
        SiteRng rng(m.seed, *m.step_ctr, (unsigned)(m.pop_off + s));
        site_collide<D, R>(m, f, nA, nB, FA, FB, [&](int J, int i, R v) {
            __builtin_nontemporal_store(
                ST::encode_sr(v, (R)Lattice<D>::W[i], (R)m.n0[J], rng.next()),
                base + (long)(J * Lattice<D>::Q + i) * m.N + s);
        });
        return;
    }
    site_collide<D, R>(m, f, nA, nB, FA, FB, [&](int J, int i, R v) {
        __builtin_nontemporal_store(ST::encode(v, (R)Lattice<D>::W[i], (R)m.n0[J]),
                                    base + (long)(J * Lattice<D>::Q + i) * m.N + s);
    });
}

// The first pass of a two-pass step advances the step counter that seeds the
// second pass's stochastic rounding (one thread of the launch).
__device__ __forceinline__ void advance_step_counter(const Member &m, bool first) {
    if (m.sr && first && threadIdx.x == 0 && threadIdx.y == 0) m.step_ctr[0] += 1u;
}

// ---- raw-buffer access with 32-bit offsets (used by the fused kernels) ----
// One buffer descriptor per component covers its Q planes; lanes pass 32-bit
// byte offsets, the plane offset goes in the scalar offset.  The hardware
// returns 0 for reads and drops writes outside the descriptor's range.
constexpr int BUF_DATA_FORMAT_32 = 0x00020000;
constexpr int BUF_NT = 2;  // cache policy: non-temporal

template <class T> struct RawBuf;
template <> struct RawBuf<float> {
    __device__ __forceinline__ static float load(__amdgpu_buffer_rsrc_t r, int v,
                                                 int s) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
    }
    __device__ __forceinline__ static float load_nt(__amdgpu_buffer_rsrc_t r, int v, int s) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, BUF_NT));
    }
    __device__ __forceinline__ static void store_nt(float x, __amdgpu_buffer_rsrc_t r,
                                                    int v, int s) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, v,
                                              s, BUF_NT);
    }
};
template <> struct RawBuf<uint16_t> {
    __device__ __forceinline__ static uint16_t load(__amdgpu_buffer_rsrc_t r, int v,
                                                    int s) {
        return __builtin_amdgcn_raw_buffer_load_b16(r, v, s, 0);
    }
    __device__ __forceinline__ static uint16_t load_nt(__amdgpu_buffer_rsrc_t r, int v, int s) {
        return __builtin_amdgcn_raw_buffer_load_b16(r, v, s, BUF_NT);
    }
    __device__ __forceinline__ static void store_nt(uint16_t x,
                                                    __amdgpu_buffer_rsrc_t r, int v,
                                                    int s) {
        __builtin_amdgcn_raw_buffer_store_b16(x, r, v, s, BUF_NT);
    }
};

template <class ST> struct PopBuf {
    __amdgpu_buffer_rsrc_t r[2];
    int plane_bytes;  // N * sizeof(T)
};

template <class ST, int Q>
__device__ __forceinline__ PopBuf<ST> make_popbuf(const typename ST::T *pop,
                                                  const Member &m) {
    using T = typename ST::T;
    PopBuf<ST> b;
    const T *base = pop + m.pop_off;
    const unsigned bytes = (unsigned)Q * (unsigned)m.N * (unsigned)sizeof(T);
    b.r[0] = __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, (int)bytes,
                                               BUF_DATA_FORMAT_32);
    b.r[1] = __builtin_amdgcn_make_buffer_rsrc((void *)(base + (long)Q * m.N), (short)0,
                                               (int)bytes, BUF_DATA_FORMAT_32);
    b.plane_bytes = m.N * (int)sizeof(T);
    return b;
}

// Cache policy of a pull through buffer descriptors.  PULL_NT_ALIGNED: the
// populations with xi_x = 0 are loaded non-temporally, as pull_site's NT.
// PULL_NT_ALL: every population is, so that the populations streaming
// through pass 1 of the moment two-pass push less of the moment field it
// writes out of the Infinity Cache before pass 2 reads it (lattices whose
// moment field comes close to that cache's size).
enum PullPolicy : int { PULL_CACHED = 0, PULL_NT_ALIGNED = 1, PULL_NT_ALL = 2 };

// Pull of site (x, y, z) through buffer descriptors (D3Q19); NT is a
// PullPolicy.  NODE: the buffer holds per-node-reference offsets, decoded
// against the reference densities m.ref of the source nodes.
template <class ST, int NT = PULL_CACHED, bool NODE = false>
__device__ __forceinline__ void pull_site_buf(const Member &m, const PopBuf<ST> &b,
                                              int x, int y, int z,
                                              typename ST::R (&f)[2][19]) {
    using L = Lattice<3>;
    using T = typename ST::T;
    using R = typename ST::R;
    const int nxy = m.nx * m.ny;
    int xo[3], yo[3], zo[3];  // index d + 1 holds coordinate + d, wrapped
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
        xo[d + 1] = wrap1(x + d, m.nx);
        yo[d + 1] = wrap1(y + d, m.ny) * m.nx;
        zo[d + 1] = wrap1(z + d, m.nz) * nxy;
    }
    const R n0A = (R)m.n0[0], n0B = (R)m.n0[1];
    float2 own = {0.f, 0.f};  // node storage: this node's reference densities
    if constexpr (NODE) own = m.ref[zo[1] + yo[1] + xo[1]];
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const int s = zo[1 - L::CZ[i]] + yo[1 - L::CY[i]] + xo[1 - L::CX[i]];
        const int voff = s * (int)sizeof(T), soff = i * b.plane_bytes;
        const R w = (R)L::W[i];
        R refA = 0, refB = 0;
        if constexpr (NODE) {
            if (i == 0) {  // the rest populations, FP32 at the node itself
                const float2 r = m.rest[s];
                f[0][0] = r.x;
                f[1][0] = r.y;
                continue;
            }
            refA = node_ref(w, own.x);
            refB = node_ref(w, own.y);
        }
        const bool nt = NT == PULL_NT_ALL || (NT == PULL_NT_ALIGNED && L::CX[i] == 0);
        const T ra = nt ? RawBuf<T>::load_nt(b.r[0], voff, soff)
                        : RawBuf<T>::load(b.r[0], voff, soff);
        const T rb = nt ? RawBuf<T>::load_nt(b.r[1], voff, soff)
                        : RawBuf<T>::load(b.r[1], voff, soff);
        if constexpr (NODE) {
            f[0][i] = ST::from_node(ra, refA);
            f[1][i] = ST::from_node(rb, refB);
        } else {
            f[0][i] = ST::decode(ra, w, n0A);
            f[1][i] = ST::decode(rb, w, n0B);
        }
    }
}

}  // namespace scmc
