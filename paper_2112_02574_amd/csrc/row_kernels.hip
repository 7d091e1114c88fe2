// row_kernels.hip -- steps of a lattice that is uniform along y and z: the
// flat interface along x (any tau, any storage rounded to nearest).
//
// From a state uniform along y and z every node of an x-plane makes the same
// step, u_y, u_z, F_y and F_z vanish by symmetry, and populations that differ
// only in the transverse part of xi stay equal.  One row of nodes with seven
// distinct populations per component then carries the whole state: rest, +x,
// -x, the transverse axes (2D: 2 of them, 3D: 4), the diagonals with
// xi_x = +1 and -1 (2 or 4 each) and the transverse diagonals (3D: 4).
//
// A row of up to 512 nodes fits the lanes of one workgroup, two lanes per
// node, one per component, with the populations in registers; what moves
// along x and the concentrations (with psi, taken once per node) pass through
// LDS, with two barriers per step, and a launch makes all steps of a call.
// A step is bound by the latency of its chain (LDS twice, FP64 exp, division),
// not by any rate: splitting the row over more CUs would add their
// synchronisation to it.  Measured at 127 nodes, FP64, E4 with psi: 0.6 us
// per step; the two passes over the full 127 x 5 x 5 box in graphs took 14.5.
#include "site_ops.h"

namespace scmc {

constexpr int ROW_MAX = 512;

// index of the representative of a group, number of its members, its weight
template <int D> struct RowSet;
template <> struct RowSet<2> {
    static constexpr int REP[7] = {0, 1, 3, 2, 5, 6, 0};
    static constexpr int NUM[7] = {1, 1, 1, 2, 2, 2, 0};
};
template <> struct RowSet<3> {
    static constexpr int REP[7] = {0, 1, 2, 3, 7, 8, 15};
    static constexpr int NUM[7] = {1, 1, 1, 4, 4, 4, 4};
};
// group of direction i
template <int D> __device__ constexpr int row_group(int i) {
    using L = Lattice<D>;
    const int t = L::CY[i] * L::CY[i] + L::CZ[i] * L::CZ[i];
    return L::CX[i] > 0 ? (t ? 4 : 1) : L::CX[i] < 0 ? (t ? 5 : 2) : t == 0 ? 0 : t == 1 ? 3 : 6;
}
// sum of W e_x over the stencil vectors with e_x = ex, weights as the
// compute type R holds them
template <int D, int ORDER, class R> __device__ constexpr double row_weight(int ex) {
    using S = Stencil<D, ORDER>;
    double w = 0;
    for (int a = 0; a < S::NE; ++a)
        if (S::T.e[a][0] == ex) w += (double)((R)S::T.W[a] * (R)ex);
    return w;
}

template <int D, int ORDER, class ST, int PSI>
__global__ void __launch_bounds__(2 * ROW_MAX)
    k_row_steps(Member m, const typename ST::T *src, typename ST::T *dst,
                int nsteps) {
    using L = Lattice<D>;
    using G = RowSet<D>;
    using T = typename ST::T;
    using R = typename ST::R;
    constexpr int NG = D == 3 ? 7 : 6;
    constexpr double C1 = row_weight<D, ORDER, R>(1), C2 = row_weight<D, ORDER, R>(2);
    __shared__ T sf[4][2 * ROW_MAX];             // +x, -x, +x diagonal, -x diagonal
    __shared__ R sn[PSI ? 2 : 1][2 * ROW_MAX];   // n, psi

    const int tid = threadIdx.x, J = tid & 1;
    const bool active = (tid >> 1) < m.nx;
    const int x = min(tid >> 1, m.nx - 1);  // lanes past the row repeat its last node
    const int l1 = 2 * wrap1(x - 1, m.nx) + J, r1 = 2 * wrap1(x + 1, m.nx) + J;
    const int l2 = 2 * wrap1(x - 2, m.nx) + J, r2 = 2 * wrap1(x + 2, m.nx) + J;
    const R gx = (R)(J ? m.g[1][0] : m.g[0][1]), gs = (R)(J ? m.g[1][1] : m.g[0][0]);
    const bool self = (m.self_on >> J) & 1, any_self = m.self_on & 3;
    const R omega = (R)m.omega[J], keep = R(1) - omega, cf = R(1) - R(0.5) * omega;
    const bool same = m.omega[0] == m.omega[1];
    const R n0 = (R)m.n0[J];

    T h[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q)
        h[q] = src[m.pop_off + ((long)J * L::Q + G::REP[q]) * m.N + x];
    for (int t = 0; t < nsteps; ++t) {
        sf[0][tid] = h[1];
        sf[1][tid] = h[2];
        sf[2][tid] = h[4];
        sf[3][tid] = h[5];
        __syncthreads();
        h[1] = sf[0][l1];
        h[2] = sf[1][r1];
        h[4] = sf[2][l1];
        h[5] = sf[3][r1];
        R f[NG];
        double nx = 0;
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            f[q] = ST::decode(h[q], (R)L::W[G::REP[q]], n0);
            nx += (double)G::NUM[q] * (double)f[q];
        }
        const double jx = ((double)f[1] - (double)f[2]) +
                          (double)G::NUM[4] * ((double)f[4] - (double)f[5]);
        const R n = (R)nx;
        sn[0][tid] = n;
        R psi = n;
        if constexpr (PSI != 0)
            if (any_self) sn[1][tid] = psi = psi_of<R, PSI>(n);
        __syncthreads();
        const R *no = sn[0], *ps = sn[PSI ? 1 : 0];
        double c = C1 * (double)(no[r1 ^ 1] - no[l1 ^ 1]), s = 0;
        if (ORDER > 4) c += C2 * (double)(no[r2 ^ 1] - no[l2 ^ 1]);
        if constexpr (PSI != 0)
            if (any_self) {
                s = C1 * (double)(ps[r1] - ps[l1]);
                if (ORDER > 4) s += C2 * (double)(ps[r2] - ps[l2]);
            }
        const R cr = (R)c;
        const R F = sc_force(gx, n, cr, gs, self ? psi : R(0), PSI == 0 ? swap_pair(cr) : (R)s);
        R u;
        if (same) {
            u = ((R)(jx + swap_pair(jx)) + R(0.5) * (F + swap_pair(F))) *
                (R(1) / (n + swap_pair(n)));
        } else {  // as site_collide
            const R v = omega * ((R)jx + R(0.5) * F), w = omega * n;
            u = (v + swap_pair(v)) * (R(1) / (w + swap_pair(w)));
        }
        const R on = omega * n;
        const R a = on * (R(1) - R(1.5) * (u * u)) - R(3) * cf * (u * F);
        const R e = a + R(4.5) * u * (on * u + R(2) * (cf * F)), o = R(3) * (on * u) + R(3) * (cf * F);
        double moving = 0;
#pragma unroll
        for (int q = 1; q < NG; ++q) {
            const R w = (R)L::W[G::REP[q]];
            const R v = keep * f[q] + w * (q == 1 || q == 4 ? e + o : q == 2 || q == 5 ? e - o : a);
            h[q] = ST::encode(v, w, n0);
            moving += (double)G::NUM[q] * (double)v;
        }
        h[0] = ST::encode((R)(nx - moving), (R)L::W[0], n0);
    }
    if (!active) return;
    T *out = dst + m.pop_off;
    for (int r = 0; r < m.ny * m.nz; ++r)
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
            out[((long)J * L::Q + i) * m.N + (long)r * m.nx + x] = h[row_group<D>(i)];
}

bool row_steps_supported(const StepKey &k, const Member &m) {
    return !k.sr && !k.node && m.nx <= ROW_MAX;
}

hipError_t launch_row_steps(const StepKey &k, const Member &m, const void *src, void *dst,
                            int nsteps, hipStream_t st) {
    hipError_t err = hipErrorInvalidValue;
    auto go = [&](auto stv, auto Dc, auto Oc) {
        using ST = decltype(stv);
        using T = typename ST::T;
        constexpr int D = decltype(Dc)::value, O = decltype(Oc)::value;
        const dim3 b((2 * m.nx + 63) / 64 * 64);
        if (k.psi)
            hipLaunchKernelGGL((k_row_steps<D, O, ST, 1>), dim3(1), b, 0, st, m, (const T *)src,
                               (T *)dst, nsteps);
        else
            hipLaunchKernelGGL((k_row_steps<D, O, ST, 0>), dim3(1), b, 0, st, m, (const T *)src,
                               (T *)dst, nsteps);
        err = hipGetLastError();
    };
    auto shape = [&](auto stv) {
        using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>;
        using O4 = std::integral_constant<int, 4>;
        using O6 = std::integral_constant<int, 6>;
        using O8 = std::integral_constant<int, 8>;
        if (k.dim == 2 && k.order == 4) go(stv, I2{}, O4{});
        if (k.dim == 2 && k.order == 6) go(stv, I2{}, O6{});
        if (k.dim == 2 && k.order == 8) go(stv, I2{}, O8{});
        if (k.dim == 3 && k.order == 4) go(stv, I3{}, O4{});
        if (k.dim == 3 && k.order == 6) go(stv, I3{}, O6{});
    };
    switch (k.storage) {
        case ST_F64: shape(StoreF64{}); break;
        case ST_F32: shape(StoreF32{}); break;
        case ST_F16: shape(StoreF16{}); break;
        case ST_BF16: shape(StoreBF16{}); break;
    }
    return err;
}

}  // namespace scmc
