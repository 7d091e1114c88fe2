// moment2d_kernels.hip -- steps of the moment two-pass that stay in the moment
// field, D2Q9 at tau = 1: several steps per launch.
//
// As in three dimensions (moment_impl.h) a step needs of its predecessor only
// the moments.  The paper's planes are small (64^2 to 512^2), so a step is
// bound by its launch and by the latency of its chain, not by any rate: a
// workgroup takes a tile of w x h nodes with a halo of (1 + R) nodes per step
// (R = the stencil's reach) and makes `steps` steps on it, the valid part
// shrinking by 1 + R each time, at the price of the halo's redundant nodes.
// Moments stay in registers, two lanes per node, one per component;
// concentrations (with psi, taken once per node) and the eight moving
// populations pass through LDS with two barriers per step.  Every population
// and sum is formed as in the two passes, so a block of steps equals single
// steps bit for bit.
#include <algorithm>

#include "fused_impl.h"  // xcd_remap
#include "site_ops.h"

namespace scmc {

constexpr int M2_THREADS = 1024, M2_EXT = M2_THREADS / 2;
constexpr int M2_BOX = 840;  // nodes of a tile with halo and the stencil's margin

template <int ORDER, class ST, int PSI>
__global__ void __launch_bounds__(M2_THREADS)
    k_mom2_steps(Member m, MomShape g, int steps, const typename ST::R *__restrict__ in,
                 typename ST::R *__restrict__ out) {
    using L = Lattice<2>;
    using S = Stencil<2, ORDER>;
    using R = typename ST::R;
    constexpr bool F64 = std::is_same<R, double>::value;
    constexpr int RR = S::R;
    __shared__ R sn[M2_BOX * 2];                    // n, with a margin of RR nodes
    __shared__ R sp[PSI ? M2_BOX * 2 : 1];          // psi, at the other component's index
    __shared__ R xb[8][M2_THREADS];

    const int t0 = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (t0 % g.ntx) * g.w, y0 = (t0 / g.ntx) * g.h;
    const int wx = min(g.w, m.nx - x0), wy = min(g.h, m.ny - y0);
    const int H = (1 + RR) * steps;
    const int tid = threadIdx.x, J = tid & 1;
    const int EW = wx + 2 * H, EH = wy + 2 * H, ET = EW * EH;
    const int e = min(tid >> 1, ET - 1);  // lanes past the halo repeat its last node
    const int ey = e / EW, ex = e - ey * EW;
    const bool inner = (tid >> 1) < ET && ex >= H && ex < H + wx && ey >= H && ey < H + wy;
    const bool edge = ex < 1 || ex > EW - 2 || ey < 1 || ey > EH - 2;
    // where arrivals are looked up (an edge node's go unused)
    const int from = edge ? 2 * (EW + 1) + J : 2 * e + J;
    auto mod = [](int v, int n) { return ((v % n) + n) % n; };
    const int s = mod(y0 - H + ey, m.ny) * m.nx + mod(x0 - H + ex, m.nx);
    const R *ib = in + m.dens_off;
    R *ob = out + m.dens_off;

    const R gx = (R)(J ? m.g[1][0] : m.g[0][1]), gs = (R)(J ? m.g[1][1] : m.g[0][0]);
    const bool self = (m.self_on >> J) & 1, any_self = m.self_on & 3;
    const R n0 = (R)m.n0[J];
    const int PW = EW + 2 * RR;
    // the other component's value at the low corner of the node's stencil box
    const int at0 = 2 * (ey * PW + ex) + (1 - J), mid = 2 * (RR * PW + RR);

    R n = ib[2L * s + J], jx = ib[2L * m.N + s], jy = ib[3L * m.N + s];
    unsigned rw = 0;  // the packed remainder of the own component
    if constexpr (!F64)
        rw = reinterpret_cast<const unsigned *>(ib + 5L * m.N)[s] >> (16 * J) & 0xFFFFu;
    for (int t = 0; t < steps; ++t) {
        sn[at0 + mid + 2 * J - 1] = n;
        R psi = n;
        if constexpr (PSI != 0)
            if (any_self) sp[at0 + mid] = psi = psi_of<R, PSI>(n);
        __syncthreads();
        auto at = [&](int dx, int dy) { return sn[at0 + 2 * ((dy + RR) * PW + dx + RR)]; };
        auto pat = [&](int dx, int dy) { return sp[at0 + 2 * ((dy + RR) * PW + dx + RR)]; };
        double c[2] = {0, 0}, ss[2] = {0, 0};
        const R no = at(0, 0);
#pragma unroll
        for (int a = S::NE / 2; a < S::NE; ++a) {
            constexpr auto T = S::T;
            const int vx = T.e[a][0], vy = T.e[a][1];
            const int e2[2] = {vx, vy};
            const R W = (R)T.W[a];
            const R d = at(vx, vy) - at(-vx, -vy);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (e2[q]) c[q] += (double)(W * (R)e2[q]) * (double)d;
            if constexpr (PSI != 0)
                if (any_self) {
                    const R p = pat(vx, vy) - pat(-vx, -vy);
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        if (e2[q]) ss[q] += (double)(W * (R)e2[q]) * (double)p;
                }
        }
        R F[3], p[3];
        const R inv = R(1) / (n + no), j[2] = {jx, jy};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const R cf = (R)c[q];
            F[q] = sc_force(gx, n, cf, gs, self ? psi : R(0), PSI == 0 ? swap_pair(cf) : (R)ss[q]);
            p[q] = fma_r(R(0.5), F[q] + swap_pair(F[q]), j[q]);
        }
        F[2] = p[2] = R(0);
        R rem = 0;
        if constexpr (!F64) rem = unpack_rem1(rw, n);
        R f[L::Q];
        collide_tau1_component<2, R>(n, rem, F, p, inv, [&](int i, R v) {
            const R w = ST::stored(v, (R)L::W[i], n0);
            if (i == 0) f[0] = w;
            else xb[i - 1][tid] = w;
            return v;
        });
        __syncthreads();
#pragma unroll
        for (int i = 1; i < L::Q; ++i) f[i] = xb[i - 1][from - 2 * (L::CX[i] + L::CY[i] * EW)];
        double nd, dx, dy, dz;
        raw_moments<2, R>(f, nd, dx, dy, dz);
        n = (R)nd;
        jx = (R)(dx + swap_pair(dx));
        jy = (R)(dy + swap_pair(dy));
        if constexpr (!F64) rw = pack_rem1(n, (R)(nd - (double)n));
    }
    if (!inner) return;
    ob[2L * s + J] = n;
    ob[(2L + J) * m.N + s] = J ? jy : jx;
    if constexpr (!F64) {
        const unsigned w = rw << 16 | (unsigned)swap_bits((int)rw);  // n_A's half low
        if (J) reinterpret_cast<unsigned *>(ob + 5L * m.N)[s] = w;
    }
}

// Tile and steps per launch.  Measured in graphs, a launch takes 2.9 us and
// each of its steps 0.15 us plus a time per wavefront that a SIMD holds, 0.27 us
// at E4, 0.37 us at E6 and 0.45 us at E8 in FP32 and about 1.3 times that in
// FP64.  All tiles that a workgroup holds are weighed for one to eight steps.
// us per step, w x h, steps per launch: 64^2 E4 FP32 4x4, 3 1.81; 4x4, 4 2.19;
// 10x10, 3 2.42; 6x4, 1 3.03; 128 x 160 E6 FP32 10x8, 2 2.99; 5x16, 1 3.62;
// 256^2 E8 FP64 16x16, 1 5.58; 13x7, 2 7.52.  The two passes of every step took
// 5.7 us at 64^2 and 11.3 us at 256^2.
static MomShape mom2_shape(const Member &m, int order, bool f64, int ncu, int *steps) {
    const int r = order == 4 ? 1 : 2;
    const double per = (order == 4 ? 0.27 : order == 6 ? 0.37 : 0.45) * (f64 ? 1.3 : 1.0);
    MomShape best{};
    double best_cost = 1e300;
    for (int t = 1; t <= 8; ++t) {
        const int H = (1 + r) * t;
        for (int w = std::min(m.nx, M2_EXT); w >= 1; --w) {
            const int ntx = (m.nx + w - 1) / w;
            if ((m.nx + ntx - 1) / ntx != w) continue;  // the balanced width of ntx tiles
            for (int h = std::min(m.ny, M2_EXT / (w + 2 * H) - 2 * H); h >= 1; --h) {
                const int nty = (m.ny + h - 1) / h;
                if ((m.ny + nty - 1) / nty != h) continue;
                if ((w + 2 * H + 2 * r) * (h + 2 * H + 2 * r) > M2_BOX) continue;
                const long waves = (2 * (w + 2 * H) * (h + 2 * H) + 63) / 64;
                const long on_cu = ((long)ntx * nty + ncu - 1) / ncu * waves;
                const double cost = 2.9 / t + 0.15 + per * (double)((on_cu + 3) / 4);
                if (cost < best_cost) {
                    best_cost = cost;
                    best = MomShape{w, h, 1, ntx, nty, 1};
                    *steps = t;
                }
            }
        }
    }
    return best;
}

bool node_mom2_steps(const StepKey &k, const Member &m, NodeLaunch *node, MomShape *shape,
                     int *steps) {
    if (k.dim != 2 || k.sr || k.node) return false;
    void *f = nullptr;
    auto go = [&](auto stv) {
        using ST = decltype(stv);
        auto order = [&](auto Oc) {
            constexpr int O = decltype(Oc)::value;
            f = k.psi ? (void *)&k_mom2_steps<O, ST, 1> : (void *)&k_mom2_steps<O, ST, 0>;
        };
        if (k.order == 4) order(std::integral_constant<int, 4>{});
        if (k.order == 6) order(std::integral_constant<int, 6>{});
        if (k.order == 8) order(std::integral_constant<int, 8>{});
    };
    switch (k.storage) {
        case ST_F64: go(StoreF64{}); break;
        case ST_F32: go(StoreF32{}); break;
        case ST_F16: go(StoreF16{}); break;
        case ST_BF16: go(StoreBF16{}); break;
    }
    if (!f) return false;
    *shape = mom2_shape(m, k.order, k.storage == ST_F64, compute_units(), steps);
    if (shape->w < 1) return false;
    const int H2 = 2 * (k.order == 4 ? 2 : 3) * *steps;
    node->func = f;
    node->grid = dim3(shape->ntx * shape->nty);
    node->block = dim3((2 * (shape->w + H2) * (shape->h + H2) + 63) / 64 * 64, 1, 1);
    node->shmem = 0;
    return true;
}

}  // namespace scmc
