// once_kernels.hip -- a single step of a small lattice in one launch (D3Q19,
// tau = 1).
//
// Pass 1 and pass 2 of a small lattice take little more than their two
// launches.  Here a workgroup owns a box of nodes: it pulls the box and the
// stencil's halo, two lanes per node, one per component, sums their moments,
// passes the concentrations (with psi, taken once per node) through LDS and
// collides the box.  Every lane pulls one node, so the step's chain is one
// round of loads, one barrier, one collision; the halo's pulls are repeated
// by the boxes around (3 to 8 times the nodes), which small lattices serve
// from the caches.  Bit for bit the two passes' result.
#include <algorithm>

#include "fused_impl.h"  // xcd_remap
#include "site_ops.h"

namespace scmc {

constexpr int ONCE_THREADS = 1024;

template <int ORDER, class ST, int PSI>
__global__ void __launch_bounds__(ONCE_THREADS)
    k_step_once(Member m, MomShape g, const typename ST::T *__restrict__ src,
                typename ST::T *__restrict__ dst) {
    using L = Lattice<3>;
    using S = Stencil<3, ORDER>;
    using R = typename ST::R;
    constexpr int RR = S::R;
    __shared__ R sn[ONCE_THREADS];
    __shared__ R sp[PSI ? ONCE_THREADS : 1];  // psi, at the other component's index

    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (b % g.ntx) * g.w, y0 = (b / g.ntx) % g.nty * g.h, z0 = b / (g.ntx * g.nty) * g.zc;
    const int wx = min(g.w, m.nx - x0), wy = min(g.h, m.ny - y0), wz = min(g.zc, m.nz - z0);
    const int EX = wx + 2 * RR, EY = wy + 2 * RR, ET = EX * EY * (wz + 2 * RR);
    const int tid = threadIdx.x, J = tid & 1;
    const int e = min(tid >> 1, ET - 1);  // lanes past the halo repeat its last node
    const int ez = e / (EX * EY), q0 = e - ez * (EX * EY), ey = q0 / EX, ex = q0 - ey * EX;
    const bool inner = (tid >> 1) < ET && ex >= RR && ex < RR + wx && ey >= RR && ey < RR + wy &&
                       ez >= RR && ez < RR + wz;
    const int x = wrap1(x0 - RR + ex, m.nx), y = wrap1(y0 - RR + ey, m.ny);
    const int z = wrap1(z0 - RR + ez, m.nz);
    const R n0 = (R)m.n0[J];

    int xo[3], yo[3], zo[3];  // index d + 1 holds coordinate + d, wrapped
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
        xo[d + 1] = wrap1(x + d, m.nx);
        yo[d + 1] = wrap1(y + d, m.ny) * m.nx;
        zo[d + 1] = wrap1(z + d, m.nz) * (m.nx * m.ny);
    }
    const typename ST::T *pop = src + m.pop_off + (long)J * L::Q * m.N;
    R f[L::Q];
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        f[i] = ST::decode(pop[i * m.N + zo[1 - L::CZ[i]] + yo[1 - L::CY[i]] + xo[1 - L::CX[i]]],
                          (R)L::W[i], n0);
    double nd, dx, dy, dz;
    raw_moments<3, R>(f, nd, dx, dy, dz);
    const R n = (R)nd;
    const R j[3] = {(R)(dx + swap_pair(dx)), (R)(dy + swap_pair(dy)), (R)(dz + swap_pair(dz))};
    R rem = 0;
    if constexpr (!std::is_same<R, double>::value)  // as the moment field keeps it
        rem = unpack_rem1(pack_rem1(n, (R)(nd - (double)n)), n);
    const bool self = (m.self_on >> J) & 1, any_self = m.self_on & 3;
    sn[tid] = n;
    R psi = n;
    if constexpr (PSI != 0)
        if (any_self) sp[tid ^ 1] = psi = psi_of<R, PSI>(n);
    __syncthreads();
    if (!inner) return;

    const int at0 = tid ^ 1;
    auto off = [&](int vx, int vy, int vz) { return 2 * (vx + EX * (vy + EY * vz)); };
    double c[3] = {0, 0, 0}, ss[3] = {0, 0, 0};
#pragma unroll
    for (int a = S::NE / 2; a < S::NE; ++a) {
        constexpr auto T = S::T;
        const int vx = T.e[a][0], vy = T.e[a][1], vz = T.e[a][2], o = off(vx, vy, vz);
        const int e3[3] = {vx, vy, vz};
        const R W = (R)T.W[a];
        const R d = sn[at0 + o] - sn[at0 - o];
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (e3[q]) c[q] += (double)(W * (R)e3[q]) * (double)d;
        if constexpr (PSI != 0)
            if (any_self) {
                const R p = sp[at0 + o] - sp[at0 - o];
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (e3[q]) ss[q] += (double)(W * (R)e3[q]) * (double)p;
            }
    }
    const R gx = (R)(J ? m.g[1][0] : m.g[0][1]), gs = (R)(J ? m.g[1][1] : m.g[0][0]);
    R F[3], p[3];
    const R inv = R(1) / (n + sn[at0]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const R cf = (R)c[q];
        F[q] = sc_force(gx, n, cf, gs, self ? psi : R(0), PSI == 0 ? swap_pair(cf) : (R)ss[q]);
        p[q] = fma_r(R(0.5), F[q] + swap_pair(F[q]), j[q]);
    }
    typename ST::T *out = dst + m.pop_off + (long)J * L::Q * m.N + (zo[1] + yo[1] + xo[1]);
    collide_tau1_component<3, R>(n, rem, F, p, inv, [&](int i, R v) {
        out[i * m.N] = ST::encode(v, (R)L::W[i], n0);
        return v;
    });
}

// Boxes of 8 x 4 x 4 nodes at E4 (360 with the halo) and 4 x 4 x 4 at E6 (512):
// of the boxes that a workgroup's lanes hold, none was faster.  One launch pays
// while the boxes fit the chip at one workgroup per CU: a workgroup is one
// round of loads and the pulls of its halo, and a second one on a CU doubles
// both.  us per call in a loop of calls, two launches against one, psi = n: FP32
// E4 24^3 (108 boxes) 8.1, 6.6; 32^3 (256) 8.5, 7.3; 33^3 (405) 9.0, 10.8; 40^3
// (500) 10.4, 11.9; E6 24^3 (216) 9.0, 7.8; 25^3 (343) 9.5, 11.5; 32^3 (512) 9.2,
// 12.5; FP16 E6 24^3 8.9, 7.1; 32^3 9.1, 10.8.  With psi the two passes take it
// of every stencil neighbour, and two workgroups per CU still pay: FP32 E4 40^3
// 13.5, 12.7; E6 24^3 14.3, 8.8; 32^3 13.9, 13.5; in FP64, whose pulls are twice
// as wide, one: E4 32^3 14.5, 11.0.  Two sides that take two launches although
// their boxes fit: E6 with psi = n in FP64 (8^3 8.4, 9.2; 24^3 11.2, 11.4;
// 16 x 32 x 32 10.7, 11.4) and what one workgroup of the two passes holds, 256
// nodes, at E6 (5^3 5.9, 7.1).
// In graphs, without the calls' own time, the sides lie as far apart (FP32 E6
// 32^3 8.8, 12.1; FP16 E4 40^3 8.8, 9.8; FP64 E6 24^3 9.9, 11.5).  A Python loop
// of scmc_step_static, 8.6 us a call with one launch, takes 11.3 with two whatever
// they do, which hides the difference (FP32 E6 32^3 11.1, 12.5; FP16 11.3, 10.5).
bool step_once_shape(const StepKey &k, const Member &m, MomShape *g) {
    if (k.dim != 3 || k.mom != 1 || k.node || k.sr || (k.order != 4 && k.order != 6)) return false;
    if (k.order == 6 && !k.psi && (k.storage == ST_F64 || m.N <= 256)) return false;
    *g = MomShape{std::min(k.order == 4 ? 8 : 4, m.nx), std::min(4, m.ny), std::min(4, m.nz)};
    g->ntx = (m.nx + g->w - 1) / g->w;
    g->nty = (m.ny + g->h - 1) / g->h;
    g->nchunks = (m.nz + g->zc - 1) / g->zc;
    const long boxes = (long)g->ntx * g->nty * g->nchunks;
    return boxes <= (k.psi && k.storage != ST_F64 ? 512 : 256);
}

hipError_t launch_step_once(const StepKey &k, const Member &m, const MomShape &g, const void *src,
                            void *dst, hipStream_t st) {
    hipError_t err = hipErrorInvalidValue;
    auto go = [&](auto stv, auto Oc) {
        using ST = decltype(stv);
        using T = typename ST::T;
        constexpr int O = decltype(Oc)::value, R2 = O == 4 ? 2 : 4;
        const int ext = (g.w + R2) * (g.h + R2) * (g.zc + R2);
        const dim3 b((2 * ext + 63) / 64 * 64), n(g.ntx * g.nty * g.nchunks);
        if (k.psi)
            hipLaunchKernelGGL((k_step_once<O, ST, 1>), n, b, 0, st, m, g, (const T *)src, (T *)dst);
        else
            hipLaunchKernelGGL((k_step_once<O, ST, 0>), n, b, 0, st, m, g, (const T *)src, (T *)dst);
        err = hipGetLastError();
    };
    auto order = [&](auto stv) {
        if (k.order == 4) go(stv, std::integral_constant<int, 4>{});
        else go(stv, std::integral_constant<int, 6>{});
    };
    switch (k.storage) {
        case ST_F64: order(StoreF64{}); break;
        case ST_F32: order(StoreF32{}); break;
        case ST_F16: order(StoreF16{}); break;
        case ST_BF16: order(StoreBF16{}); break;
    }
    return err;
}

}  // namespace scmc
