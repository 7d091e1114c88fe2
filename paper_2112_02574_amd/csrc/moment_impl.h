// moment_impl.h -- steps of the moment two-pass that stay in the moment field
// (D3Q19, tau = 1).
//
// At tau = 1 the post-collision populations f* are functions of the node's
// moments (n_A, n_B, j) and of the stencil concentrations, and the next step
// needs of them only its own moments sum_i f*_i(x - xi_i) (1, xi_i).  A call
// of k steps therefore reads the populations once (pass 1), makes k - 1 steps
// here, from one moment field to another, and stores populations once
// (pass 2).  A site then moves 24 B each way per step in FP32 instead of
// 352 B, and both fields of lattices up to about 170^3 stay in the Infinity
// Cache, so these steps are bound by vector instructions, not by memory.
//
// A workgroup marches a column of w x h nodes through a chunk of z-planes.
// Per plane it collides the column and a rim of one node (its populations
// stream in) and exchanges the 16 populations that leave the node's own
// column through LDS; each node then adds up what arrives for planes z - 1, z
// and z + 1 in FP64 registers and stores the moments of plane z - 1, which is
// complete.  The concentrations sit in an LDS ring of 2 R + 1 planes (R = the
// stencil's reach), loaded one plane ahead.  Two neighbouring lanes share a
// node, one per component: they exchange what the common velocity needs
// (force, momentum) by DPP, and the halved work per lane doubles the
// wavefronts that a column of given size offers.
//
// Every population, decoded as the storage format would hold it, and every
// sum is formed as in the two passes (collide_tau1_component, raw_moments),
// so a call of k steps equals k calls of one step bit for bit.
//
// Measured against the two passes of every step (us per step, blocks of 12 to
// 512 steps): 128^3 E6 FP32 122 -> 75, 150 x 141 x 165 FP32 334 -> 138,
// 100 x 84 x 92 FP64 101 -> 52, 192^3 FP16 348 -> 273, 63^3 E4 with psi 27.7
// -> 22.2, 96 x 104 x 112 FP16 node storage 79 -> 72.
#pragma once

#include "fused_impl.h"  // xcd_remap
#include "site_ops.h"

namespace scmc {

template <int ORDER> struct MomGeom {
    static constexpr int R = ORDER == 4 ? 1 : 2;       // stencil reach
    static constexpr int NSLOT = 2 * R + 1;            // planes of the ring
    static constexpr int PMAX = R == 1 ? 640 : 768;    // nodes of a ring plane
};

// value of the other component's lane
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

template <class R> struct RawVal;
template <> struct RawVal<float> {
    __device__ __forceinline__ static float load(__amdgpu_buffer_rsrc_t r, int v, int s) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
    }
    __device__ __forceinline__ static void store(float x, __amdgpu_buffer_rsrc_t r, int v, int s) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, v, s, 0);
    }
};
template <> struct RawVal<double> {
    __device__ __forceinline__ static double load(__amdgpu_buffer_rsrc_t r, int v, int s) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    }
    __device__ __forceinline__ static void store(double x, __amdgpu_buffer_rsrc_t r, int v, int s) {
        using U2 = unsigned __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), r, v, s, 0);
    }
};

// exchange slot of a direction that leaves the column: in-plane ones first
__device__ constexpr int mom_dir(int i) {
    constexpr int at[19] = {-1, 0, 1, 2, 3, -1, -1, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15};
    return at[i];
}

// One column chunk: collides planes z0 - 1 .. z0 + len and stores the moments
// of planes z0 .. z0 + len - 1 of the columns [x0, x0 + wx) x [y0, y0 + wy),
// (wx + 2)(wy + 2) <= MOM_EXT and (wx + 2 + 2R)(wy + 2 + 2R) <= PMAX.  The
// populations are exchanged in STAGES rounds of 16 / STAGES directions, which
// share one LDS buffer.
template <int ORDER, class ST, int PSI, bool NODE, int STAGES>
__device__ __forceinline__ void mom_column(const Member &m, const typename ST::R *__restrict__ in,
                                           typename ST::R *__restrict__ out, int in_slot,
                                           int out_slot, int x0, int y0, int z0, int wx, int wy,
                                           int len) {
    using G = MomGeom<ORDER>;
    using L = Lattice<3>;
    using S = Stencil<3, ORDER>;
    using R = typename ST::R;
    constexpr int RR = G::R, NSLOT = G::NSLOT, PMAX = G::PMAX, NT = MOM_THREADS;
    constexpr int SZ = (int)sizeof(R);
    constexpr bool F64 = std::is_same<R, double>::value;
    constexpr int ND = 16 / STAGES;
    __shared__ R ring[NSLOT][PMAX * 2];
    __shared__ R pring[PSI ? NSLOT : 1][PSI ? PMAX * 2 : 1];
    __shared__ R xb[ND][NT];

    const int tid = threadIdx.x, J = tid & 1;
    const int EW = wx + 2, ET = EW * (wy + 2);
    const int PW = EW + 2 * RR, PN = PW * (wy + 2 + 2 * RR);
    const int nxy = m.nx * m.ny;
    // whole wavefronts past the rim idle; single lanes past it repeat its last node
    const bool busy = ((tid & ~63) >> 1) < ET;
    const int e = min(tid >> 1, ET - 1);
    const int ey = e / EW, ex = e - ey * EW;
    const bool inner = (tid >> 1) < ET && ex >= 1 && ex <= wx && ey >= 1 && ey <= wy;
    const int gsite = wrap1(y0 - 1 + ey, m.ny) * m.nx + wrap1(x0 - 1 + ex, m.nx);
    // the ring values this thread loads: q and q + NT of plane order
    int pv[2];
    bool pon[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int q = tid + c * NT, s = min(q >> 1, PN - 1);
        const int py = s / PW, px = s - py * PW;
        pon[c] = (q >> 1) < PN;
        pv[c] = ((wrap1(y0 - 1 - RR + py, m.ny) * m.nx + wrap1(x0 - 1 - RR + px, m.nx)) * 2 + J) * SZ;
    }
    const int pbytes = m.N * SZ;
    const R *ib = in;
    R *ob = out;
    const __amdgpu_buffer_rsrc_t ipr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(ib + (long)in_slot * m.N), (short)0, 2 * pbytes, BUF_DATA_FORMAT_32);
    const __amdgpu_buffer_rsrc_t imr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(ib + 2L * m.N), (short)0, (F64 ? 3 : 4) * pbytes, BUF_DATA_FORMAT_32);
    const __amdgpu_buffer_rsrc_t opr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(ob + (long)out_slot * m.N), (short)0, 2 * pbytes, BUF_DATA_FORMAT_32);
    const __amdgpu_buffer_rsrc_t omr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(ob + 2L * m.N), (short)0, (F64 ? 3 : 4) * pbytes, BUF_DATA_FORMAT_32);

    const R gx = (R)(J ? m.g[1][0] : m.g[0][1]), gs = (R)(J ? m.g[1][1] : m.g[0][0]);
    const bool self = (m.self_on >> J) & 1, any_self = m.self_on & 3;
    const R n0 = (R)m.n0[J];

    auto put_ring = [&](int slot, int c, R v) {
        if (!pon[c]) return;
        const int q = tid + c * NT;
        ring[slot][q] = v;
        // psi of the own component, at the index the other lane's n has
        if constexpr (PSI != 0)
            if (any_self) pring[slot][q ^ 1] = psi_of<R, PSI>(v);
    };
    auto load_mom = [&](int z, R(&j)[3], unsigned &rem) {
        const int so = z * nxy * SZ;
#pragma unroll
        for (int c = 0; c < 3; ++c) j[c] = RawVal<R>::load(imr, gsite * SZ, so + c * pbytes);
        if constexpr (!F64)
            rem = __builtin_amdgcn_raw_buffer_load_b32(imr, gsite * SZ, so + 3 * pbytes, 0);
    };

    // ring slot k % NSLOT holds plane z0 - 1 - RR + k
#pragma unroll
    for (int k = 0; k < 2 * RR + 1; ++k) {
        const int z = wrap1(z0 - 1 - RR + k, m.nz);
#pragma unroll
        for (int c = 0; c < 2; ++c) put_ring(k, c, RawVal<R>::load(ipr, pv[c], z * nxy * 2 * SZ));
    }
    R jn[3];
    unsigned remn = 0;
    load_mom(wrap1(z0 - 1, m.nz), jn, remn);
    __syncthreads();

    int row[2 * RR + 1];  // the other component of the node's ring rows
#pragma unroll
    for (int d = -RR; d <= RR; ++d) row[d + RR] = 2 * ((ey + RR + d) * PW + ex + RR) + (1 - J);
    int slot[NSLOT];
#pragma unroll
    for (int d = 0; d < NSLOT; ++d) slot[d] = d;

    double aP[3] = {0, 0, 0}, aC[3] = {0, 0, 0};  // n, j_x, j_y of planes z - 1 and z
    double zP = 0, zC = 0;                        // what arrived from below (j_z)
    for (int k = 0; k < len + 2; ++k) {
        const R j[3] = {jn[0], jn[1], jn[2]};
        const unsigned remw = remn;
        R pre[2] = {0, 0};
        if (k < len + 1) {  // next plane's loads, waited for after the collision
            const int zp = wrap1(z0 + RR + k, m.nz);
#pragma unroll
            for (int c = 0; c < 2; ++c) pre[c] = RawVal<R>::load(ipr, pv[c], zp * nxy * 2 * SZ);
            load_mom(wrap1(z0 + k, m.nz), jn, remn);
        }
        R f[19];
        if (busy) {
            auto at = [&](int dx, int dy, int dz) {
                return ring[slot[dz + RR]][row[dy + RR] + 2 * dx];
            };
            const R n = ring[slot[RR]][row[RR] - 1 + 2 * J], no = at(0, 0, 0);
            double cs[3] = {0, 0, 0}, ss[3] = {0, 0, 0};
#pragma unroll
            for (int a = S::NE / 2; a < S::NE; ++a) {
                constexpr auto T = S::T;
                const int ex_ = T.e[a][0], ey_ = T.e[a][1], ez_ = T.e[a][2];
                const R d = at(ex_, ey_, ez_) - at(-ex_, -ey_, -ez_);
                const R W = (R)T.W[a];
                const int e3[3] = {ex_, ey_, ez_};
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (e3[c]) cs[c] += (double)(W * (R)e3[c]) * (double)d;
                if constexpr (PSI != 0)
                    if (any_self) {
                        const R q = pring[slot[ez_ + RR]][row[ey_ + RR] + 2 * ex_] -
                                    pring[slot[RR - ez_]][row[RR - ey_] - 2 * ex_];
#pragma unroll
                        for (int c = 0; c < 3; ++c)
                            if (e3[c]) ss[c] += (double)(W * (R)e3[c]) * (double)q;
                    }
            }
            R psi = R(0);
            if constexpr (PSI == 0) {
                psi = self ? n : R(0);
            } else if (self) {
                psi = pring[slot[RR]][row[RR]];
            }
            R F[3], u[3];
            const R inv = R(1) / (n + no);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const R cf = (R)cs[c];
                const R t = PSI == 0 ? swap_pair(cf) : (R)ss[c];
                F[c] = -gx * n * cf - gs * psi * t;
                u[c] = (j[c] + R(0.5) * (F[c] + swap_pair(F[c]))) * inv;
            }
            R rem = 0;
            if constexpr (!F64) rem = unpack_rem1(J ? remw >> 16 : remw, n);
            collide_tau1_component<3, R>(n, rem, F, u[0], u[1], u[2], [&](int i, R v) {
                if constexpr (NODE) {
                    if (i == 0) return f[0] = v;
                    // encoded against the density of the node it streams to
                    const R ref = node_ref((R)L::W[i], swap_pair(at(L::CX[i], L::CY[i], L::CZ[i])));
                    return f[i] = ST::from_node(ST::to_node(v, ref), ref);
                } else {
                    f[i] = ST::stored(v, (R)L::W[i], n0);
                    return v;
                }
            });
        }
        double gp = 0, g0 = 0, gm = 0, xp = 0, yp = 0;
        // what arrives at this node along xi_i, in the order of raw_moments
        auto arrive = [&](int i) {
            const int d = mom_dir(i);
            const double v = d < 0 ? f[i] : xb[d % ND][tid - 2 * (L::CX[i] + L::CY[i] * EW)];
            double &g = L::CZ[i] == 0 ? g0 : L::CZ[i] > 0 ? gp : gm;
            double &x = L::CZ[i] == 0 ? aC[1] : L::CZ[i] > 0 ? xp : aP[1];
            double &y = L::CZ[i] == 0 ? aC[2] : L::CZ[i] > 0 ? yp : aP[2];
            g += v;
            if (L::CX[i]) x += (double)L::CX[i] * v;
            if (L::CY[i]) y += (double)L::CY[i] * v;
        };
#pragma unroll
        for (int st = 0; st < STAGES; ++st) {
            if (STAGES > 1) __syncthreads();
            if (busy) {
#pragma unroll
                for (int i = 1; i < 19; ++i)
                    if (mom_dir(i) >= 0 && mom_dir(i) / ND == st) xb[mom_dir(i) % ND][tid] = f[i];
            }
            __syncthreads();
            if (st == 0 && k < len + 1) {
#pragma unroll
                for (int c = 0; c < 2; ++c) put_ring(slot[0], c, pre[c]);
            }
            if (inner) {
#pragma unroll
                for (int i = 0; i < 19; ++i)
                    if ((mom_dir(i) < 0 ? 0 : mom_dir(i) / ND) == st) arrive(i);
            }
        }
        if (inner && k >= 2) {  // plane z - 1 is complete
            const int so = wrap1(z0 + k - 2, m.nz) * nxy * SZ;
            const double nx_ = aP[0] + gm;
            const R nf = (R)nx_;
            const double jz_ = zP - gm;
            const R jx = (R)(aP[1] + swap_pair(aP[1]));
            const R jy = (R)(aP[2] + swap_pair(aP[2]));
            const R jz = (R)(jz_ + swap_pair(jz_));
            RawVal<R>::store(nf, opr, (gsite * 2 + J) * SZ, 2 * so);
            RawVal<R>::store(J ? jy : jx, omr, gsite * SZ + J * pbytes, so);
            if constexpr (F64) {
                if (J == 0) RawVal<R>::store(jz, omr, gsite * SZ, so + 2 * pbytes);
            } else {
                const unsigned own = pack_rem1(nf, (R)(nx_ - (double)nf));
                const unsigned oth = (unsigned)swap_bits((int)own);
                const unsigned w = own << 16 | oth;  // lane 1 stores it: n_A's half low
                RawVal<R>::store(J ? __builtin_bit_cast(float, w) : jz, omr,
                                 gsite * SZ + J * pbytes, so + 2 * pbytes);
            }
        }
        // the sums move on: plane z -> z - 1, z + 1 -> z
        aP[0] = aC[0] + g0;
        aP[1] = aC[1];
        aP[2] = aC[2];
        zP = zC;
        aC[0] = zC = gp;
        aC[1] = xp;
        aC[2] = yp;
        const int s0 = slot[0];
#pragma unroll
        for (int d = 0; d + 1 < NSLOT; ++d) slot[d] = slot[d + 1];
        slot[NSLOT - 1] = s0;
        if (STAGES == 1) __syncthreads();
    }
}

template <int ORDER, class ST, int PSI, bool NODE, int STAGES>
__global__ void __launch_bounds__(MOM_THREADS)
    k_mom_step(Member m, MomShape g, const typename ST::R *__restrict__ in,
               typename ST::R *__restrict__ out, int in_slot, int out_slot) {
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    const int tx = t % g.ntx, q = t / g.ntx, ty = q % g.nty, c = q / g.nty;
    const int x0 = tx * g.w, y0 = ty * g.h, z0 = c * g.zc;
    mom_column<ORDER, ST, PSI, NODE, STAGES>(m, in, out, in_slot, out_slot, x0, y0, z0,
                                             min(g.w, m.nx - x0), min(g.h, m.ny - y0),
                                             min(g.zc, m.nz - z0));
}

// The exchange of all 16 directions at once takes 64 KB of LDS in FP32 beside
// the ring's 12-61 KB.  In FP64 it would take 128 KB beside 30-61 KB (123 KB
// with psi): two rounds, or four with the E6 ring of n and psi.
template <class ST, int ORDER, int PSI> constexpr int mom_stages() {
    return sizeof(typename ST::R) == 4 ? 1 : ORDER == 6 && PSI != 0 ? 4 : 2;
}

template <class ST, int ORDER> struct MomOps {
    static void *kernel(const StepKey &k);
};

template <class ST, int ORDER> void *MomOps<ST, ORDER>::kernel(const StepKey &k) {
    auto pick = [&](auto Nc) -> void * {
        constexpr bool N = decltype(Nc)::value;
        return k.psi ? (void *)&k_mom_step<ORDER, ST, 1, N, mom_stages<ST, ORDER, 1>()>
                     : (void *)&k_mom_step<ORDER, ST, 0, N, mom_stages<ST, ORDER, 0>()>;
    };
    if (!k.node) return pick(std::false_type{});
    if constexpr (sizeof(typename ST::T) == 2) return pick(std::true_type{});
    return nullptr;
}

}  // namespace scmc
