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
// stream in).  What leaves for the eight neighbouring columns is exchanged
// through LDS as FP64 sums: a node first adds, over three planes of its march,
// the populations that arrive at the same node of a neighbouring column
// (ColumnSums: S and D per column), so 12 values per component cross instead
// of 16 and arrive already converted.  A plane's moments are complete and
// stored one plane later.  The concentrations sit in an LDS ring of 2 R + 1
// planes (R = the stencil's reach), loaded one plane ahead.  Two neighbouring
// lanes share a node, one per component: they exchange what the common velocity needs
// (force, momentum) by DPP, and the halved work per lane doubles the
// wavefronts that a column of given size offers.
//
// Every population, decoded as the storage format would hold it, and every
// sum is formed as in the two passes (collide_tau1_component, raw_moments),
// so a call of k steps equals k calls of one step bit for bit.
//
// us per step against pass 1 and pass 2 of every step: E6 128^3 FP32 122 ->
// 64, 150 x 141 x 165 FP32 337 -> 120, 192^3 FP16 343 -> 236, 100 x 84 x 92
// FP64 102 -> 37, E4 with psi 63^3 FP32 27.4 -> 17.4.  At 128^3 a lane issues
// 307 vector instructions per plane (430 with 16 exchanged populations
// instead of 12 sums), which keeps the SIMDs busy 85 % of the time; at 63^3 72 %,
// the rest of it waiting on the exchange.  FP64 with psi does not fit a lane's 128
// registers (E6 spills 33 of them, E4 3): 48^3 E4 takes 15.5 us per step, with
// psi = n 11.5, 40^3 E6 22.6, with psi = n 10.6 (step_rules.h keeps it off the
// sizes where the two passes are faster).
#pragma once

#include "fused_impl.h"  // xcd_remap
#include "site_ops.h"

namespace scmc {

// A plane of the ring holds MOM_PW x ROWS nodes: columns are at most
// MOM_PW - 2 - 2R wide and ROWS - 2 - 2R high, and MOM_EXT nodes with their
// rim.  The exchange of 12 FP64 values per lane in STAGES rounds takes
// 96 KB / STAGES of the 160 KB of LDS, the ring (and psi's) the rest.
constexpr int MOM_PW = 40;
template <int ORDER, class R, int PSI> struct MomGeom {
    static constexpr int REACH = ORDER == 4 ? 1 : 2;
    static constexpr int NSLOT = 2 * REACH + 1;
    static constexpr int STAGES = sizeof(R) == 8 && ORDER == 6 && PSI != 0 ? 4 : 1;
    static constexpr int XBYTES = 12 / STAGES * MOM_THREADS * 8;
    static constexpr int ROWBYTES = NSLOT * (PSI ? 2 : 1) * MOM_PW * 2 * (int)sizeof(R);
    static constexpr int FIT = (160 * 1024 - XBYTES) / ROWBYTES;
    static constexpr int ROWS = FIT < 25 ? FIT : 25;  // two loads per lane fill a plane
    static_assert(ROWS * MOM_PW <= MOM_THREADS && ROWS >= 12, "ring size");
};

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

// One column chunk: collides planes z0 - 1 .. z0 + len and stores the moments
// of planes z0 .. z0 + len - 1 of the columns [x0, x0 + wx) x [y0, y0 + wy).
template <int ORDER, class ST, int PSI, bool NODE>
__device__ __forceinline__ void mom_column(const Member &m, const typename ST::R *__restrict__ in,
                                           typename ST::R *__restrict__ out, int in_slot,
                                           int out_slot, int x0, int y0, int z0, int wx, int wy,
                                           int len) {
    using L = Lattice<3>;
    using S = Stencil<3, ORDER>;
    using R = typename ST::R;
    using G = MomGeom<ORDER, R, PSI>;
    constexpr bool F64 = sizeof(R) == 8;
    constexpr int RR = G::REACH, NSLOT = G::NSLOT, NT = MOM_THREADS, PW = MOM_PW;
    constexpr int PLANE = PW * G::ROWS * 2, SZ = (int)sizeof(R), NX = 12 / G::STAGES;
    __shared__ double xb[NX][NT];
    __shared__ R ring[NSLOT][PLANE];
    __shared__ R pring[PSI ? NSLOT : 1][PSI ? PLANE : 1];

    const int tid = threadIdx.x, J = tid & 1;
    const int EW = wx + 2, ET = EW * (wy + 2);
    const int PX = EW + 2 * RR, PN = PX * (wy + 2 + 2 * RR);
    const int nxy = m.nx * m.ny;
    const int e = min(tid >> 1, ET - 1);  // lanes past the rim repeat its last node
    const int ey = e / EW, ex = e - ey * EW;
    const bool inner = (tid >> 1) < ET && ex >= 1 && ex <= wx && ey >= 1 && ey <= wy;
    // where the node's arrivals are looked up (a rim lane's go unused)
    const int from = inner ? tid : 2 * (EW + 1) + J;
    const int gcol = wrap1(y0 - 1 + ey, m.ny) * m.nx + wrap1(x0 - 1 + ex, m.nx);
    // the ring values this thread loads: nodes tid / 2 and (tid + threads) / 2 of the plane
    int pv[2], pl[2];
    bool pon[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int s0 = (tid + c * (int)blockDim.x) >> 1, s = min(s0, PN - 1);
        const int py = s / PX, px = s - py * PX;
        pon[c] = s0 < PN;
        pl[c] = (py * PW + px) * 2 + J;
        pv[c] = ((wrap1(y0 - 1 - RR + py, m.ny) * m.nx + wrap1(x0 - 1 - RR + px, m.nx)) * 2 + J) * SZ;
    }
    const int pbytes = m.N * SZ;
    const __amdgpu_buffer_rsrc_t ipr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(in + m.dens_off + (long)in_slot * m.N), (short)0, 2 * pbytes, BUF_DATA_FORMAT_32);
    const __amdgpu_buffer_rsrc_t imr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(in + m.dens_off + 2L * m.N), (short)0, (F64 ? 3 : 4) * pbytes, BUF_DATA_FORMAT_32);
    const __amdgpu_buffer_rsrc_t opr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(out + m.dens_off + (long)out_slot * m.N), (short)0, 2 * pbytes, BUF_DATA_FORMAT_32);
    const __amdgpu_buffer_rsrc_t omr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(out + m.dens_off + 2L * m.N), (short)0, (F64 ? 3 : 4) * pbytes, BUF_DATA_FORMAT_32);

    const R gx = (R)(J ? m.g[1][0] : m.g[0][1]), gs = (R)(J ? m.g[1][1] : m.g[0][0]);
    const bool self = (m.self_on >> J) & 1, any_self = m.self_on & 3;
    const R n0 = (R)(J ? m.n0[1] : m.n0[0]);  // no lane's index: m stays in scalar registers
    // psi beside the collision, before the exchange's barrier, and the self sums
    // without a branch per stencil pair, over zeros where there are no self
    // couplings: us per step with psi, E4 FP32, 128^3 76.6 -> 73.5, 63^3 19.6 ->
    // 18.8, 30^3 8.7 -> 8.2.  E6 FP32 and E4 FP64, short of registers, were
    // slower that way (100 x 90 x 110: 57.9 -> 59.2, 57.0 -> 59.6).
    constexpr bool EARLY = PSI != 0 && ORDER == 4 && !F64;

    auto load_ring = [&](int z, R(&v)[2]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) v[c] = RawVal<R>::load(ipr, pv[c], z * nxy * 2 * SZ);
    };
    auto take_psi = [&](const R(&v)[2], R(&q)[2]) {
        q[0] = q[1] = R(0);
        if (any_self) {
            q[0] = psi_of<R, PSI>(v[0]);
            q[1] = psi_of<R, PSI>(v[1]);
        }
    };
    auto put_ring = [&](int slot, const R(&v)[2], const R(&q)[2]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (!pon[c]) continue;
            ring[slot][pl[c]] = v[c];
            // psi of the own component, at the index the other lane's n has
            if constexpr (EARLY)
                pring[slot][pl[c] ^ 1] = q[c];
            else if constexpr (PSI != 0)
                if (any_self) pring[slot][pl[c] ^ 1] = psi_of<R, PSI>(v[c]);
        }
    };
    auto load_mom = [&](int z, R(&j)[3], unsigned &rem) {
        const int so = z * nxy * SZ;
#pragma unroll
        for (int c = 0; c < 3; ++c) j[c] = RawVal<R>::load(imr, gcol * SZ, so + c * pbytes);
        if constexpr (!F64)
            rem = __builtin_amdgcn_raw_buffer_load_b32(imr, gcol * SZ, so + 3 * pbytes, 0);
    };

    // round k collides plane z = z0 - 1 + k; the ring's slot s holds plane z - RR + s
    auto wrapz = [&](int z) { return ((z % m.nz) + m.nz) % m.nz; };
    // all loads before the first wait: the stores to the ring are under a branch
    // that the compiler moves no load across.  us per step with a wait per
    // plane -> one wait: 25 x 26 x 23 BF16 8.3 -> 7.8, 63^3 FP32 with psi 18.1
    // -> 17.8, 192^3 FP16 244 -> 236, 128^3 FP32 64.6 -> 64.1 (124 x 142 x 148
    // with psi 96 -> 97)
    R v0[NSLOT][2], jn[3];
    unsigned remn = 0;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) load_ring(wrapz(z0 - 1 - RR + s), v0[s]);
    load_mom(wrapz(z0 - 1), jn, remn);
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
        R q[2] = {0, 0};
        if constexpr (EARLY) take_psi(v0[s], q);
        put_ring(s, v0[s], q);
    }
    __syncthreads();

    // the other component's value at the low corner of the node's stencil box
    // in a ring plane (offsets from it are non-negative, as LDS accesses take)
    const int at0 = 2 * (ey * PW + ex) + (1 - J);
    int slot[NSLOT];
#pragma unroll
    for (int d = 0; d < NSLOT; ++d) slot[d] = d;

    // on their way, per neighbouring column and for the own one (index 4): the
    // populations from below to planes z - 1 and z (up1, up2), and the sum to
    // plane z - 1 without the one from above; the diagonal columns' sums of z - 1
    double up1[5] = {0, 0, 0, 0, 0}, up2[5] = {0, 0, 0, 0, 0}, um[5] = {0, 0, 0, 0, 0};
    ColumnSums cs;
    cs.nd = cs.xd = cs.yd = 0;
    // The chunk's first plane (KIND 0) only sends up and its last (KIND 2) only
    // down: their rounds leave out the rest.
    auto round = [&](auto kind, int k) {
        constexpr int KIND = decltype(kind)::value;
        const R j[3] = {jn[0], jn[1], jn[2]};
        const unsigned remw = remn;
        R pre[2], preq[2] = {0, 0};  // the next round's loads, waited for after the collision
        if constexpr (KIND < 2) {
            load_ring(wrap1(z0 + RR + k, m.nz), pre);
            load_mom(wrap1(z0 + k, m.nz), jn, remn);
        }
        double X[12];  // S, D of plane z - 1 per column, diagonals of plane z
        double own = 0, ownD = 0;
        {
            auto at = [&](int dx, int dy, int s) {
                return ring[slot[s]][at0 + 2 * ((dy + RR) * PW + dx + RR)];
            };
            auto pat = [&](int dx, int dy, int s) {
                return pring[slot[s]][at0 + 2 * ((dy + RR) * PW + dx + RR)];
            };
            double c[3] = {0, 0, 0}, ss[3] = {0, 0, 0};
            const R n = ring[slot[RR]][at0 - 1 + 2 * J + 2 * (RR * PW + RR)], no = at(0, 0, RR);
#pragma unroll
            for (int a = S::NE / 2; a < S::NE; ++a) {
                constexpr auto T = S::T;
                const int vx = T.e[a][0], vy = T.e[a][1], vz = T.e[a][2];
                const int e3[3] = {vx, vy, vz};
                const R W = (R)T.W[a];
                const R d = at(vx, vy, RR + vz) - at(-vx, -vy, RR - vz);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (e3[q]) c[q] += (double)(W * (R)e3[q]) * (double)d;
                if constexpr (PSI != 0)
                    if (EARLY || any_self) {
                        const R p = pat(vx, vy, RR + vz) - pat(-vx, -vy, RR - vz);
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            if (e3[q]) ss[q] += (double)(W * (R)e3[q]) * (double)p;
                    }
            }
            const R psi = !self ? R(0) : PSI == 0 ? n : pat(0, 0, RR);
            R F[3], p[3];
            const R inv = R(1) / (n + no);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const R cf = (R)c[q];
                const R t = PSI == 0 ? swap_pair(cf) : (R)ss[q];
                F[q] = sc_force(gx, n, cf, gs, psi, t);
                p[q] = fma_r(R(0.5), F[q] + swap_pair(F[q]), j[q]);
            }
            R rem = 0;
            if constexpr (!F64) rem = unpack_rem1(J ? remw >> 16 : remw, n);
            double num[5], nup[5];
            auto send = [&](int q, double v) {  // for the first round of the exchange
                if (q < NX) xb[q][tid] = v;
                else X[q] = v;
            };
            // f: a population of the node as the next step pulls it
            auto give = [&](int i, R f) {
                if (KIND == 0 && L::CZ[i] != 1) return;
                if (KIND == 2 && L::CZ[i] != -1) return;
#pragma unroll
                for (int a = 0; a < 5; ++a) {
                    if (i == (a < 4 ? COL_MID[a & 3] : 0)) num[a] = up2[a] + (double)f;
                    if (i == (a < 4 ? COL_UP[a & 3] : 5)) nup[a] = f;
                    if (i != (a < 4 ? COL_DOWN[a & 3] : 6)) continue;
                    const double down = f, sum = um[a] + down, dif = up1[a] - down;
                    if (a < 4) {
                        send(a, sum);
                        send(4 + a, dif);
                    } else {
                        own = sum;
                        ownD = dif;
                    }
                }
                if (i >= 7 && i <= 10) send(i + 1, f);
            };
            collide_tau1_component<3, R>(n, rem, F, p, inv, [&](int i, R v) {
                if constexpr (NODE) {
                    R f = v;
                    if (i > 0 && (KIND == 1 || L::CZ[i] == 1 - KIND)) {  // encoded against the density of the node it streams to
                        const R ref = node_ref(
                            (R)L::W[i], swap_pair(at(L::CX[i], L::CY[i], RR + L::CZ[i])));
                        f = ST::from_node(ST::to_node(v, ref), ref);
                    }
                    give(i, f);
                    return f;
                } else {
                    give(i, ST::stored(v, (R)L::W[i], n0));
                    return v;
                }
            });
            if constexpr (KIND < 2) {
#pragma unroll
                for (int a = 0; a < 5; ++a) {
                    up1[a] = up2[a];
                    up2[a] = nup[a];
                    if (KIND == 1) um[a] = num[a];
                }
            }
        }
        if constexpr (KIND < 2 && EARLY) take_psi(pre, preq);
#pragma unroll
        for (int st = 0; st < G::STAGES; ++st) {
            if (st > 0) {
                if (KIND == 0 || (KIND == 2 && st * NX >= 8)) continue;
                __syncthreads();
#pragma unroll
                for (int q = 0; q < NX; ++q) xb[q][tid] = X[st * NX + q];
            }
            __syncthreads();
            if constexpr (KIND < 2)
                if (st == 0) put_ring(slot[0], pre, preq);
            if constexpr (KIND == 0) continue;
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                const int i = st * NX + q, d = i < 8 ? COL_MID[i & 3] : i - 1;
                if (KIND == 2 && i >= 8) continue;
                X[i] = xb[q][from - 2 * (L::CX[d] + L::CY[d] * EW)];
            }
        }
        if constexpr (KIND > 0) {
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                cs.S[a] = X[a];
                cs.D[a] = X[4 + a];
            }
            cs.own = own;
            cs.ownD = ownD;
            double nd, dx, dy, dz;
            cs.total(nd, dx, dy, dz);
            if constexpr (KIND == 1) cs.diag(X[8], X[9], X[10], X[11]);
            if (inner && k >= 2) {  // plane z - 1 is complete
                const int so = wrap1(z0 + k - 2, m.nz) * nxy * SZ;
                const R nf = (R)nd;
                const R jx = (R)(dx + swap_pair(dx)), jy = (R)(dy + swap_pair(dy));
                const R jz = (R)(dz + swap_pair(dz));
                RawVal<R>::store(nf, opr, (gcol * 2 + J) * SZ, 2 * so);
                RawVal<R>::store(J ? jy : jx, omr, gcol * SZ + J * pbytes, so);
                if constexpr (F64) {
                    if (J == 0) RawVal<R>::store(jz, omr, gcol * SZ, so + 2 * pbytes);
                } else {
                    const unsigned mine = pack_rem1(nf, (R)(nd - (double)nf));
                    const unsigned w = mine << 16 | (unsigned)swap_bits((int)mine);
                    // lane 1 stores the remainders, n_A's in the low half
                    RawVal<R>::store(J ? __builtin_bit_cast(float, w) : jz, omr,
                                     gcol * SZ + J * pbytes, so + 2 * pbytes);
                }
            }
        }
        if constexpr (KIND < 2) {
            const int s0 = slot[0];
#pragma unroll
            for (int d = 0; d + 1 < NSLOT; ++d) slot[d] = slot[d + 1];
            slot[NSLOT - 1] = s0;
            __syncthreads();
        }
    };
    round(std::integral_constant<int, 0>{}, 0);
#pragma unroll 1
    for (int k = 1; k <= len; ++k) round(std::integral_constant<int, 1>{}, k);
    round(std::integral_constant<int, 2>{}, len + 1);
}

// Block b of a member's launch: its column and chunk.
template <int ORDER, class ST, int PSI, bool NODE>
__device__ __forceinline__ void mom_block(const Member &m, const MomShape &g, int b,
                                          const typename ST::R *__restrict__ in,
                                          typename ST::R *__restrict__ out, int in_slot,
                                          int out_slot) {
    const int tx = b % g.ntx, q = b / g.ntx, ty = q % g.nty, c = q / g.nty;
    const int x0 = tx * g.w, y0 = ty * g.h, z0 = c * g.zc;
    mom_column<ORDER, ST, PSI, NODE>(m, in, out, in_slot, out_slot, x0, y0, z0,
                                     min(g.w, m.nx - x0), min(g.h, m.ny - y0),
                                     min(g.zc, m.nz - z0));
}

template <int ORDER, class ST, int PSI, bool NODE>
__global__ void __launch_bounds__(MOM_THREADS)
    k_mom_step(Member m, MomShape g, const typename ST::R *__restrict__ in,
               typename ST::R *__restrict__ out, int in_slot, int out_slot) {
    mom_block<ORDER, ST, PSI, NODE>(m, g, xcd_remap(blockIdx.x, gridDim.x), in, out, in_slot,
                                    out_slot);
}

template <int ORDER, class ST, int PSI>
__global__ void __launch_bounds__(MOM_THREADS)
    kb_mom_step(const Member *__restrict__ members, MomList list,
                const typename ST::R *__restrict__ in, typename ST::R *__restrict__ out) {
    const int b = xcd_remap(blockIdx.x, gridDim.x), lane = threadIdx.x & 63;
    const bool mine = lane < list.n && list.e[lane].first <= b;
    const int i = __builtin_amdgcn_readfirstlane(__popcll(__ballot(mine)) - 1);
    const Member m = members[list.e[i].member];
    mom_block<ORDER, ST, PSI, false>(m, list.e[i].g, b - list.e[i].first, in, out, 0, 0);
}

struct MomKernel {
    void *func = nullptr, *batch = nullptr;
    int rows = 0;  // of its ring (MomGeom::ROWS)
};

template <class ST, int ORDER> struct MomOps {
    static MomKernel kernel(const StepKey &k);
};

template <class ST, int ORDER> MomKernel MomOps<ST, ORDER>::kernel(const StepKey &k) {
    using R = typename ST::R;
    auto pick = [&](auto Pc) {
        constexpr int P = decltype(Pc)::value;
        MomKernel q;
        q.rows = MomGeom<ORDER, R, P>::ROWS;
        if (!k.node) {
            q.func = (void *)&k_mom_step<ORDER, ST, P, false>;
            q.batch = (void *)&kb_mom_step<ORDER, ST, P>;
        } else if constexpr (sizeof(typename ST::T) == 2) {
            q.func = (void *)&k_mom_step<ORDER, ST, P, true>;
        }
        return q;
    };
    return k.psi ? pick(std::integral_constant<int, 1>{}) : pick(std::integral_constant<int, 0>{});
}

}  // namespace scmc
