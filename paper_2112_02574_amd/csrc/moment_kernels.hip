// moment_kernels.hip -- launch shape and storage / order dispatch of the steps
// that stay in the moment field; the kernels are instantiated in
// moment_inst.hip (one object per storage format and stencil order).
#include <algorithm>

#include "moment_impl.h"

namespace scmc {

#define SCMC_MOM_COMBOS(X)                                                   \
    X(StoreF64, 4) X(StoreF64, 6) X(StoreF32, 4) X(StoreF32, 6)             \
    X(StoreF16, 4) X(StoreF16, 6) X(StoreBF16, 4) X(StoreBF16, 6)
#define SCMC_EXTERN(S, O) extern template struct MomOps<S, O>;
SCMC_MOM_COMBOS(SCMC_EXTERN)
#undef SCMC_EXTERN

// The launch shape.  Every node costs the collisions of its column's rim and
// of the chunk's two extra planes besides its own, and one workgroup runs per
// CU at a time (LDS).  All column sizes that a workgroup holds and all chunk
// counts are weighed by the rounds of workgroups over the CUs, times the
// planes a chunk marches (two more than it stores, and 1.5 for filling the
// ring), times the time of a plane, 1.6 us + 0.06 us per wavefront: a
// wavefront's latency and the vector instructions of all of them.  The model
// orders measured shapes (us per step of long calls, w x h x zc, the model's
// choice first): 63^3 E4 FP32 21x16x3 13.9, 32x11x3 13.6, 13x21x5 16.5, 13x13x8
// 17.6, 16x21x6 20.3, with psi 17.4, 17.2, 21.0; 128^3 E6 FP32 32x13x22 64.7,
// 26x16x22 65.2, 32x13x26 74.4, 19x16x32 75.4, 32x13x13 (two rounds) 79.9; 48^3 E6
// FP32 16x16x2 11.4, 24x10x2 11.0, 24x16x3 15.6, 24x16x4 18.2; 32^3 E4 FP32 8x16x1
// 6.4, 32x8x1 7.6, 16x16x2 9.5.  Its times are those of psi = n without 16-bit
// rounding, within about 10 % from 60^3 on (63^3 E4 15.6 against 13.9, 128^3 E6
// 65.8 against 64.7) and high below (32^3 E4 8.9 against 6.4); psi adds 10 to 30 %,
// FP64 E6 with psi doubles them.  Both fields of a step lie in the caches up to
// about 170^3, and beyond that its 48 B per site still stream faster than it
// computes.
// The search below runs over columns for a given number of planes per chunk
// (mom_columns) and over that number; the members of a batched launch share
// the chunk length, and their workgroups the rounds.
static constexpr double kWaveUs = 0.06;
static constexpr double kPlaneUs = 27, kFillPlanes = 3.5;  // in units of kWaveUs, in planes

// The fewest wavefront-planes per plane of the member: columns, largest first.
static MomShape mom_columns(const Member &m, int order, int rows) {
    const int r = order == 4 ? 1 : 2;
    MomShape best{};
    double best_cost = 1e300;
    for (int ntx = 1; ntx <= m.nx; ++ntx) {
        const int w = (m.nx + ntx - 1) / ntx;
        if (w < 8 && ntx > 1) break;
        if ((m.nx + w - 1) / w != ntx || w + 2 + 2 * r > MOM_PW) continue;
        int h = std::min({m.ny, MOM_EXT / (w + 2) - 2, rows - 2 - 2 * r});
        if (h < 1) continue;
        const int nty = (m.ny + h - 1) / h;
        h = (m.ny + nty - 1) / nty;
        const int waves = (2 * (w + 2) * (h + 2) + 63) / 64;
        const double cost = (double)ntx * nty * (kPlaneUs + waves);
        if (cost < best_cost) {
            best_cost = cost;
            best = MomShape{w, h, m.nz, ntx, nty, 1};
        }
    }
    return best;
}

static MomShape mom_shape(const Member &m, int order, int rows, int ncu, double *us) {
    const int r = order == 4 ? 1 : 2;
    MomShape best{};
    double best_cost = 1e300;
    for (int ntx = 1; ntx <= m.nx; ++ntx) {
        const int w = (m.nx + ntx - 1) / ntx;
        if (w < 8 && ntx > 1) break;
        if ((m.nx + w - 1) / w != ntx) continue;
        if (w + 2 + 2 * r > MOM_PW) continue;
        int h = std::min({m.ny, MOM_EXT / (w + 2) - 2, rows - 2 - 2 * r});
        if (h < 1) continue;
        const int nty = (m.ny + h - 1) / h;
        h = (m.ny + nty - 1) / nty;
        const int waves = (2 * (w + 2) * (h + 2) + 63) / 64;
        for (int nc = 1; nc <= m.nz; ++nc) {
            const int zc = (m.nz + nc - 1) / nc;
            if ((m.nz + zc - 1) / zc != nc) continue;
            const long blocks = (long)ntx * nty * nc;
            const double cost =
                (double)((blocks + ncu - 1) / ncu) * (zc + kFillPlanes) * (kPlaneUs + waves);
            if (cost < best_cost) {
                best_cost = cost;
                best = MomShape{w, h, zc, ntx, nty, nc};
            }
        }
    }
    *us = kWaveUs * best_cost;
    return best;
}

static MomKernel mom_kernel(const StepKey &k) {
    MomKernel f;
    if (k.dim != 3 || (k.order != 4 && k.order != 6) || k.sr) return f;
    auto go = [&](auto stv) {
        using ST = decltype(stv);
        f = k.order == 4 ? MomOps<ST, 4>::kernel(k) : MomOps<ST, 6>::kernel(k);
    };
    switch (k.storage) {
        case ST_F64: go(StoreF64{}); break;
        case ST_F32: go(StoreF32{}); break;
        case ST_F16: go(StoreF16{}); break;
        case ST_BF16: go(StoreBF16{}); break;
    }
    return f;
}

int compute_units() {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        ncu < 1)
        ncu = 256;
    return ncu;
}

// Threads of a workgroup: two lanes per node of the rimmed column; two passes
// load its ring plane.
static int mom_threads(const StepKey &k, const MomShape &g) {
    const int r2 = k.order == 4 ? 4 : 6;
    return (std::max(2 * (g.w + 2) * (g.h + 2), (g.w + r2) * (g.h + r2)) + 63) / 64 * 64;
}

bool node_mom_step(const StepKey &k, const Member &m, NodeLaunch *node, MomShape *shape,
                   double *us) {
    const MomKernel f = mom_kernel(k);
    if (!f.func) return false;
    *shape = mom_shape(m, k.order, f.rows, compute_units(), us);
    if (shape->w < 1) return false;
    node->func = f.func;
    node->grid = dim3(shape->ntx * shape->nty * shape->nchunks);
    node->block = dim3(mom_threads(k, *shape), 1, 1);
    node->shmem = 0;
    return true;
}

bool node_batch_mom_step(const StepKey &k, const std::vector<Member> &ms, int first_member,
                         NodeLaunch *node, MomList *list, double *us) {
    const MomKernel f = mom_kernel(k);
    if (!f.batch || ms.empty() || ms.size() > (size_t)MOM_LIST) return false;
    const int ncu = compute_units();
    std::vector<MomShape> g;
    int nzmax = 1, waves = 1;
    for (const Member &m : ms) {
        g.push_back(mom_columns(m, k.order, f.rows));
        if (g.back().w < 1) return false;
        nzmax = std::max(nzmax, m.nz);
        waves = std::max(waves, (2 * (g.back().w + 2) * (g.back().h + 2) + 63) / 64);
    }
    double best_cost = 1e300;
    int best = 1;
    for (int len = 1; len <= nzmax; ++len) {
        long blocks = 0;
        for (size_t i = 0; i < ms.size(); ++i)
            blocks += (long)g[i].ntx * g[i].nty * ((ms[i].nz + len - 1) / len);
        const double cost = (double)((blocks + ncu - 1) / ncu) * (len + kFillPlanes);
        if (cost < best_cost) {
            best_cost = cost;
            best = len;
        }
    }
    *us = kWaveUs * best_cost * (kPlaneUs + waves);
    list->n = (int)ms.size();
    int first = 0, threads = 64;
    for (size_t i = 0; i < ms.size(); ++i) {
        MomShape q = g[i];
        q.nchunks = (ms[i].nz + best - 1) / best;
        q.zc = (ms[i].nz + q.nchunks - 1) / q.nchunks;
        q.nchunks = (ms[i].nz + q.zc - 1) / q.zc;
        list->e[i] = MomList::Entry{first, first_member + (int)i, q};
        first += q.ntx * q.nty * q.nchunks;
        threads = std::max(threads, mom_threads(k, q));
    }
    node->func = f.batch;
    node->grid = dim3(first);
    node->block = dim3(threads, 1, 1);
    node->shmem = 0;
    return true;
}

}  // namespace scmc
