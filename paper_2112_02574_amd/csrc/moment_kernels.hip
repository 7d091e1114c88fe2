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
// orders measured shapes well (us per step, w x h x zc): 63^3 E4 FP32
// 32x11x3 19.0, 13x21x5 22.7, 16x21x6 27.6, 13x13x8 24.1; 128^3 E6 FP32
// 26x16x22 71, 32x13x13 (two rounds) 86, 19x16x32 80; 48^3 E6 FP32
// 24x10x2 11.6, 24x16x4 18.5.  Both fields of a step lie in the caches up to
// about 170^3, and beyond that its 48 B per site still stream faster than it
// computes.
static MomShape mom_shape(const Member &m, int order, int rows, int ncu) {
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
                (double)((blocks + ncu - 1) / ncu) * (zc + 3.5) * (27 + waves);
            if (cost < best_cost) {
                best_cost = cost;
                best = MomShape{w, h, zc, ntx, nty, nc};
            }
        }
    }
    return best;
}

bool node_mom_step(const StepKey &k, const Member &m, NodeLaunch *node, MomShape *shape) {
    if (k.dim != 3 || (k.order != 4 && k.order != 6) || k.sr) return false;
    MomKernel f;
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
    if (!f.func) return false;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        ncu < 1)
        ncu = 256;
    *shape = mom_shape(m, k.order, f.rows, ncu);
    if (shape->w < 1) return false;
    // two lanes per node of the rimmed column; two passes load its ring plane
    const int rim = (shape->w + 2) * (shape->h + 2), r2 = k.order == 4 ? 4 : 6;
    const int ring = (shape->w + r2) * (shape->h + r2);
    node->func = f.func;
    node->grid = dim3(shape->ntx * shape->nty * shape->nchunks);
    node->block = dim3((std::max(2 * rim, ring) + 63) / 64 * 64, 1, 1);
    node->shmem = 0;
    return true;
}

}  // namespace scmc
