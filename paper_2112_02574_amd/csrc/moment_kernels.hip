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

// The launch shape: every node costs the collisions of its column's rim and
// of the chunk's two extra planes besides its own, and one workgroup runs per
// CU at a time.  The column sizes that a workgroup holds and the chunk counts
// are all weighed: rounds of workgroups over the CUs, times the planes a
// chunk marches (two more than it stores, and about two more for filling the
// ring), times the wavefronts of a plane.
static MomShape mom_shape(const Member &m, int order, int ncu) {
    const int r = order == 4 ? 1 : 2, pmax = r == 1 ? MomGeom<4>::PMAX : MomGeom<6>::PMAX;
    MomShape best{};
    double best_cost = 1e300;
    for (int ntx = 1; ntx <= m.nx; ++ntx) {
        const int w = (m.nx + ntx - 1) / ntx;
        if (w < 8 && ntx > 1) break;
        if ((m.nx + w - 1) / w != ntx) continue;
        int h = std::min(m.ny, MOM_EXT / (w + 2) - 2);
        while (h > 0 && (w + 2 + 2 * r) * (h + 2 + 2 * r) > pmax) --h;
        if (h < 1) continue;
        const int nty = (m.ny + h - 1) / h;
        h = (m.ny + nty - 1) / nty;
        const int waves = (2 * (w + 2) * (h + 2) + 63) / 64;
        for (int nc = 1; nc <= m.nz; ++nc) {
            const int zc = (m.nz + nc - 1) / nc;
            if ((m.nz + zc - 1) / zc != nc) continue;
            const long blocks = (long)ntx * nty * nc;
            const double cost =
                (double)((blocks + ncu - 1) / ncu) * (zc + 4) * std::max(waves, 4);
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
    void *f = nullptr;
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
    if (!f) return false;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        ncu < 1)
        ncu = 256;
    *shape = mom_shape(m, k.order, ncu);
    if (shape->w < 1) return false;
    node->func = f;
    node->grid = dim3(shape->ntx * shape->nty * shape->nchunks);
    node->block = dim3(MOM_THREADS, 1, 1);
    node->shmem = 0;
    return true;
}

}  // namespace scmc
