// scmc_api.cpp -- host side of libscmc: validation, workspace planning,
// state transfer (with the pull-scheme index shift), launch sequencing,
// explicit hipGraph construction, and the FP64 post-processing of the
// pressure-tensor line (Sec. 3: closed-form minimum of sigma[R]).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <type_traits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/scmc.h"
#include "lattice.h"
#include "scmc_internal.h"
#include "step_rules.h"

using namespace scmc;

// ------------------------------------------------------------------ helpers
namespace {

constexpr size_t ALIGN = 256;
size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

int lattice_q(int lattice) { return lattice == SCMC_D2Q9 ? 9 : 19; }
int lattice_dim(int lattice) { return lattice == SCMC_D2Q9 ? 2 : 3; }
int stencil_radius(int st) { return st == SCMC_E4 ? 1 : 2; }
size_t storage_bytes(int st) {
    return st == SCMC_F64 ? 8 : st == SCMC_F32 ? 4 : 2;
}
bool node_storage(int st) { return st == SCMC_F16_NODE || st == SCMC_BF16_NODE; }
// kernel storage format of a public one (node storage keeps the 16-bit formats)
int storage_kind(int st) {
    return st == SCMC_F16_NODE ? ST_F16 : st == SCMC_BF16_NODE ? ST_BF16 : st;
}
// values per site of the density / moment field: (n_A, n_B), the momentum,
// the packed remainders and a spare; with node storage a second (n_A, n_B)
// slot (the two pair slots are the reference fields of the two buffers) and
// the FP32 rest populations
size_t field_values(int st) { return node_storage(st) ? 10 : 7; }
size_t real_bytes(int st) { return st == SCMC_F64 ? 8 : 4; }

void velocities(int lattice, int *xi, double *w) {
    if (lattice == SCMC_D2Q9) {
        using L = Lattice<2>;
        for (int i = 0; i < L::Q; ++i) {
            xi[3 * i] = L::CX[i];
            xi[3 * i + 1] = L::CY[i];
            xi[3 * i + 2] = L::CZ[i];
            w[i] = L::W[i];
        }
    } else {
        using L = Lattice<3>;
        for (int i = 0; i < L::Q; ++i) {
            xi[3 * i] = L::CX[i];
            xi[3 * i + 1] = L::CY[i];
            xi[3 * i + 2] = L::CZ[i];
            w[i] = L::W[i];
        }
    }
}

// IEEE binary16 round-to-nearest-even from binary32 (host).
uint16_t f32_to_f16_rne(float v) {
    uint32_t u;
    std::memcpy(&u, &v, 4);
    const uint32_t sign = (u >> 16) & 0x8000u;
    const uint32_t exp = (u >> 23) & 0xffu;
    uint32_t man = u & 0x7fffffu;
    if (exp == 0xff) return (uint16_t)(sign | 0x7c00u | (man ? 0x200u : 0u));
    int e = (int)exp - 127 + 15;
    if (e >= 31) return (uint16_t)(sign | 0x7c00u);
    if (e <= 0) {
        if (e < -10) return (uint16_t)sign;
        man |= 0x800000u;
        const int shift = 14 - e;
        uint32_t h = man >> shift;
        const uint32_t rem = man & ((1u << shift) - 1);
        const uint32_t half = 1u << (shift - 1);
        if (rem > half || (rem == half && (h & 1u))) ++h;
        return (uint16_t)(sign | h);
    }
    uint32_t h = ((uint32_t)e << 10) | (man >> 13);
    const uint32_t rem = man & 0x1fffu;
    if (rem > 0x1000u || (rem == 0x1000u && (h & 1u))) ++h;  // may carry
    return (uint16_t)(sign | h);
}

float f16_to_f32(uint16_t h) {
    const uint32_t sign = (uint32_t)(h & 0x8000u) << 16;
    const uint32_t exp = (h >> 10) & 0x1fu;
    uint32_t man = h & 0x3ffu;
    uint32_t u;
    if (exp == 0) {
        if (man == 0) {
            u = sign;
        } else {
            int e = -1;
            do {
                man <<= 1;
                ++e;
            } while (!(man & 0x400u));
            u = sign | ((uint32_t)(127 - 15 - e) << 23) | ((man & 0x3ffu) << 13);
        }
    } else if (exp == 31) {
        u = sign | 0x7f800000u | (man << 13);
    } else {
        u = sign | ((exp - 15 + 127) << 23) | (man << 13);
    }
    float v;
    std::memcpy(&v, &u, 4);
    return v;
}

// the single-precision offset reference used by the FP16 / BF16 formats
float offset_ref(double w, double n0) { return (float)w * (float)n0; }

// Node storage on the host, rounded as the kernels round: the reference
// w_i n_J and the decoded value are single-precision operations of their
// own (no fused multiply-add).
float node_ref_host(double w, float n) {
#pragma clang fp contract(off)
    const float wf = (float)w;
    return wf * n;
}
// FP16 node offsets are stored scaled by 2^10 (exact), as the kernels do
uint16_t node_encode(int storage, double v, float ref) {
#pragma clang fp contract(off)
    const float h = (float)v - ref;
    return storage == SCMC_F16_NODE ? f32_to_f16_rne(h * 1024.0f) : f32_to_bf16_rne(h);
}
double node_decode(int storage, uint16_t h, float ref) {
#pragma clang fp contract(off)
    const float x = storage == SCMC_F16_NODE ? f16_to_f32(h) * (1.0f / 1024.0f) : bf16_to_f32(h);
    const float d = x + ref;
    return (double)d;
}

void encode(int storage, double v, double w, double n0, void *dst, size_t i) {
    switch (storage) {
        case SCMC_F64: ((double *)dst)[i] = v; break;
        case SCMC_F32: ((float *)dst)[i] = (float)v; break;
        case SCMC_F16_OFF:
            ((uint16_t *)dst)[i] =
                f32_to_f16_rne((float)v - offset_ref(w, n0));
            break;
        default:
            ((uint16_t *)dst)[i] =
                f32_to_bf16_rne((float)v - offset_ref(w, n0));
            break;
    }
}

double decode(int storage, const void *src, size_t i, double w, double n0) {
    switch (storage) {
        case SCMC_F64: return ((const double *)src)[i];
        case SCMC_F32: return ((const float *)src)[i];
        case SCMC_F16_OFF:
            return (double)f16_to_f32(((const uint16_t *)src)[i]) +
                   (double)offset_ref(w, n0);
        default:
            return (double)bf16_to_f32(((const uint16_t *)src)[i]) +
                   (double)offset_ref(w, n0);
    }
}

}  // namespace

// ------------------------------------------------------------ shared state
struct Lat {
    scmc_problem p;
    Member m;
    int q, dim;
};

struct Common {
    StepKey key{};
    int kernel = SCMC_KERNEL_TWO_PASS;
    int tile[3] = {0, 0, 0};
    hipStream_t stream = nullptr;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    void *pop[2] = {nullptr, nullptr};
    void *dens = nullptr;
    double *dens64 = nullptr;
    double *vel64 = nullptr;
    double *velprev = nullptr;  // velocity field of the previous convergence check
    double *partials = nullptr;
    double *small = nullptr;  // stats / line / flat outputs
    unsigned *ctr = nullptr;  // step counter of the stochastic rounding
    unsigned ctr_host = 0;
    int nblocks = 0;
    int cur = 0;
    int64_t step = 0;
    bool initialized = false;
    int graph_k = 0;
    hipGraphExec_t gexec[2] = {nullptr, nullptr};
    std::string err;
};

struct scmc_sim {
    Common c;
    Lat lat;
    bool mom_ok = false;  // blocks of steps can stay in the moment field
    NodeLaunch mom_node{};
    MomShape mom_shape{};
    double mom_us = 0;  // D3Q19: a step's time by the launch model
    int mom2 = 0;  // D2Q9: the most steps that a launch of mom_node makes
    bool have_prev = false;  // convergence monitor: a previous check exists
    double prev_dP = 0;
    int64_t prev_step = 0;
};

// One launch of the batched two-pass: pass 1 or 2 over tiles [t0, t0 + n),
// one workgroup per tile; nt_all: pass 1 with every load non-temporal.
// member >= 0: the chunk is that member alone, launched like a single
// lattice (node_member_pass, with m its description) instead.
struct BatchOp {
    int pass, t0, n;
    bool nt_all = false;
    int member = -1;
    Member m{};
};

// Ops [op0, op1) of consecutive members (from `member` on), which advance a
// block of steps before the next group starts.  mom: the steps between the
// first pass 1 and the last pass 2 can stay in the moment field; they do where
// that pays (mom_steps_pay).
struct BatchGroup {
    size_t op0 = 0, op1 = 0;
    int member = 0;
    bool mom = false;
    int64_t sites = 0, ragged = 0;
    double us = 0;
    struct Launch {  // of up to MOM_LIST members; a moment step makes them all
        NodeLaunch node{};
        MomList list{};
    };
    std::vector<Launch> launches;
};

struct scmc_batch {
    Common c;
    std::vector<Lat> lats;
    Member *d_members = nullptr;
    Tile *d_tiles = nullptr;
    int ntiles = 0;
    int ntiles_cap = 0;  // tile-list capacity planned in the workspace
    int grid = 0;
    std::vector<bool> member_set;
    // The launches of one two-pass step (batch_set_ops); empty for the fused
    // designs, which run the whole list in one persistent launch.
    std::vector<BatchOp> ops;
    std::vector<BatchGroup> groups;  // runs of ops that step together
};

namespace {

int fail(Common &c, int status, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    c.err = buf;
    return status;
}

#define HIPCHK(c, expr)                                                      \
    do {                                                                     \
        hipError_t e_ = (expr);                                              \
        if (e_ != hipSuccess)                                                \
            return fail((c), SCMC_EDEVICE, "%s: %s", #expr,                  \
                        hipGetErrorString(e_));                              \
    } while (0)

// The tau = 1 designs need both relaxation times equal to one.
static bool tau_is_one(const scmc_problem &p) { return p.tau[0] == 1.0 && p.tau[1] == 1.0; }

int validate(const scmc_problem *p, std::string *why) {
    char buf[256];
    auto bad = [&](int st, const char *msg) {
        if (why) *why = msg;
        return st;
    };
    if (!p) return bad(SCMC_EINVAL, "problem is NULL");
    if (p->lattice != SCMC_D2Q9 && p->lattice != SCMC_D3Q19)
        return bad(SCMC_EINVAL, "unknown lattice");
    if (p->stencil != SCMC_E4 && p->stencil != SCMC_E6 && p->stencil != SCMC_E8)
        return bad(SCMC_EINVAL, "unknown stencil");
    if (p->lattice == SCMC_D3Q19 && p->stencil == SCMC_E8)
        return bad(SCMC_EUNSUPPORTED, "E8 stencil is 2D only");
    if (p->storage < SCMC_F64 || p->storage > SCMC_BF16_NODE)
        return bad(SCMC_EINVAL, "unknown storage");
    if (p->psi_self != SCMC_PSI_N && p->psi_self != SCMC_PSI_EXP_NEG_INV)
        return bad(SCMC_EINVAL, "unknown psi");
    if (p->kernel < SCMC_KERNEL_AUTO || p->kernel > SCMC_KERNEL_TWO_PASS_MOM)
        return bad(SCMC_EINVAL, "unknown kernel design");
    const int r = stencil_radius(p->stencil);
    if (p->lattice == SCMC_D2Q9 && p->nz != 1)
        return bad(SCMC_EINVAL, "nz must be 1 for D2Q9");
    const int ext[3] = {p->nx, p->ny, p->nz};
    for (int a = 0; a < (p->lattice == SCMC_D2Q9 ? 2 : 3); ++a)
        if (ext[a] < 2 * r + 1) {
            snprintf(buf, sizeof buf, "extent %d smaller than 2 r_F + 1 = %d",
                     ext[a], 2 * r + 1);
            if (why) *why = buf;
            return SCMC_EINVAL;
        }
    if ((double)p->nx * p->ny * p->nz * 2 * lattice_q(p->lattice) > 2.0e9)
        return bad(SCMC_EINVAL, "lattice too large for 32-bit plane indexing");
    for (int J = 0; J < 2; ++J)
        if (!std::isfinite(p->tau[J]) || !(p->tau[J] > 0.5))
            return bad(SCMC_EINVAL, "tau must be finite and > 1/2");
    if ((p->kernel == SCMC_KERNEL_FUSED_MOM || p->kernel == SCMC_KERNEL_FUSED_MOM_PIPE ||
         p->kernel == SCMC_KERNEL_TWO_PASS_MOM) &&
        !tau_is_one(*p))
        return bad(SCMC_EUNSUPPORTED, "the moment-ring designs need tau_A = tau_B = 1");
    for (int J = 0; J < 2; ++J)
        for (int K = 0; K < 2; ++K)
            if (!std::isfinite(p->g[J][K])) return bad(SCMC_EINVAL, "non-finite coupling");
    if (p->g[0][1] != p->g[1][0]) return bad(SCMC_EINVAL, "g_AB != g_BA");
    if (!std::isfinite(p->n0[0]) || !std::isfinite(p->n0[1]))
        return bad(SCMC_EINVAL, "non-finite n0");
    if (p->rounding != SCMC_ROUND_NEAREST && p->rounding != SCMC_ROUND_STOCHASTIC)
        return bad(SCMC_EINVAL, "unknown rounding");
    if (node_storage(p->storage)) {
        if (p->lattice != SCMC_D3Q19)
            return bad(SCMC_EUNSUPPORTED, "node storage runs on D3Q19");
        if (!tau_is_one(*p) ||
            (p->kernel != SCMC_KERNEL_AUTO && p->kernel != SCMC_KERNEL_TWO_PASS_MOM))
            return bad(SCMC_EUNSUPPORTED,
                       "node storage runs in the moment two-pass (tau_A = tau_B = 1)");
        if (p->rounding != SCMC_ROUND_NEAREST)
            return bad(SCMC_EUNSUPPORTED, "node storage rounds to nearest");
        if ((double)lattice_q(p->lattice) * p->nx * p->ny * p->nz * storage_bytes(p->storage) >=
            2147483648.0)
            return bad(SCMC_EUNSUPPORTED, "node storage needs 32-bit buffer offsets");
    }
    if (p->rounding == SCMC_ROUND_STOCHASTIC) {
        if (p->storage != SCMC_F16_OFF && p->storage != SCMC_BF16_OFF)
            return bad(SCMC_EINVAL, "stochastic rounding needs FP16 / BF16 offset storage");
        if (p->kernel != SCMC_KERNEL_AUTO && p->kernel != SCMC_KERNEL_TWO_PASS &&
            p->kernel != SCMC_KERNEL_TWO_PASS_MOM)
            return bad(SCMC_EUNSUPPORTED, "stochastic rounding runs in the two-pass designs");
    }
    return SCMC_OK;
}

StepKey key_of(const scmc_problem &p) {
    StepKey k;
    k.dim = lattice_dim(p.lattice);
    k.order = p.stencil;
    k.storage = storage_kind(p.storage);
    k.node = node_storage(p.storage) ? 1 : 0;
    k.sr = p.rounding == SCMC_ROUND_STOCHASTIC ? 1 : 0;
    k.psi = p.psi_self;
    switch (p.kernel) {
        case SCMC_KERNEL_FUSED_REPULL: k.repull = 1; break;
        case SCMC_KERNEL_FUSED_PIPE: k.repull = 2; break;
        case SCMC_KERNEL_FUSED_MOM: k.repull = 3; break;
        case SCMC_KERNEL_FUSED_MOM_PIPE: k.repull = 4; break;
        case SCMC_KERNEL_AUTO: k.repull = tau_is_one(p) ? 3 : 0; break;
        default: k.repull = 0;
    }
    k.mom = tau_is_one(p) && (p.kernel == SCMC_KERNEL_TWO_PASS_MOM ||
                                p.kernel == SCMC_KERNEL_AUTO);
    // TWO_PASS_MOM with a tile asks for the LDS-staged collision pass (its
    // shape is fixed at 64 x 8 columns and z-chunks of 8)
    if (p.kernel == SCMC_KERNEL_TWO_PASS_MOM && p.tile[0] != 0 && p.lattice == SCMC_D3Q19 &&
        p.storage != SCMC_F64)
        k.mom = 2;
    // node storage has no fused design: AUTO always means the moment two-pass
    if (k.node && p.kernel == SCMC_KERNEL_AUTO) k.mom = 1;
    k.big = (double)lattice_q(p.lattice) * p.nx * p.ny * p.nz * storage_bytes(p.storage) >=
            2147483648.0;
    return k;
}

Member member_of(const scmc_problem &p) {
    Member m{};
    m.nx = p.nx;
    m.ny = p.ny;
    m.nz = p.nz;
    m.znum = p.nz;
    m.N = p.nx * p.ny * p.nz;
    m.pop_off = 0;
    m.dens_off = 0;
    for (int J = 0; J < 2; ++J)
        for (int K = 0; K < 2; ++K) m.g[J][K] = p.g[J][K];
    m.omega[0] = 1.0 / p.tau[0];
    m.omega[1] = 1.0 / p.tau[1];
    m.n0[0] = p.n0[0];
    m.n0[1] = p.n0[1];
    m.psi_self = p.psi_self;
    m.self_on = (p.g[0][0] != 0.0 ? 1 : 0) | (p.g[1][1] != 0.0 ? 2 : 0);
    m.sr = p.rounding == SCMC_ROUND_STOCHASTIC;
    m.seed = p.seed;
    m.step_ctr = nullptr;  // bound to the workspace's counter by the handle
    m.ref = nullptr;       // node storage: set per launch (step_member)
    m.pair_slot = 0;
    m.rest = nullptr;
    return m;
}

// resolve the kernel design and the fused tile; own_field: the moment /
// density field belongs to the handle, and no other call writes it
int choose_kernel(const scmc_problem &p, const StepKey &k, int *kernel,
                  int *tile, bool own_field = true) {
    int t[3] = {p.tile[0], p.tile[1], p.tile[2]};
    // the default is the moment two-pass design at tau = 1 and the any-tau two
    // passes otherwise, the fastest untuned choices: us per step at tau = 0.8,
    // E6, against the fused design's default tile (64, 8, 16), 64^3 FP32 25
    // against 120, 128^3 FP32 192 against 203, FP16 101 against 133,
    // 160 x 150 x 155 FP32 345 against 591.  The autotuner may pick a fused one
    // (128^3 FP32 with (128, 4, 16): 181).  Batches, two passes on records chunk by
    // chunk against fused: twelve members of 16^3 E6 FP32 11 against 83, of 48^3 to
    // 88^3 376 against 567; where the fused tiles fit the members exactly, 24 of
    // 64^3 E6 FP16 351 against 367, E4 with psi FP32 593 against 594, BF16 432
    // against 422, two of 128^3 E4 with psi FP32 390 against 430.  The
    // allocation-free step's field is one array per GPU: there AUTO takes the
    // fused design at tau != 1, which needs no field, so that calls on several
    // streams share no memory.
    if (k.node || p.kernel == SCMC_KERNEL_TWO_PASS || p.kernel == SCMC_KERNEL_TWO_PASS_MOM ||
        (p.kernel == SCMC_KERNEL_AUTO && t[0] == 0 && (own_field || k.mom)) ||
        (p.kernel == SCMC_KERNEL_AUTO && p.rounding == SCMC_ROUND_STOCHASTIC)) {
        *kernel = SCMC_KERNEL_TWO_PASS;
        const bool lds = k.mom == 2;
        tile[0] = lds ? 64 : 0;
        tile[1] = lds ? 8 : 0;
        tile[2] = lds ? 8 : 0;
        return SCMC_OK;
    }
    if (t[0] == 0) {  // default fused tile (fits every compiled design)
        t[0] = 64;
        t[1] = 8;
        t[2] = 16;
    }
    if (fused_supported(k, t)) {
        *kernel = SCMC_KERNEL_FUSED;
        for (int a = 0; a < 3; ++a) tile[a] = t[a];
        return SCMC_OK;
    }
    if (p.kernel != SCMC_KERNEL_AUTO) return SCMC_EUNSUPPORTED;
    *kernel = SCMC_KERNEL_TWO_PASS;
    tile[0] = tile[1] = tile[2] = 0;
    return SCMC_OK;
}

// scmc_kernel value of a resolved design
int public_kernel(int kernel, int variant, int mom) {
    if (kernel == SCMC_KERNEL_TWO_PASS && mom) return SCMC_KERNEL_TWO_PASS_MOM;
    if (kernel != SCMC_KERNEL_FUSED) return kernel;
    static const int of[] = {SCMC_KERNEL_FUSED, SCMC_KERNEL_FUSED_REPULL,
                             SCMC_KERNEL_FUSED_PIPE, SCMC_KERNEL_FUSED_MOM,
                             SCMC_KERNEL_FUSED_MOM_PIPE};
    return of[variant];
}

struct Plan {
    size_t pop, dens, dens64, vel64, velprev, partials, small, ctr, members, tiles, total;
};

Plan plan_of(const std::vector<scmc_problem> &ps, int ntiles) {
    Plan pl{};
    size_t pop = 0, dens = 0, nmax = 0, nxmax = 0;
    int nb = 0;
    for (const auto &p : ps) {
        const size_t N = (size_t)p.nx * p.ny * p.nz;
        pop += align_up(2 * (size_t)lattice_q(p.lattice) * N *
                        storage_bytes(p.storage));
        dens += align_up(field_values(p.storage) * N * real_bytes(p.storage));
        nmax = std::max(nmax, N);
        nxmax = std::max(nxmax, (size_t)p.nx);
        nb = std::max(nb, stats_blocks(member_of(p)));
    }
    pl.pop = pop;
    pl.dens = dens;
    pl.dens64 = align_up(2 * nmax * 8);
    pl.vel64 = align_up(3 * nmax * 8);
    pl.velprev = ps.size() == 1 ? align_up(3 * nmax * 8) : 0;
    pl.partials = align_up((size_t)nb * 9 * 8);
    pl.small = align_up((3 * (nxmax / 2 + 1) + 3 + 2 * nxmax + 1 + 16) * 8);
    pl.ctr = align_up(sizeof(unsigned));
    pl.members = ps.size() > 1 ? align_up(ps.size() * sizeof(Member)) : 0;
    pl.tiles = ntiles > 0 ? align_up((size_t)ntiles * sizeof(Tile)) : 0;
    pl.total = 2 * pl.pop + pl.dens + pl.dens64 + pl.vel64 + pl.velprev + pl.partials +
               pl.small + pl.ctr + pl.members + pl.tiles;
    return pl;
}

void bind(Common &c, const Plan &pl, char *ws, int nblocks) {
    char *p = ws;
    c.pop[0] = p;
    p += pl.pop;
    c.pop[1] = p;
    p += pl.pop;
    c.dens = p;
    p += pl.dens;
    c.dens64 = (double *)p;
    p += pl.dens64;
    c.vel64 = (double *)p;
    p += pl.vel64;
    c.velprev = pl.velprev ? (double *)p : nullptr;
    p += pl.velprev;
    c.partials = (double *)p;
    p += pl.partials;
    c.small = (double *)p;
    p += pl.small;
    c.ctr = (unsigned *)p;
    p += pl.ctr;
    c.nblocks = nblocks;
}

void drop_graphs(Common &c) {
    for (int k = 0; k < 2; ++k)
        if (c.gexec[k]) {
            (void)hipGraphExecDestroy(c.gexec[k]);
            c.gexec[k] = nullptr;
        }
}

// ---- node storage: reference fields --------------------------------------
// The moment field of a node-storage lattice holds two (n_A, n_B) pair slots,
// at values 0 and 6N: slot b is the reference field of population buffer b,
// the densities its offsets are taken from.  Pass 1 of a step from buffer cur
// decodes against slot cur and writes the new densities into slot 1 - cur,
// against which pass 2 encodes buffer 1 - cur.
// The rest populations (f*_0^A, f*_0^B) follow as FP32 pairs at values 8N.
int pair_slot_of(int buf) { return buf ? 6 : 0; }
constexpr int kRestSlot = 8;
float *ref_field(const Common &c, const Lat &L, int buf) {
    return (float *)c.dens + (size_t)pair_slot_of(buf) * L.m.N;
}
float *rest_field(const Common &c, int N) { return (float *)c.dens + (size_t)kRestSlot * N; }
// the member as a step from buffer cur launches it (single lattice)
Member step_member(const Common &c, Member m, int cur) {
    if (c.key.node) {
        m.ref = (const float2 *)((const float *)c.dens + (size_t)pair_slot_of(cur) * m.N);
        m.pair_slot = pair_slot_of(1 - cur);
        m.rest = (float2 *)rest_field(c, m.N);
    }
    return m;
}

// ---- state transfer (single lattice member) ----------------------------
// the device buffer holds g_i(x) = f_i(x + xi_i): the post-collision values
// that the next step pulls
int upload_state(Common &c, const Lat &L, const double *f, void *dst_dev) {
    const scmc_problem &p = L.p;
    const int q = L.q;
    const size_t N = (size_t)L.m.N;
    int xi[57];
    double w[19];
    velocities(p.lattice, xi, w);
    const size_t sb = storage_bytes(p.storage);
    std::vector<unsigned char> host(2 * q * N * sb);
    if (node_storage(p.storage)) {
        // the buffer value at node y is f*_i(y) = f_i(y + xi_i); its reference
        // is the density of the node it streams to, y + xi_i, with the
        // post-collision density sum_k f*_k of a node (BGK conserves the
        // node's mass, so this is n_J of the step that produced it)
        std::vector<double> nref(2 * N, 0.0);
        std::vector<float> ref(2 * N);
        auto src_of = [&](int i, int z, int y, int x) {
            const int zs = (z + xi[3 * i + 2] + p.nz) % p.nz;
            const int ys = (y + xi[3 * i + 1] + p.ny) % p.ny;
            const int xs = (x + xi[3 * i] + p.nx) % p.nx;
            return ((size_t)zs * p.ny + ys) * p.nx + xs;
        };
        for (int J = 0; J < 2; ++J)
            for (int i = 0; i < q; ++i)
                for (int z = 0; z < p.nz; ++z)
                    for (int y = 0; y < p.ny; ++y)
                        for (int x = 0; x < p.nx; ++x)
                            nref[J * N + ((size_t)z * p.ny + y) * p.nx + x] +=
                                f[((size_t)J * q + i) * N + src_of(i, z, y, x)];
        for (size_t t = 0; t < 2 * N; ++t) ref[t] = (float)nref[t];
        uint16_t *h = (uint16_t *)host.data();
        for (int J = 0; J < 2; ++J)
            for (int i = 1; i < q; ++i)
                for (int z = 0; z < p.nz; ++z)
                    for (int y = 0; y < p.ny; ++y)
                        for (int x = 0; x < p.nx; ++x) {
                            const size_t t = ((size_t)z * p.ny + y) * p.nx + x;
                            const size_t d = src_of(i, z, y, x);  // y + xi_i
                            const double v = f[((size_t)J * q + i) * N + d];
                            h[((size_t)J * q + i) * N + t] =
                                node_encode(p.storage, v, node_ref_host(w[i], ref[J * N + d]));
                        }
        // reference field of buffer 0, as (n_A, n_B) pairs per node, and the
        // FP32 rest populations (the i = 0 planes of the buffer are unused)
        std::vector<float> pairs(2 * N), rest(2 * N);
        for (size_t t = 0; t < N; ++t) {
            pairs[2 * t] = ref[t];
            pairs[2 * t + 1] = ref[N + t];
            rest[2 * t] = (float)f[t];
            rest[2 * t + 1] = (float)f[(size_t)q * N + t];
        }
        if (dst_dev != c.pop[0])
            return fail(c, SCMC_EUNSUPPORTED, "node storage uploads into buffer 0 only");
        HIPCHK(c, hipMemcpyAsync(ref_field(c, L, 0), pairs.data(), pairs.size() * 4,
                                 hipMemcpyHostToDevice, c.stream));
        HIPCHK(c, hipMemcpyAsync(rest_field(c, L.m.N), rest.data(), rest.size() * 4,
                                 hipMemcpyHostToDevice, c.stream));
        HIPCHK(c, hipMemcpyAsync(dst_dev, host.data(), host.size(), hipMemcpyHostToDevice,
                                 c.stream));
        HIPCHK(c, hipStreamSynchronize(c.stream));
        return SCMC_OK;
    }
    for (int J = 0; J < 2; ++J)
        for (int i = 0; i < q; ++i) {
            const double *src = f + ((size_t)J * q + i) * N;
            const size_t base = ((size_t)J * q + i) * N;
            for (int z = 0; z < p.nz; ++z)
                for (int y = 0; y < p.ny; ++y) {
                    const int zs = (z + xi[3 * i + 2] + p.nz) % p.nz;
                    const int ys = (y + xi[3 * i + 1] + p.ny) % p.ny;
                    for (int x = 0; x < p.nx; ++x) {
                        const int xs = (x + xi[3 * i] + p.nx) % p.nx;
                        const double v =
                            src[((size_t)zs * p.ny + ys) * p.nx + xs];
                        encode(p.storage, v, w[i], p.n0[J], host.data(),
                               base + ((size_t)z * p.ny + y) * p.nx + x);
                    }
                }
        }
    HIPCHK(c, hipMemcpyAsync(dst_dev, host.data(), host.size(),
                             hipMemcpyHostToDevice, c.stream));
    HIPCHK(c, hipStreamSynchronize(c.stream));
    return SCMC_OK;
}

// Counter seeding the stochastic rounding: the number of steps taken.
int set_step_counter(Common &c, int64_t step) {
    c.ctr_host = (unsigned)step;
    HIPCHK(c, hipMemcpyAsync(c.ctr, &c.ctr_host, sizeof(unsigned),
                             hipMemcpyHostToDevice, c.stream));
    HIPCHK(c, hipStreamSynchronize(c.stream));
    return SCMC_OK;
}

int download_state(Common &c, const Lat &L, const void *src_dev, double *f) {
    const scmc_problem &p = L.p;
    const int q = L.q;
    const size_t N = (size_t)L.m.N;
    int xi[57];
    double w[19];
    velocities(p.lattice, xi, w);
    const size_t sb = storage_bytes(p.storage);
    std::vector<unsigned char> host(2 * q * N * sb);
    HIPCHK(c, hipMemcpyAsync(host.data(), src_dev, host.size(),
                             hipMemcpyDeviceToHost, c.stream));
    std::vector<float> pairs, rest;
    if (node_storage(p.storage)) {
        pairs.resize(2 * N);
        rest.resize(2 * N);
        const int buf = src_dev == c.pop[1] ? 1 : 0;
        HIPCHK(c, hipMemcpyAsync(pairs.data(), ref_field(c, L, buf), pairs.size() * 4,
                                 hipMemcpyDeviceToHost, c.stream));
        HIPCHK(c, hipMemcpyAsync(rest.data(), rest_field(c, L.m.N), rest.size() * 4,
                                 hipMemcpyDeviceToHost, c.stream));
    }
    HIPCHK(c, hipStreamSynchronize(c.stream));
    if (node_storage(p.storage)) {
        const uint16_t *h = (const uint16_t *)host.data();
        for (size_t t = 0; t < N; ++t) {
            f[t] = (double)rest[2 * t];
            f[(size_t)q * N + t] = (double)rest[2 * t + 1];
        }
        for (int J = 0; J < 2; ++J)
            for (int i = 1; i < q; ++i)
                for (int z = 0; z < p.nz; ++z)
                    for (int y = 0; y < p.ny; ++y) {
                        const int zs = (z - xi[3 * i + 2] + p.nz) % p.nz;
                        const int ys = (y - xi[3 * i + 1] + p.ny) % p.ny;
                        for (int x = 0; x < p.nx; ++x) {
                            const int xs = (x - xi[3 * i] + p.nx) % p.nx;
                            const size_t t = ((size_t)zs * p.ny + ys) * p.nx + xs;
                            const size_t d = ((size_t)z * p.ny + y) * p.nx + x;
                            // decoded against the densities of the pulling node
                            f[((size_t)J * q + i) * N + d] =
                                node_decode(p.storage, h[((size_t)J * q + i) * N + t],
                                            node_ref_host(w[i], pairs[2 * d + J]));
                        }
                    }
        return SCMC_OK;
    }
    for (int J = 0; J < 2; ++J)
        for (int i = 0; i < q; ++i) {
            double *dst = f + ((size_t)J * q + i) * N;
            const size_t base = ((size_t)J * q + i) * N;
            for (int z = 0; z < p.nz; ++z)
                for (int y = 0; y < p.ny; ++y) {
                    const int zs = (z - xi[3 * i + 2] + p.nz) % p.nz;
                    const int ys = (y - xi[3 * i + 1] + p.ny) % p.ny;
                    for (int x = 0; x < p.nx; ++x) {
                        const int xs = (x - xi[3 * i] + p.nx) % p.nx;
                        dst[((size_t)z * p.ny + y) * p.nx + x] = decode(
                            p.storage, host.data(),
                            base + ((size_t)zs * p.ny + ys) * p.nx + xs, w[i],
                            p.n0[J]);
                    }
                }
        }
    return SCMC_OK;
}

int set_density_impl(Common &c, const Lat &L, const double *nA,
                     const double *nB, void *dst_dev) {
    const size_t N = (size_t)L.m.N;
    const int q = L.q;
    int xi[57];
    double w[19];
    velocities(L.p.lattice, xi, w);
    for (size_t s = 0; s < N; ++s)
        if (!std::isfinite(nA[s]) || !std::isfinite(nB[s]))
            return fail(c, SCMC_EINVAL, "non-finite density at site %zu", s);
    std::vector<double> f(2 * q * N);
    for (int i = 0; i < q; ++i)
        for (size_t s = 0; s < N; ++s) {
            f[(size_t)i * N + s] = w[i] * nA[s];
            f[((size_t)q + i) * N + s] = w[i] * nB[s];
        }
    return upload_state(c, L, f.data(), dst_dev);
}

// ---- observables of one member (its populations at pop_dev) ------------
// The observable kernels get the member's own population pointer (already
// offset) and a per-call FP64 scratch, so their Member view carries no
// offsets.
Member obs_member(const Common &c, const Lat &L, const void *pop_dev) {
    Member m = L.m;
    m.pop_off = 0;
    m.dens_off = 0;
    if (c.key.node) {
        m.ref = (const float2 *)ref_field(c, L, pop_dev == c.pop[1] ? 1 : 0);
        m.rest = (float2 *)rest_field(c, L.m.N);
    }
    return m;
}

int member_obs_prep(Common &c, const Lat &L, const void *pop_dev) {
    HIPCHK(c, launch_density64(c.key, obs_member(c, L, pop_dev), pop_dev, c.dens64,
                               c.stream));
    return SCMC_OK;
}

int stats_impl(Common &c, const Lat &L, const void *pop_base, scmc_stats *out,
               int64_t step) {
    if (!out) return fail(c, SCMC_EINVAL, "out is NULL");
    const Member m = obs_member(c, L, pop_base);
    int rc = member_obs_prep(c, L, pop_base);
    if (rc) return rc;
    HIPCHK(c, launch_stats(c.key, m, pop_base, c.dens64, c.partials,
                           c.nblocks, c.small, c.stream));
    double h[9];
    HIPCHK(c, hipMemcpyAsync(h, c.small, sizeof h, hipMemcpyDeviceToHost,
                             c.stream));
    HIPCHK(c, hipStreamSynchronize(c.stream));
    out->mass[0] = h[0];
    out->mass[1] = h[1];
    out->momentum[0] = h[2];
    out->momentum[1] = h[3];
    out->momentum[2] = h[4];
    out->min_n[0] = h[5];
    out->min_n[1] = h[6];
    out->max_u = h[7];
    out->n_nonfinite = h[8];
    out->step = step;
    return SCMC_OK;
}

int fields_impl(Common &c, const Lat &L, const void *pop_base, double *nA,
                double *nB, double *u) {
    const Member m = obs_member(c, L, pop_base);
    const size_t N = (size_t)m.N;
    int rc = member_obs_prep(c, L, pop_base);
    if (rc) return rc;
    const bool both = nA && nB == nA + N;  // one array: one copy
    if (nA)
        HIPCHK(c, hipMemcpyAsync(nA, c.dens64, (both ? 2 : 1) * N * 8, hipMemcpyDeviceToHost,
                                 c.stream));
    if (nB && !both)
        HIPCHK(c, hipMemcpyAsync(nB, c.dens64 + N, N * 8,
                                 hipMemcpyDeviceToHost, c.stream));
    if (u) {
        HIPCHK(c, launch_velocity64(c.key, m, pop_base, c.dens64, c.vel64,
                                    c.stream));
        HIPCHK(c, hipMemcpyAsync(u, c.vel64, 3 * N * 8, hipMemcpyDeviceToHost,
                                 c.stream));
    }
    HIPCHK(c, hipStreamSynchronize(c.stream));
    return SCMC_OK;
}

// sigma[R] = C_d / R^(d-1) + dP R / d (the Heaviside part of eq. gen_sigma
// integrated exactly) from the probes and C_d of a P_T profile; minimum at
// R_s = (d (d-1) C_d / dP)^(1/d), and the grid scan on [R0/2, 2 R0].
void droplet_sigma(int d, double Pin, double Pout, double Cd, double R0, scmc_obs *out) {
    const double dP = Pin - Pout;
    out->P_in = Pin;
    out->P_out = Pout;
    out->dP = dP;
    out->C_d = Cd;
    out->R_s = std::pow(d * (d - 1) * Cd / dP, 1.0 / d);
    out->sigma_s = dP * out->R_s / (d - 1);
    const int nR = (int)std::floor((2.0 * R0 - 0.5 * R0) / 0.01) + 1;
    std::vector<double> sg(nR);
    int kb = 0;
    for (int k = 0; k < nR; ++k) {
        const double R = 0.5 * R0 + 0.01 * k;
        sg[k] = Cd / std::pow(R, d - 1) + dP * R / d;
        if (sg[k] < sg[kb]) kb = k;
    }
    double Rg = 0.5 * R0 + 0.01 * kb;
    if (kb > 0 && kb < nR - 1) {
        const double den = sg[kb - 1] - 2 * sg[kb] + sg[kb + 1];
        if (den != 0) Rg += 0.01 * 0.5 * (sg[kb - 1] - sg[kb + 1]) / den;
    }
    out->R_s_grid = Rg;
}

int obs_impl(Common &c, const Lat &L, const void *pop_base, int kind, double R0,
             scmc_obs *out, double *PN, double *PT, int64_t step) {
    if (!out) return fail(c, SCMC_EINVAL, "out is NULL");
    if (kind != SCMC_OBS_FLAT && kind != SCMC_OBS_DROPLET && kind != SCMC_OBS_SHELL)
        return fail(c, SCMC_EINVAL, "unknown observable kind %d", kind);
    const Member m = obs_member(c, L, pop_base);
    const int d = L.dim;
    std::memset(out, 0, sizeof *out);
    out->step = step;
    int rc = member_obs_prep(c, L, pop_base);
    if (rc) return rc;
    if (kind == SCMC_OBS_FLAT) {
        const int nx = m.nx;
        std::vector<double> h(2 * nx + 1);
        HIPCHK(c, launch_flat(c.key, m, c.dens64, c.small, c.stream));
        HIPCHK(c, hipMemcpyAsync(h.data(), c.small, h.size() * 8,
                                 hipMemcpyDeviceToHost, c.stream));
        HIPCHK(c, hipStreamSynchronize(c.stream));
        out->sigma0 = h[2 * nx];
        if (PN) std::memcpy(PN, h.data(), nx * 8);
        if (PT) std::memcpy(PT, h.data() + nx, nx * 8);
        return SCMC_OK;
    }
    if (!(R0 > 0) || !std::isfinite(R0))
        return fail(c, SCMC_EINVAL, "R0 must be positive");
    if (kind == SCMC_OBS_SHELL) {
        const int nl = shell_rmax(m, d) + 1;
        std::vector<double> h(2 * nl + 3);
        HIPCHK(c, launch_shell(c.key, m, c.dens64, c.partials, (long)c.nblocks * 9, c.small,
                               c.stream));
        HIPCHK(c, hipMemcpyAsync(h.data(), c.small, h.size() * 8, hipMemcpyDeviceToHost,
                                 c.stream));
        HIPCHK(c, hipStreamSynchronize(c.stream));
        droplet_sigma(d, h[2 * nl], h[2 * nl + 1], h[2 * nl + 2], R0, out);
        if (PN) std::memcpy(PN, h.data(), nl * 8);
        if (PT) std::memcpy(PT, h.data() + nl, nl * 8);
        return SCMC_OK;
    }
    const int rmax = m.nx / 2, nl = rmax + 1;
    std::vector<double> h(3 * nl + 3);
    HIPCHK(c, launch_line(c.key, m, c.dens64, c.small, c.stream));
    HIPCHK(c, hipMemcpyAsync(h.data(), c.small, h.size() * 8,
                             hipMemcpyDeviceToHost, c.stream));
    HIPCHK(c, hipStreamSynchronize(c.stream));
    droplet_sigma(d, h[3 * nl], h[3 * nl + 1], h[3 * nl + 2], R0, out);
    double mx = 0;
    for (int r = 0; r < nl; ++r)
        if (d == 3) mx = std::max(mx, std::fabs(h[nl + r] - h[2 * nl + r]));
    out->max_PyyPzz = mx;
    if (PN) std::memcpy(PN, h.data(), nl * 8);
    if (PT) std::memcpy(PT, h.data() + nl, nl * 8);
    return SCMC_OK;
}

// ---- stepping ------------------------------------------------------------
int direct_step_sim(scmc_sim *s) {
    Common &c = s->c;
    const void *src = c.pop[c.cur];
    void *dst = c.pop[1 - c.cur];
    hipError_t e = c.kernel == SCMC_KERNEL_FUSED
                       ? launch_fused(c.key, s->lat.m, src, dst, c.tile, c.stream)
                       : launch_two_pass(c.key, step_member(c, s->lat.m, c.cur), src,
                                         dst, c.dens, c.stream);
    if (e != hipSuccess)
        return fail(c, SCMC_EDEVICE, "step launch: %s", hipGetErrorString(e));
    c.cur ^= 1;
    return SCMC_OK;
}

StorageWidth storage_width(const StepKey &k) {
    return k.storage == ST_F64 ? WIDE_64 : k.storage == ST_F32 ? WIDE_32 : WIDE_16;
}

// sites in rows that are not a multiple of 16 (mom_steps_pay)
int64_t ragged_sites(const Member &m) { return m.nx % 16 ? m.N : 0; }

// Whether a block of k steps of this handle runs on the moment field alone.
bool mom_steps_on(const scmc_sim *s, int64_t k) {
    const StepKey &key = s->c.key;
    if (k < 2 || !s->mom_ok || s->c.kernel != SCMC_KERNEL_TWO_PASS || !key.mom || key.sr)
        return false;
    const Member &m = s->lat.m;
    return s->lat.dim == 3
               ? mom_steps_pay(storage_width(key), key.node, key.order, key.psi, m.N,
                               ragged_sites(m), s->mom_us, 1, k)
               : mom2_steps_pay(storage_width(key), key.order, key.psi, m.N, k);
}

// The launches of k >= 2 steps from buffer par that stay in the moment field:
// pass 1, k - 1 moment steps (2D: several per launch), pass 2; each goes to
// emit(launch, arguments).
// The moments alternate between the workspace's moment field, where the last
// ones must be for pass 2, and the population buffer that pass 1 does not
// read, whose contents no one needs any more and pass 2 at most overwrites
// (24 or 48 B per site of its 36 to 304).  Node storage keeps the last pairs
// as the reference field of the buffer that pass 2 fills.
template <class Emit>
int mom_steps(scmc_sim *s, int64_t k, int par, Emit &&emit) {
    Common &c = s->c;
    const Member &m = s->lat.m;
    const int last = par ^ (int)((k - 1) & 1);
    NodeLaunch p1{}, p2{};
    if (!node_two_pass(c.key, &p1, &p2, m))
        return fail(c, SCMC_EUNSUPPORTED, "no two-pass kernel for this problem");
    p1.grid = dim3(linear_blocks(m, m.nz, (int)p1.block.x));
    if (c.key.mom == 1) p2.grid = dim3(linear_blocks(m, m.nz, (int)p2.block.x));
    Member m1 = step_member(c, m, par), m2 = step_member(c, m, last);
    void *field[2] = {c.dens, c.pop[1 - par]};
    const int slot[2] = {m2.pair_slot, 0};
    // one moment step per launch in 3D; in 2D launches of equal numbers of
    // steps, at most mom2
    const int64_t nl = s->mom2 ? (k - 2 + s->mom2) / s->mom2 : k - 1;
    int at = (int)(nl & 1);  // the field that holds the current moments
    m1.pair_slot = slot[at];
    const void *src = c.pop[par], *src2 = c.pop[last];
    void *dst = c.pop[1 - last];
    std::vector<void *> a1 = {(void *)&m1, (void *)&src, (void *)&field[at]};
    int rc = emit(p1, a1);
    Member ms = m;
    MomShape shape = s->mom_shape;
    for (int64_t t = 0; t < nl && !rc; ++t, at ^= 1) {
        int si = slot[at], so = slot[1 - at];
        int steps = (int)((k - 1) / nl + (t < (k - 1) % nl ? 1 : 0));
        std::vector<void *> a = {(void *)&ms, (void *)&shape};
        if (s->mom2) a.push_back((void *)&steps);
        a.push_back((void *)&field[at]);
        a.push_back((void *)&field[1 - at]);
        if (!s->mom2) {
            a.push_back((void *)&si);
            a.push_back((void *)&so);
        }
        rc = emit(s->mom_node, a);
    }
    std::vector<void *> a2 = {(void *)&m2, (void *)&src2, (void *)&dst, (void *)&field[0]};
    return rc ? rc : emit(p2, a2);
}

// k steps of a single lattice outside graphs.
int direct_steps_sim(scmc_sim *s, int64_t k) {
    Common &c = s->c;
    if (!mom_steps_on(s, k)) {
        int rc = SCMC_OK;
        for (int64_t t = 0; t < k && !rc; ++t) rc = direct_step_sim(s);
        return rc;
    }
    const int rc = mom_steps(s, k, c.cur, [&](const NodeLaunch &nl, std::vector<void *> &args) {
        const hipError_t e =
            hipLaunchKernel(nl.func, nl.grid, nl.block, args.data(), nl.shmem, c.stream);
        return e == hipSuccess
                   ? SCMC_OK
                   : fail(c, SCMC_EDEVICE, "step launch: %s", hipGetErrorString(e));
    });
    if (!rc && (k & 1)) c.cur ^= 1;
    return rc;
}

// One op of the batched two-pass from src to dst with the moment field (its
// base, to which members add dens_off) at field.
template <class Emit>
int emit_op(scmc_batch *b, const BatchOp &o, const void *src, void *dst, void *field,
            Emit &&emit) {
    Common &c = b->c;
    std::vector<void *> args;
    NodeLaunch nl{};
    Member m = o.m;
    const Member *dm = b->d_members;
    const Tile *dt = b->d_tiles + o.t0;
    int nt = o.n;
    if (o.member >= 0) {  // a chunk of one member, as a single lattice
        if (!node_member_pass(c.key, o.m, o.pass, o.nt_all, &nl))
            return fail(c, SCMC_EUNSUPPORTED, "no kernel for a member pass");
        args = {(void *)&m, (void *)&src};
    } else {
        NodeLaunch dn{}, sn{}, dna{};
        if (!node_batch_two_pass(c.key, o.n, &dn, &sn, &dna))  // one workgroup per tile
            return fail(c, SCMC_EUNSUPPORTED, "no kernel for this batch");
        nl = o.pass == 1 ? (o.nt_all ? dna : dn) : sn;
        args = {(void *)&dm, (void *)&dt, (void *)&nt, (void *)&src};
    }
    if (o.pass == 2) args.push_back((void *)&dst);
    args.push_back((void *)&field);
    return emit(nl, args);
}

// k steps of the batched two-pass from buffer par, group by group: each group
// (whole chunks, whose pass 1 and pass 2 ops batch_set_ops pairs) advances k
// steps before the next one starts.  Members are independent lattices, so the
// order changes no bit of any member's result, and every member is k steps
// further on return; a group's next step then reads what its last one has just
// written, part of it still in the Infinity Cache, as a lattice stepped on its
// own does.  With mom set the steps between stay in the moment field, as in
// mom_steps; the second field is the group's own part of the population
// buffer that its pass 1 does not read.
template <class Emit> int batch_steps(scmc_batch *b, int64_t k, int par, Emit &&emit) {
    Common &c = b->c;
    int rc = SCMC_OK;
    for (BatchGroup &g : b->groups) {
        if (k >= 2 && g.mom &&
            mom_steps_pay(storage_width(c.key), false, c.key.order, c.key.psi, g.sites, g.ragged,
                          g.us, (int)g.launches.size(), k)) {
            const int last = par ^ (int)((k - 1) & 1);
            const Member &m0 = b->lats[g.member].m;
            const scmc_problem &p0 = b->lats[g.member].p;
            char *own = (char *)c.pop[1 - par] + m0.pop_off * (int64_t)storage_bytes(p0.storage);
            void *field[2] = {c.dens, own - m0.dens_off * (int64_t)real_bytes(p0.storage)};
            int at = (int)((k - 1) & 1);
            for (size_t j = g.op0; j < g.op1 && !rc; j += 2)
                rc = emit_op(b, b->ops[j], c.pop[par], c.pop[1 - par], field[at], emit);
            const Member *dm = b->d_members;
            for (int64_t t = 1; t < k && !rc; ++t, at ^= 1)
                for (size_t l = 0; l < g.launches.size() && !rc; ++l) {
                    std::vector<void *> a = {(void *)&dm, (void *)&g.launches[l].list,
                                             (void *)&field[at], (void *)&field[1 - at]};
                    rc = emit(g.launches[l].node, a);
                }
            for (size_t j = g.op0 + 1; j < g.op1 && !rc; j += 2)
                rc = emit_op(b, b->ops[j], c.pop[last], c.pop[1 - last], field[0], emit);
            continue;
        }
        for (size_t j = g.op0; j < g.op1 && !rc; j += 2)  // chunk by chunk
            for (int64_t t = 0; t < k && !rc; ++t) {
                const int cu = par ^ (int)(t & 1);
                rc = emit_op(b, b->ops[j], c.pop[cu], c.pop[1 - cu], c.dens, emit);
                if (!rc) rc = emit_op(b, b->ops[j + 1], c.pop[cu], c.pop[1 - cu], c.dens, emit);
            }
    }
    return rc;
}

// k steps of a batch outside graphs; the fused design (no ops) runs step by step.
int direct_steps_batch(scmc_batch *b, int64_t k) {
    Common &c = b->c;
    if (b->ops.empty()) {
        for (int64_t t = 0; t < k; ++t) {
            const hipError_t e = launch_batch_fused(c.key, b->d_members, b->d_tiles, b->ntiles,
                                                    c.pop[c.cur], c.pop[1 - c.cur], c.tile,
                                                    b->grid, c.stream);
            if (e != hipSuccess)
                return fail(c, SCMC_EDEVICE, "batch step launch: %s", hipGetErrorString(e));
            c.cur ^= 1;
        }
        return SCMC_OK;
    }
    const int rc = batch_steps(b, k, c.cur, [&](const NodeLaunch &nl, std::vector<void *> &args) {
        const hipError_t e =
            hipLaunchKernel(nl.func, nl.grid, nl.block, args.data(), nl.shmem, c.stream);
        return e == hipSuccess
                   ? SCMC_OK
                   : fail(c, SCMC_EDEVICE, "batch step launch: %s", hipGetErrorString(e));
    });
    if (!rc && (k & 1)) c.cur ^= 1;
    return rc;
}

// Build an executable graph of k steps starting from buffer `par`.
// A single lattice passes chunks {0, 0} and, to run on the moment field where
// it can, itself (sim); a batch either itself for its two-pass launches
// (two_pass) or, for the fused designs, chunks {0, ntiles}.
int build_graph(Common &c, int k, int par, bool batch, const Member &m,
                const Member *d_members, const Tile *d_tiles,
                const std::vector<int> &chunks, int grid,
                scmc_batch *two_pass = nullptr, scmc_sim *sim = nullptr) {
    hipGraph_t g = nullptr;
    HIPCHK(c, hipGraphCreate(&g, 0));
    hipGraphNode_t prev = nullptr;
    const bool fused = c.kernel == SCMC_KERNEL_FUSED;
    auto add = [&](const NodeLaunch &nl, std::vector<void *> &args) -> int {
        hipKernelNodeParams kp{};
        kp.func = nl.func;
        kp.gridDim = nl.grid;
        kp.blockDim = nl.block;
        kp.sharedMemBytes = nl.shmem;
        kp.kernelParams = args.data();
        hipGraphNode_t node;
        hipError_t e = hipGraphAddKernelNode(&node, g, prev ? &prev : nullptr, prev ? 1 : 0, &kp);
        if (e != hipSuccess) return fail(c, SCMC_EDEVICE, "graph node: %s", hipGetErrorString(e));
        prev = node;
        return SCMC_OK;
    };
    int cur = par, rc = SCMC_OK;
    if (two_pass) rc = batch_steps(two_pass, k, par, add);
    const bool mom = sim && mom_steps_on(sim, k);
    if (mom) rc = mom_steps(sim, k, par, add);
    for (int t = 0; !two_pass && !mom && t < k && !rc; ++t) {
        for (size_t ch = 0; ch + 1 < chunks.size() && !rc; ++ch) {
            const int ntiles = chunks[ch + 1] - chunks[ch];
            // persistent fused launches: at most `grid` workgroups (clamped to
            // the resident count)
            const int cgrid = batch ? std::min(grid, ntiles) : grid;
            NodeLaunch dn{}, sn{};
            const bool ok = batch ? (fused ? node_batch_fused(c.key, c.tile, cgrid, &sn)
                                           : node_batch_two_pass(c.key, cgrid, &dn, &sn))
                                  : (fused ? node_fused(c.key, c.tile, &sn, m)
                                           : node_two_pass(c.key, &dn, &sn, m));
            if (!ok) {
                rc = fail(c, SCMC_EUNSUPPORTED, "no graph node for this kernel");
                break;
            }
            // argument values, in kernel-signature order
            const Member ms = batch ? m : step_member(c, m, cur);
            Member mv = ms;
            const Member *dm = d_members;
            const Tile *dt = d_tiles ? d_tiles + chunks[ch] : nullptr;
            int nt = ntiles;
            const void *srcv = c.pop[cur];
            void *dstv = c.pop[1 - cur];
            void *densv = c.dens;
            int zc = c.tile[2];
            // the step kernel's last argument: the density field (two-pass) or
            // the z-chunk length (fused)
            void *last = fused ? (void *)&zc : (void *)&densv;
            std::vector<void *> dargs, sargs;
            if (batch) {
                dargs = {(void *)&dm, (void *)&dt, (void *)&nt, (void *)&srcv, (void *)&densv};
                sargs = {(void *)&dm, (void *)&dt, (void *)&nt, (void *)&srcv, (void *)&dstv, last};
            } else {
                dargs = {(void *)&mv, (void *)&srcv, (void *)&densv};
                sargs = {(void *)&mv, (void *)&srcv, (void *)&dstv, last};
            }
            const std::vector<SlabOp> slabs =
                batch || fused ? std::vector<SlabOp>() : slab_schedule(c.key, m);
            if (!slabs.empty()) {  // the moment two-pass in z-slabs, as launch_two_pass
                NodeLaunch pn{};
                Member mv1 = ms;
                int nb2 = 0, nb1 = 0;
                std::vector<void *> pargs = {(void *)&mv, (void *)&mv1, (void *)&nb2,
                                                   (void *)&nb1, (void *)&srcv, (void *)&dstv,
                                                   (void *)&densv};
                for (const SlabOp &o : slabs) {
                    if (rc) break;
                    mv = ms;
                    mv.zoff = o.z0;
                    mv.znum = o.nz;
                    if (o.pass == 3) {
                        if (!pn.func && !node_slab_pair(c.key, &pn)) {
                            rc = fail(c, SCMC_EUNSUPPORTED, "no graph node for the slab pair");
                            break;
                        }
                        mv1 = ms;
                        mv1.zoff = o.z1;
                        mv1.znum = o.n1;
                        nb2 = linear_blocks(m, o.nz, (int)pn.block.x);
                        nb1 = linear_blocks(m, o.n1, (int)pn.block.x);
                        NodeLaunch nl = pn;
                        nl.grid = dim3(nb2 + nb1);
                        rc = add(nl, pargs);
                        continue;
                    }
                    NodeLaunch nl = o.pass == 1 ? dn : sn;
                    nl.grid = dim3(linear_blocks(m, o.nz, (int)nl.block.x));
                    rc = add(nl, o.pass == 1 ? dargs : sargs);
                }
                continue;
            }
            if (!fused) rc = add(dn, dargs);
            if (!rc) rc = add(sn, sargs);
        }
        cur ^= 1;
    }
    if (rc) {
        (void)hipGraphDestroy(g);
        return rc;
    }
    hipError_t e = hipGraphInstantiate(&c.gexec[par], g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        c.gexec[par] = nullptr;
        return fail(c, SCMC_EDEVICE, "graph instantiate: %s",
                    hipGetErrorString(e));
    }
    return SCMC_OK;
}

// Steps outside graphs go in blocks of up to kStepBlock steps through many(k).
constexpr int64_t kStepBlock = 64;

template <class BuildFn, class ManyFn>
int run_steps(Common &c, int64_t nsteps, BuildFn build, ManyFn many) {
    if (nsteps < 0) return fail(c, SCMC_EINVAL, "nsteps < 0");
    if (!c.initialized)
        return fail(c, SCMC_ESTATE, "state not set (call set_density first)");
    int64_t left = nsteps;
    while (left > 0) {
        if (c.graph_k > 0 && left >= c.graph_k) {
            if (!c.gexec[c.cur]) {
                int rc = build(c.cur);
                if (rc) return rc;
            }
            HIPCHK(c, hipGraphLaunch(c.gexec[c.cur], c.stream));
            if (c.graph_k % 2) c.cur ^= 1;
            left -= c.graph_k;
            c.step += c.graph_k;
        } else {
            const int64_t k = std::min(left, kStepBlock);
            int rc = many(k);
            if (rc) return rc;
            left -= k;
            c.step += k;
        }
    }
    return SCMC_OK;
}

}  // namespace

// =================================================================== ABI
extern "C" {

int scmc_problem_init(scmc_problem *p) {
    if (!p) return SCMC_EINVAL;
    std::memset(p, 0, sizeof *p);
    p->lattice = SCMC_D3Q19;
    p->stencil = SCMC_E6;
    p->nx = p->ny = p->nz = 64;
    p->tau[0] = p->tau[1] = 1.0;
    p->g[0][1] = p->g[1][0] = 1.8;
    p->psi_self = SCMC_PSI_N;
    p->storage = SCMC_F32;
    p->n0[0] = p->n0[1] = 0.52;
    p->kernel = SCMC_KERNEL_AUTO;
    return SCMC_OK;
}

int scmc_velocities(int lattice, int *xi, double *w) {
    if (lattice != SCMC_D2Q9 && lattice != SCMC_D3Q19) return SCMC_EINVAL;
    if (!xi || !w) return SCMC_EINVAL;
    velocities(lattice, xi, w);
    return lattice_q(lattice);
}

int scmc_workspace_bytes(const scmc_problem *p, size_t *out) {
    if (!out) return SCMC_EINVAL;
    int rc = validate(p, nullptr);
    if (rc) return rc;
    *out = plan_of({*p}, 0).total;
    return SCMC_OK;
}

int scmc_create(const scmc_problem *p, void *d_ws, size_t ws_bytes,
                void *stream, scmc_sim **out) {
    if (!out) return SCMC_EINVAL;
    *out = nullptr;
    std::string why;
    int rc = validate(p, &why);
    if (rc) return rc;
    if (!d_ws || ((uintptr_t)d_ws % ALIGN)) return SCMC_EINVAL;
    const Plan pl = plan_of({*p}, 0);
    if (ws_bytes < pl.total) return SCMC_ENOSPACE;
    scmc_sim *s = new (std::nothrow) scmc_sim();
    if (!s) return SCMC_EINVAL;
    s->lat.p = *p;
    s->lat.m = member_of(*p);
    s->lat.q = lattice_q(p->lattice);
    s->lat.dim = lattice_dim(p->lattice);
    Common &c = s->c;
    c.key = key_of(*p);
    rc = choose_kernel(*p, c.key, &c.kernel, c.tile);
    if (rc) {
        delete s;
        return rc;
    }
    c.stream = (hipStream_t)stream;
    c.ws = (char *)d_ws;
    c.ws_bytes = ws_bytes;
    bind(c, pl, c.ws, stats_blocks(s->lat.m));
    s->lat.m.step_ctr = c.ctr;
    s->mom_ok = s->lat.dim == 3
                    ? node_mom_step(c.key, s->lat.m, &s->mom_node, &s->mom_shape, &s->mom_us)
                    : node_mom2_steps(c.key, s->lat.m, &s->mom_node, &s->mom_shape, &s->mom2);
    *out = s;
    return SCMC_OK;
}

int scmc_destroy(scmc_sim *s) {
    if (!s) return SCMC_EINVAL;
    // queued steps still write the caller's workspace: let them finish before
    // the caller may reuse that memory
    const hipError_t e = hipStreamSynchronize(s->c.stream);
    drop_graphs(s->c);
    delete s;
    return e == hipSuccess ? SCMC_OK : SCMC_EDEVICE;
}

int scmc_set_density(scmc_sim *s, const double *nA, const double *nB) {
    if (!s || !nA || !nB) return SCMC_EINVAL;
    int rc = set_density_impl(s->c, s->lat, nA, nB, s->c.pop[0]);
    if (!rc) rc = set_step_counter(s->c, 0);
    if (rc) return rc;
    s->have_prev = false;
    s->c.cur = 0;
    s->c.step = 0;
    s->c.initialized = true;
    return SCMC_OK;
}

int scmc_set_populations(scmc_sim *s, const double *f, int64_t step) {
    if (!s || !f) return SCMC_EINVAL;
    const size_t n = 2 * (size_t)s->lat.q * s->lat.m.N;
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(f[i]))
            return fail(s->c, SCMC_EINVAL, "non-finite population %zu", i);
    int rc = upload_state(s->c, s->lat, f, s->c.pop[0]);
    if (!rc) rc = set_step_counter(s->c, step);
    if (rc) return rc;
    s->have_prev = false;
    s->c.cur = 0;
    s->c.step = step;
    s->c.initialized = true;
    return SCMC_OK;
}

int scmc_get_populations(scmc_sim *s, double *f, int64_t *step) {
    if (!s || !f) return SCMC_EINVAL;
    if (!s->c.initialized) return fail(s->c, SCMC_ESTATE, "state not set");
    int rc = download_state(s->c, s->lat, s->c.pop[s->c.cur], f);
    if (rc) return rc;
    if (step) *step = s->c.step;
    return SCMC_OK;
}

int scmc_set_graph_steps(scmc_sim *s, int k) {
    if (!s || k < 0) return SCMC_EINVAL;
    drop_graphs(s->c);
    s->c.graph_k = k;
    return SCMC_OK;
}

int scmc_step(scmc_sim *s, int64_t nsteps) {
    if (!s) return SCMC_EINVAL;
    Common &c = s->c;
    return run_steps(
        c, nsteps,
        [&](int par) {
            static const std::vector<int> whole = {0, 0};
            return build_graph(c, c.graph_k, par, false, s->lat.m, nullptr,
                               nullptr, whole, 0, nullptr, s);
        },
        [&](int64_t k) { return direct_steps_sim(s, k); });
}

// ---- the allocation-free step ----------------------------------------------
// For callers that cannot allocate: the density / moment field of the
// two-pass designs lives in this file-scope device array instead of a caller
// workspace.  Host code never passes its name as an address (in host code the
// name is a host-side stand-in): static_scratch() fetches the current GPU's
// own copy with hipGetSymbolAddress, once per device, and every use goes
// through that pointer.
static __device__ __align__(256) unsigned char scratch[SCMC_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
thread_local char g_static_err[320] = "";

int static_fail(int status, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_static_err, sizeof g_static_err, fmt, ap);
    va_end(ap);
    return status;
}

// Device address of the current device's scratch array.
int static_scratch(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return static_fail(SCMC_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices)
        return static_fail(SCMC_EDEVICE, "device index %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return static_fail(SCMC_EDEVICE, "hipGetSymbolAddress(scratch) on device %d: %s",
                               dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SCMC_OK;
}

}  // namespace

int scmc_step_static(const scmc_problem *p, const void *src, void *dst, void *stream) {
    g_static_err[0] = '\0';
    if (!p || !src || !dst) return static_fail(SCMC_EINVAL, "NULL problem or population buffer");
    if (src == dst) return static_fail(SCMC_EINVAL, "src and dst must be distinct buffers");
    int rc = validate(p, nullptr);
    if (rc) return static_fail(rc, "invalid problem (%s)", scmc_status_str(rc));
    if (p->rounding == SCMC_ROUND_STOCHASTIC)
        return static_fail(SCMC_EUNSUPPORTED,
                           "stochastic rounding keeps its step counter in a workspace: use scmc_step");
    if (node_storage(p->storage))
        return static_fail(SCMC_EUNSUPPORTED,
                           "node storage keeps its reference field in a workspace: use scmc_step");
    const StepKey key = key_of(*p);
    int kernel = 0, tile[3] = {0, 0, 0};
    rc = choose_kernel(*p, key, &kernel, tile, false);
    if (rc) return static_fail(rc, "no kernel design for this problem");
    const Member m = member_of(*p);
    // the field that scmc_workspace_bytes plans for the same problem: 7
    // values of the compute precision per site
    const size_t per_site = 7 * real_bytes(p->storage);
    const size_t need = per_site * (size_t)m.N;
    if (need > (size_t)SCMC_STATIC_SCRATCH_BYTES)
        return static_fail(SCMC_ENOSPACE,
                           "%d sites need %zu bytes of scratch; the static array holds %zu "
                           "bytes (at most %zu sites with this storage)",
                           m.N, need, (size_t)SCMC_STATIC_SCRATCH_BYTES,
                           (size_t)SCMC_STATIC_SCRATCH_BYTES / per_site);
    void *scr = nullptr;
    rc = static_scratch(&scr);
    if (rc) return rc;
    const hipStream_t st = (hipStream_t)stream;
    const hipError_t e = kernel == SCMC_KERNEL_FUSED
                             ? launch_fused(key, m, src, dst, tile, st)
                             : launch_two_pass(key, m, src, dst, scr, st);
    if (e != hipSuccess) return static_fail(SCMC_EDEVICE, "step launch: %s", hipGetErrorString(e));
    return SCMC_OK;
}

int scmc_synchronize(scmc_sim *s) {
    if (!s) return SCMC_EINVAL;
    HIPCHK(s->c, hipStreamSynchronize(s->c.stream));
    return SCMC_OK;
}

int scmc_get_fields(scmc_sim *s, double *nA, double *nB, double *u) {
    if (!s) return SCMC_EINVAL;
    if (!s->c.initialized) return fail(s->c, SCMC_ESTATE, "state not set");
    return fields_impl(s->c, s->lat, s->c.pop[s->c.cur], nA, nB, u);
}

int scmc_stats_get(scmc_sim *s, scmc_stats *out) {
    if (!s) return SCMC_EINVAL;
    if (!s->c.initialized) return fail(s->c, SCMC_ESTATE, "state not set");
    int rc = stats_impl(s->c, s->lat, s->c.pop[s->c.cur], out, s->c.step);
    if (rc) return rc;
    if (out->n_nonfinite > 0)
        return fail(s->c, SCMC_ENONFINITE, "%.0f non-finite populations",
                    out->n_nonfinite);
    return SCMC_OK;
}

int scmc_observables(scmc_sim *s, int kind, double R0, scmc_obs *out,
                     double *PN, double *PT) {
    if (!s) return SCMC_EINVAL;
    if (!s->c.initialized) return fail(s->c, SCMC_ESTATE, "state not set");
    return obs_impl(s->c, s->lat, s->c.pop[s->c.cur], kind, R0, out, PN, PT,
                    s->c.step);
}

int scmc_convergence_check(scmc_sim *s, double R0, double tol_dP, double tol_du,
                           scmc_convergence *out) {
    if (!s || !out) return SCMC_EINVAL;
    Common &c = s->c;
    if (!c.initialized) return fail(c, SCMC_ESTATE, "state not set");
    const Lat &L = s->lat;
    const void *pop = c.pop[c.cur];
    const Member m = obs_member(c, L, pop);
    scmc_obs o;
    int rc = obs_impl(c, L, pop, SCMC_OBS_DROPLET, R0, &o, nullptr, nullptr, c.step);
    if (rc) return rc;  // obs_impl leaves the FP64 densities in dens64
    const long N = m.N;
    const long centre = ((long)(m.nz / 2) * m.ny + m.ny / 2) * m.nx + m.nx / 2;
    const long far = ((long)((m.nz / 2 + m.nz / 2) % m.nz) * m.ny + (m.ny / 2 + m.ny / 2) % m.ny) *
                         m.nx + (m.nx / 2 + m.nx / 2) % m.nx;
    double h[4];
    HIPCHK(c, hipMemcpyAsync(&h[0], c.dens64 + centre, 8, hipMemcpyDeviceToHost, c.stream));
    HIPCHK(c, hipMemcpyAsync(&h[1], c.dens64 + N + centre, 8, hipMemcpyDeviceToHost, c.stream));
    HIPCHK(c, hipMemcpyAsync(&h[2], c.dens64 + far, 8, hipMemcpyDeviceToHost, c.stream));
    HIPCHK(c, hipMemcpyAsync(&h[3], c.dens64 + N + far, 8, hipMemcpyDeviceToHost, c.stream));
    HIPCHK(c, hipStreamSynchronize(c.stream));
    const int rich = h[1] > h[0] ? 1 : 0;
    HIPCHK(c, launch_velocity64(c.key, m, pop, c.dens64, c.vel64, c.stream));
    HIPCHK(c, launch_monitor(m, L.dim, c.dens64, c.vel64, s->have_prev ? c.velprev : nullptr,
                             rich, h[2 + rich], c.partials, c.small, c.stream));
    double r[5];
    HIPCHK(c, hipMemcpyAsync(r, c.small, sizeof r, hipMemcpyDeviceToHost, c.stream));
    HIPCHK(c, hipMemcpyAsync(c.velprev, c.vel64, 3 * N * 8, hipMemcpyDeviceToDevice, c.stream));
    HIPCHK(c, hipStreamSynchronize(c.stream));
    const double nan = std::nan("");
    std::memset(out, 0, sizeof *out);
    out->dP = o.dP;
    out->dP_change = s->have_prev ? std::fabs(o.dP - s->prev_dP) / std::fabs(s->prev_dP) : nan;
    out->du = s->have_prev ? r[0] / (double)N : nan;
    const int ext[3] = {m.nx, m.ny, m.nz};
    out->com_offset = 0;
    for (int a = 0; a < 3; ++a) {
        const double off = a < L.dim ? r[2 + a] / r[1] : 0.0;
        out->com[a] = ext[a] / 2 + off;
        out->com_offset = std::max(out->com_offset, std::fabs(off));
    }
    out->rich = rich;
    out->step = c.step;
    out->prev_step = s->have_prev ? s->prev_step : -1;
    out->converged = s->have_prev && (out->dP_change < tol_dP || out->du < tol_du);
    s->have_prev = true;
    s->prev_dP = o.dP;
    s->prev_step = c.step;
    return SCMC_OK;
}

int scmc_run_to_convergence(scmc_sim *s, double R0, int64_t dt, int64_t max_steps,
                            double tol_dP, double tol_du, scmc_convergence *out) {
    if (!s || !out || dt < 1 || max_steps < 0) return SCMC_EINVAL;
    int rc = scmc_convergence_check(s, R0, tol_dP, tol_du, out);
    int64_t done = 0;
    while (!rc && !out->converged && done < max_steps) {
        const int64_t k = std::min(dt, max_steps - done);
        rc = scmc_step(s, k);
        done += k;
        if (!rc) rc = scmc_convergence_check(s, R0, tol_dP, tol_du, out);
        if (!rc && !std::isfinite(out->dP))
            rc = fail(s->c, SCMC_ENONFINITE, "Delta P is not finite at step %lld",
                      (long long)out->step);
    }
    return rc;
}

int scmc_curvature_fit(int n, const double *curvature, const double *sigma, double *out) {
    if (n < 3 || !curvature || !sigma || !out) return SCMC_EINVAL;
    // least squares of sigma = c0 + c1 k + c2 k^2 through the normal equations,
    // in powers of k / kmax so that the 3 x 3 system stays well scaled
    double kmax = 0;
    for (int i = 0; i < n; ++i) {
        if (!std::isfinite(curvature[i]) || !std::isfinite(sigma[i])) return SCMC_EINVAL;
        kmax = std::max(kmax, std::fabs(curvature[i]));
    }
    if (kmax == 0) return SCMC_EINVAL;
    double A[3][4] = {};
    for (int i = 0; i < n; ++i) {
        const double t = curvature[i] / kmax, b[3] = {1.0, t, t * t};
        for (int r = 0; r < 3; ++r) {
            for (int c = 0; c < 3; ++c) A[r][c] += b[r] * b[c];
            A[r][3] += b[r] * sigma[i];
        }
    }
    const double scale = A[0][0];
    for (int c = 0; c < 3; ++c) {  // Gauss-Jordan with partial pivoting
        int piv = c;
        for (int r = c + 1; r < 3; ++r)
            if (std::fabs(A[r][c]) > std::fabs(A[piv][c])) piv = r;
        if (std::fabs(A[piv][c]) <= 1e-12 * scale) return SCMC_EINVAL;  // < 3 distinct k
        for (int k = 0; k < 4; ++k) std::swap(A[c][k], A[piv][k]);
        for (int r = 0; r < 3; ++r) {
            if (r == c) continue;
            const double f = A[r][c] / A[c][c];
            for (int k = c; k < 4; ++k) A[r][k] -= f * A[c][k];
        }
    }
    const double c0 = A[0][3] / A[0][0];
    const double c1 = A[1][3] / A[1][1] / kmax;
    const double c2 = A[2][3] / A[2][2] / (kmax * kmax);
    if (!(c0 != 0) || !std::isfinite(c0)) return SCMC_EINVAL;
    out[0] = c0;
    out[1] = -c1 / (2.0 * c0);
    out[2] = c2 / c0;
    return SCMC_OK;
}

int scmc_pull_copy(scmc_sim *s, int reps, double *us) {
    if (!s || !us || reps < 1) return SCMC_EINVAL;
    Common &c = s->c;
    const Lat &L = s->lat;
    const int bytes = (int)storage_bytes(L.p.storage);
    Member m = L.m;
    hipEvent_t e0, e1;
    HIPCHK(c, hipEventCreate(&e0));
    HIPCHK(c, hipEventCreate(&e1));
    hipError_t e = launch_pull_copy(L.dim, bytes, m, c.pop[0], c.pop[1], c.stream);  // warm-up
    if (e == hipSuccess) e = hipEventRecord(e0, c.stream);
    for (int r = 0; r < reps && e == hipSuccess; ++r)
        e = launch_pull_copy(L.dim, bytes, m, c.pop[r & 1], c.pop[1 - (r & 1)], c.stream);
    if (e == hipSuccess) e = hipEventRecord(e1, c.stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    // the buffers now hold shifted copies, not a state of the method
    c.initialized = false;
    c.step = 0;
    c.cur = 0;
    s->have_prev = false;
    if (e != hipSuccess) return fail(c, SCMC_EDEVICE, "pull copy: %s", hipGetErrorString(e));
    *us = 1e3 * ms / reps;
    return SCMC_OK;
}

int scmc_config(scmc_sim *s, int *kernel, int *tile) {
    if (!s) return SCMC_EINVAL;
    if (kernel)
        *kernel = public_kernel(s->c.kernel, s->c.key.repull, s->c.key.mom);
    if (tile)
        for (int a = 0; a < 3; ++a) tile[a] = s->c.tile[a];
    return SCMC_OK;
}

const char *scmc_last_error(const scmc_sim *s) {
    if (s) return s->c.err.c_str();
    return g_static_err[0] ? g_static_err : "NULL handle";
}
const char *scmc_batch_last_error(const scmc_batch *b) {
    return b ? b->c.err.c_str() : "NULL handle";
}

const char *scmc_status_str(int st) {
    switch (st) {
        case SCMC_OK: return "ok";
        case SCMC_EINVAL: return "invalid argument";
        case SCMC_EUNSUPPORTED: return "unsupported";
        case SCMC_ENOSPACE: return "workspace too small";
        case SCMC_EDEVICE: return "device error";
        case SCMC_ENONFINITE: return "non-finite state";
        case SCMC_ESTATE: return "bad call order";
    }
    return "unknown status";
}

// ------------------------------------------------------- flat steady state
static scmc_problem flat_problem(const scmc_problem &p, int lx) {
    scmc_problem q = p;
    q.nx = lx;
    q.ny = 5;
    q.nz = p.lattice == SCMC_D2Q9 ? 1 : 5;
    q.kernel = SCMC_KERNEL_TWO_PASS;  // a few thousand sites: launch-bound
    return q;
}

// k steps of the flat interface, which stays uniform along y and z.
static int flat_steps(scmc_sim *s, int64_t k) {
    Common &c = s->c;
    if (!row_steps_supported(c.key, s->lat.m)) return scmc_step(s, k);
    const int to = c.cur ^ (int)(k & 1);
    HIPCHK(c, launch_row_steps(c.key, s->lat.m, c.pop[c.cur], c.pop[to], (int)k, c.stream));
    c.cur = to;
    c.step += k;
    return SCMC_OK;
}

int scmc_flat_workspace_bytes(const scmc_problem *p, int lx, size_t *out) {
    if (!p || !out) return SCMC_EINVAL;
    const scmc_problem q = flat_problem(*p, lx);
    return scmc_workspace_bytes(&q, out);
}

int scmc_flat_equilibrium(const scmc_problem *p, int lx, const double *guess,
                          int64_t max_steps, double tol, void *d_ws,
                          size_t ws_bytes, void *stream, double *out,
                          int64_t *steps) {
    if (!p || !out || max_steps < 0 || !(tol >= 0)) return SCMC_EINVAL;
    const double g0[4] = {1.0, 0.04, 0.04, 1.0};
    const double *g = guess ? guess : g0;
    for (int k = 0; k < 4; ++k)
        if (!std::isfinite(g[k])) return SCMC_EINVAL;
    const scmc_problem q = flat_problem(*p, lx);
    scmc_sim *s = nullptr;
    int rc = scmc_create(&q, d_ws, ws_bytes, stream, &s);
    if (rc) return rc;
    const size_t N = (size_t)q.nx * q.ny * q.nz;
    std::vector<double> nA(N), nB(N);
    for (size_t i = 0; i < N; ++i) {
        const int x = (int)(i % q.nx);
        const bool in = x >= lx / 4 && x < 3 * lx / 4;
        nA[i] = in ? g[0] : g[2];
        nB[i] = in ? g[1] : g[3];
    }
    rc = scmc_set_density(s, nA.data(), nB.data());
    if (!rc) rc = scmc_set_graph_steps(s, 256);
    // sample row y = z = 2 (any row: the state stays transverse-uniform)
    const size_t row = ((size_t)(q.nz > 1 ? 2 : 0) * q.ny + 2) * q.nx;
    double prev[4] = {0, 0, 0, 0};
    int64_t done = 0;
    bool converged = false;
    while (!rc && !converged && done < max_steps) {
        const int64_t k = std::min<int64_t>(2048, max_steps - done);
        rc = flat_steps(s, k);
        if (!rc) rc = scmc_get_fields(s, nA.data(), nB.data(), nullptr);
        if (rc) break;
        done += k;
        const double cur[4] = {nA[row + lx / 2], nB[row + lx / 2], nA[row],
                               nB[row]};
        double d = 0;
        for (int c = 0; c < 4; ++c) {
            if (!std::isfinite(cur[c])) rc = SCMC_ENONFINITE;
            d = std::max(d, std::fabs(cur[c] - prev[c]));
            prev[c] = cur[c];
        }
        converged = done > k && d <= tol;
    }
    for (int c = 0; c < 4; ++c) out[c] = prev[c];
    if (steps) *steps = done;
    scmc_destroy(s);
    return rc;
}

// ------------------------------------------------------------------ batch
// Chunks of whole members for the batched moment two-pass (see scmc_batch),
// in the order of the two-pass tile list.  A member whose moment field
// reaches kBatchChunkBytes is a chunk of its own; the others join chunks, in
// their given order, until a chunk's moment fields would pass
// kBatchChunkBytes.
static constexpr size_t kBatchChunkBytes = (size_t)48 << 20;
// Chunks that together have at most this much make their moment steps in one
// launch: both fields of its members then stay in the Infinity Cache.  Longer
// launches fill the CUs more evenly and march longer chunks: us per step of
// twelve members of 48^3 to 88^3 (one group from 91 MB on) and of 48 members
// of 48^3 to 160^3, by MB per group: 48: 164, 2 526; 112: 145, 2 416; 224:
// 145, 2 435.  The two passes of every step took 271 and 5 190.
static constexpr size_t kBatchGroupBytes = (size_t)112 << 20;

static std::vector<std::vector<int>> two_pass_chunks(const std::vector<scmc_problem> &ps) {
    std::vector<std::vector<int>> out;
    size_t bytes = 0;
    bool open = false;  // the last chunk takes more members
    for (int i = 0; i < (int)ps.size(); ++i) {
        const scmc_problem &p = ps[i];
        const size_t mb = (size_t)6 * p.nx * p.ny * p.nz * real_bytes(p.storage);
        if (mb >= kBatchChunkBytes) {
            out.push_back({i});
            open = false;
            continue;
        }
        if (!open || bytes + mb > kBatchChunkBytes) {
            out.push_back({});
            bytes = 0;
            open = true;
        }
        out.back().push_back(i);
        bytes += mb;
    }
    return out;
}

static int batch_tiles(const std::vector<scmc_problem> &ps, int kernel,
                       const int *tile, std::vector<Tile> *out) {
    out->clear();
    if (kernel != SCMC_KERNEL_FUSED) {  // runs of 256 consecutive sites, chunk by chunk
        for (const std::vector<int> &chunk : two_pass_chunks(ps))
            for (int i : chunk) {
                const int N = ps[i].nx * ps[i].ny * ps[i].nz;
                for (int s0 = 0; s0 < N; s0 += 256) out->push_back({i, s0, 0, 0});
            }
        return (int)out->size();
    }
    for (int i = 0; i < (int)ps.size(); ++i) {
        const scmc_problem &p = ps[i];
        for (int z = 0; z < p.nz; z += tile[2])
            for (int y = 0; y < p.ny; y += tile[1])
                for (int x = 0; x < p.nx; x += tile[0]) out->push_back({i, x, y, z});
    }
    return (int)out->size();
}

// The launches of a two-pass step: pass 1 and then pass 2 of each chunk in
// turn (ops[2i] and ops[2i + 1]; several steps run chunk by chunk, see
// direct_steps_batch), so that pass 2 finds the chunk's moments still cached.  (Sharing a
// launch between pass 2 of one chunk and pass 1 of the next measured no
// faster.)  A chunk of one member runs the single-lattice kernels with that
// member's description as an argument (no per-block tile and member loads).
// The any-tau two passes run by the same chunks: 24 members of 64^3 E4 with psi,
// us per step over the whole list and by chunks, FP32 632, 593, BF16 478, 432.
// The fused designs (one persistent launch), two dimensions at tau != 1 and
// stochastic rounding (whose step counter advances at the first tile of
// pass 1) run the whole list at once.
static void batch_set_ops(scmc_batch *b) {
    const Common &c = b->c;
    b->ops.clear();
    b->groups.clear();
    if (c.kernel == SCMC_KERNEL_FUSED) return;
    std::vector<std::vector<int>> members_of;  // by chunk
    bool chunked = c.key.mom || c.key.dim == 3;
    for (const Lat &L : b->lats) chunked = chunked && !L.m.sr;
    std::vector<BatchOp> ops;
    if (chunked) {
        std::vector<scmc_problem> ps;
        for (const Lat &L : b->lats) ps.push_back(L.p);
        int t = 0;
        members_of = two_pass_chunks(ps);
        for (const std::vector<int> &chunk : members_of) {
            int n = 0;
            long sites = 0;
            for (int i : chunk) {
                n += (b->lats[i].m.N + 255) / 256;  // tiles of batch_tiles
                sites += b->lats[i].m.N;
            }
            BatchOp p1{1, t, n, pass1_nt_all(c.key, sites)}, p2{2, t, n};
            NodeLaunch probe{};
            if (chunk.size() == 1 &&
                node_member_pass(c.key, b->lats[chunk[0]].m, 1, false, &probe)) {
                p1.member = p2.member = chunk[0];
                p1.m = p2.m = b->lats[chunk[0]].m;
            }
            ops.push_back(p1);
            ops.push_back(p2);
            t += n;
        }
        if (t != b->ntiles) {
            ops.clear();
            members_of.clear();
        }
    }
    if (ops.empty()) ops = {{1, 0, b->ntiles}, {2, 0, b->ntiles}};
    b->ops = ops;
    if (members_of.size() * 2 != ops.size()) {  // the whole list, not by chunks
        b->groups.push_back(BatchGroup{0, ops.size(), 0});
        return;
    }
    // groups of consecutive chunks that share a moment step's launch
    for (size_t q = 0; q < members_of.size();) {
        BatchGroup g;
        g.op0 = 2 * q;
        g.member = members_of[q][0];
        std::vector<Member> ms;
        size_t bytes = 0;
        for (; q < members_of.size(); ++q) {
            size_t more = 0;
            for (int i : members_of[q]) more += (size_t)6 * b->lats[i].m.N * real_bytes(b->lats[i].p.storage);
            if (!ms.empty() && (bytes + more > kBatchGroupBytes ||
                                ms.size() + members_of[q].size() > (size_t)MOM_LIST))
                break;
            bytes += more;
            for (int i : members_of[q]) ms.push_back(b->lats[i].m);
        }
        g.op1 = 2 * q;
        for (const Member &m : ms) {
            g.sites += m.N;
            g.ragged += ragged_sites(m);
        }
        // a chunk of more than MOM_LIST members: full launches first (129 of 24^3:
        // 64, 64 and 1 fill 256 CUs in one round each, 43 three times in two)
        g.mom = c.key.mom;
        for (size_t m0 = 0; m0 < ms.size() && g.mom; m0 += MOM_LIST) {
            const size_t m1 = std::min(ms.size(), m0 + MOM_LIST);
            BatchGroup::Launch launch;
            double us = 0;
            g.mom = node_batch_mom_step(c.key, {ms.begin() + m0, ms.begin() + m1},
                                        g.member + (int)m0, &launch.node, &launch.list, &us);
            g.us += us;
            g.launches.push_back(launch);
        }
        b->groups.push_back(g);
    }
}

// Tile-list capacity: enough for the current design, for the smallest fused
// tile and for the two-pass tiling, so that the autotuner can switch design
// and tile inside the same workspace.
static int batch_tile_capacity(const std::vector<scmc_problem> &v, int kernel,
                               const int *tile) {
    std::vector<Tile> tiles;
    const int tmin[3] = {32, 2, 8}, none[3] = {0, 0, 0};
    int nt = batch_tiles(v, kernel, tile, &tiles);
    nt = std::max(nt, batch_tiles(v, SCMC_KERNEL_FUSED, tmin, &tiles));
    nt = std::max(nt, batch_tiles(v, SCMC_KERNEL_TWO_PASS, none, &tiles));
    return std::max(nt, 1);
}

static int batch_check(const scmc_problem *ps, int count, std::string *why) {
    if (!ps || count < 1) return SCMC_EINVAL;
    for (int i = 0; i < count; ++i) {
        int rc = validate(&ps[i], why);
        if (rc) return rc;
        if (node_storage(ps[i].storage)) {
            if (why) *why = "node storage runs on single lattices";
            return SCMC_EUNSUPPORTED;
        }
        if (ps[i].lattice != ps[0].lattice || ps[i].stencil != ps[0].stencil ||
            ps[i].storage != ps[0].storage || ps[i].tau[0] != ps[0].tau[0] ||
            ps[i].tau[1] != ps[0].tau[1] ||
            ps[i].psi_self != ps[0].psi_self || ps[i].kernel != ps[0].kernel ||
            ps[i].rounding != ps[0].rounding ||
            ps[i].tile[0] != ps[0].tile[0] || ps[i].tile[1] != ps[0].tile[1] ||
            ps[i].tile[2] != ps[0].tile[2])
            return SCMC_EINVAL;
    }
    return SCMC_OK;
}

int scmc_batch_workspace_bytes(const scmc_problem *ps, int count, size_t *out) {
    if (!out) return SCMC_EINVAL;
    int rc = batch_check(ps, count, nullptr);
    if (rc) return rc;
    std::vector<scmc_problem> v(ps, ps + count);
    int kernel, tile[3];
    StepKey k0 = key_of(ps[0]);
    for (int i = 1; i < count; ++i) k0.big |= key_of(ps[i]).big;
    rc = choose_kernel(ps[0], k0, &kernel, tile);
    if (rc) return rc;
    const int nt = batch_tile_capacity(v, kernel, tile);
    *out = plan_of(v, nt).total + align_up(count * sizeof(Member));
    return SCMC_OK;
}

int scmc_batch_create(const scmc_problem *ps, int count, void *d_ws,
                      size_t ws_bytes, void *stream, scmc_batch **out) {
    if (!out) return SCMC_EINVAL;
    *out = nullptr;
    std::string why;
    int rc = batch_check(ps, count, &why);
    if (rc) return rc;
    if (!d_ws || ((uintptr_t)d_ws % ALIGN)) return SCMC_EINVAL;
    size_t need;
    rc = scmc_batch_workspace_bytes(ps, count, &need);
    if (rc) return rc;
    if (ws_bytes < need) return SCMC_ENOSPACE;
    scmc_batch *b = new (std::nothrow) scmc_batch();
    if (!b) return SCMC_EINVAL;
    Common &c = b->c;
    std::vector<scmc_problem> v(ps, ps + count);
    c.key = key_of(ps[0]);
    for (int i = 1; i < count; ++i) c.key.big |= key_of(ps[i]).big;
    rc = choose_kernel(ps[0], c.key, &c.kernel, c.tile);
    if (rc) {
        delete b;
        return rc;
    }
    std::vector<Tile> tiles;
    const int nt_max = batch_tile_capacity(v, c.kernel, c.tile);
    b->ntiles = batch_tiles(v, c.kernel, c.tile, &tiles);
    b->ntiles_cap = nt_max;
    const Plan pl = plan_of(v, nt_max);
    c.stream = (hipStream_t)stream;
    c.ws = (char *)d_ws;
    c.ws_bytes = ws_bytes;
    int nbmax = 0;
    for (auto &p : v) nbmax = std::max(nbmax, stats_blocks(member_of(p)));
    bind(c, pl, c.ws, nbmax);
    char *tail = (char *)c.ctr + pl.ctr;
    b->d_members = (Member *)tail;
    tail += align_up(count * sizeof(Member));
    b->d_tiles = (Tile *)tail;
    // members: offsets into the shared buffers
    long long pop_off = 0, dens_off = 0;
    std::vector<Member> ms;
    for (int i = 0; i < count; ++i) {
        Lat L;
        L.p = v[i];
        L.m = member_of(v[i]);
        L.q = lattice_q(v[i].lattice);
        L.dim = lattice_dim(v[i].lattice);
        L.m.pop_off = pop_off;
        L.m.dens_off = dens_off;
        L.m.step_ctr = c.ctr;
        const size_t N = (size_t)L.m.N;
        pop_off += (long long)(align_up(2 * L.q * N * storage_bytes(v[i].storage)) /
                               storage_bytes(v[i].storage));
        dens_off += (long long)(align_up(7 * N * real_bytes(v[i].storage)) /
                                real_bytes(v[i].storage));
        ms.push_back(L.m);
        b->lats.push_back(L);
    }
    b->member_set.assign(count, false);
    int dev = 0, ncu = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess)
            ncu = prop.multiProcessorCount;
    }
    b->grid = std::min(b->ntiles, ncu * 8);
    batch_set_ops(b);
    hipError_t e = hipMemcpyAsync(b->d_members, ms.data(),
                                  ms.size() * sizeof(Member),
                                  hipMemcpyHostToDevice, c.stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->d_tiles, tiles.data(), tiles.size() * sizeof(Tile),
                           hipMemcpyHostToDevice, c.stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c.stream);
    if (e != hipSuccess) {
        delete b;
        return SCMC_EDEVICE;
    }
    *out = b;
    return SCMC_OK;
}

int scmc_batch_destroy(scmc_batch *b) {
    if (!b) return SCMC_EINVAL;
    const hipError_t e = hipStreamSynchronize(b->c.stream);  // as scmc_destroy
    drop_graphs(b->c);
    delete b;
    return e == hipSuccess ? SCMC_OK : SCMC_EDEVICE;
}

static const void *member_pop(const scmc_batch *b, int i, int buf) {
    const Lat &L = b->lats[i];
    return (const char *)b->c.pop[buf] +
           L.m.pop_off * (long long)storage_bytes(L.p.storage);
}

int scmc_batch_set_density(scmc_batch *b, int i, const double *nA,
                           const double *nB) {
    if (!b || !nA || !nB || i < 0 || i >= (int)b->lats.size())
        return SCMC_EINVAL;
    Common &c = b->c;
    if (c.step != 0 || (c.cur != 0 && c.initialized))
        return fail(c, SCMC_ESTATE, "members are set before the first step");
    int rc = set_density_impl(c, b->lats[i], nA, nB,
                              (void *)member_pop(b, i, 0));
    if (!rc) rc = set_step_counter(c, 0);
    if (rc) return rc;
    b->member_set[i] = true;
    c.initialized = std::all_of(b->member_set.begin(), b->member_set.end(),
                                [](bool v) { return v; });
    return SCMC_OK;
}

int scmc_batch_set_graph_steps(scmc_batch *b, int k) {
    if (!b || k < 0) return SCMC_EINVAL;
    drop_graphs(b->c);
    b->c.graph_k = k;
    return SCMC_OK;
}

int scmc_batch_step(scmc_batch *b, int64_t nsteps) {
    if (!b) return SCMC_EINVAL;
    Common &c = b->c;
    return run_steps(
        c, nsteps,
        [&](int par) {
            const std::vector<int> whole = {0, b->ntiles};
            return build_graph(c, c.graph_k, par, true, Member{}, b->d_members, b->d_tiles,
                               whole, b->grid,
                               c.kernel == SCMC_KERNEL_FUSED ? nullptr : b);
        },
        [&](int64_t k) { return direct_steps_batch(b, k); });
}

int scmc_batch_get_fields(scmc_batch *b, int i, double *nA, double *nB,
                          double *u) {
    if (!b || i < 0 || i >= (int)b->lats.size()) return SCMC_EINVAL;
    if (!b->c.initialized) return fail(b->c, SCMC_ESTATE, "state not set");
    return fields_impl(b->c, b->lats[i], member_pop(b, i, b->c.cur), nA, nB, u);
}

int scmc_batch_get_populations(scmc_batch *b, int i, double *f, int64_t *step) {
    if (!b || !f || i < 0 || i >= (int)b->lats.size()) return SCMC_EINVAL;
    if (!b->c.initialized) return fail(b->c, SCMC_ESTATE, "state not set");
    int rc = download_state(b->c, b->lats[i], member_pop(b, i, b->c.cur), f);
    if (rc) return rc;
    if (step) *step = b->c.step;
    return SCMC_OK;
}

int scmc_batch_stats_get(scmc_batch *b, int i, scmc_stats *out) {
    if (!b || i < 0 || i >= (int)b->lats.size()) return SCMC_EINVAL;
    if (!b->c.initialized) return fail(b->c, SCMC_ESTATE, "state not set");
    int rc = stats_impl(b->c, b->lats[i], member_pop(b, i, b->c.cur), out,
                        b->c.step);
    if (rc) return rc;
    if (out->n_nonfinite > 0)
        return fail(b->c, SCMC_ENONFINITE, "%.0f non-finite populations",
                    out->n_nonfinite);
    return SCMC_OK;
}

int scmc_batch_observables(scmc_batch *b, int i, int kind, double R0,
                           scmc_obs *out, double *PN, double *PT) {
    if (!b || i < 0 || i >= (int)b->lats.size()) return SCMC_EINVAL;
    if (!b->c.initialized) return fail(b->c, SCMC_ESTATE, "state not set");
    return obs_impl(b->c, b->lats[i], member_pop(b, i, b->c.cur), kind, R0,
                    out, PN, PT, b->c.step);
}

int scmc_batch_config(scmc_batch *b, int *tile, int *grid) {
    if (!b) return SCMC_EINVAL;
    if (tile)
        for (int a = 0; a < 3; ++a) tile[a] = b->c.tile[a];
    if (grid) *grid = b->grid;
    return SCMC_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- autotuner
namespace {

struct Candidate {
    int kernel;   // SCMC_KERNEL_FUSED or SCMC_KERNEL_TWO_PASS (internal)
    int variant;  // StepKey::repull (fused)
    int mom;      // StepKey::mom (two-pass)
    int tile[3];
};

// Designs this problem can run: for kernel AUTO the population-ring fused
// designs (plain and pipelined) over the compiled tiles and three z-chunk
// lengths and, at tau = 1, the moment-ring fused designs and the moment
// two-pass design, otherwise the any-tau two passes beside a fused design (by
// themselves they leave nothing to choose); for a fixed fused design, its tiles
// only.
std::vector<Candidate> candidates(const scmc_problem &p, const StepKey &k0, int nx) {
    static const int tiles[][2] = {{64, 4}, {32, 8},  {64, 8}, {32, 16},
                                   {128, 4}, {128, 8}, {64, 16}};
    static const int chunks[] = {8, 16, 32};
    const bool tau1 = tau_is_one(p);
    std::vector<int> variants;
    if (p.kernel == SCMC_KERNEL_AUTO) {
        variants = {0, 2};
        if (tau1) variants = {0, 2, 3, 4};
    } else {
        variants = {k0.repull};
    }
    std::vector<Candidate> out;
    if (p.rounding == SCMC_ROUND_STOCHASTIC) {  // two-pass designs only
        if (p.kernel == SCMC_KERNEL_AUTO && tau1) {
            out.push_back(Candidate{SCMC_KERNEL_TWO_PASS, 0, 1, {0, 0, 0}});
            if (k0.dim == 3 && !k0.big)
                out.push_back(Candidate{SCMC_KERNEL_TWO_PASS, 0, 2, {64, 8, 8}});
        }
        return out;
    }
    for (int variant : variants)
        for (const auto &t : tiles) {
            if (t[0] > 2 * nx) continue;  // mostly idle lanes
            for (int zc : chunks) {
                Candidate c{SCMC_KERNEL_FUSED, variant, 0, {t[0], t[1], zc}};
                StepKey k = k0;
                k.repull = variant;
                if (fused_supported(k, c.tile)) out.push_back(c);
            }
        }
    if (p.kernel == SCMC_KERNEL_AUTO && !tau1 && !out.empty())
        out.push_back(Candidate{SCMC_KERNEL_TWO_PASS, 0, 0, {0, 0, 0}});
    if (p.kernel == SCMC_KERNEL_AUTO && tau1) {
        out.push_back(Candidate{SCMC_KERNEL_TWO_PASS, 0, 1, {0, 0, 0}});
        if (k0.dim == 3 && !k0.big && p.storage != SCMC_F64)  // LDS-staged collision pass
            out.push_back(Candidate{SCMC_KERNEL_TWO_PASS, 0, 2, {64, 8, 8}});
    }
    return out;
}

std::string cache_key(const scmc_problem &p, int count) {
    char buf[256];
    snprintf(buf, sizeof buf,
             "lattice=%d stencil=%d storage=%d psi=%d rounding=%d tau1=%d kernel=%d "
             "box=%dx%dx%d members=%d",
             p.lattice, p.stencil, p.storage, p.psi_self, p.rounding, tau_is_one(p) ? 1 : 0,
             p.kernel, p.nx, p.ny, p.nz, count);
    return buf;
}

bool cache_lookup(const char *path, const std::string &key, Candidate *c);

bool same(const Candidate &a, const Candidate &b) {
    return a.kernel == b.kernel && a.variant == b.variant && a.mom == b.mom &&
           a.tile[0] == b.tile[0] && a.tile[1] == b.tile[1] && a.tile[2] == b.tile[2];
}

// a cached choice is used only if this problem can still run it
bool cached_choice(const char *path, const std::string &key,
                   const std::vector<Candidate> &cands, Candidate *c) {
    Candidate t;
    if (!cache_lookup(path, key, &t)) return false;
    for (const Candidate &x : cands)
        if (same(x, t)) {
            *c = t;
            return true;
        }
    return false;
}

bool cache_lookup(const char *path, const std::string &key, Candidate *c) {
    if (!path) return false;
    FILE *f = fopen(path, "r");
    if (!f) return false;
    char line[512];
    bool found = false;
    while (fgets(line, sizeof line, f)) {
        const char *sep = strstr(line, " -> ");
        if (!sep || std::string(line, sep - line) != key) continue;
        Candidate t;
        if (sscanf(sep + 4, "kernel=%d variant=%d mom=%d tile=%d,%d,%d", &t.kernel,
                   &t.variant, &t.mom, &t.tile[0], &t.tile[1], &t.tile[2]) == 6) {
            *c = t;  // the last entry for a key wins
            found = true;
        }
    }
    fclose(f);
    return found;
}

void cache_store(const char *path, const std::string &key, const Candidate &c,
                 double us) {
    if (!path) return;
    FILE *f = fopen(path, "a");
    if (!f) return;
    fprintf(f, "%s -> kernel=%d variant=%d mom=%d tile=%d,%d,%d  (%.2f us/step)\n",
            key.c_str(), c.kernel, c.variant, c.mom, c.tile[0], c.tile[1], c.tile[2], us);
    fclose(f);
}

// Time a call of `steps` steps, step(n), on the handle's stream, in
// microseconds per step.
template <class StepFn>
int time_steps(Common &c, int warm, int steps, StepFn step, double *us) {
    hipEvent_t e0, e1;
    HIPCHK(c, hipEventCreate(&e0));
    HIPCHK(c, hipEventCreate(&e1));
    int rc = step(warm);
    if (!rc) {
        (void)hipEventRecord(e0, c.stream);
        rc = step(steps);
        (void)hipEventRecord(e1, c.stream);
        (void)hipEventSynchronize(e1);
        float ms = 0;
        (void)hipEventElapsedTime(&ms, e0, e1);
        *us = 1e3 * ms / steps;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}

void apply(Common &c, const Candidate &cand) {
    c.kernel = cand.kernel;
    c.key.repull = cand.variant;
    c.key.mom = cand.mom;
    for (int a = 0; a < 3; ++a) c.tile[a] = cand.tile[a];
    drop_graphs(c);
}

}  // namespace

extern "C" {

int scmc_autotune(scmc_sim *s, const char *cache_path, int *tile) {
    if (!s) return SCMC_EINVAL;
    Common &c = s->c;
    const scmc_problem &p = s->lat.p;
    if (p.kernel == SCMC_KERNEL_TWO_PASS || p.kernel == SCMC_KERNEL_TWO_PASS_MOM)
        return fail(c, SCMC_EUNSUPPORTED, "the two-pass design has no tile to tune");
    std::vector<Candidate> cands = candidates(p, c.key, p.nx);
    if (cands.empty())
        return fail(c, SCMC_EUNSUPPORTED, "no fused kernel for this problem");
    const std::string key = cache_key(p, 1);
    Candidate best{};
    if (!cached_choice(cache_path, key, cands, &best)) {
        // scratch state: a uniform mixture at rest
        std::vector<double> nA(s->lat.m.N, 0.5), nB(s->lat.m.N, 0.5);
        int rc = set_density_impl(c, s->lat, nA.data(), nB.data(), c.pop[0]);
        if (rc) return rc;
        c.cur = 0;
        // 20 timed steps per candidate, in two rounds over the list, each
        // candidate's faster round counting: the designs closest in speed
        // differ by a few per cent, and a single round of timings has picked
        // one 8 % slower than the best (clock and cache state drift between
        // the first candidates and the last)
        std::vector<double> t(cands.size(), 1e300);
        for (int round = 0; round < 2; ++round)
            for (size_t i = 0; i < cands.size(); ++i) {
                apply(c, cands[i]);
                double us = 0;
                rc = time_steps(c, 4, 20, [&](int k) { return direct_steps_sim(s, k); }, &us);
                if (rc) return rc;
                t[i] = std::min(t[i], us);
            }
        const size_t ib = (size_t)(std::min_element(t.begin(), t.end()) - t.begin());
        best = cands[ib];
        const double best_us = t[ib];
        // The forms of the moment two-pass make the same moment steps and differ
        // in pass 2 alone, once per call: a call of 20 steps ranks them by noise
        // (96^3 E6 FP16: 18 us apart, 0.9 per step of 35).  They are ranked by
        // single steps, where they differ at every step.
        if (best.mom) {
            double least = 1e300;
            std::vector<double> one(cands.size(), 1e300);
            for (int round = 0; round < 2; ++round)
                for (size_t i = 0; i < cands.size(); ++i) {
                    if (!cands[i].mom) continue;
                    apply(c, cands[i]);
                    double us = 0;
                    rc = time_steps(c, 4, 20, [&](int k) {
                        int e = SCMC_OK;
                        for (int q = 0; q < k && !e; ++q) e = direct_steps_sim(s, 1);
                        return e;
                    }, &us);
                    if (rc) return rc;
                    one[i] = std::min(one[i], us);
                }
            for (size_t i = 0; i < cands.size(); ++i)
                if (one[i] < least) {
                    least = one[i];
                    best = cands[i];
                }
        }
        cache_store(cache_path, key, best, best_us);
        c.initialized = false;  // the scratch state is not the caller's
        c.step = 0;
        c.cur = 0;
    }
    apply(c, best);
    if (tile)
        for (int a = 0; a < 3; ++a) tile[a] = best.tile[a];
    return SCMC_OK;
}

int scmc_batch_autotune(scmc_batch *b, const char *cache_path, int *tile) {
    if (!b) return SCMC_EINVAL;
    Common &c = b->c;
    const scmc_problem &p0 = b->lats[0].p;
    if (p0.kernel == SCMC_KERNEL_TWO_PASS || p0.kernel == SCMC_KERNEL_TWO_PASS_MOM)
        return fail(c, SCMC_EUNSUPPORTED, "the two-pass design has no tile to tune");
    int nxmin = p0.nx;
    std::vector<scmc_problem> ps;
    for (const Lat &L : b->lats) {
        nxmin = std::min(nxmin, L.p.nx);
        ps.push_back(L.p);
    }
    std::vector<Candidate> cands = candidates(p0, c.key, nxmin);
    if (cands.empty())
        return fail(c, SCMC_EUNSUPPORTED, "no fused kernel for this batch");
    const std::string key = cache_key(p0, (int)b->lats.size());
    auto use = [&](const Candidate &cand) -> int {
        std::vector<Tile> tiles;
        const int nt = batch_tiles(ps, cand.kernel, cand.tile, &tiles);
        if (nt > b->ntiles_cap)
            return fail(c, SCMC_ENOSPACE, "tile list larger than planned");
        apply(c, cand);
        b->ntiles = nt;
        batch_set_ops(b);
        HIPCHK(c, hipMemcpyAsync(b->d_tiles, tiles.data(), nt * sizeof(Tile),
                                 hipMemcpyHostToDevice, c.stream));
        HIPCHK(c, hipStreamSynchronize(c.stream));
        return SCMC_OK;
    };
    Candidate best{};
    if (!cached_choice(cache_path, key, cands, &best)) {
        for (int i = 0; i < (int)b->lats.size(); ++i) {
            std::vector<double> nA(b->lats[i].m.N, 0.5), nB(b->lats[i].m.N, 0.5);
            int rc = set_density_impl(c, b->lats[i], nA.data(), nB.data(),
                                      (void *)member_pop(b, i, 0));
            if (rc) return rc;
        }
        c.cur = 0;
        double best_us = 1e300;
        for (const Candidate &cand : cands) {
            if (cand.tile[0] > 2 * nxmin) continue;
            int rc = use(cand);
            if (rc == SCMC_ENOSPACE) continue;
            if (rc) return rc;
            double us = 0;
            rc = time_steps(c, 1, 4, [&](int k) { return direct_steps_batch(b, k); }, &us);
            if (rc) return rc;
            if (us < best_us) {
                best_us = us;
                best = cand;
            }
        }
        cache_store(cache_path, key, best, best_us);
        c.initialized = false;
        c.step = 0;
        c.cur = 0;
        std::fill(b->member_set.begin(), b->member_set.end(), false);
    }
    int rc = use(best);
    if (rc) return rc;
    if (tile)
        for (int a = 0; a < 3; ++a) tile[a] = best.tile[a];
    return SCMC_OK;
}

}  // extern "C"
