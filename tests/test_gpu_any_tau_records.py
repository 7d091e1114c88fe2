"""The any-tau two passes on per-site records against the generic kernels.

A single D3Q19 lattice of the TWO_PASS design keeps one record per site
(concentrations, and psi where it is not n); a batch of the same lattices runs
the generic tile-list kernels, which take psi of every stencil neighbour.  Both
form the same operations in the same order: equal bit for bit.
"""
import numpy as np
import pytest

from paper_2112_02574_amd import inputs, scmc

pytestmark = pytest.mark.gpu

# smallest extents, fewer and more sites than a block of 256, ragged rows
SHAPES = {4: [(3, 3, 3), (5, 7, 9), (13, 6, 70)], 6: [(5, 5, 5), (6, 7, 9), (9, 33, 20)]}


@pytest.mark.parametrize("storage", [scmc.F64, scmc.F32, scmc.F16_OFF, scmc.BF16_OFF])
@pytest.mark.parametrize("stencil", [4, 6])
@pytest.mark.parametrize("psi,g", [(scmc.PSI_N, ((-0.2, 1.8), (1.8, 0.0))),
                                   (scmc.PSI_EXP_NEG_INV, ((-1.478, 0.5), (0.5, 0.0)))])
@pytest.mark.parametrize("tau", [(0.8, 0.8), (0.9, 1.2)])
def test_records_equal_generic_kernels(storage, stencil, psi, g, tau):
    ps, states = [], []
    for shape in SHAPES[stencil]:
        nz, ny, nx = shape
        p = scmc.problem(scmc.D3Q19, stencil, shape, g=g, psi_self=psi, storage=storage,
                         kernel=scmc.KERNEL_TWO_PASS)
        p.tau[0], p.tau[1] = tau
        nA, nB = inputs.droplet(nx, ny, nz, R=max(2.0, min(shape) / 4))
        u = inputs.splitmix64_uniform_array(13, nA.size).reshape(nA.shape)
        ps.append(p)
        states.append((nA * (1 + 1e-3 * u), nB * (1 - 1e-3 * u)))
    b = scmc.Batch(ps)
    for i, st in enumerate(states):
        b.scmc_batch_set_density(i, *st)
    b.scmc_batch_step(4)
    for i, st in enumerate(states):
        for graph in (0, 2):
            s = scmc.Sim(ps[i])
            s.scmc_set_density(*st)
            s.scmc_set_graph_steps(graph)
            s.scmc_step(4)
            np.testing.assert_array_equal(s.scmc_get_fields(), b.scmc_batch_get_fields(i),
                                          err_msg=str(SHAPES[stencil][i]))
            s.close()
    b.close()
