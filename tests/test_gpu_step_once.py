"""One step of a small lattice in one launch against the two passes.

Small D3Q19 lattices at tau = 1 make a single step in one launch; graphs of one
step always run pass 1 and pass 2, which form the same operations in the same
order: the populations are equal bit for bit.
"""
import numpy as np
import pytest

from paper_2112_02574_amd import inputs, scmc

pytestmark = pytest.mark.gpu

# smallest extents, exact boxes, remainders in every direction, the largest
# lattices that take one launch and the first that do not
SHAPES = {4: [(3, 3, 3), (4, 4, 8), (5, 7, 9), (13, 6, 33), (32, 32, 32), (40, 40, 40), (41, 40, 40)],
          6: [(5, 5, 5), (8, 8, 8), (6, 7, 9), (24, 24, 24), (13, 33, 5), (32, 32, 32), (33, 32, 32)]}


@pytest.mark.parametrize("storage", [scmc.F64, scmc.F32, scmc.F16_OFF, scmc.BF16_OFF])
@pytest.mark.parametrize("stencil", [4, 6])
@pytest.mark.parametrize("psi,g", [(scmc.PSI_N, ((-0.2, 1.8), (1.8, 0.0))),
                                   (scmc.PSI_EXP_NEG_INV, ((-1.478, 0.5), (0.5, -1.2)))])
def test_one_launch_equals_two_passes(storage, stencil, psi, g):
    for shape in SHAPES[stencil]:
        nz, ny, nx = shape
        p = scmc.problem(scmc.D3Q19, stencil, shape, g=g, psi_self=psi, storage=storage)
        nA, nB = inputs.droplet(nx, ny, nz, R=max(2.0, min(shape) / 4))
        u = inputs.splitmix64_uniform_array(9, nA.size).reshape(nA.shape)
        out = []
        for graph in (0, 1):
            s = scmc.Sim(p)
            s.scmc_set_density(nA * (1 + 1e-3 * u), nB * (1 - 1e-3 * u))
            s.scmc_set_graph_steps(graph)
            for _ in range(3):
                s.scmc_step(1)
            out.append(s.scmc_get_populations()[0])
            s.close()
        np.testing.assert_array_equal(out[0], out[1], err_msg=str(shape))
