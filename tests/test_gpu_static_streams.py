"""Allocation-free steps at tau != 1 on two streams at once.

AUTO takes the fused design there, which keeps no field in the array that
the two-pass calls of a GPU share, so steps of two lattices that overlap on
two streams give what each lattice's own handle gives alone, bit for bit.
"""
import numpy as np
import pytest

from paper_2112_02574_amd import inputs, scmc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STEPS = 20


@pytest.mark.parametrize("storage", [scmc.F32, scmc.F16_OFF, scmc.BF16_OFF])
@pytest.mark.parametrize("stencil,psi,g", [(6, scmc.PSI_N, ((-0.2, 1.8), (1.8, 0.0))),
                                           (4, scmc.PSI_EXP_NEG_INV, ((-1.478, 0.5), (0.5, -1.2)))])
def test_overlapping_streams(storage, stencil, psi, g):
    lattices = []
    for shape in ((40, 40, 40), (31, 48, 70)):
        p = scmc.problem(scmc.D3Q19, stencil, shape, tau=0.8, g=g, psi_self=psi, storage=storage)
        nz, ny, nx = shape
        nA, nB = inputs.droplet(nx, ny, nz, R=8.0)
        q = scmc.problem(scmc.D3Q19, stencil, shape, tau=0.8, g=g, psi_self=psi, storage=storage,
                         kernel=scmc.KERNEL_FUSED)
        alone = scmc.Sim(q)
        alone.scmc_set_density(nA, nB)
        n = scmc.state_bytes(p)
        src = alone.ws[:n].clone()
        alone.scmc_step(STEPS)  # even: the state is back in the first buffer
        alone.scmc_synchronize()
        want = alone.ws[:n].clone()
        alone.close()
        lattices.append(dict(p=p, bufs=[src, torch.empty_like(src)], want=want,
                             stream=torch.cuda.Stream()))
    torch.cuda.synchronize()
    for k in range(STEPS):
        for c in lattices:
            a, b = c["bufs"][k % 2], c["bufs"][1 - k % 2]
            scmc.scmc_step_static(c["p"], a, b, c["stream"])
    torch.cuda.synchronize()
    for c in lattices:
        assert torch.equal(c["bufs"][0], c["want"]), (c["p"].nz, c["p"].ny, c["p"].nx)
