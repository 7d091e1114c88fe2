"""The flat interface stepped as one row of nodes against the full lattice.

scmc_flat_equilibrium steps a state uniform along y and z on a single row
(up to 512 nodes; longer rows and other cases run the full lattice).  The same
box stepped by the tau-general two-pass design from the same profile must give
the same row.  Both round every population the same number of times per step;
they add populations and stencil terms in another order and contract other
products, so they differ by a few rounding errors per step, and the errors
neither grow nor decay much over 37 steps of a smooth relaxation.  Bounds, for
values of about 2: 37 steps x 19 populations x 2 ulp = 37 * 19 * 2 * 2.2e-16 =
3e-13 in FP64 and 37 * 19 * 2 * 1.2e-7 = 1.7e-4 in FP32.  The 16-bit offsets
(below 1 in size) round to 2^-12 and 2^-9; one population per node and step may
fall on the other side of a rounding boundary: 37 * 2^-12 and 37 * 2^-9.
"""
import numpy as np
import pytest

from paper_2112_02574_amd import scmc

pytestmark = pytest.mark.gpu

TOL = {scmc.F64: 3e-13, scmc.F32: 1.7e-4, scmc.F16_OFF: 37 * 2.0 ** -12, scmc.BF16_OFF: 37 * 2.0 ** -9}
GUESS = (1.05, 0.05, 0.04, 0.98)
STEPS = 37


def _full(p, lattice, lx):
    """Two-pass steps of the whole box; returns (n_A, n_B) of a row."""
    shape = (5, lx) if lattice == scmc.D2Q9 else (5, 5, lx)
    q = scmc.problem(lattice, p.stencil, shape,
                     g=((p.g[0][0], p.g[0][1]), (p.g[1][0], p.g[1][1])), psi_self=p.psi_self,
                     storage=p.storage, kernel=scmc.KERNEL_TWO_PASS)
    q.tau[0], q.tau[1] = p.tau[0], p.tau[1]
    x = np.arange(lx)
    inside = (x >= lx // 4) & (x < 3 * lx // 4)
    nA = np.broadcast_to(np.where(inside, GUESS[0], GUESS[2]), shape).copy()
    nB = np.broadcast_to(np.where(inside, GUESS[1], GUESS[3]), shape).copy()
    s = scmc.Sim(q)
    s.scmc_set_density(nA, nB)
    s.scmc_step(STEPS)
    n = s.scmc_get_fields()
    s.close()
    return n.reshape(2, -1, lx)[:, 2]


@pytest.mark.parametrize("storage", list(TOL))
@pytest.mark.parametrize("lattice,stencil,psi", [
    (scmc.D3Q19, 4, scmc.PSI_EXP_NEG_INV), (scmc.D3Q19, 6, scmc.PSI_N),
    (scmc.D2Q9, 4, scmc.PSI_N), (scmc.D2Q9, 6, scmc.PSI_EXP_NEG_INV), (scmc.D2Q9, 8, scmc.PSI_N)])
@pytest.mark.parametrize("tau", [(1.0, 1.0), (0.8, 0.8), (0.7, 1.2)])
def test_row_equals_full_lattice(storage, lattice, stencil, psi, tau):
    g = ((-0.2, 1.8), (1.8, -0.1)) if psi == scmc.PSI_N else ((-1.0, 0.9), (0.9, -0.8))
    for lx in (2 * (1 if stencil == 4 else 2) + 1, 31, 32, 127, 512, 513):
        shape = (5, lx) if lattice == scmc.D2Q9 else (5, 5, lx)
        p = scmc.problem(lattice, stencil, shape, g=g, psi_self=psi, storage=storage)
        p.tau[0], p.tau[1] = tau
        row = _full(p, lattice, lx)
        want = [row[0, lx // 2], row[1, lx // 2], row[0, 0], row[1, 0]]
        flat = dict(lx=lx, guess=GUESS, max_steps=STEPS, tol=0.0)
        if not np.isfinite(want).all():  # a narrow box can blow up: then both do
            with pytest.raises(scmc.ScmcError):
                scmc.scmc_flat_equilibrium(p, **flat)
            continue
        got, steps = scmc.scmc_flat_equilibrium(p, **flat)
        assert steps == STEPS
        np.testing.assert_allclose(got, want, rtol=0, atol=TOL[storage], err_msg=f"lx = {lx}")
