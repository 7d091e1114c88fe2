"""Blocks of steps on the moment field (D3Q19, tau = 1) against single steps.

A call of k >= 2 steps reads the populations once, stays in the moment field
for k - 1 steps and stores populations once; a call of one step runs pass 1
and pass 2, which the other tests check against the oracle.  Both form every
population and every sum from the same operations in the same order, so their
populations are equal bit for bit: the tolerance is zero.
"""
import numpy as np
import pytest

from paper_2112_02574_amd import inputs, scmc

pytestmark = pytest.mark.gpu

ASYM = ((-0.2, 1.8), (1.8, 0.0))
PAPER = ((-1.478, 0.5), (0.5, -1.2))


def _problem(shape, stencil, storage, psi=scmc.PSI_N, g=ASYM):
    return scmc.problem(scmc.D3Q19, stencil, shape, g=g, psi_self=psi, storage=storage)


def _state(shape, seed=5):
    nz, ny, nx = shape
    nA, nB = inputs.droplet(nx, ny, nz, R=max(2.0, min(shape) / 4))
    n = nA.size
    noise = [1 + 1e-3 * (2 * inputs.splitmix64_uniform_array(seed + t, n) - 1).reshape(nA.shape)
             for t in range(2)]
    return nA * noise[0], nB * noise[1]


def _run(p, state, calls, graph=0):
    s = scmc.Sim(p)
    s.scmc_set_density(*state)
    if graph:
        s.scmc_set_graph_steps(graph)
    for k in calls:
        s.scmc_step(k)
    f = s.scmc_get_populations()
    n = s.scmc_get_fields()
    s.close()
    return f[0] if isinstance(f, tuple) else f, n


# smallest extents, one column, several columns with remainders in x, y and z,
# rows longer than a column's plane holds
SHAPES = {4: [(3, 3, 3), (4, 7, 5), (9, 33, 67), (5, 3, 300), (40, 5, 8)],
          6: [(5, 5, 5), (6, 9, 7), (19, 35, 66), (7, 5, 261), (33, 21, 20)]}
STORAGES = [scmc.F64, scmc.F32, scmc.F16_OFF, scmc.BF16_OFF, scmc.F16_NODE, scmc.BF16_NODE]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("stencil", [4, 6])
@pytest.mark.parametrize("psi,g", [(scmc.PSI_N, ASYM), (scmc.PSI_EXP_NEG_INV, PAPER)])
def test_block_equals_single_steps(storage, stencil, psi, g):
    for shape in SHAPES[stencil]:
        p, st = _problem(shape, stencil, storage, psi, g), _state(shape)
        f1, n1 = _run(p, st, [1] * 5)
        f5, n5 = _run(p, st, [5])
        np.testing.assert_array_equal(f5, f1, err_msg=str(shape))
        np.testing.assert_array_equal(n5, n1, err_msg=str(shape))
        f4, _ = _run(p, st, [2, 3])
        np.testing.assert_array_equal(f4, f1, err_msg=str(shape))


@pytest.mark.parametrize("storage", [scmc.F64, scmc.F32, scmc.F16_NODE])
def test_block_graph_equals_single_steps(storage):
    shape = (21, 30, 45)
    p, st = _problem(shape, 6, storage), _state(shape)
    f1, _ = _run(p, st, [1] * 13)
    fg, _ = _run(p, st, [7, 6], graph=3)  # two replays and a single step, then two more
    np.testing.assert_array_equal(fg, f1)


def test_block_large_lattice_equals_single_steps():
    """Many columns and chunks, moments beyond the slab threshold of FP16."""
    shape = (190, 176, 180)
    for storage in (scmc.F32, scmc.F16_OFF):
        p, st = _problem(shape, 6, storage), _state(shape)
        f1, _ = _run(p, st, [1] * 3)
        f3, _ = _run(p, st, [3])
        assert np.array_equal(f3, f1)


def _batch_equals_singles(shapes, storage, calls, stencil=6, graph=0):
    ps = [_problem(s, stencil, storage) for s in shapes]
    b = scmc.Batch(ps)
    for i, s in enumerate(shapes):
        b.scmc_batch_set_density(i, *_state(s, seed=7 + i))
    if graph:
        b.scmc_batch_set_graph_steps(graph)
    for k in calls:
        b.scmc_batch_step(k)
    for i, s in enumerate(shapes):
        _, n = _run(ps[i], _state(s, seed=7 + i), [1] * sum(calls))
        assert np.array_equal(b.scmc_batch_get_fields(i), n), (i, s)
    b.close()


@pytest.mark.parametrize("storage", [scmc.F64, scmc.F32, scmc.F16_OFF])
@pytest.mark.parametrize("graph", [0, 2])
def test_batch_block_equals_single_steps(storage, graph):
    """Ragged members in one launch; odd and even blocks from both buffers."""
    _batch_equals_singles([(5, 5, 5), (24, 31, 40), (33, 20, 70), (9, 9, 100)], storage, [3, 4], graph=graph)
    _batch_equals_singles([(3, 3, 3), (12, 40, 7)], storage, [5], stencil=4, graph=graph)


def test_batch_groups_equal_single_steps():
    """Members beyond one group (112 MB of moments, 64 members): the second
    field of a group lies in its own part of the other population buffer."""
    _batch_equals_singles([(128, 128, 130), (128, 128, 128), (90, 128, 128), (20, 20, 20)],
                          scmc.F16_OFF, [3])
    _batch_equals_singles([(5 + i % 3, 6, 7) for i in range(70)], scmc.F32, [3])


SHAPES_2D = {4: [(3, 3), (4, 70), (64, 64), (33, 130)], 6: [(5, 5), (64, 7), (61, 67)],
             8: [(5, 6), (40, 41), (200, 257)]}


@pytest.mark.parametrize("storage", [scmc.F64, scmc.F32, scmc.F16_OFF, scmc.BF16_OFF])
@pytest.mark.parametrize("stencil", [4, 6, 8])
@pytest.mark.parametrize("psi,g", [(scmc.PSI_N, ASYM), (scmc.PSI_EXP_NEG_INV, PAPER)])
def test_block_2d_equals_single_steps(storage, stencil, psi, g):
    """Blocks shorter and longer than a launch's steps, direct and in graphs."""
    for shape in SHAPES_2D[stencil]:
        p = scmc.problem(scmc.D2Q9, stencil, shape, g=g, psi_self=psi, storage=storage)
        nA, nB = inputs.droplet(shape[1], shape[0], R=max(2.0, min(shape) / 4))
        noise = [1 + 1e-3 * (2 * inputs.splitmix64_uniform_array(3 + t, nA.size) - 1).reshape(nA.shape)
                 for t in range(2)]
        st = (nA * noise[0], nB * noise[1])
        f1, n1 = _run(p, st, [1] * 21)
        f2, n2 = _run(p, st, [2, 19])
        np.testing.assert_array_equal(f2, f1, err_msg=str(shape))
        np.testing.assert_array_equal(n2, n1, err_msg=str(shape))
        f3, _ = _run(p, st, [14, 7], graph=5)
        np.testing.assert_array_equal(f3, f1, err_msg=str(shape))
