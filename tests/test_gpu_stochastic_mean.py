"""Stochastic rounding is unbiased about the value that a load gives back.

A load adds w_i n0 to the stored offset in one fused multiply-add, so the mean
of the stored offsets over many sites has to be f*_i - w_i n0 with the product
unrounded; an offset formed against the rounded product is off by the product's
rounding error, every step.  A uniform mixture at rest collides to the same
f*_i = w_i n everywhere, formed here in single precision as the step forms it.
The concentrations lie close to n0, so that one unit in the last place of an
offset, which sets the noise of the mean, is not much larger than that error:
2^-24 for FP16 (offsets in [2^-14, 2^-13), the smallest that round
stochastically) and for BF16 (offsets in [2^-17, 2^-16)).  With 2^18 sites the mean's
standard deviation is at most half a unit over 512; the bound is five of them.
"""
import numpy as np
import pytest

from paper_2112_02574_amd import scmc

pytestmark = pytest.mark.gpu

N0 = (0.52, 0.4703125)
f32 = np.float32


def _fma(a, b, c):
    """Single-precision fused multiply-add (the product is exact in FP64)."""
    return f32(np.float64(f32(a)) * np.float64(f32(b)) + np.float64(f32(c)))


@pytest.mark.parametrize("lattice,kernel,tile,tau", [
    (scmc.D3Q19, scmc.KERNEL_TWO_PASS_MOM, (0, 0, 0), 1.0),
    (scmc.D3Q19, scmc.KERNEL_TWO_PASS_MOM, (64, 8, 8), 1.0),
    (scmc.D3Q19, scmc.KERNEL_TWO_PASS, (0, 0, 0), 0.8), (scmc.D2Q9, scmc.KERNEL_TWO_PASS_MOM, (0, 0, 0), 1.0),
    (scmc.D2Q9, scmc.KERNEL_TWO_PASS, (0, 0, 0), 0.8)])
@pytest.mark.parametrize("storage", [scmc.F16_OFF, scmc.BF16_OFF])
def test_mean_offset(storage, lattice, kernel, tile, tau):
    shape = (64, 64, 64) if lattice == scmc.D3Q19 else (512, 512)
    p = scmc.problem(lattice, scmc.E4, shape, tau=tau, storage=storage, kernel=kernel, tile=tile,
                     n0=N0, rounding=scmc.ROUND_STOCHASTIC, seed=11)
    xi, w = scmc.velocities(lattice)
    q = len(w)
    wf, n0 = w.astype(f32), np.array(N0, dtype=f32)
    low, unit = (2.0 ** -14 if storage == scmc.F16_OFF else 2.0 ** -17), 2.0 ** -24
    for weight in np.unique(wf[1:]):  # offsets of 1.4 low in the directions with this weight
        n = [n0[J] + 1.4 * low / weight for J in range(2)]
        s = scmc.Sim(p)
        s.scmc_set_density(*(np.full(shape, v) for v in n))
        h0 = _offsets(s, wf, n0)
        s.scmc_step(1)
        h1 = _offsets(s, wf, n0)
        s.close()
        for J in range(2):
            f = [_fma(wf[i], n0[J], h0[J, i].flat[0]) for i in range(q)]
            total = f32(sum(np.float64(v) for v in f))
            omega = f32(1.0 / tau)
            keep, on = f32(1) - omega, omega * total
            for i in np.flatnonzero(wf == weight):
                if i == 0:
                    continue  # closes the node's mass, in another rounding
                want = wf[i] * total if tau == 1.0 else _fma(keep, f[i], f32(wf[i] * on))
                offset = np.float64(want) - np.float64(wf[i]) * np.float64(n0[J])
                assert low <= offset < 2 * low
                err = h1[J, i].mean() - offset
                assert abs(err) < 5 * 0.5 * unit / 512, (J, i, err / unit)


def _offsets(s, w, n0):
    """Stored offsets, exactly: the host adds the rounded single-precision
    product to them in FP64."""
    f, _ = s.scmc_get_populations()
    f = f.reshape(2, len(w), -1)
    return f - (w[None, :] * n0[:, None]).astype(np.float64)[:, :, None]
