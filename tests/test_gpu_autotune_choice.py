"""What the autotuner chooses from."""
import pytest

from paper_2112_02574_amd import scmc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("storage,shape", [(scmc.F64, (24, 24, 24)), (scmc.F32, (24, 24, 12))])
def test_nothing_to_choose_is_refused(storage, shape):
    """At tau != 1 without a fused design (FP64, or rows shorter than half the
    narrowest tile) the two passes are the only design."""
    p = scmc.problem(scmc.D3Q19, scmc.E6, shape, tau=0.8, storage=storage)
    for make, tune in ((lambda: scmc.Sim(p), "scmc_autotune"),
                       (lambda: scmc.Batch([p, p]), "scmc_batch_autotune")):
        s = make()
        with pytest.raises(scmc.ScmcError) as e:
            getattr(s, tune)()
        assert e.value.status == -2
        s.close()


@pytest.mark.parametrize("L", [48, 96])
def test_moment_designs_are_ranked_by_their_passes(L):
    """The LDS-staged pass 2 makes a single step 1.4 to 3 times as long at these
    sizes, which a call of 20 steps shows by 3 to 10 % only."""
    p = scmc.problem(scmc.D3Q19, scmc.E6, (L, L, L), storage=scmc.F16_OFF)
    for _ in range(3):
        s = scmc.Sim(p)
        s.scmc_autotune()
        kernel, tile = s.scmc_config()
        s.close()
        assert kernel != scmc.KERNEL_TWO_PASS_MOM or tuple(tile) == (0, 0, 0)
