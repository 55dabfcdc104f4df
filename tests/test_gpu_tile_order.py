"""The two-step launch through states larger than the memory-side cache (its
tiles' order alternates from launch to launch, the leading tiles' results are
streamed): the same state, to the bit, as launches of one step, on both sides
of each change of the streamed share, alone and in a batch."""
import numpy as np
import pytest

from slbm_workloads import configs as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slbm():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm as S
    S.lib()
    return S


# 160 (fp64) or 88 (fp32) bytes of state a site: below and above 250 and 500 MB
@pytest.mark.parametrize("precision,n", [("fp64", 1231), ("fp64", 1290), ("fp64", 1742), ("fp64", 1801),
                                         ("fp32", 1670), ("fp32", 1703), ("fp32", 2401)])
def test_large_plates_equal_single_steps(slbm, precision, n):
    p = P.moving_hole_plate(n)
    with slbm.Solver(p, precision) as a, slbm.Solver(p, precision) as b:
        b.set_launch(6, 62)
        for k, group in ((2, 0), (4, 8), (3, 0)):
            a.set_xcd_group(group)
            a.step(k)
            b.step(k)
        assert a.time() == b.time()
        assert np.array_equal(a.displacement(), b.displacement())
        for x, y in zip(a.moments(), b.moments()):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("precision,n", [("fp64", 700), ("fp64", 950), ("fp64", 1301), ("fp32", 1301)])
def test_large_batches_equal_single_steps(slbm, precision, n):
    p = P.square_clamped_pulled(n)
    solo = slbm.Solver(p, precision)
    solo.set_launch(6, 62)
    solo.step(7)
    b = slbm.Batch(8 << 30)
    slots = [b.add(p, 7, precision) for _ in range(3)]
    b.set_launch(10, 58)
    b.step(7)
    u = solo.displacement()
    for slot in slots:
        assert np.array_equal(b.solver(slot).displacement(), u)
    b.close()
    solo.close()
