"""The library's own launch (two steps per launch, rows by the plate's size)
against launches of one step: the same state, to the bit, for even and odd
step counts, on both sides of each change of the rows."""
import numpy as np
import pytest

from test_gpu_parity import mixed_plate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slbm():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm as S
    S.lib()
    return S


# 58-column strips x rows: 256 tiles of 2, 4, 6 or 8 rows and a row more
@pytest.mark.parametrize("shape,rows", [((40, 30), 2), ((232, 128), 2), ((232, 129), 4), ((464, 128), 4), ((465, 128), 6),
                                        ((928, 97), 8), ((929, 130), 10)])
@pytest.mark.parametrize("periodic", [False, True])
def test_default_launch_equals_single_steps(slbm, shape, rows, periodic):
    p = mixed_plate(*shape, seed=3, order=1, periodic=periodic)
    for prec in ("fp32", "fp64"):
        with slbm.Solver(p, prec) as a, slbm.Solver(p, prec) as b:
            assert a.launch() == (0, 0, 0) and a.boundary_lists()[0] == rows
            b.set_launch(6, 62)
            for n in (1, 2, 7, 10):
                a.step(n)
                b.step(n)
            a.sync()
            assert a.time() == b.time()
            assert np.array_equal(a.displacement(), b.displacement())
            for x, y in zip(a.moments(), b.moments()):
                assert np.array_equal(x, y)
            b.set_launch(0, 0)
            a.step(4)
            b.step(4)
            assert b.boundary_lists()[0] == rows and np.array_equal(a.displacement(), b.displacement())
