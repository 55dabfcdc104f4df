"""Up to four steps per launch (small plates under the library's own launch)
against launches of one step: the same state, to the bit, for every number of
steps a launch can take, around the edges of its tiles (50 columns, 2 rows,
256 tiles) and with more periods in a tile's reach than one."""
import numpy as np
import pytest

from slbm_workloads import geometry as G
from test_gpu_parity import mixed_plate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slbm():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm as S
    S.lib()
    return S


@pytest.mark.parametrize("shape", [(12, 9), (50, 16), (51, 17), (100, 101), (101, 100), (150, 170), (150, 171), (500, 25)])
@pytest.mark.parametrize("periodic", [False, True])
def test_four_steps_equal_single_steps(slbm, shape, periodic):
    p = mixed_plate(*shape, seed=5, order=1, periodic=periodic)
    for prec in ("fp32", "fp64"):
        with slbm.Solver(p, prec) as a, slbm.Solver(p, prec) as b:
            b.set_launch(6, 62)
            for n in (1, 2, 3, 4, 5, 11):
                a.step(n)
                b.step(n)
            a.sync()
            assert a.time() == b.time()
            assert np.array_equal(a.displacement(), b.displacement())
            for x, y in zip(a.moments(), b.moments()):
                assert np.array_equal(x, y)


def test_no_cut_links_and_changes_of_the_launch(slbm):
    p = G.build_plate(70, 60, lam=0.04, mu=0.05, tau=0.55, walls=[], groups=[], force=(1e-6, -2e-6),
                      periodic_x=True, periodic_y=True, name="bare")
    rng = np.random.default_rng(2)
    v = 1e-3 * rng.standard_normal((2, 60, 70))
    with slbm.Solver(p, "fp64") as a, slbm.Solver(p, "fp64") as b:
        b.set_launch(6, 62)
        for s in (a, b):
            s.init_fields(vel=v)
        for rows, strip in ((0, 0), (4, 58), (0, 0), (6, 64), (0, 0)):
            a.set_launch(rows, strip)
            a.step(5)
            b.step(5)
        a.autotune()
        a.step(6)
        b.step(6)
        assert np.array_equal(a.displacement(), b.displacement())
