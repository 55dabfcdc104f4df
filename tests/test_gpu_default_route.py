"""How many steps a launch takes when it is left to the library: recorded into a
graph, which is not run, and counted, on both sides of the rule's lines, above
all for plates without tile lists; and the state of such plates, bit-equal to
launches of one step."""
import dataclasses

import numpy as np
import pytest

from bench import recorded_kernels
from slbm_workloads import configs
from slbm_workloads import geometry as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm
    slbm.lib()
    return torch, slbm


def bare(nx, ny):
    return G.periodic_box(nx, ny, lam=0.04, mu=0.05, tau=0.55, force=(1e-7, 2e-7))


def holed(n, _):
    """Lists in every tile."""
    return configs.hole_plate(n, n / 8, lam=0.05, tau=0.55)


def many_groups(n, _):
    """A hole, and more groups than the lists take."""
    p = holed(n, n)
    return dataclasses.replace(p, groups=list(p.groups) + [G.BCGroup(G.NEUMANN, (0.0, 0.0))] * 65)


def cut_up(nx, ny):
    """Full-width cracks every second row: more cut links in a tile than its list takes."""
    walls = G.edge_walls(nx, ny, left=0, right=1, bottom=1, top=1)
    walls += [G.HLine(y + 0.5, 1, x_lo=-0.5, x_hi=nx - 0.5) for y in range(1, ny - 2, 2)]
    return G.build_plate(nx, ny, lam=0.04, mu=0.05, tau=0.55, walls=walls,
                         groups=[G.BCGroup(G.DIRICHLET, (0.0, 0.0)), G.BCGroup(G.NEUMANN, (1e-5, 0.0))], neumann_order=0)


@pytest.mark.parametrize("make,shape,single,double", [
    (holed, (512, 512), 2, 2), (holed, (1024, 1024), 2, 2), (bare, (80, 60), 4, 4), (bare, (256, 256), 2, 2),
    (bare, (400, 400), 2, 2), (bare, (2048, 2048), 2, 2), (bare, (116, 4000), 2, 2), (bare, (124, 4000), 1, 2),
    (bare, (62, 4000), 1, 1), (bare, (62, 1000), 2, 2), (bare, (100000, 1), 1, 2), (bare, (20000, 5), 1, 2),
    (bare, (20000, 6), 2, 2), (many_groups, (256, 256), 2, 2), (many_groups, (512, 512), 1, 1),
    (many_groups, (1024, 1024), 1, 1), (many_groups, (2048, 2048), 2, 2), (cut_up, (701, 354), 1, 1),
])
def test_steps_of_a_launch(env, make, shape, single, double):
    torch, slbm = env
    p = make(*shape)
    for prec, steps in (("fp32", single), ("fp64", double)):
        stream = torch.cuda.Stream().cuda_stream
        with slbm.Solver(p, prec, stream=stream) as s:
            assert s.launch() == (0, 0, 0)
            s.step(2)
            s.sync()
            # 16 steps: an even number of launches, as single steps, whichever is taken
            assert len(recorded_kernels(slbm.lib(), stream, lambda: s.step(16))) == 16 // steps, prec


@pytest.mark.parametrize("make,shape", [(bare, (400, 400)), (bare, (20000, 1)), (bare, (20000, 3)), (bare, (5000, 8)),
                                        (bare, (62, 2000)), (many_groups, (300, 300)), (many_groups, (520, 520))])
def test_plates_without_lists_equal_single_steps(env, make, shape):
    torch, slbm = env
    p = make(*shape)
    rng = np.random.default_rng(4)
    vel = 1e-3 * rng.standard_normal((2, p.ny, p.nx)) * p.mask
    for prec in ("fp32", "fp64"):
        with slbm.Solver(p, prec) as a, slbm.Solver(p, prec) as b:
            b.set_launch(6, 62)
            for s in (a, b):
                s.init_fields(vel=vel)
                for n in (1, 2, 5):
                    s.step(n)
            assert np.array_equal(a.displacement(), b.displacement())
            assert np.array_equal(a.moments()[3], b.moments()[3])
