"""Steps recorded into a graph: each replay advances the state by the steps
recorded, for every even number of them, whatever number of launches the
library takes for them, with eager steps in between; bit-equal to eager steps."""
import numpy as np
import pytest

from slbm_workloads import box3d as B
from slbm_workloads import geometry as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm, slbm3
    slbm.lib()
    return torch, slbm, slbm3


def check(torch, make, n):
    stream = torch.cuda.Stream()
    a, b = make(stream.cuda_stream), make(stream.cuda_stream)
    a.step(3)
    a.sync()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        a.step(n)
    a.step(4)
    b.step(7)
    for k in range(3):
        with torch.cuda.stream(stream):
            g.replay()
        stream.synchronize()
        b.step(n)
        assert np.array_equal(a.displacement(), b.displacement()), k
    a.step(5)
    b.step(5)
    assert np.array_equal(a.displacement(), b.displacement())
    a.close()
    b.close()


# plates of up to four steps per launch, and of two; no wall changes with time
@pytest.mark.parametrize("shape", [(80, 60), (300, 200)])
@pytest.mark.parametrize("n", [2, 4, 6, 8, 10, 12])
def test_plates(env, shape, n):
    torch, slbm, _ = env
    nx, ny = shape
    p = G.build_plate(nx, ny, lam=0.04, mu=0.05, tau=0.55, walls=[G.Circle(nx * 0.45, ny * 0.55, ny * 0.18, 0)],
                      groups=[G.BCGroup(G.DIRICHLET, (0.0, 0.0))], force=(1e-6, -2e-6),
                      periodic_x=True, periodic_y=True, name="held")
    check(torch, lambda s: slbm.Solver(p, "fp32", stream=s), n)


# one launch per step, slab and cut links
@pytest.mark.parametrize("kind", ["slab", "cavities"])
def test_boxes(env, kind):
    torch, _, slbm3 = env
    box = (B.slab3(96, 96, 96, B.Wall3(B.DIRICHLET), B.Wall3(B.NEUMANN, (5e-5, 0, 0)), lam=.04, mu=.05, tau=.55)
           if kind == "slab" else B.cavities_box3(128, per_axis=2))
    check(torch, lambda s: slbm3.Solver3(box, "fp32" if kind == "slab" else "fp64", stream=s), 2)
