"""Which boxes take a step in one launch (k3_march) and which in two: recorded
into a graph, which is not run, and counted.  On both sides of the rule's lines:
thin boxes, round pores, faces and short last chunks."""
import numpy as np
import pytest

from bench import recorded_kernels
from slbm_workloads import box3d as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm3
    slbm3.lib()
    return torch, slbm3


def launches(env, box, prec):
    """Launches of a step."""
    torch, slbm3 = env
    stream = torch.cuda.Stream().cuda_stream
    with slbm3.Solver3(box, prec, stream=stream) as s:
        s.step(2)
        s.sync()
        many, few = (recorded_kernels(slbm3.lib(), stream, lambda: s.step(k)) for k in (6, 4))
    return (len(many) - len(few)) / 2


PRESSED = [B.BCGroup3(B.NEUMANN, (0.0, 0.0, 0.0), 1e-5)]
COMMON = dict(lam=0.05, mu=0.05, tau=0.7, groups=PRESSED)


def slab(*d):
    return B.slab3(*d, B.Wall3(B.DIRICHLET), B.Wall3(B.NEUMANN, (5e-5, 0, 0)), lam=0.04, mu=0.05, tau=0.55)


def periodic(*d):
    return B.periodic_box3(*d, lam=0.04, force=(1e-7, 2e-7, 0))


def block(nx, ny, nz):
    return B.block_box3(nx, ny, nz, (1, 1, 1), (nx - 2, ny - 2, nz - 2), [0] * 6, PRESSED, lam=0.05, mu=0.05, tau=0.7)


def cavity(*d):
    r = 0.3 * min(d)
    return B.sphere_box3(*d, [B.Sphere3(d[0] / 2 - 0.4, d[1] / 2 - 0.3, d[2] / 2 - 0.6, r, 0)], PRESSED, lam=0.05, mu=0.05,
                         tau=0.7)


def crack(nx, ny, nz):
    return B.sphere_box3(nx, ny, nz, [], PRESSED, lam=0.05, mu=0.05, tau=0.7,
                         cracks=[B.PennyCrack3(nx / 2 + 0.3, ny / 2 + 0.1, 0.5, 0.2 * min(nx, ny), 0, 0)])


# (box, fp32, fp64): slower in one launch unless 1
@pytest.mark.parametrize("make,d,single,double", [
    (slab, (128, 128, 128), 1, 1), (periodic, (128, 128, 128), 1, 1), (periodic, (64, 64, 64), 2, 2),
    (slab, (1024, 1, 1024), 2, 2), (periodic, (1024, 1, 1024), 2, 2), (slab, (700, 2, 700), 2, 2),
    (periodic, (700, 2, 700), 1, 1), (slab, (400, 3, 800), 1, 1), (slab, (1024, 1024, 1), 2, 2),
    (periodic, (1024, 1024, 1), 2, 2), (slab, (1024, 1024, 2), 1, 2), (slab, (1024, 1024, 4), 1, 1),
    (slab, (400, 9, 240), 2, 1), (slab, (400, 8, 270), 1, 1),
    (cavity, (128, 128, 128), 1, 1), (cavity, (136, 136, 136), 2, 2), (cavity, (144, 144, 144), 2, 1),
    (cavity, (160, 160, 160), 1, 1), (crack, (1024, 1024, 3), 2, 2), (crack, (1024, 1024, 6), 1, 1),
    (slab, (130, 100, 100), 1, 1), (slab, (66, 150, 150), 2, 1), (periodic, (150, 100, 100), 2, 1),
    (periodic, (100, 150, 150), 1, 1), (slab, (96, 150, 150), 1, 1), (slab, (130, 200, 200), 2, 1),
    (periodic, (90, 200, 200), 2, 1), (slab, (190, 150, 150), 1, 1), (slab, (50, 300, 300), 1, 1),
    (cavity, (130, 200, 200), 2, 1), (cavity, (70, 260, 260), 2, 2), (cavity, (180, 180, 180), 1, 1),
    (block, (1024, 8, 512), 2, 2), (block, (512, 34, 256), 2, 2), (block, (160, 160, 160), 2, 2),
])
def test_launches_of_a_step(env, make, d, single, double):
    box = make(*d)
    assert launches(env, box, "fp32") == single
    assert launches(env, box, "fp64") == double


# k3_march's last template argument: its stores pass the caches by
@pytest.mark.parametrize("d,single,double", [((96, 96, 96), False, True), ((120, 150, 140), True, True),
                                             ((160, 160, 160), True, True), ((190, 150, 150), False, True),
                                             ((50, 300, 300), False, True), ((52, 240, 240), False, True),
                                             ((48, 300, 300), True, True)])
def test_stores_of_the_one_launch_step(env, d, single, double):
    torch, slbm3 = env
    for box in (slab(*d), periodic(*d)):
        for prec, streamed in (("fp32", single), ("fp64", double)):
            stream = torch.cuda.Stream().cuda_stream
            with slbm3.Solver3(box, prec, stream=stream) as s:
                s.step(2)
                s.sync()
                name = recorded_kernels(slbm3.lib(), stream, lambda: s.step(1))[-1]
            assert "k3_march" in name and ("Lb1EEE" in name) == streamed, (prec, name)
