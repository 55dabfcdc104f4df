"""Steps recorded into a graph, and the launch changed afterwards: the graph's
replays still take the steps they were recorded with, whatever set_launch and
the autotuner did to the plate's tile lists since, bit-equal to eager steps."""
import dataclasses

import numpy as np
import pytest

from slbm_workloads import geometry as G
from test_gpu_parity import mixed_plate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm
    slbm.lib()
    return torch, slbm


def record(torch, stream, call):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        call()
    return g


def replay(torch, stream, g):
    with torch.cuda.stream(stream):
        g.replay()
    stream.synchronize()


def plate(shape):
    """Edges, a hole and a crack; no load that changes with time, which a graph
    would repeat as recorded."""
    p = mixed_plate(*shape, seed=4, order=1, periodic=False)
    return dataclasses.replace(p, groups=[dataclasses.replace(g, profile=G.PROFILE_STEP) for g in p.groups])


# a plate of two steps per launch from tile lists, and a small one of four
@pytest.mark.parametrize("shape", [(300, 200), (70, 60)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_lists_outlive_a_change_of_the_launch(env, shape, prec):
    torch, slbm = env
    p = plate(shape)
    stream = torch.cuda.Stream()
    with slbm.Solver(p, prec, stream=stream.cuda_stream) as a, slbm.Solver(p, prec, stream=stream.cuda_stream) as b:
        b.set_launch(6, 62)
        a.step(4)
        b.step(4)
        g = record(torch, stream, lambda: a.step(8))
        changes = [lambda: a.set_launch(5, 58), a.autotune, lambda: a.set_launch(7, 58), lambda: a.set_launch(0, 0),
                   lambda: a.set_launch(6, 62)]
        for k, change in enumerate(changes):
            change()
            replay(torch, stream, g)
            a.step(4)
            replay(torch, stream, g)
            b.step(20)
            assert np.array_equal(a.displacement(), b.displacement()), k
        # no more are kept than those recorded from, and they are taken up again
        held = []
        for _ in range(3):
            for shape2 in ((5, 58), (7, 58), (0, 0)):
                a.set_launch(*shape2)
            held.append(a.device_bytes())
        assert held[0] == held[1] == held[2]
        del g


# launches of two steps asked for or found by the autotuner: an odd number of
# them would leave the state in the other buffer than the replay begins from
@pytest.mark.parametrize("rows", [4, 10, None])
@pytest.mark.parametrize("n", [2, 4, 6, 8, 10])
def test_two_steps_per_launch_recorded(env, rows, n):
    torch, slbm = env
    p = plate((300, 200))
    stream = torch.cuda.Stream()
    with slbm.Solver(p, "fp32", stream=stream.cuda_stream) as a, slbm.Solver(p, "fp32", stream=stream.cuda_stream) as b:
        b.set_launch(6, 62)
        if rows is None:
            a.autotune()
        else:
            a.set_launch(rows, 58)
        a.step(3)
        b.step(3)
        g = record(torch, stream, lambda: a.step(n))
        for k in range(3):
            replay(torch, stream, g)
            a.step(2)
            b.step(n + 2)
            assert np.array_equal(a.displacement(), b.displacement()), k
        a.step(5)
        b.step(5)
        assert np.array_equal(a.displacement(), b.displacement())
        del g


# a readout alone in a graph reads the buffer of its recording: eager steps in
# between leave the state there after every even number, as single steps do
@pytest.mark.parametrize("shape,launch", [((300, 200), (0, 0)), ((70, 60), (0, 0)), ((300, 200), (6, 58))])
@pytest.mark.parametrize("n", [2, 4, 6, 8, 10])
def test_readouts_recorded(env, shape, launch, n):
    torch, slbm = env
    p = plate(shape)
    stream = torch.cuda.Stream()
    new = lambda k: torch.zeros((k, p.ny, p.nx), dtype=torch.float64, device="cuda")
    u, v, rho, sig = new(2), new(2), new(1), new(3)
    torch.cuda.synchronize()
    with slbm.Solver(p, "fp64", stream=stream.cuda_stream) as a, slbm.Solver(p, "fp64", stream=stream.cuda_stream) as b:
        b.set_launch(6, 62)
        a.set_launch(*launch)
        a.step(3)
        b.step(3)
        g = [record(torch, stream, lambda: a.displacement_device(u.data_ptr())),
             record(torch, stream, lambda: a.displacement_device_noalloc(v.data_ptr())),
             record(torch, stream, lambda: a.moments_device(rho=rho.data_ptr(), sigma=sig.data_ptr()))]
        for k in range(2):
            a.step(n)
            b.step(n)
            for one in g:
                replay(torch, stream, one)
            m = b.moments()
            assert np.array_equal(u.cpu().numpy(), b.displacement()) and torch.equal(u, v), k
            assert np.array_equal(rho.cpu().numpy()[0], m[0]) and np.array_equal(sig.cpu().numpy(), m[3]), k
        del g, one


def test_back_to_the_librarys_launch_while_recording(env):
    """set_launch(0, 0) needs no device work of its own: it may be called
    between recorded steps."""
    torch, slbm = env
    p = plate((300, 200))
    stream = torch.cuda.Stream()
    with slbm.Solver(p, "fp32", stream=stream.cuda_stream) as a, slbm.Solver(p, "fp32", stream=stream.cuda_stream) as b:
        b.set_launch(6, 62)
        a.set_launch(10, 58)
        a.step(3)
        b.step(3)

        def call():
            a.set_launch(0, 0)
            a.step(4)

        g = record(torch, stream, call)
        for _ in range(2):
            replay(torch, stream, g)
            b.step(4)
        a.step(5)
        b.step(5)
        assert np.array_equal(a.displacement(), b.displacement())
        del g
