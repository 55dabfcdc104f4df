"""A plate left to the library's launch on a device without room for its tile
lists: creation and set_launch(0, 0) succeed and the steps take the rules site
by site, bit-equal to single steps; lists that are asked for (strip 58) are
refused, and the plate goes on."""
import numpy as np
import pytest

from slbm_workloads import geometry as G

pytestmark = pytest.mark.gpu


def pinholes(n):
    """One void site in every 8 x 8 block of an n x n periodic plate: few
    sites with cut links, all over it, so that its tile lists are large."""
    mask = np.ones((n, n), dtype=np.uint8)
    mask[4::8, 4::8] = 0
    parts = []
    for k, (cx, cy) in enumerate([(1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)], 1):
        y, x = np.nonzero((mask == 1) & (np.roll(mask, (-cy, -cx), axis=(0, 1)) == 0))
        r = np.zeros(len(y), dtype=G.LINK_DTYPE)
        r["site"], r["dir"], r["q"], r["group2"] = y * n + x, k, 0.5, -1
        r["normal"] = np.array([cx, cy]) / np.hypot(cx, cy)
        parts.append(r)
    links = np.concatenate(parts)
    links = links[np.lexsort((links["dir"], links["site"]))]
    return G.Plate(nx=n, ny=n, lam=0.04, mu=0.05, rho=1.0, tau=0.55, mask=mask, links=links,
                   groups=[G.BCGroup(G.DIRICHLET, (0.0, 0.0))], force=(1e-6, -2e-6), periodic_x=True, periodic_y=True,
                   name="pinholes", neumann_order=0)


BLOCK = 32 << 20


def fill(torch, room):
    """Takes all device memory but about `room` bytes: blocks until no more is
    had, less what the room asks for."""
    held = [torch.empty(torch.cuda.mem_get_info()[0] - (2 << 30), dtype=torch.uint8, device="cuda")]
    for _ in range(400):
        try:
            held.append(torch.empty(BLOCK, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            break
    else:
        pytest.skip("the device's memory does not end")
    del held[len(held) - room // BLOCK:]
    torch.cuda.empty_cache()
    return held


def test_no_room_for_the_tile_lists():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm
    p = pinholes(1600)
    with slbm.Solver(p, "fp64") as ref:
        ref.set_launch(6, 62)
        ref.step(7)
        want = ref.displacement()
    torch.zeros(1, device="cuda")
    free = torch.cuda.mem_get_info()[0]
    with slbm.Solver(p, "fp64") as s:
        assert s.boundary_lists()[0] == 10
        used = free - torch.cuda.mem_get_info()[0]
        lists = s.boundary_lists()[1] * 140
    assert used > 4e8 and lists > 2 * BLOCK, (used, lists)
    held = fill(torch, used - lists // 2)
    with slbm.Solver(p, "fp64") as s:
        assert s.boundary_lists() == (0, 0, 0)
        held.clear()
        torch.cuda.empty_cache()
        s.step(3)
        held = fill(torch, lists // 2)
        with pytest.raises(slbm.SlbmError) as e:
            s.set_launch(9, 58)
        assert e.value.code == -2, e.value
        s.set_launch(0, 0)
        held.clear()
        torch.cuda.empty_cache()
        s.step(4)
        assert np.array_equal(s.displacement(), want)
        s.set_launch(0, 0)
        assert s.boundary_lists()[0] == 10


def test_no_room_to_autotune():
    """The trials' larger lists are refused: the error leaves the launch, its
    lists and the state as they were."""
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm
    p = pinholes(1600)
    with slbm.Solver(p, "fp64") as s, slbm.Solver(p, "fp64") as ref:
        ref.set_launch(6, 62)
        s.step(3)
        s.autotune()                               # its scratch is there
        s.set_launch(0, 0)
        lists = s.boundary_lists()
        assert lists[0] == 10
        held = fill(torch, BLOCK)
        with pytest.raises(slbm.SlbmError) as e:
            s.autotune()
        assert e.value.code == -2, e.value
        assert s.boundary_lists() == lists and s.launch()[:2] == (0, 0)
        held.clear()
        torch.cuda.empty_cache()
        s.step(4)
        ref.step(7)
        assert np.array_equal(s.displacement(), ref.displacement())
