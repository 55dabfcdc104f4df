"""The one-launch 3-D step on boxes large enough to take it, ragged against
its 64-site chunks, its rows and its planes.  The box repeats a small one's
field periodically in y and z, so the reference steps the small one and every
repetition must match it."""
import numpy as np
import pytest

from oracle.slbm3d import Oracle3D
from slbm_workloads import box3d as B
from test_gpu_parity3d import FP32_TOL, FP64_TOL, S3, check  # noqa: F401  (S3: the fixture)

pytestmark = pytest.mark.gpu

DT = np.sqrt(1.0 / (3 * 0.05))


def box_of(kind, nx, ny, nz):
    if kind == "periodic":
        return B.periodic_box3(nx, ny, nz, lam=0.04, mu=0.05, tau=0.6, force=(1e-6, -2e-6, 0.5e-6))
    moving = B.Wall3(B.DIRICHLET, (1e-4, -5e-5, 2e-5), q=0.3, profile=B.RAMP, ramp_time=5 * DT)
    pulled = B.Wall3(B.NEUMANN, (5e-5, 1e-5, -2e-5), q=0.8)
    walls = (moving, pulled) if kind == "slab" else (pulled, moving)
    return B.slab3(nx, ny, nz, *walls, lam=0.04, mu=0.05, tau=0.6, force=(1e-6, -2e-6, 0.5e-6))


# (kind, nx, repetitions of 9 x 5 in y and z): whole chunks; one site more (its
# wall is the halo column of the last chunk); a short last chunk; one chunk
@pytest.mark.parametrize("prec,tol", [("fp64", FP64_TOL), ("fp32", FP32_TOL)])
@pytest.mark.parametrize("kind,nx,ry,rz", [("slab", 128, 13, 14), ("slab", 65, 15, 22), ("flipped", 131, 11, 15),
                                           ("slab", 61, 19, 18), ("periodic", 128, 13, 15), ("periodic", 67, 16, 20)])
def test_large_boxes_match_the_reference(S3, kind, nx, ry, rz, prec, tol):  # noqa: F811
    ny, nz = 9, 5
    small, big = box_of(kind, nx, ny, nz), box_of(kind, nx, ny * ry, nz * rz)
    assert big.n_sites >= 850000
    vel = B.random_velocity(small, 17, 1e-3)
    tile = lambda v: np.tile(v, (1, rz, ry, 1))
    ref = Oracle3D(small, extended=(prec == "fp64"))
    ref.init_fields(vel=vel)
    ref.step(7)
    with S3.Solver3(big, prec) as s:
        s.init_fields(vel=tile(vel))
        s.step(4)
        saved = s.save()
        s.step(3)
        s.sync()
        u, (rho, j, P, sig) = s.displacement(), s.moments()
        s.load(saved)                                       # the walls' parts are formed anew from the state
        s.step(3)
        assert np.array_equal(u, s.displacement())
    rr, jr, Pr, sr = ref.moments()
    check((u, (rho, j, P, sig)), (tile(ref.displacement()), (tile(rr[None])[0], tile(jr), tile(Pr), tile(sr))), tol,
          f"{kind} {nx} {prec}", big)


# states on the other side of 250 MB, where the stores change: fp64 below, fp32 above
@pytest.mark.parametrize("kind,nx,ry,rz,prec,tol", [("slab", 65, 9, 14, "fp64", FP64_TOL), ("flipped", 128, 13, 26, "fp32", FP32_TOL),
                                                    ("periodic", 129, 13, 23, "fp32", FP32_TOL)])
def test_both_kinds_of_stores_match_the_reference(S3, kind, nx, ry, rz, prec, tol):  # noqa: F811
    ny, nz = 9, 5
    small, big = box_of(kind, nx, ny, nz), box_of(kind, nx, ny * ry, nz * rz)
    state = big.n_sites * (38 * (8 if prec == "fp64" else 4) + 24)
    assert big.n_sites >= 250000 and (state < 250e6) == (prec == "fp64")
    vel = B.random_velocity(small, 19, 1e-3)
    tile = lambda v: np.tile(v, (1, rz, ry, 1))
    ref = Oracle3D(small, extended=(prec == "fp64"))
    ref.init_fields(vel=vel)
    ref.step(6)
    with S3.Solver3(big, prec) as s:
        s.init_fields(vel=tile(vel))
        s.step(6)
        s.sync()
        got = s.displacement(), s.moments()
    rr, jr, Pr, sr = ref.moments()
    check(got, (tile(ref.displacement()), (tile(rr[None])[0], tile(jr), tile(Pr), tile(sr))), tol, f"{kind} {nx} {prec}", big)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_one_launch_equals_two(S3, prec):  # noqa: F811
    """A mask without void takes the two launches: the same state as the
    periodic box's one launch, to the bit."""
    box = box_of("periodic", 71, 113, 108)
    geo = B.Box3(**{**box.__dict__, "mask": np.ones((box.nz, box.ny, box.nx), np.uint8),
                    "links": np.zeros(0, B.LINK3_DTYPE), "groups": []})
    vel = B.random_velocity(box, 5, 1e-3)
    res = []
    for b in (box, geo):
        with S3.Solver3(b, prec) as s:
            s.init_fields(vel=vel)
            s.step(6)
            s.sync()
            res.append((s.displacement(), *s.moments()))
    for x, y in zip(*res):
        np.testing.assert_array_equal(x, y)


def solid(nx, order):
    """A small solid: a pressurised and a moving cavity, one across the edge of
    the first 64-site chunk where there is one, and a loaded crack whose rows
    have more than 64 cut links; ramps."""
    ramp = lambda n: dict(profile=B.RAMP, ramp_time=n * DT)
    groups = [B.BCGroup3(B.NEUMANN, (0.0, 0.0, 0.0), 2e-4, **ramp(5)), B.BCGroup3(B.DIRICHLET, (1e-4, -5e-5, 2e-5)),
              B.BCGroup3(B.NEUMANN, (2e-5, 0.0, 1e-5)), B.BCGroup3(B.NEUMANN, (0.0, 1e-5, -3e-5), **ramp(3))]
    far = 64.3 if nx > 64 else 48.3
    spheres = [B.Sphere3(9.3, 8.2, 7.1, 4.2, 0), B.Sphere3(far, 9.6, 7.7, 3.9, 1)]
    return B.sphere_box3(nx, 27, 16, spheres, groups, lam=0.05, mu=0.05, tau=0.7, neumann_order=order,
                         force=(1e-6, -2e-6, 0.5e-6), cracks=[B.PennyCrack3(28.4, 13.2, 8.5, 11.6, 2, 3)])


def repeated(box, ry, rz):
    """The box repeated in y and z, its links with it."""
    ny, nz, nx = box.ny * ry, box.nz * rz, box.nx
    L, parts = box.links, []
    z, r = np.divmod(L["site"].astype(np.int64), box.ny * nx)
    y, x = np.divmod(r, nx)
    for j in range(rz):
        for i in range(ry):
            c = L.copy()
            c["site"] = ((z + j * box.nz) * ny + (y + i * box.ny)) * nx + x
            parts.append(c)
    links = np.concatenate(parts)
    links = links[np.lexsort((links["dir"], links["site"]))]
    return B.Box3(**{**box.__dict__, "ny": ny, "nz": nz, "links": links, "mask": np.tile(box.mask, (rz, ry, 1))})


@pytest.mark.parametrize("prec,tol", [("fp64", FP64_TOL), ("fp32", FP32_TOL)])
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("nx,ry,rz", [(60, 8, 11), (64, 8, 10), (128, 5, 8), (130, 9, 9)])
def test_large_solids_match_the_reference(S3, nx, ry, rz, order, prec, tol):  # noqa: F811
    small = solid(nx, order)
    big = repeated(small, ry, rz)
    assert big.n_sites >= 2000000
    vel = B.random_velocity(small, 23, 1e-3) * small.mask
    tile = lambda v: np.tile(v, (1, rz, ry, 1))
    ref = Oracle3D(small, extended=(prec == "fp64"))
    ref.init_fields(vel=vel)
    ref.step(6)
    with S3.Solver3(big, prec) as s:
        s.init_fields(vel=tile(vel))
        s.step(3)
        saved = s.save()
        s.step(3)
        s.sync()
        u, (rho, j, P, sig) = s.displacement(), s.moments()
        s.load(saved)
        s.step(3)
        assert np.array_equal(u, s.displacement())
    rr, jr, Pr, sr = ref.moments()
    check((u, (rho, j, P, sig)), (tile(ref.displacement()), (tile(rr[None])[0], tile(jr), tile(Pr), tile(sr))), tol,
          f"solid {nx} order {order} {prec}", big)
