"""The one-pass plate readout at the edges of its tiles (62 columns; 2, 6 or
14 rows by the plate's size) against the reference."""
import pytest

from oracle import Oracle
from test_gpu_parity import compare, mixed_plate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slbm():
    import torch
    assert torch.cuda.is_available()
    from paper_2208_04088_amd import slbm as S
    S.lib()
    return S


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("shape", [(61, 42), (62, 41), (63, 43),          # 2 rows a tile, one strip and one column more
                                   (124, 150), (125, 133),               # 6 rows, whole tiles and one row more
                                   (620, 434), (621, 435)])              # 14 rows
def test_readout_at_tile_edges(slbm, shape, periodic):
    p = mixed_plate(*shape, seed=shape[0], periodic=periodic)
    for prec, steps in (("fp64", 0), ("fp64", 7), ("fp32", 8)):
        ref = Oracle(p, extended=True)
        ref.step(steps)
        with slbm.Solver(p, prec) as s:
            s.step(steps)
            compare(s, ref, prec)
