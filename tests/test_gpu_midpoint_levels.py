"""The implicit step's elastic terms at numbers of particles per key that their
kernels walk differently: four wavefronts deal a tile's levels (none, some or all
of them have one), keys of one tile hold from none to all levels, and a support
reaches into the tiles beside.  Against the oracle at the binary64 bar."""
import pytest

from tests.test_gpu_levels import _scene
from tests.test_gpu_midpoint import SOLVER, TOL, _b, _compare, _oracle_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,degree", [(3, 2), (3, 3), (2, 2)])
@pytest.mark.parametrize("counts", [(1,), (3, 4, 5), (4, 8, 0, 9, 7, 16, 17), (33, 5, 70, 0, 1)],
                         ids=["one", "to5", "levels", "many"])
def test_levels(dim, degree, counts):
    s = _scene(dim, degree, "fp64", counts, seed=40 + len(counts))
    s.model = 1
    ds = _b().DeviceScene(s, midpoint=True)
    st = ds.step_midpoint(1, **SOLVER)
    x, v, B, F, ost = _oracle_chain(s, 1)
    print(st, ost, flush=True)
    assert st["flags"] == 0
    _compare(ds.state(), x, v, B, F, s.dx, TOL, f"midpoint {dim}d deg{degree} {counts}")
