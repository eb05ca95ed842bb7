"""The transfers at every number of particles per key the level walks treat
differently: the block of wavefronts that takes a tile walks its levels in
groups of four or eight, tiles whose busiest key holds more than 32 particles
are stored key by key, and keys of one tile may hold from none to all of them.
One step against the oracle at the bars of the parity tests (binary64 1e-12,
binary32 1e-5 relative per field)."""
import numpy as np
import pytest

from paper_1603_06188_amd import scenes
from tests.test_gpu_parity import TOL, compare_step

pytestmark = pytest.mark.gpu


def _b():
    from paper_1603_06188_amd import binding
    return binding


def _scene(dim, degree, precision, counts, seed, transfer=0):
    """counts[i] particles in the i-th of a run of base nodes that starts in one
    tile and ends in the next, the others empty."""
    rng = np.random.default_rng(seed)
    cells, dx = 16, 1.0 / 16
    low = 0.5 if degree == 2 else 1.0       # offset of a key's cell corner from its base node, in cells
    xs = []
    for i, c in enumerate(counts):
        base = np.array([3 + i % 3, 3 + (i // 3) % 3, 3 + i // 9][:dim], dtype=np.float64)
        xs.append((base + low + 0.02 + 0.96 * rng.random((c, dim))) * dx)
    x = np.concatenate(xs)
    n = x.shape[0]
    s = scenes.random_particles(n, dim=dim, cells=cells, degree=degree, seed=seed, precision=precision,
                                f_sigma=0.05, b_sigma=0.002, vel_sigma=0.3, dt=1e-4)
    s = s.with_state(x=x)
    s.transfer = transfer
    return s


@pytest.mark.parametrize("precision,compensated", [("fp64", False), ("fp64", True), ("fp32", False), ("fp32", True)])
@pytest.mark.parametrize("dim,degree", [(3, 2), (3, 3), (2, 2)])
@pytest.mark.parametrize("counts", [(1,), (1, 2, 3, 4, 5), (4, 8, 0, 9, 7, 16, 17), (32, 1, 31, 2), (33, 5, 70, 0, 1)],
                         ids=["one", "to5", "groups", "full32", "busy"])
def test_levels(dim, degree, precision, compensated, counts):
    s = _scene(dim, degree, precision, counts, seed=len(counts) + 10 * dim + degree)
    ds = _b().DeviceScene(s, compensated=compensated)
    compare_step(s, ds, TOL[precision], label=f"{dim}d deg{degree} {precision} {counts}")
