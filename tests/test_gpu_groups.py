"""The transfer to grid forms the terms of a tile's particles 64 at a time, over
groups of four levels (binary64 cubic: eight): tiles whose groups are full, lack
one particle, or go one past, against the oracle at the bars of the parity tests."""
import numpy as np
import pytest

from paper_1603_06188_amd import scenes
from tests.test_gpu_parity import TOL, compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree,precision,compensated", [(2, "fp32", True), (2, "fp32", False), (2, "fp64", False),
                                                          (3, "fp32", True), (3, "fp64", False), (3, "fp64", True)])
@pytest.mark.parametrize("per_key,drop", [(1, 63), (1, 1), (1, 0), (4, 1), (4, 0), (5, 63), (8, 1), (8, 0), (9, 31)])
def test_groups(degree, precision, compensated, per_key, drop):
    """per_key particles in each of the 64 keys of one tile, the last `drop` of them
    left out."""
    from paper_1603_06188_amd import binding as b

    rng = np.random.default_rng(10 * per_key + drop)
    low = 0.5 if degree == 2 else 1.0
    base = 4 + np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    base = np.concatenate([base] * per_key)[:64 * per_key - drop]
    x = (base + low + 0.02 + 0.96 * rng.random(base.shape)) / 16
    s = scenes.random_particles(x.shape[0], dim=3, cells=16, degree=degree, seed=per_key, precision=precision,
                                f_sigma=0.05, b_sigma=0.002, vel_sigma=0.3, dt=1e-4).with_state(x=x)
    perm = rng.permutation(s.n)
    ds = b.DeviceScene(s.subset(perm), compensated=compensated)
    compare_step(s.subset(perm), ds, TOL[precision], label=f"deg{degree} {precision} {per_key} {drop}")
