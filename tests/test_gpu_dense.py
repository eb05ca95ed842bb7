"""Many particles in few tiles, above and below the particle count from which the
key pass has a wavefront per tile where the tiles are many or not so full."""
import dataclasses

import numpy as np
import pytest

from paper_1603_06188_amd import scenes

pytestmark = pytest.mark.gpu


def _b():
    from paper_1603_06188_amd import binding
    return binding


def _dense(dim, degree, precision, n, seed):
    """n particles in a square or cube of about 1,800 per tile, in motion."""
    te, cells = (4, 48) if dim == 3 else (8, 256)
    rng = np.random.default_rng(seed)
    s = scenes.random_particles(n, dim=dim, cells=cells, degree=degree, seed=seed, precision=precision, model=0,
                                vel_sigma=0.3, b_sigma=0.002 / cells)
    width = te * (n / 1800.0) ** (1.0 / dim)
    x = (5.3 + width * rng.random((n, dim))) / cells
    return dataclasses.replace(s.with_state(x=x, v=s.v + np.array([0.5, 0.3, -0.2])[:dim]), dt=5e-3)


def _rows(ds, live):
    ids = ds.id[:live].cpu().numpy()
    assert np.array_equal(np.sort(ids), np.arange(live))
    at = np.argsort(ids)
    return ds.f[:, :live].cpu().numpy()[:, at], ds.cell[:live].cpu().numpy()[at]


@pytest.mark.parametrize("dim,degree,precision", [(3, 2, "fp32"), (3, 3, "fp32"), (3, 1, "fp64"), (2, 2, "fp64")])
def test_same_bits_on_both_sides(dim, degree, precision):
    """The same particles, and with enough more without a position to be above."""
    b = _b()
    n, extra = (1 << 19) - 300, 500
    s = _dense(dim, degree, precision, n, seed=dim + degree)
    below = b.DeviceScene(s, with_id=True, compensated=True)
    more = s.subset(np.r_[np.arange(n), np.arange(extra)])
    above = b.DeviceScene(more, with_id=True, compensated=True)
    above.f[0, n:n + extra] = float("nan")
    above.sort()
    below.sort()
    cell0 = _rows(below, n)[1]
    for ds in (below, above):
        ds.step(3)
    got, want = _rows(above, n), _rows(below, n)
    assert np.count_nonzero(want[1] != cell0) > n // 100
    assert got[0].tobytes() == want[0].tobytes() and np.array_equal(got[1], want[1])


def test_same_bits_in_a_batch():
    b = _b()
    hosts = [_dense(3, 2, "fp32", 280000, seed=k) for k in range(2)]
    alone = b.DeviceScene(hosts[1], with_id=True, compensated=True)
    alone.step(3)
    batch = b.SceneBatch([b.DeviceScene(h, with_id=True, compensated=True) for h in hosts])
    batch.step(3)
    got, want = _rows(batch.scenes[1], hosts[1].n), _rows(alone, hosts[1].n)
    assert got[0].tobytes() == want[0].tobytes() and np.array_equal(got[1], want[1])
