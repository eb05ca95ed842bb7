"""Particles that enter one key from its neighbours in one step, up to 12 of them
(lists of at most 8 are ranked from registers in 2D, longer ones by walking): where
they are stored is a function of the layout they left, so a second run, whose
atomics may run in another order, gives the same bits, and the state agrees with
the oracle (1e-11 over the steps, as for the other chained steps)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_1603_06188_amd import scenes
from tests.test_gpu_parity import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("entering", [1, 2, 7, 8, 9, 12])
def test_entering(dim, entering):
    from paper_1603_06188_amd import binding as b

    cells, dt, steps = 16, 1e-2, 3
    rng = np.random.default_rng(100 * dim + entering)
    # particles of base nodes 6 and 8 along x that enter base node 7 (quadratic: the
    # key changes at half a cell), and slow ones there and about
    low = np.array([6.5, 5.5, 5.5])[:dim]
    xa = low + np.concatenate([np.c_[0.9 + 0.05 * rng.random(entering)], rng.random((entering, dim - 1))], axis=1)
    xb = np.array([6.5, 5.5, 5.5])[:dim] + rng.random((40, dim)) * np.array([3.0, 1.0, 1.0])[:dim]
    x = np.concatenate([xa, xb]) / cells
    v = np.concatenate([np.tile(np.eye(dim)[0] * 0.3 / cells / dt, (entering, 1)), np.zeros((40, dim))])
    tmpl = scenes.random_particles(x.shape[0], dim=dim, cells=cells, degree=2, seed=5, model=0, vel_sigma=0.0,
                                   b_sigma=0.0)
    s = dataclasses.replace(tmpl.with_state(x=x, v=v, B=np.zeros_like(tmpl.B)), dt=dt)
    runs = []
    for _ in range(2):
        ds = b.DeviceScene(s)
        ds.step(steps)
        runs.append(ds.state(raw=True))
        assert ds.flags() == 0
    for key in ("id", "cell", "off", "v", "B", "F", "m"):
        assert np.array_equal(runs[0][key], runs[1][key]), key
    got = ds.state()
    g = oracle.Grid(s.dim, s.degree, s.cells, s.dx)
    x, v, B, F = s.x, s.v, s.B, s.F
    for _ in range(steps):
        r = oracle.step(g, x, v, B, F, s.m, s.V, s.model, s.mu, s.lam, s.dt, s.gravity, s.band, transfer=s.transfer)
        x, v, B, F = r["x_new"], r["v_new"], r["B_new"], r["F_new"]
    assert float(np.abs(got["x"] - x).max() / s.dx) <= 1e-11
    for key, ref in (("v", v), ("B", B), ("F", F)):
        assert rel(got[key], ref) <= 1e-11, (key, rel(got[key], ref))
