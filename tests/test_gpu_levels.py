"""The transfers at every number of particles per key the level walks treat
differently: the block of wavefronts that takes a tile walks its levels in
groups of four or eight, tiles whose busiest key holds more than 32 particles
are stored key by key, and keys of one tile may hold from none to all of them.
One step against the oracle at the bars of the parity tests (binary64 1e-12,
binary32 1e-5 relative per field)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_1603_06188_amd import scenes
from tests.test_gpu_parity import TOL, compare_step, rel

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


@pytest.mark.parametrize("dim,degree", [(3, 2), (3, 3), (2, 2)])
@pytest.mark.parametrize("crowd", [24, 60])
def test_movers_of_crowded_tiles(dim, degree, crowd):
    """Chained steps of a cloud with about `crowd` particles per key whose
    particles change key by the tenth every step: marks of many levels (24) and
    tiles stored key by key that their particles enter and leave (60), against
    the oracle in binary64 (1e-11 over the steps)."""
    b = _b()
    cells, steps, width = 16, 4, 3.0 if dim == 3 else 5.0
    n = int(crowd * width ** dim)
    s = scenes.random_particles(n, dim=dim, cells=cells, degree=degree, seed=crowd + dim + degree, model=0,
                                vel_sigma=0.3, b_sigma=0.002)
    rng = np.random.default_rng(crowd)
    x = (5.3 + width * rng.random((n, dim))) / cells
    s = dataclasses.replace(s.with_state(x=x, v=s.v + np.array([1.5, 1.0, -0.7])[:dim]), dt=1e-2)
    ds = b.DeviceScene(s)
    ds.step(steps)
    got = ds.state()
    g = oracle.Grid(s.dim, s.degree, s.cells, s.dx)
    x, v, B, F = s.x, s.v, s.B, s.F
    shift = 0.5 if degree == 2 else 0.0
    moved = 0
    for _ in range(steps):
        r = oracle.step(g, x, v, B, F, s.m, s.V, s.model, s.mu, s.lam, s.dt, s.gravity, s.band, transfer=s.transfer)
        moved += int(np.count_nonzero((np.floor(r["x_new"] / s.dx - shift) != np.floor(x / s.dx - shift)).any(axis=1)))
        x, v, B, F = r["x_new"], r["v_new"], r["B_new"], r["F_new"]
    assert moved > n // 10 and ds.flags() == 0
    assert float(np.abs(got["x"] - x).max() / s.dx) <= 1e-11
    for key, ref in (("v", v), ("B", B), ("F", F)):
        assert rel(got[key], ref) <= 1e-11, (key, rel(got[key], ref))


def test_wavefronts_per_tile_give_the_same_bits():
    """A scene below the sizes at which the key pass and the transfer to
    particles take one wavefront per tile, and the same scene in a batch above
    them: the same bits."""
    b = _b()
    hosts = []
    for k in range(3):
        s = scenes.cube3d(seed=20 + k, cells=72, precision="fp32", steps=1)
        rng = np.random.default_rng(k)
        hosts.append(dataclasses.replace(s.with_state(v=s.v + rng.normal(0.0, 2.0, size=s.v.shape)), dt=1e-3))
    assert hosts[0].n < (1 << 19) and sum(h.n for h in hosts) >= (1 << 20)
    alone = b.DeviceScene(hosts[1], compensated=True)
    alone.step(3)
    batch = b.SceneBatch([b.DeviceScene(h, compensated=True) for h in hosts])
    batch.step(3)
    ga, gb = alone.state(), batch.scenes[1].state()
    for key in ("cell", "off", "v", "B", "F", "m"):
        assert np.array_equal(ga[key], gb[key]), key
