"""Scenes of few particles per tile.  The key pass and the transfer to particles
take a block per tile or several tiles per block by the number of listed tiles and
the particles in them (3D binary64 above 768 tiles, the others above 1536), and the
grid update four wavefronts or one per tile (above 2048 to 5120): here both sides
of those lines, tile counts that leave the last block short, particles that leave
their key and some that leave the grid."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_1603_06188_amd import scenes
from tests.test_gpu_parity import rel

pytestmark = pytest.mark.gpu


def _b():
    from paper_1603_06188_amd import binding
    return binding


def _sparse(dim, degree, precision, edge, per_tile, seed, dt=1e-2):
    """About `edge` tiles along each axis and `per_tile` particles in each, moving
    by up to a few tenths of a cell a step."""
    te = 4 if dim == 3 else 8
    cells = edge * te
    rng = np.random.default_rng(seed)
    n = int(per_tile * edge ** dim)
    s = scenes.random_particles(n, dim=dim, cells=cells, degree=degree, seed=seed, precision=precision, model=0,
                                margin=3.0, vel_sigma=0.0, b_sigma=0.002 / cells ** 2 / dt)
    # each row of tiles drifts by its own velocity, the particles with it
    base = rng.uniform(-0.3, 0.3, size=(edge + 1, dim)) / cells / dt
    v = base[s.cell[:, 0] // te] + rng.normal(0.0, 0.02 / cells / dt, size=(n, dim))
    return dataclasses.replace(s.with_state(v=v), dt=dt)


@pytest.mark.parametrize("dim,degree,precision,edge,per_tile", [
    (3, 2, "fp32", 11, 12),     # 1331 tiles: a block each
    (3, 2, "fp32", 12, 9),      # 1728: a wavefront each
    (3, 1, "fp32", 13, 5),      # 2197
    (3, 2, "fp32", 18, 3),      # about 5500, the grid update by one wavefront each
    (3, 3, "fp32", 12, 9),
    (3, 2, "fp64", 9, 12),      # 729
    (3, 2, "fp64", 10, 9),      # 1000, the key pass two tiles to a block
    (3, 1, "fp64", 10, 9),
    (3, 3, "fp64", 11, 9),      # 1331: an odd number
    (2, 2, "fp32", 39, 9),      # 1521
    (2, 2, "fp32", 41, 9),      # 1681
    (2, 3, "fp64", 47, 9),      # 2209
])
def test_steps(dim, degree, precision, edge, per_tile):
    """Chained steps against the oracle (binary64 1e-11, binary32 2e-5: two steps)."""
    b = _b()
    s = _sparse(dim, degree, precision, edge, per_tile, seed=edge + dim + degree)
    steps = 2
    ds = b.DeviceScene(s, compensated=precision == "fp32")
    ds.step(steps)
    got = ds.state()
    g = oracle.Grid(s.dim, s.degree, s.cells, s.dx)
    x, v, B, F = s.x, s.v, s.B, s.F
    moved = 0
    shift = 0.5 if degree == 2 else 0.0
    for _ in range(steps):
        r = oracle.step(g, x, v, B, F, s.m, s.V, s.model, s.mu, s.lam, s.dt, s.gravity, s.band, transfer=s.transfer)
        moved += int(np.count_nonzero((np.floor(r["x_new"] / s.dx - shift) != np.floor(x / s.dx - shift)).any(axis=1)))
        x, v, B, F = r["x_new"], r["v_new"], r["B_new"], r["F_new"]
    assert moved > s.n // 20 and ds.flags() == 0
    tol = 1e-11 if precision == "fp64" else 2e-5
    assert float(np.abs(got["x"] - x).max() / s.dx) <= tol
    for key, ref in (("v", v), ("B", B), ("F", F)):
        assert rel(got[key], ref) <= tol, (key, rel(got[key], ref))


@pytest.mark.parametrize("dim,degree,precision,edge", [(3, 2, "fp32", 12), (3, 2, "fp64", 9), (3, 2, "fp64", 10),
                                                       (2, 2, "fp32", 41)])
def test_particles_that_leave_the_grid(dim, degree, precision, edge):
    """The rows of dead particles are carried bit for bit, all of them, while the
    others step as they do without them."""
    b = _b()
    s = _sparse(dim, degree, precision, edge, 7, seed=5)
    rng = np.random.default_rng(6)
    out = np.sort(rng.permutation(s.n)[:333])
    live = np.setdiff1d(np.arange(s.n), out)
    ds = b.DeviceScene(s, compensated=True)
    ds.f[0, out.tolist()] = float("nan")    # no position
    ds.sort()
    dead0 = ds.f[:, live.size:s.n].cpu().numpy()
    ds.step(2)
    ref = b.DeviceScene(s.subset(live), compensated=True)
    ref.step(2)
    assert ds.flags() & b.APIC_FLAG_NONFINITE and ref.flags() == 0
    got, want = ds.f[:, :live.size].cpu().numpy(), ref.f[:, :live.size].cpu().numpy()
    ids, ids_ref = ds.id[:live.size].cpu().numpy(), live[ref.id[:live.size].cpu().numpy()]
    assert np.array_equal(np.sort(ids), live)
    assert np.array_equal(got[:, np.argsort(ids)], want[:, np.argsort(ids_ref)])
    dead = ds.f[:, live.size:s.n].cpu().numpy()
    assert sorted(dead[1:, i].tobytes() for i in range(333)) == sorted(dead0[1:, i].tobytes() for i in range(333))


@pytest.mark.parametrize("dim,degree,precision,edge", [(3, 2, "fp32", 12), (3, 3, "fp32", 12), (3, 2, "fp64", 10),
                                                       (2, 2, "fp32", 41)])
def test_same_bits_in_a_batch(dim, degree, precision, edge):
    """A sparse scene alone (several tiles per block) and in a batch of two, where
    its part of the limit is the whole (a block per tile): the same bits."""
    b = _b()
    s = [_sparse(dim, degree, precision, edge, 7, seed=k) for k in (1, 2)]
    small = [scenes.random_particles(500, dim=dim, cells=12, degree=degree, seed=9, precision=precision)]
    alone = b.DeviceScene(s[0], compensated=True)
    alone.step(3)
    for others in ([s[1]], small, 40 * small):
        batch = b.SceneBatch([b.DeviceScene(h, compensated=True) for h in [s[0]] + others])
        batch.step(3)
        ga, gb = alone.state(), batch.scenes[0].state()
        for key in ("cell", "off", "v", "B", "F", "m"):
            assert np.array_equal(ga[key], gb[key]), (len(others), key)
