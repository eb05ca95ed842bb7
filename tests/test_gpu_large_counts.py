"""The launches whose kernels change with the particle count (2^18, 2^19, 2^20),
where the results do not: batches of such totals under every plan against
their scenes stepped alone, and scenes of many tiles on both sides of 2^19."""
import dataclasses

import numpy as np
import pytest

from paper_1603_06188_amd import scenes

pytestmark = pytest.mark.gpu


def _b():
    from paper_1603_06188_amd import binding
    return binding


def _moving(dim, degree, precision, n, cells, seed):
    rng = np.random.default_rng(seed)
    dt = 1e-2
    s = scenes.random_particles(n, dim=dim, cells=cells, degree=degree, seed=seed, precision=precision, model=0,
                                margin=3.0, vel_sigma=0.05 / cells / dt, b_sigma=0.002 / cells ** 2 / dt)
    drift = rng.uniform(-0.2, 0.2, size=(cells, dim)) / cells / dt   # by the first cell index
    return dataclasses.replace(s.with_state(v=s.v + drift[s.cell[:, 0]]), dt=dt)


@pytest.mark.parametrize("dim,degree,precision,cells", [
    (3, 2, "fp32", 28),     # 343 tiles
    (3, 2, "fp32", 56),     # 2744
    (3, 3, "fp64", 30),
    (2, 2, "fp64", 104),    # 169
    (2, 2, "fp32", 330),    # about 1700
])
def test_batches_under_every_plan(dim, degree, precision, cells):
    b = _b()
    hosts = [_moving(dim, degree, precision, n, cells, seed=k) for k, n in enumerate((89000, 90000, 30000))]
    alone = []
    for h in hosts:
        d = b.DeviceScene(h, compensated=True)
        d.step(2)
        alone.append(d.state())
    groups = [(0, 1, 2), (0, 1, 0, 2), (0, 1, 0, 1, 0, 2, 1, 2), (0, 1) * 6 + (2,)]
    totals = [sum(hosts[k].n for k in g) for g in groups]
    assert totals[0] < 1 << 18 <= totals[1] < 1 << 19 <= totals[2] < 1 << 20 <= totals[3]
    try:
        for g in groups:
            for plan in range(b.apic_batch_plan_count()):
                b.apic_batch_set_plan(plan)
                batch = b.SceneBatch([b.DeviceScene(hosts[k], compensated=True) for k in g])
                batch.step(2)
                for at in {0, 1, len(g) - 1}:
                    got, want = batch.scenes[at].state(), alone[g[at]]
                    for key in ("cell", "off", "v", "B", "F", "m"):
                        assert np.array_equal(got[key], want[key]), (len(g), plan, at, key)
    finally:
        b.apic_batch_set_plan(-1)


@pytest.mark.parametrize("dim,degree,precision,absolute", [
    (3, 2, "fp32", True),
    (3, 3, "fp32", True),
    (3, 3, "fp32", False),
    (3, 3, "fp64", False),
    (3, 1, "fp32", False),
    (2, 2, "fp32", True),
    (2, 3, "fp64", False),
])
def test_same_bits_on_both_sides(dim, degree, precision, absolute):
    """The same particles, and with enough more without a position to be above."""
    b = _b()
    n, extra = (1 << 19) - 300, 500
    s = _moving(dim, degree, precision, n, 46 if dim == 3 else 400, seed=dim + degree)
    below = b.DeviceScene(s, with_id=True, compensated=True, absolute=absolute)
    above = b.DeviceScene(s.subset(np.r_[np.arange(n), np.arange(extra)]), with_id=True, compensated=True,
                          absolute=absolute)
    above.f[0, n:n + extra] = float("nan")
    above.sort()
    below.sort()
    rows, moved = [], 0
    for ds in (below, above):
        cell0 = ds.cell[:n].cpu().numpy()[np.argsort(ds.id[:n].cpu().numpy())]
        ds.step(3)
        ids = ds.id[:n].cpu().numpy()
        assert np.array_equal(np.sort(ids), np.arange(n))
        at = np.argsort(ids)
        cell = ds.cell[:n].cpu().numpy()[at]
        moved += np.count_nonzero(cell != cell0)
        rows.append((ds.f[:, :n].cpu().numpy()[:, at].tobytes(), cell.tobytes()))
    assert moved > n // 20
    assert rows[0] == rows[1]
