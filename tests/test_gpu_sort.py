"""The order a sort leaves, for particles given in any order: of a tile's keys
level by level (key by key where a key holds more than 32), within a key by
their place before the sort, and the particles outside the grid or without a
finite position after all others.  Every row is intact, bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_levels import _scene

pytestmark = pytest.mark.gpu


def _b():
    from paper_1603_06188_amd import binding
    return binding


def _keys(cell, off, degree):
    """Tile and local index (0..63) of each particle's base node: tiles of 4x4x4
    or 8x8 base nodes, the first axis fastest."""
    base = np.where(off < 0.5, cell - 1, cell) if degree == 2 else cell - 1
    w = 4 if base.shape[1] == 3 else 8
    tile, local = np.zeros(len(base), dtype=np.int64), np.zeros(len(base), dtype=np.int64)
    for a in reversed(range(base.shape[1])):
        tile, local = tile * 64 + base[:, a] // w, local * w + base[:, a] % w
    return tile, local


def _order(tile, local):
    """Rows of one tile in the stored order, given in the order before it."""
    out = {}
    for t in np.unique(tile):
        rows = np.flatnonzero(tile == t)
        rank = np.zeros(rows.size, dtype=np.int64)
        for k in np.unique(local[rows]):
            at = np.flatnonzero(local[rows] == k)
            rank[at] = np.arange(at.size)
        busy = rank.max() >= 32
        out[t] = rows[np.lexsort((rank, local[rows]) if busy else (local[rows], rank))]
    return out


@pytest.mark.parametrize("dim,degree,precision,ids,dead,counts", [
    (3, 2, "fp32", True, 0, (1,)),
    (3, 2, "fp32", True, 7, (1, 2, 3, 4, 5)),
    (3, 3, "fp64", True, 300, (4, 8, 0, 9, 7, 16, 17)),
    (2, 2, "fp64", False, 5, (32, 1, 31, 2)),
    (2, 2, "fp32", True, 1, (33, 5, 70, 0, 1)),
    (3, 2, "fp64", True, 0, (33, 32, 400, 1, 1)),
    (3, 2, "fp32", False, 0, (90, 3, 32, 32, 32, 31)),
])
def test_order(dim, degree, precision, ids, dead, counts):
    s = _scene(dim, degree, precision, counts, seed=7 + len(counts))
    rng = np.random.default_rng(sum(counts))
    s = s.subset(rng.permutation(np.r_[np.arange(s.n), rng.integers(0, s.n, dead)]))
    ds = _b().DeviceScene(s, with_id=ids)
    n = s.n
    gone = np.zeros(n, dtype=bool)
    gone[rng.permutation(n)[:dead]] = True
    # half of them in a corner cell whose support leaves the grid, half without
    # a position
    marks = np.flatnonzero(gone)
    ds.cell[marks[::2].tolist()] = 0
    ds.f[:dim, marks[::2].tolist()] = 0.25
    ds.f[0, marks[1::2].tolist()] = float("nan")
    f0, cell0 = ds.f[:, :n].cpu().numpy(), ds.cell[:n].cpu().numpy()
    tile, local = _keys(s.cell, s.off, s.degree)
    ds.sort()
    f1, cell1 = ds.f[:, :n].cpu().numpy(), ds.cell[:n].cpu().numpy()
    b = _b()
    assert ds.flags() == ((b.APIC_FLAG_OUT_OF_DOMAIN if dead else 0) | (b.APIC_FLAG_NONFINITE if dead > 1 else 0))
    live = np.flatnonzero(~gone)
    want = {t: live[o] for t, o in _order(tile[live], local[live]).items()}
    rows = {f0[:, i].tobytes() + cell0[i].tobytes(): [] for i in range(n)}
    for i in range(n):      # a row drawn twice: by its place, the earlier first
        rows[f0[:, i].tobytes() + cell0[i].tobytes()].append(i)
    if ids:
        got = ds.id[:n].cpu().numpy()
        assert f1.tobytes() == f0[:, got].tobytes() and np.array_equal(cell1, cell0[got])
    else:
        got = np.array([rows[f1[:, i].tobytes() + cell1[i].tobytes()].pop(0) for i in range(n)])
    assert np.array_equal(np.sort(got), np.arange(n))
    assert gone[got[live.size:]].all()
    at = 0
    while at < live.size:
        w = want.pop(tile[got[at]])
        assert np.array_equal(got[at:at + w.size], w)
        at += w.size
    assert not want
