"""The grid update deals the node tiles of a key tile to four wavefronts in small
scenes and batches and leaves them to one in large ones: the same bits."""
import numpy as np
import pytest

from paper_1603_06188_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,precision", [(3, "fp32"), (2, "fp32"), (2, "fp64")])
def test_same_bits(dim, precision):
    """A scene alone, and in a batch with one that takes the whole over the line."""
    from paper_1603_06188_amd import binding as b

    line = 1 << (22 if dim == 3 else 20)
    small = scenes.random_particles(20000, dim=dim, cells=40, degree=2, seed=3, precision=precision, vel_sigma=0.3,
                                    b_sigma=0.002, dt=1e-4)
    big = scenes.random_particles(line, dim=dim, cells=96 if dim == 3 else 512, degree=2, seed=4, precision=precision,
                                  vel_sigma=0.3, b_sigma=0.002, dt=1e-4)
    alone = b.DeviceScene(small, compensated=True)
    alone.step(2)
    batch = b.SceneBatch([b.DeviceScene(small, compensated=True), b.DeviceScene(big, compensated=True)])
    batch.step(2)
    ga, gb = alone.state(), batch.scenes[0].state()
    for key in ("cell", "off", "v", "B", "F", "m"):
        assert np.array_equal(ga[key], gb[key]), key
    assert alone.flags() == 0
