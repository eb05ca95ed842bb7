"""The order a sort leaves in tiles stored key by key, with as many particles as
fit into the LDS (2048), one more, one less, and many more."""
import pytest

import tests.test_gpu_sort as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,degree,precision,ids,dead,counts", [
    (3, 2, "fp32", True, 0, (0, 1000, 1047)),
    (3, 3, "fp64", True, 3, (1, 1000, 1048)),
    (2, 2, "fp32", False, 0, (33, 1000, 1016)),
    (2, 2, "fp64", True, 40, (700, 0, 700, 2, 700, 700, 40)),
    (3, 2, "fp32", True, 2, (2100, 33, 31, 2050, 1, 2016)),
])
def test_order_busy(dim, degree, precision, ids, dead, counts):
    base.test_order(dim, degree, precision, ids, dead, counts)
