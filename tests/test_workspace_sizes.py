"""Workspaces callers hold stay large enough: a workspace of a size that
apic_workspace_bytes once gave still holds its scene, and a scene that fitted
the array of apic_step_noalloc still does.  The figures are those of the library
before the transfer to particles kept bounds per tile."""
import pytest

from paper_1603_06188_amd import binding as b

# (dim, degree, binary64, cells, compensated): bytes for 1, 1,000 and 1,000,003 particles, most
# particles without a workspace (None: none)
HELD = {
    (3, 2, 0, (16, 16, 16), 0): ((636416, 1188608, 129065472), 1040256),
    (3, 2, 0, (128, 128, 128), 1): ((140307968, 147343872, 516984832), None),
    (3, 3, 1, (61, 47, 33), 1): ((8255744, 30412544, 274180096), 386176),
    (3, 1, 0, (100, 100, 100), 0): ((68694016, 70822912, 231984384), 236224),
    (2, 2, 0, (1024, 1024), 0): ((60718336, 62001920, 160819456), 667520),
    (2, 3, 1, (63, 65), 1): ((453376, 993280, 132866304), 1010240),
    (2, 2, 1, (8, 8), 0): ((167936, 302080, 132175104), 1015488),
}


@pytest.mark.parametrize("case", HELD, ids=str)
def test_held_sizes(case):
    dim, degree, f64, cells, comp = case
    g = b.ApicGridDesc()
    g.dim, g.degree, g.dx = dim, degree, 1.0 / 64
    g.precision = b.APIC_F64 if f64 else b.APIC_F32
    g.options = b.APIC_OPT_COMPENSATED if comp else 0
    for a in range(dim):
        g.cells[a] = cells[a]
    sizes, most = HELD[case]
    for n, size in zip((1, 1000, 1000003), sizes):
        assert b.apic_workspace_bytes(g, n) <= size, n
    if most:
        assert b.apic_workspace_bytes(g, most) <= b.apic_noalloc_max_bytes()
