"""The force path's workspace over box sizes (host side only)."""
import pytest

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W


@pytest.mark.parametrize("double", [False, True])
@pytest.mark.parametrize("flags", [0, api.PAIR_FULL_SHELL, api.ACCUM_F32_ATOMIC, api.PAIR_PREDICATED])
def test_workspace_serves_a_shrinking_box(flags, double):
    """At a given number of atoms a smaller box (fewer cells) needs no more than a larger one, so a run
    at constant pressure keeps the workspace of its largest box. Around every change of the grid on
    the way from 18^3 cells to 2^3, on one axis at a time and on all."""
    base = W.small_system().params()
    for n in (1, 3000, 20000, 200000):
        last = None
        dims = [18, 18, 18]
        shapes = [tuple(dims)]
        while max(dims) > 2:
            d = dims.index(max(dims))
            dims[d] -= 1
            shapes.append(tuple(dims))
        for dims3 in shapes:
            box = tuple(12.0 * d + 6.0 for d in dims3)
            p = dict(base, box=box, flags=flags)
            lay = api.workspace_layout(p, n, double)
            assert lay["dims"] == dims3
            nb = api.workspace_bytes(p, n, double)
            assert last is None or nb <= last, (n, dims3)
            last = nb
