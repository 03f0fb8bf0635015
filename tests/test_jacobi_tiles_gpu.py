"""jacobi_2d's region tiles: the height chosen against the heights it can be
forced to, on narrow arrays above all, and what a pass over a narrow array
costs, whose tiles nearly all hold boundary cells; rows of odd length.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import DEV, say, to_dev, to_host
from paper_2107_00555_amd import inputs

pytestmark = pytest.mark.gpu


def _us(A, B, tsteps, tblock):
    """Least of several runs, us."""
    from paper_2107_00555_amd import api
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(25):
        a.record()
        api.jacobi_2d(A, B, tsteps, tblock)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


def _pair(n0, n1):
    g = torch.Generator(device=DEV).manual_seed(n0)
    return tuple(torch.rand((n0, n1), dtype=torch.float64, device=DEV, generator=g) for _ in range(2))


# runs repeat within 3%, and the rule is within 7% of the fastest height wherever
# it was measured
@pytest.mark.parametrize("shape,tblock", [((118, 9505), 8), ((200, 3000), 12), ((3000, 400), 8), ((9505, 135), 12),
                                          ((160, 9505), 4), ((1300, 1300), 12), ((3000, 3000), 12)])
def test_height_is_among_the_fastest(monkeypatch, shape, tblock):
    A, B = _pair(*shape)
    say("jacobi_2d height", shape, tblock)
    monkeypatch.setenv("DCP_TUNING", "1")
    monkeypatch.setenv("DCP_J2_MODE", "1")
    _us(A, B, 97, tblock)
    took = _us(A, B, 97, tblock)
    others = []
    for cfg in ("0", "1", "2"):  # 4, 6 and 8 rows per lane
        monkeypatch.setenv("DCP_J2_CFG", cfg)
        others.append(_us(A, B, 97, tblock))
    print(f"took {took:.1f}", [round(x, 1) for x in others])
    assert took <= 1.12 * min(others)


# runs repeat within 3%, and the rule is within 7% of the better form wherever it
# was measured
@pytest.mark.parametrize("n,tblock", [(2500, 6), (3000, 4), (3000, 8), (3500, 16), (4500, 4), (4500, 10)])
def test_form_is_the_faster(monkeypatch, n, tblock):
    A, B = _pair(n, n)
    say("jacobi_2d form", n, tblock)
    took = _us(A, B, 97, tblock)
    monkeypatch.setenv("DCP_TUNING", "1")
    both = []
    for mode in ("1", "3"):  # region tiles, row march
        monkeypatch.setenv("DCP_J2_MODE", mode)
        both.append(_us(A, B, 97, tblock))
    print(f"took {took:.1f}", [round(x, 1) for x in both])
    assert took <= 1.12 * min(both)


def test_narrow_array_moves_no_more(monkeypatch):
    # two half-steps per pass: memory bounds it; the same number of cells
    monkeypatch.setenv("DCP_TUNING", "1")
    monkeypatch.setenv("DCP_J2_MODE", "1")
    say("jacobi_2d narrow")
    square, narrow = (_us(*_pair(*s), 25, 2) for s in ((3464, 3464), (20000, 600)))
    print(f"square {square:.0f}, narrow {narrow:.0f}")
    # the column halo: 600 columns are five tiles of 124, 20 of them idle (3%)
    assert narrow <= 1.15 * square


@pytest.mark.parametrize("shape", [(257, 511), (333, 261), (40, 1001), (1001, 33), (130, 129)])
@pytest.mark.parametrize("tblock", [1, 2, 5, 8, 16])
def test_region_tiles_on_odd_rows(monkeypatch, shape, tblock):
    # the row march takes odd rows too: the tiles are forced
    from paper_2107_00555_amd import api
    monkeypatch.setenv("DCP_TUNING", "1")
    monkeypatch.setenv("DCP_J2_MODE", "1")
    A, B = inputs.jacobi_fields(2, shape[0], seed=3, n1=shape[1])
    for tsteps in (2, 14):
        say("jacobi_2d odd rows", shape, tblock, tsteps)
        a, b = to_dev(A), to_dev(B)
        api.jacobi_2d(a, b, tsteps, tblock)
        want = oracle.jacobi_2d(tsteps, A, B)
        assert np.array_equal(to_host(a), want[0]) and np.array_equal(to_host(b), want[1])
