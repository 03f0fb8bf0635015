"""Planning a run takes microseconds whatever the length of a row."""
import time

import pytest

from paper_2107_00555_amd import _lib as L


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("shape", [(1 << 24, 1, 1), (1000001, 3, 2), (100000, 8, 4), (16384, 64, 64)])
def test_a_long_row_is_planned_at_once(shape, dtype):
    best = float("inf")
    for _ in range(5):
        t = time.perf_counter()
        p = L.run_plan(dtype, *shape, 100, 3)
        best = min(best, time.perf_counter() - t)
    assert p["passes"] == [0, 2, 32]
    assert best < 1e-3  # a few thousand tiles are priced, some 10 ns each
