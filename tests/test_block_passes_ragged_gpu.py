"""Forward passes over blocks on rows that are not whole vectors: grids of at
least 2^18 points, which take them, with every remainder of a row and last blocks
cut short on each axis.  The plan is checked to be the block form's, and with
that form switched off to be another one; both give single steps' bits.
"""
import pytest
import torch

import oracle
from gpu_util import BASE, assert_normwise, assert_rel, f32_round, rand_fields, say, to_dev, to_host

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
TOL = {F64: 1e-12, F32: 1e-5}


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("shape", [(61, 67, 71), (67, 61, 65), (90, 54, 55), (95, 53, 53), (13, 170, 121)])
def test_ragged_rows_over_blocks(monkeypatch, shape, bc, dtype):
    from paper_2107_00555_amd import _lib, api
    T, code = 8, _lib.F64 if dtype == F64 else _lib.F32
    u0, f = rand_fields(shape, sum(shape))
    if dtype == F32:
        u0, f = f32_round(u0), f32_round(f)
    fd = to_dev(f, dtype)
    want, e_want, r_want = oracle.run(u0, f, BASE, T, bc)
    blocks = _lib.run_plan(code, *shape, T, 3)
    assert blocks["passes"] == [0, 1, 2] and blocks["lanes"] == 768
    states = []
    for form in ("blocks", "others"):
        say("ragged blocks", shape, bc, dtype, form)
        if form == "others":
            monkeypatch.setenv("DCP_TUNING", "1")
            monkeypatch.setenv("DCP_TBK_CFG", "0,0,0")
            assert _lib.run_plan(code, *shape, T, 3) != blocks
        for tb in (1, 2, 3):
            u = to_dev(u0, dtype)
            out = api.run(u, fd, BASE, T, bc, tblock=tb, ckpt_every=3)
            states.append((u, out["ckpt"]))
            assert_rel("E_t", to_host(out["energy"]), e_want, TOL[dtype])
            assert_rel("R_t", to_host(out["resid"]), r_want, TOL[dtype])
    assert_normwise("u_T", to_host(states[0][0]), want, TOL[dtype])
    for u, ckpt in states:
        assert torch.equal(u, states[0][0]) and torch.equal(ckpt, states[0][1])
