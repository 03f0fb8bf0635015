"""Tiles of the one-step forward kernel on either side of the 1500 workgroups
from which it takes four rows per lane: runs of planes that divide the grid
and runs that leave a shorter last one, with the norms and without.  Against
the C oracle (FP64 1e-12, FP32 1e-5), the two calls' states bit for bit equal.
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
@pytest.mark.parametrize("shape", [
    (8, 800, 240),   # 50 x 30 workgroups of 16 rows and 8 planes: the fewest with four rows per lane
    (8, 800, 239),   # a ragged last run of planes
    (8, 784, 240),   # one block of rows fewer: two rows per lane
    (9, 793, 245),   # ragged rows and blocks
])
def test_step_with_and_without_norms(shape, bc, dtype):
    from paper_2107_00555_amd import api
    say("step tiles", shape, bc, dtype)
    u0, f = rand_fields(shape, sum(shape))
    if dtype == F32:
        u0, f = f32_round(u0), f32_round(f)
    want, e_want, r_want = oracle.run(u0, f, BASE, 1, bc)
    u, fd = to_dev(u0, dtype), to_dev(f, dtype)
    plain, none = api.step(u, fd, BASE, bc)
    out, n2 = api.step(u, fd, BASE, bc, norms=True)
    ran = u.clone()
    res = api.run(ran, fd, BASE, 1, bc, tblock=1)
    assert none is None
    assert_normwise("u_1", to_host(out), want, TOL[dtype])
    assert torch.equal(plain, out) and torch.equal(ran, out)
    assert_rel("E", to_host(res["energy"]), e_want, TOL[dtype])
    assert_rel("R", to_host(res["resid"]), r_want, TOL[dtype])
    assert_rel("sum u^2", to_host(n2[:1]), e_want, TOL[dtype])
    assert_rel("sum (u_1 - u)^2", to_host(n2[1:].sqrt()), r_want, TOL[dtype])
