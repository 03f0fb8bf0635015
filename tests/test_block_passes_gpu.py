"""Passes over blocks on small grids: two and three forward steps and two
adjoint steps per pass.  Every point takes the one-step kernel's operations,
so states and dL/du0, dL/df equal single steps bit for bit; the sums are added
per block and agree with the oracle's at the stated tolerance.  The same grids
through the marching forms (blocks switched off by an empty tiling override)
give the same bits.
"""
import pytest
import torch

import oracle
from gpu_util import BASE, assert_normwise, assert_rel, f32_round, rand_fields, say, to_dev, to_host

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
TOL = {F64: 1e-12, F32: 1e-5}

# one block and many on each axis, the last ones cut short, grids smaller than
# a halo, rows of any length, the largest single round of workgroups
SHAPES = [(1, 1, 1), (2, 3, 1), (4, 2, 3), (16, 28, 8), (17, 29, 9), (64, 64, 64), (61, 67, 71), (96, 96, 96),
          (500, 7, 4), (5, 700, 3), (6, 4, 900), (90, 33, 12)]


def _api():
    from paper_2107_00555_amd import api
    return api


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_block_passes(monkeypatch, shape, bc, dtype):
    api = _api()
    T = 8  # two passes of three steps and one of two
    u0, f = rand_fields(shape, 17 + sum(shape))
    if dtype == F32:
        u0, f = f32_round(u0), f32_round(f)
    fd = to_dev(f, dtype)
    want, e_want, r_want = oracle.run(u0, f, BASE, T, bc)
    ref = None
    for blocks in (True, False):
        say("block passes", shape, bc, dtype, "blocks" if blocks else "marching")
        if not blocks:
            monkeypatch.setenv("DCP_TUNING", "1")
            monkeypatch.setenv("DCP_TBK_CFG", "0,0,0")
        for tb in (1, 2, 3):
            u = to_dev(u0, dtype)
            out = api.run(u, fd, BASE, T, bc, tblock=tb, norms=True, ckpt_every=3)
            lam = to_dev(f, dtype)
            g = api.adjoint_run(out["ckpt"], 3, fd, lam, BASE, T, bc, tblock=tb, want_f=True, want_gamma=True)
            plain = api.adjoint_run(out["ckpt"], 3, fd, lam, BASE, T, bc, tblock=tb)
            if ref is None:
                ref = (u, out, g)
                assert_normwise("u_T", to_host(u), want, TOL[dtype])
            assert torch.equal(u, ref[0]) and torch.equal(out["ckpt"], ref[1]["ckpt"])
            assert torch.equal(g["u0"], ref[2]["u0"]) and torch.equal(g["f"], ref[2]["f"])
            assert torch.equal(plain[0], g["u0"]) and torch.equal(plain[1], g["ab"])
            assert_rel("E_t", to_host(out["energy"]), e_want, TOL[dtype])
            assert_rel("R_t", to_host(out["resid"]), r_want, TOL[dtype])
            # the sums cancel: 1e-12 of the number of terms, each at most a few units
            assert torch.allclose(g["ab"], ref[2]["ab"], rtol=0, atol=1e-12 * T * u0.size + 1e-14)


@pytest.mark.parametrize("bc", [0, 1])
def test_block_passes_in_the_reverse_sweep(bc):
    # binomial checkpointing over the same passes
    api = _api()
    shape, T = (61, 40, 33), 23
    u0, f = rand_fields(shape, 3)
    fd, lam = to_dev(f), to_dev(u0)
    ck = api.run(to_dev(u0), fd, BASE, T, bc, norms=False, ckpt_every=5)["ckpt"]
    want = api.adjoint_run(ck, 5, fd, lam, BASE, T, bc, tblock=1, want_f=True, want_gamma=True)
    for s in (0, 2, 5):
        say("block passes, revolve", s, bc)
        ws = api.revolve_forward(to_dev(u0), fd, BASE, T, bc, s, reserve_sum=True)
        got = api.revolve_adjoint(ws, fd, lam, BASE, T, bc, s, want_f=True, want_gamma=True)
        assert torch.equal(got["u0"], want["u0"]) and torch.equal(got["f"], want["f"])
        assert torch.equal(got["gamma"], want["gamma"])
        assert torch.allclose(got["ab"], want["ab"], rtol=0, atol=1e-12 * T * u0.size)
