"""Rows that are not a whole number of 16-byte vectors, and fields that are
aligned to their elements only: the stencil kernels take vectors at any
element, the last one of a row overlapping the one before it.  States against
the C oracle (FP64 1e-12, FP32 1e-5, the stated tolerances), multi-step and
paired passes bit for bit against single steps, and the sums, in which an
overlapped point counts once, against the oracle's.
"""
import pytest
import torch

import oracle
from gpu_util import BASE, assert_normwise, assert_rel, f32_round, misaligned_like, rand_fields, say, to_dev, to_host

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
TOL = {F64: 1e-12, F32: 1e-5}


def _api():
    from paper_2107_00555_amd import api
    return api


def _fields(shape, seed, dtype):
    u0, f = rand_fields(shape, seed)
    return (u0, f) if dtype == F64 else (f32_round(u0), f32_round(f))


# lengths around one vector, one lane's and one wave's end, where the
# overlapping lane is the first or the last of a wave
NX = {F64: [2, 3, 5, 127, 129, 131, 255, 257, 385], F32: [4, 5, 6, 7, 253, 255, 257, 259, 513, 515, 1027]}


@pytest.mark.parametrize("dtype,nx", [(d, n) for d in NX for n in NX[d]])
@pytest.mark.parametrize("bc", [0, 1])
def test_single_steps_and_their_adjoint(dtype, nx, bc):
    api = _api()
    shape, T = (nx, 11, 5), 4
    say("ragged single steps", shape, bc, dtype)
    u0, f = _fields(shape, nx, dtype)
    u, fd = to_dev(u0, dtype), to_dev(f, dtype)
    out = api.run(u, fd, BASE, T, bc, tblock=1, norms=True, ckpt_every=1)
    want, e_want, r_want = oracle.run(u0, f, BASE, T, bc)
    assert_normwise("u_T", to_host(u), want, TOL[dtype])
    assert_rel("E_t", to_host(out["energy"]), e_want, TOL[dtype])
    assert_rel("R_t", to_host(out["resid"]), r_want, TOL[dtype])
    lam = _fields(shape, nx + 1, dtype)[0]
    g1 = api.adjoint_run(out["ckpt"], 1, fd, to_dev(lam, dtype), BASE, T, bc, tblock=1, want_f=True, want_gamma=True)
    g2 = api.adjoint_run(out["ckpt"], 1, fd, to_dev(lam, dtype), BASE, T, bc, tblock=2, want_f=True, want_gamma=True)
    w = oracle.adjoint_full(u0, f, lam, BASE, T, bc)
    assert_normwise("dL/du0", to_host(g1["u0"]), w["u0"], TOL[dtype])
    assert_normwise("dL/df", to_host(g1["f"]), w["f"], TOL[dtype])
    assert torch.equal(g1["u0"], g2["u0"]) and torch.equal(g1["f"], g2["f"])
    # the sums cancel: their error is measured against the sum of the terms' sizes
    n = u0.size * T
    for g in (g1, g2):
        for k, s in (("alpha", 6 * 0.1), ("beta", 0.1)):
            i = 0 if k == "alpha" else 1
            assert abs(float(g["ab"][i]) - w[k]) <= TOL[dtype] * s * n, (k, float(g["ab"][i]), w[k])
        assert abs(float(g["gamma"]) - w["gamma"]) <= TOL[dtype] * 0.1 * n


# at least 2^18 points, so that runs take passes of several steps (the first
# ones over blocks, those of more than about 900,000 points over x-segments):
# two and more segments, a short last one, few rows, few planes
SHAPES = [(257, 80, 61), (1031, 40, 33), (515, 66, 40), (129, 129, 70), (2051, 33, 17), (97, 333, 40), (513, 700, 3), (257, 40, 37), (131, 70, 35), (1031, 20, 17), (515, 33, 20), (2051, 13, 11), (513, 513, 3), (37, 97, 80),
          (1022, 21, 13)]


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_multi_step_passes(shape, bc, dtype):
    from paper_2107_00555_amd import _lib
    api = _api()
    T = 8
    say("ragged passes", shape, bc, dtype)
    u0, f = _fields(shape, sum(shape), dtype)
    fd = to_dev(f, dtype)
    runs = {}
    for tb in (1, 2, 3):
        u = to_dev(u0, dtype)
        runs[tb] = (u, api.run(u, fd, BASE, T, bc, tblock=tb, norms=True, ckpt_every=3))
    plan = _lib.run_plan(_lib.F64 if dtype == F64 else _lib.F32, *shape, T, 3)
    assert plan["passes"] == [0, 1, 2], plan
    want, e_want, r_want = oracle.run(u0, f, BASE, T, bc)
    for tb, (u, out) in runs.items():
        assert torch.equal(u, runs[1][0]) and torch.equal(out["ckpt"], runs[1][1]["ckpt"]), tb
        assert_rel("E_t", to_host(out["energy"]), e_want, TOL[dtype])
        assert_rel("R_t", to_host(out["resid"]), r_want, TOL[dtype])
    assert_normwise("u_T", to_host(runs[1][0]), want, TOL[dtype])


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("shape", [(128, 64, 40), (257, 40, 37), (6, 9, 4)])
def test_fields_aligned_to_their_elements(shape, dtype):
    # the same bits from fields at an odd offset as from aligned ones
    api = _api()
    say("element alignment", shape, dtype)
    u0, f = _fields(shape, 7, dtype)
    got = []
    for move in (lambda t: t, misaligned_like):
        u, fd = move(to_dev(u0, dtype)), move(to_dev(f, dtype))
        out = api.run(u, fd, BASE, 7, 1, norms=True, ckpt_every=2)
        lam = move(to_dev(u0, dtype))
        g = api.adjoint_run(out["ckpt"], 2, fd, lam, BASE, 7, 1, want_f=True)
        s, n2 = api.step(u, fd, BASE, 0, norms=True)
        got.append([u, out["energy"], out["resid"], out["ckpt"], g["u0"], g["ab"], g["f"], s, n2])
    for a, b in zip(*got):
        assert torch.equal(a, b)
