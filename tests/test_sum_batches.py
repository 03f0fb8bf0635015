"""The room for per-step sums in a run's, an adjoint's and a reverse sweep's
workspace: at most 16 MiB and the two sums of each step, whatever the number of
steps; and, on the GPU, sweeps of more steps than that holds.
"""
import pytest
import torch

from gpu_util import BASE, rand_fields, say, to_dev

MIB = 1 << 20
GRIDS = [(512, 512, 512), (1024, 1024, 512), (64, 64, 64), (33, 700, 900)]


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("shape", GRIDS)
def test_workspace_does_not_grow_with_the_steps(shape, dtype):
    from paper_2107_00555_amd import _lib as L
    many = 10000
    for tb in (1, 3):
        def run(T, norms):
            return L.workspace_bytes(L.OP_RUN, dtype, *shape, T, 1, tb, norms)
        assert run(many, True) - run(many, False) <= 16 * MIB + 512
        def adj(T):
            return L.workspace_bytes(L.OP_ADJOINT, dtype, *shape, T, 5, tb, False)
        assert adj(many) - adj(5) <= 16 * MIB + 16 * many + 512
    def rev(T):
        return L.revolve_workspace_bytes(dtype, *shape, T, 5)
    assert rev(many) - rev(5) <= 16 * MIB + 16 * many + 512


@pytest.mark.gpu
@pytest.mark.parametrize("tblock", [1, 3])
@pytest.mark.parametrize("bc", [0, 1])
def test_more_steps_than_a_batch(tblock, bc):
    """One sweep of 760 steps against two of 380: the same norms, states and
    gradient fields bit for bit, the parameter sums to rounding.  The single steps'
    1500 workgroups leave room for 699 steps."""
    from paper_2107_00555_amd import _lib as L, api
    shape, T, k = (8, 400, 240), 760, 95
    room = L.workspace_bytes(L.OP_RUN, 0, *shape, T, 1, tblock, True) - \
        L.workspace_bytes(L.OP_RUN, 0, *shape, T, 1, tblock, False)
    assert room < T * 1500 * 16
    say("sum batches", tblock, bc)
    u0, f = rand_fields(shape, 2)
    c = dict(BASE, dt=0.01)
    u, v, fd = to_dev(u0), to_dev(u0), to_dev(f)
    one = api.run(u, fd, c, T, bc, tblock=tblock, ckpt_every=k)
    two = [api.run(v, fd, c, T // 2, bc, tblock=tblock, ckpt_every=k) for _ in range(2)]
    assert torch.equal(u, v)
    for key in ("energy", "resid"):
        # (tblock 3: the halves end in passes of two steps, whose sums have another order)
        assert torch.allclose(one[key], torch.cat([r[key] for r in two]), rtol=1e-13 if tblock > 1 else 0, atol=0)
    assert torch.equal(one["ckpt"], torch.cat([r["ckpt"] for r in two]))
    lam = to_dev(f)
    whole = api.adjoint_run(one["ckpt"], k, fd, lam, c, T, bc, tblock=tblock, want_f=True)
    late = api.adjoint_run(two[1]["ckpt"], k, fd, lam, c, T // 2, bc, tblock=tblock)
    early = api.adjoint_run(two[0]["ckpt"], k, fd, late[0], c, T // 2, bc, tblock=tblock)
    assert torch.equal(whole["u0"], early[0])
    assert torch.allclose(whole["ab"], late[1] + early[1], rtol=1e-12, atol=0)
    ws = api.revolve_forward(to_dev(u0), fd, c, T, bc, 9, tblock=tblock)
    swept = api.revolve_adjoint(ws, fd, lam, c, T, bc, 9, tblock=tblock)
    assert torch.equal(swept[0], whole["u0"])
    assert torch.allclose(swept[1], whole["ab"], rtol=1e-12, atol=0)
