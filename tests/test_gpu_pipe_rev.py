"""Pipelined passes of the reverse recursion over ribbons (pipe_rev.hip)
against the CPU oracle's reverse mode."""
import numpy as np
import pytest

import oracle as O
from test_gpu_adjoint import assert_grad_close, rel_l2, ribbon_inputs
from test_gpu_parity import assert_state_close, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    return T


@pytest.fixture(scope="module")
def cheb():
    import paper_0907_3022_amd as P
    P.load_library()
    return P


# rows below, at and past a pass's eight levels and a chunk; columns below, at
# and past a strip's 112 own columns; orders at and past whole passes (a rest
# of one order, of a few, none), so that first, inner and last passes run
@pytest.mark.parametrize("edge", ["zigzag", "armchair"])
@pytest.mark.parametrize("w,l,chunks", [(1, 113, 1), (2, 2, 1), (7, 112, 1), (9, 111, 1), (30, 225, 2), (53, 114, 5)])
def test_pipelined_reverse_matches_oracle(torch, cheb, monkeypatch, edge, w, l, chunks):
    monkeypatch.setenv("CHEBTD_REV_CHUNKS", str(chunks))
    V, psi0, mask = ribbon_inputs(w, l, dense=True)
    H = O.honeycomb(w, l, V, edge=edge)
    lo, hi = H.gershgorin()
    K, dt = 2, 1.0
    for M in (8, 9, 10, 16, 29):
        say(f"[gpu] pipelined reverse {w}x{l} {edge} chunks={chunks} M={M}")
        ctx = cheb.Context()
        Vd = torch.from_numpy(V.copy()).cuda()
        ctx.honeycomb(w, l, Vd, edge=edge)
        ctx.set_bounds(lo, hi)
        ctx.plan_order(dt, M)
        ctx.reserve_adjoint(K, cheb.ADJ_REVERSE)
        psi = torch.from_numpy(psi0.copy()).cuda()
        ctx.propagate(psi, K, None, None, cheb.NO_CHECK | cheb.KEEP_CHECKPOINTS)
        gbar = (2.0 * torch.from_numpy(mask).cuda() * psi).contiguous()
        dV = torch.zeros_like(Vd)
        ctx.adjoint(gbar, dV)
        torch.cuda.synchronize()
        ctx.close()
        Lr, gr, ur = O.adjoint(H, O.Plan(lo, hi, dt, M=M), psi0, K, mask)
        assert_grad_close(dV.cpu().numpy(), gr)
        assert_state_close(gbar.cpu().numpy(), ur)


# many workgroups per pass: rows handed from wavefront to wavefront in every
# state of the pipeline, against the single-wavefront passes
@pytest.mark.parametrize("edge", ["zigzag", "armchair"])
@pytest.mark.parametrize("chunks", [2, 6, 16])
def test_pipelined_reverse_many_workgroups(torch, cheb, monkeypatch, edge, chunks):
    w, l, K = 256, 4096, 2
    V, psi0, mask = ribbon_inputs(w, l, dense=True)

    def go():
        ctx = cheb.Context()
        Vd = torch.from_numpy(V.copy()).cuda()
        ctx.honeycomb(w, l, Vd, edge=edge)
        ctx.set_bounds(-3.5, 3.5)
        ctx.plan_order(4.0, 24)
        ctx.reserve_adjoint(K, cheb.ADJ_REVERSE)
        psi = torch.from_numpy(psi0.copy()).cuda()
        ctx.propagate(psi, K, None, None, cheb.NO_CHECK | cheb.KEEP_CHECKPOINTS)
        gbar = (2.0 * torch.from_numpy(mask).cuda() * psi).contiguous()
        dV = torch.zeros_like(Vd)
        ctx.adjoint(gbar, dV)
        torch.cuda.synchronize()
        ctx.close()
        return gbar.cpu().numpy(), dV.cpu().numpy()

    monkeypatch.setenv("CHEBTD_REV_DEPTH", "5")
    ur, gr = go()
    monkeypatch.delenv("CHEBTD_REV_DEPTH")
    monkeypatch.setenv("CHEBTD_REV_CHUNKS", str(chunks))
    say(f"[gpu] pipelined reverse {w}x{l} {edge} chunks={chunks}")
    u, g = go()
    assert rel_l2(u, ur) <= 1e-12 and np.abs(u - ur).max() <= 1e-12 * np.abs(ur).max()
    assert_grad_close(g, gr, 1e-11)
