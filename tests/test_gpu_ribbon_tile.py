"""Register-resident passes over ribbons of up to 48 rows (ribbon_tile.hip)
against the CPU oracle and, bit for bit, the pipelined passes."""
import numpy as np
import pytest

import oracle as O
from test_gpu_deep import run
from test_gpu_parity import assert_state_close, honey_case, say

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


# every number of rows per wavefront (2, 4, 6), full and ragged last
# wavefronts, the most rows and one more (pipelined); columns below, at and past a strip's own (the
# depths leave 126 .. 32 of them); odd and even depths, every remainder of the
# four-order loop, one pass and several
@pytest.mark.parametrize("edge", ["zigzag", "armchair"])
@pytest.mark.parametrize("w,l", [(1, 2), (2, 3), (3, 33), (10, 200), (16, 88), (17, 89), (32, 61), (33, 130), (47, 97),
                                 (48, 32), (49, 121)])
def test_tiled_ribbons_match_oracle_and_pipeline(torch, cheb, monkeypatch, edge, w, l):
    case = honey_case(w, l, edge, state="dense")
    for M, D in ((2, 48), (5, 5), (20, 48), (20, 7), (48, 48), (67, 23)):
        say(f"[gpu] tiled ribbon {w}x{l} {edge} M={M} D={D}")
        monkeypatch.setenv("CHEBTD_TILE", str(D))
        ctx, psi, nrm, en, plan = run(torch, cheb, case, 1.0, 2, M=M)
        ctx.close()
        monkeypatch.setenv("CHEBTD_TILE", "0")
        ctx, pp, pn, pe, _ = run(torch, cheb, case, 1.0, 2, M=M)
        ctx.close()
        ref, rn, re = O.propagate(case["H"], plan, case["psi0"], 2, want_obs=True)
        assert_state_close(psi, ref)
        np.testing.assert_array_equal(psi, pp)
        np.testing.assert_allclose(nrm, rn, rtol=1e-12)
        np.testing.assert_allclose(en, re, rtol=1e-10, atol=1e-12)


# the step-end pairs of the downward adjoint schedule, and graph replay
@pytest.mark.parametrize("w,l,edge", [(9, 70, "zigzag"), (40, 150, "armchair")])
def test_tiled_ribbon_step_ends_and_graph(torch, cheb, monkeypatch, w, l, edge):
    monkeypatch.setenv("CHEBTD_TILE", "7")
    case = honey_case(w, l, edge, state="dense")
    _, p1, n1, e1, plan = run(torch, cheb, case, 1.0, 5)
    _, p2, n2, e2, _ = run(torch, cheb, case, 1.0, 5, flags=cheb.GRAPH)
    np.testing.assert_array_equal(p1, p2)
    np.testing.assert_array_equal(n1, n2)
    np.testing.assert_array_equal(e1, e2)
    import workloads as W
    from test_gpu_adjoint import assert_grad_close, gpu_adjoint
    eps, _ = W.ribbon_inputs(w, l, 0.5, 0)
    mask = W.random_weights(w * l, 3)
    H = O.honeycomb(w, l, eps, edge=edge)
    lo, hi = H.gershgorin()
    _, g, u0, prop = gpu_adjoint(torch, cheb, "honeycomb", dict(width=w, length=l, edge=edge), eps, case["psi0"], mask,
                                 (lo, hi), 1.0, 3, cheb.ADJ_REVERSE)
    _, gr, ur = O.adjoint(H, O.Plan(lo, hi, 1.0), case["psi0"], 3, mask)
    assert_grad_close(g, gr)
    assert_state_close(u0, ur)
