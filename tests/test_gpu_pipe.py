"""Pipelined many-order passes over ribbons (pipe.hip) against the CPU oracle:
every pass shape at the edges of its strips, chunks and wavefront hand-overs."""
import numpy as np
import pytest

import oracle as O
from test_gpu_deep import run
from test_gpu_parity import assert_state_close, honey_case, rel_l2, say

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


SHAPES = ["2,4", "3,4", "4,4", "5,4", "3,8"]


# rows below, at and past the orders of a pass and of a chunk; columns below,
# at and past a strip's own columns (112, 104, 96, 88 and 80 of them); M below,
# at and past the pass depth, so that inner passes and padded last ones run
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("edge", ["zigzag", "armchair"])
@pytest.mark.parametrize("w,l,chunks", [(1, 81, 1), (2, 2, 1), (7, 80, 1), (20, 89, 1), (25, 177, 1), (53, 96, 3),
                                        (70, 209, 4)])
def test_pipelined_shapes_match_oracle(torch, cheb, monkeypatch, shape, edge, w, l, chunks):
    monkeypatch.setenv("CHEBTD_PIPE", shape)
    monkeypatch.setenv("CHEBTD_PIPE_CHUNKS", str(chunks))
    dw, nw = map(int, shape.split(","))
    case = honey_case(w, l, edge, state="dense")
    for M in (3, dw * nw, dw * nw + 1, 2 * dw * nw + 5):
        say(f"[gpu] pipelined {shape} {w}x{l} {edge} chunks={chunks} M={M}")
        ctx, psi, nrm, en, plan = run(torch, cheb, case, 1.0, 2, M=M)
        ref, rn, re = O.propagate(case["H"], plan, case["psi0"], 2, want_obs=True)
        ctx.close()
        assert_state_close(psi, ref)
        np.testing.assert_allclose(nrm, rn, rtol=1e-12)
        np.testing.assert_allclose(en, re, rtol=1e-10, atol=1e-12)


# a site's arithmetic does not depend on the shape, the chunks or the number
# of passes: the same bits; and more steps than the partial sums in flight
def test_pipelined_bits_do_not_depend_on_the_shape(torch, cheb, monkeypatch):
    case = honey_case(41, 230, "zigzag", state="dense")
    first = None
    for shape in SHAPES:
        for chunks in ("1", "2"):
            monkeypatch.setenv("CHEBTD_PIPE", shape)
            monkeypatch.setenv("CHEBTD_PIPE_CHUNKS", chunks)
            say(f"[gpu] pipelined bits {shape} chunks={chunks}")
            ctx, psi, nrm, en, plan = run(torch, cheb, case, 1.0, 70)
            ctx.close()
            if first is None:
                first = psi
                _, rn, re = O.propagate(case["H"], plan, case["psi0"], 70, want_obs=True)
            np.testing.assert_array_equal(psi, first)
            np.testing.assert_allclose(nrm, rn, rtol=1e-12)
            np.testing.assert_allclose(en, re, rtol=1e-10, atol=1e-12)


# checkpoints of the pipelined head, and the steps replayed from a graph
def test_pipelined_checkpoints_and_graph(torch, cheb):
    case = honey_case(33, 190, "armchair", state="dense")
    _, p1, n1, e1, plan = run(torch, cheb, case, 1.0, 5)
    _, p2, n2, e2, _ = run(torch, cheb, case, 1.0, 5, flags=cheb.GRAPH)
    np.testing.assert_array_equal(p1, p2)
    np.testing.assert_array_equal(n1, n2)
    np.testing.assert_array_equal(e1, e2)
    from test_gpu_adjoint import gpu_adjoint
    import workloads as W
    mask = W.random_weights(33 * 190, 3)
    eps, _ = W.ribbon_inputs(33, 190, 0.5, 0)
    H = O.honeycomb(33, 190, eps, edge="armchair")
    lo, hi = H.gershgorin()
    _, g, u0, prop = gpu_adjoint(torch, cheb, "honeycomb", dict(width=33, length=190, edge="armchair"), eps,
                                 case["psi0"], mask, (lo, hi), 1.0, 3, cheb.ADJ_STEP)
    _, gr, ur = O.adjoint(H, O.Plan(lo, hi, 1.0), case["psi0"], 3, mask)
    assert rel_l2(g, gr) <= 1e-8 and rel_l2(u0, ur) <= 1e-10


# the step-end pairs v_{M-1}, v_M of a checkpointing run come from exact
# pipelined passes and, where M is no multiple of four, one pass of the rest:
# every remainder, one and several passes, through the downward adjoint
@pytest.mark.parametrize("dt", [0.42, 0.46, 0.5, 0.55, 1.0, 1.07, 1.14, 1.2, 4.0])
def test_pipelined_step_ends(torch, cheb, dt):
    import workloads as W
    from test_gpu_adjoint import assert_grad_close, gpu_adjoint
    w, l, edge = 50, 130, "zigzag"
    case = honey_case(w, l, edge, state="dense")
    eps, _ = W.ribbon_inputs(w, l, 0.5, 0)
    mask = W.random_weights(w * l, 3)
    H = O.honeycomb(w, l, eps, edge=edge)
    lo, hi = H.gershgorin()
    _, g, u0, prop = gpu_adjoint(torch, cheb, "honeycomb", dict(width=w, length=l, edge=edge), eps, case["psi0"], mask,
                                 (lo, hi), dt, 2, cheb.ADJ_REVERSE)
    say(f"[gpu] pipelined step ends dt={dt} M={prop.M}")
    _, gr, ur = O.adjoint(H, O.Plan(lo, hi, dt), case["psi0"], 2, mask)
    assert_grad_close(g, gr)
    assert_state_close(u0, ur)
