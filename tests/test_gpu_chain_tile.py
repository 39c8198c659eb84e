"""Tiled many-order passes over 1D chains (chain_tile.hip) against the CPU
oracle, at the edges of a wavefront's sites and of its orders."""
import numpy as np
import pytest

import oracle as O
from test_gpu_deep import run
from test_gpu_parity import assert_state_close, chain_case, rel_l2, say

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


# chains shorter than a wavefront's own sites, of exactly some of them and one
# more; passes of one to many orders, with every remainder of the four-order
# loop, in one pass and in several of unequal depth
@pytest.mark.parametrize("R,D", [(2, 7), (2, 40), (4, 9), (4, 64), (8, 10), (8, 61)])
@pytest.mark.parametrize("n", [2, 3, 63, 4097, 5120, 9001])
def test_tiled_passes_match_oracle(torch, cheb, monkeypatch, R, D, n):
    monkeypatch.setenv("CHEBTD_TILE", f"{R},{D}")
    case = chain_case(n, state="dense")
    for M in (2, 3, 5, D, D + 1, 2 * D + 3):
        say(f"[gpu] tiled chain n={n} R={R} D={D} M={M}")
        ctx, psi, nrm, en, plan = run(torch, cheb, case, 0.002, 2, M=M, flags=cheb.NO_PERSISTENT)
        ref, rn, re = O.propagate(case["H"], plan, case["psi0"], 2, want_obs=True)
        ctx.close()
        assert_state_close(psi, ref)
        np.testing.assert_allclose(nrm, rn, rtol=1e-12)
        np.testing.assert_allclose(en, re, rtol=1e-10, atol=1e-10 * np.abs(re).max())


def test_tiled_graph_and_driven_steps(torch, cheb):
    case = chain_case(20011, state="dense")
    ctx, p1, n1, e1, plan = run(torch, cheb, case, 0.002, 5)
    ctx.close()
    ctx, p2, n2, e2, _ = run(torch, cheb, case, 0.002, 5, flags=cheb.GRAPH)
    np.testing.assert_array_equal(p1, p2)
    np.testing.assert_array_equal(n1, n2)
    np.testing.assert_array_equal(e1, e2)
    # a constant on-site schedule through the time-dependent entry point
    V = torch.from_numpy(np.tile(case["V"], (5, 1))).cuda()
    psi = torch.from_numpy(case["psi0"].copy()).cuda()
    ctx.propagate_td(psi, V)
    np.testing.assert_array_equal(psi.cpu().numpy(), p1)
    ctx.close()


# the whole-run kernels take at most 256 steps a launch: a longer run equals
# the same run in parts, its norms, energies and end-of-call check included
@pytest.mark.parametrize("n", [129, 300, 1000])
def test_chain_run_longer_than_a_launch(torch, cheb, n):
    case = chain_case(n, state="dense")
    K = 600
    say(f"[gpu] chain run of {K} steps n={n}")
    ctx, p1, n1, e1, plan = run(torch, cheb, case, 0.001, K)
    psi = torch.from_numpy(case["psi0"].copy()).cuda()
    nrm = torch.zeros(K, dtype=torch.float64, device="cuda")
    en = torch.zeros_like(nrm)
    for a in (0, 200, 400):
        ctx.propagate(psi, 200, nrm[a:a + 200], en[a:a + 200])
    ctx.close()
    np.testing.assert_array_equal(psi.cpu().numpy(), p1)
    np.testing.assert_array_equal(nrm.cpu().numpy(), n1)
    np.testing.assert_array_equal(en.cpu().numpy(), e1)
    ref, rn, re = O.propagate(case["H"], plan, case["psi0"], K, want_obs=True)
    assert_state_close(p1, ref)
    np.testing.assert_allclose(n1, rn, rtol=1e-11)
