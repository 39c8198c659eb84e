"""Calls whose kernel or launch shape a rule picks, on either side of the rule's
lines, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from test_gpu_deep import run
from test_gpu_parity import assert_state_close, chain_case, dev, gpu_context, host, say

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


# weights in LDS, and past the orders whose weights would leave too little room
# for the runs of other streams, in memory
@pytest.mark.parametrize("M", [10050, 10300])
def test_chain_weights_in_lds_and_in_memory(torch, cheb, M):
    case = chain_case(4096, state="dense")
    lo, hi = case["H"].gershgorin()
    dt = 0.97 * M / (0.505 * (hi - lo))
    say(f"[gpu] chain n=4096 M={M}")
    ctx, psi, nrm, en, plan = run(torch, cheb, case, dt, 2, M=M)
    ctx.close()
    ref, rn, re = O.propagate(case["H"], plan, case["psi0"], 2, want_obs=True)
    assert_state_close(psi, ref)
    np.testing.assert_allclose(nrm, rn, rtol=1e-11)


# four runs of 94 workgroups each at once: all find room, each equals its run alone
def test_chain_runs_on_four_streams(torch, cheb):
    M, n = 10600, 4096
    cases = [chain_case(n, state="dense") for _ in range(4)]
    lo, hi = cases[0]["H"].gershgorin()
    dt = 0.97 * M / (0.505 * (hi - lo))
    _, alone, _, _, _ = run(torch, cheb, cases[0], dt, 2, M=M)
    streams = [torch.cuda.Stream() for _ in range(4)]
    ctxs, psis = [], []
    say("[gpu] four chain runs at once")
    for s, case in zip(streams, cases):
        with torch.cuda.stream(s):
            ctx = gpu_context(torch, cheb, case)
            ctx.set_bounds(lo, hi, 0.01)
            ctx.plan_order(dt, M)
            ctxs.append(ctx)
            psis.append(dev(torch, case["psi0"]))
    torch.cuda.synchronize()
    for ctx, psi in zip(ctxs, psis):
        ctx.propagate(psi, 2, None, None, cheb.NO_CHECK)
    torch.cuda.synchronize()
    for ctx, psi in zip(ctxs, psis):
        np.testing.assert_array_equal(host(psi), alone)
        ctx.close()
