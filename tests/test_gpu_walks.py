"""The single-wavefront passes in the split that the plan picks by itself
(CHEBTD_WALK=1: also where pipelined or tiled passes would take the steps), and
the batched ones of five and six orders (CHEBTD_BATCH_DEPTH=5), against the CPU
oracle and each other."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_batch import SMALL, batch_deep_split, make_systems
from test_gpu_deep import run
from test_gpu_parity import assert_state_close, dev, honey_case, host, say
from windows import ribbon_sample_sites, ribbon_sites

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


# every M from 2 to 30: passes of two to six orders in all their mixtures
@pytest.mark.parametrize("w,l,edge", [(21, 131, "armchair"), (70, 59, "zigzag"), (1, 300, "zigzag"), (64, 3, "armchair")])
def test_walked_splits_match_oracle(torch, cheb, monkeypatch, w, l, edge):
    monkeypatch.setenv("CHEBTD_WALK", "1")
    case = honey_case(w, l, edge, state="dense")
    for M in range(2, 31):
        say(f"[gpu] walked {w}x{l} {edge} M={M}")
        ctx, psi, nrm, en, plan = run(torch, cheb, case, 1.0, 2, M=M)
        passes = ctx.plan_passes()
        ms, name, orders = ctx.time_recursion_kernel(1)
        assert sum(passes) == M and orders in passes and name.startswith("k_deep" if orders > 2 else "k_pair")
        ctx.close()
        ref, rn, re = O.propagate(case["H"], plan, case["psi0"], 2, want_obs=True)
        assert_state_close(psi, ref)
        np.testing.assert_allclose(nrm, rn, rtol=1e-12)
        np.testing.assert_allclose(en, re, rtol=1e-10, atol=1e-12)


# the batch's passes of five and six orders are those of each system's own plan
# (M = 17 .. 22), hence the same bits at every chunk height
@pytest.mark.parametrize("rows", [None, "3", "22", "40"])
@pytest.mark.parametrize("K", [1, 2, 3])
def test_batch_deep_equals_walked_systems_bitwise(torch, cheb, monkeypatch, K, rows):
    monkeypatch.setenv("CHEBTD_BATCH_DEPTH", "5")
    monkeypatch.setenv("CHEBTD_WALK", "1")
    if rows is not None:
        monkeypatch.setenv("CHEBTD_BATCH_DEEP_ROWS", rows)
    systems = make_systems(SMALL, torch)
    ctx = cheb.Context()
    ctx.batch_create(systems, 1.0)
    ctx.batch_set_schedule(cheb.SCHED_DEEP, 1024, 256, 1)
    say(f"[gpu] batch deep K={K} rows={rows}")
    ctx.batch_propagate(K, cheb.GRAPH)
    torch.cuda.synchronize()
    Ms = [int(M) for M in ctx.batch_info()]
    assert {6, 5} <= {d for M in Ms for d in batch_deep_split(M)}
    for s, M in zip(systems, Ms):
        one = cheb.Context()
        one.honeycomb(s["width"], s["length"], s["eps"], edge=s["edge"])
        one.set_bounds(s["emin"], s["emax"])
        one.plan(1.0)
        assert one.plan_passes() == batch_deep_split(M)
        assert one.time_recursion_kernel(1)[1].startswith("k_deep")
        p = dev(torch, s["psi0"])
        one.propagate(p, K)
        np.testing.assert_array_equal(host(p), s["psi"].cpu().numpy())
        one.close()
        ref = O.propagate(s["H"], O.Plan(s["emin"], s["emax"], 1.0), s["psi0"], K)
        assert_state_close(s["psi"].cpu().numpy(), ref)
    ctx.close()


# large lattices, sampled sites: streaming stores and 52-row chunks from 16M
# sites on, and the top of the 32-bit offsets ((W + 14) L 16 B = 2^31)
@pytest.mark.parametrize("w,l,edge", [(512, 32768, "zigzag"), (2034, 65536, "zigzag"), (2034, 65536, "armchair")])
def test_walked_large_lattices_sampled(torch, cheb, monkeypatch, w, l, edge):
    monkeypatch.setenv("CHEBTD_WALK", "1")
    eps = W.anderson_disorder(w, l, 0.5, 7)
    psi0 = W.random_state(w * l, 707)
    ctx = cheb.Context()
    eps_d = torch.from_numpy(eps).cuda()
    ctx.honeycomb(w, l, eps_d, edge=edge)
    lo, hi = ctx.gershgorin()
    ctx.set_bounds(lo, hi, 0.01)
    M = ctx.plan(1.0)
    passes = ctx.plan_passes()
    assert set(passes) == {5} and sum(passes) == M
    assert ctx.time_recursion_kernel(1)[1] == f"k_deep<{int(edge == 'armchair')},5,false,true>"
    psi = torch.from_numpy(psi0).cuda()
    nrm = torch.zeros(2, dtype=torch.float64, device="cuda")
    say(f"[gpu] walked {w}x{l} {edge}, passes {passes}")
    ctx.propagate(psi, 2, nrm, None, 0)
    torch.cuda.synchronize()
    np.testing.assert_allclose(host(nrm), 1.0, rtol=1e-12)
    sites = set(ribbon_sample_sites(w, l, 16, 23))
    u = W.uniform01(29, 12)
    for k in range(6):  # the last rows, where the offsets are largest
        sites.add((w - 1 - k, int(u[2 * k] * l)))
        sites.add((w - 1 - k, l - 1 - int(u[2 * k + 1] * 64)))
    sites = sorted(sites)
    got = host(psi[torch.tensor([y * l + x for y, x in sites], device="cuda")])
    ctx.close()
    ref = ribbon_sites(w, l, edge, eps, psi0, O.Plan(lo, hi, 1.0), 2, sites)
    assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
