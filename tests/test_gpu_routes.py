"""Calls whose kernel or launch shape a rule picks, on either side of the rule's
lines, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from test_gpu_deep import run
from test_gpu_parity import _hermitian_csr, assert_state_close, chain_case, dev, gpu_context, honey_case, host, say

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


# the arrays are borrowed: a matrix of more entries, written over them after it
# was registered, is what the next call runs
def test_csr_copy_stays_inside_its_room(torch, cheb, monkeypatch):
    monkeypatch.setenv("CHEBTD_CSR_COPY", "1")
    n = 300
    rng = np.random.default_rng(3)

    def matrix(fill):
        A = np.diag(rng.standard_normal(n)).astype(np.complex128)
        for i in range(0, n - fill, 2):
            A[i, i + fill] = A[i + fill, i] = rng.standard_normal()
        rowptr, cols, vals = _hermitian_csr(A)
        return rowptr, cols.astype(np.int32), vals

    small, large = matrix(n), matrix(7)
    room = len(large[1])
    assert len(small[1]) < room
    r_d = dev(torch, small[0])
    c_d = torch.zeros(room, dtype=torch.int32, device="cuda")
    v_d = torch.zeros(room, dtype=torch.complex128, device="cuda")
    c_d[:len(small[1])] = dev(torch, small[1])
    v_d[:len(small[1])] = dev(torch, small[2])
    psi0 = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    psi0 /= np.linalg.norm(psi0)
    ctx = cheb.Context()
    ctx.csr(r_d, c_d[:len(small[1])], v_d[:len(small[1])])
    ctx.set_bounds(-12.0, 12.0)
    ctx.plan_order(0.2, 12)
    say("[gpu] csr arrays rewritten with more entries")
    for rowptr, cols, vals in (small, large):
        r_d.copy_(dev(torch, rowptr))
        c_d[:len(cols)] = dev(torch, cols)
        v_d[:len(cols)] = dev(torch, vals)
        psi = dev(torch, psi0)
        ctx.propagate(psi, 2, None, None, cheb.NO_CHECK)
        torch.cuda.synchronize()
        H = O.import_csr(rowptr, cols.astype(np.int64), vals)
        ref, _, _ = O.propagate(H, O.Plan(-12.0, 12.0, 0.2, M=12), psi0, 2, want_obs=True)
        assert_state_close(host(psi), ref)
    ctx.close()


def tridiagonal(n, off):
    """rowptr, col, val of a Hermitian tridiagonal matrix."""
    i = np.arange(n)
    col = i[:, None] + np.array([-1, 0, 1])
    val = np.broadcast_to(np.array([np.conj(off), 0.5, off]), col.shape)
    keep = (col >= 0) & (col < n)
    rowptr = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64)
    return rowptr, col[keep].astype(np.int32), val[keep].astype(np.complex128)


# the timed CSR kernel is the one that a call of one step runs
@pytest.mark.parametrize("off,M,name", [(0.3, 12, "k_iter_csr<OpCsrCopy>"), (0.3, 5, "k_iter_csr<OpCsr>"),
                                        (0.3 + 0.1j, 12, "k_iter_csr<OpCsr>")])
def test_csr_timing_names_the_kernel_that_runs(torch, cheb, off, M, name):
    n = 360000
    arrays = [dev(torch, a) for a in tridiagonal(n, off)]
    assert arrays[1].numel() > 1 << 20
    ctx = cheb.Context()
    ctx.csr(*arrays)
    ctx.set_bounds(-2.0, 2.0)
    ctx.plan_order(0.5, M)
    ms, got, orders = ctx.time_recursion_kernel(3)
    ctx.close()
    assert got == name and orders == 1 and ms > 0


# the rows' shape that the rule above counts on, found when the matrix is
# registered: one long row in every wavefront's 64 and the copy does not pay
@pytest.mark.parametrize("every,copied", [(0, True), (64, False), (360000, False)])
def test_csr_uneven_rows_are_not_copied(torch, cheb, every, copied):
    n = 360000
    rowptr, col, val = tridiagonal(n, 0.3)
    cnt = np.diff(rowptr)
    if every:
        cnt[::every] += 200
        rng = np.random.default_rng(1)
        col = rng.integers(0, n, int(cnt.sum())).astype(np.int32)
        val = np.zeros(col.size, dtype=np.complex128)
        rowptr = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
    ctx = cheb.Context()
    arrays = [dev(torch, a) for a in (rowptr, col, val)]
    ctx.csr(*arrays)
    ctx.set_bounds(-2.0, 2.0)
    ctx.plan_order(0.5, 80)
    _, name, _ = ctx.time_recursion_kernel(2)
    ctx.close()
    assert ("Copy" in name) == copied


# steps of few orders on ribbons run as walks inside the run whose sums go over
# several steps: every route with sums, checks, graphs and driven steps, more
# steps than the sums in flight
@pytest.mark.parametrize("w,l,edge,M,kernel", [(61, 300, "zigzag", 2, "k_pair"), (61, 300, "armchair", 3, "k_deep"),
                                               (130, 131, "zigzag", 5, "k_deep"), (50, 70, "armchair", 6, "k_deep"),
                                               (40, 500, "zigzag", 3, "k_deep"), (700, 9, "zigzag", 9, "k_deep"),
                                               (700, 9, "armchair", 10, "k_deep"), (61, 300, "zigzag", 7, "k_pipe"),
                                               (10, 300, "zigzag", 3, "k_ribbon_tile")])
def test_steps_of_few_orders(torch, cheb, w, l, edge, M, kernel):
    K, dt = 70, 0.05
    case = honey_case(w, l, edge, state="dense")
    say(f"[gpu] few orders {w}x{l} {edge} M={M}")
    ctx, psi, nrm, en, plan = run(torch, cheb, case, dt, K, M=M)
    assert ctx.time_recursion_kernel(2)[1].startswith(kernel)
    ref, rn, re = O.propagate(case["H"], plan, case["psi0"], K, want_obs=True)
    assert_state_close(psi, ref)
    np.testing.assert_allclose(nrm, rn, rtol=1e-12)
    np.testing.assert_allclose(en, re, rtol=1e-10, atol=1e-12)
    # checked, without sums, replayed from a graph, driven by a constant on-site term
    ctx.set_check_tol(1.0)
    p = dev(torch, case["psi0"])
    ctx.propagate(p, K)
    np.testing.assert_array_equal(host(p), psi)
    n2, e2 = torch.zeros(K, dtype=torch.float64, device="cuda"), torch.zeros(K, dtype=torch.float64, device="cuda")
    for k in (K, 5):
        p = dev(torch, case["psi0"])
        n2.zero_()
        ctx.propagate(p, k, n2, e2, cheb.GRAPH)
        np.testing.assert_array_equal(host(n2)[:k], nrm[:k])
        np.testing.assert_array_equal(host(e2)[:k], en[:k])
    p = dev(torch, case["psi0"])
    ctx.propagate_td(p, case["eps_dev"].repeat(K, 1), n2, e2)
    np.testing.assert_array_equal(host(p), psi)
    np.testing.assert_array_equal(host(n2), nrm)
    # a state that is not finite still ends with the error
    p = dev(torch, case["psi0"])
    p[w * l // 2] = float("nan")
    with pytest.raises(cheb.ChebError):
        ctx.propagate(p, 3)
    ctx.close()


# a batch of five orders everywhere takes them in one walk, as one system does
# with that depth; one system of six orders and all run pipelined
@pytest.mark.parametrize("dt,orders", [(0.004, {5}), (0.00545, {5, 6})])
def test_batch_of_few_orders(torch, cheb, monkeypatch, dt, orders):
    import test_gpu_batch as B
    specs = [(7, 300, 0.6, 2, "armchair"), (64, 513, 1.2, 9, "zigzag"), (33, 129, 0.9, 3, "zigzag"),
             (5, 1025, 0.5, 5, "armchair")]
    systems = B.make_systems(specs, torch)
    ctx = cheb.Context()
    ctx.batch_create(systems, dt)
    assert {int(M) for M in ctx.batch_info()} == orders
    ctx.batch_set_schedule(cheb.SCHED_DEEP, 1024, 256, 1)
    say(f"[gpu] batch of few orders dt={dt}")
    ctx.batch_propagate(3, cheb.GRAPH)
    torch.cuda.synchronize()
    monkeypatch.setenv("CHEBTD_DEPTH", "5")
    for s in systems:
        got = s["psi"].cpu().numpy()
        ref = O.propagate(s["H"], O.Plan(s["emin"], s["emax"], dt), s["psi0"], 3)
        assert_state_close(got, ref)
        if orders == {5}:
            one = cheb.Context()
            one.honeycomb(s["width"], s["length"], s["eps"], edge=s["edge"])
            one.set_bounds(s["emin"], s["emax"])
            one.plan(dt)
            p = dev(torch, s["psi0"])
            one.propagate(p, 3)
            np.testing.assert_array_equal(host(p), got)
            one.close()
    ctx.close()


# checkpointing runs of few orders, walked, under each adjoint schedule
@pytest.mark.parametrize("mode", ["ADJ_STEP", "ADJ_SQRTM", "ADJ_REVERSE"])
@pytest.mark.parametrize("w,l,edge,M", [(61, 130, "zigzag", 2), (61, 130, "armchair", 3), (50, 70, "zigzag", 5),
                                        (40, 90, "zigzag", 3), (700, 9, "zigzag", 9)])
def test_gradients_of_few_orders(torch, cheb, w, l, edge, M, mode):
    from test_gpu_adjoint import assert_grad_close, ribbon_inputs
    K, dt = 3, 0.05
    V, psi0, mask = ribbon_inputs(w, l, dense=True)
    H = O.honeycomb(w, l, V, edge=edge)
    lo, hi = H.gershgorin()
    say(f"[gpu] gradient of few orders {w}x{l} {edge} M={M} {mode}")
    ctx = cheb.Context()
    Vd = dev(torch, V)
    ctx.honeycomb(w, l, Vd, edge=edge)
    ctx.set_bounds(lo, hi)
    ctx.plan_order(dt, M)
    assert ctx.time_recursion_kernel(1)[1].startswith(("k_deep", "k_pair"))
    ctx.reserve_adjoint(K, getattr(cheb, mode))
    psi = dev(torch, psi0)
    ctx.propagate(psi, K, None, None, cheb.NO_CHECK | cheb.KEEP_CHECKPOINTS)
    gbar = (2.0 * dev(torch, mask) * psi).contiguous()
    dV = torch.zeros_like(Vd)
    ctx.adjoint(gbar, dV)
    torch.cuda.synchronize()
    ctx.close()
    _, gr, ur = O.adjoint(H, O.Plan(lo, hi, dt, M=M), psi0, K, mask)
    assert_grad_close(host(dV), gr)
    assert_state_close(host(gbar), ur)


# chains whose kept steps of few orders are walked, and one below
@pytest.mark.parametrize("n,M", [(600001, 2), (599999, 2), (1300007, 3), (1300007, 4)])
def test_gradients_of_few_orders_on_long_chains(torch, cheb, n, M):
    import workloads as W
    from test_gpu_adjoint import assert_grad_close
    K, dt, dx = 2, 0.05, 0.8
    V, psi0, mask = W.random_weights(n, 400 + M), W.random_state(n, 500 + M), W.random_weights(n, 600 + M)
    H = O.chain1d(V, dx)
    lo, hi = H.gershgorin()
    say(f"[gpu] gradient of few orders on a chain of {n} M={M}")
    ctx = cheb.Context()
    Vd = dev(torch, V)
    ctx.chain1d(Vd, dx)
    ctx.set_bounds(lo, hi)
    ctx.plan_order(dt, M)
    ctx.reserve_adjoint(K, cheb.ADJ_REVERSE)
    psi = dev(torch, psi0)
    ctx.propagate(psi, K, None, None, cheb.NO_CHECK | cheb.KEEP_CHECKPOINTS)
    gbar = (2.0 * dev(torch, mask) * psi).contiguous()
    dV = torch.zeros_like(Vd)
    ctx.adjoint(gbar, dV)
    torch.cuda.synchronize()
    ctx.close()
    _, gr, ur = O.adjoint(H, O.Plan(lo, hi, dt, M=M), psi0, K, mask)
    assert_grad_close(host(dV), gr)
    assert_state_close(host(gbar), ur)


# a few tall ribbons in a batch are cut into hundreds of chunks, uneven ones
# into different numbers
@pytest.mark.parametrize("dt", [0.1, 1.0, 1.6])
@pytest.mark.parametrize("specs", [[(900, 30, 0.6, 2, "armchair")],
                                   [(1501, 9, 0.6, 2, "zigzag"), (333, 120, 1.2, 9, "armchair"), (40, 41, 0.9, 3, "zigzag")]])
def test_batch_of_tall_ribbons(torch, cheb, specs, dt):
    import test_gpu_batch as B
    systems = B.make_systems(specs, torch)
    ctx = cheb.Context()
    ctx.batch_create(systems, dt)
    ctx.batch_set_schedule(cheb.SCHED_DEEP, 1024, 256, 1)
    say(f"[gpu] batch of tall ribbons dt={dt} M={ctx.batch_info()}")
    ctx.batch_propagate(3, cheb.GRAPH)
    torch.cuda.synchronize()
    for s in systems:
        ref = O.propagate(s["H"], O.Plan(s["emin"], s["emax"], dt), s["psi0"], 3)
        assert_state_close(s["psi"].cpu().numpy(), ref)
    ctx.close()


# batches whose strips fill the chip, of flat ribbons, alike and not
@pytest.mark.parametrize("dt", [0.4, 1.6])
@pytest.mark.parametrize("specs", [[(1, 120001, 0.6, 2, "armchair")],
                                   [(2, 60000, 0.6, 2, "zigzag"), (1, 70003, 1.2, 9, "armchair"), (31, 900, 0.9, 3, "zigzag")]])
def test_batch_of_flat_ribbons(torch, cheb, specs, dt):
    import test_gpu_batch as B
    systems = B.make_systems(specs, torch)
    ctx = cheb.Context()
    ctx.batch_create(systems, dt)
    ctx.batch_set_schedule(cheb.SCHED_DEEP, 1024, 256, 1)
    say(f"[gpu] batch of flat ribbons dt={dt} M={ctx.batch_info()}")
    ctx.batch_propagate(3, cheb.GRAPH)
    torch.cuda.synchronize()
    for s in systems:
        ref = O.propagate(s["H"], O.Plan(s["emin"], s["emax"], dt), s["psi0"], 3)
        assert_state_close(s["psi"].cpu().numpy(), ref)
    ctx.close()


# tall ribbons of few columns in a batch run two single-wavefront passes a step
# of ten orders, where all are such
@pytest.mark.parametrize("specs", [[(2200, 16, 0.6, 2, "zigzag"), (3001, 9, 0.6, 9, "armchair")],
                                   [(2200, 16, 0.6, 2, "zigzag"), (3001, 41, 0.6, 9, "armchair")]])
def test_batch_of_tall_narrow_ribbons(torch, cheb, specs):
    import test_gpu_batch as B
    systems = B.make_systems(specs, torch)
    dt = next(float(t) for t in np.arange(0.01, 0.2, 0.001)
              if all(O.Plan(s["emin"], s["emax"], t).M == 10 for s in systems))
    ctx = cheb.Context()
    ctx.batch_create(systems, dt)
    ctx.batch_set_schedule(cheb.SCHED_DEEP, 1024, 256, 1)
    say(f"[gpu] batch of tall narrow ribbons dt={dt} M={ctx.batch_info()}")
    ctx.batch_propagate(3, cheb.GRAPH)
    torch.cuda.synchronize()
    for s in systems:
        ref = O.propagate(s["H"], O.Plan(s["emin"], s["emax"], dt), s["psi0"], 3)
        assert_state_close(s["psi"].cpu().numpy(), ref)
    ctx.close()
