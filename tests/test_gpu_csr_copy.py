"""Calls of many orders on a CSR matrix read a copy of it if it is real
(launch_csr_copy): against the CPU oracle, and the same bits as without."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import _hermitian_csr, assert_state_close, dev, host, say

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


def matrix(n, kind, rng):
    """Dense Hermitian of a few entries a row, with empty rows; real, with one
    imaginary pair in the last rows, or complex."""
    A = np.zeros((n, n), dtype=np.complex128)
    for i in range(n):
        if i % 11 == 5:
            continue
        for j in rng.integers(0, n, size=int(rng.integers(1, 4))):
            if j % 11 != 5:
                x = rng.standard_normal() + (1j * rng.standard_normal() if kind == "complex" and i != j else 0)
                A[i, j] = x
                A[j, i] = np.conj(x)
    if kind == "one" and n > 1:
        A[n - 1, 0], A[0, n - 1] = 0.25j, -0.25j
    return A


# sizes at and around a wavefront, a block and several blocks; every flag path
@pytest.mark.parametrize("kind", ["real", "one", "complex"])
@pytest.mark.parametrize("n", [1, 63, 65, 257, 900])
def test_csr_copy_matches_oracle(torch, cheb, monkeypatch, n, kind):
    rng = np.random.default_rng(n)
    A = matrix(n, kind, rng)
    if n == 1:
        A[0, 0] = 0.5
    rowptr, cols, vals = _hermitian_csr(A)
    H = O.import_csr(rowptr, cols.astype(np.int64), vals)
    r_d, c_d, v_d = (dev(torch, a) for a in (rowptr, cols, vals))
    psi0 = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    psi0 /= np.linalg.norm(psi0)
    radius = float(np.abs(A).sum(axis=1).max()) + 1.0
    for M, K, flags in ((1, 3, 0), (9, 3, 0), (9, 4, cheb.GRAPH), (2, 5, cheb.GRAPH)):
        got = []
        for force in ("0", "1"):
            monkeypatch.setenv("CHEBTD_CSR_COPY", force)
            say(f"[gpu] csr copy n={n} {kind} M={M} K={K} force={force}")
            ctx = cheb.Context()
            ctx.csr(r_d, c_d, v_d)
            ctx.set_bounds(-radius, radius)
            ctx.plan_order(0.2, M)
            psi = dev(torch, psi0)
            nrm = torch.zeros(K, dtype=torch.float64, device="cuda")
            ctx.propagate(psi, K, nrm, None, flags | cheb.NO_CHECK)
            torch.cuda.synchronize()
            got.append((host(psi), host(nrm)))
            ctx.close()
        np.testing.assert_array_equal(got[1][0], got[0][0])
        np.testing.assert_array_equal(got[1][1], got[0][1])
        ref, _, _ = O.propagate(H, O.Plan(-radius, radius, 0.2, M=M), psi0, K, want_obs=True)
        assert_state_close(got[1][0], ref)


# the arrays are borrowed: what they hold at the next call counts
def test_csr_copy_sees_new_values(torch, cheb, monkeypatch):
    monkeypatch.setenv("CHEBTD_CSR_COPY", "1")
    rng = np.random.default_rng(7)
    A = matrix(130, "real", rng)
    rowptr, cols, vals = _hermitian_csr(A)
    r_d, c_d, v_d = (dev(torch, a) for a in (rowptr, cols, vals))
    psi0 = rng.standard_normal(130) + 1j * rng.standard_normal(130)
    psi0 /= np.linalg.norm(psi0)
    ctx = cheb.Context()
    ctx.csr(r_d, c_d, v_d)
    ctx.set_bounds(-20.0, 20.0)
    ctx.plan_order(0.2, 12)
    for scale in (1.0, 0.5):
        v_d.copy_(dev(torch, vals * scale))
        psi = dev(torch, psi0)
        ctx.propagate(psi, 2, None, None, cheb.NO_CHECK)
        torch.cuda.synchronize()
        H = O.import_csr(rowptr, cols.astype(np.int64), vals * scale)
        ref, _, _ = O.propagate(H, O.Plan(-20.0, 20.0, 0.2, M=12), psi0, 2, want_obs=True)
        assert_state_close(host(psi), ref)
    ctx.close()
