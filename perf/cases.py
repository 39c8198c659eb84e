"""The workloads this library is timed on, through its public entry points.

They follow the paper's applications (arXiv:0907.3022, Sect. 3) and the sizes
of this repository's benchmark: disordered honeycomb ribbons from a few
thousand to tens of millions of sites, the double well and longer 1D chains,
the Holstein polaron matrix-free and as a general sparse matrix, many ribbons
at once, and the gradient of a transmitted probability.  listed() names one
case per kind of use, draw() gives further ones of the same ranges, and
exact() computes a case's result in plain torch, 64 bits, without the library.
"""
import math

import numpy as np
import torch

import paper_0907_3022_amd as P

DEV = "cuda"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # one step of a small ribbon at a time, each followed by the density and the
        # transmitted probability: a program that watches a packet, bound by latency
        dict(name="stepwise_ribbon_32x512", kind="ribbon", width=32, length=512, edge="zigzag", dt=1.0, K=1, obs=True),
        # the armchair ribbon of Table 2 (10 x 1000 atoms) with its middle time step
        dict(name="table2_ribbon_10x1000", kind="ribbon", width=10, length=1000, edge="armchair", dt=10.0, K=10,
             obs=False),
        # the benchmark's ribbon: 20 steps with the norm and energy of each
        dict(name="ribbon_128x8192", kind="ribbon", width=128, length=8192, edge="zigzag", dt=1.0, K=20, obs=False),
        # a ribbon of odd sizes under an on-site term that changes from step to step
        dict(name="driven_ribbon_301x5003", kind="driven", width=301, length=5003, edge="armchair", dt=1.0, K=4),
        # a ribbon far larger than the last-level cache (33.5M sites)
        dict(name="ribbon_1024x32768", kind="ribbon", width=1024, length=32768, edge="zigzag", dt=1.0, K=2, obs=False),
        # the double well of Sect. 3.1 on 4096 points: thousands of orders per step
        dict(name="double_well_4096", kind="chain", n=4096, dt=0.5, z=0.0, K=2),
        # a chain of the benchmark's gradient workload, run forwards (order 64)
        dict(name="chain_65536", kind="chain", n=65536, dt=0.0, z=30.5, K=20),
        # the Holstein ring (1.85M states) with the polaron observables
        dict(name="holstein_ring_L10", kind="holstein", L=10, nph=10, w0=1.0, periodic=True, dt=0.1, K=5),
        # the open chain of Fig. 3 at 12 sites and 11 phonons (16.2M states)
        dict(name="polaron_L12_nph11", kind="holstein", L=12, nph=11, w0=2.0, periodic=False, dt=0.5, K=1),
        # the ring's Hamiltonian handed over as a general sparse matrix
        dict(name="csr_ring_L10", kind="csr", L=10, nph=10, w0=1.0, periodic=True, dt=0.1, K=5),
        # 64 disorder realisations of uneven ribbons in one batch
        dict(name="batch_64_ribbons", kind="batch", nsys=64, wmin=32, wmax=128, lmin=512, lmax=4096, dt=1.0, K=4),
        # forward and backward pass of the gradient workload, 4 steps of order 64
        dict(name="gradient_ribbon_256x4096", kind="gradient", geom="honeycomb", width=256, length=4096, n=0, z=30.5,
             K=4),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["ribbon", "ribbon", "ribbon", "driven", "chain", "chain", "holstein", "csr", "batch", "gradient"])
    edge = rng.choice(["zigzag", "armchair"])
    if kind in ("ribbon", "driven"):
        w, l = _log(rng, 4, 1024), _log(rng, 64, 32768)
        dt = round(math.exp(rng.uniform(math.log(0.5), math.log(20.0))), 3)
        K = _log(rng, 1, 20)
        # no more work than the largest listed ribbon's
        while K > 1 and w * l * K * max(20.0, 4.0 * dt) > 1.2e9:
            K -= 1
        if w * l * max(20.0, 4.0 * dt) > 1.2e9:
            dt = 1.0
        c = dict(kind=kind, width=w, length=l, edge=edge, dt=dt, K=min(K, 6) if kind == "driven" else K)
        if kind == "ribbon":
            c["obs"] = rng.random() < 0.3
        return c
    if kind == "chain":
        if rng.random() < 0.5:  # the double well's lengths
            return dict(kind="chain", n=_log(rng, 150, 4096), dt=round(rng.uniform(0.02, 0.5), 3), z=0.0,
                        K=rng.randint(1, 2))
        return dict(kind="chain", n=_log(rng, 4500, 1 << 20), dt=0.0, z=round(rng.uniform(8.0, 80.0), 2),
                    K=rng.randint(1, 20))
    if kind in ("holstein", "csr"):
        while True:
            L, nph = rng.randint(4, 12), rng.randint(3, 11)
            states = L * math.comb(L + nph, nph)
            if 2000 <= states <= (16300000 if kind == "holstein" else 2000000):
                break
        return dict(kind=kind, L=L, nph=nph, w0=rng.choice([1.0, 2.0]), periodic=rng.random() < 0.5,
                    dt=rng.choice([0.1, 0.2, 0.5]), K=rng.randint(1, 5) if states < 4000000 else 1)
    if kind == "batch":
        wmin, lmin = rng.randint(8, 64), _log(rng, 128, 1024)
        return dict(kind="batch", nsys=_log(rng, 2, 64), wmin=wmin, wmax=wmin + rng.randint(0, 64), lmin=lmin,
                    lmax=lmin + rng.randint(0, 3000), dt=1.0, K=rng.randint(1, 4))
    z = round(rng.uniform(5.0, 30.5), 2)
    if rng.random() < 0.5:
        return dict(kind="gradient", geom="chain", width=0, length=0, n=_log(rng, 4500, 65536), z=z, K=rng.randint(1, 4))
    return dict(kind="gradient", geom="honeycomb", width=_log(rng, 8, 256), length=_log(rng, 64, 4096), n=0, z=z,
                K=rng.randint(1, 4))


# --------------------------------------------------------------------------
# inputs, made on the GPU from the seed
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(seed, count):
    """A few numbers in [0, 1) of the seed, on the host."""
    return np.random.RandomState(seed & 0x7FFFFFFF).random_sample(count)


def _ribbon_inputs(w, l, seed, strength=0.5):
    """Disorder in [-strength/2, strength/2) and a Gaussian packet moving in x,
    injected about a quarter of the length in."""
    u = _uniform(seed, 3)
    eps = strength * (torch.rand(w * l, generator=_gen(seed), device=DEV, dtype=torch.float64) - 0.5)
    sigma, x0, y0, k0 = min(20.0, w / 4.0), l * (0.2 + 0.1 * u[0]), (w - 1) / 2.0, 0.8 + 0.4 * u[1]
    y = torch.arange(w, device=DEV, dtype=torch.float64)[:, None]
    x = torch.arange(l, device=DEV, dtype=torch.float64)[None, :]
    env = torch.exp(-((x - x0) ** 2 + (y - y0) ** 2) / (4.0 * sigma * sigma))
    env = env / env.square().sum().sqrt()
    psi = torch.complex(env * torch.cos(k0 * x), env * torch.sin(k0 * x)).reshape(-1).contiguous()
    return eps, psi


def _chain_inputs(n, seed):
    """The quartic double well on [-20, 20] and a packet in its left well."""
    u = _uniform(seed, 3)
    dx = 40.0 / (n - 1)
    x = -20.0 + dx * torch.arange(n, device=DEV, dtype=torch.float64)
    V = 0.05 * (x * x - (4.8 + 0.4 * u[0]) ** 2) ** 2
    env = torch.exp(-((x + 5.0 - 0.5 * u[1]) ** 2) / 4.0)
    env = env / env.square().sum().sqrt()
    k0 = 0.8 + 0.4 * u[2]
    return dx, V, torch.complex(env * torch.cos(k0 * x), env * torch.sin(k0 * x))


def _holstein_inputs(c, seed):
    """Couplings, site energies and a bare electron packet in the phonon vacuum."""
    L, u = c["L"], _uniform(seed, c["L"] + 2)
    g = np.full(L, math.sqrt(0.5 + 0.5 * u[L]))
    delta = 0.2 * (u[:L] - 0.5)
    nconf = math.comb(L + c["nph"], c["nph"])
    i = np.arange(L)
    e = np.exp(-((i - L / 3.0) ** 2) / 8.0 + 1j * (0.2 + 0.3 * u[L + 1]) * i)
    psi = torch.zeros(L * nconf, dtype=torch.complex128, device=DEV)
    psi[::nconf] = torch.from_numpy(e / np.linalg.norm(e)).to(DEV)
    return g, delta, psi


def _batch_sizes(c, seed):
    u = _uniform(20000, 2 * c["nsys"])  # the shapes are the case's, not the seed's
    return [(c["wmin"] + int(u[2 * s] * (c["wmax"] - c["wmin"] + 1)), c["lmin"] + int(u[2 * s + 1] * (c["lmax"] - c["lmin"] + 1)))
            for s in range(c["nsys"])]


def _batch_seed(seed, s):
    return seed * 1009 + 7 * s


def _ahead(geom, c, x=None):
    """1 ahead of the packet's start, 0 behind it."""
    if geom == "chain":
        return (x > -5.0).to(torch.float64)
    return (torch.arange(c["length"], device=DEV) > c["length"] / 4.0).to(torch.float64).repeat(c["width"])


def _chain_dt(c, lo, hi):
    return c["dt"] if c["z"] == 0.0 else c["z"] / (0.5 * 1.01 * (hi - lo))


def _ribbon_bounds(width, length, eps, edge):
    with P.Context() as probe:
        probe.honeycomb(width, length, eps, edge=edge)
        return probe.gershgorin()


def prepare(case, seed):
    c, kind = case, case["kind"]
    st = dict(case=case)
    if kind in ("ribbon", "driven"):
        eps, psi = _ribbon_inputs(c["width"], c["length"], seed)
        ctx = P.Context()
        ctx.honeycomb(c["width"], c["length"], eps, edge=c["edge"])
        lo, hi = ctx.gershgorin()
        if kind == "driven":  # a gate voltage ahead of the packet, ramped over the steps
            ramp = torch.linspace(0.1, 0.4, c["K"], device=DEV, dtype=torch.float64)[:, None]
            st["onsite"] = (eps[None, :] + ramp * _ahead("honeycomb", c)[None, :]).contiguous()
            hi += 0.4
        ctx.set_bounds(lo, hi)
        ctx.plan(c["dt"])
        st.update(ctx=ctx, psi=psi, norm=torch.zeros(c["K"], dtype=torch.float64, device=DEV),
                  energy=torch.zeros(c["K"], dtype=torch.float64, device=DEV))
        if c.get("obs"):
            st["mask"] = _ahead("honeycomb", c).to(torch.uint8)
    elif kind == "chain":
        dx, V, psi = _chain_inputs(c["n"], seed)
        ctx = P.Context()
        ctx.chain1d(V, dx)
        lo, hi = ctx.gershgorin()
        ctx.set_bounds(lo, hi)
        ctx.plan(_chain_dt(c, lo, hi))
        st.update(ctx=ctx, psi=psi, norm=torch.zeros(c["K"], dtype=torch.float64, device=DEV))
    elif kind in ("holstein", "csr"):
        g, delta, psi = _holstein_inputs(c, seed)
        ctx = P.Context()
        if kind == "holstein":
            ctx.holstein(c["L"], c["nph"], 1.0, c["w0"], g, delta, c["periodic"])
        else:
            rowptr, col, val = P.holstein_csr_host(c["L"], c["nph"], 1.0, c["w0"], g, delta, c["periodic"])
            ctx.csr(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV), torch.from_numpy(val).to(DEV))
        ctx.set_bounds(*ctx.gershgorin())
        ctx.plan(c["dt"])
        st.update(ctx=ctx, psi=psi, norm=torch.zeros(c["K"], dtype=torch.float64, device=DEV))
    elif kind == "batch":
        systems = []
        for s, (w, l) in enumerate(_batch_sizes(c, seed)):
            eps, psi = _ribbon_inputs(w, l, _batch_seed(seed, s))
            lo, hi = _ribbon_bounds(w, l, eps, "zigzag")
            systems.append(dict(width=w, length=l, eps=eps, psi=psi, emin=lo, emax=hi))
        ctx = P.Context()
        ctx.batch_create(systems, c["dt"])
        ctx.batch_set_schedule(P.SCHED_DEEP, 4096, 512, 1)  # what the autotuner picks and its cache file holds
        st.update(ctx=ctx, psi=[s["psi"] for s in systems])
    else:
        if c["geom"] == "chain":
            dx, V, psi0 = _chain_inputs(c["n"], seed)
            with P.Context() as probe:
                probe.chain1d(V, dx)
                lo, hi = probe.gershgorin()
            mask = _ahead("chain", c, torch.linspace(-20.0, 20.0, c["n"], device=DEV, dtype=torch.float64))
            prop = P.Propagator("chain", c["z"] / (0.5 * 1.01 * (hi - lo)), c["K"], (lo, hi), dx=dx)
        else:
            V, psi0 = _ribbon_inputs(c["width"], c["length"], seed)
            lo, hi = _ribbon_bounds(c["width"], c["length"], V, "zigzag")
            mask = _ahead("honeycomb", c)
            prop = P.Propagator("honeycomb", c["z"] / (0.5 * 1.01 * (hi - lo)), c["K"], (lo, hi), width=c["width"],
                                length=c["length"])
        st.update(prop=prop, V=V.requires_grad_(True), psi=psi0.requires_grad_(True), mask=mask)
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(st):
    c, kind = st["case"], st["case"]["kind"]
    if kind == "ribbon":
        ctx, psi = st["ctx"], st["psi"]
        ctx.propagate(psi, c["K"], st["norm"], st["energy"])
        out = dict(psi=psi, norm=st["norm"], energy=st["energy"])
        if c["obs"]:
            out["density"] = ctx.density(psi)
            out["transmitted"] = ctx.region_sum(psi, st["mask"])
        return out
    if kind == "driven":
        st["ctx"].propagate_td(st["psi"], st["onsite"], st["norm"], st["energy"])
        return dict(psi=st["psi"], norm=st["norm"], energy=st["energy"])
    if kind in ("chain", "csr"):
        st["ctx"].propagate(st["psi"], c["K"], st["norm"])
        return dict(psi=st["psi"], norm=st["norm"])
    if kind == "holstein":
        st["ctx"].propagate(st["psi"], c["K"], st["norm"])
        n_i, nph, chi = st["ctx"].holstein_obs(st["psi"])
        return dict(psi=st["psi"], norm=st["norm"], n=n_i, nph=nph, chi=chi)
    if kind == "batch":
        st["ctx"].batch_propagate(c["K"], P.GRAPH)
        return dict(psi=list(st["psi"]))
    V, psi0 = st["V"], st["psi"]
    psi = P.ChebPropagate.apply(V, psi0, st["prop"])
    loss = (st["mask"] * torch.view_as_real(psi).square().sum(-1)).sum()
    dV, dpsi0 = torch.autograd.grad(loss, (V, psi0))
    return dict(psi=psi.detach(), loss=loss.detach(), dV=dV, dpsi0=dpsi0)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _order(z):
    """Orders a step of spectral half-width times dt = z needs to 1e-15."""
    return int(z + 9.5 * max(z, 1.0) ** (1.0 / 3.0) + 3.0)


def work(case):
    c, kind = case, case["kind"]
    if kind == "batch":
        n = sum(w * l for w, l in _batch_sizes(c, 0))
        return dict(bytes=40.0 * n, flops=20.0 * n * _order(3.3 * c["dt"]) * c["K"])
    if kind in ("ribbon", "driven", "chain"):
        n = c["n"] if kind == "chain" else c["width"] * c["length"]
        if kind == "chain":
            dx = 40.0 / (c["n"] - 1)
            z = c["z"] or 0.505 * c["dt"] * (2.0 / dx ** 2 + 7031.0)
        else:
            z = 3.3 * c["dt"]
        per = 32.0 + 8.0 * (c["K"] if kind == "driven" else 1) + (9.0 if c.get("obs") else 0.0)
        return dict(bytes=per * n, flops=(20.0 if kind != "chain" else 18.0) * n * _order(z) * c["K"])
    if kind in ("holstein", "csr"):
        n = c["L"] * math.comb(c["L"] + c["nph"], c["nph"])
        z = c["dt"] * 0.505 * (c["nph"] * c["w0"] + 4.0 + 2.0 * c["w0"] * math.sqrt(c["nph"]))
        per = 32.0 if kind == "holstein" else 32.0 + 8.0 + 4.0 * 20.0
        return dict(bytes=per * n, flops=(30.0 if kind == "holstein" else 48.0) * n * _order(z) * c["K"])
    n = c["n"] if c["geom"] == "chain" else c["width"] * c["length"]
    return dict(bytes=(16.0 + 8.0 + 16.0 + 8.0 + 8.0 + 16.0) * n, flops=3 * 20.0 * n * _order(c["z"]) * c["K"])


# --------------------------------------------------------------------------
# the same results in plain torch
# --------------------------------------------------------------------------
def _bessel(z):
    """J_0 .. J_m(z) by Miller's backward recurrence, m where they fall below 1e-18."""
    m = int(z + 14.0 * max(z, 1.0) ** (1.0 / 3.0) + 20.0)
    j, up, cur = [0.0] * (m + 2), 0.0, 1e-280
    for k in range(m + 1, 0, -1):
        j[k] = cur
        up, cur = cur, 2.0 * k / z * cur - up
        if abs(cur) > 1e250:
            up, cur = up * 1e-250, cur * 1e-250
            j[k:] = [v * 1e-250 for v in j[k:]]
    j[0] = cur
    norm = j[0] + 2.0 * math.fsum(j[2::2])
    j = [v / norm for v in j]
    while len(j) > 2 and abs(j[-1]) < 1e-18:
        j.pop()
    return j


def _plan(lo, hi, dt):
    a, b = 0.5 * 1.02 * (hi - lo), 0.5 * (hi + lo)
    j = _bessel(a * dt)
    phase = complex(math.cos(b * dt), -math.sin(b * dt))
    return a, b, [phase * (2.0 if k else 1.0) * (-1j) ** (k % 4) * v for k, v in enumerate(j)]


def _step(H, psi, plan):
    a, b, g = plan
    prev, cur = psi, (H(psi) - b * psi) / a
    out = g[0] * prev + g[1] * cur
    for w in g[2:]:
        prev, cur = cur, (2.0 / a) * (H(cur) - b * cur) - prev
        out = out + w * cur
    return out


def _ribbon_h(w, l, edge):
    par = (torch.arange(w, device=DEV)[:, None] + torch.arange(l, device=DEV)[None, :]) % 2

    def apply(v, eps):
        v = v.view(w, l)
        zr, zc = torch.zeros_like(v[:1]), torch.zeros_like(v[:, :1])
        down, up = torch.cat((v[1:], zr)), torch.cat((zr, v[:-1]))
        right, left = torch.cat((v[:, 1:], zc), 1), torch.cat((zc, v[:, :-1]), 1)
        if edge == "zigzag":
            s = left + right + torch.where(par == 0, down, up)
        else:
            s = down + up + torch.where(par == 0, right, left)
        return (eps.view(w, l) * v - s).reshape(-1)

    return apply


def _chain_h(V, dx):
    z = torch.zeros(1, dtype=torch.complex128, device=DEV)
    return lambda v, pot: (1.0 / dx ** 2 + pot) * v - (0.5 / dx ** 2) * (torch.cat((z, v[:-1])) + torch.cat((v[1:], z)))


def _ne(H, psi):
    return torch.stack((psi.abs().square().sum(), torch.vdot(psi, H(psi)).real))


def _holstein_h(c, g, delta):
    """Configurations by total then lexicographically, each found by its key."""
    L, nph, B = c["L"], c["nph"], c["nph"] + 2
    key, tot = torch.zeros(1, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    for _ in range(L):
        reps = nph - tot + 1
        first = torch.repeat_interleave(torch.cumsum(reps, 0) - reps, reps)
        digit = torch.arange(first.numel(), device=DEV) - first
        key, tot = torch.repeat_interleave(key, reps) * B + digit, torch.repeat_interleave(tot, reps) + digit
    top = B ** L
    key = (tot * top + key).sort().values
    tot = key // top
    up, dn, ru, rd = [], [], [], []
    for s in range(L):
        p = B ** (L - 1 - s)
        n = (key // p) % B
        iu = torch.searchsorted(key, key + top + p).clamp(max=key.numel() - 1)
        idn = torch.searchsorted(key, key - top - p).clamp(max=key.numel() - 1)
        up.append(iu)
        dn.append(idn)
        ru.append(torch.where(tot < nph, (n + 1).double().sqrt(), 0.0))
        rd.append(n.double().sqrt())
    tot = tot.double()
    occ = [v.square() for v in rd]

    def apply(v):
        v = v.view(L, -1)
        out = torch.empty_like(v)
        for s in range(L):
            hop = torch.zeros_like(v[s])
            for q in (s - 1, s + 1):
                if c["periodic"] or 0 <= q < L:
                    hop = hop + v[q % L]
            ph = ru[s] * v[s][up[s]] + rd[s] * v[s][dn[s]]
            out[s] = (float(delta[s]) + c["w0"] * tot) * v[s] - hop - float(g[s]) * c["w0"] * ph
        return out.reshape(-1)

    def observables(v):
        v = v.view(L, -1)
        d = v.abs().square()
        every = d.sum(0)
        n = d.sum(1)
        ph = torch.stack([(occ[s] * every).sum() for s in range(L)])
        chi = torch.stack([2.0 * (v[s].conj() * ru[s] * v[s][up[s]]).real.sum() for s in range(L)])
        return n, ph, chi

    span = float(np.abs(g).max()) * c["w0"] * (2.0 * math.sqrt(nph) + 1.0) + 2.0
    return apply, observables, float(delta.min()) - span, float(delta.max()) + nph * c["w0"] + span


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("ribbon", "driven"):
        eps, psi = _ribbon_inputs(c["width"], c["length"], seed)
        H = _ribbon_h(c["width"], c["length"], c["edge"])
        plan = _plan(float(eps.min()) - 3.0, float(eps.max()) + 3.4, c["dt"])
        ramp = torch.linspace(0.1, 0.4, c["K"], device=DEV, dtype=torch.float64)
        ne = []
        for k in range(c["K"]):
            e = eps + ramp[k] * _ahead("honeycomb", c) if kind == "driven" else eps
            ne.append(_ne(lambda v: H(v, e), psi))
            psi = _step(lambda v: H(v, e), psi, plan)
        ne = torch.stack(ne)
        out = dict(psi=psi, norm=ne[:, 0], energy=ne[:, 1])
        if c.get("obs"):
            out["density"] = psi.abs().square()
            out["transmitted"] = (out["density"] * _ahead("honeycomb", c)).sum().reshape(1)
        return out
    if kind == "chain":
        dx, V, psi = _chain_inputs(c["n"], seed)
        lo, hi = float(V.min()), 2.0 / dx ** 2 + float(V.max())
        H = _chain_h(V, dx)
        glo, ghi = _chain_gershgorin(V, dx)
        plan, norm = _plan(lo, hi, _chain_dt(c, glo, ghi)), []
        if len(plan[2]) * c["K"] > 40000:
            return None
        for _ in range(c["K"]):
            norm.append(psi.abs().square().sum())
            psi = _step(lambda v: H(v, V), psi, plan)
        return dict(psi=psi, norm=torch.stack(norm))
    if kind in ("holstein", "csr"):
        g, delta, psi = _holstein_inputs(c, seed)
        H, observables, lo, hi = _holstein_h(c, g, delta)
        plan, norm = _plan(lo, hi, c["dt"]), []
        for _ in range(c["K"]):
            norm.append(psi.abs().square().sum())
            psi = _step(H, psi, plan)
        out = dict(psi=psi, norm=torch.stack(norm))
        if kind == "holstein":
            out["n"], out["nph"], out["chi"] = observables(psi)
        return out
    if kind == "batch":
        out = []
        for s, (w, l) in enumerate(_batch_sizes(c, seed)):
            eps, psi = _ribbon_inputs(w, l, _batch_seed(seed, s))
            H = _ribbon_h(w, l, "zigzag")
            plan = _plan(float(eps.min()) - 3.0, float(eps.max()) + 3.0, c["dt"])
            for _ in range(c["K"]):
                psi = _step(lambda v: H(v, eps), psi, plan)
            out.append(psi)
        return dict(psi=out)
    # the gradient, by torch's own differentiation of the recursion
    if c["geom"] == "chain":
        dx, V, psi0 = _chain_inputs(c["n"], seed)
        lo, hi = _chain_gershgorin(V, dx)
        H, mask = _chain_h(V, dx), _ahead("chain", c, torch.linspace(-20.0, 20.0, c["n"], device=DEV, dtype=torch.float64))
    else:
        V, psi0 = _ribbon_inputs(c["width"], c["length"], seed)
        lo, hi = _ribbon_gershgorin(c["width"], c["length"], V)
        H, mask = _ribbon_h(c["width"], c["length"], "zigzag"), _ahead("honeycomb", c)
    plan = _plan(lo, hi, c["z"] / (0.5 * 1.01 * (hi - lo)))
    V, psi0 = V.requires_grad_(True), psi0.requires_grad_(True)
    psi = psi0
    for _ in range(c["K"]):
        psi = _step(lambda v: H(v, V), psi, plan)
    loss = (mask * torch.view_as_real(psi).square().sum(-1)).sum()
    dV, dpsi0 = torch.autograd.grad(loss, (V, psi0))
    return dict(psi=psi.detach(), loss=loss.detach(), dV=dV, dpsi0=dpsi0)


def _chain_gershgorin(V, dx):
    """Diagonal minus and plus the neighbours' magnitudes, as the step dt = z / a is defined by."""
    d = 1.0 / dx ** 2 + V
    r = torch.full_like(V, 1.0 / dx ** 2)
    r[0] = r[-1] = 0.5 / dx ** 2
    return float((d - r).min()), float((d + r).max())


def _ribbon_gershgorin(w, l, eps):
    """The same of a zigzag ribbon: every bond of a site counts 1."""
    x, y = torch.arange(l, device=DEV)[None, :], torch.arange(w, device=DEV)[:, None]
    r = (x > 0).long() + (x + 1 < l).long() + torch.where((x + y) % 2 == 0, y + 1 < w, y > 0).long()
    return float((eps.view(w, l) - r).min()), float((eps.view(w, l) + r).max())
