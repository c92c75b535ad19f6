"""Performance cases: what a program that uses this library has it do, through
its public entry points, over the range of sizes it is used at.

Kinds of a case (each a grid of N buses, B lines, G generators over T periods):
  sweep    one replay of the evaluation sweep's graph: objective, gradient,
           constraints, Jacobian, Hessian, J^T v and condensed matrix
  batch    the same sweep over k uneven instances in one model
  adjoint  constraints and their backward pass through torch.autograd
  iterate  the evaluation half of an interior-point iteration: gradient,
           constraints, condensed right-hand side, J + H + K, step recovery
  newton   the linear-algebra half: factorization of K and one solve
  solve    one more solve with a factorization that is already there
  ipm      the first iterations of a whole interior-point solve
Everything is FP64, the library's only type.  Inputs come from the seed;
"tuned" cases take their launch shapes from the committed tuning file,
as bench.py does, the others run on the library's defaults.
"""
import dataclasses
import math
import os

import numpy as np
import torch

from paper_2405_14032_amd import capi, synth
from paper_2405_14032_amd.autograd import OpfCons

TUNE = os.path.join(os.path.dirname(capi.__file__), "tune", "mi355x.json")


def listed():
    return [
        # the smallest grid, called in a loop: launches and latency are all there is
        dict(name="sweep_tiny", kind="sweep", N=14, B=20, G=5, T=4, tuned=False),
        # a transmission grid over one day: an ordinary evaluation
        dict(name="sweep_mid", kind="sweep", N=2000, B=3200, G=400, T=24, tuned=False),
        # a continental grid over a week of hours: the benchmark's headline workload
        dict(name="sweep_paper", kind="sweep", N=10000, B=13000, G=2000, T=168, tuned=True),
        # 64 uneven grids in one model (scenario sets): ragged tiles
        dict(name="batch64", kind="batch", k=64, tuned=True),
        # forward and backward of the constraints inside a torch program
        dict(name="adjoint16", kind="adjoint", k=16, N=2000, B=3200, G=400, T=24, tuned=True),
        # an interior-point iteration's evaluation, a day-ahead grid over a week
        dict(name="iterate_week", kind="iterate", N=2000, B=3200, G=400, T=168, tuned=False),
        # factorization and solve: the smallest grid
        dict(name="newton_tiny", kind="newton", N=14, B=20, G=5, T=4),
        # the ordinary grid over one day
        dict(name="newton_mid", kind="newton", N=2000, B=3200, G=400, T=24),
        # a small grid over ten weeks of hours: a long chain of small fronts
        dict(name="newton_long", kind="newton", N=118, B=186, G=54, T=1680),
        # the continental grid over a week: the largest factorization
        dict(name="newton_paper", kind="newton", N=10000, B=13000, G=2000, T=168),
        # further right-hand sides on one factorization
        dict(name="solve_week", kind="solve", N=2000, B=3200, G=400, T=168),
        # the first iterations of a whole solve, loads capped so that it has a feasible point
        dict(name="ipm_mid", kind="ipm", N=2000, B=3200, G=400, T=24, iters=3),
    ]


def draw(rng):
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["sweep", "sweep", "batch", "adjoint", "iterate", "newton", "newton", "newton", "solve", "ipm"])
    if kind == "batch":
        return dict(kind=kind, k=rng.randint(3, 48), tuned=False)
    most = {"sweep": 10000, "adjoint": 2000, "iterate": 6000}.get(kind, 3000)
    N = logu(14, most)
    c = dict(kind=kind, N=N, B=int(N * rng.uniform(1.3, 1.6)), G=max(1, int(N * rng.uniform(0.18, 0.46))),
             T=logu(1, 168))
    if kind in ("sweep", "adjoint", "iterate"):
        c["tuned"] = False
    if kind == "adjoint":
        c.update(k=rng.randint(1, 12), T=min(c["T"], 48))
    if kind == "ipm":
        c.update(iters=rng.randint(1, 3), T=min(c["T"], 48))
    return c


def networks(case, seed):
    """The grids of a case: the topology is the user's own and stays, the loads of an interior-point solve are
    the seed's day."""
    if case["kind"] == "batch":
        return synth.batched_networks(case["k"])
    nets = [synth.make_network(case["N"], case["B"], case["G"], case["T"], synth.ADJOINT_SEED0 + i)
            for i in range(case.get("k", 1))]
    if case["kind"] == "ipm":
        day = np.random.default_rng(seed).uniform(0.9, 1.1, (case["T"], case["N"]))
        nets = [synth.cap_load(dataclasses.replace(n, pd=n.pd * day, qd=n.qd * day), 0.3) for n in nets]
    return nets


class Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.dev = torch.device("cuda:0")
        self.g = torch.Generator(device=self.dev).manual_seed(1 + seed)

    def uniform(self, shape, lo=0.0, hi=1.0):
        u = torch.rand(shape, generator=self.g, device=self.dev, dtype=torch.float64)
        return lo + (hi - lo) * u

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device=self.dev, dtype=torch.float64)

    def logu(self, n, lo, hi):
        return 10.0 ** self.uniform((n,), lo, hi)

    def point(self, net):
        t = lambda a: torch.as_tensor(a, device=self.dev)
        T = net.T
        u = lambda lo, hi: t(lo) + (t(hi) - t(lo)) * self.uniform((T, len(lo)))
        parts = [self.uniform((T, net.N), 0.9, 1.1), self.uniform((T, net.N), -0.5, 0.5),
                 u(net.pmin, net.pmax), u(net.qmin, net.qmax)]
        parts += [u(-net.rate, net.rate) for _ in range(4)]
        return torch.cat(parts, dim=1).reshape(-1)


def inputs(case, seed):
    """Grids and input tensors of a case, without the library."""
    nets, d = networks(case, seed), Draw(seed)
    n, m = sum(k.n for k in nets), sum(k.m for k in nets)
    s = {"x": torch.cat([d.point(k) for k in nets])}
    kind = case["kind"]
    if kind in ("sweep", "batch"):
        # weights over eight decades, as the condensation meets them
        s.update(lam=d.normal(m), v=d.normal(m), diag_x=d.logu(n, -4, 4), dcon=d.logu(m, -4, 4))
    elif kind == "adjoint":
        t = lambda key: torch.cat([torch.as_tensor(getattr(k, key), device=d.dev).reshape(-1) for k in nets])
        s.update(pd=t("pd"), qd=t("qd"), gc=d.normal(m))
    elif kind in ("newton", "solve"):
        # objective-only Hessian (the multipliers of a first iterate are 0): K is positive definite
        s.update(diag_x=d.logu(n, -3, 3), dcon=d.logu(m, -3, 3), want=d.normal(n))
    elif kind == "iterate":
        s.update(bounds_draws=[d.uniform((n,), 0.05, 0.95), d.uniform((m,), 0.05, 0.95), d.normal(n), d.normal(m)],
                 mult=[d.logu(k, -3, 1) for k in (n, n, m, m)], y=d.normal(m), dx=1e-2 * d.normal(n))
    return nets, s


def inside(lo, hi, u, z):
    """Strictly inside [lo, hi]; entries without bounds take z (bounds come in pairs or with one side infinite)."""
    fl, fh = torch.isfinite(lo), torch.isfinite(hi)
    both = lo.nan_to_num(posinf=0, neginf=0) + u * (hi - lo).nan_to_num(posinf=0, neginf=0)
    out = torch.where(fl & fh, both, z)
    out = torch.where(fl & ~fh, lo + z.abs() + 0.05, out)
    return torch.where(~fl & fh, hi - z.abs() - 0.05, out)


def bounds_of(nets, dev):
    """Variable and row bounds of the grids, in the library's order."""
    lx, ux, lc, uc = [], [], [], []
    inf = np.inf
    for k in nets:
        one, big = np.ones, 1e-4
        lx.append(np.tile(np.concatenate([k.vmin, -inf * one(k.N), k.pmin, k.qmin, -inf * one(4 * k.B)]), k.T))
        ux.append(np.tile(np.concatenate([k.vmax, inf * one(k.N), k.pmax, k.qmax, inf * one(4 * k.B)]), k.T))
        eq = one(2 * k.N + 1 + 4 * k.B) * big  # equality rows, relaxed to +-1e-4
        lc += [np.tile(np.concatenate([-eq, -inf * one(2 * k.B), k.angmin]), k.T), np.tile(-k.ramp, k.T - 1)]
        uc += [np.tile(np.concatenate([eq, k.rate ** 2, k.rate ** 2, k.angmax]), k.T), np.tile(k.ramp, k.T - 1)]
    return [torch.as_tensor(np.concatenate(a), device=dev) for a in (lx, ux, lc, uc)]


def iterate_state(nets, s):
    """An interior iterate of the lifted method."""
    xl, xu, sl, su = bounds_of(nets, s["x"].device)
    ux, us, zx, zs = s["bounds_draws"]
    keep = lambda a, b: torch.where(torch.isfinite(b), a, torch.zeros_like(a))
    zl, zu, vl, vu = (keep(a, b) for a, b in zip(s["mult"], (xl, xu, sl, su)))
    return dict(x=inside(xl, xu, ux, zx), s=inside(sl, su, us, zs), y=s["y"], zl=zl, zu=zu, vl=vl, vu=vu,
                xl=xl, xu=xu, sl=sl, su=su), dict(mu=0.1, delta_w=1e-4, delta_c=1e-6)


def prepare(case, seed):
    nets, s = inputs(case, seed)
    M = capi.Model(nets, device=0)
    M.use_current_torch_stream()
    if case.get("tuned"):
        M.autotune(TUNE)
    e = lambda k: torch.empty(k, dtype=torch.float64, device="cuda:0")
    st = {"kind": case["kind"], "M": M, **s}
    kind = case["kind"]
    if kind in ("sweep", "batch"):
        out = dict(f=e(M.ninst), grad=e(M.n), c=e(M.m), jvals=e(M.nnz_jac), hvals=e(M.nnz_hess), jtv=e(M.n),
                   kvals=e(M.nnz_kkt))
        st["out"] = out
        st["args"] = M.sweep_args(x=s["x"], lam=s["lam"], sigma=1.0, v=s["v"], diag_x=s["diag_x"], dcon=s["dcon"], **out)
    elif kind == "adjoint":
        for k in ("x", "pd", "qd"):
            st[k].requires_grad_(True)
    elif kind == "iterate":
        keep, par = iterate_state(nets, s)
        st["iter"], st["cst"] = keep, M.ipm_state(**keep, **par)
        st["ly"] = -keep["y"]
        st["out"] = dict(grad=e(M.n), c=e(M.m), diag_x=e(M.n), dcon=e(M.m), rhs=e(M.n), jvals=e(M.nnz_jac),
                         hvals=e(M.nnz_hess), kvals=e(M.nnz_kkt), ds=e(M.m), dy=e(M.m), dzl=e(M.n), dzu=e(M.n),
                         dvl=e(M.m), dvu=e(M.m))
    elif kind in ("newton", "solve"):
        jv, hv, kv = e(M.nnz_jac), e(M.nnz_hess), e(M.nnz_kkt)
        M.eval_jhk(s["x"], torch.zeros(M.m, dtype=torch.float64, device="cuda:0"), 1.0, s["diag_x"], s["dcon"],
                   jv, hv, kv)
        del jv
        # the right-hand side of a known solution: b = K want = (H + diag + J^T D J) want
        jw, b = e(M.m), e(M.n)
        M.jprod(s["x"], s["want"], jw)
        M.jtprod(s["x"], jw.mul_(s["dcon"]), b)
        b += s["diag_x"] * s["want"]
        for k, net in enumerate(nets):  # the objective's diagonal on the generators
            p = slice(int(M.x_off[k]), int(M.x_off[k + 1]))
            g = slice(2 * net.N, 2 * net.N + net.G)
            c2 = torch.as_tensor(net.c2, device="cuda:0")
            b[p].view(net.T, -1)[:, g] += 2.0 * c2 * s["want"][p].view(net.T, -1)[:, g]
        st.update(kv=kv, b=b, dx=e(M.n), npert=torch.zeros(1, dtype=torch.int32, device="cuda:0"), F=capi.Chol(M))
        for k in ("x", "diag_x", "dcon", "want"):
            del st[k]
        if kind == "solve":
            st["F"].factor(kv, 0.0, 1.0, st["npert"])
    elif kind == "ipm":
        st.update(F=capi.Chol(M), iters=case["iters"], xo=e(M.n), yo=e(M.m))
    return st


def run(st):
    M, kind = st["M"], st["kind"]
    if kind in ("sweep", "batch"):
        M.sweep_graph(st["args"])
        return st["out"]
    if kind == "adjoint":
        st["x"].grad = st["pd"].grad = st["qd"].grad = None
        c = OpfCons.apply(st["x"], st["pd"], st["qd"], M)
        c.backward(st["gc"])
        return dict(c=c.detach(), gx=st["x"].grad, gpd=st["pd"].grad, gqd=st["qd"].grad)
    if kind == "iterate":
        o, x = st["out"], st["iter"]["x"]
        M.eval_grad(x, o["grad"])
        M.eval_cons(x, o["c"])
        M.condensed_rhs(st["cst"], o["grad"], o["c"], o["diag_x"], o["dcon"], o["rhs"])
        M.eval_jhk(x, st["ly"], 1.0, o["diag_x"], o["dcon"], o["jvals"], o["hvals"], o["kvals"])
        M.recover_step(st["cst"], o["c"], st["dx"], o["ds"], o["dy"], o["dzl"], o["dzu"], o["dvl"], o["dvu"])
        return o
    if kind == "newton":
        st["F"].factor(st["kv"], 0.0, 1.0, st["npert"])
        st["F"].solve(st["b"], st["dx"])
        return dict(dx=st["dx"], npert=st["npert"])
    if kind == "solve":
        st["F"].solve(st["b"], st["dx"])
        return dict(dx=st["dx"], npert=st["npert"])
    r = capi.ipm_solve(M, st["F"], st["xo"], st["yo"], max_iter=st["iters"])
    return dict(x=st["xo"], y=st["yo"], objective=r["objective"], iterations=r["iterations"],
                factorizations=r["factorizations"])


def work(case):
    nets = networks(case, 0)
    sm = lambda f: float(sum(f(k) for k in nets))
    n, m = sm(lambda k: k.n), sm(lambda k: k.m)
    nj = sm(lambda k: k.T * (2 * k.G + 30 * k.B + 1) + 2 * k.G * (k.T - 1))
    nh = sm(lambda k: k.T * (k.G + 40 * k.B))
    BT, NT = sm(lambda k: k.B * k.T), sm(lambda k: k.N * k.T)
    kind = case["kind"]
    if kind == "adjoint":
        # x, loads in, c out; x, cotangent in, three gradients out
        return {"bytes": 8 * (3 * n + 2 * m + 4 * NT), "flops": 150.0 * BT}
    M = capi.Model(nets, device=-1)
    nk = float(M.nnz_kkt)
    if kind in ("sweep", "batch"):
        # x, v, diag_x, D, six multipliers per line and period, loads in; everything else out
        return {"bytes": 8 * (4 * n + 3 * m + 6 * BT + 2 * NT + nj + nh + nk), "flops": 700.0 * BT}
    if kind == "iterate":
        # the state once, its outputs once, x and y again as little as can be
        return {"bytes": 8 * (13 * n + 13 * m + 2 * NT + nj + nh + nk), "flops": 900.0 * BT}
    i = capi.Chol(M).info()  # the analysis' own count of operations and factor entries
    fac, ent = float(i["flops"]), float(i["factor_entries"])
    if kind == "newton":
        return {"bytes": 8 * (nk + 2 * n + ent), "flops": fac + 4 * ent}
    if kind == "solve":
        return {"bytes": 8 * (ent + 2 * n), "flops": 4 * ent}
    its = case["iters"]
    return {"bytes": its * 8 * (26 * n + 26 * m + nj + nh + 2 * nk + ent), "flops": its * (fac + 4 * ent + 900.0 * BT)}


# ---- the same quantities in plain torch, in 64 bits

def split(net, x):
    return x.view(net.T, -1).split([net.N, net.N, net.G, net.G] + [net.B] * 4, dim=1)


def flows(net, vi, vj, d):
    """Pi-model flows leaving the two ends (pf, qf, pt, qt) of every line."""
    t = lambda a: torch.as_tensor(a, device=vi.device)
    y = 1.0 / (net.r + 1j * net.x)
    g, b, h = t(y.real), t(y.imag), t(net.b_charge / 2)
    w, cs, sn = vi * vj, torch.cos(d), torch.sin(d)
    return (g * vi * vi - w * (g * cs + b * sn), -(b + h) * vi * vi - w * (g * sn - b * cs),
            g * vj * vj - w * (g * cs - b * sn), -(b + h) * vj * vj + w * (g * sn + b * cs))


def rows(net, x, pd, qd):
    """All constraint rows."""
    vm, va, pg, qg, pf, qf, pt, qt = split(net, x)
    ix = lambda a: torch.as_tensor(np.asarray(a, dtype=np.int64), device=x.device)
    f, t, gb = ix(net.f_bus), ix(net.t_bus), ix(net.gen_bus)
    d = va[:, f] - va[:, t]
    phi = flows(net, vm[:, f], vm[:, t], d)
    bal = lambda gen, a, b, load: (torch.zeros_like(load).index_add(1, gb, gen).index_add(1, f, -a).index_add(1, t, -b)
                                   - load)
    per = torch.cat([bal(pg, pf, pt, pd), bal(qg, qf, qt, qd), va[:, net.ref_bus:net.ref_bus + 1]]
                    + [a - b for a, b in zip((pf, qf, pt, qt), phi)]
                    + [pf * pf + qf * qf, pt * pt + qt * qt, d], dim=1)
    return torch.cat([per.reshape(-1), (pg[1:] - pg[:-1]).reshape(-1)])


def cost(net, x):
    c2, c1, c0 = (torch.as_tensor(a, device=x.device) for a in (net.c2, net.c1, net.c0))
    pg = split(net, x)[2]
    return (c2 * pg * pg + c1 * pg + c0).sum()


def derivatives(net, x, lam, sigma):
    """Jacobian and lower Hessian values in the library's order."""
    vm, va, pg, qg, pf, qf, pt, qt = split(net, x)
    ix = lambda a: torch.as_tensor(np.asarray(a, dtype=np.int64), device=x.device)
    f, t = ix(net.f_bus), ix(net.t_bus)
    z = [a.detach().clone().requires_grad_(True) for a in (vm[:, f], vm[:, t], va[:, f], va[:, t])]
    per = lam[:net.T * net.m_period].view(net.T, -1)[:, 2 * net.N + 1:].split([net.B] * 7, dim=1)
    one = torch.ones_like(pf)
    jb = [torch.ones_like(torch.cat([pg, qg], 1)), -one, -one, -one, -one, one[:, :1]]
    hb = [torch.as_tensor(2.0 * sigma * net.c2, device=x.device).expand(net.T, net.G)]
    for k, phi in enumerate(flows(net, z[0], z[1], z[2] - z[3])):
        g1 = torch.autograd.grad(phi.sum(), z, create_graph=True, allow_unused=True)
        jb += [one] + [-a.detach() for a in g1]
        skip = (1, 1) if k < 2 else (0, 0)
        for r in range(4):
            g2 = torch.autograd.grad(g1[r].sum(), z, retain_graph=True, allow_unused=True)
            hb += [-per[k] * (g2[q].detach() if g2[q] is not None else 0.0 * one) for q in range(r + 1) if (r, q) != skip]
    jb += [2 * pf, 2 * qf, 2 * pt, 2 * qt, one, -one]
    hb += [2 * per[4], 2 * per[4], 2 * per[5], 2 * per[5]]
    ramp = torch.ones((net.T - 1, 2 * net.G), dtype=torch.float64, device=x.device)
    ramp[:, net.G:] = -1.0
    return torch.cat([torch.cat(jb, 1).reshape(-1), ramp.reshape(-1)]), torch.cat(hb, 1).reshape(-1)


def indices(net):
    """COO indices of the Jacobian and the lower Hessian, in the library's order."""
    N, B, G, T, r = net.N, net.B, net.G, net.T, lambda o, k: o + np.arange(k)
    f, t, gb = (np.asarray(a, dtype=np.int64) for a in (net.f_bus, net.t_bus, net.gen_bus))
    xo = {k: o for k, o in zip(("vm", "va", "pg", "qg", "pf", "qf", "pt", "qt"),
                               np.cumsum([0, N, N, G, G, B, B, B]))}
    co = 2 * N + 1
    four = [f, t, N + f, N + t]
    jr = [gb, N + gb, f, N + f, t, N + t, np.array([2 * N])]
    jc = [r(xo["pg"], G), r(xo["qg"], G)] + [r(xo[k], B) for k in ("pf", "qf", "pt", "qt")] + [np.array([N + net.ref_bus])]
    hr, hc = [r(xo["pg"], G)], [r(xo["pg"], G)]
    for k, name in enumerate(("pf", "qf", "pt", "qt")):
        jr += [r(co + k * B, B)] * 5
        jc += [r(xo[name], B)] + four
        for a in range(4):
            for b in range(a + 1):
                if (a, b) != ((1, 1) if k < 2 else (0, 0)):
                    hr.append(np.maximum(four[a], four[b]))
                    hc.append(np.minimum(four[a], four[b]))
    for k, name in enumerate(("pf", "qf", "pt", "qt")):
        jr.append(r(co + (4 + k // 2) * B, B))
        jc.append(r(xo[name], B))
        hr.append(r(xo[name], B))
        hc.append(r(xo[name], B))
    jr += [r(co + 6 * B, B)] * 2
    jc += [N + f, N + t]
    cat = np.concatenate
    shift = lambda a, step: (cat(a)[None, :] + step * np.arange(T)[:, None]).reshape(-1)
    rr = (T * net.m_period + np.arange((T - 1) * G)).reshape(T - 1, G)
    pg = xo["pg"] + np.arange(G) + net.n_period * np.arange(T)[:, None]
    jr = cat([shift(jr, net.m_period), cat([rr, rr], 1).reshape(-1)])
    jc = cat([shift(jc, net.n_period), cat([pg[1:], pg[:-1]], 1).reshape(-1)])
    return jr, jc, shift(hr, net.n_period), shift(hc, net.n_period)


def condensed(net, jv, hv, diag_x, dcon):
    """lower(H + diag(diag_x) + J^T D J) in CSR order."""
    import scipy.sparse as sp
    jr, jc, hr, hc = indices(net)
    n, m = net.n, net.m
    jv, hv, diag_x, dcon = (a.cpu().numpy() for a in (jv, hv, diag_x, dcon))
    mat = lambda v, i, j, shape: sp.csr_matrix((v, (i, j)), shape=shape)
    J1, J = mat(np.ones(len(jr)), jr, jc, (m, n)), mat(jv, jr, jc, (m, n))
    pat = sp.tril(J1.T @ J1 + mat(np.ones(len(hr)), hr, hc, (n, n)) + sp.identity(n)).tocoo()
    val = sp.tril(J.T @ sp.diags(dcon) @ J + mat(hv, hr, hc, (n, n)) + sp.diags(diag_x)).tocoo()
    keys = np.sort(pat.row.astype(np.int64) * n + pat.col)
    out = np.zeros(len(keys))
    out[np.searchsorted(keys, val.row.astype(np.int64) * n + val.col)] = val.data
    return torch.as_tensor(out)


def vjp(net, x, v, pd, qd):
    """c, J^T v and the gradients on the loads."""
    a = [k.detach().clone().requires_grad_(True) for k in (x, pd, qd)]
    c = rows(net, *a)
    return (c.detach(), *torch.autograd.grad((c * v).sum(), a))


def jvp(net, x, v, pd, qd):
    """J v, as the derivative of u -> u^T J v."""
    x = x.detach().clone().requires_grad_(True)
    c = rows(net, x, pd, qd)
    u = torch.zeros_like(c, requires_grad=True)
    g, = torch.autograd.grad((c * u).sum(), x, create_graph=True)
    return torch.autograd.grad((g * v).sum(), u)[0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "ipm":
        return None
    nets, s = inputs(case, seed)
    if kind in ("newton", "solve"):
        return dict(dx=s["want"], npert=None)
    dev = s["x"].device
    t = lambda a: torch.as_tensor(a, device=dev)
    if kind == "iterate":
        net, pd, qd = nets[0], t(nets[0].pd), t(nets[0].qd)
        k, par = iterate_state(nets, s)
        mu, dw, dc = par["mu"], par["delta_w"], par["delta_c"]
        x, y = k["x"], k["y"]
        xg = x.clone().requires_grad_(True)
        grad, = torch.autograd.grad(cost(net, xg), xg)
        c, jty, _, _ = vjp(net, x, y, pd, qd)
        jv, hv = derivatives(net, x, -y, 1.0)

        def side(z, gap):
            fin = torch.isfinite(gap)
            g = torch.where(fin, gap, torch.ones_like(gap))
            zf = torch.where(fin, z, torch.zeros_like(z))
            p = torch.where(fin, zf * g - mu, torch.zeros_like(z))
            return zf / g, p / g, zf, g, p

        lx, hx = side(k["zl"], x - k["xl"]), side(k["zu"], k["xu"] - x)
        ls, hs = side(k["vl"], k["s"] - k["sl"]), side(k["vu"], k["su"] - k["s"])
        sig_s = ls[0] + hs[0]
        diag_x = dw + lx[0] + hx[0]
        C = 1.0 / (dc * sig_s + 1.0 + dc * dw)
        D = (sig_s + dw) * C
        qs = (-ls[2] + hs[2] + y) + ls[1] - hs[1]
        qy = c - k["s"]
        rhs = (grad - jty - lx[2] + hx[2]) + lx[1] - hx[1] + vjp(net, x, C * qs + D * qy, pd, qd)[1]
        dx = s["dx"]
        ds = C * (jvp(net, x, dx, pd, qd) + dc * qs - qy)
        return dict(grad=grad, c=c, diag_x=diag_x, dcon=D, rhs=rhs, jvals=jv, hvals=hv,
                    kvals=condensed(net, jv, hv, diag_x, D) if net.n <= 500_000 else None,
                    ds=ds, dy=(sig_s + dw) * ds - qs,
                    dzl=(-lx[2] * dx + lx[4]) / lx[3], dzu=(hx[2] * dx + hx[4]) / hx[3],
                    dvl=(-ls[2] * ds + ls[4]) / ls[3], dvu=(hs[2] * ds + hs[4]) / hs[3])
    xo, co, lo = 0, 0, 0
    got = []
    small = sum(k.n for k in nets) <= 500_000
    for net in nets:
        xs, cs = slice(xo, xo + net.n), slice(co, co + net.m)
        xo, co = xs.stop, cs.stop
        if kind == "adjoint":
            ls = slice(lo, lo + net.T * net.N)
            lo = ls.stop
            c, gx, gp, gq = vjp(net, s["x"][xs], s["gc"][cs], s["pd"][ls].view(net.T, -1), s["qd"][ls].view(net.T, -1))
            got.append(dict(c=c, gx=gx, gpd=gp.reshape(-1), gqd=gq.reshape(-1)))
            continue
        x, lam = s["x"][xs], s["lam"][cs]
        xg = x.clone().requires_grad_(True)
        f = cost(net, xg)
        grad, = torch.autograd.grad(f, xg)
        c, jtv, _, _ = vjp(net, x, s["v"][cs], t(net.pd), t(net.qd))
        jv, hv = derivatives(net, x, lam, 1.0)
        o = dict(f=f.detach().reshape(1), grad=grad, c=c, jvals=jv, hvals=hv, jtv=jtv)
        if small:
            o["kvals"] = condensed(net, jv, hv, s["diag_x"][xs], s["dcon"][cs])
        got.append(o)
    return {k: torch.cat([g[k] for g in got]) for k in got[0]}
