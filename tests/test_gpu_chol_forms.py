"""The forms of the Cholesky's pg chain (from both ends, by cyclic reduction)
and the rule that picks one: what cyclic reduction adds in memory is held over
the whole batch and never refuses a model that the chain from both ends takes.
Bitwise against the single instance in the form that the rule gives it, and
against the oracle (tolerances as in test_gpu_chol: backward error 1e-11, 1e-8
forward for the well conditioned family)."""
import numpy as np
import pytest

from paper_2405_14032_amd import synth

from test_gpu_chol import _check, _gpu_solve, _inputs, dev  # noqa: F401

pytestmark = pytest.mark.gpu


def _solve(nets, inps, torch, dev):  # noqa: F811
    from paper_2405_14032_amd import capi
    M = capi.Model(nets, device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    x, npert = _gpu_solve(M, F, inps, torch, dev, repeat=2)
    F.close()
    M.close()
    assert npert == 0
    return x


def _added(net):
    """Bytes beyond the chain's: G^2 per period, one level's 2G x 2G blocks."""
    return 8 * net.G ** 2 * net.T, 8 * ((net.T + 1) // 2) * 4 * net.G ** 2


@pytest.mark.parametrize("spare,expect", [(-1, "second"), (0, "first"), (1, "first"), ("all", "both")])
def test_memory_bound_holds_over_the_batch(spare, expect, dev, monkeypatch):  # noqa: F811
    """Either side of what the first instance adds, and what both do (the
    update blocks shared)."""
    import torch
    nets = [synth.make_network(40, 56, 9, 70, 3), synth.make_network(31, 45, 7, 66, 4)]
    print(f"memory bound {spare}", flush=True)
    inps = _inputs(nets, "well", 29)
    monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", "0")
    chain = [_solve([k], [i], torch, dev) for k, i in zip(nets, inps)]
    monkeypatch.delenv("OPF_CHOL_CYCLIC_BYTES")
    cyclic = [_solve([k], [i], torch, dev) for k, i in zip(nets, inps)]
    assert not any(np.array_equal(a, b) for a, b in zip(chain, cyclic))
    (f0, b0), (f1, b1) = (_added(k) for k in nets)
    monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", str(f0 + f1 + max(b0, b1) if spare == "all" else f0 + b0 + spare))
    got = _solve(nets, inps, torch, dev)
    # (below the first one's need the second, smaller one still has room)
    want = {"second": [chain[0], cyclic[1]], "first": [cyclic[0], chain[1]], "both": cyclic}[expect]
    assert np.array_equal(got, np.concatenate(want))
    _check(nets, inps, got, "well", f"memory bound {spare}")


def test_failed_allocation_takes_the_chain(dev, monkeypatch):  # noqa: F811
    import torch
    nets = [synth.make_network(40, 56, 9, 70, 3), synth.make_network(31, 45, 7, 6, 4)]
    inps = _inputs(nets, "well", 31)
    monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", "0")
    chain = _solve(nets, inps, torch, dev)
    monkeypatch.delenv("OPF_CHOL_CYCLIC_BYTES")
    assert not np.array_equal(chain, _solve(nets, inps, torch, dev))
    monkeypatch.setenv("OPF_TEST_FAIL_ALLOC", "cyclic")
    got = _solve(nets, inps, torch, dev)
    assert np.array_equal(got, chain)
    _check(nets, inps, got, "well", "failed allocation")


def _counts(net, tr, cyclic):
    """Stored factor doubles and flops of an instance by enumeration: the
    interior fronts of its tree, then the pg fronts one by one."""
    p = tr["npiv"].astype(np.int64)
    u = np.diff(tr["rowptr"]).astype(np.int64)
    G, T = net.G, net.T

    def diag(k):  # 64 x 64 diagonal blocks, the last one as it is
        return sum(min(64, k - j) ** 2 for j in range(0, k, 64))

    def work(a, b):
        return a ** 3 / 3 + a * a * b + a * b * b

    ent = int(np.sum((p + u) * p)) + sum(diag(int(k)) for k, v in zip(p, u) if k + v > 64)
    flops = float(sum(work(float(k), float(v)) for k, v in zip(p, u))) * T
    ent = (ent + (3 if cyclic else 2) * G * G + diag(G)) * T
    if not cyclic:
        return ent, flops + (T - 1) * work(G, G) + work(G, 0)
    left = list(range(T))  # every other one of the fronts left, from the first
    while left:
        gone, stay = left[::2], left[1::2]
        for _ in gone:
            flops += work(G, 2 * G if len(gone) > 1 else (G if stay else 0))
        left = stay
    return ent, flops


@pytest.mark.parametrize("T,cyclic", [(63, False), (64, True), (70, True), (70, False)])
def test_info_counts_the_form_in_use(T, cyclic, dev, monkeypatch):  # noqa: F811
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(90, 130, 70, T, 8), synth.make_network(31, 45, 7, 6, 4)]
    if T >= 64 and not cyclic:
        monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", "0")
    host, M = capi.Model(nets, device=-1), capi.Model(nets, device=0)
    H, F = capi.Chol(host), capi.Chol(M)
    want = [_counts(k, F.tree(i), cyclic and i == 0) for i, k in enumerate(nets)]
    info, plan = F.info(), H.info()
    assert info["factor_entries"] == sum(w[0] for w in want)
    assert abs(info["flops"] - sum(w[1] for w in want)) <= 1e-12 * info["flops"]
    assert info["arena_entries"] >= plan["arena_entries"]
    assert info["flops"] >= plan["flops"] and info["factor_entries"] > plan["factor_entries"]
    for o in (F, H, M, host):
        o.close()


def test_info_counts_separate_update_blocks(dev, monkeypatch):  # noqa: F811
    """With a workspace of one period per chunk the reduction's update blocks
    do not fit it: one block for both instances, counted with the workspace."""
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(40, 56, 9, 70, 3), synth.make_network(31, 45, 7, 66, 4)]
    monkeypatch.setenv("OPF_CHOL_ARENA_BYTES", "1")
    M = capi.Model(nets, device=0)
    F = capi.Chol(M)
    both = F.info()["arena_entries"]
    F.close()
    monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", "0")
    F = capi.Chol(M)
    assert both - F.info()["arena_entries"] == max(_added(k)[1] for k in nets) // 8
    F.close()
    M.close()



@pytest.mark.parametrize("G,T", [(1, 1), (5, 3), (16, 4), (17, 3), (20, 1), (33, 2), (54, 3), (64, 1), (65, 3), (70, 1),
                                 (130, 2), (257, 1), (17, 64), (70, 65), (5, 64)])
def test_infinite_pivots_anywhere_in_a_panel(G, T, dev):  # noqa: F811
    """A generator held fixed by an infinite diagonal entry gets 0 wherever its
    pivot lies in the pg front, the last of a part-filled panel included, and
    the others the solution without it (well conditioned family, 1e-8)."""
    import torch
    from oracle import opf_oracle as O
    from paper_2405_14032_amd import capi
    from test_gpu_chol import _oracle_k
    net = synth.make_network(max(14, G), int(1.4 * max(14, G)), G, T, 9)
    M = capi.Model([net], device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    inp = _inputs([net], "well", 37)[0]
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    e = lambda k: torch.empty(k, dtype=torch.float64, device=dev)
    jv, hv, kv, x = e(M.nnz_jac), e(M.nnz_hess), e(M.nnz_kkt), e(M.n)
    M.eval_jhk(t(inp["x"]), t(inp["lam"]), 1.0, t(inp["diag_x"]), t(inp["dcon"]), jv, hv, kv)
    rp, ci = torch.empty(M.n + 1, dtype=torch.int64, device=dev), torch.empty(M.nnz_kkt, dtype=torch.int32, device=dev)
    M.kkt_structure(rp, ci)
    npert = torch.zeros(1, dtype=torch.int32, device=dev)
    n, orp, oci, okv = _oracle_k(net, inp)
    K = O.kkt_full(n, orp, oci, okv).tocsc()
    import scipy.sparse.linalg as sla
    np_ = M.n // T
    for g in sorted({0, G // 2, max(0, G - 2), G - 1}):
        for tt in sorted({0, T // 2, T - 1}):
            at = tt * np_ + 2 * net.N + g
            k2 = kv.clone()
            k2[rp[at + 1] - 1] = float("inf")
            F.factor(k2, 0.0, 1.0, npert)
            F.solve(t(inp["b"]), x)
            torch.cuda.synchronize()
            got = x.cpu().numpy()
            keep = np.arange(n) != at
            ref = np.zeros(n)
            ref[keep] = sla.spsolve(K[keep][:, keep].tocsc(), inp["b"][keep])
            assert int(npert.item()) == 0 and got[at] == 0.0, (g, tt)
            assert np.max(np.abs(got - ref)) <= 1e-8 * np.max(np.abs(ref)), (g, tt)
    F.close()
    M.close()


@pytest.mark.parametrize("G,T", [(1, 1), (5, 1), (17, 1), (33, 1), (64, 1), (65, 1), (257, 1), (5, 2), (70, 2)])
def test_infinite_right_hand_side_stays_in_its_place(G, T, dev):  # noqa: F811
    """A diagonal K and an infinite entry at the variable eliminated last: it
    comes out infinite, not NaN (nothing is taken from it afterwards), no
    entry that is coupled to it finite, and the other instance of the batch is
    not touched."""
    import torch
    from paper_2405_14032_amd import capi
    net, other = synth.make_network(max(14, G), int(1.4 * max(14, G)), G, T, 9), synth.make_network(14, 20, 5, 2, 10)
    M = capi.Model([net, other], device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    rp, ci = torch.empty(M.n + 1, dtype=torch.int64, device=dev), torch.empty(M.nnz_kkt, dtype=torch.int32, device=dev)
    M.kkt_structure(rp, ci)
    kv = torch.zeros(M.nnz_kkt, dtype=torch.float64, device=dev)
    kv[rp[1:] - 1] = 4.0
    last = 2 * net.N + G - 1  # the last pg variable of the chain's middle period, (T - 1) / 2 = 0
    b, x = torch.ones(M.n, dtype=torch.float64, device=dev), torch.empty(M.n, dtype=torch.float64, device=dev)
    npert = torch.zeros(1, dtype=torch.int32, device=dev)
    F.factor(kv, 0.0, 1.0, npert)
    for v in (np.inf, -np.inf):
        b[last] = v
        F.solve(b, x)
        torch.cuda.synchronize()
        got = x.cpu().numpy()
        assert int(npert.item()) == 0 and got[last] == v
        assert not np.any(np.isfinite(got[2 * net.N:2 * net.N + G]))
        assert np.array_equal(got[net.n:], np.full(M.n - net.n, 0.25))
    F.close()
    M.close()


@pytest.mark.parametrize("G", [1, 5, 17, 33, 64, 65, 70])
def test_zero_pivot_below_a_negative_threshold(G, dev):  # noqa: F811
    """A threshold below 0 lets a zero pivot stand: not counted, its root 0 and
    the reciprocal infinite, as sqrt(0) and 1 / 0 round, so the last variable
    eliminated comes out infinite (a diagonal K); another instance of the batch
    is not touched."""
    import torch
    from paper_2405_14032_amd import capi
    net, other = synth.make_network(max(14, G), int(1.4 * max(14, G)), G, 1, 9), synth.make_network(14, 20, 5, 2, 10)
    M = capi.Model([net, other], device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    rp, ci = torch.empty(M.n + 1, dtype=torch.int64, device=dev), torch.empty(M.nnz_kkt, dtype=torch.int32, device=dev)
    M.kkt_structure(rp, ci)
    kv = torch.zeros(M.nnz_kkt, dtype=torch.float64, device=dev)
    kv[rp[1:] - 1] = 4.0
    last = 2 * net.N + G - 1  # the last pg variable
    kv[rp[last + 1] - 1] = 0.0
    b, x = torch.ones(M.n, dtype=torch.float64, device=dev), torch.empty(M.n, dtype=torch.float64, device=dev)
    b[last] = -1.0
    npert = torch.full((1,), -7, dtype=torch.int32, device=dev)
    F.factor(kv, -1.0, 1.0, npert)
    F.solve(b, x)
    torch.cuda.synchronize()
    got = x.cpu().numpy()
    assert int(npert.item()) == 0 and got[last] == -np.inf
    assert np.array_equal(got[net.n:], np.full(M.n - net.n, 0.25))
    F.factor(kv, 0.0, 2.0, npert)  # counted and replaced where the threshold is not below it
    F.solve(b, x)
    torch.cuda.synchronize()
    want = np.full(M.n, 0.25)
    want[last] = -0.5
    assert int(npert.item()) == 1 and np.max(np.abs(x.cpu().numpy() - want)) <= 1e-15
    F.close()
    M.close()


# solves of two and more 256-column launches a front, one and two 1024-column
# steps of the factorization, the last size that is reduced and the next one
@pytest.mark.parametrize("G,T,reduced", [(257, 64, True), (400, 66, True), (513, 65, True), (1030, 64, True),
                                         (1536, 64, True), (1537, 64, False)])
def test_both_forms_on_large_fronts(G, T, reduced, dev, monkeypatch):  # noqa: F811
    """The same K by cyclic reduction and by the chain: backward error in K of
    each (1e-11), so two eliminations in different orders that agree to twice
    the forward tolerance (2e-8); beyond the reduction's sizes both are the
    chain, bit for bit."""
    import scipy.sparse as sp
    import torch
    from paper_2405_14032_amd import capi
    net = synth.make_network(G, int(1.3 * G), G, T, 61)
    print(f"both forms G={G} T={T}", flush=True)
    inp = _inputs([net], "well", 41)[0]
    M = capi.Model([net], device=0)
    M.use_current_torch_stream()
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    e = lambda k: torch.empty(k, dtype=torch.float64, device=dev)
    jv, hv, kv, x, b = e(M.nnz_jac), e(M.nnz_hess), e(M.nnz_kkt), e(M.n), t(inp["b"])
    M.eval_jhk(t(inp["x"]), t(inp["lam"]), 1.0, t(inp["diag_x"]), t(inp["dcon"]), jv, hv, kv)
    rp, ci = torch.empty(M.n + 1, dtype=torch.int64, device=dev), torch.empty(M.nnz_kkt, dtype=torch.int32, device=dev)
    M.kkt_structure(rp, ci)
    npert = torch.zeros(1, dtype=torch.int32, device=dev)
    got, flops = [], []
    for budget in (None, "0"):
        if budget:
            monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", budget)
        F = capi.Chol(M)
        flops.append(F.info()["flops"])
        for _ in range(2):
            F.factor(kv, 0.0, 1.0, npert)
            F.solve(b, x)
        torch.cuda.synchronize()
        assert int(npert.item()) == 0
        got.append(x.cpu().numpy().copy())
        F.close()
    lower = sp.csr_matrix((kv.cpu().numpy(), ci.cpu().numpy(), rp.cpu().numpy()), shape=(M.n, M.n))
    M.close()
    K = (lower + sp.tril(lower, -1).T).tocsr()
    for v in got:
        assert np.max(np.abs(K @ v - inp["b"])) <= 1e-11 * (abs(K).max() * np.max(np.abs(v)) + np.max(np.abs(inp["b"])))
    assert (flops[0] > flops[1]) == reduced
    if reduced:
        assert 0.0 < np.max(np.abs(got[0] - got[1])) <= 2e-8 * np.max(np.abs(got[1]))
    else:
        assert np.array_equal(got[0], got[1])


def test_static_pivots_in_both_forms(dev, monkeypatch):  # noqa: F811
    """Whether a static pivot is taken is a property of K (indefinite or not):
    the same answer from both forms with fronts of several panels, full and
    stopped at the first."""
    import torch
    from paper_2405_14032_amd import capi
    net = synth.make_network(300, 420, 270, 65, 61)
    inps = _inputs([net], "well", 43)
    neg = inps[0]["diag_x"].copy()
    neg.reshape(net.T, -1)[40, 2 * net.N + 269] = -1e6  # one generator of one period
    M = capi.Model([net], device=0)
    M.use_current_torch_stream()
    for budget in (None, "0"):
        if budget:
            monkeypatch.setenv("OPF_CHOL_CYCLIC_BYTES", budget)
        F = capi.Chol(M)
        assert _gpu_solve(M, F, inps, torch, dev)[1] == 0
        for stop in (False, True):
            F.set_stop_on_pivot(stop)
            assert _gpu_solve(M, F, [dict(inps[0], diag_x=neg)], torch, dev)[1] >= 1
        x, n = _gpu_solve(M, F, inps, torch, dev)
        assert n == 0
        _check([net], inps, x, "backward error only", f"static pivots, budget {budget}")
        F.close()
    M.close()
