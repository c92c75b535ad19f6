"""The Cholesky's blocked fronts and its pg chain at the sizes where their
kernels can go wrong: pg fronts of 1 .. 257 pivots (edges of the 16-column
blocks, the 64-column panels, the 128- and 256-column updates and the 32- and
64-row tiles), horizons around the switch from the two-ended chain to cyclic
reduction and around powers of two, static pivots in both, and a batch that
mixes them.  K from the library's own kernels, solutions against the oracle's
sparse LU of the oracle's K: backward error 1e-11 (a backward stable
elimination of fronts of a few hundred rows leaves some 1e-14, K agrees to
1e-12 per entry) and, for the well conditioned family, 1e-8 forward."""
import numpy as np
import pytest

from paper_2405_14032_amd import synth

from test_gpu_chol import _check, _gpu_solve, _inputs, dev  # noqa: F401

pytestmark = pytest.mark.gpu

# (N, B, G, T): the front's edges on the chain, then the horizon's on both forms
SHAPES = [(max(g, 14), int(1.3 * max(g, 14)), g, 3) for g in (1, 15, 16, 17, 63, 64, 65, 127, 129, 193, 257)]
SHAPES += [(20, 28, g, 64) for g in (1, 16, 17)] + [(70, 95, 65, 66), (140, 190, 130, 67)]
SHAPES += [(14, 20, 5, t) for t in (1, 2, 62, 63, 64, 65, 95, 96, 127, 128, 129)]


@pytest.mark.parametrize("family", ["well", "wide"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N%d_B%d_G%d_T%d" % s)
def test_front_and_horizon_edges(shape, family, dev):  # noqa: F811
    import torch
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(*shape, 61)]
    print(f"fronts: {shape} {family}", flush=True)
    M = capi.Model(nets, device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    inps = _inputs(nets, family, 17)
    xg, npert = _gpu_solve(M, F, inps, torch, dev, repeat=2)
    assert npert == 0
    _check(nets, inps, xg, family, str(shape))
    F.close()
    M.close()


def test_mixed_batch_and_chunks(dev, monkeypatch):  # noqa: F811
    """A batch of a chain and a cyclic instance, each bitwise equal to its own
    single-instance solve, and to itself with the periods factored one per
    chunk."""
    import torch
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(40, 56, 9, 70, 3), synth.make_network(31, 45, 7, 6, 4),
            synth.make_network(90, 130, 66, 64, 5)]
    inps = _inputs(nets, "well", 23)

    def solve(ns, ins):
        M = capi.Model(ns, device=0)
        M.use_current_torch_stream()
        F = capi.Chol(M)
        x, n = _gpu_solve(M, F, ins, torch, dev)
        assert n == 0
        F.close()
        M.close()
        return x

    whole = solve(nets, inps)
    parts = [solve([k], [i]) for k, i in zip(nets, inps)]
    assert np.array_equal(whole, np.concatenate(parts))
    monkeypatch.setenv("OPF_CHOL_ARENA_BYTES", "1")
    assert np.array_equal(whole, solve(nets, inps))


@pytest.mark.parametrize("T", [5, 70])
def test_static_pivots_and_early_stop(T, dev):  # noqa: F811
    """Negative diagonal entries are counted in both forms of the chain, with
    the early stop at least one, and the next factorization is exact."""
    import torch
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(90, 130, 70, T, 8)]
    inps = _inputs(nets, "well", 9)
    bad = [dict(inps[0], diag_x=np.where(np.arange(len(inps[0]["diag_x"])) % 7 == 0, -1e6, inps[0]["diag_x"]))]
    M = capi.Model(nets, device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    _, full = _gpu_solve(M, F, bad, torch, dev)
    xa, n0 = _gpu_solve(M, F, inps, torch, dev)
    F.set_stop_on_pivot(True)
    _, part = _gpu_solve(M, F, bad, torch, dev)
    assert full >= 1 and 1 <= part <= full
    xb, n1 = _gpu_solve(M, F, inps, torch, dev)
    assert n0 == 0 and n1 == 0 and np.array_equal(xa, xb)
    _check(nets, inps, xb, "well", "after static pivots")
    F.close()
    M.close()


def test_pivots_of_extreme_size(dev):  # noqa: F811
    """Pivots far outside the range the pivot chain takes without scaling: K
    scaled by 2^-900 and by 2^900 solves to the same bits times the inverse
    power (every step of the elimination scales exactly), and an infinite
    diagonal entry gives its variable the value 0."""
    import torch
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(90, 130, 70, 3, 8)]
    M = capi.Model(nets, device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    inps = _inputs(nets, "well", 9)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    e = lambda k: torch.empty(k, dtype=torch.float64, device=dev)
    jv, hv, kv, x = e(M.nnz_jac), e(M.nnz_hess), e(M.nnz_kkt), e(M.n)
    i = inps[0]
    M.eval_jhk(t(i["x"]), t(i["lam"]), 1.0, t(i["diag_x"]), t(i["dcon"]), jv, hv, kv)
    npert = torch.zeros(1, dtype=torch.int32, device=dev)
    b = t(i["b"])

    def solve(k):
        F.factor(k, 0.0, 1.0, npert)
        F.solve(b, x)
        torch.cuda.synchronize()
        assert int(npert.item()) == 0
        return x.cpu().numpy()

    ref = solve(kv)
    for p in (-900, 900):
        got = solve(kv * 2.0 ** p)
        assert np.array_equal(got * 2.0 ** p, ref), p
    rp, ci = torch.empty(M.n + 1, dtype=torch.int64, device=dev), torch.empty(M.nnz_kkt, dtype=torch.int32, device=dev)
    M.kkt_structure(rp, ci)
    pg = 2 * nets[0].N + 33  # a generator variable of the first period: a pivot of the blocked chain
    kv[int(rp[pg + 1]) - 1] = float("inf")
    got = solve(kv)
    assert got[pg] == 0.0 and np.all(np.isfinite(got))
    F.close()
    M.close()


# either side of the chain's forms by wavefronts (8 / 9, 16 / 17, 32 / 33,
# 48 / 49, 64 / 65 generators; horizons with none, one and more fronts on a side, and the last
# one before cyclic reduction)
@pytest.mark.parametrize("G", [1, 8, 9, 16, 17, 32, 33, 48, 49, 64, 65])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 63])
def test_chain_by_wavefronts(G, T, dev):  # noqa: F811
    """Against the oracle, and the static pivots' count the same with and
    without a second factorization in between."""
    import torch
    from paper_2405_14032_amd import capi
    nets = [synth.make_network(max(40, G), max(56, int(1.4 * G)), G, T, 71)]
    print(f"chain by wavefronts: G={G} T={T}", flush=True)
    M = capi.Model(nets, device=0)
    M.use_current_torch_stream()
    F = capi.Chol(M)
    inps = _inputs(nets, "well", 19)
    bad = [dict(inps[0], diag_x=np.where(np.arange(len(inps[0]["diag_x"])) % 3 == 0, -1e6, inps[0]["diag_x"]))]
    _, full = _gpu_solve(M, F, bad, torch, dev)
    x, npert = _gpu_solve(M, F, inps, torch, dev, repeat=2)
    _, again = _gpu_solve(M, F, bad, torch, dev)
    F.set_stop_on_pivot(True)
    _, part = _gpu_solve(M, F, bad, torch, dev)
    F.close()
    M.close()
    assert npert == 0 and full == again and full >= 1 and 1 <= part <= full
    _check(nets, inps, x, "well", f"chain by wavefronts G={G} T={T}")
