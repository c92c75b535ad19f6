"""Calls whose path depends on sizes or on earlier calls: the whole sweep's
default tiles at the edges of the rule that picks them (against the oracle),
the load profile of several instances, and the interior-point loop's kept work
vectors (both bit for bit against a fresh object)."""
import dataclasses

import numpy as np
import pytest

from paper_2405_14032_amd import synth

import gpu_common as GC

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available()
    return torch.device("cuda:0")


# 128 / 129 lines and 256 / 257 buses: blocks of 256 or of one wavefront; 190
# lines and 30 generators are 4 wavefronts a period: at 256 periods 1024 (one
# period per tile), above two periods, from 385 (1540) on blocks of 256
@pytest.mark.parametrize("N,B,G,T", [(100, 128, 20, 3), (100, 129, 20, 3), (256, 300, 40, 2), (257, 300, 40, 2),
                                     (120, 190, 30, 256), (120, 190, 30, 257), (120, 190, 30, 384),
                                     (120, 190, 30, 385)])
def test_sweep_default_tiles(N, B, G, T, dev):
    import torch
    from paper_2405_14032_amd import capi
    print(f"sweep case {(N, B, G, T)}", flush=True)
    net = synth.make_network(N, B, G, T, 77)
    pt = synth.make_point(net, 77, stress=True)
    M = capi.Model([net], device=0)
    out = GC.gpu_all(M, pt.x, pt.lam, pt.sigma, pt.lam, pt.diag_x, pt.dcon, torch, dev, graph=True)
    M.close()
    GC.compare(out, GC.oracle_all(net, pt), f"sweep {(N, B, G, T)}")


@pytest.mark.parametrize("sizes", [[(14, 20, 5, 4)], [(1, 0, 1, 1), (64, 90, 13, 13), (300, 420, 60, 7)]])
def test_set_load_equals_a_fresh_model(sizes, dev):
    import torch
    from paper_2405_14032_amd import capi
    import pins
    print(f"set_load case {sizes}", flush=True)
    nets = [synth.make_network(*s, 80 + i) if s[1] else
            pins.manual_network(1, [], [], [], [], [], [0], T=s[3], pd=np.full((s[3], 1), 0.4))
            for i, s in enumerate(sizes)]
    rng = np.random.default_rng(5)
    new = [dataclasses.replace(n, pd=rng.normal(size=n.pd.shape), qd=rng.normal(size=n.qd.shape)) for n in nets]
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev)

    def cons(M):
        M.use_current_torch_stream()
        x = t(np.random.default_rng(6).normal(size=M.n))
        c = torch.full((M.m,), float("nan"), dtype=torch.float64, device=dev)
        M.eval_cons(x, c)
        torch.cuda.synchronize()
        return c.cpu().numpy()

    M, R = capi.Model(nets, device=0), capi.Model(new, device=0)
    M.use_current_torch_stream()
    M.set_load(t(np.concatenate([n.pd.ravel() for n in new])), t(np.concatenate([n.qd.ravel() for n in new])))
    a, b = cons(M), cons(R)
    M.close()
    R.close()
    assert np.array_equal(a, b)


@pytest.mark.parametrize("first,second", [(0, 1), (1, 0)])
def test_ipm_solves_share_a_factor_object(first, second, dev):
    import torch
    from paper_2405_14032_amd import capi
    print(f"ipm case line_search {first} then {second}", flush=True)
    net = synth.config_network("tiny")

    def solve(M, F, ls):
        x = torch.full((M.n,), float("nan"), dtype=torch.float64, device=dev)
        y = torch.full((M.m,), float("nan"), dtype=torch.float64, device=dev)
        r = capi.ipm_solve(M, F, x, y, line_search=ls, max_iter=8)
        torch.cuda.synchronize()
        return r["iterations"], x.cpu().numpy(), y.cpu().numpy()

    M = capi.Model([net], device=0)
    M.use_current_torch_stream()
    F, F2 = capi.Chol(M), capi.Chol(M)
    solve(M, F, first)
    again, fresh = solve(M, F, second), solve(M, F2, second)
    F.close()
    F2.close()
    M.close()
    assert again[0] == fresh[0]
    assert np.array_equal(again[1], fresh[1]) and np.array_equal(again[2], fresh[2])
