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
