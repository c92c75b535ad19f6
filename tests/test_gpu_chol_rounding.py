"""How the Cholesky rounds one pivot and one product, bit for bit against
exact arithmetic: the square root and its reciprocal as sqrt() and the division
round them, in every kernel that takes pivots (the kernels refine a hardware
estimate instead of calling the two), and one update as one fused
multiply-add, on the vector units and the matrix cores alike.  K is made of
pivots that nothing couples, or of coupled pairs, so that each entry of the
solution depends on one pivot or one pair."""
from fractions import Fraction

import numpy as np
import pytest

from paper_2405_14032_amd import synth

from test_gpu_chol import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# chain by wavefronts (pg fronts of up to 32 rows), pg fronts of one and of
# several panels, interior fronts of both kinds
SIZES = [(60, 85, 7, 2), (60, 85, 16, 2), (90, 130, 70, 2), (1500, 2100, 300, 1)]


class Setup:
    def __init__(self, size, dev):  # noqa: F811
        import torch
        from paper_2405_14032_amd import capi
        self.torch, self.dev = torch, dev
        self.net = synth.make_network(*size, 91)
        host = capi.Model([self.net], device=-1)
        self.rp, self.ci = host.kkt_structure_host()
        host.close()
        self.M = capi.Model([self.net], device=0)
        self.M.use_current_torch_stream()
        self.F = capi.Chol(self.M)
        tr = self.F.tree(0)
        n_p, n_int = self.net.n_period, self.net.n_period - self.net.G
        # of every variable of a period: its elimination position, its front, and
        # whether the front is one of a wavefront (order <= 64)
        self.pos = np.empty(n_p, dtype=np.int64)
        self.pos[tr["perm"]] = np.arange(n_p)
        node = np.full(n_p, -1)
        node[:n_int] = np.repeat(np.arange(len(tr["first"])), tr["npiv"])
        self.first = np.append(tr["first"], n_int)[node]  # of the front that eliminates the position
        order = tr["npiv"] + np.diff(tr["rowptr"])
        small = np.append(order <= 64, False)[node]
        self.node, self.small = node, small

    def local(self, i):
        return self.pos[np.asarray(i) % self.net.n_period]

    def solve(self, kv, b):
        t = lambda a: self.torch.tensor(a, dtype=self.torch.float64, device=self.dev)
        x = self.torch.empty(self.M.n, dtype=self.torch.float64, device=self.dev)
        npert = self.torch.full((1,), -1, dtype=self.torch.int32, device=self.dev)
        self.F.factor(t(kv), 0.0, 1.0, npert)
        self.F.solve(t(b), x)
        self.torch.cuda.synchronize()
        assert int(npert.item()) == 0
        return x.cpu().numpy()

    def close(self):
        self.F.close()
        self.M.close()


def _expected(s, small):
    """1 / s / s as the solves take it: the small fronts divide twice, the
    others multiply twice by the reciprocal."""
    r = 1.0 / s
    return np.where(small, r / s, r * r)


@pytest.mark.parametrize("size", SIZES, ids=lambda s: "N%d_B%d_G%d_T%d" % s)
def test_roots_round_as_sqrt(size, dev):  # noqa: F811
    S = Setup(size, dev)
    rng = np.random.default_rng(92)
    diag = S.rp[1:] - 1
    small = S.small[S.local(np.arange(S.M.n))]
    print(f"roots {size}: {small.sum()} pivots of small fronts, {(~small).sum()} of others", flush=True)
    for top in (1, 400, 980):  # the last one beyond the range the pivot chain takes without scaling
        d = np.ldexp(rng.uniform(1.0, 4.0, S.M.n), rng.integers(-top, top, S.M.n))
        kv = np.zeros(len(S.ci))
        kv[diag] = d
        got = S.solve(kv, np.ones(S.M.n))
        assert np.array_equal(got, _expected(np.sqrt(d), small)), top
    S.close()


@pytest.mark.parametrize("size", SIZES[:2] + SIZES[3:], ids=lambda s: "N%d_B%d_G%d_T%d" % s)
def test_update_of_a_pair_is_one_fused_multiply_add(size, dev):  # noqa: F811
    """Pairs (p, q) of one front (of a blocked one: of one 64-column panel), p
    first: L = a rd(1 / rd(sqrt(d_p))), then d_q - L^2 with one rounding."""
    S = Setup(size, dev)
    rng = np.random.default_rng(93)
    n = S.M.n
    rows = np.repeat(np.arange(n), np.diff(S.rp))
    off = np.flatnonzero(S.ci != rows)
    pr, pc = S.local(rows[off]), S.local(S.ci[off])
    same = (rows[off] // S.net.n_period == S.ci[off] // S.net.n_period) & (S.node[pr] == S.node[pc])
    same &= S.small[pr] | ((pr - S.first[pr]) // 64 == (pc - S.first[pc]) // 64)
    off = off[same]
    seen = {"small": 0, "same 16 columns": 0, "other 16 columns": 0}
    for _ in range(12):
        used = np.zeros(n, dtype=bool)
        pairs = []
        for e in rng.permutation(off):
            i, j = int(rows[e]), int(S.ci[e])
            if not used[i] and not used[j]:
                used[i] = used[j] = True
                pairs.append((e, j, i) if S.local(j) < S.local(i) else (e, i, j))
        d = np.ldexp(rng.uniform(1.0, 4.0, n), rng.integers(-200, 200, n))
        kv, b, want = np.zeros(len(S.ci)), np.zeros(n), {}
        for e, p, q in pairs:
            a = float(np.ldexp(rng.uniform(-2.0, 2.0), int(rng.integers(-100, 100))))
            ell = a * (1.0 / np.sqrt(d[p]))
            d[q] = ell * ell * rng.uniform(1.1, 4.0)
            kv[e], b[q] = a, 1.0
            s = np.sqrt(float(Fraction(d[q]) - Fraction(ell) ** 2))
            lp, lq = S.local(p), S.local(q)
            want[q] = float(_expected(s, S.small[lq]))
            f = S.first[lp]
            seen["small" if S.small[lp] else "same 16 columns" if (lp - f) // 16 == (lq - f) // 16
                 else "other 16 columns"] += 1
        kv[S.rp[1:] - 1] = d
        got = S.solve(kv, b)
        bad = [q for q, w in want.items() if got[q] != w]
        assert not bad, (len(bad), len(want), bad[:5])
    print(f"pairs {size}: {seen}", flush=True)
    assert seen["small"] > 0 and (size != SIZES[3] or min(seen.values()) > 0)
    S.close()


def test_sums_run_in_ascending_order(dev):  # noqa: F811
    """Several variables p of one front and one 64-column panel coupled to one
    later q of the front: within a small front or q's own panel one chain of
    fused multiply-adds on d_q, ascending in p (also where the matrix cores
    take 16 columns at once); from an earlier panel such a chain from 0,
    subtracted once."""
    S = Setup(SIZES[3], dev)
    rng = np.random.default_rng(94)
    n = S.M.n
    rows = np.repeat(np.arange(n), np.diff(S.rp))
    off = np.flatnonzero(S.ci != rows)
    a, b = rows[off], S.ci[off].astype(np.int64)
    swap = S.local(b) > S.local(a)
    q, p = np.where(swap, b, a), np.where(swap, a, b)
    lq, lp = S.local(q), S.local(p)
    panel = lambda l: np.where(S.small[l], 0, (l - S.first[l]) // 64)
    same = S.node[lq] == S.node[lp]
    by = {}
    for e, i, j in zip(off[same], q[same], p[same]):
        by.setdefault((int(i), int(panel(S.local(j)))), []).append((int(S.local(j)), int(e), int(j)))
    stars = [(i, k, sorted(v)) for (i, k), v in by.items() if len(v) > 1]
    seen = {"small": 0, "same panel": 0, "earlier panel": 0}
    for _ in range(12):
        used = np.zeros(n, dtype=bool)
        d = np.ldexp(rng.uniform(1.0, 4.0, n), rng.integers(-30, 30, n))
        kv, b, want = np.zeros(len(S.ci)), np.zeros(n), {}
        for s in rng.permutation(len(stars)):
            i, k, ps = stars[s]
            if used[i] or any(used[j] for _, _, j in ps):
                continue
            used[i] = True
            ells = []
            for _, e, j in ps:
                used[j] = True
                kv[e] = float(np.sqrt(d[j]) * rng.uniform(-2.0, 2.0))
                ells.append(kv[e] * (1.0 / np.sqrt(d[j])))
            d[i] = sum(l * l for l in ells) * rng.uniform(1.1, 4.0)
            li = S.local(i)
            own = bool(S.small[li]) or int(panel(li)) == k
            y = float(d[i]) if own else 0.0
            for l in ells:
                y = float(Fraction(y) - Fraction(l) ** 2)
            y = y if own else float(d[i]) + y
            want[i] = float(_expected(np.sqrt(y), S.small[li]))
            b[i] = 1.0
            seen["small" if S.small[li] else "same panel" if own else "earlier panel"] += 1
        kv[S.rp[1:] - 1] = d
        got = S.solve(kv, b)
        bad = [i for i, w in want.items() if got[i] != w]
        assert not bad, (len(bad), len(want), bad[:5])
    print(f"stars: {seen}", flush=True)
    assert min(seen.values()) > 0
    S.close()
