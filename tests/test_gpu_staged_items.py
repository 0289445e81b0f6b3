"""Cell and face targets of merged levels with four items per wave (8192 items or
more, the last workgroup in part empty) against the forms that take one item per
wave (the update with the next cell stage, the persistent step): the same states
bit for bit; and with one item per wave at fewer items, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle.solver import Solver as Oracle
from tests.parity import state_error

pytestmark = pytest.mark.gpu


def _levels(p):
    # the base grid, and a level with 2 x 2 merges away from the middle
    nb = p.nv // 2
    far = np.abs(np.arange(nb) - (nb - 1) / 2)
    kappa = (np.maximum(far[:, None], far[None, :]) > nb / 4 + 0.4).astype(np.uint8)
    return np.stack([np.zeros(nb * nb, np.uint8), kappa.ravel()])


def _solver(p, kap, cl, precision, fuse, monkeypatch, **kw):
    import paper_2609_35258_amd as m
    monkeypatch.setenv("MLVS_FUSE", fuse)
    s = m.Solver.from_problem(p, precision=precision, **kw)
    s.set_levels(kap, cl)
    return s


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("ni,nj", [(131, 63), (64, 128)])
def test_many_items(ni, nj, precision, monkeypatch):
    p = W.perturb(W.periodic_box(ni, nj, Ly=0.5, nv=10, vmax=5.0, kind="sine", amp=0.3), seed=3)
    kap, cl = _levels(p), W.striped_levels(ni, nj, 2, 0)
    print("case many", ni, nj, precision, flush=True)
    staged = _solver(p, kap, cl, precision, "0", monkeypatch)
    fused = _solver(p, kap, cl, precision, "1", monkeypatch)
    pers = _solver(p, kap, cl, precision, "1", monkeypatch, graph=True)
    pers.set_persistent(True)
    for s in (staged, fused, pers):
        s.step(3)
    a = staged.get_state()
    assert all(np.isfinite(x[0]).all() and np.isfinite(x[1]).all() for x in a)
    for s in (fused, pers):
        for x, y in zip(a, s.get_state()):
            assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1])
    for s in (staged, fused, pers):
        s.close()


@pytest.mark.parametrize("precision", [64, 32])
def test_few_items(precision, monkeypatch):
    # FP64 1e-12 of the largest value; FP32 two steps of at most ten roundings
    # of 2^-24 to a stored value, 1.2e-6, taken as 2e-6
    p = W.perturb(W.periodic_box(9, 5, Ly=0.5, nv=16, vmax=5.0, kind="sine", amp=0.3), seed=3)
    kap, cl = _levels(p), W.striped_levels(9, 5, 2, 0)
    print("case few", precision, flush=True)
    s = _solver(p, kap, cl, precision, "0", monkeypatch)
    o = Oracle(p, compat=4)
    o.set_levels(list(kap), cl)
    for k in range(2):
        s.step(1)
        o.step()
        e = state_error(s.get_state(), o.g, o.h)
        assert max(e) < (1e-12 if precision == 64 else 2e-6), (k, e)
    s.close()
