"""The four-moment correction as sums over the two axes of the tensor base grid
(level sets of the base grid alone) against the oracle's sums over all points
and against the general path, which the same grid takes where a second level
stands beside it: axes shorter than, equal to and longer than the sixteen lanes
of a group with remainders, one and two dimensions, Gauss-Hermite and uniform
nodes, corrections at the faces on and off, states far from the grid's middle.

Tolerances: FP64 1e-12 of the largest value, as for every step of this solver;
FP32, two steps with at most ten roundings of 2^-24 each to a stored value,
1.2e-6, taken as 2e-6."""
import numpy as np
import pytest

import workloads as W
from oracle.solver import Solver as Oracle
from tests.parity import state_error

pytestmark = pytest.mark.gpu

CASES = {
    "sod_5": (lambda: W.sod_1d(9, Kn=0.1, nv=5, vmax=4.0), 0.1),
    "sod_17": (lambda: W.sod_1d(11, Kn=0.1, nv=17, vmax=6.0), 0.3),
    "sod_101": (lambda: W.sod_1d(6, Kn=0.01, nv=101), 0.3),
    "gh_8": (lambda: W.cavity(4, nv=8), 0.1),
    "gh_28": (lambda: W.cavity(5, nv=28), 0.3),
    "nc_16": (lambda: W.periodic_box(5, 3, nv=16, vmax=5.0, kind="sine", amp=0.5), 0.3),
    "nc_33": (lambda: W.periodic_box(3, 3, nv=33, vmax=5.0, kind="sine"), 0.3),
}


def _shifted(case):
    make, amp = CASES[case]
    p = W.perturb(make(), seed=23, amp=amp)
    p.u0 = p.u0 + 0.5
    return p


@pytest.mark.parametrize("face_compat", [True, False])
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("case", sorted(CASES))
def test_axis_sums_match_the_oracle(case, precision, face_compat):
    import paper_2609_35258_amd as m
    p = _shifted(case)
    print("case", case, precision, face_compat, flush=True)
    o = Oracle(p, compat=4, face_compat=face_compat)
    g = m.Solver.from_problem(p, precision=precision, compat=4, face_compat=face_compat)
    for k in range(2):
        o.step()
        g.step(1)
        e = state_error(g.get_state(), o.g, o.h)
        assert max(e) < (1e-12 if precision == 64 else 2e-6), (k, e)
    g.close()


@pytest.mark.parametrize("chunk", ["64", None])
@pytest.mark.parametrize("case", ["sod_5", "sod_101", "gh_8", "nc_16"])
def test_correction_off(case, chunk, monkeypatch):
    # five nodes hold the Maxwellian's moments so badly that a correction shows
    import paper_2609_35258_amd as m
    if chunk:
        monkeypatch.setenv("MLVS_CHUNK", chunk)
    else:
        monkeypatch.delenv("MLVS_CHUNK", raising=False)
    p = _shifted(case)
    print("case off", case, chunk, flush=True)
    o = Oracle(p, compat=0)
    g = m.Solver.from_problem(p, precision=64, compat=0)
    for k in range(2):
        o.step()
        g.step(1)
        e = state_error(g.get_state(), o.g, o.h)
        assert max(e) < 1e-12, (k, e)
    g.close()


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("case", ["gh_8", "gh_28", "nc_16"])
def test_axis_sums_match_the_general_path(case, precision):
    # the base grid twice in the catalogue, all cells on the first copy
    import paper_2609_35258_amd as m
    p = _shifted(case)
    print("case", case, precision, flush=True)
    a = m.Solver.from_problem(p, precision=precision, compat=4)
    b = m.Solver.from_problem(p, precision=precision, compat=4)
    n = b.n_cells
    st = b.get_state()
    b.set_levels(np.zeros((2, b.n_blocks), np.uint8), np.zeros(n, np.int32))
    for (g, h), (g2, h2) in zip(st, b.get_state()):
        assert np.array_equal(g, g2) and np.array_equal(h, h2)
    a.step(2)
    b.step(2)
    e = state_error(b.get_state(), *zip(*a.get_state()))
    assert max(e) < (1e-12 if precision == 64 else 2e-6), e
    a.close()
    b.close()
