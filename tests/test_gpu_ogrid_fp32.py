"""FP32 steps on a small O-grid, curved faces whose normals lie at any angle to
the velocities, against the oracle at every step.  The nodes of the velocity
grids are floats (multiples of 1 or 1/2), so that FP32 storage holds the same
velocities as the oracle: with nodes of 4/3 their rounding alone gives 6.3e-6 on
this mesh.  Rows of 169 and of 1089 points, in one chunk and in chunks of 64.

Tolerance: three steps with at most ten roundings of 2^-24 each to a stored
value, 1.8e-6, taken as 2e-6."""
import pytest

import workloads as W
from oracle.solver import Solver as Oracle
from tests.parity import state_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", ["64", None])
@pytest.mark.parametrize("nv,vmax", [(13, 6.0), (33, 8.0)])
def test_ogrid_fp32_on_float_velocities(nv, vmax, chunk, monkeypatch):
    import paper_2609_35258_amd as m
    if chunk:
        monkeypatch.setenv("MLVS_CHUNK", chunk)
    else:
        monkeypatch.delenv("MLVS_CHUNK", raising=False)
    p = W.perturb(W.cylinder(12, 5, nv=nv, vmax=vmax, dr1=0.2), seed=11)
    o = Oracle(p, compat=4)
    g = m.Solver.from_problem(p, precision=32, compat=4)
    for k in range(3):
        o.step()
        g.step(1)
        e = state_error(g.get_state(), o.g, o.h)
        assert max(e) < 2e-6, (k, e)
    g.close()
