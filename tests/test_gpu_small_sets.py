"""Which form the correction of a small level set takes, on both sides of each
line of the rule, against the oracle: axis sums or sums over all points on the
base grid (1-D: FP64 from 3500 cells on; 2-D: 512 cells or more than 512 points),
face targets by a wave each in the fused step, with four and eight moments, over
levels that merge nothing and a catalogue of two.

Tolerances: FP64 1e-12 of the largest value, as for every step of this solver;
FP32, two steps with at most ten roundings of 2^-24 each to a stored value,
1.2e-6, taken as 2e-6."""
import numpy as np
import pytest

import workloads as W
from oracle.solver import Solver as Oracle
from tests.parity import state_error

pytestmark = pytest.mark.gpu

AXES, WAVE = 64, 256
CASES = {
    "sod_3499": (lambda: W.sod_1d(3499, Kn=0.1, nv=17, vmax=6.0), WAVE, WAVE),
    "sod_3500": (lambda: W.sod_1d(3500, Kn=0.1, nv=17, vmax=6.0), AXES, WAVE),
    "sod_5": (lambda: W.sod_1d(9, Kn=0.1, nv=5, vmax=4.0), WAVE, WAVE),
    "cavity_22": (lambda: W.cavity(22, nv=8), WAVE, WAVE),
    "cavity_23": (lambda: W.cavity(23, nv=8), AXES, AXES),
    "points_484": (lambda: W.cavity(3, nv=22), WAVE, WAVE),
    "points_576": (lambda: W.cavity(3, nv=24), AXES, AXES),
}


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("case", sorted(CASES))
def test_base_grid_on_both_sides_of_the_rule(case, precision):
    import paper_2609_35258_amd as m
    make, f64, f32 = CASES[case]
    p = W.perturb(make(), seed=23, amp=0.1)
    print("case", case, precision, flush=True)
    o = Oracle(p, compat=4)
    g = m.Solver.from_problem(p, precision=precision, compat=4)
    assert "face" in g.step_stages()
    assert g.variant_form("face", 1) & (AXES | WAVE) == (f64 if precision == 64 else f32)
    for k in range(2):
        o.step()
        g.step(1)
        e = state_error(g.get_state(), o.g, o.h)
        assert max(e) < (1e-12 if precision == 64 else 2e-6), (k, e)
    g.close()


@pytest.mark.parametrize("make", [lambda: W.cavity(2, nv=41, vel_kind="nc", vmax=5.0),
                                  lambda: W.sod_1d(600, Kn=0.1, nv=1201, vmax=6.0)], ids=["cells_4", "sod_600"])
def test_chosen_chunks_fp64(make):
    # rows longer than the fused step's: chunks of 256 points and a remainder for
    # four cells, one chunk of the whole row for 600
    import paper_2609_35258_amd as m
    p = W.perturb(make(), seed=7)
    o = Oracle(p, compat=4)
    g = m.Solver.from_problem(p, compat=4)
    assert "face_rec" in g.step_stages()
    for k in range(2):
        o.step()
        g.step(1)
        e = state_error(g.get_state(), o.g, o.h)
        assert max(e) < 1e-12, (k, e)
    g.close()


@pytest.mark.parametrize("compat", [0, 4, 8])
@pytest.mark.parametrize("mesh", ["cavity", "triangles"])
def test_wave_targets_over_two_levels_fp64(mesh, compat):
    import paper_2609_35258_amd as m
    p = W.perturb(W.cavity(5, nv=12, vel_kind="nc", vmax=4.5), seed=8)
    if mesh == "triangles":
        p = W.as_unstructured(p, split="random", seed=6)
    nb = p.nv // 2
    # 2 x 2 merges away from the middle
    far = np.abs(np.arange(nb) - (nb - 1) / 2) > 1.6
    kap = np.stack([np.zeros(nb * nb, np.uint8), (far[:, None] | far[None, :]).astype(np.uint8).ravel()])
    cl = (np.arange(p.n_cells) // 3 % 2).astype(np.int32)
    o = Oracle(p, compat=compat)
    g = m.Solver.from_problem(p, compat=compat)
    o.set_levels(list(kap), cl)
    g.set_levels(kap, cl)
    assert g.variant_form("face", 1) & WAVE
    for k in range(2):
        o.step()
        g.step(1)
        e = state_error(g.get_state(), o.g, o.h)
        assert max(e) < 1e-12, (k, e)
    g.close()


@pytest.mark.parametrize("case", ["sod", "cavity", "two_levels"])
def test_persistent_step_of_a_small_mesh(case):
    # one workgroup per four faces, in eights, where fewer than fit the device;
    # no neighbour rows and no barrier behind them except over two levels
    import paper_2609_35258_amd as m
    p = W.sod_1d(37, Kn=0.1, nv=33, vmax=6.0) if case == "sod" else W.cavity(6, nv=12, vel_kind="nc", vmax=4.5)
    p = W.perturb(p, seed=4)
    a, b = (m.Solver.from_problem(p, graph=True) for _ in range(2))
    if case == "two_levels":
        nb = p.nv // 2
        far = np.abs(np.arange(nb) - (nb - 1) / 2) > 1.6
        kap = np.stack([np.zeros(nb * nb, np.uint8), (far[:, None] | far[None, :]).astype(np.uint8).ravel()])
        for s in (a, b):
            s.set_levels(kap, (np.arange(p.n_cells) // 3 % 2).astype(np.int32))
    b.set_persistent(True)
    for k in range(4):
        a.step(1)
        b.step(1)
        for x, y in zip(a.get_state(), b.get_state()):
            assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]), k
    info = b.graph_info()
    faces = 38 if case == "sod" else 84
    assert info["error"] == 0 and info["grid"] == 8 * -(-faces // 32)
    a.close()
    b.close()
