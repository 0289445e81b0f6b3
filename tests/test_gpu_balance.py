"""What the step conserves in FP32 storage, where the targets that it evaluates
and the sums that normalise them have to be the same functions.

One diffuse-walled cell at rest in the wall's equilibrium, one step so long that
a hundred times its mass goes through the walls: the net mass flux over the
outgoing one.  Outflow and inflow hold the same products up to roundings that
differ from point to point, ten of them at most, and the one rounding of the
wall density with the Maxwellian's factor, which all points share: the bound is
2^-24 + 4 sigma, sigma = sqrt(10) 2^-24/sqrt(3) sqrt(sum (w v g)^2)/sum w |v| g
over the points that cross a wall, four walls independent of each other.

A closed cavity over 300 steps: the total mass.  A step multiplies it by the
difference of the FP32 weights 4/3 and 1/3, 1 + 2^-25; roundings of a cell's
weights and target, different in each cell, add at most 2^-24 a step.

One periodic cell that relaxes at once (Kn -> 0), where the new state's moments
are the target's: mass, velocity and energy of 60 random states, with the
correction from sums over the two axes (the base grid alone) and from sums over
all points (the same grid twice in the catalogue).  The rms error of the first
may exceed that of the second by three standard deviations of a ratio of two
rms of 60 samples, a factor 1 + 3/sqrt(60) = 1.39."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

U24 = 2.0 ** -24


def _nodes(p):
    import paper_2609_35258_amd as m
    x, w = m.gauss_hermite(p.nv, p.R, p.gh_scale_T) if p.vel_kind == "gh" else m.newton_cotes(p.nv, p.vmax)
    return np.tile(x, p.nv), np.repeat(x, p.nv), np.outer(w, w).ravel()


@pytest.mark.parametrize("levels", ["base", "twice"])
@pytest.mark.parametrize("grid", ["gh28", "nc33", "nc101"])
def test_wall_mass_balance_fp32(grid, levels):
    # "twice": the base grid twice in the catalogue, the staged wall sums
    import paper_2609_35258_amd as m
    p0 = {"gh28": lambda: W.cavity(1, nv=28), "nc33": lambda: W.cavity(1, nv=33, vel_kind="nc", vmax=5.0),
          "nc101": lambda: W.cavity(1, nv=101, vel_kind="nc", vmax=6.0)}[grid]()
    x, y, w = _nodes(p0)
    dt = 100.0
    for T in np.linspace(0.6, 1.5, 40):
        p = dataclasses.replace(p0, bcs=[W.BC(W.WALL, T=T), W.BC(W.WALL, T=T)], T0=p0.T0 * T, u0=0.0 * p0.u0)
        g = m.Solver.from_problem(p, precision=32, compat=4, dt=dt)
        if levels == "twice":
            g.set_levels(np.zeros((2, g.n_blocks), np.uint8), np.zeros(1, np.int32))
        m0 = np.sum(w * np.asarray(g.get_state()[0][0], float))
        g.step(1)
        m1 = np.sum(w * np.asarray(g.get_state()[0][0], float))
        g.close()
        f = w * np.abs(x) * np.exp(-(x * x + y * y) / (2 * p.R * T)) / (2 * np.pi * p.R * T)
        out = np.sum(f[x > 0])
        sigma = np.sqrt(10 / 3) * U24 * np.sqrt(np.sum(f[x > 0] ** 2)) / out / 2
        net = (m1 - m0) / (4 * dt * out)
        assert abs(net) < U24 + 4 * sigma, (T, net, U24 + 4 * sigma)


def test_closed_cavity_keeps_its_mass_fp32():
    import paper_2609_35258_amd as m
    p = W.perturb(W.cavity(16, nv=28), seed=3, amp=0.2)
    g = m.Solver.from_problem(p, precision=32, compat=4)
    m0 = g.totals()[0]
    for n in (100, 200, 300):
        g.step(100)
        assert abs(g.totals()[0] / m0 - 1) < n * (U24 + U24 / 2), n
    g.close()


@pytest.mark.parametrize("nv,vmax", [(24, 5.0), (33, 5.0), (64, 6.0), (101, 6.0), (101, 10.0)])
def test_axis_sums_conserve_as_the_sums_over_all_points_fp32(nv, vmax):
    import paper_2609_35258_amd as m
    rng = np.random.default_rng(17)
    p = W.periodic_box(1, 1, Ly=1.0, Kn=1e-7, nv=nv, vmax=vmax)
    x, y, w = _nodes(p)

    def moments(s):
        g, h = (np.asarray(q, float) for q in s.get_state()[0])
        rho = np.sum(w * g)
        return np.array([rho, np.sum(w * x * g) / rho, np.sum(w * y * g) / rho,
                         0.5 * np.sum(w * ((x * x + y * y) * g + h))])

    sq = np.zeros((2, 4))
    for k in range(60):
        q = dataclasses.replace(p, rho0=np.full((1, 1), rng.uniform(0.2, 2.0)),
                                u0=np.full((1, 1), rng.uniform(-0.5, 0.5)),
                                v0=np.full((1, 1), rng.uniform(-0.5, 0.5)),
                                T0=np.full((1, 1), rng.uniform(0.7, 1.6)))
        for twice in (0, 1):
            s = m.Solver.from_problem(q, precision=32, compat=4)
            if twice:
                s.set_levels(np.zeros((2, s.n_blocks), np.uint8), np.zeros(1, np.int32))
            s.step(1)
            a = moments(s)
            s.step(1)
            b = moments(s)
            s.close()
            sq[twice] += [(b[0] / a[0] - 1) ** 2, (b[1] - a[1]) ** 2, (b[2] - a[2]) ** 2, (b[3] / a[3] - 1) ** 2]
    rms = np.sqrt(sq / 60)
    print("rms axes", rms[0], "all points", rms[1], flush=True)
    assert np.all(rms[0] < (1 + 3 / np.sqrt(60)) * rms[1])
