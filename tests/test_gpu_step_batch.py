"""Several steps replayed as one graph: the states, step counts and adaptations
of long graph runs equal those of directly launched steps, bit for bit, where
the batches begin (after 64 single replays of a level set), where a call has
fewer steps left than a batch, and where the next adaptation is nearer."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interval,calls", [(0, (64, 8, 7, 9, 40)), (75, (72, 2, 30, 61)), (10, (35, 50))])
def test_batched_replay_matches_direct_steps(interval, calls):
    import torch
    import paper_2609_35258_amd as m
    p = W.perturb(W.periodic_box(6, 4, Lx=1.0, Ly=0.5, Kn=0.05, nv=16, vmax=5.0, kind="sine", amp=0.5), seed=5)
    ap = dict(C_split=5e-3, C_merge=2.5e-3, eps_merge=1e-3, tau_clust=0.02, flux_test=True, interval=interval)
    print("case interval", interval, "calls", calls, flush=True)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        a = m.Solver.from_problem(p, adapt=ap)
    b = m.Solver.from_problem(p, adapt=ap, graph=True)
    for n in calls:
        a.step(n)
        b.step(n)
        assert a.counters() == b.counters(), n
        for x, y in zip(a.get_state(), b.get_state()):
            assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]), n
    launches = b.graph_info()["launches"]
    assert launches < sum(calls) if interval != 10 else launches <= sum(calls)
    a.close()
    b.close()
