"""The tuner times what launches something of its own, once, and a stored choice
is used only where its variants launch the same kernels."""
import ctypes
import json

import numpy as np
import pytest

import paper_2609_35258_amd as m
import paper_2609_35258_amd.autotune as at
import workloads as W


class Stub:
    """A solver of one stage whose variants launch `forms`; variant 3 is the fastest."""

    def __init__(self, forms):
        self.forms, self.set, self.timed = forms, [], []

    def stage_size(self, st):
        return 1000, 500000.0

    def variants(self, st):
        return len(self.forms)

    def variant_form(self, st, v):
        return self.forms[v]

    def set_variant(self, st, v):
        self.set.append(v)

    def time_stage(self, st, reps):
        v = self.set[-1] if self.set else 1
        self.timed.append(v)
        return 1.0 if v == 3 else 2.0


@pytest.fixture
def tuner(monkeypatch, tmp_path):
    monkeypatch.setattr(at, "_arch", lambda: "gfx950")
    monkeypatch.setattr(at, "_lib_tag", lambda: "0")
    path = tmp_path / "t.json"
    return lambda s: at.autotune(s, 32, stages=["cell"], cache=str(path))["cell"], path


def test_every_variant_of_its_own_is_timed_and_stored(tuner):
    tune, path = tuner
    s = Stub([0, 1, 2, 3, 4])
    assert tune(s)["variant"] == 3 and sorted(set(s.timed)) == [0, 1, 2, 3, 4]
    again = Stub([0, 1, 2, 3, 4])
    assert tune(again)["from_cache"] and again.set == [3] and not again.timed
    # another kernel family of the same size does not take that choice
    other = Stub([64, 65, 66, 67, 68])
    assert not tune(other)["from_cache"]
    assert len(json.loads(path.read_text())) == 2


def test_equal_launches_are_timed_once(tuner):
    tune, _ = tuner
    s = Stub([0, 0, 2, 0, 0])
    tune(s)
    assert sorted(set(s.timed)) == [0, 2]


def test_one_launch_is_neither_swept_nor_stored(tuner):
    tune, path = tuner
    s = Stub([16] * 5)
    r = tune(s)
    assert s.set == [] and not r["from_cache"] and r["ms"] == 2.0
    assert json.loads(path.read_text()) == {}


def test_form_rejects_bad_arguments():
    f = ctypes.c_int()
    assert m.lib().mlvs_variant_form(None, 0, 0, ctypes.byref(f)) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("mesh,compat,merged", [("box", 4, False), ("box", 4, True), ("box", 8, True),
                                                ("tri", 4, True)])
def test_forms_follow_the_dispatch(mesh, compat, merged):
    p = W.periodic_box(6, 4, Lx=1.0, Ly=0.5, nv=36, kind="sine")
    if mesh == "tri":
        p = W.as_unstructured(W.cavity(4, nv=36, vel_kind="nc", vmax=4.5), split="random", seed=3)
    s = m.Solver.from_problem(p, compat=compat)
    if merged:
        s.set_levels(np.zeros((2, s.n_blocks), np.uint8), np.zeros(s.n_cells, np.int32))
    n = {st: len({s.variant_form(st, v) for v in range(s.variants(st))}) for st in at.TUNABLE}
    assert n["update"] == 5 and n["update_cell"] == 5
    assert n["face_rec"] == (1 if mesh == "tri" else 5)
    assert n["xface"] == (1 if mesh == "tri" else 2)
    assert n["cell"] == (1 if compat == 8 else 5)
    assert n["face_target"] == (5 if merged and compat == 4 else 1)
    assert (s.variant_form("cell", 1) & 511 == 1) == (merged and compat == 4)
    s.close()
