"""The bench line's traffic: the kernels that a stage launches, by name, and their
counters looked up among those of every variant that the tuner's sweep ran."""
import hashlib
import os
import re
import subprocess

import pytest

import bench
import paper_2609_35258_amd as m

STAGED = [0, 1, 2, 3, 4, 16, 128]
CACHED = ("cell", "face_rec", "face", "update")          # with 512: rows kept in the caches
FORMS = {"cell": STAGED + [64, 65, 66, 67, 68], "face_rec": [0, 1, 2, 3, 4, 32], "face_target": STAGED + [64],
         "face": [0, 1, 2, 3, 4, 64, 65, 66, 67, 68, 256, 257, 258, 259, 260, 272, 288, 304], "xface": [0, 2, 32], "update": [0, 1, 2, 3, 4],
         "update_cell": [0, 1, 2, 3, 4, 16, 17, 18, 19, 20], "criterion": [0]}

FORMS = {st: f + ([512 | x for x in f] if st in CACHED else []) for st, f in FORMS.items()}


def test_every_kernel_named_is_in_the_library():
    out = subprocess.run(["nm", "-C", m.LIB_PATH], capture_output=True, text=True, check=True).stdout
    have = {x.replace(" ", "") for x in re.findall(r"mlvs::__device_stub__(k_\w+<[^>]*>)", out)}
    for stage, forms in FORMS.items():
        for form in forms:
            for precision in (32, 64):
                names = bench.stage_kernels(stage, form, precision)
                assert names and set(names) <= have, (stage, form, precision, names)


def test_traffic_of_the_chosen_variant_among_all(tmp_path, monkeypatch):
    src = tmp_path / "paper_2609_35258_amd" / "csrc" / "kernels.hip"
    os.makedirs(src.parent)
    src.write_text("kernels")
    h = hashlib.sha256(b"kernels").hexdigest()[:16]
    os.makedirs(tmp_path / "profiles")
    rows = [("k_update<float,1,4>", 1), ("k_update<float,2,3>", 2), ("k_update<double,2,3>", 3),
            ("k_face_rec<float,3,0>", 10), ("k_face_target<float,2,4,4,4>", 20), ("k_face_target<float,2,4,4,1>", 40)]
    (tmp_path / "profiles" / "traffic.txt").write_text(
        "# comment\n" + "".join("%s jet mlvs::%s %d\n" % (h, k, v) for k, v in rows) + "0000 jet mlvs::k_x<float> 5\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic("jet", "update", 32, 1) == 2
    assert bench.measured_traffic("jet", "update", 64, 1) == 3
    assert bench.measured_traffic("jet", "update", 32, 2) is None
    assert bench.measured_traffic("jet", "face", 32, 129) == 30          # both launches of the stage
    assert bench.measured_traffic("other", "update", 32, 1) is None
    assert bench.measured_traffic("jet", "update", 32, None) is None
    src.write_text("changed")
    assert bench.measured_traffic("jet", "update", 32, 1) is None


@pytest.mark.gpu
def test_forms_reach_the_bench():
    import workloads as W
    p = W.periodic_box(6, 4, Lx=1.0, Ly=0.5, nv=36, kind="sine")
    s, _, _, _ = bench.run_gpu(p, 2, 1, 32, None)
    for st, form in bench._forms(s.tuned).items():
        assert form in FORMS[st], (st, form)
    s.close()
