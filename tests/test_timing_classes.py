"""What the kernel timing classes stand for in the benchmark's accounts and the
profile summaries (no GPU needed)."""
import os
import re

import bench
import workloads as W
from paper_2002_01392_amd import Solver, profsummary

CSRC = os.path.join(os.path.dirname(profsummary.__file__), "csrc")


def test_one_launch_is_counted_once():
    # where small planes ran in one launch, the four classes that report it too go
    rep = {k: (0, 0.0) for k in Solver.TIMING_CLASSES}
    for k in ("y_back_dy", "y_back_dz", "x_nl", "y_fwd", "plane_nl"):
        rep[k] = (4, 0.06)
    rep["z_pass"] = (4, 0.1)
    assert bench.timed_launches(rep) == {"plane_nl": (4, 0.06), "z_pass": (4, 0.1)}
    rep["plane_nl"] = (0, 0.0)
    assert set(bench.timed_launches(rep)) == {"y_back_dy", "y_back_dz", "x_nl", "y_fwd", "z_pass"}


def test_every_class_has_its_bytes():
    w = W.get("channel_32x32x33")
    M, _ = bench.field_bytes(w)
    for k in Solver.TIMING_CLASSES:
        assert bench.algorithmic_bytes(w, k, 1) > 0
    assert bench.algorithmic_bytes(w, "plane_nl", 1) == 3 * w.nfields * M


def test_profile_summaries_know_every_kernel_of_the_nonlinear_term():
    for fn in ("xypass.hip", "plane.hip"):
        src = open(os.path.join(CSRC, fn)).read()
        names = re.findall(r"__global__[^;{]*?void\s+(k_(?:x|y|plane)\w*)\(", src)
        assert names
        for n in names:
            assert f"fcns::{n}<" in profsummary.CLASSES, n
