"""The benchmark's counter figures of the paired dedispersion kernel: used for
the workload, tiling and source they were taken on, and for no other."""
import hashlib
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402
from sps_inputs import workloads  # noqa: E402

DEFAULT = dict(m=4, dpw=1, nw=16, cs=16, waves_per_eu=4)


def _summary(tmp_path, sha, kernel="sps::dedisperse_pairs_kernel<4>"):
    (tmp_path / "profiles").mkdir(exist_ok=True)
    src = os.path.join("paper_2511_02328_amd", "csrc")
    (tmp_path / src).mkdir(parents=True, exist_ok=True)
    (tmp_path / src / "dedisperse.hip").write_text("kernel source\n")
    (tmp_path / "profiles" / "full_scale_pairs_counters.txt").write_text(
        f"# summary\ndedisperse_pairs_source_sha256_16: {sha}\ndedisperse_kernel_name: {kernel}\n"
        "dedisperse_hbm_bytes_calibrated: 1.25e+11\n"
        "dedisperse_valu_lane_ops_per_sample_add: 0.3\n")


def test_figures_of_the_present_source_are_used(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    wl = workloads.FULL_SCALE
    sha = hashlib.sha256(b"kernel source\n").hexdigest()[:16]
    _summary(tmp_path, sha)
    assert bench.measured_counters(wl, DEFAULT) == {"traffic": 1.25e11, "ops_per_add": 0.3}
    # not for another workload, time tile or number of waves
    assert bench.measured_counters(workloads.SINGLE_BEAM, DEFAULT) is None
    assert bench.measured_counters(wl, dict(DEFAULT, m=3)) is None
    assert bench.measured_counters(wl, dict(DEFAULT, nw=8, cs=8)) is None
    # nor of another source or kernel
    _summary(tmp_path, "0" * 16)
    assert bench.measured_counters(wl, DEFAULT) is None
    _summary(tmp_path, sha, "sps::dedisperse_kernel<4, 1, 16, 16, 3, 4, false>")
    assert bench.measured_counters(wl, DEFAULT) is None
