"""The benchmark's roofline: a launch is held against the peak of the matrix
instructions that it takes, and the stored HBM counters against every source
file that its kernels come from (CPU only)."""
import hashlib

import bench
from workload import CONFIGS


def test_peak_is_that_of_the_instructions_that_run():
    assert bench.gemm_peak(CONFIGS["next7b_b16"])[1:] == (4, 4)
    assert abs(bench.gemm_peak(CONFIGS["next7b_b16"])[0] - bench.F6_PEAK_TOPS) < 1e-6
    assert bench.gemm_peak(CONFIGS["next7b_b1_k320"])[1] == 0
    assert abs(bench.gemm_peak(CONFIGS["next7b_b1_k320"])[0] - bench.INT8_PEAK_TOPS) < 1e-6
    phases = {"gemm": [1.0], "select": [0.1]}
    res = bench.config_result(CONFIGS["next7b_b16"], 1.1, phases, 4000.0)
    assert abs(res["gemm_frac_int8_peak"] - 2 * res["gemm_frac_peak"]) < 2e-4
    assert "gemm_frac_measured_mfma_peak" not in res      # an int8 ceiling
    assert "gemm_frac_measured_mfma_peak" in bench.config_result(CONFIGS["next7b_b1_k320"], 1.1, phases, 4000.0)


def test_traffic_of_changed_sources_is_not_reported(tmp_path, monkeypatch):
    names = ("w4a4_gemm.hip", "w4a4_f6.hip", "gemm_device.h")
    csrc = tmp_path / "paper_2609_34867_amd" / "csrc"
    csrc.mkdir(parents=True)
    for n in names:
        (csrc / n).write_text(f"// {n}\n")
    sha = hashlib.sha256(b"".join((csrc / n).read_bytes() for n in names)).hexdigest()
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "hbm_traffic_w4a4_gemm_llava_next_b16.md").write_text(
        f"- hbm bytes per launch: 123\n- {' + '.join(names)} sha256: {sha}\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.traffic_from_profile() == 123
    for n in names:
        text = (csrc / n).read_text()
        (csrc / n).write_text(text + "// changed\n")
        assert bench.traffic_from_profile() is None, n
        (csrc / n).write_text(text)
