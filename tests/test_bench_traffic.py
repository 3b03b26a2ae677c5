"""The benchmark reports a kernel's counted HBM traffic only for the sources that it was counted on.  No GPU."""
import os
import shutil

import pytest

import bench


@pytest.mark.parametrize("kernel,source", [("k_res_gemm", "gemm_residue.hip"), ("k_limb_gemm_lds", "gemm_limb.hip")])
def test_fingerprint_covers_the_shared_header(kernel, source, tmp_path, monkeypatch):
    csrc = os.path.dirname(bench.API_SOURCE)
    for f in (source, "packed.h", "api.cpp"):
        shutil.copy(os.path.join(csrc, f), tmp_path)
    monkeypatch.setattr(bench, "API_SOURCE", str(tmp_path / "api.cpp"))
    was = bench.kernel_fingerprint(kernel)
    for f in (source, "packed.h"):
        text = (tmp_path / f).read_text()
        (tmp_path / f).write_text(text + "\n// a comment\n")
        assert bench.kernel_fingerprint(kernel) == was
        (tmp_path / f).write_text(text + "\nint changed;\n")
        assert bench.kernel_fingerprint(kernel) != was
        (tmp_path / f).write_text(text)


def test_traffic_of_the_benchmarks_kernel_is_current():
    """The kernel that the benchmark's finish runs."""
    traffic, algorithmic = bench.measured_traffic("k_res_gemm")
    assert traffic and algorithmic and traffic > algorithmic
