"""Host-side check of bench.py: a committed traffic figure is reported only while the headers that
hold the kernel's main loop, staging and epilogue are those it was measured on, too."""
import hashlib
import json
import os
import re
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNELS = ["gemm_f32_simt", "gemm_bf16_tn", "gemm_bf16x3_tn", "gemm_bf16_direct", "gemm_bf16x3_direct", "gemm_fp8r_tn",
           "gemm_fp8r_tiles", "gemm_fp6x3_tn", "gemm_fp6x3_tiles"]


@pytest.mark.parametrize("name", KERNELS)
def test_a_changed_header_drops_the_figure(name, tmp_path, monkeypatch):
    import bench
    csrc = "paper_2311_03543_amd/csrc"
    shutil.copytree(os.path.join(ROOT, csrc), tmp_path / csrc)
    sha = lambda rel: hashlib.sha256((tmp_path / rel).read_bytes()).hexdigest()
    src = bench.KERNEL_SOURCES[name]
    # the kernel headers that the source includes (kernels.h holds launch interfaces and host rules)
    used = {f"{csrc}/{h}" for h in re.findall(r'#include "(\w+\.h)"', (tmp_path / src).read_text())} - {f"{csrc}/kernels.h"}
    rec = {"hbm_bytes_per_launch": 7.0, "source_sha256": sha(src), "headers_sha256": {h: sha(h) for h in used}}
    os.makedirs(tmp_path / "profiles")
    (tmp_path / "profiles" / "hbm_traffic_n64.json").write_text(json.dumps({"kernels": {name: rec}}))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic(name, 64) == 7.0
    for h in used:
        text = (tmp_path / h).read_text()
        (tmp_path / h).write_text(text + "// changed\n")
        assert bench.measured_traffic(name, 64) is None, h
        (tmp_path / h).write_text(text)
    assert bench.measured_traffic(name, 64) == 7.0
    del rec["headers_sha256"]                              # a record that does not tell its headers
    (tmp_path / "profiles" / "hbm_traffic_n64.json").write_text(json.dumps({"kernels": {name: rec}}))
    assert bench.measured_traffic(name, 64) is None


def test_fp32_kernel_is_bound_by_the_matrix_instructions():
    import bench
    bound, work, peak, unit = bench.kernel_roofline("gemm_f32_simt", 64, 64, 64)
    assert (bound, work, peak, unit) == ("mfma", 2 * 64 ** 3, 157.3, "TFLOP/s")
