"""The byte counts that bench.py replays from profiles/ belong to the kernels they were recorded with."""

import os
import shutil

import pytest

import bench

CSRC = os.path.join("paper_2504_02921_amd", "csrc")


@pytest.mark.parametrize("source", ["hr_gemm_mfma.hip", "hr_attn_mfma.hip", "hr_kernels_generic.hip", "hr_attn_common.h", "hr_gemm_tiles.h",
                                    "hr_layout.h", "hr_device_types.h"])
def test_a_record_of_bytes_is_dropped_when_device_code_changes(source, tmp_path, monkeypatch):
    """Each source and each header with device code of the recorded kernels counts."""
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.kernel_sources_sha()
    with open(tmp_path / CSRC / source, "a") as f:
        f.write("// another line\n")
    assert bench.kernel_sources_sha() != before
