"""The counted GEMM traffic is reported only while every GEMM source is the one
it was counted on: kernels, epilogues, tile shapes and their choice.
"""
import glob
import os
import shutil

import pytest

import bench
from paper_2509_16248_amd.prof_summary import CSRC, gemm_sources_sha256

NAMES = sorted(os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "gm_gemm*")))


@pytest.mark.parametrize("name", NAMES)
def test_every_source_counts(name, tmp_path):
    for n in NAMES:
        shutil.copy(os.path.join(CSRC, n), tmp_path / n)
    assert gemm_sources_sha256(tmp_path) == gemm_sources_sha256()
    with open(tmp_path / name, "a") as fh:
        fh.write("\n")
    assert gemm_sources_sha256(tmp_path) != gemm_sources_sha256()


def test_record_of_other_sources_is_not_reported(monkeypatch):
    monkeypatch.setattr("paper_2509_16248_amd.prof_summary.gemm_sources_sha256", lambda: "other")
    assert bench.measured_traffic("decoder_4096") is None
