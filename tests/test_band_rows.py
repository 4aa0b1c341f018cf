"""Rows of the padded input that a band of the backward-weights reduction touches
(csrc/band_rows.h, host arithmetic of every call's plan): the few bands it looks
at give the maximum that a scan of all bands gives, over output sizes with and
without factors of two, images of less than a band, strides, paddings and segment
lengths, and cost little where the scan was long."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_band_rows_max_against_scan(tmp_path):
    exe = str(tmp_path / "band_rows_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_1802_00930_amd", "csrc"),
                           os.path.join(ROOT, "tests", "helpers", "band_rows_check.cpp"), "-o", exe])
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout
