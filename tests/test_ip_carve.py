"""LDS of the inner-product scan (no GPU): the kernel's addresses and the launcher's request come from
one description, walked here over every shape."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_inner_product_scan_regions_fit_their_allocation(tmp_path):
    exe = str(tmp_path / "ip_carve")
    cmd = ["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2312_01712_amd", "csrc"),
           os.path.join(ROOT, "tests", "sanitize", "ip_carve_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "clean" in r.stdout, r.stdout
