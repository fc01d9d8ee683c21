"""How the 24-field kernel deals its units to workgroups, for many numbers of units (no GPU needed)."""
import os
import subprocess


def test_units_are_dealt_once_and_a_held_compute_unit_costs_little(tmp_path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    csrc = os.path.join(root, "paper_2007_12792_amd", "csrc")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp_path / "rounds_check")
    cc = subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", os.path.join(root, "include"),
                         "-I", csrc, os.path.join(root, "tests", "host_logic", "rounds_check.cpp"), "-o", exe], capture_output=True, text=True, timeout=300)
    assert cc.returncode == 0, cc.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "units dealt\n", r.stdout
