"""Resource limits of the 24-field kernel with two points per thread, from the compiler's report (no GPU needed): one workgroup of 512
threads on a compute unit has 256 registers a thread and 160 KB of LDS; a spilled register would be waited for together with all
loads that are on their way."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_12792_amd", "csrc")


def test_no_spills():
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-x", "hip", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-c", "-o", os.devnull,
                        "-Rpass-analysis=kernel-resource-usage", os.path.join(CSRC, "brick.hip")], capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-2000:]
    def values(key):
        return [int(v) for v in re.findall(r"remark:\s+%s: (\d+)" % re.escape(key), r.stderr)]
    names = re.findall(r"Function Name: \S*k_brickILi(\d)ELb(\d)ELb(\d)E", r.stderr)
    # epilogue, operands and results non-temporal: the stages with operands have one instance more
    assert sorted(names) == sorted([("1", "0", "0"), ("1", "0", "1"), ("2", "0", "0"), ("2", "0", "1"), ("3", "0", "0"), ("3", "1", "0"), ("3", "1", "1"),
                                    ("4", "0", "0"), ("4", "1", "0"), ("4", "1", "1")])
    assert max(values("VGPRs")) <= 256 and not any(values("VGPRs Spill")) and not any(values("ScratchSize [bytes/lane]"))
    assert max(values("LDS Size [bytes/block]")) <= 160 * 1024
