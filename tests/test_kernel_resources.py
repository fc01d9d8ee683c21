"""Resource limits that the kernels' speed depends on, read from the compiler's own report (no GPU needed).

The right-hand-side kernels of the kinds other than the 24-field system are compiled for 64 registers and 40 KB of LDS
so that four workgroups share a compute unit; at that occupancy a kernel that spills even a few registers was measured
a quarter slower.  The two-block kernel of the 24-field system needs 128 registers (the one with two points per thread:
test_brick_resources.py).  A change that breaks one of these silently costs tens of per cent, so the build is checked here.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_12792_amd", "csrc")


@pytest.fixture(scope="module")
def usage():
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-x", "hip", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-c",
           "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]
    kernels, cur, lines = {}, None, []
    for src in ("kernels.hip", "pair.hip"):
        r = subprocess.run(cmd + [os.path.join(CSRC, src)], capture_output=True, text=True, timeout=900)
        assert r.returncode == 0, r.stderr[-2000:]
        lines += r.stderr.splitlines()
    for line in lines:
        m = re.search(r"remark:\s+(.*?)\s+\[-Rpass", line)
        if not m:
            continue
        key, _, val = m.group(1).partition(":")
        key, val = key.strip(), val.strip()
        if key == "Function Name":
            cur = kernels.setdefault(val, {})
        elif cur is not None and val.isdigit():
            cur[key] = int(val)
    assert kernels
    return kernels


def instances(usage, name):
    """template arguments -> resources of the instances of a kernel template, from the mangled names"""
    out = {}
    for mangled, res in usage.items():
        m = re.search(r"\d%sI((?:L[bi]\dE)+)E" % name, mangled)
        if m:
            out[tuple(int(g) for g in re.findall(r"L[bi](\d)E", m.group(1)))] = res
    return out


def check(res, what, vgprs, lds):
    assert res["VGPRs"] + res.get("AGPRs", 0) <= vgprs, (what, res)
    assert res["LDS Size [bytes/block]"] <= lds, (what, res)
    assert res["ScratchSize [bytes/lane]"] == 0 and res["VGPRs Spill"] == 0, (what, res)


def test_small_kinds_fit_four_workgroups_per_compute_unit_without_spilling(usage):
    plain = instances(usage, "k_rhs")                                              # kind, zipped input, epilogue
    stream = instances(usage, "k_rhs_stream")                                      # kind, epilogue
    # on zipped input: DERIVS one epilogue, the others that and three stages; on padded input one each
    padded_stream = instances(usage, "k_rhs_padded_stream")                        # kind
    assert len(plain) == 9 + 3 and len(stream) == 9 and len(padded_stream) == 3
    for key, res in list(plain.items()) + list(stream.items()) + list(padded_stream.items()):
        check(res, key, 64, 160 * 1024 // 4)


def test_two_block_kernel_fits_one_compute_unit(usage):
    """1,024 threads, so 128 registers at most, and all the LDS from one compute unit's 160 KB; one instance per epilogue"""
    ks = instances(usage, "k_pair_wide")
    assert sorted(ks) == [(1,), (2,), (3,), (4,)]
    for key, res in ks.items():
        check(res, key, 128, 160 * 1024)


def test_every_kernel_is_looked_at(usage):
    names = ["k_rhs", "k_rhs_stream", "k_rhs_padded_stream", "k_pair_wide", "k_unzip", "k_virtual", "k_virtual_centred", "k_virtual_centred_few", "k_zip"]      # and no kernel that nothing needs
    other = [n for n in usage if not any(re.search(r"\d%s[IE]" % k, n) for k in names)]
    assert not other, other


def test_fill_kernels_fit_three_workgroups_per_compute_unit(usage):
    names = [n for n in usage if "k_unzip" in n or "k_virtual" in n]
    assert len(names) == 1 + 2 * 3                              # the fills also non-temporally
    for n in names:
        assert usage[n]["LDS Size [bytes/block]"] <= 160 * 1024 // 3, n
        assert usage[n]["VGPRs Spill"] == 0, n
