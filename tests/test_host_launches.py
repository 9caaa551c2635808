"""The attention launchers' host code on stand-ins for the HIP runtime (no GPU): a
failed launch ends its call, and no launch reaches 2^32 threads (tests/native/
launch_check.cpp)."""
import os
import subprocess

import pytest

from paper_2608_02504_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_launch_errors_and_sizes(tmp_path):
    try:
        hipcc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    flags = [f for f in B.COMMON if f not in ("-O3", "-Wall")] + ["-O1", "-w"]
    objs = []
    for src in ("attn_bf16.hip", "attn_f32.hip"):
        objs.append(str(tmp_path / (src + ".o")))
        cmd = [hipcc, *flags, "--cuda-host-only", "-c", os.path.join(B.CSRC, src), "-o", objs[-1]]
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-4000:]
    exe = str(tmp_path / "launch_check")
    # (the device code is not linked: only its registration, a stand-in here, names it)
    cmd = ["g++", "-std=c++17", "-O1", "-w", "-no-pie", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           f"-I{B.INCLUDE}", f"-I{B.CSRC}", os.path.join(HERE, "native", "launch_check.cpp"), *objs, "-o", exe,
           "-Wl,--unresolved-symbols=ignore-all"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-2000:]
    assert "launches: ok" in run.stdout
