"""dm_set_params when the device runs out of memory or a copy fails: the
library's host code, compiled for the host alone, on a stand-in of the HIP
runtime (tests/host/set_params_failures.cpp).  CPU only."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1411_3487_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ROCM = os.path.dirname(os.path.dirname(os.path.realpath(HIPCC)))


def test_a_failed_call_leaves_nothing_to_step_with(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    from paper_1411_3487_amd.build import SOURCES
    jobs, objs = [], []
    for src in SOURCES + [os.path.join(ROOT, "tests", "host", "set_params_failures.cpp")]:
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        objs.append(obj)
        if src.endswith(".hip"):
            cmd = [HIPCC, "-O0", "-std=c++17", "--offload-host-only", "-x", "hip"]
        else:
            cmd = ["g++", "-O0", "-std=c++17", "-I", os.path.join(ROCM, "include")]
        jobs.append(subprocess.Popen([*cmd, "-c", os.path.join(CSRC, src), "-o", obj]))
    assert all(j.wait() == 0 for j in jobs)
    exe = str(tmp_path / "failures")
    # the compiler's own helpers (bfloat16 conversion) are in its runtime
    # library; the device images and calls that the program does not reach
    # stay unresolved
    builtins = subprocess.run([HIPCC, "--rtlib=compiler-rt", "-print-libgcc-file-name"],
                              capture_output=True, text=True, check=True).stdout.split()[-1]
    subprocess.run(["g++", "-no-pie", "-o", exe, *objs, builtins,
                    "-Wl,--unresolved-symbols=ignore-all"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
