"""The gradient-pointer table after a write that failed part way, on the CPU:
the library's host code over stand-ins of the HIP calls and the launchers,
with address and undefined-behaviour sanitizers."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_30342_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_failed_table_write_leaves_no_mixed_table(tmp_path):
    exe = str(tmp_path / "grad_table_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    "-o", exe, os.path.join(HERE, "grad_table_check.cpp"),
                    os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "plan.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
