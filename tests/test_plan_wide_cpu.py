"""Index checks of the tables of mostly ragged sets and of split row items
on the CPU, with address and undefined-behaviour sanitizers."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_30342_amd", "csrc")


def test_ragged_tiles_and_split_items(tmp_path):
    exe = str(tmp_path / "plan_wide_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-o", exe,
                    os.path.join(HERE, "plan_wide_check.cpp"), os.path.join(CSRC, "plan.cpp")],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
