"""Memory that waits between contexts (csrc/dynlp_kept.h, compiled for the host with a runtime and a clock of its own): which block a
request gets, the bounds in bytes and blocks, how long a block waits, what happens when the runtime has no memory left, threads."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_06596_amd", "csrc")


def test_the_list_of_kept_memory(tmp_path):
    exe = str(tmp_path / "kept")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "kept_memory_test.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), r.stdout + r.stderr
