"""Plan creation's rules over a layout (csrc/ef_layout.h), on the host alone: tests/layout_rules_driver.cpp."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1905_10936_amd", "csrc")


def test_layout_rules(tmp_path):
    exe = str(tmp_path / "layout_rules")
    built = subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                            os.path.join(HERE, "layout_rules_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
