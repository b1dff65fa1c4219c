"""What the persistent kernels' waits go by, compiled for the host (csrc/dg4_wait.h)."""
import os
import subprocess

from paper_2502_01681_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def compile_and_run(tmp_path, name, *args):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", build.CSRC, os.path.join(HERE, name + ".cpp"), "-o", exe], check=True)
    return subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)


def test_a_wait_gives_up_only_when_the_sweep_stands_still(tmp_path):
    r = compile_and_run(tmp_path, "wait_check")
    assert r.returncode == 0, r.stdout
