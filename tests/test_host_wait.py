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


def test_groups_form_from_whichever_workgroups_run(tmp_path):
    # with places of its XCD missing for as long as the sweep lasts, or two sweeps sharing the device, every ticket is
    # finished by whole groups and every workgroup leaves
    r = compile_and_run(tmp_path, "groups_check", 10)
    assert r.returncode == 0, r.stdout
