"""Host checks of index rules that the kernels use, compiled from the library's
own headers (tests/native)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1908_03634_amd", "csrc")


def _run(name, tmp_path):
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC,
                           os.path.join(HERE, "native", name + ".cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_nodes_beside_a_wall_have_the_other_colour(tmp_path):
    _run("nodal_axis", tmp_path)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_pair_sweep_boxes_fit_their_lds_array(tmp_path):
    _run("pair_box", tmp_path)
