"""Arithmetic that the kernels and launchers share with the host, run on the CPU in small C++ programs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_02647_amd", "csrc")


def run(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I" + CSRC, "-o", exe, os.path.join(ROOT, "tests", "host", name + ".cpp")])
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert p.returncode == 0, p.stdout
    return p.stdout


def test_halves_of_a_listed_tile_stay_inside_it(tmp_path):
    assert "clean" in run(tmp_path, "half_tile")
