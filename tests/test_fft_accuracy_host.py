"""Rounding of the transforms against double precision (host build of csrc/fft.hpp and col_fft.hpp): the
split column transforms stay as accurate as the staged ones, and the plans of 64 and 96 points as other
radices; the split of 800-point halves phase by phase."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_02624_amd", "csrc")


@pytest.fixture(scope="module")
def figures(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path_factory.mktemp("fft") / "col_accuracy"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", os.path.join(HERE, "host_fft"), "-I", CSRC,
                    os.path.join(HERE, "host_fft", "col_accuracy.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout  # slots and banks of the 800-point halves
    return {k: float(v) for k, v in (line.split() for line in run.stdout.splitlines())}


def test_split_columns_round_no_more_than_staged_ones(figures):
    # means over enough columns that their ratio is known to about half a per cent
    ratios = {k: v for k, v in figures.items() if k.startswith("split")}
    assert len(ratios) == 16
    assert all(v < 1.02 for v in ratios.values()), ratios


def test_plans_of_short_lengths(figures):
    ratios = {k: v for k, v in figures.items() if k.startswith("plan")}
    assert len(ratios) == 4
    assert all(v < 1.01 for v in ratios.values()), ratios


def test_halves_of_800_points(figures):
    # a few half-ulp roundings (6e-8) per butterfly level, eight levels in quadrature
    assert figures["forward800"] < 4e-7
