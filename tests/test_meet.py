"""The few-token kernel's meetings over flags in the workspace, stepped on the
host: tests/meet_model.cpp runs the steps of csrc/meet.hpp, which the kernel
runs too, through every order of their accesses, over launches that carry one
tag as the replays of a graph do, on flags that hold old data at first."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_19528_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("meet") / "meet_model")
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "meet_model.cpp"), "-o", exe],
                   check=True)

    def run(*args):
        p = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        assert p.returncode in (0, 1), p.stderr
        return p.returncode == 0, p.stdout

    return run


@pytest.mark.parametrize("tiles,parts", [(1, 2), (1, 3), (2, 1), (3, 1), (2, 2)])
def test_every_order_of_two_launches(model, tiles, parts):
    """Each tile finished once, from this launch's shares only, every flag down."""
    ok, out = model(tiles, parts, 2, "claim", "taken")
    assert ok, out


def test_model_finds_a_second_finisher(model):
    """Without the exchange that picks one finisher, a tile finished twice leaves
    its flag up for the replay, whose last meeting then reads an old share."""
    ok, out = model(2, 2, 2, "all", "taken")
    assert not ok and ("flag is still up" in out or "share was read" in out), out


def test_model_finds_old_data_taken_for_a_flag(model):
    """A tag that counts launches is a word that the workspace may hold."""
    ok, out = model(1, 3, 1, "claim", "counted")
    assert not ok, out


def test_tags_are_no_data(model):
    ok, first = model("tags", 100000)
    assert ok, first
    ok, other = model("tags", 100000)
    assert ok and other != first  # (each process starts elsewhere)
