"""Geometry of the tile lists, by brute force on the host.

csrc/list_geometry.h holds the rules that say which tiles a node is listed for
when a tile's block has moved it: its class (near or far) for each of the eight
neighbours, whether it may reach a tile beyond them, and which tiles around a
tile whose list overflowed hold every node that it needs.  list_geometry.cpp
compiles them for the host and compares them with the cells that the kernels
read, for every axis length of up to six tiles of 16 (111 cells) or 32 (191),
every filter radius 1..8, with and without two-layer markers, one-kernel step
and separate kernels: no class is weaker than needed, no reached tile is missed,
no tile gets a node twice.
"""
import os
import subprocess

import pytest

from paper_2607_02954_amd import build as mc_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("geometry") / "list_geometry")
    res = subprocess.run(
        [mc_build.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", mc_build.CSRC, "-I", mc_build.INCLUDE,
         "-o", exe, os.path.join(HERE, "list_geometry.cpp")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


@pytest.mark.parametrize("side", [16, 32])
def test_lists_hold_what_the_kernels_read(program, side):
    res = subprocess.run([program, str(side)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert res.stdout.endswith(" checks\n") and int(res.stdout.split()[0]) > 1e6, res.stdout
