"""Tiles that several workgroups finish together: whatever order their events come in, and whichever of them give up waiting, every
slice is finished once, from parts that are all there, and the count is back at zero.  The kernel's own count
(lords_meet.h), compiled for the host."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("meet") / "meet_count.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "meet_count.cpp")], check=True)
    return ctypes.CDLL(out)


@pytest.fixture(scope="module")
def orders(library):
    return library.meet_orders


@pytest.mark.parametrize("log", [1, 2])
@pytest.mark.parametrize("may_give_up", [0, 1])
def test_every_order_of_two_and_four(orders, log, may_give_up):
    assert orders(log, may_give_up, 0) == 0


@pytest.mark.parametrize("may_give_up", [0, 1])
def test_drawn_orders_of_eight(orders, may_give_up):
    assert orders(3, may_give_up, 200000) == 0


@pytest.mark.parametrize("log", [0, 1, 2, 3])
def test_every_part_has_one_workgroup(library, log):
    assert [(xcd, tiles) for xcd in range(8) for tiles in range(1, 300) if library.meet_places_wrong(xcd, tiles, log)] == []
