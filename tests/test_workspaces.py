"""The kept workspaces (csrc/workspace.cpp) on the CPU, against a recording
stand-in for the HIP calls: what a graph captured stays allocated, a capture
keeps nothing, a reservation that fails leaves everything as it was."""
import ctypes
import os
import subprocess

import pytest

from paper_2101_09808_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
MIB = 1 << 20


@pytest.fixture()
def ws(tmp_path):
    """A fresh instance of the library's workspaces (its own copy per test)."""
    lib = str(tmp_path / "workspaces.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", *build.HOST_FLAGS, "-I", build.INCLUDE, "-I",
                    build.CSRC, os.path.join(HERE, "workspace_harness.cpp"),
                    os.path.join(build.CSRC, "workspace.cpp"), "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    for f, args, res in (("t_call", [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64], ctypes.c_uint64),
                         ("t_reserve", [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64], None),
                         ("t_release", [ctypes.c_uint64], ctypes.c_int), ("t_room", [ctypes.c_uint64], None),
                         ("t_live", [ctypes.c_uint64], ctypes.c_int), ("t_used", [], ctypes.c_uint64)):
        getattr(L, f).argtypes = args
        getattr(L, f).restype = res
    return L


@pytest.mark.parametrize("grow", ["t_call", "t_reserve"])
def test_a_captured_buffer_outlives_growth(ws, grow):
    a = ws.t_call(0, 3 * MIB, 7)
    ws.t_capturing(1)
    assert ws.t_call(0, 3 * MIB, 7) == a and ws.t_graph_allocs() == 0
    ws.t_capturing(0)
    for k in range(4, 40):  # larger and larger calls: the graph's buffer stays
        getattr(ws, grow)(0, k * MIB, 7)
        assert ws.t_live(a)
    b = ws.t_call(0, 39 * MIB, 7)
    assert b != a and ws.t_used() <= 3 * MIB + 40 * MIB
    assert ws.t_release(7) == 0 and ws.t_used() == 0 and ws.t_bad_frees() == 0


def test_retained_buffers_are_bounded_by_the_kept_one(ws):
    held = []
    for k in range(1, 60):  # a capture after every growth
        held.append(ws.t_call(0, k * MIB, 7))
        ws.t_capturing(1)
        assert ws.t_call(0, k * MIB, 7) == held[-1]
        ws.t_capturing(0)
    assert all(ws.t_live(p) for p in held)
    assert ws.t_used() <= 4 * 59 * MIB  # kept: at most twice what was asked; retained: less than that
    ws.t_release(7)
    assert ws.t_used() == 0 and ws.t_bad_frees() == 0


def test_a_capture_without_a_kept_buffer_keeps_nothing(ws):
    ws.t_call(0, MIB, 7)
    ws.t_capturing(1)
    a = ws.t_call(0, 5 * MIB, 7)
    assert a and ws.t_graph_allocs() == 1 and ws.t_graph_frees() == 1  # inside the graph
    ws.t_capturing(0)
    assert ws.t_call(0, 5 * MIB, 7) != a
    assert ws.t_release(7) == 0 and ws.t_bad_frees() == 0


def test_a_reservation_without_room_changes_nothing(ws):
    a = ws.t_call(0, 2 * MIB, 7)
    ws.t_room(4 * MIB)
    ws.t_reserve(0, 3 * MIB, 7)
    assert ws.t_last_error() == 0  # a launch after it reports its own errors only
    assert ws.t_live(a) and ws.t_call(0, 2 * MIB, 7) == a
    b = ws.t_call(0, 3 * MIB, 7)  # a call that needs it gives the old buffer back first
    assert b and not ws.t_live(a) and ws.t_last_error() == 0
    assert ws.t_call(0, 9 * MIB, 7) == 0
