"""What a session holds on the device (maze_device_bytes), without a device:
resident solves keep their exchange in memory that the session has anyway, but for a part on the
smallest grids."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2505_20418_amd", "libmaze.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libmaze.so not built")


def device_bytes(N, precision, flags):
    from paper_2505_20418_amd import maze
    cfg = maze.maze_config(216, 2, 0.4 * N, 0.4, 1e-9, 100, precision, 0, flags, 1.0, None)
    n = maze.lib().maze_device_bytes(ctypes.byref(cfg))
    assert n > 0
    return n


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("flags", [0, 16, 1])
def test_resident_solves_take_no_memory_of_their_own(monkeypatch, precision, flags):
    for N in (45, 48, 64, 72, 76, 80, 96, 100, 112, 120, 128, 129, 160, 256):
        if flags == 1 and N in (45, 76, 100, 120, 129):
            continue  # no multigrid hierarchy
        monkeypatch.delenv("MAZE_PERSIST", raising=False)
        a = device_bytes(N, precision, flags)
        monkeypatch.setenv("MAZE_PERSIST", "0")
        assert a == device_bytes(N, precision, flags), N


@pytest.mark.parametrize("precision", [0, 1])
def test_small_grids_take_less_than_half_a_megabyte(monkeypatch, precision):
    for N in range(4, 45):
        monkeypatch.delenv("MAZE_PERSIST", raising=False)
        a = device_bytes(N, precision, 0)
        monkeypatch.setenv("MAZE_PERSIST", "0")
        assert 0 <= a - device_bytes(N, precision, 0) <= 1 << 19, N
