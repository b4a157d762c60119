"""How a call's launches are shaped, host core alone (no GPU)."""
import ctypes

import pytest

from tests import core_lib

K = 1 << 10


@pytest.mark.parametrize("run_bytes,lanes", [
    (16, 64), (1008, 64), (1024, 64), (1040, 128), (2 * K, 128), (2 * K + 16, 256), (4 * K, 256),
    (4 * K + 16, 512), (6 * K, 512), (8 * K, 512), (10 * K, 512), (16 * K - 16, 512),
    (16 * K, 1024), (40 * K, 1024), (64 * K, 1024), (1 << 30, 1024), (0, 64)])
def test_lanes_follow_the_mean_run(run_bytes, lanes):
    """One vector per lane below 16 KiB, 1024 lanes from there up; capped
    grids always 1024."""
    fn = core_lib.lib().aqua_core_run_threads
    fn.argtypes, fn.restype = [ctypes.c_uint64, ctypes.c_int32], ctypes.c_uint32
    assert fn(run_bytes, 0) == lanes
    assert fn(run_bytes, 1) == 1024
