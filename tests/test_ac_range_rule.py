"""How many knot intervals a wavefront of the A/C pass takes: the host's rule, at
shapes whose times for 1, 2, 4 and 8 intervals were measured."""
import ctypes
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1112_4139_amd", "libagis.so")


@pytest.fixture(scope="module")
def rule():
    if not os.path.exists(LIB):
        pytest.skip("libagis.so not built")
    f = ctypes.CDLL(LIB).agis_ac_pass_range
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_int64, ctypes.c_void_p]

    def of(counts):
        off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        return f(off.size - 1, off.ctypes.data)
    return of


# (intervals, mean records, ranges within 2% of the fastest one)
@pytest.mark.parametrize("n,mean,near", [
    (4383, 6099, {1}), (8766, 3049, {1}), (17532, 1525, {1}), (39447, 678, {2}), (78894, 339, {2, 4}),
    (4383, 1016, {1}), (13149, 339, {1, 2}), (39447, 113, {4}), (4383, 113, {1, 2}), (17532, 28, {4}),
    (39447, 13, {4, 8}), (17532, 17, {8}), (4383, 20329, {1}), (52596, 282, {2, 4}), (473364, 141, {4, 8})])
def test_measured_shapes(rule, n, mean, near):
    counts = np.random.default_rng(n).poisson(mean, n)
    assert rule(counts) in near


def test_part_of_a_mission(rule):
    """Records in few of a mission's knot intervals: those count, not the mean."""
    counts = np.zeros(400000, np.int64)
    counts[1000:1500] = 20000
    assert rule(counts) == 1
    assert rule(np.zeros(1, np.int64)) in (1, 2, 4, 8) and rule(np.array([7])) in (1, 2, 4, 8)
