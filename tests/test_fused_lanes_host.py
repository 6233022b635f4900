"""The fused decoder's automatic lanes per workgroup (no GPU needed): equal lanes
take the number whose workgroups are resident at once, uneven ones the number
that ends first."""
import ctypes as C
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(ROOT, "paper_2511_11337_amd", "libboa.so")),
                                reason="libboa.so not built")
DT = {"f32": 0, "bf16": 1, "fp8": 2}


def _choice(lens, D=256, dtype="bf16", layers=3, max_lanes=None):
    from paper_2511_11337_amd import _lib
    fn = _lib.load().boa_test_fused_lanes
    fn.restype = C.c_int
    fn.argtypes = [C.c_uint32, C.c_uint32, C.c_uint32, _lib.U64P, C.c_uint64, C.c_uint32, C.c_uint64]
    cl = np.ascontiguousarray(lens, dtype=np.uint64)
    return fn(D, layers, DT[dtype], cl.ctypes.data_as(_lib.U64P), cl.size, max_lanes or cl.size, 160 * 1024)


@pytest.mark.parametrize("D", [64, 128, 256, 512])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_equal_lanes(D, dtype):
    two_a_cu = D == 64 and dtype != "f32"                # one-lane workgroups of which a CU holds two
    for lanes, want in [(1, 1), (256, 1), (257, 1 if two_a_cu else 2), (512, 1 if two_a_cu else 2), (513, 4), (1024, 4),
                        (1025, 8), (2048, 8)]:
        assert _choice(np.full(lanes, 1000), D, dtype) == want, lanes


@pytest.mark.parametrize("lanes", [300, 384, 511])
def test_uneven_lanes_take_one(lanes):
    """The short lanes of a second round run behind the first one's, while the longest lane sets the end."""
    assert _choice(np.linspace(16, 1024, lanes).astype(np.uint64)) == 1
    assert _choice(np.r_[np.full(lanes - 1, 9), 5000]) == 1


def test_many_long_lanes_take_more():
    assert _choice(np.full(5000, 300)) == 8              # three rounds of 8 before two of 16
    assert _choice(np.full(4096, 300)) == 16
    assert _choice(np.full(8192, 300)) == 16
    assert _choice(np.full(8192, 300), D=512, layers=4, dtype="fp8") == 8


def test_lds_bounds_the_choice():
    from paper_2511_11337_amd import _lib
    fn = _lib.load().boa_test_fused_lanes
    cl = np.full(4096, 50, dtype=np.uint64)
    assert fn(256, 3, 1, cl.ctypes.data_as(_lib.U64P), cl.size, 4096, 65536) < 16


@pytest.mark.parametrize("D,dtype,lens,want", [
    (128, "fp8", np.full(2514, 200), 16),                # 4 lanes: 15.2 ms, 8: 14.7, 16: 13.3
    (512, "bf16", np.linspace(158, 436, 1746), 8),       # 4: 123, 8: 117
    (128, "bf16", np.linspace(69, 902, 2824), 8),        # 4: 33.9, 8: 29.0, 16: 48.7
    (64, "fp8", np.linspace(28, 96, 7237), 16)])         # 8: 7.5, 16: 7.1
def test_a_last_round_of_few_workgroups_steps_faster(D, dtype, lens, want):
    """A step's time depends on how many workgroups run beside it."""
    assert _choice(lens.astype(np.uint64), D, dtype, layers={64: 2, 128: 2, 256: 3, 512: 4}[D]) == want
