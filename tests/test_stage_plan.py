"""Which kernel a grid's LIM stages run on (host query of the library): 3D grids
of few y rows take their stages one per launch where the columns of the blocked
launches would hold mostly rows that are no cells, all others in blocks."""
import ctypes

import pytest

from paper_2106_00282_amd import tlim

GENERAL, LINE, TILES, MARCH, BLOCKED_MARCH = range(5)


class Plan(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int32) for k in ("kernel", "stages", "tile_x", "tile_y")]


def stage_plan(n, precision="fp64", face=0, count=23, coeffs=False, bc=None):
    lib, g, p = tlim.load_library(), tlim.make_grid(n, bc=bc), Plan()
    assert lib.tlim_stage_plan(ctypes.byref(g), tlim.FP32 if precision == "fp32" else tlim.FP64, face, count,
                               int(coeffs), ctypes.byref(p)) == 0
    return p


@pytest.mark.parametrize("face", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(1000, 1, 1000), (64, 1, 20000), (700, 2, 700), (2000, 1, 2000), (1, 1, 60000)])
def test_few_rows_take_one_stage_per_launch(n, precision, face):
    p = stage_plan(n, precision, face)
    assert (p.kernel, p.stages) == (MARCH, 1)
    assert stage_plan(n, precision, face, count=2).kernel == MARCH  # every launch of a pass


@pytest.mark.parametrize("face", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(128, 128, 128), (150, 131, 97), (512, 512, 512), (20, 20, 20), (256, 1, 256), (1, 5, 200),
                               (256, 8, 256), (1, 256, 256), (200, 200, 30)])
def test_other_grids_take_blocks(n, precision, face):
    p = stage_plan(n, precision, face)
    assert (p.kernel, p.stages) == (BLOCKED_MARCH, 4 if precision == "fp32" else 3)
    assert stage_plan(n, precision, face, count=2).stages == 2


def test_flat_grids():
    assert stage_plan((1000,)).kernel == LINE
    assert stage_plan((100, 31)).kernel == GENERAL
    assert stage_plan((100, 32)).kernel == TILES


def reverse_plan(n, face=0):
    return tlim.load_library().tlim_reverse_plan(ctypes.byref(tlim.make_grid(n)), face)


@pytest.mark.parametrize("n,kernel", [((1000, 1, 1000), MARCH), ((64, 3, 20000), MARCH), ((700, 2, 700), MARCH),
                                      ((20000, 20000, 2), MARCH), ((1000, 4, 1000), BLOCKED_MARCH),
                                      ((128, 128, 128), BLOCKED_MARCH), ((256, 1, 256), BLOCKED_MARCH),
                                      ((100, 40), TILES), ((100, 31), GENERAL), ((1000,), GENERAL)])
def test_reverse_stages(n, kernel):
    assert reverse_plan(n) == kernel
    assert reverse_plan(n, face=1) == GENERAL
