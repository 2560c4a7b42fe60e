"""The fp16 map of the grids: a point's cell, found in fp16 as the kernel finds it, against the box that the lists were built
for.  Exhaustive over the fp16 numbers of one axis, for scales and offsets of all sizes that the kernel accepts."""
import os
import re

import numpy as np
import pytest

from paper_2504_03661_amd import build as lib_build

HEADER = open(os.path.join(lib_build.CSRC, "pq_nearest_grid.h")).read()
H = np.float16


def _constant(name):
    return float(re.search(r"\bconstexpr float " + name + r" = ([0-9.e+-]+)f?;", HEADER).group(1))


BIAS, WIDER, WIDER_F16, UNIT = (_constant("GRID_" + n) for n in ("BIAS", "WIDER", "WIDER_F16", "F16_UNIT"))
X = np.arange(65536, dtype=np.uint16).view(H)
X = X[np.isfinite(X)]


def cells(x, s, o):
    """pq_grid_cell_f16, one axis, s and o in units of UNIT: a fused multiply-add, an addition and a minimum in fp16, then bits"""
    exact = x.astype(np.float64) * float(s) + float(o)                  # (a product of two halves and a sum: exact in a double
    with np.errstate(over="ignore"):                                    # unless it leaves the map by far)
        u = exact.astype(H)
        w = np.minimum((np.abs(u) + H(BIAS / UNIT)).astype(H), np.uint16(0x2fff).view(H))
    bits = (w.view(np.uint16) >> 5) ^ np.where(np.signbit(u), 0xffff, 0).astype(np.uint16)
    return ((bits & 0xfc) >> 2).astype(np.int64)


def _box(e):
    """pq_grid_box of one cell"""
    k = np.where(e < 32, e, e - 64)
    edge = lambda k: np.sign(k) * ((np.uint32(0x40000000) + (np.abs(k).astype(np.uint32) << np.uint32(20))).astype(np.uint32).view(np.float32) - 2.0)
    lo, hi = edge(k).astype(np.float64), edge(k + 1).astype(np.float64)
    half = 0.5 * (hi - lo) + WIDER + (np.maximum(-lo, hi) + BIAS) * WIDER_F16
    return 0.5 * (lo + hi), half


@pytest.mark.parametrize("scale", [1.1e-4, 0.003, 0.11, 1.0, 5.59, 47.3, 913.0, 60000.0, 7.1e5, 60000.0 * 256])
@pytest.mark.parametrize("offset", [0.0, 0.37, -1.93, 27.9, -311.0, 4093.0, -16383.0])
def test_every_point_lies_in_the_box_of_its_cell(scale, offset):
    s, o = H(scale / UNIT), H(offset / UNIT)
    cell, u = cells(X, s, o), (X.astype(np.float64) * float(s) + float(o)) * UNIT
    inside = (cell != 31) & (cell != 32)
    centre, half = _box(cell[inside])
    assert (np.abs(u[inside] - centre) <= half).all()
    assert (np.abs(u[~inside]) > 27.9).all()                            # the outermost cells take nothing else
    assert ((cell >= 32) == (u < 0))[u != 0].all()
