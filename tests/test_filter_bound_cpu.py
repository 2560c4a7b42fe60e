"""The encode and the k-means assignment decide codes in fp64 but first filter centroids with fp32 matrix-core sums; the
filter is safe if every centroid that it does not mark is farther than the nearest one.  This test forms the sums as the
kernels do (with the constants of csrc/pq_filter_constants.h, which they include) under the WORST rounding the bound allows
for — every fp32 addition truncated toward zero, terms added one after the other — on random inputs of very different
magnitudes, and marks centroids by the kernels' rule."""
import os
import re

import numpy as np
import pytest

_HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_03661_amd", "csrc",
                       "pq_filter_constants.h")


def _constant(name):
    """The value the kernels are compiled with: parsed from the header they include."""
    m = re.search(r"^#define\s+" + name + r"\s+([0-9.eE+-]+)f\s*$", open(_HEADER).read(), re.M)
    assert m, name
    return np.float32(m.group(1))


K_ABS, X2F, NEAR = _constant("PQ_FILTER_TAU_ABS"), _constant("PQ_FILTER_X2_FACTOR"), _constant("PQ_FILTER_TAU_NEAR")


def trunc32(v):
    """float64 -> the float32 obtained by truncating toward zero."""
    f = np.asarray(v, dtype=np.float64).astype(np.float32)
    over = np.abs(f.astype(np.float64)) > np.abs(v)
    return np.where(over, np.nextafter(f, np.float32(0)), f).astype(np.float32)


def offset_columns(x2):
    """|x|^2 / 2 with half a per cent on top and a floor, rounded up to o_0 + 2^15 o_1, one of them zero: float16 values."""
    up = (X2F * x2 + np.float32(3) * K_ABS) * np.float32(1.003) + np.float32(6.0e-8)
    large = ~(X2F * x2 + np.float32(3) * K_ABS < np.float32(60000))
    o0 = np.where(large, np.float32(0), up).astype(np.float16)
    o1 = np.where(large, up * np.float32(1 / 32768), np.float32(0)).astype(np.float16)
    return o0, o1


@pytest.mark.parametrize("ds", [2, 4])
@pytest.mark.parametrize("c_scale,x_scale", [(1.0, 1.0), (1e-3, 1e-3), (30.0, 1.0), (1.0, 200.0), (30.0, 100.0), (1e-5, 3.0), (30.0, 30.0),
                                             (60.0, 60.0), (0.01, 0.01)])
def test_unmarked_centroids_are_farther_under_the_worst_rounding(ds, c_scale, x_scale):
    rng = np.random.default_rng(int(1000 * ds + 7 * c_scale + x_scale) % 2**31)
    c = (rng.standard_normal((256, ds)) * c_scale).astype(np.float16).astype(np.float32)
    c[128:160] = c[:32]                                       # ties and ...
    steps = lambda v, most: (v + rng.integers(-most, most + 1, v.shape) * np.spacing(np.abs(v).astype(np.float16)).astype(np.float32)).astype(np.float16)
    c[160:] = steps(c[:96], 2)                                # ... pairs a few fp16 steps apart
    x = (rng.standard_normal((512, ds)) * x_scale).astype(np.float16).astype(np.float32)
    if c_scale == x_scale:
        x[::2] = steps(c[rng.integers(0, 96, 256)], 3)        # ... with tokens around them
    e = max(int(np.frexp(np.abs(c).max())[1]), -11)           # a codebook of small numbers: the values' gain, a power of four
    gain = np.float32(2.0 ** (4 - 2 * e)) if np.abs(c).max() < 2 else np.float32(1)
    # centroid rows as the kernels build them
    n = np.zeros(256, np.float32)
    for j in range(ds):
        n = n + c[:, j] * c[:, j]
    h = np.float32(0.5) * gain * n
    hh = h.astype(np.float16)
    hl = (h - hh.astype(np.float32)).astype(np.float16)
    rows = (c * gain).astype(np.float16)
    assert (rows.astype(np.float64) == c.astype(np.float64) * float(gain)).all() and (h < 60000).all()
    # token columns
    xg = x * gain
    x2 = np.zeros(len(x), np.float32)
    for j in range(ds):
        x2 = xg[:, j] * xg[:, j] + x2
    x2 = x2 / gain
    inside = X2F * x2 + np.float32(3) * K_ABS < np.float32(2e9)     # others send their chunk through the fp64 scan
    assert inside.all() or c_scale < 1e-4 * x_scale
    x, x2 = x[inside], x2[inside]
    o0, o1 = offset_columns(x2)
    # the instruction's sum, every add truncated: the products are exact in fp32
    products = [-(x[:, j].astype(np.float64)[:, None] * rows[:, j].astype(np.float64)[None]) for j in range(ds)]
    products += [np.broadcast_to(hh.astype(np.float64), (len(x), 256)), np.broadcast_to(hl.astype(np.float64), (len(x), 256)),
                 np.broadcast_to(o0.astype(np.float64)[:, None], (len(x), 256)),
                 np.broadcast_to(o1.astype(np.float64)[:, None] * 32768, (len(x), 256))]
    true = ((x.astype(np.float64)[:, None] - c.astype(np.float64)[None]) ** 2).sum(2)
    nearest = true.min(1)
    for order in (range(len(products)), reversed(range(len(products)))):
        acc = np.zeros((len(x), 256), np.float32)
        for k in order:
            acc = trunc32(acc.astype(np.float64) + products[k])
        assert (acc > 0).all()                                # positive: they compare as integers
        best = acc.min(1)
        limit = (best.astype(np.float64) * (1 + float(NEAR)) + (float(NEAR) * x2.astype(np.float64) + float(K_ABS))).astype(np.float32)
        marked = acc <= limit[:, None]
        assert (marked | (true > nearest[:, None])).all()     # every nearest centroid is marked, all of a tie
        if c_scale >= x_scale:                                # a filter, not a pass-through
            assert marked.sum(1).mean() <= 4 and marked.sum(1).max() <= 96


def test_truncation_helper():
    v = np.array([1.0 + 2.0 ** -24, -(1.0 + 2.0 ** -24), 1.0 + 3 * 2.0 ** -24, 0.1])
    t = trunc32(v)
    assert t[0] == np.float32(1.0) and t[1] == np.float32(-1.0) and t[2] == np.float32(1.0 + 2.0 ** -23)
    assert abs(float(t[3])) <= 0.1
