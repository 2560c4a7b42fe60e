"""The grid that names, for every cell of a subspace's plane, the centroids that can be the nearest of a point in it (long
appends and large trainings at two dims per subspace).  On the CPU: the cell lists, built as the kernel builds them for fp16 and
for fp32 codebooks, hold the fp64-nearest centroid of every point.  On the GPU: codes and trained codebooks against the oracle."""
import ctypes
import functools
import os
import re
import subprocess
import tempfile

import numpy as np
import pytest
import torch

from oracle import pq_kmeans_oracle as K
from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V
from paper_2504_03661_amd import binding as B
from paper_2504_03661_amd import build as lib_build
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W
from tests import test_grid_map as map16
from tests.test_gpu_kmeans import gpu_fit, make_ctx

F = np.float32
KINDS = ["normal", "lattice", "duplicates", "outliers", "line", "tiny", "two clusters", "far from zero", "diagonal", "stretched",
         "heavy tails", "equal", "sixteen values"]


def codebook_and_points(kind, n, seed, dtype=np.float16):
    """256 centroids of one kind and n points: of the same distribution, centroids themselves, the middles between two
    neighbouring ones (ties), points far outside, zeros."""
    rng = np.random.default_rng(seed)
    normal = lambda m: rng.standard_normal((m, 2))
    draw = {
        "normal": normal,
        "lattice": lambda m: rng.integers(-8, 8, (m, 2)) * 0.25,
        "duplicates": normal,
        "outliers": lambda m: np.where(rng.random((m, 2)) < 0.02, 20.0, 1.0) * normal(m),
        "line": lambda m: normal(m) * [1, 0] + [0, 0.5],
        "tiny": lambda m: normal(m) * 1e-4,
        "two clusters": lambda m: normal(m) * 0.01 + np.where(rng.random((m, 1)) < 0.5, -30.0, 30.0),
        "far from zero": lambda m: normal(m) * 0.1 + [50, -3],
        "diagonal": lambda m: normal(m)[:, :1] * [1, 1] + normal(m) * 0.01,
        "stretched": lambda m: normal(m) * [100, 0.3],
        "heavy tails": lambda m: np.clip(rng.standard_cauchy((m, 2)), -3e4, 3e4),
        "equal": lambda m: normal(m) * 0 + 0.75,
        "sixteen values": lambda m: rng.integers(0, 4, (m, 2)) * 0.5,
        "smallest": lambda m: normal(m) * 1e-5,
        "far and narrow": lambda m: normal(m) * [0.1, 0.01] + [70, -7],
    }[kind]
    c = draw(256)
    if kind == "lattice":
        c = np.stack(np.meshgrid(np.arange(-8, 8), np.arange(-8, 8)), -1).reshape(256, 2) * 0.25
    if kind == "duplicates":
        c[200:] = c[:56]
    c = c.astype(dtype)
    x = draw(n)
    share = n // 8
    x[:share] = c[rng.integers(0, 256, share)]
    wide = c.astype(np.float64)
    neighbour = np.argsort(((wide[:, None] - wide[None]) ** 2).sum(-1), 1)[:, 1]
    first = rng.integers(0, 256, share)
    x[share:2 * share] = 0.5 * (wide[first] + wide[neighbour[first]])
    x[2 * share:2 * share + 40] *= 50
    x[2 * share + 40:2 * share + 60] = 0
    if dtype == np.float16:
        x = np.clip(x, -65504, 65504)
    return c, rng.permutation(x).astype(dtype)


HEADER = open(os.path.join(lib_build.CSRC, "pq_nearest_grid.h")).read()


def _constant(name):
    """A number the kernels are compiled with, from their header."""
    m = re.search(r"\bconstexpr (?:float|int) " + name + r" = ([0-9.e+-]+)f?;", HEADER)
    assert m, name
    return F(m.group(1))


COVER, DEVIATIONS, LOWERED, MARGIN, WIDER, WIDER_F16, UNIT = (
    _constant("GRID_" + n) for n in ("COVER", "DEVIATIONS", "LOWERED", "MARGIN", "WIDER", "WIDER_F16", "F16_UNIT"))
LONGEST = int(_constant("GRID_LONGEST"))


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * b + c).astype(F)


def _edge(k):
    e = (np.uint32(0x40000000) + (np.abs(k).astype(np.uint32) << np.uint32(20))).astype(np.uint32).view(F) - F(2)
    return np.where(k < 0, -e, e)


def _rounded(v):
    """A factor of the fp16 map: an fp16 number in units of UNIT."""
    return (v / UNIT).astype(np.float16).astype(F) * UNIT


def _cells(x, s, o):
    if x.dtype == np.float16:
        return map16.cells(x, s / UNIT, o / UNIT)
    u = _fma(x, s, o)
    b = np.minimum((np.abs(u) + F(2)).astype(F).view(np.uint32), np.uint32(0x41ffffff))
    e = ((b >> np.uint32(20)) & np.uint32(63)).astype(np.int64)
    return np.where(np.signbit(u), 63 - e, e)


def _box(e, n, dtype):
    """Centre and half side of cell coordinates e .. e + n - 1."""
    k = np.where(e < 32, e, e - 64)
    lo, hi = _edge(k), _edge(k + n)
    half = F(0.5) * (hi - lo) + WIDER
    if dtype == np.float16:
        half = _fma(np.maximum(-lo, hi) + F(2), WIDER_F16, half)
    return F(0.5) * (lo + hi), half


def _repeats(c):
    """The centroids that pq_grid_take_out finds to be equal to one before them: the first with their hash."""
    bits = c.view(np.uint16 if c.dtype == np.float16 else np.uint32).astype(np.uint64)
    h = bits[:, 0] | bits[:, 1] << np.uint64(16) if c.dtype == np.float16 else bits[:, 0] * np.uint64(0x85ebca6b) & np.uint64(0xffffffff) ^ bits[:, 1]
    h = (h * np.uint64(0x9e3779b1) & np.uint64(0xffffffff)) >> np.uint64(24)
    first = np.array([np.nonzero(h == v)[0][0] for v in h])
    return (first < np.arange(256)) & (c[first] == c).all(1)


def _lists(c):
    """The steps of pq_grid_tables, pq_grid_take_out and pq_grid_lists -> (s, o, candidates [64, 64, 256] bool, which cells have a
    list, fill code of every cell); None: no grid for this codebook."""
    dtype, exact, again, c = c.dtype, c.astype(np.float64), _repeats(c), c.astype(F)
    mean, end = np.zeros(2, F), np.full(2, 3e38, F)
    for _ in range(2):
        near = np.abs(c - mean) <= end
        n = near.sum(0).astype(F)
        new = (c * near).sum(0, dtype=F) / n
        dev = (np.abs(c - new) * near).sum(0, dtype=F) / n
        mean, end = new, F(3) * dev
    if not (dev > 1e-30).all():
        return None
    s = COVER / (DEVIATIONS * dev)
    if dtype == np.float16:
        s = _rounded(np.minimum(s, F(60000) * UNIT))
        if not ((s > 1e-4).all() and (np.abs(mean * s) < 16384).all()):
            return None
    o = -mean * s
    if dtype == np.float16:
        o = _rounded(o)
    w = F(s[0] / s[1]) ** 2
    u = _fma(c, s, o)
    if not (np.abs(u) < 1e6).all() or not 1e-9 < w < 1e9:
        return None
    ax, ay = u[:, 0], w * u[:, 1]
    norm = F(0.5) * (u[:, 0] * ax + u[:, 1] * ay)
    low = np.where(again, F(1e30), norm * (F(1) - LOWERED))
    exact = np.where(again[:, None], np.inf, exact)
    lists, listed, fills = np.zeros((64, 64, 256), bool), np.zeros((64, 64), bool), np.zeros((64, 64), np.int64)
    lowest, largest = (-60000, 60000) if dtype == np.float16 else (-3e37, 3e37)
    for bx in range(16):
        for by in range(16):
            # the block's list: all centroids against the one nearest to its centre
            (gx, hx), (gy, hy) = _box(np.int64(4 * bx), 4, dtype), _box(np.int64(4 * by), 4, dtype)
            p = np.clip([(gx - o[0]) / s[0], (gy - o[1]) / s[1]], lowest, largest).astype(dtype).astype(np.float64)
            r = int(((exact - p) ** 2).sum(1).argmin())
            value = lambda k: _fma(-gy, ay[k], _fma(-gx, ax[k], low[k]))
            far_x, far_y = np.abs(gx) + hx, np.abs(gy) + hy
            limit = value(r) + MARGIN * (norm[r] + far_x * far_x + w * far_y * far_y)
            t = _fma(-np.abs(ay - ay[r]), hy, _fma(-np.abs(ax - ax[r]), hx, value(slice(None))))
            k = np.nonzero(t <= limit)[0]
            free = np.setdiff1d(np.arange(32), np.concatenate([k, np.nonzero(again)[0]]))
            if len(k) > LONGEST or len(free) == 0:
                continue
            # its cells' lists: the block's candidates against the one nearest to the cell's centre, found in numbers whose
            # low bits hold the place in the list
            e = np.arange(4)
            (gx, hx), (gy, hy) = _box(4 * bx + e, 1, dtype), _box(4 * by + e, 1, dtype)
            gx, hx, gy, hy = (np.repeat(gx, 4), np.repeat(hx, 4), np.tile(gy, 4), np.tile(hy, 4))
            half = F(0.5) * (gx * gx + w * gy * gy)
            v = _fma(ay[k], -gy[:, None], _fma(ax[k], -gx[:, None], low[k] + half[:, None]))
            cut = v.view(np.int32) & ~(31 if len(k) <= 32 else 63)
            first = cut.argmin(1)
            ref, nearest = k[first], cut[np.arange(16), first].view(F)
            far = (np.abs(gx) + hx) ** 2 + w * (np.abs(gy) + hy) ** 2
            limit = nearest + MARGIN * (F(2) * np.abs(nearest) + norm[ref] + far)
            t = _fma(-np.abs(ax[k] - ax[ref][:, None]), hx[:, None], v)
            t = _fma(-np.abs(ay[k] - ay[ref][:, None]), hy[:, None], t)
            rows, cols = 4 * bx + np.repeat(e, 4), 4 * by + np.tile(e, 4)
            mask = np.zeros((16, 256), bool)
            mask[:, k] = t <= limit[:, None]
            lists[rows, cols], listed[rows, cols], fills[rows, cols] = mask, True, free[0]
    listed[31:33] = listed[:, 31:33] = False
    return s, o, lists, listed, fills


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("kind", KINDS + ["smallest", "far and narrow"])
def test_lists_hold_the_nearest_centroid_of_every_point(kind, dtype):
    """With all ties but the centroids that repeat one before them, which are no codes."""
    for seed in range(3):
        c, x = codebook_and_points(kind, 8000, seed, dtype)
        grid = _lists(c)
        if grid is None:
            assert kind in ("line", "equal")
            continue
        s, o, lists, listed, fills = grid
        ix, iy = _cells(x[:, 0], s[0], o[0]), _cells(x[:, 1], s[1], o[1])
        inside = listed[ix, iy]
        d = ((x.astype(np.float64)[:, None] - c.astype(np.float64)[None]) ** 2).sum(-1)
        nearest = d == d.min(1)[:, None]
        again = _repeats(c)
        assert not again[d.argmin(1)].any()
        assert not (nearest & ~again & ~lists[ix, iy])[inside].any()
        assert not lists[:, :, again].any()
        assert not nearest[np.arange(len(x)), fills[ix, iy]][inside].any()
        if kind in ("normal", "tiny") or (kind == "smallest" and dtype == np.float32):
            assert inside.mean() > 0.98 and (lists[ix, iy].sum(1) > 4)[inside].mean() < 0.15


def test_the_kinds_reach_every_form_of_list():
    """Blocks of up to 32, of 33 to 64 and of more candidates; cells of up to 4, of more, and of more than 32; a pool that is too
    small: what the kernel treats in different ways, in the codebooks that the GPU tests use as well."""
    seen = set()
    for kind in KINDS:
        grid = _lists(codebook_and_points(kind, 8000, 0)[0])
        if grid is None:
            seen.add("no grid")
            continue
        _, _, lists, listed, _ = grid
        n = lists.sum(2)[listed]
        seen |= {"cells " + size for size, any_ in (("<= 4", (n <= 4).any()), ("> 4", ((n > 4) & (n <= 32)).any()), ("> 32", (n > 32).any())) if any_}
        if listed.sum() < 62 * 62:
            seen.add("blocks > 64")
        if ((n + 3) // 4)[n > 4].sum() > _constant("GRID_POOL"):
            seen.add("pool too small")
    assert seen == {"no grid", "cells <= 4", "cells > 4", "cells > 32", "blocks > 64", "pool too small"}


@functools.cache
def _rule():
    """The launchers' rule (slices of the tokens for the grid kernels, 0: the filter), compiled from its source."""
    text = "".join(re.search(what, HEADER, re.S | re.M).group(0) for what in (r"^struct pq_grid_price {.*?^};", r"^inline int pq_grid_slices\(.*?^}"))
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "rule.cpp"), "w") as f:
            f.write("#include <cstdint>\n" + text + "\nextern \"C\" int rule(int64_t c, int64_t f, int64_t g, int n, int kept, uint32_t price) "
                    "{ return pq_grid_slices(c, f, g, n, kept, {price >> 16, price & 65535}); }\n")
        lib = os.path.join(d, "rule.so")
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", lib, f.name], check=True)
        fn = ctypes.CDLL(lib).rule
    fn.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 2 + [ctypes.c_uint32]
    return lambda chunks, filter_chunks, groups, n_cu, kept=False, price=18 << 16 | 72: fn(chunks, filter_chunks, groups, n_cu, kept, price)


def encode_slices(Hkv, B_, n_new, n_cu=256):
    return _rule()(B_ * ((n_new + 126) >> 6), (B_ * n_new + 63) // 64, 2 * Hkv * 16, n_cu)


def train_slices(Hkv, n, n_cu=256):
    return _rule()((n + 63) // 64, (n + 63) // 64, Hkv * 16, n_cu)


LONG_APPENDS = [
    (2, 1, 68001, np.float16, [0], 68001),
    (8, 3, 23003, np.float16, [0, 77, 63], 23070),                # K codes by lane quads; the second sequence overflows
    (2, 2, 34000, np.float32, [5, 64], 40000),
]
TRAININGS = [(2, 80003, 1), (5, 45000, 2)]


def test_the_rule_takes_the_cheapest_of_all_divisions():
    """What the launchers' rule gives without a walk over them for appends too short to gain."""
    rng = np.random.default_rng(0)
    seen = set()
    for _ in range(3000):
        n, b, heads, n_cu = (int(np.exp(rng.uniform(0, top))) for top in (11, 4, 5, 6.3))
        kept, price = bool(rng.integers(2)), (18, 72) if rng.random() < 0.5 else (int(rng.integers(18, 600)), int(rng.integers(72, 500)))
        chunks, through_filter, groups = b * ((n + 126) >> 6), (b * n + 63) // 64, heads * 32
        times = {s: -(-groups * s // n_cu) * ((900 if kept else 7400) + -(-chunks // s) * price[0]) for s in range(1, 33)}
        best = min(times, key=times.get)
        want = best if times[best] < through_filter * groups * price[1] // n_cu else 0
        assert _rule()(chunks, through_filter, groups, n_cu, kept, price[0] << 16 | price[1]) == want
        seen.add(min(want, 2))
    assert seen == {0, 1, 2}


def test_codebooks_that_the_grids_do_not_serve_are_left_to_the_filter():
    """The rule for kept grids, told that none of the subspaces are the filter's, one of four, all."""
    useless = [int(v) for v in re.search(r"if \(pq_grid_useless\(m\)\)\s+return {(\d+)u, (\d+)u};", HEADER).groups()]
    none, some, all_ = (((4 - k) * 18 + k * useless[0]) // 4 << 16 | ((4 - k) * 72 + k * useless[1]) // 4 for k in (0, 1, 4))
    sizes = [(32, 1, n) for n in (1200, 2000, 4000, 9000, 32768)] + [(8, 1, 4000), (8, 3, 30000), (4, 64, 2000)]
    kept = lambda H, b, n, c: _rule()(b * ((n + 126) >> 6), (b * n + 63) // 64, 2 * H * 16, 256, True, c)
    assert all(kept(*s, none) > 0 and kept(*s, all_) == 0 for s in sizes)
    assert all(kept(*s, some) > 0 for s in sizes[1:])


def test_the_sizes_below_take_the_grid():
    assert all(encode_slices(2, B_, n_new) > 1 for _, B_, n_new, *_ in LONG_APPENDS)
    assert all(train_slices(Hkv, n) > 1 for Hkv, n, _ in TRAININGS)
    assert encode_slices(32, 1, 9000) == 1 and encode_slices(32, 1, 8000) == 0 and encode_slices(1, 1, 20000) == 0
    assert train_slices(32, 9000) == 1 and train_slices(32, 4000) == 0 and train_slices(2, 68003) == 0


def _data(Hq, Hkv, B_, n_new, dtype, start, kinds=KINDS):
    w = W.Workload("grid", B_, Hq, Hkv, 128, 64, 64, "f16" if dtype == np.float16 else "f32", n_new=8, seed=n_new)
    data = W.generate(w)
    for book, new in (("k_codebook", "new_k"), ("v_codebook", "new_v")):
        cb = np.empty((Hkv, 64, 256, 2), dtype)
        x = np.empty((B_, Hkv, n_new, 128), dtype)
        for h in range(Hkv):
            for i in range(64):
                c, p = codebook_and_points(kinds[(i + h) % len(kinds)], B_ * n_new, 1000 * h + i + len(book), dtype)
                cb[h, i] = c
                x[:, h, :, 2 * i:2 * i + 2] = p.reshape(B_, n_new, 2)
        if book == "k_codebook" and kinds is KINDS:
            cb[0, 20, 7, 1] = np.inf
        data[book], data[new] = cb, x
    data["ctx_len"] = np.asarray(start, np.int32)
    return data


def _n_cu():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,B_,n_new,dtype,start,room", LONG_APPENDS)
def test_long_appends_equal_the_oracle(Hq, B_, n_new, dtype, start, room):
    assert encode_slices(2, B_, n_new, _n_cu()) > 0
    data = _data(Hq, 2, B_, n_new, dtype, start)
    with PQSession(data, Hq, "f16" if dtype == np.float16 else "f32", max_context=room) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got = {"k": s.unpack(PQ_CODES_K, room), "v": s.unpack(PQ_CODES_V, room)}
        assert s.ctx_len.cpu().tolist() == [min(room, n + n_new) for n in start]
    for name, codes in got.items():
        want = O.encode(data["new_" + name], data[name + "_codebook"])
        for b, n in enumerate(start):
            wrong = codes[b, :, n:n + n_new] != want[b, :, :room - n]
            assert not wrong.any(), [(h, KINDS[(i + h) % len(KINDS)]) for h, i in set(zip(*np.nonzero(wrong.any(1))))]


WITHOUT_A_GRID = ["sixteen values", "equal", "two clusters", "line"]   # no subspace of a workgroup has one
LEFT_TO_THE_FILTER = ["heavy tails", "outliers", "normal", "duplicates"]   # many tokens outside the map, or with two nearest ones


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [WITHOUT_A_GRID, LEFT_TO_THE_FILTER])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_what_the_grid_leaves_to_the_filter(kinds, dtype):
    """Unsure tokens by the hundreds per wavefront and subspace: 64 at a time, the rest of all wavefronts together."""
    assert encode_slices(2, 2, 34007, _n_cu()) > 0
    data = _data(2, 2, 2, 34007, dtype, [3, 0], kinds)
    with PQSession(data, 2, "f16" if dtype == np.float16 else "f32", max_context=34010) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got = {"k": s.unpack(PQ_CODES_K, 34010), "v": s.unpack(PQ_CODES_V, 34010)}
    for name, codes in got.items():
        want = O.encode(data["new_" + name], data[name + "_codebook"])
        for b, n in enumerate([3, 0]):
            wrong = codes[b, :, n:n + 34007] != want[b]
            assert not wrong.any(), [(h, kinds[(i + h) % len(kinds)]) for h, i in set(zip(*np.nonzero(wrong.any(1))))]


@pytest.mark.gpu
def test_rows_that_start_off_a_16_byte_address():
    assert encode_slices(2, 1, 68001, _n_cu()) > 0
    data = _data(2, 2, 1, 68001, np.float16, [0])
    shifted = {}
    for name in ("new_k", "new_v"):
        flat = torch.empty(data[name].size + 1, dtype=torch.float16, device="cuda")
        shifted[name] = flat[1:].view(data[name].shape)
        shifted[name].copy_(torch.from_numpy(data[name]))
    with PQSession(data, 2, "f16", max_context=68001) as s:
        s.append(shifted["new_k"], shifted["new_v"])
        torch.cuda.synchronize()
        off = [s.unpack(kind, 68001) for kind in (PQ_CODES_K, PQ_CODES_V)]
        s.ctx_len.zero_()
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        for kind, codes in zip((PQ_CODES_K, PQ_CODES_V), off):
            np.testing.assert_array_equal(codes, s.unpack(kind, 68001))


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [KINDS, WITHOUT_A_GRID, LEFT_TO_THE_FILTER])
@pytest.mark.parametrize("Hkv,n,iters", TRAININGS)
def test_training_on_many_samples_equals_the_oracle(Hkv, n, iters, kinds):
    if kinds is not KINDS:
        iters = 1
    assert train_slices(Hkv, n, _n_cu()) > 0
    samples = np.empty((Hkv, n, 128), np.float16)
    init = np.empty((Hkv, 64, 256, 2), np.float16)
    for h in range(Hkv):
        for i in range(64):
            init[h, i], samples[h, :, 2 * i:2 * i + 2] = codebook_and_points(kinds[(i + 3 * h) % len(kinds)], n, 100 * h + i)
    ctx = make_ctx(Hkv, 64)
    try:
        got = gpu_fit(ctx, samples, init, iters)
    finally:
        B.pq_attn_destroy(ctx)
    want, _ = K.kmeans_lloyd(samples, init, iters)
    wrong = (got.view(np.uint16) != want.view(np.uint16)).any((2, 3))
    assert not wrong.any(), [(h, kinds[(i + 3 * h) % len(kinds)]) for h, i in zip(*np.nonzero(wrong))]


def _span_us(f):
    """Shortest of five spans of five calls."""
    begin, end = torch.cuda.Event(True), torch.cuda.Event(True)
    best = float("inf")
    for _ in range(6):                                          # the first warms up
        begin.record()
        for _ in range(5):
            f()
        end.record()
        end.synchronize()
        best = min(best, begin.elapsed_time(end) * 200) if _ else best
    return best


def _rows(kind, shape, gen):
    x = torch.randn(shape, generator=gen, device="cuda")
    if kind == "laplace":
        u = torch.rand(shape, generator=gen, device="cuda") - 0.5
        x = -torch.sign(u) * torch.log1p(-1.9999 * u.abs())
    if kind == "2 % times 20":
        x = torch.where(torch.rand(shape, generator=gen, device="cuda") < 0.02, 20 * x, x)
    if kind == "few values":
        x = (2 * x).round() / 4
    return x.half()


# What the data make of the grids, beside the same call through the filter, which takes rows that start off a 16-byte address:
# appends with kept grids, appends and trainings that build them in place.
# Heavy tails: 0.38, 0.91 and 0.78 measured; 1.55 in place and 1.35 in training with the tokens outside the map one by one.  Few
# values, ties all over: 0.51, 0.63 and 0.49; 2.3 and 1.9 with their tokens one by one, 1.2 and 0.95 with repeated centroids left in.
@pytest.mark.gpu
@pytest.mark.parametrize("kind,most_kept,most", [("laplace", 0.5, 1.15), ("2 % times 20", 0.5, 1.15), ("few values", 0.7, 0.85)])
def test_data_that_the_grids_do_not_serve_cost_little(kind, most_kept, most):
    n, H, gen = 9000, 32, torch.Generator(device="cuda").manual_seed(1)
    assert encode_slices(H, 1, n, _n_cu()) > 0 and train_slices(H, n, _n_cu()) > 0
    cfg = B.PQAttnConfig(batch=1, n_q_heads=H, n_kv_heads=H, n_subspaces=64, max_context=n)
    ctx = B.pq_attn_create(cfg)
    x = [_rows(kind, (H, n, 128), gen) for _ in range(2)]
    books = [t[:, :256].reshape(H, 256, 64, 2).transpose(1, 2).contiguous() for t in x]
    B.pq_attn_set_codebooks(ctx, *books)
    codes = torch.zeros((2, B.pq_attn_codes_bytes(cfg)), dtype=torch.uint8, device="cuda")
    length = torch.zeros(1, dtype=torch.int32, device="cuda")
    nbytes = B.pq_kmeans_workspace_bytes(ctx)
    workspace, book = torch.empty(nbytes, dtype=torch.uint8, device="cuda"), books[0].clone()

    def encode(k, v, own=(None, None)):
        length.zero_()
        B.pq_encode_append(ctx, k, v, n, *own, codes[0], codes[1], length)

    def train(k):
        book.copy_(books[0])
        B.pq_kmeans_fit(ctx, k, n, book, 1, workspace, nbytes)

    off = []
    for t in x:
        flat = torch.empty(t.numel() + 2, dtype=t.dtype, device="cuda")
        off.append(flat[2:].view(t.shape))
        off[-1].copy_(t)
    kept, through_filter = _span_us(lambda: encode(*x)), _span_us(lambda: encode(*off))
    in_place, again = _span_us(lambda: encode(*x, books)), _span_us(lambda: encode(*off, books))    # (none are kept of these)
    trained, trained_by_filter = _span_us(lambda: train(x[0])), _span_us(lambda: train(off[0]))
    B.pq_attn_destroy(ctx)
    print(f"{kind}: kept {kept / through_filter:.2f}, in place {in_place / again:.2f}, training {trained / trained_by_filter:.2f}")
    assert kept <= most_kept * through_filter and in_place <= most * again, (kept, through_filter, in_place, again)
    assert trained <= most * trained_by_filter, (trained, trained_by_filter)


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1e-4, 1e-5])
def test_small_numbers_keep_their_grids(scale):
    """Appends whose context keeps grids, of small numbers and of unit scale: 1.0 measured; 4.3 at 1e-5 where the fp16 map ended at
    deviations of 9e-5 (and 2.1 at 3e-5)."""
    n, H, gen = 9000, 32, torch.Generator(device="cuda").manual_seed(2)
    cfg = B.PQAttnConfig(batch=1, n_q_heads=H, n_kv_heads=H, n_subspaces=64, max_context=n)
    codes = torch.zeros((2, B.pq_attn_codes_bytes(cfg)), dtype=torch.uint8, device="cuda")
    length, times = torch.zeros(1, dtype=torch.int32, device="cuda"), []
    for factor in (1.0, scale):
        ctx = B.pq_attn_create(cfg)
        x = [(torch.randn((H, n, 128), generator=gen, device="cuda") * factor).half() for _ in range(2)]
        B.pq_attn_set_codebooks(ctx, *[t[:, :256].reshape(H, 256, 64, 2).transpose(1, 2).contiguous() for t in x])

        def encode():
            length.zero_()
            B.pq_encode_append(ctx, *x, n, None, None, codes[0], codes[1], length)

        times.append(_span_us(encode))
        B.pq_attn_destroy(ctx)
    assert times[1] <= 1.4 * times[0], times
