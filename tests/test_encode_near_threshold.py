"""The 8-bit nearest-centroid filter keeps every centroid whose computed value lies within
tau = PQ_FILTER_TAU_NEAR (|x|^2 + best) + PQ_FILTER_TAU_ABS of the best one.  On the CPU: tau against sums whose errors
are as large, and of such signs, as the bound allows.  On the GPU: the codes at the edges of the token mapping and of the
offset's range."""
import numpy as np
import pytest
import torch

from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W
from tests.test_filter_bound_cpu import K_ABS, X2F, _constant

NEAR = float(_constant("PQ_FILTER_TAU_NEAR"))
EPS = 11.5 * 2.0 ** -23


@pytest.mark.parametrize("ds", [2, 4])
@pytest.mark.parametrize("c_scale,x_scale,outliers", [(1, 1, 0), (1e-3, 1e-3, 0), (30, 1, 0), (1, 200, 0), (1, 1, 60), (1e-5, 3, 0)])
def test_worst_case_errors_never_hide_the_nearest_centroid(ds, c_scale, x_scale, outliers):
    rng = np.random.default_rng(ds + int(100 * x_scale) + outliers)
    c = rng.standard_normal((256, ds)) * c_scale
    c[::50] *= max(1, outliers)
    c[128:] = c[:128] + rng.standard_normal((128, ds)) * c_scale * 10.0 ** rng.uniform(-6, -2, (128, 1))     # close pairs
    c = c.astype(np.float16).astype(np.float64)
    x = (rng.standard_normal((2000, ds)) * x_scale).astype(np.float16).astype(np.float64)
    pair = rng.integers(0, 128, 1000)
    x[:1000] = (0.5 * (c[pair] + c[pair + 128])).astype(np.float16)
    x2 = (x * x).sum(1)
    off = (float(X2F) * x2 + 3 * float(K_ABS))[:, None] * 1.001
    true = off + 0.5 * (c * c).sum(1)[None] - x @ c.T
    size = off + 0.5 * (c * c).sum(1)[None] + np.abs(x) @ np.abs(c).T
    err = EPS * size + 2.0 ** -25
    nearest = true.argmin(1)
    rows = np.arange(len(x))
    assert (true - err > 0).all()
    # the nearest centroid computed as high as it may be, every other one as low
    computed = true - err
    computed[rows, nearest] = true[rows, nearest] + err[rows, nearest]
    best = computed.min(1)
    tau = NEAR * (x2 + best) + float(K_ABS)
    assert (computed[rows, nearest] <= best + tau).all()


@pytest.mark.gpu
@pytest.mark.parametrize("M", [64, 32])
@pytest.mark.parametrize("B_,n_new", [(3, 56), (3, 57), (2, 63), (2, 64), (2, 65), (3, 113), (3, 114), (1, 70), (40, 7)])
def test_codes_at_the_edges_of_the_mapping_and_of_the_offset(M, B_, n_new):
    """Token counts on both sides of the rule that gives every sequence its own 64-token chunks (57 and 114 are the first
    to have them), remainders, several chunks per wavefront's job; sub-vectors up to the largest fp16 (beyond a length of
    345 the offset moves to its second slot, beyond 6e4 the chunk takes the full scan)."""
    ds = 128 // M
    lens = tuple(int(v) for v in np.random.default_rng(B_).integers(0, 90, B_))
    w = W.Workload("edge", B_, 4, 4, 128, M, 90 + n_new, "f16", n_new=n_new, seed=70 + M + n_new, ctx_lens=lens)
    data = W.generate(w, ctx_cap=90 + n_new)
    for x in (data["new_k"], data["new_v"]):
        x[:, :, ::3, :ds] = np.float16(340.0) * np.sign(x[:, :, ::3, :ds])
        x[:, :, ::4, ds:2 * ds] *= np.float16(900.0)
        x[:, :, ::5, 2 * ds:3 * ds] = np.float16(65504.0)
        x[:, :, 1::5, 2 * ds:3 * ds] = np.float16(-30000.0)
        x[:, :, ::2, 3 * ds:4 * ds] = 0
    with PQSession(data, 4, "f16", max_context=90 + n_new) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        assert s.ctx_len.cpu().tolist() == [n + n_new for n in lens]
        got_k, got_v = s.unpack(PQ_CODES_K, 90 + n_new), s.unpack(PQ_CODES_V, 90 + n_new)
    exp_k, exp_v = O.encode(data["new_k"], data["k_codebook"]), O.encode(data["new_v"], data["v_codebook"])
    for b, n in enumerate(lens):
        np.testing.assert_array_equal(got_k[b, :, n:n + n_new], exp_k[b])
        np.testing.assert_array_equal(got_v[b, :, n:n + n_new], exp_v[b])
        np.testing.assert_array_equal(got_k[b, :, :n], data["k_codes"][b, :, :n])
