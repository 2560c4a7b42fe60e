"""The nearest-centroid filter at the scales that keys and values have: a codebook of small numbers gets a gain, so that the
filter stays as selective and the codes the same.  On the CPU: the bound with the gain.  On the GPU: codes and codebooks
against the oracle, and the time against that of unit scale."""
import numpy as np
import pytest
import torch

import paper_2504_03661_amd as P
from oracle import pq_kmeans_oracle as K
from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W
from tests.test_encode_few import takes_the_few_token_kernel
from tests.test_encode_near_threshold import EPS, NEAR
from tests.test_filter_bound_cpu import K_ABS, X2F
from tests.test_gpu_kmeans import gpu_fit, make_ctx


def gain_of(c_max):
    """pq_filter_scale of an fp16 codebook."""
    e = max(int(np.frexp(np.float32(c_max))[1]), -11)
    return 2.0 ** (4 - 2 * e) if 0 < c_max < 2 else 1.0


@pytest.mark.parametrize("c_max", [6e-8, 1e-4, 2.0 ** -12, 2.0 ** -11, 0.01, 0.4, 0.999, 1.0, 1.5, 1.999])
def test_the_gain_keeps_every_coordinate_exact(c_max):
    g = gain_of(np.float16(c_max))
    c = np.arange(0, int(np.float16(c_max).view(np.uint16)) + 1, dtype=np.uint16).view(np.float16)      # every value up to it
    scaled = c.astype(np.float64) * g
    assert np.log2(g) % 2 == 0 and scaled.max() < 2 ** 15 and (scaled.astype(np.float16) == scaled).all()


@pytest.mark.parametrize("ds", [2, 4])
@pytest.mark.parametrize("scale", [1.0, 0.3, 0.05, 0.01, 1e-3, 1e-4])
def test_the_filter_is_safe_and_selective_at_every_scale(ds, scale):
    """Errors as large, and of such signs, as the bound allows, as in test_encode_near_threshold; and of random tokens few
    have a second candidate within tau.  (fp16 numbers of 1e-4 are 600 of the smallest steps: tokens coincide.)"""
    rng = np.random.default_rng(ds)
    c = (rng.standard_normal((256, ds)) * scale).astype(np.float16).astype(np.float64)
    x = (rng.standard_normal((4000, ds)) * scale).astype(np.float16).astype(np.float64)
    x[3000:] *= 20
    g = gain_of(np.abs(c).max())
    x2 = g * (x * x).sum(1)
    off = (float(X2F) * x2 + 3 * float(K_ABS))[:, None] * 1.001
    norm = 0.5 * g * (c * c).sum(1)[None]
    true = off + norm - x @ (g * c).T
    err = EPS * (off + norm + np.abs(x) @ np.abs(g * c).T) + 2.0 ** -25
    nearest, rows = true.argmin(1), np.arange(len(x))
    assert (true - err > 0).all()
    computed = true - err
    computed[rows, nearest] = true[rows, nearest] + err[rows, nearest]
    best = computed.min(1)
    assert (computed[rows, nearest] <= best + NEAR * (x2 + best) + float(K_ABS)).all()
    best = true.min(1)
    near = (true <= (best + NEAR * (x2 + best) + float(K_ABS))[:, None]).sum(1)
    assert (near[:3000] > 1).mean() <= 0.05, (near > 1).mean()


@pytest.mark.gpu
@pytest.mark.parametrize("M,C,B_,n_new", [(64, 256, 1, 200), (32, 256, 3, 40), (32, 256, 4, 40), (32, 256, 2, 150),
                                            (32, 4096, 1, 100), (32, 4096, 1, 300)])
def test_codes_at_every_scale(M, C, B_, n_new):
    """Every subspace has its own scale, from subnormal codebooks to 30, tokens of the codebook's scale, far larger ones and
    zeros, an infinite centroid in a codebook of small and in one of large numbers.  (3 x 40 tokens are the few-token kernel's.)"""
    assert C == 4096 or takes_the_few_token_kernel(2, B_ * n_new, M) == ((B_, n_new) == (3, 40))
    ds = 128 // M
    w = W.Workload("scales", B_, 2, 2, 128, M, n_new, "f16", n_new=n_new, seed=9 + M + n_new, n_centroids=C)
    data = W.generate(w)
    rng = np.random.default_rng(M)
    scales = np.array([1e-7, 1e-6, 1e-5, 1e-4, 2.5e-4, 5e-4, 1e-3, 3e-3, 0.01, 0.03, 0.1, 0.3, 0.49, 0.51, 1, 2, 30], np.float32)
    for cb, x in ((data["k_codebook"], data["new_k"]), (data["v_codebook"], data["new_v"])):
        for i in range(M):
            s = scales[i % len(scales)]
            cb[:, i] = (cb[:, i].astype(np.float32) * s).astype(np.float16)
            part = x[..., i * ds:(i + 1) * ds].astype(np.float32) * s
            part[:, :, ::7] *= rng.choice([0, 50, 2000, 1e6])
            x[..., i * ds:(i + 1) * ds] = np.clip(part, -65504, 65504).astype(np.float16)
        cb[0, 6, 17, 0] = np.inf
        cb[0, 15, 3, 1] = -np.inf
        cb[1, 15, 5] = 65504
    with PQSession(data, 2, "f16") as s:
        s.ctx_len.zero_()
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got_k, got_v = s.unpack(PQ_CODES_K, n_new), s.unpack(PQ_CODES_V, n_new)
    np.testing.assert_array_equal(got_k, O.encode(data["new_k"], data["k_codebook"]))
    np.testing.assert_array_equal(got_v, O.encode(data["new_v"], data["v_codebook"]))


@pytest.mark.gpu
@pytest.mark.parametrize("C,M,scale", [(256, 64, 0.01), (256, 32, 1e-3), (4096, 32, 0.01)])
def test_training_at_small_scales(C, M, scale):
    d = W.training_samples(2, 4500, 128, M, seed=M + C, duplicate_init=3, n_centroids=C)
    small = lambda a: (a.astype(np.float32) * np.float32(scale)).astype(np.float16)
    samples, init = small(d["samples"]), small(d["init"])
    want, _ = K.kmeans_lloyd(samples, init, 2)
    ctx = make_ctx(2, M, n_centroids=C)
    try:
        got = gpu_fit(ctx, samples, init, 2)
    finally:
        P.pq_attn_destroy(ctx)
    assert (got.view(np.uint16) == want.view(np.uint16)).all()


def _encode_ms(M, C, scale):
    cfg = P.PQAttnConfig(batch=1, n_q_heads=8, n_kv_heads=8, n_subspaces=M, n_centroids=C, max_context=4096)
    ctx = P.pq_attn_create(cfg)
    gen = torch.Generator(device="cuda").manual_seed(M)
    normal = lambda *shape: (torch.randn(shape, generator=gen, device="cuda") * scale).half()
    P.pq_attn_set_codebooks(ctx, normal(8, M, C, 128 // M), normal(8, M, C, 128 // M))
    x = normal(2, 1, 8, 4096, 128)
    codes = torch.empty(2, P.pq_attn_codes_bytes(cfg), dtype=torch.uint8, device="cuda")
    n, best = torch.zeros(1, dtype=torch.int32, device="cuda"), float("inf")
    begin, end = torch.cuda.Event(True), torch.cuda.Event(True)
    for rep in range(5):
        begin.record()
        for _ in range(4):
            n.zero_()
            P.pq_encode_append(ctx, x[0], x[1], 4096, None, None, codes[0], codes[1], n)
        end.record()
        end.synchronize()
        best = min(best, begin.elapsed_time(end))
    P.pq_attn_destroy(ctx)
    return best


@pytest.mark.gpu
@pytest.mark.parametrize("M,C", [(64, 256), (32, 256), (32, 4096)])
def test_small_numbers_take_no_longer(M, C):
    """The same random numbers times 0.01 and 0.001; a quarter more is allowed, the runs differ by a few per cent."""
    unit = _encode_ms(M, C, 1.0)
    for scale in (0.01, 1e-3):
        assert _encode_ms(M, C, scale) <= 1.25 * unit, scale


@pytest.mark.gpu
def test_a_codebook_of_equal_centroids_takes_one_scan():
    """All numbers zero, so every centroid is as near as any: the scan of all costs 4.8 times a pass of the filter, a walk over
    all of its 64 quads 6.9 times."""
    assert _encode_ms(64, 256, 0.0) <= 5.8 * _encode_ms(64, 256, 1.0)


@pytest.mark.gpu
@pytest.mark.parametrize("M,dtype", [(64, "f16"), (32, "f16"), (64, "f32"), (32, "f32")])
def test_tokens_as_near_to_many_quads(M, dtype):
    """1 to 64 quads with the token's nearest centroid, several times inside some: an even and an odd number, 40 and 41, in one
    lane half or both; the lowest index of all is the code."""
    ds, n_new = 128 // M, 150
    assert not takes_the_few_token_kernel(2, n_new, M)
    w = W.Workload("quads", 1, 2, 2, 128, M, n_new, dtype, n_new=n_new, seed=M)
    data = W.generate(w)
    rng = np.random.default_rng(M)
    lowest = np.zeros((2, 2, M), int)
    for t, (cb, x) in enumerate(((data["k_codebook"], data["new_k"]), (data["v_codebook"], data["new_v"]))):
        for h in range(2):
            for i in range(M):
                n = [1, 2, 3, 4, 7, 16, 31, 32, 33, 39, 40, 41, 42, 63, 64][i % 15]
                quads = np.sort(rng.choice(64, n, False)) if i % 2 else np.sort(rng.permutation(np.r_[0:64:2, 1:64:2][:max(n, 32)])[:n])
                at = np.unique(4 * quads[:, None] + rng.integers(0, 4, (n, 2)))
                point = cb[h, i, at[0]].copy()
                cb[h, i, at] = point
                lowest[t, h, i] = at.min()
                x[0, h, ::2, i * ds:(i + 1) * ds] = point
    with PQSession(data, 2, dtype) as s:
        s.ctx_len.zero_()
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got = s.unpack(PQ_CODES_K, n_new), s.unpack(PQ_CODES_V, n_new)
    for t, (x, cb) in enumerate(((data["new_k"], data["k_codebook"]), (data["new_v"], data["v_codebook"]))):
        np.testing.assert_array_equal(got[t], O.encode(x, cb))
        assert (got[t][0, :, ::2] == lowest[t][:, None]).all()
