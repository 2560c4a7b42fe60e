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
from tests.test_encode_few import takes_the_few_token_kernel
from tests.test_filter_bound_cpu import K_ABS, X2F, _constant

NEAR, NEAR_F32 = float(_constant("PQ_FILTER_TAU_NEAR")), float(_constant("PQ_FILTER_TAU_NEAR_F32"))
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


@pytest.mark.parametrize("ds", [2, 4])
@pytest.mark.parametrize("c_scale,x_scale", [(1, 1), (1, 30), (1, 1e-4), (1e-12, 1e-12), (1e9, 1e8)])
def test_split_operands_never_hide_the_nearest_centroid(ds, c_scale, x_scale):
    """fp32 inputs: the filter's sums from split fp16 operands, as the kernel forms them, in fp32 arithmetic and with a
    further error of 16 x 2^-23 of the terms of either sign."""
    rng = np.random.default_rng(ds + abs(int(np.log10(c_scale) * 10)))
    c = (rng.standard_normal((256, ds)) * c_scale).astype(np.float32)
    c[128:] = (c[:128] * (1 + 10.0 ** rng.uniform(-7, -2, (128, ds)))).astype(np.float32)                  # close pairs
    x = (rng.standard_normal((2000, ds)) * x_scale).astype(np.float32)
    pair = rng.integers(0, 128, 1000)
    if c_scale == x_scale:
        x[:1000] = 0.5 * (c[pair] + c[pair + 128])
    scale = np.float32(2.0) ** (6 - np.frexp(np.abs(c).max())[1])
    assert 32 <= np.abs(c).max() * scale < 64
    cs, xs = c * scale, x * scale
    split = lambda v: (v.astype(np.float16), (v - v.astype(np.float16).astype(np.float32)).astype(np.float16))
    (c1, c2), (x1, x2) = split(cs), split(xs)
    half_norm = (np.float32(0.5) * (cs * cs).sum(1, dtype=np.float32)).astype(np.float32)
    h1, h2 = split(half_norm)
    length2 = (xs * xs).sum(1, dtype=np.float32)
    off = (X2F * length2 + 3 * K_ABS).astype(np.float64)[:, None] * 1.001
    d = lambda v: v.astype(np.float64)
    terms = np.concatenate([np.broadcast_to(off[:, :, None], (len(x), 256, 1)),
                            np.broadcast_to(d(h1)[None, :, None], (len(x), 256, 1)),
                            np.broadcast_to(d(h2)[None, :, None], (len(x), 256, 1)),
                            -d(x1)[:, None] * d(c1)[None], -d(x1)[:, None] * d(c2)[None], -d(x2)[:, None] * d(c1)[None]], axis=2)
    computed, slack = terms.sum(2), 16 * 2.0 ** -23 * np.abs(terms).sum(2)
    nearest = ((d(x)[:, None] - d(c)[None]) ** 2).sum(2).argmin(1)
    rows = np.arange(len(x))
    low = computed - slack
    assert (low > 0).all()
    low[rows, nearest] = computed[rows, nearest] + slack[rows, nearest]
    best = low.min(1)
    tau = NEAR_F32 * (length2 + best) + float(K_ABS)
    assert (low[rows, nearest] <= best + tau).all()


@pytest.mark.gpu
@pytest.mark.parametrize("M", [64, 32])
def test_fp32_codes_over_magnitudes_and_near_ties(M):
    """fp32 contexts: codebooks from 1e-30 to 1e15, all zero, with outliers, with pairs of centroids a few fp32 steps
    apart and tokens on their midpoints, tokens far longer than the codebook."""
    ds, n_new = 128 // M, 300
    w = W.Workload("f32", 2, 4, 2, 128, M, n_new, "f32", n_new=n_new, seed=5 + M)
    data = W.generate(w)
    rng = np.random.default_rng(M)
    for cb in (data["k_codebook"], data["v_codebook"]):
        for i, s in enumerate((1e-30, 1e-12, 1e-4, 300.0, 1e15)):
            cb[:, i] *= np.float32(s)
        cb[:, 5] = 0
        cb[:, 6, ::40] *= np.float32(1000.0)
        cb[:, 7, 128:] = cb[:, 7, :128] * (1 + rng.integers(-4, 5, cb[:, 7, :128].shape) * np.float32(2.0) ** -23)
        cb[:, 8, 255] = cb[:, 8, 3]
        cb[:, 10] *= np.float32(1e-39)                                          # subnormal fp32
    for x in (data["new_k"], data["new_v"]):
        for i, s in enumerate((1e-30, 1e-12, 1e-4, 300.0, 1e15)):
            x[..., i * ds:(i + 1) * ds] *= np.float32(s)
        pair = rng.integers(0, 128, x.shape[:3])
        cb7 = data["k_codebook"][:, 7]
        hk = np.arange(x.shape[1])[None, :, None]
        x[..., 7 * ds:8 * ds] = 0.5 * (cb7[hk, pair] + cb7[hk, pair + 128])
        x[..., 8 * ds:9 * ds] = data["k_codebook"][:, 8, 3][None, :, None]
        x[:, :, ::50, 9 * ds:10 * ds] *= np.float32(1e6)
    with PQSession(data, 4, "f32") as s:
        s.ctx_len.zero_()
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got_k, got_v = s.unpack(PQ_CODES_K, n_new), s.unpack(PQ_CODES_V, n_new)
    exp_k = O.encode(data["new_k"], data["k_codebook"])
    assert (exp_k[..., 5] == 0).all() and (exp_k[..., 8] == 3).all()
    np.testing.assert_array_equal(got_k, exp_k)
    np.testing.assert_array_equal(got_v, O.encode(data["new_v"], data["v_codebook"]))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("M", [64, 32])
@pytest.mark.parametrize("B_,n_new", [(3, 56), (3, 57), (2, 63), (2, 64), (2, 65), (3, 113), (3, 114), (1, 70), (40, 7),
                                      (1, 6), (6, 1), (1, 7), (7, 1), (2, 3), (4, 2), (1, 56), (2, 28), (1, 57), (3, 19), (1, 72),
                                      (8, 9), (1, 73), (73, 1)])
def test_codes_at_the_edges_of_the_mapping_and_of_the_offset(M, B_, n_new, dtype):
    """Token counts on both sides of the rule that gives every sequence its own 64-token chunks (57 and 114 are the first
    to have them) and of the one between the few-token kernel and the filter (4 heads: up to 56 tokens per head at M = 64, 72 at
    M = 32), remainders; sub-vectors up to the largest fp16 (beyond a length of 345 the offset moves to its second slot, beyond 6e4 the chunk
    takes the full scan)."""
    assert takes_the_few_token_kernel(4, B_ * n_new, M) == (B_ * n_new <= (56 if M == 64 else 72))
    ds = 128 // M
    lens = tuple(int(v) for v in np.random.default_rng(B_).integers(0, 90, B_))
    w = W.Workload("edge", B_, 4, 4, 128, M, 90 + n_new, dtype, n_new=n_new, seed=70 + M + n_new, ctx_lens=lens)
    data = W.generate(w, ctx_cap=90 + n_new)
    for x in (data["new_k"], data["new_v"]):
        x[:, :, ::3, :ds] = x.dtype.type(340.0) * np.sign(x[:, :, ::3, :ds])
        x[:, :, ::4, ds:2 * ds] *= x.dtype.type(900.0)
        x[:, :, ::5, 2 * ds:3 * ds] = 65504.0
        x[:, :, 1::5, 2 * ds:3 * ds] = -30000.0
        x[:, :, ::2, 3 * ds:4 * ds] = 0
    with PQSession(data, 4, dtype, max_context=90 + n_new) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        assert s.ctx_len.cpu().tolist() == [n + n_new for n in lens]
        got_k, got_v = s.unpack(PQ_CODES_K, 90 + n_new), s.unpack(PQ_CODES_V, 90 + n_new)
    exp_k, exp_v = O.encode(data["new_k"], data["k_codebook"]), O.encode(data["new_v"], data["v_codebook"])
    for b, n in enumerate(lens):
        np.testing.assert_array_equal(got_k[b, :, n:n + n_new], exp_k[b])
        np.testing.assert_array_equal(got_v[b, :, n:n + n_new], exp_v[b])
        np.testing.assert_array_equal(got_k[b, :, :n], data["k_codes"][b, :, :n])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("M,B_,Hkv,n_new,per_seq", [(64, 64, 32, 5, False), (64, 40, 32, 70, False), (32, 70, 32, 11, False),
                                                    (32, 130, 16, 37, False), (64, 1, 16, 1100, True), (64, 5, 32, 127, True),
                                                    (32, 2, 32, 600, True)])
def test_codes_with_several_chunks_per_wavefront(M, B_, Hkv, n_new, per_seq, dtype):
    """Enough 64-token chunks that a wavefront takes two or more in a row: the step from one to the next, where the tokens of
    all sequences are in a row (several sequences or none passed on the way) and where every sequence has its own chunks."""
    seq_chunks = (n_new + 63) // 64
    assert per_seq == (seq_chunks * 512 <= n_new * 9 or B_ == 1)                # the launcher's rule, and ...
    chunks = B_ * seq_chunks if per_seq else (B_ * n_new + 63) // 64
    assert Hkv * chunks * M * 2 // 8192 >= 2                                    # ... its chunks per wavefront
    lens = tuple(int(v) for v in np.random.default_rng(B_).integers(0, 20, B_))
    w = W.Workload("rounds", B_, Hkv, Hkv, 128, M, 20 + n_new, dtype, n_new=n_new, seed=M + n_new, ctx_lens=lens)
    data = W.generate(w, ctx_cap=20 + n_new)
    with PQSession(data, Hkv, dtype, max_context=20 + n_new) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        assert s.ctx_len.cpu().tolist() == [n + n_new for n in lens]
        got_k, got_v = s.unpack(PQ_CODES_K, 20 + n_new), s.unpack(PQ_CODES_V, 20 + n_new)
    exp_k, exp_v = O.encode(data["new_k"], data["k_codebook"]), O.encode(data["new_v"], data["v_codebook"])
    for b, n in enumerate(lens):
        np.testing.assert_array_equal(got_k[b, :, n:n + n_new], exp_k[b])
        np.testing.assert_array_equal(got_v[b, :, n:n + n_new], exp_v[b])
        np.testing.assert_array_equal(got_k[b, :, :n], data["k_codes"][b, :, :n])
