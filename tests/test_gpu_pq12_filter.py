"""12-bit encode through the matrix-core filter: token counts at the edges of its paths (8 / 9 tokens per head: per-token
kernel / split; 64 / 65; 128 / 129: split / unsplit; several chunks per wavefront), with ties inside a block of 16, across
the interleaved blocks of the two lane halves and across rows and columns of blocks, near-ties, a codebook of norms
beyond fp16, subnormals, and tokens up to the largest fp16."""
import numpy as np
import pytest
import torch

from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,n_new", [(1, 2, 4), (5, 2, 1), (1, 3, 1), (4, 2, 2), (9, 2, 1), (1, 2, 64), (5, 1, 13), (2, 1, 64), (1, 1, 129), (3, 2, 171),
                                         (1, 8, 1700)])
def test_codes_of_every_path_are_the_oracles(B, Hkv, n_new):
    rng = np.random.default_rng(B + n_new)
    lens = tuple(int(v) for v in rng.integers(0, 200, B))
    w = W.Workload("f12", B, Hkv, Hkv, 128, 32, 200 + n_new, "f16", n_new=n_new, seed=31 + n_new, ctx_lens=lens, n_centroids=4096)
    data = W.generate(w, ctx_cap=200 + n_new)
    for cb in (data["k_codebook"], data["v_codebook"]):
        cb[:, 0, [5, 7]] = cb[:, 0, 6][:, None]                     # a tie inside a quad
        cb[:, 1, [100, 104]] = cb[:, 1, 99][:, None]                # quads of both lane halves, one instruction
        cb[:, 2, [40, 300, 4000, 2050, 2055]] = cb[:, 2, 3][:, None]   # several rows and columns of blocks
        base = cb[:, 3, 0].astype(np.float32)                       # 4096 near-ties, a few fp16 steps apart
        steps = rng.integers(-3, 4, size=(cb.shape[0], 4096, 4)).astype(np.float32)
        cb[:, 3] = (base[:, None] + steps * np.abs(np.spacing(base.astype(np.float16)))[:, None].astype(np.float32)).astype(np.float16)
        cb[:, 4] = (cb[:, 4].astype(np.float32) * 1e-6).astype(np.float16)
        cb[:, 5] = (cb[:, 5].astype(np.float32) * 150.0).astype(np.float16)
        d = rng.standard_normal((cb.shape[0], 2048, 4)).astype(np.float32) * 0.01
        cb[:, 6, 2048:] = (cb[:, 6, :2048].astype(np.float32) + d).astype(np.float16)
    for x in (data["new_k"], data["new_v"]):
        for i, c in ((0, 6), (1, 104), (2, 4000), (3, 0)):
            x[..., 4 * i:4 * i + 4] = data["k_codebook"][:, i, c][None, :, None, :]
        x[..., 16:20] = (x[..., 16:20].astype(np.float32) * 1e-6).astype(np.float16)
        pair = rng.integers(0, 2048, size=x.shape[:3])
        cb6 = data["k_codebook"][:, 6].astype(np.float32)
        hk = np.arange(x.shape[1])[None, :, None]
        x[..., 24:28] = (0.5 * (cb6[hk, pair] + cb6[hk, pair + 2048])).astype(np.float16)
        x[:, :, ::3, 28:32] *= np.float16(300.0)
        x[:, :, ::7, 32:36] = 65504.0
    with PQSession(data, Hkv, "f16", max_context=200 + n_new) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        assert s.ctx_len.cpu().tolist() == [n + n_new for n in lens]
        got_k, got_v = s.unpack(PQ_CODES_K, 200 + n_new), s.unpack(PQ_CODES_V, 200 + n_new)
    exp_k, exp_v = O.encode(data["new_k"], data["k_codebook"]), O.encode(data["new_v"], data["v_codebook"])
    assert (exp_k[..., 0] == 5).all() and (exp_k[..., 1] == 99).all() and (exp_k[..., 2] == 3).all()
    for b, n in enumerate(lens):
        np.testing.assert_array_equal(got_k[b, :, n:n + n_new], exp_k[b])
        np.testing.assert_array_equal(got_v[b, :, n:n + n_new], exp_v[b])
        np.testing.assert_array_equal(got_k[b, :, :n], data["k_codes"][b, :, :n])


@pytest.mark.parametrize("n_new", [1, 5, 8, 9])
def test_tokens_and_centroids_that_are_not_finite(n_new):
    """The lowest index among the least distances, infinite ones and NaN never below another: code 0 if there is none."""
    w = W.Workload("f12n", 1, 2, 2, 128, 32, 64, "f16", n_new=n_new, seed=n_new, ctx_lens=(9,), n_centroids=4096)
    data = W.generate(w, ctx_cap=64)
    for cb in (data["k_codebook"], data["v_codebook"]):
        cb[:, 0, 1:3000] = np.nan
        cb[:, 1, 1::2, 1] = np.inf
        cb[:, 2] = -np.inf
        cb[:, 3, 4095] = np.nan
    for x in (data["new_k"], data["new_v"]):
        x[..., 16:20] = np.nan
        x[..., 20] = -np.inf
    with PQSession(data, 2, "f16", max_context=64) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got_k, got_v = s.unpack(PQ_CODES_K, 64), s.unpack(PQ_CODES_V, 64)
    exp_k, exp_v = O.encode(data["new_k"], data["k_codebook"]), O.encode(data["new_v"], data["v_codebook"])
    assert (exp_k[..., 2] == 0).all() and (exp_k[..., 4] == 0).all()
    np.testing.assert_array_equal(got_k[0, :, 9:9 + n_new], exp_k[0])
    np.testing.assert_array_equal(got_v[0, :, 9:9 + n_new], exp_v[0])
