"""Appends of a few tokens per KV head (one wavefront per subspace and group of tokens): the launcher's rule, compiled from
its source, and the codes against the oracle, exact, where fp32 distances decide and where they do not."""
import ctypes
import functools
import os
import re
import subprocess
import tempfile

import numpy as np
import pytest
import torch

from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V
from paper_2504_03661_amd import build as lib_build
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W


@functools.cache
def _per_wave():
    text = open(os.path.join(lib_build.CSRC, "pq_encode.hip")).read()
    text = re.search(r"^inline int pq_encode_few_per_wave\(.*?^}", text, re.S | re.M).group(0)
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "rule.cpp"), "w") as f:
            f.write("#include <cstdint>\n" + text + '\nextern "C" int rule(int64_t t, int64_t r, int M) { return pq_encode_few_per_wave(t, r, M); }\n')
        lib = os.path.join(d, "rule.so")
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", lib, f.name], check=True)
        fn = ctypes.CDLL(lib).rule
    fn.argtypes, fn.restype = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int], ctypes.c_int
    return fn


def takes_the_few_token_kernel(Hkv, tokens, M):
    """Whether the launcher gives an append of so many tokens per head (of all sequences) to the few-token kernel: the other tests
    of the filter ask, so that their sizes reach it."""
    return _per_wave()(tokens, Hkv * M * 2, M) > 0


@pytest.fixture
def per_wave():
    return _per_wave()


@pytest.mark.parametrize("M", [32, 64])
@pytest.mark.parametrize("heads", [1, 2, 4, 5, 8, 28, 32, 64, 128, 1000, 100000])
def test_groups_cover_the_tokens_and_a_wavefront_has_at_most_64(per_wave, heads, M):
    rows = heads * M * 2
    took = [per_wave(t, rows, M) for t in range(1, 3000)]
    few = sum(n > 0 for n in took)
    assert few >= 6 and all(n > 0 for n in took[:few]) and not any(took[few:])     # one line between the two kernels
    for t, n in zip(range(1, few + 1), took):
        groups = -(-t // n)
        assert 1 <= n <= 64 and (groups - 1) * n < t and groups * 2 < 65536


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("M,B_,Hkv,n_new,share", [(64, 1, 32, 1, 1), (64, 13, 32, 1, 7), (64, 2, 32, 7, 7), (64, 3, 2, 31, 4),
                                                  (64, 1, 1, 70, 2), (32, 5, 32, 3, 5), (32, 16, 32, 1, 6), (32, 2, 4, 33, 3),
                                                  (32, 70, 4, 1, 3)])
def test_codes_of_few_tokens(per_wave, M, B_, Hkv, n_new, share, dtype):
    """One token, a last group with fewer tokens than the others, groups that begin inside a sequence, the largest appends
    of the kernel.  Subspaces with equal centroids in one lane's four and in others', near-ties, coordinates whose squares
    underflow (fp32) or are subnormal (fp16), tokens on centroids and far outside."""
    assert per_wave(B_ * n_new, Hkv * M * 2, M) == share
    ds = 128 // M
    lens = tuple(int(v) for v in np.random.default_rng(B_).integers(0, 90, B_))
    cap = 88 + n_new                                                            # (some tokens are beyond it)
    w = W.Workload("few", B_, Hkv, Hkv, 128, M, cap, dtype, n_new=n_new, seed=M + n_new, ctx_lens=tuple(min(n, cap) for n in lens))
    data = W.generate(w, ctx_cap=cap)
    rng = np.random.default_rng(M + n_new)
    tiny = 1e-38 if dtype == "f32" else 1e-6
    for cb in (data["k_codebook"], data["v_codebook"]):
        cb[:, 0, 1] = cb[:, 0, 0]                                               # equal: neighbours, and in two lanes
        cb[:, 1, 130] = cb[:, 1, 7]
        cb[:, 2] = cb[:, 2, :1]                                                 # all equal
        cb[:, 3, 128:] = (cb[:, 3, :128].astype(np.float32) * (1 + rng.integers(-4, 5, cb[:, 3, :128].shape) *
                                                               np.float32(2.0) ** -23)).astype(cb.dtype)
        cb[:, 4] = (cb[:, 4].astype(np.float64) * tiny).astype(cb.dtype)
    for x, cb in ((data["new_k"], data["k_codebook"]), (data["new_v"], data["v_codebook"])):
        hk = np.arange(Hkv)[None, :, None]
        pick = rng.integers(0, 128, x.shape[:3])
        x[..., :ds] = cb[:, 0, 1][None, :, None]
        x[..., ds:2 * ds] = cb[:, 1, 7][None, :, None]
        x[..., 3 * ds:4 * ds] = (0.5 * (cb[hk, 3, pick].astype(np.float32) + cb[hk, 3, pick + 128].astype(np.float32))).astype(x.dtype)
        x[..., 4 * ds:5 * ds] = (x[..., 4 * ds:5 * ds].astype(np.float64) * tiny).astype(x.dtype)
        x[..., 5 * ds:6 * ds] = cb[hk, 5, pick]
        x[:, :, ::2, 6 * ds:7 * ds] = 60000.0
    with PQSession(data, Hkv, dtype, max_context=cap) as s:
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        assert s.ctx_len.cpu().tolist() == [min(n + n_new, cap) for n in w.ctx_lens]
        got = s.unpack(PQ_CODES_K, cap), s.unpack(PQ_CODES_V, cap)
    for codes, old, x, cb in ((got[0], data["k_codes"], data["new_k"], data["k_codebook"]),
                              (got[1], data["v_codes"], data["new_v"], data["v_codebook"])):
        want = O.encode(x, cb)
        assert (want[..., 0] == 0).all() and (want[..., 1] == 7).all() and (want[..., 2] == 0).all()
        for b, n in enumerate(w.ctx_lens):
            np.testing.assert_array_equal(codes[b, :, n:n + n_new], want[b, :, :cap - n])
            np.testing.assert_array_equal(codes[b, :, :n], old[b, :, :n])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("M,B_,n_new,few", [(64, 1, 1, True), (64, 3, 5, True), (32, 2, 7, True), (64, 3, 300, False), (32, 3, 300, False)])
def test_codes_of_infinities_and_nans(per_wave, M, B_, n_new, few, dtype):
    """No distance of such a token is below infinity, so its code is 0, also where a single one is not NaN; and centroids at
    infinity are never a finite token's.  The filter of longer appends on the same data."""
    assert (per_wave(B_ * n_new, 2 * M * 2, M) > 0) == few
    ds = 128 // M
    w = W.Workload("not finite", B_, 2, 2, 128, M, n_new, dtype, n_new=n_new, seed=M + n_new)
    data = W.generate(w)
    for cb, x in ((data["k_codebook"], data["new_k"]), (data["v_codebook"], data["new_v"])):
        cb[:, 0, :, 0] = np.inf
        cb[:, 0, 37, 0] = 0.5                              # infinite tokens: infinitely far, NaN to all others
        cb[:, 1, ::3, 1] = -np.inf
        cb[:, 2, 5:, ds - 1] = np.inf
        for i, v in ((0, np.inf), (1, -np.inf), (2, np.inf), (3, np.inf), (4, -np.inf), (5, np.nan)):
            x[:, :, ::2, i * ds + (ds - 1 if i == 2 else i & 1)] = v
        x[:, :, ::2, 6 * ds:7 * ds] = np.inf
    with PQSession(data, 2, dtype) as s:
        s.ctx_len.zero_()
        s.append(torch.from_numpy(data["new_k"]).cuda(), torch.from_numpy(data["new_v"]).cuda())
        torch.cuda.synchronize()
        got = s.unpack(PQ_CODES_K, n_new), s.unpack(PQ_CODES_V, n_new)
    for codes, x, cb in ((got[0], data["new_k"], data["k_codebook"]), (got[1], data["new_v"], data["v_codebook"])):
        want = O.encode(x, cb)
        assert (want[:, :, ::2, :7] == 0).all()
        np.testing.assert_array_equal(codes, want)
