"""Contexts keep the grids of their codebooks once their appends have paid for them: codes against the oracle for repeated
appends, codebooks registered again in between and handed to the call, and replays of a graph between them."""
import numpy as np
import pytest
import torch

from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V, pq_attn_set_codebooks
from paper_2504_03661_amd.harness import PQSession
from tests.test_nearest_grid import _data, _n_cu, _rule, encode_slices

pytestmark = pytest.mark.gpu


def _appended(s, n_new, **kw):
    """the codes of an append of the new rows at position 0"""
    for t in (s.ctx_len, s.k_codes[0], s.v_codes[0]):
        t.zero_()
    s.append(s.new[0], s.new[1], **kw)
    return s.unpack(PQ_CODES_K, n_new), s.unpack(PQ_CODES_V, n_new)


@pytest.mark.parametrize("dtype,B_,n_new", [(np.float16, 2, 34007), (np.float32, 2, 34007), (np.float16, 1, 9003)])
def test_appends_with_kept_grids_equal_the_oracle(dtype, B_, n_new):
    """One append of 2 x 34007 tokens pays for the grids, it takes several of 9003, which go through the filter until then."""
    first = next(n for n in range(1, 100) if _rule()(*[n * (B_ * n_new + 63) // 64] * 2, 64, _n_cu()) > 0)
    assert (first == 1) == (encode_slices(2, B_, n_new, _n_cu()) > 0) == (n_new > 10000)
    kind = "f16" if dtype == np.float16 else "f32"
    data = _data(2, 2, B_, n_new, dtype, [0] * B_)              # (codebooks of all kinds, some without a useful grid)
    want = {books: [O.encode(data["new_" + n], data[m + "_codebook"]) for n, m in zip("kv", books)] for books in ("kv", "vk")}
    with PQSession(data, 2, kind, max_context=n_new) as s:
        s.new = [torch.from_numpy(data["new_" + n]).cuda() for n in "kv"]

        def check(books, **kw):
            for got, ref in zip(_appended(s, n_new, **kw), want[books]):
                np.testing.assert_array_equal(got, ref)

        for _ in range(first + 2):
            check("kv")
        pq_attn_set_codebooks(s.ctx, s.v_codebook, s.k_codebook)
        for _ in range(first + 1):
            check("vk")
        check("kv", pass_codebooks=True)                        # none are kept of these
        check("kv")
        pq_attn_set_codebooks(s.ctx, s.v_codebook, s.k_codebook)
        check("vk")


def test_a_recorded_append_follows_the_registration_in_force():
    n_new = 34007
    data = _data(2, 2, 2, n_new, np.float16, [0, 0])
    want = {books: [O.encode(data["new_" + n], data[m + "_codebook"]) for n, m in zip("kv", books)] for books in ("kv", "vk")}
    with PQSession(data, 2, "f16", max_context=n_new) as s:
        s.new = [torch.from_numpy(data["new_" + n]).cuda() for n in "kv"]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        _appended(s, n_new)                                     # (pays for the grids)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            s.ctx_len.zero_()
            s.append(s.new[0], s.new[1])
        for rep, books in enumerate(("kv", "kv", "vk", "kv", "kv")):
            for t in (s.k_codes[0], s.v_codes[0]):              # eager work between the replays
                t.fill_(255)
            g.replay()
            torch.cuda.synchronize()
            for kind, ref in zip((PQ_CODES_K, PQ_CODES_V), want[books]):
                np.testing.assert_array_equal(s.unpack(kind, n_new), ref)
            if books == "vk":                                   # back, by a call that builds no grids
                _appended(s, n_new, pass_codebooks=True)
            elif rep == 1:
                pq_attn_set_codebooks(s.ctx, s.v_codebook, s.k_codebook)
