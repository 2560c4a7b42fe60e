"""Long appends of many heads store the codes of a chunk together: every byte of the code tensors against the same tokens appended in
pieces that store them one by one, and two heads' codes against the oracle."""
import numpy as np
import pytest
import torch

from oracle import pq_oracle as O
from paper_2504_03661_amd import PQ_CODES_K, PQ_CODES_V
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W

pytestmark = pytest.mark.gpu


# chunks that are not full at both ends; tokens beyond the capacity; the skew of K by lanes (16 query heads) and by quads (64)
@pytest.mark.parametrize("Hq,start,n_new,room", [(16, 0, 16384, 16384), (16, 37, 16421, 16453), (64, 63, 16450, 16600)])
def test_wide_codes_equal_single_ones(Hq, start, n_new, room):
    assert 2 * 16 * 16 >= 2 * torch.cuda.get_device_properties(0).multi_processor_count and (n_new + 126) >> 6 >= 256
    data = W.generate(W.Workload("wide", 1, Hq, 16, 128, 64, 64, "f16", n_new=8, seed=n_new))
    data["ctx_len"] = np.asarray([start], np.int32)
    data["v_codebook"][3, 20, :, 1] = 0.5                    # no useful grid
    data["k_codebook"][9, 40:44, 1:] = data["k_codebook"][9, 40:44, :1]
    g = torch.Generator(device="cuda").manual_seed(n_new)
    new = []
    for book in ("k_codebook", "v_codebook"):
        spread = torch.from_numpy(data[book].astype(np.float32).std(axis=2).reshape(16, 1, 128)).cuda()
        x = torch.randn((1, 16, n_new, 128), generator=g, device="cuda") * spread
        x *= 1 + 4 * (torch.rand(x.shape, generator=g, device="cuda") < 0.02)   # (some outside the grids)
        new.append(x.half())
    with PQSession(data, Hq, "f16", max_context=room) as s:
        codes = s.k_codes[0], s.v_codes[0]

        def appended(step):
            s.ctx_len.fill_(start)
            for t in codes:
                t.fill_(0xa5)
            for t0 in range(0, n_new, step):
                s.append(*(x[:, :, t0:t0 + step].contiguous() for x in new))
            assert s.ctx_len.tolist() == [min(room, start + n_new)]
            return [t.clone() for t in codes]

        single = appended(2047)
        for _ in range(3):                                   # (the first may build its grids)
            for got, ref in zip(appended(n_new), single):
                assert torch.equal(got, ref)
        n = min(room, start + n_new) - start
        for kind, book, x in zip((PQ_CODES_K, PQ_CODES_V), ("k_codebook", "v_codebook"), new):
            got = s.unpack(kind, room)[:, [3, 9], start:start + n]
            ref = O.encode(x[:, [3, 9], :n].cpu().numpy(), data[book][[3, 9]])
            np.testing.assert_array_equal(got, ref)
