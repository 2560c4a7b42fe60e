"""What the library's own choice for a batch costs: memory of a context, and time against the same call with the splits
asked for that the context reports."""
import pytest
import torch

import paper_2504_03661_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv", [(63, 4, 4), (31, 8, 8), (60, 16, 4)])
def test_contexts_of_a_batch_hold_one_partial_per_head_and_job(B, Hq, Hkv):
    """A row's partials of 528 bytes for 64 (32, 64) jobs per head, not for every sequence and job: 8 contexts take a few
    MiB (codebooks, rounded-up small allocations) instead of 68, 34 and 259."""
    cfg = P.PQAttnConfig(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, max_context=64)
    P.pq_attn_destroy(P.pq_attn_create(cfg))        # the process's first context loads the code objects: not counted
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    contexts = [P.pq_attn_create(cfg) for _ in range(8)]
    used = before - torch.cuda.mem_get_info()[0]
    for c in contexts:
        P.pq_attn_destroy(c)
    codebooks = 8 * 4 * Hkv * 256 * 128 * 2
    assert used <= codebooks + (16 << 20), used
