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


def _ratio(B, Hq, Hkv, lengths, M=64, dtype=torch.float16, recent=0, layers=4):
    """Time of a decode at the library's own choice over that of the same call with the reported splits asked for; each
    side has `layers` contexts that take turns, as a model's layers do, with codebooks and codes of their own."""
    gen = torch.Generator(device="cuda").manual_seed(B + Hq + M)
    cfg = P.PQAttnConfig(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, n_subspaces=M, max_context=max(lengths), max_recent=recent,
                         dtype=P.PQ_F16 if dtype == torch.float16 else P.PQ_F32)
    sides = [[P.pq_attn_create(cfg) for _ in range(layers)]]
    cfg.n_splits = P.pq_attn_n_splits(sides[0][0])
    sides.append([P.pq_attn_create(cfg) for _ in range(layers)])
    normal = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)
    codes = torch.randint(0, 256, (layers, 2, P.pq_attn_codes_bytes(cfg)), generator=gen, device="cuda", dtype=torch.uint8)
    q, out = normal(B, Hq, 128), torch.empty(B, Hq, 128, device="cuda")
    n = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    rows = [None] * 3 if recent == 0 else [normal(B, Hkv, recent, 128), normal(B, Hkv, recent, 128), torch.full_like(n, recent)]
    for side in sides:
        for c in side:
            P.pq_attn_set_codebooks(c, normal(Hkv, M, 256, 128 // M), normal(Hkv, M, 256, 128 // M))
    best = [float("inf")] * 2
    begin, end = torch.cuda.Event(True), torch.cuda.Event(True)
    for rep in range(8):                                    # in turn; the first round warms up
        for k, side in enumerate(sides):
            begin.record()
            for i in range(60):
                j = i % layers
                P.pq_attn_decode(side[j], q, codes[j][0], codes[j][1], n, None, None, *rows, 0.088, out)
            end.record()
            end.synchronize()
            if rep:
                best[k] = min(best[k], begin.elapsed_time(end))
    for side in sides:
        for c in side:
            P.pq_attn_destroy(c)
    return best[0] / best[1]


# the two sides do the same work, so what is allowed is a tenth to a quarter of the time: the runs of one side differ by a few per cent

@pytest.mark.parametrize("B,Hq,Hkv", [(63, 1, 1), (24, 1, 1), (48, 2, 2), (48, 8, 1), (30, 8, 2)])
def test_few_heads_have_the_whole_chip(B, Hq, Hkv):
    """Batches of few heads: the workgroups of a head are its share of the compute units, however many that are."""
    assert _ratio(B, Hq, Hkv, [8192] * B) <= 1.25


def test_workgroups_that_share_codes_are_neighbours():
    """More query heads per KV head than one workgroup takes: those of the same job read the same codes out of one L2."""
    assert _ratio(31, 8, 1, [4096] * 31, dtype=torch.float32) <= 1.25


@pytest.mark.parametrize("B", [2, 3])
def test_a_heads_workgroups_share_an_xcd_in_any_grid(B):
    """28 heads have 9 workgroups each: 252 of them, which 8 does not divide."""
    assert _ratio(B, 28, 28, [200] * B) <= 1.25


def _spread(lo, hi, n):
    return [lo + (hi - lo) * (7 * k % n) // (n - 1) for k in range(n)]


@pytest.mark.parametrize("B,Hq,Hkv", [(40, 8, 1), (12, 28, 4)])
def test_the_long_sequences_of_a_batch_are_spread_over_the_xcds(B, Hq, Hkv):
    """A KV head whose sequences lie on several XCDs, one workgroup each, longest first."""
    assert _ratio(B, Hq, Hkv, _spread(1000, 10000, B), dtype=torch.float32) <= 1.1


@pytest.mark.parametrize("B,Hq,Hkv,lo,hi", [(5, 32, 8, 30, 200), (63, 8, 1, 60, 60), (2, 4, 4, 500, 16000), (63, 4, 4, 1000, 1000)])
def test_dealing_costs_little_where_it_gains_little(B, Hq, Hkv, lo, hi):
    """Short sequences keep one workgroup, a long one gets no more splits than its merge is worth, equal lengths are cut
    without a search."""
    assert _ratio(B, Hq, Hkv, _spread(lo, hi, B)) <= 1.15


@pytest.mark.parametrize("B,Hq,Hkv,M", [(63, 32, 8, 64), (15, 32, 32, 32)])
def test_short_sequences_are_not_ranked(B, Hq, Hkv, M):
    assert _ratio(B, Hq, Hkv, _spread(30, 200, B), M=M) <= 1.1
