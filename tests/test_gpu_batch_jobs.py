"""Batches whose workgroups follow the sequences' lengths: fewer sequences than a head's share of the compute units (the
workgroups are dealt out by length), more (workgroups that walk several sequences, or one each, longest first).  Against the
oracle, and twice on one context (the tickets are back at zero)."""
import numpy as np
import pytest

from oracle import pq_oracle as O
from paper_2504_03661_amd.harness import PQSession
from synth import workloads as W

pytestmark = pytest.mark.gpu


def _lengths(kind, B, longest, rng):
    if kind == "equal":
        return [longest] * B
    if kind == "one long":                     # one long sequence, the others a token or none
        return [longest] + [b % 2 for b in range(1, B)]
    if kind == "powers":
        return [max(longest >> b, 0) for b in range(B)]
    return [int(v) for v in rng.integers(0, longest + 1, B)]


@pytest.mark.parametrize("M,dtype", [(64, "f16"), (32, "f16"), (64, "f32"), (32, "f32")])
@pytest.mark.parametrize("B,Hq,Hkv,longest", [(2, 2, 2, 3000), (3, 8, 2, 2500), (7, 16, 16, 700), (63, 4, 4, 1500), (64, 4, 4, 300),
                                              (5, 14, 2, 1200), (10, 32, 32, 400), (40, 32, 8, 260), (9, 32, 32, 130),
                                              (17, 32, 32, 200), (40, 20, 20, 90), (64, 32, 32, 70)])
@pytest.mark.parametrize("kind", ["equal", "one long", "powers", "random"])
def test_batches_of_any_lengths(M, dtype, B, Hq, Hkv, longest, kind):
    rng = np.random.default_rng(B + Hq + longest + M)
    lens = _lengths(kind, B, longest, rng)
    w = W.Workload("jobs", B, Hq, Hkv, 128, M, longest, dtype, recent_cap=40, recent_uniform=True, seed=B + Hq + M,
                   ctx_lens=tuple(lens))
    data = W.generate(w)
    scale = W.attention_scale(w)
    ref = O.decode(data["q"], data["k_codes"], data["v_codes"], data["ctx_len"], data["k_codebook"], data["v_codebook"],
                   data["recent_k"], data["recent_v"], data["recent_len"], scale=scale)
    with PQSession(data, Hq, dtype) as s:
        for call in range(2):
            s.out.fill_(float("nan"))
            out = s.decode(scale).cpu().numpy().astype(np.float64)
            err, norm = np.abs(out - ref).max(), np.linalg.norm(ref)
            # fp32 sums against double: 1e-6 relative, a few 1e-6 absolute on values of order one
            assert np.isfinite(out).all() and err <= 2e-5 and np.linalg.norm(out - ref) <= 1e-5 * norm, (call, err)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("B,Hq,Hkv", [(2, 1, 1), (3, 4, 1), (2, 2, 2)])
def test_a_sequence_takes_no_more_splits_than_a_merge_holds(B, Hq, Hkv, dtype):
    """More jobs per head (128, 256) than one sequence may have splits (64), and a sequence long enough to ask for more."""
    test_batches_of_any_lengths(64, dtype, B, Hq, Hkv, 40000, "one long")


@pytest.mark.parametrize("M,dtype,B,Hq,Hkv", [(64, "f32", 12, 28, 4), (64, "f32", 40, 8, 1), (64, "f32", 44, 8, 1), (32, "f16", 16, 20, 20),
                                              (32, "f32", 18, 20, 20), (64, "f16", 33, 32, 4), (64, "f16", 60, 12, 3), (64, "f32", 13, 20, 20)])
def test_one_workgroup_per_sequence_and_head_in_any_numbering(M, dtype, B, Hq, Hkv):
    """Heads whose sequences lie on 1, 2 or 8 XCDs, one, two, three and more workgroups per KV head and sequence, pair counts
    that 8 divides and does not."""
    for kind in ("random", "powers"):
        test_batches_of_any_lengths(M, dtype, B, Hq, Hkv, 150, kind)
