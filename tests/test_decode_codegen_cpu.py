"""What the compiler makes of the 8-bit decode kernels, cross-compiled to gfx950 assembly (no GPU needed): the kernels whose
workgroups take whole sequences exchange nothing, and the kernels that choose a sequence by the lengths keep as much in
registers as the one that does not."""
import re

import pytest

from tests.test_exchange_codegen_cpu import assembly, kernels


@pytest.fixture(scope="module", params=["pq_decode.hip", "pq_decode_grouped.hip"])
def listing(request, tmp_path_factory):
    return assembly(request.param, tmp_path_factory.mktemp("asm"))


def test_kernels_of_whole_sequences_exchange_nothing(listing):
    whole = {k: v for k, v in kernels(listing).items() if "whole_kernel" in k}
    assert whole
    for name, body in whole.items():
        assert not re.search(r"\bglobal_atomic|\bsc1\b", body), name


def test_no_kernel_keeps_what_it_should_work_out_again(listing):
    """Registers spilled, of 128 per lane in the kernels of 16 wavefronts: 21 to 23 where the addresses of the fp32 codebook
    images stayed alive through the scan."""
    spills = dict(re.findall(r"\.name:\s+(\S+)\s.*?\.vgpr_spill_count:\s+(\d+)", listing, re.S))
    spills = {k: int(v) for k, v in spills.items() if "pq_decode" in k}
    assert len(spills) >= 8
    assert max(spills.values()) <= 8, spills
