"""How many 64-token chunks a wavefront of the encode's filter kernel takes in a row: the launcher's rule, compiled from its
source.  The workgroups of a head go to the XCDs in turn, so a head's wavefronts have to get about the same number."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2504_03661_amd import build as lib_build


@pytest.fixture(scope="module")
def rounds(tmp_path_factory):
    text = open(os.path.join(lib_build.CSRC, "pq_encode.hip")).read()
    text = re.search(r"^inline int64_t pq_encode_rounds\(.*?^}", text, re.S | re.M).group(0)
    d = tmp_path_factory.mktemp("rounds")
    (d / "rule.cpp").write_text("#include <cstdint>\n" + text +
                                '\nextern "C" int64_t rule(int64_t c, int64_t r) { return pq_encode_rounds(c, r); }\n')
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(d / "rule.so"), str(d / "rule.cpp")], check=True)
    fn = ctypes.CDLL(str(d / "rule.so")).rule
    fn.argtypes, fn.restype = [ctypes.c_int64] * 2, ctypes.c_int64
    return fn


@pytest.mark.parametrize("M", [32, 64])
@pytest.mark.parametrize("heads", [1, 2, 3, 4, 5, 8, 16, 28, 32, 40, 64])
def test_wavefronts_of_a_head_take_about_the_same_number_of_chunks(rounds, heads, M):
    rows = heads * M * 2
    for n in range(1, 4000):
        r = rounds(n, rows)
        jobs = -(-n // r)
        assert 1 <= r <= max(1, min(32, n))
        if rows * n <= 16384:
            assert jobs * r - n <= n / 7, (n, r)
            assert r == 1 or 3072 <= rows * jobs, (n, r)
        assert r * (jobs - 1) < n and rows * jobs >= min(rows * n, 3072)


def test_chunks_at_named_sizes(rounds):
    assert [rounds(n, 32 * 64) for n in (1, 2, 3, 4, 5, 6, 7, 8)] == [1, 1, 1, 2, 1, 3, 4, 4]       # M = 32, 32 heads
    assert [rounds(n, 32 * 128) for n in (1, 2, 3, 4, 63)] == [1, 2, 3, 4, 21]                       # M = 64
    assert rounds(9, 8 * 64) == 1 and rounds(11, 8 * 64) == 2
