"""Where inline assembly writes VCC or scalar registers with a vector instruction and reads them with one, it has to keep
the wait states that the compiler puts in by itself on gfx950: two between the write and the read.  Checked in the assembly of
the sources that hold such blocks, cross-compiled (no GPU needed)."""
import re

import pytest

from tests.test_exchange_codegen_cpu import assembly, kernels

WAIT_STATES = 2
TWO_RESULTS = re.compile(r"_co_|^v_div_scale|^v_mad_[iu]64_[iu]32")    # the second operand is written as well


def scalars(operand):
    """The scalar registers in an operand, one by one."""
    operand = operand.split()[0].strip("|-")
    if operand in ("vcc", "vcc_lo", "vcc_hi"):
        return {"vcc_lo", "vcc_hi"} if operand == "vcc" else {operand}
    m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    first, last = (m[1], m[1]) if m[1] else (m[2], m[3])
    return {f"s{k}" for k in range(int(first), int(last) + 1)}


def too_early(body):
    """(write, read) pairs of vector instructions with fewer than the wait states between them."""
    found, recent = [], []                                               # recent: (wait states since, written, line)
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.endswith(":") or line.startswith("."):
            continue
        name, _, rest = line.partition(" ")
        written = set()
        if name.startswith("v_"):
            operands = [o.strip() for o in rest.split(",") if o.strip()]
            n_results = 2 if TWO_RESULTS.search(name) else 1
            for o in operands[:n_results]:
                written |= scalars(o)
            read = set().union(*[scalars(o) for o in operands[n_results:]])
            if name.startswith("v_div_fmas"):
                read |= {"vcc_lo", "vcc_hi"}
            found += [(w, line) for _, regs, w in recent if regs & read]
        passed = int(rest, 0) + 1 if name == "s_nop" else 1
        recent = [(n + passed, regs - written, w) for n, regs, w in recent if n + passed < WAIT_STATES]
        if written:
            recent.append((0, written, line))
    return found


def test_the_reader_of_assembly_sees_what_it_looks_for():
    early = "v_cmp_le_f32_e32 vcc, v1, v2\n\tv_addc_co_u32_e32 v0, vcc, v0, v0, vcc"
    assert len(too_early(early)) == 1
    assert len(too_early("v_cmp_le_f32_e64 s[4:5], v1, v2\n\ts_nop 0\n\tv_cndmask_b32_e64 v0, v1, v2, s[4:5]")) == 1
    assert len(too_early("v_readlane_b32 s5, v1, 3\n\tv_mov_b32_e32 v9, v8\n\tv_fma_f32 v0, |s5|, v1, v2")) == 1
    assert not too_early(early.replace("\n", "\n\ts_nop 1\n"))
    assert not too_early("v_cmp_le_f32_e64 s[4:5], v1, v2\n\tv_mov_b32_e32 v9, v8\n\ts_mov_b32 s8, 0\n\tv_cndmask_b32_e64 v0, v1, v2, s[4:5]")


@pytest.mark.parametrize("source", ["pq_encode.hip", "pq_kmeans.hip"])
def test_vector_reads_of_scalars_wait(source, tmp_path):
    text = assembly(source, tmp_path)
    bodies = kernels(text)
    assert any("grid_kernel" in name for name in bodies)
    early = {name: pairs for name, pairs in ((n, too_early(b)) for n, b in bodies.items()) if pairs}
    assert not early, {name: (len(pairs), pairs[:3]) for name, pairs in early.items()}
