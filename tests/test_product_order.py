"""The check that keeps matrix products of two formats apart in the compiled kernels."""
import os

import pytest

from paper_2201_03478_amd import build, product_order

FP8 = "v_mfma_f32_16x16x32_fp8_fp8 v[0:3], v[20:21], v[22:23], %s"
F16 = "v_mfma_f32_16x16x32_f16 v[0:3], v[24:27], v[28:31], v[0:3]"
OTHER = "v_mfma_f32_16x16x32_f16 v[4:7], v[24:27], v[28:31], v[4:7]"


def _listing(lines):
    """Listing of a function of 8-byte instructions; a branch names its target line."""
    out = ["0000000000001000 <kern>:"]
    for i, s in enumerate(lines):
        op, _, arg = s.partition(" -> ")
        out.append("\t%s // %012X: 00000000%s" % (op, 0x1000 + 8 * i, " <kern+0x%x>" % (8 * int(arg)) if arg else ""))
    return "\n".join(out + ["\ts_endpgm // %012X: BF810000" % (0x1000 + 8 * len(lines))])


@pytest.mark.parametrize("lines,bad", [
    ([FP8 % "0", F16], [1]),                                      # back to back
    ([FP8 % "0", "s_nop 7", "v_add_f32_e32 v9, v9, v9", F16], [3]),  # too short a wait
    ([FP8 % "0", "s_nop 15", F16], []),
    ([FP8 % "0", "s_nop 7", "s_nop 7", F16], []),
    ([FP8 % "0", OTHER, F16], []),                                # another accumulator in between
    ([FP8 % "0", F16, F16], [1]),                                 # one format: no distance needed
    ([F16, FP8 % "v[0:3]"], [1]),                                 # the other way round
    ([F16, "v_mfma_f32_16x16x32_fp8_fp8 v[8:11], v[20:21], v[22:23], v[2:5]"], [1]),  # part of the result
    ([F16, FP8 % "0"], []),                                       # a fresh accumulator
    # round a loop: the FP16 product at its end meets the FP8 product at its start
    ([FP8 % "v[0:3]", "s_nop 15", F16, "s_cbranch_scc1 65532 -> 0"], [0]),
    ([FP8 % "v[0:3]", "s_nop 15", F16, "s_nop 15", "s_cbranch_scc1 65532 -> 0"], []),
    # a branch around the wait
    ([FP8 % "0", "s_cbranch_scc1 1 -> 3", "s_nop 15", F16], [3]),
    ([FP8 % "0", "s_branch 1 -> 3", F16, "s_nop 15", F16], []),
])
def test_adjacent_formats(lines, bad):
    assert [b[1] for b in product_order.adjacent_formats(_listing(lines))] == [8 * i for i in bad]


def test_built_gather_keeps_formats_apart():
    obj = os.path.join(build.BUILD, "k_gather.o")
    if not os.path.exists(obj):
        os.makedirs(build.BUILD, exist_ok=True)
        build._compile("k_gather.hip")
    text = product_order.disassemble(obj)
    assert "v_mfma_f32_16x16x32_fp8_fp8" in text and "v_mfma_f32_16x16x32_f16" in text
    assert product_order.adjacent_formats(text) == []
