"""csrc/off_ladder.hpp keeps the products beyond its sixteen accumulators in ordinary registers, by matrix instructions written out in the
source, whose hazards the compiler does not look after.  What that rests on, checked on the built kernels."""
import re

import pytest

import listing

pytestmark = pytest.mark.skipif(not listing.AVAILABLE, reason="no LLVM tools")


def test_products_in_ordinary_registers_are_touched_by_their_matrix_instructions_alone():
    kernels = 0
    for symbol in listing.texts():
        if "off_ladder_kernel" not in symbol or not re.search(r"^\s+v_mfma\S+ v\[", listing.texts()[symbol], flags=re.M):
            continue
        kernels += 1
        code = listing.instructions(symbol)
        index = {i.at: n for n, i in enumerate(code)}
        mine = [n for n, i in enumerate(code) if re.match(r"v_mfma\S+ v\[", i.text)]
        loops = [(index[i.target], n) for n, i in enumerate(code) if i.target is not None and i.target <= i.at]
        inner = {max((lo, hi) for lo, hi in loops if lo < n < hi) for n in mine}         # the stage loops
        assert 2 <= len(inner) <= 4 and all(sum(lo < n < hi for lo, hi in inner) == 1 for n in mine)
        for lo, hi in inner:
            held = set()
            for n in mine:
                if lo < n < hi:
                    product, summand = re.match(r"v_mfma\S+ (v\[\d+:\d+\]),.*, (v\[\d+:\d+\])$", code[n].text).groups()
                    assert product == summand                         # in place: what the next one of the same slot reads is what this one wrote
                    assert code[n - 1].text == "s_nop 1"              # behind a write of a source, or the two steps of an INT8 product
                    held |= listing.vector_registers(product)
            for n in range(lo, hi + 1):
                assert n in mine or not listing.vector_registers(code[n].text) & held, (symbol, code[n].text)
            # behind the loop: 32 wait states before anything touches them
            at = hi + 1
            while [i.text for i in code[at:at + 2]] != ["s_nop 15", "s_nop 15"]:
                assert "s_cbranch" not in code[at].text and not listing.vector_registers(code[at].text) & held, (symbol, code[at].text)
                at = index[code[at].target] if code[at].target is not None else at + 1
    assert kernels == 8                                               # FP8 with 11 to 13 slices, INT8 with 11; two forms each


def test_the_check_finds_a_stranger():
    assert listing.vector_registers("v_mov_b64_e32 v[4:5], v[20:21]") == {4, 5, 20, 21}
    assert listing.vector_registers("v_mov_b32_e32 v17, 0") == {17} and not listing.vector_registers("v_accvgpr_write_b32 a17, 0")
