"""Operands of the plain FP32 form, read from the gfx950 code object inside the
built liblensmap.so (no GPU).

Its rays evaluate the cell's Taylor polynomial each, so the 2 (P - 1)
coefficients are operands of most of a ray's instructions outside the lens loop,
and an instruction with a scalar operand takes twice the issue time of one whose
operands are vector registers: the coefficients must be held in vectors."""
import re

import pytest

from paper_2308_14278_amd import codeobj

KERNELS = ("k_shoot_mapILi1ELi1ELi%dELi%dE", "k_shoot_batchILi1ELi1ELi%dELi%dELi0E")


def _scalar_fmas(part):
    code = codeobj.kernel_code(part)
    assert code, "kernel not in the code object"
    fma = [ins for _, ins, _ in code if re.match(r"v_(fma|fmac)_f32", ins)]
    return len(fma), sum(1 for ins in fma if re.search(r"[ ,|-]s(\d|\[)", ins))


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("nr", [4, 16])
def test_taylor_coefficients_are_vector_operands(kernel, nr):
    if not codeobj.tools_available():
        pytest.skip("ROCm LLVM tools not found")
    (all2, s2), (all7, s7) = (_scalar_fmas(kernel % (nr, p)) for p in (2, 7))
    # five more terms add 4 FMAs each to every ray (linear and fold model, whole and
    # partial groups); none of them may take a scalar operand
    assert all7 - all2 >= 4 * 5 * nr
    assert s7 <= s2
