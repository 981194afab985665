"""Order of loads in the far-field coefficients, read from the gfx950 code object
inside the built liblensmap.so (no GPU).

A lens's data come through the scalar cache and a wave over a lattice of few cells has
nothing to hide them behind but its own sums: the next lenses must be read before the
current ones are summed, in the untested ranges and in the tested ones, where such a
lattice has most of its lenses."""
import pytest

from paper_2308_14278_amd import codeobj


@pytest.mark.parametrize("terms", [3, 4, 7])
def test_next_lenses_are_read_ahead(terms):
    if not codeobj.tools_available():
        pytest.skip("ROCm LLVM tools not found")
    code = [ins for _, ins, _ in codeobj.kernel_code("k_coeffsILi0ELi%dE" % terms)]
    assert code
    # runs of scalar loads whose first wait comes after a lens's reciprocal
    ahead, k = 0, 0
    while k < len(code):
        if not code[k].startswith("s_load"):
            k += 1
            continue
        sums = 0
        while k < len(code) and not (code[k].startswith("s_waitcnt") and "lgkmcnt(0)" in code[k]):
            sums += code[k].startswith("v_rcp_f64")
            k += 1
        ahead += sums >= 2
    # two in the loop of each kind of range
    assert ahead >= 4
    meta = [v for n, v in codeobj.kernel_metadata().items() if "k_coeffsILi0ELi%dE" % terms in n]
    assert int(meta[0]["private_segment_fixed_size"]) == 0 and int(meta[0]["vgpr_count"]) <= 128
