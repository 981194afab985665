"""Resources of the direct sum's shooting kernels, read from the metadata of the
gfx950 code object inside the built liblensmap.so (no GPU).

Four workgroups to a CU need at most 128 VGPRs and 40 KiB of LDS.  The instances for
16 rays per lane take one block of lenses and must not touch scratch memory: a launch
of few lenses paid 2 us for its set-up, and the lens loop ran among spills."""
import pytest

from paper_2308_14278_amd import codeobj

MAP = "_ZN12_GLOBAL__N_111k_shoot_mapILi0ELi%dELi%dELi1EEEv6LmDesc"
BATCH = "_ZN12_GLOBAL__N_113k_shoot_batchILi0ELi%dELi%dELi1ELi0EEEvPK6LmDescPKlPKiiPy"


@pytest.mark.parametrize("name", [MAP, BATCH])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nr,spills", [(4, 0), (8, 16), (16, 0)])
def test_direct_kernels_fit_four_workgroups(name, precision, nr, spills):
    if not codeobj.tools_available():
        pytest.skip("ROCm LLVM tools not found")
    k = codeobj.kernel_metadata()[name % (precision, nr)]
    assert int(k["vgpr_count"]) + int(k["agpr_count"]) <= 128
    assert int(k["group_segment_fixed_size"]) <= 40 * 1024
    # 8 rays per lane keep the compensation of several blocks of lenses
    assert int(k["vgpr_spill_count"]) <= spills
    assert int(k["private_segment_fixed_size"]) <= 4 * spills
