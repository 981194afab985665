"""Resources of the shooting kernels that run 16 rays per lane by default beside the
plain FP32 ones: centred sums (four waves per SIMD: 128 VGPRs and 40 KiB of LDS a
workgroup) and FP64 sums (three: 168 VGPRs, a third of 160 KiB), read from the gfx950
code object inside the built liblensmap.so (no GPU).  What they spill to scratch memory
is held once per unit and must stay out of the lens loops."""
import re

import pytest

from paper_2308_14278_amd import codeobj

MAP = "_ZN12_GLOBAL__N_111k_shoot_mapILi1ELi%dELi16ELi%dEEEv6LmDesc"
BATCH = "_ZN12_GLOBAL__N_113k_shoot_batchILi1ELi%dELi16ELi%dELi0EEEvPK6LmDescPKlPKiiPy"


@pytest.fixture(scope="module")
def metadata():
    if not codeobj.tools_available():
        pytest.skip("ROCm LLVM tools not found")
    return codeobj.kernel_metadata()


@pytest.mark.parametrize("name", [MAP, BATCH])
@pytest.mark.parametrize("precision,vgprs,lds", [(4, 128, 40 * 1024), (2, 168, 160 * 1024 // 3)])
@pytest.mark.parametrize("terms,spills", [(4, 8), (7, 20)])
def test_resources(metadata, name, precision, vgprs, lds, terms, spills):
    k = metadata[name % (precision, terms)]
    assert int(k["vgpr_count"]) + int(k["agpr_count"]) <= vgprs
    assert int(k["group_segment_fixed_size"]) <= lds
    assert int(k["vgpr_spill_count"]) <= spills


def _blocks(code):
    """Basic blocks: instructions between branches and their targets."""
    start = code[0][0]
    targets = {start + int(m.group(1), 16) for _, ins, note in code if "branch" in ins
               for m in [re.search(r"\+0x([0-9a-f]+)>", note)] if m}
    block = []
    for addr, ins, _ in code:
        if addr in targets and block:
            yield block
            block = []
        block.append(ins)
        if "branch" in ins:
            yield block
            block = []
    yield block


@pytest.mark.parametrize("precision,rcp", [(4, "v_rcp_f32"), (2, "v_rcp_f64")])
@pytest.mark.parametrize("terms", [4, 7])
@pytest.mark.parametrize("kernel", ["k_shoot_mapILi1ELi%dELi16ELi%dE",
                                    "k_shoot_batchILi1ELi%dELi16ELi%dELi0E"])
def test_lens_loops_touch_no_scratch(metadata, kernel, precision, terms, rcp):
    code = codeobj.kernel_code(kernel % (precision, terms))
    # a step of the lens loop: its reciprocals and the FMAs of its columns
    loops = [b for b in _blocks(code) if sum(i.startswith(rcp) for i in b) >= 8
             and sum(i.startswith(("v_fma", "v_fmac", "v_pk_fma")) for i in b) >= 32]
    assert loops
    for b in loops:
        assert not any(i.startswith(("scratch_", "buffer_load", "buffer_store")) for i in b)
