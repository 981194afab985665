"""Order of memory in the peak statistics' hand-off, read from the gfx950 code
object inside the built liblensmap.so (no GPU).

The last workgroup of k_peak_stats takes the histograms over from all others, so
every wave's additions must have reached memory before its workgroup counts
itself as finished.  One thread of one wave does that behind a barrier, and the
barrier waits for no outstanding memory operation: each wave has to wait for its
own before it."""
import re

import pytest

from paper_2308_14278_amd import codeobj


def test_every_wave_waits_for_its_additions_before_the_barrier():
    if not codeobj.tools_available():
        pytest.skip("ROCm LLVM tools not found")
    code = codeobj.kernel_code("k_peak_stats")
    assert code, "kernel not in the code object"
    at = {addr: k for k, (addr, _, _) in enumerate(code)}
    adds = [k for k, (_, ins, _) in enumerate(code) if ins.startswith("global_atomic_add_x2")]
    assert len(adds) >= 2
    # no path from an addition to a barrier without a wait for all memory operations
    todo, seen = list(adds), set()
    while todo:
        k = todo.pop()
        if k in seen:
            continue
        seen.add(k)
        addr, ins, note = code[k]
        assert not ins.startswith("s_barrier"), \
            "the barrier is reached with additions outstanding (0x%x)" % addr
        if ins.startswith("s_endpgm") or (ins.startswith("s_waitcnt") and "vmcnt(0)" in ins):
            continue
        if "branch" in ins:
            todo.append(at[code[0][0] + int(re.search(r"\+0x([0-9a-f]+)>", note).group(1), 16)])
        if not ins.startswith("s_branch"):
            todo.append(k + 1)
