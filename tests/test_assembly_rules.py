"""Rules that the assembly of every kernel of the library keeps, read off one listing."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_06199_amd import build as hip_build
from test_wait_states import HIPCC, Kernel, _fail_if, _regs


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("needs hipcc")
    out = tmp_path_factory.mktemp("isa") / "flashprefill.s"
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
    subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out)] +
                   [os.path.join(hip_build.CSRC, s) for s in hip_build.SOURCES], check=True, capture_output=True)
    return out.read_text()


@pytest.fixture(scope="module")
def kernels(listing):
    return {m.group(1): Kernel(m.group(1), m.group(2).split("\n"))
            for m in re.finditer(r"^(_ZN2fp\w+):.*?\n(.*?)^\s*\.section", listing, re.S | re.M)}


def test_no_scratch_no_spills(listing):
    """Compute calls allocate nothing, and scratch memory would be the runtime's to provide at a launch."""
    notes = listing.split("amdhsa.kernels:")[1].split("\namdhsa.")[0]
    found = {}
    for k in re.split(r"^  - ", notes, flags=re.M)[1:]:
        get = lambda key: re.search(rf"\.{key}:\s*(\S+)", k).group(1)
        found[get("symbol")] = (int(get("private_segment_fixed_size")), int(get("vgpr_spill_count")))
    # 10 attention kernels, 4 with two waves per 32 queries, 20 of the search, 5 of pooling, 2 of the threshold
    assert len(found) == 41, sorted(found)
    assert not {k: v for k, v in found.items() if v != (0, 0)}


def test_search_holds_its_query_fragments(kernels):
    """The search holds every query fragment of its head dimension back until Q has landed, and no more than there are: one empty
    statement per fragment."""
    search = {n: k for n, k in kernels.items() if "search_kernel" in n}
    assert len(search) == 20      # head dimension and block, scores or lists, one or two groups of waves
    held = {n: sum(not region for region in k.regions) for n, k in search.items()}
    assert held == {n: 2 * int(re.search(r"ILi(\d+)E", n).group(1)) // 16 for n in search}     # 32 queries each, 16 dims each


# Register swaps between halves and rows of a wave (v_permlane32_swap, v_permlane16_swap) are asm statements:
#   before   two wait states stand in the same statement, for a vector instruction that has just written an operand
#   after    within two wait states nothing reads a result through DPP or as an operand of an MFMA: the compiler, which does not see
#            what the statement holds, may have left them out (any other vector instruction may read it at once)
def swap_faults(k):
    """(number of swaps, complaints) of one kernel."""
    bad, swaps = [], 0
    for region in k.regions:
        states = 0
        for i in region:
            if "permlane" in k.ins[i].op and "swap" in k.ins[i].op:
                swaps += 1
                if states < 2:
                    bad.append(f"{k.name}: {k.ins[i].text}: {states} wait states before it in its statement")
                result = _regs(k.ins[i].args)
                bad += [f"{k.name}: {k.ins[i].text} -> {u.text}" for u in k.after(i, 2)
                        if ("_dpp" in u.op or u.mfma) and _regs(u.args[1:]) & result]
            # a statement's own earlier vector instructions are as close as any
            states = states + k.ins[i].states if not k.ins[i].valu else 0
    assert swaps == sum("permlane" in i.op and "swap" in i.op for i in k.ins), f"{k.name}: a swap outside of a statement"
    return swaps, bad


def test_swaps(kernels):
    found = {n: swap_faults(k) for n, k in kernels.items()}
    _fail_if([b for _, bad in found.values() for b in bad])
    for kernel, number in (("attn_kernel", 10), ("attn_pair_kernel", 4), ("search_kernel", 20), ("threshold_kernel", 2)):
        swaps = [s for n, (s, _) in found.items() if kernel in n]
        assert len(swaps) == number and min(swaps) > 0, kernel


@pytest.mark.parametrize("text,complaints", (
    (("v_mov_b32_e32 v4, v11", "#ASMSTART", "s_nop 1", "v_permlane16_swap_b32 v4, v11", "#ASMEND", "v_max_f32_e32 v4, v4, v11"), 0),
    (("#ASMSTART", "s_nop 0", "v_permlane16_swap_b32 v4, v11", "#ASMEND", "v_max_f32_e32 v4, v4, v11"), 1),
    (("#ASMSTART", "v_permlane32_swap_b32 v4, v11", "#ASMEND", "s_nop 1", "v_max_f32_dpp v4, v4, v4 row_ror:8"), 1),
    (("#ASMSTART", "s_nop 1", "v_permlane32_swap_b32 v4, v11", "#ASMEND", "s_nop 0", "v_max_f32_dpp v1, v2, v11 row_ror:8"), 1),
    (("#ASMSTART", "s_nop 1", "v_permlane32_swap_b32 v4, v11", "#ASMEND", "v_mov_b32_e32 v0, v1", "s_nop 0", "v_max_f32_dpp v1, v2, v11 row_ror:8"), 0),
    (("#ASMSTART", "s_nop 1", "v_permlane32_swap_b32 v4, v11", "#ASMEND", "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[0:3], 0"), 1),
))
def test_swap_rules_themselves(text, complaints):
    swaps, bad = swap_faults(Kernel("k", list(text) + ["s_endpgm"]))
    assert swaps == 1 and len(bad) == complaints
