"""Wait states around the register swaps between halves and rows of a wave (v_permlane32_swap, v_permlane16_swap), which are written as
asm statements, in the assembly of every kernel that reduces over a wave:

  before   two wait states stand in the same statement, for a vector instruction that has just written an operand
  after    within two wait states nothing reads a result through DPP or as an operand of an MFMA: the compiler, which does not see what
           the statement holds, may have left them out (any other vector instruction may read it at once)
"""
import pytest

from test_wait_states import Kernel, _fail_if, _regs, assembly  # noqa: F401  (assembly: a fixture)


def faults(k):
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


def test_swaps(assembly):  # noqa: F811
    found = {n: faults(Kernel(n, lines)) for n, lines in assembly.items()}
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
def test_the_rules_themselves(text, complaints):
    swaps, bad = faults(Kernel("k", list(text) + ["s_endpgm"]))
    assert swaps == 1 and len(bad) == complaints
