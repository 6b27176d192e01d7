"""The rules of test_wait_states.py for the attention kernel with two waves per 32 queries, read off its assembly in the same way."""
import pytest

from test_wait_states import MFMA_RESULT, Kernel, _fail_if, assembly  # noqa: F401  (assembly: a fixture)


@pytest.fixture(scope="module")
def pair(assembly):  # noqa: F811
    kernels = [Kernel(n, lines) for n, lines in assembly.items() if "attn_pair_kernel" in n]
    assert len(kernels) == 4 and all(any(i.mfma for i in k.ins) for k in kernels)
    return kernels


def test_exponentials_and_mfma_results(pair):
    n, bad = 0, []
    for k in pair:
        for region in k.regions:
            for at, i in enumerate(region):
                e = k.ins[i]
                if e.op.startswith("v_exp_f32"):
                    n += 1
                    if at + 1 == len(region) or e.writes & k.ins[region[at + 1]].reads:
                        bad.append(f"{k.name}: {e.text}: no wait state behind it in its statement")
        for i, p in enumerate(k.ins):
            if p.mfma:
                bad += [f"{k.name}: {p.text} -> {u.text}" for u in k.after(i, MFMA_RESULT)
                        if not u.mfma and u.asm and (u.reads | u.writes) & p.writes]
    _fail_if(bad)
    assert n >= 4 * 16 * 7       # the steps' variants and the last tile


def test_loads(pair):
    queries, tiles, bad = 0, 0, []
    for k in pair:
        for i, p in enumerate(k.ins):
            if p.asm and p.op == "global_load_dwordx4":
                queries += 1
                todo, seen = list(k.next[i]), set()
                while todo:
                    j = todo.pop()
                    u = k.ins[j]
                    if j in seen or (u.op == "s_waitcnt" and "vmcnt" in u.text):
                        continue
                    seen.add(j)
                    if (u.reads | u.writes) & p.writes:
                        bad.append(f"{k.name}: {p.text} -> {u.text}")
                    todo += k.next[j]
            sgprs = {r for r in p.writes if r[0] == "s"} if p.valu else set()
            if sgprs:
                bad += [f"{k.name}: {p.text} -> {u.text}" for u in k.after(i, 5)
                        if u.asm and u.op.startswith("global_load") and u.reads & sgprs]
        for region in k.regions:
            ops = [k.ins[i] for i in region]
            if any(o.op.startswith("global_load_lds") for o in ops):
                tiles += 1
                if not (len(ops) == 3 and ops[0].text.startswith("s_mov_b32 m0") and ops[2].op.startswith("global_load_lds")):
                    bad.append(f"{k.name}: {[o.text for o in ops]}")
    _fail_if(bad)
    assert queries == 2 * (4 + 8) and tiles > 40
