"""The search holds every query fragment of its head dimension back until Q has landed, and no more than there are: one empty statement
per fragment in the assembly of each of its kernels."""
import re

from test_wait_states import Kernel, assembly  # noqa: F401  (assembly: a fixture)


def test_all_fragments_and_no_others(assembly):  # noqa: F811
    kernels = {n: Kernel(n, lines) for n, lines in assembly.items() if "search_kernel" in n}
    assert len(kernels) == 20      # head dimension and block, scores or lists, one or two groups of waves
    held = {n: sum(not region for region in k.regions) for n, k in kernels.items()}
    want = {n: 2 * int(re.search(r"ILi(\d+)E", n).group(1)) // 16 for n in kernels}     # 32 queries each, 16 dims each
    assert held == want
