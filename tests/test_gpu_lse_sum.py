"""Precision of the softmax row sum, seen through lse.  All keys but the first have the same logit, so every
addition to a long running sum rounds the same way and the errors add up instead of averaging out.  The
kernel sums each tile on its own and adds it once to the running sum; a sum that takes the exponentials in
one by one is 8 (32-key tiles) or 16 times as many roundings and misses the bound.

Bound, u = 2^-24, T tiles: the running sum grows evenly, so its T roundings of at most u times its value are
u T / 2 of the result; a tile's chain of 16, the sums of two chains and of two half waves and the
first tile's head start are less than 16 u; the exponential's argument (one rounding, |argument| < 16) and
result (1 ulp) are the same for every key, (0.7 * 16 + 2) u.  log2 of that times log2 e, and the three fp32
operations on a result below 16 that end in lse, 16 u each and 1 ulp of the logarithm."""
import numpy as np
import pytest

from paper_2603_06199_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 2.0 ** -24
LOG2E = 1.4426950408889634


@pytest.mark.parametrize("head_dim,block", [(64, 128), (128, 128), (256, 128), (128, 64), (128, 256)])
def test_row_sum_of_equal_terms(head_dim, block):
    n, gains = 16384, [1.25, 1.75, 2.0, 2.5, 3.5, 4.0, 5.0, 6.0]
    print(f"\n[case] head_dim {head_dim} block {block}", flush=True)
    # logit of key 0: 4 gain; of every other key: 0 (exact in bf16 and in the products)
    Q = torch.zeros((n, len(gains), head_dim), dtype=torch.bfloat16, device="cuda")
    Q[:, :, 0] = torch.tensor(gains, dtype=torch.bfloat16, device="cuda")
    K = torch.zeros((n, 1, head_dim), dtype=torch.bfloat16, device="cuda")
    K[0, 0, 0] = 4.0
    V = torch.ones_like(K)
    plan = B.Plan(np.array([0, n], np.int32), len(gains), 1, head_dim=head_dim, block=block)
    O, lse = plan.fp_dense_prefill(Q, K, V)
    torch.cuda.synchronize()
    plan.close()

    c = np.float32(1.0) / np.sqrt(np.float32(head_dim)) * np.float32(LOG2E)
    first = 4.0 * np.array(gains)[:, None] * float(c)
    keys = np.arange(1, n + 1)[None, :]
    ref = first + np.log2(1.0 + (keys - 1) * np.exp2(-first))
    tiles = keys // (64 if block > 64 else 32) + 1
    bound = U * (LOG2E * (tiles / 2 + 16 + 0.7 * 16 + 2) + 4 * 16)
    worst = (np.abs(lse.cpu().numpy() - ref) / bound).max(axis=1)
    assert worst.max() <= 1.0, f"error / bound by head: {worst}"
    assert torch.all((O.float() - 1.0).abs() <= 2.0 ** -7)      # V = 1: O is 1 but for the rounding of the probabilities
