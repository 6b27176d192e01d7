"""The attention kernel deals (KV head, row) pairs to the XCDs in an order that depends on the number of KV heads and rows.  Every pair
is served, once and rightly, whatever the numbers: each KV head's outputs equal those of that head on its own, bit for bit."""
import numpy as np
import pytest

from paper_2603_06199_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# divisors and multiples of the eight XCDs, and numbers that are neither
@pytest.mark.parametrize("hkv", (1, 2, 3, 4, 5, 6, 8, 12, 16, 24))
# one row, fewer and more than the XCDs, ragged ends; a packed batch
@pytest.mark.parametrize("lens", ((77,), (128 * 7,), (128 * 8 + 1,), (128 * 19, 300, 128 * 2)))
def test_heads_alone_and_together(hkv, lens):
    group = 2
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    print(f"[case] hkv={hkv} lens={lens}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(hkv)
    Q = torch.randn((cu[-1], group * hkv, 128), generator=gen, device="cuda").bfloat16()
    K, V = (torch.randn((cu[-1], hkv, 128), generator=gen, device="cuda").bfloat16() for _ in range(2))
    O = torch.full_like(Q, float("nan"))
    together, alone = B.Plan(cu, group * hkv, hkv), B.Plan(cu, group, 1)
    O, lse = together.fp_dense_prefill(Q, K, V, O)
    for h in range(hkv):
        Oh, lh = alone.fp_dense_prefill(Q[:, group * h:group * (h + 1)].contiguous(), K[:, h:h + 1].contiguous(), V[:, h:h + 1].contiguous())
        assert torch.equal(O[:, group * h:group * (h + 1)], Oh) and torch.equal(lse[group * h:group * (h + 1)], lh)
    assert bool(torch.isfinite(O).all())
    together.close(); alone.close()


# lists of one KV head several times as long as the others': few rows and many, one and more workgroups per CU
@pytest.mark.parametrize("hkv,tokens", ((4, 128 * 5), (2, 128 * 40 + 9), (3, 128 * 31), (8, 128 * 29 + 1), (4, 128 * 64), (4, 128 * 65), (8, 128 * 90 + 77)))
@pytest.mark.parametrize("head_dim,block", ((128, 128), (64, 128), (256, 128), (128, 64), (128, 256)))
def test_sparse_heads_of_unequal_density(hkv, tokens, head_dim, block):
    group = 4
    rows = -(-tokens // block)
    print(f"[case] hkv={hkv} tokens={tokens} D={head_dim} block={block}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(tokens + hkv)
    Q = torch.randn((tokens, group * hkv, head_dim), generator=gen, device="cuda").bfloat16()
    K, V = (torch.randn((tokens, hkv, head_dim), generator=gen, device="cuda").bfloat16() for _ in range(2))
    rng = np.random.default_rng(tokens)
    keep = rng.random((group * hkv, rows, rows)) < np.where(np.arange(group * hkv) // group == hkv // 2, 0.9, 0.2)[:, None, None]
    keep[:, np.arange(rows), np.arange(rows)] = True
    keep &= np.tri(rows, dtype=bool)
    cnt = torch.from_numpy(keep.sum(2).astype(np.int32)).cuda()
    idx = torch.from_numpy(np.argsort(~keep, axis=2, kind="stable").astype(np.int32)).cuda()
    O = torch.full_like(Q, float("nan"))
    together, alone = (B.Plan([0, tokens], group * n, n, head_dim=head_dim, block=block) for n in (hkv, 1))
    O, lse = together.fp_sparse_prefill(Q, K, V, idx, cnt, O)
    for h in range(hkv):
        q = slice(group * h, group * (h + 1))
        Oh, lh = alone.fp_sparse_prefill(Q[:, q].contiguous(), K[:, h:h + 1].contiguous(), V[:, h:h + 1].contiguous(), idx[q].contiguous(), cnt[q].contiguous())
        assert torch.equal(O[:, q], Oh) and torch.equal(lse[q], lh)
    assert bool(torch.isfinite(O).all())
    together.close(); alone.close()
