"""Launches with few workgroups run attention with two waves per 32 queries.  Both kernels form every sum in the same order:
a sequence on its own (few workgroups) equals the same sequence repeated in a packed batch (many), bit for bit."""
import numpy as np
import pytest

from paper_2603_06199_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _both(head_dim, n, prefix, gain, lists):
    """Outputs of the sequence alone and of its first copy in a batch, dense and (per list rule) sparse."""
    hq, hkv, block = 4, 2, 128
    gen = torch.Generator(device="cuda").manual_seed(n + prefix + head_dim)
    Q = (gain * torch.randn((n, hq, head_dim), generator=gen, device="cuda")).bfloat16()
    K, V = (torch.randn((n + prefix, hkv, head_dim), generator=gen, device="cuda").bfloat16() for _ in range(2))
    one = B.Plan([0, n], hq, hkv, head_dim=head_dim, cu_seqlens_k=[0, n + prefix])
    rows, width = one.m_total, one.n_max
    copies = 128 // (rows * hq) + 1
    many = B.Plan(np.arange(copies + 1) * n, hq, hkv, head_dim=head_dim, cu_seqlens_k=np.arange(copies + 1) * (n + prefix))
    assert one.m_total * hq <= 128 < many.m_total * hq        # two waves per 32 queries, one
    rep = lambda t: t.repeat(copies, 1, 1)
    yield one.fp_dense_prefill(Q, K, V), many.fp_dense_prefill(rep(Q), rep(K), rep(V)), n
    rng = np.random.default_rng(n)
    for rule in lists:
        idx, cnt = np.zeros((hq, rows, width), np.int32), np.zeros((hq, rows), np.int32)
        for h in range(hq):
            for r in range(rows):
                I = r + prefix // block
                keep = rule(rng, h, r, I)
                idx[h, r, :len(keep)], cnt[h, r] = keep, len(keep)
        i1, c1 = torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()
        yield (one.fp_sparse_prefill(Q, K, V, i1, c1),
               many.fp_sparse_prefill(rep(Q), rep(K), rep(V), i1.repeat(1, copies, 1).contiguous(), c1.repeat(1, copies).contiguous()), n)
    one.close(); many.close()


# list lengths 0, 1, 2, .. in turn, with and without the diagonal block; random lists of any length
def _counted(rng, h, r, I):
    k = min((h + r) % 10, I + 1)
    keep = rng.choice(I + 1, size=k, replace=False)
    return sorted(set(keep.tolist()) | ({I} if k and (h + r) % 2 else set()))


def _any(rng, h, r, I):
    return sorted(rng.choice(I + 1, size=int(rng.integers(1, I + 2)), replace=False).tolist())


@pytest.mark.parametrize("head_dim", (64, 128))
# 1 token to several blocks, ends on and beside block and 64-query boundaries, a prefix
@pytest.mark.parametrize("n,prefix", ((1, 0), (64, 0), (65, 0), (128, 0), (300, 0), (1024, 0), (1100, 0), (3937, 0), (200, 128 * 37), (128, 128 * 6)))
# logits of ordinary size, and large ones, which move the reference point of the softmax often
@pytest.mark.parametrize("gain", (1.0, 30.0))
def test_pair_equals_plain_bitwise(head_dim, n, prefix, gain):
    print(f"[case] D={head_dim} n={n} prefix={prefix} gain={gain}", flush=True)
    for (O, lse), (Om, lsem), n in _both(head_dim, n, prefix, gain, (_counted, _any)):
        assert torch.equal(O.view(torch.int16), Om[:n].view(torch.int16))
        assert torch.equal(lse, lsem[:, :n])
