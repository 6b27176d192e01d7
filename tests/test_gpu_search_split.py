"""A launch of the search with few workgroups gives each row to two groups of waves.  The results do not depend on
that: a chunk's rows (few workgroups) equal the same rows of a plain prefill (many), bit for bit, for the scores, and so do
the one-pass lists."""
import numpy as np
import pytest

from paper_2603_06199_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# key blocks: two tiles of 32 with one block in the second, two full ones, an odd count, the longest row scored with both
# planes in the one-pass search and the first that is not
@pytest.mark.parametrize("blocks", (33, 64, 97, 128, 129))
@pytest.mark.parametrize("head_dim,block", ((128, 128), (64, 128), (256, 128), (128, 64), (128, 256)))
@pytest.mark.parametrize("last", ("full", "ragged"))
def test_chunk_equals_plain_search_bitwise(head_dim, block, blocks, last):
    hq, hkv, new = 32, 8, 3
    n = blocks * block - (0 if last == "full" else block // 2 + 5)
    q = n - (blocks - new) * block
    wg_per_row = hkv * -(-(hq // hkv) // (4 if block == 64 else 2 if block == 128 else 1))
    assert blocks * wg_per_row > 256 >= new * wg_per_row       # one group for the whole sequence, two for the chunk
    print(f"[case] D={head_dim} block={block} blocks={blocks} {last}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(blocks + block + head_dim)
    hot = torch.randn((head_dim,), generator=gen, device="cuda") / head_dim ** 0.5
    mark = (torch.rand((blocks,), generator=gen, device="cuda") < 0.1).float().repeat_interleave(block)[:n]
    Q = (torch.randn((n, hq, head_dim), generator=gen, device="cuda") + 4.0 * hot).bfloat16()
    K = (torch.randn((n, hkv, head_dim), generator=gen, device="cuda") + 3.0 * mark[:, None, None] * hot).bfloat16()
    whole = B.Plan([0, n], hq, hkv, head_dim=head_dim, block=block)
    chunk = B.Plan([0, q], hq, hkv, head_dim=head_dim, block=block, cu_seqlens_k=[0, n])
    Qc = Q[n - q:].contiguous()
    for eps in (1e-10, 0.5):                                      # without and with the pairs' maxima
        P, Pc = whole.fp_block_search(Q, K, eps=eps), chunk.fp_block_search(Qc, K, eps=eps)
        assert torch.equal(P[:, blocks - new:], Pc)
    idx, cnt = whole.fp_search_select(Q, K, 0.2)
    idc, cnc = chunk.fp_search_select(Qc, K, 0.2)
    assert torch.equal(cnt[:, blocks - new:], cnc)
    valid = torch.arange(blocks, device="cuda")[None, None] < cnc[:, :, None]
    assert torch.equal(idx[:, blocks - new:][valid], idc[valid])
    assert int(cnc.min()) >= 1 and int(cnc.max()) <= blocks
    whole.close(); chunk.close()
