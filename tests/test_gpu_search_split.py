"""A launch of the search with few workgroups and long rows gives each row to two groups of waves (from 96 key blocks on at head
dimension 64, 224 to 416 elsewhere).  The results do not depend on
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


# every form in two groups: an odd number of tiles, an even one with one block in the last, and the same one tile on
@pytest.mark.parametrize("blocks", (416, 417, 448, 449))
@pytest.mark.parametrize("head_dim,block", ((128, 128), (64, 128), (256, 128), (128, 64), (128, 256)))
@pytest.mark.parametrize("last", ("full", "ragged"))
def test_long_rows_bitwise(head_dim, block, blocks, last):
    test_chunk_equals_plain_search_bitwise(head_dim, block, blocks, last)


# even and odd numbers of tiles in the hi-plane pass, whose first group re-scores all of a row's pairs, 32 at a time, while the second
# takes the barriers: key blocks that differ by little, alpha in the middle of their scores
@pytest.mark.parametrize("blocks", (192, 448, 600))
@pytest.mark.parametrize("head_dim,block", ((128, 128), (64, 128), (256, 128), (128, 64), (128, 256)))
def test_many_rescored_pairs(head_dim, block, blocks):
    hq, hkv, new = 32, 8, 3
    wg_per_row = hkv * -(-(hq // hkv) // (4 if block == 64 else 2 if block == 128 else 1))
    assert blocks * wg_per_row > 256 >= new * wg_per_row
    print(f"[case] D={head_dim} block={block} blocks={blocks}", flush=True)
    n, q = blocks * block, new * block
    gen = torch.Generator(device="cuda").manual_seed(blocks + block + head_dim)
    Q = torch.randn((n, hq, head_dim), generator=gen, device="cuda").bfloat16()
    K = torch.randn((block, hkv, head_dim), generator=gen, device="cuda").repeat(blocks, 1, 1)
    K = (K + 0.05 * torch.randn((n, hkv, head_dim), generator=gen, device="cuda")).bfloat16()
    whole = B.Plan([0, n], hq, hkv, head_dim=head_dim, block=block)
    chunk = B.Plan([0, q], hq, hkv, head_dim=head_dim, block=block, cu_seqlens_k=[0, n])
    Qc = Q[n - q:].contiguous()
    P = chunk.fp_block_search(Qc, K)
    ratio = P / P.amax(2, keepdim=True)
    alpha = float(ratio[ratio > 0].median())
    # nearer to the threshold than the hi plane can tell: |lo| is about 2^-10 of a pooled key, whose logits reach |q| |k| log2 e / sqrt(d) of
    # 1 to 2, hence 1e-3 and more in log2
    assert float((((ratio / alpha).log2().abs() < 1e-3).sum(2) > 32).float().mean()) > 0.75
    idx, cnt = whole.fp_search_select(Q, K, alpha)
    idc, cnc = chunk.fp_search_select(Qc, K, alpha)
    assert torch.equal(cnt[:, blocks - new:], cnc)
    valid = torch.arange(blocks, device="cuda")[None, None] < cnc[:, :, None]
    assert torch.equal(idx[:, blocks - new:][valid], idc[valid])
    assert blocks / 4 < float(cnc.float().mean()) < 3 * blocks / 4
    # scores of both planes decide: the lists are those of the two stages.  Both form 2^(t - T) / sum from the same t; exp2, division and
    # product round by 2^-24 or two each, so that only a score within 1e-6 of the threshold may go either way
    idt, cnt2 = chunk.fp_threshold(P, alpha)
    kept = []
    for i, c in ((idc, cnc), (idt, cnt2)):
        mask = torch.zeros((hq, new, blocks + 1), dtype=torch.bool, device="cuda")
        listed = torch.arange(blocks, device="cuda")[None, None] < c[:, :, None]
        mask.scatter_(2, torch.where(listed, i, blocks).long(), True)
        kept.append(mask[:, :, :blocks])
    assert float((ratio[kept[0] != kept[1]] / alpha - 1).abs().sum()) <= 1e-6 * int((kept[0] != kept[1]).sum())
    whole.close(); chunk.close()


# two groups' buffers and a row of so many key blocks do not fit the LDS at head dimension 256: one group, as in a launch of many rows
def test_row_too_long_for_two_groups():
    head_dim, blocks, many = 256, 4096, 257
    n = blocks * 128
    gen = torch.Generator(device="cuda").manual_seed(1)
    hot = 8.0 * torch.nn.functional.normalize(torch.randn((head_dim,), generator=gen, device="cuda"), dim=0)
    mark = (torch.rand((blocks,), generator=gen, device="cuda") < 0.05).float().repeat_interleave(128)
    Q = (torch.randn((many * 128, 2, head_dim), generator=gen, device="cuda") + hot).bfloat16()
    K = (torch.randn((n, 1, head_dim), generator=gen, device="cuda") + mark[:, None, None] * hot).bfloat16()
    rows = B.Plan([0, many * 128], 2, 1, head_dim=head_dim, cu_seqlens_k=[0, n])
    one = B.Plan([0, 128], 2, 1, head_dim=head_dim, cu_seqlens_k=[0, n])
    Q1 = Q[-128:].contiguous()
    assert torch.equal(rows.fp_block_search(Q, K)[:, -1:], one.fp_block_search(Q1, K))
    (idx, cnt), (id1, cn1) = rows.fp_search_select(Q, K, 0.2), one.fp_search_select(Q1, K, 0.2)
    assert torch.equal(cnt[:, -1:], cn1) and 1 <= int(cn1.min()) and int(cn1.max()) < blocks
    valid = torch.arange(blocks, device="cuda")[None, None] < cn1[:, :, None]
    assert torch.equal(idx[:, -1:][valid], id1[valid])
    rows.close(); one.close()
