"""GPU parity of the attention kernels over the length of a row's list.  A row runs its list as plain steps,
masked steps and two closing steps, in pairs of tiles; which of them occur, and how often, depends on the
number of listed blocks, on whether the diagonal block is among them and on whether the sequence ends
inside it.  Lists of 0 .. 6 blocks with and without the diagonal one, and of all of a row's 1 .. 9 blocks, on full and
ragged last blocks, at every head dimension and block size, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2603_06199_amd import binding as B
import synth

from gpu_util import LSE_ATOL, compare_O, dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tail", [0, 1, 33])
@pytest.mark.parametrize("head_dim,block", [(64, 128), (128, 128), (256, 128), (128, 64), (128, 256)])
def test_rows_of_every_length(head_dim, block, tail):
    hq, hkv = 8, 2
    lens = [8 * block + tail, block + tail]
    print(f"\n[case] head_dim {head_dim} block {block} tail {tail}", flush=True)
    Q, K, V = synth.random_qkv(lens, hq, hkv, head_dim, seed=5)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    m_total, n_max, ro = oracle.layout(cu, block=block)[:3]
    idx = np.zeros((hq, m_total, n_max), np.int32)
    cnt = np.zeros((hq, m_total), np.int32)
    rng = np.random.default_rng(9)
    for s in range(len(lens)):
        for r in range(ro[s], ro[s + 1]):
            I = int(r - ro[s])
            for h in range(hq):
                want = min(h if h < 7 else I + 1, I + 1)       # head h lists h blocks, the last one all
                blocks = rng.permutation(I + 1)[:want]
                if want and h % 2 == 0:                        # even heads see the diagonal block
                    blocks[0] = I if I not in blocks else blocks[0]
                blocks = np.unique(blocks)
                idx[h, r, :blocks.size], cnt[h, r] = blocks, blocks.size
    O_ref, lse_ref = oracle.sparse_prefill(Q, K, V, cu, idx, cnt, block=block)
    plan = B.Plan(cu, hq, hkv, head_dim=head_dim, block=block)
    O, lse = plan.fp_sparse_prefill(dev(Q), dev(K), dev(V), torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda())
    torch.cuda.synchronize()
    compare_O(O, O_ref)
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=LSE_ATOL, rtol=0)
    plan.close()
