"""Softmax-sum selection where many blocks tie: every score equal, or a few distinct
values, so that lists overflow and are cut again and again and the picks are
decided by the block index alone.  Scores are exact here (one feature, powers of
two), so the selection must equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,d,top_k", [(1, 64, 12), (2, 128, 12), (2, 64, 32), (4, 128, 5), (8, 64, 16), (1, 128, 31)])
@pytest.mark.parametrize("kind", ["ties", "two_values"])
def test_softmax_sum_ties(G, d, top_k, kind):
    B, Hkv, m, T, Lq = 1, 2, 16, 700, 150
    log(f"[softmax-sum] {kind} G={G} d={d} k={top_k}")
    kc = torch.zeros(B, Hkv, T, d)
    if kind == "two_values":
        kc[..., 0] = (torch.arange(T) % 9 < 2).float()   # 156 blocks tie at the top
    q = torch.zeros(B, Lq, G * Hkv, d)
    q[..., 0] = 4.0                                      # every head alike: a block's probability is monotone in kc
    cfg = phsa.Config(block_size=m, top_k=top_k, n_init_blocks=1, window=32, softmax_sum=True)
    sel = phsa.select(q.bfloat16().cuda(), kc.cuda(), T * m, cfg).cpu().numpy()
    ref, _, _ = oracle.select(q.numpy(), kc.double().numpy(), m, top_k, 1, 32, d ** -0.5, T * m, mode=oracle.SOFTMAX_SUM)
    np.testing.assert_array_equal(sel, ref)
