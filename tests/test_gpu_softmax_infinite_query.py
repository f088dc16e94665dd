"""Softmax-sum selection (bf16) of rows with an infinite query in one head: that head's
probabilities are NaN, and with them every score of the row, so such a row keeps its forced
blocks alone, whatever the size of the group; the other rows are not touched."""
import pytest
import torch

from paper_2601_02819_amd import phsa
from tests.gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("Lq", [300, 4200])     # one and two row tiles per wave
@pytest.mark.parametrize("top_k", [5, 20])
@pytest.mark.parametrize("G,d", [(1, 128), (2, 128), (2, 64), (4, 64), (8, 128)])
def test_infinite_query(G, d, top_k, Lq, value):
    B, Hkv, m, T = 1, 8, 64, 80
    log(f"[select] softmax sum, query {value}: G={G} d={d} top_k={top_k} Lq={Lq}")
    g = torch.Generator().manual_seed(G + d + top_k)
    q = torch.randn(B, Lq, G * Hkv, d, generator=g)
    kc = torch.randn(B, Hkv, T, d, generator=g).cuda()
    cfg = phsa.Config(block_size=m, top_k=top_k, n_init_blocks=1, window=0, softmax_sum=True)
    want = phsa.select(q.bfloat16().cuda(), kc, T * m, cfg).cpu()
    q[:, ::7, 0, 3] = value                      # head 0: group 0
    sel = phsa.select(q.bfloat16().cuda(), kc, T * m, cfg).cpu()
    odd = torch.zeros(Lq, dtype=torch.bool)
    odd[::7] = True
    assert torch.equal(sel[:, :, ~odd], want[:, :, ~odd]) and torch.equal(sel[:, 1:], want[:, 1:])
    cur = (T * m - Lq + torch.arange(Lq)) // m
    assert (cur > 1).all()
    row = sel[0, 0, odd]
    assert (row[:, 0] == 0).all() and torch.equal(row[:, 1], cur[odd].int()) and (row[:, 2:] == -1).all()
