"""bf16 selection with one and with two row tiles per wave (by the number of row tiles
of all (b, g)), on either side of the line: against the oracle with ragged last tiles,
windows, and many equal scores.  Calls that large are split over (b, g) here, so
that rows and blocks stay few."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import check_sel, log, to_np

pytestmark = pytest.mark.gpu


def run(B, Hkv, G, d, Lq, T, top_k, window, ties, softmax_sum):
    m, n_init = 16, 2
    log(f"[select] R={B * Hkv} G={G} d={d} Lq={Lq} T={T} k={top_k} ties={ties} softmax_sum={softmax_sum}")
    g = torch.Generator().manual_seed(Lq + G)
    q = torch.randn(B, Lq, G * Hkv, d, generator=g)
    kc = torch.randn(B, Hkv, T, d, generator=g) * 0.3
    if ties:   # exact scores: one feature, few values, every head alike
        q = torch.zeros_like(q)
        q[..., 0] = 4.0
        kc = torch.zeros_like(kc)
        kc[..., 0] = (torch.arange(T) % 7 < 3).float()
    cfg = phsa.Config(block_size=m, top_k=top_k, n_init_blocks=n_init, window=window, softmax_sum=softmax_sum)
    sel = phsa.select(q.bfloat16().cuda(), kc.cuda(), T * m, cfg).cpu().numpy()
    mode = oracle.SOFTMAX_SUM if softmax_sum else oracle.SUM_LOGITS
    qh, kch = to_np(q.bfloat16()), kc.double().numpy()
    ref, kth, gap = oracle.select(qh, kch, m, top_k, n_init, window, d ** -0.5, T * m, mode=mode)
    if ties:
        np.testing.assert_array_equal(sel, ref)
    else:
        check_sel(sel, ref, kth, gap, lambda i: oracle.score_row(qh, kch, m, d ** -0.5, T * m, *(i[0], i[2], i[1]), mode=mode))


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("B,Hkv,G,d,Lq,T,top_k,window", [
    (8, 8, 2, 128, 500, 90, 12, 0),      # 256 tiles of 128 rows: one per wave
    (8, 8, 2, 128, 513, 90, 12, 32),     # 320: two, the last tile one row
    (8, 12, 8, 64, 400, 70, 16, 0),      # 384 at d = 64: one
    (8, 13, 2, 64, 500, 60, 9, 0),       # 416 at d = 64, few blocks: one
    (8, 13, 2, 64, 500, 66, 9, 0),       # 416 at d = 64: two
    (8, 8, 1, 64, 900, 130, 5, 0),       # 512 at d = 64: two, chunks past the first 64 blocks
    (5, 13, 4, 128, 600, 80, 16, 64),    # 325: two
])
def test_summed_logits(B, Hkv, G, d, Lq, T, top_k, window, ties):
    run(B, Hkv, G, d, Lq, T, top_k, window, ties, False)


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("B,Hkv,G,d,Lq,T,top_k,window", [
    (8, 8, 2, 128, 256, 90, 12, 0),      # 256 workgroups of 128 pairs: one tile per wave
    (8, 8, 2, 128, 257, 90, 12, 32),     # 320: two, the last workgroup one token
    (8, 8, 4, 64, 256, 130, 16, 0),      # 512 at d = 64: one
    (8, 9, 4, 64, 257, 130, 5, 64),      # 648: two
    (5, 13, 8, 128, 65, 80, 16, 0),      # 325: two
    (8, 8, 1, 128, 700, 80, 12, 0),      # one head per group: one
    (8, 8, 2, 64, 600, 80, 20, 0),       # more than 16 picks: one
])
def test_softmax_sum(B, Hkv, G, d, Lq, T, top_k, window, ties):
    run(B, Hkv, G, d, Lq, T, top_k, window, ties, True)
