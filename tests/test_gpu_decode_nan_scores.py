"""Decode with NaN among the candidates' scores (a NaN in a representative): such a block
ranks last, whichever way the candidates are scored and ranked, and every row lists k
different blocks."""
import numpy as np
import pytest
import torch

from paper_2601_02819_amd import phsa
from tests.gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [64, 1024])     # blocks of cache: 1024 are scored in slices
@pytest.mark.parametrize("equal", [False, True])  # all scores alike
@pytest.mark.parametrize("length", [24, 60])
@pytest.mark.parametrize("bad", [[3], [1, 2, 3, 7, 11], list(range(1, 20))])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_nan_ranks_last(cap, equal, length, bad, dtype):
    m, d, G, k = 64, 128, 2, 5
    log(f"[decode] NaN scores: cap={cap} equal={equal} length={length} bad={len(bad)} {dtype}")
    g = torch.Generator().manual_seed(length)
    q = torch.randn(1, 1, G, d, generator=g).to(dtype)
    kc = torch.randn(1, 1, cap, d, generator=g)
    if equal:
        kc[:] = kc[:, :, :1]
    kc[0, 0, bad, 5] = float("nan")
    kv = torch.randn(1, cap * m, 1, d, generator=g).to(dtype).cuda()
    cfg = phsa.Config(block_size=m, top_k=k, n_init_blocks=1, window=0)
    lens = torch.tensor([length * m], dtype=torch.int32).cuda()
    sel = phsa.decode_varlen(q.cuda(), kv, kv, kc.cuda(), lens, cfg)[0][0, 0, 0].tolist()
    score = (q.double().sum(2)[0, 0] @ kc[0, 0].double().T).numpy()
    if equal:
        score[:] = 0.0
        score[bad] = np.nan
    cand = sorted(range(1, length - 1), key=lambda t: (np.isnan(score[t]), -score[t] if score[t] == score[t] else 0, t))
    assert sel == [0, *sorted(cand[:k]), length - 1]


def test_nan_hides_no_score():
    """More than 64 equal scores, ranked one pick after another: the best block is found in a
    lane whose lower candidate (64 blocks before it) is NaN."""
    m, d, T, k = 64, 64, 160, 4
    q = torch.zeros(1, 1, 1, d)
    q[..., 0] = 1
    kc = torch.zeros(1, 1, T, d)
    kc[0, 0, 1 + 7 + 64, 0] = 1                 # candidate 71, of lane 7
    kc[0, 0, 1 + 7, 0] = float("nan")           # candidate 7, of lane 7 too
    kv = torch.ones(1, T * m, 1, d).bfloat16().cuda()
    cfg = phsa.Config(block_size=m, top_k=k, n_init_blocks=1, window=0)
    sel = phsa.decode(q.bfloat16().cuda(), kv, kv, kc.cuda(), cfg)[0][0, 0, 0].tolist()
    assert sel == [0, 1, 2, 3, 72, T - 1]
