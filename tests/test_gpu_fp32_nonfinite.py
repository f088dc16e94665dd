"""float32 backward with infinities and NaN: a row's Q or dO, or a key's K or V, reaches
the gradients of the pairs it takes part in and no others.  Every row attends to
block 0 and its own block, so a value planted past the middle of a block must leave
the keys after its row, and the rows before its key, as the oracle has them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import log, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,G,d", [(16, 2, 64), (32, 1, 128), (64, 4, 64), (64, 8, 128)])
@pytest.mark.parametrize("what", ["q", "k", "v", "do"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_masked_pairs_stay_out(m, G, d, what, value):
    L, Hkv, B = 5 * m, 2, 1
    log(f"[fp32 non-finite] {what} {value} m={m} G={G} d={d}")
    g = torch.Generator().manual_seed(m + G)
    x = {"q": torch.randn(B, L, G * Hkv, d, generator=g), "k": torch.randn(B, L, Hkv, d, generator=g),
         "v": torch.randn(B, L, Hkv, d, generator=g), "do": torch.randn(B, L, G * Hkv, d, generator=g)}
    i = 3 * m + m // 2 + 1   # a row (or key) past the middle of block 3
    x[what][0, i, 0, 5] = value
    cur = torch.arange(L) // m
    sel = torch.stack([torch.zeros_like(cur), torch.where(cur > 0, cur, -1)], 1).int().expand(B, Hkv, L, 2).contiguous()
    cfg = phsa.Config(block_size=m, top_k=0, n_init_blocks=1, window=0)
    dev = {n: t.cuda() for n, t in x.items()}
    o, lse = phsa.attn_fwd(dev["q"], dev["k"], dev["v"], sel.cuda(), cfg)
    got = phsa.attn_bwd(dev["q"], dev["k"], dev["v"], o, dev["do"], lse, sel.cuda(), cfg)
    ref = oracle.attn_bwd(*(x[n].numpy() for n in ("q", "k", "v", "do")), sel.numpy(), m, d ** -0.5)
    for name, a, r in zip(("dQ", "dK", "dV"), got, ref):
        a = to_np(a)
        fine = np.isfinite(r)
        assert fine.mean() > 0.5
        assert np.isfinite(a[fine]).all(), f"{name}: {np.argwhere(~np.isfinite(a) & fine)[:4].tolist()}"
        np.testing.assert_allclose(a[fine], r[fine], atol=1e-4, rtol=0, err_msg=name)
