"""float32 forward: a row with a NaN or +inf score beside others has no weights, and its O is
NaN in every feature (not 0, which is what a row without keys gets); the other rows are not
touched."""
import pytest
import torch

from paper_2601_02819_amd import phsa
from tests.gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where,value", [("q", float("inf")), ("k", float("inf")), ("k", float("nan"))])
@pytest.mark.parametrize("G,d,m", [(1, 64, 16), (2, 128, 64), (4, 64, 32), (8, 128, 16)])
def test_rows_without_weights(G, d, m, where, value):
    L, Hkv, at = 3 * m, 2, m + 3
    log(f"[fp32] {where} {value}: G={G} d={d} m={m}")
    g = torch.Generator().manual_seed(G)
    q, k, v = (torch.randn(1, L, h, d, generator=g) for h in (G * Hkv, Hkv, Hkv))
    q[..., 5] = q[..., 5].abs() + 0.1
    k[..., 5] = k[..., 5].abs() + 0.1
    sel = torch.arange(3).expand(1, Hkv, L, 3)
    sel = torch.where(sel <= (torch.arange(L) // m)[None, None, :, None], sel, -1).int().contiguous().cuda()
    sel[:, :, 5] = -1                                    # a row without blocks
    cfg = phsa.Config(block_size=m, top_k=1, n_init_blocks=1, window=0)
    want = phsa.attn_fwd(q.cuda(), k.cuda(), v.cuda(), sel, cfg)[0].cpu()
    bad = torch.zeros(1, L, G * Hkv, dtype=torch.bool)
    if where == "q":
        q[0, at, 0, 5] = value
        bad[0, at, 0] = True
    else:
        k[0, at, 1, 5] = value
        bad[0, at:, G:] = True                           # every later row sees the key
    o = phsa.attn_fwd(q.cuda(), k.cuda(), v.cuda(), sel, cfg)[0].cpu()
    assert torch.isnan(o[bad]).all() and torch.equal(o[~bad], want[~bad])
    assert (o[0, 5] == 0).all()
