"""float32 attention takes every valid slot of a sel row, wherever it stands and however
often a block is listed, in the forward, dQ, dK and dV alike.  (Rows of that kind are
outside what the header asks for; the gradients must still be those of the forward.)"""
import pytest
import torch

from paper_2601_02819_amd import phsa
from tests.gpu_common import log

pytestmark = pytest.mark.gpu


def rows_of(form, T, L, m, g):
    sel = torch.full((L, 4), -1, dtype=torch.int32)
    for i in range(L):
        cur = i // m
        pick = torch.randint(0, cur + 1, (2,), generator=g).tolist()
        sel[i] = torch.tensor({"holes": [-1, pick[0], T + 3, cur] if pick[0] != cur else [-1, cur, -1, -1],
                               "future": [cur + 1, 0 if cur else -1, cur, cur + 2],
                               "any_order": [cur, *([] if cur == 0 else [0]), *([] if cur < 2 else [1]), -1, -1, -1][:4],
                               "copies": [pick[0], cur, pick[1], cur]}[form])
    return sel


@pytest.mark.parametrize("form", ["holes", "future", "any_order", "copies"])
@pytest.mark.parametrize("m,G,d,T", [(16, 1, 64, 20), (32, 4, 128, 5), (64, 2, 64, 5)])
def test_gradients_of_the_forward(form, m, G, d, T):
    L, Hkv = T * m, 2
    log(f"[fp32 sel] {form} m={m} G={G} d={d} T={T}")
    g = torch.Generator().manual_seed(m)
    q, do = (torch.randn(1, L, G * Hkv, d, generator=g) for _ in "qo")
    k, v = (torch.randn(1, L, Hkv, d, generator=g) for _ in "kv")
    sel = torch.stack([rows_of(form, T, L, m, g) for _ in range(Hkv)])[None].contiguous()
    cfg = phsa.Config(block_size=m, top_k=2, n_init_blocks=1, window=0)
    o, lse = phsa.attn_fwd(q.cuda(), k.cuda(), v.cuda(), sel.cuda(), cfg)
    got = (o, *phsa.attn_bwd(q.cuda(), k.cuda(), v.cuda(), o, do.cuda(), lse, sel.cuda(), cfg))
    # float64: the softmax with each key counted as often as its block is listed
    times = torch.zeros(Hkv, L, T, dtype=torch.float64)
    for s in range(4):
        t = sel[0, :, :, s].long()
        ok = (t >= 0) & (t <= torch.arange(L) // m) & (t < T)
        times.scatter_add_(2, t.clamp(0, T - 1)[..., None], ok.double()[..., None])
    times = times.repeat_interleave(m, 2) * (torch.arange(L)[None, :] <= torch.arange(L)[:, None])
    qd, kd, vd = (x.double().requires_grad_(True) for x in (q, k, v))
    out = []
    for h in range(G * Hkv):
        p = torch.exp(qd[0, :, h] @ kd[0, :, h // G].T * d ** -0.5) * times[h // G]
        out.append((p / p.sum(1, keepdim=True)) @ vd[0, :, h // G])
    ref = torch.stack(out, 1)[None]
    for name, a, r in zip(("O", "dQ", "dK", "dV"), got,
                          (ref.detach(), *torch.autograd.grad(ref, (qd, kd, vd), do.double()))):
        err = ((a.cpu().double() - r).norm() / r.norm()).item()
        assert err < 1e-5, f"{name}: {err}"
