"""Forward attention and decode with infinite keys and values, against the oracle: a key
that scores -inf has weight 0 beside any finite score, and an infinite value shows in
its own features only."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import O_TOL, log, to_np

pytestmark = pytest.mark.gpu
DT = {"bf16": torch.bfloat16, "fp32": torch.float32}


def same_where_finite(a, r, tol, name):
    fine = np.isfinite(r)
    assert fine.any()
    assert np.isfinite(a[fine]).all(), f"{name}: {np.argwhere(~np.isfinite(a) & fine)[:4].tolist()}"
    np.testing.assert_allclose(a[fine], r[fine], atol=tol, rtol=0, err_msg=name)


@pytest.mark.parametrize("G,d,m", [(1, 64, 16), (2, 128, 64), (8, 64, 32)])
def test_fp32_forward_keys_at_minus_infinity(G, d, m):
    L, Hkv = 3 * m, 2
    log(f"[-inf key] forward G={G} d={d} m={m}")
    g = torch.Generator().manual_seed(G)
    q, k, v = (torch.randn(1, L, h, d, generator=g) for h in (G * Hkv, Hkv, Hkv))
    q[..., 5] = q[..., 5].abs() + 0.1
    k[0, ::2, :, 5] = float("-inf")   # every other key: row 1 sees one such key and one finite one
    sel = torch.arange(3).expand(1, Hkv, L, 3)
    sel = torch.where(sel <= (torch.arange(L) // m)[None, None, :, None], sel, -1).int().contiguous()
    cfg = phsa.Config(block_size=m, top_k=1, n_init_blocks=1, window=0)
    o, lse = phsa.attn_fwd(q.cuda(), k.cuda(), v.cuda(), sel.cuda(), cfg)
    o_r, lse_r = oracle.attn_fwd(q.numpy(), k.numpy(), v.numpy(), sel.numpy(), m, d ** -0.5)
    same_where_finite(to_np(o)[:, 1:], o_r[:, 1:], O_TOL["fp32"], "O")
    same_where_finite(to_np(lse)[..., 1:], lse_r[..., 1:], O_TOL["fp32"], "LSE")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("G,d,m,n", [(1, 64, 16, 2), (2, 128, 16, 18), (4, 64, 64, 67), (8, 128, 32, 34)])
def test_decode_keys_at_minus_infinity(dtype, G, d, m, n):
    L, Hkv, B = 8 * m, 2, 2
    log(f"[-inf key] decode {dtype} G={G} d={d} m={m} length {n}")
    g = torch.Generator().manual_seed(n)
    q = torch.randn(B, 1, G * Hkv, d, generator=g)
    q[..., 5] = q[..., 5].abs() + 0.1
    k, v = (torch.randn(B, L, Hkv, d, generator=g) for _ in "kv")
    kc = phsa.compress(k.to(DT[dtype]).cuda(), torch.zeros(B, L, dtype=torch.uint8).cuda(),
                       phsa.Config(block_size=m, top_k=2))
    k[:, ::2, :, 5] = float("-inf")
    q, k, v = (x.to(DT[dtype]) for x in (q, k, v))
    cfg = phsa.Config(block_size=m, top_k=2, n_init_blocks=1, window=0)
    sel, o, lse = phsa.decode_varlen(q.cuda(), k.cuda(), v.cuda(), kc, torch.full((B,), n, dtype=torch.int32).cuda(), cfg)
    pad = -(-n // m) * m
    o_r, lse_r = oracle.attn_fwd(to_np(q), to_np(k)[:, :pad], to_np(v)[:, :pad], sel.cpu().numpy(), m, d ** -0.5,
                                 q_pos0=n - 1)
    same_where_finite(to_np(o), o_r, O_TOL[dtype], "O")
    same_where_finite(to_np(lse), lse_r, O_TOL[dtype], "LSE")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("mode", ["plain", "softmax_sum", "sliced"])
@pytest.mark.parametrize("G,d,m,n", [(1, 64, 16, 5), (2, 128, 16, 300), (4, 64, 64, 200), (8, 128, 32, 1000)])
def test_decode_infinite_values(dtype, mode, G, d, m, n):
    """Values of +-inf at the query's own position, inside a selected block and both
    signs in one feature (NaN there): O as the oracle has it, finite elsewhere."""
    L, Hkv, B = (512 if mode == "sliced" else 64) * m, 2, 2
    log(f"[inf value] decode {dtype} {mode} G={G} d={d} m={m} length {n}")
    g = torch.Generator().manual_seed(n + G)
    q = (torch.randn(B, 1, G * Hkv, d, generator=g) * 0.3).to(DT[dtype])
    k, v = (torch.randn(B, L, Hkv, d, generator=g) for _ in "kv")
    v[:, n - 1, :, 3] = float("inf")
    v[:, 1, :, 7] = float("-inf")
    v[:, n - 1, 0, 9], v[:, 2, 0, 9] = float("inf"), float("-inf")
    k, v = k.to(DT[dtype]), v.to(DT[dtype])
    cfg = phsa.Config(block_size=m, top_k=3, n_init_blocks=1, window=0, softmax_sum=mode == "softmax_sum")
    kc = phsa.compress(k.cuda(), torch.zeros(B, L, dtype=torch.uint8).cuda(), cfg)
    sel, o, lse = phsa.decode_varlen(q.cuda(), k.cuda(), v.cuda(), kc, torch.full((B,), n, dtype=torch.int32).cuda(), cfg)
    pad = -(-n // m) * m
    o_r, lse_r = oracle.attn_fwd(to_np(q), to_np(k)[:, :pad], to_np(v)[:, :pad], sel.cpu().numpy(), m, d ** -0.5,
                                 q_pos0=n - 1)
    assert np.isinf(o_r).sum() == (2 * G * Hkv) * B and np.isnan(o_r).sum() == G * B
    np.testing.assert_allclose(to_np(o), o_r, atol=O_TOL[dtype], rtol=0)
    np.testing.assert_allclose(to_np(lse), lse_r, atol=O_TOL[dtype], rtol=0)
