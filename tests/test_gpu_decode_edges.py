"""Decode at the edges of its dispatch, against the oracle: candidate ranges scored by
one workgroup and by slices (odd numbers of candidates, slices that come out
empty, more picks than a slice holds), every group size and head dim, and the
selection's order on ties and on scores that leave all winners in one lane or in
one slice."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import O_TOL, check_sel, log, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,d,m,T,top_k,n_init,window,dtype", [
    (1, 64, 64, 9, 4, 1, 0, "bf16"), (2, 128, 16, 700, 16, 8, 512, "bf16"), (8, 64, 32, 1000, 7, 2, 64, "bf16"),
    (8, 128, 16, 513, 32, 1, 0, "bf16"), (4, 128, 16, 2048, 1, 0, 16, "bf16"), (1, 128, 16, 1999, 12, 1, 0, "bf16"),
    (2, 64, 64, 130, 31, 3, 128, "bf16"), (4, 64, 16, 64, 0, 1, 0, "bf16"), (2, 128, 16, 900, 16, 1, 0, "fp32"),
    (8, 64, 16, 530, 9, 1, 32, "fp32"),
])
@pytest.mark.parametrize("varlen", [False, True])
def test_decode_matches_oracle(G, d, m, T, top_k, n_init, window, dtype, varlen):
    B, Hkv, L = 3, 2, T * m
    log(f"[decode] G={G} d={d} m={m} T={T} k={top_k} {dtype} varlen={varlen}")
    g = torch.Generator().manual_seed(T + G)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q = torch.randn(B, 1, G * Hkv, d, generator=g).to(dt)
    k, v = (torch.randn(B, L, Hkv, d, generator=g).to(dt) for _ in "kv")
    punct = (torch.rand(B, L, generator=g) < 0.1).to(torch.uint8)
    cfg = phsa.Config(block_size=m, top_k=top_k, n_init_blocks=n_init, window=window)
    lens = [L, L // 2 + 1, 1] if varlen else [L] * B
    kc = phsa.compress(k.cuda(), punct.cuda(), cfg)
    if varlen:
        sel, o, lse = phsa.decode_varlen(q.cuda(), k.cuda(), v.cuda(), kc, torch.tensor(lens, dtype=torch.int32).cuda(),
                                         cfg)
    else:
        sel, o, lse = phsa.decode(q.cuda(), k.cuda(), v.cuda(), kc, cfg)
    qh, kh, vh, kch = (to_np(x) for x in (q, k, v, kc))
    for b, n in enumerate(lens):
        pad = -(-n // m) * m
        one = slice(b, b + 1)
        ref, kth, gap = oracle.select(qh[one], kch[one, :, :pad // m], m, top_k, n_init, window, d ** -0.5, pad,
                                      q_pos0=n - 1)
        check_sel(sel[one].cpu().numpy(), ref, kth, gap,
                  lambda i: oracle.score_row(qh[one], kch[one, :, :pad // m], m, d ** -0.5, pad, 0, 0, i[1]))
        o_r, lse_r = oracle.attn_fwd(qh[one], kh[one, :pad], vh[one, :pad], sel[one].cpu().numpy(), m, d ** -0.5,
                                     q_pos0=n - 1)
        np.testing.assert_allclose(to_np(o[one]), o_r, atol=O_TOL[dtype], rtol=0)
        np.testing.assert_allclose(to_np(lse[one]), lse_r, atol=O_TOL[dtype], rtol=0)


@pytest.mark.parametrize("T,top_k", [(100, 5), (500, 16), (2048, 16), (2048, 32), (1100, 12)])
@pytest.mark.parametrize("kind", ["ties", "few_values", "one_lane", "one_slice"])
def test_decode_selection_order(T, top_k, kind):
    B, Hkv, d, m = 2, 2, 128, 16
    log(f"[decode] order {kind} T={T} k={top_k}")
    t = torch.arange(T, dtype=torch.float64)
    f = {"ties": torch.zeros(T, dtype=torch.float64), "few_values": (t * 7 % 5) / 8,
         "one_lane": torch.where(t % 64 == 9, 2.0 + t / 4096, t / 8192),
         "one_slice": torch.where((t > T // 3) & (t < T // 3 + 40), 2.0 - t / 4096, t / 8192)}[kind]
    kc = torch.zeros(B, Hkv, T, d)
    kc[..., 0] = f.float()
    q = torch.zeros(B, 1, 2 * Hkv, d)
    q[..., 0] = 1.0
    kv = torch.zeros(B, T * m, Hkv, d, dtype=torch.bfloat16)
    cfg = phsa.Config(block_size=m, top_k=top_k, n_init_blocks=1, window=0)
    sel, _, _ = phsa.decode(q.bfloat16().cuda(), kv.cuda(), kv.cuda(), kc.cuda(), cfg)
    ref, _, _ = oracle.select(q.numpy(), kc.double().numpy(), m, top_k, 1, 0, d ** -0.5, T * m)
    np.testing.assert_array_equal(sel.cpu().numpy(), ref)
