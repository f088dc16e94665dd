"""phsa_cache_append over its range of widths (16-byte chunks per token row, key slices
per chunk), block sizes and types: the token's rows, flag and length, the
representatives of the blocks it completes against the oracle, and nothing else
touched."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import log, to_np

pytestmark = pytest.mark.gpu


def check(B, Hkv, d, m, dtype):
    cap = 4 * m
    log(f"[append] B={B} Hkv={Hkv} d={d} m={m} {dtype}")
    g = torch.Generator().manual_seed(Hkv * d + m)
    kc0 = torch.randn(B, Hkv, cap // m, d, generator=g)
    k, v = (torch.randn(B, cap, Hkv, d, generator=g).to(dtype) for _ in "kv")
    kn, vn = (torch.randn(B, Hkv, d, generator=g).to(dtype) for _ in "kv")
    p = (torch.rand(B, cap, generator=g) < 0.2).to(torch.uint8)
    p[1], p[2] = 0, 1                                          # a block without flags, one with all
    pn = torch.tensor([1, 0, 1, 0, 1, 1, 0, 1], dtype=torch.uint8).repeat(B // 8)
    p[5, :m], p[5, 2 * m:] = 0, 0                              # its only flag is the newest token's
    # one token short of a block's end, of the cache's end, in a block, at its start, full
    lens = torch.tensor([m - 1, 2 * m - 1, 3 * m - 1, 4 * m - 1, 2 * m - 2, m - 1, 2 * m, 4 * m],
                        dtype=torch.int32).repeat(B // 8)
    dk, dv, dp, dl, dkc = (x.clone().cuda() for x in (k, v, p, lens, kc0))
    cfg = phsa.Config(block_size=m, top_k=2, lam=0.3)
    phsa.cache_append(kn.cuda(), vn.cuda(), pn.cuda(), dk, dv, dp, dl, dkc, cfg)
    for b, n in enumerate(lens.tolist()):
        if n < cap:
            k[b, n], v[b, n], p[b, n] = kn[b], vn[b], pn[b]
    assert torch.equal(dk.cpu(), k) and torch.equal(dv.cpu(), v) and torch.equal(dp.cpu(), p)
    assert dl.tolist() == [min(n + 1, cap) for n in lens.tolist()]
    got, want = dkc.cpu().numpy(), kc0.numpy().copy()
    done = np.zeros(want.shape[:3], bool)
    ref = oracle.compress(to_np(k), p.numpy(), m, 0.3)
    for b, n in enumerate(lens.tolist()):
        if n < cap and (n + 1) % m == 0:
            done[b, :, n // m] = True
    np.testing.assert_array_equal(got[~done], want[~done])
    # float32 sums of at most 64 keys of size about 4 in any order: 64 * 4 * 2^-23
    np.testing.assert_allclose(got[done], ref[done], atol=4e-5, rtol=0)


@pytest.mark.parametrize("Hkv", [1, 3, 8, 16, 72])   # 72: more chunks than threads (d 128, float32: 2304)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("m", [16, 32, 64])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_append_completes_blocks(Hkv, d, m, dtype):
    check(8, Hkv, d, m, dtype)


@pytest.mark.parametrize("B", [256, 264, 512, 520])   # workgroups of 1024, 512, 512 and 256 threads
@pytest.mark.parametrize("Hkv,d,m,dtype", [(1, 64, 64, torch.bfloat16), (3, 128, 16, torch.bfloat16),
                                           (4, 128, 64, torch.bfloat16), (5, 128, 32, torch.float32)])
def test_many_sequences(B, Hkv, d, m, dtype):
    check(B, Hkv, d, m, dtype)
