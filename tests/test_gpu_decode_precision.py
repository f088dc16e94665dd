"""bf16 decode sums its probabilities times values at float32 precision: O is the bf16
rounding of the exact value, but for values within a float32 error of a rounding
boundary.  That error is some 2^-22 of O's scale against a spacing of 2^-8 between bf16
values, so a few in 10000 may round the other way (measured 0 to 4e-4, the largest
on the fewest values); weights of 16 bits round 1.6e-3 to 2.6e-3 wrongly."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_02819_amd import phsa
from tests.gpu_common import log, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("softmax_sum", [False, True])
@pytest.mark.parametrize("G,d,m,L", [(2, 128, 64, 4096), (8, 64, 16, 8192), (1, 128, 32, 2048), (4, 128, 16, 16384)])
def test_output_is_rounded_once(G, d, m, L, softmax_sum):
    B, Hkv = (16, 8) if L <= 8192 else (2, 4)   # the second: scored in slices unless softmax_sum
    g = torch.Generator().manual_seed(L + G)
    q = torch.randn(B, 1, G * Hkv, d, generator=g).bfloat16()
    k, v = (torch.randn(B, L, Hkv, d, generator=g).bfloat16() for _ in "kv")
    cfg = phsa.Config(block_size=m, top_k=12, n_init_blocks=1, window=2 * m, softmax_sum=softmax_sum)
    kc = phsa.compress(k.cuda(), torch.zeros(B, L, dtype=torch.uint8).cuda(), cfg)
    sel, o, _ = phsa.decode(q.cuda(), k.cuda(), v.cuda(), kc, cfg)
    ref, _ = oracle.attn_fwd(to_np(q), to_np(k), to_np(v), sel.cpu().numpy(), m, d ** -0.5)
    wrong = float((o.cpu() != torch.from_numpy(ref).bfloat16()).double().mean())
    log(f"[decode] G={G} d={d} m={m} L={L}: {wrong:.2e} of {o.numel()} values rounded the other way")
    assert wrong < 1e-3
