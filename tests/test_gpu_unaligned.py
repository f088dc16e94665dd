"""Tensors that start at any element, not at a multiple of 16 bytes: the sparse forward and
decode, which copy K and V tiles straight into LDS, take them by way of registers then, and
every result is bit for bit that of the same tensors aligned."""
import pytest
import torch

from paper_2601_02819_amd import phsa
from tests.gpu_common import log

pytestmark = pytest.mark.gpu


def shifted(x, off):
    """A contiguous copy of x that starts `off` elements past a 16-byte boundary."""
    y = torch.empty(x.numel() + 16, dtype=x.dtype, device="cuda")
    y = y[off:off + x.numel()].view(x.shape)
    assert y.data_ptr() % 16 == off * x.element_size() % 16
    return y.copy_(x)


@pytest.mark.parametrize("off", [1, 2, 4])
@pytest.mark.parametrize("G,d,m,dtype", [(2, 128, 64, torch.bfloat16), (4, 64, 16, torch.bfloat16),
                                         (8, 128, 16, torch.bfloat16), (1, 64, 64, torch.bfloat16),
                                         (2, 64, 32, torch.float32), (4, 128, 64, torch.float32)])
def test_any_start(G, d, m, dtype, off):
    B, Hkv, L = 2, 2, 832
    g = torch.Generator().manual_seed(G + d + m)
    q, do = (torch.randn(B, L, G * Hkv, d, generator=g).to(dtype).cuda() for _ in "qd")
    k, v = (torch.randn(B, L, Hkv, d, generator=g).to(dtype).cuda() for _ in "kv")
    punct = (torch.rand(B, L, generator=g) < 0.1).to(torch.uint8).cuda()
    lens = torch.tensor([700, 832], dtype=torch.int32).cuda()
    cfg = phsa.Config(block_size=m, top_k=5, n_init_blocks=1, window=0)

    def calls(q, k, v, do):
        kc, sel, o, lse = phsa.forward(q, k, v, punct, cfg)
        one = q[:, -1:].contiguous()
        return (kc, sel, o, lse, *phsa.attn_bwd(q, k, v, o, do, lse, sel, cfg), *phsa.decode(one, k, v, kc, cfg),
                *phsa.decode_varlen(one, k, v, kc, lens, cfg))

    log(f"[unaligned] G={G} d={d} m={m} {dtype} off={off}")
    names = "kc sel o lse dq dk dv dsel do dlse vsel vo vlse".split()
    for name, a, b in zip(names, calls(q, k, v, do), calls(*(shifted(x, off) for x in (q, k, v, do)))):
        assert torch.equal(a, b), name


@pytest.mark.parametrize("B,Hkv,G,d,L,softmax_sum", [
    (33, 8, 2, 128, 512, False),    # more workgroups than CUs: 8 waves
    (33, 8, 4, 64, 512, True),
    (2, 3, 2, 64, 640, True),       # 16 waves
    (1, 2, 2, 128, 40960, False),   # 640 blocks: scored in slices where V is aligned
])
def test_decode_any_start(B, Hkv, G, d, L, softmax_sum):
    g = torch.Generator(device="cuda").manual_seed(B + L)
    q = torch.randn(B, 1, G * Hkv, d, generator=g, device="cuda").bfloat16()
    k, v = (torch.randn(B, L, Hkv, d, generator=g, device="cuda").bfloat16() for _ in "kv")
    cfg = phsa.Config(block_size=64, top_k=5, n_init_blocks=1, window=64, softmax_sum=softmax_sum)
    kc = phsa.compress(k, torch.zeros(B, L, dtype=torch.uint8, device="cuda"), cfg)
    log(f"[unaligned] decode B={B} Hkv={Hkv} G={G} d={d} L={L} softmax_sum={softmax_sum}")
    want = phsa.decode(q, k, v, kc, cfg)
    for name, a, b in zip(("sel", "o", "lse"), want, phsa.decode(q, shifted(k, 3), shifted(v, 5), kc, cfg)):
        assert torch.equal(a, b), name
