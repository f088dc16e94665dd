"""The float32 kernels at their edges, against the oracle (1e-4): every group size
and head dim, blocks of 16, 32 and 64 tokens (four, two and one row tiles per
chunk), lists of one, several and no work units, an odd number of blocks, tail
query rows and a single row."""
import pytest

from paper_2601_02819_amd.inputs import Workload
from tests.test_gpu_parity import run_full

pytestmark = pytest.mark.gpu


def wl(G, d, m, Lq, Lk, B=1, Hkv=1, top_k=3, n_init=1, window=0):
    return Workload(f"fp32_g{G}_d{d}_m{m}_{Lq}of{Lk}", B, Lq, Lk, Hkv * G, Hkv, d, m, top_k, n_init, window, "fp32")


@pytest.mark.parametrize("case", [
    wl(1, 64, 16, 272, 272), wl(2, 128, 16, 336, 336), wl(4, 64, 16, 130, 1040), wl(8, 128, 16, 208, 208),
    wl(1, 128, 32, 352, 352), wl(2, 64, 32, 33, 800), wl(4, 128, 32, 160, 160, window=64), wl(8, 64, 32, 224, 224),
    wl(1, 64, 64, 320, 320), wl(4, 128, 64, 192, 192), wl(8, 128, 64, 192, 192), wl(2, 128, 64, 1, 640),
    wl(2, 64, 64, 577, 704, B=2, Hkv=2, top_k=8, n_init=2), wl(8, 64, 64, 17, 128),
], ids=lambda c: c.name)
def test_fp32_matches_oracle(case):
    run_full(case)
