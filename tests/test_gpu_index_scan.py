"""Both ways to sum the index's tile counts, by the fill's workgroups and by the scan
kernel (more than 512 workgroups), with one tile per (b, g), with several and a
ragged last one, with fewer rows than keys and with the most LDS that a tile takes
(2048 blocks, 64 slots); float32 takes the same index."""
import pytest

from paper_2601_02819_amd.inputs import Workload
from tests.test_gpu_parity import run_full

pytestmark = pytest.mark.gpu


def wl(name, B, Lq, Lk, Hq, Hkv, d, m, top_k, dtype="bf16", n_init=1):
    return Workload(name, B, Lq, Lk, Hq, Hkv, d, m, top_k, n_init, 0, dtype)


@pytest.mark.parametrize("case", [
    wl("fill_512", 64, 64, 128, 8, 8, 64, 64, 1),
    wl("scan_520_of_1_tile", 65, 64, 128, 8, 8, 64, 64, 1),
    wl("scan_172_of_3_tiles", 43, 520, 576, 8, 4, 64, 64, 2),
    wl("scan_9_of_65_tiles_fp32", 9, 16400, 16400, 1, 1, 64, 16, 1, "fp32"),
    wl("most_lds_fp32", 1, 300, 32768, 1, 1, 64, 16, 32, "fp32", n_init=31),
], ids=lambda c: c.name)
def test_index_scan_forms(case):
    run_full(case)
