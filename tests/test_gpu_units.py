"""Work units of the sparse attention kernels at the edges of their sizes, against
the oracle (the bars of test_gpu_parity): lists of exactly one unit, one entry
more and one less, a single entry, many units per list, and more blocks than the
list scan's workgroup has threads."""
import pytest

from paper_2601_02819_amd.inputs import Workload
from tests.test_gpu_parity import run_full

pytestmark = pytest.mark.gpu


def wl(name, Lq, Lk, Hq, Hkv, d, top_k, n_init=1):
    return Workload(name, 1, Lq, Lk, Hq, Hkv, d, 64, top_k, n_init, 0, "bf16")


# Block 0 is on every row's list, so its list has Lq entries; small problems have
# forward units of 64 / G and backward units of 128 / G entries.
@pytest.mark.parametrize("case", [
    wl("unit_g1", 128, 1024, 1, 1, 128, 2),
    wl("unit_g1_less", 127, 1024, 1, 1, 128, 2),
    wl("unit_g1_more", 129, 1024, 1, 1, 128, 2),
    wl("unit_g8", 17, 512, 8, 1, 64, 3),
    wl("unit_g4_many", 1537, 1600, 8, 2, 64, 5),
    wl("one_slot", 300, 320, 2, 1, 64, 0, n_init=0),  # Ksel = 1
    wl("tiles_33", 8300, 8320, 1, 1, 64, 3),          # 33 index tiles: the fill sums two batches of counts per block
    wl("tiles_65", 16500, 16512, 1, 1, 64, 3),        # 65 tiles: three batches
    wl("blocks_1030", 130, 1030 * 64, 2, 1, 64, 6),   # 1030 blocks: three rounds of the 512-thread scan
], ids=lambda c: c.name)
def test_units_match_oracle(case):
    run_full(case)
