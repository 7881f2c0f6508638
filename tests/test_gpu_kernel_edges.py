"""Parity at the edges of kernel variants and dispatch rules: sizes on either side of a tile, of a remainder and of
the line between two kernels, against the oracle with the tolerances of test_gpu_parity."""
import pytest

from paper_2603_08055_amd import workloads
from tests.test_gpu_parity import layer_case, s3r  # noqa: F401  (s3r: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,block,views,tpv,special,heads", [
    ("bf16", 16, 1, 230, 6, 2),       # 14 blocks = 3.5 units + 1 special unit: the last unit of a split is short
    ("bf16", 16, 2, 250, 3, 1),       # 8 + 1 units, two splits; the second ends in the special-token segment
    ("bf16", 32, 3, 401, 2, 3),       # blocks of 32, odd number of them
    ("bf16", 16, 5, 611, 61, 2),      # 305 special rows: three row groups, five special units
    ("bf16", 64, 2, 700, 1, 1),       # one row group of two rows over many splits
    ("f32", 32, 2, 411, 2, 2),        # fp32 operand parts
])
def test_special_rows_in_key_splits(s3r, oracle, dtype, block, views, tpv, special, heads):  # noqa: F811
    wl = workloads.Workload(f"splits_{dtype}_{block}_{views}x{tpv}_{special}", views, tpv, heads, 64, dtype, block, 3,
                            93, "normal")
    layer_case(s3r, oracle, wl, special, with_gate=True)
