"""fp32 grouped products at the sizes where their two forms can go wrong, against the fp64 oracle (every tensor, 1e-4).

The sliced form (at most 512 output tiles of 64 x 64) cuts an expert's rows into 32-row tiles and the reduction into 16-deep
chunks over 16 wavefronts; the tiled form (more tiles) works in 64 x 64 x 32 blocks through two LDS buffers.  The shapes end
tiles after one row, reductions inside a chunk, before the last wavefront gets a chunk, and after an odd number of
blocks; the largest lies just above the line between the forms.
"""
import pytest

from test_gpu_parity import _full_check
from paper_2103_13262_amd.synth import Workload

pytestmark = pytest.mark.gpu

CASES = [
    Workload("one_row", 1, 32, 32, 1, 1, "f32", 0.0, 501),
    Workload("one_row_past_a_tile", 33, 32, 544, 1, 1, "f32", 0.0, 502, 0.1),
    Workload("reduction_of_17_rows", 17, 544, 32, 1, 1, "f32", 0.0, 503),
    Workload("reduction_of_257_rows", 257, 96, 288, 1, 1, "f32", 0.0, 504),
    Workload("empty_and_small_experts", 70, 64, 96, 70, 2, "f32", 0.8, 505, 0.1),     # (over 64 experts: the longer search)
    Workload("sliced_largest", 1984, 32, 512, 2, 2, "f32", 0.0, 506),
    Workload("tiled_smallest", 2100, 32, 512, 3, 2, "f32", 0.7, 507),
    Workload("tiled_odd_blocks_skewed", 1500, 352, 480, 90, 3, "f32", 1.0, 508, 0.1),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_f32_products(w):
    _full_check(w)
