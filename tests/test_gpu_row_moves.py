"""The row movements at the edges of their kernels: k with a form of its own (1, 2, 4) and without (3, 8), one piece of 16 bytes to
several wavefronts' worth per row, one token, and more pieces than one round of the largest grid (8192 workgroups of 256) takes.
Bar and references are those of test_gpu_reorder.py.
"""
import pytest

import test_gpu_reorder as reorder
from paper_2103_13262_amd.synth import Workload

pytestmark = pytest.mark.gpu

CASES = [(1, 32, 3, 1, "f32"), (1, 32, 8, 8, "bf16"), (7, 96, 4, 4, "bf16"), (65, 1056, 5, 4, "f32"), (33, 288, 9, 8, "f32"),
         (129, 544, 6, 3, "bf16"), (257, 2048, 4, 2, "bf16"), (31000, 544, 11, 2, "bf16"), (16500, 512, 7, 1, "f32")]


@pytest.mark.parametrize("N,d,E,k,dtype", CASES, ids=lambda v: str(v))
def test_row_moves_at_the_edges(N, d, E, k, dtype):
    reorder.test_scatter_gather_and_their_backwards(Workload("moves", N, d, 32, E, k, dtype, 0.0, 900 + N % 89))
