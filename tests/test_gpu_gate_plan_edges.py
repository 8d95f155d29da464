"""Routing (gate, selection, counting, placing) at the sizes where its kernels change over, bit for bit against the oracle.

The gate takes a workgroup per token for small batches (pieces of 16 bytes that hold one feature or several; one or more pieces
per expert row; up to 1024 experts; two workgroups per compute unit above 256 tokens); where it stops doing so is
test_gpu_gate_paths.py's subject.  The plan counts the assignments itself up
to 8192, from chunk histograms above, orders up to 256 experts by counting and more by sorting, and makes its chunks longer than 1024
assignments above 262144.  Inputs are small integers with duplicated gate columns and a zero row: exact ties everywhere.
"""
import numpy as np
import pytest

from harness import GpuRun, check_plan_exact
from paper_2103_13262_amd.synth import Workload, f32_to_bf16_bits, make_inputs

pytestmark = pytest.mark.gpu

CASES = [(N, d, E, k, dt, False) for N, d, E, k, dt in (
    (1, 32, 1, 1, "bf16"), (1, 32, 1, 1, "f32"), (3, 64, 3, 2, "bf16"), (2, 2048, 16, 2, "bf16"), (5, 96, 9, 8, "f32"),
    (256, 160, 57, 3, "bf16"), (257, 160, 57, 3, "bf16"), (300, 128, 64, 2, "bf16"), (7, 512, 256, 1, "bf16"), (9, 96, 257, 4, "bf16"),
    (40, 64, 1023, 8, "bf16"), (40, 64, 1024, 8, "f32"), (520, 64, 1000, 2, "f32"), (130, 992, 255, 2, "f32"), (512, 32, 20, 4, "bf16"),
    (1024, 32, 12, 8, "bf16"), (1025, 32, 12, 8, "bf16"), (4096, 32, 300, 2, "bf16"), (8193, 32, 5, 1, "f32"),
    (33000, 32, 11, 8, "bf16"))] + [(17, 64, 40, 2, "bf16", True), (300, 96, 130, 3, "f32", True), (1, 32, 700, 8, "bf16", True)]


@pytest.mark.parametrize("N,d,E,k,dtype,score_all", CASES, ids=lambda v: str(v))
def test_routing_at_the_edges(N, d, E, k, dtype, score_all):
    w = Workload("edges", N, d, 32, E, k, dtype, 0.0, 700 + N % 97, 0.0, score_all)
    inputs = make_inputs(w, with_dy=False)
    g = np.random.default_rng(N * 31 + E)
    X = g.integers(-3, 4, (N, d)).astype(np.float32)
    Wg = g.integers(-2, 3, (d, E)).astype(np.float32)
    X[N // 2] = 0
    Wg[:, E - 1] = Wg[:, 0]
    if E > 4:
        Wg[:, E // 2] = Wg[:, 1]
    cast = f32_to_bf16_bits if dtype == "bf16" else (lambda a: a)
    inputs.update(X=cast(X), Wg=cast(Wg), bg=np.zeros(E, np.float32))
    run = GpuRun(w, inputs)
    run.plan()
    run.torch.cuda.synchronize()
    run.check_guards()
    check_plan_exact(run, inputs)
