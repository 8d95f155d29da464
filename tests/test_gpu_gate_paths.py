"""Which gate kernel a batch gets, and that every one of them routes as the oracle does: a workgroup per token up to a token count that
depends on sizes and type, tiled kernels above.  Every pair below lies on the two sides of that line for one tiled kernel:
up to 16 experts; 17 to 32 with logits in fp64 (fp32, or logits stored); bf16 with a block of 64, 128 and 256 experts; and blocks
of 64 experts in fp64, with features that end in a partial slab.  The kernels leave their mark in the list of tokens whose every logit was
evaluated in fp64: the workgroup per token lists all of them, the bf16 kernel the few that it could not settle, the others
leave the list alone.  Inputs are small integers with duplicated gate columns and a zero row: exact ties everywhere.
"""
import numpy as np
import pytest

from harness import GpuRun, check_plan_exact
from paper_2103_13262_amd import binding as B
from paper_2103_13262_amd.synth import Workload, f32_to_bf16_bits, make_inputs

pytestmark = pytest.mark.gpu

# largest batch of the small kernel, d, E, k, dtype, stored logits ("": none, "scores": scores over all experts, "balance": statistics)
LINES = [(512, 1024, 8, 2, "bf16", ""), (512, 512, 12, 2, "f32", ""), (256, 96, 12, 1, "bf16", "scores"),
         (1024, 64, 24, 2, "f32", ""), (1024, 96, 29, 3, "f32", "scores"), (768, 64, 32, 4, "bf16", "scores"), (512, 64, 24, 2, "bf16", "balance"),
         (1024, 64, 40, 3, "bf16", ""), (768, 64, 100, 2, "bf16", ""), (1280, 64, 200, 8, "bf16", ""),
         (1024, 6144, 64, 8, "bf16", ""),       # (rows that do not fit the LDS of the tiled kernel for few tokens)
         (2048, 160, 70, 3, "f32", ""), (1536, 288, 70, 2, "bf16", "scores"), (1024, 288, 300, 3, "bf16", "")]
# and far beyond it: several workgroups per compute unit
CASES = [(n + more, *rest, more == 0) for n, *rest in LINES for more in (0, 1)] + [
    (9000, 64, 24, 2, "f32", "", False), (5000, 96, 29, 3, "bf16", "balance", False), (5000, 64, 32, 8, "f32", "scores", False)]


@pytest.mark.parametrize("N,d,E,k,dtype,stored,small", CASES, ids=lambda v: str(v))
def test_gate_on_both_sides_of_the_line(N, d, E, k, dtype, stored, small):
    print(f"[case] N {N} d {d} E {E} k {k} {dtype} {stored or 'plain'}", flush=True)
    w = Workload("paths", N, d, 32, E, k, dtype, 0.0, 700 + N % 97, 0.0, stored == "scores")
    inputs = make_inputs(w, with_dy=False)
    g = np.random.default_rng(N * 31 + E)
    X = g.integers(-3, 4, (N, d)).astype(np.float32)
    Wg = g.integers(-2, 3, (d, E)).astype(np.float32) / 16
    X[N // 2] = 0
    Wg[:, E - 1] = Wg[:, 0]
    Wg[:, E // 2] = Wg[:, 1]
    cast = f32_to_bf16_bits if dtype == "bf16" else (lambda a: a)
    inputs.update(X=cast(X), Wg=cast(Wg), bg=np.zeros(E, np.float32))
    run = GpuRun(w, inputs, balance_stats=int(stored == "balance"))
    off, n = B.moe_workspace_region(run.desc, "gate_uncertified")
    listed = run.workspace[off:off + n].view(run.torch.int32)
    listed.fill_(-1)
    run.plan()
    run.torch.cuda.synchronize()
    run.check_guards()
    ref = check_plan_exact(run, inputs)
    count = int(listed[0])
    if small:
        assert count == N and bool((listed[1:] == run.torch.arange(N, dtype=run.torch.int32, device=run.device)).all())
    elif dtype == "bf16" and 16 < E <= 256 and not stored:
        assert 1 <= count < N and N // 2 in listed[1:1 + count].tolist()      # (the zero row: all logits equal)
    else:
        assert count == -1
    if stored:                                                               # the probabilities that the backward pass and the statistics read
        prob = run.torch.empty(E, device=run.device)
        B.moe_balance_stats(run.desc, run.plan_struct, None, prob, None, run.workspace, run.ws_bytes, run.stream())
        p = np.exp(ref["logits"] - ref["logits"].max(1, keepdims=True))
        # fp64 throughout, one rounding to fp32 (2^-24) at the end
        np.testing.assert_allclose(prob.cpu().numpy(), (p / p.sum(1, keepdims=True)).mean(0), rtol=1e-6, atol=1e-12)
