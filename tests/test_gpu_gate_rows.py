"""The bf16 gate kernel that keeps its tokens' rows in LDS (up to some thousand tokens): its routing against the oracle's, bit for bit, at the edges of its
forms: 32, 64, 128 and 256 experts and one more, features that are no multiple of its 128-wide groups, the widest rows that fit the LDS and one step more
(where the slab kernel takes over), a last workgroup of one token, the tokens at which the slab kernel takes over, and many tokens whose every
logit has to be evaluated in fp64 (zero rows, equal gate columns), 16 in one workgroup among them.  Inputs are small integers: exact ties everywhere."""
import numpy as np
import pytest

from harness import GpuRun, check_plan_exact
from paper_2103_13262_amd import binding as B
from paper_2103_13262_amd.synth import Workload, f32_to_bf16_bits, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,E,k", [(1601, 256, 17, 2), (1601, 288, 32, 1), (1601, 416, 33, 3), (1700, 992, 64, 2), (1601, 1056, 65, 8), (1601, 544, 128, 2),
                                     (1601, 320, 129, 4), (1650, 256, 256, 2), (1601, 4480, 24, 2), (1601, 4512, 24, 2), (4096, 256, 40, 2), (4097, 256, 40, 2),
                                     (8192, 1024, 20, 1), (8193, 1024, 40, 1)])
def test_routing(N, d, E, k):
    print(f"[case] N {N} d {d} E {E} k {k}", flush=True)
    w = Workload("rows", N, d, 32, E, k, "bf16", 0.0, 900 + E)
    inputs = make_inputs(w, with_dy=False)
    g = np.random.default_rng(N + d + E)
    X = g.integers(-3, 4, (N, d)).astype(np.float32)
    Wg = g.integers(-2, 3, (d, E)).astype(np.float32) / 16
    zero = np.unique(np.concatenate([np.arange(32, 48), g.integers(0, N, 40), [N - 1]]))
    X[zero] = 0
    Wg[:, E - 1] = Wg[:, 0]
    Wg[:, E // 2] = Wg[:, 1]
    inputs.update(X=f32_to_bf16_bits(X), Wg=f32_to_bf16_bits(Wg), bg=np.zeros(E, np.float32))
    run = GpuRun(w, inputs)
    run.plan()
    run.torch.cuda.synchronize()
    run.check_guards()
    check_plan_exact(run, inputs)
    off, n = B.moe_workspace_region(run.desc, "gate_uncertified")
    listed = run.workspace[off:off + n].view(run.torch.int32)
    count = int(listed[0])
    assert len(zero) <= count < N and set(zero.tolist()) <= set(listed[1:1 + count].tolist())
