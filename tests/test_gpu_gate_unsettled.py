"""The bf16 gate kernel that keeps its tokens' rows in LDS, on tokens that its error bound cannot settle (every logit in fp64): equal gate columns, zero rows, and
rows and weights that are not finite, which unsettle all 16 tokens of a workgroup.  At 17 to 256 experts and few features, where some of the reduction's parts are
empty, against fp64 logits with ties to the lower expert; and a launch with a workgroup full of such tokens takes no more than four times as long as one without."""
import numpy as np
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["equal columns", "rows", "weights"])
@pytest.mark.parametrize("N,d,E,k", [(1601, 32, 17, 2), (1601, 96, 32, 3), (1601, 32, 64, 1), (1700, 160, 40, 8), (1601, 288, 100, 2), (1601, 32, 128, 4), (1601, 64, 129, 2),
                                     (1601, 1024, 256, 2)])
def test_routing(N, d, E, k, kind):
    import torch

    print(f"[case] {kind}: N {N} d {d} E {E} k {k}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(N + d + E)
    X = torch.empty((N, d), dtype=torch.bfloat16, device=dev).normal_(generator=g)
    Wg = torch.empty((d, E), dtype=torch.bfloat16, device=dev).normal_(0, 0.05, generator=g)
    bg = torch.linspace(0.1, 0.0, E, device=dev)
    rows = [3, 16, 31, 700, N - 1]                        # one of a workgroup, its first and last, the last workgroup's only one
    if kind == "equal columns":
        Wg[:, :17] = Wg[:, :1]
        bg[:17] = 20.0                                    # (17 equal logits, the largest of nearly every token)
    elif kind == "rows":
        X[rows[0], d - 1], X[rows[1], 0], X[rows[2], 5] = float("nan"), float("inf"), -float("inf")
        X[rows[3]], X[rows[4]] = float("nan"), 0
    else:
        Wg[1, E - 1], Wg[d - 1, 2], Wg[7, 5] = float("inf"), -float("inf"), float("nan")
    desc = B.make_desc(N, d, 32, E, k)
    buf = B.MoeLayerBuffers(desc, dev)
    B.moe_plan(desc, X, Wg, bg, buf.plan, buf.workspace, buf.ws_bytes, buf.stream())
    off, n = B.moe_workspace_region(desc, "gate_uncertified")
    listed = buf.workspace[off:off + n].view(torch.int32)
    count = int(listed[0])
    listed = set(listed[1:1 + count].tolist())
    assert len(listed) == count
    if kind == "rows":                                    # all 16 tokens around each row that is not finite
        around = {t for r in rows[:4] for t in range(r // 16 * 16, r // 16 * 16 + 16)}
        assert around <= listed and count < N
    else:
        assert count == N if kind == "weights" else count > N // 2
    logits = (X.double() @ Wg.double()).cpu().numpy() + bg.double().cpu().numpy()
    if kind == "equal columns":
        logits[:, :17] = logits[:, :1]                    # (the reference's sums differ in their last bits)
    logits[np.isnan(logits)] = -np.inf
    order = np.argsort(-logits, axis=1, kind="stable")[:, :k]
    idx = buf.topk_idx[:N * k].view(N, k).cpu().numpy()
    np.testing.assert_array_equal(idx, order)
    chosen = np.take_along_axis(logits, order, 1)
    finite = np.isfinite(chosen).all(1)
    assert finite.sum() > N // 8 or kind == "weights"
    p = np.exp(chosen[finite] - chosen[finite, :1])
    p /= p.sum(1, keepdims=True)
    w = buf.topk_w[:N * k].view(N, k).cpu().numpy()[finite]
    # one rounding to fp32; both sides' fp64 logits are off by up to d 2^-53 of their terms' size (at most some hundred)
    assert (np.abs(w - p) <= p * (2.0 ** -24 * 1.01 + 2 * d * 2.0 ** -53 * 300)).all()


def test_time():
    import torch

    N, d, E, dev = 1500, 1024, 256, torch.device("cuda:0")
    X = torch.empty((N, d), dtype=torch.bfloat16, device=dev).normal_()
    Z = X.clone()
    Z[320:336] = 0
    Wg = torch.empty((d, E), dtype=torch.bfloat16, device=dev).normal_(0, 0.02)
    desc = B.make_desc(N, d, 32, E, 2)
    buf = B.MoeLayerBuffers(desc, dev)
    times = {}
    for _ in range(5):
        for name, x in (("settled", X), ("zero rows", Z)):
            B.moe_profile_enable(True)
            for _ in range(5):
                B.moe_plan(desc, x, Wg, None, buf.plan, buf.workspace, buf.ws_bytes, buf.stream())
            torch.cuda.synchronize()
            launches, ms = B.moe_profile_read()["gate_topk"]
            B.moe_profile_enable(False)
            times.setdefault(name, []).append(ms / launches)
    print({n: f"{min(t) * 1e3:.1f} us" for n, t in times.items()})
    assert min(times["zero rows"]) <= 4 * min(times["settled"])
