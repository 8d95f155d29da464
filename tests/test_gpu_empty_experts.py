"""Backward pass of a layer most of whose experts have no rows: their gradients are zeros (or stay as they were, accumulating), and writing them takes
many workgroups: the gate's part of the pass takes no longer than twice as long as moe_scatter_backward, which has a workgroup per expert for its sums."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


def _layer(torch, N, d, h, E, k, dtype, accumulate):
    print(f"[case] N {N} d {d} h {h} E {E} k {k} {dtype} accumulate {accumulate}", flush=True)
    dev = torch.device("cuda:0")
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    dt = B.MOE_BF16 if dtype == "bf16" else B.MOE_F32
    grad = torch.float32 if accumulate else act
    g = torch.Generator(device=dev)
    g.manual_seed(N + d + E)
    new = lambda *s: torch.empty(s, dtype=act, device=dev).normal_(generator=g)
    X, Wg, dY, W1, W2 = new(N, d), new(d, E), new(N, d), new(E, d, h), new(E, h, d)
    desc = B.make_desc(N, d, h, E, k, dt, B.MOE_F32 if accumulate else dt, accumulate)
    buf = B.MoeLayerBuffers(desc, dev)
    ws = (buf.workspace, buf.ws_bytes, buf.stream())
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws)
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, torch.empty_like(X), *ws)
    new_grad = lambda *s: torch.full(s, 0.5, dtype=grad, device=dev)
    dW1, dW2 = new_grad(E, d, h), new_grad(E, h, d)

    def outputs():
        return torch.empty_like(X), new_grad(d, E), torch.full((max(E, 4),), 0.5, device=dev)

    def backward(dX, dWg, dbg):
        B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, dbg, dW1, dW2, *ws)

    def region(name, dtype_):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(dtype_)

    def separate(dX, dWg, dbg):
        Xs, dXs, dl = region("Xs", act).clone(), region("dXs", act).clone(), region("dl", torch.float32).clone()
        return lambda: B.moe_scatter_backward(desc, buf.plan, Wg, Xs, dXs, dl, dX, dWg, dbg, *ws)

    return desc, buf, ws, outputs, backward, separate, region


@pytest.mark.parametrize("dtype,accumulate", [("bf16", 0), ("f32", 0), ("bf16", 1)])
@pytest.mark.parametrize("N,d,h,E,k", [(8, 2048, 96, 256, 2), (100, 2080, 64, 1000, 1), (1, 544, 1056, 17, 1), (40, 32, 32, 1024, 3), (3, 1024, 32, 33, 2)])
def test_gradients(N, d, h, E, k, dtype, accumulate):
    import torch

    desc, buf, ws, outputs, backward, separate, region = _layer(torch, N, d, h, E, k, dtype, accumulate)
    empty = buf.counts[:E] == 0
    assert int(empty.sum()) > E // 3
    got, want = outputs(), outputs()
    backward(*got)
    separate(*want)()
    for a, b in zip(got, want):
        assert torch.equal(a[:E] if a.dim() == 1 else a, b[:E] if b.dim() == 1 else b)
    rest = 0.5 if accumulate else 0.0
    assert bool((got[1][:, empty] == rest).all()) and bool((got[2][:E][empty] == rest).all())
    db1, db2 = (torch.full((E, w), 0.5, device=buf.counts.device) for w in (h, d))
    B.moe_bias_backward(desc, buf.plan, db1, db2, *ws)
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    for db, name in ((db1, "dZ"), (db2, "dYs")):
        rows = region(name, act).view(N * k, -1).double()
        sums = torch.stack([s.sum(0) for s in rows.split(buf.counts[:E].tolist())])
        size = torch.stack([s.abs().sum(0) for s in rows.split(buf.counts[:E].tolist())])
        # fp32 sums of at most N k terms and what was there
        assert bool(((db.double() - sums - rest).abs() <= (size + rest) * (N * k + 1) * 2.0 ** -24).all())
        assert bool((db[empty] == rest).all())


def test_time():
    import torch

    desc, buf, ws, outputs, backward, separate, _ = _layer(torch, 100, 2048, 32, 1000, 2, "bf16", 0)
    out = outputs()
    backward(*out)
    call = separate(*outputs())
    whole, two = [], []
    for _ in range(5):
        B.moe_profile_enable(True)
        for _ in range(5):
            backward(*out)
        torch.cuda.synchronize()
        launches, ms = B.moe_profile_read()["gate_bwd"]
        B.moe_profile_enable(False)
        whole.append(ms / launches)
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(5):
            call()
        end.record()
        torch.cuda.synchronize()
        two.append(start.elapsed_time(end) / 5)
    print(f"gate backward {min(whole) * 1e3:.1f} us, moe_scatter_backward {min(two) * 1e3:.1f} us")
    assert min(whole) <= 2 * min(two)
