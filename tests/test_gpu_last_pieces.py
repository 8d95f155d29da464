"""Backward pair launches whose big tiles leave few workgroups free: the last pieces behind them, against torch in fp32.

An expert's whole blocks of 256 rows run in 256 x 256 tiles, its last piece in 128 x 256 tiles behind them: on the
workgroups that the big tiles' last round left free while those get at most two each, round all workgroups otherwise.  With 32
workgroups per XCD the rows below leave 1, 4 (exactly two tiles each, and one tile more), and all of them free.
"""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,E,rest", [(62, 20, 5), (56, 16, 128), (56, 17, 1), (64, 9, 100)])
def test_last_pieces(blocks, E, rest):
    import torch

    print(f"[case] blocks {blocks} E {E} rest {rest}", flush=True)
    d, h, dev = 1024, 2048, torch.device("cuda:0")
    rows = [256 * (blocks // E + (e < blocks % E)) + rest for e in range(E)]
    N = sum(rows)
    g = torch.Generator(device=dev)
    g.manual_seed(blocks + E)
    normal = lambda shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, std, generator=g)
    expert = torch.repeat_interleave(torch.arange(E, device=dev), torch.tensor(rows, device=dev))[torch.randperm(N, generator=g, device=dev)]
    X, Wg = normal((N, d)), torch.zeros((d, E), dtype=torch.bfloat16, device=dev)
    X[:, :E] = 0                                   # one feature per expert decides: the experts' row counts are exact
    X[torch.arange(N, device=dev), expert] = 1
    Wg[torch.arange(E), torch.arange(E)] = 1
    W1, W2, dY = normal((E, d, h), 0.02), normal((E, h, d), 0.02), normal((N, d))
    desc = B.make_desc(N, d, h, E, 1)
    buf = B.MoeLayerBuffers(desc, dev)
    Y, dX, dWg, dW1, dW2 = (torch.empty_like(t) for t in (dY, X, Wg, W1, W2))
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws, st)
    B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, torch.empty(max(E, 4), device=dev), dW1, dW2, *ws, st)
    assert buf.counts.tolist() == rows

    def region(name, width):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(torch.bfloat16).view(N, width)

    dZ, dXs, Xs = region("dZ", h), region("dXs", d), region("Xs", d)
    r0 = 0
    for e, n in enumerate(rows):
        seg = slice(r0, r0 + n)
        r0 += n
        a, w, x = dZ[seg].float(), W1[e].float(), Xs[seg].float()
        for name, got, ref, size, depth in (("dXs", dXs[seg], a @ w.T, a.abs() @ w.T.abs(), h), ("dW1", dW1[e], x.T @ a, x.T.abs() @ a.abs(), n)):
            # exact products; both sums round by at most depth * 2^-24 of the terms' size each, the result to bf16 by 2^-9 of itself
            bound = 2 * depth * 2.0 ** -24 * size + 2.0 ** -8 * ref.abs() + 1e-30
            assert bool(((got.float() - ref).abs() <= bound).all()), (name, e)
