"""Weight gradients in tiles of 128 x 256 (few tiles, or fp32 gradients that are added to), in launches of their own and behind the rows products, there also with an
expert's rows cut into ranges (CUT: thousands of rows in one expert, none, one or a few blocks of 32 in others, so that some ranges hold no block; that the rule cuts them is
checked with the rule itself, compiled for the host): edges of a tile in both directions, experts without rows, with one, 31 to 33
and more rows, stored in bf16 or fp32, added to or not, twice with the same result, against fp64 sums of the same bf16 operands.  The operands are small integers, so every product and
every sum is exact in fp32; the only rounding is the result's to bf16 (2^-9 of its magnitude)."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu

ROWS = {5: [0, 1, 31, 33, 200], 3: [64, 65, 700], 1: [300], 2: [2100, 33], 4: [1, 4000, 0, 321], 6: [9000, 0, 1, 33, 700, 1],
        "one": [9768], "two": [9000, 1], "three": [9000, 0, 1], "blocks": [6000, 70, 3001]}
CUT = [("one", 384, 1408), ("two", 128, 96), ("three", 128, 96), ("three", 288, 544), ("blocks", 160, 320)]


@pytest.mark.parametrize("grad,accumulate", [("bf16", 0), ("f32", 0), ("f32", 1), ("bf16", 1)])
@pytest.mark.parametrize("rows_of,d,h", [(5, 128, 256), (5, 160, 288), (3, 384, 4096), (1, 1056, 2080), (3, 32, 64), (5, 96, 544), (2, 160, 1056), (4, 544, 288), (2, 1088, 2080), (6, 128, 96), *CUT])
def test_weight_gradients(rows_of, d, h, grad, accumulate):
    import torch

    rows = ROWS[rows_of]
    E = len(rows)
    print(f"[case] rows {rows} d {d} h {h} {grad} accumulate {accumulate}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(E * d + h)
    N = sum(rows)
    expert = torch.repeat_interleave(torch.arange(E, device=dev), torch.tensor(rows, device=dev))[torch.randperm(N, generator=g, device=dev)]
    X, Wg = torch.randint(-2, 3, (N, d), generator=g, device=dev).bfloat16(), torch.zeros((d, E), dtype=torch.bfloat16, device=dev)
    X[:, :E] = 0
    X[torch.arange(N, device=dev), expert] = 1     # one feature per expert decides: the experts' row counts are exact
    Wg[torch.arange(E), torch.arange(E)] = 1
    gt = torch.float32 if grad == "f32" else torch.bfloat16
    # weights in the place of their own gradients: every gradient gets a launch of its own (up to 1000 rows; with more, beside the weights)
    desc = B.make_desc(N, d, h, E, 1, B.MOE_BF16, B.MOE_F32 if grad == "f32" else B.MOE_BF16, accumulate)
    buf = B.MoeLayerBuffers(desc, dev)
    ws = (buf.workspace, buf.ws_bytes, buf.stream())
    size = E * d * h
    mem1, mem2 = (torch.zeros(size, dtype=gt, device=dev) for _ in range(2))
    if accumulate:
        for m in (mem1, mem2):
            m.view(torch.bfloat16)[:size] = torch.randint(-2, 3, (size,), generator=g, device=dev).bfloat16() / 64
    W1, W2 = mem1.view(torch.bfloat16)[:size].view(E, d, h), mem2.view(torch.bfloat16)[:size].view(E, h, d)
    if N > 1000:
        W1, W2 = (torch.randint(-2, 3, w.shape, generator=g, device=dev).bfloat16() / 64 for w in (W1, W2))
    dY = torch.randint(-2, 3, (N, d), generator=g, device=dev).bfloat16()
    Y, dX, dWg, dbg = torch.empty_like(X), torch.empty_like(X), torch.zeros((d, E), dtype=gt, device=dev), torch.zeros(max(E, 4), device=dev)
    before = [m.clone().double() for m in (mem1, mem2)]
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws)
    assert buf.counts[:E].tolist() == rows
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws)

    def region(name, width):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(torch.bfloat16).view(N, width)

    region("H", h).copy_(torch.randint(-2, 3, (N, h), generator=g, device=dev))
    backward = lambda: B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, dbg, mem1, mem2, *ws)
    backward()
    if N > 1000:                                   # (up to that many the first call has overwritten the weights)
        first = [m.clone() for m in (mem1, mem2)]
        for m, was in zip((mem1, mem2), before):
            m.copy_(was)
        backward()
        assert torch.equal(first[0], mem1) and torch.equal(first[1], mem2)
    perm = buf.perm[:N].long()
    for mem, was, a, b in ((mem1, before[0], X[perm], region("dZ", h)), (mem2, before[1], region("H", h), dY[perm])):
        want = torch.stack([x.double().T @ y.double() for x, y in zip(a.split(rows), b.split(rows))])
        bound = torch.stack([x.double().abs().T @ y.double().abs() for x, y in zip(a.split(rows), b.split(rows))]) * 2.0 ** -24 * (max(rows) + 1)
        if accumulate:
            want = want + was.view_as(want)
            bound = bound + want.abs() * 2.0 ** -24
        if grad == "bf16":
            bound = bound + want.abs() * 2.0 ** -8
        got = mem.view_as(want).double()
        assert bool(((got - want).abs() <= bound).all()), float(((got - want).abs() - bound).max())
