"""bf16 products whose operands lie further apart than the main loop's 32-bit offsets reach: rows of 2^22 values and more (the
kernels with 64-bit offsets, in 64 x 256 tiles and in size classes), and rows gathered from an X of more than 4 GB (the same kernels: no scattered
copy is written)."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


def _close(got, a, b, what):
    """got = a @ b with exact products: the sum rounds by at most depth * 2^-24 of the terms' size, the result to bf16."""
    a, b = a.float(), b.float()
    bound = 2 * a.shape[1] * 2.0 ** -24 * (a.abs() @ b.abs()) + 2.0 ** -8 * (a @ b).abs() + 1e-30
    assert bool(((got.float() - a @ b).abs() <= bound).all()), what


# 70: 64 x 256 tiles (below 96 rows per expert); 300: FC1 and dZ in size classes (a whole block and a last piece), FC2 and dXs, with few tiles, not
@pytest.mark.parametrize("N", [70, 300])
def test_rows_of_millions_of_values(N):
    import torch

    d, h, E, dev = 32, 1 << 22, 1, torch.device("cuda:0")
    print(f"[case] N {N} d {d} h {h}", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, 0.3, generator=g)
    # hidden units that are not zero: few, so that their sums can be stated; first and last among them
    at = torch.cat([torch.tensor([0, 31, h // 2, h - 33, h - 1], device=dev), torch.randint(64, h - 64, (60,), generator=g, device=dev)]).unique()
    X, dY, Wg = normal(N, d), normal(N, d), normal(d, E)
    W1, W2 = torch.zeros((E, d, h), dtype=torch.bfloat16, device=dev), torch.zeros((E, h, d), dtype=torch.bfloat16, device=dev)
    W1[0][:, at], W2[0][at] = normal(d, len(at)), normal(len(at), d)
    desc = B.make_desc(N, d, h, E, 1)
    buf = B.MoeLayerBuffers(desc, dev)
    Y, dX, dWg, dW1, dW2 = (torch.full_like(t, 7) for t in (dY, X, Wg, W1, W2))
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws, st)
    B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, torch.empty(4, device=dev), dW1, dW2, *ws, st)

    def region(name, width):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(torch.bfloat16).view(N, width)

    Z, H, dZ, dXs = region("Z", h), region("H", h), region("dZ", h), region("dXs", d)
    for name, whole, part in (("Z", Z, Z[:, at]), ("H", H, H[:, at]), ("dZ", dZ, dZ[:, at]), ("dW1", dW1, dW1[0][:, at]), ("dW2", dW2, dW2[0][at])):
        assert int(whole.count_nonzero()) == int(part.count_nonzero()) > 0, name
    _close(Z[:, at], X, W1[0][:, at], "Z")
    _close(Y, H[:, at], W2[0][at], "Y")
    _close(dXs, dZ[:, at], W1[0][:, at].T, "dXs")
    _close(dW1[0][:, at], X.T, dZ[:, at], "dW1")
    _close(dW2[0][at], H[:, at].T, dY, "dW2")


def test_a_reduction_over_millions_in_size_classes():
    import torch

    N, d, h, E, dev = 1600, 32, 1 << 22, 1, torch.device("cuda:0")        # six whole blocks and a last piece of 64 rows
    print(f"[case] N {N} d {d} h {h}", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, 0.3, generator=g)
    at = torch.randint(0, h, (60,), generator=g, device=dev).unique()
    X, Wg, W1 = normal(N, d), normal(d, E), torch.zeros((E, d, h), dtype=torch.bfloat16, device=dev)
    W2 = torch.zeros((E, h, d), dtype=torch.bfloat16, device=dev)
    W1[0][:, at], W2[0][at] = normal(d, len(at)), normal(len(at), d)
    desc = B.make_desc(N, d, h, E, 1)
    buf = B.MoeLayerBuffers(desc, dev)
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
    Y = torch.full_like(X, 7)
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws, st)
    off, n = B.moe_workspace_region(desc, "H")
    _close(Y, buf.workspace[off:off + n].view(torch.bfloat16).view(N, h)[:, at], W2[0][at], "Y")


def test_x_of_more_than_4_gb():
    import torch

    d, h, E, dev = 2048, 32, 2, torch.device("cuda:0")
    N = (1 << 20) + 33
    print(f"[case] N {N} d {d} h {h}", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(6)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, 0.1, generator=g)
    X, Wg, W1, W2 = normal(N, d), normal(d, E), normal(E, d, h), normal(E, h, d)
    desc = B.make_desc(N, d, h, E, 1)
    buf = B.MoeLayerBuffers(desc, dev)
    Y = torch.empty_like(X)
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
    off, n = B.moe_workspace_region(desc, "Xs")
    Xs = buf.workspace[off:off + n].view(torch.int32)
    Xs.fill_(0x5a5a5a5a)
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws, st)
    assert bool((Xs == 0x5a5a5a5a).all())
    at = torch.cat([torch.arange(40, device=dev), torch.arange(N - 40, N, device=dev), torch.randint(0, N, (400,), generator=g, device=dev)])
    row, expert = buf.pos[:N].long()[at], buf.topk_idx[:, 0].long()[at]

    def region(name, width):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(torch.bfloat16).view(N, width)[row]

    Z, H = region("Z", h), region("H", h)
    for e in range(E):
        m = expert == e
        assert int(m.sum()) > 50
        _close(Z[m], X[at][m], W1[e], "Z")
        _close(Y[at][m], H[m], W2[e], "Y")
