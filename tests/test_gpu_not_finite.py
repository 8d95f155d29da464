"""Pre-activations that are not finite, in the backward products' small tiles: dZ = dH GeLU'(Z) is NaN where Z is NaN, dH or an exact zero
where Z is an infinity, and as without them elsewhere."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


# rows on average below 96 with columns that fill 256-wide tiles badly and more than 48 MB of weights; a deep reduction with few big tiles
@pytest.mark.parametrize("N,d,h,E", [(480, 1024, 544, 48), (500, 2048, 96, 4)])
def test_factor_at_nan_and_infinities(N, d, h, E):
    import torch

    print(f"[case] N {N} d {d} h {h} E {E}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(N)
    normal = lambda shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, std, generator=g)
    X, Wg, W1, W2, dY = normal((N, d)), normal((d, E)), normal((E, d, h), 0.02), normal((E, h, d), 0.02), normal((N, d))
    b1, b2 = torch.zeros((E, h), dtype=torch.bfloat16, device=dev), torch.zeros((E, d), dtype=torch.bfloat16, device=dev)
    desc = B.make_desc(N, d, h, E, 1)

    def run():
        buf = B.MoeLayerBuffers(desc, dev)
        ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
        Y, dX, dWg, dW1, dW2 = (torch.empty_like(t) for t in (dY, X, Wg, W1, W2))
        B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
        B.moe_forward(desc, buf.plan, X, W1, W2, b1, b2, Y, *ws, st)
        B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, torch.empty(max(E, 4), device=dev), dW1, dW2, *ws, st)
        off, n = B.moe_workspace_region(desc, "dZ")
        return buf.workspace[off:off + n].view(torch.bfloat16).view(N, h).clone()

    clean = run()
    b1[:, 3], b1[:, 32], b1[:, h - 1] = float("nan"), float("inf"), float("-inf")
    dZ = run()
    same = torch.ones(h, dtype=torch.bool, device=dev)
    same[[3, 32, h - 1]] = False
    assert torch.equal(dZ[:, same], clean[:, same])
    assert bool(dZ[:, 3].isnan().all())
    assert bool(dZ[:, 32].isfinite().all()) and int(dZ[:, 32].count_nonzero()) > 0
    assert int(dZ[:, h - 1].count_nonzero()) == 0
