"""Weight gradients added to what is there, in fp32 and in bf16, at the edges of their tiles: the new sum against the old one plus the
gradient on its own."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f32", [True, False], ids=["fp32", "bf16"])
@pytest.mark.parametrize("N,d,h,E", [(70, 32, 96, 3), (600, 288, 544, 4), (1500, 224, 800, 5), (300, 256, 256, 40)])
def test_added_to(N, d, h, E, f32):
    import torch

    print(f"[case] N {N} d {d} h {h} E {E} fp32 {f32}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(N)
    normal = lambda shape, std=1.0, t=torch.bfloat16: torch.empty(shape, dtype=t, device=dev).normal_(0.0, std, generator=g)
    X, Wg, W1, W2, dY = normal((N, d)), normal((d, E), 0.1), normal((E, d, h), 0.1), normal((E, h, d), 0.1), normal((N, d))
    kind = torch.float32 if f32 else torch.bfloat16
    before = {"dW1": normal((E, d, h), 1.0, kind), "dW2": normal((E, h, d), 1.0, kind)}

    def run(accumulate, grads):
        desc = B.make_desc(N, d, h, E, 2, B.MOE_BF16, B.MOE_F32 if f32 else B.MOE_BF16, accumulate)
        buf = B.MoeLayerBuffers(desc, dev)
        ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
        Y, dX, dWg = torch.empty_like(X), torch.empty_like(X), torch.zeros((d, E), dtype=kind, device=dev)
        B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
        B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws, st)
        B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, torch.zeros(max(E, 4), device=dev), grads["dW1"], grads["dW2"], *ws, st)
        return grads

    # (strips behind the gradients: nothing is written past them)
    strips = {n: torch.full((t.numel() + 512,), 3.0, dtype=kind, device=dev) for n, t in before.items()}
    summed = {n: strips[n][:t.numel()].view(t.shape).copy_(t) for n, t in before.items()}
    alone = run(0, {n: torch.empty_like(t) for n, t in before.items()})
    run(1, summed)
    for n, was in before.items():
        # fp32: one rounding of the sum; bf16: the gradient's own rounding alone, and the sum's
        ref = was.double() + alone[n].double()
        unit = 2.0 ** -24 if f32 else 2.0 ** -8
        bound = 1.01 * unit * (ref.abs() + (0 if f32 else alone[n].double().abs())) + 1e-30
        over = float(((summed[n].double() - ref).abs() - bound).max())
        assert over <= 0, (n, over)
        assert bool((strips[n][was.numel():] == 3.0).all()), n
